"""The Python binding's two routes agree: the extension for plain tensors, and
the ctypes path for everything else (tensor subclasses, function modes, errors)."""
import numpy as np
import pytest
import torch

from paper_2609_30656_amd import eb
from test_parity_gpu import _custom, _table, dev, say  # noqa: F401  (dev: the fixture)

pytestmark = pytest.mark.gpu


class Sub(torch.Tensor):
    pass


class Mode(torch.overrides.TorchFunctionMode):
    def __torch_function__(self, func, types, args=(), kwargs=None):
        return func(*args, **(kwargs or {}))


def _calls(w, h, wrap=lambda x: x):
    """Every entry point once, as {name: outputs}."""
    D = w.tables[0].dim
    dev_ = w.indices.device
    i, o = wrap(w.indices), wrap(w.offsets)
    wt = wrap(w.weights)
    out, fm = torch.empty((w.batch, w.sum_dim), device=dev_), torch.empty(w.batch, device=dev_)
    got = {"forward": eb.eb_forward(h, i, o, wt, "sum", wrap(out)).clone()}
    eb.eb_forward(h, i, o, None, "mean", wrap(out))
    got["mean"] = out.clone()
    got["fm_cross"] = eb.eb_fm_cross(h, wrap(out), wrap(fm)).clone()
    eb.eb_forward_fm(h, i, o, wt, 0, wrap(out), wrap(fm))
    got["forward_fm"], got["fm"] = out.clone(), fm.clone()
    got["seq"] = eb.eb_forward_seq(h, i, o, wrap(torch.empty((w.indices.numel(), D), device=dev_))).clone()
    g = torch.Generator(device=dev_).manual_seed(1)
    grad = torch.randn((w.batch, w.sum_dim), generator=g, device=dev_)
    before = [t.rows.clone() for t in w.tables]
    for name in ("workspace", "given", "noalloc"):
        state = torch.zeros(sum(t.num_rows for t in w.tables), device=dev_)
        for t, b in zip(w.tables, before):
            t.rows.copy_(b)
        args = (h, i, o, wt, "sum", wrap(grad), "rowwise_adagrad", 0.1, 1e-6, wrap(state))
        if name == "noalloc":
            eb.eb_backward_update_noalloc(*args)
        else:
            ws = torch.empty(eb.eb_backward_workspace_size(h, w.indices.numel()), dtype=torch.uint8, device=dev_)
            eb.eb_backward_update(*args, workspace=wrap(ws) if name == "given" else None)
        torch.cuda.synchronize()
        got["rows " + name] = torch.cat([t.rows.float().view(-1) for t in w.tables])
        got["state " + name] = state.clone()
    for t, b in zip(w.tables, before):
        t.rows.copy_(b)
    return {k: v.as_subclass(torch.Tensor) for k, v in got.items()}


def test_routes_agree(dev):  # noqa: F811
    say("[bind] routes agree")
    rng = np.random.default_rng(2)
    w = _custom(dev, [_table(dev, "f32", 300, 16), _table(dev, "f16", 200, 16, seed=1)],
                [rng.integers(0, 30, 40) for _ in range(2)], weighted=True)
    with eb.eb_create_tables(w.tables) as h:
        plain = _calls(w, h)
        sub = _calls(w, h, lambda x: x.as_subclass(Sub))
        param = _calls(w, h, lambda x: torch.nn.Parameter(x, requires_grad=False))
        with Mode():
            mode = _calls(w, h)
    for other in (sub, param, mode):
        for k in plain:
            assert torch.equal(plain[k].view(torch.int32), other[k].view(torch.int32)), k


def test_errors_are_the_same(dev):  # noqa: F811
    say("[bind] errors")
    w = _custom(dev, [_table(dev, "f32", 300, 16)], [np.full(8, 3)])
    out = torch.empty((8, 16), device=dev)
    with eb.eb_create_tables(w.tables) as h:
        for bad, what in ((w.indices.cpu(), "on the handle's GPU"), (w.indices.repeat(2)[::2], "contiguous")):
            with pytest.raises(ValueError, match=what):
                eb.eb_forward(h, bad, w.offsets, None, "sum", out)
        for kw in (dict(i=w.indices.double()), dict(o=w.offsets.to(torch.int32)), dict(out=out.half())):
            with pytest.raises(eb.EBError) as e:
                eb.eb_forward(h, kw.get("i", w.indices), kw.get("o", w.offsets), None, "sum", kw.get("out", out))
            assert e.value.status == eb.EB_ERR_DTYPE
        with pytest.raises(eb.EBError) as e:
            eb.eb_forward(h, w.indices, w.offsets, None, 7, out)
        assert e.value.status == eb.EB_ERR_INVALID_ARG
        with pytest.raises(KeyError):
            eb.eb_forward(h, w.indices, w.offsets, None, "max", out)
        with pytest.raises(KeyError):
            eb.eb_backward_update_noalloc(h, w.indices, w.offsets, None, "sum", out, "adam")
        with pytest.raises(AttributeError):
            eb.eb_forward(h, [1, 2], w.offsets, None, "sum", out)
    with pytest.raises(eb.EBError) as e:  # a destroyed handle
        eb.eb_forward(h, w.indices, w.offsets, None, "sum", out)
    assert e.value.status == eb.EB_ERR_INVALID_ARG
