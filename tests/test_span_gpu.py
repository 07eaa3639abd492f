"""GPU parity of the span kernel and its fix-up: batches of at least 64 lookups
per bag on average, cut into spans of the index stream whatever bags they fall
in.  Same bar as test_parity_gpu.py."""
import numpy as np
import pytest
import torch

from test_parity_gpu import WIDTHS, _custom, _table, dev, full_check, run_gpu, say  # noqa: F401  (dev: the fixture)

pytestmark = pytest.mark.gpu

# bag lengths around the edges of chunks (64) and spans (256 and more), empty
# and one-row bags, a run of empty bags longer than the 64 offsets a wavefront
# holds, a bag of many spans, and empty bags at both ends
EDGES = ([0, 0, 1, 63, 64, 65, 255, 256, 257, 0, 511, 512, 513] + [0] * 150 + [20000, 1, 0, 1, 0, 4097, 300, 0])


def _lens(rng, edges):
    lens = np.array(edges)
    return np.concatenate([lens, rng.integers(60, 200, 2 * len(lens))]) if edges is EDGES else lens


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("mode", ["sum", "mean", "weighted"])
@pytest.mark.parametrize("dtype,D", [("f32", 64), ("f16", 128), ("int8_rowwise", 64), ("int8_rowwise_split", 128),
                                     ("f32", 4), ("f16", 520), ("f32", 1028)])
def test_one_kind(dev, monkeypatch, dtype, D, mode, bits):  # noqa: F811
    say(f"[span] {dtype} D={D} {mode} {bits}-bit")
    monkeypatch.delenv("EB_LONG_BAG", raising=False)
    rng = np.random.default_rng(3)
    tables = [_table(dev, dtype, 5000, D), _table(dev, dtype, 3000, D, seed=1)]
    lens = [_lens(rng, EDGES), _lens(rng, EDGES)[::-1].copy()]
    assert np.mean(lens) >= 64
    w = _custom(dev, tables, lens, weighted=(mode == "weighted"), pooling="mean" if mode == "mean" else "sum",
                index_dtype=torch.int32 if bits == 32 else torch.int64)
    got = full_check(w, f"span {dtype} {mode}")
    assert np.array_equal(got.view(np.uint32), run_gpu(w).cpu().numpy().view(np.uint32))


@pytest.mark.parametrize("mode", ["sum", "mean", "weighted"])
def test_every_width_in_one_handle(dev, monkeypatch, mode):  # noqa: F811
    # spans that cross from table to table, of other storage types and widths
    say(f"[span] every width, {mode}")
    monkeypatch.delenv("EB_LONG_BAG", raising=False)
    rng = np.random.default_rng(4)
    tables = [_table(dev, dt, 300 + 7 * i, D, seed=i) for i, (dt, D) in enumerate(WIDTHS)]
    lens = [rng.permutation([0, 1, 64, 129, 700, 0, 90, 15, 300, 0, 33]) for _ in tables]
    w = _custom(dev, tables, lens, weighted=(mode == "weighted"), pooling="mean" if mode == "mean" else "sum")
    full_check(w, f"span widths {mode}")


@pytest.mark.parametrize("lens", [[64], [100], [70000], [0, 0, 0, 300], [4000, 0, 0, 0], [0] * 40000 + [2600000]])
def test_few_bags(dev, monkeypatch, lens):  # noqa: F811
    say(f"[span] {len(lens)} bags, the longest {max(lens)}")
    monkeypatch.delenv("EB_LONG_BAG", raising=False)
    assert np.mean(lens) >= 64
    full_check(_custom(dev, [_table(dev, "f32", 1000, 16)], [np.array(lens)]), "span few bags")
