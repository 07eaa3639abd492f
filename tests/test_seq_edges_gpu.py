"""The un-pooled lookup where its chunks, pieces and output end: bit equality
with the oracle, and nothing written past an output that is too small."""
import numpy as np
import pytest
import torch

from conftest import oracle_tables
from oracle import ebo_forward_seq
from paper_2609_30656_amd import eb
from test_parity_gpu import _custom, _table, dev, say  # noqa: F401  (dev: the fixture)
from test_seq_gpu import full_seq_check, seq_numel

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("bits", [32, 64])
@pytest.mark.parametrize("dtype,D", [("f32", 4), ("f32", 64), ("f32", 260), ("f16", 8), ("f16", 72), ("f16", 128),
                                     ("f16", 1032), ("int8_rowwise", 16), ("int8_rowwise", 112),
                                     ("int8_rowwise_split", 128), ("int8_rowwise_split", 1040)])
def test_chunk_edges(dev, dtype, D, bits):  # noqa: F811
    say(f"[seq] chunk edges {dtype} D={D}")
    tables = [_table(dev, dtype, 200, D, seed=i) for i in range(4)]
    for n in (1, 63, 64, 65, 127, 129):
        lens = [np.array([0, n, 0]), np.array([0, 0, 0]), np.array([n + 1, 0, 2]), np.array([0, 0, n])]
        full_seq_check(_custom(dev, tables, lens, index_dtype=torch.int32 if bits == 32 else torch.int64),
                       f"{dtype} D={D} n={n}")


@pytest.mark.parametrize("short", [4, 8, 64, 100, 128, 1000])
def test_output_too_small(dev, short):  # noqa: F811
    # an output within the host's range but smaller than these offsets need:
    # what fits is written, nothing after it
    say(f"[seq] output {short} values too small")
    tables = [_table(dev, "f32", 50, 8), _table(dev, "f16", 50, 64, seed=1), _table(dev, "int8_rowwise", 50, 16, seed=2)]
    w = _custom(dev, tables, [np.full(40, 3)] * 3)
    n = seq_numel(w)
    buf = torch.full((n,), 7.0, device=dev)
    with eb.eb_create_tables(w.tables) as h:
        eb.eb_forward_seq(h, w.indices, w.offsets, buf[:n - short])
        torch.cuda.synchronize()
    assert bool((buf[n - short:] == 7.0).all())
    ref = ebo_forward_seq(oracle_tables(w), w.indices.cpu().numpy(), w.offsets.cpu().numpy())
    whole = (n - short) // 64 * 64 - 64  # every row before the last that fits
    assert np.array_equal(buf[:whole].cpu().numpy().view(np.uint32), ref[:whole].view(np.uint32))


@pytest.mark.parametrize("n", [(1 << 26) - 64, (1 << 26) - 63, (1 << 26) + 65])
def test_two_chunks_per_wavefront(dev, n):  # noqa: F811
    # the last size of one chunk per wavefront and the first of two, with a
    # table's end inside a chunk; fp32 rows come out as they are stored
    say(f"[seq] {n} positions")
    tables = [torch.randn((1000, 4), device=dev) for _ in range(2)]
    cut = n // 2 // 64 * 64 + 31
    indices = torch.randint(0, 1000, (n,), device=dev, dtype=torch.int32)
    offsets = torch.tensor([0, cut, n], device=dev, dtype=torch.int32)
    out = torch.full((4 * n,), 7.0, device=dev)
    with eb.eb_create_tables([(t, 4, "f32") for t in tables]) as h:
        eb.eb_forward_seq(h, indices, offsets, out)
        torch.cuda.synchronize()
    for t, (a, b) in enumerate(((0, cut), (cut, n))):
        assert torch.equal(out[4 * a:4 * b].view(-1, 4), tables[t][indices[a:b].long()])
