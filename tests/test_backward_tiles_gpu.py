"""GPU parity of the backward's tiles where runs meet the edges of lane groups,
wavefronts and tiles: runs of chosen lengths in chosen places, every width of a
lane group, both storage types, both optimizers.  Same bounds as
test_backward_gpu.py."""
import numpy as np
import pytest
import torch

from paper_2609_30656_amd import eb
from paper_2609_30656_amd.workload import Table, Workload
from test_backward_gpu import dev, run_and_check, say  # noqa: F401  (dev: the fixture)

pytestmark = pytest.mark.gpu

# rows occur these many times, in row order, so the sorted positions hold runs
# of these lengths: inside a group, exactly a group, wavefront (64) or tile
# (256), one more, one less, and whole tiles in one run
RUNS = ([1, 2, 3, 1, 1, 4, 7, 8, 9, 15, 16, 17, 1, 31, 32, 33, 63, 1, 64, 65, 1, 2] + [1] * 70 +
        [127, 1, 255, 256, 257, 3, 1, 1000, 1, 1, 513, 5])


def _workload(dev, specs, runs, pooling, weighted, bits, seed=0):  # noqa: F811
    """Tables (dtype, D) whose row i occurs runs[t][i] times, at shuffled positions of 50 bags."""
    g = torch.Generator(device="cpu")
    g.manual_seed(seed)
    B, tables, lens, idx = 50, [], [], []
    for (dtype, D), r in zip(specs, runs):
        rows = torch.randn((len(r) + 3, D), generator=g)
        tables.append(Table((rows * 0.1).half().to(dev) if dtype == "f16" else rows.to(dev), D, dtype))
        i = torch.repeat_interleave(torch.arange(len(r)), torch.tensor(r))
        i = i[torch.randperm(i.numel(), generator=g)]
        cuts, _ = torch.sort(torch.randint(0, i.numel() + 1, (B - 1,), generator=g))
        edges = torch.cat([torch.zeros(1, dtype=torch.int64), cuts, torch.tensor([i.numel()])])
        lens.append(edges[1:] - edges[:-1])
        idx.append(i)
    lens, idx = torch.cat(lens), torch.cat(idx)
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64)
    torch.cumsum(lens, 0, out=off[1:])
    dt = torch.int32 if bits == 32 else torch.int64
    w = torch.rand(idx.numel(), generator=g).to(dev) if weighted else None
    return Workload("runs", tables, B, idx.to(dt).to(dev), off.to(dt).to(dev), w, pooling, lens.to(dev))


@pytest.mark.parametrize("chunks", ["0", "1", "16"])
@pytest.mark.parametrize("optimizer", ["sgd", "rowwise_adagrad"])
@pytest.mark.parametrize("dtype", ["f32", "f16"])
def test_runs_of_every_length(dev, monkeypatch, dtype, optimizer, chunks):  # noqa: F811
    monkeypatch.setenv("EB_BWD_TILE_CHUNKS", chunks)
    unit = 4 if dtype == "f32" else 8
    for k, D in enumerate([unit, 8, 16, 24, 32, 64, 72, 128, 136, 256]):
        bits, pooling, weighted = (32, "mean", False) if k % 3 == 1 else (64, "sum", k % 3 == 2)
        runs = RUNS if k % 2 == 0 else RUNS[::-1]
        w = _workload(dev, [(dtype, D), (dtype, D)], [runs, [700] + runs[5:40]], pooling, weighted, bits, seed=k)
        run_and_check(w, dev, optimizer, label=f"runs {dtype} D={D} chunks={chunks}")


def test_runs_over_mixed_tables(dev):  # noqa: F811
    specs = [("f32", 4), ("f16", 256), ("f32", 256), ("f16", 64), ("f32", 36), ("f16", 128)]
    runs = [RUNS, RUNS[::-1], [3000, 1, 1], RUNS[10:], [1] * 300, [256, 256, 256, 1]]
    run_and_check(_workload(dev, specs, runs, "sum", True, 64), dev, "rowwise_adagrad", label="runs, mixed tables")


def test_gradient_past_4gib(dev):  # noqa: F811
    """A gradient matrix of more than 4 GiB is read with 64-bit addresses: 70
    tables of 256 values, batch 65 536, lookups in the first and last examples."""
    say("[bwd] gradient past 4 GiB")
    T, D, B, R, L = 70, 256, 65536, 40, 60
    g = torch.Generator(device=dev)
    g.manual_seed(3)
    rows = [torch.randn((R, D), generator=g, device=dev) for _ in range(T)]
    tables = [Table(r if t % 2 else r.mul(0.1).half(), D, "f32" if t % 2 else "f16") for t, r in enumerate(rows)]
    lens = torch.zeros((T, B), dtype=torch.int64, device=dev)
    lens[:, 0], lens[:, B - 1] = 5, L - 5
    off = torch.zeros(T * B + 1, dtype=torch.int64, device=dev)
    torch.cumsum(lens.view(-1), 0, out=off[1:])
    idx = torch.randint(0, R, (T * L,), generator=g, device=dev)
    grad = torch.randn((B, T * D), generator=g, device=dev)
    assert grad.numel() * 4 > 1 << 32
    want = []
    for t, tb in enumerate(tables):
        i = idx[t * L:(t + 1) * L]
        G = torch.zeros((R, D), dtype=torch.float64, device=dev)
        G.index_add_(0, i[:5], grad[:1, t * D:(t + 1) * D].double().expand(5, D))
        G.index_add_(0, i[5:], grad[B - 1:, t * D:(t + 1) * D].double().expand(L - 5, D))
        want.append(tb.rows.double() - 0.5 * G)
    with eb.eb_create_tables(tables) as h:
        eb.eb_backward_update(h, idx, off, None, "sum", grad, "sgd", 0.5)
        torch.cuda.synchronize()
    for t, tb in enumerate(tables):
        err = (tb.rows.double() - want[t]).abs().max().item()
        # one rounding to the storage type of values up to about 20, fp32 sums of up to L terms
        bound = np.abs(want[t].cpu().numpy()).max() * (2.0 ** -11 if tb.dtype == "f16" else L * 2.0 ** -24) + 1e-5
        assert err <= bound, (t, err, bound)


@pytest.mark.parametrize("weighted", [False, True])
@pytest.mark.parametrize("most", [3_000_000, 100_000, 300])
def test_tables_of_every_pass_count(dev, monkeypatch, most, weighted):  # noqa: F811
    """Tables whose rows take one to three sort passes, next to one whose rows
    set the launch's: each starts at its own pass, with its own digit bits; an
    index outside its table among them."""
    say(f"[bwd] tables of up to {most} rows")
    g = torch.Generator(device="cpu")
    g.manual_seed(most)
    sizes = [r for r in (1, 2, 3, 127, 128, 255, 256, 511, 512, 5000, 65535, 65536, 262143, 262144, most) if r <= most]
    tables = [Table(torch.randn((r, 4), generator=g).to(dev), 4, "f32") for r in sizes]
    B = 37
    lens = torch.randint(0, 60, (len(sizes) * B,), generator=g)
    off = torch.zeros(lens.numel() + 1, dtype=torch.int64)
    torch.cumsum(lens, 0, out=off[1:])
    parts = []
    for t, r in enumerate(sizes):
        n = int(lens[t * B:(t + 1) * B].sum())
        i = torch.randint(0, r, (n,), generator=g)
        i[torch.rand(n, generator=g) < 0.2] = r - 1
        parts.append(i)
    idx = torch.cat(parts)
    w = torch.rand(idx.numel(), generator=g).to(dev) if weighted else None
    run_and_check(Workload("passes", tables, B, idx.to(dev), off.to(dev), w, "sum", lens.to(dev)), dev,
                  "rowwise_adagrad", label=f"passes, up to {most} rows")


@pytest.mark.parametrize("dtype,D", [("f32", 4), ("f32", 32), ("f16", 128), ("f32", 256)])
def test_run_of_many_tiles(dev, dtype, D):  # noqa: F811
    # runs that cover 64 tiles of 256 positions after their own, one more, the
    # fix-up's first full batch of partials, and an odd rest of it
    for tiles, rest in ((64, 1), (65, 1), (66, 200), (73, 255), (200, 3)):
        runs = [100, 256 * tiles + rest, 30]
        w = _workload(dev, [(dtype, D)], [runs], "sum", tiles % 2 == 0, 64, seed=tiles)
        run_and_check(w, dev, "sgd", label=f"run over {tiles} tiles {dtype} D={D}")
