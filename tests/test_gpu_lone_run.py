"""The whole-wave run of a wave's last lane against the oracle: calls of one
genotype, so that every run of theirs is made that way, over grids of both
layouts and their halves' borders (the 32 x 32 grid's rows lie on two lanes,
split at x = 16), long runs (several blocks of random words), the sixteenth
oriented tile, 16 colours, and every class; then a call in which one long run
outlasts its wave's others, whose lists and grids must be left as they were."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def records(rec):
    torch.cuda.synchronize()
    return rec.cpu().numpy().view(ref.RECORD).reshape(-1)


def pool(t, c, grid, seed):
    """Genotypes whose first run is long, of every class, and a plain sample."""
    from tests.test_gpu_bonds import symmetric_genomes
    rng = np.random.default_rng(seed)
    bits = 4 * t * (3 if c == 8 else 4)
    gs = rng.integers(0, 1 << min(bits, 63), size=120_000, dtype=np.uint64)
    gs = np.concatenate([gs, symmetric_genomes(rng, 30_000, t, c)])
    one = ref.classify(gs, t, c=c, grid=grid, runs=1, seed=1)
    order = np.argsort(-one["steps"], kind="stable")
    pick = [order[:60], rng.choice(len(gs), 60)]
    for cls in (0, 1, 3):
        pick.append(order[one["cls"][order] == cls][:40])
    return gs[np.unique(np.concatenate(pick))]


@pytest.mark.parametrize("t,c,grid", [(2, 8, 16), (3, 8, 32), (4, 8, 32), (4, 16, 32), (4, 16, 16),
                                      (4, 8, 10), (3, 8, 18), (4, 8, 24), (1, 8, 8)])
def test_calls_of_one_genotype(t, c, grid):
    import paper_2205_15311_amd as jt
    gs = pool(t, c, grid, 7 * t + c + grid)
    want = ref.classify(gs, t, c=c, grid=grid, runs=12, seed=1)
    dev = torch.from_numpy(gs.view(np.int64)).cuda()
    out = torch.empty((len(gs), 4), dtype=torch.int32, device="cuda")
    for i in range(len(gs)):
        jt.classify(dev[i:i + 1], t, c, grid, 12, 1, out=out[i:i + 1])
    got = records(out)
    assert np.array_equal(got, want), np.nonzero(got != want)[0][:5]


@pytest.mark.parametrize("t,grid", [(2, 16), (3, 32), (4, 32)])
def test_one_long_run_among_short_ones(t, grid):
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(t + grid)
    gs = rng.integers(0, 1 << min(12 * t, 63), size=200_000, dtype=np.uint64)
    one = ref.classify(gs, t, grid=grid, runs=1, seed=1)
    order = np.argsort(-one["steps"], kind="stable")
    waves = [np.concatenate([gs[order[k:k + 1]], gs[rng.choice(order[5000:], 63)]])
             for k in range(40)]
    for w in waves:
        rng.shuffle(w)
        want = ref.classify(w, t, grid=grid, runs=20, seed=1)
        # as one wave's items, and twice over through the pipeline
        dev = torch.from_numpy(w.view(np.int64)).cuda()
        with jt.Batch(len(w)) as b:
            assert np.array_equal(records(b.classify(dev, t, 8, grid, 20, 1)), want)
            b.set_refill(25)
            assert np.array_equal(records(b.classify(dev, t, 8, grid, 20, 1)), want)
            assert np.array_equal(records(b.classify(dev, t, 8, grid, 20, 1)), want)
