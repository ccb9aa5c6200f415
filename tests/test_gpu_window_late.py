"""Items of G > 16 whose first run stays in the 16 x 16 window and ends cleanly, and
which leave it in a later run: the repeat runs list them for the rerun in their own
grid, under every repeat mapping.  The four-tile genotypes below are such at R = 20,
seed 1 (checked here on the oracle: at G = 16 their first run is clean and a later
one exposes a bondable site outside the box); in their own grids they end in
different ways.  Records must equal the oracle's, the tally the records' classes."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

LATE = np.array([0x3173088a0c, 0x31735281ca, 0x3173fcaa0c, 0x6827e0029e86, 0xe9a340ebe0fc,
                 0x845103e85fce, 0x5a0f01f85fda], dtype=np.uint64)


def records(rec):
    torch.cuda.synchronize()
    return rec.cpu().numpy().view(ref.RECORD).reshape(-1)


def test_these_leave_the_window_late():
    first = ref.classify(LATE, 4, grid=16, runs=1, seed=1)
    all_runs = ref.classify(LATE, 4, grid=16, runs=20, seed=1)
    assert (first["cls"] == ref.DET).all() and (all_runs["cls"] == ref.UNBOUND).all()
    own = ref.classify(LATE, 4, grid=32, runs=20, seed=1)
    assert len(np.unique(own["cls"])) == 3


@pytest.mark.parametrize("mapping", [0, 1, 2])
@pytest.mark.parametrize("runs", [2, 3, 5, 9, 20, 33])
def test_lists_that_leave_the_window_late(mapping, runs):
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(runs)
    gs = np.concatenate([np.resize(LATE, 3000), rng.integers(0, 1 << 48, size=3000, dtype=np.uint64)])
    gs = gs[rng.permutation(len(gs))]
    x = torch.from_numpy(gs.view(np.int64)).cuda()
    with jt.Batch(len(gs)) as b:
        b.set_tuning(16, repeat_mapping=mapping)
        b.set_tuning(32, wide_layout=2, repeat_mapping=mapping)
        for grid in (18, 20, 24, 32):
            want = ref.classify(gs, 4, grid=grid, runs=runs, seed=1)
            tally = torch.zeros(4, dtype=torch.int64, device="cuda")
            assert np.array_equal(records(b.classify(x, 4, 8, grid, runs, 1, tally=tally)), want)
            assert tally.cpu().tolist() == np.bincount(want["cls"], minlength=4).tolist()


@pytest.mark.parametrize("n", [6000, (1 << 20) + 77])
def test_mixed_items_that_leave_the_window_late(n):
    """Above 2^20 items the window is the default."""
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(n)
    gs = np.concatenate([np.resize(LATE, 2000), rng.integers(0, 1 << 48, size=4000, dtype=np.uint64)])
    g = rng.choice([14, 16, 18, 24, 32], size=len(gs)).astype(np.uint8)
    want = np.empty(len(gs), dtype=ref.RECORD)
    for side in np.unique(g):
        want[g == side] = ref.classify(np.ascontiguousarray(gs[g == side]), 4, grid=int(side), runs=20,
                                       seed=1)
    at = np.resize(rng.permutation(len(gs)), n)
    items = torch.from_numpy(jt.make_items(gs[at], 4, g[at])).cuda()
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    with jt.Batch(n) as b:
        if n <= 1 << 20:
            b.set_tuning(32, wide_layout=2)
        got = records(b.classify_items(items, tally=tally))
    assert np.array_equal(got, want[at])
    assert tally.cpu().tolist() == np.bincount(want[at]["cls"], minlength=4).tolist()
