"""The one-launch classification against the oracle, where its lists can go
wrong: calls of one item up to a few per wave, run counts on both sides of
each change of the repeat rounds, lists that hold only candidates the proof
fails on (the wave's list fills up and is worked off early), shapes too large
to pack, lost tile ids, mixed and invalid items, and the enumeration that
counts shapes in the kernel.  The pipeline (asked for by a launch parameter)
gives the same records."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def records(rec):
    torch.cuda.synchronize()
    return rec.cpu().numpy().view(ref.RECORD).reshape(-1)


def device(gs):
    return torch.from_numpy(np.ascontiguousarray(gs).view(np.int64)).cuda()


def unproven(n, seed=3):
    """Two-tile genotypes that run 0 calls deterministic and 20 runs do not."""
    rng = np.random.default_rng(seed)
    gs = rng.integers(0, 1 << 24, size=400_000, dtype=np.uint64)
    one = ref.classify(gs, 2, grid=16, runs=1, seed=1)
    many = ref.classify(gs, 2, grid=16, runs=20, seed=1)
    gs = gs[(one["cls"] == 3) & (many["cls"] != 3)]
    assert len(gs) > 500
    return np.resize(gs, n)


@pytest.mark.parametrize("n", [1, 2, 63, 64, 65, 3073, 200_001])
@pytest.mark.parametrize("t,grid", [(2, 16), (3, 32)])
def test_call_sizes(n, t, grid):
    import paper_2205_15311_amd as jt
    gs = np.random.default_rng(n).integers(0, 1 << (12 * t), size=n, dtype=np.uint64)
    want = ref.classify(gs, t, grid=grid, runs=20, seed=4)
    assert np.array_equal(records(jt.classify(device(gs), t, 8, grid, 20, 4)), want)
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    with jt.Batch(n) as b:
        assert np.array_equal(records(b.classify(device(gs), t, 8, grid, 20, 4, tally=tally)), want)
    assert tally.cpu().tolist() == np.bincount(want["cls"], minlength=4).tolist()


@pytest.mark.parametrize("runs", [1, 2, 3, 4, 5, 7, 8, 9, 12, 20, 33, 64])
def test_lists_of_unproven_candidates(runs):
    import paper_2205_15311_amd as jt
    gs = unproven(60_000)
    want = ref.classify(gs, 2, grid=16, runs=runs, seed=1)
    with jt.Batch(len(gs)) as b:
        assert np.array_equal(records(b.classify(device(gs), 2, 8, 16, runs, 1)), want)
        b.set_refill(25)   # the pipeline
        assert np.array_equal(records(b.classify(device(gs), 2, 8, 16, runs, 1)), want)
    assert np.array_equal(records(jt.classify(device(gs), 2, 8, 16, runs, 1)), want)


@pytest.mark.parametrize("t,c,grid", [(3, 8, 32), (4, 8, 16), (4, 16, 16), (4, 8, 32), (3, 8, 16)])
def test_large_shapes_and_lost_ids(t, c, grid):
    import paper_2205_15311_amd as jt
    from tests.test_gpu_bonds import symmetric_genomes
    gs = symmetric_genomes(np.random.default_rng(t * c + grid), 60_000, t, c)
    one = ref.classify(gs, t, c=c, grid=grid, runs=1, seed=2)
    gs = gs[(one["cls"] == 3) & (one["size"] > 6)][:4000]
    assert len(gs) > 100
    want = ref.classify(gs, t, c=c, grid=grid, runs=20, seed=2)
    assert np.array_equal(records(jt.classify(device(gs), t, c, grid, 20, 2)), want)
    with jt.Batch(len(gs)) as b:
        for refill in (24, 25):
            b.set_refill(refill)
            assert np.array_equal(records(b.classify(device(gs), t, c, grid, 20, 2)), want)


def test_mixed_and_invalid_items():
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(8)
    n = 5000
    t = rng.integers(1, 4, size=n).astype(np.uint8)
    g = rng.choice([8, 10, 16, 18, 32], size=n).astype(np.uint8)
    gs = rng.integers(0, 1 << 36, size=n, dtype=np.uint64) >> (
        np.uint64(36) - np.uint64(12) * t.astype(np.uint64))
    items = jt.make_items(gs, t, g)
    want = np.empty(n, dtype=ref.RECORD)
    for tt in (1, 2, 3):
        for side in (8, 10, 16, 18, 32):
            at = np.nonzero((t == tt) & (g == side))[0]
            want[at] = ref.classify(np.ascontiguousarray(gs[at]), tt, grid=side, runs=9, seed=1)
    bad = rng.choice(n, 40, replace=False)
    items[bad[:20], 16] = 9      # tile count
    items[bad[20:], 17] = 15     # grid
    want[bad] = np.array([(-1, 0, 0, 0)], dtype=ref.RECORD)[0]
    order = torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda()
    with jt.Batch(n) as b:
        for o in (None, order):
            got = records(b.classify_items(torch.from_numpy(items).cuda(), runs=9, order=o))
            assert np.array_equal(got, want)


@pytest.mark.parametrize("first,n,slices,runs", [(0, 1 << 18, 8, 20), (5_000_001, 99_991, 3, 5),
                                                 (123, 1, 5, 20)])
def test_enumeration_counts_shapes(first, n, slices, runs):
    import paper_2205_15311_amd as jt
    total = n * slices
    want = ref.classify_range(first, total, 2, grid=16, runs=runs, seed=1)
    det = want[want["cls"] == 3]
    keys, counts = np.unique(det[["size", "hash"]], return_counts=True)
    for with_out in (False, True):
        out = torch.empty((total, 4), dtype=torch.int32, device="cuda") if with_out else None
        tally = torch.tensor([1, 2, 3, 4], dtype=torch.int64, device="cuda")
        table = torch.zeros((4096, 2), dtype=torch.int64, device="cuda")
        with jt.Batch(n) as b:
            for _ in range(2):
                b.enumerate(first, n, slices, 2, 8, 16, runs, 1, out=out, tally=tally,
                            shapes=table)
            torch.cuda.synchronize()
        if with_out:
            assert np.array_equal(records(out), want)
        got = jt.shape_table_to_numpy(table)
        assert len(got) == len(keys) and (got["count"] == 2 * counts).all()
        assert (got["size"] == keys["size"]).all() and (got["hash"] == keys["hash"]).all()
        assert tally.cpu().tolist() == (
            np.array([1, 2, 3, 4]) + 2 * np.bincount(want["cls"], minlength=4)).tolist()
