"""The pipeline at call sizes that the one-launch kernel takes by default: the same
inputs through both routes, against the oracle.  (Chosen launch parameters make a
call run the pipeline.)  And calls just above the size from which the pipeline runs
by default, for G > 16 through the 16 x 16 window, against the call without a
workspace, which always takes the one launch, and the oracle."""
import numpy as np
import pytest

from oracle import ref
from tests import inputs

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def jt():
    import paper_2205_15311_amd as pkg
    return pkg


@pytest.fixture(params=["one", "pipeline"])
def batch(request, jt):
    with jt.Batch((1 << 20) + 77) as b:
        if request.param == "pipeline":
            b.set_refill(25)
        yield b


def records(rec):
    torch.cuda.synchronize()
    return rec.cpu().numpy().view(ref.RECORD).reshape(-1)


def device(a):
    return torch.from_numpy(np.ascontiguousarray(a).view(np.int64)).cuda()


@pytest.mark.parametrize("t,grid,runs", [(2, 16, 20), (3, 16, 20), (3, 32, 20), (2, 32, 20),
                                         (4, 16, 5), (2, 16, 1), (2, 16, 2), (2, 16, 64),
                                         (3, 10, 33), (1, 8, 20), (4, 24, 20)])
def test_lists(batch, t, grid, runs):
    n = 30_000 if grid <= 16 else 8_000
    gs = np.random.default_rng(70 * t + grid + runs).integers(0, 1 << (12 * t), size=n,
                                                              dtype=np.uint64)
    want = ref.classify(gs, t, grid=grid, runs=runs, seed=1)
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    assert np.array_equal(records(batch.classify(device(gs), t, 8, grid, runs, 1, tally=tally)), want)
    assert tally.cpu().tolist() == np.bincount(want["cls"], minlength=4).tolist()


@pytest.mark.parametrize("c,t,grid", [(2, 2, 16), (4, 2, 16), (4, 4, 32), (16, 3, 16), (16, 4, 20)])
def test_colour_counts(batch, c, t, grid):
    bits = 4 * t * (c.bit_length() - 1)
    gs = np.random.default_rng(c + t).integers(0, 1 << min(bits, 63), size=8000, dtype=np.uint64)
    want = ref.classify(gs, t, c=c, grid=grid, runs=20, seed=5)
    assert np.array_equal(records(batch.classify(device(gs), t, c, grid, 20, 5)), want)


@pytest.mark.parametrize("n", [0, 1, 2, 63, 65, 1000, 4097])
def test_ranges(batch, n):
    for t, first, grid in ((2, 9_000_000, 16), (3, 12_345_678_901, 32)):
        got = records(batch.classify_range(first, n, t, 8, grid, 20, 1))
        if n:
            assert np.array_equal(got, ref.classify_range(first, n, t, grid=grid, runs=20, seed=1))


def test_one_tile_space(batch):
    got = records(batch.classify_range(0, 4096, 1, 8, 16, 20, 1))
    assert np.array_equal(got, ref.classify_range(0, 4096, 1, grid=16, runs=20, seed=1))


def test_items_and_orders(batch, jt):
    n = 20_000
    rng = np.random.default_rng(2027)
    gs, t, grid = inputs.mixed_stream(n, key=23)
    rid = gs | (t.astype(np.uint64) << np.uint64(56))
    rid[::5] ^= rng.integers(0, 1 << 40, size=rid[::5].shape[0], dtype=np.uint64)
    items = jt.make_items(gs, t, grid, rid)
    want_items = np.zeros(n, dtype=ref.ITEM)
    want_items["genome"], want_items["rng_id"], want_items["t"], want_items["grid"] = gs, rid, t, grid
    want = ref.classify_items(want_items, c=8, runs=20, seed=1)
    items[17, 16] = 9
    items[18, 17] = 11
    want[17:19] = np.array([(-1, 0, 0, 0)], dtype=ref.RECORD)[0]
    dev = torch.from_numpy(items).cuda()
    for order in (None, np.arange(n)[::-1], rng.permutation(n), np.argsort(-grid.astype(np.int64))):
        o = None if order is None else torch.from_numpy(order.astype(np.int32)).cuda()
        tally = torch.zeros(4, dtype=torch.int64, device="cuda")
        assert np.array_equal(records(batch.classify_items(dev, 8, 20, 1, tally=tally, order=o)), want)
        assert tally.cpu().tolist() == [int((want["cls"] == k).sum()) for k in range(4)]
    order = torch.from_numpy(rng.permutation(n).astype(np.int32)).cuda()
    got = records(batch.classify_range_ordered(5_000_000, n, order, 2, 8, 16, 20, 1))
    assert np.array_equal(got, ref.classify_range(5_000_000, n, 2, grid=16, runs=20, seed=1))


@pytest.mark.parametrize("grid", [16, 32])
def test_rare_paths_of_three_tiles(batch, grid):
    gs = np.random.default_rng(124 + grid).integers(0, 1 << 36, size=200_000, dtype=np.uint64)
    want = ref.classify(gs, 3, grid=grid, runs=20, seed=1)
    assert (want["cls"] == ref.ND_RUNS).sum() > 5
    assert ((want["cls"] == ref.DET) & (want["size"] >= 20)).sum() > 5
    assert np.array_equal(records(batch.classify(device(gs), 3, 8, grid, 20, 1)), want)


@pytest.mark.parametrize("t,grid", [(2, 16), (3, 16), (4, 16), (3, 32), (2, 24), (4, 32)])
def test_calls_above_the_one_launch(jt, t, grid):
    n = (1 << 20) + 77
    gs = np.random.default_rng(t + grid).integers(0, 1 << (12 * t), size=n, dtype=np.uint64)
    x = device(gs)
    one = records(jt.classify(x, t, 8, grid, 20, 1))
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    with jt.Batch(n) as b:
        assert np.array_equal(records(b.classify(x, t, 8, grid, 20, 1, tally=tally)), one)
    assert tally.cpu().tolist() == np.bincount(one["cls"], minlength=4).tolist()
    sample = np.random.default_rng(4).choice(n, 20_000, replace=False)
    assert np.array_equal(one[sample], ref.classify(gs[sample], t, grid=grid, runs=20, seed=1))


def test_first_call_under_capture(jt):
    """A call without a workspace in a graph, replayed between other work; and the
    static call, which has to have been made once before."""
    gs = torch.arange(4096, dtype=torch.int64, device="cuda") * 4093
    out = torch.zeros((4096, 4), dtype=torch.int32, device="cuda")
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    want = jt.classify_static(gs, 2, 8, 16, 20, 1)
    torch.cuda.synchronize()
    graphs = []
    for call in (lambda: jt.classify(gs, 2, 8, 16, 20, 1, out=out),
                 lambda: jt.classify_static(gs, 2, 8, 16, 20, 1, out=out, tally=tally)):
        graph = torch.cuda.CUDAGraph()
        with torch.cuda.graph(graph, stream=torch.cuda.Stream()):
            call()
        graphs.append(graph)
    counts = torch.bincount(want[:, 0].long(), minlength=4)
    for k in range(1, 4):
        for graph in graphs:
            out.zero_()
            graph.replay()
            torch.cuda.synchronize()
            assert torch.equal(out, want)
            jt.classify_static(gs[:777], 2, 8, 16, 7, 1)
        assert torch.equal(tally, k * counts)
