"""Which candidates have a proof: none in the one launch up to four runs at G <= 16, and
in the pipeline's queue those with lost ids only where a chunk of it holds enough of
them.  Lists of candidates on both sides of either line, equal to the oracle's records."""
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


@pytest.mark.parametrize("runs", [1, 2, 3, 4, 5])
@pytest.mark.parametrize("t,grid", [(2, 8), (2, 16), (3, 10), (4, 16)])
def test_few_runs(t, grid, runs):
    import paper_2205_15311_amd as jt
    from tests.test_gpu_bonds import symmetric_genomes
    rng = np.random.default_rng(10 * t + grid + runs)
    gs = rng.integers(0, 1 << 24, size=200_000, dtype=np.uint64) if t == 2 \
        else symmetric_genomes(rng, 60_000, t, 8)
    one = ref.classify(gs, t, grid=grid, runs=1, seed=1)
    gs = np.concatenate([gs[(one["cls"] == 3) & (one["size"] > 2)], gs[:500]])
    want = ref.classify(gs, t, grid=grid, runs=runs, seed=1)
    assert (want["cls"] == 3).sum() > 1000
    if runs > 1:   # candidates that a later run decides
        assert (want["cls"][:-500] != 3).sum() > 100
    for n in (len(gs), 250_000):   # a few a wave, and more than a list's length
        at = np.resize(rng.permutation(len(gs)), n)
        x = device(gs[at])
        assert np.array_equal(records(jt.classify(x, t, 8, grid, runs, 1)), want[at]), n
        tally = torch.zeros(4, dtype=torch.int64, device="cuda")
        with jt.Batch(n) as b:
            assert np.array_equal(records(b.classify(x, t, 8, grid, runs, 1, tally=tally)),
                                  want[at]), n
        assert tally.tolist() == [int((want["cls"][at] == k).sum()) for k in range(4)]


@pytest.mark.parametrize("share", [0.3, 0.5, 1.0])
@pytest.mark.parametrize("n", [40_000, 300_000])   # fewer chunks than waves, and more
def test_queues_with_lost_ids(n, share):
    import paper_2205_15311_amd as jt
    from tests.test_gpu_sixteenth_tile import structured, triples
    rng = np.random.default_rng(n + int(10 * share))
    rows = [np.resize(np.array(triples(q), dtype=np.uint64), 20_000) for q in (3, 2)]
    lost = np.concatenate([structured(rng, 20_000), rows[0]])
    kept = np.concatenate([rng.integers(0, 1 << 48, size=20_000, dtype=np.uint64), rows[1]])
    both = []
    for gs in (lost, kept):
        one = ref.classify(gs, 4, grid=16, runs=1, seed=1)
        gs = gs[(one["cls"] == 3) & (one["size"] > 2)]
        both.append((gs, ref.classify(gs, 4, grid=16, runs=20, seed=1)))
    from_lost = rng.random(n) < share
    gs, want = np.empty(n, dtype=np.uint64), np.empty(n, dtype=ref.RECORD)
    for mask, (pool, rec) in ((from_lost, both[0]), (~from_lost, both[1])):
        at = rng.integers(0, len(pool), size=int(mask.sum()))
        gs[mask], want[mask] = pool[at], rec[at]
    with jt.Batch(n) as b:
        b.set_refill(25)   # launch parameters of the caller's: the pipeline
        assert np.array_equal(records(b.classify(device(gs), 4, 8, 16, 20, 1)), want)
