"""More than 32 runs, where a wave's long list of unproven candidates has a pass of 16
runs between the first four and all of them: lists of candidates on both sides of
the length from which it does, decided by a witness in each of the passes or by
none, against the oracle."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("runs", [32, 33, 48, 64])
@pytest.mark.parametrize("t", [2, 4])
def test_long_lists_of_candidates(runs, t):
    import paper_2205_15311_amd as jt
    from tests.test_gpu_bonds import symmetric_genomes
    rng = np.random.default_rng(runs + t)
    gs = rng.integers(0, 1 << 24, size=300_000, dtype=np.uint64) if t == 2 \
        else symmetric_genomes(rng, 120_000, 4, 8)
    one = ref.classify(gs, t, grid=16, runs=1, seed=1)
    gs = gs[(one["cls"] == 3) & (one["size"] > 2)]
    want = ref.classify(gs, t, grid=16, runs=runs, seed=1)
    first = ref.classify(gs, t, grid=16, runs=4, seed=1)
    # few proven ones among them: those that 4 runs leave open or decide otherwise
    pick = np.nonzero((want["cls"] != 3) | (first["steps"] != (first["size"] - 1) * 4))[0]
    late = np.nonzero((first["cls"] == 3) & (want["cls"] != 3))[0]
    assert len(pick) > 300 and len(late) > 10
    pick = np.concatenate([pick, np.resize(late, len(pick)), np.arange(len(gs))[:len(pick)]])
    for n in (len(pick), 400_000):   # one or a few a wave, and more than a list's length
        at = np.resize(rng.permutation(pick), n)
        x = torch.from_numpy(gs[at].view(np.int64)).cuda()
        rec = jt.classify(x, t, 8, 16, runs, 1)
        torch.cuda.synchronize()
        assert np.array_equal(rec.cpu().numpy().view(ref.RECORD).reshape(-1), want[at]), n
