"""The breadth-first search behind the true class against one written from the
from-scratch model of tests/brute_force.py, level by level: class, size and the
number of states, for searches on both sides of sixteen states a level (where
the search moves from LDS to device memory), every end a search can have, and
limits on the states and on the states of a level."""
import numpy as np
import pytest

from oracle import ref
from tests import brute_force as bf

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def levels(genome, t, c, grid, cap, max_level):
    """(class, size, states, widest level): the search by levels."""
    m = bf.Model(int(genome), t, c, grid)
    level = [{m.centre: m.seed_tile}]
    total, widest, shape = 1, 1, None
    while True:
        analysed = [m.analyse(s) for s in level]
        if any(e is not None for e, _ in analysed):
            return 1, 0, total, widest
        nxt = {}
        for state, (_, frontier) in zip(level, analysed):
            for q, tile in frontier.items():
                s = dict(state)
                s[q] = tile
                nxt[frozenset(s.items())] = s
        if len(nxt) > max_level:
            return -2, 0, total, max(widest, len(nxt))
        widest = max(widest, len(nxt))
        for state, (_, frontier) in zip(level, analysed):
            if not frontier:
                shape = shape or set(state)
                if set(state) != shape:
                    return 1, 0, total, widest
        if total + len(nxt) > cap:
            return -2, 0, total, widest
        if not nxt:
            return 3, len(shape), total, widest
        level = list(nxt.values())
        total += len(level)


def candidates(t, c, grid, n, seed):
    """Genotypes that 20 runs call deterministic, with a choice of sites."""
    from tests.test_gpu_bonds import symmetric_genomes
    rng = np.random.default_rng(seed)
    pool = rng.integers(0, 1 << (4 * t * (3 if c == 8 else 4)) if t < 4 or c == 8 else 1 << 63,
                        size=300_000, dtype=np.uint64)
    pool = np.concatenate([pool, symmetric_genomes(rng, 60_000, t, c)])
    rec = ref.classify(pool, t, c=c, grid=grid, runs=1, seed=1)
    return pool[(rec["cls"] == ref.DET) & (rec["size"] >= 3) & (rec["size"] <= 14)][:n]


@pytest.mark.parametrize("t,c,grid", [(2, 8, 16), (3, 8, 16), (4, 8, 16), (4, 16, 32),
                                      (2, 8, 32), (3, 8, 32)])
def test_levels(t, c, grid):
    import paper_2205_15311_amd as jt
    gs = candidates(t, c, grid, 20_000, 5 * t + c + grid)
    dev = torch.from_numpy(gs.view(np.int64)).cuda()
    cap = 150
    seen = set()
    for max_level in (4096, 3, 16, 17):
        with jt.Truth(len(gs), max_level=max_level, waves=16) as w:
            rec = w.true_class(dev, t, c, grid, cap=cap)
            torch.cuda.synchronize()
            rec = rec.cpu().numpy().view(ref.RECORD).reshape(-1)
        searched = np.nonzero(rec["steps"] > 0)[0]
        assert len(searched) > 0
        # the widest searches, the ones at the limits and a plain sample
        many = searched[np.argsort(rec["steps"][searched])[-25:]]
        few = searched[:: max(1, len(searched) // 40)]
        for i in np.unique(np.concatenate([many, few])):
            cls, size, total, widest = levels(gs[i], t, c, grid, cap, max_level)
            assert (rec["cls"][i], rec["size"][i], rec["steps"][i]) == (cls, size, total), \
                (hex(int(gs[i])), max_level, widest)
            seen.add((cls, widest > 16))
    assert (1, False) in seen
    print(t, c, grid, sorted(seen))
