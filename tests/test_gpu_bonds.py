"""Bond lookup by colour and the four-sites-at-once placement, through the ABI.

The cases are where a table of bonds per colour can go wrong: tiles that
look the same after a quarter or half turn, tiles that repeat an earlier
tile's orbit, two tiles that bond to one colour, every colour count (16
colours take a table of two halves), and grids whose box ends inside, at and
beyond a word of the layouts.  Records must equal the oracle's bit for bit.
"""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def symmetric_genomes(rng, n, t, c):
    """Genomes of t tiles with period-1, period-2, repeated, turned and
    ordinary tiles mixed, colours drawn from a few bonding pairs so that
    structures grow."""
    bits = c.bit_length() - 1
    pool = min(c, 6)
    sides = rng.integers(0, pool, size=(n, t, 4))
    kind = rng.integers(0, 5, size=(n, t))
    for i in range(t):
        one, two = kind[:, i] == 0, kind[:, i] == 1
        sides[one, i, 1:] = sides[one, i, :1]
        sides[two, i, 2:] = sides[two, i, :2]
        if i > 0:
            again = kind[:, i] == 2
            sides[again, i] = np.roll(sides[again, i - 1], int(rng.integers(0, 4)), axis=1)
    g = np.zeros(n, dtype=np.uint64)
    for i in range(t):
        for d in range(4):
            g = (g << np.uint64(bits)) | sides[:, i, d].astype(np.uint64)
    return g


@pytest.mark.parametrize("t,c,grid", [(1, 8, 16), (2, 8, 8), (2, 8, 16), (2, 4, 14), (3, 8, 16),
                                      (4, 8, 16), (4, 16, 16), (2, 16, 12), (4, 2, 16),
                                      (3, 8, 18), (3, 8, 32), (4, 16, 32), (2, 16, 30)])
def test_symmetric_and_repeated_tiles(t, c, grid):
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(100 * t + 10 * c + grid)
    gs = symmetric_genomes(rng, 4000, t, c)
    want = ref.classify(gs, t, c=c, grid=grid, runs=12, seed=9)
    # over two colours nothing bonds: every genotype is its seed
    assert len(np.unique(want["cls"])) >= (1 if c == 2 else 2)
    dev = torch.from_numpy(gs.view(np.int64)).cuda()
    plain = jt.classify(dev, t, c, grid, 12, 9)
    with jt.Batch(len(gs)) as b:
        records = [plain, b.classify(dev, t, c, grid, 12, 9)]
        if grid > 16:
            b.set_tuning(32, wide_layout=2)
            records.append(b.classify(dev, t, c, grid, 12, 9))
        torch.cuda.synchronize()
    for rec in records:
        assert np.array_equal(rec.cpu().numpy().view(ref.RECORD).reshape(-1), want)
