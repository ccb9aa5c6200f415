"""True-class searches of more than sixteen states a level, which go on in device
memory, one wave each: genotypes picked for it (levels of up to 551 states), their
verdicts and state counts against the search by levels and the oracle's, with
limits on the states and on the states of a level that end the search in device
memory too.  (All of these find an event or a second shape: no deterministic
genotype among 10^8 needed a search that wide, since guarded shapes need none.)"""
import numpy as np
import pytest

from oracle import ref
from tests.test_gpu_truth_levels import levels

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

WIDE = {
    (3, 16): [0xdb6a01086, 0x9240b4543, 0x6dbf53220, 0x492073ca6, 0x249efa831],
    (3, 32): [0xdb6e2c3bb, 0x249bd9957, 0xb6d86cdd0, 0x9246adb39],
    (4, 16): [0x6eb2069e8610, 0x9345fb1b9a20, 0x864ffa265383, 0xa45f4c237fda, 0xd863d8164110,
              0x6de64742f106],
    (4, 32): [0xc9978e83ccf, 0xec368423edc5, 0xb620ffe6cdd4, 0xb4d184bd0ec8, 0x79f83f919c5],
}


@pytest.mark.parametrize("t,grid", sorted(WIDE))
@pytest.mark.parametrize("waves", [1, 64])
def test_wide_searches(t, grid, waves):
    import paper_2205_15311_amd as jt
    # among genotypes that need no search or a narrow one
    rng = np.random.default_rng(t * grid)
    gs = np.concatenate([np.array(WIDE[t, grid], dtype=np.uint64),
                         rng.integers(0, 1 << (12 * t), size=500, dtype=np.uint64)])
    order = rng.permutation(len(gs))
    x = torch.from_numpy(gs[order].view(np.int64)).cuda()
    seen = set()
    for max_level, cap in ((4096, 2000), (4096, 150), (4096, 250), (60, 2000), (17, 2000)):
        with jt.Truth(len(gs), max_level=max_level, waves=waves) as w:
            rec = w.true_class(x, t, 8, grid, cap=cap)
            torch.cuda.synchronize()
        got = np.empty(len(gs), dtype=ref.RECORD)
        got[order] = rec.cpu().numpy().view(ref.RECORD).reshape(-1)
        if (max_level, cap) == (4096, 2000):
            # (the oracle searches every genotype, so it may reach its own limit on the
            # states of one that the library proves)
            want = ref.true_class(gs, t, grid=grid, cap=cap)
            decided = want["cls"] != ref.TRUE_CAPPED
            assert decided.sum() > 490
            for f in ("cls", "size", "hash"):
                assert np.array_equal(got[f][decided], want[f][decided]), f
        for i, genome in enumerate(WIDE[t, grid]):
            cls, size, total, widest = levels(genome, t, 8, grid, cap, max_level)
            assert (got["cls"][i], got["size"][i], got["hash"][i], got["steps"][i]) == \
                (cls, size, 0, total), (hex(genome), max_level, cap)
            seen.add((cls, widest > 16))
    assert seen >= {(1, True), (-2, True)}
