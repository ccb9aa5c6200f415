"""Top-k selection against a sort at the edges of its pieces: threads and blocks
(256 items a step, 1,024 a block, 128 blocks until each has 8,192), one and all of
the scores, scores that differ only in one digit of the radix select, that are all
equal, and that hold NaN, infinities and both zeros."""
import numpy as np
import pytest

from tests.test_gpu_screen import top_k_reference

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


def scores(kind, n, rng):
    if kind == "normal":
        return rng.standard_normal(n).astype(np.float32)
    if kind == "equal":
        return np.full(n, -0.25, dtype=np.float32)
    if kind == "special":
        s = rng.choice(np.array([np.nan, np.inf, -np.inf, 0.0, -0.0, 1.0], dtype=np.float32), n)
        return s
    # neighbours in the key: one of the three digits varies
    shift = {"low": 0, "middle": 10, "high": 21}[kind]
    u = np.uint32(0x3F800000) ^ (rng.integers(0, 700, size=n, dtype=np.uint32) << np.uint32(shift))
    return u.view(np.float32)


@pytest.mark.parametrize("kind", ["normal", "equal", "special", "low", "middle", "high"])
def test_select_top_at_edges(kind):
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(len(kind))
    sizes = [1, 255, 256, 257, 1023, 1024, 1025, 5000, 131_071, 131_072, 131_073, 1_048_579]
    with jt.GA(max(sizes)) as ga:
        for n in sizes:
            s = scores(kind, n, rng)
            dev = torch.from_numpy(s).cuda()
            for k in {1, max(1, n // 3), n}:
                got = ga.select_top(dev, k).cpu().numpy()
                assert np.array_equal(got, top_k_reference(s, k)), (n, k)


def test_select_top_of_many_blocks():
    import paper_2205_15311_amd as jt
    n = (1 << 23) + 12_345   # the largest number of blocks
    s = np.random.default_rng(2).integers(0, 5000, size=n).astype(np.float32)
    with jt.GA(n) as ga:
        got = ga.select_top(torch.from_numpy(s).cuda(), n // 2).cpu().numpy()
    assert np.array_equal(got, top_k_reference(s, n // 2))
