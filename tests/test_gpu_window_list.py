"""The list of items that leave the 16 x 16 window, and the tally's counter
sets, through the ABI: some, none and all of a call's items leave, alone or
mixed with items of G <= 16, under every repeat mapping.  (Items that leave only
in a later run, after a clean first one, are listed by the repeat rounds; none
was found among millions of genotypes, where such growth always meets an
ambiguous site first.)  Records must equal the oracle's and the tally the
records' classes, added to what the caller held."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mapping", [0, 1, 2])
@pytest.mark.parametrize("pick", ["mixed", "none", "all"])
def test_items_that_leave_the_window(mapping, pick):
    import paper_2205_15311_amd as jt
    rng = np.random.default_rng(77)
    n, grid = 60_000, 32
    gs = rng.integers(0, 1 << 36, size=n, dtype=np.uint64)
    small = ref.classify(gs, 3, grid=16, runs=20, seed=1)   # the window's records
    gone = small["cls"] == 0
    keep = {"mixed": np.ones(n, bool), "none": ~gone, "all": gone}[pick]
    gs = np.ascontiguousarray(gs[keep][:20_000])
    g = np.full(len(gs), grid, dtype=np.uint8)
    if pick == "mixed":
        g[rng.random(len(gs)) < 0.4] = 14
    items = jt.make_items(gs, 3, g)
    want = np.empty(len(gs), dtype=ref.RECORD)
    for side in (14, grid):
        at = g == side
        if at.any():
            want[at] = ref.classify(np.ascontiguousarray(gs[at]), 3, grid=side, runs=20, seed=1)
    tally = torch.tensor([5, 6, 7, 8], dtype=torch.int64, device="cuda")
    with jt.Batch(len(gs)) as b:
        b.set_tuning(16, repeat_mapping=mapping)
        b.set_tuning(32, wide_layout=2, repeat_mapping=mapping)
        for _ in range(2):
            rec = b.classify_items(torch.from_numpy(items).cuda(), tally=tally)
        torch.cuda.synchronize()
    got = rec.cpu().numpy().view(ref.RECORD).reshape(-1)
    assert np.array_equal(got, want)
    counts = np.bincount(want["cls"], minlength=4)
    assert tally.cpu().tolist() == (np.array([5, 6, 7, 8]) + 2 * counts).tolist()
