"""Shape counts of the one-launch enumeration where many deterministic shapes do
not fit an 8 x 8 bitmap (rows of nine cells and more): each wave collects them
by hash and size, eight at a time, before they go to the table.  Counts against
the oracle's records; and collecting them must not cost more than the
classification itself (one atomic each on one word of the table did)."""
import numpy as np
import pytest

from oracle import ref

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("t,first,n,slices,grid", [
    (3, (1 << 33) + (3 << 23), 1 << 16, 3, 16),     # rows of nine: one shape for many
    (3, (1 << 33) + (3 << 23) + 12345, 9_973, 5, 16),
    (4, 0x320000000000, 1 << 16, 1, 16),
    (3, 5 << 30, 1 << 16, 2, 12)])
def test_counts_of_large_shapes(t, first, n, slices, grid):
    import paper_2205_15311_amd as jt
    total = n * slices
    want = ref.classify_range(first, total, t, grid=grid, runs=20, seed=1)
    det = want[want["cls"] == 3]
    keys, counts = np.unique(det[["size", "hash"]], return_counts=True)
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    table = torch.zeros((4096, 2), dtype=torch.int64, device="cuda")
    with jt.Batch(n) as b:
        for _ in range(2):
            b.enumerate(first, n, slices, t, 8, grid, 20, 1, tally=tally, shapes=table)
        torch.cuda.synchronize()
    got = jt.shape_table_to_numpy(table)
    assert len(got) == len(keys) and (got["count"] == 2 * counts).all()
    assert (got["size"] == keys["size"]).all() and (got["hash"] == keys["hash"]).all()
    assert tally.cpu().tolist() == (2 * np.bincount(want["cls"], minlength=4)).tolist()


def test_counting_shapes_costs_less_than_finding_them():
    import paper_2205_15311_amd as jt
    n, first = 1 << 22, 1 << 33   # 75,000 rows of nine cells in eight slices
    tally = torch.zeros(4, dtype=torch.int64, device="cuda")
    table = torch.zeros((4096, 2), dtype=torch.int64, device="cuda")

    def ms(b, shapes):
        best = float("inf")
        for _ in range(6):
            x, y = torch.cuda.Event(enable_timing=True), torch.cuda.Event(enable_timing=True)
            x.record()
            b.enumerate(first, n, 8, 3, 8, 16, 20, 1, tally=tally, shapes=shapes)
            y.record()
            y.synchronize()
            best = min(best, x.elapsed_time(y))
        return best

    with jt.Batch(n) as b:
        plain, counted = ms(b, None), ms(b, table)
    print(f"{plain:.2f} ms without, {counted:.2f} ms with shape counts")
    assert counted < 2 * plain   # 1.0 times; 3.2 times with an atomic for each
