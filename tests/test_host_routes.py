"""Which kernels a classification call launches, by its size and the workspace's
parameters: the host code alone, with stand-ins for the launches.  The records
are the same on every route; the autotuner has to time one of them only, and what
it finds must not take the faster route away from small calls."""
import ctypes

import pytest

from tests import host_api

SMALL, LARGE = 1 << 12, (1 << 20) + 1
ONE, PIPE = (1, 0, 0, 0), (0, 1, 0, 0)


class Tuning(ctypes.Structure):
    _fields_ = [(n, ctypes.c_int) for n in (
        "refill", "first_waves", "repeat_waves", "wide_layout", "claim_share", "claim_chunks",
        "repeat_mapping")]


@pytest.fixture(scope="module")
def lib(tmp_path_factory):
    return host_api.build(tmp_path_factory.mktemp("host"))


@pytest.fixture
def host(lib):
    h = host_api.Host(lib)
    h.solo_ms, h.pipeline_ms, h.fast_refill = 1.0, 2.0, 0
    return h


class Batch:
    def __init__(self, host):
        self.host, self.lib = host, host.lib
        self.h = ctypes.c_void_p()
        assert self.lib.jatam_batch_create(ctypes.c_int64(LARGE), ctypes.byref(self.h)) == 0
        self.mem = ctypes.create_string_buffer(64)   # an address; nothing is read or written

    def tuning(self, grid):
        t = Tuning()
        assert self.lib.jatam_batch_get_tuning(self.h, grid, ctypes.byref(t)) == 0
        return t

    def set_tuning(self, grid, **fields):
        t = self.tuning(grid)
        for k, v in fields.items():
            setattr(t, k, v)
        assert self.lib.jatam_batch_set_tuning(self.h, grid, ctypes.byref(t)) == 0

    def range_(self, n, grid):
        return self.host.count(lambda: self.lib.jatam_batch_classify_range(
            self.h, ctypes.c_uint64(0), ctypes.c_int64(n), 2, 8, grid, 20, ctypes.c_uint64(1),
            self.mem, None, None))

    def list_(self, n, grid, t=2, c=8):
        return self.host.count(lambda: self.lib.jatam_batch_classify(
            self.h, self.mem, ctypes.c_int64(n), t, c, grid, 20, ctypes.c_uint64(1), self.mem,
            None, None))

    def items(self, n, tune=None):
        pair = (Tuning * 2)(*tune) if tune else None
        return self.host.count(lambda: self.lib.jatam_classify_batch(
            self.h, self.mem, ctypes.c_int64(n), 8, 20, ctypes.c_uint64(1), None, pair, self.mem,
            None, None))

    def enumerate_(self, slice_n, slices, grid, shapes=True):
        return self.host.count(lambda: self.lib.jatam_batch_enumerate(
            self.h, ctypes.c_uint64(0), ctypes.c_int64(slice_n), ctypes.c_int64(slices), 2, 8,
            grid, 20, ctypes.c_uint64(1), None, self.mem, self.mem if shapes else None,
            ctypes.c_int64(64 if shapes else 0), None))

    def autotune(self, n, grid=16):
        best = Tuning()
        got = self.host.count(lambda: self.lib.jatam_batch_autotune(
            self.h, ctypes.c_uint64(0), ctypes.c_int64(n), 2, 8, grid, 20, ctypes.c_uint64(1),
            self.mem, ctypes.byref(best), None))
        return best, got


@pytest.fixture
def batch(host):
    b = Batch(host)
    yield b
    host.lib.jatam_batch_destroy(b.h)


@pytest.mark.parametrize("t,c,grid,most", [
    (1, 8, 8, 1 << 20), (2, 8, 16, 1 << 20), (4, 16, 16, 1 << 20), (2, 8, 18, 1 << 18),
    (1, 8, 32, 1 << 18), (3, 8, 18, (1 << 20) - 1), (4, 8, 32, (1 << 20) - 1),
    (2, 16, 32, (1 << 20) - 1)])
def test_size_decides_by_default(batch, t, c, grid, most):
    for n in (1, SMALL, most):
        assert batch.list_(n, grid, t, c) == ONE
    for n in (most + 1, LARGE):
        assert batch.list_(n, grid, t, c) == PIPE
    assert batch.range_(SMALL, grid) == ONE and batch.range_(LARGE, grid) == PIPE


def test_size_decides_for_items(batch):
    assert batch.items(SMALL) == ONE and batch.items((1 << 20) - 1) == ONE
    assert batch.items(1 << 20) == PIPE and batch.items(LARGE) == PIPE


@pytest.mark.parametrize("n", [SMALL, 1 << 20, LARGE])
@pytest.mark.parametrize("grid", [16, 32])
def test_autotuner_times_the_pipeline_only(batch, host, n, grid):
    host.fast_refill = 32
    best, got = batch.autotune(n, grid)
    assert got[0] == 0 and got[1] >= 4 * 8       # baseline and trials alike
    assert best.refill == 32                     # found although the one launch is faster
    assert batch.tuning(grid).refill == 32


def test_tuned_parameters_leave_small_calls_the_one_launch(batch, host):
    host.fast_refill = 32
    for n in (SMALL, LARGE):
        batch.autotune(n)
        assert batch.range_(SMALL, 16) == ONE and batch.items(SMALL) == ONE
        assert batch.range_(LARGE, 16) == PIPE and host.last_refill == 32


def test_cached_parameters_leave_small_calls_the_one_launch(batch, host, tmp_path):
    host.fast_refill = 32
    path = str(tmp_path / "tuning.jsonl").encode()
    batch.set_tuning(16, refill=64)
    for hit in (0, 1):
        from_cache = ctypes.c_int(-1)
        assert host.lib.jatam_batch_autotune_cached(
            batch.h, path, ctypes.c_uint64(0), ctypes.c_int64(SMALL), 2, 8, 16, 20,
            ctypes.c_uint64(1), batch.mem, None, ctypes.byref(from_cache), None) == 0
        assert from_cache.value == hit and batch.tuning(16).refill == 32
        assert batch.range_(SMALL, 16) == ONE
        batch.set_tuning(16, refill=64)
        assert batch.range_(SMALL, 16) == PIPE and host.last_refill == 64


def test_chosen_parameters_run_the_pipeline_in_their_class(batch, host):
    batch.set_tuning(32, refill=8)
    assert batch.range_(SMALL, 16) == ONE        # the other class's parameters
    assert batch.range_(SMALL, 32) == PIPE and host.last_refill == 8
    assert batch.items(SMALL) == PIPE            # items may have either
    batch.set_tuning(32, refill=24)              # the defaults again
    assert batch.range_(SMALL, 32) == ONE and batch.items(SMALL) == ONE
    assert host.lib.jatam_batch_set_refill(batch.h, 25) == 0
    assert batch.range_(SMALL, 16) == PIPE and batch.list_(SMALL, 32) == PIPE


def test_parameters_of_one_call(batch, host):
    default = [batch.tuning(16), batch.tuning(32)]
    other = [batch.tuning(16), batch.tuning(32)]
    other[1].repeat_mapping = 1
    assert batch.items(SMALL, default) == ONE
    assert batch.items(SMALL, other) == PIPE
    batch.set_tuning(16, refill=25)
    assert batch.items(SMALL, default) == ONE and batch.items(SMALL) == PIPE


@pytest.mark.parametrize("grid", [16, 32])
def test_enumeration_runs_on_the_parameters_the_caller_chose(batch, host, grid):
    """One launch over all slices for G <= 16, or with chosen parameters of its
    class the slice pipeline, captured once and replayed."""
    one = ONE if grid == 16 else (0, 1, 1, 8)
    assert batch.enumerate_(SMALL, 8, grid) == one
    batch.set_tuning(48 - grid, refill=8)        # the other class's parameters
    assert batch.enumerate_(SMALL, 8, grid) == one
    host.fast_refill = 32
    batch.autotune(SMALL, grid)
    assert batch.enumerate_(SMALL, 8, grid) == one
    batch.set_tuning(grid, refill=25, repeat_mapping=1)
    assert batch.enumerate_(SMALL, 8, grid) == (0, 1, 1, 8)
    assert (host.last_refill, host.last_mapping, host.last_n) == (25, 1, SMALL)
    assert batch.enumerate_(SMALL, 8, grid, shapes=False) == (0, 1, 0, 8)
