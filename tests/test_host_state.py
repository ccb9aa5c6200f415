"""What a call leaves behind when a launch or a runtime query of it fails: the host
code alone, with stand-ins for them (tests/host_stubs.cpp)."""
import ctypes

import pytest

from tests import host_api


@pytest.fixture
def host(tmp_path):
    """A copy of the library of its own: what it remembers belongs to one test."""
    return host_api.Host(host_api.build(tmp_path))


def test_failed_training_step_keeps_the_step_count(host):
    lib, net, mem = host.lib, ctypes.c_void_p(), ctypes.create_string_buffer(64)
    assert lib.jatam_mlp_create(ctypes.c_int64(64), 8, ctypes.byref(net)) == 0

    def train(lr):
        return lib.jatam_mlp_train_step(net, mem, None, 3, mem, ctypes.c_int64(8),
                                        ctypes.c_float(lr), None, None)

    assert train(1e-3) == 0 and host.last_step == 1
    host.fail_train = 2
    assert train(1e-3) == host_api.E_HIP and host.last_step == 2
    assert train(1e-3) == host_api.E_HIP and host.last_step == 2
    assert train(1e-3) == 0 and host.last_step == 2
    assert train(0.0) == 0 and host.last_step == 2      # gradients only
    assert train(1e-3) == 0 and host.last_step == 3
    lib.jatam_mlp_destroy(net)


def test_failed_device_query_is_asked_again(host):
    mem = ctypes.create_string_buffer(64)

    def classify():
        return host.lib.jatam_classify(mem, ctypes.c_int64(8), 2, 8, 16, 20, ctypes.c_uint64(1), mem,
                                       None)

    host.fail_attribute = 2
    assert classify() == host_api.E_HIP and classify() == host_api.E_HIP
    assert host.solo_launches == 0
    assert classify() == 0 and host.solo_launches == 1
    host.fail_attribute = 1          # known by now
    assert classify() == 0 and host.solo_launches == 2
