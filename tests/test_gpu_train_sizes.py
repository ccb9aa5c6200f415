"""A training step's loss and gradients against the reference network at the
edges of the kernels' pieces: sixteen samples a workgroup, operand blocks of 32,
chunks of 128, and the splits of the batch (one below 512 samples, sixteen from
4096 on), one network taking them in an order that leaves a larger call's
activations behind each smaller one; and that a step has one result.

Tolerance: that of test_gpu_mlp.py for whole batches, plus four activations
that round to the other bf16 neighbour (2^-8 of one of 256 n values), which
small batches do not average away."""
import numpy as np
import pytest

from oracle import mlp_ref as M
from tests.test_gpu_mlp import GRAD_MAX, GRAD_REL, rel, sample, to_dev

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

SIZES = [5000, 4097, 4096, 1, 545, 15, 16, 513, 512, 17, 511, 31, 129, 33, 127, 128, 32, 2111]


def test_gradients_at_every_edge():
    import paper_2205_15311_amd as jt
    p = M.random_params(5, scale=0.7)
    with jt.MLP(5000) as net:
        net.set_params(torch.from_numpy(M.flatten(p).astype(np.float32)).cuda())
        for n in SIZES:
            g, t, cls, size = sample(n, n)
            dg, dt, lab = to_dev(g, t, cls, size)
            got = []
            for _ in range(2):
                loss = torch.full((1,), 7.0, device="cuda")
                net.train_step(dg, dt, lab, lr=0.0, loss=loss)
                _, grads = net.get_params(grads=True)
                got.append((loss.item(), grads.cpu().numpy()))
            assert got[0][0] == got[1][0] and np.array_equal(got[0][1], got[1][1]), n
            grads = M.unflatten(got[0][1].astype(np.float64))
            want_loss, want, _ = M.loss_and_grads(p, g, t, cls, size)
            assert abs(got[0][0] - want_loss) <= 1e-6 * abs(want_loss) + 2.0 ** -8 / n, n
            for k in M.ORDER:
                assert rel(grads[k], want[k]) <= GRAD_REL + 2.0 ** -8 * (4 / (256 * n)) ** 0.5, \
                    (n, k, rel(grads[k], want[k]))
                assert np.abs(grads[k] - want[k]).max() <= \
                    (GRAD_MAX + 2.0 ** -7 / n ** 0.5) * np.abs(want[k]).max(), (n, k)


@pytest.mark.parametrize("n", [1, 15, 17, 33, 300])
def test_forward_is_the_same_alone(n):
    import paper_2205_15311_amd as jt
    g, t, cls, size = sample(400, 3)
    dg, dt, _ = to_dev(g, t, cls, size)
    with jt.MLP(64) as net:      # pieces of at most 64 samples
        net.init(9)
        full = net.forward(dg, dt)
        part = net.forward(dg[:n].contiguous(), dt[:n].contiguous())
        assert torch.equal(full[:n], part)
