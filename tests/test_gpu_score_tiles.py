"""A sample's predicted score does not depend on the call it is in: the same
bits whether the call gives a wave 16, 32 or 64 samples, at tile edges, alone or
among others, for every kind, with per-sample tile counts (out of range ones
read as no tiles) or one for all.  The scores themselves are checked against a
reference network in test_gpu_screen.py; here the largest call is, too."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = pytest.mark.gpu

N = 200_003   # more samples than one round of 64 a wave on 256 CUs


@pytest.mark.parametrize("t", [1, 2, 3, None])
def test_scores_do_not_depend_on_the_call(t):
    import paper_2205_15311_amd as jt
    g = torch.Generator().manual_seed(11)
    genomes = torch.randint(0, 1 << (12 * (t or 3)), (N,), generator=g, dtype=torch.int64).cuda()
    tiles = t if t is not None else torch.randint(0, 6, (N,), generator=g,
                                                  dtype=torch.uint8).cuda()
    at = (lambda a, b: t) if t is not None else (lambda a, b: tiles[a:b].contiguous())
    net = jt.MLP(64)
    net.init(3)
    for kind in (jt.PREDICT_SCREEN, jt.PREDICT_COST, jt.PREDICT_P_UNBOUND):
        full = net.predict(genomes, tiles, kind)
        for n in (1, 15, 16, 17, 64, 65, 4097, 32_768, 32_769, 65_536, 65_537, 131_136):
            for a in (0, N - n):
                part = net.predict(genomes[a:a + n].contiguous(), at(a, a + n), kind)
                assert torch.equal(part.view(torch.int32), full[a:a + n].view(torch.int32)), \
                    (kind, n, a)
        # the training path's outputs: h1 and h2 can round the other way in
        # their last bf16 bit where the fp32 sums' order matters
        o = net.forward(genomes[:4096].contiguous(), at(0, 4096)).double().cpu()
        p = torch.softmax(o[:, :3], dim=1)
        want = {jt.PREDICT_SCREEN: p[:, 2] * o[:, 3].exp() - 1.0,
                jt.PREDICT_COST: o[:, 3].exp() - 1.0,
                jt.PREDICT_P_UNBOUND: p[:, 0]}[kind]
        err = (full[:4096].double().cpu() - want).abs() / (1.0 + want.abs())
        assert err.max() < 1e-2 and np.median(err.numpy()) < 1e-5
