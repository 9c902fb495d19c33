"""The gradient's fused column pass (forward DFT, times H_d, inverse DFT in one
launch), used for small problems and for one distance, and the loss summed beside
the accumulate pass: gradient and data term against the FP64 oracle at the stated
1e-5 on both sides of the sizes where the pass is chosen (2^18 elements over all
distances; 2^21 for one distance) and at the shortest and longest columns."""
import numpy as np
import pytest

from _parity import ELEM_TOL, elem, rel
from oracle import pr as opr

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("m,n,D", [(32, 32, 1), (32, 64, 3), (128, 32, 5), (256, 256, 1), (256, 256, 4), (256, 256, 5),
                                   (2048, 512, 1), (4096, 64, 1), (64, 4096, 1), (1024, 2048, 1)])
def test_gradient_matches_oracle_on_both_sides_of_the_rule(m, n, D):
    import paper_2109_05496_amd as ctv
    rng = np.random.default_rng(m + n + D)
    dists, lam, pix = [1e-3 + 4e-4 * d for d in range(D)], 532e-9, 4e-6
    x = (rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))).astype(np.complex64)
    y = (rng.random((D, m, n)) * 2.0).astype(np.float32)
    Hs = [opr.transfer(m, n, d, lam, pix) for d in dists]
    sy = [np.sqrt(v.astype(np.float64)) for v in y]
    xt, yt = torch.as_tensor(x).cuda(), torch.as_tensor(y).cuda()
    g, loss = ctv.pr_gradient(xt, yt, dists, lam, pix)
    gref = opr.grad_F(x.astype(np.complex128), sy, Hs)
    lref = opr.data_term(x.astype(np.complex128), sy, Hs)
    assert rel(g.cpu().numpy(), gref) <= 1e-5 and elem(g.cpu().numpy(), gref) <= ELEM_TOL
    assert abs(float(loss.cpu()[0]) - lref) <= 1e-5 * lref
