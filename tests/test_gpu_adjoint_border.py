"""Reverse-step tiles at the image's border (row buffers, zero steps): gradients at
sizes that put the last row and column first, last and alone in a tile (outputs of
a tile: 64 - 2 halo columns, 32 - 2 halo rows, halo 2 .. 6) against the
FP64 oracle's reverse pass, at the stated relative 1e-4."""
import numpy as np
import pytest

from oracle import adjoint

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


@pytest.mark.parametrize("shape", [(1, 1), (1, 53), (21, 1), (20, 52), (21, 53), (41, 105), (40, 104)])
@pytest.mark.parametrize("kind,ckpt", [("1i", 9), ("1a", 1), ("2i", 4), ("2a", 5)])
def test_border_gradients_match_the_oracle(shape, kind, ckpt):
    import paper_2109_05496_amd as ctv
    m, n = shape
    rng = np.random.default_rng(m * 100 + n)
    b = (rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))).astype(np.complex64)
    gx = (rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))).astype(np.complex64)
    mask = (rng.random((m, n)) < 0.8).astype(np.uint8)
    K, lam, alpha = 9, 0.2, 0.4
    for support in (None, mask):
        mt = None if support is None else torch.as_tensor(support).cuda()
        kw = dict(kind=kind, alpha=alpha, support=mt, iters=K, ckpt_every=ckpt)
        _, saved = ctv.denoise(torch.as_tensor(b).cuda(), lam, **kw)
        gb, gl = ctv.denoise_backward(torch.as_tensor(b).cuda(), lam, torch.as_tensor(gx).cuda(), saved, **kw)
        _, rb, rl = adjoint.fgp_vjp(b.astype(np.complex128), lam, K, gx.astype(np.complex128), kind, alpha, "modulus",
                                    support)
        assert np.linalg.norm(gb.cpu().numpy() - rb) <= 1e-4 * max(np.linalg.norm(rb), 1e-3)
        assert abs(float(gl[0]) - rl) <= 1e-4 * max(abs(rl), 1.0)
