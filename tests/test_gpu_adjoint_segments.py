"""The gradient does not depend on how the iterations are cut into recomputed segments:
segments of one launch and of several (more than 12 iterations), one and many reverse
launches, with and without a final state kept for the output step."""
import pytest

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("shape", [(1, 1, 1), (2, 30, 62), (1, 31, 63), (1, 95, 190)])
@pytest.mark.parametrize("kind,masked", [("1i", False), ("1a", True), ("2i", False), ("2a", True)])
def test_gradients_do_not_depend_on_the_segments(shape, kind, masked):
    import torch
    import paper_2109_05496_amd as ctv
    from paper_2109_05496_amd.api import denoise_backward
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    B, m, n = shape
    K, lam = 29, [0.07] * B
    g = torch.Generator(device="cuda").manual_seed(m * n)
    draw = lambda: torch.view_as_complex(torch.randn(B, m, n, 2, device="cuda", generator=g)).contiguous()
    b, gx = draw(), draw()
    support = (torch.rand(m, n, device="cuda", generator=g) < 0.6).to(torch.uint8) if masked else None
    got = []
    for ckpt in (1, 4, 6, 13, 14, 27, 29, 40):
        x, saved = ctv.denoise(b, lam, kind=kind, alpha=0.4, support=support, iters=K, ckpt_every=ckpt)
        gb, gl = denoise_backward(b, lam, gx, saved, kind, 0.4, "modulus", support, K, 0, ckpt, "fgp")
        torch.cuda.synchronize()
        got.append((torch.view_as_real(gb).clone(), gl.double().clone()))
    for gb, gl in got[1:]:
        assert torch.equal(gb, got[0][0])
        # float64 partial sums in another order, rounded once to float32
        assert torch.all((gl - got[0][1]).abs() <= 2.0**-23 * got[0][1].abs().clamp(min=1.0))
