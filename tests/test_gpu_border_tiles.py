"""Column tiles at the image's border (every tile of a small image): their rows
are read and written through bounds-checked row buffers and the differences that
leave the image have a zero step instead of selects. x and the dual state must
equal the LDS-staged tile's bit for bit (its border handling is by selects), and
nothing may be written past x. Sizes put the last row and column first, last and
alone in a tile (outputs of a tile: 64 - 2 halo columns and rows)."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

GUARD = 4096
SHAPES = [(1, 1), (1, 59), (59, 1), (57, 59), (58, 58), (59, 57), (64, 64), (115, 117), (117, 115)]


@pytest.mark.parametrize("kind", ["1i", "1a", "2i", "2a"])
@pytest.mark.parametrize("shape", SHAPES)
def test_border_tiles_equal_the_lds_tile_and_stay_inside(kind, shape):
    import paper_2109_05496_amd as ctv
    m, n = shape
    rng = np.random.default_rng(m * 1000 + n)
    b = torch.as_tensor((rng.standard_normal((2, m, n)) + 1j * rng.standard_normal((2, m, n))).astype(np.complex64)).cuda()
    mask = torch.as_tensor((rng.random((m, n)) < 0.7).astype(np.uint8)).cuda()
    for constraint in ("modulus", "none"):
        for support in (None, mask):
            kw = dict(kind=kind, alpha=0.35, constraint=constraint, support=support, iters=7, return_state=True)
            ref, st_ref = ctv.denoise(b, 0.07, fuse=3, tile=(-1, 8), **kw)
            for tile in ((8, 8), (12, 4), (8, 4)):
                flat = torch.full((2 * GUARD + b.numel(),), 7.0, dtype=torch.complex64, device="cuda")
                out = flat[GUARD:GUARD + b.numel()].view(2, m, n)
                x, st = ctv.denoise(b, 0.07, fuse=3, tile=tile, out=out, **kw)
                torch.cuda.synchronize()
                assert torch.equal(torch.view_as_real(x).view(torch.int32), torch.view_as_real(ref).view(torch.int32)), tile
                assert torch.equal(st.view(torch.int32), st_ref.view(torch.int32)), tile
                assert bool((flat[:GUARD] == 7.0).all()) and bool((flat[GUARD + b.numel():] == 7.0).all()), tile
