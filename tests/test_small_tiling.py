"""The automatic tile shape and fusion depth of small problems (one or two tiles per
CU): host-side, every choice is a supported shape whose tiles fit the 256 CUs once
(tiles of 4 rows a wave: twice), or the default depth and region; on the GPU, an automatic call equals the 8 x 8 tile with 8
fused iterations bit for bit at the sizes where the choice changes."""
import numpy as np
import pytest

import paper_2109_05496_amd as ctv

SHAPES = {(8, 8), (12, 4), (8, 4), (16, 4)}


def tiles(m, n, batch, T, rows):
    return -(-n // (64 - 2 * T)) * -(-m // (rows - 2 * T)) * min(batch, 32)


@pytest.mark.parametrize("batch", [1, 3, 31, 40])
def test_choice_fits_the_cus_or_is_the_default(batch):
    ctv.tune_cache_clear()
    rng = np.random.default_rng(batch)
    sizes = [(1, 1), (1, 100000), (64, 64), (700, 700), (705, 700), (2048, 2048)]
    sizes += [tuple(int(v) for v in np.exp(rng.uniform(0, np.log(3000), 2))) for _ in range(60)]
    seen = set()
    for m, n in sizes:
        m, n = max(m, 1), max(n, 1)
        for K in (1, 2, 7, 20, 100):
            T, rows, w, rp = ctv.tiling(0, K, m, n, batch=batch, detail=True)
            assert (w, rp) in SHAPES and rows == w * rp and 1 <= T <= K and T < rows // 2 - 1
            if (w * rp, T) != (64, min(8, K)):
                two = rp == 4 and (w < 16 or T >= 8)
                assert tiles(m, n, batch, T, rows) <= (512 if two else 256), (m, n, K)
            seen.add((w, rp))
    assert len(seen) > 1


@pytest.mark.gpu
@pytest.mark.parametrize("batch,m,n", [(1, 9, 70), (1, 64, 64), (1, 200, 129), (2, 330, 332), (1, 700, 700), (1, 705, 700), (1, 850, 850),
                                       (33, 64, 65)])
def test_automatic_choice_equals_the_default_tile(batch, m, n):
    import torch
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctv.tune_cache_clear()
    g = torch.Generator(device="cuda").manual_seed(m + n)
    b = torch.view_as_complex(torch.randn(batch, m, n, 2, device="cuda", generator=g)).contiguous()
    mask = (torch.rand(m, n, device="cuda", generator=g) < 0.6).to(torch.uint8)
    mask[m // 3:] = 0
    for kind, support, K in (("1i", None, 23), ("2a", mask, 23), ("1a", mask, 5), ("2i", None, 1)):
        kw = dict(kind=kind, alpha=0.3, support=support, iters=K)
        x, gap = ctv.denoise(b, 0.06, gap=True, **kw)
        ref, gap_ref = ctv.denoise(b, 0.06, gap=True, fuse=8, tile=(8, 8), **kw)
        torch.cuda.synchronize()
        assert torch.equal(torch.view_as_real(x).view(torch.int32), torch.view_as_real(ref).view(torch.int32)), (kind, K)
        assert torch.equal(gap, gap_ref)
    xc, saved = ctv.denoise(b, 0.06, iters=23, ckpt_every=6)
    ref, saved_ref = ctv.denoise(b, 0.06, iters=23, ckpt_every=6, fuse=8, tile=(8, 8))
    assert torch.equal(torch.view_as_real(xc), torch.view_as_real(ref)) and torch.equal(saved, saved_ref)
