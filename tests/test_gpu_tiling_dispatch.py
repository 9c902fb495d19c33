"""The automatic tilings, each asserted to be the one that runs and compared bit for bit
with the 8 x 8 tile: 16 x 4 above three tiles per CU, an interval of 9 to 11 iterations
between checkpoints in one launch, and the list of live tiles with a fixed tile."""
import ctypes

import numpy as np
import pytest

from paper_2109_05496_amd import _lib

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]


def choice(m, n, iters, batch, ckpt):
    p = _lib.make_params("1i", iters=iters)
    out = [ctypes.c_int32() for _ in range(3)]
    _lib.call("ctv_tune_cache_clear")
    _lib.call("ctv_debug_tiling", ctypes.byref(p), batch, m, n, ckpt, 0, *(ctypes.byref(o) for o in out))
    return tuple(o.value for o in out)


def bits(t):
    t = torch.view_as_real(t) if t.is_complex() else t
    return t.contiguous().view(torch.int32) if t.dtype == torch.float32 else t


def inputs(batch, m, n, masked):
    g = torch.Generator(device="cuda").manual_seed(m * 7 + n)
    b = torch.view_as_complex(torch.randn(batch, m, n, 2, device="cuda", generator=g)).contiguous()
    if not masked:
        return b, None
    support = (torch.rand(m, n, device="cuda", generator=g) < 0.6).to(torch.uint8)
    support[m // 2:, : n // 2] = 0
    return b, support


@pytest.mark.parametrize("batch,m,n", [(1, 1500, 1345), (4, 769, 817), (30, 241, 337)])
@pytest.mark.parametrize("kind,masked", [("1i", False), ("1a", True), ("2i", True), ("2a", False)])
def test_16x4_above_three_tiles_per_cu(batch, m, n, kind, masked):
    import paper_2109_05496_amd as ctv
    assert choice(m, n, 17, batch, 0) == (8, 16, 4)
    b, support = inputs(batch, m, n, masked)
    for constraint in ("modulus", "none"):
        kw = dict(kind=kind, alpha=0.3, support=support, constraint=constraint, iters=17, gap=True, return_state=True)
        x, gap, st = ctv.denoise(b, 0.06, **kw)
        rx, rgap, rst = ctv.denoise(b, 0.06, fuse=8, tile=(8, 8), **kw)
        assert torch.equal(bits(x), bits(rx)) and torch.equal(gap, rgap) and torch.equal(bits(st), bits(rst))


@pytest.mark.parametrize("ckpt", [8, 9, 10, 11, 12])
@pytest.mark.parametrize("masked", [False, True])
def test_checkpoint_interval(ckpt, masked):
    import paper_2109_05496_amd as ctv
    batch, m, n = 4, 769, 817
    b, support = inputs(batch, m, n, masked)
    for kind, K in (("1i", 2 * ckpt), ("2a", 2 * ckpt + 3), ("2i", ckpt + 1)):
        assert choice(m, n, K, batch, ckpt) == (ckpt if 9 <= ckpt <= 11 else 8, 16, 4)
        kw = dict(kind=kind, alpha=0.3, support=support, iters=K, ckpt_every=ckpt, gap=True)
        x, gap, saved = ctv.denoise(b, 0.06, **kw)
        rx, rgap, rsaved = ctv.denoise(b, 0.06, fuse=8, tile=(8, 8), **kw)
        assert torch.equal(bits(x), bits(rx)) and torch.equal(gap, rgap) and torch.equal(bits(saved), bits(rsaved))


@pytest.mark.parametrize("shape,T", [((8, 8), 8), ((16, 4), 8), ((8, 4), 7)])
def test_supports_of_one_pixel_and_of_nothing_with_live_tiles(shape, T):
    """Tiles of at least 16 x 16 output pixels, which the lists are for; the automatic
    choice for this size has fewer rows and runs every tile."""
    import paper_2109_05496_amd as ctv
    m, n, K = 130, 190, 25
    b, _ = inputs(1, m, n, False)
    one = torch.zeros(m, n, dtype=torch.uint8, device="cuda")
    nothing = one.clone()
    one[77, 101] = 1
    ws_bytes = ctv.workspace_size(m, n, 1, iters=K)[0]
    for support in (nothing, one):
        kw = dict(kind="2i", support=support, iters=K)
        x = ctv.denoise(b, 0.1, **kw)
        for fill in (0xFF, 0):
            ws = torch.full((ws_bytes,), fill, dtype=torch.uint8, device="cuda")
            y = ctv.denoise(b, 0.1, tile=shape, fuse=T, workspace=ws, **kw)
            assert torch.equal(bits(x), bits(y)) and not bool(y[0][support == 0].any())
        _, saved = ctv.denoise(b, 0.1, tile=shape, fuse=T, ckpt_every=10, **kw)
        for s, k in enumerate((10, 20)):
            _, st = ctv.denoise(b, 0.1, tile=shape, fuse=T, return_state=True, **dict(kw, iters=k))
            assert torch.equal(bits(saved.view(2, -1)[s]), bits(st).view(-1))


@pytest.mark.parametrize("kind,ckpt", [("1i", 4), ("2a", 10)])
def test_backward_of_a_sparse_support_takes_nothing_from_the_workspace(kind, ckpt):
    """Three and more reverse launches: the adjoint state outside the live tiles is what
    the call itself put there, whatever the workspace held."""
    import paper_2109_05496_amd as ctv
    batch, m, n, K = 2, 260, 310, 23
    b, _ = inputs(batch, m, n, False)
    gx, _ = inputs(batch, n, m, False)
    gx = gx.transpose(1, 2).contiguous()
    support = torch.zeros(m, n, dtype=torch.uint8, device="cuda")
    support[90:130, 70:120] = 1
    support[m - 1, n - 1] = 1
    kw = dict(kind=kind, alpha=0.4, iters=K, support=support, ckpt_every=ckpt)
    _, saved = ctv.denoise(b, 0.06, **kw)
    p = _lib.make_params(kind, 0.4, "modulus", K)
    size = ctypes.c_size_t()
    _lib.call("ctv_backward_workspace_size", ctypes.byref(p), batch, m, n, ckpt, ctypes.byref(size))
    out = []
    for fill in (0xFF, 0x00, 0x3F):
        ws = torch.full((size.value,), fill, dtype=torch.uint8, device="cuda")
        gb, gl = torch.empty_like(b), torch.empty(batch, device="cuda")
        lam = (ctypes.c_float * batch)(0.06, 0.06)
        ptr = lambda t: ctypes.c_void_p(t.data_ptr())
        _lib.call("ctv_denoise_backward", ctypes.byref(p), batch, m, n, ptr(b), lam, ptr(support), ckpt, ptr(saved),
                  ptr(gx), ptr(gb), ptr(gl), ptr(ws), ws.numel(),
                  ctypes.c_void_p(torch.cuda.current_stream().cuda_stream))
        torch.cuda.synchronize()
        out.append((gb, gl))
    assert bool(out[0][0].abs().sum() > 0) and not bool(out[0][0][:, support == 0].any())
    for gb, gl in out[1:]:
        assert torch.equal(bits(gb), bits(out[0][0])) and torch.equal(gl, out[0][1])
