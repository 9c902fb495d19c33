"""More tiles than CUs: the automatic 64 x 64 region runs as 16 waves x 4 rows. Results
equal the 8 x 8 form's bit for bit (plain, masked, checkpointed, continued from a
state, ragged plans), on images whose last tiles hold one row or column, and fewer."""
import numpy as np
import pytest

pytestmark = pytest.mark.gpu


def bits(t):
    import torch
    t = torch.view_as_real(t) if t.is_complex() else t
    return t.contiguous().view(torch.int32) if t.dtype == torch.float32 else t


@pytest.mark.parametrize("batch,m,n", [(1, 769, 817), (1, 1500, 1345), (30, 97, 145), (32, 49, 480)])
@pytest.mark.parametrize("kind,masked", [("1i", False), ("1a", True), ("2i", False), ("2a", True)])
def test_automatic_equals_8x8(batch, m, n, kind, masked):
    import torch
    import paper_2109_05496_amd as ctv
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctv.tune_cache_clear()
    g = torch.Generator(device="cuda").manual_seed(m + n)
    b = torch.view_as_complex(torch.randn(batch, m, n, 2, device="cuda", generator=g)).contiguous()
    support = (torch.rand(m, n, device="cuda", generator=g) < 0.6).to(torch.uint8) if masked else None
    if masked:
        support[m // 2:] = 0
    for constraint in ("modulus", "none"):
        kw = dict(kind=kind, alpha=0.3, support=support, constraint=constraint, iters=17)
        x, gap, st = ctv.denoise(b, 0.06, gap=True, return_state=True, **kw)
        rx, rgap, rst = ctv.denoise(b, 0.06, gap=True, return_state=True, fuse=8, tile=(8, 8), **kw)
        assert torch.equal(bits(x), bits(rx)) and torch.equal(gap, rgap) and torch.equal(bits(st), bits(rst))
    y = ctv.denoise(b, 0.06, state=st, k0=17, **kw)
    ry = ctv.denoise(b, 0.06, state=rst, k0=17, fuse=8, tile=(8, 8), **kw)
    assert torch.equal(bits(y), bits(ry))
    z, saved = ctv.denoise(b, 0.06, ckpt_every=5, **kw)
    rz, rsaved = ctv.denoise(b, 0.06, ckpt_every=5, fuse=8, tile=(8, 8), **kw)
    assert torch.equal(bits(z), bits(rz)) and torch.equal(bits(saved), bits(rsaved))


@pytest.mark.parametrize("ckpt", [8, 9, 11, 12])
def test_checkpoint_interval_in_one_launch_equals_8x8(ckpt):
    import torch
    import paper_2109_05496_amd as ctv
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctv.tune_cache_clear()
    g = torch.Generator(device="cuda").manual_seed(ckpt)
    b = torch.view_as_complex(torch.randn(2, 601, 517, 2, device="cuda", generator=g)).contiguous()
    support = (torch.rand(601, 517, device="cuda", generator=g) < 0.6).to(torch.uint8)
    support[:100] = 0
    for kind, mask, K in (("1i", None, 2 * ckpt), ("2a", support, 2 * ckpt + 3), ("1a", support, ckpt), ("2i", None, 7)):
        kw = dict(kind=kind, alpha=0.3, support=mask, iters=K, ckpt_every=ckpt, gap=True)
        x, gap, saved = ctv.denoise(b, 0.06, **kw)
        rx, rgap, rsaved = ctv.denoise(b, 0.06, fuse=8, tile=(8, 8), **kw)
        assert torch.equal(bits(x), bits(rx)) and torch.equal(gap, rgap), (kind, K)
        assert (saved is None and rsaved is None) or torch.equal(bits(saved), bits(rsaved)), (kind, K)


@pytest.mark.parametrize("count,lo,hi", [(3, 500, 700), (60, 40, 200)])
def test_ragged_plan_equals_8x8(count, lo, hi):
    import torch
    import paper_2109_05496_amd as ctv
    if not torch.cuda.is_available():
        pytest.skip("needs a GPU")
    ctv.tune_cache_clear()
    rng = np.random.default_rng(count)
    kinds = ("1i", "1a", "2i", "2a")
    imgs = [dict(m=int(rng.integers(lo, hi)), n=int(rng.integers(lo, hi)), lam=float(rng.uniform(0.02, 0.2)),
                 kind=kinds[i % 4], alpha=0.4, iters=int(rng.integers(9, 30)), has_support=i % 3 == 0)
            for i in range(count)]
    g = torch.Generator(device="cuda").manual_seed(count)
    cuda = dict(device="cuda", generator=g)
    bs = [torch.view_as_complex(torch.randn(i["m"], i["n"], 2, **cuda)).cpu().numpy() for i in imgs]
    masks = [(torch.rand(i["m"], i["n"], **cuda) < 0.6).to(torch.uint8) for i in imgs if i["has_support"]]
    out = []
    for kw in (dict(), dict(fuse=8, tile=(8, 8))):
        plan = ctv.BatchedPlan(imgs, **kw)
        out.append(bits(plan.run(plan.pack(bs), plan.pack_support(masks))).clone())
        if not kw:
            assert plan.tiling == (8, 16, 4)
        torch.cuda.synchronize()
        plan.close()
    assert torch.equal(out[0], out[1])
