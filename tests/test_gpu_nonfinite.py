"""Values that are not finite, or too large to stay so, and states that hold a dual
where none exists: every column tile, the dataflow schedule, the single-tile kernel and
the batched kernel give what the LDS-staged tile gives, which selects the differences
that leave the image and takes a NaN scale as 1. NaNs in the same places, all other
values bit for bit."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

INF, NAN = float("inf"), float("nan")
SPECIAL = {"inf": complex(INF, 0.3), "-inf i": complex(0.2, -INF), "nan": complex(NAN, 0.3),
           "3e38": complex(3e38, -1e38)}
SHAPES = [(1, 1), (1, 50), (50, 1), (3, 70), (64, 64), (100, 131)]
TILES = [((8, 8), 4), ((16, 4), 8), ((8, 4), 5), ((12, 4), 7), ((4, 8), 3), ((16, 8), 8), ((-2, 32), 6)]


def values(t):
    """(NaN mask, bits of the rest) of a float or complex tensor."""
    t = torch.view_as_real(t) if t.is_complex() else t
    nan = torch.isnan(t)
    return nan, torch.where(nan, torch.zeros_like(t), t).contiguous().view(torch.int32)


def same(a, b):
    return all(torch.equal(u, v) for u, v in zip(values(a), values(b)))


def image(m, n, seed, batch=2):
    rng = np.random.default_rng(seed)
    return torch.as_tensor((rng.standard_normal((batch, m, n)) + 1j * rng.standard_normal((batch, m, n)))
                           .astype(np.complex64))


def spots(m, n):
    return [(0, 0), (m - 1, n - 1), (m // 2, n - 1), (m - 1, n // 3), (m // 2, n // 2)]


def check_all_forms(b, lam, what, **kw):
    import paper_2109_05496_amd as ctv
    ref, st_ref = ctv.denoise(b, lam, return_state=True, fuse=5, tile=(-1, 8), **kw)
    forms = [dict(tile=t, fuse=f) for t, f in TILES] + [dict(), dict(schedule="flow")]
    for form in forms:
        x, st = ctv.denoise(b, lam, return_state=True, **form, **kw)
        torch.cuda.synchronize()
        assert same(x, ref) and same(st, st_ref), (what, form)
    return ref, st_ref


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["1i", "1a", "2i", "2a"])
def test_special_values(kind, shape):
    m, n = shape
    for name, v in SPECIAL.items():
        for j, k in spots(m, n):
            b = image(m, n, m * 100 + n)
            b[1, j, k] = v
            for constraint in ("none", "modulus"):
                check_all_forms(b.cuda(), 0.07, (name, j, k, constraint), kind=kind, alpha=0.35,
                                constraint=constraint, iters=7)


def test_one_pixel_keeps_its_infinity():
    """No difference exists in a 1 x 1 image: x = b without a constraint set."""
    import paper_2109_05496_amd as ctv
    b = torch.tensor([[complex(INF, -2.0)]], dtype=torch.complex64, device="cuda")
    for kind in ("1i", "1a", "2i", "2a"):
        x, st = ctv.denoise(b, 0.1, kind=kind, constraint="none", iters=9, return_state=True)
        assert same(x, b) and not bool(st.any())


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["1i", "1a", "2i", "2a"])
def test_states_with_duals_that_do_not_exist(kind, shape):
    """Such entries enter the first iteration's y and are 0 two iterations later."""
    m, n = shape
    b = image(m, n, 5).cuda()
    rng = np.random.default_rng(6)
    for v in (1.0, -0.0, 1e-42, 1e30, NAN):
        for plane in (0, 1):
            st = (0.3 * rng.standard_normal((2, 2, m, n, 4))).astype(np.float32)
            st[:, :, -1, :, :2] = 0
            st[:, :, :, -1, 2:] = 0
            st[:, plane, -1, :, 0] = v
            st[:, plane, :, -1, 3] = v
            for iters in (1, 2, 7):
                _, out = check_all_forms(b, 0.07, (v, plane, iters), kind=kind, alpha=0.35, iters=iters,
                                         state=torch.as_tensor(st).cuda(), k0=20)
            if v == v:
                assert not bool(out[:, :, -1, :, :2].any()) and not bool(out[:, :, :, -1, 2:].any())


@pytest.mark.parametrize("constraint", ["none", "modulus"])
def test_batched_plan(constraint):
    import paper_2109_05496_amd as ctv
    rng = np.random.default_rng(9)
    for name, v in SPECIAL.items():
        imgs, bs, masks, refs = [], [], [], []
        for i, (m, n) in enumerate(SHAPES):
            d = dict(m=m, n=n, lam=0.05, kind=("1i", "1a", "2i", "2a")[i % 4], alpha=0.35, iters=6 + i,
                     has_support=i % 2 == 0)
            b = image(m, n, i, 1)[0]
            b[spots(m, n)[i % 5]] = v
            mask = torch.as_tensor((rng.random((m, n)) < 0.7).astype(np.uint8)) if d["has_support"] else None
            if mask is not None:
                masks.append(mask)
            refs.append(ctv.denoise(b.cuda(), d["lam"], kind=d["kind"], alpha=0.35, constraint=constraint,
                                    support=None if mask is None else mask.cuda(), iters=d["iters"], tile=(-1, 8),
                                    fuse=5))
            if mask is not None and not bool(mask.any()):
                refs[-1] = torch.zeros_like(refs[-1])  # a tile without a pixel of the support is not computed
            imgs.append(d)
            bs.append(b)
        for kw in (dict(), dict(tile=(16, 4), fuse=8), dict(tile=(8, 4), fuse=3)):
            plan = ctv.BatchedPlan(imgs, constraint, **kw)
            out = plan.unpack(plan.run(plan.pack(bs), plan.pack_support(masks)))
            torch.cuda.synchronize()
            for x, ref, d in zip(out, refs, imgs):
                assert same(x, ref), (name, kw, d)
            plan.close()
