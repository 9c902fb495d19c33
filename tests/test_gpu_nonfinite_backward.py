"""The backward pass with values that are not finite: which entries of the gradients are
NaN or infinite is what a float64 evaluation gives that selects the differences that leave
the image and takes a NaN scale as 1, so a NaN reaches no gradient through a dual that
does not exist."""
import numpy as np
import pytest

torch = pytest.importorskip("torch")
pytestmark = [pytest.mark.gpu,
              pytest.mark.skipif(not torch.cuda.is_available(), reason="needs a GPU")]

INF, NAN = float("inf"), float("nan")
SHAPES = [(1, 1), (1, 50), (50, 1), (3, 70), (64, 64), (100, 131)]


def scale(n2, rho=1.0):
    """min(1, rho / |v|); 1 for a NaN, 0 for rho = 0."""
    s = np.minimum(1.0, rho / np.sqrt(np.where(n2 == 0, 1e-300, n2)))
    return np.where(np.isnan(n2), 1.0, s)


class Reference:
    """The K-step map of one image and its transpose; duals are arrays [4, m, n]."""

    def __init__(self, kind, alpha, constraint, mask, lam):
        self.kind, self.mod, self.lam = kind, constraint == "modulus", lam
        self.ra, self.sa = (alpha, 1 - alpha) if kind[0] == "2" else (1.0, 1.0)
        self.mask, self.c = mask, 1 / (8 * lam)

    @staticmethod
    def diff(y):
        """L y, 0 where the neighbour does not exist; [4, m, n] of [2, m, n]."""
        d = np.zeros((4,) + y.shape[1:])
        d[0:2, :-1] = y[:, :-1] - y[:, 1:]
        d[2:4, :, :-1] = y[:, :, :-1] - y[:, :, 1:]
        return d

    @staticmethod
    def div(v):
        up, left = np.zeros_like(v[0:2]), np.zeros_like(v[2:4])
        up[:, 1:] = v[0:2, :-1]
        left[:, :, 1:] = v[2:4, :, :-1]
        return (v[0:2] - up) + (v[2:4] - left)

    @staticmethod
    def exists(v):
        v = v.copy()
        v[0:2, -1] = 0
        v[2:4, :, -1] = 0
        return v

    def project(self, w):
        if not self.mod:
            return np.where(self.mask, w, 0.0), np.ones(w.shape[1:])
        s = scale(w[0] * w[0] + w[1] * w[1])
        return w * np.where(self.mask, s, 0.0), s

    def project_vjp(self, w, s, yb):
        o = yb
        if self.mod:
            d = (w[0] * yb[0] + w[1] * yb[1]) * (s * s)
            o = np.where(s < 1, s * (yb - w * d), yb)
        return np.where(self.mask, o, 0.0)

    def groups(self):
        return {"1i": [((0, 1, 2, 3), 1.0)], "1a": [((0, 1), 1.0), ((2, 3), 1.0)],
                "2i": [((0, 2), self.ra), ((1, 3), self.sa)],
                "2a": [((0,), self.ra), ((1,), self.sa), ((2,), self.ra), ((3,), self.sa)]}[self.kind]

    def ball(self, g):
        o = np.empty_like(g)
        for ix, rho in self.groups():
            v = g[list(ix)]
            if self.kind == "2a":
                o[ix[0]] = np.where(np.isnan(v[0]), -rho, np.clip(v[0], -rho, rho))
            else:
                o[list(ix)] = v * scale((v * v).sum(0), rho)
        return o

    def ball_vjp(self, g, a):
        o = np.empty_like(g)
        for ix, rho in self.groups():
            v, x = g[list(ix)], a[list(ix)]
            if self.kind == "2a":
                o[ix[0]] = np.where(np.abs(v[0]) <= rho, x[0], 0.0)
                continue
            n2 = (v * v).sum(0)
            s = scale(n2, rho)
            d = (v * x).sum(0) * (s * s) if self.kind == "1i" else (v * x).sum(0) / np.where(s < 1, n2, 1.0)
            o[list(ix)] = np.where(s < 1, s * (x - v * d), x)
        return o

    def gradients(self, b, xbar, K):
        q = r = np.zeros((4,) + b.shape[1:])
        rs, betas, t = [], [], 1.0
        for _ in range(K):
            rs.append(r)
            y, _ = self.project(b - self.lam * self.div(r))
            g = self.exists(r + self.c * self.diff(y))
            tn = (1 + np.sqrt(1 + 4 * t * t)) / 2
            d = self.ball(g) - q
            betas.append((t - 1) / tn)
            q = q + d
            r, t = q + betas[-1] * d, tn
        dd = self.div(q)
        w = b - self.lam * dd
        _, s = self.project(w)
        wbar = self.project_vjp(w, s, xbar)
        bbar, lbar = wbar, -(wbar * dd).sum()
        A, B = -self.lam * self.diff(wbar), np.zeros_like(q)
        for k in range(K - 1, -1, -1):
            r, beta = rs[k], betas[k - 1] if k else 0.0
            dd = self.div(r)
            w = b - self.lam * dd
            y, s = self.project(w)
            l = self.diff(y)
            gbar = self.exists(self.ball_vjp(self.exists(r + self.c * l), A))
            lbar -= (gbar * l).sum() / (8 * self.lam ** 2)
            wbar = self.project_vjp(w, s, self.c * self.div(gbar))
            bbar = bbar + wbar
            lbar -= (wbar * dd).sum()
            rbar = self.exists(gbar - self.lam * self.diff(wbar))
            A, B = B + (1 + beta) * rbar, -beta * rbar
        return bbar, lbar


def pair(z):
    return np.stack([z.real, z.imag]).astype(np.float64)


@pytest.mark.parametrize("shape", SHAPES)
@pytest.mark.parametrize("kind", ["1i", "1a", "2i", "2a"])
@pytest.mark.parametrize("constraint", ["none", "modulus"])
def test_gradients_of_special_values(kind, constraint, shape):
    import paper_2109_05496_amd as ctv
    m, n = shape
    rng = np.random.default_rng(m * 1000 + n)
    for K, ckpt, masked in ((1, 10, False), (7, 3, False), (12, 10, True)):
        mask = rng.random(shape) < 0.8 if masked else np.ones(shape, bool)
        for name, v in (("inf", complex(INF, 0.3)), ("nan i", complex(0.2, NAN))):
            for j, k in ((0, 0), (m - 1, n - 1), (m // 2, n - 1), (0, n // 2)):
                for where in ("b", "grad"):
                    z = [(rng.standard_normal(shape) + 1j * rng.standard_normal(shape)).astype(np.complex64)
                         for _ in range(2)]
                    z[where == "grad"][j, k] = v
                    b, gx = (torch.as_tensor(a).cuda() for a in z)
                    kw = dict(kind=kind, alpha=0.35, constraint=constraint, iters=K, ckpt_every=ckpt,
                              support=torch.as_tensor(mask.astype(np.uint8)).cuda() if masked else None)
                    _, saved = ctv.denoise(b, 0.07, **kw)
                    gb, gl = ctv.denoise_backward(b, 0.07, gx, saved, **kw)
                    torch.cuda.synchronize()
                    with np.errstate(all="ignore"):
                        eb, el = Reference(kind, 0.35, constraint, mask, 0.07).gradients(pair(z[0]), pair(z[1]), K)
                    what = (K, ckpt, masked, name, j, k, where)
                    gb = pair(gb.cpu().numpy())
                    assert np.array_equal(np.isnan(gb), np.isnan(eb)), what
                    assert np.array_equal(np.isinf(gb), np.isinf(eb)), what
                    assert np.isnan(gl.item()) == np.isnan(el), what
                    # One projection that rounding switches changes a few pixels by O(1): only
                    # in the largest image is that a small part of the norm.
                    ok = np.isfinite(eb)
                    if m * n > 10000:
                        assert np.linalg.norm(gb[ok] - eb[ok]) <= 0.05 * np.linalg.norm(eb[ok]), what


def test_one_pixel():
    """No difference exists in a 1 x 1 image: x = b, so dL/db = dL/dx and dL/dlambda = 0."""
    import paper_2109_05496_amd as ctv
    gx = torch.tensor([[0.7 - 1.3j]], dtype=torch.complex64, device="cuda")
    for v in (complex(INF, -2.0), complex(NAN, 1.0)):
        b = torch.tensor([[v]], dtype=torch.complex64, device="cuda")
        for kind in ("1i", "1a", "2i", "2a"):
            kw = dict(kind=kind, constraint="none", iters=7, ckpt_every=3)
            _, saved = ctv.denoise(b, 0.1, **kw)
            gb, gl = ctv.denoise_backward(b, 0.1, gx, saved, **kw)
            assert torch.equal(gb, gx) and gl.item() == 0.0


def test_checkpoint_with_duals_that_do_not_exist():
    """Such entries of a checkpoint enter the first y only, whatever the interval's launches."""
    import paper_2109_05496_amd as ctv
    rng = np.random.default_rng(3)
    m, n, K, ckpt = 40, 75, 6, 3
    b, gx = (torch.as_tensor((rng.standard_normal((m, n)) + 1j * rng.standard_normal((m, n))).astype(np.complex64)).cuda()
             for _ in range(2))
    for kind in ("1i", "2i"):
        kw = dict(kind=kind, alpha=0.4, iters=K, ckpt_every=ckpt)
        _, saved = ctv.denoise(b, 0.07, **kw)
        plain = ctv.denoise_backward(b, 0.07, gx, saved, **kw)[0]
        st = saved.view(1, 2, m, n, 4).clone()
        st[:, 0, -1, :, 0] = 0.5   # q: gone after one iteration, and r = q + beta (q - q') with it
        st[:, 0, :, -1, 3] = 0.5
        other = ctv.denoise_backward(b, 0.07, gx, st.view(-1), **kw)[0]
        torch.cuda.synchronize()
        assert bool(torch.isfinite(torch.view_as_real(other)).all())
        # far from the last row and column (6 iterations, 6 reverse steps) nothing changes
        assert torch.equal(plain[:m - 14, :n - 14], other[:m - 14, :n - 14])
