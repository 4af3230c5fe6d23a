"""One adjoint layer of the generalized-SP2 network against FP64, element by element.

With one layer nothing propagates: G_0 = W (G X + X G) + B G and the three gradients follow from the
FP32 operands in FP64, and each output has a bound of its own from its chain of FP32 operations.
The bounds are narrow enough to see one wrong 32 x 32 tile, which the CPU test checks on an FP32
stand-in and on mistakes planted in the reference."""
import numpy as np
import pytest

from paper_2101_06385_amd import sp2

U, U64 = 2.0**-24, 2.0**-53
W, B, C = 0.7, -0.4, 0.3


def _operands(n, signed):
    """G and X (FP32, symmetric).  Positive entries: no sum cancels, so a tile left out of a sum is
    far outside the sum's bound; signed ones: typical of training."""
    rng = np.random.default_rng(3000 + n)
    def sym():
        a = rng.standard_normal((n, n)) if signed else rng.uniform(0.25, 1.0, (n, n))
        return ((a + a.T) / (2 * np.sqrt(n))).astype(np.float32)
    return sym(), sym()


class _Reference:
    """FP64 values of (G_0, dW, dB, dC) and the bounds of the kernel's results."""

    def __init__(self, g32, x32):
        n = len(g32)
        w, b = float(np.float32(W)), float(np.float32(B))
        g, x = g32.astype(np.float64), x32.astype(np.float64)
        gx = g @ x
        self.terms = g, x, gx + gx.T
        m_abs = np.abs(g) @ np.abs(x)
        m_abs = m_abs + m_abs.T
        self.g0 = w * (gx + gx.T) + b * g
        # per element: n products and n sums in each of two chains, the sum of the chains, W M + B G
        self.g0_bound = (2 * n + 8) * U * (abs(w) * m_abs + abs(b) * np.abs(g)) + 1e-30
        # FP64 sums of FP32 values, rounded once; dW of the FP32 M
        self.dc, self.db, self.dw = np.trace(g), (g * x).sum(), 0.5 * ((gx + gx.T) * x).sum()
        sums = 2 * (n * n + 1) * U64
        self.dc_bound = U * abs(self.dc) + sums * np.abs(np.diag(g)).sum() + 1e-30
        self.db_bound = U * abs(self.db) + sums * (np.abs(g) * np.abs(x)).sum() + 1e-30
        self.dw_bound = U * abs(self.dw) + ((2 * n + 8) * U + sums) * 0.5 * (m_abs * np.abs(x)).sum() + 1e-30

    def without_tile(self, i, j):
        """The values with the 32 x 32 tile (i, j) of M, and its mirror, left out."""
        g, x, m = self.terms
        n = len(g)
        keep = np.ones((n, n))
        keep[32 * i:32 * i + 32, 32 * j:32 * j + 32] = 0.0
        keep[32 * j:32 * j + 32, 32 * i:32 * i + 32] = 0.0
        return self.g0 * keep, 0.5 * (m * x * keep).sum(), (g * x * keep).sum(), np.trace(g * keep)

    def wrong(self, g0, dw, db, dc):
        """Names of the outputs that are outside their bounds."""
        out = [k for k, bad in (("g0", np.any(np.abs(g0 - self.g0) > self.g0_bound)),
                                ("dw", abs(dw - self.dw) > self.dw_bound), ("db", abs(db - self.db) > self.db_bound),
                                ("dc", abs(dc - self.dc) > self.dc_bound)) if bad]
        return out


def _stand_in(g, x):
    """The layer in numpy's FP32."""
    gx = g @ x
    m = gx + gx.T
    w, b = np.float32(W), np.float32(B)
    gd, xd = g.astype(np.float64), x.astype(np.float64)
    return (w * m + b * g, np.float32(0.5 * (m.astype(np.float64) * xd).sum()), np.float32((gd * xd).sum()),
            np.float32(np.trace(gd)))


# one ragged tile, several cut ones (all of them up to 1408), whole 64-tiles with cut ones (1409: 256 + 20)
SIZES = [1, 31, 33, 65, 200, 1408, 1409]


@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("n", SIZES)
def test_bounds_hold_for_fp32_and_see_one_wrong_tile(n, signed):
    g, x = _operands(n, signed)
    ref = _Reference(g, x)
    assert ref.wrong(*_stand_in(g, x)) == []
    last = (n - 1) // 32
    whole = max(n // 32 - 1, 0)
    for i, j in {(0, 0), (0, last), (last // 2, last), (last, last), (0, whole), (whole, whole)}:
        wrong = ref.wrong(*ref.without_tile(i, j))
        assert "g0" in wrong, (i, j)
        # the sums see every tile of 32 columns (one of a single column is 1e-6 of dW at n = 1409)
        if not signed and 32 * (j + 1) <= max(n, 32):
            assert wrong == ["g0", "dw", "db"] + (["dc"] if i == j else []), (i, j)


@pytest.mark.gpu
@pytest.mark.parametrize("signed", [False, True])
@pytest.mark.parametrize("n", SIZES + [2050])
def test_adjoint_layer_elements_match_fp64(n, signed):
    import torch

    g, x = _operands(n, signed)
    dev = "cuda:0"
    w, b, c = (torch.tensor([v], dtype=torch.float32, device=dev) for v in (W, B, C))
    x0, gk = torch.from_numpy(x).to(dev), torch.from_numpy(g).to(dev)
    _, ws = sp2.net_forward(x0, w, b, c, precision="fp32")
    dw, db, dc, g0 = sp2.net_backward(gk, w, b, c, ws, precision="fp32")
    g0 = g0.cpu().numpy().astype(np.float64)
    assert np.array_equal(g0, g0.T)
    assert _Reference(g, x).wrong(g0, float(dw[0]), float(db[0]), float(dc[0])) == []
