"""The fp32 products on the f16 matrix units, at the edges of their tiles and scales.

Bounds.  A product is hi hi + hi lo + lo hi of two-part f16 operands: each operand is off by at
most 2^-23 of itself (test_parts_carry_24_bits), the missing lo lo by 2^-24 of the product, and a
sum over K runs through at most 3 ceil(K / 16) fp32 additions, each off by 2^-24 of the terms'
absolute sum S: |error| <= (3 ceil(K / 16) + SLACK) 2^-24 S.  SLACK covers the operands (8), the
k-split's sums and the epilogue; inputs that the library normalises add 4 roundings of the row.
"""
import numpy as np
import pytest
import torch

U = 2.0 ** -24
SLACK = 24


def bound(k, terms):
    return (3 * -(-k // 16) + SLACK) * U * terms


def row_scale(x):
    """The power of two that brings the largest |x| of each row to [2^14, 2^15)."""
    return 2.0 ** (14 - np.floor(np.log2(np.abs(x).max(axis=1, keepdims=True))))


def test_parts_carry_24_bits():
    rng = np.random.default_rng(0)
    x = (rng.normal(size=(64, 4096)) * 2.0 ** rng.integers(-30, 30, (64, 1))).astype(np.float32)
    x[:, ::7] *= np.float32(2.0 ** -20)
    p = row_scale(x.astype(np.float64))
    xp = x.astype(np.float64) * p
    hi = xp.astype(np.float16)
    assert np.isfinite(hi).all()
    lo = (xp - hi.astype(np.float64)).astype(np.float16)
    off = np.abs(xp - hi.astype(np.float64) - lo.astype(np.float64))
    assert (off <= np.maximum(2.0 ** -23 * np.abs(xp), 2.0 ** -25)).all()


def lib():
    import paper_2404_08573_amd as P
    return P


def make_layer(P, W, b):
    return P.Layer(torch.from_numpy(W).cuda(), torch.from_numpy(b).cuda())


def forward(P, W, b, x, normalised):
    n, m = x.shape[0], W.shape[0]
    h, g = torch.empty(n, m, device="cuda"), torch.empty(n, device="cuda")
    P.ff_layer_forward(make_layer(P, W, b), P.HParams(), torch.from_numpy(x).cuda(), normalised,
                       h_out=h, goodness=g)
    torch.cuda.synchronize()
    return h.cpu().numpy().astype(np.float64), g.cpu().numpy().astype(np.float64)


# rows, d_in, d_out: a single tile and its edges, k tails, then every rung of the forward tiles
# (64x64, 128x64, 128x128, 256x128)
FORWARD = [(1, 4, 4), (63, 60, 68), (65, 132, 64), (129, 20, 132), (300, 784, 500),
           (1024, 68, 2000), (2048, 36, 2000), (2050, 68, 2004), (4100, 100, 1028)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_in,d_out", FORWARD)
@pytest.mark.parametrize("normalised", [False, True])
def test_forward(rows, d_in, d_out, normalised):
    P = lib()
    rng = np.random.default_rng(rows + d_in)
    W = (rng.normal(size=(d_out, d_in)) * 10.0 ** rng.uniform(-6, 4, (d_out, 1))).astype(np.float32)
    b = rng.normal(size=d_out).astype(np.float32) * 0.1
    x = (np.maximum(rng.normal(size=(rows, d_in)), 0) *
         10.0 ** rng.uniform(-5, 5, (rows, 1))).astype(np.float32)
    x[rows // 2] = 0
    h, g = forward(P, W, b, x, normalised)
    xh = x.astype(np.float64)
    if not normalised:
        xh /= np.linalg.norm(xh, axis=1, keepdims=True) + 1e-8
    z = xh @ W.T.astype(np.float64) + b
    S = np.abs(xh) @ np.abs(W.T.astype(np.float64)) + np.abs(b)
    tol = bound(d_in, S) + (0 if normalised else 4 * U * S)
    assert (np.abs(h - np.maximum(z, 0)) <= tol + 1e-37).all()
    np.testing.assert_allclose(g, np.square(h).sum(1), rtol=1e-5, atol=1e-30)


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_in,d_out", [(70, 68, 132), (1024, 36, 2000), (2050, 36, 2004)])
def test_forward_not_finite(rows, d_in, d_out):
    """inf, NaN and the largest floats give what fp32 sums give: relu(+inf) = inf, NaN -> 0."""
    P = lib()
    rng = np.random.default_rng(5)
    W = rng.normal(size=(d_out, d_in)).astype(np.float32)
    W[3, 5], W[7, 2], W[d_out - 1, d_in - 1] = np.inf, np.nan, 3.3e38
    x = rng.uniform(0.01, 0.1, (rows, d_in)).astype(np.float32)
    x[:, 5][::2] = 0
    x[11, 3], x[rows - 1, 0] = -np.inf, np.nan
    b = np.zeros(d_out, np.float32)
    h, _ = forward(P, W, b, x, True)
    with np.errstate(all="ignore"):
        z = np.stack([(x.astype(np.float64) * w).sum(1) for w in W.astype(np.float64)], 1)
        S = np.stack([np.abs(x.astype(np.float64) * w).sum(1) for w in W.astype(np.float64)], 1)
    want = np.where(np.isnan(z), 0, np.maximum(np.nan_to_num(z, posinf=np.inf, neginf=-np.inf), 0))
    fin = np.isfinite(want) & np.isfinite(S)
    assert np.array_equal(np.isposinf(h), np.isposinf(want))
    assert (h[~np.isfinite(S) & np.isfinite(want)] == 0).all()
    # the fp32 instructions add one product after another: d_in additions
    assert (np.abs(h[fin] - want[fin]) <= (d_in + SLACK) * U * S[fin]).all()


def ref_step(W, x, n_pos, theta, normalised):
    """c, h, x_hat of the FF step in 64 bits, and the bound of the device's error in h."""
    xh = x.astype(np.float64)
    if not normalised:
        xh = xh / (np.linalg.norm(xh, axis=1, keepdims=True) + 1e-8)
    h = np.maximum(xh @ W.T.astype(np.float64), 0)
    g = np.square(h).sum(1)
    n = x.shape[0]
    e = np.where(np.arange(n) < n_pos, theta - g, g - theta)
    s = np.where(e > 0, 1 / (1 + np.exp(-np.abs(e))), np.exp(-np.abs(e)) / (1 + np.exp(-np.abs(e))))
    c = np.where(np.arange(n) < n_pos, -2 * s / n_pos, 2 * s / (n - n_pos))
    return c, h, xh, bound(x.shape[1] + 16, np.abs(xh) @ np.abs(W.T.astype(np.float64)))


# rows, d_in, d_out: one tile and its edges, the 2048-row factor table's end, then the
# weight-gradient rungs (64x64, 128x64 on eight waves, on four)
STEP = [(2, 4, 4), (70, 68, 132), (33, 132, 60), (2047, 36, 68), (2100, 68, 36), (4100, 20, 24),
        (150, 784, 2000), (130, 1028, 2004)]


@pytest.mark.gpu
@pytest.mark.parametrize("rows,d_in,d_out", STEP)
@pytest.mark.parametrize("normalised", [False, True])
def test_step_gradient(rows, d_in, d_out, normalised):
    """From zero moments, mW = 0.1 dW and mb = 0.1 db after one step.  c carries the goodness'
    rounding (under 1e-5 of c here)."""
    P = lib()
    rng = np.random.default_rng(rows + d_out)
    W = (rng.normal(size=(d_out, d_in)) / np.sqrt(d_out)).astype(np.float32)
    x = np.maximum(rng.normal(size=(rows, d_in)), 0).astype(np.float32) + np.float32(1e-3)
    x *= (rng.uniform(0.2, 1.5, (rows, 1)) / np.linalg.norm(x, axis=1, keepdims=True)).astype(
        np.float32)
    n_pos = max(1, rows // 3)
    L = make_layer(P, W, np.zeros(d_out, np.float32))
    P.ff_layer_step(L, P.HParams(theta=0.7), torch.from_numpy(x).cuda(), n_pos, rows - n_pos,
                    normalised)
    torch.cuda.synchronize()
    c, h, xh, eh = ref_step(W, x, n_pos, 0.7, normalised)
    dz, dh = c[:, None] * h, np.abs(c[:, None]) * eh
    for got, want, terms, slack in (
            (L.mW, dz.T @ xh, np.abs(dz).T @ np.abs(xh), dh.T @ np.abs(xh)),
            (L.mb, dz.sum(0), np.abs(dz).sum(0), dh.sum(0))):
        off = np.abs(got.cpu().numpy().astype(np.float64) * 10 - want)
        assert (off <= bound(rows, terms) + rows * U * terms + 2e-5 * terms + slack + 1e-37).all()


@pytest.mark.gpu
@pytest.mark.parametrize("d_in,d_out", [(68, 132), (784, 2000), (1028, 2004)])
def test_step_not_finite(d_in, d_out):
    """A NaN input feature: its row's activities come out 0, and 0 * NaN makes its weight column's
    gradient NaN in every unit; the other columns are what they are without that row."""
    P = lib()
    rng = np.random.default_rng(9)
    rows, bad = 90, 17
    W = (rng.normal(size=(d_out, d_in)) / np.sqrt(d_out)).astype(np.float32)
    x = rng.uniform(0.0, 1.0, (rows, d_in)).astype(np.float32)
    x /= np.linalg.norm(x, axis=1, keepdims=True)
    xn = x.copy()
    xn[4, bad] = np.nan
    L = make_layer(P, W, np.zeros(d_out, np.float32))
    P.ff_layer_step(L, P.HParams(theta=0.7), torch.from_numpy(xn).cuda(), 45, 45, True)
    torch.cuda.synchronize()
    m = L.mW.cpu().numpy().astype(np.float64) * 10
    assert np.isnan(m[:, bad]).all()
    c, h, xh, eh = ref_step(W, x, 45, 0.7, True)
    h[4] = 0
    dz, keep = c[:, None] * h, np.arange(d_in) != bad
    want, terms = dz.T @ xh, np.abs(dz).T @ np.abs(xh)
    slack = 2e-5 * terms + (np.abs(c[:, None]) * eh).T @ np.abs(xh) + 1e-37
    assert (np.abs(m - want) <= (rows + SLACK) * U * terms + slack)[:, keep].all()


@pytest.mark.gpu
def test_step_rows_of_very_different_weight():
    """Rows whose gradient coefficients differ by 2^-60 and rows without any activity: the
    neurons that only the light rows reach keep their relative accuracy."""
    P = lib()
    rng = np.random.default_rng(3)
    d, rows = 64, 96
    W = np.zeros((2 * d, 2 * d), np.float32)
    W[:d, :d] = np.abs(rng.normal(size=(d, d))) * 0.9   # reached by the light rows (g large)
    W[d:, d:] = np.abs(rng.normal(size=(d, d))) * 0.01  # by the heavy ones
    x = np.zeros((rows, 2 * d), np.float32)
    x[:48, :d] = rng.uniform(0.5, 1, (48, d))
    x[48:, d:] = rng.uniform(0.5, 1, (48, d))
    x[40:44] = 0
    x /= np.maximum(np.linalg.norm(x, axis=1, keepdims=True), 1e-30)
    L = make_layer(P, W, np.zeros(2 * d, np.float32))
    g = torch.empty(rows, device="cuda")
    theta = 2.0
    P.ff_layer_step(L, P.HParams(theta=theta), torch.from_numpy(x).cuda(), 48, 48, True, goodness=g)
    torch.cuda.synchronize()
    c, h, xh, eh = ref_step(W, x, 48, theta, True)
    dz = c[:, None] * h
    want, terms = dz.T @ xh, np.abs(dz).T @ np.abs(xh)
    got = L.mW.cpu().numpy().astype(np.float64) * 10
    # c = exp(theta - g) of the light rows carries the goodness' absolute rounding
    slack = (2e-5 + 8 * U * g.cpu().numpy().max()) * terms
    slack += (np.abs(c[:, None]) * eh).T @ np.abs(xh)
    assert (np.abs(got - want) <= bound(rows, terms) + slack + 1e-37).all()
