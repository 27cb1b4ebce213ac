"""GPU parity of MuonH (puro_muonh_step, puro_newton_schulz_bf16) against the
oracle (oracle/muonh.py), through the C ABI.

* One Newton-Schulz step, from each of the oracle's own BF16 iterates: every
  element of X' lies in the band that binary32 accumulation (1e-5 of
  sum |ab| per product), the coefficients' binary32 rounding and the BF16
  roundings of A and B allow, propagated through the three products; and
  99% of them are within one BF16 step of the oracle's BF16 evaluation
  (a rounding flip in A or B moves X' by far less than a step).
* The step with no Newton-Schulz iterations: the momentum buffer bit for bit,
  X_0 = V / (||V|| + eps) within its binary32 evaluation (relative 2^-22
  before the BF16 rounding), and W' within the first-order bound of the
  hyperball step around the oracle's, given the width of X_0's band.
* The full step: the momentum bit for bit, the direction u within twice the
  BF16 noise of the oracle's own BF16 evaluation (its distance from the
  float64 definition), W' on the sphere of radius R and within the bound
  that this u tolerance gives through the hyperball step.
* The Qwen2-1.5B shapes in the launch configuration the benchmark times (28
  matrices per call): the last matrix of each call checked as above, every
  matrix's radius and momentum.
"""

import numpy as np
import pytest

from oracle import bf16, muonh
from paper_2608_27370_amd import inputs

from gpu_util import bf16_bits, host, to_dev, to_dev_bf16

pytestmark = pytest.mark.gpu

A32, B32, C32 = (float(np.float32(v)) for v in muonh.COEFFS)
F32 = 2.0 ** -23          # binary32 rounding of a sum or product, with margin


@pytest.fixture(scope="module")
def P():
    from paper_2608_27370_amd import puro
    puro.lib()
    return puro


def f64(bits):
    return muonh.to_f64(bits)


def band(val, dev):
    """BF16 ends of [val - dev, val + dev] and the largest distance of an
    accepted value from val."""
    lo, hi = bf16.from_f64_rne(val - dev), bf16.from_f64_rne(val + dev)
    return lo, hi, np.maximum(np.abs(f64(lo) - val), np.abs(f64(hi) - val))


def in_band(got, lo, hi):
    g = f64(got)
    return (g >= f64(lo)) & (g <= f64(hi))


def ns_step_band(X_bits):
    """The BF16 values one GPU Newton-Schulz step may give from X."""
    a, b, c = muonh.COEFFS
    X = f64(X_bits)
    aX = np.abs(X)
    A = X @ X.T
    _, _, wA = band(A, 1e-5 * (aX @ aX.T))
    aA = np.abs(A)
    AA = aA @ aA.T
    B = b * A + c * (A @ A)
    tB = (abs(b) * wA + abs(c) * (wA @ aA.T + aA @ wA.T + wA @ wA.T) + abs(c) * 1e-5 * ((aA + wA) @ (aA + wA).T)
          + abs(b - B32) * aA + abs(c - C32) * AA + F32 * (abs(b) * aA + abs(c) * AA))
    _, _, wB = band(B, tB)
    aB = np.abs(B)
    Xn = a * X + B @ X
    tX = wB @ aX + 1e-5 * ((aB + wB) @ aX) + abs(a - A32) * aX + F32 * (abs(a) * aX + aB @ aX)
    lo, hi, _ = band(Xn, tX)
    return lo, hi


def ulp_distance(x_bits, y_bits):
    """|x - y| in BF16 steps of the larger magnitude."""
    x, y = f64(x_bits), f64(y_bits)
    m = np.maximum(np.abs(x), np.abs(y))
    _, e = np.frexp(np.where(m > 0, m, 1.0))
    step = np.ldexp(1.0, np.maximum(e - 1, -126) - 7)
    return np.abs(x - y) / step


@pytest.mark.parametrize("r,c,count", [(128, 384, 2), (256, 256, 1), (256, 640, 3)])
def test_newton_schulz_one_step(P, r, c, count):
    Vs = [inputs.muonh_matrix(r, c, key=100 + i)[1] for i in range(count)]
    X = np.stack([muonh.ns_start_bf16(V) for V in Vs])
    for k in range(muonh.STEPS):
        got = bf16_bits(P.newton_schulz_bf16(to_dev_bf16(X), steps=1))
        for i in range(count):
            lo, hi = ns_step_band(X[i])
            ok = in_band(got[i], lo, hi)
            assert ok.all(), "step %d matrix %d: %d outside the band" % (k, i, (~ok).sum())
            want = muonh.ns_step_bf16(X[i])[2]
            assert np.mean(ulp_distance(got[i], want) <= 1.0) >= 0.99, (k, i)
        X = np.stack([muonh.ns_step_bf16(X[i])[2] for i in range(count)])


@pytest.mark.timeout(300)
def test_newton_schulz_batch_of_ragged_large_tiles(P):
    """A batch whose symmetric products take 256x256 tiles (20 matrices of 896
    rows: 200 tiles of 256, 560 of 128) though its rows end inside the last of
    them; the first and last matrices in the band."""
    r, count = 896, 20
    rng = np.random.default_rng(7)
    X = bf16.from_f64_rne(rng.standard_normal((count, r, r)).astype(np.float32).astype(np.float64) / r)
    for i in (0, count - 1):
        X[i] = muonh.ns_start_bf16(inputs.muonh_matrix(r, r, key=150 + i)[1])
    print("newton-schulz: GPU step of %d [%d, %d]" % (count, r, r), flush=True)
    got = bf16_bits(P.newton_schulz_bf16(to_dev_bf16(X), steps=1))
    for i in (0, count - 1):
        lo, hi = ns_step_band(X[i])
        ok = in_band(got[i], lo, hi)
        assert ok.all(), "matrix %d: %d outside the band" % (i, (~ok).sum())


def _run_step(P, W, G, buf, R, eta, steps, mu=0.95):
    torch = __import__("torch")
    Wd, Gd, bd = to_dev(W), to_dev(G), to_dev(buf)
    Rd = to_dev(np.asarray(R, dtype=np.float32))
    wb = torch.empty(W.shape, dtype=torch.bfloat16, device="cuda")
    ud = torch.empty(W.shape, dtype=torch.bfloat16, device="cuda")
    P.muonh_step(Wd, Gd, bd, Rd, eta, mu=mu, ns_steps=steps, w_bf16=wb, u_out=ud)
    return host(Wd), host(bd), bf16_bits(wb), bf16_bits(ud)


def hyperball_bound(W, u, du, eta, R):
    """Elementwise first-order bound on |W'(u + du) - W'(u)| plus the
    binary32 evaluation of W' (k1 = eta R / ||u||, k2 = R / ||W~||, each
    rounded, and W' = k2 (W - k1 u) with a fused multiply-add)."""
    nu = np.linalg.norm(u)
    k1 = eta * R / nu
    Wt = W - k1 * u
    nt = np.linalg.norm(Wt)
    d1 = k1 * (np.abs(du) + np.abs(u) * np.linalg.norm(du) / nu)
    dW = (R / nt) * (d1 + np.abs(Wt) * np.linalg.norm(d1) / nt)
    return dW + 4 * F32 * (R / nt) * (np.abs(W) + k1 * np.abs(u))


def _check_common(Wn, bn, wb, W, G, buf, R, mu, what):
    want_buf = muonh.momentum(buf, G, mu)[0]
    assert np.array_equal(bn.view(np.uint32), want_buf.view(np.uint32)), what + ": momentum"
    assert abs(np.linalg.norm(Wn.astype(np.float64)) - R) <= 1e-6 * R, what + ": radius"
    assert np.array_equal(wb, bf16.from_f64_rne(Wn.astype(np.float64))), what + ": BF16 copy of W'"


@pytest.mark.parametrize("rows,cols", [(256, 384), (384, 256), (128, 128)])
def test_muonh_start_and_hyperball(P, rows, cols):
    """ns_steps = 0: the hyperball step along X_0 itself."""
    count, eta, mu = 2, 0.02, 0.95
    mats = [inputs.muonh_matrix(rows, cols, key=200 + i) for i in range(count)]
    W = np.stack([m[0] for m in mats]); G = np.stack([m[1] for m in mats]); buf = np.stack([m[2] for m in mats])
    R = [float(np.float32(np.linalg.norm(W[i].astype(np.float64)))) for i in range(count)]
    Wn, bn, wb, u = _run_step(P, W, G, buf, R, eta, 0, mu)
    for i in range(count):
        _, V = muonh.momentum(buf[i], G[i], mu)
        V64 = V.astype(np.float64)
        x0 = V64 / (np.linalg.norm(V64) + muonh.EPS)
        lo, hi, _ = band(x0, 2.0 ** -22 * np.abs(x0))
        assert in_band(u[i], lo, hi).all(), "X_0 of matrix %d" % i
        _check_common(Wn[i], bn[i], wb[i], W[i], G[i], buf[i], R[i], mu, "matrix %d" % i)
        uo = f64(bf16.from_f64_rne(x0))
        ref = muonh.hyperball(W[i], uo, eta, R[i])
        # the kernel's X_0 may be any value of the band: its distance from uo
        du = np.maximum(np.abs(f64(lo) - uo), np.abs(f64(hi) - uo))
        tol = hyperball_bound(W[i].astype(np.float64), uo, du, eta, R[i])
        assert np.all(np.abs(Wn[i] - ref) <= tol), np.max(np.abs(Wn[i] - ref) / tol)


def _check_full(Wn, bn, wb, u, W, G, buf, R, eta, mu, what):
    _check_common(Wn, bn, wb, W, G, buf, R, mu, what)
    _, V = muonh.momentum(buf, G, mu)
    u64 = muonh.newton_schulz(V)
    uem = f64(muonh.newton_schulz_bf16(V))
    noise = np.linalg.norm(uem - u64)
    dev = np.linalg.norm(f64(u) - u64)
    assert dev <= 2.0 * noise + 2.0 ** -9 * np.linalg.norm(u64), (what, dev, noise)
    # W' around the hyperball step along the float64 direction: |du| is
    # bounded in norm only, so the bound is in norm
    ref = muonh.hyperball(W, u64, eta, R)
    nu = np.linalg.norm(u64)
    Wt = W.astype(np.float64) - eta * R * u64 / nu
    bound = (R / np.linalg.norm(Wt)) * eta * R * 2.0 * (2.0 * noise + 2.0 ** -9 * nu) / nu * 2.0 + 1e-6 * R
    assert np.linalg.norm(Wn - ref) <= bound, (what, np.linalg.norm(Wn - ref), bound)


@pytest.mark.parametrize("rows,cols", [(256, 512), (512, 256)])
def test_muonh_full_step(P, rows, cols):
    count, eta, mu = 2, 0.01, 0.95
    mats = [inputs.muonh_matrix(rows, cols, key=300 + i) for i in range(count)]
    W = np.stack([m[0] for m in mats]); G = np.stack([m[1] for m in mats]); buf = np.stack([m[2] for m in mats])
    R = [float(np.float32(np.linalg.norm(W[i].astype(np.float64)))) for i in range(count)]
    Wn, bn, wb, u = _run_step(P, W, G, buf, R, eta, muonh.STEPS, mu)
    for i in range(count):
        _check_full(Wn[i], bn[i], wb[i], u[i], W[i], G[i], buf[i], R[i], eta, mu, "matrix %d" % i)


def test_muonh_zero_gradient_only_projects(P):
    rows, cols = 128, 256
    W = inputs.muonh_matrix(rows, cols, key=400)[0]
    G = np.zeros_like(W)
    buf = np.zeros_like(W)
    R = 0.5 * float(np.float32(np.linalg.norm(W.astype(np.float64))))
    Wn, bn, wb, u = _run_step(P, W[None], G[None], buf[None], [R], 0.02, muonh.STEPS)
    assert not np.any(bn) and not np.any(f64(u))
    ref = muonh.hyperball(W, np.zeros_like(W), 0.02, R)
    assert np.all(np.abs(Wn[0] - ref) <= 4 * F32 * np.abs(ref) + 1e-30)


@pytest.mark.timeout(900)
@pytest.mark.parametrize("name,rows,cols", [(n, r, c) for n, r, c in inputs.LAYER_LINEARS])
def test_muonh_layer_shapes_28_matrices(P, name, rows, cols):
    """The 28 layers' matrices of one kind in one call, as the benchmark
    runs them: matrices 0..26 come from torch's generator on the device (they
    are checked for radius and momentum only); the last from the seeded
    generator, checked in full."""
    torch = __import__("torch")
    count, eta, mu = inputs.LAYERS, 0.01, 0.95
    gen = torch.Generator(device="cuda").manual_seed(11)
    W = torch.randn(count, rows, cols, device="cuda", generator=gen) * 0.02
    G = torch.randn(count, rows, cols, device="cuda", generator=gen) * 1e-3
    buf = torch.randn(count, rows, cols, device="cuda", generator=gen) * 1e-3
    w0, g0, b0 = inputs.muonh_matrix(rows, cols, key=500)
    W[-1].copy_(torch.from_numpy(w0)); G[-1].copy_(torch.from_numpy(g0)); buf[-1].copy_(torch.from_numpy(b0))
    R = torch.linalg.vector_norm(W.double(), dim=(1, 2)).float()
    R[-1] = float(np.float32(np.linalg.norm(w0.astype(np.float64))))
    W_h, G_h, b_h, R_h = host(W), host(G), host(buf), host(R)
    wb = torch.empty(W.shape, dtype=torch.bfloat16, device="cuda")
    ud = torch.empty(W.shape, dtype=torch.bfloat16, device="cuda")
    print("muonh %s: GPU step of %d [%d, %d]" % (name, count, rows, cols), flush=True)
    P.muonh_step(W, G, buf, R, eta, mu=mu, ns_steps=muonh.STEPS, w_bf16=wb, u_out=ud)
    Wn, bn = host(W), host(buf)
    for i in range(count):
        want = muonh.momentum(b_h[i], G_h[i], mu)[0]
        assert np.array_equal(bn[i].view(np.uint32), want.view(np.uint32)), i
        assert abs(np.linalg.norm(Wn[i].astype(np.float64)) - R_h[i]) <= 1e-6 * R_h[i], i
    print("muonh %s: oracle of the last matrix" % name, flush=True)
    _check_full(Wn[-1], bn[-1], bf16_bits(wb[-1]), bf16_bits(ud[-1]), w0, g0, b0, float(R_h[-1]), eta, mu,
                "%s last" % name)
