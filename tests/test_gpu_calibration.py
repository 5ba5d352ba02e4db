"""GPU parity of the offline density-matched calibration (App. "Offline Threshold
Calibration via 1/t-Weighted Histograms"; Alg. "Density-Matched Offline
Threshold Calibration"); needs an MI355X.

The GPU computes scores on the matrix cores in fp32 and bins them in fp32; a
score within its error bound of a bin edge may land in the next bin.  The
oracle therefore also bins every pair at S - delta and S + delta with
  delta = d 2^-24 sum_i |q_i k_i| / sqrt(d) + 8 2^-24 (|lo| + |hi| + S_max)
(the classical bound for d fp32 additions of exact products, plus the binning
arithmetic; S_max = max |q| max |k| / sqrt(d) by Cauchy-Schwarz), and the
GPU's cumulative histogram must lie between those two.  The target densities
agree to the gate's slope (beta / 4) times the largest delta; the constants
solve the oracle's equation g(c) = target up to the change that moving the
ambiguous mass to a neighbouring bin can make in g (beta w / 4 per unit of
mass).  Accumulation is in integers, so it is exactly reproducible and
additive over calls.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_support import require_gpu, say
from paper_2609_20888_amd import eta
from synth import as_numpy, calib_stream

pytestmark = pytest.mark.gpu

U = 2.0 ** -24


@pytest.fixture(autouse=True)
def _gpu(request):
    require_gpu()
    say(f"\n[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()


def _gpu_calibrate(cs, *, beta, lo, hi, nb, splits=1):
    Hq, Hkv, d = cs.q.shape[1], cs.k.shape[1], cs.q.shape[3]
    cal = eta.Calibrator(Hq, Hkv, d, beta=beta, lo=lo, hi=hi, num_bins=nb, device="cuda")
    N = cs.q.shape[0]
    cuts = np.linspace(0, N, splits + 1).astype(int)
    for a, b in zip(cuts[:-1], cuts[1:]):
        cal.accumulate(cs.q[a:b].contiguous(), cs.k[a:b].contiguous(), cs.tau[a:b].contiguous())
    c, target = cal.solve()
    torch.cuda.synchronize()
    hist = cal.hist.cpu().numpy().view(np.uint64)
    dens = cal.density.cpu().numpy().view(np.uint64)
    return hist, dens, c.cpu().numpy(), target.cpu().numpy()


CASES = [
    # N, Hq, Hkv, T, d, beta, lo, hi, nb
    (3, 8, 2, 200, 128, 4.0, -4.0, 8.0, 256),
    (2, 4, 4, 77, 64, 2.0, -3.0, 6.0, 1024),
    (1, 8, 1, 33, 128, 8.0, -5.0, 10.0, 64),
    (2, 16, 2, 130, 128, 4.0, -2.0, 2.0, 4096),
]


@pytest.mark.parametrize("case", range(len(CASES)))
def test_calibration_matches_oracle(case):
    _check_calibration(*CASES[case], seed=100 + case)


def _check_calibration(N, Hq, Hkv, T, d, beta, lo, hi, nb, *, seed):
    cs = calib_stream(N=N, Hq=Hq, Hkv=Hkv, T=T, d=d, seed=seed, device="cuda")
    hist, dens, c, target = _gpu_calibrate(cs, beta=beta, lo=lo, hi=hi, nb=nb)
    qn, kn = as_numpy(cs.q), as_numpy(cs.k)
    tau = cs.tau.cpu().numpy().astype(np.float64)
    s_max = float(cs.q.float().norm(dim=-1).max() * cs.k.float().norm(dim=-1).max()) / math.sqrt(d)
    eps_abs = 8 * U * (abs(lo) + abs(hi) + s_max)
    delta_max = d * U * s_max + eps_abs
    r = oracle.calib_hist(qn, kn, tau, beta=beta, lo=lo, hi=hi, nb=nb, gamma=d * U,
                          eps_abs=eps_abs, brackets=True)
    H = hist.astype(np.float64) / eta.CALIB_UNIT
    total = N * T
    # weights: one per step, up to the fixed-point rounding of each 1/(t+1)
    np.testing.assert_allclose(H.sum(axis=1), r.total, rtol=0, atol=1e-6)
    cg, cl, ch = np.cumsum(H, axis=1), np.cumsum(r.hist_lo, axis=1), np.cumsum(r.hist_hi, axis=1)
    assert np.all(cg <= cl + 1e-6) and np.all(cg >= ch - 1e-6)
    amb = (cl - ch).sum(axis=1) / total                    # mass that may sit one bin over
    w = (hi - lo) / nb
    # target density: gate slope <= beta / 4 times the score error; fp32 gate rounding
    tgt_tol = beta / 4 * delta_max + 1e-6
    np.testing.assert_allclose(target, r.target, rtol=0, atol=tgt_tol)
    np.testing.assert_allclose(dens.astype(np.float64) / eta.CALIB_UNIT / total, r.target, atol=tgt_tol)
    worst = 0.0
    for h in range(Hq):
        resid = abs(oracle.calib_g(r.hist[h], lo, hi, beta, float(c[h])) - r.target[h])
        tol = amb[h] * beta * w / 4 + tgt_tol + beta / 4 * abs(float(c[h])) * U + 1e-9
        assert resid <= tol, (h, resid, tol)
        worst = max(worst, resid)
    c_orc = np.array([oracle.calib_solve(r.hist[h], lo, hi, beta, r.target[h]) for h in range(Hq)])
    say(f"[gpu] calibration {N}x{T}, {Hq}/{Hkv}, d={d}: max |c_gpu - c_oracle| {np.max(np.abs(c - c_orc)):.2e}, "
        f"max g residual {worst:.2e}, ambiguous mass {amb.max():.2e}")


def test_calibration_is_reproducible_and_additive():
    cs = calib_stream(N=4, Hq=8, Hkv=2, T=150, d=128, seed=7, device="cuda")
    kw = dict(beta=4.0, lo=-4.0, hi=8.0, nb=512)
    a = _gpu_calibrate(cs, **kw)
    b = _gpu_calibrate(cs, **kw)
    c = _gpu_calibrate(cs, splits=3, **kw)
    for x, y, z in zip(a, b, c):
        assert np.array_equal(x, y) and np.array_equal(x, z)


def test_constant_dynamic_threshold_is_recovered():
    """Calibrating a predictor that always outputs tau0_h returns tau0_h to within a bin."""
    tau0 = [0.25 * h - 0.5 for h in range(8)]
    cs = calib_stream(N=2, Hq=8, Hkv=2, T=256, d=128, seed=8, tau_const=tau0, device="cuda")
    lo, hi, nb = -6.0, 10.0, 4096
    _, _, c, _ = _gpu_calibrate(cs, beta=4.0, lo=lo, hi=hi, nb=nb)
    assert np.all(np.abs(c - np.array(tau0)) <= (hi - lo) / nb), c


@pytest.mark.parametrize("T,N,Hq,Hkv,d,nb", [(1, 2, 2, 1, 64, 1), (15, 1, 2, 2, 128, 777),
                                             (64, 1, 4, 1, 64, 4096), (65, 2, 2, 1, 128, 1000),
                                             (256, 1, 2, 2, 128, 1024), (321, 1, 8, 1, 64, 1025)])
def test_calibration_block_edges(T, N, Hq, Hkv, d, nb):
    """Steps around the 16-query groups, 64-query blocks and 256-query workgroups; bins
    around the solver's 1024 threads."""
    _check_calibration(N, Hq, Hkv, T, d, 4.0, -6.0, 10.0, nb, seed=100 + len(CASES))


def test_calibration_adds_up_over_calls_with_several_workgroups_per_head():
    cs = calib_stream(N=5, Hq=4, Hkv=2, T=700, d=64, seed=17, device="cuda")
    kw = dict(beta=4.0, lo=-8.0, hi=24.0, nb=1024)
    a = _gpu_calibrate(cs, **kw)
    for splits in (2, 5):
        for x, y in zip(a, _gpu_calibrate(cs, splits=splits, **kw)):
            assert np.array_equal(x, y)


def _slope(hist, lo, hi, beta, c):
    """-g'(c) / beta in [0, 1/4]."""
    s = lo + (np.arange(hist.size) + 0.5) * (hi - lo) / hist.size
    e = np.exp(-np.abs(beta * (s - c)))
    return float(np.sum(hist * (e / (1 + e) ** 2)) / np.sum(hist))


@pytest.mark.parametrize("tau", [-60.0, 60.0, 1e30])
def test_saturated_gates_solve_to_the_end_of_the_bracket(tau):
    """Every gate fully open or shut (1e30: the gate's exponential overflows): the
    density is 1 or 0 and the solution runs to an end of the bracket, as in the oracle's
    bisection of the same histogram and density."""
    cs = calib_stream(N=1, Hq=2, Hkv=1, T=100, d=64, seed=5, tau_const=[tau, tau], device="cuda")
    lo, hi, nb = -8.0, 24.0, 512
    hist, dens, c, target = _gpu_calibrate(cs, beta=4.0, lo=lo, hi=hi, nb=nb)
    for h in range(2):
        assert abs(target[h] - (1.0 if tau < 0 else 0.0)) <= 1e-7
        ref = oracle.calib_solve(hist[h] / eta.CALIB_UNIT, lo, hi, 4.0, float(target[h]))
        # the solver's last interval, one rounding to fp32, and what 32 fp64 roundings of g
        # move a root this far out by
        sl = _slope(hist[h] / eta.CALIB_UNIT, lo, hi, 4.0, ref)
        tol = 1e-9 / 4.0 + abs(ref) * U
        if 0 < target[h] < 1:
            tol += 32 * 2.0 ** -53 / sl / 4.0
        assert abs(c[h] - ref) <= tol, (h, c[h], ref)


def _solve_counts(hist, dens, *, beta, lo, hi):
    """eta_calib_solve of given integer accumulators: hist [H][nb], dens [H]."""
    H, nb = hist.shape
    cal = eta.Calibrator(H, H, 64, beta=beta, lo=lo, hi=hi, num_bins=nb, device="cuda")
    cal.hist.copy_(torch.from_numpy(hist.astype(np.int64)))
    cal.density.copy_(torch.from_numpy(dens.astype(np.int64)))
    c, target = cal.solve()
    torch.cuda.synchronize()
    return c.cpu().numpy().astype(np.float64), target.cpu().numpy()


@pytest.mark.parametrize("nb", [1, 2, 777, 1025, 4096])
@pytest.mark.parametrize("beta", [0.0625, 4.0, 300.0])     # (exact in fp32, as the descriptor holds it)
def test_solve_returns_the_root(nb, beta):
    """The constant is the root of g(c) = target that bisection of the same histogram and
    density finds: within 1e-9 / beta (the solver's last step), what 32 fp64 roundings of
    g move the root by, and one rounding to fp32."""
    rng = np.random.default_rng(nb)
    lo, hi, H = -8.0, 24.0, 8
    hist = (rng.random((H, nb)) ** 4 * 2.0 ** 40).astype(np.int64) + 1
    hist[1::2, nb // 3: 2 * nb // 3] = 0                 # a gap in every other head
    frac = np.array([1e-4, 0.01, 0.1, 0.3, 0.6, 0.9, 0.99, 0.9999])
    dens = np.rint(hist.sum(axis=1) * frac).astype(np.int64)
    c, target = _solve_counts(hist, dens, beta=beta, lo=lo, hi=hi)
    for h in range(H):
        H64 = hist[h].astype(np.float64)
        ref = oracle.calib_solve(H64, lo, hi, beta, float(target[h]))
        sl = _slope(H64, lo, hi, beta, ref)
        tol = (1e-9 + 32 * 2.0 ** -53 / max(sl, 1e-300)) / beta + abs(ref) * U
        assert abs(c[h] - ref) <= tol, (h, c[h], ref, sl, tol)


@pytest.mark.parametrize("beta", [4.0, 64.0])
def test_solve_on_a_flat_stretch_ends_where_bisection_ends(beta):
    """Where g equals the target over a stretch (two clusters of scores far apart, the
    density one cluster's share; or every score counted, density the whole), every point
    of it is a root, and bisection's is the stretch's lower end: where the nearer cluster
    below still adds a rounding of g, anything from a quarter to a whole one with the order
    of g's additions (a factor of 4 in that cluster's exponential: log 4 / beta).  Heads 2
    and 3 count every score: the bracket's lower end."""
    lo, hi, nb = -8.0, 24.0, 512
    hist = np.zeros((4, nb), dtype=np.int64)
    hist[0, 10], hist[0, 500] = 1 << 40, 1 << 40
    hist[1, 0:4], hist[1, 508:512] = 3 << 38, 1 << 38
    hist[2, 256] = 1 << 44
    hist[3, :] = 1 << 36
    dens = np.array([1 << 40, 4 << 38, 1 << 44, nb << 36], dtype=np.int64)
    c, target = _solve_counts(hist, dens, beta=beta, lo=lo, hi=hi)
    for h in range(4):
        ref = oracle.calib_solve(hist[h].astype(np.float64), lo, hi, beta, float(target[h]))
        tol = 1e-9 / beta + abs(ref) * U + (math.log(4.0) / beta if h < 2 else 0.0)
        assert abs(c[h] - ref) <= tol, (h, c[h], ref)
