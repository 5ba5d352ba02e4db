"""GPU parity of the gated prefill / training forward (App. "Hardware-Aligned
Forward Kernel") against the oracle; needs an MI355X.

Outputs per (sequence, head) row: max_c |o_gpu - o_ref| / max |o_ref| over a
head's rows (over the row, for sampled rows) <= 2e-2 (bf16 operands, softmax weights rounded to bf16 for p.V);
gate row sums R to 1e-4 relative (fp32 sums of gates whose scores differ from
fp64 by fp32 accumulation); log-sum-exp L to 1e-4 absolute.  Rows past a
sequence's length are zero / 0 / -inf.
"""
import math

import numpy as np
import pytest
import torch

import oracle
from gpu_support import require_gpu, say
from paper_2609_20888_amd import eta
from synth import as_numpy

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    require_gpu()
    say(f"\n[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()


def _inputs(B, Hq, Hkv, T, d, seed, tau_mode="normal", q_scale=1.0):
    gen = torch.Generator().manual_seed(seed)
    q = (q_scale * torch.randn(B, Hq, T, d, generator=gen)).to(torch.bfloat16)
    k = torch.randn(B, Hkv, T, d, generator=gen).to(torch.bfloat16)
    v = torch.randn(B, Hkv, T, d, generator=gen).to(torch.bfloat16)
    if tau_mode == "normal":
        tau = 0.5 + 0.5 * torch.randn(B, Hq, T, generator=gen)
    elif tau_mode == "ungated":
        tau = torch.full((B, Hq, T), float("-inf"))
    else:
        tau = torch.full((B, Hq, T), float("inf"))
    return q, k, v, tau.float()


CASES = {
    # name: (B, Hq, Hkv, T, d, seq_lens, beta, additive, C, tau_mode)
    "gqa2_d128_ragged": (2, 4, 2, 200, 128, [200, 131], 4.0, False, 0.0, "normal"),
    "gqa8_d64": (1, 8, 1, 256, 64, [256], 4.0, False, 0.0, "normal"),
    "mha_d128_additive": (1, 2, 2, 160, 128, [150], 2.0, True, 3.0, "normal"),
    "ungated_is_causal_softmax": (1, 4, 4, 130, 64, [130], 4.0, False, 0.0, "ungated"),
    "closed_gates_diagonal_only": (1, 4, 2, 96, 128, [96], 4.0, False, 0.0, "closed"),
    "short_and_empty": (3, 4, 2, 70, 128, [1, 0, 65], 4.0, False, 0.0, "normal"),
}


@pytest.mark.parametrize("name", sorted(CASES))
def test_prefill_matches_oracle(name):
    B, Hq, Hkv, T, d, lens, beta, add, C, tm = CASES[name]
    q, k, v, tau = _inputs(B, Hq, Hkv, T, d, seed=hash(name) % 1000, tau_mode=tm)
    dev = torch.device("cuda")
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    out, R, L = eta.gated_prefill(q.to(dev), k.to(dev), v.to(dev), tau.to(dev), sl, beta=beta,
                                  additive=add, C=C)
    torch.cuda.synchronize()
    r = oracle.prefill(as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64), lens,
                       beta=beta, additive=add, C=C)
    o = out.float().cpu().numpy()
    Rg, Lg = R.cpu().numpy(), L.cpu().numpy()
    worst = 0.0
    for b in range(B):
        n = lens[b]
        assert np.all(o[b, :, n:] == 0) and np.all(Rg[b, :, n:] == 0) and np.all(np.isneginf(Lg[b, :, n:]))
        if n == 0:
            continue
        for h in range(Hq):
            ref = r.o[b, h, :n]
            err = float(np.max(np.abs(o[b, h, :n] - ref)) / np.max(np.abs(ref)))
            worst = max(worst, err)
            assert err <= 2e-2, (b, h, err)
        np.testing.assert_allclose(Rg[b, :, :n], r.r[b, :, :n], rtol=1e-4, atol=1e-5)
        np.testing.assert_allclose(Lg[b, :, :n], r.lse[b, :, :n], rtol=0, atol=1e-4)
    say(f"[gpu] prefill {name}: worst output rel err {worst:.2e}")


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("Hq,Hkv", [(8, 2), (6, 3)])      # Hq % 8 == 0: head order by XCD
@pytest.mark.parametrize("T,lens", [(1, [1, 1]), (32, [32, 31]), (33, [33, 1]), (64, [64, 63]),
                                    (97, [96, 97]), (128, [128, 65]), (300, [33, 300])])
def test_prefill_unit_edges(d, Hq, Hkv, T, lens):
    """Lengths around the 32-key units, 64-key blocks and 128-row workgroups, the
    unit before the first (no weights) and sequences that end inside a wavefront."""
    q, k, v, tau = _inputs(2, Hq, Hkv, T, d, seed=31 * T + d + Hq)
    dev = torch.device("cuda")
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    for add in (False, True):
        out, R, L = eta.gated_prefill(q.to(dev), k.to(dev), v.to(dev), tau.to(dev), sl, beta=4.0,
                                      additive=add, C=2.0)
        torch.cuda.synchronize()
        r = oracle.prefill(as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64),
                           lens, beta=4.0, additive=add, C=2.0)
        o, Rg, Lg = out.float().cpu().numpy(), R.cpu().numpy(), L.cpu().numpy()
        for b in range(2):
            n = lens[b]
            assert np.all(o[b, :, n:] == 0) and np.all(Rg[b, :, n:] == 0)
            assert np.all(np.isneginf(Lg[b, :, n:]))
            for h in range(Hq):
                ref = r.o[b, h, :n]
                assert np.max(np.abs(o[b, h, :n] - ref)) <= 2e-2 * np.max(np.abs(ref)), (add, b, h)
            np.testing.assert_allclose(Rg[b, :, :n], r.r[b, :, :n], rtol=1e-4, atol=1e-5)
            np.testing.assert_allclose(Lg[b, :, :n], r.lse[b, :, :n], rtol=0, atol=1e-4)


def _prefill_vs_oracle(q, k, v, tau, lens, **kw):
    """Launch and compare every row (module docstring's tolerances); returns (out, R, L)."""
    dev = torch.device("cuda")
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    out, R, L = eta.gated_prefill(q.to(dev), k.to(dev), v.to(dev), tau.to(dev), sl, beta=4.0, **kw)
    torch.cuda.synchronize()
    return out.float().cpu().numpy(), R.cpu().numpy(), L.cpu().numpy()


def _check_all(got, r, lens, tag="", lse_atol=1e-4):
    o, Rg, Lg = got
    for b, n in enumerate(lens):
        assert np.all(o[b, :, n:] == 0) and np.all(Rg[b, :, n:] == 0)
        assert np.all(np.isneginf(Lg[b, :, n:]))
        for h in range(o.shape[1] if n else 0):
            ref = r.o[b, h, :n]
            err = np.max(np.abs(o[b, h, :n] - ref), axis=1) / np.max(np.abs(ref), axis=1)
            assert np.max(err) <= 2e-2, (tag, b, h, int(np.argmax(err)), float(np.max(err)))
        np.testing.assert_allclose(Rg[b, :, :n], r.r[b, :, :n], rtol=1e-4, atol=1e-5)
        np.testing.assert_allclose(Lg[b, :, :n], r.lse[b, :, :n], rtol=0, atol=lse_atol)


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T", [1, 33, 64, 97, 200])
@pytest.mark.parametrize("mode", ["open_32", "open_64", "open_all", "closed_additive"])
def test_prefill_rows_whose_first_keys_score_very_low(mode, T, d):
    """The first 32, 64 or all keys score about -103 (2^-149 below weight one: past where
    an fp32 exponential of the reference's move overflows) with the gates open, or every
    key but the row's own is shut 100 below by the additive gate.  The reference of the
    first unit must not be scaled into the empty accumulators.  (Scores near 110: d fp32
    additions add up to d 2^-24 110 to the log-sum-exp's tolerance.)"""
    gen = torch.Generator().manual_seed(T + d)
    q = 0.3 * torch.randn(1, 2, T, d, generator=gen)
    k = 0.3 * torch.randn(1, 1, T, d, generator=gen)
    v = torch.randn(1, 1, T, d, generator=gen).to(torch.bfloat16)
    kw = {}
    if mode == "closed_additive":
        tau = torch.full((1, 2, T), float("inf"))
        kw = dict(additive=True, C=100.0)
    else:
        tau = torch.full((1, 2, T), float("-inf"))
        low = {"open_32": 32, "open_64": 64, "open_all": T}[mode]
        q[..., 0] = 8.0
        k[..., 0] = -2.0 * math.sqrt(d) / 8.0
        k[:, :, :low, 0] = -103.0 * math.sqrt(d) / 8.0
    q, k = q.to(torch.bfloat16), k.to(torch.bfloat16)
    got = _prefill_vs_oracle(q, k, v, tau, [T], **kw)
    r = oracle.prefill(as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64), [T],
                       beta=4.0, **kw)
    _check_all(got, r, [T], mode, lse_atol=1e-4 + d * 2.0 ** -24 * 110)


@pytest.mark.parametrize("d", [64, 128])
def test_prefill_largest_weight_of_the_first_64_keys_is_exact(d):
    """Key 40 outweighs all others (by 2^4 .. 2^7.5, another fraction in every row) and only
    its value is not zero, so an output row is v times one weight over the sum.  The
    reference maximum covers the first 64 keys, so that weight is exactly one in bf16 and
    the row's mean relative error is that of the output's own rounding: each value's is
    uniform within 2^-8 (values in [1, 2)), a row's mean of d of them has a standard
    deviation below 2^-8 / sqrt(3 d) <= 2.9e-4.  Rounding the weight would add up to 2^-8
    (rms 1.6e-3) to every value of a row alike."""
    T = 64
    q, k = torch.zeros(1, 2, T, d), torch.zeros(1, 1, T, d)
    # scores S = q0 k0 / sqrt(d), 4 .. 7.5 in base-2 units, steps that bf16 q0 resolves
    k[..., 40, 0] = 1.0
    x = torch.linspace(4.0, 7.5, 2 * T).view(1, 2, T) * math.log(2.0) * math.sqrt(d)
    q[..., 0] = x
    v = torch.zeros(1, 1, T, d)
    gen = torch.Generator().manual_seed(d)
    v[..., 40, :] = (1.0 + torch.rand(d, generator=gen)) * (1 - 2 * torch.randint(0, 2, (d,), generator=gen))
    q, k, v = (t.to(torch.bfloat16) for t in (q, k, v))
    tau = torch.full((1, 2, T), float("-inf"))
    o, _, _ = _prefill_vs_oracle(q, k, v, tau, [T])
    r = oracle.prefill(as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64), [T],
                       beta=4.0)
    mean = (o[0, :, 40:] / r.o[0, :, 40:] - 1.0).mean(axis=-1)
    rms = float(np.sqrt(np.mean(mean ** 2)))
    say(f"[gpu] prefill d={d}: rms over rows of the mean relative error {rms:.2e}")
    assert rms <= 5e-4


@pytest.mark.parametrize("d", [64, 128])
@pytest.mark.parametrize("T,lens", [(130, [33, 65, 0]), (200, [97, 1, 200]), (64, [63, 32, 64]),
                                    (256, [129, 191, 128])])
def test_prefill_ignores_what_lies_past_the_sequence(d, T, lens):
    """A cache's rows past a sequence's end hold anything: NaN in q, k and tau and NaN or
    infinities in v there change nothing."""
    q, k, v, tau = _inputs(3, 4, 2, T, d, seed=T + d)
    clean = [as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64)]
    for b, n in enumerate(lens):
        for t in (q, k, v, tau):
            t[b, :, n:] = float("nan")
        v[b, :, n::3] = float("inf")
    got = _prefill_vs_oracle(q, k, v, tau, lens)
    r = oracle.prefill(*clean, lens, beta=4.0)
    _check_all(got, r, lens)


def _check_rows(o, R, L, r, rows, lens):
    worst = 0.0
    for n, (b, h, i) in enumerate(rows):
        if i >= lens[b]:
            assert np.all(o[n] == 0) and R[n] == 0 and np.isneginf(L[n])
            continue
        err = float(np.max(np.abs(o[n] - r.o[n])) / np.max(np.abs(r.o[n])))
        worst = max(worst, err)
        assert err <= 2e-2, (b, h, i, err)
        np.testing.assert_allclose(R[n], r.r[n], rtol=1e-4, atol=1e-5, err_msg=str((b, h, i)))
        np.testing.assert_allclose(L[n], r.lse[n], rtol=0, atol=1e-4, err_msg=str((b, h, i)))
    return worst


def test_prefill_long_rows_with_rescaling():
    """1100 tokens (9 query tiles, 18 key blocks, a ragged end) with queries scaled
    up so that the row maxima keep growing and the running reference moves often;
    both gate forms."""
    B, Hq, Hkv, T, d, lens = 1, 4, 1, 1100, 128, [1037]
    q, k, v, tau = _inputs(B, Hq, Hkv, T, d, seed=321, q_scale=3.0)
    dev = torch.device("cuda")
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    rng = np.random.default_rng(5)
    rows = np.array([[0, h, i] for h in range(Hq)
                     for i in sorted({0, 63, 64, 127, 128, 1023, 1036, 1037, 1099}
                                     | set(rng.integers(0, T, 24).tolist()))])
    for add, C in ((False, 0.0), (True, 4.0)):
        out, R, L = eta.gated_prefill(q.to(dev), k.to(dev), v.to(dev), tau.to(dev), sl, beta=4.0,
                                      additive=add, C=C)
        torch.cuda.synchronize()
        r = oracle.prefill_rows(as_numpy(q), as_numpy(k), as_numpy(v),
                                tau.numpy().astype(np.float64), lens, rows, beta=4.0,
                                additive=add, C=C)
        idx = tuple(rows.T)
        worst = _check_rows(out.float().cpu().numpy()[idx], R.cpu().numpy()[idx],
                            L.cpu().numpy()[idx], r, rows, lens)
        say(f"[gpu] prefill long additive={add}: worst output rel err {worst:.2e}")


def test_prefill_full_size_sampled_rows():
    """The benchmarked prefill workload (16384 tokens, 32 query / 8 KV heads, d=128,
    bf16, causal) in the same launch, checked on sampled rows: tile edges, the first
    and last rows, and random rows of every head."""
    B, Hq, Hkv, T, d, lens = 1, 32, 8, 16384, 128, [16384]
    say("[gpu] prefill full size: building inputs")
    q, k, v, tau = _inputs(B, Hq, Hkv, T, d, seed=2024)
    dev = torch.device("cuda")
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    out, R, L = eta.gated_prefill(q.to(dev), k.to(dev), v.to(dev), tau.to(dev), sl, beta=4.0)
    torch.cuda.synchronize()
    rng = np.random.default_rng(6)
    fixed = [0, 1, 63, 64, 127, 128, 4095, 8192, 16255, 16256, 16383]
    rows = np.array([[0, h, i] for h in range(Hq)
                     for i in sorted(set(fixed[h % 4::4]) | set(rng.integers(0, T, 3).tolist()))])
    say(f"[gpu] prefill full size: oracle on {len(rows)} rows")
    r = oracle.prefill_rows(as_numpy(q), as_numpy(k), as_numpy(v), tau.numpy().astype(np.float64),
                            lens, rows, beta=4.0)
    idx = tuple(rows.T)
    worst = _check_rows(out.float().cpu().numpy()[idx], R.cpu().numpy()[idx], L.cpu().numpy()[idx],
                        r, rows, lens)
    say(f"[gpu] prefill full size: worst output rel err {worst:.2e} over {len(rows)} rows")
