"""GPU parity of the block-index variants: the sub-block variance envelope and
the incremental decode-time update (needs an MI355X).

  * envelope sigma against the oracle's Eq. (subblock_envelope_appx) for every
    (head dim, block, dtype) kernel shape and sub-block lengths below, equal to
    and above the rows one load covers; mu and M are the flat build's, bit for
    bit; sub_block = block_size reproduces the flat sigma bit for bit;
  * the update writes exactly the records of the blocks completed since
    prev_lens (capped at max_new_blocks), equal bit for bit to a full build,
    and leaves every other entry alone; a token-by-token decode loop ends with
    the full build's index;
  * a decode step on envelope summaries matches the oracle run on the oracle's
    own envelope summaries.
"""
import numpy as np
import pytest
import torch

import oracle
from gpu_support import (calibrate_bias, compare, oracle_inputs, oracle_summaries, require_gpu,
                         run_gpu, run_oracle, say)
from paper_2609_20888_amd import eta
from synth import as_numpy, make_workload

pytestmark = pytest.mark.gpu


@pytest.fixture(autouse=True)
def _gpu(request):
    require_gpu()
    say(f"\n[gpu] {request.node.nodeid}")
    yield
    torch.cuda.synchronize()


def _np(s: eta.Summaries):
    return s.mu.cpu().numpy(), s.sigma.cpu().numpy(), s.max_norm.cpu().numpy()


ENVELOPE_CASES = [
    # B, Hkv, d, b, lens, dtype, sub_blocks
    (1, 2, 128, 64, [64 * 40 + 9], torch.bfloat16, (1, 2, 4, 8, 16)),
    (1, 1, 128, 128, [128 * 35], torch.bfloat16, (4, 32)),
    (2, 1, 64, 64, [64 * 33, 64 * 7 + 1], torch.bfloat16, (2, 4, 8, 16)),
    (1, 1, 64, 128, [128 * 20], torch.bfloat16, (4, 64)),
    (1, 1, 128, 64, [64 * 30], torch.float32, (1, 4, 16)),
    (1, 1, 64, 64, [64 * 30], torch.float32, (2, 4, 32)),
]


@pytest.mark.parametrize("dt,d,b,sub,n_cap", [
    (torch.bfloat16, 64, 64, 0, 16384), (torch.bfloat16, 128, 64, 8, 14336),
    (torch.bfloat16, 64, 128, 0, 12288), (torch.float32, 64, 64, 0, 8192)])
@pytest.mark.parametrize("stat", [torch.float32, torch.float16])
def test_wide_and_narrow_workgroups_write_the_same_records(stat, dt, d, b, sub, n_cap):
    """The same keys in a short cache (4 blocks per workgroup) and in one long enough for 32
    (n_cap blocks in all, two heads): equal records, nothing past the last full block."""
    n = 75
    T, cap = n * b + 11, n_cap // 2 * b
    gen = torch.Generator(device="cuda").manual_seed(d + b)
    k = (torch.randn(1, 2, T, d, generator=gen, device="cuda") + 1.0).to(dt)
    big = torch.zeros(1, 2, cap, d, device="cuda", dtype=dt)
    big[:, :, :T] = k
    sl = torch.tensor([T], dtype=torch.int32, device="cuda")
    a = eta.build_block_summaries(k, sl, b, sub_block=sub, stat_dtype=stat)
    w = eta.Summaries.empty(1, 2, d, cap // b, "cuda", stat)
    for t in (w.mu, w.sigma, w.max_norm):
        t.fill_(-7.0)
    eta.build_block_summaries(big, sl, b, out=w, sub_block=sub)
    torch.cuda.synchronize()
    for x, y in zip((a.mu, a.sigma, a.max_norm), (w.mu, w.sigma, w.max_norm)):
        assert torch.equal(x[..., :n], y[..., :n])
        assert torch.all(y[..., n:] == -7.0)


@pytest.mark.parametrize("case", range(len(ENVELOPE_CASES)))
def test_envelope_matches_oracle(case):
    _check_envelope(*ENVELOPE_CASES[case], seed=40 + case)


def _check_envelope(B, Hkv, d, b, lens, dt, subs, *, seed):
    wl = make_workload(B=B, Hq=Hkv, Hkv=Hkv, d=d, block=b, seq_lens=lens, dtype=dt,
                       planted={"frac": 0.1}, predictor=False, tau_const=1.0, seed=seed)
    dev = torch.device("cuda")
    k = wl.k.to(dev)
    sl = torch.tensor(lens, dtype=torch.int32, device=dev)
    fmu, fsg, fmx = _np(eta.build_block_summaries(k, sl, b))
    kn = as_numpy(wl.k)
    for sub in subs:
        mu, sg, mx = _np(eta.build_block_summaries(k, sl, b, sub_block=sub))
        for bb in range(B):
            N = lens[bb] // b
            np.testing.assert_array_equal(mu[bb, :, :, :N], fmu[bb, :, :, :N])
            np.testing.assert_array_equal(mx[bb, :, :N], fmx[bb, :, :N])
            for g in range(Hkv):
                omu, _, _ = oracle.summaries(kn[bb, g, :lens[bb]], b)
                env = oracle.envelope(kn[bb, g, :lens[bb]], b, sub, omu)
                np.testing.assert_allclose(sg[bb, g, :, :N].T, env, rtol=1e-5, atol=1e-5,
                                           err_msg=f"sub_block {sub}")
                # the envelope dominates the flat sigma up to rounding (mean of sub-block MSDs <= max)
                assert np.all(sg[bb, g, :, :N] >= fsg[bb, g, :, :N] * (1 - 1e-5) - 1e-6)


@pytest.mark.parametrize("d,b,dt", [(128, 128, torch.bfloat16), (64, 64, torch.bfloat16),
                                    (128, 64, torch.float32)])
def test_envelope_of_one_sub_block_is_flat_sigma(d, b, dt):
    wl = make_workload(B=1, Hq=2, Hkv=2, d=d, block=b, seq_lens=[b * 50 + 3], dtype=dt,
                       planted={"frac": 0.1}, predictor=False, tau_const=1.0, seed=47)
    dev = torch.device("cuda")
    k = wl.k.to(dev)
    sl = torch.tensor(wl.seq_lens, dtype=torch.int32, device=dev)
    flat = _np(eta.build_block_summaries(k, sl, b))
    env = _np(eta.build_block_summaries(k, sl, b, sub_block=b))
    N = wl.seq_lens[0] // b
    for x, y in zip(flat, env):
        np.testing.assert_array_equal(x[..., :N], y[..., :N])


def _sentinel(B, Hkv, d, ncap, dev):
    s = eta.Summaries.empty(B, Hkv, d, ncap, dev)
    for t in (s.mu, s.sigma, s.max_norm):
        t.fill_(float("nan"))
    return s


UPDATE_CASES = [
    # d, b, dtype, prev lens, new lens, max_new_blocks, sub_block
    (128, 128, torch.bfloat16, [128 * 30 + 127, 128 * 9], [128 * 31, 128 * 9 + 5], 1, 0),
    (128, 64, torch.bfloat16, [64 * 20 + 3, 64 * 5, 0], [64 * 23 + 1, 64 * 5 + 63, 64 * 2], 3, 0),
    (128, 64, torch.bfloat16, [64 * 20 + 3, 64 * 40], [64 * 23 + 1, 64 * 35], 2, 0),     # cap; shrink
    (64, 64, torch.float32, [64 * 10], [64 * 50 + 7], 64, 4),                              # > 32 blocks
    (64, 128, torch.bfloat16, [128 * 3 + 1], [128 * 4], 1, 8),
]


@pytest.mark.parametrize("case", range(len(UPDATE_CASES)))
def test_update_writes_exactly_the_completed_blocks(case):
    d, b, dt, prev, new, max_new, sub = UPDATE_CASES[case]
    B, Hkv = len(prev), 2
    T_cap = b * 64
    wl = make_workload(B=B, Hq=4, Hkv=Hkv, d=d, block=b, seq_lens=[T_cap] * B, T_cap=T_cap,
                       dtype=dt, planted={"frac": 0.1}, predictor=False, tau_const=1.0,
                       seed=50 + case)
    dev = torch.device("cuda")
    k = wl.k.to(dev)
    pl = torch.tensor(prev, dtype=torch.int32, device=dev)
    nl = torch.tensor(new, dtype=torch.int32, device=dev)
    ncap = T_cap // b
    full = _np(eta.build_block_summaries(k, nl, b, sub_block=sub))
    s = eta.build_block_summaries(k, pl, b, sub_block=sub, out=_sentinel(B, Hkv, d, ncap, dev))
    before = _np(s)
    eta.update_block_summaries(k, pl, nl, s, b, max_new_blocks=max_new, sub_block=sub)
    after = _np(s)
    for bb in range(B):
        p_n, n_n = prev[bb] // b, new[bb] // b
        hi = min(n_n, p_n + max_new)
        written = np.zeros(ncap, bool)
        written[p_n:max(hi, p_n)] = True
        for x_full, x_before, x_after in zip(full, before, after):
            xa = np.moveaxis(x_after[bb], -1, 0) if x_after.ndim == 4 else x_after[bb].T
            xb = np.moveaxis(x_before[bb], -1, 0) if x_before.ndim == 4 else x_before[bb].T
            xf = np.moveaxis(x_full[bb], -1, 0) if x_full.ndim == 4 else x_full[bb].T
            # block axis first
            np.testing.assert_array_equal(xa[written], xf[written])
            np.testing.assert_array_equal(xa[~written], xb[~written])
        say(f"[gpu] seq {bb}: blocks {p_n}..{hi - 1} written")


@pytest.mark.parametrize("sub", [0, 4])
def test_token_by_token_decode_loop_rebuilds_the_index(sub):
    d, b = 128, 64
    L0, steps = 64 * 6 + 50, 3 * 64 + 20
    wl = make_workload(B=2, Hq=8, Hkv=2, d=d, block=b, seq_lens=[L0 + steps, L0 + steps],
                       T_cap=L0 + steps + 64, planted={"frac": 0.1}, predictor=False,
                       tau_const=1.0, seed=60)
    dev = torch.device("cuda")
    k = wl.k.to(dev)
    lens = torch.tensor([L0, L0 - 30], dtype=torch.int32, device=dev)
    s = eta.build_block_summaries(k, lens, b, sub_block=sub)
    for _ in range(steps):
        prev = lens.clone()
        lens += 1
        eta.update_block_summaries(k, prev, lens, s, b, max_new_blocks=1, sub_block=sub)
    ref = _np(eta.build_block_summaries(k, lens, b, sub_block=sub))
    got = _np(s)
    for bb in range(2):
        N = int(lens[bb]) // b
        for x, y in zip(got, ref):
            np.testing.assert_array_equal(x[bb, ..., :N], y[bb, ..., :N])


@pytest.mark.parametrize("sub,lwb", [(4, 2), (16, 0)])
def test_decode_on_envelope_summaries_matches_oracle(sub, lwb):
    wl = make_workload(B=2, Hq=8, Hkv=2, d=128, block=64, seq_lens=[20000, 9001],
                       planted={"frac": 0.05}, predictor=False, tau_const=2.0, lwb=lwb,
                       seed=70 + sub)
    np_in = oracle_inputs(wl)
    calibrate_bias(wl, np_in)
    g = run_gpu(wl, sub_block=sub)
    summ = oracle_summaries(wl, np_in[1], sub_block=sub)
    orc, tau_o = run_oracle(wl, np_in, summaries=summ)
    stats = compare(wl, g, orc, tau_o, np_inputs=np_in, union_counts=g.union_counts)
    frac = float(g.mask.float().mean())
    say(f"[gpu] envelope sub {sub} lwb {lwb}: {stats}, mask density {frac:.3f}")


@pytest.mark.parametrize("d,b,sub", [(64, 64, 1), (64, 64, 32), (64, 64, 64), (64, 128, 2), (64, 128, 8),
                                     (64, 128, 128), (128, 64, 64), (128, 128, 2)])
def test_envelope_sub_block_edges(d, b, sub):
    """Sub-blocks below, at and above the row groups that one load covers."""
    _check_envelope(2, 1, d, b, [b * 9 + 5, b * 2], torch.bfloat16, (sub,), seed=40 + len(ENVELOPE_CASES))


@pytest.mark.parametrize("d,b,sub,rec", [(128, 128, 0, torch.float32), (128, 64, 4, torch.float16),
                                         (64, 64, 4, torch.float8_e4m3fn), (64, 64, 0, torch.float32),
                                         (64, 128, 8, torch.float16)])
def test_large_and_small_builds_write_the_same_records(d, b, sub, rec):
    """A cache large enough for 32 blocks per workgroup and its first part alone, built with
    4 per workgroup: the same bits, ragged ends included."""
    T = 512 * 1024 * 1024 // (4 * d * 2) + 3 * b + 7          # 4 kv heads, over 512 MiB
    cut = 45 * b + 3
    gen = torch.Generator(device="cuda").manual_seed(d + b + sub)
    k = torch.empty(1, 4, T, d, device="cuda", dtype=torch.bfloat16)
    for h in range(4):
        k[0, h] = torch.randn(T, d, generator=gen, device="cuda").to(torch.bfloat16)
    kw = dict(sub_block=sub, stat_dtype=rec)
    big = eta.build_block_summaries(k, torch.tensor([T], dtype=torch.int32, device="cuda"), b, **kw)
    part = eta.build_block_summaries(k[:, :, :cut], torch.tensor([cut], dtype=torch.int32, device="cuda"),
                                     b, **kw)
    first = T // b - 11                          # the last blocks: a shorter workgroup
    end = eta.build_block_summaries(k[:, :, first * b:],
                                    torch.tensor([T - first * b], dtype=torch.int32, device="cuda"), b, **kw)
    n = cut // b
    bits = lambda t: t.contiguous().view(torch.uint8)
    for name in ("mu", "sigma"):
        assert torch.equal(bits(getattr(big, name)[..., :n]), bits(getattr(part, name)[..., :n]))
    assert torch.equal(big.max_norm[..., :n], part.max_norm[..., :n])
    for name in ("mu", "sigma", "max_norm"):
        assert torch.equal(bits(getattr(big, name)[..., first:]), bits(getattr(end, name)[..., :11]))
