"""The work a program has this library do, as a fixed list of measurable cases.

A case is one call path at one size: a decode step over an existing cache, the
block index built after a prefill, the gated prefill itself, the dense decode,
or the offline threshold calibration.  ``listed()`` holds the sizes of the
benchmark's and the tests' own workloads (and the head shape of the paper's
kernel table); ``draw`` gives more cases of the same ranges.

Every input is drawn on the GPU from the seed alone, in plain torch: N(0, 1)
queries, keys and values, a share of the blocks "planted" along the group's
query direction, predictor weights N(0, 0.02^2) and a bias that leaves a given
share of each head's blocks above the threshold.  ``exact`` recomputes what
``run`` returns in 64 bits from the same inputs with torch alone.
"""
import math

import torch

from paper_2609_20888_amd import eta

DEV = "cuda"
REC = {"f32": torch.float32, "f16": torch.float16, "fp8": torch.float8_e4m3fn}
WINDOW = {64: 128, 128: 64}       # rescue window (blocks) for each block size
BETA = 4.0


# ---------------------------------------------------------------- the cases

def listed():
    return [
        # one short chat: 4K tokens, MHA, fp32 cache, frozen per-head thresholds; all latency
        dict(name="step_4k_mha_fp32", kind="step", B=1, Hq=4, Hkv=4, d=64, block=64, T=4096,
             ragged=False, dtype="f32", rec="f32", survival=0.125, planted=0.125, z=1.0,
             predictor=False, update=False),
        # one 32K conversation, a serving loop's token: the token completes a block, so the
        # index is updated, then the step runs
        dict(name="step_32k_update", kind="step", B=1, Hq=16, Hkv=4, d=128, block=64, T=32768,
             ragged=False, dtype="bf16", rec="f32", survival=0.10, planted=0.05, z=1.0,
             predictor=True, update=True),
        # eight 128K documents side by side
        dict(name="step_128k_b8", kind="step", B=8, Hq=16, Hkv=4, d=128, block=64, T=131072,
             ragged=False, dtype="bf16", rec="f32", survival=0.10, planted=0.07, z=1.0,
             predictor=True, update=False),
        # the benchmark's step: one 512K context, 20% of the blocks per head
        dict(name="step_512k", kind="step", B=1, Hq=16, Hkv=4, d=128, block=128, T=524288,
             ragged=False, dtype="bf16", rec="f32", survival=0.20, planted=0.01, z=1.0,
             predictor=True, update=False),
        # a serving batch: 32 sequences of 16K..64K tokens, compact fp16 records
        dict(name="step_ragged_b32_f16", kind="step", B=32, Hq=32, Hkv=8, d=128, block=64,
             T=65536, ragged=True, dtype="bf16", rec="f16", survival=0.10, planted=0.0, z=2.0,
             predictor=True, update=False),
        # the paper's kernel table: batch 32 at 64K, eight query heads per kv head, d = 64
        dict(name="step_paper_b32_64k_d64", kind="step", B=32, Hq=32, Hkv=4, d=64, block=64,
             T=65536, ragged=False, dtype="bf16", rec="f16", survival=0.10, planted=0.08, z=1.0,
             predictor=True, update=False),
        # layers that keep plain softmax attention: ragged batch, every token read
        dict(name="dense_b8_32k", kind="dense", B=8, Hq=16, Hkv=4, d=128, block=64, T=32768,
             ragged=True, dtype="bf16"),
        # block index of one 512K cache after its prefill
        dict(name="index_512k", kind="index", B=1, Hkv=4, d=128, block=128, T=524288,
             ragged=False, dtype="bf16", rec="f32", sub=0),
        # the paper's b = 64 index: sub-block envelope (sub-blocks of 4), fp16 records, d = 64,
        # a batch of ragged prompts
        dict(name="index_envelope_b8_d64", kind="index", B=8, Hkv=4, d=64, block=64, T=32000,
             ragged=True, dtype="bf16", rec="f16", sub=4),
        # gated prefill of one long prompt
        dict(name="prefill_16k", kind="prefill", B=1, Hq=32, Hkv=8, d=128, T=16384,
             ragged=False, additive=False),
        # gated training forward (additive mask) on a batch of short ragged sequences, d = 64
        dict(name="prefill_b4_2k_d64", kind="prefill", B=4, Hq=32, Hkv=4, d=64, T=2000,
             ragged=True, additive=True),
        # offline calibration of the static thresholds: eight sequences of 2048 steps, then solved
        dict(name="calib_8x2k", kind="calib", B=8, Hq=32, Hkv=8, d=128, T=2048, bins=1024),
    ]


def _loguniform(rng, lo, hi):
    return int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))


def draw(rng):
    kind = rng.choice(["step", "step", "step", "dense", "index", "prefill", "calib"])
    G = rng.choice([1, 2, 4, 8])
    d = rng.choice([64, 128, 128])
    if kind == "step":
        if rng.random() < 0.25:                # a short fp32 cache, any length
            Hkv = rng.choice([2, 4, 8])
            return dict(kind="step", B=rng.choice([1, 1, 2]), Hq=G * Hkv, Hkv=Hkv, d=d, block=64,
                        T=_loguniform(rng, 1000, 16384), ragged=False, dtype="f32", rec="f32",
                        survival=rng.uniform(0.05, 0.3), planted=0.05, z=1.0,
                        predictor=rng.random() < 0.5, update=rng.random() < 0.5)
        block = rng.choice([64, 64, 128])
        Hkv = rng.choice([2, 4, 8])
        B = rng.choice([1, 2, 5, 8, 16, 32])
        most = min(524288, 32 * 65536 * 8 * 128 // (B * Hkv * d) // 2)
        return dict(kind="step", B=B, Hq=G * Hkv, Hkv=Hkv, d=d, block=block,
                    T=_loguniform(rng, 2000, most), ragged=B > 1 and rng.random() < 0.5,
                    dtype="bf16", rec=rng.choice(["f32", "f32", "f16", "fp8"]),
                    survival=rng.uniform(0.03, 0.3), planted=0.03, z=rng.choice([1.0, 2.0]),
                    predictor=rng.random() < 0.8, update=rng.random() < 0.3)
    Hkv = rng.choice([2, 4, 8])
    if kind == "dense":
        B = rng.choice([1, 2, 5, 8])
        return dict(kind="dense", B=B, Hq=G * Hkv, Hkv=Hkv, d=d, block=64,
                    T=_loguniform(rng, 1000, 65536), ragged=B > 1, dtype="bf16")
    if kind == "index":
        B = rng.choice([1, 2, 8])
        block = rng.choice([64, 128])
        return dict(kind="index", B=B, Hkv=Hkv, d=d, block=block,
                    T=_loguniform(rng, 2000, 524288 // B), ragged=B > 1,
                    dtype=rng.choice(["bf16", "bf16", "bf16", "f32"]),
                    rec=rng.choice(["f32", "f16", "fp8"]), sub=rng.choice([0, 0, 4, block // 16]))
    if kind == "prefill":
        B = rng.choice([1, 2, 4])
        return dict(kind="prefill", B=B, Hq=G * Hkv, Hkv=Hkv, d=d,
                    T=_loguniform(rng, 300, 8192 if B == 1 else 4096), ragged=B > 1,
                    additive=rng.random() < 0.3)
    return dict(kind="calib", B=rng.choice([1, 2, 4]), Hq=G * Hkv, Hkv=Hkv, d=d,
                T=_loguniform(rng, 300, 2048), bins=rng.choice([256, 1000, 1024, 4096]))


# ---------------------------------------------------------------- inputs

def _lens(c, gen):
    """Lengths of the batch: all T, or uniform in T/4..T (the first one T)."""
    if not c["ragged"]:
        return [c["T"]] * c["B"]
    r = torch.rand(c["B"], generator=gen, device=DEV).tolist()
    lens = [c["T"] // 4 + int(x * (c["T"] - c["T"] // 4)) for x in r]
    lens[0] = c["T"]
    return lens


def _gen(c, seed):
    return torch.Generator(device=DEV).manual_seed(int(seed))


def _randn(gen, *shape):
    return torch.randn(*shape, generator=gen, device=DEV, dtype=torch.float32)


def _stats(kf, block, rec, sub=0):
    """Block records of one (sequence, kv head): kf [T][d] in fp32 or fp64 -> mu, sigma
    rounded to the record type (in kf's type), largest norm."""
    n = kf.shape[0] // block
    x = kf[:n * block].view(n, block, -1)
    mu = x.mean(1)
    dev2 = (x - mu[:, None]).square()
    if sub:
        sg = dev2.view(n, block // sub, sub, -1).mean(2).amax(1).sqrt()
    else:
        sg = dev2.mean(1).sqrt()
    M = x.square().sum(2).amax(1).sqrt()
    if rec != "f32":
        mu, sg = (t.to(torch.float32).to(REC[rec]).to(kf.dtype) for t in (mu, sg))
    return mu, sg, M


def _bounds(qg, mu, sg, M, z):
    """Screening bound of every block for the group's queries qg [G][d] -> [G][n]."""
    g = qg @ mu.t() + z * (qg.square() @ sg.square().t()).sqrt()
    return torch.minimum(g, qg.norm(dim=1)[:, None] * M[None]) / math.sqrt(qg.shape[1])


def _step_inputs(c, seed):
    """q, k, v, lengths, W (head-major) and bias of a decode step."""
    gen = _gen(c, seed)
    B, Hq, Hkv, d, T, blk = c["B"], c["Hq"], c["Hkv"], c["d"], c["T"], c["block"]
    G = Hq // Hkv
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    lens = _lens(c, gen)
    q = _randn(gen, B, Hq, d).to(dt)
    k = torch.empty(B, Hkv, T, d, device=DEV, dtype=dt)
    v = torch.empty(B, Hkv, T, d, device=DEV, dtype=dt)
    W = 0.02 * _randn(gen, Hq, Hq * d) if c["predictor"] else None
    qf = q.float()
    qW = torch.zeros(B, Hq, device=DEV) if W is None else qf.view(B, -1) @ W.t()
    rel = [[] for _ in range(Hkv)]               # bound - qW, per kv head: [G][blocks of b]
    for b in range(B):
        n = lens[b] // blk
        for g in range(Hkv):
            kk = _randn(gen, T, d)
            if c["planted"] and n:
                hot = torch.rand(n, generator=gen, device=DEV) < c["planted"]
                u = qf[b, g * G:(g + 1) * G].sum(0)
                shift = hot.float()[:, None, None] * (3.0 * math.sqrt(d) * u / u.norm())
                kk[:n * blk].view(n, blk, d).add_(shift)
            k[b, g] = kk.to(dt)
            v[b, g] = _randn(gen, T, d).to(dt)
            mu, sg, M = _stats(k[b, g, :lens[b]].float(), blk, c["rec"])
            rel[g].append(_bounds(qf[b, g * G:(g + 1) * G], mu, sg, M, c["z"])
                          - qW[b, g * G:(g + 1) * G, None])
    # the bias leaves about `survival` of each head's blocks (over the batch) above the
    # threshold; of the cuts within half a percent of that count, the widest gap is taken,
    # so that no bound sits at its threshold
    bias = torch.empty(Hq, device=DEV)
    for g in range(Hkv):
        x = torch.cat(rel[g], dim=1).sort(dim=1, descending=True).values      # [G][n]
        n = x.shape[1]
        kk = min(max(int(c["survival"] * n), 1), n - 1)
        w = max(2, n // 200)
        lo, hi = max(1, kk - w), min(n - 1, kk + w)
        gaps = x[:, lo - 1:hi] - x[:, lo:hi + 1]
        at = (lo - 1 + gaps.argmax(dim=1))[:, None]
        bias[g * G:(g + 1) * G] = (0.5 * (x.gather(1, at) + x.gather(1, at + 1)))[:, 0]
    return q, k, v, lens, W, bias


def _dense_inputs(c, seed):
    gen = _gen(c, seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    lens = _lens(c, gen)
    q = _randn(gen, c["B"], c["Hq"], c["d"]).to(dt)
    k = _randn(gen, c["B"], c["Hkv"], c["T"], c["d"]).to(dt)
    v = _randn(gen, c["B"], c["Hkv"], c["T"], c["d"]).to(dt)
    return q, k, v, lens


def _index_inputs(c, seed):
    gen = _gen(c, seed)
    dt = torch.float32 if c["dtype"] == "f32" else torch.bfloat16
    lens = _lens(c, gen)
    # keys with a mean per coordinate, as real keys have, so mu is not all rounding
    k = (_randn(gen, c["B"], c["Hkv"], c["T"], c["d"])
         + _randn(gen, c["B"], c["Hkv"], 1, c["d"])).to(dt)
    return k, lens


def _prefill_inputs(c, seed):
    gen = _gen(c, seed)
    B, Hq, Hkv, T, d = c["B"], c["Hq"], c["Hkv"], c["T"], c["d"]
    lens = _lens(c, gen)
    q = _randn(gen, B, Hq, T, d).to(torch.bfloat16)
    k = _randn(gen, B, Hkv, T, d).to(torch.bfloat16)
    v = _randn(gen, B, Hkv, T, d).to(torch.bfloat16)
    tau = 0.5 + 0.5 * _randn(gen, B, Hq, T)
    return q, k, v, tau, lens


CALIB_LO, CALIB_HI = -8.0, 24.0


def _calib_inputs(c, seed):
    """Queries and keys of every step, 5% of the keys along the group's mean query
    direction (the score stream's right tail), and the dynamic thresholds."""
    gen = _gen(c, seed)
    N, Hq, Hkv, T, d = c["B"], c["Hq"], c["Hkv"], c["T"], c["d"]
    q = _randn(gen, N, Hq, T, d)
    k = _randn(gen, N, Hkv, T, d)
    u = q.view(N, Hkv, Hq // Hkv, T, d).sum(dim=(2, 3))
    u = u / u.norm(dim=-1, keepdim=True)
    hot = torch.rand(N, Hkv, T, generator=gen, device=DEV) < 0.05
    k = torch.where(hot[..., None], 3.0 * math.sqrt(d) * u[:, :, None] + k, k)
    mean = torch.linspace(0.5, 2.0, Hq, device=DEV)
    tau = mean[None, :, None] + 0.3 * _randn(gen, N, Hq, T)
    return q.to(torch.bfloat16), k.to(torch.bfloat16), tau.contiguous()


def _i32(lens):
    return torch.tensor(lens, dtype=torch.int32, device=DEV)


# ---------------------------------------------------------------- prepare and run

def prepare(case, seed):
    c = case
    if c["kind"] == "step":
        q, k, v, lens, W, bias = _step_inputs(c, seed)
        sl = _i32(lens)
        summ = eta.build_block_summaries(k, sl, c["block"], num_q_heads=c["Hq"],
                                         stat_dtype=REC[c["rec"]])
        p = eta.decode_params(beta=BETA, z=c["z"], rescue_window=WINDOW[c["block"]])
        step = eta.DecodeStep(q, k, v, sl, summ, W, bias, block_size=c["block"], params=p)
        return dict(c=c, step=step, k=k, sl=sl, prev=sl - 1, summ=summ)
    if c["kind"] == "dense":
        q, k, v, lens = _dense_inputs(c, seed)
        ws = eta.alloc_workspace(eta.dense_workspace_size(eta.kv_desc(k, c["Hq"], c["block"])), DEV)
        return dict(c=c, q=q, k=k, v=v, sl=_i32(lens), ws=ws, out=torch.empty_like(q))
    if c["kind"] == "index":
        k, lens = _index_inputs(c, seed)
        summ = eta.Summaries.empty(c["B"], c["Hkv"], c["d"], c["T"] // c["block"], DEV,
                                   REC[c["rec"]])
        return dict(c=c, k=k, sl=_i32(lens), summ=summ)
    if c["kind"] == "prefill":
        q, k, v, tau, lens = _prefill_inputs(c, seed)
        R = torch.empty(tau.shape, device=DEV)
        return dict(c=c, q=q, k=k, v=v, tau=tau, sl=_i32(lens), out=torch.empty_like(q), R=R,
                    L=torch.empty_like(R))
    q, k, tau = _calib_inputs(c, seed)
    return dict(c=c, q=q, k=k, tau=tau)


def run(state):
    s, c = state, state["c"]
    if c["kind"] == "step":
        st = s["step"]
        r = {}
        if c["update"]:
            eta.update_block_summaries(s["k"], s["prev"], s["sl"], s["summ"], c["block"],
                                       max_new_blocks=1, num_q_heads=c["Hq"])
            r = {"mu": s["summ"].mu, "sigma": s["summ"].sigma, "max_norm": s["summ"].max_norm}
        st.run()
        r.update(out=st.out, mask=st.mask, counts=st.counts, union_counts=st.union_counts,
                 tau=st.tau)
        return r
    if c["kind"] == "dense":
        return eta.dense_decode(s["q"], s["k"], s["v"], s["sl"], block_size=c["block"],
                                out=s["out"], workspace=s["ws"])
    if c["kind"] == "index":
        u = eta.build_block_summaries(s["k"], s["sl"], c["block"], out=s["summ"],
                                      sub_block=c["sub"])
        return {"mu": u.mu, "sigma": u.sigma, "max_norm": u.max_norm}
    if c["kind"] == "prefill":
        o, R, L = eta.gated_prefill(s["q"], s["k"], s["v"], s["tau"], s["sl"], beta=BETA,
                                    additive=c["additive"], C=3.0, out=s["out"], R=s["R"],
                                    L=s["L"])
        return {"out": o, "R": R, "L": L}
    cal = eta.Calibrator(c["Hq"], c["Hkv"], c["d"], beta=BETA, lo=CALIB_LO, hi=CALIB_HI,
                         num_bins=c["bins"], device=DEV)
    cal.accumulate(s["q"], s["k"], s["tau"])
    thr, target = cal.solve()
    # the histogram and the gate density as weights, the way a calibration report keeps them
    return {"c": thr, "target": target, "hist": cal.hist.double() / eta.CALIB_UNIT,
            "density": cal.density.double() / eta.CALIB_UNIT}


# ---------------------------------------------------------------- work

def _mean_len(c):
    return c["T"] * (0.625 if c["ragged"] else 1.0)


def work(case):
    c = case
    if c["kind"] == "calib":
        pairs = c["B"] * c["Hq"] * c["T"] * (c["T"] + 1) / 2
        return {"bytes": c["B"] * c["T"] * ((c["Hq"] + c["Hkv"]) * c["d"] * 2 + c["Hq"] * 4)
                + c["Hq"] * (c["bins"] * 8 + 20), "flops": 2.0 * c["d"] * pairs}
    if c["kind"] == "prefill":
        n2 = c["B"] * c["Hq"] * (c["T"] ** 2) * (0.4375 if c["ragged"] else 1.0) / 2
        n = c["B"] * c["T"]
        return {"bytes": n * c["d"] * 2 * (2 * c["Hq"] + 2 * c["Hkv"]) + n * c["Hq"] * 12,
                "flops": 4.0 * c["d"] * n2}
    e = 4 if c["dtype"] == "f32" else 2
    tok = c["B"] * c["Hkv"] * _mean_len(c)
    if c["kind"] == "dense":
        return {"bytes": 2 * tok * c["d"] * e + 2 * c["B"] * c["Hq"] * c["d"] * e,
                "flops": 4.0 * c["d"] * tok * (c["Hq"] // c["Hkv"])}
    rec = 2 * c["d"] * {"f32": 4, "f16": 2, "fp8": 1}[c["rec"]] + 4
    nblk = tok / c["block"]
    if c["kind"] == "index":
        return {"bytes": tok * c["d"] * e + nblk * rec, "flops": 6.0 * tok * c["d"]}
    G = c["Hq"] // c["Hkv"]
    pl = min(c["planted"], c["survival"])        # planted blocks survive for every head
    r = (c["survival"] - pl) / (1 - pl)
    union = pl + (1 - pl) * (1 - (1 - r) ** G)
    small = c["B"] * c["Hq"] * (2 * c["d"] * e + c["T"] // c["block"] + 12)
    if c["predictor"]:
        small += c["Hq"] * c["Hq"] * c["d"] * 4
    return {"bytes": 2 * union * tok * c["d"] * e + nblk * rec + small,
            "flops": 4.0 * G * nblk * c["d"] + 4.0 * c["d"] * c["survival"] * tok * G}


# ---------------------------------------------------------------- tolerance

def tolerance(case):
    c = case
    if c["kind"] in ("step", "dense"):
        # bf16 results differ by their own rounding (2^-9); fp32 ones by the order of the sums.
        # A block whose bound is within fp32 rounding of its threshold may go either way.
        if c["dtype"] == "f32":
            return {"rel": 2e-5, "max": 2e-4, "differ": 0.002}
        return {"rel": 5e-3, "max": 5e-2, "differ": 0.002}
    if c["kind"] == "index":
        # a record may round the other way when its fp32 statistic moves by an ulp
        return {"f32": {"rel": 1e-6, "max": 1e-5}, "f16": {"rel": 2e-4, "max": 4e-3},
                "fp8": {"rel": 1e-2, "max": 0.3}}[c["rec"]]
    if c["kind"] == "prefill":
        return {"rel": 1e-2, "max": 0.1}
    # scores at a bin's edge may fall in the next bin (an early step's pair weighs up to 1)
    return {"rel": 2e-4, "max": 0.05}


# ---------------------------------------------------------------- 64 bits

def _softmax_rows(s, v):
    m = s.amax(dim=1, keepdim=True)
    m = torch.where(torch.isinf(m), torch.zeros_like(m), m)
    p = torch.exp(s - m)
    l = p.sum(1, keepdim=True)
    return torch.where(l > 0, (p @ v) / l, torch.zeros_like(l))


def _exact_step(c, seed):
    q, k, v, lens, W, bias = _step_inputs(c, seed)
    B, Hq, Hkv, d, blk = c["B"], c["Hq"], c["Hkv"], c["d"], c["block"]
    G = Hq // Hkv
    qd = q.double()
    tau = bias.double().expand(B, Hq)
    if W is not None:
        tau = tau + qd.view(B, -1) @ W.double().t()
    out = torch.zeros(B, Hq, d, dtype=torch.float64, device=DEV)
    for b in range(B):
        T = lens[b]
        n = T // blk
        for g in range(Hkv):
            hs = slice(g * G, (g + 1) * G)
            kd = k[b, g, :T].double()
            t = tau[b, hs, None]
            bd = _bounds(qd[b, hs], *_stats(kd, blk, c["rec"]), c["z"])
            sel = bd >= t
            w = min(WINDOW[blk], n)
            if w:
                lost = ~sel[:, :w].any(dim=1)
                first = bd[:, :w].argmax(dim=1)
                sel[torch.arange(G, device=DEV)[lost], first[lost]] = True
            s = qd[b, hs] @ kd.t() / math.sqrt(d)
            s = s * torch.sigmoid(BETA * (s - t))
            on = torch.cat([sel.repeat_interleave(blk, dim=1),
                            torch.ones(G, T - n * blk, dtype=torch.bool, device=DEV)], dim=1)
            out[b, hs] = _softmax_rows(s.masked_fill(~on, -math.inf), v[b, g, :T].double())
    r = {"out": out, "mask": None, "counts": None, "union_counts": None, "tau": tau.contiguous()}
    if c["update"]:
        r.update(mu=None, sigma=None, max_norm=None)
    return r


def exact(case, seed):
    c = case
    if c["kind"] == "step":
        return _exact_step(c, seed)
    if c["kind"] == "dense":
        q, k, v, lens = _dense_inputs(c, seed)
        G = c["Hq"] // c["Hkv"]
        out = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
        for b in range(c["B"]):
            for g in range(c["Hkv"]):
                hs = slice(g * G, (g + 1) * G)
                s = q[b, hs].double() @ k[b, g, :lens[b]].double().t() / math.sqrt(c["d"])
                out[b, hs] = _softmax_rows(s, v[b, g, :lens[b]].double())
        return out
    if c["kind"] == "index":
        k, lens = _index_inputs(c, seed)
        B, Hkv, d, n = c["B"], c["Hkv"], c["d"], c["T"] // c["block"]
        mu, sg = (torch.zeros(B, Hkv, d, n, dtype=torch.float64, device=DEV) for _ in range(2))
        M = torch.zeros(B, Hkv, n, dtype=torch.float64, device=DEV)
        for b in range(B):
            for g in range(Hkv):
                m, s, x = _stats(k[b, g, :lens[b]].double(), c["block"], "f32", c["sub"])
                j = m.shape[0]
                mu[b, g, :, :j], sg[b, g, :, :j], M[b, g, :j] = m.t(), s.t(), x
        return {"mu": mu, "sigma": sg, "max_norm": M}
    if c["kind"] == "prefill":
        q, k, v, tau, lens = _prefill_inputs(c, seed)
        B, Hq, T, d = q.shape
        G = Hq // c["Hkv"]
        out = torch.zeros(q.shape, dtype=torch.float64, device=DEV)
        R = torch.zeros(B, Hq, T, dtype=torch.float64, device=DEV)
        L = torch.full((B, Hq, T), -math.inf, dtype=torch.float64, device=DEV)
        for b in range(B):
            for h in range(Hq):
                kd, vd = k[b, h // G].double(), v[b, h // G].double()
                for r0 in range(0, lens[b], 4096):
                    r1 = min(r0 + 4096, lens[b])
                    s = q[b, h, r0:r1].double() @ kd[:r1].t() / math.sqrt(d)
                    i = torch.arange(r0, r1, device=DEV)[:, None]
                    j = torch.arange(r1, device=DEV)[None]
                    gate = torch.sigmoid(BETA * (s - tau[b, h, r0:r1, None].double()))
                    x = s + 3.0 * gate - 3.0 if c["additive"] else s * gate
                    x = torch.where(i == j, s, x).masked_fill_(j > i, -math.inf)
                    R[b, h, r0:r1] = gate.masked_fill_(j > i, 0.0).sum(1)
                    L[b, h, r0:r1] = torch.logsumexp(x, dim=1)
                    out[b, h, r0:r1] = _softmax_rows(x, vd[:r1])
        return {"out": out, "R": R, "L": L}
    q, k, tau = _calib_inputs(c, seed)
    N, Hq, T, d = q.shape
    G, nb = Hq // c["Hkv"], c["bins"]
    wt = 1.0 / torch.arange(1, T + 1, device=DEV, dtype=torch.float64)
    hist = torch.zeros(Hq, nb, dtype=torch.float64, device=DEV)
    dens = torch.zeros(Hq, dtype=torch.float64, device=DEV)
    low = torch.ones(T, T, dtype=torch.bool, device=DEV).tril()
    ww = wt[:, None].expand(T, T)[low]
    width = (CALIB_HI - CALIB_LO) / nb
    for x in range(N):
        for h in range(Hq):
            s = q[x, h].double() @ k[x, h // G].double().t() / math.sqrt(d)
            bins = ((s[low] - CALIB_LO) / width).floor().clamp(0, nb - 1).long()
            hist[h] += torch.bincount(bins, weights=ww, minlength=nb)
            gate = torch.sigmoid(BETA * (s - tau[x, h, :, None].double()))
            dens[h] += (gate * wt[:, None])[low].sum()
    total = float(N * T)
    target = dens / total
    mid = CALIB_LO + (torch.arange(nb, device=DEV, dtype=torch.float64) + 0.5) * width
    lo = torch.full((Hq,), CALIB_LO - 60.0 / BETA, dtype=torch.float64, device=DEV)
    hi = torch.full((Hq,), CALIB_HI + 60.0 / BETA, dtype=torch.float64, device=DEV)
    for _ in range(80):
        m = 0.5 * (lo + hi)
        g = (hist / total * torch.sigmoid(BETA * (mid[None] - m[:, None]))).sum(1)
        lo, hi = torch.where(g > target, m, lo), torch.where(g > target, hi, m)
    return {"c": 0.5 * (lo + hi), "target": target, "hist": hist, "density": dens}
