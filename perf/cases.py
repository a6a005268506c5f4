"""Workloads the library's speed is measured on, through its Python entry points.

Every case is one thing a serving or calibration program does with the library:

  prune      occam.prune: score, threshold, compact and gather in one call
             (``call = "steps"``: occam.score / threshold / select / gather in turn)
  topk       occam.score, occam.select_topk, occam.gather: the fixed-budget variant
  redirect   occam.register_redirect on an MLP activation, in place
  calibrate  occam.match_lambda on a calibration batch's scores

Inputs are drawn on the GPU from the seed: Gaussian queries and keys, a few high-norm sink
keys per sample, and keys aligned with an anchor row, as in the package's synthetic
workloads.  lambda is calibrated on the drawn batch the way budget matching does it (the
geometric midpoint between two neighbouring ratios, here the widest gap near the wanted
count), so that rounding in the last bits of a score cannot move a survivor.
"""
from __future__ import annotations

import math
import random

import torch

from paper_2605_29657_amd import occam

DEV = "cuda"
TDT = {"bf16": torch.bfloat16, "f32": torch.float32}
ESZ = {"bf16": 2, "f32": 4}


def _prune(name=None, **kw):
    c = dict(kind="prune", stage="vis", B=1, R=4, H=16, Hkv=16, d=64, T=1, T_lo=0, N=576, N_lo=0,
             dtype="bf16", hidden=1024, kv_rows=False, keep=0.18, lse=False, mapped=False,
             call="prune", sizes=0)
    c.update(kw)
    return dict(c, name=name) if name else c


def listed():
    return [
        # One LLaVA-1.5 image through the float32 vision tower: the smallest call, latency.
        _prune("cls_image_f32", dtype="f32", keep=0.43),
        # LLaVA-NeXT batch, vision stage: five tiles of 576 tokens per image.
        _prune("cls_next", B=32, N=2880),
        # A 12-head encoder over images of mixed sizes, vision stage: ragged batch.
        _prune("cls_ragged_12h", B=24, R=1, H=12, Hkv=12, N=1200, N_lo=97, hidden=768, keep=0.25,
               sizes=3),
        # Fixed token budget on a ragged Qwen3-VL-shaped vision batch (head dim 72).
        dict(name="topk_ragged", kind="topk", B=64, R=4, H=16, Hkv=16, d=72, N=4096, N_lo=256,
             dtype="bf16", hidden=1152, k_keep=96, sizes=5),
        # One LLaVA-NeXT image, text stage: a single request being served.
        _prune("text_image", stage="txt", B=1, H=32, Hkv=32, d=128, T=128, N=2880, hidden=4096,
               kv_rows=True, keep=0.014),
        # LLaVA-NeXT batch, text stage: the headline batch.
        _prune("text_next", stage="txt", B=32, H=32, Hkv=32, d=128, T=128, N=2880, hidden=4096,
               kv_rows=True, keep=0.014),
        # Ragged batch (images and prompts of all lengths) on a grouped-query model.
        _prune("text_ragged_gqa", stage="txt", B=64, H=32, Hkv=8, d=128, T=512, T_lo=16, N=4096,
               N_lo=256, hidden=4096, kv_rows=True, keep=0.11, sizes=7),
        # Text stage over the tokens a vision stage kept, with the attention kernel's own
        # normalisers and the original token indices: one pass over few keys.
        _prune("text_chained_lse", stage="txt", B=32, H=32, Hkv=32, d=128, T=128, N=1100, N_lo=64,
               hidden=4096, kv_rows=True, keep=0.09, lse=True, mapped=True, sizes=11),
        # Eight videos of 8 x 2048 tokens, text stage: the longest samples.
        _prune("text_video", stage="txt", B=8, R=8, H=32, Hkv=32, d=128, T=256, N=16384,
               hidden=4096, kv_rows=True, keep=0.02),
        # Mutual scoring (encoder without a CLS row): every token is an anchor row.
        _prune("mutual_ragged", stage="mut", B=16, H=16, Hkv=16, d=72, N=4096, N_lo=256,
               hidden=1152, keep=0.18, sizes=13),
        # Register construction on the vision MLP activations of the LLaVA-NeXT batch.
        dict(name="redirect_next", kind="redirect", B=32, R=4, N=2880, N_lo=0, width=4096,
             channels=10, dtype="bf16", sizes=0),
        # Budget matching on a calibration batch of 64 LLaVA-NeXT images.
        dict(name="calibrate", kind="calibrate", B=64, R=4, N=2880, N_lo=0, keep=0.2, sizes=0),
    ]


def _log_int(rng, lo, hi):
    return max(lo, min(hi, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


# A drawn case does at most the work of the largest listed one of its kind.
MAX_TEXT_FLOPS = 2.5e11
MAX_MUTUAL_FLOPS = 1.5e11
MAX_KEYS = 140000


def draw(rng):
    kind = rng.choice(["cls", "cls", "cls", "topk", "text", "text", "text", "text", "text",
                       "mutual", "redirect", "calibrate"])
    sizes = rng.randrange(1, 1 << 20)
    B = _log_int(rng, 1, 64)
    R = rng.choice([1, 4, 4, 8])
    N = _log_int(rng, 64, 4096)
    N_lo = max(16, N // rng.randint(2, 16)) if rng.random() < 0.5 else 0
    while B * (N + R) > MAX_KEYS:
        B -= 1
    if kind in ("cls", "topk"):
        H, d = rng.choice([(16, 64), (16, 64), (16, 72), (12, 64), (16, 80), (20, 64)])
        dtype = "f32" if kind == "cls" and rng.random() < 0.25 else "bf16"
        if kind == "topk":
            return dict(kind="topk", B=B, R=R, H=H, Hkv=H, d=d, N=N, N_lo=N_lo, dtype=dtype,
                        hidden=H * d, k_keep=min(_log_int(rng, 8, 256), (N_lo or N) // 2),
                        sizes=sizes)
        return _prune(B=B, R=R, H=H, Hkv=H, d=d, N=N, N_lo=N_lo, dtype=dtype, hidden=H * d,
                      keep=round(rng.uniform(0.1, 0.45), 3), sizes=sizes,
                      call="steps" if rng.random() < 0.2 else "prune")
    if kind == "text":
        H = rng.choice([16, 32, 32])
        Hkv = rng.choice([H, H, H // 4])
        d = rng.choice([128, 128, 128, 96, 64])
        T = _log_int(rng, 12, 512)
        T_lo = max(2, T // rng.randint(2, 16)) if N_lo and rng.random() < 0.6 else 0
        if rng.random() < 0.2:
            N, N_lo, T_lo = _log_int(rng, 4096, 16384), 0, 0
        while B > 1 and (B * (N + R) > MAX_KEYS or 2.0 * B * T * (N + R) * H * d > MAX_TEXT_FLOPS):
            B -= 1
        lse = rng.random() < 0.25
        return _prune(stage="txt", B=B, R=R, H=H, Hkv=Hkv, d=d, T=T, T_lo=T_lo, N=N, N_lo=N_lo,
                      hidden=H * d, kv_rows=True, keep=round(rng.uniform(0.012, 0.12), 3), lse=lse,
                      mapped=lse, sizes=sizes, call="steps" if rng.random() < 0.2 else "prune")
    if kind == "mutual":
        H, d = rng.choice([(16, 64), (16, 72), (16, 72), (12, 64)])
        while B > 1 and 2.0 * B * (N + R) ** 2 * H * d > MAX_MUTUAL_FLOPS:
            B -= 1
        return _prune(stage="mut", B=B, R=R, H=H, Hkv=H, d=d, N=N, N_lo=N_lo, hidden=H * d,
                      keep=round(rng.uniform(0.1, 0.45), 3), sizes=sizes)
    if kind == "redirect":
        width = rng.choice([3072, 4096, 4304, 5120])
        return dict(kind="redirect", B=B, R=R, N=N, N_lo=N_lo, width=width,
                    channels=_log_int(rng, 1, 64), dtype=rng.choice(["bf16", "bf16", "f32"]),
                    sizes=sizes)
    B = _log_int(rng, 8, 100)
    while B * (N + R) > 2 * MAX_KEYS:
        B -= 1
    return dict(kind="calibrate", B=B, R=R, N=N, N_lo=N_lo, keep=round(rng.uniform(0.02, 0.4), 3),
                sizes=sizes)


# ------------------------------------------------------------------------------- shapes
def _counts(case):
    """(anchor rows, candidates) of every sample: part of the case, not of the seed."""
    r = random.Random(case["sizes"])
    B, R = case["B"], case["R"]
    lo = case["N_lo"]
    N = [r.randint(lo, case["N"]) if lo else case["N"] for _ in range(B)]
    if case.get("stage") == "mut":
        return [n + R for n in N], N
    t_lo = case.get("T_lo", 0)
    T = [r.randint(t_lo, case["T"]) if t_lo else case.get("T", 1) for _ in range(B)]
    return T, N


def _prefix(xs):
    out = [0]
    for x in xs:
        out.append(out[-1] + x)
    return out


def work(case):
    T, N = _counts(case)
    R, B = case["R"], case["B"]
    S = [n + R for n in N]
    if case["kind"] == "redirect":
        e = ESZ[case["dtype"]]
        # The listed channels of every visual row are read and cleared, one row written.
        return {"bytes": float(sum(N) * 2 + B) * case["channels"] * e, "flops": 0.0}
    if case["kind"] == "calibrate":
        return {"bytes": 4.0 * sum(S), "flops": 0.0}
    e, H, Hkv, d = ESZ[case["dtype"]], case["H"], case["Hkv"], case["d"]
    kept = B * case["k_keep"] if case["kind"] == "topk" else case["keep"] * sum(N)
    row = case["hidden"] * e + (2 * Hkv * d * e if case.get("kv_rows") else 0)
    b = sum(S) * Hkv * d * e + sum(T) * H * d * e + 4.0 * sum(S) + kept * (2 * row + 4) + 8.0 * B
    if case.get("lse"):
        b += 4.0 * sum(T) * H
    if case.get("mapped"):
        b += 4.0 * kept
    return {"bytes": float(b), "flops": 2.0 * sum(t * s for t, s in zip(T, S)) * H * d}


# ------------------------------------------------------------------------------- inputs
def _aligned(k, idx, direction, cos, gen):
    """Turn the keys ``idx`` to ``cos`` against ``direction`` ([n, heads, d]), norms kept."""
    old = k[idx].float()
    dhat = torch.nn.functional.normalize(direction.float(), dim=-1)
    u = torch.randn(old.shape, generator=gen, device=DEV)
    u = torch.nn.functional.normalize(u - (u * dhat).sum(-1, keepdim=True) * dhat, dim=-1)
    c = cos.view(-1, 1, 1)
    k[idx] = (old.norm(dim=-1, keepdim=True) * (c * dhat + torch.sqrt(1 - c * c) * u)).to(k.dtype)


def _scores(case, x, dt, row_lse=None, want_lse=False):
    """Scores by plain torch in ``dt``: softmax over the sample's keys of every (row, head),
    mean over heads, max (text) or mean (mutual) over rows, registers by the mean."""
    T, N = _counts(case)
    R, H, Hkv, d = case["R"], case["H"], case["Hkv"], case["d"]
    scale = 1.0 / math.sqrt(d)
    out, lses, qo, ko = [], [], 0, 0
    for t, n in zip(T, N):
        q = x["q"][qo:qo + t].to(dt).view(t, Hkv, H // Hkv, d).permute(1, 2, 0, 3)
        k = x["k"][ko:ko + R + n].to(dt).permute(1, 2, 0).contiguous()
        l = torch.bmm(q.reshape(Hkv, -1, d), k).view(H, t, R + n).mul_(scale)
        lse = torch.logsumexp(l, -1) if row_lse is None else row_lse[qo:qo + t].to(dt).t()
        p = l.sub_(lse.unsqueeze(-1)).exp_().mean(0)
        s = p.mean(0)
        if case.get("stage") != "mut":
            s[R:] = p[:, R:].max(0).values
        out.append(s)
        lses.append(lse.t())
        qo, ko = qo + t, ko + R + n
    return (torch.cat(out), torch.cat(lses)) if want_lse else torch.cat(out)


def _calibrated(ratios, keep):
    """lambda: the geometric midpoint of the widest gap between neighbouring ratios within
    2 % of the wanted count."""
    r = torch.sort(ratios.double(), descending=True).values
    m = r.numel()
    c = max(1, min(m - 1, int(keep * m)))
    w = max(4, int(0.02 * c))
    lo, hi = max(0, c - w), min(m - 1, c + w)
    gap = (r[lo:hi] / r[lo + 1:hi + 1])
    j = lo + int(torch.argmax(gap))
    return math.sqrt(float(r[j]) * float(r[j + 1]))


def _anchor_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    cpu = random.Random(int(seed))
    T, N = _counts(case)
    B, R, H, Hkv, d = (case[n] for n in ("B", "R", "H", "Hkv", "d"))
    dt = TDT[case["dtype"]]
    ko, qo, co = _prefix([n + R for n in N]), _prefix(T), _prefix(N)
    x = dict(q=torch.randn(qo[-1], H, d, generator=gen, device=DEV).to(dt),
             k=torch.randn(ko[-1], Hkv, d, generator=gen, device=DEV).to(dt),
             hidden=torch.randn(co[-1], case["hidden"], generator=gen, device=DEV).to(dt))
    sinks, rel, rows, cos = [], [], [], []
    for b in range(B):
        n_rel = case["k_keep"] - 3 if case["kind"] == "topk" else (
            cpu.randint(5, 40) if case["stage"] == "txt" else 20 * N[b] // 576)
        pick = cpu.sample(range(N[b]), min(N[b], 3 + n_rel))
        sinks += [ko[b] + R + v for v in pick[:3]]
        rel += [ko[b] + R + v for v in pick[3:]]
        rows += [qo[b] + (cpu.randrange(T[b]) if T[b] > 1 else 0) for _ in pick[3:]]
        cos += [cpu.uniform(0.45, 0.6) if case["kind"] == "topk" else 0.6 for _ in pick[3:]]
    if rel:
        idx = torch.tensor(rel, device=DEV)
        _aligned(x["k"], idx, x["q"][torch.tensor(rows, device=DEV)][:, ::H // Hkv],
                 torch.tensor(cos, device=DEV), gen)
    x["k"][torch.tensor(sinks, device=DEV)] *= 8.0
    if case.get("kv_rows"):
        x["v"] = torch.randn(ko[-1], Hkv * d, generator=gen, device=DEV).to(dt)
    if case["kind"] == "topk":
        return x
    s, lse = _scores(case, x, torch.float32, want_lse=True)
    if case["lse"]:
        # The attention kernel's normaliser also covers the prompt's text keys.
        more = torch.rand(lse.shape, generator=gen, device=DEV)
        x["row_lse"] = (lse + torch.log1p(more)).contiguous()
        s = _scores(case, x, torch.float32, row_lse=x["row_lse"])
    if case["mapped"]:
        # Original indices of the tokens an earlier stage kept: ascending, with gaps.
        x["index_map"] = torch.cat([torch.cumsum(torch.randint(
            1, 6, (n,), generator=gen, device=DEV, dtype=torch.int32), 0) for n in N]).int()
    ratio = torch.cat([s[ko[b] + R:ko[b + 1]] / s[ko[b]:ko[b] + R].mean() for b in range(B)])
    x["lam"] = _calibrated(ratio, case["keep"])
    return x


def _i32(xs):
    return torch.tensor(xs, dtype=torch.int32, device=DEV)


def _problem(case):
    T, N = _counts(case)
    rr = occam.ROWS_MEAN if case.get("stage") == "mut" else occam.ROWS_MAX
    ragged_n, ragged_t = bool(case["N_lo"]), len(set(T)) > 1
    return occam.Problem(
        case["B"], case.get("H", 1), case.get("Hkv", 1), case.get("d", 64), case["R"], rows=T[0],
        cands=N[0], q_offsets=_i32(_prefix(T)) if ragged_t else None,
        key_offsets=_i32(_prefix([n + case["R"] for n in N])) if ragged_n else None,
        max_rows=max(T), max_cands=max(N), dtype=case.get("dtype", "f32"), visual_row_reduce=rr)


def prepare(case, seed):
    T, N = _counts(case)
    B, R = case["B"], case["R"]
    st = dict(case=case, problem=_problem(case))
    if case["kind"] == "redirect":
        st.update(_redirect_inputs(case, seed))
        return st
    if case["kind"] == "calibrate":
        st["scores"] = _calibration_scores(case, seed)
        st["ws"] = occam.workspace(st["problem"])
        st["lam"] = torch.zeros(1, device=DEV)
        st["mean"] = torch.zeros(1, device=DEV)
        return st
    x = _anchor_inputs(case, seed)
    st.update(x)
    keys, cands = sum(N) + R * B, sum(N)
    st["ws"] = occam.workspace(st["problem"])
    # Outputs of worst-case size, cleared once: the unused ends stay zero.
    st["out"] = dict(scores=torch.zeros(keys, device=DEV), tau=torch.zeros(B, device=DEV),
                     kept_idx=_i32([0]).repeat(cands), kept_count=_i32([0] * B),
                     kept_offsets=_i32([0] * (B + 1)))
    src = [(x["hidden"], 0, 0)]
    if case.get("kv_rows"):
        src += [(x["k"].view(keys, -1), R, R), (x["v"], R, R)]
    st["dst"] = [torch.zeros(cands, s.shape[1], dtype=s.dtype, device=DEV) for s, _, _ in src]
    st["rows"] = [occam.Rows(s, o, src_pad_rows=pad, src_row0=row0)
                  for (s, pad, row0), o in zip(src, st["dst"])]
    return st


def _redirect_inputs(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    _, N = _counts(case)
    rows = sum(N) + case["R"] * case["B"]
    h = torch.empty(rows, case["width"], dtype=TDT[case["dtype"]], device=DEV)
    for r in range(0, rows, 1 << 14):
        m = min(1 << 14, rows - r)
        h[r:r + m] = torch.nn.functional.gelu(torch.randn(m, case["width"], generator=gen, device=DEV))
    ch = torch.randperm(case["width"], generator=gen, device=DEV)[:case["channels"]]
    return dict(h=h, channels=ch.int().contiguous())


def _calibration_scores(case, seed):
    gen = torch.Generator(device=DEV).manual_seed(int(seed))
    _, N = _counts(case)
    rows = sum(N) + case["R"] * case["B"]
    # A mean over heads of exponentiated logits, on the scale of a softmax over N keys.
    return torch.randn(rows, 16, generator=gen, device=DEV).exp().mean(1) / (1.6 * case["N"])


# ------------------------------------------------------------------------------- passes
def run(state):
    c, p = state["case"], state["problem"]
    if c["kind"] == "redirect":
        # In place: a second pass on the same state finds the channels already cleared.
        occam.register_redirect(p, state["h"], state["channels"])
        return state["h"]
    if c["kind"] == "calibrate":
        occam.match_lambda(p, state["scores"], c["keep"] * c["N"], state["lam"], state["ws"],
                           mean_kept=state["mean"])
        return dict(lam=state["lam"], mean=state["mean"])
    o, ws, rows = state["out"], state["ws"], state["rows"]
    lists = (o["kept_idx"], o["kept_count"], o["kept_offsets"])
    if c["kind"] == "topk":
        occam.score(p, state["q"], state["k"], o["scores"], ws)
        occam.select_topk(p, o["scores"], c["k_keep"], *lists, ws)
        occam.gather(p, rows, o["kept_idx"], o["kept_offsets"])
    elif c["call"] == "steps":
        occam.score(p, state["q"], state["k"], o["scores"], ws, row_lse=state.get("row_lse"))
        occam.threshold(p, o["scores"], state["lam"], occam.REG_MEAN, o["tau"])
        occam.select(p, o["scores"], o["tau"], *lists, ws)
        occam.gather(p, rows, o["kept_idx"], o["kept_offsets"])
    else:
        occam.prune(p, state["q"], state["k"], state["lam"], *lists, ws, rows=rows,
                    scores=o["scores"], tau=o["tau"], row_lse=state.get("row_lse"),
                    index_map=state.get("index_map"))
    return dict(o, rows=state["dst"])


def tolerance(case):
    if case["kind"] == "redirect":
        return "exact"
    # Scores and thresholds are float32 sums of products that are exact in float32 (bf16
    # inputs) or rounded once (float32 inputs): measured 1e-7 to 7e-7 from float64 over all
    # forms.  The survivors and their rows do not move (the calibrated gap).
    return {"rel": 3e-6, "max": 3e-5}


def exact(case, seed):
    """Scores, thresholds, the redirected activation, the matched lambda in 64 bits.
    Survivor lists and gathered rows are whole values and copies."""
    _, N = _counts(case)
    B, R = case["B"], case["R"]
    ko = _prefix([n + R for n in N])
    if case["kind"] == "redirect":
        x = _redirect_inputs(case, seed)
        h, ch = x["h"].double(), x["channels"].long()
        for b in range(B):
            vis = h[ko[b] + R:ko[b + 1]]
            h[ko[b], ch] = vis[:, ch].max(0).values
            vis[:, ch] = 0.0
        return h
    if case["kind"] == "calibrate":
        s = _calibration_scores(case, seed).double()
        r = torch.cat([s[ko[b] + R:ko[b + 1]] / s[ko[b]:ko[b] + R].mean() for b in range(B)])
        r = torch.sort(r, descending=True).values
        t = case["keep"] * case["N"] * B
        n = max(1, min(r.numel() - 1, math.ceil(t - 0.5)))
        return dict(lam=torch.sqrt(r[n - 1] * r[n]).view(1), mean=torch.tensor([n / B]).double())
    x = _anchor_inputs(case, seed)
    s = _scores(case, x, torch.float64, row_lse=x.get("row_lse"))
    tau = None
    if case["kind"] == "prune":
        tau = x["lam"] * torch.stack([s[ko[b]:ko[b] + R].mean() for b in range(B)])
    return dict(scores=s, tau=tau, kept_idx=None, kept_count=None, kept_offsets=None, rows=None)
