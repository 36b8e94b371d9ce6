"""The work that a serving program has this library do, as timed cases.

A decode step of one layer scores the whole projected-key cache, selects a token budget per query
head and attends over the selected rows; between predictions a kept selection is reused.  Prompts
are projected once when they have been read, and a producer layer's predictor makes the importance
queries.  The cases below are these calls at the sizes of this repository's configurations and
tests: the smallest one, the named long-context ones, ragged ones and the largest row that the
selection takes.  Everything goes through ``paper_2503_07518_amd.binding`` and ``interval``.
"""
import math

import torch

from paper_2503_07518_amd import binding as tb
from paper_2503_07518_amd import interval, workloads

DEV = "cuda"
CACHE_BYTES_MAX = 6 << 30  # K and V of a drawn case, so that several states fit a card easily


# ---- the cases ------------------------------------------------------------------------------------
def _step(name, **kw):
    c = dict(name=name, kind="step", sink=0, window=0, zipf=False)
    c.update(kw)
    return c


def listed():
    return [
        # One prediction step of the tiny fp32 configuration: a call bound by launches and latency.
        _step("step_tiny_f32", dtype="f32", B=1, Hq=8, Hkv=8, D=64, N=1024, Dimp=16, k=128),
        # Interactive decoding, one sequence at 32K context: the headline configuration.
        _step("step_32k", dtype="bf16", B=1, Hq=32, Hkv=8, D=128, N=32768, Dimp=32, k=3277),
        # A serving batch of 16 sequences at 16K context.
        _step("step_batch16_16k", dtype="bf16", B=16, Hq=32, Hkv=8, D=128, N=16384, Dimp=32, k=2048),
        # Long contexts on a model with 64 query heads, projected keys of very uneven magnitude.
        _step("step_128k_64heads", dtype="bf16", B=4, Hq=64, Hkv=8, D=128, N=131072, Dimp=32, k=4096, zipf=True),
        # The longest row the selection takes: one sequence of 1M tokens, an 8K budget.
        _step("step_1m", dtype="bf16", B=1, Hq=32, Hkv=8, D=128, N=1 << 20, Dimp=32, k=8192),
        # A small mixed batch in the middle of decoding: an odd length, 16 projected dimensions, sink
        # prefix and local window kept as the selection policy asks.
        _step("step_ragged_d16", dtype="bf16", B=3, Hq=32, Hkv=8, D=128, N=20011, Dimp=16, k=2049, sink=128, window=256),
        # A whole prediction interval with neighbour fetching: 8 new rows projected, one prediction
        # step, the selection widened, 7 steps that reuse it plus the rows appended since.
        dict(name="interval_64k", kind="interval", dtype="bf16", B=4, Hq=32, Hkv=8, D=128, N=65536, Dimp=32, k=4096,
             sink=0, window=0, P=8, radius=1, mode=0),
        # The three-buffer layout over one interval of 16 steps and the step at which the local
        # window's ring is full: its keys are projected in one batch and a prediction follows.
        dict(name="ring_16k", kind="ring", dtype="bf16", B=2, Hq=32, Hkv=8, D=128, N=16384, Dimp=16, k=1024,
             sink=128, ring=256, P=16, radius=1, mode=1),
        # The variant with one importance head: one list per sequence for all heads.
        dict(name="headless_32k", kind="headless", dtype="bf16", B=4, Hq=32, Hkv=8, D=128, N=32768, Dimp=32, k=3277,
             sink=128, window=256),
        # After the prompt: the keys of the whole cache are projected.
        dict(name="prefill_projection", kind="project", dtype="bf16", B=1, Hkv=8, D=128, N=32768, Dimp=32, per_head=False),
        # A producer layer's query predictor for one sequence and for a batch.
        dict(name="predict_b1", kind="predict", dtype="bf16", B=1, E=4096, hidden=512, G=4, Hq=32, Dimp=32),
        dict(name="predict_b16", kind="predict", dtype="bf16", B=16, E=4096, hidden=512, G=4, Hq=32, Dimp=32),
    ]


def _log_int(rng, lo, hi):
    """A whole number spread over the logarithm of [lo, hi]."""
    return min(hi, max(lo, int(round(math.exp(rng.uniform(math.log(lo), math.log(hi)))))))


def _cache_bytes(c):
    return 2 * c["B"] * c["Hkv"] * c["N"] * c["D"] * _elt(c)


def _draw_decode(rng, kind):
    # (the interval and ring loops run several steps a pass: shorter rows and smaller batches)
    most_n = {"step": 1 << 20, "headless": 1 << 17, "interval": 1 << 16, "ring": 1 << 15}[kind]
    g = rng.choice((1, 2, 4, 4, 4, 8))
    hkv = rng.choice((1, 2, 4, 8, 8, 8))
    n = _log_int(rng, 1024, most_n)
    if rng.random() < 0.3:
        n = max(1024, n // 1024 * 1024)  # (cache lengths are as often round as they are odd)
    c = dict(kind=kind, dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), B=_log_int(rng, 1, 16 if kind in ("step", "headless") else 4),
             Hq=g * hkv, Hkv=hkv, D=rng.choice((64, 128, 128, 128)), N=n, Dimp=rng.choice((16, 32, 32, 64)),
             k=max(32, min(8192, int(n * math.exp(rng.uniform(math.log(0.01), math.log(0.2)))))),
             sink=rng.choice((0, 4, 128)), window=rng.choice((0, 64, 256)))
    if kind == "step":
        c["zipf"] = rng.random() < 0.15
    if kind in ("interval", "ring"):
        c["P"], c["radius"], c["mode"] = rng.choice((4, 8, 16)), rng.choice((1, 1, 2)), rng.choice((0, 0, 1))
    if kind == "ring":
        c["ring"] = c["P"] * rng.choice((2, 4, 16))
        del c["window"]
    return c


def draw(rng):
    most = {}
    for c in listed():
        most[c["kind"]] = max(most.get(c["kind"], 0.0), work(c)["bytes"])
    while True:
        kind = rng.choice(("step", "step", "step", "step", "interval", "ring", "headless", "project", "predict", "predict"))
        if kind == "project":
            c = dict(kind=kind, dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), B=_log_int(rng, 1, 16), Hkv=rng.choice((1, 4, 8, 8)),
                     D=rng.choice((64, 128, 128)), N=_log_int(rng, 512, 131072), Dimp=rng.choice((16, 32, 32, 64)),
                     per_head=rng.random() < 0.25)
        elif kind == "predict":
            c = dict(kind=kind, dtype=rng.choice(("bf16", "bf16", "bf16", "f32")), B=_log_int(rng, 1, 64), E=rng.choice((2048, 3072, 4096, 5120, 8192)),
                     hidden=rng.choice((256, 512, 512, 520, 1024)), G=rng.choice((1, 2, 4, 4)), Hq=rng.choice((8, 16, 32, 32, 64)), Dimp=rng.choice((16, 32, 32)))
            if c["dtype"] == "f32" or c["E"] > 4096:
                c["B"] = min(c["B"], 24)
            if work(c)["bytes"] <= 8 * most[kind]:
                return c
            continue
        else:
            c = _draw_decode(rng, kind)
        if kind != "project" and _cache_bytes(c) > CACHE_BYTES_MAX:
            continue
        limit = 8 * most[kind] if kind in ("project", "ring", "headless") else most[kind]
        if work(c)["bytes"] <= limit:
            return c


# ---- inputs ---------------------------------------------------------------------------------------
def _elt(c):
    return 4 if c["dtype"] == "f32" else 2


def _torch_dtype(c):
    return torch.float32 if c["dtype"] == "f32" else torch.bfloat16


def _layer(c, seed, steps=1):
    """One layer's cache as the workload generator draws it (planted heavy tokens, queries that
    the importance queries follow), its prompt's keys projected."""
    heavy = max(1, min(c["N"] // 100, c["N"] // max(1, steps) // 4))
    cfg = workloads.DecodeConfig(c["kind"], B=c["B"], Hq=c["Hq"], Hkv=c["Hkv"], D=c["D"], N=c["N"], Dimp=c["Dimp"], k=c["k"],
                                 dtype=c["dtype"], heavy_per_kv_head=heavy, steps=steps, zipf_kimp=bool(c.get("zipf")))
    data = workloads.make_layer(cfg, seed=seed, device=DEV)
    K, V = data["K"], data["V"]
    Kimp = torch.zeros((c["B"], c["Hkv"], K.shape[2], c["Dimp"]), dtype=K.dtype, device=DEV)
    tb.tb_project_keys(tb.make_desc(c["N"], c["Hq"], K=K, V=V, Kimp=Kimp), K, data["W"], Kimp, 0, c["N"])
    workloads.apply_kimp_row_scale(Kimp, data["kimp_row_scale"])
    return cfg, data, K, V, Kimp


def _padded(n):
    return (n + 3) // 4 * 4


def _prepare_step(c, seed):
    cfg, data, K, V, Kimp = _layer(c, seed)
    B, Hq, N = c["B"], c["Hq"], c["N"]
    cap = tb.policy_count(N, c["k"], c["sink"], c["window"])
    desc = tb.make_desc(N, Hq, K=K, V=V, Kimp=Kimp)
    return dict(case=c, desc=desc, K=K, V=V, Kimp=Kimp, q=data["q"][0].contiguous(), q_imp=data["q_imp"][0].contiguous(), sm=cfg.sm_scale,
                scores=torch.zeros((B, Hq, _padded(N)), dtype=torch.float32, device=DEV),
                idx=torch.zeros((B, Hq, cap), dtype=torch.int32, device=DEV), cnt=torch.zeros((B, Hq), dtype=torch.int32, device=DEV),
                out=torch.empty((B, Hq, c["D"]), dtype=torch.float32, device=DEV), lse=torch.empty((B, Hq), dtype=torch.float32, device=DEV),
                ws=tb.new_workspace(tb.TB_OP_DECODE_STEP, desc, cap))


def _run_step(s):
    c = s["case"]
    tb.tb_decode_step(s["desc"], s["q_imp"], s["Kimp"], 1.0, s["q"], s["K"], s["V"], c["k"], c["sink"], c["window"], s["sm"],
                      s["scores"], s["idx"], s["cnt"], s["out"], s["lse"], s["ws"])
    return s["scores"], s["idx"], s["cnt"], s["out"], s["lse"]


def _prepare_interval(c, seed):
    cfg, data, K, V, Kimp = _layer(c, seed, steps=c["P"])
    dec = interval.IntervalDecoder(K, V, data["W"], Kimp, c["Hq"], c["k"], c["P"], c["radius"], sink=c["sink"], window=c["window"],
                                   sm_scale=cfg.sm_scale, mode=c["mode"])
    return dict(case=c, dec=dec, q=[t.contiguous() for t in data["q"]], q_imp=[t.contiguous() for t in data["q_imp"]])


def _run_interval(s):
    c, dec = s["case"], s["dec"]
    dec.projected_upto = c["N"] - c["P"]  # the rows of the interval before this one are still to be projected
    outs = []
    for t in range(c["P"]):
        out, lse = dec.step(t, c["N"] + t, s["q"][t], s["q_imp"][t])
        outs.append(out.clone())  # (the decoder's own buffers hold until the next step only)
    return outs, lse, dec.scores[:, :, :c["N"]], dec.idx, dec.cnt, dec.exp_idx, dec.exp_cnt, dec.Kimp[:, :, c["N"] - c["P"]:c["N"]]


def _prepare_ring(c, seed):
    R, P = c["ring"], c["P"]
    cfg, data, K, V, Kimp = _layer(c, seed, steps=R + 1)
    dec = interval.RingLayoutDecoder(K, V, data["W"], Kimp, c["Hq"], c["k"], P, c["radius"], R, sink=c["sink"], sm_scale=cfg.sm_scale,
                                     mode=c["mode"])
    # the ring as the steps before this interval have filled it
    dec.aux_K[:, :, c["sink"]:].copy_(K[:, :, c["N"]:c["N"] + R])
    dec.aux_V[:, :, c["sink"]:].copy_(V[:, :, c["N"]:c["N"] + R])
    first = R - P
    return dict(case=c, dec=dec, q=[data["q"][t].contiguous() for t in range(first, R + 1)],
                q_imp=[data["q_imp"][t].contiguous() for t in range(first, R + 1)])


def _run_ring(s):
    c, dec = s["case"], s["dec"]
    first = c["ring"] - c["P"]
    outs = []
    for i in range(c["P"] + 1):
        t = first + i
        out, lse = dec.step(t, c["N"] + t, s["q"][i], s["q_imp"][i])
        outs.append(out.clone())
    return outs, lse, dec.scores[:, :, :c["N"]], dec.idx, dec.cnt, dec.exp_idx, dec.exp_cnt, dec.imp_cnt, dec.Kimp[:, :, c["N"]:c["N"] + c["ring"]]


def _prepare_headless(c, seed):
    cfg, data, K, V, Kimp = _layer(c, seed)
    B, Hq, N = c["B"], c["Hq"], c["N"]
    Kimp = Kimp[:, :1].contiguous()  # one importance head: the first KV head's projected keys
    q_imp = data["q_imp"][0][:, :1].contiguous()
    cap = tb.policy_count(N, c["k"], c["sink"], c["window"])
    d1 = tb.make_desc(N, 1, Kimp=Kimp)
    desc = tb.make_desc(N, Hq, K=K, V=V, Dimp=c["Dimp"])
    return dict(case=c, d1=d1, desc=desc, K=K, V=V, Kimp=Kimp, q=data["q"][0].contiguous(), q_imp=q_imp, sm=cfg.sm_scale, cap=cap,
                scores=torch.zeros((B, 1, _padded(N)), dtype=torch.float32, device=DEV),
                idx=torch.zeros((B, 1, cap), dtype=torch.int32, device=DEV), cnt=torch.zeros((B, 1), dtype=torch.int32, device=DEV),
                out=torch.empty((B, Hq, c["D"]), dtype=torch.float32, device=DEV), lse=torch.empty((B, Hq), dtype=torch.float32, device=DEV),
                sel_ws=tb.new_workspace(tb.TB_OP_SELECT, d1, cap), ws=tb.new_workspace(tb.TB_OP_ATTN, desc, cap))


def _run_headless(s):
    c = s["case"]
    tb.tb_score(s["d1"], s["q_imp"], s["Kimp"], 1.0, s["scores"])
    tb.tb_select_topk(s["d1"], s["scores"], c["k"], c["sink"], c["window"], s["idx"], s["cnt"], s["sel_ws"])
    tb.tb_sparse_decode_attn_shared(s["desc"], s["q"], s["K"], s["V"], s["idx"], s["cnt"], s["cap"], s["sm"], s["out"], s["lse"], s["ws"])
    return s["scores"], s["idx"], s["cnt"], s["out"], s["lse"]


def _prepare_project(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    td = _torch_dtype(c)
    K = torch.randn((c["B"], c["Hkv"], c["N"], c["D"]), generator=gen, device=DEV).to(td)
    W = (torch.randn((c["Hkv"] if c["per_head"] else 1, c["D"], c["Dimp"]), generator=gen, device=DEV) / math.sqrt(c["D"])).to(td)
    Kimp = torch.zeros((c["B"], c["Hkv"], c["N"], c["Dimp"]), dtype=td, device=DEV)
    return dict(case=c, desc=tb.make_desc(c["N"], c["Hkv"], K=K, Kimp=Kimp), K=K, W=W, Kimp=Kimp)


def _run_project(s):
    tb.tb_project_keys(s["desc"], s["K"], s["W"], s["Kimp"], 0, s["case"]["N"])
    return s["Kimp"]


def _prepare_predict(c, seed):
    gen = torch.Generator(device=DEV).manual_seed(seed)
    td = _torch_dtype(c)

    def r(*shape, scale=1.0, shift=0.0):
        return (torch.randn(shape, generator=gen, device=DEV) * scale + shift).to(td)

    B, E, hidden, n_out = c["B"], c["E"], c["hidden"], c["G"] * c["Hq"] * c["Dimp"]
    return dict(case=c, h=r(B, E, scale=2.0, shift=0.5), gamma=r(E, scale=0.2, shift=1.0), beta=r(E, scale=0.2),
                W1=r(hidden, E, scale=E ** -0.5), b1=r(hidden, scale=0.3), W2=r(n_out, hidden, scale=hidden ** -0.5), b2=r(n_out, scale=0.3),
                hidden_act=torch.empty((B, hidden), dtype=torch.float32, device=DEV), ln_act=torch.empty((B, E), dtype=torch.float32, device=DEV),
                q_imp=torch.empty((c["G"], B, c["Hq"], c["Dimp"]), dtype=td, device=DEV))


def _run_predict(s):
    c = s["case"]
    tb.tb_predict_queries(s["h"], s["gamma"], s["beta"], s["W1"], s["b1"], s["W2"], s["b2"], c["G"], c["Hq"], c["Dimp"], s["hidden_act"],
                          s["ln_act"], s["q_imp"])
    return s["q_imp"], s["hidden_act"]


PREPARE = dict(step=_prepare_step, interval=_prepare_interval, ring=_prepare_ring, headless=_prepare_headless, project=_prepare_project,
               predict=_prepare_predict)
RUN = dict(step=_run_step, interval=_run_interval, ring=_run_ring, headless=_run_headless, project=_run_project, predict=_run_predict)


def prepare(case, seed):
    return PREPARE[case["kind"]](case, seed)


def run(state):
    return RUN[state["case"]["kind"]](state)


# ---- what a pass cannot do without ------------------------------------------------------------------
def _attended(c, rows):
    """Bytes and flops of attention over `rows` listed rows per query head.  A row that several
    heads of a KV group list is needed once: with lists that do not depend on each other, a group of
    g heads lists N (1 - (1 - rows / N)^g) different rows."""
    g = c["Hq"] // c["Hkv"]
    n = float(c["N"])
    rows = min(float(rows), n)
    distinct = n * (1.0 - (1.0 - rows / n) ** g)
    bytes_ = c["B"] * c["Hkv"] * distinct * 2 * c["D"] * _elt(c) + c["B"] * c["Hq"] * (c["D"] * (4 + _elt(c)) + 4)
    return bytes_, 4.0 * c["B"] * c["Hq"] * rows * c["D"]


def _predicted(c, heads, kv_heads, window):
    """Scoring and selection: projected keys read, scores and lists written."""
    n, count = c["N"], tb.policy_count(c["N"], c["k"], c["sink"], window)
    bytes_ = c["B"] * (kv_heads * n * c["Dimp"] * _elt(c) + heads * (c["Dimp"] * _elt(c) + 4 * n + 4 * count + 4))
    return bytes_, 2.0 * c["B"] * heads * n * c["Dimp"], count


def work(case):
    c = case
    if c["kind"] == "project":
        rows = c["B"] * c["Hkv"] * c["N"]
        w = (c["Hkv"] if c["per_head"] else 1) * c["D"] * c["Dimp"]
        return {"bytes": (rows * (c["D"] + c["Dimp"]) + w) * _elt(c), "flops": 2.0 * rows * c["D"] * c["Dimp"]}
    if c["kind"] == "predict":
        n_out = c["G"] * c["Hq"] * c["Dimp"]
        weights = c["hidden"] * c["E"] + n_out * c["hidden"]
        bytes_ = (weights + c["hidden"] + n_out + 2 * c["E"] + c["B"] * (c["E"] + n_out)) * _elt(c) + c["B"] * c["hidden"] * 4
        return {"bytes": bytes_, "flops": 2.0 * c["B"] * weights}
    if c["kind"] == "headless":
        pb, pf, count = _predicted(c, 1, 1, c["window"])
        # one list per sequence: every head of a KV group reads the same rows
        ab = c["B"] * c["Hkv"] * count * 2 * c["D"] * _elt(c) + c["B"] * c["Hq"] * (c["D"] * (4 + _elt(c)) + 4)
        return {"bytes": pb + ab, "flops": pf + 4.0 * c["B"] * c["Hq"] * count * c["D"]}
    window = c["ring"] if c["kind"] == "ring" else c["window"]
    pb, pf, count = _predicted(c, c["Hq"], c["Hkv"], window)
    ab, af = _attended(c, count)
    if c["kind"] == "step":
        return {"bytes": pb + ab, "flops": pf + af}
    # the widened list: the sink and window entries, and k tokens with their neighbours (about as
    # many positions as the rule adds, less what neighbouring picks share)
    frac = c["k"] / c["N"]
    wide = count + (c["N"] * (1.0 - (1.0 - frac) ** (2 * c["radius"] + 1)) - c["k"] if c["mode"] == 0 else c["k"])
    eb = 4.0 * c["B"] * c["Hq"] * (count + wide)  # list read, widened list written
    wb, wf = _attended(c, wide)
    proj_rows = c["P"] if c["kind"] == "interval" else c["ring"]
    jb = c["B"] * c["Hkv"] * proj_rows * (c["D"] + c["Dimp"]) * _elt(c)
    jf = 2.0 * c["B"] * c["Hkv"] * proj_rows * c["D"] * c["Dimp"]
    if c["kind"] == "interval":
        return {"bytes": pb + ab + eb + jb + (c["P"] - 1) * wb, "flops": pf + af + jf + (c["P"] - 1) * wf}
    # ring: two predictions, each moving the widened list's rows into the per-head buffers; every step reads them
    moved = c["B"] * c["Hq"] * max(0.0, wide - c["sink"] - c["ring"]) * 2 * c["D"] * _elt(c)
    aux = c["B"] * c["Hkv"] * (c["sink"] + c["ring"]) * 2 * c["D"] * _elt(c)
    return {"bytes": 2 * (pb + eb + wb + moved) + jb + (c["P"] + 1) * (moved + aux), "flops": 2 * pf + jf + (c["P"] + 1) * wf}


def tolerance(case):
    # About four times what the results differ by from the same path evaluated in 64 bits, on the
    # listed sizes.  Scores, attention and hidden activations are fp32 sums whatever the storage type
    # (seen: 3e-7, largest 2e-6); lists of positions follow from the scores, and two scores that
    # differ only by rounding may change places.
    if case["kind"] in ("step", "headless") or case["dtype"] == "f32":
        return {"rel": 2e-6, "max": 2e-5, "differ": 0.001}
    # Results stored as bf16: a sum that rounds to the other neighbour is one unit in the last place
    # off (2^-7 of the value at most).  Predicted queries: seen 1e-4, the activations enter the
    # matrix cores as two bf16 numbers; projected keys: seen 1e-5.
    return {"rel": 5e-4 if case["kind"] == "predict" else 5e-5, "max": 0.02, "differ": 0.001}


# ---- the same numbers in 64 bits --------------------------------------------------------------------
def _exact_scores(q_imp, Kimp, n):
    """One batch element: [Hq, d'] queries, [Hkv, N, d'] projected keys -> [Hq, n] and the size of the
    sums' terms."""
    hq, hkv = q_imp.shape[0], Kimp.shape[0]
    q = q_imp.double().view(hkv, hq // hkv, -1)
    k = Kimp[:, :n].double()
    return torch.matmul(q, k.transpose(1, 2)).view(hq, n), torch.matmul(q.abs(), k.abs().transpose(1, 2)).view(hq, n)


def _exact_lists(scores, size, c):
    """[heads, N] scores -> the policy's lists [heads, count], or None where two scores at the budget's
    edge are closer than 32-bit sums resolve (either list is right then)."""
    n = scores.shape[1]
    lo = min(c["sink"], n)
    hi = max(lo, n - c["window"])
    kk = min(c["k"], hi - lo)
    pick = torch.topk(scores[:, lo:hi], min(kk + 1, hi - lo), dim=1)
    if kk < hi - lo:
        edge = lo + pick.indices[:, kk - 1:kk + 1]
        if bool((pick.values[:, kk - 1] - pick.values[:, kk] < 1e-6 * size.gather(1, edge).amax(1)).any()):
            return None
    keep = torch.zeros_like(scores, dtype=torch.bool)
    keep[:, :lo], keep[:, hi:] = True, True
    keep[:, lo:hi].scatter_(1, pick.indices[:, :kk], True)
    return keep.nonzero()[:, 1].view(scores.shape[0], -1)


def _exact_attention(q, K, V, lists, sm):
    """One batch element: [Hq, D] queries, [Hkv, N, D] rows, [Hq, count] lists."""
    hq, g = q.shape[0], q.shape[0] // K.shape[0]
    out, lse = [], []
    for h in range(hq):
        k, v = K[h // g][lists[h]].double(), V[h // g][lists[h]].double()
        x = torch.mv(k, q[h].double()) * sm
        lse.append(torch.logsumexp(x, 0))
        out.append(torch.mv(v.t().contiguous(), torch.softmax(x, 0)))
    return torch.stack(out), torch.stack(lse)


def _exact_decode(c, s):
    scores, outs, lses = [], [], []
    for b in range(c["B"]):
        sc, size = _exact_scores(s["q_imp"][b], s["Kimp"][b], c["N"])
        lists = _exact_lists(sc, size, c) if outs is not None else None
        full = torch.zeros(s["scores"].shape[1:], dtype=torch.float64, device=DEV)  # (the padding of a row stays 0)
        full[:, :c["N"]] = sc
        scores.append(full)
        if lists is None:
            outs = None
            continue
        o, l = _exact_attention(s["q"][b], s["K"][b], s["V"][b], lists.expand(c["Hq"], -1), s["sm"])
        outs.append(o)
        lses.append(l)
    return torch.stack(scores), None, None, None if outs is None else torch.stack(outs), None if outs is None else torch.stack(lses)


def exact(case, seed):
    c, s = case, prepare(case, seed)
    if c["kind"] in ("step", "headless"):
        return _exact_decode(c, s)
    if c["kind"] == "project":
        return torch.stack([torch.matmul(s["K"][b].double(), s["W"].double()) for b in range(c["B"])])
    if c["kind"] == "predict":
        d = {name: s[name].double() for name in ("h", "gamma", "beta", "W1", "b1", "W2", "b2")}
        x = torch.nn.functional.layer_norm(d["h"], (c["E"],), d["gamma"], d["beta"], 1e-5)
        z = torch.nn.functional.gelu(x @ d["W1"].t() + d["b1"])
        y = z @ d["W2"].t() + d["b2"]
        return y.view(c["B"], c["G"], c["Hq"], c["Dimp"]).transpose(0, 1).contiguous(), z
    # The loops' lists hang on scores of keys that were rounded to their storage type on the way, so
    # one value either side of a rounding boundary changes what follows; their projected rows do not.
    dec = s["dec"]
    first, last = (c["N"] - c["P"], c["N"]) if c["kind"] == "interval" else (c["N"], c["N"] + c["ring"])
    rows = torch.matmul(dec.K[:, :, first:last].double(), dec.W.double())
    outs = [None] * (c["P"] if c["kind"] == "interval" else c["P"] + 1)
    return (outs, None, None, None, None, None, None, rows) if c["kind"] == "interval" else (outs, None, None, None, None, None, None, None, rows)
