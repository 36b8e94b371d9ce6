"""The entry points under HIP graph capture: a captured call, replayed several times with the
program's own eager work and synchronisations between the replays, must reproduce the eager
result bit for bit on every replay (the library clears its counters and scratch with kernels of
its own, never with memset nodes)."""
import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from gpu_util import DEV, np_of
from paper_2503_07518_amd import binding as tb
from paper_2503_07518_amd import interval, workloads


def _capture(fn):
    g = torch.cuda.CUDAGraph()
    side = torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        with torch.cuda.graph(g, stream=side):
            fn()
    torch.cuda.current_stream().wait_stream(side)
    return g


def _layer(cfg, layer):
    data = workloads.make_layer(cfg, layer=layer, device=DEV)
    K, V = data["K"], data["V"]
    Kimp = torch.zeros((cfg.B, cfg.Hkv, cfg.N, cfg.Dimp), dtype=K.dtype, device=DEV)
    d = tb.make_desc(cfg.N, cfg.Hq, K=K, V=V, Kimp=Kimp)
    tb.tb_project_keys(d, K, data["W"], Kimp, 0, cfg.N)
    need = tb.policy_count(cfg.N, cfg.k, 0, 0)
    stride = (cfg.N + 3) // 4 * 4
    bufs = dict(
        d=d, K=K, V=V, Kimp=Kimp, q=data["q"][0].contiguous(), q_imp=data["q_imp"][0].contiguous(), need=need,
        scores=torch.zeros((cfg.B, cfg.Hq, stride), dtype=torch.float32, device=DEV),
        idx=torch.zeros((cfg.B, cfg.Hq, need), dtype=torch.int32, device=DEV),
        cnt=torch.zeros((cfg.B, cfg.Hq), dtype=torch.int32, device=DEV),
        out=torch.zeros((cfg.B, cfg.Hq, cfg.D), dtype=torch.float32, device=DEV),
        lse=torch.zeros((cfg.B, cfg.Hq), dtype=torch.float32, device=DEV),
        ws=tb.new_workspace(tb.TB_OP_DECODE_STEP, d, need))
    return bufs


def _step(cfg, b):
    tb.tb_decode_step(b["d"], b["q_imp"], b["Kimp"], 1.0, b["q"], b["K"], b["V"], cfg.k, 0, 0, cfg.sm_scale,
                      b["scores"], b["idx"], b["cnt"], b["out"], b["lse"], b["ws"])


@pytest.mark.parametrize("name,kw", [
    ("split attention, one selection workgroup per row", dict(B=1, N=8192, k=800)),
    ("a short step in one launch", dict(B=1, N=1024, k=100, heavy_per_kv_head=10)),
    ("selection by pieces (workspace scratch in the graph)", dict(B=2, N=70001, k=4096, heavy_per_kv_head=64)),
])
def test_decode_step_graph_replays_match_eager(name, kw):
    print(f"[case] graph replay: {name}", flush=True)
    cfg = workloads.C2.scaled(name="C2_graph", **kw)
    a, other = _layer(cfg, 0), _layer(cfg, 1)
    _step(cfg, a)
    torch.cuda.synchronize()
    ref = {k: a[k].clone() for k in ("scores", "idx", "cnt", "out", "lse")}
    assert int(ref["cnt"].min()) == a["need"]
    g = _capture(lambda: _step(cfg, a))
    for r in range(4):
        for k in ("scores", "out", "lse"):
            a[k].fill_(float("nan"))
        a["idx"].fill_(-1)
        a["cnt"].fill_(-1)
        _step(cfg, other)            # eager work of the same library between the replays
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        for k, v in ref.items():
            got = a[k][..., :cfg.N] if k == "scores" else a[k]      # (the padding of a score row is not written)
            want = v[..., :cfg.N] if k == "scores" else v
            assert torch.equal(got, want), f"replay {r}: {k} differs from the eager call"


def test_static_scratch_attention_in_a_graph():
    """The entry point for callers that cannot allocate, used the way such a caller would: captured."""
    print("[case] graph replay: attention on the library's own scratch", flush=True)
    cfg = workloads.C2.scaled(name="C2_graph_static", B=1, N=8192, k=800)
    a = _layer(cfg, 0)
    _step(cfg, a)
    torch.cuda.synchronize()
    ref_out, ref_lse = a["out"].clone(), a["lse"].clone()

    def call():
        tb.tb_sparse_decode_attn_static(a["d"], a["q"], a["K"], a["V"], a["idx"], a["cnt"], a["need"], cfg.sm_scale,
                                        a["out"], a["lse"])
    g = _capture(call)
    for r in range(3):
        a["out"].fill_(float("nan"))
        a["lse"].fill_(float("nan"))
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert torch.equal(a["out"], ref_out) and torch.equal(a["lse"], ref_lse), f"replay {r} differs"
        call()                       # and an eager call on the same scratch in between
        torch.cuda.synchronize()
        assert torch.equal(a["out"], ref_out)


def test_three_buffer_steps_in_a_graph():
    """A prediction step, whose rows migrate on the way, and a reuse step of the three-buffer layout, each with a row that arrives."""
    print("[case] graph replay: three-buffer layout, a prediction and a reuse step", flush=True)
    cfg = workloads.C4.scaled(name="C4_graph_ring", B=2, N=4096, k=256, steps=6, P=4, heavy_per_kv_head=8)
    data = workloads.make_layer(cfg, device=DEV)
    K, V = data["K"], data["V"]
    Kimp = torch.zeros((cfg.B, cfg.Hkv, K.shape[2], cfg.Dimp), dtype=K.dtype, device=DEV)
    tb.tb_project_keys(tb.make_desc(cfg.N, cfg.Hq, K=K, V=V, Kimp=Kimp), K, data["W"], Kimp, 0, cfg.N)
    dec = interval.RingLayoutDecoder(K, V, data["W"], Kimp, cfg.Hq, cfg.k, cfg.P, cfg.radius, 8, sink=16, sm_scale=cfg.sm_scale)
    q, q_imp = [[t.contiguous() for t in data[n]] for n in ("q", "q_imp")]

    def steps(which):
        return [tuple(x.clone() for x in dec.step(t, cfg.N + t, q[t], q_imp[t])) for t in which]
    first = steps(range(4))
    ref = steps((4, 5))
    kept = {name: getattr(dec, name).clone() for name in ("aux_K", "aux_V", "imp_cnt", "exp_cnt")}
    mask = (torch.arange(dec.exp_cap, device=DEV) < kept["imp_cnt"][:, :, None])[..., None]
    rows = [torch.where(mask, b, 0) for b in (dec.Kbuf, dec.Vbuf)]
    got = [torch.empty_like(x) for pair in ref for x in pair]

    def call():
        for i, t in enumerate((4, 5)):
            out, lse = dec.step(t, cfg.N + t, q[t], q_imp[t])
            got[2 * i].copy_(out)
            got[2 * i + 1].copy_(lse)
    g = _capture(call)
    for r in range(3):
        assert all(torch.equal(a, b) for x, y in zip(steps(range(4)), first) for a, b in zip(x, y))  # eager steps between the replays
        for x in got + [dec.Kbuf, dec.Vbuf]:
            x.fill_(float("nan"))
        dec.aux_K[:, :, 16 + 3:], dec.aux_V[:, :, 16 + 3:] = float("nan"), float("nan")  # the slots that the two steps fill, and those behind
        torch.cuda.synchronize()
        g.replay()
        torch.cuda.synchronize()
        assert all(torch.equal(a, b) for a, b in zip(got, [x for pair in ref for x in pair])), f"replay {r} differs"
        for name in ("imp_cnt", "exp_cnt"):
            assert torch.equal(getattr(dec, name), kept[name]), name
        assert torch.equal(dec.aux_K[:, :, :16 + 5], kept["aux_K"][:, :, :16 + 5]) and torch.equal(dec.aux_V[:, :, :16 + 5], kept["aux_V"][:, :, :16 + 5])
        assert all(torch.equal(torch.where(mask, b, 0), want) for b, want in zip((dec.Kbuf, dec.Vbuf), rows))
