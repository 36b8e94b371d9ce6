"""The paper's physical buffer layout (Sec. 3.3): migration of the selected rows into
per-query-head buffers and attention over the buffers plus the local window, against the
oracle and against the fused-gather attention (which must agree bit for bit)."""
import math

import numpy as np
import pytest
import torch

from gpu_util import DEV, assert_attention, attn_plan, dtype_name, gpu_attn, np_of
from paper_2503_07518_amd import binding as tb, interval, workloads

pytestmark = pytest.mark.gpu


def say(msg):
    print(f"[case] {msg}", flush=True)


def make_lists(B, Hq, N, cap, seed, full=False):
    g = torch.Generator().manual_seed(seed)
    idx = torch.stack([torch.stack([torch.randperm(N, generator=g)[:cap].sort().values for _ in range(Hq)])
                       for _ in range(B)]).to(torch.int32)
    cnt = torch.full((B, Hq), cap, dtype=torch.int32) if full else torch.randint(0, cap + 1, (B, Hq), generator=g).to(torch.int32)
    cnt[0, 0] = cap
    if Hq > 1:
        cnt[0, 1] = 0
    return idx.to(DEV), cnt.to(DEV)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,N,cap", [
    (torch.bfloat16, 2, 8, 2, 128, 3000, 517),
    (torch.float32, 1, 4, 4, 64, 700, 130),
    (torch.bfloat16, 1, 4, 1, 64, 90, 64),
    (torch.float32, 1, 2, 2, 128, 33, 1),
])
def test_gather_kv_and_buffered_attention(oracle, dtype, B, Hq, Hkv, D, N, cap):
    say(f"gather + buffered attention dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} N={N} cap={cap}")
    g = torch.Generator().manual_seed(11)
    K = torch.randn((B, Hkv, N, D), generator=g).to(dtype).to(DEV)
    V = torch.randn((B, Hkv, N, D), generator=g).to(dtype).to(DEV)
    q = torch.randn((B, Hq, D), generator=g).to(dtype).to(DEV)
    idx, cnt = make_lists(B, Hq, N - 8, cap, 12)
    buf_cap = cap + 3
    Kbuf = torch.full((B, Hq, buf_cap, D), 7.0, dtype=dtype, device=DEV)
    Vbuf = torch.full((B, Hq, buf_cap, D), 7.0, dtype=dtype, device=DEV)
    d = tb.make_desc(N, Hq, K=K, V=V)
    tb.tb_gather_kv(d, K, V, idx, cnt, cap, Kbuf, Vbuf)
    torch.cuda.synchronize()
    rK, rV = oracle.gather_kv(np_of(K), np_of(V), np_of(idx), np_of(cnt), buf_cap)
    mask = (np.arange(buf_cap)[None, None, :] < np_of(cnt)[..., None])[..., None]
    seven = np_of(torch.full((1,), 7.0, dtype=dtype))[0]
    assert np.array_equal(np.where(mask, np_of(Kbuf), 0), rK) and np.array_equal(np.where(mask, np_of(Vbuf), 0), rV)
    assert np.all(np.where(mask, seven, np_of(Kbuf)) == seven), "rows beyond the count stay untouched"

    sm = 1.0 / math.sqrt(D)
    tail = (N - 8, N - 1)
    ws = tb.new_workspace(tb.TB_OP_ATTN, d, cap + 7)
    out = torch.full((B, Hq, D), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((B, Hq), float("nan"), dtype=torch.float32, device=DEV)
    tb.tb_buffered_decode_attn(d, q, Kbuf, Vbuf, cnt, cap, K, V, sm, out, lse, ws, tail[0], tail[1])
    fused_out, fused_lse = gpu_attn(q, K, V, idx, cnt, N, sm, max_count=cap, tail=tail)
    torch.cuda.synchronize()
    assert torch.equal(out, fused_out) and torch.equal(lse, fused_lse), "same rows in the same order: same bits"
    # oracle: the list followed by the tail rows
    cn = np_of(cnt)
    full = np.zeros((B, Hq, cap + 7), dtype=np.int32)
    for b in range(B):
        for h in range(Hq):
            c = cn[b, h]
            full[b, h, :c] = np_of(idx)[b, h, :c]
            full[b, h, c:c + 7] = np.arange(tail[0], tail[1])
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), full, cn + 7, dtype_name(K), sm)
    assert_attention(np_of(out), ro, dtype_name(K), np_of(lse), rl)


def test_buffered_interval_matches_fused_interval(oracle):
    say("interval loop with migrated buffers against the fused-gather loop, scaled-down C4")
    cfg = workloads.C4.scaled(name="C4_small_buf", B=2, N=4096, k=256, steps=12, P=4, heavy_per_kv_head=8)
    data = workloads.make_layer(cfg, device=DEV)
    K, V, W = data["K"], data["V"], data["W"]
    Kimp = torch.zeros((cfg.B, cfg.Hkv, K.shape[2], cfg.Dimp), dtype=K.dtype, device=DEV)
    tb.tb_project_keys(tb.make_desc(cfg.N, cfg.Hq, K=K, V=V, Kimp=Kimp), K, W, Kimp, 0, cfg.N)
    fused = interval.IntervalDecoder(K, V, W, Kimp, cfg.Hq, cfg.k, cfg.P, cfg.radius, sm_scale=cfg.sm_scale)
    buffered = interval.IntervalDecoder(K, V, W, Kimp.clone(), cfg.Hq, cfg.k, cfg.P, cfg.radius, sm_scale=cfg.sm_scale,
                                        buffered=True)
    for t in range(cfg.steps):
        q, qi = data["q"][t].contiguous(), data["q_imp"][t].contiguous()
        o1, l1 = fused.step(t, cfg.N + t, q, qi)
        o1, l1 = o1.clone(), l1.clone()
        o2, l2 = buffered.step(t, cfg.N + t, q, qi)
        torch.cuda.synchronize()
        assert torch.equal(o1, o2) and torch.equal(l1, l2), f"step {t}"


def test_gather_important_skips_sink_and_window_entries(oracle):
    say("migration of the middle of a list (sink and window entries left out)")
    B, Hq, Hkv, D, N, cap = 2, 4, 2, 128, 900, 200
    g = torch.Generator().manual_seed(5)
    K = torch.randn((B, Hkv, N, D), generator=g).to(torch.bfloat16).to(DEV)
    V = torch.randn((B, Hkv, N, D), generator=g).to(torch.bfloat16).to(DEV)
    idx, cnt = make_lists(B, Hq, N, cap, 6)
    cnt[1, 0] = 7  # shorter than what is skipped: nothing is migrated
    d = tb.make_desc(N, Hq, K=K, V=V)
    for front, back in ((0, 0), (5, 9), (16, 0), (0, 33)):
        Kbuf = torch.full((B, Hq, cap, D), 7.0, dtype=torch.bfloat16, device=DEV)
        Vbuf = torch.full_like(Kbuf, 7.0)
        n_out = torch.full((B, Hq), -3, dtype=torch.int32, device=DEV)
        tb.tb_gather_important(d, K, V, idx, cnt, cap, front, back, Kbuf, Vbuf, n_out)
        torch.cuda.synchronize()
        want_cnt = np.maximum(np_of(cnt) - front - back, 0)
        assert np.array_equal(np_of(n_out), want_cnt)
        shifted = np.zeros_like(np_of(idx))
        shifted[..., : cap - front] = np_of(idx)[..., front:]
        rK, rV = oracle.gather_kv(np_of(K), np_of(V), shifted, want_cnt, cap)
        mask = (np.arange(cap)[None, None, :] < want_cnt[..., None])[..., None]
        seven = np_of(torch.full((1,), 7.0, dtype=torch.bfloat16))[0]
        assert np.array_equal(np.where(mask, np_of(Kbuf), 0), rK) and np.array_equal(np.where(mask, np_of(Vbuf), 0), rV)
        assert np.all(np.where(mask, seven, np_of(Kbuf)) == seven), "rows beyond the count stay untouched"


@pytest.mark.parametrize("mode", [0, 1])
def test_ring_layout_interval_loop(oracle, mode):
    """Sink Buffer + Local Window ring + Important Buffer with the projection deferred to the
    wraps of the ring (Sec. 3.3 "Inference Setup"), over more than two wraps, every step against
    the oracle's driver in ring mode: selection, widened list and migrated row counts bit-exact,
    attention to the bar.  The projected-key cache starts with the post-prefill rows only."""
    check_ring_layout(oracle, mode, sink=16)


def test_ring_layout_without_sink(oracle):
    """No sink rows, the decoder's default: the first step attends to nothing but the Important Buffer."""
    check_ring_layout(oracle, mode=0, sink=0)


def check_ring_layout(oracle, mode, sink):
    ring = 8
    cfg = workloads.C4.scaled(name="C4_small_ring", B=2, N=4096, k=256, steps=21, P=4, heavy_per_kv_head=8)
    say(f"ring layout: ring={ring} sink={sink} P={cfg.P} steps={cfg.steps} neighbour rule {mode}")
    data = workloads.make_layer(cfg, device=DEV)
    K, V, W = data["K"], data["V"], data["W"]
    B, Hq, Hkv, N0, D = cfg.B, cfg.Hq, cfg.Hkv, cfg.N, cfg.D
    Kimp = torch.zeros((B, Hkv, K.shape[2], cfg.Dimp), dtype=K.dtype, device=DEV)
    tb.tb_project_keys(tb.make_desc(N0, Hq, K=K, V=V, Kimp=Kimp), K, W, Kimp, 0, N0)  # post-prefill state
    dec = interval.RingLayoutDecoder(K, V, W, Kimp, Hq, cfg.k, cfg.P, cfg.radius, ring, sink=sink,
                                     sm_scale=cfg.sm_scale, mode=mode)
    recs = []
    for t in range(cfg.steps):
        out, lse = dec.step(t, N0 + t, data["q"][t].contiguous(), data["q_imp"][t].contiguous())
        pred = t % cfg.P == 0
        recs.append((out.clone(), lse.clone(), dec.imp_cnt.clone(),
                     dec.idx.clone() if pred else None, dec.cnt.clone() if pred else None,
                     dec.exp_idx.clone() if pred else None, dec.exp_cnt.clone() if pred else None,
                     dec.scores[:, :, : N0 + t].clone() if pred else None))
    torch.cuda.synchronize()
    assert dec.projections == (cfg.steps - 1) // ring and dec.projections >= 2
    # the deferred batches left the same projected keys as one projection of the whole cache
    # (rows past the last wrap are still unprojected)
    upto = N0 + dec.projections * ring
    ref_kimp = oracle.project_keys(np_of(K)[:, :, :upto], np_of(W), cfg.dtype)
    assert np.mean(np_of(Kimp)[:, :, :upto] == ref_kimp) > 0.99 and not np_of(Kimp)[:, :, upto:].any()
    Kn, Vn, Kin = np_of(K), np_of(V), np_of(Kimp)
    drv = oracle.IntervalDriver(cfg.dtype, cfg.k, cfg.P, cfg.radius, sink=sink, sm_scale=cfg.sm_scale, mode=mode,
                                ring=ring)
    for t in range(cfg.steps):
        N_t, W_t = N0 + t, min(ring, t)
        u_idx, u_cnt = drv.lists(t, N_t, np_of(data["q_imp"][t]), Kin)
        if t % cfg.P == 0:
            g_idx, g_cnt = np_of(recs[t][3]), np_of(recs[t][4])
            s_idx, s_cnt = oracle.select_topk(np_of(recs[t][7]), cfg.k, sink, W_t)
            assert np.array_equal(s_cnt, g_cnt) and np.array_equal(s_idx, g_idx[..., : s_idx.shape[-1]])
            e_idx, e_cnt = oracle.expand_neighbors(g_idx, g_cnt, N_t, cfg.radius, cap_out=recs[t][5].shape[-1], mode=mode)
            assert np.array_equal(np_of(recs[t][6]), e_cnt)
            mask = np.arange(e_idx.shape[-1])[None, None] < e_cnt[..., None]
            assert np.array_equal(np.where(mask, np_of(recs[t][5]), -1), np.where(mask, e_idx, -1))
            drv.exp_idx, drv.exp_cnt = e_idx, e_cnt  # continue the oracle from the GPU's selection
            u_idx, u_cnt = e_idx, e_cnt
            W_p = W_t
        else:
            assert np.array_equal(u_cnt, drv.exp_cnt - W_p + W_t)
        assert np.array_equal(np_of(recs[t][2]), drv.exp_cnt - sink - W_p), f"step {t}: rows in the Important Buffer"
        ro, rl = oracle.sparse_decode_attn(np_of(data["q"][t]), Kn[:, :, :N_t], Vn[:, :, :N_t], u_idx, u_cnt, cfg.dtype,
                                           cfg.sm_scale)
        assert_attention(np_of(recs[t][0]), ro, cfg.dtype, np_of(recs[t][1]), rl, what=f"step {t}")


@pytest.mark.parametrize("dtype,D,rows", [(torch.bfloat16, 64, 1), (torch.bfloat16, 128, 1), (torch.float32, 128, 1), (torch.float32, 64, 37)])
def test_append_kv(dtype, D, rows):
    """Rows of strided caches into a buffer: the named rows change, byte for byte, and nothing else."""
    say(f"append rows dtype={dtype} D={D} rows={rows}")
    B, Hkv, N, R = 3, 2, 90, 50
    g = torch.Generator().manual_seed(71)
    K, V = (torch.randn((B, N, Hkv, D), generator=g).to(dtype).to(DEV).transpose(1, 2) for _ in range(2))  # strides of their own
    dK, dV = (torch.randn((B, Hkv, R, D), generator=g).to(dtype).to(DEV) for _ in range(2))
    rK, rV = dK.clone(), dV.clone()
    rK[:, :, 5:5 + rows] = K[:, :, 40:40 + rows]
    rV[:, :, 5:5 + rows] = V[:, :, 40:40 + rows]
    src, dst = tb.make_desc(N, Hkv, K=K, V=V), tb.make_desc(R, Hkv, K=dK, V=dV)
    tb.tb_append_kv(src, K, V, 40, dst, dK, dV, 5, rows)
    torch.cuda.synchronize()
    assert torch.equal(dK, rK) and torch.equal(dV, rV)
    for bad in ((N - rows + 1, 0), (0, R - rows + 1), (-1, 0)):
        with pytest.raises(tb.TbError):
            tb.tb_append_kv(src, K, V, bad[0], dst, dK, dV, bad[1], rows)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,cap,counts,tail,slot", [
    (torch.bfloat16, 2, 8, 2, 128, 300, (300, 0, 17), (0, 96), 95),    # splits of a head, the row in the last tile
    (torch.bfloat16, 1, 8, 1, 128, 3000, (3000, 129), (0, 64), 0),
    (torch.bfloat16, 1, 8, 1, 128, 5000, (5000, 129), (0, 64), 0),     # from here on the list in shares, one per XCD
    (torch.float32, 1, 16, 2, 64, 5000, (4093, 5000, 2), (3, 128), 127),
    (torch.float32, 3, 4, 4, 64, 40, (40, 1, 0), (5, 60), 33),
    (torch.float32, 1, 16, 2, 128, 1, (1, 0), (10, 20), 3),            # the row outside the attended range
    (torch.bfloat16, 9, 16, 8, 64, 700, (700, 64, 1), (0, 128), 77),
])
def test_append_with_buffered_attention(dtype, B, Hq, Hkv, D, cap, counts, tail, slot):
    """The row that arrives with the attention: the same bytes in the buffer and the same bits as the two calls, where the
    place it goes to holds what must not be seen."""
    say(f"append with attention dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} cap={cap} tail={tail} slot={slot}")
    g = torch.Generator().manual_seed(81)
    N, R = 50, 128
    K, V = (torch.randn((B, N, Hkv, D), generator=g).to(dtype).to(DEV).transpose(1, 2) for _ in range(2))  # strides of their own
    aK, aV = (torch.randn((B, Hkv, R, D), generator=g).to(dtype).to(DEV) for _ in range(2))
    aK[:, :, slot], aV[:, :, slot] = float("nan"), float("inf")
    Kb, Vb = (torch.randn((B, Hq, cap, D), generator=g).to(dtype).to(DEV) for _ in range(2))
    q = torch.randn((B, Hq, D), generator=g).to(dtype).to(DEV)
    cnt = torch.tensor([counts[i % len(counts)] for i in range(B * Hq)], dtype=torch.int32, device=DEV).view(B, Hq)
    assert cap < 5000 or attn_plan(dtype, B, Hq, Hkv, D, cap + tail[1] - tail[0])[1], "the plan has changed: these shapes were chosen for theirs"
    src, dst = tb.make_desc(N, Hq, K=K, V=V), tb.make_desc(R, Hq, K=aK, V=aV)
    ws = tb.new_workspace(tb.TB_OP_ATTN, dst, cap + R)
    res = []
    for fused in (True, False):
        k, v = aK.clone(), aV.clone()
        out, lse = (torch.full(s, float("nan"), device=DEV) for s in ((B, Hq, D), (B, Hq)))
        if fused:
            tb.tb_append_buffered_decode_attn(src, K, V, 41, dst, q, Kb, Vb, cnt, cap, k, v, slot, 0.1, out, lse, ws, *tail)
        else:
            tb.tb_append_kv(src, K, V, 41, dst, k, v, slot)
            tb.tb_buffered_decode_attn(dst, q, Kb, Vb, cnt, cap, k, v, 0.1, out, lse, ws, *tail)
        torch.cuda.synchronize()
        res.append((k, v, out, lse))
    assert all(torch.equal(a, b) for a, b in zip(*res)) and bool(torch.isfinite(res[0][2]).all())
    assert torch.equal(res[0][0][:, :, slot], K[:, :, 41]) and torch.equal(res[0][1][:, :, slot], V[:, :, 41])
    for bad in ((N, slot), (41, R), (-1, slot)):
        with pytest.raises(tb.TbError):
            tb.tb_append_buffered_decode_attn(src, K, V, bad[0], dst, q, Kb, Vb, cnt, cap, aK, aV, bad[1], 0.1, out, lse, ws, *tail)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,cap,counts,front,back,tail,slot", [
    (torch.bfloat16, 2, 8, 2, 128, 300, (300, 0, 17, 40), 16, 9, (0, 96), 95),      # lists shorter than what is left out, a row that arrives
    (torch.bfloat16, 1, 8, 1, 128, 3000, (3000, 129), 4, 64, (0, 64), -1),          # most rows listed by several heads
    (torch.float32, 3, 4, 4, 64, 40, (40, 1, 0), 0, 0, (5, 60), 33),
    (torch.float32, 1, 16, 2, 128, 1, (1, 0), 0, 1, (10, 20), -1),                  # nothing migrates
    (torch.bfloat16, 9, 16, 8, 64, 700, (700, 64, 1), 128, 256, (0, 128), 77),
    (torch.float32, 5, 8, 1, 128, 1100, (1100, 777), 3, 5, (7, 7), -1),             # no dense range
])
def test_migration_with_buffered_attention(dtype, B, Hq, Hkv, D, cap, counts, front, back, tail, slot):
    """Rows that migrate with the attention: buffers (past the migrated rows untouched), counts, ring and results the same bits as
    the separate calls, for lists with entries outside the cache, too."""
    check_migration(dtype, B, Hq, Hkv, D, 2 * cap + 50, cap, counts, front, back, tail, slot)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,Hq,Hkv,sparse,slot", [(64, 8, 2, True, 77), (128, 8, 1, True, 0), (64, 16, 2, False, 127), (128, 4, 2, False, 5)])
def test_migration_in_shares(dtype, D, Hq, Hkv, sparse, slot):
    """Few KV groups: the lists go in shares, one per XCD.  Rows that few heads list (read non-temporally) and many, with a row that
    arrives; infinite and NaN rows among those that are listed, and in row 0, which slots past the end load and no list holds."""
    cap, front, back, tail = 5001, 16, 40, (3, 128)
    _, in_shares = attn_plan(dtype, 1, Hq, Hkv, D, cap + tail[1] - tail[0])
    assert in_shares, "the plan has changed: these shapes were chosen for theirs"
    N, g = (40 if sparse else 2) * cap, Hq // Hkv
    p = (cap - front - back) / N
    assert (g * p / (1 - (1 - p) ** g) <= 1.3) == sparse  # (readers a row up to which rows are not kept in the caches)
    check_migration(dtype, 1, Hq, Hkv, D, N, cap, (cap, 3333, 2 * cap // 3 + 2, 30), front, back, tail, slot, infinite=True)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,cap,sparse", [(torch.bfloat16, 2, 8, 8, 128, 700, True), (torch.float32, 2, 16, 8, 64, 333, False)])
def test_migration_of_infinite_rows(dtype, B, Hq, Hkv, D, cap, sparse):
    """The same without shares."""
    assert not attn_plan(dtype, B, Hq, Hkv, D, cap + 90)[1]
    check_migration(dtype, B, Hq, Hkv, D, (20 if sparse else 2) * cap, cap, (cap, 3, cap // 2 + 1), 2, 1, (10, 100), 64, infinite=True)


def same(a, b):
    """Equal bits, one NaN being like another."""
    nan = torch.isnan(a) if a.is_floating_point() else torch.zeros_like(a, dtype=torch.bool)
    return torch.equal(nan, torch.isnan(b) if b.is_floating_point() else nan) and torch.equal(a.masked_fill(nan, 0), b.masked_fill(nan, 0))


def check_migration(dtype, B, Hq, Hkv, D, N, cap, counts, front, back, tail, slot, infinite=False):
    say(f"migration with attention dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} N={N} cap={cap} front={front} back={back} tail={tail} slot={slot}")
    g = torch.Generator().manual_seed(82)
    R = 128
    K, V = (torch.randn((B, N, Hkv, D), generator=g).to(dtype).to(DEV).transpose(1, 2) for _ in range(2))  # strides of their own
    aK, aV = (torch.randn((B, Hkv, R, D), generator=g).to(dtype).to(DEV) for _ in range(2))
    q = torch.randn((B, Hq, D), generator=g).to(dtype).to(DEV)
    idx = torch.rand((B, Hq, N), generator=g)
    idx[:, :, 0] = 0.0 if infinite else idx[:, :, 0]
    idx = idx.topk(cap, dim=-1).indices.sort(-1).values.to(torch.int32)
    idx[0, 0, :2], idx[-1, -1, -2:] = -5, N + 7
    if infinite:
        idx.clamp_(min=1)
        V[:, :, 0, 1], V[:, :, 0, 2], V[:, :, 0, 3], K[:, :, 0, 5] = float("inf"), -float("inf"), float("nan"), float("inf")
        V[0, 0, int(idx[0, 0, cap // 2]), 7], V[0, -1, int(idx[0, -1, front]), 9] = float("inf"), float("nan")
        V[:, :, N - 1, 11] = -float("inf")
    idx, cnt = idx[:, :, :cap].contiguous().to(DEV), torch.tensor([counts[i % len(counts)] for i in range(B * Hq)], dtype=torch.int32, device=DEV).view(B, Hq)
    src, dst = tb.make_desc(N, Hq, K=K, V=V), tb.make_desc(R, Hq, K=aK, V=aV)
    ws = tb.new_workspace(tb.TB_OP_ATTN, dst, cap + R)
    res = []
    for fused in (True, False):
        k, v = aK.clone(), aV.clone()
        Kb, Vb = (torch.full((B, Hq, cap, D), 3.5, dtype=dtype, device=DEV) for _ in range(2))
        out, lse = (torch.full(s, float("nan"), device=DEV) for s in ((B, Hq, D), (B, Hq)))
        n_out = torch.full((B, Hq), -7, dtype=torch.int32, device=DEV)
        if fused:
            tb.tb_migrate_buffered_decode_attn(src, K, V, idx, cnt, cap, front, back, n_out, 41 if slot >= 0 else -1, dst, q, Kb, Vb, k, v, slot, 0.1,
                                               out, lse, ws, *tail)
        else:
            tb.tb_gather_important(src, K, V, idx, cnt, cap, front, back, Kb, Vb, n_out)
            if slot >= 0:
                tb.tb_append_kv(src, K, V, 41, dst, k, v, slot)
            tb.tb_buffered_decode_attn(dst, q, Kb, Vb, n_out, cap, k, v, 0.1, out, lse, ws, *tail)
        torch.cuda.synchronize()
        res.append((k, v, Kb, Vb, n_out, out, lse))
    assert all(same(a, b) for a, b in zip(*res))
    finite = torch.isfinite(res[0][5])
    if infinite:  # only where a listed row makes it so, never from row 0
        assert bool(finite[:, :, (1, 2, 3, 5)].all()) and 0 < int((~finite).sum()) <= 3 * B * Hq and bool(torch.isfinite(res[0][6]).all())
    else:
        assert bool(finite.all())
    assert torch.equal(res[0][4], (cnt - front - back).clamp(min=0))
    for bad in (dict(cap=cap + 1), dict(front=-1), dict(src_row=N), dict(dst_row=R)):
        with pytest.raises(tb.TbError):
            tb.tb_migrate_buffered_decode_attn(src, K, V, idx, cnt, bad.get("cap", cap), bad.get("front", front), back, n_out, bad.get("src_row", 41), dst, q,
                                               Kb, Vb, k, v, bad.get("dst_row", 0), 0.1, out, lse, ws, *tail)
