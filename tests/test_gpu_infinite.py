"""Infinite and NaN elements of V: a column of the output is infinite (or NaN) where an attended row makes it so and nowhere
else, whatever the split of the list over workgroups and waves, and whatever lies in the slots past the list's end."""
import math

import numpy as np
import pytest
import torch

from gpu_util import DEV, assert_attention, attn_plan, gpu_attn, gpu_decode_step, group_plan, np_of
from paper_2503_07518_amd import binding as tb

pytestmark = pytest.mark.gpu

INF = float("inf")


def say(msg):
    print(f"[case] {msg}", flush=True)


def check(out, lse, ref, ref_lse, dn):
    got = np_of(out)
    assert np.array_equal(np.isnan(got), np.isnan(ref)), "NaN elsewhere than in the oracle"
    assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)])
    fin = np.isfinite(ref)
    assert 0 < fin.sum() < fin.size
    assert_attention(np.where(fin, got, 0.0), np.where(fin, ref, 0.0), dn, np_of(lse), ref_lse)


def shared_attn(q, K, V, idx, cnt, N, sm, max_count):
    B, Hq, D = q.shape
    d = tb.make_desc(N, Hq, K=K, V=V)
    ws = tb.new_workspace(tb.TB_OP_ATTN, d, max_count)
    out = torch.full((B, Hq, D), float("nan"), dtype=torch.float32, device=DEV)
    lse = torch.full((B, Hq), float("nan"), dtype=torch.float32, device=DEV)
    tb.tb_sparse_decode_attn_shared(d, q, K, V, idx, cnt, max_count, sm, out, lse, ws)
    return out, lse


def tensors(dtype, B, Hq, Hkv, N, D, seed):
    gen = torch.Generator().manual_seed(seed)
    K, V = (torch.randn((B, Hkv, N, D), generator=gen).to(dtype) for _ in range(2))
    return torch.randn((B, Hq, D), generator=gen).to(dtype), K, V, gen


@pytest.mark.parametrize("dtype,D,B,Hkv,g,unit,splits,shared", [
    # a list per head: `unit` rows are two tiles for each of a workgroup's four waves; either side of the numbers of splits that
    # fill the thread groups which add them up (8, 16, 32 with D = 128, 16, 32, 64 with D = 64), where the plan has such numbers
    *[(torch.bfloat16, 128, 1, 8, 1, 128, n, False) for n in (2, 8, 9, 15, 16, 17, 31)],
    *[(torch.bfloat16, 128, 1, 4, 1, 128, n, False) for n in (32, 33, 47)],
    *[(torch.float32, 128, 1, 4, 1, 64, n, False) for n in (7, 10, 21, 33)],
    *[(torch.bfloat16, 64, 1, 2, 4, 256, n, False) for n in (5, 16, 24)],
    *[(torch.float32, 64, 1, 2, 2, 128, n, False) for n in (13, 32, 40)],
    # one list for all heads, a workgroup per KV group: matrix cores (steps of 256 rows), vector form
    *[(torch.bfloat16, 128, 4, 8, 4, 256, n, True) for n in (4, 5, 7)],
    *[(torch.bfloat16, 64, 2, 8, 8, 256, n, True) for n in (13, 15)],
    *[(torch.float32, 128, 4, 8, 2, 64, n, True) for n in (4, 6, 13)],
    *[(torch.float32, 128, 4, 8, 8, 64, n, True) for n in (3, 12)],
    *[(torch.bfloat16, 64, 8, 8, 2, 256, n, True) for n in (3, 6)],
])
def test_infinite_values_of_every_split(oracle, dtype, D, B, Hkv, g, unit, splits, shared):
    """Every split attends a row with an infinite element in a column of its own; the list ends with a whole tile."""
    say(f"infinite values of every split dtype={dtype} D={D} B={B} Hkv={Hkv} g={g} splits={splits} shared={shared}")
    Hq = g * Hkv
    plan = (lambda rows: group_plan(dtype, B, Hq, Hkv, D, rows)) if shared else (lambda rows: attn_plan(dtype, B, Hq, Hkv, D, rows)[0])
    rows = next((r for r in range(unit // 2, 100 * unit, unit // 2) if (p := plan(r)) and p.nsplit == splits), None)
    assert rows, "the plan has no such number of splits"
    N, dn = rows + 40, "f32" if dtype == torch.float32 else "bf16"
    q, K, V, gen = tensors(dtype, B, Hq, Hkv, N, D, splits + D)
    idx = torch.stack([torch.randperm(N, generator=gen)[:rows].sort().values for _ in range(B)]).to(torch.int32)
    cnt = torch.full((B,), rows, dtype=torch.int32)
    for b in range(B):
        for j in range(2 * rows // unit):  # (half a unit is the least that one split takes in a row)
            V[b, :, int(idx[b, j * unit // 2 + j % 8]), j % (D - 4)] = INF if j % 3 else -INF
        V[b, :, int(idx[b, rows - 1]), D - 1] = INF
        V[b, :, int(idx[b, rows // 2]), D - 2] = float("nan")
    sm = 1.0 / math.sqrt(D)
    if shared:
        out, lse = shared_attn(q.to(DEV), K.to(DEV), V.to(DEV), idx.to(DEV), cnt.to(DEV), N, sm, rows)
        ref, ref_lse = oracle.sparse_decode_attn_shared(np_of(q), np_of(K), np_of(V), idx.numpy(), cnt.numpy(), dn, sm)
    else:
        lists, counts = idx[:, None].expand(B, Hq, rows).contiguous(), cnt[:, None].expand(B, Hq).contiguous()
        out, lse = gpu_attn(q.to(DEV), K.to(DEV), V.to(DEV), lists.to(DEV), counts.to(DEV), N, sm)
        ref, ref_lse = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), lists.numpy(), counts.numpy(), dn, sm)
    check(out, lse, ref, ref_lse, dn)


def past_the_end(V, lists, counts, Hq):
    """Infinite elements where a slot past a list's end may look: the lowest listed row of every list, and row 0, which no
    list holds."""
    B, Hkv = V.shape[:2]
    for b in range(B):
        for h in range(lists.shape[1]):
            assert int(lists[b, h, 0]) > 0 and int(counts[b, h]) >= 1
            hkv = h // (Hq // Hkv)
            V[b, hkv if lists.shape[1] == Hq else slice(None), int(lists[b, h, 0]), 4 + h % 8] = INF if h % 2 else -INF
    V[:, :, 0, 1], V[:, :, 0, 2], V[:, :, 0, 3] = INF, -INF, float("nan")


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,g,Hkv,rows", [(128, 1, 3, 1), (64, 4, 2, 37), (128, 4, 8, 130), (128, 8, 1, 1277), (64, 2, 8, 2050)])
def test_infinite_values_past_the_end(oracle, dtype, D, g, Hkv, rows):
    """Lists that end inside a tile: per head, from per-head buffers with a dense tail, and one list for all heads."""
    say(f"infinite values past the end dtype={dtype} D={D} g={g} Hkv={Hkv} rows={rows}")
    B, Hq, N, tail = 4, g * Hkv, rows + 300, 5
    dn, sm = "f32" if dtype == torch.float32 else "bf16", 1.0 / math.sqrt(D)
    q, K, V, gen = tensors(dtype, B, Hq, Hkv, N, D, rows + D)

    def draw(heads):
        picks = [1 + torch.randperm(N - tail - 1, generator=gen)[:rows].sort().values for _ in range(B * heads)]
        return torch.stack(picks).to(torch.int32).view(B, heads, rows)

    idx, cnt, V1 = draw(Hq), torch.full((B, Hq), rows, dtype=torch.int32), V.clone()
    past_the_end(V1, idx, cnt, Hq)
    dev = dict(q=q.to(DEV), K=K.to(DEV), V=V1.to(DEV))
    out, lse = gpu_attn(dev["q"], dev["K"], dev["V"], idx.to(DEV), cnt.to(DEV), N, sm)
    ref, ref_lse = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V1), idx.numpy(), cnt.numpy(), dn, sm)
    check(out, lse, ref, ref_lse, dn)

    Kbuf, Vbuf = (torch.zeros((B, Hq, rows, D), dtype=dtype, device=DEV) for _ in range(2))
    d = tb.make_desc(N, Hq, K=dev["K"], V=dev["V"])
    tb.tb_gather_kv(d, dev["K"], dev["V"], idx.to(DEV), cnt.to(DEV), rows, Kbuf, Vbuf)
    out, lse = torch.full_like(out, float("nan")), torch.full_like(lse, float("nan"))
    ws = tb.new_workspace(tb.TB_OP_ATTN, d, rows + tail)
    tb.tb_buffered_decode_attn(d, dev["q"], Kbuf, Vbuf, cnt.to(DEV), rows, dev["K"], dev["V"], sm, out, lse, ws, N - tail, N)
    dense = torch.arange(N - tail, N, dtype=torch.int32).expand(B, Hq, tail)
    ref, ref_lse = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V1), torch.cat([idx, dense], dim=2).numpy(), (cnt + tail).numpy(), dn, sm)
    check(out, lse, ref, ref_lse, dn)

    idx, cnt, V1 = draw(1), torch.full((B, 1), rows, dtype=torch.int32), V.clone()
    past_the_end(V1, idx, cnt, Hq)
    out, lse = shared_attn(dev["q"], dev["K"], V1.to(DEV), idx[:, 0].contiguous().to(DEV), cnt[:, 0].contiguous().to(DEV), N, sm, rows)
    ref, ref_lse = oracle.sparse_decode_attn_shared(np_of(q), np_of(K), np_of(V1), idx[:, 0].numpy(), cnt[:, 0].numpy(), dn, sm)
    check(out, lse, ref, ref_lse, dn)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,Dimp,g,Hkv,N,k", [(64, 16, 1, 2, 200, 1), (64, 16, 1, 8, 1024, 127), (128, 32, 4, 2, 1500, 150), (128, 16, 2, 2, 4095, 333),
                                               (128, 32, 4, 2, 9001, 901), (128, 16, 2, 2, 70001, 1003)])
def test_infinite_values_in_a_step(oracle, dtype, D, Dimp, g, Hkv, N, k):
    """A whole step, in one launch and in several, with infinite elements in the lowest selected row of every head and in a row
    0 that no head selects."""
    say(f"infinite values in a step dtype={dtype} D={D} Dimp={Dimp} g={g} N={N} k={k}")
    B, Hq, dn, sm = 2, g * Hkv, "f32" if dtype == torch.float32 else "bf16", 1.0 / math.sqrt(D)
    q, K, V, gen = tensors(dtype, B, Hq, Hkv, N, D, N + k)
    q_imp = torch.randn((B, Hq, Dimp), generator=gen).abs().to(dtype)
    Kimp = torch.randn((B, Hkv, N, Dimp), generator=gen).to(dtype)
    Kimp[:, :, 0] = -50.0
    dev = [t.to(DEV) for t in (q, q_imp, K, V, Kimp)]
    _, idx, cnt, _, _ = gpu_decode_step(*dev, N, k, 0, 0, sm)
    V1 = V.clone()
    past_the_end(V1, idx.cpu(), cnt.cpu(), Hq)
    dev[3] = V1.to(DEV)
    _, idx1, cnt1, out, lse = gpu_decode_step(*dev, N, k, 0, 0, sm)
    assert torch.equal(idx1, idx) and torch.equal(cnt1, cnt)
    ref, ref_lse = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V1), np_of(idx), np_of(cnt), dn, sm)
    check(out, lse, ref, ref_lse, dn)
