"""GPU parity: every exported operation, called through the C ABI, against the CPU oracle on
the same bytes.  Sizes span several tiles and ragged tails; edge cases are listed per op.

The bars (index lists bit-exact; scores, attention, log-sum-exp and projected keys within the
tolerances of the benchmark definition) are stated once, in gpu_util.py."""
import math

import numpy as np
import pytest
import torch

pytestmark = pytest.mark.gpu

from paper_2503_07518_amd import binding as tb
from gpu_util import (ATTN_TOL, DEV, assert_attention, assert_projection, assert_scores, attn_plan, dtype_name, gpu_attn,
                      gpu_decode_step, gpu_expand, gpu_project, gpu_score, gpu_select, np_of, projection_magnitude,
                      score_magnitude)


def say(msg):
    print(f"[case] {msg}", flush=True)


def randn(shape, dtype, seed, scale=1.0):
    g = torch.Generator(device="cpu").manual_seed(seed)
    return (torch.randn(shape, generator=g) * scale).to(dtype).to(DEV)


# --------------------------------------------------------------------------- projection

@pytest.mark.parametrize("dtype,D,Dimp,N,Hw", [
    (torch.float32, 64, 16, 1000, 1),
    (torch.bfloat16, 128, 32, 1037, 1),
    (torch.bfloat16, 128, 32, 300, 3),
    (torch.bfloat16, 64, 64, 129, 1),
    (torch.float32, 128, 64, 65, 3),
    (torch.bfloat16, 128, 16, 1, 1),
    # up to four rows: the one-wave-per-row form of the decode-step append
    (torch.float32, 64, 64, 3, 3),
    (torch.bfloat16, 128, 32, 2, 1),
    (torch.bfloat16, 64, 16, 4, 3),
    (torch.float32, 128, 32, 5, 1),
    # enough rows for the matrix-core form (bf16, Dimp 32), ragged last tile
    (torch.bfloat16, 128, 32, 4133, 1),
    (torch.bfloat16, 64, 32, 2501, 3),
    (torch.bfloat16, 128, 32, 2048, 3),
    (torch.bfloat16, 128, 16, 3000, 1),   # the paper's interaction dimension, on the same tile
    (torch.bfloat16, 64, 16, 2111, 3),
])
def test_project_keys(oracle, dtype, D, Dimp, N, Hw):
    say(f"project dtype={dtype} D={D} Dimp={Dimp} N={N} Hw={Hw}")
    B, Hkv = 2, 3
    K = randn((B, Hkv, N + 5, D), dtype, 1)
    W = randn((Hw, D, Dimp), dtype, 2, 1 / math.sqrt(D))
    Kimp = gpu_project(K, W, N)
    torch.cuda.synchronize()
    dn = dtype_name(K)
    ref = oracle.project_keys(np_of(K)[:, :, :N], np_of(W), dn)
    got = np_of(Kimp)
    assert not got[:, :, N:].any(), "rows beyond N must stay untouched"
    mag = projection_magnitude(oracle, np_of(K)[:, :, :N], np_of(W), dn, Hkv)
    assert_projection(oracle, got[:, :, :N], ref, mag, dn)
    if dn == "bf16":
        assert np.mean(got[:, :, :N] == ref) > 0.99  # and nearly always the same bits


@pytest.mark.parametrize("N,n_begin,n_end", [(500, 70, 391), (5000, 70, 4391)])
def test_project_identity_and_row_range(oracle, N, n_begin, n_end):
    say(f"project identity W, row range [{n_begin}, {n_end}) of {N}")
    B, Hkv, D, Dimp = 1, 2, 128, 32
    K = randn((B, Hkv, N, D), torch.bfloat16, 3)
    W = torch.zeros((1, D, Dimp), dtype=torch.bfloat16, device=DEV)
    W[0, 3:3 + Dimp, :] = torch.eye(Dimp, dtype=torch.bfloat16)
    Kimp = torch.full((B, Hkv, N, Dimp), 7.0, dtype=torch.bfloat16, device=DEV)
    gpu_project(K, W, N, n_begin=n_begin, n_end=n_end, Kimp=Kimp)
    torch.cuda.synchronize()
    assert torch.equal(Kimp[:, :, n_begin:n_end], K[:, :, n_begin:n_end, 3:3 + Dimp])
    assert torch.all(Kimp[:, :, :n_begin] == 7.0) and torch.all(Kimp[:, :, n_end:] == 7.0)


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("D,Dimp,B,Hkv,n_begin,n_end", [
    (128, 32, 2, 2, 3, 8), (64, 16, 1, 3, 0, 15), (128, 64, 1, 2, 7, 24),     # below, at and past one 16-row tile
    (128, 16, 2, 2, 1, 65), (64, 64, 1, 2, 0, 129),                           # past the four tiles of a workgroup
    (128, 32, 16, 8, 5, 600), (64, 32, 16, 8, 2, 531),                        # two tiles a wave, the last ones ragged
    (64, 16, 16, 8, 0, 8200),                                                 # four tiles a wave
])
def test_project_tile_edges(oracle, dtype, D, Dimp, B, Hkv, n_begin, n_end):
    """Row ranges around the tiles of project_kernel, into rows with a stride of their own; what lies
    outside the range keeps its bytes."""
    say(f"project tile edges dtype={dtype} D={D} Dimp={Dimp} B={B} Hkv={Hkv} rows [{n_begin}, {n_end})")
    N = n_end + 3
    K = randn((B, Hkv, N, D), dtype, 61)
    W = randn((Hkv if B == 2 else 1, D, Dimp), dtype, 62, 1.0 / math.sqrt(D))
    store = torch.full((B, Hkv, N, Dimp + 8), 7.0, dtype=dtype, device=DEV)
    gpu_project(K, W, N, n_begin=n_begin, n_end=n_end, Kimp=store[..., :Dimp])
    torch.cuda.synchronize()
    got, dn = np_of(store[..., :Dimp]), dtype_name(K)
    ref = oracle.project_keys(np_of(K), np_of(W), dn)
    mag = projection_magnitude(oracle, np_of(K), np_of(W), dn, Hkv)
    rows = slice(n_begin, n_end)
    assert_projection(oracle, got[:, :, rows], ref[:, :, rows], mag[:, :, rows], dn)
    assert bool((store[:, :, :n_begin] == 7).all()) and bool((store[:, :, n_end:] == 7).all()) and bool((store[..., Dimp:] == 7).all())


def test_project_strided_cache(oracle):
    say("project into a strided (over-allocated) cache")
    B, Hkv, N, D, Dimp = 2, 2, 200, 128, 32
    Kbig = randn((B, Hkv, 256, D + 8), torch.bfloat16, 4)
    K = Kbig[:, :, :, :D]  # row stride D+8
    W = randn((1, D, Dimp), torch.bfloat16, 5, 0.1)
    Kimp_big = torch.zeros((B, Hkv, 256, Dimp + 8), dtype=torch.bfloat16, device=DEV)
    Kimp = Kimp_big[:, :, :, :Dimp]
    gpu_project(K, W, N, Kimp=Kimp)
    torch.cuda.synchronize()
    ref = oracle.project_keys(np_of(K)[:, :, :N], np_of(W), "bf16")
    mag = projection_magnitude(oracle, np_of(K)[:, :, :N], np_of(W), "bf16", Hkv)
    assert_projection(oracle, np_of(Kimp)[:, :, :N], ref, mag, "bf16")
    assert not np_of(Kimp_big)[..., Dimp:].any()


# --------------------------------------------------------------------------- scoring

@pytest.mark.parametrize("dtype,B,Hq,Hkv,Dimp,N", [
    (torch.float32, 1, 8, 8, 16, 1024),
    (torch.bfloat16, 1, 32, 8, 32, 5000),
    (torch.bfloat16, 2, 16, 2, 32, 1025),
    (torch.bfloat16, 1, 4, 2, 16, 63),
    (torch.float32, 1, 2, 2, 64, 300),
    (torch.bfloat16, 1, 4, 4, 64, 1),
    (torch.float32, 2, 8, 2, 32, 4097),
    (torch.bfloat16, 1, 4, 4, 32, 257),    # the matrix-core form (bf16, 32 projected dims): one query head per KV head
    (torch.bfloat16, 3, 6, 3, 32, 70),     # ... two, a ragged single workgroup
    (torch.bfloat16, 1, 8, 1, 32, 9),      # ... eight, fewer rows than one matrix tile
])
def test_score(oracle, dtype, B, Hq, Hkv, Dimp, N):
    say(f"score dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} Dimp={Dimp} N={N}")
    q_imp = randn((B, Hq, Dimp), dtype, 6)
    Kimp = randn((B, Hkv, N + 3, Dimp), dtype, 7)
    scale = 0.7
    s = gpu_score(q_imp, Kimp, N, scale)
    torch.cuda.synchronize()
    dn = dtype_name(Kimp)
    ref = oracle.score(np_of(q_imp), np_of(Kimp)[:, :, :N], dn, scale)
    got = np_of(s)
    assert_scores(got[:, :, :N], ref, score_magnitude(oracle, np_of(q_imp), np_of(Kimp)[:, :, :N], dn, Hq // Hkv), scale)
    assert np.isnan(got[:, :, N:]).all(), "padding beyond N must stay untouched"


# --------------------------------------------------------------------------- selection

def check_select(oracle, scores_t, N, k, sink, window, ws=None):
    idx, cnt = gpu_select(scores_t, N, k, sink, window, ws=ws)
    torch.cuda.synchronize()
    s_np = np_of(scores_t)[:, :, :N]
    ridx, rcnt = oracle.select_topk(s_np, k, sink, window)
    gi, gc = np_of(idx), np_of(cnt)
    assert np.array_equal(gc, rcnt)
    width = ridx.shape[-1]
    mask = np.arange(width)[None, None, :] < rcnt[..., None]
    assert np.array_equal(np.where(mask, gi[..., :width], -1), np.where(mask, ridx, -1))
    assert np.all(gi[..., :width][~mask] == -7), "entries beyond count must stay untouched"
    return gi, gc


@pytest.mark.parametrize("N", [1, 2, 63, 64, 65, 1000, 1025, 4096, 4097, 8192, 20000, 40000, 65536, 70001])
def test_select_sizes_random_scores(oracle, N):
    say(f"select random N={N}")
    B, Hq = 2, 3
    scores = randn((B, Hq, (N + 3) // 4 * 4), torch.float32, 100 + N)
    for k in sorted({1, max(1, N // 10), N - 1, N, N + 5} - {0}):
        check_select(oracle, scores, N, k, 0, 0)
    if N > 20:
        check_select(oracle, scores, N, max(1, N // 7), 5, 9)
        check_select(oracle, scores, N, 0, 3, 4)


@pytest.mark.parametrize("N", [700, 2047, 2049, 4095, 4097, 8193, 12289, 16385, 20481, 24577, 32769, 40961, 49153, 65535])
def test_select_register_forms(oracle, N):
    """Either side of every size at which the one-workgroup selection takes another number of waves or of tiles per
    wave, with scores that lead it through each of its paths: thresholds above and below zero, a wave's span that keeps
    (almost) everything, ties, NaN and infinities, and a sample that misleads."""
    say(f"select register forms N={N}")
    s = randn((1, 9, (N + 3) // 4 * 4), torch.float32, 300 + N)
    inf, nan = float("inf"), float("nan")
    s[0, 1] -= 100.0                                                    # thresholds below zero
    s[0, 2] = torch.arange(s.shape[-1], dtype=torch.float32).to(DEV)     # the kept scores crowd into the last waves
    s[0, 3] = (s[0, 3] * 4).round() / 4                                   # ties (and both zeros) at the threshold
    s[0, 4, ::3], s[0, 4, 1::3], s[0, 4, 2::97] = nan, -inf, inf          # thresholds at +-inf, NaN among what ties with -inf
    s[0, 5] = torch.where(s[0, 5] > 1.0, torch.full_like(s[0, 5], -0.0), s[0, 5].abs() * 1e-42)  # denormals and -0
    s[0, 6, ::5] = -nan
    threads = 512 if N <= 4096 else 1024
    pos = (torch.arange(threads // 4) * N // (threads // 4) // 4 * 4).view(-1, 1) + torch.arange(4)
    pos = pos.view(-1)[pos.view(-1) < N].unique().to(DEV)
    s[0, 7, pos], s[0, 8, pos] = 1e30, -1e30                              # the sample sees nothing but these
    for k in sorted({1, N // 40, N // 10, N // 2 - 3, N - 1}):
        check_select(oracle, s, N, k, 0, 0)
    check_select(oracle, s, N, N // 7, 5, 9)
    check_select(oracle, s, N, N // 9, N // 3, 70)


@pytest.mark.parametrize("N,ks", [
    (65537, (1, 4096, 8192)),            # one score more than a workgroup holds in registers
    (70001, (4096, 8000, 35000)),        # a short last piece
    (131072, (4096, 13000, 65536)),      # streamed rows: the bracket's keys fit the LDS list
    (300001, (1, 4096, 30000, 150000)),  # ... and overflow it for the larger budgets
    (1 << 20, (4096, 104857)),           # longest supported row
])
def test_select_streamed_rows(oracle, N, ks):
    say(f"select streamed N={N}")
    from paper_2503_07518_amd import binding as tb
    scores = randn((1, 2, (N + 3) // 4 * 4), torch.float32, 200 + N % 1000)
    d = tb.tb_cache_desc()
    d.B, d.Hq, d.Hkv, d.D, d.Dimp, d.dtype, d.N = 1, 2, 2, 128, 32, tb.TB_F32, N
    d.k_stride_n = d.v_stride_n = 128
    d.ki_stride_n = 32
    assert tb.tb_workspace_bytes(tb.TB_OP_SELECT, d, ks[0]) > 0, "a long row on two heads is cut into pieces"
    # with the workspace that tb_workspace_bytes asks for, the row is selected piecewise by
    # several workgroups; with a smaller one, a single workgroup streams the whole row
    small = torch.zeros(256, dtype=torch.uint8, device=DEV)
    g = torch.Generator().manual_seed(N)
    tied = torch.randint(0, 50, scores.shape, generator=g).to(torch.float32).to(DEV)  # heavy ties at the threshold
    asc = torch.arange(scores.shape[-1], dtype=torch.float32).view(1, 1, -1).to(DEV)  # every kept key in one span
    for ws in (None, small):
        for k in ks:
            check_select(oracle, scores, N, k, 0, 0, ws=ws)
        check_select(oracle, scores, N, ks[0], 128, 256, ws=ws)
        check_select(oracle, tied, N, ks[0], 0, 0, ws=ws)
        check_select(oracle, tied, N, ks[-1], 3, 5, ws=ws)
        check_select(oracle, asc, N, ks[0], 0, 0, ws=ws)
        check_select(oracle, -asc, N, ks[0], 2, 0, ws=ws)
    # rows whose sample misleads the first stage: huge values exactly where it looks -> the pieces
    # keep fewer keys than the budget; hugely negative ones exactly there -> the pieces keep far
    # more than they have room for.  Both must end in the same lists (the second stage then
    # selects on the whole row).
    pos = sample_positions(N)
    huge = scores.clone()
    huge[:, :, pos.to(DEV)] = 1e30
    check_select(oracle, huge, N, min(N // 8, 3 * len(pos)), 0, 0)
    low = scores.clone()
    low[:, :, pos.to(DEV)] = -1e30
    check_select(oracle, low, N, ks[0], 0, 0)


def sample_positions(N, lo=0, hi=None, places=1024):
    """Positions that the first stage of a selection by pieces may sample: four adjacent scores at
    each of up to 1024 places spread evenly over the candidates (a workgroup of T threads looks at
    the places t * span / T, T = 256, 512 or 1024: all on this grid; the larger samples look at 2048)."""
    hi = N if hi is None else hi
    span = hi - lo
    start = torch.tensor([(lo + (t * span) // places) & ~3 for t in range(places)])
    pos = (start[:, None] + torch.arange(4)[None, :]).reshape(-1)
    return torch.unique(pos[pos < N])


def test_select_pieces_row_count_not_a_multiple_of_eight(oracle):
    """The first stage places the pieces of a row on one XCD and pads its launch to a multiple of
    eight rows: 6 and 11 rows, sink and window, a ragged last piece."""
    say("select by pieces, 6 and 11 rows")
    for B, Hq, N in ((2, 3, 66003), (1, 11, 81925)):
        scores = randn((B, Hq, (N + 3) // 4 * 4), torch.float32, 300 + Hq)
        check_select(oracle, scores, N, 4096, 0, 0)
        check_select(oracle, scores, N, 2000, 64, 100)


@pytest.mark.parametrize("N,rows,k,sink,window", [((1 << 20) - 3, 2, 8192, 0, 0), (1 << 20, 1, 6000, 128, 256), (900001, 3, 8000, 4, 0)])
def test_select_pieces_row_sampled_once(oracle, N, rows, k, sink, window):
    """A small budget of a very long row: the bracket comes from a kernel of its own.  Plain scores,
    a ramp (the last pieces keep nearly all of their scores), few distinct values with NaN and -inf
    among them, and scores that are large only where the sample looks (too little is kept: the whole
    row is selected on) or only where it does not (too much is kept)."""
    say(f"select by pieces, row sampled once, N={N} rows={rows}")
    stride = (N + 3) // 4 * 4
    scores = randn((1, rows, stride), torch.float32, 88)
    check_select(oracle, scores, N, k, sink, window)
    ramp = (scores + torch.arange(stride, dtype=torch.float32, device=DEV) * 1e-4).contiguous()
    check_select(oracle, ramp, N, k, sink, window)
    few = torch.round(scores * 4) / 4
    few[:, :, ::7] = float("nan")
    few[:, :, 3::7] = -float("inf")
    check_select(oracle, few, N, k, sink, window)
    lo, hi = sink, N - window
    places = (lo + torch.arange(2048, device=DEV) * (hi - lo) // 2048) // 4 * 4
    seen = scores.clone()
    for c in range(4):
        seen[:, :, (places + c).clamp(max=N - 1)] += 50.0
    check_select(oracle, seen, N, k, sink, window)
    unseen = scores.clone() + 50.0
    for c in range(4):
        unseen[:, :, (places + c).clamp(max=N - 1)] -= 50.0
    check_select(oracle, unseen, N, k, sink, window)


def test_select_pieces_many_rows(oracle):
    """Enough long rows that the pieces take their widest form (512 threads, 16384 scores)."""
    say("select by pieces, 128 rows")
    N, k = 70001, 4096
    stride = (N + 3) // 4 * 4
    scores = randn((2, 64, stride), torch.float32, 77)
    check_select(oracle, scores, N, k, 0, 0)
    check_select(oracle, scores, N, 7000, 128, 256)
    # every kept score in one wave's span: its LDS region overflows and the piece takes the slower path
    asc = torch.arange(stride, dtype=torch.float32).view(1, 1, -1).expand(2, 64, stride).contiguous().to(DEV)
    check_select(oracle, asc, N, k, 0, 0)
    mixed = scores.clone()
    mixed[:, ::2, 20000:23000] += 100.0  # a dense block of large scores in every other row
    check_select(oracle, mixed, N, k, 3, 9)
    pos = sample_positions(N)
    low = scores.clone()
    low[:, :, pos.to(DEV)] = -1e30
    check_select(oracle, low, N, k, 0, 0)
    # flat distributions put several budgets' worth of scores into one coarse bin around the
    # threshold (the kept scores are cut inside that bin), a ramp towards recent positions puts
    # nearly all kept scores into the last piece (its waves' LDS regions overflow)
    g = torch.Generator().manual_seed(5)
    flat = (1.0 + torch.rand((2, 64, stride), generator=g)).to(DEV)
    check_select(oracle, flat, N, k, 0, 0)
    ramp = (torch.arange(stride, dtype=torch.float32).view(1, 1, -1) * (8.0 / N) + torch.randn((2, 64, stride), generator=g)).to(DEV)
    check_select(oracle, ramp, N, k, 16, 32)
    nan = scores.clone()
    nan[:, :, ::5] = float("nan")
    nan[:, :, 1::5] = float("-inf")
    check_select(oracle, nan, N, 60000, 0, 0)  # the threshold falls among the NaN / -inf ties


@pytest.mark.parametrize("N", [777, 9000, 66000])
def test_select_ties_and_special_values(oracle, N):
    say(f"select ties/specials N={N}")
    g = torch.Generator(device="cpu").manual_seed(N)
    stride = (N + 3) // 4 * 4
    # heavy ties: scores quantised to a handful of values, threshold lands inside a tie block
    q = torch.randint(-3, 4, (1, 4, stride), generator=g).float() * 0.5
    for k in (1, N // 3, N // 2, N - 1):
        check_select(oracle, q.to(DEV), N, k, 0, 0)
    check_select(oracle, q.to(DEV), N, N // 3, 17, 33)
    # all equal
    same = torch.full((1, 2, stride), 1.25)
    check_select(oracle, same.to(DEV), N, N // 5, 0, 0)
    check_select(oracle, same.to(DEV), N, N // 5, 11, 7)
    # special values: +-inf, NaN (ranks with -inf), -0 / +0, denormals, huge and tiny magnitudes
    sp = torch.randn((1, 3, stride), generator=g)
    pos = torch.randperm(N, generator=g)
    vals = [float("inf"), float("-inf"), float("nan"), -0.0, 0.0, 1e-42, -1e-42, 3e38, -3e38, 1e-30]
    for i, v in enumerate(vals):
        sp[:, :, pos[i::len(vals)][: max(1, N // 40)]] = v
    for k in (1, N // 20, N // 2, N - 2):
        check_select(oracle, sp.to(DEV), N, k, 0, 0)
    # all NaN / all -inf mixture: index order decides
    nn = torch.full((1, 1, stride), float("nan"))
    nn[0, 0, ::3] = float("-inf")
    check_select(oracle, nn.to(DEV), N, N // 2, 0, 0)
    # sorted ascending and descending
    asc = torch.arange(stride, dtype=torch.float32).view(1, 1, stride)
    check_select(oracle, asc.to(DEV), N, N // 4, 0, 0)
    check_select(oracle, (-asc).to(DEV), N, N // 4, 2, 2)
    # values that agree in the top 11 and top 22 key bits: every radix level has to refine
    base = torch.full((1, 2, stride), 1.0)
    base = (base.view(torch.int32) + torch.randint(0, 700, (1, 2, stride), generator=g, dtype=torch.int32)).view(torch.float32)
    check_select(oracle, base.to(DEV), N, N // 3, 0, 0)


def test_select_sink_window_cover_everything(oracle):
    say("select sink+window >= N")
    N = 300
    scores = randn((1, 2, 300), torch.float32, 9)
    gi, gc = check_select(oracle, scores, N, 10, 200, 200)
    assert np.all(gc == N)
    gi, gc = check_select(oracle, scores, N, 10, 400, 0)
    assert np.all(gc == N)


def test_select_repeatable_and_workspace_reuse(oracle):
    say("select repeated calls share one workspace")
    from paper_2503_07518_amd import binding as tb
    N, k = 30000, 3000
    scores = randn((2, 8, N), torch.float32, 10)
    d = tb.tb_cache_desc()
    d.B, d.Hq, d.Hkv, d.D, d.Dimp, d.dtype, d.N = 2, 8, 8, 128, 32, tb.TB_F32, N
    d.k_stride_n = d.v_stride_n = 128
    d.ki_stride_n = 32
    ws = tb.new_workspace(tb.TB_OP_SELECT, d)
    first = None
    for _ in range(4):
        idx, cnt = gpu_select(scores, N, k, ws=ws)
        torch.cuda.synchronize()
        if first is None:
            first = (idx.clone(), cnt.clone())
        assert torch.equal(idx, first[0]) and torch.equal(cnt, first[1])
    ridx, rcnt = oracle.select_topk(np_of(scores), k)
    assert np.array_equal(np_of(first[0]), ridx) and np.array_equal(np_of(first[1]), rcnt)
    assert not ws.any(), "the workspace is left zeroed"


# --------------------------------------------------------------------------- neighbours

def random_lists(B, Hq, N, count_max, seed, cap=None):
    rng = np.random.default_rng(seed)
    cap = cap or max(count_max, 1)
    idx = np.full((B, Hq, cap), -1, np.int32)
    cnt = np.zeros((B, Hq), np.int32)
    for b in range(B):
        for h in range(Hq):
            c = int(rng.integers(0, count_max + 1)) if (b + h) % 3 else count_max
            c = min(c, N)
            idx[b, h, :c] = np.sort(rng.choice(N, c, replace=False))
            cnt[b, h] = c
    return idx, cnt


@pytest.mark.parametrize("N,count_max,radius", [(50, 20, 1), (1000, 300, 1), (1000, 999, 2), (70000, 5000, 1),
                                                (4096, 4096, 3), (10, 0, 1), (100000, 7, 5), (5000, 2500, 0)])
@pytest.mark.parametrize("mode", [0, 1])
def test_expand_neighbors(oracle, N, count_max, radius, mode):
    say(f"expand N={N} count_max={count_max} r={radius} mode={mode}")
    idx, cnt = random_lists(2, 3, N, count_max, seed=N + radius)
    # clustered input as well: runs of consecutive positions and picks at both ends
    if count_max >= 8 and N > 64:
        run = np.arange(N - 6, N, dtype=np.int32)
        idx[0, 0, :] = -1
        head = np.array([0, 1, 2], np.int32)
        mid = np.arange(N // 2, N // 2 + min(count_max - 9, 40), dtype=np.int32)
        lst = np.concatenate([head, mid, run])
        idx[0, 0, : len(lst)] = lst
        cnt[0, 0] = len(lst)
    out, oc = gpu_expand(torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV), N, radius, mode)
    torch.cuda.synchronize()
    ro, rc = oracle.expand_neighbors(idx, cnt, N, radius, cap_out=out.shape[-1], mode=mode)
    go, gc = np_of(out), np_of(oc)
    assert np.array_equal(gc, rc)
    mask = np.arange(go.shape[-1])[None, None, :] < rc[..., None]
    assert np.array_equal(np.where(mask, go, -1), np.where(mask, ro, -1))
    assert np.all(go[~mask] == -7)


@pytest.mark.parametrize("mode", [0, 1])
def test_expand_capacity_beyond_30_bits(oracle, mode):
    """Lists that lie more than 2^30 entries apart: every unit reads its own."""
    say(f"expand, lists 2^30 + 16 entries apart, mode={mode}")
    cap, N = (1 << 30) + 16, 1000
    idx = torch.zeros((1, 2, cap), dtype=torch.int32, device=DEV)
    lists = [[3, 4, 500, 999], [7, 100, 101, 102, 640]]
    cnt = torch.tensor([[len(l) for l in lists]], dtype=torch.int32, device=DEV)
    for u, l in enumerate(lists):
        idx[0, u, :len(l)] = torch.tensor(l, dtype=torch.int32)
    small = np_of(idx[:, :, :8])
    out, oc = gpu_expand(idx, cnt, N, 1, mode)
    torch.cuda.synchronize()
    del idx
    torch.cuda.empty_cache()
    ro, rc = oracle.expand_neighbors(small, np_of(cnt), N, 1, cap_out=N, mode=mode)
    assert np.array_equal(np_of(oc), rc)
    for u in range(2):
        assert np.array_equal(np_of(out)[0, u, :rc[0, u]], ro[0, u, :rc[0, u]])


@pytest.mark.parametrize("N,cap,counts", [
    (100000, 16319, (16319, 9000, 0)), (100000, 16320, (16320, 16319, 1)),   # the longest lists staged in LDS
    (100000, 16321, (16321, 16320, 2)), (100000, 16384, (16384, 16383, 5)),  # and the shortest that are not
    (70000, 60000, (60000, 59999, 1023)), (50000, 50000, (50000, 1025, 1)),  # several tens of entries a thread; every position
])
@pytest.mark.parametrize("mode", [0, 1])
def test_expand_long_lists(oracle, N, cap, counts, mode):
    """Either side of the length up to which a list is staged, and well beyond it."""
    say(f"expand long lists N={N} cap={cap} counts={counts} mode={mode}")
    rng = np.random.default_rng(N + cap)
    idx = np.full((1, len(counts), cap), -1, np.int32)
    for u, c in enumerate(counts):
        idx[0, u, :c] = np.sort(rng.choice(N, c, replace=False))
    cnt = np.asarray([counts], np.int32)
    out, oc = gpu_expand(torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV), N, 1, mode)
    torch.cuda.synchronize()
    ro, rc = oracle.expand_neighbors(idx, cnt, N, 1, cap_out=out.shape[-1], mode=mode)
    go = np_of(out)
    assert np.array_equal(np_of(oc), rc)
    mask = np.arange(go.shape[-1])[None, None, :] < rc[..., None]
    assert np.array_equal(np.where(mask, go, -1), np.where(mask, ro, -1)) and np.all(go[~mask] == -7)


# --------------------------------------------------------------------------- attention

@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,N,count_max", [
    (torch.float32, 1, 8, 8, 64, 1024, 128),
    (torch.bfloat16, 1, 32, 8, 128, 5000, 700),
    (torch.bfloat16, 2, 8, 2, 128, 3000, 3000),
    (torch.float32, 1, 4, 2, 128, 777, 333),
    (torch.bfloat16, 1, 4, 4, 64, 900, 65),
    (torch.bfloat16, 1, 2, 2, 128, 40, 1),
    (torch.bfloat16, 3, 16, 2, 128, 9000, 2049),
])
def test_sparse_decode_attn(oracle, dtype, B, Hq, Hkv, D, N, count_max):
    say(f"attn dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} N={N} count_max={count_max}")
    q = randn((B, Hq, D), dtype, 11)
    K = randn((B, Hkv, N + 2, D), dtype, 12)
    V = randn((B, Hkv, N + 2, D), dtype, 13)
    idx, cnt = random_lists(B, Hq, N, count_max, seed=14)
    cnt[0, 0] = 0  # an empty list
    sm = 1 / math.sqrt(D)
    out, lse = gpu_attn(q, K, V, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV), N, sm)
    torch.cuda.synchronize()
    dn = dtype_name(K)
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K)[:, :, :N], np_of(V)[:, :, :N], idx, cnt, dn, sm)
    go, gl = np_of(out), np_of(lse)
    assert_attention(go, ro, dn, gl, rl)
    assert not go[0, 0].any() and gl[0, 0] == -np.inf


def test_attn_full_budget_equals_dense_and_tail(oracle):
    say("attn full list == dense; list + dense tail")
    B, Hq, Hkv, D, N = 1, 8, 2, 128, 2500
    q = randn((B, Hq, D), torch.bfloat16, 15)
    K = randn((B, Hkv, N, D), torch.bfloat16, 16)
    V = randn((B, Hkv, N, D), torch.bfloat16, 17)
    sm = 1 / math.sqrt(D)
    full = torch.arange(N, dtype=torch.int32, device=DEV).expand(B, Hq, N).contiguous()
    cnt = torch.full((B, Hq), N, dtype=torch.int32, device=DEV)
    out, _ = gpu_attn(q, K, V, full, cnt, N, sm)
    torch.cuda.synchronize()
    dense = oracle.dense_decode_attn(np_of(q), np_of(K), np_of(V), "bf16", sm)
    assert_attention(np_of(out), dense, "bf16", what="full list against dense attention")
    # a list over the first part plus the rest as a dense tail gives the same result
    idx, c = random_lists(B, Hq, 2000, 300, seed=18)
    out_t, lse_t = gpu_attn(q, K, V, torch.from_numpy(idx).to(DEV), torch.from_numpy(c).to(DEV), N, sm,
                            tail=(2000, N))
    torch.cuda.synchronize()
    cap = idx.shape[-1] + (N - 2000)
    joined = np.full((B, Hq, cap), -1, np.int32)
    for h in range(Hq):
        joined[0, h, : c[0, h]] = idx[0, h, : c[0, h]]
        joined[0, h, c[0, h]: c[0, h] + N - 2000] = np.arange(2000, N)
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), joined, c + (N - 2000), "bf16", sm)
    assert_attention(np_of(out_t), ro, "bf16", np_of(lse_t), rl)


@pytest.mark.parametrize("dtype,g,Hkv,D", [(torch.bfloat16, 8, 1, 128), (torch.bfloat16, 4, 2, 64), (torch.float32, 2, 4, 128)])
@pytest.mark.parametrize("cap,counts", [(1500, (1500, 1, 127)), (3000, (129, 2999, 0)), (3000, (1023, 1025, 2048)), (5000, (129, 4999, 0)), (5000, (1023, 1025, 5000))])
def test_attn_few_groups_shares(oracle, dtype, g, Hkv, D, cap, counts):
    """Few KV groups, whose longer lists are cut into one share per XCD: lists of every length below their
    capacity, with a tail, and the buffered form the same bit for bit."""
    assert cap < 5000 or attn_plan(dtype, 1, g * Hkv, Hkv, D, cap + 7)[1], "the plan has changed: these shapes were chosen for theirs"
    say(f"attn shares dtype={dtype} g={g} Hkv={Hkv} D={D} counts={counts}")
    B, Hq, N = 1, g * Hkv, 2 * cap + 9
    q, K, V = randn((B, Hq, D), dtype, 26), randn((B, Hkv, N, D), dtype, 27), randn((B, Hkv, N, D), dtype, 28)
    tail, sm = (N - 9, N - 2), 1 / math.sqrt(D)
    idx, cnt = random_lists(B, Hq, N - 9, cap, seed=29)
    for h in range(Hq):
        c = counts[h % 3]
        idx[0, h, :c] = np.sort(np.random.default_rng(h).choice(N - 9, c, replace=False))
        cnt[0, h] = c
    ti, tc = torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)
    out, lse = gpu_attn(q, K, V, ti, tc, N, sm, tail=tail)
    Kbuf, Vbuf = (torch.zeros((B, Hq, cap, D), dtype=dtype, device=DEV) for _ in range(2))
    d = tb.make_desc(N, Hq, K=K, V=V)
    ws = tb.new_workspace(tb.TB_OP_ATTN, d, cap + 7)
    out_b, lse_b = torch.empty_like(out), torch.empty_like(lse)
    tb.tb_gather_kv(d, K, V, ti, tc, cap, Kbuf, Vbuf)
    tb.tb_buffered_decode_attn(d, q, Kbuf, Vbuf, tc, cap, K, V, sm, out_b, lse_b, ws, tail_begin=tail[0], tail_end=tail[1])
    torch.cuda.synchronize()
    joined = np.full((B, Hq, cap + 7), -1, np.int32)
    for h in range(Hq):
        joined[0, h, :cnt[0, h]] = idx[0, h, :cnt[0, h]]
        joined[0, h, cnt[0, h]:cnt[0, h] + 7] = np.arange(*tail)
    dn = dtype_name(K)
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), joined, cnt + 7, dn, sm)
    assert_attention(np_of(out), ro, dn, np_of(lse), rl)
    assert torch.equal(out, out_b) and torch.equal(lse, lse_b)


def test_attn_strided_cache_and_max_count_truncation(oracle):
    say("attn on a strided cache view; max_count truncates longer lists")
    B, Hq, Hkv, D, N = 2, 4, 2, 128, 1200
    q = randn((B, Hq, D), torch.bfloat16, 19)
    Kbig = randn((B, Hkv, N, 2 * D), torch.bfloat16, 20)
    K, V = Kbig[..., :D], Kbig[..., D:]  # interleaved K|V rows, stride 2D
    idx, cnt = random_lists(B, Hq, N, 500, seed=21)
    sm = 0.1
    out, lse = gpu_attn(q, K, V, torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV), N, sm, max_count=260)
    torch.cuda.synchronize()
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), idx, np.minimum(cnt, 260), "bf16", sm)
    assert_attention(np_of(out), ro, "bf16", np_of(lse), rl)


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,rows", [
    (torch.bfloat16, 2, 8, 8, 128, 300),    # lists of their own, several splits
    (torch.float32, 1, 8, 1, 64, 2100),     # in shares, one per XCD
    (torch.float32, 1, 2, 2, 128, 1),
    (torch.bfloat16, 4, 32, 8, 128, 0),     # nothing is named: only the dense range
    (torch.bfloat16, 4, 32, 8, 128, 3300),  # one list for all heads: a workgroup per KV group, on the matrix cores
    (torch.float32, 4, 32, 8, 128, 400),
])
def test_attn_lists_that_are_columns_of_an_array(dtype, B, Hq, Hkv, D, rows):
    """Lists that are the last columns of a wider array: the last of them ends with the array, and nothing behind the entries
    that the call names is read (what lies in front of the next list is a row number outside the cache).  The same bits as for
    lists of their own."""
    say(f"attn lists in columns dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} rows={rows}")
    N, before, tail = rows + 90, 700, (rows + 80, rows + 90)
    q, K, V = randn((B, Hq, D), dtype, 55), randn((B, Hkv, N, D), dtype, 56), randn((B, Hkv, N, D), dtype, 57)
    gen = torch.Generator().manual_seed(58)
    wide = torch.full((B, Hq, before + rows), 1 << 30, dtype=torch.int32)
    wide[:, :, before:] = torch.rand((B, Hq, N), generator=gen).topk(rows, dim=-1).indices.sort(-1).values.to(torch.int32)
    wide = wide.to(DEV)
    idx, cnt = wide[:, :, before:] if rows else wide, torch.full((B, Hq), rows, dtype=torch.int32, device=DEV)
    ws = tb.new_workspace(tb.TB_OP_ATTN, tb.make_desc(N, Hq, K=K, V=V), rows + 10)
    res = [gpu_attn(q, K, V, lists, cnt, N, 0.1, max_count=rows, tail=tail, ws=ws) for lists in (idx, idx.contiguous())]
    shared = []
    for lists in (idx[:, -1], idx[:, -1].contiguous()):  # (one list per batch element, Hq lists of the array apart)
        out, lse = torch.full((B, Hq, D), float("nan"), device=DEV), torch.full((B, Hq), float("nan"), device=DEV)
        tb.tb_sparse_decode_attn_shared(tb.make_desc(N, Hq, K=K, V=V), q, K, V, lists, cnt[:, 0].contiguous(), rows, 0.1, out, lse, ws, *tail)
        shared.append((out, lse))
    torch.cuda.synchronize()
    for a, b in (res, shared):
        assert torch.equal(a[0], b[0]) and torch.equal(a[1], b[1]) and bool(torch.isfinite(a[0]).all())


# splits a head for the full lists of the test below, and whether they are one share of the list per XCD
SPLIT_COUNTS = {(3, 32, 8, 128, 1100): (5, False), (22, 8, 1, 128, 1030): (4, False), (9, 32, 8, 64, 2049): (3, False), (20, 16, 4, 128, 640): (3, False),
                (1, 4, 4, 64, 385): (3, False), (41, 64, 8, 64, 257): (1, False), (22, 8, 1, 128, 2070): (8, True), (1, 16, 2, 64, 8200): (32, True),
                (5, 8, 4, 128, 4000): (24, True)}


@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,N,rows", [
    (torch.bfloat16, 3, 32, 8, 128, 3000, 1100),   # 5 splits, 480 workgroups
    (torch.bfloat16, 22, 8, 1, 128, 1500, 1030),   # more heads than half the compute units, four splits
    (torch.bfloat16, 9, 32, 8, 64, 2500, 2049),    # more heads than compute units, split
    (torch.float32, 20, 16, 4, 128, 700, 640),
    (torch.float32, 1, 4, 4, 64, 400, 385),
    (torch.bfloat16, 41, 64, 8, 64, 300, 257),     # one split a head, several rounds
    (torch.bfloat16, 22, 8, 1, 128, 2500, 2070),   # eight splits: one share of the list per XCD
    (torch.bfloat16, 1, 16, 2, 64, 9000, 8200),    # shares of two workgroups and more
    (torch.float32, 5, 8, 4, 128, 4100, 4000),
])
def test_attn_split_counts(oracle, dtype, B, Hq, Hkv, D, N, rows):
    """Numbers of heads either side of the compute units and of whole rounds of them: full lists, a list that ends before most
    splits begin, one entry, an empty one; one workspace for every length."""
    say(f"attn split counts dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} N={N} rows={rows}")
    dn, sm, g = "f32" if dtype == torch.float32 else "bf16", 1 / math.sqrt(D), Hq // Hkv
    q, K, V = randn((B, Hq, D), dtype, 51), randn((B, Hkv, N, D), dtype, 52), randn((B, Hkv, N, D), dtype, 53)
    gen = torch.Generator().manual_seed(54)
    idx = torch.rand((B, Hq, N), generator=gen).topk(rows, dim=-1).indices.sort(-1).values.to(torch.int32)
    plan, in_shares = attn_plan(dtype, B, Hq, Hkv, D, rows)
    assert (plan.nsplit, in_shares) == SPLIT_COUNTS[B, Hq, Hkv, D, rows], "the plan has changed: these shapes were chosen for theirs"
    ws = tb.new_workspace(tb.TB_OP_ATTN, tb.make_desc(N, Hq, K=K, V=V), rows)
    for most in (rows, rows // 3, 70):
        cnt = torch.full((B, Hq), most, dtype=torch.int32)
        cnt[0, 0], cnt[0, 1], cnt[-1, -1] = 0, 1, min(65, most)
        out, lse = gpu_attn(q, K, V, idx.to(DEV), cnt.to(DEV), N, sm, max_count=most, ws=ws)
        torch.cuda.synchronize()
        for b, h in {(0, 0), (0, 1), (0, Hq - 1), (B // 2, Hq // 2), (B - 1, 0), (B - 1, Hq - 1)}:
            ro, rl = oracle.sparse_decode_attn(np_of(q[b:b + 1, h:h + 1]), np_of(K[b:b + 1, h // g:h // g + 1]), np_of(V[b:b + 1, h // g:h // g + 1]),
                                               idx[b:b + 1, h:h + 1].numpy(), cnt[b:b + 1, h:h + 1].numpy(), dn, sm)
            assert_attention(np_of(out[b, h]), ro[0, 0], dn, np_of(lse[b, h]), rl[0, 0])
        assert bool(torch.isfinite(out).all())


@pytest.mark.parametrize("dtype,B,Hq,Hkv,rows,rooms", [
    (torch.bfloat16, 3, 32, 8, 5000, (7, 6, 5)),         # eight splits planned, six asked for
    (torch.float32, 5, 8, 1, 4000, (20, 16, 14, 13, 12)),  # 24 in shares, one per XCD; thirteen asked for
])
def test_attn_workspace_with_room_for_fewer_splits(oracle, dtype, B, Hq, Hkv, rows, rooms):
    """A workspace made for a shorter list serves with fewer splits as long as it holds what is asked for at least."""
    D, N = 128, rows + 70
    q, K, V = randn((B, Hq, D), dtype, 61), randn((B, Hkv, N, D), dtype, 62), randn((B, Hkv, N, D), dtype, 63)
    plan, _ = attn_plan(dtype, B, Hq, Hkv, D, rows)
    gen = torch.Generator().manual_seed(64)
    idx = torch.rand((B, Hq, N), generator=gen).topk(rows, dim=-1).indices.sort(-1).values.to(torch.int32).to(DEV)
    cnt = torch.full((B, Hq), rows, dtype=torch.int32, device=DEV)
    d, dn = tb.make_desc(N, Hq, K=K, V=V), dtype_name(K)
    ref = None
    for room in (plan.nsplit, *rooms):
        say(f"attn workspace dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} rows={rows}: room for {room} of {plan.nsplit} splits, least {plan.least}")
        shorter = next(r for r in range(1, rows + 1) if attn_plan(dtype, B, Hq, Hkv, D, r)[0].max_split >= room)
        assert attn_plan(dtype, B, Hq, Hkv, D, shorter)[0].max_split == room
        ws = tb.new_workspace(tb.TB_OP_ATTN, d, shorter)
        if room < plan.least:
            with pytest.raises(tb.TbError):
                gpu_attn(q, K, V, idx, cnt, N, 0.1, ws=ws)
            continue
        out, lse = gpu_attn(q, K, V, idx, cnt, N, 0.1, ws=ws)
        torch.cuda.synchronize()
        if ref is None:
            b, h, ref = B - 1, Hq - 1, (out, lse)
            ro, rl = oracle.sparse_decode_attn(np_of(q[b:, h:]), np_of(K[b:, Hkv - 1:]), np_of(V[b:, Hkv - 1:]), np_of(idx[b:, h:]), np_of(cnt[b:, h:]), dn, 0.1)
            assert_attention(np_of(out[b:, h:]), ro, dn, np_of(lse[b:, h:]), rl)
        # fp32 sums in another order: 4000 terms err by a few 1e-6 of the largest at most
        assert float((out - ref[0]).abs().max()) <= 1e-5 and float((lse - ref[1]).abs().max()) <= 1e-5 * float(ref[1].abs().max())


@pytest.mark.parametrize("B,Hq,Hkv,N,k", [(1, 32, 8, 32768, 3277), (16, 32, 8, 16384, 2048)])
def test_attn_split_handover_repeatable(oracle, B, Hq, Hkv, N, k):
    """The split attention hands partial results from workgroup to workgroup (last arriver
    combines): 200 launches on the shapes of the single-sequence and the batched benchmark
    configuration, each compared bit for bit with the first, which is checked against the
    oracle.  Stops at the first mismatch."""
    say(f"attn hand-over: 200 launches, B={B} Hq={Hq} N={N} k={k}")
    D = 128
    q = randn((B, Hq, D), torch.bfloat16, 22)
    K = randn((B, Hkv, N, D), torch.bfloat16, 23)
    V = randn((B, Hkv, N, D), torch.bfloat16, 24)
    rng = np.random.default_rng(25)  # full lists: the largest number of splits
    idx = np.stack([np.stack([np.sort(rng.choice(N, k, replace=False)).astype(np.int32) for _ in range(Hq)])
                    for _ in range(B)])
    cnt = np.full((B, Hq), k, np.int32)
    ti, tc = torch.from_numpy(idx).to(DEV), torch.from_numpy(cnt).to(DEV)
    from paper_2503_07518_amd import binding as tb
    d = tb.make_desc(N, Hq, K=K, V=V)
    ws = tb.new_workspace(tb.TB_OP_ATTN, d, k)
    sm = 1 / math.sqrt(D)
    out, lse = gpu_attn(q, K, V, ti, tc, N, sm, ws=ws)
    torch.cuda.synchronize()
    ref = (out.clone(), lse.clone())
    # the oracle on a sample of units (all of them for the single sequence)
    rng = np.random.default_rng(7)
    units = [(b, h) for b in range(B) for h in range(Hq)] if B == 1 else [
        (int(rng.integers(B)), int(rng.integers(Hq))) for _ in range(64)]
    g = Hq // Hkv
    for b, h in units:
        ro, rl = oracle.sparse_decode_attn(np_of(q[b:b + 1, h:h + 1]), np_of(K[b:b + 1, h // g:h // g + 1]),
                                           np_of(V[b:b + 1, h // g:h // g + 1]), idx[b:b + 1, h:h + 1],
                                           cnt[b:b + 1, h:h + 1], "bf16", sm)
        assert_attention(np_of(out[b, h]), ro[0, 0], "bf16", np_of(lse[b, h]), rl[0, 0])
    for it in range(200):
        out, lse = gpu_attn(q, K, V, ti, tc, N, sm, ws=ws)
        if it % 20 == 19:
            print(f"[case]   launch {it + 1}", flush=True)
        torch.cuda.synchronize()
        assert torch.equal(out, ref[0]) and torch.equal(lse, ref[1]), f"launch {it} differs from the first"


# --------------------------------------------------------------------------- fused step

@pytest.mark.parametrize("dtype,B,Hq,Hkv,D,Dimp,N,k,sink,window", [
    (torch.float32, 1, 8, 8, 64, 16, 1024, 128, 0, 0),
    (torch.bfloat16, 1, 32, 8, 128, 32, 6000, 600, 0, 0),
    (torch.bfloat16, 2, 16, 2, 128, 32, 3001, 300, 16, 32),
    (torch.bfloat16, 1, 8, 2, 128, 32, 500, 500, 0, 0),
    (torch.bfloat16, 1, 8, 2, 128, 32, 500, 0, 4, 4),
])
def test_decode_step_matches_separate_calls_and_oracle(oracle, dtype, B, Hq, Hkv, D, Dimp, N, k, sink, window):
    say(f"decode_step dtype={dtype} B={B} Hq={Hq} Hkv={Hkv} D={D} Dimp={Dimp} N={N} k={k} S={sink} W={window}")
    q = randn((B, Hq, D), dtype, 26)
    q_imp = randn((B, Hq, Dimp), dtype, 27)
    K = randn((B, Hkv, N, D), dtype, 28)
    V = randn((B, Hkv, N, D), dtype, 29)
    W = randn((1, D, Dimp), dtype, 30, 1 / math.sqrt(D))
    Kimp = gpu_project(K, W, N)
    sm = 1 / math.sqrt(D)
    s, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, V, Kimp, N, k, sink, window, sm)
    s2 = gpu_score(q_imp, Kimp, N)
    idx2, cnt2 = gpu_select(s2, N, k, sink, window, Hkv=Hkv)
    out2, lse2 = gpu_attn(q, K, V, idx2, cnt2, N, sm, max_count=idx2.shape[-1])
    torch.cuda.synchronize()
    assert torch.equal(s[:, :, :N], s2[:, :, :N])
    assert torch.equal(cnt, cnt2) and torch.equal(idx, idx2)
    assert torch.equal(out, out2) and torch.equal(lse, lse2)
    dn = dtype_name(K)
    ridx, rcnt = oracle.select_topk(np_of(s)[:, :, :N], k, sink, window)
    assert np.array_equal(np_of(cnt), rcnt)
    assert np.array_equal(np_of(idx)[..., : ridx.shape[-1]], ridx)
    ro, rl = oracle.sparse_decode_attn(np_of(q), np_of(K), np_of(V), np_of(idx), np_of(cnt), dn, sm)
    assert_attention(np_of(out), ro, dn, np_of(lse), rl)


@pytest.mark.parametrize("dtype,B,g,Hkv,D,N,k,sink,window", [
    (torch.float32, 4, 1, 8, 128, 5003, 3000, 37, 101),
    (torch.bfloat16, 8, 2, 8, 64, 9601, 3700, 0, 160),
    (torch.bfloat16, 16, 4, 8, 128, 4001, 483, 5, 0),
])
def test_decode_step_large_lists(oracle, dtype, B, g, Hkv, D, N, k, sink, window):
    """Lists of more than 100 MB of rows, just selected, are gathered non-temporally; handed in, like any others: the same
    bits, with an infinite row that is in nobody's list; without a sink it is the one that a tile's empty slots load.  One unit
    against the oracle."""
    say(f"decode_step large lists dtype={dtype} B={B} g={g} Hkv={Hkv} D={D} N={N} k={k} S={sink} W={window}")
    Hq, Dimp, sm = g * Hkv, 16, 1 / math.sqrt(D)
    q, q_imp = randn((B, Hq, D), dtype, 36), randn((B, Hq, Dimp), dtype, 37)
    gen = torch.Generator(device=DEV).manual_seed(38)
    K, V = (torch.randn((B, Hkv, N, D), generator=gen, device=DEV).to(dtype) for _ in range(2))
    Kimp = torch.randn((B, Hkv, N, Dimp), generator=gen, device=DEV).to(dtype)
    low = sink + 1 if sink else 0  # (never selected: the only row with a score that is not finite; an empty slot loads row 0)
    Kimp[:, :, low], V[:, :, low] = float("nan"), float("inf")
    s, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, V, Kimp, N, k, sink, window, sm)
    out2, lse2 = gpu_attn(q, K, V, idx, cnt, N, sm, max_count=idx.shape[-1])
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(lse, lse2) and bool(torch.isfinite(out).all())
    b, h = B - 1, Hq - 1
    ro, rl = oracle.sparse_decode_attn(np_of(q[b:b + 1, h:h + 1]), np_of(K[b:b + 1, h // g:h // g + 1]), np_of(V[b:b + 1, h // g:h // g + 1]),
                                       np_of(idx[b:b + 1, h:h + 1]), np_of(cnt[b:b + 1, h:h + 1]), dtype_name(K), sm)
    assert_attention(np_of(out[b, h]), ro[0, 0], dtype_name(K), np_of(lse[b, h]), rl[0, 0])


@pytest.mark.parametrize("dtype", [torch.bfloat16, torch.float32])
@pytest.mark.parametrize("g,Hkv,B,D,Dimp,N,k,sink,window", [
    (1, 1, 1, 64, 16, 1, 1, 0, 0),
    (2, 3, 1, 128, 32, 65, 9, 1, 2),
    (4, 8, 4, 128, 32, 1023, 130, 4, 64),      # 128 heads, one and two splits of the attention
    (8, 8, 4, 64, 16, 4095, 400, 128, 256),    # 256 heads: the most
    (8, 8, 4, 64, 64, 800, 90, 0, 0),
    (1, 8, 1, 64, 16, 1024, 128, 0, 0),
    (2, 2, 1, 128, 32, 2051, 500, 0, 0),       # bf16: three splits
    (4, 1, 1, 128, 16, 4096, 511, 0, 0),       # the longest row
    (4, 1, 1, 64, 16, 4096, 300, 0, 0),
    (2, 1, 1, 128, 64, 1025, 200, 2, 0),
    (4, 1, 1, 128, 64, 2051, 500, 0, 0),       # more bytes than one workgroup takes: separate kernels
    (4, 2, 1, 64, 32, 700, 700, 0, 0),         # everything kept
    (8, 1, 1, 128, 32, 300, 0, 0, 0),          # nothing kept
    (4, 8, 9, 64, 32, 500, 50, 0, 0),          # 288 heads, and a row of 4097: separate kernels
    (4, 1, 1, 64, 32, 4097, 100, 0, 0),
])
def test_decode_step_short_rows(oracle, dtype, g, Hkv, B, D, Dimp, N, k, sink, window):
    """A short step is one launch: scores, lists, outputs must be those of the separate calls bit for bit (projected keys with
    ties, NaN and infinities among them), in caches with strides of their own."""
    say(f"decode_step short rows dtype={dtype} g={g} Hkv={Hkv} B={B} D={D} Dimp={Dimp} N={N} k={k}")
    Hq, cap = g * Hkv, N + 5
    K, V = randn((B, cap, Hkv, D + 8), dtype, 41).transpose(1, 2)[..., :D], randn((B, Hkv, cap, D), dtype, 42)
    Kimp = randn((B, Hkv, cap, Dimp + 16), dtype, 43)[..., :Dimp]
    q, q_imp = randn((B, Hq, D), dtype, 44), randn((B, Hq, Dimp), dtype, 45)
    tied, odd = Kimp.clone(), Kimp.clone()
    tied[:, :, 1::2] = tied[:, :, :1]
    odd[:, :, ::5, 0], odd[:, :, 1::7, 1], odd[:, :, 2::9, 2] = float("nan"), -float("inf"), float("inf")
    for name, keys, scale in (("random", Kimp, 1.0), ("negative", Kimp, -0.5), ("tied", tied, 1.0), ("odd", odd, 1.0)):
        s, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, V, keys, N, k, sink, window, 0.1, scale=scale)
        s2 = gpu_score(q_imp, keys, N, scale)
        idx2, cnt2 = gpu_select(s2, N, k, sink, window, Hkv=Hkv)
        out2, lse2 = gpu_attn(q, K, V, idx2, cnt2, N, 0.1, max_count=tb.policy_count(N, k, sink, window))
        ridx, rcnt = oracle.select_topk(np_of(s2)[:, :, :N], k, sink, window)
        need = tb.policy_count(N, k, sink, window)
        assert np.array_equal(np_of(s)[:, :, :N].view(np.uint32), np_of(s2)[:, :, :N].view(np.uint32)), name
        assert np.array_equal(np_of(cnt), rcnt) and np.array_equal(np_of(idx)[..., :need], ridx[..., :need]), name
        assert torch.equal(cnt, cnt2) and torch.equal(idx, idx2), name
        assert torch.equal(out, out2) and torch.equal(lse, lse2), name


@pytest.mark.parametrize("dtype,g,Hkv,D,Dimp,N,k,sink,window", [
    (torch.bfloat16, 4, 1, 64, 16, 4096, 1200, 0, 0),   # the longest row, all four splits
    (torch.bfloat16, 2, 2, 64, 32, 3001, 1100, 3, 21),
    (torch.float32, 1, 2, 64, 16, 2051, 650, 0, 0),
    (torch.float32, 2, 1, 64, 16, 2600, 600, 5, 0),
])
def test_decode_step_short_rows_misleading_sample(oracle, dtype, g, Hkv, D, Dimp, N, k, sink, window):
    """One launch, with scores that are huge or tiny exactly where its selection takes a sample (four adjacent ones at each of
    256 places): the bracket misses the threshold and is widened."""
    say(f"decode_step short rows, misleading sample dtype={dtype} g={g} Hkv={Hkv} N={N} k={k}")
    Hq, lo, span = g * Hkv, sink, N - window - sink
    K, V, Kimp = randn((1, Hkv, N, D), dtype, 51), randn((1, Hkv, N, D), dtype, 52), randn((1, Hkv, N, Dimp), dtype, 53)
    q = randn((1, Hq, D), dtype, 54)
    q_imp = randn((1, Hkv, Dimp), dtype, 55).repeat_interleave(g, dim=1)  # (one direction a KV group: its heads agree on what is huge)
    pos = torch.tensor([((lo + t * span // 256) & ~3) + c for t in range(256) for c in range(4)])
    pos = torch.unique(pos[(pos >= lo) & (pos < lo + span)])
    rank, share = k * len(pos) / span, k / span
    past = rank + 6 * math.sqrt(rank * (1 - share)) + 4  # the sample's rank for the bracket's lower end
    n_high = min(len(pos), int(past + k) // 2)
    assert past + 2 < n_high < k, "the sample puts the threshold among the huge scores, the row does not"
    high, low = Kimp.clone(), Kimp.clone()
    high[:, :, pos[torch.randperm(len(pos), generator=torch.Generator().manual_seed(N))[:n_high]].to(DEV)] = 30 * q_imp[:, ::g, None]
    low[:, :, pos.to(DEV)] = -30 * q_imp[:, ::g, None]
    for name, keys, kk in (("misled high", high, k), ("misled low", low, min(k, (span - len(pos)) // 2)), ("misled high, negative", low, -(-k // 2))):
        scale = -1.0 if "negative" in name else 1.0
        s, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, V, keys, N, kk, sink, window, 0.1, scale=scale)
        s2 = gpu_score(q_imp, keys, N, scale)
        need = tb.policy_count(N, kk, sink, window)
        ridx, rcnt = oracle.select_topk(np_of(s2)[:, :, :N], kk, sink, window)
        assert np.array_equal(np_of(s)[:, :, :N].view(np.uint32), np_of(s2)[:, :, :N].view(np.uint32)), name
        assert np.array_equal(np_of(cnt), rcnt) and np.array_equal(np_of(idx)[..., :need], ridx[..., :need]), name
        idx2, cnt2 = gpu_select(s2, N, kk, sink, window, Hkv=Hkv)
        out2, lse2 = gpu_attn(q, K, V, idx2, cnt2, N, 0.1, max_count=need)
        assert torch.equal(out, out2) and torch.equal(lse, lse2), name


@pytest.mark.parametrize("dtype,g,Hkv,Dimp,N,sink,window", [(torch.bfloat16, 4, 2, 16, (1 << 20) - 5, 0, 0), (torch.float32, 2, 1, 16, 1 << 20, 128, 257),
                                                            (torch.bfloat16, 2, 1, 32, 900001, 4, 0)])
def test_decode_step_long_rows_larger_sample(oracle, dtype, g, Hkv, Dimp, N, sink, window):
    """A hundredth of a very long row kept: the bracket comes from 8192 scored rows.  Scores in no order, huge ones exactly at
    the sampled places (too little is kept) and tiny ones there (too much is): the second stage then selects on the whole row.
    Outputs are those of the separate calls: the attention's partial sums take the place of the kept scores."""
    say(f"decode_step long rows, larger sample dtype={dtype} g={g} Hkv={Hkv} Dimp={Dimp} N={N}")
    Hq, k, D = g * Hkv, N // 100, 64
    K, V, Kimp = randn((1, Hkv, N, D), dtype, 61), randn((1, Hkv, N, D), dtype, 62), randn((1, Hkv, N, Dimp), dtype, 63)
    q = randn((1, Hq, D), dtype, 64)
    q_imp = randn((1, Hkv, Dimp), dtype, 65).repeat_interleave(g, dim=1)
    pos = sample_positions(N, sink, N - window, places=2048).to(DEV)
    assert len(pos) < k
    high, low = Kimp.clone(), Kimp.clone()
    high[:, :, pos], low[:, :, pos] = 30 * q_imp[:, ::g, None], -30 * q_imp[:, ::g, None]
    need = tb.policy_count(N, k, sink, window)
    for name, keys in (("random", Kimp), ("misled high", high), ("misled low", low)):
        scores, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, V, keys, N, k, sink, window, 0.125)
        separate = gpu_score(q_imp, keys, N)
        ridx, rcnt = oracle.select_topk(np_of(separate)[:, :, :N], k, sink, window)
        assert np.array_equal(np_of(scores)[:, :, :N].view(np.uint32), np_of(separate)[:, :, :N].view(np.uint32)), name
        assert np.array_equal(np_of(cnt), rcnt) and np.array_equal(np_of(idx)[..., :need], ridx[..., :need]), name
        out2, lse2 = gpu_attn(q, K, V, idx, cnt, N, 0.125, max_count=need)
        assert torch.equal(out, out2) and torch.equal(lse, lse2), name


@pytest.mark.parametrize("dtype,g,Hkv,B,Dimp,N", [
    (torch.bfloat16, 1, 3, 1, 16, 65537),     # one row past the separate calls, a last piece of one row
    (torch.float32, 2, 1, 2, 16, 70003),      # two of four waves have a head
    (torch.bfloat16, 2, 3, 1, 32, 66001),
    (torch.bfloat16, 4, 1, 1, 32, 131072),
    (torch.float32, 8, 1, 1, 16, 131073),     # two heads a wave
    (torch.bfloat16, 8, 3, 1, 32, 100001),    # a number of KV groups that is no multiple of eight
    (torch.bfloat16, 4, 2, 1, 16, (1 << 20) - 5),  # pieces of sixteen blocks; the larger sample where a hundredth is kept
    (torch.float32, 4, 1, 1, 16, 1 << 20),
    (torch.bfloat16, 1, 2, 1, 32, 66001),     # either side of the rule: scores and selection stay apart
    (torch.float32, 8, 1, 1, 32, 66001),
])
def test_decode_step_long_rows(oracle, dtype, g, Hkv, B, Dimp, N):
    """Rows of more than 65536 scores: the scoring kernel keeps the scores that a sampled bracket does not rule out.  The
    scores must be those of the scoring call, bit for bit, and the lists the oracle's on them, with thresholds
    above and below zero, ties, NaN, ascending rows (all that is kept crowds into the last pieces) and a sample that misleads; a
    workspace too small for the lists of the pieces gives the same results."""
    say(f"decode_step long rows dtype={dtype} g={g} Hkv={Hkv} B={B} Dimp={Dimp} N={N}")
    Hq = g * Hkv
    cap = N + 3
    K = torch.zeros((B, Hkv, cap, 64), dtype=dtype, device=DEV)  # (the attention is not what is tested)
    Kimp = randn((B, Hkv, cap, Dimp), dtype, 31)
    q_imp, q = randn((B, Hq, Dimp), dtype, 32), randn((B, Hq, 64), dtype, 33)
    inf, nan = float("inf"), float("nan")
    ramp = torch.zeros_like(Kimp)
    ramp[..., 0] = (torch.arange(cap, device=DEV) // 256).to(dtype)  # (256 equal scores a block: ties at every threshold)
    odd = Kimp.clone()
    odd[:, :, ::5, 0], odd[:, :, 1::5, 1], odd[:, :, 2::997, 2] = nan, -inf, inf
    lie, low = Kimp.clone(), Kimp.clone()
    pos = sample_positions(N).to(DEV)
    lie[:, :, pos], low[:, :, pos] = 30 * q_imp[:, ::g, None], -30 * q_imp[:, ::g, None]
    d = tb.make_desc(N, Hq, K=K, V=K, Kimp=Kimp)
    some = min(N // 8, 5000)
    for name, keys, scale, k, sink, window in (
            ("random", Kimp, 0.5, some, 0, 0), ("random", Kimp, -1.0, N // 100, 128, 257), ("random", Kimp, 1.0, 1, 3, 0),
            ("ramp", ramp, 1.0, some, 4, 64), ("ramp", ramp, -1.0, some, 0, 0), ("odd", odd, 1.0, some, 0, 5),
            ("constant", torch.zeros_like(Kimp), 1.0, some, 1, 1), ("misled high", lie, 1.0, some, 0, 0), ("misled low", low, 1.0, some, 0, 0)):
        separate = gpu_score(q_imp, keys, N, scale)
        ridx, rcnt = oracle.select_topk(np_of(separate)[:, :, :N], k, sink, window)
        need = tb.policy_count(N, k, sink, window)
        small = tb.new_workspace(tb.TB_OP_ATTN, d, need)
        for ws in (None, small):
            scores, idx, cnt, out, lse = gpu_decode_step(q, q_imp, K, K, keys, N, k, sink, window, 1.0, scale=scale, ws=ws)
            assert np.array_equal(np_of(scores)[:, :, :N].view(np.uint32), np_of(separate)[:, :, :N].view(np.uint32)), name
            assert np.array_equal(np_of(cnt), rcnt), name
            assert np.array_equal(np_of(idx)[..., :need], ridx[..., :need]), name


def test_read_stream_probe_reads_and_writes_nothing():
    """The bandwidth calibration kernel: any size (also below one vector, and ragged), the
    source and the sink word stay as they were."""
    from paper_2503_07518_amd import binding as tb
    print("[case] read-stream probe", flush=True)
    for nbytes in (8, 16, 100, 4096 * 33 + 16, 1 << 22):
        src = torch.arange(max(nbytes, 16), dtype=torch.int64, device=DEV).to(torch.uint8)[:max(nbytes, 16)].contiguous()
        before = src.clone()
        sink = torch.full((4,), 7, dtype=torch.int32, device=DEV)
        tb.tb_read_stream_probe(src[:nbytes], sink)
        torch.cuda.synchronize()
        assert torch.equal(src, before) and torch.all(sink == 7)
