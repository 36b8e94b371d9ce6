"""Host-side checks of the C ABI that need no GPU: the library loads, exports every symbol the
header declares, and rejects bad arguments on the host before anything is launched."""
import ctypes
import os
import re

import pytest

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


@pytest.fixture(scope="module")
def tb():
    from paper_2503_07518_amd import binding

    if not os.path.exists(binding.LIB_PATH):
        from paper_2503_07518_amd import build

        build.build(force=True)
    binding.load_library()
    return binding


def declared_symbols():
    text = open(os.path.join(ROOT, "include", "tokenbutler.h")).read()
    text = re.sub(r"/\*.*?\*/", "", text, flags=re.S)
    return sorted(set(re.findall(r"\b(tb_[a-z_]+)\s*\(", text)))


def test_header_symbols_are_exported(tb):
    names = declared_symbols()
    assert set(names) == set(tb.EXPORTS), (names, tb.EXPORTS)
    lib = tb.load_library()
    for n in names:
        assert getattr(lib, n) is not None
    # nothing else takes up a name without a namespace, which a program's own function of that name would stand in for
    for n in ("sparse_attn", "buffered_attn", "check_gather", "check_append"):
        assert not hasattr(lib, n), n


def test_version_and_status_strings(tb):
    assert tb.tb_version() >= 100
    assert tb.status_string(0) == "ok"
    for code in (1, 2, 3, 4):
        assert tb.status_string(code) not in ("ok", "unknown status")
    assert tb.status_string(99) == "unknown status"


def desc(tb, **kw):
    d = tb.tb_cache_desc()
    base = dict(B=1, Hq=8, Hkv=2, D=128, Dimp=32, dtype=tb.TB_BF16, N=1000,
                k_stride_b=2 * 1024 * 128, k_stride_h=1024 * 128, k_stride_n=128,
                v_stride_b=2 * 1024 * 128, v_stride_h=1024 * 128, v_stride_n=128,
                ki_stride_b=2 * 1024 * 32, ki_stride_h=1024 * 32, ki_stride_n=32)
    base.update(kw)
    for k, v in base.items():
        setattr(d, k, v)
    return d


P = ctypes.c_void_p(0x10000)  # never dereferenced: every call below must fail validation first
NULL = None


def test_workspace_sizes(tb):
    d = desc(tb)
    sel = tb.tb_workspace_bytes(tb.TB_OP_SELECT, d, 0)
    att = tb.tb_workspace_bytes(tb.TB_OP_ATTN, d, 500)
    step = tb.tb_workspace_bytes(tb.TB_OP_DECODE_STEP, d, 500)
    assert sel == 0 and att >= 8 * 256 and step == att
    assert tb.tb_workspace_bytes(99, d, 0) == 0
    assert tb.tb_workspace_bytes(tb.TB_OP_ATTN, desc(tb, D=96), 10) == 0
    assert tb.tb_workspace_bytes(tb.TB_OP_ATTN, d, -1) == 0
    # long rows on few heads are selected in two stages and need room for the candidates
    long_row = desc(tb, N=1 << 20)
    need = tb.tb_workspace_bytes(tb.TB_OP_SELECT, long_row, 8192)
    assert need >= 8 * 8 * 8192 * 8 and tb.tb_workspace_bytes(tb.TB_OP_DECODE_STEP, long_row, 8192) >= need
    assert tb.tb_workspace_bytes(tb.TB_OP_SELECT, long_row, 0) == 0


@pytest.mark.parametrize("B,Hq,Hkv,Dimp,k", [(14, 32, 8, 32, 2000), (1, 32, 8, 32, 2000), (1, 8, 8, 32, 1000), (3, 24, 3, 16, 5000), (16, 64, 8, 64, 8192),
                                               (5, 1, 1, 32, 30000)])
def test_workspace_of_a_capacity_serves_fewer_rows(tb, B, Hq, Hkv, Dimp, k):
    """A workspace made for a cache's capacity is enough for every number of rows on the way there."""
    rows = sorted({*range(1024, 1 << 20, 9973), *range(65535, 90000, 61), 74877, 74941, 1 << 17, (1 << 17) + 1, 1 << 20})
    for op in (tb.TB_OP_SELECT, tb.TB_OP_ATTN, tb.TB_OP_DECODE_STEP):
        sizes = [tb.tb_workspace_bytes(op, desc(tb, B=B, Hq=Hq, Hkv=Hkv, Dimp=Dimp, N=n), k) for n in rows]
        assert sizes == sorted(sizes), (op, next((rows[i], sizes[i], rows[i + 1], sizes[i + 1]) for i in range(len(sizes) - 1) if sizes[i] > sizes[i + 1]))


def rounded(rows, want, granule):
    """`want` splits or a few less: as many as equal shares of whole granules make."""
    share = -(-rows // want)
    return -(-rows // (-(-share // granule) * granule))


@pytest.mark.parametrize("f32,B,Hq,Hkv,rows,splits", [
    (False, 1, 8, 2, 3277, 24), (False, 1, 16, 4, 8384, 32), (True, 1, 8, 1, 8196, 64), (False, 1, 16, 4, 3350, 24), (False, 2, 4, 2, 6890, 32),
    (False, 1, 8, 1, 2050, 16), (False, 1, 8, 1, 3100, 24), (False, 1, 32, 4, 3100, 16)])
def test_attention_plan_in_shares(tb, f32, B, Hq, Hkv, rows, splits):
    """Where the plan counts on the list being cut into one share per XCD, the number of splits is a multiple of them."""
    import torch
    from gpu_util import attn_plan
    p, in_shares = attn_plan(torch.float32 if f32 else torch.bfloat16, B, Hq, Hkv, 128, rows)
    assert (p.nsplit, in_shares) == (splits, True)


@pytest.mark.parametrize("f32,B,Hq,Hkv,D,rows,splits", [(False, 1, 8, 2, 128, 1590, 12), (False, 1, 16, 4, 128, 1590, 12), (True, 1, 16, 2, 64, 1590, 12),
                                                        (False, 2, 4, 1, 128, 1300, 10)])
def test_attention_plan_of_few_short_lists(tb, f32, B, Hq, Hkv, D, rows, splits):
    """In a launch of one round the shares' gain is small: eight of them do not take the place of half as many splits again."""
    import torch
    from gpu_util import attn_plan
    p, in_shares = attn_plan(torch.float32 if f32 else torch.bfloat16, B, Hq, Hkv, D, rows)
    assert (p.nsplit, in_shares) == (splits, False)


@pytest.mark.parametrize("f32,B,Hq,Hkv,D,rows,splits", [(True, 9, 8, 2, 64, 5000, 16), (True, 20, 8, 1, 64, 1000, 4), (True, 9, 16, 2, 128, 660, 8),
                                                        (False, 9, 16, 2, 64, 2327, 8), (False, 3, 32, 4, 128, 1000, 4), (True, 3, 32, 4, 128, 400, 4)])
def test_attention_plan_of_one_list_for_all_heads(tb, f32, B, Hq, Hkv, D, rows, splits):
    """Heads that read the same list meet on an XCD with a multiple of four splits."""
    import torch
    from gpu_util import attn_plan
    assert attn_plan(torch.float32 if f32 else torch.bfloat16, B, Hq, Hkv, D, rows, one_list=True)[0].nsplit == splits


def test_attention_plan_and_workspace(tb):
    """For every length: no more splits than a workspace made for that length has room for, no more asked for than two
    workgroups a compute unit (which every workspace held that was made for as many rows), and from 32 splits on in shares."""
    import torch
    from gpu_util import attn_plan
    for dtype, D in ((torch.bfloat16, 128), (torch.bfloat16, 64), (torch.float32, 128)):
        tile = {(torch.bfloat16, 128): 64, (torch.bfloat16, 64): 128, (torch.float32, 128): 32}[dtype, D]
        for B, Hq, Hkv in ((1, 1, 1), (1, 8, 1), (1, 8, 8), (1, 16, 2), (3, 8, 1), (1, 32, 4), (1, 32, 8), (3, 32, 8), (5, 40, 5), (2, 256, 256), (20, 64, 8)):
            units, longest = B * Hq, 0
            for rows, one_list in ((r, one) for r in range(1, 12000, 41) for one in (False, True)):
                p, in_shares = attn_plan(dtype, B, Hq, Hkv, D, rows, one_list)
                before = rounded(rows, max(1, min(-(-512 // units), rows // (2 * tile))), tile // 4)
                assert 1 <= p.least <= min(p.nsplit, before) and p.nsplit <= p.max_split, (units, rows, tile)
                assert longest <= p.max_split
                longest = p.max_split
                assert p.multiple in ((1, 2, 4, 8) if one_list else (1, 8)) and p.nsplit % p.multiple == 0
                if not one_list and Hq > Hkv and B * Hkv % 8 and p.nsplit >= 32:
                    assert in_shares, (units, rows, tile)


def test_rejects_bad_arguments_without_launching(tb):
    L = tb.load_library()
    d = desc(tb)
    r = ctypes.byref
    # null pointers
    assert L.tb_score(r(d), NULL, P, 1.0, P, 1000, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_project_keys(r(d), P, NULL, 1, P, 0, 10, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_select_topk(r(d), P, 1000, 10, 0, 0, NULL, P, 100, P, 1 << 20, None) == tb.TB_ERR_INVALID_ARG
    # inconsistent shapes
    assert L.tb_score(r(desc(tb, Hq=7)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_score(r(desc(tb, N=-1)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_score(r(d), P, P, 1.0, P, 996, None) == tb.TB_ERR_INVALID_ARG  # stride < N
    # unsupported shapes / alignment
    assert L.tb_score(r(desc(tb, Dimp=24)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_score(r(desc(tb, D=96)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_score(r(desc(tb, Hq=6, Hkv=2)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_score(r(d), P, P, 1.0, P, 1002, None) == tb.TB_ERR_UNSUPPORTED  # stride % 4
    assert L.tb_score(r(d), ctypes.c_void_p(0x10004), P, 1.0, P, 1000, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_score(r(desc(tb, ki_stride_n=36)), P, P, 1.0, P, 1000, None) == tb.TB_ERR_UNSUPPORTED
    # projection ranges
    assert L.tb_project_keys(r(d), P, P, 1, P, 5, 4, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_project_keys(r(d), P, P, 1, P, 0, 1001, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_project_keys(r(d), P, P, 3, P, 0, 10, None) == tb.TB_ERR_INVALID_ARG  # Hw not 1 or Hkv
    assert L.tb_project_keys(r(d), P, P, 1, P, 7, 7, None) == tb.TB_OK  # empty range: no-op
    # selection: negative budget, capacity too small, missing workspace, N too large
    assert L.tb_select_topk(r(d), P, 1000, -1, 0, 0, P, P, 100, P, 1 << 20, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_select_topk(r(d), P, 1000, 10, 4, 4, P, P, 17, P, 1 << 20, None) == tb.TB_ERR_INVALID_ARG
    big = desc(tb, N=(1 << 20) + 4)
    assert L.tb_select_topk(r(big), P, (1 << 20) + 4, 10, 0, 0, P, P, 10, P, 1 << 20, None) == tb.TB_ERR_UNSUPPORTED
    # neighbours: output capacity, mode, aliasing
    assert L.tb_expand_neighbors(1, 8, 1000, 1, 0, P, P, 100, ctypes.c_void_p(0x20000), P, 299, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_expand_neighbors(1, 8, 1000, 1, 2, P, P, 100, ctypes.c_void_p(0x20000), P, 300, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_expand_neighbors(1, 8, 1000, 1, 0, P, P, 100, P, P, 300, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_expand_neighbors(1, 8, 1000, -1, 0, P, P, 100, ctypes.c_void_p(0x20000), P, 300, None) == tb.TB_ERR_INVALID_ARG
    # attention: max_count beyond capacity, tail outside the cache, workspace too small
    assert L.tb_sparse_decode_attn(r(d), P, P, P, P, P, 100, 101, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_sparse_decode_attn(r(d), P, P, P, P, P, 100, 100, 990, 1001, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_sparse_decode_attn(r(d), P, P, P, P, P, 100, 100, 0, 0, 1.0, P, NULL, P, 64, None) == tb.TB_ERR_WORKSPACE
    assert L.tb_sparse_decode_attn(r(desc(tb, k_stride_n=100)), P, P, P, P, P, 100, 100, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    # the head-less form takes the same checks
    assert L.tb_sparse_decode_attn_shared(r(d), P, P, P, P, P, 100, 101, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_sparse_decode_attn_shared(r(d), P, P, P, NULL, P, 100, 100, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_sparse_decode_attn_shared(r(d), P, P, P, P, P, 100, 100, 0, 0, 1.0, P, NULL, P, 64, None) == tb.TB_ERR_WORKSPACE
    # fused step inherits all of the above
    assert L.tb_decode_step(r(d), P, P, 1.0, P, P, P, 10, 0, 0, 1.0, P, 1000, P, P, 9, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_decode_step(r(d), P, P, 1.0, P, P, P, 10, 0, 0, 1.0, P, 1000, P, P, 10, P, NULL, P, 64, None) == tb.TB_ERR_WORKSPACE
    # buffer migration and buffered attention: capacities, null buffers, workspace
    assert L.tb_gather_kv(r(d), P, P, P, P, 100, 101, P, P, 200, None) == tb.TB_ERR_INVALID_ARG  # max_count > idx_cap
    assert L.tb_gather_kv(r(d), P, P, P, P, 100, 100, P, P, 99, None) == tb.TB_ERR_INVALID_ARG   # buffer too small
    assert L.tb_gather_kv(r(d), P, P, P, P, 100, 100, NULL, P, 100, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_gather_kv(r(d), P, P, P, P, 100, 100, ctypes.c_void_p(0x10008), P, 100, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_buffered_decode_attn(r(d), P, NULL, P, 100, P, 100, P, P, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_buffered_decode_attn(r(d), P, P, P, 100, P, 101, P, P, 0, 0, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_buffered_decode_attn(r(d), P, P, P, 100, P, 100, P, P, 0, 1001, 1.0, P, NULL, P, 1 << 24, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_buffered_decode_attn(r(d), P, P, P, 100, P, 100, P, P, 0, 0, 1.0, P, NULL, P, 64, None) == tb.TB_ERR_WORKSPACE
    # query predictor: shapes, null pointers, sizes outside the supported range
    pd = tb.tb_predictor_desc(4096, 512, 4, 32, 32, tb.TB_BF16, 1e-5)
    args = (P, P, P, P, P, P, P, P, P, P)
    assert L.tb_predict_queries(r(pd), 1, NULL, *args[1:], None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_predict_queries(r(pd), -1, *args, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_predict_queries(r(tb.tb_predictor_desc(4100, 512, 4, 32, 32, tb.TB_BF16, 1e-5)), 1, *args, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_predict_queries(r(tb.tb_predictor_desc(16384, 512, 4, 32, 32, tb.TB_BF16, 1e-5)), 1, *args, None) == tb.TB_ERR_UNSUPPORTED
    assert L.tb_predict_queries(r(tb.tb_predictor_desc(4096, 512, 0, 32, 32, tb.TB_BF16, 1e-5)), 1, *args, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_predict_queries(r(tb.tb_predictor_desc(4096, 512, 4, 32, 32, 7, 1e-5)), 1, *args, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_predict_queries(r(pd), 0, *args, None) == tb.TB_OK  # empty batch: no-op
    # workspace init
    assert L.tb_workspace_init(NULL, 16, None) == tb.TB_ERR_INVALID_ARG
    assert L.tb_workspace_init(P, 6, None) == tb.TB_ERR_INVALID_ARG


def migrate(tb, src, dst, idx_cap=100, max_count=100, front=0, back=0, src_row=-1, dst_row=0, buf_cap=100, tail=(0, 0), ws_bytes=64):
    """tb_migrate_buffered_decode_attn with a workspace that is too small: a call that gets so far has passed every other check."""
    r = ctypes.byref
    return tb.load_library().tb_migrate_buffered_decode_attn(r(src), P, P, P, P, idx_cap, max_count, front, back, P, src_row, r(dst), P, P, P, buf_cap, P, P,
                                                             dst_row, *tail, 1.0, P, NULL, P, ws_bytes, None)


@pytest.mark.parametrize("rows,want", [(1 << 30, "TB_ERR_WORKSPACE"), ((1 << 30) + 1, "TB_ERR_UNSUPPORTED"), (1 << 33, "TB_ERR_UNSUPPORTED")])
def test_migration_refuses_rows_that_its_numbers_cannot_name(tb, rows, want):
    """Bit 30 of a row number says which cache the row is in: a source of more rows than that is refused."""
    strides = dict(k_stride_b=0, k_stride_h=0, v_stride_b=0, v_stride_h=0)
    assert migrate(tb, desc(tb, N=rows, **strides), desc(tb)) == getattr(tb, want)


def test_missing_library_is_an_error(tb, monkeypatch, tmp_path):
    """The product path has no fallback: without the HIP library the ops raise."""
    monkeypatch.setattr(tb, "_lib", None)
    monkeypatch.setattr(tb, "LIB_PATH", str(tmp_path / "libtokenbutler.so"))
    with pytest.raises(ImportError):
        tb.tb_version()


def test_current_stream_without_the_raw_handle(tb, monkeypatch):
    """A torch that lacks the function that gives a stream's bare handle still gives the stream."""
    import torch

    class Stream:
        cuda_stream = 77
    monkeypatch.setattr(tb, "_raw_stream", None)
    monkeypatch.setattr(torch.cuda, "current_stream", lambda: Stream)
    assert tb._stream() == 77 and tb._stream(Stream) == 77
    monkeypatch.setattr(tb, "_raw_stream", lambda device: 1000 + device)
    monkeypatch.setattr(torch.cuda, "current_device", lambda: 3)
    assert tb._stream() == 1003 and tb._stream(Stream) == 77
