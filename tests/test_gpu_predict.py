"""Query predictor (LN + two-layer MLP, Sec. 3.1) through the C ABI against the fp64 oracle."""
import numpy as np
import pytest
import torch

from gpu_util import DEV, dtype_name, np_of
from paper_2503_07518_amd import binding as tb

pytestmark = pytest.mark.gpu


def make(B, E, hidden, G, Hq, Dimp, dtype, seed):
    g = torch.Generator().manual_seed(seed)
    r = lambda *shape, scale=1.0, shift=0.0: ((torch.randn(shape, generator=g) * scale + shift).to(dtype).to(DEV))
    return dict(h=r(B, E, scale=2.0, shift=0.5), gamma=r(E, shift=1.0, scale=0.2), beta=r(E, scale=0.2),
                W1=r(hidden, E, scale=E ** -0.5), b1=r(hidden, scale=0.3),
                W2=r(G * Hq * Dimp, hidden, scale=hidden ** -0.5), b2=r(G * Hq * Dimp, scale=0.3))


@pytest.mark.parametrize("dtype,B,E,hidden,G,Hq,Dimp", [
    (torch.bfloat16, 1, 4096, 512, 4, 32, 32),   # Llama-3-8B shape, the paper's predictor
    (torch.bfloat16, 5, 4096, 512, 4, 32, 16),   # odd batch: a half-filled batch chunk
    (torch.float32, 3, 1024, 256, 2, 8, 16),
    (torch.float32, 1, 8192, 2048, 1, 4, 8),     # largest supported sizes
    (torch.bfloat16, 2, 64, 8, 3, 2, 8),         # rows shorter than one pass of a wave
    # larger batches: tiles of 16 sequences
    (torch.bfloat16, 16, 4096, 512, 4, 32, 32),  # one full tile of sequences
    (torch.bfloat16, 8, 4096, 512, 4, 32, 32),   # half a tile
    (torch.bfloat16, 20, 1024, 256, 2, 8, 16),   # two tiles per workgroup, the second ragged
    (torch.bfloat16, 45, 512, 64, 1, 4, 16),     # two workgroup groups along the batch
    (torch.bfloat16, 9, 96, 32, 3, 2, 8),        # smallest sizes the tiles divide
    (torch.bfloat16, 16, 4096, 520, 4, 32, 32),  # hidden size not a multiple of 32: ragged last tile and step
    (torch.float32, 16, 1024, 256, 2, 8, 16),    # one full tile of sequences, fp32
])
def test_predict_queries(oracle, dtype, B, E, hidden, G, Hq, Dimp):
    print(f"[case] predictor dtype={dtype} B={B} E={E} hidden={hidden} G={G} Hq={Hq} Dimp={Dimp}", flush=True)
    p = make(B, E, hidden, G, Hq, Dimp, dtype, 21)
    z = torch.full((B, hidden), float("nan"), dtype=torch.float32, device=DEV)
    q_imp = torch.zeros((G, B, Hq, Dimp), dtype=dtype, device=DEV)
    xln = torch.empty((B, E), dtype=torch.float32, device=DEV)
    tb.tb_predict_queries(p["h"], p["gamma"], p["beta"], p["W1"], p["b1"], p["W2"], p["b2"], G, Hq, Dimp, z, xln, q_imp)
    torch.cuda.synchronize()
    dn = dtype_name(p["h"])
    rq, rz = oracle.predict_queries(*(np_of(p[k]) for k in ("h", "gamma", "beta", "W1", "b1", "W2", "b2")), G, Hq, Dimp, dn)
    # hidden activations: fp32 sums of E products after an fp32 LayerNorm
    assert np.abs(np_of(z) - rz).max() <= 2e-4 * max(1.0, np.abs(rz).max())
    got = np_of(q_imp)
    if dn == "bf16":
        g64, r64 = oracle.bf16_to_f64(got), oracle.bf16_to_f64(rq)
        assert np.all(np.abs(g64 - r64) <= 2.0 ** -7 * np.abs(r64) + 2e-3)
        assert np.mean(got == rq) > 0.97  # and nearly always the same bits
    else:
        assert np.abs(got - rq).max() <= 2e-4 * max(1.0, np.abs(rq).max())


@pytest.mark.parametrize("dtype,B,E,hidden,G,Hq,Dimp", [
    (torch.bfloat16, 1, 4096, 512, 1, 8, 16),    # eight slices, summed by the output kernel
    (torch.bfloat16, 2, 4096, 264, 1, 3, 8),     # just past what it sums itself; ragged tiles on both sides
    (torch.bfloat16, 3, 8192, 2048, 1, 4, 8),    # largest sizes: 16 waves, several chunks of steps
    (torch.bfloat16, 17, 1000, 40, 1, 5, 8),     # a second M tile with one row; pieces past E in the last step
    (torch.bfloat16, 33, 264, 520, 2, 4, 16),    # more hidden units than inputs: one slice
    (torch.float32, 1, 5120, 512, 1, 8, 16),
    (torch.float32, 7, 3000, 520, 2, 4, 16),     # ragged last step and slice
    (torch.float32, 33, 64, 8, 3, 2, 8),         # two workgroup groups along the batch, sizes below one step
    # several slices and few hidden activations: more than two sequences still get LN(h)
    (torch.bfloat16, 4, 4096, 128, 1, 4, 8),
    (torch.float32, 3, 2048, 160, 1, 4, 8),
    (torch.bfloat16, 16, 1024, 32, 1, 4, 8),
    (torch.float32, 2, 4096, 128, 1, 4, 8),      # two sequences: summed by the output kernel
    (torch.bfloat16, 1, 2048, 520, 1, 4, 8),     # ... two elements a thread
    (torch.bfloat16, 1, 2048, 1024, 1, 5, 8),    # ... four elements a thread
    (torch.float32, 2, 2304, 1000, 1, 5, 8),     # ... as many as it takes, the last round ragged
    # large batches: two and four tiles of a layer per workgroup, the last ones ragged
    (torch.bfloat16, 520, 264, 520, 1, 67, 8),
    (torch.bfloat16, 1030, 264, 520, 1, 67, 8),
    (torch.float32, 1030, 264, 520, 1, 67, 8),
    (torch.float32, 520, 264, 520, 1, 67, 8),
])
def test_predict_split_layers(oracle, dtype, B, E, hidden, G, Hq, Dimp):
    """Edges of the tiles, steps and slices; z starts 4 bytes off a 16-byte boundary.  Bars of
    test_predict_queries; LN(h) is an fp32 evaluation of a few operations on values of size <= 10."""
    print(f"[case] predictor split dtype={dtype} B={B} E={E} hidden={hidden} G={G} Hq={Hq} Dimp={Dimp}", flush=True)
    p = make(B, E, hidden, G, Hq, Dimp, dtype, 24)
    z = torch.full((B * hidden + 1,), float("nan"), dtype=torch.float32, device=DEV)[1:].view(B, hidden)
    q_imp = torch.zeros((G, B, Hq, Dimp), dtype=dtype, device=DEV)
    xln = torch.full((B, E), float("nan"), dtype=torch.float32, device=DEV)
    tb.tb_predict_queries(p["h"], p["gamma"], p["beta"], p["W1"], p["b1"], p["W2"], p["b2"], G, Hq, Dimp, z, xln, q_imp)
    torch.cuda.synchronize()
    dn = dtype_name(p["h"])
    rq, rz = oracle.predict_queries(*(np_of(p[k]) for k in ("h", "gamma", "beta", "W1", "b1", "W2", "b2")), G, Hq, Dimp, dn)
    # fp32 sums of E products, seen 2e-7 relative to the largest: an eighth of the general bar
    assert np.abs(np_of(z) - rz).max() <= 2.5e-5 * max(1.0, np.abs(rz).max())
    got = np_of(q_imp)
    if dn == "bf16":
        g64, r64 = oracle.bf16_to_f64(got), oracle.bf16_to_f64(rq)
        assert np.all(np.abs(g64 - r64) <= 2.0 ** -7 * np.abs(r64) + 1e-4)
        assert np.mean(got == rq) > 0.97
    else:
        assert np.abs(got - rq).max() <= 2.5e-5 * max(1.0, np.abs(rq).max())
    if B > 2:
        ln = torch.nn.functional.layer_norm(p["h"].double().cpu(), (E,), p["gamma"].double().cpu(), p["beta"].double().cpu(), 1e-5)
        assert (xln.double().cpu() - ln).abs().max() <= 1e-5


@pytest.mark.parametrize("dtype,B", [(torch.bfloat16, 1), (torch.bfloat16, 3), (torch.bfloat16, 20), (torch.float32, 2)])
def test_predict_infinite_weights(oracle, dtype, B):
    """An infinite weight makes the sums it enters infinite (NaN where a hidden activation's argument is
    -inf, by the oracle's formula) and no others.  Its inputs have few bits (beta alone; gelu(20) = 20), so
    that the lower of the three bf16 parts they are split into are 0."""
    print(f"[case] predictor infinite weights dtype={dtype} B={B}", flush=True)
    E, hidden, G, Hq, Dimp = 2048, 64, 1, 4, 8
    p = make(B, E, hidden, G, Hq, Dimp, dtype, 25)
    inf, at = float("inf"), [5, 40, 62, 63]
    p["gamma"][at] = 0.0
    p["W1"][at], p["b1"][at] = 0.0, 20.0
    for where in ("W1", "W2"):
        w = dict(p)
        w[where] = p[where].clone()
        w[where][3, 5], w[where][7, 40], w[where][12, 63] = inf, -inf, inf
        w[where][12, 62] = -inf  # both signs in one row: NaN or infinite, as the signs of the inputs have it
        z = torch.zeros((B, hidden), dtype=torch.float32, device=DEV)
        xln = torch.zeros((B, E), dtype=torch.float32, device=DEV)
        q_imp = torch.zeros((G, B, Hq, Dimp), dtype=dtype, device=DEV)
        tb.tb_predict_queries(w["h"], w["gamma"], w["beta"], w["W1"], w["b1"], w["W2"], w["b2"], G, Hq, Dimp, z, xln, q_imp)
        torch.cuda.synchronize()
        dn = dtype_name(w["h"])
        rq, rz = oracle.predict_queries(*(np_of(w[k]) for k in ("h", "gamma", "beta", "W1", "b1", "W2", "b2")), G, Hq, Dimp, dn)
        pairs = [(np_of(z).astype(np.float64), np.asarray(rz, np.float64))]
        if where == "W2":
            pairs.append(tuple(oracle.bf16_to_f64(x) if dn == "bf16" else np.asarray(x, np.float64) for x in (np_of(q_imp), rq)))
        for got, ref in pairs:
            assert np.array_equal(np.isnan(got), np.isnan(ref))
            assert np.array_equal(got[np.isinf(ref)], ref[np.isinf(ref)]) and not np.isinf(got[~np.isinf(ref)]).any()
        assert not np.isfinite(pairs[-1][1]).all() and np.isfinite(pairs[-1][1]).any()


def test_predicted_slot_feeds_scoring(oracle):
    """Slot s of the predictor's output is laid out as tb_score's q_imp."""
    print("[case] predictor slot -> tb_score", flush=True)
    from gpu_util import gpu_score, score_tolerance
    B, E, hidden, G, Hq, Hkv, Dimp, N = 2, 512, 64, 4, 8, 2, 32, 3000
    p = make(B, E, hidden, G, Hq, Dimp, torch.bfloat16, 22)
    z = torch.empty((B, hidden), dtype=torch.float32, device=DEV)
    q_imp = torch.zeros((G, B, Hq, Dimp), dtype=torch.bfloat16, device=DEV)
    xln = torch.empty((B, E), dtype=torch.float32, device=DEV)
    tb.tb_predict_queries(p["h"], p["gamma"], p["beta"], p["W1"], p["b1"], p["W2"], p["b2"], G, Hq, Dimp, z, xln, q_imp)
    Kimp = (torch.randn((B, Hkv, N, Dimp), generator=torch.Generator().manual_seed(23))).to(torch.bfloat16).to(DEV)
    s = gpu_score(q_imp[2], Kimp, N)
    torch.cuda.synchronize()
    ref = oracle.score(np_of(q_imp[2]), np_of(Kimp), "bf16", 1.0)
    guard = score_tolerance(oracle, np_of(q_imp[2]), np_of(Kimp), "bf16", 1.0, Hq // Hkv)
    assert np.all(np.abs(np_of(s)[:, :, :N] - ref) <= 1e-4 * np.abs(ref) + guard)
