"""GPU parity of the pieces around the layer of Section 3.1, each through the C ABI against the
CPU oracle: the post-training quantised shared expert (Section 4.3), the block of Eq.1-2
(normalisation prologue, residual epilogue), the load-balancing statistic (Eq.12), the 1-bit
routed-expert quantiser (Table 5) and the straight-through gradients of Section 3.2."""
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from oracle import mote_oracle as O
from tests.mote_testlib import GpuProblem, OracleProblem, bits, error_metrics

pytestmark = pytest.mark.gpu

MAX_ABS_TOL = 2e-2          # bf16 output against the oracle's unrounded fp32 output
REL_L2_TOL = 5e-3
# The quantised shared expert sums integer-valued bf16 codes in fp32 and scales afterwards, the
# oracle sums dequantised weights in fp64: the pre-activations agree to about 1e-6 relative, so a
# rounding of h_s to bf16 (half a unit = 2^-9 relative) flips for well under one value in a hundred.
HS_FLIP_RATE = 1e-2


def _m():
    import paper_2506_14435_amd as M
    M.load_library()
    return M


def _log(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------------------ packing
@pytest.mark.parametrize("bits_", [8, 4])
@pytest.mark.parametrize("shape", [(32, 128), (96, 384), (64, 2048), (512, 256)])
def test_pack_rtn_bit_exact(shape, bits_):
    M = _m()
    g = torch.Generator().manual_seed(shape[0] * 7 + shape[1] + bits_)
    w = (torch.randn(*shape, generator=g) * 0.02).to(torch.bfloat16)
    w[3] = 0.0                                         # a zero row: clamped scale, zero codes
    w[5, 7] = 1.0                                      # an outlier that sets its row's scale
    packed, scales = M.mote_pack_rtn(w.cuda(), bits_)
    torch.cuda.synchronize()
    q, s = O.rtn_quantize(W.bf16_bits(w), bits_)
    assert np.array_equal(scales.cpu().numpy(), s)
    assert np.array_equal(packed.cpu().numpy(), O.pack_rtn(q, bits_))
    assert packed.numel() == M.mote_rtn_packed_bytes(*shape, bits_) == O.rtn_packed_bytes(*shape, bits_)


def test_pack_binary_bit_exact():
    M = _m()
    g = torch.Generator().manual_seed(77)
    w = torch.randn(96, 256, generator=g) * 0.02
    w[0, :5] = 0.0                                     # sign(0) = +1
    for t in (w, w.to(torch.bfloat16)):
        packed, alpha = M.mote_pack_ternary(t.cuda(), binary=True)
        torch.cuda.synchronize()
        tb, a = O.binarize(t.float().numpy())
        assert alpha.item() == a
        assert np.array_equal(packed.cpu().numpy().view(np.uint32), O.pack_int2(tb))


def test_layer_with_binary_experts():
    """1-bit routed experts (Table 5) through the unchanged forward: integer stages bit-exact."""
    M = _m()
    cfg = W.MoteConfig("binary_experts", 256, 384, 4, 2, 90, seed=41)
    gp, op = GpuProblem(cfg, binary_experts=True), OracleProblem(cfg, binary_experts=True)
    taps = M.alloc_taps(gp.layer, cfg.n_tokens, ("topk_idx", "row_of", "acc_gate", "acc_up", "acc_down", "q_h"))
    out = M.mote_layer_forward(gp.layer, gp.x, taps=taps)
    torch.cuda.synchronize()
    ref = op.forward()
    flat = taps["row_of"].cpu().numpy().reshape(-1)
    assert np.array_equal(taps["topk_idx"].cpu().numpy(), ref["idx"])
    for n in ("acc_gate", "acc_up"):
        assert np.array_equal(taps[n].cpu().numpy()[flat].reshape(cfg.n_tokens, cfg.top_k, -1), ref[n])
    max_abs, rel_l2 = error_metrics(bits(out), ref["out_f32"])
    _log(f"  binary experts: max-abs-err {max_abs:.3e} rel-L2 {rel_l2:.3e}")
    assert max_abs <= MAX_ABS_TOL and rel_l2 <= REL_L2_TOL


# ------------------------------------------------------------------ load balancing (Eq.12)
@pytest.mark.parametrize("T,d,E,k,bias", [(64, 256, 4, 2, False), (1, 256, 4, 1, False), (300, 384, 8, 2, True),
                                           (2048, 896, 8, 2, False), (5000, 256, 16, 2, True), (333, 128, 33, 3, False),
                                           (8192, 2048, 16, 2, False)])
def test_router_balance_matches_oracle(T, d, E, k, bias):
    M = _m()
    g = torch.Generator().manual_seed(T + d + E)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16)
    wr = (torch.randn(d, E, generator=g) * d ** -0.5).to(torch.bfloat16)
    b = (torch.randn(E, generator=g) * 0.5) if bias else None
    idx, p, counts, gate_p, gate_sum, loss = M.mote_router_balance(x.cuda(), wr.cuda(), k, None if b is None else b.cuda())
    torch.cuda.synchronize()
    _, p_o, idx_o, w_o = O.router(W.bf16_bits(x), W.bf16_bits(wr), None if b is None else b.numpy(), k)
    t_o, s_o, loss_o = O.load_balance(p_o, idx_o)
    assert np.array_equal(idx.cpu().numpy(), idx_o)
    assert np.allclose(p.cpu().numpy(), w_o, rtol=2e-6, atol=1e-9)
    assert np.array_equal(counts.cpu().numpy(), t_o)
    assert np.allclose(gate_p.cpu().numpy(), p_o, rtol=2e-6, atol=1e-9)
    assert np.allclose(gate_sum.cpu().numpy(), s_o, rtol=1e-6)
    assert loss.item() == pytest.approx(loss_o, rel=1e-6)
    # the same routing as the plain router entry point
    idx2, p2, counts2 = M.mote_router_topk(x.cuda(), wr.cuda(), k, None if b is None else b.cuda())
    assert torch.equal(idx, idx2) and torch.equal(p, p2) and torch.equal(counts, counts2)


# column groups of the balance kernel: 16-byte groups that do and do not divide the workgroup, single experts,
# rows that end inside a pass of the workgroup, fewer rows than lanes; eight and sixteen loads in flight (up to 24576
# probabilities or indices, and more)
@pytest.mark.parametrize("T,d,E,k", [(1030, 128, 12, 2), (2050, 128, 64, 8), (3, 128, 64, 1), (1025, 128, 1, 1),
                                     (7, 128, 5, 2), (9000, 128, 4, 2), (4096, 128, 6, 2), (4097, 128, 6, 2), (3073, 128, 8, 8)])
def test_router_balance_column_groups(T, d, E, k):
    M = _m()
    g = torch.Generator().manual_seed(T + E)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16)
    wr = (torch.randn(d, E, generator=g) * d ** -0.5).to(torch.bfloat16)
    idx, p, counts, gate_p, gate_sum, loss = M.mote_router_balance(x.cuda(), wr.cuda(), k)
    torch.cuda.synchronize()
    _, p_o, idx_o, _ = O.router(W.bf16_bits(x), W.bf16_bits(wr), None, k)
    t_o, s_o, loss_o = O.load_balance(p_o, idx_o)
    assert np.array_equal(idx.cpu().numpy(), idx_o) and np.array_equal(counts.cpu().numpy(), t_o)
    # the sums of the GPU's own fp32 probabilities differ from their fp64 sums by one fp32 rounding (2^-24)
    own = gate_p.double().sum(0).cpu().numpy()
    assert (np.abs(gate_sum.cpu().numpy() - own) <= 2.0 ** -23 * own).all()
    assert np.allclose(gate_sum.cpu().numpy(), s_o, rtol=1e-6) and loss.item() == pytest.approx(loss_o, rel=1e-6)


# ------------------------------------------------------------------------- block (Eq.1-2)
def _norm_inputs(cfg, kind, seed):
    g = torch.Generator().manual_seed(seed)
    gamma = (1.0 + 0.1 * torch.randn(cfg.d_model, generator=g)).to(torch.bfloat16)
    beta = (0.05 * torch.randn(cfg.d_model, generator=g)).to(torch.bfloat16) if kind == "layer" else None
    return gamma, beta


BLOCK_CASES = [
    (W.C1, "rms"), (W.C1, "layer"),
    (W.C1.with_tokens(1, name="c1_T1"), "rms"),
    (W.C1.with_tokens(300, name="c1_T300"), "rms"),
    (W.MoteConfig("ragged_mid", 384, 640, 8, 2, 211, seed=11, outlier_channels=2), "layer"),
    (W.MoteConfig("decode_like", 512, 1408, 16, 2, 16, seed=13, bias_kind="subset", bias_subset=4), "rms"),
    (W.MoteConfig("wide_row", 2560, 256, 4, 2, 70, seed=51), "rms"),          # more chunks than threads per row
]


@pytest.mark.parametrize("cfg,kind", BLOCK_CASES, ids=lambda c: getattr(c, "name", str(c)))
def test_block_forward_matches_oracle(cfg, kind):
    """x^a is the workload's x scaled and shifted (an un-normalised hidden state); LN(x^a) bit-exact,
    routing and integer stages on LN(x^a) bit-exact, block output within the layer's tolerances."""
    M = _m()
    _log(f"block {cfg.name} {kind}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    gamma, beta = _norm_inputs(cfg, kind, cfg.seed + 5)
    x_a = (gp.x.float() * 3.0 + 0.25).to(torch.bfloat16)
    op.x = W.bf16_bits(x_a.cpu())
    eps = 1e-6 if kind == "rms" else 1e-5
    names = ("topk_idx", "row_of", "q_x", "beta_x", "acc_gate", "acc_up", "xn", "out_f32")
    taps = M.alloc_taps(gp.layer, cfg.n_tokens, names)
    out = M.mote_block_forward(gp.layer, x_a, gamma.cuda(), None if beta is None else beta.cuda(), eps=eps, taps=taps)
    torch.cuda.synchronize()
    norm = ("rms", W.bf16_bits(gamma), eps) if kind == "rms" else ("layer", W.bf16_bits(gamma), W.bf16_bits(beta), eps)
    ref = op.block_forward(norm)
    assert np.array_equal(bits(taps["xn"]), ref["xn"])
    assert np.array_equal(taps["topk_idx"].cpu().numpy(), ref["idx"])
    assert np.array_equal(taps["q_x"].cpu().numpy(), ref["q_x"])
    flat = taps["row_of"].cpu().numpy().reshape(-1)
    assert np.array_equal(taps["acc_gate"].cpu().numpy()[flat].reshape(cfg.n_tokens, cfg.top_k, -1), ref["acc_gate"])
    assert np.array_equal(bits(out), O.f32_to_bf16(taps["out_f32"].cpu().numpy()))
    max_abs, rel_l2 = error_metrics(bits(out), ref["block_f32"])
    # the residual raises |out|: the final bf16 rounding alone is half a unit in the last place of the largest value
    ulp = 2.0 ** (np.floor(np.log2(np.abs(ref["block_f32"]).max())) - 8)
    _log(f"  max-abs-err {max_abs:.3e} rel-L2 {rel_l2:.3e} max|ref| {np.abs(ref['block_f32']).max():.2f} half-ulp {ulp:.3e}")
    assert max_abs <= MAX_ABS_TOL + ulp and rel_l2 <= REL_L2_TOL
    # without the residual and the norm it is the layer: block(x) - x == layer(LN(x)) up to the one rounding
    lay = M.mote_layer_forward(gp.layer, taps["xn"])
    torch.cuda.synchronize()
    diff = (out.float() - x_a.float() - lay.float()).abs().max().item()
    assert diff <= 4 * ulp + 2e-2


def test_block_forward_rejects_bad_norms():
    import ctypes
    M = _m()
    lib = M.load_library()
    cfg = W.C1
    gp = GpuProblem(cfg)
    ws = gp.layer.workspace(cfg.n_tokens)
    out = torch.empty_like(gp.x)
    B = M.binding
    for norm in (B.MoteNormStruct(0, 256, None, 1e-6), B.MoteNormStruct(1, None, None, 1e-6),
                 B.MoteNormStruct(2, 256, None, 1e-5)):
        rc = lib.mote_block_forward(ctypes.byref(gp.layer.struct), ctypes.byref(norm), ctypes.c_void_p(gp.x.data_ptr()),
                                    cfg.n_tokens, ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(ws.data_ptr()),
                                    ws.numel(), None, None)
        assert rc == 1
    assert lib.mote_block_forward(ctypes.byref(gp.layer.struct), None, ctypes.c_void_p(gp.x.data_ptr()), cfg.n_tokens,
                                  ctypes.c_void_p(out.data_ptr()), ctypes.c_void_p(ws.data_ptr()), ws.numel(), None, None) == 1


# ------------------------------------------------------- quantised shared expert (Section 4.3)
def _check_rtn_layer(cfg, bits_, gp, op, tokens=None):
    M = _m()
    T = cfg.n_tokens
    names = ("topk_idx", "row_of", "acc_gate", "acc_down", "h_s", "y_s", "out_f32")
    taps = M.alloc_taps(gp.layer, T, names)
    out = M.mote_layer_forward(gp.layer, gp.x, taps=taps)
    torch.cuda.synchronize()
    ref = op.forward(tokens=tokens)
    sel = np.arange(T) if tokens is None else np.asarray(tokens)
    sel_t = torch.from_numpy(sel.astype(np.int64)).cuda()
    assert np.array_equal(taps["topk_idx"].cpu().numpy(), ref["idx"])
    hs = bits(taps["h_s"][sel_t])
    neq = hs != ref["h_s"]
    if neq.any():     # a flip moves the value by one bf16 step; sums that cancel to nearly zero keep the fp32
        a = O.bf16_to_f32(hs[neq]).astype(np.float64)          # accumulation error of their terms instead
        b = O.bf16_to_f32(ref["h_s"][neq]).astype(np.float64)
        h_max = np.abs(O.bf16_to_f32(ref["h_s"])).max()
        assert (np.abs(a - b) <= np.maximum(np.abs(a), np.abs(b)) * 2.0 ** -7 + 1e-5 * h_max).all()
    assert neq.mean() <= HS_FLIP_RATE, neq.mean()
    y_s = taps["y_s"][sel_t].cpu().numpy()
    assert np.allclose(y_s, ref["y_s"], rtol=0, atol=2e-3 + 2e-3 * np.abs(ref["y_s"]).max())
    max_abs, rel_l2 = error_metrics(bits(out[sel_t]), ref["out_f32"])
    _log(f"  INT{bits_} shared expert, T={T}: h_s flip rate {neq.mean():.2e}, max-abs-err {max_abs:.3e}, rel-L2 {rel_l2:.3e}")
    assert max_abs <= MAX_ABS_TOL and rel_l2 <= REL_L2_TOL
    return out


RTN_SMALL = [
    W.C1, W.C1.with_tokens(1, name="c1_T1"), W.C1.with_tokens(9, name="c1_T9"), W.C1.with_tokens(24, name="c1_T24"),
    W.C1.with_tokens(64, name="c1_T64"), W.C1.with_tokens(65, name="c1_T65"), W.C1.with_tokens(300, name="c1_T300"),
    W.MoteConfig("ragged_mid", 384, 640, 8, 2, 211, seed=11, outlier_channels=2),
    W.MoteConfig("decode_like", 512, 1408, 16, 2, 16, seed=13, bias_kind="subset", bias_subset=4),
    W.MoteConfig("shared_wider_T9", 256, 384, 4, 2, 9, seed=31, d_ff_shared=640),
    W.MoteConfig("shared_wider_T1100", 256, 512, 4, 2, 1100, seed=33, d_ff_shared=1152),
    W.MoteConfig("decode_wide", 2560, 1280, 8, 2, 12, seed=17),
]


@pytest.mark.parametrize("bits_", [8, 4])
@pytest.mark.parametrize("cfg", RTN_SMALL, ids=lambda c: c.name)
def test_layer_rtn_shared_small(cfg, bits_):
    _log(f"layer {cfg.name} with an INT{bits_} shared expert")
    gp, op = GpuProblem(cfg, shared_bits=bits_), OracleProblem(cfg, shared_bits=bits_)
    # the GPU's packed codes and scales are the oracle's
    for m in range(3):
        q, s = op.shared[2 * m], op.shared[2 * m + 1]
        assert np.array_equal(gp.shared[m].cpu().numpy(), O.pack_rtn(q, bits_))
        assert np.array_equal(gp.shared_scales[m].cpu().numpy(), s)
    out = _check_rtn_layer(cfg, bits_, gp, op)
    M = _m()
    out2 = M.mote_layer_forward(gp.layer, gp.x)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)


@pytest.mark.parametrize("bits_", [8, 4])
@pytest.mark.parametrize("T,n", [(1, 2), (4, 4), (16, 8), (64, 16)])
def test_layer_rtn_shared_config4_decode(T, n, bits_):
    """The decode shape (3B width) with a quantised shared expert: every token against the oracle."""
    cfg = W.decode_config(T, n)
    _log(f"layer {cfg.name} with an INT{bits_} shared expert")
    gp, op = GpuProblem(cfg, shared_bits=bits_), OracleProblem(cfg, shared_bits=bits_)
    _check_rtn_layer(cfg, bits_, gp, op)


@pytest.mark.parametrize("bits_", [8, 4])
def test_layer_rtn_shared_prefill_width_sampled(bits_):
    """3B width, 2048 tokens (the large-batch path: codes expanded to integer-valued bf16, scales in
    the GEMM epilogue): tokens of every 256-row tile of the shared GEMMs, first and last row of each."""
    cfg = dataclasses.replace(W.C3, name=f"c3_T2048_int{bits_}", n_tokens=2048)
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg, shared_bits=bits_), OracleProblem(cfg, shared_bits=bits_)
    tokens = np.unique(np.concatenate([np.arange(0, 2048, 256), np.arange(255, 2048, 256), [1000, 1001]]))
    _check_rtn_layer(cfg, bits_, gp, op, tokens=tokens)


def test_rtn_layer_arguments_are_validated():
    import ctypes
    M = _m()
    lib = M.load_library()
    L = M.binding.MoteLayerStruct(256, 512, 512, 4, 2, *([ctypes.c_void_p(256)] * 1), None, *([ctypes.c_void_p(256)] * 7), 3)
    assert lib.mote_layer_workspace_bytes(ctypes.byref(L), 8) == 0                      # shared_bits must be 0, 8 or 4
    L.shared_bits = 8                                                                    # scales missing
    assert lib.mote_layer_forward(ctypes.byref(L), ctypes.c_void_p(256), 8, ctypes.c_void_p(256), ctypes.c_void_p(256),
                                  1 << 30, None, None) == 1
    assert lib.mote_pack_rtn(ctypes.c_void_p(256), 32, 128, 5, ctypes.c_void_p(256), ctypes.c_void_p(256), None) == 1
    assert lib.mote_pack_rtn(ctypes.c_void_p(256), 33, 128, 8, ctypes.c_void_p(256), ctypes.c_void_p(256), None) == 2
    assert lib.mote_rtn_packed_bytes(32, 128, 5) == 0


# -------------------------------------------------- straight-through gradients (Section 3.2)
def _ste_problem(R, N, K, E, seed, cuts=None):
    """Seeded inputs of one grouped ternary linear layer on its way back: latent weights ~ N(0, 0.02)
    packed on the GPU (the pack is bit-exact against the oracle elsewhere), activations ~ N(0, 1)
    quantised by the oracle's Q_a, gradient rows ~ N(0, 1) in bf16, ragged expert groups."""
    M = _m()
    g = torch.Generator().manual_seed(9000 + seed)
    rng = np.random.default_rng(9000 + seed)
    if cuts is None:
        cuts = np.sort(rng.integers(0, R + 1, E - 1))
    offsets = np.concatenate([[0], np.asarray(cuts, np.int64), [R]]).astype(np.int64)
    latents = [torch.randn(N, K, generator=g) * 0.02 for _ in range(E)]
    packed, alpha = [], []
    for w in latents:
        p, a = M.mote_pack_ternary(w.cuda())
        packed.append(p.view(torch.uint8).reshape(-1))
        alpha.append(a)
    x = torch.randn(R, K, generator=g).numpy()
    q, beta = O.absmax_int8(x)
    dy = torch.randn(R, N, generator=g).to(torch.bfloat16)
    experts = [O.ternarize(w.numpy()) for w in latents]
    return dict(offsets=offsets, packed=torch.cat(packed), alpha=torch.cat(alpha), q=q, beta=beta.reshape(-1), dy=dy,
                experts=experts)


def _ste_tight_bound(terms):
    """terms [n, S]: the products of S sampled outputs in contraction order.  The kernel adds them in
    that order, 16 at a time, in fp32: every rounding is at most 2^-24 of the running sum, which
    stays below the largest prefix sum plus one group of 16 products."""
    n = terms.shape[0]
    running = np.abs(np.cumsum(terms, axis=0)).max(axis=0) + 16.0 * np.abs(terms).max(axis=0)
    return (n / 16 + 4) * 2.0 ** -24 * running + 1e-30


def _ste_check(p, dx, dw, N, K, experts_checked=None, rows_per_expert=None):
    """dx and dw against the oracle.  Every element within the worst-case bound of an fp32 sum of
    exact products (a bf16 value times a ternary value or an int8 code; 2^-24 of sum |terms| per
    rounding), and a sample of outputs within the much tighter bound of the running sum, which is
    far below a single product: a dropped or mis-signed term would show."""
    offsets, dy_bits = p["offsets"], W.bf16_bits(p["dy"])
    E = len(p["experts"])
    for e in (range(E) if experts_checked is None else experts_checked):
        lo, hi = int(offsets[e]), int(offsets[e + 1])
        rng = np.random.default_rng(100 + e)
        rows = np.arange(lo, hi)
        if rows_per_expert is not None and len(rows) > rows_per_expert:
            rows = np.unique(np.concatenate([[lo, hi - 1], rng.choice(rows, rows_per_expert - 2, replace=False)]))
        t, alpha = p["experts"][e]
        # dX on the chosen rows, dW from all rows of the expert
        sub_dx, _, _ = O.ste_linear_backward(dy_bits[rows], [0, len(rows)], [(t, alpha)], p["q"][rows], p["beta"][rows])
        _, sub_dw, dys = O.ste_linear_backward(dy_bits[lo:hi], [0, hi - lo], [(t, alpha)], p["q"][lo:hi], p["beta"][lo:hi])
        got_dw = dw[e].cpu().numpy().astype(np.float64)
        if hi == lo:
            assert not got_dw.any(), f"expert {e} without rows"
            continue
        got_dx = dx[torch.from_numpy(rows).cuda()].cpu().numpy().astype(np.float64)
        g = O.bf16_to_f32(dy_bits[rows]).astype(np.float64)
        a64, t64 = float(alpha), t.astype(np.float64)
        bound_dx = a64 * (np.abs(g) @ np.abs(t64)) * ((N / 16 + 4) * 2.0 ** -24) + 1e-30
        assert (np.abs(got_dx - sub_dx) <= bound_dx).all(), (e, np.abs(got_dx - sub_dx).max())
        gs = O.bf16_to_f32(dys).astype(np.float64)
        q64 = p["q"][lo:hi].astype(np.float64)
        bound_dw = (np.abs(gs).T @ np.abs(q64)) * (((hi - lo) / 16 + 4) * 2.0 ** -24) + 1e-30
        assert (np.abs(got_dw - sub_dw[0]) <= bound_dw).all(), (e, np.abs(got_dw - sub_dw[0]).max())
        # sampled outputs against the bound of the running sum
        n_s = 96
        ri, ci = rng.integers(0, len(rows), n_s), rng.integers(0, K, n_s)
        terms = g[ri].T * t64[:, ci]                                  # [N, n_s]
        tight = a64 * _ste_tight_bound(terms) + np.abs(sub_dx[ri, ci]) * 2.0 ** -23
        assert (np.abs(got_dx[ri, ci] - sub_dx[ri, ci]) <= tight).all(), (e, "dx")
        assert np.median(tight) < 0.05 * a64 * np.median(np.abs(g)), (np.median(tight), a64)
        ni, ci = rng.integers(0, N, n_s), rng.integers(0, K, n_s)
        terms = gs[:, ni] * q64[:, ci]                                # [rows of e, n_s]
        tight = _ste_tight_bound(terms)
        assert (np.abs(got_dw[ni, ci] - sub_dw[0][ni, ci]) <= tight).all(), (e, "dw")
        if hi - lo >= 8:
            assert np.median(tight) < 0.05 * np.median(np.abs(gs)) * np.median(np.abs(q64)), np.median(tight)


@pytest.mark.parametrize("R,N,K,E,cuts", [(300, 256, 128, 3, None), (1000, 512, 384, 4, None),
                                          (77, 128, 256, 5, [0, 10, 10, 64]), (64, 128, 128, 1, None),
                                          (513, 384, 256, 2, [512]),
                                          (200, 128, 128, 3, [120, 200]),          # the last expert without rows
                                          (1018, 256, 256, 4, [256, 506, 762]),    # near-equal: every block padded to the longest
                                          # near-equal and unequal groups (dW: one launch, the experts are its K ranges)
                                          (1024, 256, 256, 4, [250, 510, 770]),
                                          (2100, 128, 384, 8, [300, 600, 900, 900, 1200, 1500, 1800])])
def test_ste_linear_backward_matches_oracle(R, N, K, E, cuts):
    M = _m()
    _log(f"ste backward R={R} N={N} K={K} E={E}")
    p = _ste_problem(R, N, K, E, seed=R + N + K, cuts=cuts)
    dx, dw = M.mote_ste_linear_backward(p["dy"].cuda(), p["offsets"], p["packed"].cuda(), p["alpha"].cuda(), 1,
                                        torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    _ste_check(p, dx, dw, N, K)


def test_ste_linear_backward_3b_gate_matrix_sampled():
    """The gate matrices of configuration 3's width (N = 11008, K = 2048) with eight experts and
    4096 dispatch rows: two experts through the oracle, every row tile boundary of theirs in dX."""
    M = _m()
    R, N, K, E = 4096, 11008, 2048, 8
    _log(f"ste backward R={R} N={N} K={K} E={E}")
    p = _ste_problem(R, N, K, E, seed=77)
    dx, dw = M.mote_ste_linear_backward(p["dy"].cuda(), p["offsets"], p["packed"].cuda(), p["alpha"].cuda(), 1,
                                        torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    sizes = np.diff(p["offsets"])
    chosen = [int(np.argmax(sizes)), int(np.argsort(sizes)[len(sizes) // 2])]
    _ste_check(p, dx, dw, N, K, experts_checked=chosen, rows_per_expert=24)


@pytest.mark.parametrize("R,N,K,E,cuts,what", [
    # 32 row tiles of 256 x 8 channel tiles = one round of workgroups: one K plane
    (7816, 1024, 2048, 4, [1000, 2030, 5030], "one plane"),
    # 34 row tiles x 8 channel tiles = a full round and a nearly empty one: its two row tiles in two K planes, added afterwards
    (8192, 2048, 2048, 8, [1000, 2100, 3100, 4200, 5200, 6150, 7170], "two planes of the last two row tiles")])
def test_ste_linear_backward_grouped_dx_on_256_row_tiles(R, N, K, E, cuts, what):
    """dX of all experts in one grouped GEMM on 256 x 256 tiles: groups that end inside a tile, tiles
    that read the next group's rows, the last tile clamped at R."""
    M = _m()
    _log(f"ste backward, grouped dX on 256-row tiles ({what}) R={R} N={N} K={K} E={E}")
    p = _ste_problem(R, N, K, E, seed=R + N + E, cuts=cuts)
    dx, dw = M.mote_ste_linear_backward(p["dy"].cuda(), p["offsets"], p["packed"].cuda(), p["alpha"].cuda(), 1,
                                        torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    assert torch.isfinite(dx).all()
    _ste_check(p, dx, dw, N, K, experts_checked=[0, 1, E - 1], rows_per_expert=40)


def test_ste_linear_backward_dx_in_batches_of_experts():
    """With the limit on expanded weights per grouped dX launch lowered to 1 MiB the six experts go
    through in batches of two: one batch with an expert without rows, one without any row."""
    M = _m()
    R, N, K, E = 900, 512, 768, 6
    _log(f"ste backward in batches of experts R={R} N={N} K={K} E={E}")
    p = _ste_problem(R, N, K, E, seed=4242, cuts=[0, 400, 400, 400, 700])
    M.mote_tuning_set("ste_batch_mib", 1)
    try:
        dx, dw = M.mote_ste_linear_backward(p["dy"].cuda(), p["offsets"], p["packed"].cuda(), p["alpha"].cuda(), 1,
                                            torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
        torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("ste_batch_mib", 4095)
    _ste_check(p, dx, dw, N, K)


def test_ste_linear_backward_arguments_are_validated():
    M = _m()
    lib = M.load_library()
    import ctypes
    offs = (ctypes.c_int32 * 3)(0, 5, 9)
    buf = torch.zeros(1 << 20, dtype=torch.uint8, device="cuda")
    ptr = ctypes.c_void_p(buf.data_ptr())
    call = lambda o, R, N, K, E, ws_bytes: lib.mote_ste_linear_backward(ptr, o, ptr, ptr, 1, ptr, ptr, R, N, K, E, ptr, ptr, ptr,
                                                                       ctypes.c_size_t(ws_bytes), None)
    assert call(offs, 9, 100, 128, 2, 1 << 20) == 2          # N not a multiple of 128
    assert call(offs, 10, 128, 128, 2, 1 << 20) == 1         # offsets do not end at R
    assert call((ctypes.c_int32 * 3)(0, 9, 5), 5, 128, 128, 2, 1 << 20) == 1   # not ascending
    assert call(offs, 9, 128, 128, 2, 16) == 3               # workspace too small
    assert lib.mote_ste_backward_workspace_bytes(9, 128, 128, 2) > 0
    assert lib.mote_ste_backward_workspace_bytes(9, 100, 128, 2) == 0


# The 2-bit operand of dX: exact sums (integer gradients, sums below 2^24) make every code's place visible.
# 128 channels: half a 256-wide tile; 640: a last tile of half a width, on 256-row tiles; 128 output rows: one
# workgroup of the re-blocking kernel; a group of one row and an empty one; groups whose last 128-row tile has up to 64 rows
# (half of its wavefronts without any) and one more, several such tiles in turn per workgroup.
@pytest.mark.parametrize("R,N,K,E,cuts", [(70, 128, 128, 3, [1, 1]), (300, 384, 640, 2, [130]), (16700, 128, 640, 2, [16600]),
                                          (129, 1408, 256, 4, [0, 64, 128]),
                                          (642, 1024, 5120, 8, [64, 129, 257, 386, 387, 387, 450])])
def test_ste_dx_of_integer_gradients_is_exact(R, N, K, E, cuts):
    M = _m()
    p = _ste_problem(R, N, K, E, seed=77 + R, cuts=cuts)
    dy = torch.randint(-8, 9, (R, N), generator=torch.Generator().manual_seed(R)).float()
    dx, _ = M.mote_ste_linear_backward(dy.to(torch.bfloat16).cuda(), p["offsets"], p["packed"].cuda(), p["alpha"].cuda(), 1,
                                       torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    alpha = p["alpha"].cpu().numpy().reshape(-1)
    for e in range(E):
        a, b = int(p["offsets"][e]), int(p["offsets"][e + 1])
        ref = (dy[a:b].numpy() @ p["experts"][e][0].astype(np.float32)).astype(np.float32)   # |sums| <= 8 N: exact
        assert np.array_equal(dx[a:b].cpu().numpy(), ref * np.float32(alpha[e]))


# The last row tiles in K planes of their own: 36 row tiles of 256 x 8 channel tiles, the last four row tiles (from the
# middle of a group on) in four planes; 33 row tiles, a group of 40 rows in two planes (K steps: 32).  128-row tiles of up to 64
# rows and of 65 in four planes.  All rows of 256-row tiles in two planes, where no whole rounds can be cut off: 21 row tiles x 14
# channel tiles (294 tiles fill two rounds of 256 workgroups to 57 %, twice as many half as long ones three to 77 %) with an empty
# group, and 19 x 16 (59 and 79 %).  Every plane is multiplied by alpha before they are added, so alpha is a power of two here
# and everything stays exact.
@pytest.mark.parametrize("R,N,K,E,cuts", [(8700, 4096, 2048, 3, [2900, 5800]), (8232, 2048, 2048, 3, [0, 8192]),
                                          (150, 4096, 640, 3, [64, 129]),
                                          (5000, 2048, 3584, 4, [700, 2500, 2500]), (4400, 2048, 4096, 2, [300])])
def test_ste_dx_with_the_last_row_tiles_in_planes_is_exact(R, N, K, E, cuts):
    M = _m()
    p = _ste_problem(R, N, K, E, seed=5 + R, cuts=cuts)
    dy = torch.randint(-8, 9, (R, N), generator=torch.Generator().manual_seed(R)).float()
    alpha = torch.full_like(p["alpha"], 2.0 ** -6)
    dx, _ = M.mote_ste_linear_backward(dy.to(torch.bfloat16).cuda(), p["offsets"], p["packed"].cuda(), alpha.cuda(), 1,
                                       torch.from_numpy(p["q"]).cuda(), torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    for e in range(E):
        a, b = int(p["offsets"][e]), int(p["offsets"][e + 1])
        ref = dy[a:b].numpy() @ p["experts"][e][0].astype(np.float32)   # |sums| <= 8 N: exact
        assert np.array_equal(dx[a:b].cpu().numpy(), ref * np.float32(2.0 ** -6))


def test_ste_gradients_of_rows_beyond_32_bit_offsets():
    """Gradient rows of 4.33 GB (each expert's below 2 GiB): the experts of one launch of either GEMM stay below 4 GiB, which
    is as far as its byte offsets reach.  An expert without rows, unequal ones; integer gradients and an activation scale of
    one, so every sum is an integer below 2^24, and exact times a power of two (in K planes too)."""
    M = _m()
    R, N, K, E = 131200, 16512, 128, 9
    cuts = [16400, 32800, 32800, 49200, 65600, 82000, 98400, 114801]
    assert R * N * 2 > 1 << 32
    _log(f"ste backward R={R} N={N} K={K} E={E}")
    offsets = [0, *cuts, R]
    g = torch.Generator(device="cuda").manual_seed(9)
    latent = [torch.randn(N, K, device="cuda", generator=g) * 0.02 for _ in range(E)]
    packed = torch.cat([M.mote_pack_ternary(w)[0] for w in latent])
    alpha = torch.tensor([2.0 ** -(e % 3) for e in range(E)], device="cuda")
    dy = torch.randint(-2, 3, (R, N), dtype=torch.int8, device="cuda", generator=g).to(torch.bfloat16)
    q = torch.randint(-4, 5, (R, K), dtype=torch.int8, device="cuda", generator=g)
    dx, dw = M.mote_ste_linear_backward(dy, offsets, packed, alpha, 1, q,
                                        torch.full((R,), 127.0, device="cuda"), N, K)
    torch.cuda.synchronize()
    for e in range(E):
        a, b = offsets[e], offsets[e + 1]
        t = torch.from_numpy(O.ternarize(latent[e].cpu().numpy())[0].astype(np.float32)).cuda()
        rows = dy[a:b].float()
        assert torch.equal(dx[a:b], (rows @ t) * alpha[e]), e
        assert torch.equal(dw[e], rows.t() @ q[a:b].float()), e


# Sums near both ends of the fp32 range: the contraction and the scale keep the exponents of dy, t and alpha.  Every
# row of dy follows the signs of one channel at 2^120, so its own sum is 2^120 times that channel's number of
# non-zero codes (above 2^127 for more than 128 of 256); every product and partial sum is exact, as is alpha's value.
@pytest.mark.parametrize("alpha", [0.0173, float(np.float32(2.0 ** -126) * np.float32(1 + 2.0 ** -23))])
def test_ste_dx_keeps_the_fp32_range(alpha):
    M = _m()
    R, N, K = 40, 256, 128
    p = _ste_problem(R, N, K, 1, seed=5)
    t = p["experts"][0][0].astype(np.float64)
    own = np.arange(R) % K
    dy = t[:, own].T * 2.0 ** 120
    sums = dy @ t
    mine = sums[np.arange(R), own]
    assert (mine >= 2.0 ** 127).all() and (np.abs(sums) < 2.0 ** 128).all()
    dx, _ = M.mote_ste_linear_backward(torch.from_numpy(dy).to(torch.bfloat16).cuda(), p["offsets"], p["packed"].cuda(),
                                       torch.tensor([alpha], device="cuda"), 1, torch.from_numpy(p["q"]).cuda(),
                                       torch.from_numpy(p["beta"]).cuda(), N, K)
    torch.cuda.synchronize()
    ref = (sums.astype(np.float32) * np.float32(alpha)).astype(np.float32)
    assert np.isfinite(ref).all() and np.array_equal(dx.cpu().numpy(), ref)


# More than 64 tokens through the streaming kernels of a quantised shared expert, 64 at a time: one token in the
# last chunk, whole chunks, a last chunk of few rows, the most tokens a shape takes this way and one more.
@pytest.mark.parametrize("bits_", [8, 4])
@pytest.mark.parametrize("d,F,Ts", [(256, 512, (65, 128, 200, 512, 513)), (896, 4864, (128, 129)), (1536, 8960, (192, 193))])
def test_rtn_shared_expert_streamed_in_chunks_of_64_tokens(d, F, Ts, bits_):
    M = _m()
    for T in Ts:
        cfg = W.MoteConfig(f"rtn_chunks_{d}_{T}", d, F, 4, 1, T, seed=T + d)
        gp, op = GpuProblem(cfg, shared_bits=bits_), OracleProblem(cfg, shared_bits=bits_)
        tokens = None if d == 256 else sorted({0, 63, 64, T // 2, T - 2, T - 1})
        out = _check_rtn_layer(cfg, bits_, gp, op, tokens=tokens)
        # one workspace sized for more tokens serves this batch with the same result
        ws = torch.empty(gp.layer.workspace_bytes(T + 70), dtype=torch.uint8, device="cuda")
        again = M.mote_layer_forward(gp.layer, gp.x, workspace=ws)
        torch.cuda.synchronize()
        assert torch.equal(out, again)


# Kernel launches of a decode step: five with the router, the row quantiser and the dispatch plan inside the large
# kernels, seven with only the plan inside the gate-up kernel, eight otherwise.  Wherever the forward would not fork it
# takes the five: between the batches that fork for their few tokens and those that fork for their work (3B width, T = 17
# to 23; quantised 1.5B width, T = 33 to 38), with the helper stream switched off, and on the static scratch; and in bf16
# wherever the head kernel's workgroups fit two per CU.
LAUNCH_CASES = [(2048, 11008, 4, 0, 16, "", 5), (2048, 11008, 4, 0, 20, "", 5), (2048, 11008, 4, 0, 24, "", 5),
                (2048, 11008, 4, 0, 32, "no_fork", 5), (2048, 11008, 4, 0, 33, "static", 5), (1536, 8960, 4, 8, 33, "", 5),
                (1536, 8960, 4, 4, 64, "", 5), (2048, 11008, 4, 4, 33, "", 8), (256, 512, 17, 0, 8, "", 8),
                (3584, 18944, 4, 0, 1, "", 8), (3584, 18944, 4, 0, 8, "", 8), (2304, 16384, 16, 0, 8, "", 7), (2304, 14592, 4, 0, 8, "", 5), (3584, 18944, 4, 0, 64, "", 8),
                (3584, 18944, 4, 8, 33, "", 7), (3584, 18944, 4, 4, 16, "", 5), (3584, 18944, 4, 4, 33, "", 8),
                (3584, 18944, 4, 8, 64, "no_fork", 5)]


@pytest.mark.parametrize("d,F,E,bits_,T,how,launches", LAUNCH_CASES)
def test_decode_step_kernel_launches(d, F, E, bits_, T, how, launches):
    import ctypes
    M = _m()
    lib = M.load_library()
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(*s, dtype=dtype, device="cuda")
    shared, scales = [z(F, d), z(F, d), z(d, F)], None
    if bits_:
        shared = [z(F * d * bits_ // 8, dtype=torch.uint8) for _ in range(3)]
        scales = tuple(z(n, dtype=torch.float32) for n in (F, F, d))
    layer = M.MoteLayer(z(d, E), *shared, *[z(E, d * F // 16, dtype=torch.int32) for _ in range(3)],
                        z(E, 3, dtype=torch.float32), 1, shared_bits=bits_, shared_scales=scales)
    x, out = z(T, d), z(T, d)
    ws = layer.workspace(T)
    call = lambda: (M.mote_layer_forward_static(layer, x, out) if how == "static"
                    else M.mote_layer_forward(layer, x, out=out, workspace=ws))
    stream, graph, n = torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    try:
        M.mote_tuning_set("no_fork", int(how == "no_fork"))
        with torch.cuda.stream(stream):
            call()                                  # helper stream and kernel attributes exist from here on
            torch.cuda.synchronize()
            handle = ctypes.c_void_p(stream.cuda_stream)
            assert lib.hipStreamBeginCapture(handle, 2) == 0
            call()
            assert lib.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
        assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        assert n.value == launches
    finally:
        M.mote_tuning_set("no_fork", 0)
        if graph:
            lib.hipGraphDestroy(graph)


def _captured_kernels(call):
    """Names of the kernels that call() launches, in no particular order: the kernel nodes of a captured graph."""
    import ctypes

    class Params(ctypes.Structure):      # hipKernelNodeParams
        _fields_ = [("block", ctypes.c_uint * 3), ("extra", ctypes.c_void_p), ("func", ctypes.c_void_p),
                    ("grid", ctypes.c_uint * 3), ("args", ctypes.c_void_p), ("lds", ctypes.c_uint)]
    lib = _m().load_library()
    lib.hipKernelNameRefByPtr.restype = ctypes.c_char_p
    stream, graph, n = torch.cuda.Stream(), ctypes.c_void_p(), ctypes.c_size_t()
    with torch.cuda.stream(stream):
        call()                           # helper stream and kernel attributes exist from here on
        torch.cuda.synchronize()
        handle = ctypes.c_void_p(stream.cuda_stream)
        assert lib.hipStreamBeginCapture(handle, 2) == 0
        call()
        assert lib.hipStreamEndCapture(handle, ctypes.byref(graph)) == 0
    try:
        assert lib.hipGraphGetNodes(graph, None, ctypes.byref(n)) == 0
        nodes = (ctypes.c_void_p * n.value)()
        assert lib.hipGraphGetNodes(graph, nodes, ctypes.byref(n)) == 0
        names = []
        for node in nodes:
            p = Params()
            assert lib.hipGraphKernelNodeGetParams(ctypes.c_void_p(node), ctypes.byref(p)) == 0
            names.append(lib.hipKernelNameRefByPtr(ctypes.c_void_p(p.func), handle).decode())
        return names
    finally:
        lib.hipGraphDestroy(graph)


def _zero_layer(M, d, F, E, k, bits_):
    z = lambda *s, dtype=torch.bfloat16: torch.zeros(*s, dtype=dtype, device="cuda")
    shared, scales = [z(F, d), z(F, d), z(d, F)], None
    if bits_:
        shared = [z(F * d * bits_ // 8, dtype=torch.uint8) for _ in range(3)]
        scales = tuple(z(n, dtype=torch.float32) for n in (F, F, d))
    return M.MoteLayer(z(d, E), *shared, *[z(E, d * F // 16, dtype=torch.int32) for _ in range(3)],
                       z(E, 3, dtype=torch.float32), k, shared_bits=bits_, shared_scales=scales)


# The batches up to which a quantised shared expert's codes are streamed, on both sides of each limit.
@pytest.mark.parametrize("d,F,T,streamed", [(256, 512, 512, True), (256, 512, 513, False), (896, 1024, 384, True),
                                            (896, 1024, 385, False), (1024, 8192, 128, True), (1024, 8192, 129, False),
                                            (1536, 8960, 192, True), (1536, 8960, 193, False), (2304, 14592, 320, True),
                                            (2304, 14592, 321, False)])
def test_quantised_shared_expert_is_streamed_up_to_a_limit_by_shape(d, F, T, streamed):
    M = _m()
    layer = _zero_layer(M, d, F, 8, 1, 8)
    x = torch.zeros(T, d, dtype=torch.bfloat16, device="cuda")
    out, ws = torch.empty_like(x), layer.workspace(T)
    names = _captured_kernels(lambda: M.mote_layer_forward(layer, x, out=out, workspace=ws))
    assert any("shared_qwave_kernel" in n for n in names) == streamed
    assert any("rtn_dequant_kernel" in n for n in names) == (not streamed)


# Rows per expert (T * k / E) up to which a layer with d > 2048 runs on 32-row tiles, on both sides of each limit.
@pytest.mark.parametrize("F,E,k,bits_,T,decode", [(640, 4, 2, 0, 96, True), (640, 4, 2, 8, 98, False), (5760, 4, 1, 0, 112, True),
                                                  (5760, 4, 1, 0, 113, False), (14592, 4, 1, 0, 80, True), (14592, 4, 1, 0, 81, False),
                                                  (14592, 2, 1, 0, 56, True), (14592, 2, 1, 0, 57, False), (14592, 4, 1, 8, 96, True),
                                                  (14592, 4, 1, 8, 97, False), (640, 32, 4, 0, 192, True), (640, 32, 4, 0, 193, False),
                                                  (6144, 64, 8, 0, 128, True), (6144, 64, 8, 0, 129, False), (6144, 64, 8, 4, 192, True)])
def test_tile_height_of_wide_layers(F, E, k, bits_, T, decode):
    M = _m()
    layer = _zero_layer(M, 2304, F, E, k, bits_)
    x = torch.zeros(T, 2304, dtype=torch.bfloat16, device="cuda")
    out, ws = torch.empty_like(x), layer.workspace(T)
    names = _captured_kernels(lambda: M.mote_layer_forward(layer, x, out=out, workspace=ws))
    assert any("routed_decode_kernel" in n for n in names) == decode
    assert any("routed_gemm_kernel" in n for n in names) == (not decode)
