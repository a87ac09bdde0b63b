"""GPU parity: the HIP path (through the C ABI) against the CPU oracle, element by element
on the same seeded inputs.

Bar: bit-exact for router indices, dispatch order, packed weights, int8 codes and int32
accumulators; bf16 layer output within max-abs-err <= 2e-2 and rel-L2 <= 5e-3 of the
oracle's unrounded fp32 output.  Integer parity is stage-wise: the SwiGLU feeds a
quantiser, and the kernel's exp/divide differ from the oracle's in the last fp32 bit, so a
rare bf16 rounding of h flips; q_h and the down accumulators are therefore checked bit-exact
against the oracle applied to the GPU's own h, and h itself against the oracle's h with a
bounded flip rate."""
import ctypes
import dataclasses

import numpy as np
import pytest
import torch

import workloads as W
from oracle import mote_oracle as O
from tests.mote_testlib import GpuProblem, OracleProblem, bits, error_metrics

pytestmark = pytest.mark.gpu

MAX_ABS_TOL = 2e-2
REL_L2_TOL = 5e-3
H_FLIP_RATE = 1e-3


def _m():
    import paper_2506_14435_amd as M
    return M


def _log(msg):
    print(msg, flush=True)


# ------------------------------------------------------------------------------- pack
@pytest.mark.parametrize("shape,dtype", [((32, 128), "f32"), ((96, 384), "f32"), ((512, 256), "f32"),
                                         ((256, 512), "bf16"), ((4864, 896), "f32"), ((896, 4864), "f32")])
def test_pack_ternary_bit_exact(shape, dtype):
    M = _m()
    _log(f"pack {shape} {dtype}")
    g = torch.Generator().manual_seed(shape[0] * 7 + shape[1])
    w = torch.randn(*shape, generator=g) * 0.02
    if dtype == "bf16":
        wt = w.to(torch.bfloat16)
        w_np = O.bf16_to_f32(W.bf16_bits(wt))
    else:
        wt, w_np = w, w.numpy()
    packed, alpha = M.mote_pack_ternary(wt.cuda())
    t, a = O.ternarize(w_np)
    assert alpha.cpu().numpy()[0] == a
    want = O.pack_int2(t)
    got = packed.cpu().numpy().view(np.uint32)
    assert got.nbytes == M.mote_packed_bytes(*shape) == O.packed_bytes(*shape)
    assert np.array_equal(got, want)


def test_pack_ternary_degenerate_matrices():
    M = _m()
    packed, alpha = M.mote_pack_ternary(torch.zeros(64, 256, device="cuda"))
    assert alpha.item() == np.float32(1e-5)
    assert (packed.cpu().numpy().view(np.uint32) == 0x55555555).all()
    # exact ties in both directions and a constant matrix
    w = torch.tensor([0.75, -0.75, 0.25, -0.25]).repeat(32, 32)
    packed, alpha = M.mote_pack_ternary(w.cuda())
    t, a = O.ternarize(w.numpy())
    assert alpha.item() == a == np.float32(0.5)
    assert np.array_equal(packed.cpu().numpy().view(np.uint32), O.pack_int2(t))
    w = torch.full((32, 128), -3.0)
    packed, alpha = M.mote_pack_ternary(w.cuda())
    assert alpha.item() == 3.0 and (packed.cpu().numpy().view(np.uint32) == 0).all()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("shape", [(32, 128), (64, 384), (160, 2048)])
def test_pack_ternary_at_the_rounding_threshold(shape, dtype):
    """Weights within 64 units in the last place of alpha / 2 on both sides (fp32; the few nearest bf16
    values else): every code must be what the rounded division gives, and every position of a tile is hit."""
    M = _m()
    rng = np.random.default_rng(shape[0] + shape[1])
    n = shape[0] * shape[1]
    a = np.float32(0.0173)
    if dtype == "f32":
        half = (np.float32(a / 2).view(np.int32) + rng.integers(-64, 65, n // 2).astype(np.int32)).view(np.float32)
    else:
        half = ((np.float32(a / 2).view(np.int32) >> 16) + rng.integers(-2, 3, n // 2).astype(np.int32) << 16).view(np.float32)
    w = np.concatenate([half, (2 * a - half).astype(np.float32)]) * rng.choice(np.float32([-1, 1]), n)   # mean |w| = a
    wt = torch.from_numpy(rng.permutation(w).reshape(shape)).to(torch.bfloat16 if dtype == "bf16" else torch.float32)
    packed, alpha = M.mote_pack_ternary(wt.cuda())
    t, al = O.ternarize(wt.float().numpy())
    assert alpha.item() == al
    assert (t[np.abs(wt.float().numpy()) < a] == 0).any() and (np.abs(t[np.abs(wt.float().numpy()) < a]) == 1).any()
    assert np.array_equal(packed.cpu().numpy().view(np.uint32), O.pack_int2(t))


# ----------------------------------------------------------------------------- router
@pytest.mark.parametrize("T,d,E,k,bias", [(64, 256, 4, 2, False), (1, 256, 4, 1, False), (37, 384, 8, 2, True),
                                          (515, 896, 8, 2, False), (130, 2048, 16, 2, True),
                                          (33, 256, 6, 3, False), (70, 512, 32, 4, True), (9, 128, 64, 8, False),
                                          (16, 128, 16, 16, False),
                                          # above 1024 tokens (256 for d <= 1024), E <= 16: 16 tokens per workgroup on the
                                          # fp64 matrix instruction (ragged last workgroup; E not a multiple of 8; a last
                                          # block of 128 channels; the widest register variant), the kernels on
                                          # either side of both limits, and wider rows of many tokens
                                          (4099, 384, 6, 3, True), (4112, 896, 8, 2, True), (4100, 3584, 16, 2, False),
                                          (4096, 128, 16, 1, False), (4097, 4096, 2, 2, True), (4200, 256, 16, 8, False),
                                          (256, 896, 8, 2, False), (257, 1024, 12, 2, True), (1024, 1152, 16, 2, False),
                                          (1025, 1152, 16, 2, True), (2049, 4224, 13, 2, False)])
def test_router_topk_matches_oracle(T, d, E, k, bias):
    M = _m()
    _log(f"router T={T} d={d} E={E} k={k} bias={bias}")
    cfg = W.MoteConfig("router_case", d, 128, E, min(k, 8), T, seed=100 + T + E)
    k = min(k, 8)
    x, wr = W.make_x(cfg), W.make_router(cfg)
    b = None
    if bias:
        b = torch.randn(E, generator=torch.Generator().manual_seed(E)) * 2.0
    idx, p, counts = M.mote_router_topk(x.cuda(), wr.cuda(), k, None if b is None else b.cuda())
    torch.cuda.synchronize()
    logits, p_all, idx_o, w_o = O.router(W.bf16_bits(x), W.bf16_bits(wr), None if b is None else b.numpy(), k)
    srt = np.sort(logits, axis=1)[:, ::-1]
    assert np.diff(srt[:, : k + 1], axis=1).max() < -1e-9      # no near-ties in this seeded case
    assert np.array_equal(idx.cpu().numpy(), idx_o)
    assert np.allclose(p.cpu().numpy(), w_o, rtol=2e-6, atol=1e-9)
    assert np.array_equal(counts.cpu().numpy(), np.bincount(idx_o.ravel(), minlength=E))


def test_router_exact_ties_lower_index_and_empty_batch():
    M = _m()
    cfg = W.MoteConfig("tie_case", 256, 128, 4, 2, 19, seed=5)
    x = W.make_x(cfg)
    col = W.make_router(cfg)[:, :1]
    wr = col.repeat(1, 4).contiguous()
    idx, p, _ = M.mote_router_topk(x.cuda(), wr.cuda(), 2)
    assert (idx.cpu().numpy() == np.array([0, 1])).all()
    assert np.allclose(p.cpu().numpy(), 0.25, rtol=1e-6)
    idx, p, _ = M.mote_router_topk(x[:0].cuda(), wr.cuda(), 2)
    assert idx.shape == (0, 2)


def test_router_non_finite_hidden_states_select_valid_experts():
    """NaN and infinite logits (from non-finite hidden states) still select k distinct experts
    below E: an index beyond E would send the later stages out of bounds.  Only the router entry
    point runs here; it writes the k indices per token and reads nothing through them."""
    M = _m()
    for E, k in ((2, 2), (4, 2), (5, 3), (16, 2), (3, 3)):
        d = 256
        g = torch.Generator().manual_seed(40 + E)
        x = torch.randn(6, d, generator=g).to(torch.bfloat16)
        wr = (torch.randn(d, E, generator=g) * d ** -0.5).to(torch.bfloat16)
        x[1, 3] = float("nan")
        x[2, 7] = float("inf")
        x[3, 9] = float("-inf")
        x[4, :] = float("nan")
        bias = torch.zeros(E)
        bias[E - 1] = float("nan")
        for b in (None, bias.cuda()):
            idx, p, _ = M.mote_router_topk(x.cuda(), wr.cuda(), k, router_bias=b, want_counts=False)
            idx = idx.cpu().numpy()
            assert idx.min() >= 0 and idx.max() < E, (E, k, idx)
            assert all(len(set(row)) == k for row in idx.tolist()), (E, k, idx)
        # finite tokens are untouched by their neighbours
        ref = O.router(W.bf16_bits(x[:1]), W.bf16_bits(wr), None, k)
        idx, p, _ = M.mote_router_topk(x.cuda(), wr.cuda(), k, want_counts=False)
        assert np.array_equal(idx.cpu().numpy()[:1], ref[2])


def test_router_non_finite_hidden_states_many_tokens():
    """The same on the kernel of many tokens (above 256 at this width): a non-finite token touches neither
    its 15 neighbours in the accumulator tile nor the range of the indices."""
    M = _m()
    T, d, E, k = 4100, 256, 5, 3
    g = torch.Generator().manual_seed(77)
    x = torch.randn(T, d, generator=g).to(torch.bfloat16)
    wr = (torch.randn(d, E, generator=g) * d ** -0.5).to(torch.bfloat16)
    bad = [1, 17, 18, 4097]
    x[1, 3] = float("nan")
    x[17, 7] = float("inf")
    x[18, 9] = float("-inf")
    x[4097, :] = float("nan")
    idx, p, _ = M.mote_router_topk(x.cuda(), wr.cuda(), k, want_counts=False)
    idx, p = idx.cpu().numpy(), p.cpu().numpy()
    assert idx.min() >= 0 and idx.max() < E
    assert all(len(set(row)) == k for row in idx[bad].tolist())
    good = np.setdiff1d(np.arange(T), bad)
    _, _, idx_o, w_o = O.router(W.bf16_bits(x[good]), W.bf16_bits(wr), None, k)
    assert np.array_equal(idx[good], idx_o)
    assert np.allclose(p[good], w_o, rtol=2e-6, atol=1e-9)


# ------------------------------------------------------------------------ whole layer
def _run_layer(gp, taps_names):
    M = _m()
    T = gp.x.shape[0]
    taps = M.alloc_taps(gp.layer, T, taps_names)
    for t in taps.values():
        t.zero_()
    out = M.mote_layer_forward(gp.layer, gp.x, taps=taps)
    torch.cuda.synchronize()
    return out, taps


def _check_stagewise(cfg, gp, op, ref, out, taps):
    """Full stage-wise comparison for cases where the oracle evaluates every token."""
    T, k, E = cfg.n_tokens, cfg.top_k, cfg.n_experts
    R = T * k
    # routing and dispatch order: bit-exact
    assert np.array_equal(taps["topk_idx"].cpu().numpy(), ref["idx"])
    assert np.allclose(taps["topk_p"].cpu().numpy(), ref["w"], rtol=2e-6, atol=1e-9)
    assert np.array_equal(taps["counts"].cpu().numpy(), ref["counts"])
    row_of = taps["row_of"].cpu().numpy()
    assert np.array_equal(row_of, ref["row_of"])
    assert np.array_equal(taps["tok_of"].cpu().numpy(), ref["tok_of"])
    # Q_a(x): bit-exact
    assert np.array_equal(taps["q_x"].cpu().numpy(), ref["q_x"])
    assert np.array_equal(taps["beta_x"].cpu().numpy(), ref["beta_x"])
    # gate / up accumulators: bit-exact (dispatch-row order on the GPU, [t, j] in the oracle)
    flat = row_of.reshape(-1)
    acc_gate = taps["acc_gate"].cpu().numpy()[flat].reshape(T, k, -1)
    acc_up = taps["acc_up"].cpu().numpy()[flat].reshape(T, k, -1)
    assert np.array_equal(acc_gate, ref["acc_gate"])
    assert np.array_equal(acc_up, ref["acc_up"])
    # h: identical up to rare one-step bf16 rounding flips
    h_gpu = bits(taps["h"])                                           # [R, F]
    h_ref = ref["h"].reshape(R, -1)
    h_g = h_gpu[flat]
    neq = h_g != h_ref
    flip_rate = neq.mean()
    if neq.any():
        a = O.bf16_to_f32(h_g[neq]).astype(np.float64)
        b = O.bf16_to_f32(h_ref[neq]).astype(np.float64)
        assert (np.abs(a - b) <= np.maximum(np.abs(a), np.abs(b)) * 2.0 ** -7 + 1e-30).all()
    assert flip_rate <= H_FLIP_RATE, flip_rate
    # Q_a(h) from the GPU's own h: bit-exact
    q_h_want, beta_h_want = O.absmax_int8(O.bf16_to_f32(h_gpu))
    q_h = taps["q_h"].cpu().numpy()
    assert np.array_equal(q_h, q_h_want)
    assert np.array_equal(taps["beta_h"].cpu().numpy(), beta_h_want[:, 0])
    # down accumulators from the GPU's own q_h: bit-exact
    acc_down = taps["acc_down"].cpu().numpy()
    tok_of = ref["tok_of"]
    offs = np.concatenate([[0], np.cumsum(ref["counts"])])
    for e in range(E):
        lo, hi = offs[e], offs[e + 1]
        if hi > lo:
            t_down = op.experts(e)[4]
            assert np.array_equal(acc_down[lo:hi], O.ternary_matmul_int(t_down, q_h[lo:hi])), f"expert {e}"
    # end-to-end q_h mismatch against the oracle's own chain: bounded
    qh_ref = ref["q_h"].reshape(R, -1)
    dq = np.abs(q_h[flat].astype(np.int32) - qh_ref.astype(np.int32))
    _log(f"  h flip rate {flip_rate:.2e}; q_h mismatch rate {np.mean(dq != 0):.2e}, max |dq| {dq.max()}")
    # shared expert
    hs_neq = (bits(taps["h_s"]) != ref["h_s"]).mean()
    assert hs_neq <= 5e-3, hs_neq
    assert np.allclose(taps["y_s"].cpu().numpy(), ref["y_s"], rtol=0, atol=2e-3 + 2e-3 * np.abs(ref["y_s"]).max())
    # output
    out_f32 = taps["out_f32"].cpu().numpy()
    assert np.array_equal(bits(out), O.f32_to_bf16(out_f32))           # the final rounding is RNE
    max_abs, rel_l2 = error_metrics(bits(out), ref["out_f32"])
    _log(f"  out: max-abs-err {max_abs:.3e} rel-L2 {rel_l2:.3e} max|ref| {np.abs(ref['out_f32']).max():.3f}")
    assert np.abs(ref["out_f32"]).max() < 8.0
    assert max_abs <= MAX_ABS_TOL and rel_l2 <= REL_L2_TOL


SMALL_CASES = [
    W.C1,
    W.C1.with_tokens(1, name="c1_T1"),
    W.C1.with_tokens(5, name="c1_T5"),
    W.C1.with_tokens(33, name="c1_T33"),
    W.C1.with_tokens(131, name="c1_T131"),
    W.C1.with_tokens(300, name="c1_T300"),
    dataclasses.replace(W.C1, name="paper_shape_top1", top_k=1, n_tokens=77),        # Section 4.1: E=4, top-1
    dataclasses.replace(W.C1, name="k_equals_E", top_k=4, n_tokens=40),              # Eq.4 as written (dense sum)
    dataclasses.replace(W.C1, name="single_expert", n_experts=1, top_k=1, n_tokens=50),
    W.MoteConfig("ragged_mid", 384, 640, 8, 2, 211, seed=11, outlier_channels=2),
    W.MoteConfig("e16_skew", 256, 384, 16, 2, 500, seed=12, bias_kind="zipf", zipf_tau=0.8),
    W.MoteConfig("decode_like", 512, 1408, 16, 2, 16, seed=13, bias_kind="subset", bias_subset=4),
    W.C1.with_tokens(24, name="c1_T24"),                                              # 17..32 tokens: its own shared decode variant
    W.MoteConfig("decode_wide", 2560, 1280, 8, 2, 12, seed=17),                     # decode with d > 2048: register-ring gate-up kernel
    W.MoteConfig("one_k_step", 128, 256, 4, 2, 200, seed=14),                        # d = 128: a single 128-channel K step
    # about 75 rows per expert: just above the decode kernels' range, 128-row tiles mostly half empty
    W.MoteConfig("rows75", 512, 640, 8, 2, 300, seed=20),
    W.MoteConfig("rows75_skew_wide", 1024, 2048, 16, 2, 600, seed=21, bias_kind="zipf", zipf_tau=0.5),
    W.MoteConfig("e64_k8", 256, 256, 64, 8, 100, seed=18),                           # the largest expert count and top-k the library takes
    W.MoteConfig("e32_k4_large_batch", 256, 384, 32, 4, 1200, seed=19, bias_kind="zipf", zipf_tau=0.6),   # 64-expert router variant, large-batch kernels, empty experts likely
    # 34 row tiles x 64 channel tiles on 512 workgroups: the gate-up tiles are drawn from the
    # counters (and taken from other XCDs' lists at the end); every output is checked
    W.MoteConfig("drawn_tiles", 256, 8192, 4, 2, 2048, seed=15),
    # 76 row tiles x 8 channel tiles of the down projection on 512 workgroups with fixed shares:
    # the 8-16 pairs left for the last round of each XCD's list are cut into two K planes
    W.MoteConfig("split_last_round", 2048, 2048, 8, 2, 4608, seed=16),
    # shared and routed experts of different hidden widths (the boundary keeps two fields): decode
    # kernels, mid-size and large-batch kernels
    W.MoteConfig("shared_wider_T9", 256, 384, 4, 2, 9, seed=31, d_ff_shared=640),
    W.MoteConfig("shared_narrower_T150", 384, 640, 8, 2, 150, seed=32, d_ff_shared=256),
    W.MoteConfig("shared_wider_T1100", 256, 512, 4, 2, 1100, seed=33, d_ff_shared=1152),
]


@pytest.mark.parametrize("cfg", SMALL_CASES, ids=lambda c: c.name)
def test_layer_stagewise_small(cfg):
    _log(f"layer {cfg.name} T={cfg.n_tokens} d={cfg.d_model} F={cfg.d_ff} E={cfg.n_experts} k={cfg.top_k}")
    M = _m()
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, M.TAP_FIELDS)
    ref = op.forward()
    _check_stagewise(cfg, gp, op, ref, out, taps)
    # determinism: a second run is bit-identical
    out2 = M.mote_layer_forward(gp.layer, gp.x)
    torch.cuda.synchronize()
    assert torch.equal(out, out2)


@pytest.mark.parametrize("T", [3, 64, 300, 2048])
def test_dispatch_plan_follows_the_input_on_a_reused_workspace(T):
    """Alternating two inputs on one workspace, the dispatch plan of every call is the stable
    expert-major order of that call's own top-k indices (nothing of the call before survives in
    the plan arrays, counters or caches)."""
    M = _m()
    cfg = W.C1.with_tokens(T, name=f"c1_T{T}")
    _log(f"plan on reused workspace {cfg.name}")
    gp = GpuProblem(cfg)
    xs = [gp.x.clone(), gp.x.flip(0).contiguous() * 0.5 + gp.x * 0.5]
    seen = []
    for it in range(6):
        x = xs[it & 1]
        taps = M.alloc_taps(gp.layer, T, ("topk_idx", "counts", "row_of", "tok_of"))
        M.mote_layer_forward(gp.layer, x, taps=taps)
        torch.cuda.synchronize()
        idx = taps["topk_idx"].cpu().numpy().reshape(-1)
        order = np.argsort(idx, kind="stable")
        row_of = np.empty_like(order)
        row_of[order] = np.arange(order.size)
        assert np.array_equal(taps["row_of"].cpu().numpy().reshape(-1), row_of), it
        assert np.array_equal(taps["tok_of"].cpu().numpy(), order // cfg.top_k), it
        assert np.array_equal(taps["counts"].cpu().numpy(), np.bincount(idx, minlength=cfg.n_experts)), it
        seen.append(idx)
    assert np.array_equal(seen[0], seen[2]) and np.array_equal(seen[1], seen[3])
    if T > 3:
        assert not np.array_equal(seen[0], seen[1])


def _random_config(seed):
    rng = np.random.default_rng(1000 + seed)
    d = int(rng.choice([128, 256, 384, 512, 640, 1024]))
    f = int(rng.choice([128, 256, 384, 640, 896, 1152]))
    e = int(rng.integers(1, 17))
    k = int(rng.integers(1, min(e, 4) + 1))
    t = int(rng.choice([1, 2, 3, 7, 17, 40, 65, 129, 260, 511, 700]))
    kind = ["none", "zipf", "subset"][int(rng.integers(0, 3))]
    kw = {}
    if kind == "zipf":
        kw = dict(bias_kind="zipf", zipf_tau=float(rng.uniform(0.3, 1.0)))
    elif kind == "subset" and e > 1:
        kw = dict(bias_kind="subset", bias_subset=int(rng.integers(max(k, 1), e + 1)))
    return W.MoteConfig(f"random_{seed}_d{d}_F{f}_E{e}_k{k}_T{t}_{kind}", d, f, e, k, t, seed=200 + seed, **kw)


@pytest.mark.parametrize("seed", range(40))
def test_layer_random_shapes(seed):
    """Seeded random small shapes (widths, expert counts, top-k, batch sizes from one token to a few
    hundred, uniform / skewed / restricted routing): every output against the oracle, stage by stage."""
    cfg = _random_config(seed)
    _log(f"layer {cfg.name}")
    M = _m()
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, M.TAP_FIELDS)
    _check_stagewise(cfg, gp, op, op.forward(), out, taps)


def test_layer_pack_parity_config1_all_experts():
    cfg = W.C1
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    for e in range(cfg.n_experts):
        ex = op.experts(e)
        for m in range(3):
            assert np.array_equal(gp.wt[m][e].cpu().numpy().view(np.uint32), O.pack_int2(ex[2 * m]))
            assert gp.alpha[e, m].item() == ex[2 * m + 1]


def test_layer_zero_token_and_zero_rows_are_handled():
    M = _m()
    cfg = W.C1.with_tokens(8, name="c1_T8")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out = M.mote_layer_forward(gp.layer, gp.x[:0].contiguous())
    assert out.shape == (0, cfg.d_model)
    # an all-zero token: beta clamps to 1e-5, routed part is zero, output = shared(0) = 0
    gp.x[3].zero_()
    op.x[3] = 0
    out, taps = _run_layer(gp, M.TAP_FIELDS)
    ref = op.forward()
    _check_stagewise(cfg, gp, op, ref, out, taps)
    assert not bits(out)[3].any() or np.abs(O.bf16_to_f32(bits(out)[3])).max() == 0


@pytest.mark.parametrize("cfg", [W.C1, W.C1.with_tokens(300, name="c1_T300")], ids=lambda c: c.name)
def test_layer_each_tap_is_optional_on_its_own(cfg):
    """Every member of the tap struct may be NULL independently of the others (small-batch and
    large-batch kernel families)."""
    M = _m()
    _log(f"single taps {cfg.name}")
    gp = GpuProblem(cfg)
    out_all, taps_all = _run_layer(gp, M.TAP_FIELDS)
    for name in M.TAP_FIELDS:
        out, taps = _run_layer(gp, (name,))
        assert torch.equal(out, out_all), name
        assert torch.equal(taps[name], taps_all[name]), name


# ------------------------------------------------- full-size configurations (sampled)
def _sample_tokens(ref_router, experts_allowed, n_max, seed):
    idx = ref_router
    ok = np.isin(idx, experts_allowed).all(axis=1)
    cand = np.flatnonzero(ok)
    rng = np.random.default_rng(seed)
    if len(cand) > n_max:
        cand = np.sort(rng.choice(cand, n_max, replace=False))
    return cand


def _check_sampled(cfg, n_sample, n_allowed_experts, out, taps, op):
    """Full-size run: routing / dispatch / Q_a(x) for all tokens, experts on sampled tokens."""
    T, k, E = cfg.n_tokens, cfg.top_k, cfg.n_experts
    logits, _, idx_o, w_o = O.router(op.x, op.w_router, op.bias, k)
    srt = np.sort(logits, axis=1)[:, ::-1]
    margin = -np.diff(srt[:, : min(k + 1, E)], axis=1).max()
    _log(f"  smallest top-k margin {margin:.3e}")
    assert margin > 1e-9
    assert np.array_equal(taps["topk_idx"].cpu().numpy(), idx_o)
    assert np.allclose(taps["topk_p"].cpu().numpy(), w_o, rtol=2e-6, atol=1e-9)
    counts, row_of_o, tok_of_o = O.dispatch_order(idx_o, E)
    _log(f"  expert loads {counts.tolist()}")
    assert np.array_equal(taps["counts"].cpu().numpy(), counts)
    row_of = taps["row_of"].cpu().numpy()
    assert np.array_equal(row_of, row_of_o)
    assert np.array_equal(taps["tok_of"].cpu().numpy(), tok_of_o)
    q_x_o, beta_x_o = O.absmax_int8(O.bf16_to_f32(op.x))
    assert np.array_equal(taps["q_x"].cpu().numpy(), q_x_o)
    assert np.array_equal(taps["beta_x"].cpu().numpy(), beta_x_o[:, 0])
    # experts with the largest loads are the ones the oracle evaluates
    allowed = np.argsort(-counts, kind="stable")[:n_allowed_experts]
    tokens = _sample_tokens(idx_o, allowed, n_sample, seed=cfg.seed)
    assert len(tokens) >= min(8, T)
    ref = op.forward(tokens=tokens)
    rows = row_of[tokens].reshape(-1)
    rows_t = torch.from_numpy(rows.astype(np.int64)).cuda()
    acc_gate = taps["acc_gate"][rows_t].cpu().numpy().reshape(len(tokens), k, -1)
    acc_up = taps["acc_up"][rows_t].cpu().numpy().reshape(len(tokens), k, -1)
    assert np.array_equal(acc_gate, ref["acc_gate"])
    assert np.array_equal(acc_up, ref["acc_up"])
    h_g = bits(taps["h"][rows_t])
    flip = (h_g != ref["h"].reshape(len(rows), -1)).mean()
    assert flip <= H_FLIP_RATE, flip
    q_h_want, beta_h_want = O.absmax_int8(O.bf16_to_f32(h_g))
    q_h = taps["q_h"][rows_t].cpu().numpy()
    assert np.array_equal(q_h, q_h_want)
    assert np.array_equal(taps["beta_h"][rows_t].cpu().numpy(), beta_h_want[:, 0])
    acc_down = taps["acc_down"][rows_t].cpu().numpy()
    e_of_row = idx_o[tokens].reshape(-1)
    for e in np.unique(e_of_row):
        sel = np.flatnonzero(e_of_row == e)
        assert np.array_equal(acc_down[sel], O.ternary_matmul_int(op.experts(int(e))[4], q_h[sel])), f"expert {e}"
    tok_t = torch.from_numpy(tokens.astype(np.int64)).cuda()
    max_abs, rel_l2 = error_metrics(bits(out[tok_t]), ref["out_f32"])
    _log(f"  {len(tokens)} sampled tokens over experts {sorted(allowed.tolist())}: h flip rate {flip:.2e}, "
         f"max-abs-err {max_abs:.3e}, rel-L2 {rel_l2:.3e}, max|ref| {np.abs(ref['out_f32']).max():.3f}")
    assert np.abs(ref["out_f32"]).max() < 8.0
    assert max_abs <= MAX_ABS_TOL and rel_l2 <= REL_L2_TOL
    return ref


def _check_down_rows(cfg, op, taps, rows):
    """Down accumulators of the given dispatch rows against W_down . q_h (exact), whatever tile or K plane computed them."""
    k = cfg.top_k
    row_of = taps["row_of"].cpu().numpy().reshape(-1)
    idx = taps["topk_idx"].cpu().numpy().reshape(-1)
    flat_of_row = np.empty_like(row_of)
    flat_of_row[row_of] = np.arange(row_of.size)
    e_of_row = idx[flat_of_row[rows]]
    rows_t = torch.from_numpy(rows.astype(np.int64)).cuda()
    q_h = taps["q_h"][rows_t].cpu().numpy()
    acc_down = taps["acc_down"][rows_t].cpu().numpy()
    for e in np.unique(e_of_row):
        sel = np.flatnonzero(e_of_row == e)
        assert np.array_equal(acc_down[sel], O.ternary_matmul_int(op.experts(int(e))[4], q_h[sel])), f"expert {e}"


def _check_rows_of_every_expert(cfg, op, taps, tile_m=128, keep=()):
    """Full-size run: for EVERY expert, dispatch rows of its first, a middle and its last row tile
    (first and last row of each) go through the oracle's ternary expert: gate / up accumulators
    bit-exact, h up to rare one-step flips, Q_a(h) bit-exact on the GPU's own h, down accumulators
    bit-exact on the GPU's own q_h.  One expert is ternarised at a time."""
    E = cfg.n_experts
    counts = taps["counts"].cpu().numpy()
    tok_of = taps["tok_of"].cpu().numpy()
    offs = np.concatenate([[0], np.cumsum(counts)])
    x = O.bf16_to_f32(op.x)
    seen = []
    for e in range(E):
        n = int(counts[e])
        if n == 0:
            continue
        n_tiles = (n + tile_m - 1) // tile_m
        local = set()
        for t in sorted({0, n_tiles // 2, n_tiles - 1}):
            local.update({t * tile_m, min(t * tile_m + tile_m - 1, n - 1)})
        rows = offs[e] + np.array(sorted(local))
        rows_t = torch.from_numpy(rows.astype(np.int64)).cuda()
        r = O.ternary_expert(x[tok_of[rows]], *op.experts(e))
        assert np.array_equal(taps["acc_gate"][rows_t].cpu().numpy(), r["acc_gate"]), f"expert {e}"
        assert np.array_equal(taps["acc_up"][rows_t].cpu().numpy(), r["acc_up"]), f"expert {e}"
        h_g = bits(taps["h"][rows_t])
        neq = h_g != r["h"]
        assert neq.mean() <= 5 * H_FLIP_RATE, (e, neq.mean())        # a few rows: the rate itself is noisy
        if neq.any():
            a, b = O.bf16_to_f32(h_g[neq]).astype(np.float64), O.bf16_to_f32(r["h"][neq]).astype(np.float64)
            assert (np.abs(a - b) <= np.maximum(np.abs(a), np.abs(b)) * 2.0 ** -7 + 1e-30).all()
        q_h_want, beta_h_want = O.absmax_int8(O.bf16_to_f32(h_g))
        q_h = taps["q_h"][rows_t].cpu().numpy()
        assert np.array_equal(q_h, q_h_want), f"expert {e}"
        assert np.array_equal(taps["beta_h"][rows_t].cpu().numpy(), beta_h_want[:, 0]), f"expert {e}"
        assert np.array_equal(taps["acc_down"][rows_t].cpu().numpy(),
                              O.ternary_matmul_int(op.experts(e)[4], q_h)), f"expert {e}"
        seen.append(e)
        if e not in keep and cfg.n_experts * cfg.d_model * cfg.d_ff > 5e8:
            op._experts.pop(e, None)                                  # the largest shape: one expert's matrices at a time
    _log(f"  rows of the first / middle / last row tile checked for experts {seen}")
    assert seen == [e for e in range(E) if counts[e] > 0]


def _check_shared_tiles(cfg, op, taps, tile=256):
    """Shared expert at full size: first and last token of every row tile of the shared GEMMs."""
    T = cfg.n_tokens
    toks = np.unique(np.concatenate([np.arange(0, T, tile), np.minimum(np.arange(tile - 1, T + tile - 1, tile), T - 1)]))
    tok_t = torch.from_numpy(toks.astype(np.int64)).cuda()
    h_ref, y_ref = O.shared_expert(op.x[toks], *op.shared)
    hs_neq = (bits(taps["h_s"][tok_t]) != h_ref).mean()
    assert hs_neq <= 5e-3, hs_neq
    y = taps["y_s"][tok_t].cpu().numpy()
    assert np.allclose(y, y_ref, rtol=0, atol=2e-3 + 2e-3 * np.abs(y_ref).max())
    _log(f"  shared expert on {len(toks)} tokens (both ends of every {tile}-row tile): h_s flip rate {hs_neq:.2e}, "
         f"max |dy_s| {np.abs(y - y_ref).max():.2e}")


FULL_TAPS = ("topk_idx", "topk_p", "counts", "row_of", "tok_of", "q_x", "beta_x", "acc_gate", "acc_up", "h", "q_h",
             "beta_h", "acc_down")


def test_layer_config2_full():
    """Qwen2.5-0.5B-shaped layer, T = 2048, outlier channels: every token against the oracle."""
    cfg = W.C2
    _log(f"layer {cfg.name}")
    M = _m()
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, M.TAP_FIELDS)
    ref = op.forward()
    _check_stagewise(cfg, gp, op, ref, out, taps)
    assert ref["counts"].max() / ref["counts"].min() < 2.5          # near-uniform load


def test_layer_config3_prefill_sampled():
    cfg = W.C3
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS + ("h_s", "y_s"))
    _check_sampled(cfg, 48, 3, out, taps, op)
    _check_rows_of_every_expert(cfg, op, taps, keep=np.argsort(-taps["counts"].cpu().numpy(), kind="stable")[:3])
    _check_shared_tiles(cfg, op, taps)
    # The last round of the down projection's tile lists is nearly empty at this shape: its row
    # tiles (the last ones in dispatch order) are cut into K planes.  Rows of the first and of
    # the last tiles, all channels.
    R = cfg.n_tokens * cfg.top_k
    rng = np.random.default_rng(7)
    rows = np.concatenate([rng.choice(1024, 16, replace=False), R - 1 - rng.choice(1400, 48, replace=False)])
    _check_down_rows(cfg, op, taps, np.sort(rows))


@pytest.mark.parametrize("T", [256, 320, 448, 512, 768, 1024, 1536])
def test_layer_3b_width_mid_size_batches(T):
    """The 3B width (the weights of configuration 3) between decode and prefill: 32 to 192 rows per
    expert.  T = 256, 320 and 448 run the wave-streaming kernel on 64-row tiles (at 448 some experts
    have more than 64 rows, i.e. a second, short tile); 512 and 768 the large-batch kernels whose
    partly filled row tiles skip their empty fragments; 1024 and 1536 the down projection in two K
    planes.  Routing for all tokens, rows of every expert's first / middle / last row tile, sampled
    tokens end to end, both ends of every shared row tile."""
    cfg = W.C3.with_tokens(T, name=f"c3_qwen3b_T{T}")
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS + ("h_s", "y_s"))
    _check_sampled(cfg, 24, 4, out, taps, op)
    _check_rows_of_every_expert(cfg, op, taps, tile_m=64 if T <= 480 else 128)
    _check_shared_tiles(cfg, op, taps, tile=128)
    R = cfg.n_tokens * cfg.top_k
    rng = np.random.default_rng(T)
    _check_down_rows(cfg, op, taps, np.sort(rng.choice(R, 48, replace=False)))


def test_layer_64_row_tiles_with_units_cut_into_equal_runs():
    """A wider expert (d_ff = 14336: seven K planes in the down projection) at T = 480: 20 row tiles of
    64 rows give 140 (row tile, K plane) groups for 256 workgroups, so the wave-streaming down kernel
    cuts the (group, fragment) units into equal runs and a workgroup ends one group and starts the
    next (asserted from the expert counts)."""
    cfg = W.MoteConfig("mid_equal_runs_T480", 2048, 14336, 16, 2, 480, seed=31, sigma_shared=0.012)
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS + ("h_s", "y_s"))
    counts = taps["counts"].cpu().numpy()
    groups = int(np.sum((counts + 63) // 64)) * 7
    assert 128 < groups < 192, groups          # one workgroup per group would leave more than a quarter of 256 idle
    _check_sampled(cfg, 24, 4, out, taps, op)
    _check_rows_of_every_expert(cfg, op, taps, tile_m=64)
    R = cfg.n_tokens * cfg.top_k
    _check_down_rows(cfg, op, taps, np.sort(np.random.default_rng(480).choice(R, 48, replace=False)))


@pytest.mark.parametrize("T", [136, 192, 240])
def test_layer_1p5b_width_64_row_tiles(T):
    """The paper's 1.5B layer (four experts, top-1) with 34 to 60 rows per expert: 64-row tiles whose
    planes are shorter than the kernel's 16 K steps (gate-up 12 steps, down 14), so the padding
    steps are exercised."""
    cfg = W.P15.with_tokens(T, name=f"paper_1.5b_top1_T{T}")
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS + ("h_s", "y_s"))
    _check_sampled(cfg, 24, 4, out, taps, op)
    _check_rows_of_every_expert(cfg, op, taps, tile_m=64)
    R = cfg.n_tokens * cfg.top_k
    rng = np.random.default_rng(T)
    _check_down_rows(cfg, op, taps, np.sort(rng.choice(R, 32, replace=False)))


@pytest.mark.parametrize("cfg", [W.P05, W.P15, W.P3], ids=lambda c: c.name)
def test_layer_paper_shape_top1_sampled(cfg):
    """The paper's own layer (Section 4.1): four routed experts, top-1 gating (the combine weight is
    the raw softmax probability), 2048 tokens, at the 0.5B / 1.5B / 3B widths."""
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS)
    _check_sampled(cfg, 32, 4, out, taps, op)


def _random_mid_config(seed):
    rng = np.random.default_rng(5000 + seed)
    d = int(rng.choice([512, 768, 1024, 1536, 2048]))
    f = int(rng.choice([1024, 1536, 2048, 3072, 4096]))
    e = int(rng.choice([2, 4, 6, 8, 12]))
    k = int(rng.integers(1, min(e, 3) + 1))
    t = int(rng.choice([1000, 1537, 2048, 3000, 4100, 6000]))
    kw = dict(bias_kind="zipf", zipf_tau=float(rng.uniform(0.2, 0.8))) if rng.integers(0, 2) else {}
    return W.MoteConfig(f"random_mid_{seed}_d{d}_F{f}_E{e}_k{k}_T{t}", d, f, e, k, t, seed=300 + seed,
                        sigma_shared=0.012, **kw)


@pytest.mark.parametrize("seed", range(8))
def test_layer_random_mid_size_sampled(seed):
    """Seeded random mid-size shapes on the large-batch kernels (fixed and drawn tile shares, K planes,
    cut last rounds): routing and dispatch for every token, the experts on sampled tokens, and the
    down accumulators of the first and last dispatch rows on every channel."""
    cfg = _random_mid_config(seed)
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS)
    _check_sampled(cfg, 24, min(cfg.n_experts, 3 + 2 * cfg.top_k), out, taps, op)
    R = cfg.n_tokens * cfg.top_k
    rng = np.random.default_rng(seed)
    rows = np.unique(np.concatenate([rng.choice(256, 8, replace=False), R - 1 - rng.choice(600, 24, replace=False)]))
    _check_down_rows(cfg, op, taps, rows)


@pytest.mark.parametrize("T,n", [(1, 2), (4, 4), (16, 8), (64, 16)])
def test_layer_config4_decode(T, n):
    cfg = W.decode_config(T, n)
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS)
    _, _, idx_o, _ = O.router(op.x, op.w_router, op.bias, cfg.top_k)
    assert len(np.unique(idx_o)) == n                                # the step touches exactly n experts
    _check_sampled(cfg, 12, n, out, taps, op)


def test_layer_decode_with_64_experts_tile_list_beyond_one_wavefront():
    """64 experts at the 3B width (d_ff = 8192), 64 tokens of which the biased router sends to six
    experts: the bound on the row tiles (R / 32 + E = 68) exceeds the 64 entries the wave-streaming
    kernel can fetch as one table, so it reads the tile list entry by entry."""
    cfg = W.MoteConfig("decode_64_experts", 2048, 8192, 64, 2, 64, seed=41, sigma_shared=0.015,
                       bias_kind="subset", bias_subset=6)
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS)
    _, _, idx_o, _ = O.router(op.x, op.w_router, op.bias, cfg.top_k)
    n = len(np.unique(idx_o))
    assert 2 <= n <= 6
    _check_sampled(cfg, 16, n, out, taps, op)


def test_layer_config5_skewed_sampled():
    cfg = W.C5
    _log(f"layer {cfg.name}")
    gp, op = GpuProblem(cfg), OracleProblem(cfg)
    out, taps = _run_layer(gp, FULL_TAPS + ("h_s", "y_s"))
    _check_sampled(cfg, 24, 2, out, taps, op)
    counts = taps["counts"].cpu().numpy()
    assert 6.0 <= counts.max() / counts.min() <= 14.0                # loads imbalanced about 10x
    # every expert at its real load (7037 down to 708 rows): both ends and the middle of its row tiles
    _check_rows_of_every_expert(cfg, op, taps)
    _check_shared_tiles(cfg, op, taps)
    # down accumulators of the first and of the last dispatch rows on every channel (the tiles of the
    # last round are the ones a drawn or cut schedule treats differently)
    R = cfg.n_tokens * cfg.top_k
    rng = np.random.default_rng(11)
    rows = np.concatenate([rng.choice(1024, 16, replace=False), R - 1 - rng.choice(1400, 32, replace=False)])
    _check_down_rows(cfg, op, taps, np.sort(rows))


# ------------------------------------------------------------------------ error paths
def test_bad_arguments_are_rejected_before_any_launch():
    M = _m()
    lib = M.load_library()
    gp = GpuProblem(W.C1.with_tokens(4, name="c1_T4"))
    L = gp.layer.struct
    ws = gp.layer.workspace(4)
    out = torch.empty_like(gp.x)
    fwd = lambda layer, T, wsb: lib.mote_layer_forward(ctypes.byref(layer), gp.x.data_ptr(), T, out.data_ptr(),
                                                       ws.data_ptr(), wsb, None, None)
    assert fwd(L, 4, ws.numel()) == 0
    assert fwd(L, 4, 16) == 3                                         # workspace too small
    assert fwd(L, -1, ws.numel()) == 1
    bad = type(L)()
    ctypes.memmove(ctypes.byref(bad), ctypes.byref(L), ctypes.sizeof(L))
    bad.d_model = 200
    assert fwd(bad, 4, ws.numel()) == 2                               # unsupported shape
    ctypes.memmove(ctypes.byref(bad), ctypes.byref(L), ctypes.sizeof(L))
    bad.top_k = 9
    assert fwd(bad, 4, ws.numel()) == 2
    ctypes.memmove(ctypes.byref(bad), ctypes.byref(L), ctypes.sizeof(L))
    bad.wt_up = None
    assert fwd(bad, 4, ws.numel()) == 1
    assert lib.mote_layer_workspace_bytes(ctypes.byref(bad), -3) == 0
    w = torch.zeros(33, 128, device="cuda")
    p = torch.zeros(1024, dtype=torch.int32, device="cuda")
    a = torch.zeros(1, device="cuda")
    assert lib.mote_pack_ternary(w.data_ptr(), 0, 33, 128, p.data_ptr(), a.data_ptr(), None) == 2
    assert lib.mote_pack_ternary(w.data_ptr(), 7, 32, 128, p.data_ptr(), a.data_ptr(), None) == 1
    assert lib.mote_pack_ternary(None, 0, 32, 128, p.data_ptr(), a.data_ptr(), None) == 1
    assert lib.mote_router_topk(gp.x.data_ptr(), gp.w_router.data_ptr(), None, 4, 256, 4, 5, p.data_ptr(),
                                a.data_ptr(), None, None) == 2
    assert M.load_library().mote_status_string(2) == b"unsupported shape"
    torch.cuda.synchronize()


@pytest.mark.parametrize("cfg", [W.C1, W.C1.with_tokens(300, name="c1_T300")], ids=lambda c: c.name)
def test_forward_graph_replays_match_eager(cfg):
    """The forward captured into a HIP graph (helper stream included) gives the eager result on
    every replay, with eager work and synchronisations between the replays."""
    M = _m()
    _log(f"graph {cfg.name}")
    gp = GpuProblem(cfg)
    want = M.mote_layer_forward(gp.layer, gp.x).clone()
    torch.cuda.synchronize()
    x = gp.x.clone()
    out = torch.empty_like(x)
    ws = gp.layer.workspace(cfg.n_tokens)
    fg = M.ForwardGraph(gp.layer, x, out, ws)
    for it in range(4):
        out.zero_()
        torch.cuda.synchronize()
        got = fg.replay()
        torch.cuda.synchronize()
        assert torch.equal(got, want), it
        eager = M.mote_layer_forward(gp.layer, gp.x)          # eager work between the replays
        torch.cuda.synchronize()
        assert torch.equal(eager, want), it
    # new input in the captured buffer: the replay follows it
    x.copy_(gp.x.flip(0))
    want2 = M.mote_layer_forward(gp.layer, gp.x.flip(0).contiguous())
    got2 = fg.replay()
    torch.cuda.synchronize()
    assert torch.equal(got2, want2)


@pytest.mark.parametrize("cfg", [W.C1, W.C1.with_tokens(300, name="c1_T300"), W.decode_config(4, 4)], ids=lambda c: c.name)
def test_forward_on_a_caller_stream_and_changing_batch_sizes(cfg):
    """The forward is ordered on the caller's stream (a non-default one here, with work queued before
    and after it on that stream), and one layer serves batches of different sizes one after the other."""
    M = _m()
    _log(f"caller stream {cfg.name}")
    gp = GpuProblem(cfg)
    want = M.mote_layer_forward(gp.layer, gp.x).clone()
    torch.cuda.synchronize()
    side = torch.cuda.Stream()
    with torch.cuda.stream(side):
        x = torch.zeros_like(gp.x)
        x.copy_(gp.x, non_blocking=True)                 # producer of x on the same stream
        got = M.mote_layer_forward(gp.layer, x)
        doubled = got.float() * 2                         # consumer on the same stream
    side.synchronize()
    assert torch.equal(got, want)
    assert torch.equal(doubled, want.float() * 2)
    T = cfg.n_tokens
    for t in (max(1, T // 3), T, max(1, T - 1)):          # smaller, equal, ragged: same workspace object
        part = M.mote_layer_forward(gp.layer, gp.x[:t].contiguous())
        torch.cuda.synchronize()
        assert torch.equal(part, want[:t]), t


@pytest.mark.parametrize("cfg,n", [(W.C2, 60), (W.decode_config(64, 16), 120), (W.decode_config(4, 4), 120),
                                   (W.C1.with_tokens(300, name="c1_T300"), 120)], ids=lambda c: getattr(c, "name", str(c)))
def test_back_to_back_forwards_with_alternating_inputs(cfg, n):
    """Forwards queued back to back, without a synchronisation between them and with two inputs
    taking turns on one workspace: every output equals the one of a forward that was waited for
    (the fork and join between the caller's stream and the helper stream order all data)."""
    M = _m()
    _log(f"back to back {cfg.name}")
    gp = GpuProblem(cfg)
    xs = [gp.x, (gp.x.flip(0) * 0.5 + gp.x * 0.5).contiguous()]
    refs = []
    for x in xs:
        refs.append(M.mote_layer_forward(gp.layer, x).clone())
        torch.cuda.synchronize()
    assert not torch.equal(refs[0], refs[1])
    outs = [torch.empty_like(gp.x) for _ in range(n)]
    for i in range(n):
        M.mote_layer_forward(gp.layer, xs[i & 1], out=outs[i])
    torch.cuda.synchronize()
    assert [i for i in range(n) if not torch.equal(outs[i], refs[i & 1])] == []


@pytest.mark.parametrize("cfg,n", [(W.C2, 30), (W.decode_config(4, 4), 60)], ids=lambda c: getattr(c, "name", str(c)))
def test_forward_after_async_host_to_device_copy(cfg, n):
    """x is refilled from pinned host memory by an asynchronous copy on the caller's stream right
    before each forward (three inputs taking turns): the helper stream, too, sees the new x."""
    M = _m()
    _log(f"host copy {cfg.name}")
    gp = GpuProblem(cfg)
    xs = [gp.x.clone(), (gp.x.flip(0) * 0.5 + gp.x * 0.5).contiguous(), (gp.x * 0.25).contiguous()]
    refs = []
    for x in xs:
        refs.append(M.mote_layer_forward(gp.layer, x).clone())
        torch.cuda.synchronize()
    hosts = [x.cpu().pin_memory() for x in xs]
    xdev = torch.empty_like(gp.x)
    outs = [torch.empty_like(gp.x) for _ in range(n)]
    for i in range(n):
        xdev.copy_(hosts[i % 3], non_blocking=True)
        M.mote_layer_forward(gp.layer, xdev, out=outs[i])
    torch.cuda.synchronize()
    assert [i for i in range(n) if not torch.equal(outs[i], refs[i % 3])] == []


def test_stage_timing_reports_every_stage():
    M = _m()
    gp = GpuProblem(W.C1)
    M.mote_stage_timing(True)
    try:
        M.mote_layer_forward(gp.layer, gp.x)
        times = M.mote_stage_times()
    finally:
        M.mote_stage_timing(False)
    assert set(times) == set(M.STAGE_NAMES) and all(v > 0 for v in times.values())
    src = torch.arange(1 << 16, dtype=torch.int32, device="cuda")
    dst = torch.zeros_like(src)
    M.mote_calib_copy(dst, src)
    torch.cuda.synchronize()
    assert torch.equal(src, dst)


# A decode step with the router, the row quantiser and the dispatch plan inside the large kernels against
# the same step with kernels of their own: same arithmetic per element, so every tap is equal to the bit.
# Tokens at the edges of the token-row templates (8, 16, 32), top-k up to the most dispatch rows (512) and
# one row, expert counts that are no power of two and the most (16), one tile and several per expert (and 64-row tiles), one
# chunk sweep of a hidden row and a second one (F > 20480), a gate-up kernel for d <= 2048 and one above.
ROLE_CASES = [(1, 256, 512, 4, 1), (1, 256, 512, 16, 8), (8, 384, 640, 5, 2), (9, 512, 1408, 16, 2), (16, 256, 512, 2, 1),
              (17, 2176, 1280, 8, 2), (32, 256, 20608, 3, 1), (33, 1536, 8960, 16, 2), (63, 128, 128, 16, 8),
              (64, 2048, 11008, 16, 2), (64, 256, 512, 16, 8), (64, 384, 640, 1, 1), (64, 1536, 8960, 4, 2)]


@pytest.mark.parametrize("shared_bits", [0, 8, 4])
@pytest.mark.parametrize("T,d,F,E,k", ROLE_CASES)
def test_decode_step_with_small_kernels_inside_the_large_ones(T, d, F, E, k, shared_bits):
    M = _m()
    g = torch.Generator(device="cuda").manual_seed(T * 1000 + d + E)
    rnd = lambda *s, std=1.0: torch.randn(*s, device="cuda", generator=g) * std
    shared = [rnd(*s, std=0.02).to(torch.bfloat16) for s in ((F, d), (F, d), (d, F))]
    scales = None
    if shared_bits:
        packed = [M.mote_pack_rtn(w, shared_bits) for w in shared]
        shared, scales = [p for p, _ in packed], tuple(s for _, s in packed)
    wt = [torch.empty(E, d * F // 16, dtype=torch.int32, device="cuda") for _ in range(3)]
    alpha = torch.empty(3, E, 1, dtype=torch.float32, device="cuda")
    for e in range(E):
        for m in range(3):
            M.mote_pack_ternary(rnd(*((F, d) if m < 2 else (d, F)), std=0.02), packed=wt[m][e], alpha=alpha[m, e])
    bias = None if E < 4 else torch.linspace(0.0, 2.0, E, device="cuda")     # uneven loads: empty and full tiles
    layer = M.MoteLayer(rnd(d, E, std=d ** -0.5).to(torch.bfloat16), *shared, *wt, alpha[:, :, 0].t().contiguous(), k,
                        router_bias=bias, shared_bits=shared_bits, shared_scales=scales)
    x = rnd(T, d).to(torch.bfloat16)
    names = ("topk_idx", "topk_p", "counts", "row_of", "tok_of", "q_x", "beta_x", "acc_gate", "acc_up", "h", "q_h",
             "beta_h", "acc_down", "h_s", "y_s", "out_f32")
    taps = {}
    try:
        for mode in (0, 2):
            M.mote_tuning_set("decode_roles", mode)
            taps[mode] = M.alloc_taps(layer, T, names)
            taps[mode]["out"] = M.mote_layer_forward(layer, x, taps={n: t for n, t in taps[mode].items()})
            torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("decode_roles", 1)
    for n in taps[0]:
        a, b = taps[0][n], taps[2][n]
        assert torch.equal(a, b), n


@pytest.mark.parametrize("T", [32, 34, 36, 94, 96, 98])
def test_layer_rows_longer_than_a_plane_on_either_tile_height(T):
    """d > 2048 with 16, 17 and 47 to 49 rows per expert: the 128-row kernel from 17 and from 49 rows on, equal to the bit to
    the 32-row kernels (integer accumulators; the shared expert runs the same kernels either way)."""
    M = _m()
    cfg = W.MoteConfig(f"wide_T{T}", 2304, 640, 4, 2, T, seed=500 + T)
    gp = GpuProblem(cfg)
    names = ("topk_idx", "row_of", "acc_gate", "acc_up", "h", "q_h", "acc_down", "y_s", "out_f32")
    taps = {}
    try:
        for rows in (48, 16, -1):
            M.mote_tuning_set("decode_rows", rows)
            taps[rows] = M.alloc_taps(gp.layer, T, names)
            out = M.mote_layer_forward(gp.layer, gp.x, taps=taps[rows])
            torch.cuda.synchronize()
            taps[rows]["out"] = out
    finally:
        M.mote_tuning_set("decode_rows", -1)
    for n in taps[48]:
        assert torch.equal(taps[48][n], taps[16][n]) and torch.equal(taps[48][n], taps[-1][n]), n


# Steps of the widest layers keep the forked shared expert and make only the dispatch plan inside the gate-up kernel (the
# K-split one, d > 2048): against the plan kernel, by the default rule, with the shared chain on the
# helper stream.  Two, eight and 32 tokens, one and several tiles per expert, experts without rows (bias).
@pytest.mark.parametrize("T,k,shared_bits", [(2, 1, 0), (8, 2, 0), (1, 2, 8), (7, 2, 8), (32, 2, 8), (3, 2, 4), (8, 4, 4)])
def test_decode_step_with_the_plan_alone_inside_the_gate_up_kernel(T, k, shared_bits):
    M = _m()
    d, F, E = 2304, 16384, 16
    g = torch.Generator(device="cuda").manual_seed(T * 100 + k)
    rnd = lambda *s, std=1.0: torch.randn(*s, device="cuda", generator=g) * std
    shared, scales = [rnd(*s, std=0.01).to(torch.bfloat16) for s in ((F, d), (F, d), (d, F))], None
    if shared_bits:
        packed = [M.mote_pack_rtn(w, shared_bits) for w in shared]
        shared, scales = [p for p, _ in packed], tuple(s for _, s in packed)
    wt = [torch.empty(E, d * F // 16, dtype=torch.int32, device="cuda") for _ in range(3)]
    alpha = torch.empty(3, E, 1, dtype=torch.float32, device="cuda")
    for e in range(E):
        for m in range(3):
            M.mote_pack_ternary(rnd(*((F, d) if m < 2 else (d, F)), std=0.02), packed=wt[m][e], alpha=alpha[m, e])
    layer = M.MoteLayer(rnd(d, E, std=d ** -0.5).to(torch.bfloat16), *shared, *wt, alpha[:, :, 0].t().contiguous(), k,
                        router_bias=torch.tensor([0.0, 3.0, 30.0] + 13 * [-2.0], device="cuda"), shared_bits=shared_bits, shared_scales=scales)
    x = rnd(T, d).to(torch.bfloat16)
    names = ("topk_idx", "topk_p", "counts", "row_of", "tok_of", "acc_gate", "acc_up", "h", "q_h", "acc_down", "h_s", "y_s", "out_f32")
    taps = {}
    try:
        for mode in (0, 1):
            M.mote_tuning_set("decode_roles", mode)
            for again in range(3):      # a step right behind the last one: the two streams meet different kernels
                taps[mode] = M.alloc_taps(layer, T, names)
                taps[mode]["out"] = M.mote_layer_forward(layer, x, taps=dict(taps[mode]))
            torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("decode_roles", 1)
    assert taps[0]["counts"].sum() == T * k
    for n in taps[0]:
        assert torch.equal(taps[0][n], taps[1][n]), n


def _small_layer(M, d, F, E, k, w_router, shared_bits=0, seed=0):
    g = torch.Generator(device="cuda").manual_seed(seed)
    rnd = lambda *s, std=1.0: torch.randn(*s, device="cuda", generator=g) * std
    shared, scales = [rnd(*s, std=0.02).to(torch.bfloat16) for s in ((F, d), (F, d), (d, F))], None
    dense = [w.double() for w in shared]
    if shared_bits:
        q = [O.rtn_quantize(W.bf16_bits(w.cpu()), shared_bits) for w in shared]
        dense = [torch.from_numpy(c).cuda().double() * torch.from_numpy(s).cuda().double()[:, None] for c, s in q]
        packed = [M.mote_pack_rtn(w, shared_bits) for w in shared]
        shared, scales = [p for p, _ in packed], tuple(s for _, s in packed)
    wt = [torch.empty(E, d * F // 16, dtype=torch.int32, device="cuda") for _ in range(3)]
    alpha = torch.empty(3, E, 1, dtype=torch.float32, device="cuda")
    for e in range(E):
        for m in range(3):
            M.mote_pack_ternary(rnd(*((F, d) if m < 2 else (d, F)), std=0.02), packed=wt[m][e], alpha=alpha[m, e])
    layer = M.MoteLayer(w_router, *shared, *wt, alpha[:, :, 0].t().contiguous(), k, shared_bits=shared_bits, shared_scales=scales)
    layer.shared_dense = dense
    return layer


# The router inside the decode kernel reads a chunk's router rows as whole 16-byte runs, 8-byte runs of an aligned matrix
# or single elements: expert counts of each kind, and matrices that begin 2 and 4 bytes past an 8-byte boundary.  The same
# experts, weights and codes as the router kernel of its own, to the bit (same sums in the same order).  At most 31 rows per
# expert: with more the routed GEMMs may leave the decode kernels, and the router would have a kernel of its own in both modes.
@pytest.mark.parametrize("E,k,offset", [(16, 2, 0), (8, 1, 0), (12, 2, 0), (4, 4, 0), (12, 2, 1), (4, 1, 2), (6, 2, 0), (13, 3, 0), (1, 1, 1)])
@pytest.mark.parametrize("T,d,shared_bits", [(1, 128, 0), (5, 2176, 0), (64, 384, 8)])
def test_router_rows_of_every_alignment_inside_the_decode_kernel(E, k, offset, T, d, shared_bits):
    M = _m()
    T = min(T, 31 * E // k)
    g = torch.Generator(device="cuda").manual_seed(E * 100 + T)
    w = torch.empty(d * E + 8, dtype=torch.bfloat16, device="cuda")[offset:offset + d * E].view(d, E)
    w.copy_(torch.randn(d, E, device="cuda", generator=g) * d ** -0.5)
    layer = _small_layer(M, d, 256, E, k, w, shared_bits=shared_bits, seed=E)
    x = torch.randn(T, d, device="cuda", generator=g).to(torch.bfloat16)
    names = ("topk_idx", "topk_p", "q_x", "beta_x", "out_f32")
    taps = {}
    try:
        for mode in (0, 2):
            M.mote_tuning_set("decode_roles", mode)
            taps[mode] = M.alloc_taps(layer, T, names)
            M.mote_layer_forward(layer, x, taps=taps[mode])
            torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("decode_roles", 1)
    for n in names:
        assert torch.equal(taps[0][n], taps[2][n]), n


# Batches of up to 64 tokens with at most two experts per token have a combine kernel of their own; with the fp32 output
# tapped the general one runs.  Same sums in the same order: equal to the bit, with the residual of a block too.
# One token and the most, one more, one channel group per row tile and a wide row, one and several planes of either kind.
@pytest.mark.parametrize("T,d,F,E,k", [(1, 128, 256, 4, 1), (64, 256, 512, 4, 2), (65, 256, 512, 4, 2), (3, 2176, 640, 4, 2), (2, 128, 4096, 4, 2),
                                       (63, 1536, 8960, 4, 1), (5, 256, 512, 4, 3)])
@pytest.mark.parametrize("shared_bits", [0, 4])
def test_combine_of_few_tokens_equals_the_general_one(T, d, F, E, k, shared_bits):
    M = _m()
    g = torch.Generator(device="cuda").manual_seed(T + d)
    layer = _small_layer(M, d, F, E, k, (torch.randn(d, E, device="cuda", generator=g) * d ** -0.5).to(torch.bfloat16), shared_bits, T)
    x = torch.randn(T, d, device="cuda", generator=g).to(torch.bfloat16)
    gamma = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    for call in (lambda **kw: M.mote_layer_forward(layer, x, **kw), lambda **kw: M.mote_block_forward(layer, x, gamma, None, eps=1e-6, **kw)):
        taps = M.alloc_taps(layer, T, ("out_f32",))
        plain, general = call(), call(taps=taps)
        torch.cuda.synchronize()
        assert torch.equal(plain, general) and torch.equal(general, taps["out_f32"].to(torch.bfloat16))
        assert general.float().abs().max() > 0


def _unpacked(words, n_rows, n_cols):
    """Ternary matrix of the packed words (layout of O.pack_int2), as float64 on the device."""
    w = words.view(n_rows // 32, n_cols // 128, 2, 32, 4)                       # row tile, K tile, g, r, s
    code = torch.stack([(w >> (8 * (i % 4) + 2 * (i // 4))) & 3 for i in range(16)], dim=-1)
    return (code.permute(0, 3, 1, 4, 2, 5).reshape(n_rows, n_cols) - 1).double()


# Routed tiles run K loops of 32, 64, 96 or 128 rows: tiles of every height at and beside those limits, alone and behind a
# full tile, an expert without rows, one K plane and several.  Integer accumulators, exact.
@pytest.mark.parametrize("counts", [(1, 32, 33, 64, 65, 96, 97, 128), (129, 160, 161, 225, 256, 300, 0, 31)])
@pytest.mark.parametrize("d,F", [(128, 256), (384, 640), (256, 4096), (2176, 384)])
def test_routed_tiles_of_every_height(d, F, counts):
    M = _m()
    E, T = len(counts), sum(counts)
    g = torch.Generator(device="cuda").manual_seed(d + T)
    w = torch.zeros(d, E, device="cuda")
    w[torch.arange(E), torch.arange(E)] = 1.0                    # channel e alone decides for expert e
    layer = _small_layer(M, d, F, E, 1, w.to(torch.bfloat16), seed=d)
    expert = torch.repeat_interleave(torch.arange(E), torch.tensor(counts))[torch.randperm(T, generator=torch.Generator().manual_seed(T))]
    x = torch.randn(T, d, device="cuda", generator=g)
    x[:, :E] = 0
    x[torch.arange(T), expert] = 6.0
    taps = M.alloc_taps(layer, T, ("counts", "tok_of", "q_x", "acc_gate", "acc_up", "q_h", "acc_down"))
    M.mote_layer_forward(layer, x.to(torch.bfloat16), taps=taps)
    torch.cuda.synchronize()
    assert tuple(taps["counts"].tolist()) == counts
    q_x, tok_of, q_h = taps["q_x"].double(), taps["tok_of"].long(), taps["q_h"].double()
    lo = 0
    for e, n in enumerate(counts):
        if n:
            t = [_unpacked(layer.tensors[m][e], *((F, d) if m != "wt_down" else (d, F))) for m in ("wt_gate", "wt_up", "wt_down")]
            rows = q_x[tok_of[lo:lo + n]]
            assert torch.equal(taps["acc_gate"][lo:lo + n].double(), rows @ t[0].T), e
            assert torch.equal(taps["acc_up"][lo:lo + n].double(), rows @ t[1].T), e
            assert torch.equal(taps["acc_down"][lo:lo + n].double(), q_h[lo:lo + n] @ t[2].T), e
        lo += n


# The shared expert's GEMM tiles (128 x 128, 128 x 256 and 256 x 256, by the cost model and each of them forced): token and
# channel remainders of every tile, two K chunks (the fewest a shape has) and more, K planes of the down projection, and the scaled epilogue of
# a quantised expert whose expanded codes take the same kernels.
@pytest.mark.parametrize("variant", [0, 1, 2, 3])
@pytest.mark.parametrize("T,d,F,shared_bits", [(65, 128, 256, 0), (129, 384, 640, 0), (300, 256, 4096, 0), (257, 896, 1152, 0),
                                               (1025, 256, 384, 0), (513, 256, 640, 8), (520, 384, 512, 4)])
def test_shared_gemm_tiles(variant, T, d, F, shared_bits):
    M = _m()
    g = torch.Generator(device="cuda").manual_seed(T + d)
    layer = _small_layer(M, d, F, 4, 1, (torch.randn(d, 4, device="cuda", generator=g) * d ** -0.5).to(torch.bfloat16), shared_bits, T)
    x = torch.randn(T, d, device="cuda", generator=g).to(torch.bfloat16)
    w = layer.shared_dense
    taps = M.alloc_taps(layer, T, ("h_s", "y_s"))
    try:
        M.mote_tuning_set("shared_variant", variant)
        M.mote_layer_forward(layer, x, taps=taps)
        torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("shared_variant", 0)
    xd = x.double()
    gate = xd @ w[0].T
    h_ref = (gate * torch.sigmoid(gate) * (xd @ w[1].T)).float().to(torch.bfloat16)
    h = taps["h_s"]
    neq = h != h_ref                     # fp32 sums against fp64: a rounding flips now and then, by one bf16 step
    a, b = h[neq].double(), h_ref[neq].double()
    assert neq.double().mean() <= 5e-3
    assert ((a - b).abs() <= torch.maximum(a.abs(), b.abs()) * 2.0 ** -7 + 1e-5 * h_ref.abs().max().double()).all()
    # F products summed in fp32 in any order: at most F roundings of 2^-24, each of no more than the sum of magnitudes
    hd = h.double()
    bound = F * 2.0 ** -24 * (hd.abs() @ w[2].abs().T) + 1e-30
    assert ((taps["y_s"].double() - hd @ w[2].T).abs() <= bound).all()


# Narrow layers whose shared gate-up GEMM has a 256 x 256 tile for every CU start the shared expert behind the router, others (128 x 256
# tiles, fifth and sixth) in front of it, those of more than 16 experts (the last two) already with either tile for most CUs: the fewest such tiles and a row of them less, a quantised expert (its expansion goes first), a block,
# alternating inputs without a wait between them, and replays of a captured forward.  Equal to one stream, to the bit.
@pytest.mark.parametrize("T,d,F,E,k,shared_bits", [(4096, 128, 2048, 8, 2, 0), (3840, 128, 2048, 8, 2, 0), (4090, 256, 2048, 4, 1, 8), (8192, 256, 1024, 16, 3, 0),
                                                   (2048, 512, 2048, 8, 2, 0), (8192, 256, 512, 4, 2, 4),
                                                   (2000, 512, 2048, 32, 2, 0), (6144, 256, 1024, 17, 1, 8)])
def test_shared_expert_started_behind_the_router(T, d, F, E, k, shared_bits):
    M = _m()
    g = torch.Generator(device="cuda").manual_seed(T + d)
    layer = _small_layer(M, d, F, E, k, (torch.randn(d, E, device="cuda", generator=g) * d ** -0.5).to(torch.bfloat16), shared_bits, T)
    xs = [torch.randn(T, d, device="cuda", generator=g).to(torch.bfloat16) for _ in range(2)]
    gamma = torch.ones(d, dtype=torch.bfloat16, device="cuda")
    try:
        M.mote_tuning_set("no_fork", 1)
        want = [M.mote_layer_forward(layer, x) for x in xs] + [M.mote_block_forward(layer, xs[0], gamma, None, eps=1e-6)]
        torch.cuda.synchronize()
    finally:
        M.mote_tuning_set("no_fork", 0)
    outs = [M.mote_layer_forward(layer, xs[i % 2]) for i in range(12)]
    block = M.mote_block_forward(layer, xs[0], gamma, None, eps=1e-6)
    torch.cuda.synchronize()
    assert all(torch.equal(o, want[i % 2]) for i, o in enumerate(outs)) and torch.equal(block, want[2])
    x, out = xs[0].clone(), torch.empty_like(xs[0])
    graph = M.ForwardGraph(layer, x, out, layer.workspace(T))
    for i in (1, 0, 1):
        x.copy_(xs[i])
        out.zero_()
        graph.replay()
        torch.cuda.synchronize()
        assert torch.equal(out, want[i])


# Many tokens go through the fp64 matrix kernel, with router rows read by 16 or 8 bytes or by elements: every such kind and
# register bound (d = 1024, 2048, 4096), a number of channel steps that is no multiple of those in flight, a last
# workgroup of one token, and a matrix that begins 2 bytes past an 8-byte boundary.  Against the kernel of smaller batches.
@pytest.mark.parametrize("d,E,k,offset", [(128, 16, 2, 0), (896, 8, 2, 0), (1024, 12, 2, 1), (1152, 4, 1, 0), (2048, 12, 3, 0), (2048, 13, 2, 0),
                                          (2176, 16, 2, 0), (3584, 6, 2, 0), (4096, 1, 1, 0), (4096, 16, 8, 0)])
def test_router_many_tokens_equals_smaller_batches(d, E, k, offset):
    M = _m()
    T = 4096 + 17
    g = torch.Generator(device="cuda").manual_seed(d + E)
    w = torch.empty(d * E + 8, dtype=torch.bfloat16, device="cuda")[offset:offset + d * E].view(d, E)
    w.copy_(torch.randn(d, E, device="cuda", generator=g) * d ** -0.5)
    x = torch.randn(T, d, device="cuda", generator=g).to(torch.bfloat16)
    x[5, 3], x[4100, d - 1] = float("inf"), float("nan")
    idx, p, counts = M.mote_router_topk(x, w, k)
    parts = [M.mote_router_topk(x[i:i + 128], w, k) for i in range(0, T, 128)]
    torch.cuda.synchronize()
    keep = torch.ones(T, dtype=torch.bool, device="cuda")
    keep[5] = keep[4100] = False                        # not finite: some valid expert
    assert torch.equal(idx[keep], torch.cat([q[0] for q in parts])[keep])
    assert torch.allclose(p[keep], torch.cat([q[1] for q in parts])[keep], rtol=2e-6, atol=1e-9)   # as against the oracle
    assert (idx >= 0).all() and (idx < E).all() and counts.sum().item() == T * k
