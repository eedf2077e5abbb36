"""GPU parity of the individual C-ABI calls against the CPU oracle:
d2c_attention, d2c_refresh_layer, d2c_influence, d2c_select.  Same seeded inputs on
both sides; floats within rel-L2 1e-5 (fp32) / 2e-2 (bf16), index sets bit-exact."""
import numpy as np
import pytest
import torch

from oracle import d2cache_oracle as O
from paper_2509_23094_amd import workloads as W

from gpu_util import TOL, host, oracle_dims, rel_l2, say, topk_margin

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2509_23094_amd import binding
    return binding


def _ctx_for(B, wd, max_seq, n_layers=1, seed=0, tiny_vocab=None, tunables=None):
    dims = W.with_layers(wd, n_layers)
    if tiny_vocab is not None:
        from dataclasses import replace
        dims = replace(dims, vocab=tiny_vocab)
    mdl = W.model_weights(dims, seed)
    return B.Context(dims, mdl, max_seq, tunables=tunables), dims, mdl


# ------------------------------------------------------------------ the ragged-row projection
LINEAR_CASES = [
    # dtype, m, N, K
    ("f32", 1, 16, 16), ("f32", 72, 768, 256), ("f32", 128, 1376, 256), ("f32", 37, 256, 688), ("f32", 5, 40, 20),
    ("f32", 200, 100, 132),
    ("bf16", 1, 64, 128), ("bf16", 83, 1024, 512), ("bf16", 17, 40, 72), ("bf16", 96, 4096, 1408),
    ("bf16", 130, 200, 264), ("bf16", 300, 3000, 520), ("bf16", 64, 33000, 256),
    ("bf16", 185, 1000, 392), ("bf16", 192, 4096, 512), ("bf16", 200, 520, 256),   # 12 row tiles in one chunk; two chunks
]


@pytest.mark.parametrize("dtype,m,N,K", LINEAR_CASES)
def test_linear_parity(B, dtype, m, N, K, tunables=None):
    say(f"linear dtype={dtype} m={m} N={N} K={K} tunables={tunables}")
    wd = W.ModelDims(1, 256, 4, 4, 64, 80, 64, dtype=dtype)
    ctx, _, _ = _ctx_for(B, wd, max_seq=max(m, 16), tunables=tunables)
    a = W.hidden_rows(11, m, K)
    w = W.hidden_rows(12, N, K, std=0.05)
    if dtype == "bf16":
        a, w = W.round_bf16(a), W.round_bf16(w)
    out = torch.full((m, N), 7.0, dtype=torch.float32, device="cuda")
    ctx.d2c_linear(B.to_device(a, dtype), B.to_device(w, dtype), m, N, K, out)
    torch.cuda.synchronize()
    ref = a.astype(np.float64) @ w.astype(np.float64).T          # exact inputs on both sides: fp32 accumulation only
    assert rel_l2(host(out), ref) < 1e-5
    ctx.close()


@pytest.mark.parametrize("waves", [4, 6, 7, 8, 10])
@pytest.mark.parametrize("dtype,m,N,K", [("f32", 37, 250, 132), ("bf16", 70, 1000, 520), ("bf16", 9, 176, 4096)])
def test_linear_parity_every_workgroup_width(B, waves, dtype, m, N, K):
    """The planner picks 6, 8 or 10 waves per workgroup by shape; here each width (and the 4-wave one) is
    forced on shapes whose column count is no multiple of the workgroup's columns."""
    test_linear_parity(B, dtype, m, N, K, tunables={"gemm_waves": waves})


@pytest.mark.parametrize("N", [64, 63])
@pytest.mark.parametrize("splits", [2, 3, 4, 5, 6, 7, 8])
def test_linear_parity_every_split_count(B, splits, N):
    """The partial sums of 2 to 8 splits of k added in pieces of 16 bytes (20 x 64) and value by value (21 x 63)."""
    m, K = 20 if N == 64 else 21, 256 * splits
    assert B.d2c_plan_projection("bf16", m, N, K)["splits"] == splits
    test_linear_parity(B, "bf16", m, N, K)


# ------------------------------------------------------------------ attention (config "C2" and edge shapes)
ATTN_CASES = [
    # dtype, H, Hkv, dh, L, m, kernels ("few": the few-row kernels, "tiled": the LDS-tiled ones, "default":
    # the library's own choice, "": fp32)
    ("bf16", 32, 32, 128, 2048, 256, "tiled"),    # the isolated selective-refresh attention workload, full size
    ("bf16", 32, 32, 128, 2048, 256, "few"),
    ("bf16", 28, 4, 128, 768, 83, "few"),         # Dream geometry (GQA 28/4), ragged m
    ("bf16", 28, 4, 128, 768, 83, "tiled"),       # two query tiles per wave, split key range, ragged last block
    ("bf16", 4, 2, 64, 203, 37, "few"),           # head_dim 64, ragged L and m
    ("bf16", 4, 2, 64, 203, 37, "tiled"),
    ("bf16", 8, 8, 128, 17, 1, "few"),            # one query, L smaller than a workgroup's key span
    ("bf16", 8, 8, 128, 17, 1, "tiled"),          # a single, mostly empty key block
    ("bf16", 4, 4, 128, 130, 130, "few"),         # every row selected
    ("bf16", 4, 4, 128, 130, 130, "tiled"),
    ("bf16", 32, 32, 128, 3072, 300, "tiled"),    # long-context shape: no key split, 3 query blocks, 48 key blocks
    ("bf16", 3, 1, 64, 1000, 129, "tiled"),       # odd head count (A-bar loop tail), head_dim 64, 3 query blocks
    ("bf16", 6, 3, 64, 100, 20, "few"),           # 3 kv heads: neither divides nor is divided by the 8 XCDs
    ("bf16", 16, 2, 128, 600, 50, "few"),         # 4 XCDs per kv head, 8 query heads each; L above 512
    ("bf16", 32, 32, 128, 512, 46, "few"),        # the LLaDA-8B decode step: 96 (tile, head) pairs
    ("bf16", 5, 5, 128, 300, 16, "few"),          # 5 kv heads: plain placement
    ("bf16", 28, 4, 128, 1824, 93, "default"),    # the long-generation decode step late on: too long for the
                                                  # per-head probability rows, so the tiled kernels from 48 rows on
    ("bf16", 28, 4, 128, 1824, 40, "default"),    # same length, fewer rows: the tiled kernels as well
    ("bf16", 28, 4, 128, 1824, 40, "few"),        # and the few-row kernels with their second launch
    ("f32", 4, 4, 64, 128, 73, ""),               # the small fp32 model's geometry
    ("f32", 4, 2, 8, 19, 5, ""),
]


@pytest.mark.parametrize("dtype,H,Hkv,dh,L,m,kernels", ATTN_CASES)
def test_attention_parity(B, dtype, H, Hkv, dh, L, m, kernels):
    say(f"attention dtype={dtype} H={H} Hkv={Hkv} dh={dh} L={L} m={m} kernels={kernels}")
    tun = {"attn_tiled_min_m": 1 if kernels == "tiled" else 1 << 30} if kernels in ("tiled", "few") else None
    _attention_parity(B, dtype, H, Hkv, dh, L, m, tunables=tun)


def test_attention_short_sequence_in_a_long_context(B):
    """A context sized for 2048 positions serving L = 256: the short sequence is split into more head groups
    and key ranges than the longest one, so the scratch buffers must be sized over every L, not max_seq."""
    say("attention L=256 m=200 in a max_seq=2048 context")
    _attention_parity(B, "bf16", 8, 8, 128, 256, 200, max_seq=2048, tunables={"attn_tiled_min_m": 1})


def _attention_parity(B, dtype, H, Hkv, dh, L, m, max_seq=None, tunables=None):
    wd = W.ModelDims(1, H * dh, H, Hkv, dh, 64, 64, dtype=dtype)
    ctx, dims, _ = _ctx_for(B, wd, max_seq=max_seq or L, tunables=tunables)
    case = W.attention_case(1, H, Hkv, dh, L, m, dtype=dtype)
    tdt = B.torch_dtype(dtype)
    q = B.to_device(case["q"], dtype)
    kc, vc = B.to_device(case["k_cache"], dtype), B.to_device(case["v_cache"], dtype)
    nk, nv = B.to_device(case["new_k"], dtype), B.to_device(case["new_v"], dtype)
    idx = torch.from_numpy(case["idx"]).cuda()
    out = torch.zeros((m, H * dh), dtype=tdt, device="cuda")
    abar = torch.zeros((m, L), dtype=torch.float32, device="cuda")
    ctx.d2c_attention(q, idx, m, nk, nv, kc, vc, L, out, abar)
    torch.cuda.synchronize()

    k_ref, v_ref = case["k_cache"].astype(np.float64), case["v_cache"].astype(np.float64)
    k_ref[case["idx"]] = case["new_k"]
    v_ref[case["idx"]] = case["new_v"]
    # the scatter is a copy: bit-exact
    np.testing.assert_array_equal(host(kc), k_ref.astype(np.float32))
    np.testing.assert_array_equal(host(vc), v_ref.astype(np.float32))
    o_ref, a_ref = O.selective_attention(case["q"], k_ref, v_ref, H, Hkv, dh)
    og, ag = host(out), host(abar)
    for r in range(m):
        assert rel_l2(og[r], o_ref[r]) < TOL[dtype], f"output row {r}"
        assert rel_l2(ag[r], a_ref[r]) < TOL[dtype], f"A-bar row {r}"
    np.testing.assert_allclose(host(abar).sum(axis=1), 1.0, atol=2e-3 if dtype == "bf16" else 1e-5)

    # without the head average the output must not change; run-to-run the bits must not change
    out2 = torch.zeros_like(out)
    ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, out2, None)
    abar3, out3 = torch.zeros_like(abar), torch.zeros_like(out)
    ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, out3, abar3)
    torch.cuda.synchronize()
    assert torch.equal(out, out2) and torch.equal(out, out3) and torch.equal(abar, abar3)
    ctx.close()


# ------------------------------------------------------------------ one block on the selected rows
LAYER_CASES = [
    # name, dims, L, m, tolerance-scale
    ("C1-f32", W.DIMS["C1"], 128, 72),
    ("C1-f32-all", W.DIMS["C1"], 128, 128),
    ("tiny-f32-gqa", W.ModelDims(1, 64, 4, 2, 16, 80, 64, dtype="f32"), 33, 7),
    ("bf16-small", W.ModelDims(1, 512, 4, 4, 128, 1408, 64, dtype="bf16"), 200, 45),
    ("bf16-gqa", W.ModelDims(1, 512, 8, 2, 64, 1024, 64, dtype="bf16"), 300, 150),
    ("bf16-185-rows", W.ModelDims(1, 512, 4, 4, 128, 1408, 64, dtype="bf16"), 260, 185),   # 12 row tiles in one chunk
    ("C3-width", W.DIMS["C3"], 512, 83),     # one LLaDA-8B-shaped layer at full width
    ("C4-width", W.DIMS["C4"], 768, 100),    # one Dream-7B-shaped layer at full width
    # more than 256 rows: 128 x 64 outputs per wave in every projection (all widths are whole chunk pairs)
    ("bf16-330-rows", W.ModelDims(1, 512, 4, 4, 128, 1536, 64, dtype="bf16"), 400, 330),
    ("tiny-f32-odd-ffn", W.ModelDims(1, 64, 4, 4, 16, 72, 64, dtype="f32"), 40, 9),   # FFN width not a multiple of 16
]
# the same block with the caller's row-major weights (no pre-tiled copies, separate SwiGLU launch)
LAYER_CASES_ROW_MAJOR = ["C1-f32", "bf16-small", "C3-width"]


@pytest.mark.parametrize("name,wd,L,m", LAYER_CASES, ids=[c[0] for c in LAYER_CASES])
def test_refresh_layer_parity(B, name, wd, L, m):
    _refresh_layer_parity(B, name, wd, L, m)


@pytest.mark.parametrize("name", LAYER_CASES_ROW_MAJOR)
def test_refresh_layer_parity_row_major_weights(B, name):
    case = [c for c in LAYER_CASES if c[0] == name][0]
    _refresh_layer_parity(B, *case, tunables={"gemm_preshuffle": 0})


@pytest.mark.parametrize("waves", [6, 7, 10])
@pytest.mark.parametrize("name", ["C1-f32", "bf16-small", "tiny-f32-odd-ffn"])
def test_refresh_layer_parity_forced_workgroup_width(B, name, waves):
    """The gated epilogue pairs neighbouring waves: checked for the 6- and 10-wave workgroups on shapes where
    the planner would not pick them by itself."""
    case = [c for c in LAYER_CASES if c[0] == name][0]
    _refresh_layer_parity(B, *case, tunables={"gemm_waves": waves})


@pytest.mark.parametrize("mt", [6, 7, 8])
def test_refresh_layer_parity_forced_rows_per_workgroup(B, mt):
    """Many rows: 6, 7 or 8 row tiles for each half of a workgroup of the wide projection shape, whatever the planner would take."""
    case = [c for c in LAYER_CASES if c[0] == "bf16-330-rows"][0]
    _refresh_layer_parity(B, *case, tunables={"gemm_wide_mt": mt})


@pytest.mark.parametrize("m", [299, 300, 304])
def test_refresh_layer_parity_many_rows_from_inside_a_tile(B, m):
    """gemm_wide_min_rows inside a 16-row tile: two plans for one tile count, workspace for both."""
    case = [c for c in LAYER_CASES if c[0] == "bf16-small"][0]
    _refresh_layer_parity(B, f"bf16-{m}-rows", case[1], 304, m, tunables={"gemm_wide_min_rows": 300})


def _refresh_layer_parity(B, name, wd, L, m, tunables=None):
    say(f"refresh_layer {name} L={L} m={m} tunables={tunables}")
    ctx, dims, mdl = _ctx_for(B, wd, max_seq=L, tiny_vocab=64, tunables=tunables)
    od = oracle_dims(dims)
    dtype = dims.dtype
    S = W.distinct_sorted_rows(3, L, m)
    h0 = W.hidden_rows(4, m, dims.d_model, std=0.5)
    kc0 = W.hidden_rows(5, L, dims.d_kv, std=1.0, extra=1)
    vc0 = W.hidden_rows(5, L, dims.d_kv, std=1.0, extra=2)
    if dtype == "bf16":
        kc0, vc0 = W.round_bf16(kc0), W.round_bf16(vc0)
    roll0 = np.abs(W.hidden_rows(6, m, L)).astype(np.float32)           # an arbitrary incoming block for layer > 0

    hidden = torch.from_numpy(h0).cuda()
    kc, vc = B.to_device(kc0, dtype), B.to_device(vc0, dtype)
    idx = torch.from_numpy(S).cuda()
    abar = torch.zeros((m, L), dtype=torch.float32, device="cuda")
    roll = torch.from_numpy(roll0).cuda()
    ctx.d2c_refresh_layer(0, hidden, idx, S, kc, vc, L, abar, roll)
    torch.cuda.synchronize()

    k_ref, v_ref = kc0.astype(np.float64), vc0.astype(np.float64)
    h_ref, a_ref = O.refresh_layer(od, mdl["layers"][0], h0, S, k_ref, v_ref)
    tol = TOL[dtype]
    # row by row: one wrong row must not hide in a norm over the whole tensor
    for r in range(m):
        assert rel_l2(host(hidden)[r], h_ref[r]) < tol, f"hidden row {r}"
        assert rel_l2(host(abar)[r], a_ref[r]) < tol, f"A-bar row {r}"
    kg, vg = host(kc), host(vc)
    for i in S:
        assert rel_l2(kg[i], k_ref[i]) < tol and rel_l2(vg[i], v_ref[i]) < tol, f"K/V row {i}"
    rest = np.setdiff1d(np.arange(L), S)
    np.testing.assert_array_equal(host(kc)[rest], kc0[rest])             # reused rows: untouched bits
    np.testing.assert_array_equal(host(vc)[rest], vc0[rest])
    # layer 0 starts the rollout from the identity: C_S = (A-bar + one-hot) / 2
    c_ref = O.rollout([a_ref], S, L)[S]
    assert rel_l2(host(roll), c_ref) < tol
    ctx.close()


@pytest.mark.parametrize("d,H,dh,F,m", [(64, 32, 64, 208, 17), (128, 16, 64, 80, 33), (128, 32, 64, 208, 17), (192, 16, 64, 208, 16),
                                        (192, 8, 128, 80, 5), (252, 8, 64, 80, 70), (256, 4, 128, 80, 20), (256, 12, 64, 208, 40),
                                        (256, 32, 64, 208, 31)])
def test_refresh_layer_parity_split_sums_in_the_norm_and_apart(B, d, H, dh, F, m):
    """Small float layers whose O projection has 2 to 8 splits: summed inside gate/up's norm, or by a launch in front of it where
    that is the faster, behind a QKV projection with the norm inside or (heads of 128) without."""
    _refresh_layer_parity(B, f"f32 d={d} heads {H} x {dh}", W.ModelDims(1, d, H, H, dh, F, 64, dtype="f32"), m + 20, m)


@pytest.mark.parametrize("d,H,Hkv,dh,F,L,m", [(256, 4, 4, 64, 688, 128, 1), (256, 4, 2, 64, 688, 150, 128), (60, 6, 3, 2, 80, 40, 17),
                                              (132, 3, 1, 32, 48, 70, 33), (20, 2, 1, 16, 16, 20, 16), (192, 6, 2, 4, 208, 300, 127)])
def test_refresh_layer_parity_fused_norm_and_rope(B, d, H, Hkv, dh, F, L, m):
    """Float layers whose projections make the norm in front and RoPE and the cache update behind: ragged contractions, column
    blocks with several heads and with a last head cut off, one row and all eight row tiles; and what a bias adds."""
    wd = W.ModelDims(1, d, H, Hkv, dh, F, 64, dtype="f32")
    _refresh_layer_parity(B, f"f32 d={d} heads {H}/{Hkv} x {dh}", wd, L, m)
    mdl = W.model_weights(wd, 0)
    mdl["layers"][0]["bqkv"] = W.hidden_rows(9, 1, wd.d_q + 2 * wd.d_kv)[0]
    ctx = B.Context(wd, mdl, L)
    S, h0 = W.distinct_sorted_rows(3, L, m), W.hidden_rows(4, m, d, std=0.5)
    kc, vc = (W.hidden_rows(5, L, wd.d_kv, extra=e).astype(np.float64) for e in (1, 2))
    hidden, kd, vd = torch.from_numpy(h0).cuda(), B.to_device(kc, "f32"), B.to_device(vc, "f32")
    ctx.d2c_refresh_layer(0, hidden, torch.from_numpy(S).cuda(), S, kd, vd, L, None, None)
    torch.cuda.synchronize()
    h_ref, _ = O.refresh_layer(oracle_dims(wd), mdl["layers"][0], h0, S, kc, vc)
    assert rel_l2(host(hidden), h_ref) < TOL["f32"] and rel_l2(host(kd), kc) < TOL["f32"] and rel_l2(host(vd), vc) < TOL["f32"]
    ctx.close()


def test_refresh_layer_rollout_chain_and_influence(B):
    """Three layers in a row on the same rows: the compact rollout block and c_j against the literal L x L rollout."""
    wd = W.ModelDims(3, 256, 4, 4, 64, 688, 64, dtype="f32")
    L, m = 96, 29
    say(f"rollout chain L={L} m={m}")
    mdl = W.model_weights(wd, 2)
    ctx = B.Context(wd, mdl, L)
    od = oracle_dims(wd)
    S = W.distinct_sorted_rows(7, L, m)
    h0 = W.hidden_rows(8, m, wd.d_model, std=0.5)
    hidden = torch.from_numpy(h0).cuda()
    idx = torch.from_numpy(S).cuda()
    kcs = [W.hidden_rows(9, L, wd.d_kv, extra=l) for l in range(3)]
    vcs = [W.hidden_rows(10, L, wd.d_kv, extra=l) for l in range(3)]
    roll = torch.zeros((m, L), dtype=torch.float32, device="cuda")
    abar = torch.zeros((m, L), dtype=torch.float32, device="cuda")
    h_ref, abars = h0.astype(np.float64), []
    for l in range(3):
        kc, vc = B.to_device(kcs[l], "f32"), B.to_device(vcs[l], "f32")
        ctx.d2c_refresh_layer(l, hidden, idx, S, kc, vc, L, abar, roll)
        h_ref, a = O.refresh_layer(od, mdl["layers"][l], h_ref, S, kcs[l].astype(np.float64), vcs[l].astype(np.float64))
        abars.append(a)
    infl = torch.zeros(L, dtype=torch.float32, device="cuda")
    ctx.d2c_influence(roll, idx, m, L, infl)
    torch.cuda.synchronize()
    C = O.rollout(abars, S, L)
    assert rel_l2(host(hidden), h_ref) < 1e-5
    assert rel_l2(host(roll), C[S]) < 1e-5
    assert rel_l2(host(infl), O.influence(C)) < 1e-5
    assert abs(float(host(infl).sum()) - L) < 1e-3
    ctx.close()


def test_refresh_layer_empty_and_errors(B):
    wd = W.ModelDims(1, 64, 4, 2, 16, 80, 64, dtype="f32")
    L = 20
    ctx, dims, _ = _ctx_for(B, wd, max_seq=L)
    say("refresh_layer m=0 and argument errors")
    hidden = torch.ones((4, 64), device="cuda")
    kc = torch.randn((L, dims.d_kv), device="cuda")
    vc = torch.randn((L, dims.d_kv), device="cuda")
    kc0, vc0, h0 = kc.clone(), vc.clone(), hidden.clone()
    idx = torch.tensor([1, 5, 6, 9], dtype=torch.int32, device="cuda")
    empty = np.zeros(0, np.int32)
    ctx.d2c_refresh_layer(0, hidden, idx, empty, kc, vc, L, None, None)                # m = 0: nothing touched
    torch.cuda.synchronize()
    assert torch.equal(kc, kc0) and torch.equal(vc, vc0) and torch.equal(hidden, h0)
    for bad in ([5, 1, 6, 9], [1, 5, 5, 9], [1, 5, 6, 20], [-1, 5, 6, 9]):
        with pytest.raises(B.D2CError) as ei:
            ctx.d2c_refresh_layer(0, hidden, idx, np.array(bad, np.int32), kc, vc, L, None, None)
        assert ei.value.code == B.D2C_EINVAL
    with pytest.raises(B.D2CError) as ei:
        ctx.d2c_refresh_layer(0, hidden, idx, np.array([1, 5, 6, 9], np.int32), kc, vc, L + 1, None, None)
    assert ei.value.code == B.D2C_ESHAPE
    with pytest.raises(B.D2CError) as ei:
        ctx.d2c_refresh_layer(3, hidden, idx, np.array([1, 5, 6, 9], np.int32), kc, vc, L, None, None)
    assert ei.value.code == B.D2C_EINVAL
    torch.cuda.synchronize()
    assert torch.equal(kc, kc0) and torch.equal(vc, vc0) and torch.equal(hidden, h0)   # nothing written on error
    ctx.close()


# ------------------------------------------------------------------ selection
def _run_select(B, ctx, prm, logits, logit_pos, y, is_masked, P, conf, pred, c, score_over_influence=False):
    L = len(y)
    dev = "cuda"
    t = {
        "tokens": torch.from_numpy(y.astype(np.int32)).to(dev), "is_masked": torch.from_numpy(is_masked.astype(np.uint8)).to(dev),
        "conf": torch.from_numpy(conf.astype(np.float32)).to(dev), "pred": torch.from_numpy(pred.astype(np.int32)).to(dev),
        "influence": torch.from_numpy(c.astype(np.float32)).to(dev),
    }
    for name in ("mstar", "u_set", "decode_idx", "s_next", "s_rows_next"):
        t[name] = torch.full((L,), -1, dtype=torch.int32, device=dev)
    t["counts"] = torch.zeros(B.N_COUNTS, dtype=torch.int32, device=dev)
    t["score"] = t["influence"] if score_over_influence else torch.zeros(L, dtype=torch.float32, device=dev)
    lg = torch.from_numpy(logits).to(dev) if len(logit_pos) else None
    lp = torch.from_numpy(logit_pos.astype(np.int32)).to(dev) if len(logit_pos) else None
    ctx.d2c_select(prm, lg, lp, len(logit_pos), t["tokens"], t["is_masked"], L, P, t["conf"], t["pred"], t["influence"],
                   t["mstar"], t["u_set"], t["decode_idx"], t["s_next"], t["s_rows_next"], t["counts"], t["score"])
    torch.cuda.synchronize()
    cnt = t["counts"].cpu().numpy()
    res = {k: v.cpu().numpy() for k, v in t.items()}
    res["mstar"] = res["mstar"][: cnt[B.CNT_MSTAR]]
    res["u_set"] = res["u_set"][: cnt[B.CNT_U]]
    res["decode_idx"] = res["decode_idx"][: cnt[B.CNT_DECODE]]
    res["s_next"] = res["s_next"][: cnt[B.CNT_S]]
    res["s_rows_next"] = res["s_rows_next"][: cnt[B.CNT_NEXT_ROWS]]
    return res, cnt


SELECT_CASES = [
    # L, P, vocab, block_len, k, n_unmask, p, sigma, frac_known, cand_mode, skewed[, threshold, conf_decode]
    (128, 64, 1024, 32, 8, 1, 0.9, 10.0, 0.0, 0, False),
    (128, 64, 1024, 32, 8, 1, 0.9, 10.0, 0.4, 0, True),
    (512, 256, 126464, 32, 32, 1, 0.1, 10.0, 0.3, 0, True),      # LLaDA-8B-shaped step, full vocabulary
    (768, 512, 152064, 32, 32, 1, 0.1, 10.0, 0.6, 0, False),     # Dream-7B-shaped
    (3072, 2048, 4096, 64, 32, 2, 0.1, 10.0, 0.5, 0, True),      # long context
    (3072, 2048, 4096, 1024, 32, 2, 0.1, 40.0, 0.5, 0, True),    # fully non-autoregressive: one block
    (333, 100, 777, 50, 7, 3, 0.35, 3.0, 0.5, 1, True),          # ragged everything, literal candidate mode
    (64, 8, 64, 16, 100, 100, 1.0, 10.0, 0.2, 0, False),         # select-all switch, unmask the whole block
    (40, 40, 64, 8, 4, 1, 0.5, 10.0, 0.0, 0, False),             # nothing masked
    (97, 0, 64, 32, 5, 1, 0.0, 10.0, 0.1, 0, True),              # no prompt, p = 0
    (512, 256, 4096, 32, 8, 1, 0.1, 10.0, 0.3, 0, True, 0.5, 0),     # parallel decoding: threshold on s^i
    (512, 256, 4096, 32, 8, 2, 0.1, 10.0, 0.3, 0, True, 0.0, 1),     # decode by confidence alone
    (300, 100, 512, 64, 4, 1, 0.2, 5.0, 0.5, 1, False, 0.9, 1),      # both, literal candidate mode
]


@pytest.mark.parametrize("case", SELECT_CASES, ids=[str(i) for i in range(len(SELECT_CASES))])
def test_select_parity(B, case):
    L, P, V, blk, k, nu, p, sigma, frac, mode, skew = case[:11]
    thr, cdec = (case[11], case[12]) if len(case) > 11 else (0.0, 0)
    say(f"select L={L} P={P} V={V} block={blk} k={k} n_unmask={nu} p={p} sigma={sigma} mode={mode} thr={thr} cdec={cdec}")
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
    mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)      # the selection never touches them
    ctx = B.Context(wd, mdl, L)
    seed = L + V
    is_masked = W.random_mask(seed, L, P, frac).astype(bool) if L > P else np.zeros(L, bool)
    y = np.where(is_masked, wd.mask_id, 7).astype(np.int32)
    conf0 = W.random_scores(seed, L)
    pred0 = (np.arange(L) * 7 % V).astype(np.int32)
    c = W.skewed_influence(seed, L) if skew else (W.random_scores(seed + 1, L) + np.float32(0.5))
    c[3 % L] = c[(L // 2)] = c[L - 1]                                     # exact ties in the influence
    masked_pos = np.flatnonzero(is_masked)
    logit_pos = masked_pos[:: 3][:16]                                     # rows that were in this step's forward
    logits = W.logits_rows(seed, len(logit_pos), V) if len(logit_pos) else np.zeros((0, V), np.float32)
    if len(logit_pos) > 1:
        logits[1, 5] = logits[1, 2] = logits[1].max() + 1.0               # tied maxima: lowest index wins
    prm = B.make_params(sigma, k, p, blk, nu, mode, thr, cdec)
    res, cnt = _run_select(B, ctx, prm, logits, logit_pos, y, is_masked, P, conf0, pred0, c)

    # Eq. 1
    conf_ref, pred_ref = conf0.astype(np.float64), pred0.copy()
    if len(logit_pos):
        s, xh = O.confidence(logits)
        conf_ref[logit_pos], pred_ref[logit_pos] = s, xh
    np.testing.assert_array_equal(res["pred"], pred_ref)
    np.testing.assert_allclose(res["conf"], conf_ref, rtol=1e-5)
    # Eq. 3: scores within tolerance
    oprm = O.Params(sigma=sigma, k=k, p=p, block_len=blk, n_unmask=nu, cand_mode=mode, threshold=thr, conf_decode=cdec)
    sel = O.select(oprm, is_masked, P, conf_ref.astype(np.float32), c)
    lo, hi = sel["block"]
    cand1 = np.array([i for i in range(lo, hi) if is_masked[i]], np.int64)
    assert (cnt[B.CNT_BLOCK_LO], cnt[B.CNT_BLOCK_HI]) == (lo, hi)
    if len(cand1):
        np.testing.assert_allclose(res["score"][cand1], sel["score"][cand1], rtol=1e-5)
    # Eq. 4 and the decode set: integer-exact on the score array the GPU itself produced
    np.testing.assert_array_equal(res["mstar"], O.top_k_select(res["score"], cand1, k))
    dec_ref = O.top_k_select(res["conf"] if cdec else res["score"], cand1, nu)      # on the GPU's own float arrays
    if thr > 0:
        dec_ref = np.union1d(dec_ref, cand1[res["conf"][cand1] > np.float32(thr)]).astype(np.int32)
    np.testing.assert_array_equal(res["decode_idx"], dec_ref)
    if topk_margin(sel["score"], cand1, k) > 1e-4:
        np.testing.assert_array_equal(res["mstar"], sel["mstar"])
    conf_margin = np.min(np.abs(conf_ref[cand1] - thr) / max(thr, 1e-9)) if thr > 0 and len(cand1) else 1.0
    if topk_margin(conf_ref if cdec else sel["score"], cand1, nu) > 1e-4 and conf_margin > 1e-4:
        np.testing.assert_array_equal(res["decode_idx"], sel["decode"])
    # stage 2 is decided on the given float32 influence array: bit-exact always
    cand2 = np.flatnonzero(~is_masked) if mode == 0 else np.setdiff1d(np.arange(L), res["mstar"])
    np.testing.assert_array_equal(res["u_set"], O.top_p_select(c, cand2, p))
    np.testing.assert_array_equal(res["s_next"], np.union1d(np.union1d(res["mstar"], res["decode_idx"]), res["u_set"]))
    # Eq. 2
    y_ref, m_ref = y.copy(), is_masked.copy()
    y_ref[res["decode_idx"]] = pred_ref[res["decode_idx"]]
    m_ref[res["decode_idx"]] = False
    np.testing.assert_array_equal(res["tokens"], y_ref)
    np.testing.assert_array_equal(res["is_masked"].astype(bool), m_ref)
    np.testing.assert_array_equal(res["s_rows_next"], np.flatnonzero(m_ref[res["s_next"]]))
    assert cnt[B.CNT_MASKED] == int(m_ref.sum())
    ctx.close()


def test_select_large_equal_scores_and_errors(B):
    """All scores equal: top-k takes the lowest indices, top-p the first floor(p n)+1 known tokens."""
    L, P, V = 256, 100, 64
    say("select equal scores")
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(wd, 0)
    ctx = B.Context(wd, mdl, L)
    is_masked = np.zeros(L, bool); is_masked[P:] = True
    y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
    # conf chosen so that D * conf is the same float for every candidate is impossible in general (D varies);
    # sigma huge makes D constant instead
    conf = np.full(L, 0.25, np.float32)
    c = np.ones(L, np.float32)
    prm = B.make_params(1e6, 5, 0.25, L, 2, 0)
    res, cnt = _run_select(B, ctx, prm, np.zeros((0, V), np.float32), np.zeros(0, np.int32), y, is_masked, P, conf,
                           np.zeros(L, np.int32), c)
    assert list(res["mstar"]) == [P, P + 1, P + 2, P + 3, P + 4]
    assert list(res["decode_idx"]) == [P, P + 1]
    assert list(res["u_set"]) == list(range(int(0.25 * P) + 1))
    for bad in (dict(sigma=0.0), dict(k=-1), dict(block_len=0), dict(p=-0.5), dict(cand_mode=2), dict(threshold=-1.0),
                dict(conf_decode=3), dict(rollout_layers=-2)):
        kw = dict(sigma=10.0, k=4, p=0.1, block_len=32, n_unmask=1, cand_mode=0)
        kw.update(bad)
        with pytest.raises(B.D2CError) as ei:
            _run_select(B, ctx, B.make_params(**kw), np.zeros((0, V), np.float32), np.zeros(0, np.int32), y, is_masked,
                        P, conf, np.zeros(L, np.int32), c)
        assert ei.value.code == B.D2C_EINVAL
    ctx.close()


@pytest.mark.parametrize("P,blk,inside", [(20, 8, 17), (20, 8, 3), (5, 8, 2)])
def test_select_masked_position_inside_prompt(B, P, blk, inside):
    """A masked position before the end of the prompt (legal input, not produced by the decoding loop): blocks
    are counted from the prompt's end in both directions, so the current block is the one holding it."""
    L, V = 64, 64
    say(f"select with a masked prompt position P={P} block={blk} inside={inside}")
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    ctx = B.Context(wd, W.model_weights(wd, 0), L)
    is_masked = np.zeros(L, bool)
    is_masked[[inside, inside + 1, 40, 41]] = True
    y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
    conf = W.random_scores(P, L)
    c = W.random_scores(P + 1, L) + np.float32(0.5)
    res, cnt = _run_select(B, ctx, B.make_params(3.0, 1, 0.2, blk, 1, 0), np.zeros((0, V), np.float32),
                           np.zeros(0, np.int32), y, is_masked, P, conf, np.zeros(L, np.int32), c)
    sel = O.select(O.Params(sigma=3.0, k=1, p=0.2, block_len=blk, n_unmask=1), is_masked, P, conf, c)
    assert (cnt[B.CNT_BLOCK_LO], cnt[B.CNT_BLOCK_HI]) == sel["block"]
    lo, hi = sel["block"]
    assert lo <= inside < hi
    cand1 = np.array([i for i in range(lo, hi) if is_masked[i]], np.int64)
    np.testing.assert_array_equal(res["mstar"], O.top_k_select(res["score"], cand1, 1))
    np.testing.assert_array_equal(res["decode_idx"], O.top_k_select(res["score"], cand1, 1))
    np.testing.assert_array_equal(res["u_set"], sel["u"])
    ctx.close()


def test_tunables_belong_to_a_context(B):
    """Two live contexts with different tunables give the launch shapes each asked for, a live context can be
    re-tuned, and the pre-tiled weight copies can only be chosen at init."""
    say("per-context tunables")
    wd = W.ModelDims(1, 256, 4, 4, 64, 80, 64, dtype="bf16")
    mdl = W.model_weights(wd, 0)
    ctx_a = B.Context(wd, mdl, 64, tunables={"gemm_waves": 4, "gemm_max_splits": 1})
    ctx_b = B.Context(wd, mdl, 64)
    m, N, K = 40, 1000, 520
    a = W.round_bf16(W.hidden_rows(11, m, K))
    w = W.round_bf16(W.hidden_rows(12, N, K, std=0.05))
    ref = a.astype(np.float64) @ w.astype(np.float64).T
    outs = []
    for ctx in (ctx_a, ctx_b, ctx_a):
        out = torch.zeros((m, N), dtype=torch.float32, device="cuda")
        ctx.d2c_linear(B.to_device(a, "bf16"), B.to_device(w, "bf16"), m, N, K, out)
        torch.cuda.synchronize()
        assert rel_l2(host(out), ref) < 1e-5
        outs.append(out)
    assert torch.equal(outs[0], outs[2])                       # context a is unaffected by what b ran in between
    ctx_b.set_tunable("gemm_waves", 10)
    out = torch.zeros((m, N), dtype=torch.float32, device="cuda")
    ctx_b.d2c_linear(B.to_device(a, "bf16"), B.to_device(w, "bf16"), m, N, K, out)
    torch.cuda.synchronize()
    assert rel_l2(host(out), ref) < 1e-5
    with pytest.raises(B.D2CError) as ei:
        ctx_b.set_tunable("gemm_preshuffle", 0)
    assert ei.value.code == B.D2C_EINVAL
    with pytest.raises(B.D2CError) as ei:
        ctx_b.set_tunable("no_such_knob", 1)
    assert ei.value.code == B.D2C_EINVAL
    info = ctx_a.memory_info()
    assert info["total_bytes"] == ctx_a.workspace_bytes() and 0 < info["pretiled_weight_bytes"] < info["total_bytes"]
    ctx_a.close()
    ctx_b.close()


SELECT_EDGES = [
    # as SELECT_CASES: word and workgroup edges of the bitmaps, ranking by counting / by radix (256 candidates), long and
    # short.  Every candidate has a known token within 9 sigma (exp(-40)), so that no score is subnormal: there the
    # relative bound of 1e-5 on the score says nothing (one unit in the last place is more)
    (1, 0, 16, 4, 3, 1, 0.1, 10.0, 0.0, 0, False),
    (65, 1, 16, 64, 8, 2, 0.3, 10.0, 0.2, 0, True),
    (2048, 1024, 64, 256, 40, 3, 0.2, 30.0, 0.0, 0, True),
    (2049, 700, 64, 1349, 300, 7, 0.5, 10.0, 0.3, 1, True),
    (4096, 500, 64, 3596, 257, 256, 0.05, 15.0, 0.1, 0, False),
    (4096, 500, 64, 3596, 5, 40, 0.999, 300.0, 0.1, 1, True, 0.9, 1),
    (1500, 100, 64, 1400, 0, 0, 0.1, 1e6, 0.4, 0, True),
]


@pytest.mark.parametrize("case", SELECT_EDGES, ids=[str(c[0]) + "-" + str(i) for i, c in enumerate(SELECT_EDGES)])
def test_select_parity_at_the_edges(B, case):
    test_select_parity(B, case)


@pytest.mark.parametrize("L", [1, 64, 512, 513, 1024, 1025, 2048, 2049, 4096])
def test_select_halves_in_one_launch_and_in_two(B, L):
    """With logit rows the half of the selection that needs none runs beside Eq. 1, in another launch: the same sets and the same
    bits as in one launch (no logit rows; the confidences those of the first call)."""
    say(f"select in halves L={L}")
    V = 8196
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
    mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)
    ctx = B.Context(wd, mdl, L)
    rng = np.random.default_rng(L)
    for P, blk, k, nu, p, sigma, cdec in ((0, L, 300, 5, 0.3, 10.0, 0), (L // 3, 64, 8, 1, 0.1, 25.0, 1), (L // 2, 16, 0, 2, 1.0, 1e5, 0)):
        is_masked = rng.random(L) < 0.6; is_masked[:P] = False; is_masked[L - 1] = True
        y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
        pos = np.flatnonzero(is_masked)[:5]
        prm = B.make_params(sigma, k, p, blk, nu, 0, conf_decode=cdec)
        conf, c = rng.random(L).astype(np.float32), W.skewed_influence(L, L)
        two, _ = _run_select(B, ctx, prm, W.logits_rows(L, len(pos), V), pos, y, is_masked, P, conf, np.zeros(L, np.int32), c)
        one, _ = _run_select(B, ctx, prm, np.zeros((0, V), np.float32), pos[:0], y, is_masked, P, two["conf"], two["pred"], c)
        for name in two:
            np.testing.assert_array_equal(two[name], one[name], err_msg=name)
    ctx.close()


@pytest.mark.parametrize("rows", [1, 3, 6])
@pytest.mark.parametrize("V", [40, 8192, 8196, 20001, 40000])
def test_select_chunks_beside_a_first_half_and_alone(B, V, rows):
    """Eq. 1's chunks in the launch that does the first half as well (cand_mode 0) and in one of their own (1): odd and even counts
    of chunks, whole and ragged ones, rows that 16-byte loads take and rows that they do not.  Same bits, and the oracle's values."""
    say(f"select chunks V={V} rows={rows}")
    L = 64
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
    mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)
    ctx = B.Context(wd, mdl, L)
    is_masked = np.arange(L) >= 32
    y, pos = np.where(is_masked, wd.mask_id, 3).astype(np.int32), np.arange(32, 32 + rows)
    logits, zero = W.logits_rows(V, rows, V), np.zeros(L, np.int32)
    conf, pred = [], []
    for mode in (0, 1):
        res, _ = _run_select(B, ctx, B.make_params(10.0, 4, 0.3, 32, 1, mode), logits, pos, y, is_masked, 32, zero, zero, W.skewed_influence(L, L))
        conf.append(res["conf"]), pred.append(res["pred"])
    np.testing.assert_array_equal(conf[0], conf[1])
    np.testing.assert_array_equal(pred[0], pred[1])
    x = logits.astype(np.float64)
    np.testing.assert_array_equal(pred[0][pos], x.argmax(1))
    ref = 1.0 / np.exp(x - x.max(1, keepdims=True)).sum(1)
    np.testing.assert_allclose(conf[0][pos], ref, rtol=1e-5)          # sums of up to 40000 positive floats in chunks
    ctx.close()


@pytest.mark.parametrize("rows", [0, 5])
@pytest.mark.parametrize("mode", [0, 1])
@pytest.mark.parametrize("L", [100, 700, 2100])
def test_select_scores_over_the_influence(B, L, mode, rows):
    """score_out may be the influence's own buffer: the influence is read before the scores are written."""
    say(f"select, scores over the influence L={L} mode={mode} rows={rows}")
    V = 1024
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    ctx = B.Context(wd, W.model_weights(wd, 0), L)
    rng = np.random.default_rng(L)
    is_masked = rng.random(L) < 0.5; is_masked[: L // 3] = False; is_masked[L - 1] = True
    y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
    pos = np.flatnonzero(is_masked)[:rows]
    prm = B.make_params(10.0, 8, 0.3, 64, 1, mode)
    conf, c = rng.random(L).astype(np.float32), W.skewed_influence(L, L)
    args = (B, ctx, prm, W.logits_rows(L, rows, V), pos, y, is_masked, L // 3, conf, np.zeros(L, np.int32), c)
    apart, over = (_run_select(*args, score_over_influence=o)[0] for o in (False, True))
    for name in apart:
        if name != "influence":
            np.testing.assert_array_equal(apart[name], over[name], err_msg=name)
    ctx.close()


@pytest.mark.parametrize("L,n_masked", [(640, 600), (3000, 2900)])
def test_select_ties_beyond_the_counting_limit(B, L, n_masked):
    """More than 256 candidates, runs of equal scores and of equal influence: the lowest index of a run goes first."""
    say(f"select ties L={L}")
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, 64, dtype="f32")
    ctx = B.Context(wd, W.model_weights(wd, 0), L)
    is_masked = np.zeros(L, bool); is_masked[L - n_masked:] = True
    y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
    rng = np.random.default_rng(L)
    conf = rng.integers(1, 4, size=L).astype(np.float32) / 4
    c = rng.integers(0, 3, size=L).astype(np.float32)                       # masses 0, 1, 2: long runs, some of no mass
    for k, nu, p, mode in ((257, 9, 0.4, 1), (n_masked - 1, 300, 0.0, 0), (1, 1, 0.99999, 1)):
        prm = B.make_params(1e6, k, p, L, nu, mode, conf_decode=1)
        res, _ = _run_select(B, ctx, prm, np.zeros((0, 64), np.float32), np.zeros(0, np.int32), y, is_masked, L - n_masked, conf,
                             np.zeros(L, np.int32), c)
        cand1 = np.flatnonzero(is_masked)
        np.testing.assert_array_equal(res["mstar"], O.top_k_select(res["score"], cand1, k))
        np.testing.assert_array_equal(res["decode_idx"], O.top_k_select(conf, cand1, nu))
        cand2 = np.flatnonzero(~is_masked) if mode == 0 else np.setdiff1d(np.arange(L), res["mstar"])
        np.testing.assert_array_equal(res["u_set"], O.top_p_select(c, cand2, p))
    ctx.close()


@pytest.mark.parametrize("V", [40000, 126464, 8192 * 33])
def test_confidence_does_not_depend_on_the_other_rows(B, V):
    """A row's confidence and prediction have the same bits whether the call merges them inside the selection (up to 256
    rows) or in a launch of its own (more)."""
    L = 640
    say(f"confidence of the same rows in calls of 1, 256, 257 and 600 rows V={V}")
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
    mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)
    ctx = B.Context(wd, mdl, L)
    is_masked = np.ones(L, bool)
    y, zero = np.full(L, wd.mask_id, np.int32), np.zeros(L, np.float32)
    g = torch.Generator(device="cuda")
    g.manual_seed(3)
    logits = torch.randn((600, V), generator=g, device="cuda") * 2.0
    got = []
    for n in (1, 256, 257, 600):
        res, _ = _run_select(B, ctx, B.make_params(n_unmask=0), logits[:n].cpu().numpy(), np.arange(n), y, is_masked, 0, zero,
                             np.zeros(L, np.int32), zero + 1.0)
        got.append((res["conf"][:n], res["pred"][:n]))
    for conf, pred in got[:-1]:
        np.testing.assert_array_equal(conf, got[-1][0][: len(conf)])
        np.testing.assert_array_equal(pred, got[-1][1][: len(pred)])
    ctx.close()


def test_workspace_holds_the_chunk_triples_of_the_vocabulary(B):
    """Eq. 1's chunk triples are held for every row of a group and every chunk that the vocabulary has, no more: 8192 entries
    (one chunk) against 65536 (eight), 4 sequences of 512 positions."""
    say("workspace of two vocabularies")
    ws = []
    for V in (8192, 65536):
        wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
        mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
        mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)
        ctx = B.Context(wd, mdl, 512, max_batch=4)
        info = ctx.memory_info()
        ws.append(info["total_bytes"] - info["pretiled_weight_bytes"])
        ctx.close()
    head_rows = 256
    assert ws[1] - ws[0] == head_rows * (65536 - 8192) * 4 + 4 * 512 * (8 - 1) * 3 * 4


@pytest.mark.parametrize("n_rows,V", [(1, 8192), (17, 8193), (256, 40000), (257, 40000), (40, 8192 * 33)])
def test_select_merges_every_logit_row(B, n_rows, V):
    """Eq. 1 with the chunks merged beside the selection (up to 256 rows, up to 32 chunks or more) and by a launch of its own."""
    say(f"select rows {n_rows} x {V}")
    L = 600
    wd = W.ModelDims(1, 64, 4, 4, 16, 80, V, dtype="f32")
    mdl = W.model_weights(W.ModelDims(1, 64, 4, 4, 16, 80, 8, dtype="f32"), 0)
    mdl["tok_emb"] = mdl["lm_head"] = np.zeros((V, 64), np.float32)
    ctx = B.Context(wd, mdl, L)
    is_masked = np.zeros(L, bool); is_masked[100:] = True
    y = np.where(is_masked, wd.mask_id, 3).astype(np.int32)
    pos = (100 + np.arange(n_rows)).astype(np.int32)
    logits = W.logits_rows(n_rows, n_rows, V)
    logits[0, V - 1] = logits[0, 1] = logits[0].max() + 1.0                  # tied maxima in the first and last chunk
    prm = B.make_params(10.0, 32, 0.1, 32, 1, 0)
    res, _ = _run_select(B, ctx, prm, logits, pos, y, is_masked, 100, np.zeros(L, np.float32), np.zeros(L, np.int32),
                         W.skewed_influence(1, L))
    s, xh = O.confidence(logits)
    np.testing.assert_array_equal(res["pred"][pos], xh)
    np.testing.assert_allclose(res["conf"][pos], s, rtol=1e-5)
    ctx.close()


@pytest.mark.parametrize("H,Hkv,dh,L,m", [(4, 4, 64, 1, 1), (4, 2, 64, 129, 17), (6, 3, 128, 100, 33), (3, 1, 64, 1000, 129),
                                          (2, 2, 128, 16, 16), (4, 4, 64, 143, 128)])
def test_attention_parity_f32_tiles(B, H, Hkv, dh, L, m):
    """fp32 on the matrix cores: one key, ragged last key and query tiles, waves without a key tile, grouped heads."""
    say(f"attention f32 tiles H={H} Hkv={Hkv} dh={dh} L={L} m={m}")
    _attention_parity(B, "f32", H, Hkv, dh, L, m)


def test_attention_f32_unaligned_rows(B):
    """Buffers that are not 16-byte aligned take the per-row kernels: the same result up to summation order."""
    H, dh, L, m = 4, 64, 77, 19
    say("attention f32 unaligned")
    wd = W.ModelDims(1, H * dh, H, H, dh, 64, 64, dtype="f32")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L)
    case = W.attention_case(1, H, H, dh, L, m, dtype="f32")
    idx = torch.from_numpy(case["idx"]).cuda()
    got = []
    for off in (0, 1):
        def put(a):
            t = torch.zeros(a.size + 4, device="cuda")[off: off + a.size].view(a.shape)
            t.copy_(torch.from_numpy(a))
            return t
        q, kc, vc = put(case["q"]), put(case["k_cache"]), put(case["v_cache"])
        out, abar = torch.zeros_like(q), torch.zeros((m, L), device="cuda")
        ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, out, abar)
        torch.cuda.synchronize()
        got.append((host(out), host(abar)))
    assert rel_l2(got[0][0], got[1][0]) < 1e-6 and rel_l2(got[0][1], got[1][1]) < 1e-6
    ctx.close()


@pytest.mark.parametrize("dh", [64, 128])
@pytest.mark.parametrize("low", [-np.inf, np.finfo(np.float32).min])
def test_attention_f32_scores_of_minus_infinity(B, dh, low):
    """Keys whose scores are -inf, a whole key tile and the whole of a wave's keys among them, weigh nothing: the softmax of
    the others (K holds -inf, or the type's lowest value, which overflows in the product)."""
    H, L, m = 2, 300, 17
    say(f"attention f32 scores of -inf dh={dh} low={low}")
    wd = W.ModelDims(1, H * dh, H, H, dh, 64, 64, dtype="f32")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L)
    case = W.attention_case(5, H, H, dh, L, m, dtype="f32")
    q, k = np.abs(case["q"]) + 1.0, case["k_cache"].copy()
    gone = np.zeros(L, bool)
    gone[0:40] = gone[128:144] = gone[256:272] = gone[299] = True      # tiles 0, 8 and 16: all keys of the first wave
    k[gone, 3] = k[gone, dh + 3] = low
    out, abar = torch.zeros((m, H * dh), device="cuda"), torch.zeros((m, L), device="cuda")
    ctx.d2c_attention(torch.from_numpy(q).cuda(), torch.from_numpy(case["idx"]).cuda(), m, None, None, torch.from_numpy(k).cuda(),
                      torch.from_numpy(case["v_cache"]).cuda(), L, out, abar)
    torch.cuda.synchronize()
    o_ref, a_ref = O.selective_attention(q, k[~gone].astype(np.float64), case["v_cache"][~gone].astype(np.float64), H, H, dh)
    for r in range(m):
        assert rel_l2(host(out)[r], o_ref[r]) < TOL["f32"] and rel_l2(host(abar)[r, ~gone], a_ref[r]) < TOL["f32"], f"row {r}"
    assert (host(abar)[:, gone] == 0.0).all()
    ctx.close()


@pytest.mark.parametrize("L,m", [(1, 1), (40, 16), (131, 64), (200, 65), (791, 768), (800, 769), (1900, 1793)])
def test_rollout_update_and_influence_at_the_size_rules(B, L, m):
    """The second layer's rollout update for every form of it (operand gathered, dense, strip in LDS or not) and Eq. 9,
    against the formula in fp64 on the GPU's own head averages.  Bound: sums of at most 1793 terms of a row that sums to
    one, in fp32 (1793 roundings of 6e-8 of a value below 1, most of which cancel): 1e-5 relative to the row."""
    say(f"rollout L={L} m={m}")
    wd = W.ModelDims(2, 64, 4, 4, 16, 64, 64, dtype="f32")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L, n_layers=2)
    S = W.distinct_sorted_rows(1, L, m)
    idx = torch.from_numpy(S).cuda()
    h = torch.from_numpy(W.hidden_rows(1, m, 64)).cuda()
    kc, vc = (torch.from_numpy(W.hidden_rows(s, 2 * L, 64).reshape(2, L, 64)).cuda() for s in (2, 3))
    avg, roll = torch.zeros((m, L), device="cuda"), torch.full((m, L), 7.0, device="cuda")
    got = []
    for l in range(2):
        ctx.d2c_refresh_layer(l, h, idx, S, kc[l], vc[l], L, avg, roll)
        got.append((host(avg).astype(np.float64), host(roll).astype(np.float64)))
    c = torch.zeros(L, device="cuda")
    ctx.d2c_influence(roll, idx, m, L, c)
    torch.cuda.synchronize()
    eye = np.zeros((m, L)); eye[np.arange(m), S] = 1.0
    outside = np.ones(L); outside[S] = 0.0
    prev = eye
    for a, r in got:
        ref = 0.5 * (a[:, S] @ prev + a * outside + prev)
        for i in range(m):
            assert rel_l2(r[i], ref[i]) < 1e-5, f"rollout row {i}"
        prev = r
    np.testing.assert_allclose(host(c), outside + prev.sum(0), rtol=1e-5)
    ctx.close()


@pytest.mark.parametrize("kernel", [2, 3])
@pytest.mark.parametrize("m,N,K", [(257, 40, 256), (289, 1000, 512), (385, 264, 768), (513, 256, 2304), (777, 72, 256), (1153, 520, 512),
                                   (289, 16391, 2304), (513, 8200, 4352), (1500, 200, 1280), (900, 3000, 1536)])
def test_linear_parity_many_rows(B, m, N, K, kernel):
    """Row-major weights in both kernels for many rows (gemm_wide_tiles 2: two row chunks per workgroup, 3: one): odd counts of
    row chunks, 5 to 8 row tiles, 256 and 192 columns, ragged rows and columns, one chunk pair of k and several splits."""
    test_linear_parity(B, "bf16", m, N, K, tunables={"gemm_wide_tiles": kernel})


@pytest.mark.parametrize("kernel", [0, 2, 3])
def test_linear_many_rows_start_chunk(B, kernel):
    """gemm_rot moves the first chunk of a workgroup's walk over k in every kernel for many rows: the same sums in another
    order, so other low bits somewhere in 300 x 1000 results of 2304 products (one in four rounds differently), same values."""
    m, N, K = 300, 1000, 2304
    say(f"linear many rows, start chunk, kernel {kernel}")
    wd = W.ModelDims(1, 256, 4, 4, 64, 80, 64, dtype="bf16")
    ctx, _, _ = _ctx_for(B, wd, max_seq=m, tunables={"gemm_wide_tiles": kernel, "gemm_max_splits": 1})
    a, w = W.round_bf16(W.hidden_rows(11, m, K)), W.round_bf16(W.hidden_rows(12, N, K, std=0.05))
    ad, wdv = B.to_device(a, "bf16"), B.to_device(w, "bf16")
    ref = a.astype(np.float64) @ w.astype(np.float64).T
    got = []
    for rot in (0, 5):
        ctx.set_tunable("gemm_rot", rot)
        out = torch.full((m, N), 7.0, device="cuda")
        ctx.d2c_linear(ad, wdv, m, N, K, out)
        torch.cuda.synchronize()
        assert rel_l2(host(out), ref) < 1e-5
        got.append(out)
    assert not torch.equal(got[0], got[1]) and torch.equal(got[0][:, :128], got[1][:, :128])     # the first column block starts at 0
    ctx.close()


@pytest.mark.parametrize("m,N,K", [(193, 40, 128), (200, 520, 640), (256, 1000, 384)])
def test_linear_parity_two_row_chunks(B, m, N, K):
    """193-256 rows as one workgroup row of the same kernel, counts of 128-element chunks that are odd among them."""
    test_linear_parity(B, "bf16", m, N, K, tunables={"gemm_wide_tiles": 2})


@pytest.mark.parametrize("m,N,K", [(300, 33000, 1280), (400, 520, 512), (256, 512 * 96, 128)])
def test_linear_parity_many_rows_by_shape(B, m, N, K):
    """The planner's own choice (two row chunks per workgroup, two column tiles per wave, 193-256 rows that fill the chip)."""
    test_linear_parity(B, "bf16", m, N, K)


@pytest.mark.parametrize("kernel", [2, 3])
@pytest.mark.parametrize("m", [257, 300, 449, 700])
def test_refresh_layer_parity_many_rows(B, m, kernel):
    """The same with pre-tiled weights and the gated epilogue; widths that leave the last column block ragged."""
    _refresh_layer_parity(B, f"bf16-{m}-rows", W.ModelDims(1, 512, 4, 4, 128, 1280, 64, dtype="bf16"), m + 30, m,
                          tunables={"gemm_wide_tiles": kernel})


@pytest.mark.parametrize("m,F", [(257, 1280), (300, 208), (449, 1024)])
def test_gated_epilogue_of_large_gates(B, m, F):
    """Gates far beyond 87, where exp(-g) leaves the range of a float, beside ordinary ones: whole waves of either, and mixed ones."""
    say(f"gated epilogue, large gates m={m} F={F}")
    wd = W.ModelDims(1, 512, 4, 4, 128, F, 64, dtype="bf16")
    mdl = W.model_weights(wd, 0)
    gate = mdl["layers"][0]["w_gate_up"]
    gate[: F // 3] *= 400.0                                                 # gates with a standard deviation of 180
    gate[F // 2: F: 7] *= 100.0
    mdl["layers"][0]["w_gate_up"] = W.round_bf16(gate)
    ctx = B.Context(wd, mdl, m, tunables={"gemm_wide_tiles": 2})
    S, h0 = np.arange(m, dtype=np.int32), W.hidden_rows(4, m, wd.d_model, std=0.5)
    kc, vc = (np.zeros((m, wd.d_kv)) for _ in range(2))
    hidden, kd, vd = torch.from_numpy(h0).cuda(), B.to_device(kc, "bf16"), B.to_device(vc, "bf16")
    ctx.d2c_refresh_layer(0, hidden, torch.from_numpy(S).cuda(), S, kd, vd, m, None, None)
    torch.cuda.synchronize()
    h_ref, _ = O.refresh_layer(oracle_dims(wd), mdl["layers"][0], h0, S, kc, vc)
    for r in range(m):
        assert rel_l2(host(hidden)[r], h_ref[r]) < TOL["bf16"], f"hidden row {r}"
    ctx.close()


@pytest.mark.parametrize("m,F", [(200, 208), (200, 1040), (250, 208), (250, 1040)])
def test_refresh_layer_parity_gated_pairs_in_one_wave(B, m, F):
    """193-256 rows in the kernel for many rows: four column tiles a wave, 7 and 8 row tiles, cut-off rows and column blocks."""
    _refresh_layer_parity(B, f"bf16-{m}-rows-{F}", W.ModelDims(1, 512, 4, 4, 128, F, 64, dtype="bf16"), m + 30, m,
                          tunables={"gemm_wide_tiles": 2})


@pytest.mark.parametrize("m,F", [(257, 1280), (300, 208), (449, 1024), (200, 208), (250, 1040)])
def test_gated_epilogue_of_ordinary_gates_beside_large_ones(B, m, F):
    """Every seventh hidden column has gates far beyond 87 and half of the output columns do not see those: the ordinary gates of
    mixed waves on their own.  200 and 250 rows: four column tiles a wave, the others three."""
    say(f"gated epilogue, ordinary gates beside large ones m={m} F={F}")
    wd = W.ModelDims(1, 512, 4, 4, 128, F, 64, dtype="bf16")
    mdl = W.model_weights(wd, 0)
    layer, half = mdl["layers"][0], wd.d_model // 2
    layer["w_gate_up"][0:F:7] = W.round_bf16(layer["w_gate_up"][0:F:7] * 400.0)
    layer["w_down"][:half, 0:F:7] = 0.0
    layer["w_down"][:half] *= 16.0                                          # 2^4: the values stay bf16; the FFN is most of the sum
    ctx = B.Context(wd, mdl, m, tunables={"gemm_wide_tiles": 2})
    S, h0 = np.arange(m, dtype=np.int32), W.hidden_rows(4, m, wd.d_model, std=0.5)
    kc, vc = (np.zeros((m, wd.d_kv)) for _ in range(2))
    hidden, kd, vd = torch.from_numpy(h0).cuda(), B.to_device(kc, "bf16"), B.to_device(vc, "bf16")
    ctx.d2c_refresh_layer(0, hidden, torch.from_numpy(S).cuda(), S, kd, vd, m, None, None)
    torch.cuda.synchronize()
    h_ref, _ = O.refresh_layer(oracle_dims(wd), layer, h0, S, kc, vc)
    for r in range(m):
        assert rel_l2(host(hidden)[r, :half], h_ref[r, :half]) < TOL["bf16"], f"hidden row {r}"
        assert rel_l2(host(hidden)[r, half:], h_ref[r, half:]) < TOL["bf16"], f"hidden row {r}, large gates"
    ctx.close()


@pytest.mark.parametrize("m,F", [(300, 16400), (457, 16400), (200, 16400), (250, 16400)])
def test_gated_epilogue_of_a_row_depends_on_that_row_alone(B, m, F):
    """A row of each 16 gets gates beyond 87: every other row keeps its bits.  The rows meet in no other place: without q, K and V
    of their own all of them attend alike.  300 and 457 rows: pairs of column tiles across two waves; 200 and 250: inside one.
    As many values as it takes for the last place of a float to show, which changes one bf16 value in 65536."""
    say(f"gated epilogue, rows apart m={m} F={F}")
    wd = W.ModelDims(1, 256, 4, 4, 64, F, 64, dtype="bf16")
    mdl = W.model_weights(wd, 0)
    layer = mdl["layers"][0]
    layer["wqkv"][:] = 0.0
    layer["wo"][0] = 0.0                                                    # column 0 of the residual stays what it is
    layer["w_gate_up"][:F, 0] = W.round_bf16(W.hidden_rows(7, 1, F, std=20.0)[0])      # and adds to the gates where it is not 0
    ctx = B.Context(wd, mdl, m, tunables={"gemm_wide_tiles": 2})
    S, moved = np.arange(m, dtype=np.int32), np.arange(5, m, 16)
    idx, others = torch.from_numpy(S).cuda(), np.setdiff1d(S, moved)
    for seed in range(8):
        h0, got = W.hidden_rows(seed, m, wd.d_model, std=0.5), []
        for x in (0.0, 20.0):
            h0[:, 0] = 0.0
            h0[moved, 0] = x
            hidden = torch.from_numpy(h0).cuda()
            kd, vd = (B.to_device(np.zeros((m, wd.d_kv)), "bf16") for _ in range(2))
            ctx.d2c_refresh_layer(0, hidden, idx, S, kd, vd, m, None, None)
            torch.cuda.synchronize()
            got.append(host(hidden))
        np.testing.assert_array_equal(got[0][others], got[1][others], err_msg=f"rows of draw {seed}")
        assert (got[0][moved] != got[1][moved]).any(axis=1).all()
    ctx.close()


@pytest.mark.parametrize("m,N,K", [(300, 520, 512), (449, 264, 2304), (230, 520, 640)])
def test_linear_many_rows_unaligned(B, m, N, K):
    """Activations that are not 16-byte aligned cannot be staged straight into LDS: gemm_wide_kernel's splits by another kernel
    (one row chunk per workgroup, or two column tiles per wave where a split is no pair of chunks)."""
    say(f"linear many rows, unaligned activations m={m} N={N} K={K}")
    wd = W.ModelDims(1, 512, 4, 4, 128, 512, 64, dtype="bf16")
    ctx, _, _ = _ctx_for(B, wd, max_seq=m, tunables={"gemm_wide_tiles": 2})
    a_np, w_np = (W.round_bf16(W.hidden_rows(s, r, K)) for s, r in ((1, m), (2, N)))
    a0, w = (torch.from_numpy(x).to(torch.bfloat16).cuda() for x in (a_np, w_np))
    ref = a_np.astype(np.float64) @ w_np.astype(np.float64).T
    for off in (0, 1):
        a = torch.zeros(m * K + 8, dtype=torch.bfloat16, device="cuda")[off: off + m * K].view(m, K)
        a.copy_(a0)
        out = torch.full((m, N), 7.0, device="cuda")
        ctx.d2c_linear(a, w, m, N, K, out)
        torch.cuda.synchronize()
        assert rel_l2(host(out), ref) < 1e-5
    ctx.close()


@pytest.mark.parametrize("H,Hkv,dh,L,m", [(8, 8, 128, 1, 1), (8, 2, 128, 33, 15), (8, 8, 128, 257, 1), (8, 2, 128, 289, 15),
                                          (32, 32, 128, 513, 17), (28, 4, 128, 1025, 47), (4, 4, 64, 511, 16), (4, 1, 64, 351, 33),
                                          (40, 8, 128, 1024, 120), (40, 8, 128, 351, 113), (40, 8, 128, 350, 113)])
def test_attention_parity_staged_rows(B, H, Hkv, dh, L, m):
    """The few-row kernel with K and Q staged through LDS (always where two workgroups share the columns, from 351 keys on
    elsewhere): one key, ragged pairs, waves without a pair, with one and with several, both widths of the output share; and the
    same values with a K cache that is not 16-byte aligned (loads in operand order), bit for bit."""
    say(f"attention staged H={H} Hkv={Hkv} dh={dh} L={L} m={m}")
    _attention_parity(B, "bf16", H, Hkv, dh, L, m, tunables={"attn_tiled_min_m": 1 << 30})
    wd = W.ModelDims(1, H * dh, H, Hkv, dh, 64, 64, dtype="bf16")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L, tunables={"attn_tiled_min_m": 1 << 30})
    case = W.attention_case(1, H, Hkv, dh, L, m, dtype="bf16")
    idx = torch.from_numpy(case["idx"]).cuda()
    got = []
    for off in (0, 1):
        kc = torch.zeros(L * Hkv * dh + 8, dtype=torch.bfloat16, device="cuda")[off: off + L * Hkv * dh].view(L, Hkv * dh)
        kc.copy_(B.to_device(case["k_cache"], "bf16"))
        q, vc = B.to_device(case["q"], "bf16"), B.to_device(case["v_cache"], "bf16")
        out = torch.zeros_like(q)
        ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, out, None)
        torch.cuda.synchronize()
        got.append(out)
    assert torch.equal(got[0], got[1])
    ctx.close()


@pytest.mark.parametrize("dtype,m,N,K", [("bf16", 1, 16, 392), ("bf16", 97, 1007, 1160), ("bf16", 113, 2600, 392), ("bf16", 145, 333, 1032),
                                         ("f32", 77, 2505, 68), ("f32", 120, 1000, 516), ("f32", 33, 26001, 196)])
def test_linear_parity_staged_weights(B, dtype, m, N, K):
    """Row-major weights staged through LDS (unsplit contractions of three chunks and more, float with five row tiles or a full
    round of workgroups): ragged last chunk and last rows, three slots, two slots (many rows, 10 waves) and none; and weights
    that are not 16-byte aligned, which take the loads in operand order: the same bits."""
    assert dtype == "bf16" or B.d2c_plan_projection(dtype, m, N, K, True)["waves"] != 4          # not the one-tile kernel's
    tun = {"gemm_max_splits": 1}
    test_linear_parity(B, dtype, m, N, K, tunables=tun)
    if dtype == "bf16":
        test_linear_parity(B, dtype, m, N, K, tunables={"gemm_waves": 10, **tun})
    wd = W.ModelDims(1, 128, 2, 2, 64, 128, 64, dtype=dtype)
    ctx, _, _ = _ctx_for(B, wd, max_seq=m, tunables=tun)
    t = B.torch_dtype(dtype)
    a = B.to_device(W.round_bf16(W.hidden_rows(1, m, K)), dtype)
    w0 = B.to_device(W.round_bf16(W.hidden_rows(2, N, K)), dtype)
    got = []
    for off in (0, 1):
        w = torch.zeros(N * K + 8, dtype=t, device="cuda")[off: off + N * K].view(N, K)
        w.copy_(w0)
        out = torch.zeros((m, N), device="cuda")
        ctx.d2c_linear(a, w, m, N, K, out)
        torch.cuda.synchronize()
        got.append(out)
    assert torch.equal(got[0], got[1])
    ctx.close()


@pytest.mark.parametrize("H,Hkv,dh,L,m", [(3, 1, 128, 1, 1), (4, 2, 64, 33, 15), (32, 32, 128, 513, 17), (28, 4, 128, 1025, 47),
                                          (6, 3, 64, 511, 33), (3, 1, 128, 257, 1), (3, 1, 128, 256, 1), (3, 3, 128, 8, 2),
                                          (5, 5, 64, 897, 3), (5, 5, 64, 896, 15), (5, 5, 64, 17, 16)])
def test_attention_average_staged_rows(B, H, Hkv, dh, L, m):
    """The head average with Q and K staged through LDS against a K cache that is not 16-byte aligned (loads in operand order):
    the same contraction order, so the same bits; waves without a head, heads that share K, ragged queries and keys."""
    say(f"attention average staged H={H} Hkv={Hkv} dh={dh} L={L} m={m}")
    _attention_parity(B, "bf16", H, Hkv, dh, L, m, tunables={"attn_tiled_min_m": 1 << 30})
    wd = W.ModelDims(1, H * dh, H, Hkv, dh, 64, 64, dtype="bf16")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L, tunables={"attn_tiled_min_m": 1 << 30})
    case = W.attention_case(1, H, Hkv, dh, L, m, dtype="bf16")
    idx = torch.from_numpy(case["idx"]).cuda()
    got = []
    for off in (0, 1):
        kc = torch.zeros(L * Hkv * dh + 8, dtype=torch.bfloat16, device="cuda")[off: off + L * Hkv * dh].view(L, Hkv * dh)
        kc.copy_(B.to_device(case["k_cache"], "bf16"))
        q, vc = B.to_device(case["q"], "bf16"), B.to_device(case["v_cache"], "bf16")
        avg = torch.zeros((m, L), device="cuda")
        ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, torch.zeros_like(q), avg)
        torch.cuda.synchronize()
        got.append(avg)
    assert torch.equal(got[0], got[1])
    ctx.close()


@pytest.mark.parametrize("H,Hkv,dh,L,m,waves", [(4, 2, 128, 1, 1, 0), (4, 2, 128, 64, 65, 4), (3, 1, 64, 65, 129, 0), (4, 4, 128, 128, 257, 8),
                                                (2, 1, 128, 193, 200, 8), (28, 4, 128, 777, 97, 0), (5, 5, 64, 320, 255, 8),
                                                (2, 2, 128, 1025, 33, 4)])
def test_attention_tiled_rows_straight_into_lds(B, H, Hkv, dh, L, m, waves):
    """The tiled kernels at the edges of their key blocks, query tiles and buffers, K and V rows staged straight into LDS; the
    same caches off their 16-byte alignment come through registers in the same order, so with the same bits."""
    say(f"attention tiled staging H={H} Hkv={Hkv} dh={dh} L={L} m={m} waves={waves}")
    m = min(m, L)
    tun = {"attn_tiled_min_m": 1, "attn_waves": waves}
    _attention_parity(B, "bf16", H, Hkv, dh, L, m, tunables=tun)
    wd = W.ModelDims(1, H * dh, H, Hkv, dh, 64, 64, dtype="bf16")
    ctx, _, _ = _ctx_for(B, wd, max_seq=L, tunables=tun)
    case = W.attention_case(1, H, Hkv, dh, L, m, dtype="bf16")
    idx = torch.from_numpy(case["idx"]).cuda()
    q = B.to_device(case["q"], "bf16")
    got = []
    for off_k, off_v in ((0, 0), (2, 0), (0, 4)):
        def put(a, off):
            t = torch.zeros(a.size + 8, dtype=torch.bfloat16, device="cuda")[off: off + a.size].view(a.shape)
            t.copy_(B.to_device(a, "bf16"))
            return t
        kc, vc = put(case["k_cache"], off_k), put(case["v_cache"], off_v)
        out, avg = torch.zeros_like(q), torch.zeros((m, L), device="cuda")
        ctx.d2c_attention(q, idx, m, None, None, kc, vc, L, out, avg)
        torch.cuda.synchronize()
        got.append((out, avg))
    for out, avg in got[1:]:
        assert torch.equal(out, got[0][0]) and torch.equal(avg, got[0][1])
    ctx.close()


@pytest.mark.parametrize("m,N,K", [(1, 1, 4), (15, 40, 60), (16, 63, 64), (17, 64, 68), (31, 65, 128), (33, 100, 132), (64, 250, 192),
                                   (65, 130, 196), (128, 1376, 256), (100, 256, 260), (128, 96, 688), (81, 60, 2048), (81, 60, 2052)])
def test_linear_f32_one_tile_per_wave(B, m, N, K):
    """Few rows and a short contraction in float: edges of rows, columns, chunks, splits, and the first contraction past them."""
    test_linear_parity(B, "f32", m, N, K)


@pytest.mark.parametrize("m", [1, 17, 128])
@pytest.mark.parametrize("wd", [W.ModelDims(1, 132, 2, 1, 32, 208, 64, dtype="f32"), W.ModelDims(1, 260, 4, 4, 16, 528, 64, dtype="f32")],
                         ids=["132", "260"])
def test_refresh_layer_f32_one_tile_per_wave(B, wd, m):
    """The same with pre-tiled weights and the gated epilogue: ragged last chunks, one contraction in one split and in two."""
    _refresh_layer_parity(B, f"f32-{wd.d_model}", wd, 131, m)


@pytest.mark.parametrize("dtype,m,N,K", [("bf16", 1, 650, 2048), ("bf16", 17, 3000, 4096), ("bf16", 70, 1000, 8192), ("bf16", 150, 520, 2048),
                                         ("bf16", 256, 300, 4096), ("bf16", 300, 1030, 2048), ("f32", 40, 3000, 1024), ("f32", 130, 200, 2048)])
def test_linear_rows_a_power_of_two_apart(B, dtype, m, N, K):
    """Row-major weights whose workgroups start their walks over k at different chunks."""
    for rot in (1, 3):
        test_linear_parity(B, dtype, m, N, K, tunables={"gemm_rot": rot})


@pytest.mark.parametrize("H,Hkv,dh,L,m", [(32, 32, 128, 1536, 16), (32, 32, 128, 1536, 17), (28, 4, 128, 1791, 47), (28, 4, 128, 1792, 17),
                                          (4, 2, 64, 1535, 1), (3, 1, 64, 2050, 40), (5, 5, 128, 1537, 1)])
def test_attention_few_rows_on_long_key_ranges(B, H, Hkv, dh, L, m):
    """Both sides of the lines between the few-row and the tiled kernels past 1024 keys, as the library chooses by itself."""
    say(f"attention few rows, long H={H} Hkv={Hkv} dh={dh} L={L} m={m}")
    _attention_parity(B, "bf16", H, Hkv, dh, L, m)


def _f32_parts(s):
    """float32 values as three bf16 pieces hi + mid / 2^8 + lo / 2^16, without a rounding"""
    s = np.asarray(s, np.float32)
    out = []
    for _ in range(3):
        hi = (s.view(np.uint32) & np.uint32(0xffff0000)).view(np.float32)
        out.append(hi)
        s = ((s - hi) * np.float32(256.0)).astype(np.float32)
    assert not s.any()
    return out


@pytest.mark.parametrize("dh", [64, 128])
def test_attention_row_does_not_depend_on_its_neighbours(B, dh):
    """A row's reference is raised by the row's own scores: here its second block of keys exceeds the reference by 8 within a
    rounding of the comparison, alone and beside a row that raises its own reference there; what was decided shows in the roundings
    of a third block 4.3 above the second."""
    scale = np.float32(1.0) / np.sqrt(np.float32(dh))
    c2 = np.float32(scale * np.float32(1.44269504088896341))
    rng = np.random.default_rng(3)
    pairs = {True: [], False: []}                            # (first block's maximum, second block's), by which rounding exceeds 8
    while min(len(p) for p in pairs.values()) < 6:
        s0 = np.float32(rng.uniform(20.0, 60.0))
        ref = np.float32(s0 * c2)
        s1 = np.float32((float(ref) + 8.0) / float(c2))
        for _ in range(4):
            fused = bool(np.float32(float(s1) * float(c2) - float(ref)) > 8.0)
            if fused != bool(np.float32(s1 * c2) > np.float32(ref + np.float32(8.0))):
                pairs[fused].append((s0, s1))
            s1 = np.nextafter(s1, np.float32(1e9))
    say(f"attention row beside another, head dimension {dh}")
    ctx, _, _ = _ctx_for(B, W.ModelDims(1, dh, 1, 1, dh, 64, 64, dtype="bf16"), max_seq=192, tunables={"attn_tiled_min_m": 1, "attn_max_splits": 1})
    q = np.zeros((2, dh), np.float32)
    q[0, :3] = 1.0, 2.0 ** -8, 2.0 ** -16
    q[1] = 2.0 * q[0]
    v = B.to_device(W.round_bf16(W.hidden_rows(21, 192, dh)), "bf16")
    for s0, s1 in pairs[True][:6] + pairs[False][:6]:
        s = np.concatenate([rng.uniform(0.0, s0, 64), rng.uniform(s0, 0.99 * s1, 64), rng.uniform(s0, s1, 64)]).astype(np.float32)
        s[10], s[70], s[150] = s0, s1, s1 + np.float32(4.3) / c2
        k = np.zeros((192, dh), np.float32)
        k[:, :3] = np.stack(_f32_parts(s), 1)
        kc, out = B.to_device(k, "bf16"), []
        for m in (1, 2):
            o = torch.zeros((m, dh), dtype=torch.bfloat16, device="cuda")
            ctx.d2c_attention(B.to_device(q[:m], "bf16"), None, m, None, None, kc, v, 192, o, None)
            torch.cuda.synchronize()
            out.append(o[0])
        p = np.exp((s.astype(np.float64) - s[150]) * float(scale))
        assert rel_l2(host(out[0]), p @ host(v).astype(np.float64) / p.sum()) < TOL["bf16"]
        assert torch.equal(out[0], out[1]), f"scores {s0} and {s1}"
    ctx.close()


def test_infinite_weight_in_a_short_last_split(B):
    """A down projection of 11 chunks in splits of 4, 4 and 3 (float, pre-tiled): an infinite weight in the last chunk gives
    infinities of the products' signs in its column, which 1e30 shows, and changes no other column."""
    wd = W.ModelDims(1, 256, 4, 4, 64, 688, 64, dtype="f32")
    m, L = 37, 64
    plan = B.d2c_plan_projection("f32", m, 256, 688)
    assert (plan["splits"], plan["k_per_split"], plan["waves"]) == (3, 256, 4)
    say("infinite weight in a short last split")
    dims = W.with_layers(wd, 1)
    idx_host = np.arange(m, dtype=np.int32)
    got = []
    for value in (1e30, np.inf):
        mdl = W.model_weights(dims, 0)
        mdl["layers"][0]["w_down"][5, 680] = value
        ctx = B.Context(dims, mdl, L)
        h = torch.from_numpy(W.hidden_rows(4, m, 256, std=0.5)).cuda()
        kc, vc = torch.zeros((L, 256), device="cuda"), torch.zeros((L, 256), device="cuda")
        ctx.d2c_refresh_layer(0, h, torch.from_numpy(idx_host).cuda(), idx_host, kc, vc, L)
        torch.cuda.synchronize()
        got.append(host(h))
        ctx.close()
    large, inf = got
    np.testing.assert_array_equal(inf[:, 5], np.copysign(np.inf, large[:, 5]).astype(np.float32))
    np.testing.assert_array_equal(np.delete(inf, 5, 1), np.delete(large, 5, 1))


@pytest.mark.parametrize("tun", [{"attn_waves": 8}, {"attn_waves": 8, "attn_qt": 1}], ids=["by-rows", "one-tile"])
@pytest.mark.parametrize("L,m", [(1536, 16), (1792, 1), (1792, 40), (2050, 47)])
def test_attention_few_rows_with_eight_waves_asked_for(B, L, m, tun):
    """attn_waves = 8 is a shape of more than 64 rows: fewer rows on long key ranges stay with the few-row kernels, and where the
    tiled ones are asked for as well the call is refused."""
    say(f"attention few rows, long, L={L} m={m} {tun}")
    _attention_parity(B, "bf16", 4, 2, 128, L, m, tunables=tun)
    with pytest.raises(B.D2CError):
        _attention_parity(B, "bf16", 4, 2, 128, L, m, tunables={"attn_tiled_min_m": 1, **tun})


@pytest.mark.parametrize("min_m,L,m,few", [(1 << 30, 1792, 40, True), (97, 1536, 16, True), (97, 3000, 47, True), (97, 1100, 48, False),
                                           (96, 1792, 40, False), (64, 1536, 1, False), (1, 1100, 1, False)])
def test_attention_few_rows_asked_for_on_long_key_ranges(B, min_m, L, m, few):
    """attn_tiled_min_m above its default keeps calls of fewer than 48 rows in the few-row kernels, whose head average is a
    launch of its own, on every key range."""
    say(f"attention families min_m={min_m} L={L} m={m}")
    tun = {"attn_tiled_min_m": min_m}
    _attention_parity(B, "bf16", 4, 2, 64, L, m, tunables=tun)
    ctx, _, _ = _ctx_for(B, W.ModelDims(1, 256, 4, 2, 64, 64, 64, dtype="bf16"), max_seq=L, tunables=tun)
    case = W.attention_case(1, 4, 2, 64, L, m, dtype="bf16")
    q, kc, vc = (B.to_device(case[n], "bf16") for n in ("q", "k_cache", "v_cache"))
    ctx.d2c_profile_begin()
    ctx.d2c_attention(q, None, m, None, None, kc, vc, L, torch.zeros_like(q), torch.zeros((m, L), device="cuda"))
    assert ctx.d2c_profile_end()["attn_avg"]["launches"] == (1 if few else 0)
    ctx.close()


def _start_chunks(B, dtype, m, N, K, rots, tunables=None):
    """d2c_linear's results under each gemm_rot (None: as the library chooses)"""
    ctxs = {rot: _ctx_for(B, W.ModelDims(1, 4096, 4, 4, 64, 80, 64, dtype=dtype), max_seq=1024,
                          tunables={**(tunables or {}), **({} if rot is None else {"gemm_rot": rot})})[0] for rot in rots}
    gen = torch.Generator(device="cuda").manual_seed(11)
    a, w = (torch.empty((r, K), dtype=B.torch_dtype(dtype), device="cuda").normal_(generator=gen) for r in (m, N))
    got = {}
    for rot, ctx in ctxs.items():
        got[rot] = torch.full((m, N), 7.0, device="cuda")
        ctx.d2c_linear(a, w, m, N, K, got[rot])
        torch.cuda.synchronize()
        ctx.close()
        ref = a.double() @ w.double().T
        assert ((got[rot].double() - ref).norm() / ref.norm()).item() < 1e-5
    return got


@pytest.mark.parametrize("dtype,m,N,K,chunks", [("bf16", 17, 1000, 4096, 32), ("f32", 17, 1000, 2048, 32), ("bf16", 70, 1000, 8192, 64)])
def test_linear_no_start_chunk_asked_for(B, dtype, m, N, K, chunks):
    """gemm_rot = 0: every workgroup starts where k starts, as with a whole turn (a multiple of the chunks), also where the library
    moves the starts by itself."""
    say(f"linear gemm_rot=0 {dtype} m={m} N={N} K={K}")
    got = _start_chunks(B, dtype, m, N, K, (None, 0, chunks), {"gemm_max_splits": 1})
    assert torch.equal(got[0], got[chunks]) and not torch.equal(got[0], got[None])


@pytest.mark.parametrize("dtype,m,N,K,starts", [
    ("bf16", 17, 24576, 2048, 3), ("bf16", 17, 12288, 2048, 0), ("bf16", 1, 8192, 4096, 0), ("bf16", 40, 12288, 4096, 1), ("bf16", 17, 12288, 8192, 1),
    ("bf16", 40, 4096, 32768, 1), ("bf16", 64, 4096, 32768, 0), ("bf16", 150, 8192, 8192, 1), ("bf16", 192, 16384, 4096, 0), ("bf16", 192, 4096, 32768, 0),
    ("bf16", 192, 65536, 2048, 3),
    ("bf16", 200, 1024, 4096, 0), ("bf16", 256, 49152, 2048, 3), ("bf16", 300, 24576, 4096, 1), ("bf16", 300, 12288, 4096, 0),
    ("bf16", 600, 24576, 4096, 0), ("f32", 1, 33000, 1024, 0), ("f32", 17, 12288, 4096, 1)])
def test_linear_start_chunks_by_shape(B, dtype, m, N, K, starts):
    """Row-major weights a power of two apart: how many chunks apart the library lets neighbouring workgroups start."""
    say(f"linear start chunks {dtype} m={m} N={N} K={K}")
    got = _start_chunks(B, dtype, m, N, K, (None, 0, 1, 3))
    assert [rot for rot in (0, 1, 3) if torch.equal(got[rot], got[None])] == [starts]


@pytest.mark.parametrize("H,Hkv,L,m,splits", [(32, 32, 1024, 400, 2), (32, 32, 2048, 200, 4), (16, 2, 2048, 400, 4), (32, 32, 777, 130, 4)])
def test_attention_key_splits_of_64_wide_heads(B, H, Hkv, L, m, splits):
    """Heads of 64: the tiled kernels take the shape that was measured the faster (4 waves and the fewer splits)."""
    say(f"attention key splits H={H} Hkv={Hkv} L={L} m={m}")
    wd = W.ModelDims(1, H * 64, H, Hkv, 64, 64, 64, dtype="bf16")
    case = W.attention_case(1, H, Hkv, 64, L, m, dtype="bf16")
    q, kc, vc = (B.to_device(case[n], "bf16") for n in ("q", "k_cache", "v_cache"))
    got = []
    for tun in (None, {"attn_waves": 4, "attn_max_splits": splits}, {"attn_waves": 4, "attn_max_splits": splits - 1}):
        ctx, _, _ = _ctx_for(B, wd, max_seq=L, tunables=tun)
        out = torch.zeros_like(q)
        ctx.d2c_attention(q, None, m, None, None, kc, vc, L, out, None)
        torch.cuda.synchronize()
        got.append(out)
        ctx.close()
    assert torch.equal(got[0], got[1]) and not torch.equal(got[0], got[2])


def test_attention_key_splits_with_units_without_end(B):
    """attn_target_wgs at the largest value an int holds plans as any value does that no launch reaches."""
    say("attention key splits, attn_target_wgs = 2^31 - 1")
    case = W.attention_case(1, 4, 4, 128, 2048, 200, dtype="bf16")
    q, kc, vc = (B.to_device(case[n], "bf16") for n in ("q", "k_cache", "v_cache"))
    got = []
    for units in (1 << 20, (1 << 31) - 1):
        ctx, _, _ = _ctx_for(B, W.ModelDims(1, 512, 4, 4, 128, 64, 64, dtype="bf16"), max_seq=2048, tunables={"attn_target_wgs": units})
        out = torch.zeros_like(q)
        ctx.d2c_attention(q, None, 200, None, None, kc, vc, 2048, out, None)
        torch.cuda.synchronize()
        got.append(out)
        ctx.close()
    assert torch.equal(got[0], got[1])
