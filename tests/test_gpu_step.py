"""GPU parity of d2c_step (the whole denoising step) against the CPU oracle.

Teacher-forced runs feed both sides the same S_t, tokens and cached confidences
at every step, compare every float output within the dtype's tolerance, and check
the index sets bit-exactly on the GPU's own score arrays; free-running runs compare
the sets directly for as long as the oracle's decision margins are wide."""
import numpy as np
import pytest
import torch

from oracle import d2cache_oracle as O
from paper_2509_23094_amd import workloads as W

from gpu_util import TOL, host, oracle_dims, oracle_params, rel_l2, say, topk_margin, topp_margin

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def B():
    from paper_2509_23094_amd import binding
    return binding


def _gpu_params(B, prm: O.Params):
    return B.make_params(prm.sigma, prm.k, prm.p, prm.block_len, prm.n_unmask, prm.cand_mode, prm.threshold,
                         prm.conf_decode, prm.rollout_layers)


def _sets(B, seq):
    cnt = seq.counts.cpu().numpy()
    return {
        "mstar": seq.mstar.cpu().numpy()[: cnt[B.CNT_MSTAR]],
        "u": seq.u_set.cpu().numpy()[: cnt[B.CNT_U]],
        "decode": seq.decode_idx.cpu().numpy()[: cnt[B.CNT_DECODE]],
        "s_next": seq.s_idx.cpu().numpy()[: cnt[B.CNT_S]],
        "rows_next": seq.s_rows.cpu().numpy()[: cnt[B.CNT_NEXT_ROWS]],
        "block": (int(cnt[B.CNT_BLOCK_LO]), int(cnt[B.CNT_BLOCK_HI])),
    }


def _force(seq, st: O.SeqState):
    """Put the oracle's state (tokens, mask, cached Eq. 1 values, S_{t+1}) into the GPU sequence."""
    seq.tokens.copy_(torch.from_numpy(st.y.astype(np.int32)))
    seq.is_masked.copy_(torch.from_numpy(st.is_masked.astype(np.uint8)))
    seq.conf.copy_(torch.from_numpy(st.conf))
    seq.pred.copy_(torch.from_numpy(st.pred))
    S = st.S.astype(np.int32)
    seq.set_selection(S, np.flatnonzero(st.is_masked[S]).astype(np.int32))
    seq.c.n_masked = int(st.is_masked.sum())


def _rows_close(got, ref, rows, tol, what):
    """Every row on its own: max over the rows of the per-row relative L2 error.  One wrong row among
    hundreds fails here; it would vanish in a norm over the whole tensor."""
    got, ref = np.asarray(got, np.float64), np.asarray(ref, np.float64)
    for r in rows:
        e = rel_l2(got[r], ref[r])
        assert e < tol, f"{what}: row {int(r)} rel-L2 {e:.3g} >= {tol}"


def _teacher_forced(B, dims, mdl, su, prm, n_steps, seed=0, check_free_run=True, n_seqs=1, prompt_lens=None,
                    max_batch=None, tunables=None):
    """Teacher-forced comparison of d2c_step with the oracle for n_seqs independent sequences that go
    through every d2c_step call together (max_batch of them share the projection launches).

    Floats are compared row by row: final hidden rows, logits rows, the refreshed K/V rows S_t of every
    layer (per row and layer), all within the dtype's tolerance; the cache rows outside S_t must keep the
    bits they had before the step.  Index sets are checked bit-exactly by running the oracle's integer
    selection on the GPU's own float arrays.  The direct comparison with the oracle's sets only runs while
    the oracle's decision margins exceed 50 x the tolerance; in bf16 (tolerance 2e-2) that would need
    relative margins above 1, which no score gap has, so there the sets are verified through the GPU's own
    arrays only -- the float scores those sets are drawn from are themselves compared with the oracle's."""
    od = oracle_dims(dims, len(mdl["layers"]))
    tol = TOL[dims.dtype]
    prompt_lens = prompt_lens or [su.prompt_len] * n_seqs
    Ls = [P + su.gen_len for P in prompt_lens]
    ctx = B.Context(dims, mdl, max(Ls), max_batch=max_batch or n_seqs, tunables=tunables)
    gp = _gpu_params(B, prm)
    sts, seqs = [], []
    for b in range(n_seqs):
        sub = W.DecodeSetup(prompt_lens[b], su.gen_len, su.block_len, su.n_unmask, su.k, su.p, su.sigma)
        y0, m0 = W.initial_sequence(dims, sub, seed, seq=b)
        sts.append(O.new_state(od, y0, m0, sub.prompt_len))
        seqs.append(B.Sequence_(ctx, y0, m0, sub.prompt_len, trace=True, max_trace_rows=su.gen_len))
        assert (seqs[b].n_s, seqs[b].n_rows, seqs[b].n_masked) == (Ls[b], su.gen_len, su.gen_len)
    free_running = check_free_run
    for t in range(n_steps):
        if not any(st.is_masked.any() for st in sts):
            break
        say(f"d2c_step teacher-forced t={t} m={[len(st.S) for st in sts]} dtype={dims.dtype} d={dims.d_model} L={Ls}")
        before = []
        for st, seq in zip(sts, seqs):
            before.append((st.is_masked.copy(), host(seq.k_cache), host(seq.v_cache)))
            if st.is_masked.any():
                O.d2cache_step(od, mdl, prm, st)
        ctx.d2c_step(gp, seqs)
        for b, (st, seq) in enumerate(zip(sts, seqs)):
            masked_before, k_prev, v_prev = before[b]
            if not masked_before.any():
                continue
            L = Ls[b]
            tr = st.trace
            S, m = tr["S"], len(tr["S"])
            rows = tr["logit_rows"]
            # --- floats, row by row
            _rows_close(host(seq.hidden_out)[:m], tr["hidden"], range(m), tol, f"hidden seq={b} t={t}")
            if len(rows):
                _rows_close(host(seq.logits_out)[: len(rows)], tr["logits"], range(len(rows)), tol, f"logits seq={b} t={t}")
            k_now, v_now = host(seq.k_cache), host(seq.v_cache)
            rest = np.setdiff1d(np.arange(L), S)
            for l in range(od.n_layers):
                _rows_close(k_now[l], st.k_cache[l], S, tol, f"K layer={l} seq={b} t={t}")
                _rows_close(v_now[l], st.v_cache[l], S, tol, f"V layer={l} seq={b} t={t}")
                np.testing.assert_array_equal(k_now[l][rest], k_prev[l][rest])     # reused rows: untouched bits
                np.testing.assert_array_equal(v_now[l][rest], v_prev[l][rest])
            infl = host(seq.influence)
            assert rel_l2(infl, tr["c"]) < tol and np.max(np.abs(infl - tr["c"])) < tol * max(1.0, tr["c"].max()), f"c t={t}"
            conf_g, pred_g = host(seq.conf), seq.pred.cpu().numpy()
            if len(rows):
                np.testing.assert_allclose(conf_g[rows], st.conf[rows], rtol=max(tol, 1e-5) * 5, err_msg=f"conf t={t}")
                lg = tr["logits"]
                picked = lg[np.arange(len(rows)), pred_g[rows]]
                assert np.all(lg.max(axis=1) - picked <= 4 * tol * np.abs(lg).max() + 1e-12), f"pred t={t}"
                if dims.dtype == "f32":
                    np.testing.assert_array_equal(pred_g[rows], st.pred[rows])
            g = _sets(B, seq)
            assert g["block"] == tr["block"]
            score_g = host(seq.score)
            cand1 = np.array([i for i in range(*tr["block"]) if masked_before[i]], np.int64)
            if len(cand1):
                np.testing.assert_allclose(score_g[cand1], tr["score"][cand1], rtol=max(tol, 1e-5) * 5)
            # --- index sets, integer-exact on the GPU's own float arrays
            np.testing.assert_array_equal(g["mstar"], O.top_k_select(score_g, cand1, prm.k))
            dec_ref = O.top_k_select(conf_g if prm.conf_decode else score_g, cand1, prm.n_unmask)
            if prm.threshold > 0:
                dec_ref = np.union1d(dec_ref, cand1[conf_g[cand1] > np.float32(prm.threshold)]).astype(np.int32)
            np.testing.assert_array_equal(g["decode"], dec_ref)
            cand2 = np.flatnonzero(~masked_before)
            np.testing.assert_array_equal(g["u"], O.top_p_select(infl, cand2, prm.p))
            np.testing.assert_array_equal(g["s_next"], np.union1d(np.union1d(g["mstar"], g["decode"]), g["u"]))
            # --- the same sets against the oracle's, while its margins are wide (fp32 only in practice)
            if free_running:
                safe = (topk_margin(tr["score"], cand1, prm.k) > 50 * tol and
                        topk_margin(tr["score"], cand1, prm.n_unmask) > 50 * tol and
                        topp_margin(tr["c"], cand2, prm.p) > 50 * tol and prm.threshold == 0 and not prm.conf_decode)
                if safe:
                    np.testing.assert_array_equal(g["mstar"], tr["mstar"])
                    np.testing.assert_array_equal(g["decode"], tr["decode"])
                    np.testing.assert_array_equal(g["u"], tr["u"])
            _force(seq, st)
    ctx.close()


def test_step_c1_teacher_forced_all_steps(B):
    """The small fp32 model: every one of its 64 steps."""
    wd, su = W.DIMS["C1"], W.SETUP["C1"]
    mdl = W.model_weights(wd, 0)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=su.gen_len)


def test_step_c1_free_running(B):
    """No forcing: the GPU decodes the whole response on its own; sets and tokens must match the oracle's
    as long as the oracle's own decisions are not near-ties."""
    wd, su = W.DIMS["C1"], W.SETUP["C1"]
    mdl = W.model_weights(wd, 0)
    # N(0, 0.02) weights give an almost uniform influence c_j, so the p = 0.9 cut falls between candidates
    # that differ by ~1e-6 of the mass: a tie by construction.  Four times wider weights give attention
    # enough structure for the cut to be decided by more than rounding for the first twenty steps.
    for lw in mdl["layers"]:
        for name in ("wqkv", "wo", "w_gate_up", "w_down"):
            lw[name] = lw[name] * np.float32(4.0)
    mdl["tok_emb"], mdl["lm_head"] = mdl["tok_emb"] * np.float32(4.0), mdl["lm_head"] * np.float32(4.0)
    od, prm = oracle_dims(wd), oracle_params(su)
    ctx = B.Context(wd, mdl, su.seq_len)
    y0, m0 = W.initial_sequence(wd, su, 0)
    st = O.new_state(od, y0, m0, su.prompt_len)
    seq = B.Sequence_(ctx, y0, m0, su.prompt_len, trace=True, max_trace_rows=su.gen_len)
    gp = _gpu_params(B, prm)
    compared = 0
    margin = 2e-5            # twenty times the fp32 path's rounding level
    for t in range(su.gen_len):
        say(f"d2c_step free-running t={t}")
        masked_before = st.is_masked.copy()
        O.d2cache_step(od, mdl, prm, st)
        ctx.d2c_step(gp, [seq])
        tr = st.trace
        cand1 = np.array([i for i in range(*tr["block"]) if masked_before[i]], np.int64)
        cand2 = np.flatnonzero(~masked_before)
        lg = np.sort(tr["logits"], axis=1) if len(tr["logit_rows"]) else np.zeros((0, 2))
        safe = (topk_margin(tr["score"], cand1, prm.k) > margin and
                topk_margin(tr["score"], cand1, prm.n_unmask) > margin and
                topp_margin(tr["c"], cand2, prm.p) > margin and
                (len(lg) == 0 or np.min(lg[:, -1] - lg[:, -2]) > margin * np.abs(lg).max()))
        if not safe:
            break
        g = _sets(B, seq)
        np.testing.assert_array_equal(g["s_next"], st.S)
        np.testing.assert_array_equal(g["decode"], tr["decode"])
        np.testing.assert_array_equal(seq.tokens.cpu().numpy(), st.y)
        np.testing.assert_array_equal(seq.is_masked.cpu().numpy().astype(bool), st.is_masked)
        compared += 1
    assert compared >= 8, "the oracle's margins were too narrow to compare even a few steps"
    if compared == su.gen_len:
        assert seq.n_masked == 0
    ctx.close()


def test_step_select_all_equals_full_recomputation(B):
    """k >= |M|, p = 1, one block: d2c_step must reproduce the oracle's separate full forward every step."""
    wd = W.with_layers(W.DIMS["C1"], 2)
    su = W.DecodeSetup(24, 16, 16, 1, k=10 ** 6, p=1.0)
    mdl = W.model_weights(wd, 5)
    od = oracle_dims(wd)
    ctx = B.Context(wd, mdl, su.seq_len)
    y0, m0 = W.initial_sequence(wd, su, 1)
    seq = B.Sequence_(ctx, y0, m0, su.prompt_len, trace=True)
    gp = B.make_params(10.0, su.seq_len, 1.0, su.gen_len, 1, 0)
    for t in range(su.gen_len):
        say(f"select-all step t={t}")
        y_in = seq.tokens.cpu().numpy()
        masked = seq.is_masked.cpu().numpy().astype(bool)
        assert seq.n_s == su.seq_len
        ctx.d2c_step(gp, [seq])
        full = O.full_forward(od, mdl, y_in)
        assert rel_l2(host(seq.hidden_out), full["hidden"]) < 1e-5
        assert rel_l2(host(seq.k_cache), full["k"]) < 1e-5 and rel_l2(host(seq.v_cache), full["v"]) < 1e-5
        rows = np.flatnonzero(masked)
        assert rel_l2(host(seq.logits_out)[: len(rows)], full["logits"][rows]) < 1e-5
    assert seq.n_masked == 0
    ctx.close()


def test_step_select_none_leaves_cache_unchanged(B):
    wd = W.with_layers(W.DIMS["C1"], 2)
    su = W.DecodeSetup(16, 16, 8, 1, k=4, p=0.5)
    mdl = W.model_weights(wd, 6)
    ctx = B.Context(wd, mdl, su.seq_len)
    y0, m0 = W.initial_sequence(wd, su, 2)
    seq = B.Sequence_(ctx, y0, m0, su.prompt_len, trace=True)
    gp = B.make_params(10.0, su.k, su.p, su.block_len, 1, 0)
    say("select-none: step 0")
    ctx.d2c_step(gp, [seq])
    snap = [t.clone() for t in (seq.k_cache, seq.v_cache, seq.conf, seq.pred)]
    seq.set_selection(np.zeros(0, np.int32), np.zeros(0, np.int32))
    say("select-none: empty S")
    ctx.d2c_step(gp, [seq])
    for a, b in zip(snap, (seq.k_cache, seq.v_cache, seq.conf, seq.pred)):
        assert torch.equal(a, b)
    np.testing.assert_array_equal(host(seq.influence), np.ones(su.seq_len, np.float32))     # S = {} => c = 1
    ctx.close()


def test_step_bf16_small_teacher_forced(B):
    """A narrow bf16 model (GQA, head_dim 64), 24 steps, two blocks."""
    wd = W.ModelDims(3, 512, 8, 2, 64, 1408, 2048, dtype="bf16")
    su = W.DecodeSetup(40, 24, 12, 1, k=6, p=0.3)
    mdl = W.model_weights(wd, 3)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=24)


def test_step_bf16_small_on_two_streams(B):
    """The same narrow bf16 model with the second stream switched on: head means and the rollout chain run
    beside the last layer's projections and the LM head, and the selection waits for them."""
    wd = W.ModelDims(3, 512, 8, 2, 64, 1408, 2048, dtype="bf16")
    su = W.DecodeSetup(40, 24, 12, 1, k=6, p=0.3)
    mdl = W.model_weights(wd, 3)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=8, tunables={"side_stream": 1})


def test_step_long_sequence_few_rows_on_two_streams(B):
    """The long-generation regime (second Q K^T launch per layer for the head average) with that launch on the
    second stream."""
    wd = W.ModelDims(2, 512, 8, 2, 64, 1024, 1024, dtype="bf16")
    su = W.DecodeSetup(1040, 64, 32, 1, k=16, p=0.02)
    mdl = W.model_weights(wd, 9)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=2, tunables={"side_stream": 1})


def test_step_bf16_many_rows_per_step(B):
    """A bf16 model whose steps select more than 96 rows (k = 64 masked + half the known tokens): the
    LDS-tiled attention kernels, whose finishing launch also writes the head average, inside d2c_step."""
    wd = W.ModelDims(2, 512, 4, 4, 128, 1408, 2048, dtype="bf16")
    su = W.DecodeSetup(160, 96, 96, 2, k=64, p=0.6)
    mdl = W.model_weights(wd, 5)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=6)


def test_step_bf16_long_sequence_few_rows(B):
    """More than 1024 positions with a few dozen selected rows per step (the long-generation regime): the
    few-row attention kernel cannot keep its scores, so every layer runs the second Q K^T pass for the head
    average; grouped-query geometry (8 query heads on 2 kv heads)."""
    wd = W.ModelDims(2, 512, 8, 2, 64, 1024, 1024, dtype="bf16")
    su = W.DecodeSetup(1040, 64, 32, 1, k=16, p=0.02)
    mdl = W.model_weights(wd, 9)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=3)


def test_step_at_the_maximum_length(B):
    """L = 4096, the longest sequence the selection and the rollout chain take: step 0 over all 4096 rows
    (the dense chain blocks at their largest) and two decode steps, against the oracle's literal L x L
    rollout.  One more position is refused at d2c_init."""
    wd = W.ModelDims(2, 256, 4, 2, 64, 512, 512, dtype="bf16")
    su = W.DecodeSetup(4096 - 64, 64, 32, 1, k=16, p=0.02)
    mdl = W.model_weights(wd, 13)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=2)
    with pytest.raises(B.D2CError) as err:
        B.Context(wd, mdl, 4097)
    assert err.value.code == -4                      # D2C_ESHAPE


def test_step_batch_of_ragged_sequences(B):
    """Two independent sequences of different length in one d2c_step call equal two separate calls."""
    wd = W.ModelDims(2, 256, 4, 4, 64, 688, 512, dtype="bf16")
    mdl = W.model_weights(wd, 4)
    ctx = B.Context(wd, mdl, 96)
    sus = [W.DecodeSetup(32, 32, 16, 2, k=8, p=0.2), W.DecodeSetup(64, 32, 32, 2, k=8, p=0.2)]
    gp = B.make_params(10.0, 8, 0.2, 16, 2, 0)
    pairs = []
    for b, su in enumerate(sus):
        y0, m0 = W.initial_sequence(wd, su, 7, seq=b)
        pairs.append((B.Sequence_(ctx, y0, m0, su.prompt_len), B.Sequence_(ctx, y0, m0, su.prompt_len)))
    for t in range(6):
        say(f"batched d2c_step t={t}")
        ctx.d2c_step(gp, [p[0] for p in pairs])
        for p in pairs:
            ctx.d2c_step(gp, [p[1]])
        for a, b in pairs:
            assert (a.n_s, a.n_rows, a.n_masked) == (b.n_s, b.n_rows, b.n_masked)
            assert a.n_masked == a.L - a.prompt_len - 2 * (t + 1)
            for name in ("tokens", "is_masked", "k_cache", "v_cache", "conf", "pred", "influence"):
                assert torch.equal(getattr(a, name), getattr(b, name)), name
            assert torch.equal(a.s_idx[: a.n_s], b.s_idx[: b.n_s])
    ctx.close()


def test_step_grouped_projections_match_separate_calls(B):
    """max_batch = 3: the rows of three ragged sequences share the projection launches.  The split plan of
    a projection depends on the row count, so the floats may differ from separate calls in the last bits:
    sets must be identical (fp32 model with widened weights: no near-ties), floats within the fp32 bar."""
    wd = W.DIMS["C1"]
    mdl = W.model_weights(wd, 3)
    for lw in mdl["layers"]:
        for name in ("wqkv", "wo", "w_gate_up", "w_down"):
            lw[name] = lw[name] * np.float32(4.0)
    sus = [W.DecodeSetup(24, 32, 16, 1, k=8, p=0.5), W.DecodeSetup(64, 48, 16, 1, k=8, p=0.5),
           W.DecodeSetup(40, 16, 16, 1, k=8, p=0.5)]
    gp = B.make_params(10.0, 8, 0.5, 16, 1, 0)
    ctx_g = B.Context(wd, mdl, 112, max_batch=3)
    ctx_1 = B.Context(wd, mdl, 112)
    grouped, single = [], []
    for b, su in enumerate(sus):
        y0, m0 = W.initial_sequence(wd, su, 11, seq=b)
        grouped.append(B.Sequence_(ctx_g, y0, m0, su.prompt_len))
        single.append(B.Sequence_(ctx_1, y0, m0, su.prompt_len))
    for t in range(20):                    # the third sequence is fully decoded after 16 steps and is skipped from then on
        say(f"grouped d2c_step t={t}")
        ctx_g.d2c_step(gp, grouped)
        for q in single:
            ctx_1.d2c_step(gp, [q])
        for a, b in zip(grouped, single):
            assert (a.n_s, a.n_rows, a.n_masked) == (b.n_s, b.n_rows, b.n_masked)
            assert torch.equal(a.s_idx[: a.n_s], b.s_idx[: b.n_s])
            assert torch.equal(a.tokens, b.tokens) and torch.equal(a.is_masked, b.is_masked)
            assert torch.equal(a.pred, b.pred)
            for name in ("k_cache", "v_cache", "conf", "influence"):
                assert rel_l2(host(getattr(a, name)), host(getattr(b, name))) < TOL["f32"], name
    ctx_g.close()
    ctx_1.close()


@pytest.mark.parametrize("cand_mode", [0, 1])
def test_step_more_sequences_than_a_launch_takes(B, cand_mode):
    """Ten sequences in one group, more than RoPE and the selection take in a launch: both halves of a selection in one kernel, the
    QKV projection's output turned by launches of its own.  At step 0 the group's masked rows go through the head in pieces."""
    wd = W.DIMS["C1"]
    mdl = W.model_weights(wd, 3)
    for lw in mdl["layers"]:
        for name in ("wqkv", "wo", "w_gate_up", "w_down"):
            lw[name] = lw[name] * np.float32(4.0)
    sus = [W.DecodeSetup(8 + 3 * b, 24 + 2 * (b % 4), 16, 1, k=8, p=0.5) for b in range(10)]
    gp = B.make_params(10.0, 8, 0.5, 16, 1, cand_mode)
    ctx_g, ctx_1 = B.Context(wd, mdl, 72, max_batch=10), B.Context(wd, mdl, 72)
    grouped, single = [], []
    for b, su in enumerate(sus):
        y0, m0 = W.initial_sequence(wd, su, 11, seq=b)
        grouped.append(B.Sequence_(ctx_g, y0, m0, su.prompt_len))
        single.append(B.Sequence_(ctx_1, y0, m0, su.prompt_len))
    for t in range(5):
        say(f"group of ten, cand_mode={cand_mode} t={t}")
        ctx_g.d2c_step(gp, grouped)
        for a, b in zip(grouped, single):
            ctx_1.d2c_step(gp, [b])
            assert (a.n_s, a.n_rows, a.n_masked) == (b.n_s, b.n_rows, b.n_masked)
            assert torch.equal(a.s_idx[: a.n_s], b.s_idx[: b.n_s]) and torch.equal(a.s_rows[: a.n_rows], b.s_rows[: b.n_rows])
            assert torch.equal(a.tokens, b.tokens) and torch.equal(a.is_masked, b.is_masked) and torch.equal(a.pred, b.pred)
            for name in ("k_cache", "v_cache", "conf", "influence"):
                assert rel_l2(host(getattr(a, name)), host(getattr(b, name))) < TOL["f32"], name
    ctx_g.close()
    ctx_1.close()


def test_step_llada_shape_reduced_depth(B):
    """LLaDA-8B geometry at full width and full vocabulary, 2 of the 32 layers: step 0 (all 512 rows)
    and two d2Cache steps, teacher-forced."""
    wd, su = W.with_layers(W.DIMS["C3"], 2), W.SETUP["C3"]
    mdl = W.model_weights(wd, 0)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=3)


def _spread_model(wd, seed):
    """The small fp32 model with wider weights, so that the confidences of the masked positions spread
    around a threshold and the attention has structure."""
    mdl = W.model_weights(wd, seed)
    for name in ("tok_emb", "lm_head"):
        mdl[name] = mdl[name] * np.float32(16.0)
    for lw in mdl["layers"]:
        for name in ("wqkv", "wo", "w_gate_up", "w_down"):
            lw[name] = lw[name] * np.float32(4.0)
    return mdl


def test_step_parallel_decoding_by_threshold(B):
    """Parallel decoding by confidence threshold alone (1 to several tokens per step)."""
    wd, su = W.DIMS["C1"], W.DecodeSetup(32, 48, 16, 1, k=8, p=0.5)
    _teacher_forced(B, wd, _spread_model(wd, 1), su, oracle_params(su, threshold=0.5), n_steps=su.gen_len)


def test_step_confidence_only_decoding(B):
    """The decode set ranked by the confidence alone; M* still by D(i) s^i."""
    wd, su = W.DIMS["C1"], W.DecodeSetup(32, 48, 16, 1, k=8, p=0.5)
    _teacher_forced(B, wd, _spread_model(wd, 1), su, oracle_params(su, conf_decode=1), n_steps=su.gen_len)


@pytest.mark.parametrize("r", [1, 2, 5])
def test_step_rollout_over_first_layers_f32(B, r):
    """Rollout over the first r layers of a 3-layer fp32 model (r = 5 exceeds the depth: all layers)."""
    wd, su = W.with_layers(W.DIMS["C1"], 3), W.DecodeSetup(32, 48, 16, 1, k=8, p=0.5)
    _teacher_forced(B, wd, _spread_model(wd, 2), su, oracle_params(su, rollout_layers=r), n_steps=12)


@pytest.mark.parametrize("regime", ["few_rows", "many_rows", "long_sequence"])
def test_step_rollout_over_first_layers_bf16(B, regime):
    """bf16, 4 layers, rollout over the first 2: the later layers run the attention kernel that keeps no
    probability rows and skip the head average.  few_rows: the attention launch itself writes the per-head
    rows (fewer than 96 selected rows, L <= 1024); many_rows: the LDS-tiled kernels; long_sequence: more
    than 1024 positions with few rows per step."""
    if regime == "few_rows":
        wd = W.ModelDims(4, 512, 8, 2, 64, 1408, 2048, dtype="bf16")
        su = W.DecodeSetup(40, 24, 12, 1, k=6, p=0.3)
        steps = 10
    elif regime == "many_rows":
        wd = W.ModelDims(4, 512, 4, 4, 128, 1408, 2048, dtype="bf16")
        su = W.DecodeSetup(160, 96, 96, 2, k=64, p=0.6)
        steps = 4
    else:
        wd = W.ModelDims(4, 512, 8, 2, 64, 1024, 1024, dtype="bf16")
        su = W.DecodeSetup(1040, 64, 32, 1, k=16, p=0.02)
        steps = 3
    mdl = W.model_weights(wd, 13)
    _teacher_forced(B, wd, mdl, su, oracle_params(su, rollout_layers=2), n_steps=steps)


def test_step_parallel_confidence_and_short_rollout_together(B):
    """All three switches at once (the combination a parallel-decoding run with the lightweight rollout uses)."""
    wd, su = W.DIMS["C1"], W.DecodeSetup(32, 48, 16, 1, k=8, p=0.5)
    prm = oracle_params(su, threshold=0.5, conf_decode=1, rollout_layers=1)
    _teacher_forced(B, wd, _spread_model(wd, 1), su, prm, n_steps=su.gen_len)


def test_step_dream_shape_reduced_depth(B):
    """Dream-7B geometry (28 query heads on 4 kv heads, d_model 3584, FFN 18944) at full width and full
    vocabulary (152064), 2 of the 28 layers: step 0 (all 768 rows) and two d2Cache steps, teacher-forced."""
    wd, su = W.with_layers(W.DIMS["C4"], 2), W.SETUP["C4"]
    mdl = W.model_weights(wd, 0)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=3)


def test_step_long_context_batch_regime(B):
    """The long-context batch regime: two sequences with different prompts (2048 and 1984 tokens) and
    1024 generated positions each, blocks of 64, two tokens unmasked per step, sigma 10 / k 32 / p 0.1,
    projected together (max_batch = 2); 2 layers of 8 x 128 heads so that the CPU side stays within a
    minute.  Step 0 over all ~3000 rows per sequence, then two d2Cache steps of a few hundred ragged rows
    each (the LDS-tiled attention kernels at L ~ 3072, the rollout chain at that length)."""
    wd = W.ModelDims(2, 1024, 8, 8, 128, 2816, 8192, dtype="bf16")
    su = W.SETUP["C5"]
    mdl = W.model_weights(wd, 21)
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=3, n_seqs=2, prompt_lens=[2048, 1984], max_batch=2)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_step_with_qkv_bias(B, dtype):
    """A model whose QKV projection has a bias (the Qwen2.5 / Dream geometry), grouped-query heads."""
    if dtype == "f32":
        wd = W.ModelDims(2, 256, 4, 2, 64, 688, 1024, dtype="f32")
    else:
        wd = W.ModelDims(2, 512, 8, 2, 64, 1408, 2048, dtype="bf16")
    su = W.DecodeSetup(40, 24, 12, 1, k=6, p=0.3)
    mdl = W.model_weights(wd, 17)
    for l, lw in enumerate(mdl["layers"]):
        lw["bqkv"] = W.hidden_rows(17, 1, wd.d_q + 2 * wd.d_kv, std=0.5, extra=100 + l)[0]
    _teacher_forced(B, wd, mdl, su, oracle_params(su), n_steps=6)


@pytest.mark.parametrize("workload", ["C3", "C4", "C5"])
def test_step_full_depth_properties_and_sampled_rows(B, workload):
    """The benchmark's own configurations (LLaDA-8B and Dream-7B shapes at full depth, weights drawn on the
    device as bench.py draws them; the long-context batch of four sequences projected together),
    free-running for step 0 and three d2Cache steps.  A CPU forward at this size
    takes minutes, so the check is what holds at any size plus sampled outputs the oracle computes row by
    row: the influence scores sum to L and are at least 1 outside S (Eq. 6-9 with rows of W summing to
    1), every index set is reproduced bit-exactly by the oracle's integer selection from the GPU's own
    float arrays, the layer-0 key rows of sampled refreshed positions equal RoPE(W_k RMSNorm(Emb[y_i])),
    and a second run from the same inputs is bit-identical."""
    import bench
    dims, su = W.DIMS[workload], W.SETUP[workload]
    mdl = bench.device_model(W, dims, 0, torch)
    ctx = B.Context(dims, mdl, su.seq_len, device_weights=True, max_batch=su.batch)
    od = oracle_dims(dims, dims.n_layers)
    prm = oracle_params(su)
    gp = _gpu_params(B, prm)
    inits = [W.initial_sequence(dims, su, b) for b in range(su.batch)]
    L, dq, dkv = su.seq_len, dims.d_q, dims.d_kv
    wk = mdl["layers"][0]["wqkv"][dq: dq + dkv].float().cpu().numpy().astype(np.float64)      # [d_kv, d]
    emb = mdl["tok_emb"]
    gain = np.ones(dims.d_model)
    finals = []
    for rep in range(2):
        seqs = [B.Sequence_(ctx, y0, m0, su.prompt_len, trace=True, max_trace_rows=su.gen_len) for y0, m0 in inits]
        for t in range(4):
            say(f"full-depth {workload} shape rep={rep} t={t} m={[q.n_s for q in seqs]}")
            before = [(q.is_masked.cpu().numpy().astype(bool), q.s_idx.cpu().numpy()[: q.n_s].astype(np.int64),
                       q.tokens.cpu().numpy()) for q in seqs]
            ctx.d2c_step(gp, seqs)
            torch.cuda.synchronize()
            for seq, (masked_before, S, tokens_in) in zip(seqs, before):
                infl = host(seq.influence)
                if rep == 0:
                    # Eq. 9 invariants
                    assert abs(float(infl.astype(np.float64).sum()) - L) < 1e-3 * L, f"sum of influence t={t}"
                    outside = np.setdiff1d(np.arange(L), S)
                    assert np.all(infl[outside] >= 1.0 - 1e-4) and np.all(infl >= 0.0)
                    # index sets: integer-exact on the GPU's own float arrays
                    g = _sets(B, seq)
                    score_g, conf_g = host(seq.score), host(seq.conf)
                    lo, hi = g["block"]
                    assert (lo, hi) == O.current_block(masked_before, su.prompt_len, su.block_len)
                    cand1 = np.array([i for i in range(lo, hi) if masked_before[i]], np.int64)
                    np.testing.assert_array_equal(g["mstar"], O.top_k_select(score_g, cand1, prm.k))
                    np.testing.assert_array_equal(g["decode"], O.top_k_select(score_g, cand1, prm.n_unmask))
                    cand2 = np.flatnonzero(~masked_before)
                    np.testing.assert_array_equal(g["u"], O.top_p_select(infl, cand2, prm.p))
                    np.testing.assert_array_equal(g["s_next"], np.union1d(np.union1d(g["mstar"], g["decode"]), g["u"]))
                    assert seq.n_masked == su.gen_len - su.n_unmask * (t + 1)
                    # Eq. 1 on sampled rows, from the logits this step produced
                    rows = np.array([i for i in S if masked_before[i]], np.int64)
                    if len(rows):
                        lg = host(seq.logits_out)[: len(rows)]
                        s_ref, x_ref = O.confidence(lg[:4])
                        np.testing.assert_allclose(conf_g[rows[:4]], s_ref, rtol=1e-4)
                        np.testing.assert_array_equal(seq.pred.cpu().numpy()[rows[:4]], x_ref)
                    # layer-0 key rows of sampled refreshed positions
                    kc0 = seq.k_cache[0].float().cpu().numpy()
                    for i in S[:: max(1, len(S) // 3)][:3]:
                        x = emb[int(tokens_in[i])].float().cpu().numpy().astype(np.float64)[None, :]
                        a = W.round_bf16(O.rmsnorm(x, gain, od.rms_eps).astype(np.float32)).astype(np.float64)
                        k = (a @ wk.T).reshape(1, dims.n_kv_heads, dims.head_dim)
                        k = O.rope(k, np.array([i]), od.rope_theta).reshape(-1)
                        assert rel_l2(kc0[i], k) < TOL["bf16"], f"layer-0 key row {i} t={t}"
        finals.append([{n: getattr(q, n).clone() for n in ("tokens", "is_masked", "k_cache", "v_cache", "conf", "pred",
                                                            "influence", "s_idx")} for q in seqs])
        del seqs
    for fa, fb in zip(finals[0], finals[1]):
        for n in fa:
            assert torch.equal(fa[n], fb[n]), f"run-to-run difference in {n}"
    ctx.close()
