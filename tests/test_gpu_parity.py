"""GPU parity: the HIP path behind the C ABI against the CPU oracle, on the same seeded inputs.

Accept lengths and token ids must be bit-exact on inputs whose compared rows clear a
top-1/top-2 logit margin of 1e-2 in the oracle; logits and hidden states must agree within
max|gpu-ref|/max|ref| <= 1e-4 (fp32 models) or 2e-2 (bf16 models).
"""
import copy

import numpy as np
import pytest

import synth
from oracle import ee_oracle as eo
from hs_common import (MARGIN, TOL, OracleSide, bf16_d128, bf16_small, gpu_side, max_rel, note,
                       check_state as _check_state, pick_drafts as _pick_drafts, run_round as _round, setup as _setup,
                       tag as _tag, trial_round as _trial_round)

pytestmark = pytest.mark.gpu


# ------------------------------------------------------------------------------------------------
# inputs: device generator == host generator, bit for bit
# ------------------------------------------------------------------------------------------------
@pytest.mark.parametrize("cfg", [synth.tiny_config(), bf16_small(), bf16_d128(gamma=(1.0, 0.5, 0.25)),
                                 synth.tiny_config(head_rank=24, gamma=(1.0, 0.5, 0.25)), bf16_small(head_rank=96)],
                         ids=["tiny_f32", "bf16_small", "bf16_d128", "tiny_f32_heads", "bf16_small_heads"])
def test_device_weights_equal_host_generator(cfg):
    import paper_2510_01336_amd as hs
    model = hs.Model(cfg, 4242)
    names = synth.model.GLOBAL_TENSORS + synth.model.LAYER_TENSORS + (synth.model.EXIT_TENSORS if cfg.head_rank else ())
    for name in names:
        shape = synth.tensor_shape(cfg, name)
        layers = [0] if name in synth.model.GLOBAL_TENSORS else ([0, 1] if name in synth.model.EXIT_TENSORS else [0, cfg.n_layers - 1])
        for layer in layers:
            want = synth.gen_tensor(cfg, 4242, name, layer)
            rows, cols = shape[0], (shape[1] if len(shape) == 2 else 1)
            got = model.tensor_rows(name, layer, 0, rows, cols).reshape(want.shape)
            nbad = int(np.count_nonzero(got.view(np.uint32) != want.view(np.uint32)))
            assert nbad == 0, (name, layer, nbad)
    model.close()


def test_set_tensor_roundtrip():
    import paper_2510_01336_amd as hs
    cfg = bf16_small()
    model = hs.Model(cfg, 1)
    rng = np.random.default_rng(0)
    for name in ("wup", "wk", "g2", "emb"):
        shape = synth.tensor_shape(cfg, name)
        vals = rng.normal(size=shape).astype(np.float32)
        model.set_tensor(name, 1, vals)
        want = synth.bf16_bits_to_f32(synth.f32_to_bf16_bits(vals))
        got = model.tensor_rows(name, 1, 0, shape[0], shape[1] if len(shape) == 2 else 1).reshape(shape)
        assert np.array_equal(got, want), name
    # neighbours in the fused / interleaved matrices are untouched
    assert np.array_equal(model.tensor_rows("wgate", 1, 0, 688, 256), synth.gen_tensor(cfg, 1, "wgate", 1))
    assert np.array_equal(model.tensor_rows("wq", 1, 0, 512, 256), synth.gen_tensor(cfg, 1, "wq", 1))
    model.close()


# ------------------------------------------------------------------------------------------------
# verify-step parity
# ------------------------------------------------------------------------------------------------
CASES = [
    # cfg, ctx lengths (ragged; > 64 spans KV pages), k, bonus modes
    ("tiny_f32", synth.tiny_config(gamma=(1.0, 0.3, 0.3)), [32], 4, (True, True)),
    ("tiny_f32_batch", synth.tiny_config(gamma=(1.0, 0.3, 0.3)), [40, 7, 129], 4, (True, False)),
    ("bf16_small", bf16_small(), [150], 8, (True, True)),
    ("bf16_small_batch", bf16_small(), [70, 5, 200, 64], 8, (True, True)),
    ("bf16_small_nobonus", bf16_small(), [33, 130], 5, (False, False)),
    ("bf16_d128", bf16_d128(), [100, 260], 8, (True, True)),
    ("bf16_d128_k16", bf16_d128(), [300], 16, (True, True)),
    # more than 64 block rows in one call: the row-tiled GEMM (8 and 12 row tiles), ragged contexts
    ("bf16_small_batch10", bf16_small(), [70, 5, 200, 64, 33, 129, 17, 90, 150, 260], 8, (True, True)),
    ("bf16_d128_batch16", bf16_d128(), [100, 260, 31, 64, 65, 7, 190, 128, 40, 77, 300, 12, 55, 201, 99, 160], 8, (True, True)),
    # auxiliary low-rank exit heads at L_d and L_i (skinny and row-tiled GEMM paths)
    ("tiny_f32_heads", synth.tiny_config(gamma=(1.0, 0.3, 0.3), head_rank=24), [32, 70], 4, (True, True)),
    ("bf16_small_heads", bf16_small(head_rank=64), [150, 40], 8, (True, True)),
    ("bf16_d128_heads_batch16", bf16_d128(head_rank=96), [100, 260, 31, 64, 65, 7, 190, 128, 40, 77, 300, 12, 55, 201, 99, 160], 8, (True, True)),
    # K shares of the weight-streaming GEMM that end in every way its pipeline distinguishes: d_ffn 3584 = 4 shares
    # of 28 k-tiles (a pair of full groups of 8, then a full and a short one), d_ffn 2560 = 4 x 20 (a pair, then one short
    # group); 9 rows (one row tile, 8 k-tiles per register set) and 18 rows (two row tiles, 4 per set)
    ("bf16_k_tail_28", bf16_small(d_ffn=3584), [90], 8, (True, True)),
    ("bf16_k_tail_28_rows18", bf16_small(d_ffn=3584), [90, 41], 8, (True, True)),
    ("bf16_k_tail_20", bf16_small(d_ffn=2560), [70, 33], 8, (True, True)),
]


@pytest.mark.parametrize("name,cfg,ctx,k,bonus", CASES, ids=[c[0] for c in CASES])
def test_verify_rounds_match_oracle(name, cfg, ctx, k, bonus):
    tol = TOL[cfg.dtype]
    max_rows = 3 * (k + 1) + 2
    O, model, sess, first, gfirst = _setup(cfg, 777, ctx, max_rows, bonus, plain=True)
    assert gfirst.tolist() == first.tolist()
    # the last prefill pass covered the last sequence: its final row is the oracle's last hidden row
    for side in O.sides():
        assert max_rel(sess.last_hidden()[-1:], side.o.last_hidden) <= tol
        assert max_rel(sess.last_logits()[-1:], side.o.last_logits) <= tol
    rng = np.random.default_rng(5)
    # round 1: intermediate only; round 2: intermediate then full; round 3: both again
    _round(O, sess, k, 0.8, rng, False, tol)
    _round(O, sess, k, 0.8, rng, True, tol)
    _round(O, sess, k, 0.6, rng, True, tol)
    sess.close(); model.close()


@pytest.mark.parametrize("ctx,k", [([70], 7), ([70, 33], 8)], ids=["rows8", "rows18"])
@pytest.mark.parametrize("d,ffn", [(256, 14336), (272, 14304), (272, 14352), (272, 6160), (272, 5136), (256, 3088)])
def test_strips_dealt_in_every_shape(d, ffn, ctx, k):
    """Gate/up matrices of 1792 and 1788 strips (one strip a wave, seven waves a workgroup: even, and a last workgroup of three), of
    1794 and 770 (four waves a workgroup, a last one of two), 642 (four strips a wave, K over eight waves, the last strips a pair) and
    386 (two strips a wave, K over four); K of 8 k-tiles and of 9, whose shares leave waves without any.  The shapes are checked
    in test_strips_host.py."""
    tol = TOL["bf16"]
    O, model, sess, first, gfirst = _setup(bf16_small(n_layers=3, exit_draft=1, exit_inter=2, d_model=d, d_ffn=ffn), 41, ctx, 3 * (k + 1) + 2)
    assert gfirst.tolist() == first.tolist()
    _round(O, sess, k, 0.8, np.random.default_rng(5), True, tol)
    sess.close(); model.close()


@pytest.mark.parametrize("batch", [4, 10])
def test_seven_weight_tiles_a_workgroup_match_oracle(batch):
    """Gate/up of 3580 weight tiles at 36 and 90 rows: 512 workgroups of seven, the last of three."""
    k, tol = 8, TOL["bf16"]
    O, model, sess, first, gfirst = _setup(bf16_small(n_layers=3, exit_draft=1, exit_inter=2, d_model=272, d_ffn=28640), 41,
                                           [20 + 9 * b for b in range(batch)], 3 * (k + 1) + 2)
    assert gfirst.tolist() == first.tolist()
    _round(O, sess, k, 0.8, np.random.default_rng(5), True, tol)
    sess.close(); model.close()


@pytest.mark.parametrize("row_tiles", [0, 4, 8, 16, 104, 108])
def test_both_forms_of_the_narrow_projection_gemm_match_oracle(row_tiles):
    """The narrow projections (O, down, QKV, adapters) of a call with more than 32 rows run either with K shares and
    a reduction pass (0) or in blocks of row_tiles*16 rows (+100: eight weight tiles per workgroup): each form forced in turn on a case whose context build
    fills whole 512-row passes and ends in a ragged one, and whose verify calls hold 144 rows and 17..64 rows."""
    name, cfg, ctx, k, bonus = next(c for c in CASES if c[0] == "bf16_d128_heads_batch16")
    import paper_2510_01336_amd as hs
    tol = TOL[cfg.dtype]
    hs.ee_debug_gemm_row_blocks(row_tiles)
    try:
        O, model, sess, first, gfirst = _setup(cfg, 777, ctx, 3 * (k + 1) + 2, bonus)
        assert gfirst.tolist() == first.tolist()
        assert max_rel(sess.last_hidden()[-1:], O.o.last_hidden) <= tol
        rng = np.random.default_rng(5)
        _round(O, sess, k, 0.8, rng, True, tol)
        sess.close(); model.close()
    finally:
        hs.ee_debug_gemm_row_blocks(-1)


def test_more_than_512_rows_in_one_call():
    """60 sequences x 9 block rows = 540 rows: beyond the row-tiled GEMM's 512, so the projections run blocked or as 512 rows and the
    rest.  With so many sequences some deciding row is always a near-tie, so every sequence
    is compared as far as its own rows clear the margin (and dropped once the two sides may have parted)."""
    cfg, k, tol = bf16_small(), 8, TOL["bf16"]
    ctx = [5 + (7 * i) % 60 for i in range(60)]
    B, max_rows = len(ctx), 3 * (k + 1) + 2
    max_ctx = max(ctx) + 4 * max_rows
    O = OracleSide(cfg, 777)
    model, sess = gpu_side(cfg, 777, B, max_ctx, max_rows)
    sess.enable_logits(True)
    prompts = [synth.gen_prompt(cfg.vocab, n, 100 + b) for b, n in enumerate(ctx)]
    first, margins = O.prefill(prompts, max_ctx)
    gfirst = sess.prefill(prompts)
    good = np.ones(B, bool)
    for b in range(B):
        if margins[b] > MARGIN:
            assert gfirst[b] == first[b], b
        elif gfirst[b] != first[b]:
            good[b] = False
    rng = np.random.default_rng(3)
    drafts = np.stack([synth.make_draft_block(O.greedy(s, k, cfg.exit_inter), k, 0.7, cfg.vocab, rng) for s in O.seqs])
    sess.draft_inject(drafts)
    ga, gn = sess.verify_intermediate()
    assert sess.last_logits().shape[0] >= B * (k + 1) > 512
    glog, r0, compared_i = sess.last_logits(), 0, 0
    for b, s in enumerate(O.seqs):
        O.o.draft_inject(s, drafts[b])
        a, nxt = O.o.verify_intermediate(s)
        rows = len(O.o.last_logits)
        clear = eo.top2_margin(O.o.last_logits)[:a + 1].min() > MARGIN
        if good[b] and clear:
            assert (int(ga[b]), int(gn[b])) == (a, nxt), b
            assert max_rel(glog[r0:r0 + rows], O.o.last_logits) <= tol
            compared_i += 1
        elif (int(ga[b]), int(gn[b])) != (a, nxt):
            good[b] = False
        r0 += rows
    gf, gn, gcom = sess.verify_full()
    compared_f = 0
    for b, s in enumerate(O.seqs):
        f, nxt, F = O.o.verify_full(s)
        clear = eo.top2_margin(O.o.last_logits)[:f + 1].min() > MARGIN
        if good[b] and clear:
            assert (int(gf[b]), int(gn[b]), gcom[b]) == (f, nxt, F), b
            compared_f += 1
    assert compared_i >= 40 and compared_f >= 30, (compared_i, compared_f)
    sess.close(); model.close()


def test_all_correct_and_wrong_first_blocks():
    cfg = bf16_small()
    k = 8
    O, model, sess, first, gfirst = _setup(cfg, 31, [90], 3 * (k + 1) + 2)
    rng = np.random.default_rng(9)
    s = O.seqs[0]
    for first_mismatch, want_a in ((k, k), (0, 0), (3, 3)):
        S = _pick_drafts(O, sess, k, 0.5, rng, False, first_mismatch=first_mismatch)[0]
        greedy = O.greedy(s, k + 1, cfg.exit_inter)
        sess.draft_inject(S[None])
        ga, gn = sess.verify_intermediate()
        O.o.draft_inject(s, S)
        a, nxt = O.o.verify_intermediate(s)
        assert (int(ga[0]), int(gn[0])) == (a, nxt) == (want_a, greedy[want_a])
    _check_state(O, sess)
    sess.close(); model.close()


def test_self_drafting_matches_oracle():
    """ee_draft (k sequential shallow passes on the device) against the oracle's Generate(L_d, ., k)."""
    # (model, weight seed): the seeds are ones whose first rounds clear the margin filter below
    for cfg, seed in ((synth.tiny_config(gamma=(1.0, 0.3, 0.3)), 99), (bf16_small(), 99), (bf16_small(head_rank=64), 7)):
        k = 4
        O, model, sess, first, gfirst = _setup(cfg, seed, [50, 20], 3 * (k + 1) + 2)
        assert gfirst.tolist() == first.tolist()
        compared = 0
        for rnd in range(6):
            trial = [copy.deepcopy(s) for s in O.seqs]
            clear = True
            for t in trial:
                O.o.draft(t, k)
                clear &= eo.top2_margin(O.o.last_logits).min() > MARGIN
                a, _ = O.o.verify_intermediate(t)
                m = eo.top2_margin(O.o.last_logits)
                clear &= m[:min(a + 1, len(m))].min() > MARGIN
            if clear:
                gS = sess.draft(k)
                for b, s in enumerate(O.seqs):
                    assert gS[b].tolist() == O.o.draft(s, k)
                compared += 1
            else:   # keep both sides moving with a teacher-forced block instead
                drafts = _pick_drafts(O, sess, k, 0.7, np.random.default_rng(rnd), False)
                sess.draft_inject(drafts)
                for b, s in enumerate(O.seqs):
                    O.o.draft_inject(s, drafts[b])
            ga, gn = sess.verify_intermediate()
            for b, s in enumerate(O.seqs):
                assert (int(ga[b]), int(gn[b])) == O.o.verify_intermediate(s)
            if rnd % 2 == 1:
                full_clear = True
                trial = [copy.deepcopy(s) for s in O.seqs]
                for t in trial:
                    f, _, _ = O.o.verify_full(t)
                    m = eo.top2_margin(O.o.last_logits)
                    full_clear &= m[:min(f + 1, len(m))].min() > MARGIN
                if not full_clear:
                    break
                gf, gn, gcom = sess.verify_full()
                for b, s in enumerate(O.seqs):
                    f, nxt, F = O.o.verify_full(s)
                    assert (int(gf[b]), int(gn[b]), gcom[b]) == (f, nxt, F)
            _check_state(O, sess)
        assert compared >= 1
        sess.close(); model.close()


# ------------------------------------------------------------------------------------------------
# cache alignment, rollback, batching
# ------------------------------------------------------------------------------------------------
def test_kv_cache_matches_oracle_and_dead_entries_never_leak():
    cfg = bf16_small()
    k = 8
    O, model, sess, _, _ = _setup(cfg, 55, [100, 30], 3 * (k + 1) + 2, plain=True)
    rng = np.random.default_rng(2)
    tol = TOL["bf16"]
    for rnd in range(4):
        for b in range(2):
            sess.poison_dead_kv(b)          # NaN in every pruned / never-written slot
        _round(O, sess, k, 0.7, rng, rnd % 2 == 1, tol)
        assert np.isfinite(sess.last_logits()).all()
    for side in O.sides():          # every KV entry against the rounding oracle and against the plain model
        for b, s in enumerate(side.seqs):
            for g in range(3):
                for l in cfg.group_layers(g):
                    n = s.len[g]
                    gk, gv = sess.read_kv(b, l, 0, n)
                    ek, ev = max_rel(gk, s.cache.K[l, :n]), max_rel(gv, s.cache.V[l, :n])
                    note(f"bf16_kv_vs_{_tag(side)}", max(ek, ev))
                    assert ek <= tol and ev <= tol, (_tag(side), b, l, ek, ev)
    sess.close(); model.close()


def test_explicit_rollback_restores_prefix_and_continues():
    cfg = bf16_small()
    k = 6
    O, model, sess, _, _ = _setup(cfg, 56, [80], 3 * (k + 1) + 2)
    rng = np.random.default_rng(3)
    tol = TOL["bf16"]
    s = O.seqs[0]
    before = sess.read_kv(0, 0, 0, 80)
    _round(O, sess, k, 0.9, rng, True, tol)
    _round(O, sess, k, 0.9, rng, True, tol)
    assert len(s.C) > 82
    sess.rollback(0, 0b111, 81)
    O.o.rollback(s, 0b111, 81)
    _check_state(O, sess)
    after = sess.read_kv(0, 0, 0, 80)
    assert np.array_equal(before[0], after[0]) and np.array_equal(before[1], after[1])   # no KV bytes moved
    sess.poison_dead_kv(0)
    _round(O, sess, k, 0.8, rng, True, tol)
    # tentative-only cut
    _round(O, sess, k, 1.0, rng, False, tol)
    cut = s.len[0] - 2
    sess.rollback(0, 0b011, cut)
    O.o.rollback(s, 0b011, cut)
    _check_state(O, sess)
    _round(O, sess, k, 0.8, rng, True, tol)
    sess.close(); model.close()


@pytest.mark.parametrize("pinned", [True, False], ids=["same_kv_splits", "free_kv_splits"])
def test_batched_equals_solo(pinned):
    """Per-sequence acceptance: each sequence of a ragged batch behaves exactly as when run alone.  With the
    attention's KV split length pinned, a sequence's context is cut alike alone and in the batch and everything
    it computes -- every logit of both verifications -- is bit-identical to its solo run: the neighbours change
    nothing.  Left free, the split length follows the shape of the whole call, a row's softmax partials are summed
    in another order, a last-bit difference in an fp32 sum can flip the bf16 rounding of an activation, and the
    two runs agree to bf16 accuracy (decisions still equal on these margin-filtered inputs)."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small()
    k = 8
    # pinned: contexts of 33..512 tokens, so that alone and together the context build runs the row-tiled GEMM,
    # whose narrow-projection form is held to K shares as well (it otherwise follows the row count of the pass)
    ctx = [70, 33, 200] if pinned else [70, 5, 200]
    hs.ee_debug_attention_split_pages(2 if pinned else 0)
    hs.ee_debug_gemm_row_blocks(0 if pinned else -1)
    try:
        O, model, sess, _, _ = _setup(cfg, 57, ctx, 3 * (k + 1) + 2)
        rng = np.random.default_rng(4)
        drafts = _pick_drafts(O, sess, k, 0.7, rng, True)
        prompts = [np.array(s.C[:-1], np.int32) for s in O.seqs]     # (a nudge may have shortened a context)
        sess.draft_inject(drafts)
        ga, gn = sess.verify_intermediate()
        blog = sess.last_logits().copy()
        gf, gfn, gcom = sess.verify_full()
        flog = sess.last_logits().copy()
        r0 = f0 = 0
        for b in range(3):
            solo = hs.Session(model, 1, sess.max_ctx, sess.max_rows)
            solo.enable_logits(True)
            solo.prefill([prompts[b]])
            solo.draft_inject(drafts[b:b + 1])
            a, n = solo.verify_intermediate()
            assert (a[0], n[0]) == (ga[b], gn[b])
            sl = solo.last_logits()
            if pinned:
                assert np.array_equal(sl, blog[r0:r0 + len(sl)]), b
            else:
                assert max_rel(sl, blog[r0:r0 + len(sl)].astype(np.float64)) <= TOL["bf16"]
            r0 += len(sl)
            f, fn, com = solo.verify_full()
            assert (f[0], fn[0], com[0]) == (gf[b], gfn[b], gcom[b])
            sl = solo.last_logits()
            if pinned:
                assert np.array_equal(sl, flog[f0:f0 + len(sl)]), b
            f0 += len(sl)
            solo.close()
        sess.close(); model.close()
    finally:
        hs.ee_debug_attention_split_pages(0)
        hs.ee_debug_gemm_row_blocks(-1)


def _equal_in_a_forked_process(arrays, want):
    """A forked process compares the arrays and reports by its exit code."""
    import os
    pid = os.fork()
    if pid == 0:
        code = 1
        try:
            code = 0 if all(np.array_equal(a, w) for a, w in zip(arrays, want)) else 2
        finally:
            os._exit(code)
    return os.waitstatus_to_exitcode(os.waitpid(pid, 0)[1]) == 0


def test_returned_rows_outlive_later_calls_and_the_session():
    """Rows come back in page-locked blocks that are lent to one array at a time: eight arrays held at once (more than there
    are blocks), a view of the first kept alone, then the session closed -- every one still holds what its call returned, here
    and in a forked process.  A call without a number of rows gets a block too; a closed session raises the library's error."""
    import threading
    import paper_2510_01336_amd as hs
    cfg = bf16_small(vocab=4096)               # (18 rows of logits: 295 KB, above the least size that gets a block)
    k = 8
    O, model, sess, _, _ = _setup(cfg, 58, [60, 40], 3 * (k + 1) + 2)
    assert not sess._logits.blocks and not sess._hidden.blocks       # (made by the calls that need them)
    held, want = [], []
    for i in range(8):
        sess.draft_inject(np.random.default_rng(i).integers(0, cfg.vocab, (2, k)).astype(np.int32))
        sess.verify_intermediate()
        rows = sess.last_logits(18)
        assert rows.shape == (18, cfg.vocab) and all(not np.shares_memory(rows, h) for h in held)
        held.append(rows); want.append(rows.copy())
        assert np.array_equal(sess.last_logits(7), rows[:7])
        for b in range(2):
            sess.rollback(b, 0b111, O.seqs[b].len[0])
    assert any(not np.array_equal(want[0], w) for w in want[1:])
    view = held[0][3:5]
    del held[0], rows
    again = sess.last_logits(18)
    assert not np.shares_memory(again, view) and np.array_equal(again, want[7])
    assert len(sess._logits.blocks) == sess._logits.BLOCKS
    assert _equal_in_a_forked_process([view] + held, [want[0][3:5]] + want[1:])
    got = [None] * 4                           # several threads read one session
    def read(i):
        got[i] = [sess.last_logits(18) for _ in range(5)]
    threads = [threading.Thread(target=read, args=(i,)) for i in range(4)]
    for t in threads: t.start()
    for t in threads: t.join()
    assert all(np.array_equal(x, want[7]) for g in got for x in g)
    del got
    held = held[3:]; want[1:] = want[4:]
    default = sess.last_logits()               # (a larger request: up to 512 rows)
    assert default.shape == (18, cfg.vocab) and np.array_equal(default, want[-1]) and default.base is not None
    assert any(b[0].numel() == 512 * cfg.vocab * 4 for b in sess._logits.blocks)
    sess.close()
    for call in (sess.last_logits, sess.last_hidden):
        with pytest.raises(hs.EEError):
            call(18)
        with pytest.raises(hs.EEError):
            call()
    model.close()
    assert _equal_in_a_forked_process([view, default] + held, [want[0][3:5], want[-1]] + want[1:])
    assert np.array_equal(view, want[0][3:5])
    for h, w in zip(held, want[1:]):
        assert np.array_equal(h, w)


@pytest.mark.parametrize("batch", [3, 4, 5, 8, 9, 13, 16])
def test_rows_of_every_quad_equal_a_lone_row(batch):
    """A few rows are read in quads of four, the rows past the last one standing in for those that are not there: one prompt in
    every slot of a batch, decoded by one row each, gives every slot the logits and hidden row of the prompt alone."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small()
    model = hs.Model(cfg, 58)
    prompt = synth.gen_prompt(cfg.vocab, 2, 3)
    got = []
    hs.ee_debug_attention_form(2)
    try:
        for n in (1, batch):
            sess = hs.Session(model, n, 64, 12)
            sess.enable_logits(True)
            sess.prefill([prompt] * n)
            tokens = sess.decode_ar(1)
            got.append((tokens, sess.last_logits(n), sess.last_hidden(n)))
            sess.close()
    finally:
        hs.ee_debug_attention_form(-1)
    model.close()
    for alone, rows in zip(*got):
        assert np.array_equal(np.repeat(alone, batch, axis=0), rows)


@pytest.mark.parametrize("batch", [17, 27, 32])
@pytest.mark.parametrize("shape", [dict(d_model=256, d_ffn=14336, vocab=28672), dict(n_q_heads=96, n_kv_heads=16),
                                   dict(d_model=3584, d_ffn=8192)], ids=["1792_strips", "512_strips", "224_strips_256_ktiles"])
def test_a_row_has_the_same_bits_beside_any_number_of_others(batch, shape):
    """Matrices below 128 MB, whose rows are summed in one order from 1 to 32 rows: gate/up and head of 1792 strips, QKV of 512 strips
    and 8 k-tiles, down of 224 strips and 256 k-tiles.  One prompt of one token in every slot of a batch, built and decoded by one row each."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_layers=3, exit_draft=1, exit_inter=2, **shape)
    model = hs.Model(cfg, 58)
    prompt = synth.gen_prompt(cfg.vocab, 1, 3)
    got = []
    hs.ee_debug_attention_form(2)
    try:
        for n in (1, batch):
            sess = hs.Session(model, n, 64, 12)
            sess.enable_logits(True)
            sess.prefill([prompt] * n)
            tokens = sess.decode_ar(1)
            got.append((tokens, sess.last_logits(n), sess.last_hidden(n)))
            sess.close()
    finally:
        hs.ee_debug_attention_form(-1)
    model.close()
    for alone, rows in zip(*got):
        assert np.array_equal(np.repeat(alone, batch, axis=0), rows)


@pytest.mark.parametrize("batch", [18, 27, 32])
@pytest.mark.parametrize("shape", [dict(d_model=8192, n_q_heads=64, head_dim=128, n_kv_heads=8, d_ffn=28672, vocab=32000),
                                   dict(d_model=2400, d_ffn=14320, vocab=28632), dict(d_model=2720, d_ffn=14320, vocab=28632),
                                   dict(d_model=3104, d_ffn=11008, vocab=28632)], ids=["70b", "75_ktiles", "85_ktiles", "97_ktiles"])
def test_17_to_32_rows_of_large_matrices_agree_with_a_row_alone(batch, shape):
    """Matrices of 128 MB and more, which get strips or the row-tiled kernel.  70B width: QKV and head of the row-tiled one (QKV in K
    shares), down of either, gate/up as seven strips a wave (32 k-tiles a K share).  Then gate/up and head of 1790 strips, seven a wave with a
    last workgroup of five, in K shares of 10 k-tiles and a last one of 5, of 11 and 8, of 13 and 6; 1376 strips a wave short of an even deal.
    Another order of the sums over K than one row alone: bf16 accuracy.  The shapes are checked in test_strips_host.py."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_layers=3, exit_draft=1, exit_inter=2, sigma=0.02, **shape)
    model = hs.Model(cfg, 58)
    prompt = synth.gen_prompt(cfg.vocab, 1, 3)
    got = []
    for n in (1, batch):
        sess = hs.Session(model, n, 64, 12)
        sess.enable_logits(True)
        sess.prefill([prompt] * n)
        got.append((sess.last_logits(n), sess.last_hidden(n)))
        sess.close()
    model.close()
    for alone, rows in zip(*got):
        assert max_rel(rows[0], alone[0].astype(np.float64)) <= TOL["bf16"]
        assert all(np.array_equal(rows[0], r) for r in rows[1:])       # (the same row in every slot)


def test_forced_row_tiled_forms_reach_large_matrices_from_17_rows():
    """18 rows of a model whose gate/up and head hold 128 MB and more: strips as the library runs them, and each forced form of the
    row-tiled kernels, agree to bf16 accuracy; a forced form is another order of sums, so that some bits differ."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_layers=3, exit_draft=1, exit_inter=2, sigma=0.02, d_model=2720, d_ffn=14320, vocab=28632)
    model = hs.Model(cfg, 58)
    prompts = [synth.gen_prompt(cfg.vocab, 1, b) for b in range(18)]
    got = {}
    try:
        for form in ("strips", "shares", "blocks"):
            hs.ee_debug_gemm_row_blocks(0 if form == "shares" else -1)
            hs.ee_debug_gemm_block_tiles(16 if form == "blocks" else 0)
            sess = hs.Session(model, 18, 64, 12)
            sess.enable_logits(True)
            sess.prefill(prompts)
            got[form] = sess.last_logits(18)
            sess.close()
    finally:
        hs.ee_debug_gemm_row_blocks(-1); hs.ee_debug_gemm_block_tiles(0)
    model.close()
    for form in ("shares", "blocks"):
        assert max_rel(got[form], got["strips"].astype(np.float64)) <= TOL["bf16"]
        assert not np.array_equal(got[form], got["strips"])


@pytest.mark.parametrize("pages", [136, 137, 648, 649])
def test_metadata_of_every_size_reaches_the_kernels(pages):
    """A call of nine rows whose metadata holds 256, 260, 768 and 772 integers (the block table makes up the size): stored by
    a kernel of 256 or 768 integers, or copied.  The rounds equal those of a session with a short table bit for bit."""
    import paper_2510_01336_amd as hs
    cfg, k, rows = bf16_small(), 8, 29
    model = hs.Model(cfg, 58)
    prompt, drafts = synth.gen_prompt(cfg.vocab, 60, 3), np.random.default_rng(2).integers(0, cfg.vocab, (1, k)).astype(np.int32)
    got = []
    for n in (4, pages):
        sess = hs.Session(model, 1, n * 64, rows, 4)
        sess.enable_logits(True)
        first = sess.prefill([prompt])
        sess.draft_inject(drafts)
        vi = sess.verify_intermediate()
        li = sess.last_logits(k + 1)
        vf = sess.verify_full()
        got.append((first, vi, li, vf[0], vf[1], vf[2][0], sess.last_logits(2 * k)))
        sess.close()
    model.close()
    for a, b in zip(*got):
        assert np.array_equal(a, b)


def test_rerun_is_bit_identical():
    cfg = bf16_d128()
    k = 8
    O, model, sess, _, _ = _setup(cfg, 58, [200], 3 * (k + 1) + 2)
    drafts = _pick_drafts(O, sess, k, 0.8, np.random.default_rng(6), False)
    n0 = O.seqs[0].len[0]
    outs = []
    for _ in range(3):
        sess.draft_inject(drafts)
        a, n = sess.verify_intermediate()
        outs.append((a.copy(), n.copy(), sess.last_logits().copy()))
        sess.rollback(0, 0b011, n0)
    for o in outs[1:]:
        assert np.array_equal(o[0], outs[0][0]) and np.array_equal(o[1], outs[0][1]) and np.array_equal(o[2], outs[0][2])
    sess.close(); model.close()


# ------------------------------------------------------------------------------------------------
# error behaviour
# ------------------------------------------------------------------------------------------------
def test_error_codes_leave_state_untouched():
    import paper_2510_01336_amd as hs
    cfg = synth.tiny_config()
    model, sess = gpu_side(cfg, 1, 1, 128, 12)
    with pytest.raises(hs.EEError) as e:
        sess.draft(2)
    assert e.value.code == -2                       # no context yet
    sess.prefill([synth.gen_prompt(cfg.vocab, 20, 1)])
    with pytest.raises(hs.EEError) as e:
        sess.verify_intermediate()
    assert e.value.code == -2                       # nothing drafted
    with pytest.raises(hs.EEError) as e:
        sess.verify_full()
    assert e.value.code == -2                       # nothing tentative
    with pytest.raises(hs.EEError) as e:
        sess.draft(40)
    assert e.value.code == -1                       # more rows than max_rows
    with pytest.raises(hs.EEError) as e:
        sess.rollback(0, 0b111, 25)
    assert e.value.code == -1                       # growing is not a rollback
    with pytest.raises(hs.EEError) as e:
        sess.rollback(0, 0b001, 5)
    assert e.value.code == -1
    with pytest.raises(hs.EEError) as e:
        sess.draft_inject(np.array([[cfg.vocab]]))
    assert e.value.code == -1
    assert sess.lengths().tolist() == [[20, 20, 20]]
    sess.draft(3)
    with pytest.raises(hs.EEError) as e:
        sess.draft(3)
    assert e.value.code == -2                       # a block is already pending
    sess.verify_intermediate()
    # capacity: a context that cannot grow any further
    small = hs.Session(model, 1, 24, 12)
    small.prefill([synth.gen_prompt(cfg.vocab, 20, 1)])
    with pytest.raises(hs.EEError) as e:
        small.draft(4)
    assert e.value.code == -3
    with pytest.raises(hs.EEError) as e:
        hs.Session(model, 1, 100000, 12)            # fp32 sessions are limited to 8192 positions
    small.close(); sess.close(); model.close()


# ------------------------------------------------------------------------------------------------
# one sequence leaves, another takes its slot
# ------------------------------------------------------------------------------------------------
def test_sequence_restart_keeps_the_others():
    import paper_2510_01336_amd as hs
    cfg = bf16_small()
    k = 6
    O, model, sess, first, gfirst = _setup(cfg, 31, [90, 40, 130], 3 * (k + 1) + 2)
    assert gfirst.tolist() == first.tolist()
    rng = np.random.default_rng(8)
    _round(O, sess, k, 0.7, rng, True, TOL["bf16"])
    before = [(sess.lengths()[b].tolist(), sess.tokens(b).tolist(), sess.read_kv(b, 3, 0, int(sess.lengths()[b][0]))) for b in (0, 2)]
    # sequence 1 is replaced by a longer prompt; the margin of its first token is checked like any other
    for attempt in range(20):
        prompt = synth.gen_prompt(cfg.vocab, 150, 900 + attempt)
        s_new = eo.Sequence_(O.model.spec, O.seqs[0].cache.capacity)
        f_new = O.o.prefill(s_new, prompt)
        if eo.top2_margin(O.o.last_logits)[0] > MARGIN:
            break
    assert sess.prefill_seq(1, prompt) == f_new
    O.seqs[1] = s_new
    for (lens, toks, (kk, vv)), b in zip(before, (0, 2)):
        assert sess.lengths()[b].tolist() == lens and sess.tokens(b).tolist() == toks
        k2, v2 = sess.read_kv(b, 3, 0, lens[0])
        assert np.array_equal(kk, k2) and np.array_equal(vv, v2)
    _check_state(O, sess)
    _round(O, sess, k, 0.7, rng, True, TOL["bf16"])          # all three go on together
    sess.close(); model.close()
    # a pool too small for the newcomer: refused, nothing changes
    model, sess = gpu_side(cfg, 31, 2, 400, 3 * (k + 1) + 2)
    sess.close()
    sess = hs.Session(model, 2, 400, 3 * (k + 1) + 2, total_pages=5)
    sess.prefill([synth.gen_prompt(cfg.vocab, 100, 1), synth.gen_prompt(cfg.vocab, 100, 2)])      # 2 + 2 pages
    lens = sess.lengths().tolist()
    with pytest.raises(hs.EEError):
        sess.prefill_seq(0, synth.gen_prompt(cfg.vocab, 300, 3))                                   # would need 5 of 3 + 2 free
    assert sess.lengths().tolist() == lens
    assert isinstance(sess.prefill_seq(0, synth.gen_prompt(cfg.vocab, 150, 3)), int)               # 3 pages fit
    sess.close(); model.close()


def test_released_slot_idles_while_the_batch_goes_on():
    """ee_seq_release: the pages go back to the pool, the slot takes no part in the batch-wide calls (which
    report -1 for it), the other sequences verify exactly as the oracle says, and the
    slot can be started again."""
    cfg = bf16_small()
    k, tol = 6, TOL["bf16"]
    O, model, sess, first, gfirst = _setup(cfg, 31, [90, 40, 130], 3 * (k + 1) + 2)
    rng = np.random.default_rng(12)
    _round(O, sess, k, 0.7, rng, True, tol)
    free0, held = sess.free_pages(), -(-(int(sess.lengths()[1].max()) + 1) // 64)
    sess.release(1)
    assert sess.free_pages() == free0 + held
    assert sess.lengths()[1].tolist() == [0, 0, 0] and sess.tokens(1).tolist() == []
    live, B = (0, 2), 3
    for rnd in range(2):
        drafts = np.full((B, k), -7, np.int32)               # the idle slot's entries are never read
        for b in live:
            s = O.seqs[b]
            greedy = O.greedy(s, k, cfg.exit_inter)
            for _ in range(25):
                S = synth.make_draft_block(greedy, k, 0.7, cfg.vocab, rng, first_mismatch=synth.draw_first_mismatch(k, 0.7, rng))
                if _trial_round(O, [s], [S], True) > MARGIN:
                    break
            else:
                pytest.fail("no draft block cleared the margin filter")
            drafts[b] = S
        sess.draft_inject(drafts)
        ga, gn = sess.verify_intermediate()
        for b in range(B):
            if b in live:
                O.o.draft_inject(O.seqs[b], drafts[b])
                assert (int(ga[b]), int(gn[b])) == O.o.verify_intermediate(O.seqs[b])
            else:
                assert (int(ga[b]), int(gn[b])) == (-1, -1)
        gf, gn, gcom = sess.verify_full()
        for b in range(B):
            if b in live:
                f, nxt, F = O.o.verify_full(O.seqs[b])
                assert (int(gf[b]), int(gn[b]), gcom[b]) == (f, nxt, F)
            else:
                assert (int(gf[b]), int(gn[b]), list(gcom[b])) == (-1, -1, [])
        lens = sess.lengths()
        for b in live:
            assert list(lens[b]) == O.seqs[b].len and sess.tokens(b).tolist() == O.seqs[b].T
        assert lens[1].tolist() == [0, 0, 0]
    # self-drafting and vanilla steps skip the idle slot as well
    gS = sess.draft(2)
    assert gS[1].tolist() == [-1, -1] and all(0 <= t < cfg.vocab for b in live for t in gS[b])
    sess.verify_intermediate(); sess.verify_full()
    before = sess.lengths().copy()
    out = sess.decode_ar(2)
    assert out[1].tolist() == [-1, -1] and sess.lengths()[1].tolist() == [0, 0, 0]
    for b in live:
        assert (sess.lengths()[b] == before[b].max() + 2).all()
    # bring the oracle's live sequences to where the GPU now stands by replaying the GPU's committed streams
    # through the oracle's own prefill (they are inputs from here on), then start the slot again
    import paper_2510_01336_amd as hs
    for b in live:
        toks = sess.tokens(b).tolist()
        s_new = eo.Sequence_(O.model.spec, O.seqs[b].cache.capacity)
        O.o.prefill(s_new, toks[:-1])
        s_new.C[-1] = toks[-1]
        O.seqs[b] = s_new
    for attempt in range(20):
        prompt = synth.gen_prompt(cfg.vocab, 70, 500 + attempt)
        s_new = eo.Sequence_(O.model.spec, O.seqs[0].cache.capacity)
        f_new = O.o.prefill(s_new, prompt)
        if eo.top2_margin(O.o.last_logits)[0] > MARGIN:
            break
    assert sess.prefill_seq(1, prompt) == f_new
    O.seqs[1] = s_new
    _check_state(O, sess)
    _round(O, sess, k, 0.7, rng, True, tol)
    # nothing started: the batch-wide calls say so
    for b in range(B):
        sess.release(b)
    with pytest.raises(hs.EEError):
        sess.draft(2)
    with pytest.raises(hs.EEError):
        sess.decode_ar(1)
    sess.close(); model.close()


@pytest.mark.gpu
def test_read_floor_times_plain_reads():
    """The measurement entry point behind bench.py's read_floor: every region gets a positive time, a region sixteen times
    the size takes longer, and the implied rate stays below the chip's 8 TB/s."""
    import torch
    import paper_2510_01336_amd as hs
    sizes = [8 << 20, 128 << 20]
    buf = torch.full((sum(sizes),), 5, dtype=torch.uint8, device="cuda")
    torch.cuda.synchronize()
    us = hs.ee_debug_read_floor(buf.data_ptr(), sizes, 5, 0)
    assert len(us) == 2 and 0.5 < us[0] < us[1] < 1e4
    assert sizes[1] / (us[1] * 1e-6) < 8.0e12
    with pytest.raises(hs.EEError):
        hs.ee_debug_read_floor(buf.data_ptr() + 4, sizes, 5, 0)


@pytest.mark.parametrize("rows", [257, 512, 513, 767, 1025])
@pytest.mark.parametrize("name", ["bf16_wide", "bf16_d128"])
def test_context_build_in_blocks_matches_the_512_row_passes(name, rows):
    """Context builds of more than 256 / 512 rows as the library runs them (blocked GEMMs, attention by the shape of the call)
    against the forms that the hooks force (K shares, 512-row passes, KV splits of four pages): rows around the block edges
    and a ragged last block, both ways within the bf16 bound of each other and the same first token, on a prompt whose last
    row clears the margin."""
    import paper_2510_01336_amd as hs
    # 2 * d_ffn / 16 weight tiles: 1546 (the wide form's floor is 1536, 1546 = 96 * 16 + 10) with few k-tiles, or narrow only
    cfg = bf16_small(d_ffn=12368, sigma=0.02) if name == "bf16_wide" else bf16_d128()
    model = hs.Model(cfg, 31)
    sess = hs.Session(model, 2, rows + 40, 12)
    sess.enable_logits(True)
    for seed in range(12):
        prompts = [synth.gen_prompt(cfg.vocab, n, 70 + seed + n) for n in (rows - 30, 30)]       # (two sequences share the pass)
        first = sess.prefill(prompts)
        got, hid = sess.last_logits()[-1:].astype(np.float64), sess.last_hidden()[-1:].copy()
        if eo.top2_margin(got)[0] > 4 * MARGIN:
            break
    else:
        raise AssertionError("no prompt cleared the margin")
    step = sess.decode_ar(1)
    after = sess.last_logits(2).astype(np.float64)
    hs.ee_debug_gemm_row_blocks(0); hs.ee_debug_gemm_row_blocks(1000); hs.ee_debug_attention_split_pages(4)
    try:
        assert sess.prefill(prompts)[1] == first[1]
        ref = sess.last_logits()[-1:].astype(np.float64)
        assert max_rel(got, ref) <= TOL["bf16"] and max_rel(hid, sess.last_hidden()[-1:].astype(np.float64)) <= TOL["bf16"]
        if int(first[0]) == int(sess.tokens(0)[-1]):            # (the first sequence's token may be a near-tie)
            sess.decode_ar(1)
            assert max_rel(after, sess.last_logits(2).astype(np.float64)) <= TOL["bf16"]           # every cached row enters here
    finally:
        hs.ee_debug_gemm_row_blocks(-1); hs.ee_debug_attention_split_pages(0)
    assert step.shape == (2, 1)
    sess.close(); model.close()


@pytest.mark.parametrize("lens,passes", [
    ([700], 0), ([513], 0), ([1041], 0), ([527, 530], 0),                       # one sequence reaches into the reported piece
    ([40, 600, 3, 530, 17], 0), ([5, 5, 509, 200], 0), ([1, 511, 1, 300], 0),     # prompts that end in front of it; a piece that starts with a sequence
    ([300, 300, 200, 1], 0), ([100] * 7 + [900], 0),
    ([700, 30, 1100], 512), ([1500, 9], 512),                                  # several passes, some of which end no prompt
])
@pytest.mark.parametrize("name", ["bf16_small", "bf16_rep3"])
def test_last_layer_of_a_context_build_over_the_rows_that_are_read(name, lens, passes):
    """A context build runs its last layer over the rows that end a prompt and the reported piece alone: first tokens, the reported hidden
    rows and every cached K and V row of all layers against the oracle, as a session is by default and once more with logits kept,
    which are compared too, and a decoding step behind it."""
    import re

    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_layers=3, exit_draft=1, exit_inter=2) if name == "bf16_small" else bf16_small(n_layers=3, exit_draft=1, exit_inter=2, n_q_heads=6)
    W = synth.WeightStore(cfg, 41)
    spec = eo.ModelSpec.from_config(cfg, round_mode="bf16")
    m = eo.EEModel(spec, W)
    hidden, firsts, prompts, caches = [], [], [], []
    for b, n in enumerate(lens):
        for seed in range(40):
            prompt = synth.gen_prompt(cfg.vocab, n, 900 + 50 * b + seed)
            cache = eo.KVCache(spec, n)
            x = m.run_layers(range(cfg.n_layers), m.embed(prompt), np.arange(n), cache)
            logits = m.exit_logits(x[-1:])
            if eo.top2_margin(logits)[0] > 2 * MARGIN:
                break
        else:
            raise AssertionError("no prompt whose first token is decided clearly")
        caches.append(cache); prompts.append(prompt); hidden.append(x); firsts.append(int(eo.argmax_rows(logits)[0]))
    model = hs.Model(cfg, 41)
    least = None
    if passes:                                                 # the smallest arena: passes of 512 rows
        with pytest.raises(hs.EEError) as e:
            hs.Session(model, len(lens), max(lens) + 20, 8, arena_bytes=1 << 12)
        least = int(re.search(r"< (\d+)", str(e.value)).group(1))
    sess = hs.Session(model, len(lens), max(lens) + 20, 8, arena_bytes=least)
    # rows of the last pass in packing order, the last 512-row piece of them
    if not passes:
        rows = np.concatenate(hidden)
    else:
        left, done = list(lens), [0] * len(lens)
        while any(left):
            room, rows = 512, []
            for b in range(len(lens)):
                n = min(left[b], room)
                rows += list(hidden[b][done[b]:done[b] + n]); left[b] -= n; done[b] += n; room -= n
        rows = np.array(rows)
    want = rows[(len(rows) - 1) // 512 * 512:]
    for logits in (False, True):
        sess.enable_logits(logits)
        assert sess.prefill(prompts).tolist() == firsts
        got = sess.last_hidden()
        assert got.shape == want.shape
        assert max_rel(got.astype(np.float64), want) <= TOL["bf16"]
        for b, n in enumerate(lens):
            for layer in range(cfg.n_layers):
                gk, gv = sess.read_kv(b, layer, 0, n)
                assert max_rel(gk, caches[b].K[layer]) <= TOL["bf16"] and max_rel(gv, caches[b].V[layer]) <= TOL["bf16"], (b, layer)
    assert max_rel(sess.last_logits().astype(np.float64), m.exit_logits(want)) <= TOL["bf16"]
    sess.decode_ar(1)
    step = sess.last_hidden(len(lens)).astype(np.float64)
    for b, n in enumerate(lens):
        x, _ = m.forward_nocache(list(prompts[b]) + [firsts[b]], cfg.n_layers)
        assert max_rel(step[b:b + 1], x[-1:]) <= TOL["bf16"], b
    sess.close(); model.close()


@pytest.mark.parametrize("rows", [2, 9, 16, 17, 32])
@pytest.mark.parametrize("heads", [(60, 5), (120, 8)], ids=["280_strips", "544_strips"])
def test_qkv_in_half_strips_matches_oracle(heads, rows):
    """QKV matrices whose strips do not fill the compute units evenly: pairs of workgroups share 3 or 5 strips, the last pair fewer
    (280 = 93 * 3 + 1, 544 = 108 * 5 + 4).  A block behind a short context, its logits and its cached K and V against the oracle."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_layers=3, exit_draft=1, exit_inter=2, d_model=2048, n_q_heads=heads[0], n_kv_heads=heads[1], d_ffn=256, sigma=0.02)
    W = synth.WeightStore(cfg, 5)
    m = eo.EEModel(eo.ModelSpec.from_config(cfg, round_mode="bf16"), W)
    model = hs.Model(cfg, 5)
    sess = hs.Session(model, 1, 128, 2 * rows + 4)
    sess.enable_logits(True)
    prompt = synth.gen_prompt(cfg.vocab, 21, 3)
    c0 = int(sess.prefill([prompt])[0])
    block = np.random.default_rng(rows).integers(0, cfg.vocab, (1, rows - 1)).astype(np.int32)
    sess.draft_inject(block)
    tokens = [int(t) for t in prompt] + [c0] + [int(t) for t in block[0]]
    cache = eo.KVCache(m.spec, len(tokens))
    x = m.run_layers(range(cfg.exit_inter), m.embed(tokens), np.arange(len(tokens)), cache)[len(prompt):]
    gk, gv = sess.read_kv(0, 0, 0, len(tokens))
    assert max_rel(gk, cache.K[0]) <= TOL["bf16"] and max_rel(gv, cache.V[0]) <= TOL["bf16"]
    sess.verify_intermediate()
    assert max_rel(sess.last_hidden().astype(np.float64), x) <= TOL["bf16"]
    assert max_rel(sess.last_logits().astype(np.float64), m.exit_logits(x)) <= TOL["bf16"]
    sess.close(); model.close()


_BLOCK_CFGS = {
    # weight tiles: QKV 48, O / down 16, gate/up 1546 (96 * 16 + 10); down over 387 k-tiles
    "long_k": lambda: bf16_small(d_ffn=12368, sigma=0.02),
    # QKV 80, O / down 32, head 128
    "d128": lambda: bf16_d128(),
    # QKV 40, O / down 17 over 12 and 4 k-tiles (fewer than the stages of the ring), gate/up 14, head 1537; adapters of rank 32
    "ragged": lambda: bf16_small(d_model=272, n_q_heads=6, d_ffn=100, vocab=24592, sigma=0.1, head_rank=32),
}


@pytest.mark.parametrize("rows", [40, 177, 256, 257, 497, 512, 785])
@pytest.mark.parametrize("name", list(_BLOCK_CFGS))
def test_blocked_gemm_in_every_form(name, rows):
    """The blocked GEMM with 8, 12 and 16 weight and 8, 12 and 16 row tiles per workgroup, every epilogue in every form it is built with, at row
    blocks that are full, partly filled and hold one row, groups of weight tiles that are not, and parts short enough for
    norm factors to be left to the consumer elsewhere: the forms sum K in one order, so logits, hidden rows and cached K and V
    are the same bits; against the row-tiled forms they agree to bf16 accuracy."""
    import paper_2510_01336_amd as hs
    cfg = _BLOCK_CFGS[name]()
    model = hs.Model(cfg, 31)
    k = 40 if rows < 300 else 8
    lens = [rows - 17, 17]
    drafts = np.random.default_rng(rows).integers(0, cfg.vocab, (2, k)).astype(np.int32)
    for seed in range(12):
        prompts = [synth.gen_prompt(cfg.vocab, n, 70 + seed + n) for n in lens]
        got = {}
        hs.ee_debug_attention_split_pages(4)
        try:
            for form in ("rows", 8, 12, 808, 1208, 1212, 16):
                hs.ee_debug_gemm_block_tiles(0 if form == "rows" else form)
                if form == "rows":
                    hs.ee_debug_gemm_row_blocks(0); hs.ee_debug_gemm_row_blocks(1000)
                else:
                    hs.ee_debug_gemm_row_blocks(-1)
                sess = hs.Session(model, 2, rows + 2 * k + 40, 2 * k + 6)
                sess.enable_logits(True)
                first = sess.prefill(prompts)
                out = [sess.last_logits(), sess.last_hidden()]
                sess.draft_inject(drafts)
                sess.verify_intermediate()
                out += [sess.last_logits(), sess.last_hidden()]
                for b in range(2):
                    for l in range(cfg.n_layers):
                        out += list(sess.read_kv(b, l, 0, lens[b]))
                got[form] = (first, out)
                sess.close()
        finally:
            hs.ee_debug_gemm_block_tiles(0); hs.ee_debug_gemm_row_blocks(-1); hs.ee_debug_attention_split_pages(0)
        if np.array_equal(got["rows"][0], got[16][0]):         # (else a first token is a near-tie: another prompt)
            break
    else:
        raise AssertionError("no prompt whose first tokens are decided clearly")
    for form in (8, 12, 808, 1208, 1212):
        for i, (x, y) in enumerate(zip(got[form][1], got[16][1])):
            assert np.array_equal(x, y), (form, i)
    for i, (x, y) in enumerate(zip(got[16][1], got["rows"][1])):
        assert np.isfinite(x).all() and max_rel(x, y.astype(np.float64)) <= TOL["bf16"], i
    model.close()


@pytest.mark.parametrize("batch", [16, 17, 18, 20, 21, 32, 33])
@pytest.mark.parametrize("name", list(_BLOCK_CFGS))
def test_calls_beyond_512_rows_in_every_route(name, batch):
    """Batch-wide calls of 512 to 1056 rows as the library runs them -- one blocked launch, or 512 rows and the rest, whose last
    part holds 32 rows (skinny kernel), up to 128, and up to 512 (row-tiled forms, K shares) -- against the blocked kernel
    throughout: the same block of drafts behind the same contexts, through the adapters and heads as well."""
    import paper_2510_01336_amd as hs
    cfg = _BLOCK_CFGS[name]()
    model = hs.Model(cfg, 31)
    k = 31
    sess = hs.Session(model, batch, 60, k + 5)
    sess.enable_logits(True)
    sess.prefill([synth.gen_prompt(cfg.vocab, 5 + b % 3, b) for b in range(batch)])
    drafts = np.random.default_rng(batch).integers(0, cfg.vocab, (batch, k)).astype(np.int32)
    got = []
    hs.ee_debug_attention_form(0)
    try:
        for tiles in (0, 16):
            hs.ee_debug_gemm_block_tiles(tiles)
            sess.draft_inject(drafts)
            sess.verify_intermediate()
            got.append([sess.last_logits(), sess.last_hidden()])
            assert len(got[-1][0]) == 32 * batch
            for b in range(batch):
                sess.rollback(b, 0b111, 5 + b % 3)
    finally:
        hs.ee_debug_gemm_block_tiles(0); hs.ee_debug_attention_form(-1)
    for x, y in zip(*got):
        assert np.isfinite(x).all()
        for r0 in range(0, 32 * batch, 32):                     # (sequence by sequence: no part hides behind the others' scale)
            assert max_rel(x[r0:r0 + 32], y[r0:r0 + 32].astype(np.float64)) <= TOL["bf16"], r0
    sess.close(); model.close()


# bytes of the session arenas of these shapes where a context-build pass never had more than 512 rows
@pytest.mark.parametrize("batch,max_ctx,max_rows,nbytes", [(2, 3000, 20, 24127744), (64, 100, 12, 66178816)])
def test_arena_of_512_row_passes_is_accepted(batch, max_ctx, max_rows, nbytes):
    """An arena too small for passes of 4096 rows gets shorter ones: the context build of prompts that take several of them
    (rows behind cached ones, prompts cut by a pass) against the build in passes of 4096, then a block of all rows at once
    (more than 512 for the larger batch) and a vanilla step; an arena that holds no pass at all is refused."""
    import paper_2510_01336_amd as hs
    cfg = synth.EEConfig(n_layers=3, d_model=256, n_q_heads=8, n_kv_heads=2, head_dim=64, d_ffn=688, vocab=1000, exit_draft=1, exit_inter=2,
                         dtype="bf16", sigma=0.05, gamma=(1.0, 0.2, 0.2))
    model = hs.Model(cfg, 31)
    assert hs.ee_session_bytes(model.handle, batch, max_ctx, max_rows, 0) > nbytes
    rng = np.random.default_rng(2)
    k = max_rows - 3
    lens = [1500, 1190] if batch == 2 else [max_ctx - 2 * max_rows - 1 - b % 7 for b in range(batch)]
    prompts = [synth.gen_prompt(cfg.vocab, n, 40 + b) for b, n in enumerate(lens)]
    drafts = rng.integers(0, cfg.vocab, (batch, k)).astype(np.int32)
    got = []
    for size in (None, nbytes):
        sess = hs.Session(model, batch, max_ctx, max_rows, arena_bytes=size)
        sess.enable_logits(True)
        first = sess.prefill(prompts)
        last = sess.last_hidden()
        sess.draft_inject(drafts)
        sess.verify_intermediate()
        block = sess.last_logits().astype(np.float64)
        kv = [sess.read_kv(b, 0, 0, lens[b]) for b in (0, batch - 1)]
        got.append((first, last, block, kv))
        sess.close()
    (f0, l0, b0, kv0), (f1, l1, b1, kv1) = got
    assert len(l0) == len(l1) == (sum(lens) - 1) % 512 + 1
    assert max_rel(l1, l0.astype(np.float64)) <= TOL["bf16"]
    assert np.mean(f0 == f1) >= 0.9                       # (a near-tie may fall either way)
    same = np.repeat(f0 == f1, k + 1)                     # the block starts with the first token
    assert max_rel(b1[same], b0[same]) <= TOL["bf16"]
    for (k0, v0), (k1, v1) in zip(kv0, kv1):
        assert max_rel(k1, k0.astype(np.float64)) <= TOL["bf16"] and max_rel(v1, v0.astype(np.float64)) <= TOL["bf16"]
    with pytest.raises(hs.EEError) as e:
        hs.Session(model, batch, max_ctx, max_rows, arena_bytes=nbytes // 2)
    assert e.value.code == -3 and "arena too small" in str(e.value)
    model.close()


@pytest.mark.parametrize("d,ffn,heads,vocab", [(66, 70, (2, 1), 130), (68, 41, (4, 2), 1001), (256, 100, (3, 3), 77)])
def test_fp32_projections_at_odd_widths_match_oracle(d, ffn, heads, vocab):
    """The fused fp32 projections where their 16-byte loads do not apply (widths that are no multiple of four), at row counts
    around the four rows of a wave and with unit counts that leave waves idle: against the oracle, fp32 bound."""
    cfg = synth.EEConfig(n_layers=4, d_model=d, n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=32, d_ffn=ffn, vocab=vocab,
                         exit_draft=1, exit_inter=2, dtype="f32", sigma=0.1, gamma=(1.0, 0.3, 0.3))
    tol, k = TOL["f32"], 4
    O, model, sess, first, gfirst = _setup(cfg, 5, [9, 66], 3 * (k + 1) + 2)
    assert gfirst.tolist() == first.tolist()
    assert max_rel(sess.last_logits()[-1:], O.o.last_logits) <= tol
    rng = np.random.default_rng(8)
    _round(O, sess, k, 0.8, rng, True, tol)
    sess.close(); model.close()


@pytest.mark.parametrize("dim", [2, 16, 40, 48, 80, 254])
def test_fp32_heads_of_any_even_size_match_oracle(dim):
    """fp32 heads whose size is no multiple of the page's tiles of 32 dimensions (padded there): rounds against the oracle over
    a page edge, and every cached K and V entry, with the dead ones poisoned."""
    cfg = synth.EEConfig(n_layers=4, d_model=64, n_q_heads=4, n_kv_heads=2, head_dim=dim, d_ffn=96, vocab=300, exit_draft=1,
                         exit_inter=2, dtype="f32", sigma=0.1, gamma=(1.0, 0.3, 0.3))
    tol, k = TOL["f32"], 4
    O, model, sess, first, gfirst = _setup(cfg, 5, [61, 130], 3 * (k + 1) + 2)
    assert gfirst.tolist() == first.tolist()
    rng = np.random.default_rng(8)
    for do_full in (False, True, True):
        for b in range(2):
            sess.poison_dead_kv(b)
        _round(O, sess, k, 0.8, rng, do_full, tol)
    for b, s in enumerate(O.seqs):
        for l in range(cfg.n_layers):
            n = s.len[0 if l < 1 else (1 if l < 2 else 2)]
            gk, gv = sess.read_kv(b, l, 0, n)
            assert max_rel(gk, s.cache.K[l, :n]) <= tol and max_rel(gv, s.cache.V[l, :n]) <= tol, (b, l)
    sess.close(); model.close()


_ATTN_CASES = {
    # contexts that end at, before and behind page edges: one page, an odd and an even number of them
    "edges": (lambda: bf16_small(), [1, 63, 64, 65, 127, 128, 129, 193, 256], 8),
    # eleven and eight pages, 41 block rows of four query heads per KV head: more than one block of 128 query rows behind a context
    "rep4": (lambda: bf16_small(), [700, 449], 40),
    "rep8_d128": (lambda: bf16_d128(), [577, 130], 24),
    "rep1": (lambda: bf16_small(n_q_heads=4, n_kv_heads=4), [321, 64], 60),
}


def _compare_kv(O, sess, tol):
    for b, s in enumerate(O.seqs):
        for g in range(3):
            for l in O.cfg.group_layers(g):
                n = s.len[g]
                gk, gv = sess.read_kv(b, l, 0, n)
                assert max_rel(gk, s.cache.K[l, :n]) <= tol and max_rel(gv, s.cache.V[l, :n]) <= tol, (b, l)


@pytest.mark.parametrize("name", list(_ATTN_CASES))
@pytest.mark.parametrize("form", [0, 1, 2], ids=["split", "block", "tile"])
def test_forced_attention_matches_oracle(form, name):
    """Each attention kernel on every call of a context build and two rounds, against the oracle: hidden rows and logits of the
    last rows, decisions, and all cached K and V (which carry the attention of every row of the layers below)."""
    import paper_2510_01336_amd as hs
    make, ctx, k = _ATTN_CASES[name]
    cfg, tol = make(), TOL["bf16"]
    hs.ee_debug_attention_form(form)
    try:
        O, model, sess, first, gfirst = _setup(cfg, 31, ctx, 3 * (k + 1) + 2)
        assert hs.ee_debug_last_attention(sess.handle) == form
        assert gfirst.tolist() == first.tolist()
        assert max_rel(sess.last_logits()[-1:], O.o.last_logits) <= tol and max_rel(sess.last_hidden()[-1:], O.o.last_hidden) <= tol
        _compare_kv(O, sess, tol)
        rng = np.random.default_rng(4)
        for _ in range(2):
            for b in range(len(ctx)):
                sess.poison_dead_kv(b)
            _round(O, sess, k, 0.8, rng, True, tol)
            assert hs.ee_debug_last_attention(sess.handle) == form
        _compare_kv(O, sess, tol)
        sess.close(); model.close()
    finally:
        hs.ee_debug_attention_form(-1)


@pytest.mark.parametrize("batch,ctx,k,build,block", [
    (1, 60, 4, False, False), (1, 120, 4, True, False),          # one page: the ring; two: blocks
    (100, 600, 24, True, True), (100, 600, 32, True, False),     # 7 q-tiles: 2 rounds of the ring, 1 of blocks; 9: 2 and 2
    (60, 600, 32, True, False)])                                 # 9 q-tiles in one round either way
def test_blocks_are_chosen_where_they_need_fewer_rounds(batch, ctx, k, build, block):
    """The rule between the ring kernel and the block kernel for calls that fill the chip unsplit, in a context build and behind
    it, and the chosen form's results against the other one's."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small()
    model = hs.Model(cfg, 31)
    sess = hs.Session(model, batch, ctx + k + 8, k + 6)
    sess.enable_logits(True)
    sess.prefill([synth.gen_prompt(cfg.vocab, ctx, b) for b in range(batch)])
    assert (hs.ee_debug_last_attention(sess.handle) == 1) == build
    drafts = np.random.default_rng(k).integers(0, cfg.vocab, (batch, k)).astype(np.int32)
    got = []
    try:
        for form in (-1, 0 if block else 1):
            hs.ee_debug_attention_form(form)
            sess.draft_inject(drafts)
            sess.verify_intermediate()
            got.append((hs.ee_debug_last_attention(sess.handle), sess.last_logits()))
            for b in range(batch):
                sess.rollback(b, 0b111, ctx)
    finally:
        hs.ee_debug_attention_form(-1)
    assert (got[0][0] == 1) == block
    assert max_rel(got[0][1], got[1][1].astype(np.float64)) <= TOL["bf16"]
    sess.close(); model.close()


@pytest.mark.parametrize("form", [-1, 1], ids=["chosen", "block"])
@pytest.mark.parametrize("make", [bf16_small, bf16_d128], ids=["d64", "d128"])
def test_context_build_over_several_passes_matches_oracle(make, form):
    """A context build whose later passes start behind cached positions (512-row passes, which the smallest arena gives): a
    prompt cut by two pass ends and a short one that shares the last pass, against the oracle."""
    import re

    import paper_2510_01336_amd as hs
    cfg, tol, lens = make(), TOL["bf16"], [1100, 37]
    O = OracleSide(cfg, 31)
    prompts = []
    for b, n in enumerate(lens):
        for attempt in range(20):
            prompts.append(synth.gen_prompt(cfg.vocab, n, 100 + 1000 * attempt + b))
            if O.prefill_one(prompts[-1], n + 64)[1] > MARGIN:
                break
            O.drop_last(); prompts.pop()
    assert len(prompts) == 2
    model = hs.Model(cfg, 31)
    with pytest.raises(hs.EEError) as e:
        hs.Session(model, 2, 1200, 12, arena_bytes=1 << 12)
    least = int(re.search(r"< (\d+)", str(e.value)).group(1))
    hs.ee_debug_attention_form(form)
    try:
        sess = hs.Session(model, 2, 1200, 12, arena_bytes=least)
        assert sess.prefill(prompts).tolist() == [s.C[-1] for s in O.seqs]
        assert form < 0 or hs.ee_debug_last_attention(sess.handle) == form
        _compare_kv(O, sess, tol)
        sess.close(); model.close()
    finally:
        hs.ee_debug_attention_form(-1)


@pytest.mark.parametrize("heads,dim,k,ctx", [
    ((8, 2), 64, 8, [1, 63, 64, 65]), ((8, 2), 64, 16, [447, 448, 449, 0, 512, 513]), ((8, 1), 128, 1, [575, 576, 577]),
    ((8, 1), 128, 8, [832, 0, 130, 1]), ((8, 8), 64, 8, [700, 2500, 90, 2561, 2300, 0, 2496, 2559, 2560])],
    ids=["one_page", "eight_pages", "nine_pages_d128", "ragged_d128", "split"])
def test_few_rows_over_short_contexts_match_the_split_kernel(heads, dim, k, ctx):
    """The attention of few rows over short contexts (a wave per page, one launch) against the ring kernel with its KV splits
    and merge, on the same cache: contexts whose last position lies at, before and behind a page edge, fewer pages than waves
    and more, several q-tiles, an idle slot (context 0) and a batch long and wide enough that this form is split too.  The
    two sum a row's softmax in another order and agree to bf16 accuracy."""
    import paper_2510_01336_amd as hs
    cfg = bf16_small(n_q_heads=heads[0], n_kv_heads=heads[1], head_dim=dim)
    B, rows = len(ctx), k + 1
    model = hs.Model(cfg, 91)
    rng = np.random.default_rng(3)
    drafts = rng.integers(0, cfg.vocab, (B, k)).astype(np.int32)
    # ctx counts the positions behind the block: prompt, first token, drafts
    prompts = [synth.gen_prompt(cfg.vocab, max(1, n - rows if n > rows else n), 40 + b) for b, n in enumerate(ctx)]
    got = {}
    try:
        for form in (0, 4):                                     # 0: the form the call itself chooses
            hs.ee_debug_attention_split_pages(4)
            sess = hs.Session(model, B, max(ctx) + 4 * rows, B * (rows + 2))
            sess.enable_logits(True)
            for b, p in enumerate(prompts):
                if ctx[b]:
                    sess.prefill_seq(b, p)
            sess.draft_inject(drafts)
            hs.ee_debug_attention_split_pages(form)
            a, _ = sess.verify_intermediate()
            assert ((a >= 0) == (np.array(ctx) > 0)).all()
            got[form] = sess.last_logits().astype(np.float64)
            assert got[form].shape[0] == rows * sum(n > 0 for n in ctx)
            sess.close()
    finally:
        hs.ee_debug_attention_split_pages(0)
    assert np.isfinite(got[0]).all() and max_rel(got[0], got[4]) <= TOL["bf16"]
    assert not np.array_equal(got[0], got[4])                   # (the forms differ, or the choice never left the ring kernel)
    model.close()
