"""CPU-side checks of the library: it loads, exports every symbol the headers
declare, its schedule generator agrees with the oracle's, and the slot allocator /
validator return the documented error codes (dry-run stages: no kernel runs)."""
import os
import re

import pytest

from oracle import stage_oracle as O
from paper_2007_01045_amd import binding as B

ROOT = os.path.dirname(os.path.dirname(os.path.abspath(__file__)))


def _declared(header):
    txt = open(os.path.join(ROOT, "include", header)).read()
    txt = re.sub(r"/\*.*?\*/", "", txt, flags=re.S)
    return set(re.findall(r"\b((?:stage|dapple|pipeline)_[a-z0-9_]+)\s*\(", txt))


def test_library_exports_every_declared_symbol():
    lib = B.load()
    names = _declared("dapple_stage.h") | _declared("dapple_kernels.h") | _declared("dapple_pipeline.h")
    assert len(names) >= 20
    for n in names:
        assert hasattr(lib, n), n
    assert names == set(B.SYMBOLS), names ^ set(B.SYMBOLS)


@pytest.mark.parametrize("order", [O.GPIPE, O.EARLY_BACKWARD])
def test_schedule_matches_oracle(order):
    for M in range(1, 12):
        for K in range(1, 12):
            assert B.stage_schedule_ops(M, K, order) == O.schedule_ops(M, K, order)


def test_schedule_bad_arguments():
    for args in [(0, 1, 1), (3, 0, 1), (3, 2, 5)]:
        with pytest.raises(B.StageError) as e:
            B.stage_schedule_ops(*args)
        assert e.value.code == B.STAGE_E_BAD_ORDER


def dry(max_slots=2, **kw):
    base = dict(n_layers=2, hidden=64, n_heads=4, ffn=256, seq=16, micro_batch=2, max_slots=max_slots,
                dtype=B.DTYPE_F32, flags=B.FLAG_DRY_RUN)
    base.update(kw)
    return B.make_config(**base)


def test_config_errors():
    for kw in [dict(n_heads=5), dict(hidden=0), dict(max_slots=0), dict(dtype=7), dict(hidden=66, n_heads=6),
               dict(ln_eps=-1.0), dict(hidden=8192, n_heads=8)]:
        with pytest.raises(B.StageError) as e:
            B.stage_query_sizes(dry(**kw))
        assert e.value.code == B.STAGE_E_CONFIG, kw
    # not a dry run and no device memory given
    cfg = dry(); cfg.flags = 0
    with pytest.raises(B.StageError) as e:
        B.stage_init(cfg, None, None, 0)
    assert e.value.code == B.STAGE_E_NULL
    with pytest.raises(B.StageError) as e:          # arena too small (pointer never dereferenced)
        B.stage_init(cfg, 4096, 4096, 1024)
    assert e.value.code == B.STAGE_E_ARENA_SMALL


def test_recompute_keeps_only_the_boundary_per_slot():
    # section VI-E: with re-computation a resident micro-batch keeps its input only; the activation
    # buffers (one for the forward tasks, one per backward lane) do not scale with the slots
    full = B.stage_query_sizes(dry(2))
    rc2 = B.stage_query_sizes(dry(2, flags=B.FLAG_DRY_RUN | B.FLAG_RECOMPUTE))
    rc8 = B.stage_query_sizes(dry(8, flags=B.FLAG_DRY_RUN | B.FLAG_RECOMPUTE))
    T, H = 2 * 16, 64
    assert rc2.slot_bytes == T * H * 4 < full.slot_bytes
    assert rc8.arena_bytes - rc2.arena_bytes == 6 * rc2.slot_bytes
    assert rc2.workspace_bytes >= full.workspace_bytes + full.slot_bytes          # a backward lane's buffer
    grads_and_slots = lambda q, k: q.grad_bytes + k * q.slot_bytes
    assert rc2.arena_bytes - grads_and_slots(rc2, 2) >= 2 * rc2.workspace_bytes + full.slot_bytes   # + the forward tasks' buffer
    one = B.stage_query_sizes(dry(2, flags=B.FLAG_DRY_RUN | B.FLAG_RECOMPUTE | B.FLAG_ONE_STREAM))
    assert one.arena_bytes - grads_and_slots(one, 2) < rc2.arena_bytes - grads_and_slots(rc2, 2) - full.slot_bytes
    # first stage: token ids; last stage: input and targets
    emb = B.stage_query_sizes(dry(2, flags=B.FLAG_DRY_RUN | B.FLAG_RECOMPUTE, has_embedding=1, vocab=100, max_pos=16))
    assert emb.slot_bytes == 256          # T int32 ids, rounded up to the 256-byte granule
    head = B.stage_query_sizes(dry(2, flags=B.FLAG_DRY_RUN | B.FLAG_RECOMPUTE, has_mlm_head=1, vocab=100))
    assert head.slot_bytes == T * H * 4 + 256


def test_sizes_scale_with_slots_only():
    a, b = B.stage_query_sizes(dry(2)), B.stage_query_sizes(dry(4))
    assert a.slot_bytes == b.slot_bytes and a.grad_bytes == b.grad_bytes
    assert b.arena_bytes - a.arena_bytes == 2 * a.slot_bytes
    H, F = 64, 256
    assert a.n_params == 2 * (4 * (H * H + H) + 2 * H * F + F + H + 4 * H)


def _workspaces(cfg):
    """The arena's workspace in units of one micro-batch's."""
    q = B.stage_query_sizes(cfg)
    return (q.arena_bytes - q.grad_bytes - cfg.max_slots * q.slot_bytes) / q.workspace_bytes


@pytest.mark.parametrize("vocab,group", [(30522, 4), (131008, 4), (131072, 3), (200000, 2), (400000, 1)])
def test_a_group_of_micro_batches_stays_addressable(vocab, group):
    """The gradient of the logits of a group, 2048 rows a micro-batch: from 2 GiB on the matrix-core products no longer
    address it, so the group must end below that."""
    cfg = dry(4, n_layers=1, hidden=1024, n_heads=16, ffn=4096, seq=512, micro_batch=4, dtype=B.DTYPE_BF16,
              has_mlm_head=1, vocab=vocab)
    assert group == 1 or group * 2048 * vocab * 2 < 2 ** 31
    assert group - 1 < _workspaces(cfg) <= group + 0.001
    launches = []
    for M in (4, 1):
        h = B.stage_init(cfg, None, None, 0)
        try:
            B.stage_reset_stats(h)
            B.stage_run_schedule(h, M, M, B.ORDER_GPIPE)
            launches.append(B.stage_stats(h).kernel_launches)
        finally:
            B.stage_destroy(h)
    assert launches[0] == launches[1] * -(-4 // group)


@pytest.mark.parametrize("slots,group", [(1, 1), (2, 2), (4, 4), (7, 7), (8, 8), (12, 8)])
def test_no_workspace_beyond_the_slots(slots, group):
    # 1024 tokens a micro-batch: eight of them make the 8192 rows a group may have
    assert _workspaces(dry(slots, n_layers=12, hidden=1024, n_heads=16, ffn=4096, seq=512, dtype=B.DTYPE_BF16)) <= group + 0.001


@pytest.mark.parametrize("kw,sets", [
    (dict(flags=B.FLAG_DRY_RUN | B.FLAG_ONE_STREAM), 1),
    (dict(micro_batch=16), 1),                 # 8192 tokens: every product fills the chip by itself
    (dict(micro_batch=2), 6),                  # a side stream takes the weight gradients: a set for each of the six layers
])
def test_one_set_of_gradient_buffers_where_one_stream_runs_a_task(kw, sets):
    """What the weight gradients read (six widths and one ffn width of a micro-batch's rows, and partial sums) is kept per
    layer only where a side stream reads it behind the task's back."""
    base = dict(n_layers=6, hidden=1024, n_heads=16, ffn=4096, seq=512, dtype=B.DTYPE_BF16, micro_batch=2)
    q6, q1 = B.stage_query_sizes(dry(1, **{**base, **kw})), B.stage_query_sizes(dry(1, **{**base, **kw, "n_layers": 1}))
    T = 512 * {**base, **kw}["micro_batch"]
    one = T * (5 * 1024 + 4096) * 2 + 2 * (T // 8) * 3 * 1024 * 4
    assert q6.workspace_bytes - q1.workspace_bytes == (sets - 1) * one


def test_slot_allocator_error_paths():
    h = B.stage_init(dry(2), None, None, 0)
    try:
        B.stage_fwd(h, 0, None, None)
        with pytest.raises(B.StageError) as e:
            B.stage_fwd(h, 0, None, None)
        assert e.value.code == B.STAGE_E_DUP_MB
        B.stage_fwd(h, 1, None, None)
        with pytest.raises(B.StageError) as e:      # K+1-th forward without a backward
            B.stage_fwd(h, 2, None, None)
        assert e.value.code == B.STAGE_E_NO_SLOT
        with pytest.raises(B.StageError) as e:
            B.stage_bwd(h, 5, None, None)
        assert e.value.code == B.STAGE_E_NOT_RESIDENT
        st = B.stage_stats(h)
        assert st.live_slots == 2 and st.peak_live_slots == 2 and st.fwd_tasks == 2
        B.stage_bwd(h, 0, None, None)
        B.stage_fwd(h, 2, None, None)               # reuses the slot B_0 released
        with pytest.raises(B.StageError) as e:
            B.stage_bwd(h, 0, None, None)
        assert e.value.code == B.STAGE_E_NOT_RESIDENT
        B.stage_bwd(h, 1, None, None)
        B.stage_bwd(h, 2, None, None)
        st = B.stage_stats(h)
        assert st.live_slots == 0 and st.peak_live_slots == 2 and st.bwd_tasks == 3
        assert st.peak_activation_bytes == 2 * st.slot_bytes
    finally:
        B.stage_destroy(h)


@pytest.mark.parametrize("M,K", [(1, 1), (4, 2), (8, 4), (16, 4), (5, 7)])
def test_peak_is_K_for_early_backward_and_M_for_gpipe(M, K):
    slots = max(M, K)
    h = B.stage_init(dry(slots), None, None, 0)
    try:
        B.stage_run_schedule(h, M, K, B.ORDER_EARLY_BACKWARD)
        st = B.stage_stats(h)
        assert st.peak_live_slots == min(K, M) and st.live_slots == 0
        assert st.fwd_tasks == M and st.bwd_tasks == M
        B.stage_reset_stats(h)
        B.stage_run_schedule(h, M, K, B.ORDER_GPIPE)
        assert B.stage_stats(h).peak_live_slots == M
    finally:
        B.stage_destroy(h)


@pytest.mark.parametrize("M,K,order,groups", [
    (10, 5, "early", 4), (14, 7, "early", 4), (9, 3, "early", 3), (8, 4, "early", 2), (11, 5, "early", 5),
    (4, 5, "early", 1), (9, 9, "gpipe", 3), (7, 1, "early", 7),
])
def test_resident_counts_that_a_group_does_not_divide(M, K, order, groups):
    """2048 tokens a micro-batch, four of them to a group: any resident count is served by full groups and a smaller
    one, K micro-batches resident at most and every one forward and backward once."""
    cfg = dry(max(M, K), n_layers=1, hidden=1024, n_heads=16, ffn=4096, seq=512, micro_batch=4, dtype=B.DTYPE_BF16)
    h = B.stage_init(cfg, None, None, 0)
    try:
        B.stage_reset_stats(h)
        B.stage_run_schedule(h, 1, 1, B.ORDER_EARLY_BACKWARD)
        one = B.stage_stats(h).kernel_launches
        B.stage_reset_stats(h)
        B.stage_run_schedule(h, M, K, B.ORDER_GPIPE if order == "gpipe" else B.ORDER_EARLY_BACKWARD)
        st = B.stage_stats(h)
        assert st.kernel_launches == groups * one
        assert st.peak_live_slots == (M if order == "gpipe" else min(K, M))
        assert st.fwd_tasks == M and st.bwd_tasks == M and st.live_slots == 0
    finally:
        B.stage_destroy(h)


def _launches_with_buffers(M, K, xs, dys, ys, dxs, order=B.ORDER_EARLY_BACKWARD):
    """Launches of an iteration whose buffers lie at the given places of one address range (a dry run: no buffer is
    touched), 2048 x 1024 bf16 a micro-batch, four micro-batches to a group."""
    cfg = dry(max(M, K), n_layers=1, hidden=1024, n_heads=16, ffn=4096, seq=512, micro_batch=4, dtype=B.DTYPE_BF16)
    at = lambda places: [(1 << 40) + int(p * 2048 * 1024 * 2) for p in places]
    h = B.stage_init(cfg, None, None, 0)
    try:
        B.stage_reset_stats(h)
        B.stage_run_schedule(h, M, K, order, at(xs), at(dys), at(ys), at(dxs))
        return B.stage_stats(h).kernel_launches
    finally:
        B.stage_destroy(h)


def test_overlapping_buffers_are_not_grouped_across_a_dependence():
    M, K = 8, 4
    n = lambda first: list(range(first, first + M))
    base = dict(xs=n(0), dys=n(10), ys=n(20), dxs=n(30))
    one = _launches_with_buffers(1, 1, [0], [10], [20], [30])
    run = lambda **kw: _launches_with_buffers(M, K, **{**base, **kw}) // one
    assert run() == 2                                        # two groups of four
    # the output of a forward is the input of the next one; of a backward, of the next one; partly
    assert run(ys=n(1)) == M and run(dxs=n(11)) == M and run(ys=[v + 0.75 for v in n(0)]) == M
    # what groups cannot show: in place, all outputs in one buffer, all inputs in one buffer, the output as its own
    # gradient, a ring of K outputs, an output that replaces an input read before it
    assert run(ys=n(0)) == 2 and run(dxs=n(10)) == 2 and run(ys=[20] * M, dxs=[30] * M) == 2 and run(xs=[0] * M) == 2
    assert run(ys=n(10)) == 2 and run(ys=[10 + m % K for m in range(M)], dys=[10 + m % K for m in range(M)]) == 2
    assert run(ys=[v - 1 for v in n(0)]) == 2
    # F_5 is listed before B_2 and overwrites what that one reads: grouped, it would come after
    assert run(ys=n(20)[:4] + [11] + n(20)[5:]) == M
    # the GPipe order has no such pair, but the chain of forwards
    gp = lambda **kw: _launches_with_buffers(M, K, **{**base, **kw}, order=B.ORDER_GPIPE) // one
    assert gp() == 2 and gp(ys=n(1)) == M and gp(ys=n(20)[:4] + [11] + n(20)[5:]) == 2


def test_run_schedule_rejects_bad_orders_before_running_anything():
    h = B.stage_init(dry(2), None, None, 0)
    try:
        bad = [
            (4, 2, B.ORDER_GPIPE, None),                                   # needs 4 slots, stage has 2
            (4, 3, B.ORDER_EARLY_BACKWARD, None),                          # K > max_slots
            (2, 2, B.ORDER_EXPLICIT, [("B", 0), ("F", 0), ("F", 1), ("B", 1)]),   # B before F
            (2, 2, B.ORDER_EXPLICIT, [("F", 0), ("F", 0), ("B", 0), ("B", 0)]),   # twice
            (3, 2, B.ORDER_EXPLICIT, [("F", 0), ("F", 1), ("F", 2), ("B", 0), ("B", 1), ("B", 2)]),  # 3 resident
            (2, 2, B.ORDER_EXPLICIT, [("F", 0), ("B", 0)]),                # incomplete
            (0, 1, B.ORDER_GPIPE, None),
        ]
        for M, K, order, ops in bad:
            with pytest.raises(B.StageError) as e:
                B.stage_run_schedule(h, M, K, order, explicit_ops=ops)
            assert e.value.code == B.STAGE_E_BAD_ORDER, (M, K, order, ops)
            assert B.stage_stats(h).fwd_tasks == 0
        # a steady phase that ran the forward first would need K+1 slots
        fb = [("F", 0), ("F", 1), ("F", 2), ("B", 0), ("B", 1), ("F", 3), ("B", 2), ("B", 3)]
        with pytest.raises(B.StageError):
            B.stage_run_schedule(h, 4, 2, B.ORDER_EXPLICIT, explicit_ops=fb)
        # descending backwards are a valid explicit order
        ok = [("F", 0), ("F", 1), ("B", 1), ("B", 0)]
        B.stage_run_schedule(h, 2, 2, B.ORDER_EXPLICIT, explicit_ops=ok)
        assert B.stage_stats(h).bwd_tasks == 2
        # leftovers from single calls block a schedule run
        B.stage_fwd(h, 9, None, None)
        with pytest.raises(B.StageError) as e:
            B.stage_run_schedule(h, 2, 2, B.ORDER_GPIPE)
        assert e.value.code == B.STAGE_E_BAD_ORDER
    finally:
        B.stage_destroy(h)


def test_null_handle_and_error_text():
    with pytest.raises(B.StageError) as e:
        B.stage_fwd(None, 0, None, None)
    assert e.value.code == B.STAGE_E_NULL and "NULL" in str(e.value)


def test_pipeline_host_functions_follow_the_oracle():
    import random
    from oracle import pipeline_oracle as PO
    rng = random.Random(7)
    for _ in range(300):
        S, M = rng.randint(1, 6), rng.randint(1, 12)
        F = [rng.uniform(0.2, 3.0) for _ in range(S)]
        Bt = [rng.uniform(0.2, 6.0) for _ in range(S)]
        if rng.random() < 0.3:
            F[0] *= 4; Bt[0] *= 4
        assert B.pipeline_pivot_stage(M, F, Bt) == PO.pivot_stage(F, Bt, M)
        assert B.pipeline_latency_model(M, F, Bt) == pytest.approx(PO.latency_model(F, Bt, M), rel=1e-13)
        Q = rng.randrange(S)
        assert B.pipeline_latency_model(M, F, Bt, Q) == pytest.approx(PO.latency_model(F, Bt, M, Q), rel=1e-13)
        for pol, name in ((B.POLICY_A, "A"), (B.POLICY_B, "B")):
            D = rng.choice([0, 1, 2, 5, 100])
            assert B.pipeline_warmup_depths(S, M, pol, D) == PO.warmup_depths(S, M, name, None if D == 0 else D)
    with pytest.raises(B.StageError):
        B.pipeline_latency_model(3, [1.0, 1.0], [1.0, 1.0], Q=2)
    assert B.pipeline_boundary_bytes(3, 4, 1000) == 2 * 2 * 4 * 1024


def plan(*a, **kw):
    """The launch dapple_gemm would make (host only: the pointers are never read)."""
    return B.dapple_gemm_plan(B.DTYPE_BF16, gemm_desc(*a, **kw))


def gemm_desc(M, N, Ks, nseg=1, akS=False, bkS=False, epi=0, tile=0):
    d = B.dapple_gemm_desc()
    d.A = d.B = d.C = d.aux = d.bsum = 1 << 20
    d.M, d.N, d.K, d.kseg_len, d.segA, d.segB = M, N, Ks * nseg, Ks, 8 * M * Ks, 8 * N * Ks
    d.lda, d.ldb, d.ldc, d.ldaux = (M if akS else Ks), (N if bkS else Ks), N, N
    d.a_kstrided, d.b_kstrided, d.epi, d.tile = int(akS), int(bkS), epi, tile
    return d


@pytest.mark.parametrize("akS,bkS", [(False, False), (False, True), (True, False), (True, True)])
def test_segments_of_a_product_share_the_turns_of_a_ring(akS, bkS):
    # tiles of which a unit holds one workgroup: less than one turn of k-tiles of zeros in all, whatever a segment's length
    for tile, ring in ((1, 4), (2, 3), (6, 5)) + (() if akS else ((12, 4),)):
        for Ks in range(64, 64 * 19, 64):
            for nseg in (1, 2, 3, 4):
                rows, cols, depth, tiles = plan(600, 320, Ks, nseg, akS, bkS, B.EPI_ADD, tile)
                assert tiles == -(-nseg * Ks // depth // ring) * ring, (tile, Ks, nseg, rows, cols, depth, tiles)
    # the others: whole turns per segment
    for tile, ring in ((3, 2), (4, 3), (7, 4)):
        for Ks in range(64, 64 * 19, 64):
            for nseg in (1, 2, 3, 4):
                tiles = plan(600, 320, Ks, nseg, akS, bkS, B.EPI_ADD, tile)[3]
                assert tiles == nseg * -(-Ks // 64 // ring) * ring, (tile, Ks, nseg, tiles)


def test_the_gradient_of_the_attention_input_runs_no_more_than_a_turn_of_zeros():
    for H in range(640, 1088, 64):   # 256x128 tiles in a ring of three
        rows, cols, depth, tiles = plan(8192, H, H, 3, epi=B.EPI_ADD)
        if (rows, cols, depth) == (256, 128, 64):
            assert tiles == -(-3 * H // 64 // 3) * 3, (H, tiles)
    assert plan(8192, 1024, 1024, 3, epi=B.EPI_ADD) == (256, 128, 64, 48)
    assert plan(4096, 1024, 1024, 3, epi=B.EPI_ADD) == (128, 128, 64, 50)


def test_every_layout_has_the_tile_that_is_chosen_for_it():
    # A k-strided, B k-contiguous: where 128x128 tiles reach three quarters of the units and fit them, they are taken
    for M, N in ((2048, 1536), (2048, 1920), (1792, 1792), (2048, 2048)):
        for K in (256, 512, 1024, 1536, 2048):
            assert plan(M, N, K, akS=True)[:3] == (128, 128, 64), (M, N, K)
    # any product and any named tile has a launch (one that is not in the list: the 64x64 tile)
    for akS, bkS in ((False, False), (False, True), (True, False), (True, True)):
        for tile in range(-1, 15):
            for M, N in ((64, 64), (600, 320), (1024, 1024), (2048, 1536), (8192, 1024), (8192, 4096)):
                for K in (200, 512, 2048):
                    assert plan(M, N, K, akS=akS, bkS=bkS, tile=tile) is not None
        for tile in (11, 13, 14):
            assert plan(600, 320, 320, akS=akS, bkS=bkS, tile=tile)[:3] == (64, 64, 64)
    for epi in (B.EPI_ACC32, B.EPI_ACC32 | B.EPI_BSUM):
        for tile in range(-1, 15):
            assert plan(600, 320, 320, akS=True, bkS=True, epi=epi, tile=tile) is not None


def test_the_plan_of_a_product_is_the_named_tile():
    for tile, shape in {1: (256, 256, 32), 2: (256, 128, 64), 3: (128, 128, 64), 4: (128, 64, 64), 6: (128, 128, 64),
                        7: (64, 64, 64), 8: (128, 128, 32), 9: (32, 64, 64), 10: (32, 32, 64), 12: (128, 64, 64)}.items():
        assert plan(600, 320, 320, tile=tile)[:3] == shape
    d = B.dapple_gemm_desc()
    with pytest.raises(B.StageError):
        B.dapple_gemm_plan(B.DTYPE_BF16, d)
    assert plan(600, 322, 320) is None   # a row of C that is no multiple of 4: the plain kernel


def test_128x64_tiles_take_four_stages_where_a_unit_has_one():
    # 65 k-tiles are 66 in a ring of three and 68 in one of four
    K = 64 * 65
    for M, N, want in ((2048, 1024, 68), (1296, 1024, 68), (2048 + 8, 1024, 66), (2560, 1024, 66)):
        for bkS in (False, True):
            assert plan(M, N, K, bkS=bkS, epi=B.EPI_ADD) == (128, 64, 64, want), (M, N, bkS)
    assert plan(2048, 1024, K, akS=True)[:3] == (128, 64, 64)
    assert plan(600, 320, K, tile=12) == (128, 64, 64, 68)


def launch(M, N, K, units=0, shared=False, **kw):
    """Rows and columns of the tile, waves and stages of the launch a stage would make."""
    p = B.dapple_gemm_plan_beside(B.DTYPE_BF16, gemm_desc(M, N, K, **kw), units, shared)
    return p[:2] + p[4:]


def test_lines_of_the_128x64_tile_and_the_units_they_move_with():
    # a data gradient and a forward product; U units, a width of 1024 on all of them
    for bkS in (False, True):
        for U, N, kw in ((256, 1024, {}), (256, 1024, {"units": 256}), (128, 512, {"units": 128}), (64, 512, {"units": 64})):
            per = N // 64                          # tiles in a row of them
            rows = lambda tiles, h: tiles // per * h   # the most rows that make so many tiles of height h
            for K in (2048, 4096):
                for shared in (False, True):
                    kw2 = dict(kw, bkS=bkS, shared=shared)
                    assert launch(rows(U, 64), N, K, **kw2) == (64, 64, 4, 4)
                    # from one tile of 64x64 more than units on: 128x64, in eight waves
                    assert launch(rows(U, 64) + 8, N, K, **kw2)[:3] == (128, 64, 8)
                    assert launch(rows(U, 64) + 8, N, K, **kw2)[3] == (3 if shared else 4)
                    # four stages where a unit has at most one tile and no other stream's products run beside it
                    assert launch(rows(U, 128) - 8, N, K, **kw2) == (128, 64, 8, 3 if shared else 4)
                    assert launch(rows(U, 128) + 8, N, K, **kw2) == (128, 64, 8, 3)
                    # up to three quarters of the units in 128x128 tiles
                    t = 3 * U // 4 // (N // 128)
                    assert launch(128 * (t - 1), N, K, **kw2) == (128, 64, 8, 3)
                    assert launch(128 * t, N, K, **kw2)[:2] == (128, 128)
            assert launch(rows(U, 64) + 8, N, 2048 - 64, bkS=bkS, **kw) == (64, 64, 4, 4)   # short sums
    assert launch(1536, 1024, 4096, akS=True) == (128, 64, 4, 3)


def test_k_segments_that_are_no_multiple_of_64_run_in_eight_waves():
    for bkS in (False, True):
        for shared in (False, True):
            for M, N, K in ((64, 64, 200), (600, 768, 3000), (1536, 1024, 2040), (2560, 1024, 4008)):
                assert launch(M, N, K, shared=shared, bkS=bkS) == (128, 64, 8, 3)
                for tile in (4, 7, 12):
                    assert launch(M, N, K, shared=shared, bkS=bkS, tile=tile) == (128, 64, 8, 3)
            assert launch(3072, 1024, 4008, shared=shared, bkS=bkS) == (128, 128, 8, 2)


def test_the_plan_beside_another_stream_checks_its_arguments():
    d = gemm_desc(600, 320, 320)
    for units, code in ((-1, B.STAGE_E_CONFIG),):
        with pytest.raises(B.StageError) as e:
            B.dapple_gemm_plan_beside(B.DTYPE_BF16, d, units)
        assert e.value.code == code
    assert B.dapple_gemm_plan_beside(B.DTYPE_BF16, d)[:4] == B.dapple_gemm_plan(B.DTYPE_BF16, d)
    assert B.dapple_gemm_plan_beside(B.DTYPE_F32, d) is None
