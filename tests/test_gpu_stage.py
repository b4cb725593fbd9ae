"""GPU parity of the whole stage against the oracle, through the C ABI: every
y_m, dx_m and every parameter-gradient tensor, both schedule orders, bit-identity
across orders, and peak activation memory bounded by K."""
import numpy as np
import pytest

from oracle import stage_oracle as O
from paper_2007_01045_amd import binding as B
from paper_2007_01045_amd import inputs as I
from tests.stage_util import c_config, compare, make_inputs, run_gpu, run_oracle, to_np

pytestmark = pytest.mark.gpu
torch = pytest.importorskip("torch")

# spec tolerances: relative L2 per tensor
TOL_F32, TOL_BF16 = 1e-4, 2e-2
SEED = I.DEFAULT_SEED


def check_config(cfg, M, K, tol, loss_scale=1.0):
    theta, mbs = make_inputs(cfg, SEED, M)
    st, ref = run_oracle(cfg, theta, mbs, M, K, loss_scale=loss_scale)
    eb = run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD, loss_scale=loss_scale)
    gp = run_gpu(cfg, theta, mbs, M, K, B.ORDER_GPIPE, loss_scale=loss_scale)
    rep = {}
    worst = compare(cfg, st, ref, eb, tol, M, mbs, rep)
    compare(cfg, st, ref, gp, tol, M, mbs)
    print(f"[{cfg.name or 'stage'} M={M} K={K}] worst rel-L2 {worst[1]:.3e} ({worst[0]}), worst element "
          f"{rep['worst_elem'][1]:.3e} rms ({rep['worst_elem'][0]}), worst table rows {rep['rows']}", flush=True)
    # the two orders run the same kernels on the same data and add the micro-batch
    # gradients in the same sequence: results must agree bit for bit
    assert np.array_equal(eb["grads"], gp["grads"])
    for m in range(M):
        assert np.array_equal(eb["ys"][m], gp["ys"][m])
        if eb["dxs"] is not None:
            assert np.array_equal(eb["dxs"][m], gp["dxs"][m])
    # peak activation memory: K slots against M slots
    assert eb["stats"]["peak_live"] == min(K, M) and gp["stats"]["peak_live"] == M
    assert eb["stats"]["peak_bytes"] == min(K, M) * eb["stats"]["slot_bytes"]
    assert gp["stats"]["peak_bytes"] == M * gp["stats"]["slot_bytes"]
    assert ref["peak_live"] == min(K, M)
    return worst


def test_tiny_fp32_config():
    cfg = I.CONFIGS["tiny"]
    worst = check_config(cfg, cfg.M, cfg.K, TOL_F32)
    print("tiny fp32 worst:", worst)


def test_fp32_ragged_shapes():
    # sizes that are not multiples of the kernels' tiles, several blocks
    cfg = I.StageConfig(2, 72, 6, 100, 19, 3, 3, 2, "f32", ln_eps=1e-5)
    check_config(cfg, 3, 2, TOL_F32)


def test_bf16_mfma_path_small():
    # d = 64, s multiple of 64: MFMA GEMMs and MFMA attention; T = 384 gives ragged tiles
    cfg = I.StageConfig(2, 256, 4, 512, 192, 2, 5, 2, "bf16")
    worst = check_config(cfg, 5, 2, TOL_BF16)
    print("bf16 small worst:", worst)


def test_bf16_plain_fallback_shapes():
    # head dim 32 and a sequence that is no multiple of a block
    cfg = I.StageConfig(1, 64, 2, 128, 24, 2, 2, 1, "bf16")
    check_config(cfg, 2, 1, TOL_BF16)


def test_K_equal_one_and_K_above_M():
    cfg = I.CONFIGS["tiny"]
    theta, mbs = make_inputs(cfg, SEED, 3)
    st, ref = run_oracle(cfg, theta, mbs, 3, 1)
    a = run_gpu(cfg, theta, mbs, 3, 1, B.ORDER_EARLY_BACKWARD)
    b = run_gpu(cfg, theta, mbs, 3, 7, B.ORDER_EARLY_BACKWARD, max_slots=7)
    compare(cfg, st, ref, a, TOL_F32, 3)
    assert a["stats"]["peak_live"] == 1 and b["stats"]["peak_live"] == 3
    assert np.array_equal(a["grads"], b["grads"])


def test_explicit_order_descending_backwards_within_tolerance():
    cfg = I.CONFIGS["tiny"]
    theta, mbs = make_inputs(cfg, SEED, 4)
    st, ref = run_oracle(cfg, theta, mbs, 4, 4)
    ops = [("F", m) for m in range(4)] + [("B", m) for m in reversed(range(4))]
    g = run_gpu(cfg, theta, mbs, 4, 4, B.ORDER_EXPLICIT, max_slots=4, explicit_ops=ops)
    compare(cfg, st, ref, g, TOL_F32, 4)


def test_repeat_runs_are_bit_identical_and_zero_grads_works():
    cfg = I.StageConfig(2, 256, 4, 512, 128, 2, 3, 2, "bf16")
    theta, mbs = make_inputs(cfg, SEED, 3)
    a = run_gpu(cfg, theta, mbs, 3, 2, B.ORDER_EARLY_BACKWARD)
    b = run_gpu(cfg, theta, mbs, 3, 2, B.ORDER_EARLY_BACKWARD)
    assert np.array_equal(a["grads"], b["grads"])
    # two iterations without zeroing accumulate; with zeroing they do not
    r = B.StageRunner(__import__("tests.stage_util", fromlist=["c_config"]).c_config(cfg, 2), theta)
    try:
        T, H = cfg.tokens, cfg.hidden
        xs = [r.to_dev(mb["x"].reshape(T, H)) for mb in mbs]
        dys = [r.to_dev(mb["dy"].reshape(T, H)) for mb in mbs]
        r.run(3, 2, B.ORDER_EARLY_BACKWARD, xs, dys)
        r.run(3, 2, B.ORDER_EARLY_BACKWARD, xs, dys)
        torch.cuda.synchronize()
        twice = r.grads.cpu().numpy().astype(np.float64)
        assert np.linalg.norm(twice - 2 * a["grads"]) <= 1e-5 * np.linalg.norm(twice)
        B.stage_zero_grads(r.h)
        r.run(3, 2, B.ORDER_EARLY_BACKWARD, xs, dys)
        torch.cuda.synchronize()
        assert np.array_equal(r.grads.cpu().numpy(), a["grads"])
    finally:
        r.close()


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_first_stage_with_embeddings_small(dtype):
    # repeated ids inside a micro-batch (vocab smaller than b*s) exercise the ordered scatter-add
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    cfg = I.StageConfig(2, 256, 4, 512, 128, 2, 3, 2, dtype, has_embedding=True, vocab=97, max_pos=128, ln_eps=1e-5)
    worst = check_config(cfg, 3, 2, tol)
    print("embedding stage worst:", dtype, worst)
    cfg = I.StageConfig(1, 64, 4, 128, 24, 3, 2, 1, dtype, has_embedding=True, vocab=1000, max_pos=32, ln_eps=1e-5)
    check_config(cfg, 2, 1, tol)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_last_stage_with_mlm_head_small(dtype):
    tol = TOL_F32 if dtype == "f32" else TOL_BF16
    # vocab not a multiple of 4 or 64: padded columns, ragged tiles
    cfg = I.StageConfig(2, 256, 4, 512, 128, 2, 3, 2, dtype, has_mlm_head=True, vocab=1022, ln_eps=1e-5)
    worst = check_config(cfg, 3, 2, tol, loss_scale=1.0 / 117)
    print("head stage worst:", dtype, worst)
    cfg = I.StageConfig(1, 64, 4, 128, 24, 3, 2, 1, dtype, has_mlm_head=True, vocab=50, ln_eps=1e-5)
    check_config(cfg, 2, 1, tol, loss_scale=0.5)


def test_first_stage_full_shapes_reduced_M():
    """Layer and vocabulary shapes of the first-stage configuration (12 layers, H 1024, seq 512,
    micro-batch 2, vocab 30522), with M = 3, K = 2 so that the oracle stays within a minute."""
    cfg = I.CONFIGS["first_stage"]
    worst = check_config(cfg, 3, 2, TOL_BF16)
    print("first_stage worst:", worst)


def test_last_stage_full_shapes_reduced_M():
    cfg = I.CONFIGS["last_stage"]
    worst = check_config(cfg, 3, 2, TOL_BF16, loss_scale=1.0 / (3 * 154))
    print("last_stage worst:", worst)


def test_bert48_quarter_full_shapes_reduced_M():
    cfg = I.CONFIGS["bert48_quarter"]
    worst = check_config(cfg, 5, 4, TOL_BF16)
    print("bert48_quarter worst:", worst)


def _full_config(name, loss_scale=1.0):
    """A named configuration at its stated M and K against the oracle, both orders, plus a run without lanes
    (one stream) that must give the same bits: the steady state of the schedule (M - K slot reuses, alternating
    backward lanes, the side lane's accumulation order) at full shapes."""
    cfg = I.CONFIGS[name]
    print(f"{name}: oracle for M={cfg.M}, K={cfg.K} ...", flush=True)
    worst = check_config(cfg, cfg.M, cfg.K, TOL_BF16, loss_scale=loss_scale)
    theta, mbs = make_inputs(cfg, SEED, cfg.M)
    eb = run_gpu(cfg, theta, mbs, cfg.M, cfg.K, B.ORDER_EARLY_BACKWARD, loss_scale=loss_scale)
    one = run_gpu(cfg, theta, mbs, cfg.M, cfg.K, B.ORDER_EARLY_BACKWARD, loss_scale=loss_scale, flags=B.FLAG_ONE_STREAM)
    assert np.array_equal(eb["grads"], one["grads"])
    for m in range(cfg.M):
        assert np.array_equal(eb["ys"][m], one["ys"][m])
        if eb["dxs"] is not None:
            assert np.array_equal(eb["dxs"][m], one["dxs"][m])
    assert one["stats"]["peak_live"] == cfg.K and one["stats"]["peak_bytes"] == cfg.K * one["stats"]["slot_bytes"]
    return worst


def test_bert48_quarter_at_stated_M_and_K():
    _full_config("bert48_quarter")


def test_first_stage_at_stated_M_and_K():
    _full_config("first_stage")


def test_last_stage_at_stated_M_and_K():
    cfg = I.CONFIGS["last_stage"]
    _full_config("last_stage", loss_scale=1.0 / (cfg.M * 154))


def test_bert_large_shaped_stage_full_size():
    """The benchmark's configuration at full size: 6 layers, H 1024, 16 heads, FFN 4096,
    seq 512, micro-batch 4, M 8, K 4 (the oracle needs about a minute of CPU)."""
    cfg = I.CONFIGS["bert_large"]
    worst = check_config(cfg, cfg.M, cfg.K, TOL_BF16)
    print("bert_large worst:", worst)


# ---- re-computation (section VI-E, Table VI "+ RC"): same numbers, a fraction of the memory
def _recompute_case(cfg, M, K, order):
    theta, mbs = make_inputs(cfg, SEED, M)
    a = run_gpu(cfg, theta, mbs, M, K, order)
    b = run_gpu(cfg, theta, mbs, M, K, order, flags=B.FLAG_RECOMPUTE)
    assert np.array_equal(a["grads"], b["grads"])          # the same kernels on the same values
    for m in range(M):
        assert np.array_equal(a["ys"][m], b["ys"][m])
        if a["dxs"] is not None:
            assert np.array_equal(a["dxs"][m], b["dxs"][m])
    return a["stats"], b["stats"]


def test_recompute_matches_stored_activations_bitwise_and_keeps_only_the_boundary():
    cfg = I.StageConfig(3, 256, 4, 512, 128, 2, 5, 2, "bf16")
    for order in (B.ORDER_EARLY_BACKWARD, B.ORDER_GPIPE):
        full, rc = _recompute_case(cfg, 5, 2, order)
        T, H = cfg.tokens, cfg.hidden
        assert rc["slot_bytes"] == T * H * 2                # the stage input, nothing else
        live = 2 if order == B.ORDER_EARLY_BACKWARD else 5
        assert rc["peak_live"] == full["peak_live"] == live
        # K boundary tensors + one activation buffer for the forward tasks and one per backward lane,
        # against K full slots
        assert rc["peak_bytes"] == live * rc["slot_bytes"] + 3 * full["slot_bytes"]
    # and against the oracle
    theta, mbs = make_inputs(cfg, SEED, 5)
    st, ref = run_oracle(cfg, theta, mbs, 5, 2)
    g = run_gpu(cfg, theta, mbs, 5, 2, B.ORDER_EARLY_BACKWARD, flags=B.FLAG_RECOMPUTE)
    compare(cfg, st, ref, g, TOL_BF16, 5)


def test_recompute_fp32_first_and_last_stage():
    _recompute_case(I.CONFIGS["tiny"], 4, 2, B.ORDER_EARLY_BACKWARD)
    emb = I.StageConfig(2, 128, 2, 256, 64, 2, 3, 2, "bf16", has_embedding=True, vocab=512, max_pos=64)
    _recompute_case(emb, 3, 2, B.ORDER_EARLY_BACKWARD)
    head = I.StageConfig(2, 128, 2, 256, 64, 2, 3, 2, "bf16", has_mlm_head=True, vocab=520)
    _recompute_case(head, 3, 2, B.ORDER_EARLY_BACKWARD)


# ---- two stages chained on one GPU: y of stage 0 is x of stage 1, dx of stage 1 is dy of stage 0
def _chained(cfg6, M, dtype_tol):
    """Split a 6-layer stage in two 3-layer stages, run both in their own early-backward orders
    (K_0 = 2, K_1 = 1: policy A of section V-C for two stages) with a task interleaving that
    respects the pipeline's data dependences, through stage_fwd / stage_bwd."""
    import torch
    half = I.StageConfig(cfg6.n_layers // 2, cfg6.hidden, cfg6.n_heads, cfg6.ffn, cfg6.seq, cfg6.micro_batch,
                         M, 2, cfg6.dtype, ln_eps=cfg6.ln_eps)
    theta, mbs = make_inputs(cfg6, SEED, M)
    nh = I.n_params(half)
    assert 2 * nh == theta.size
    T, H = cfg6.tokens, cfg6.hidden
    r0, r1 = B.StageRunner(c_config(half, 2), theta[:nh]), B.StageRunner(c_config(half, 1), theta[nh:])
    try:
        xs = [r0.to_dev(mb["x"].reshape(T, H)) for mb in mbs]
        dys = [r1.to_dev(mb["dy"].reshape(T, H)) for mb in mbs]
        mid = [r0.empty_act() for _ in range(M)]       # the message forward: y of stage 0
        ys = [r1.empty_act() for _ in range(M)]
        dmid = [r1.empty_act() for _ in range(M)]      # the message backward: dx of stage 1
        dxs = [r0.empty_act() for _ in range(M)]
        lists = [B.stage_schedule_ops(M, 2, B.ORDER_EARLY_BACKWARD), B.stage_schedule_ops(M, 1, B.ORDER_EARLY_BACKWARD)]
        pos, done = [0, 0], set()
        while pos[0] < 2 * M or pos[1] < 2 * M:
            progressed = False
            for s in (1, 0):                           # the last stage first: it unblocks backwards
                if pos[s] == 2 * M:
                    continue
                kind, m = lists[s][pos[s]]
                need = ("F", 0, m) if (s == 1 and kind == "F") else (("B", 1, m) if (s == 0 and kind == "B") else None)
                if need is not None and need not in done:
                    continue
                if s == 0 and kind == "F":
                    B.stage_fwd(r0.h, m, xs[m].data_ptr(), mid[m].data_ptr())
                elif s == 1 and kind == "F":
                    B.stage_fwd(r1.h, m, mid[m].data_ptr(), ys[m].data_ptr())
                elif s == 1:
                    B.stage_bwd(r1.h, m, dys[m].data_ptr(), dmid[m].data_ptr())
                else:
                    B.stage_bwd(r0.h, m, dmid[m].data_ptr(), dxs[m].data_ptr())
                done.add((kind, s, m))
                pos[s] += 1
                progressed = True
            assert progressed, "the two task lists deadlock"
        B.stage_sync(r0.h); B.stage_sync(r1.h)
        torch.cuda.synchronize()
        assert B.stage_stats(r0.h).peak_live_slots == min(2, M) and B.stage_stats(r1.h).peak_live_slots == 1
        got = dict(ys=[to_np(y) for y in ys], dxs=[to_np(d) for d in dxs],
                   grads=np.concatenate([r0.grads.cpu().numpy(), r1.grads.cpu().numpy()]))
    finally:
        r0.close(); r1.close()
    st, ref = run_oracle(cfg6, theta, mbs, M, 2)
    compare(cfg6, st, ref, got, dtype_tol, M)
    return theta, mbs, got


def test_two_chained_stages_fp32_equal_the_single_stage_bitwise():
    cfg6 = I.StageConfig(6, 64, 4, 128, 16, 2, 3, 2, "f32", ln_eps=1e-5)
    theta, mbs, got = _chained(cfg6, 3, TOL_F32)
    one = run_gpu(cfg6, theta, mbs, 3, 2, B.ORDER_EARLY_BACKWARD)
    assert np.array_equal(one["grads"], got["grads"])
    for m in range(3):
        assert np.array_equal(one["ys"][m], got["ys"][m]) and np.array_equal(one["dxs"][m], got["dxs"][m])


def test_two_chained_stages_bf16_follow_the_oracle():
    # the boundary tensor is bf16 here, inside one stage the residual stream stays fp32: not bitwise
    _chained(I.StageConfig(6, 256, 4, 512, 128, 2, 3, 2, "bf16"), 3, TOL_BF16)


@pytest.mark.parametrize("M,K", [(1, 1), (2, 1), (3, 2), (5, 3), (7, 2), (4, 4), (6, 8)])
def test_lanes_do_not_change_a_bit_for_any_depth(M, K):
    # (tasks this small stay on one stream: test_streams_change_no_bit has those that do not)
    cfg = I.StageConfig(2, 128, 2, 256, 64, 2, M, K, "bf16")
    theta, mbs = make_inputs(cfg, SEED, M)
    a = run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD)
    b = run_gpu(cfg, theta, mbs, M, K, B.ORDER_GPIPE)
    c = run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD, flags=B.FLAG_RECOMPUTE)
    assert np.array_equal(a["grads"], b["grads"]) and np.array_equal(a["grads"], c["grads"])
    for m in range(M):
        assert np.array_equal(a["ys"][m], b["ys"][m]) and np.array_equal(a["dxs"][m], b["dxs"][m])
        assert np.array_equal(a["dxs"][m], c["dxs"][m])
    assert a["stats"]["peak_live"] == min(K, M) and b["stats"]["peak_live"] == M


def test_graph_replays_equal_the_eager_iteration_bitwise():
    # one HIP graph of the whole iteration (all lanes): replayed several times with eager work and
    # synchronisations in between, every replay must reproduce the eager result
    import torch
    cfg = I.StageConfig(3, 256, 4, 512, 128, 2, 5, 2, "bf16")
    M, K = 5, 2
    theta, mbs = make_inputs(cfg, SEED, M)
    eager = run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD)
    T, H = cfg.tokens, cfg.hidden
    with torch.cuda.stream(torch.cuda.Stream()):
        r = B.StageRunner(c_config(cfg, K), theta)
        try:
            xs = [r.to_dev(mb["x"].reshape(T, H)) for mb in mbs]
            dys = [r.to_dev(mb["dy"].reshape(T, H)) for mb in mbs]
            ys = [r.empty_act() for _ in range(M)]
            dxs = [r.empty_act() for _ in range(M)]
            ptr = lambda ts: [t.data_ptr() for t in ts]
            args = (r.h, M, K, B.ORDER_EARLY_BACKWARD, ptr(xs), ptr(dys), ptr(ys), ptr(dxs))
            with pytest.raises(B.StageError) as e:          # nothing ran eagerly yet
                B.stage_graph_capture(*args)
            assert e.value.code == B.STAGE_E_BAD_ORDER
            with pytest.raises(B.StageError):               # nothing captured yet
                B.stage_graph_launch(r.h)
            B.stage_run_schedule(*args)
            B.stage_sync(r.h)
            B.stage_graph_capture(*args, zero_grads_first=True)
            for rep in range(3):
                for t in ys + dxs:
                    t.zero_()                               # eager work between the replays
                r.grads.fill_(float(rep + 1))               # the graph clears the accumulators itself
                B.stage_graph_launch(r.h)
                B.stage_sync(r.h)
                torch.cuda.synchronize()
                assert np.array_equal(r.grads.cpu().numpy(), eager["grads"]), rep
                for m in range(M):
                    assert np.array_equal(to_np(ys[m]), eager["ys"][m]) and np.array_equal(to_np(dxs[m]), eager["dxs"][m])
                # an eager iteration in between still works and agrees
                B.stage_zero_grads(r.h)
                B.stage_run_schedule(*args)
                B.stage_sync(r.h)
                assert np.array_equal(r.grads.cpu().numpy(), eager["grads"])
            st = B.stage_stats(r.h)
            assert st.fwd_tasks == 7 * M and st.bwd_tasks == 7 * M and st.live_slots == 0
        finally:
            r.close()


def test_graph_capture_needs_a_real_stream():
    cfg = I.CONFIGS["tiny"]
    theta, mbs = make_inputs(cfg, SEED, 2)
    r = B.StageRunner(c_config(cfg, 2), theta)     # torch's default stream is the NULL stream
    try:
        T, H = cfg.tokens, cfg.hidden
        xs = [r.to_dev(mb["x"].reshape(T, H)) for mb in mbs]
        ys = [r.empty_act() for _ in range(2)]
        ptr = lambda ts: [t.data_ptr() for t in ts]
        B.stage_run_schedule(r.h, 2, 2, B.ORDER_EARLY_BACKWARD, ptr(xs), ptr(xs), ptr(ys), ptr(ys))
        B.stage_sync(r.h)
        with pytest.raises(B.StageError) as e:
            B.stage_graph_capture(r.h, 2, 2, B.ORDER_EARLY_BACKWARD, ptr(xs), ptr(xs), ptr(ys), ptr(ys))
        assert e.value.code == B.STAGE_E_CONFIG
    finally:
        r.close()


def test_one_stream_flag_changes_no_bit():
    cfg = I.StageConfig(3, 256, 4, 512, 128, 2, 5, 2, "bf16")
    theta, mbs = make_inputs(cfg, SEED, 5)
    a = run_gpu(cfg, theta, mbs, 5, 2, B.ORDER_EARLY_BACKWARD)
    b = run_gpu(cfg, theta, mbs, 5, 2, B.ORDER_EARLY_BACKWARD, flags=B.FLAG_ONE_STREAM)
    assert np.array_equal(a["grads"], b["grads"])
    for m in range(5):
        assert np.array_equal(a["ys"][m], b["ys"][m]) and np.array_equal(a["dxs"][m], b["dxs"][m])


@pytest.mark.parametrize("M,K", [(1, 1), (5, 3), (4, 4)])
@pytest.mark.parametrize("kind", ["bf16", "f32", "first", "last"])
def test_streams_change_no_bit(kind, M, K):
    """Tasks that go to several streams (a layer's forward between 12 and 150 GFLOP; fp32 from 0.75 on): the side stream
    with the weight gradients' list cut in two, and under re-computation the forward lane and two backward lanes,
    against the same stage on one stream."""
    shape = (2, 256, 4, 1024, 128, 4) if kind == "f32" else (2, 1024, 16, 4096, 256, 2)
    cfg = I.StageConfig(*shape, M, K, "f32" if kind == "f32" else "bf16", has_embedding=kind == "first",
                        has_mlm_head=kind == "last", vocab=500, max_pos=256)
    T, H, F = cfg.tokens, cfg.hidden, cfg.ffn
    gflop = (8 * H * H + 4 * H * F) * T * 1e-9
    assert gflop >= 0.75 if kind == "f32" else 12 <= gflop and gflop * min(M, K, 8192 // T) < 150
    theta, mbs = make_inputs(cfg, SEED, M)
    ref = _bits(run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD, flags=B.FLAG_ONE_STREAM))
    ops = B.stage_schedule_ops(M, K, B.ORDER_EARLY_BACKWARD)
    for flags in (0, B.FLAG_RECOMPUTE, B.FLAG_RECOMPUTE | B.FLAG_ONE_STREAM):
        for kw in (dict(order=B.ORDER_EARLY_BACKWARD), dict(order=B.ORDER_GPIPE), dict(order=B.ORDER_EXPLICIT, explicit_ops=ops)):
            got = _bits(run_gpu(cfg, theta, mbs, M, K, flags=flags, **kw))
            assert all(np.array_equal(x, y) for x, y in zip(ref, got)), (flags, kw)


@pytest.mark.parametrize("shape", [(2, 512, 8, 2048, 512, 4), (2, 768, 12, 3072, 200, 3)])
def test_narrow_stages_on_either_side_of_the_side_streams_line(shape):
    # a layer's forward of 12.9 and 8.5 GFLOP for one micro-batch (its tasks keep the weight gradients) and more than 20 for
    # three (the side stream takes them); 6 GFLOP is the line under re-computation
    cfg = I.StageConfig(*shape, 4, 3, "bf16")
    T, H, F = cfg.tokens, cfg.hidden, cfg.ffn
    gflop = (8 * H * H + 4 * H * F) * T * 1e-9
    assert 6 <= gflop < 20 <= 3 * gflop and -(-H // 128) * -(-F // 128) < 256
    theta, mbs = make_inputs(cfg, SEED, 4)
    ref = _bits(run_gpu(cfg, theta, mbs, 4, 3, B.ORDER_EARLY_BACKWARD, flags=B.FLAG_ONE_STREAM))
    for K, flags in ((3, 0), (1, 0), (3, B.FLAG_RECOMPUTE)):
        got = _bits(run_gpu(cfg, theta, mbs, 4, K, B.ORDER_EARLY_BACKWARD, flags=flags))
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), (K, flags)


@pytest.mark.parametrize("s", [256, 320])
def test_the_attention_backward_of_a_group_has_the_bits_of_its_tasks(s):
    """16 heads of 64, 4 sequences: the heads of four micro-batches fill the 256 units (a workgroup per head, which adds the
    two blocks of 32 columns of delta itself), those of one do not, but fill 64 of them.  The same bits as a group, task by
    task, and both ways on a quarter of the units."""
    M = 4
    cfg = I.StageConfig(1, 1024, 16, 2048, s, 4, M, M, "bf16")
    heads = cfg.micro_batch * cfg.n_heads
    assert heads < 192 <= M * heads and 4 * heads >= 3 * 64 and M * cfg.tokens <= 8192
    theta, mbs = make_inputs(cfg, SEED, M)
    ops = B.stage_schedule_ops(M, M, B.ORDER_EARLY_BACKWARD)
    ways = (dict(order=B.ORDER_EARLY_BACKWARD), dict(order=B.ORDER_EXPLICIT, explicit_ops=ops))
    ref, one = (_bits(run_gpu(cfg, theta, mbs, M, M, **kw)) for kw in ways)
    assert all(np.array_equal(x, y) for x, y in zip(ref, one))
    st = B.pipeline_partition_stream_create(0, 4)
    try:
        for kw in ways:
            r = B.StageRunner(c_config(cfg, M), theta, stream_ptr=st)
            try:
                xs, dys = ([r.to_dev(mb[k].reshape(cfg.tokens, cfg.hidden)) for mb in mbs] for k in ("x", "dy"))
                torch.cuda.synchronize()   # the stage runs on a stream of its own
                ys, dxs = r.run(M, M, xs=xs, dys=dys, **kw)
                B.stage_sync(r.h)
                torch.cuda.synchronize()
                got = _bits(dict(ys=[to_np(y) for y in ys], dxs=[to_np(d) for d in dxs], grads=r.grads.detach().cpu().numpy().copy()))
                assert all(np.array_equal(x, y) for x, y in zip(ref, got)), kw
            finally:
                r.close()
    finally:
        B.pipeline_partition_stream_destroy(st)


@pytest.mark.parametrize("s,stages", [(131, 4), (257, 3)])
def test_the_added_layernorm_of_the_128x64_tiles_follows_the_oracle(s, stages):
    """A stage on 64 units whose FFN products take the 128x64 tile in eight waves, in four stages and in three: the forward
    one adds the LayerNorm of its fp32 residual; ragged rows."""
    cfg = I.StageConfig(1, 256, 4, 2048, s, 8, 1, 1, "bf16")
    d = B.dapple_gemm_desc()
    d.A = d.B = d.C = d.aux = 1 << 20
    d.M, d.N, d.K, d.lda, d.ldb, d.ldc, d.ldaux = cfg.tokens, cfg.hidden, cfg.ffn, cfg.ffn, cfg.hidden, cfg.hidden, cfg.hidden
    d.b_kstrided, d.epi = 1, B.EPI_ADD | B.EPI_AUX32 | B.EPI_OUT32
    assert B.dapple_gemm_plan_beside(B.DTYPE_BF16, d, 64)[:2] == (128, 64) and cfg.tokens % 128
    assert B.dapple_gemm_plan_beside(B.DTYPE_BF16, d, 64)[4:] == (8, stages)
    theta, mbs = make_inputs(cfg, SEED, 1)
    st = B.pipeline_partition_stream_create(0, 4)
    try:
        r = B.StageRunner(c_config(cfg, 1), theta, stream_ptr=st)
        try:
            xs, dys = ([r.to_dev(mb[k].reshape(cfg.tokens, cfg.hidden)) for mb in mbs] for k in ("x", "dy"))
            torch.cuda.synchronize()   # the stage runs on a stream of its own
            ys, dxs = r.run(1, 1, B.ORDER_EARLY_BACKWARD, xs, dys)
            B.stage_sync(r.h)
            torch.cuda.synchronize()
            got = dict(ys=[to_np(y) for y in ys], dxs=[to_np(d) for d in dxs], grads=r.grads.detach().cpu().numpy().copy())
        finally:
            r.close()
    finally:
        B.pipeline_partition_stream_destroy(st)
    oracle, ref = run_oracle(cfg, theta, mbs, 1, 1)
    compare(cfg, oracle, ref, got, TOL_BF16, 1)


@pytest.mark.parametrize("kind", ["recompute", "first_stage", "last_stage", "gpipe_order", "side_stream", "recompute_lanes"])
def test_graph_replays_of_the_other_stage_kinds(kind):
    """A captured iteration of a re-computing stage, a first stage (token ids in), a last stage (losses out), of
    the GPipe order, and of stages large enough for a side stream and for the lanes: two replays with an eager iteration between them, each equal to the eager result bit for bit."""
    import torch
    flags, order = 0, B.ORDER_EARLY_BACKWARD
    if kind == "first_stage":
        cfg = I.StageConfig(2, 128, 2, 256, 64, 2, 4, 2, "bf16", has_embedding=True, vocab=500, max_pos=64)
    elif kind == "last_stage":
        cfg = I.StageConfig(2, 128, 2, 256, 64, 2, 4, 2, "bf16", has_mlm_head=True, vocab=520)
    else:
        cfg = I.StageConfig(3, 256, 4, 512, 128, 2, 4, 2, "bf16")
        if kind in ("side_stream", "recompute_lanes"):   # 6.4 GFLOP a layer and micro-batch
            cfg = I.StageConfig(2, 1024, 16, 4096, 256, 1, 4, 2, "bf16")
        flags = B.FLAG_RECOMPUTE if kind.startswith("recompute") else 0
        order = B.ORDER_GPIPE if kind == "gpipe_order" else order
    M, K = 4, 2
    slots = M if order == B.ORDER_GPIPE else K
    theta, mbs = make_inputs(cfg, SEED, M)
    eager = run_gpu(cfg, theta, mbs, M, K, order, flags=flags)
    T, H = cfg.tokens, cfg.hidden
    emb, head = cfg.has_embedding, cfg.has_mlm_head
    with torch.cuda.stream(torch.cuda.Stream()):
        r = B.StageRunner(c_config(cfg, slots, flags=flags), theta)
        try:
            xs = [r.to_dev(mb["ids"].reshape(T).astype(np.int32)) if emb else r.to_dev(mb["x"].reshape(T, H)) for mb in mbs]
            dys = None if head else [r.to_dev(mb["dy"].reshape(T, H)) for mb in mbs]
            auxs = [r.to_dev(mb["targets"].reshape(T).astype(np.int32)) for mb in mbs] if head else None
            ys = [torch.zeros(1, dtype=torch.float32, device="cuda") if head else r.empty_act() for _ in range(M)]
            dxs = None if emb else [r.empty_act() for _ in range(M)]
            ptr = lambda ts: None if ts is None else [t.data_ptr() for t in ts]
            args = (r.h, M, K, order, ptr(xs), ptr(dys), ptr(ys), ptr(dxs), ptr(auxs))
            B.stage_zero_grads(r.h)
            B.stage_run_schedule(*args)
            B.stage_sync(r.h)
            B.stage_graph_capture(*args, zero_grads_first=True)
            for rep in range(2):
                for t in ys + (dxs or []):
                    t.zero_()
                r.grads.fill_(3.0)
                B.stage_graph_launch(r.h)
                B.stage_sync(r.h)
                torch.cuda.synchronize()
                assert np.array_equal(r.grads.cpu().numpy(), eager["grads"]), rep
                for m in range(M):
                    assert np.array_equal(to_np(ys[m]), eager["ys"][m])
                    assert emb or np.array_equal(to_np(dxs[m]), eager["dxs"][m])
                B.stage_zero_grads(r.h)
                B.stage_run_schedule(*args)
                B.stage_sync(r.h)
                assert np.array_equal(r.grads.cpu().numpy(), eager["grads"])
        finally:
            r.close()


@pytest.mark.parametrize("kind", ["middle", "first", "last", "f32", "odd"])
@pytest.mark.parametrize("M,K,order", [(7, 4, "early"), (5, 3, "early"), (8, 6, "early"), (5, 5, "gpipe")])
def test_groups_of_micro_batches_change_no_bit(kind, M, K, order):
    """Several micro-batches per set of launches (buffers one behind the other: what the built-in orders make of
    them) against the same list task by task, separate buffers: group sizes that divide K, a short last group, token
    counts that are no multiple of 8 or of a k-tile, every stage kind."""
    s, b = (37, 3) if kind == "odd" else (60, 2)
    cfg = I.StageConfig(2, 128, 2, 256, s, b, M, K, "f32" if kind == "f32" else "bf16", has_embedding=kind == "first",
                        has_mlm_head=kind == "last", vocab=200, max_pos=64)
    groups_against_tasks(cfg, M, K, B.ORDER_GPIPE if order == "gpipe" else B.ORDER_EARLY_BACKWARD)


@pytest.mark.parametrize("kind", ["middle", "first", "last", "f32"])
@pytest.mark.parametrize("M,K,order", [(20, 9, "early"), (23, 11, "early"), (11, 11, "gpipe")])
def test_uneven_groups_change_no_bit(kind, M, K, order):
    """More resident micro-batches than a group takes (eight), in runs of slots of different length: 8 + 1 and 8 + 3, a
    short last group."""
    cfg = I.StageConfig(1, 128, 2, 256, 20, 2, M, K, "f32" if kind == "f32" else "bf16", has_embedding=kind == "first",
                        has_mlm_head=kind == "last", vocab=200, max_pos=64)
    groups_against_tasks(cfg, M, K, B.ORDER_GPIPE if order == "gpipe" else B.ORDER_EARLY_BACKWARD)


@pytest.mark.parametrize("order", [B.ORDER_EARLY_BACKWARD, B.ORDER_GPIPE])
def test_outputs_that_are_the_next_inputs(order):
    """ys[m] is xs[m+1] and dxs[m] is dys[m+1]: the same numbers as task by task, the tasks called one after the other."""
    M, K = 4, 4
    cfg = I.StageConfig(1, 128, 2, 256, 60, 2, M, K, "bf16")
    theta, mbs = make_inputs(cfg, SEED, 1)
    T, H = cfg.tokens, cfg.hidden
    out = []
    for driven in (False, True):
        r = B.StageRunner(c_config(cfg, K), theta)
        try:
            x, d = (torch.zeros(M + 1, T, H, dtype=torch.bfloat16, device="cuda") for _ in range(2))
            x[0], d[0] = r.to_dev(mbs[0]["x"].reshape(T, H)), r.to_dev(mbs[0]["dy"].reshape(T, H))
            torch.cuda.synchronize()
            p = lambda t: [t[m].data_ptr() for m in range(M + 1)]
            if driven:
                for kind, m in B.stage_schedule_ops(M, K, order):
                    if kind == "F":
                        B.stage_fwd(r.h, m, p(x)[m], p(x)[m + 1])
                    else:
                        B.stage_bwd(r.h, m, p(d)[m], p(d)[m + 1])
            else:
                B.stage_run_schedule(r.h, M, K, order, p(x)[:M], p(d)[:M], p(x)[1:], p(d)[1:])
            B.stage_sync(r.h)
            out.append((to_np(x), to_np(d), r.grads.cpu().numpy().copy()))
        finally:
            r.close()
    assert all(np.array_equal(a, b) for a, b in zip(*out))
    assert np.linalg.norm(out[0][0][M]) > 0


@pytest.mark.parametrize("H,dtype", [(384, "bf16"), (512, "bf16"), (1024, "bf16"), (1024, "f32")])
def test_weight_gradients_over_three_micro_batches(H, dtype):
    """The weight gradients of a group in one launch, at the widths that take each of its tile shapes: every
    micro-batch's sum goes to the accumulator on its own, 39 rows each (no multiple of a k-tile)."""
    groups_against_tasks(I.StageConfig(1, H, H // 64, 4 * H, 39, 1, 3, 3, dtype), 3, 3, B.ORDER_GPIPE)


def groups_against_tasks(cfg, M, K, ordr):
    import torch
    kind = cfg.dtype
    theta, mbs = make_inputs(cfg, SEED, M)
    ops = B.stage_schedule_ops(M, K, ordr)
    ref = run_gpu(cfg, theta, mbs, M, K, B.ORDER_EXPLICIT, max_slots=K, explicit_ops=ops)
    T, H = cfg.tokens, cfg.hidden
    r = B.StageRunner(c_config(cfg, K), theta)
    try:
        td = torch.float32 if kind == "f32" else torch.bfloat16
        stack = lambda key, shape, dt: torch.stack([torch.as_tensor(mb[key]).reshape(shape) for mb in mbs]).to(dt).cuda().contiguous()
        emb, head = cfg.has_embedding, cfg.has_mlm_head
        xs = stack("ids", (T,), torch.int32) if emb else stack("x", (T, H), td)
        dys = None if head else stack("dy", (T, H), td)
        auxs = stack("targets", (T,), torch.int32) if head else None
        ys = torch.zeros(M, 1, device="cuda") if head else torch.zeros(M, T, H, dtype=td, device="cuda")
        dxs = None if emb else torch.zeros(M, T, H, dtype=td, device="cuda")
        ptr = lambda t: None if t is None else [t[m].data_ptr() for m in range(M)]
        B.stage_run_schedule(r.h, M, K, ordr, ptr(xs), ptr(dys), ptr(ys), ptr(dxs), ptr(auxs))
        B.stage_sync(r.h)
        st = B.stage_stats(r.h)
        assert st.peak_live_slots == K and st.fwd_tasks == M and st.bwd_tasks == M
        assert st.kernel_launches < ref["stats"]["launches"]
        assert np.array_equal(r.grads.cpu().numpy(), ref["grads"])
        for m in range(M):
            assert np.array_equal(to_np(ys[m]), ref["ys"][m])
            assert emb or np.array_equal(to_np(dxs[m]), ref["dxs"][m])
    finally:
        r.close()


def _bits(run):
    return (run["grads"], *run["ys"], *(run["dxs"] or []))


@pytest.mark.parametrize("H,F,s,b", [
    (512, 2048, 128, 2),    # one micro-batch: 32 tiles of 64x64 in a product of width 512, eight of them 256
    (256, 1024, 64, 2),
    (768, 3072, 100, 2),
    (520, 2080, 101, 2),    # ragged rows, columns and K in the large tiles that keep the small ones' sums
    (384, 8192, 64, 1),     # the weight gradients' list cut in two where a side stream takes them
])
def test_fp32_sums_do_not_depend_on_how_a_stage_is_driven(H, F, s, b):
    """fp32 products add in one of two orders; which one must follow from one micro-batch, not from how many of them
    share a launch: early-backward groups two of them, GPipe eight, an explicit list and re-computation one."""
    M, K = 8, 2
    cfg = I.StageConfig(1, H, H // 64 if H % 64 == 0 else 10, F, s, b, M, K, "f32", ln_eps=1e-5)
    theta, mbs = make_inputs(cfg, SEED, M)
    ref = _bits(run_gpu(cfg, theta, mbs, M, K, B.ORDER_EARLY_BACKWARD))
    single = [op for m in range(M) for op in (("F", m), ("B", m))]
    others = [dict(order=B.ORDER_GPIPE), dict(order=B.ORDER_EXPLICIT, explicit_ops=single),
              dict(order=B.ORDER_EARLY_BACKWARD, flags=B.FLAG_RECOMPUTE),
              dict(order=B.ORDER_EARLY_BACKWARD, flags=B.FLAG_ONE_STREAM)]
    for kw in others:
        got = _bits(run_gpu(cfg, theta, mbs, M, K, **kw))
        assert all(np.array_equal(x, y) for x, y in zip(ref, got)), kw


def test_fp32_head_sums_do_not_depend_on_the_group():
    M = 8
    cfg = I.StageConfig(1, 256, 4, 1024, 64, 2, M, 2, "f32", has_mlm_head=True, vocab=1022, ln_eps=1e-5)
    theta, mbs = make_inputs(cfg, SEED, M)
    a = _bits(run_gpu(cfg, theta, mbs, M, 2, B.ORDER_EARLY_BACKWARD))
    b = _bits(run_gpu(cfg, theta, mbs, M, 2, B.ORDER_GPIPE))
    assert all(np.array_equal(x, y) for x, y in zip(a, b))
