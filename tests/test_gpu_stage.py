"""GPU parity of the whole stage path against the fp64 oracle, through the C ABI.

Bounds are the ones the benchmark definition states: forward activations <= 2e-2, weight and
input gradients <= 3e-2 (relative Frobenius, per tensor, max over tensors), Adam fp32 master
state <= 1e-6."""
import numpy as np
import pytest

import oracle
from oracle import transformer as OT
from paper_2110_13005_amd import binding as B
from paper_2110_13005_amd.inputs import CONFIGS, StageShape, make_stage_inputs, make_adam_inputs
from paper_2110_13005_amd.stage import Stage
from helpers import (rel_fro, dev_bf16, dev_f32, host, parity, round_elem, run_direct, check_batch, passes_of, schedules,
                     FWD_TOL, GRAD_TOL, ADAM_TOL, EPS)

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("perturb", [False, True])
@pytest.mark.parametrize("fp32_acc", [1, 0])
def test_tiny_config_parity(perturb, fp32_acc):
    """Config 1 of the benchmark definition, seed 0; also with non-trivial LayerNorm
    parameters and biases so that those gradient paths carry signal."""
    sh = CONFIGS["tiny"]
    layers, xs, dys = make_stage_inputs(sh, seed=0, perturb=perturb)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    with Stage(sh, grad_accum_fp32=fp32_acc) as st:
        st.load_params(layers)
        outs, dxs, grads = run_direct(st, xs, dys)
    if not perturb:
        # biases start at zero and LayerNorm shifts at zero: their gradients are still non-zero
        assert np.linalg.norm(ref[2][0]["b_qkv"]) > 0
    check_batch(outs, dxs, grads, ref)


def test_split_input_qkv_projection_parity_and_effect():
    """qkv_input_split: same result within the bounds, and a strictly smaller q/k error where the
    logits are large (weights N(0, 0.08) at h = 256 give logits of standard deviation ~3)."""
    sh = StageShape(2, 256, 2, 128, 2, 2)
    layers, xs, dys = make_stage_inputs(sh, seed=5, perturb=True, weight_std=0.08)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    errs = []
    for split in (0, 1):
        with Stage(sh, qkv_input_split=split) as st:
            st.load_params(layers)
            outs, dxs, grads = run_direct(st, xs, dys)
        errs.append(check_batch(outs, dxs, grads, ref))
    assert errs[1]["grad"] < errs[0]["grad"] and errs[1]["fwd"] < errs[0]["fwd"], errs


@pytest.mark.parametrize("sh", [
    StageShape(1, 128, 2, 72, 1, 2),          # one layer, ragged sequence, head dim 64
    StageShape(3, 384, 3, 200, 2, 3, 1000),   # head dim 128, ragged T = 400, ffn not 4h
    StageShape(1, 64, 1, 8, 1, 1),            # smallest supported shape
    StageShape(2, 376, 2, 136, 2, 2),         # head dim 188 as in the paper's Table 1 (4512 / 24)
    StageShape(2, 264, 6, 80, 1, 2),          # head dim 44
], ids=["ragged72", "ragged200_ffn1000", "minimal", "headdim188", "headdim44"])
def test_ragged_and_degenerate_shapes(sh):
    layers, xs, dys = make_stage_inputs(sh, seed=3, perturb=True)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    with Stage(sh) as st:
        st.load_params(layers)
        outs, dxs, grads = run_direct(st, xs, dys)
    check_batch(outs, dxs, grads, ref)


@pytest.mark.parametrize("mask", [15, 0])
def test_parity_through_the_large_problem_gemm_kernels(mask):
    """The weight-gradient kernels of large problems also add up the bias gradients, from the tiles they multiply.
    With the launcher's threshold lowered the small shapes go through them too (the copying kernels, mask 15, in their
    variant with a short last k-tile where the token count is no multiple of 64; the register-staged ones, mask 0),
    element by element against the oracle."""
    try:
        B.axonn_tuning(B.TUNE_GEMM_COPY_MASK, mask)
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, 1)
        for sh, fp32_acc, seed in ((CONFIGS["tiny"], 1, 0), (CONFIGS["tiny"], 0, 0),
                                   (StageShape(3, 384, 3, 200, 2, 3, 1000), 0, 3),      # ragged T = 400
                                   (StageShape(1, 64, 1, 8, 1, 1), 1, 3)):              # one block of 8 tokens
            layers, xs, dys = make_stage_inputs(sh, seed=seed, perturb=True)
            ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
            with Stage(sh, grad_accum_fp32=fp32_acc) as st:
                st.load_params(layers)
                outs, dxs, grads = run_direct(st, xs, dys)
            check_batch(outs, dxs, grads, ref)
    finally:
        for knob in (B.TUNE_GEMM_COPY_MASK, B.TUNE_GEMM_BIG_MIN_TILES):
            B.axonn_tuning(knob, -1)


def test_launch_timing_counts_the_launches_of_a_batch():
    """The launch-timing aid (what bench.py's `kernels` and `roofline` fields are made of): per category the launches of
    one batch of direct calls, and a positive time wherever something was launched.  The bias gradients have no
    launches of their own."""
    import torch
    sh = CONFIGS["tiny"]
    L, M = sh.n_layers, sh.n_microbatches
    layers, xs, dys = make_stage_inputs(sh, seed=0)
    with Stage(sh, grad_accum_fp32=0) as st:
        st.load_params(layers)
        torch.cuda.synchronize()
        B.axonn_profile_enable(True)
        try:
            run_direct(st, xs, dys)
            torch.cuda.synchronize()
            got = B.axonn_profile_collect()
        finally:
            B.axonn_profile_enable(False)
    assert "colsum" not in got
    launches = {k: v[1] for k, v in got.items()}
    assert launches["gemm_fwd"] == 4 * L * M and launches["gemm_dgrad"] == 4 * L * M
    assert launches["attention_fwd"] == L * M and launches["attention_bwd"] == L * M
    assert launches["layernorm_fwd"] == 2 * L * M and launches["layernorm_bwd"] == 2 * L * M
    assert launches["copy_in"] == 2 * M                      # the input and the upstream gradient of every microbatch
    assert launches["gemm_wgrad"] > 0 and launches["gemm_wgrad"] % (4 * L) == 0
    for k, (ms, n) in got.items():
        assert (ms > 0) == (n > 0), (k, ms, n)
    assert B.axonn_profile_collect()["gemm_fwd"] == (0.0, 0)   # collect cleared the records


def test_zero_output_projections_give_identity():
    """Degenerate case of the method: W_o = W_fc2 = 0 (and zero biases) makes every layer the
    identity, forward and backward, bit for bit."""
    sh = StageShape(2, 256, 4, 128, 1, 1)
    layers, xs, dys = make_stage_inputs(sh, seed=1)
    for p in layers:
        p["w_o"][:] = 0
        p["w_fc2"][:] = 0
    with Stage(sh) as st:
        st.load_params(layers)
        outs, dxs, _ = run_direct(st, xs, dys)
    assert np.array_equal(outs[0].reshape(xs[0].shape), xs[0].astype(np.float64))
    assert np.array_equal(dxs[0].reshape(dys[0].shape), dys[0].astype(np.float64))


def test_schedule_independence_direct_calls():
    """The paper's correctness claim (Sec. 7.1): scheduling must not change the result.  Every
    valid interleaving gives the oracle's result, and the interleavings agree with each other
    up to accumulation order."""
    sh = CONFIGS["tiny"]
    layers, xs, dys = make_stage_inputs(sh, seed=0, perturb=True)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    results = {}
    with Stage(sh) as st:
        st.load_params(layers)
        for name, order in schedules(sh.n_microbatches, sh.n_microbatches).items():
            results[name] = run_direct(st, xs, dys, order)
            check_batch(*results[name], ref)
        rng = np.random.default_rng(0)
        # seeded random valid order: a backward may only follow its own forward
        order, fwd_done, pending_b = [], 0, []
        while len(order) < 2 * sh.n_microbatches:
            choices = ([("f", fwd_done)] if fwd_done < sh.n_microbatches else []) + [("b", i) for i in pending_b]
            k, i = choices[rng.integers(len(choices))]
            if k == "f":
                order.append((0, i)); pending_b.append(i); fwd_done += 1
            else:
                order.append((1, i)); pending_b.remove(i)
        results["random"] = run_direct(st, xs, dys, order)
        check_batch(*results["random"], ref)
    base = results["warmup1"]
    for name, r in results.items():
        for a, b in zip(r[0] + r[1], base[0] + base[1]):
            assert np.array_equal(a, b), name          # per-microbatch tensors do not depend on order
        for ga, gb in zip(r[2], base[2]):
            for k in ga:
                assert rel_fro(ga[k], gb[k]) <= 1e-3, (name, k)


@pytest.mark.parametrize("n_streams", [1, 2, 3])
def test_message_driven_run_matches_oracle_and_respects_pipeline_limit(n_streams):
    import torch
    sh = CONFIGS["tiny"]
    M, P = sh.n_microbatches, 2
    layers, xs, dys = make_stage_inputs(sh, seed=0, perturb=True)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    with Stage(sh, pipeline_limit=P) as st:
        st.load_params(layers)
        X = [dev_bf16(x) for x in xs]; DY = [dev_bf16(d) for d in dys]
        Y = [torch.zeros_like(X[0]) for _ in range(M)]; DX = [torch.zeros_like(X[0]) for _ in range(M)]
        st.zero_grad()
        # all forward messages are posted first: the scheduler must hold forwards back once P are
        # in flight and take the backward messages that free a slot
        for i in range(M):
            st.post(0, i, X[i], Y[i])
        for i in range(M):
            st.post(1, i, DY[i], DX[i])
        st.run(n_streams)
        st.join()
        torch.cuda.synchronize()
        log = B.axonn_stage_dispatch_log(st.handle)
        assert len(log) == 2 * M and sorted(log) == sorted([(i, k) for i in range(M) for k in (0, 1)])
        live, peak = set(), 0
        for mb, kind in log:
            if kind == 0:
                live.add(mb)
            else:
                assert mb in live
                live.remove(mb)
            peak = max(peak, len(live))
        assert peak == P                                  # steady state holds exactly pipeline_limit
        check_batch([host(y) for y in Y], [host(d) for d in DX], st.grads_numpy(), ref)


@pytest.mark.parametrize("sh,limit,passes,opts", [
    (StageShape(2, 256, 4, 128, 2, 5), 5, 1, dict(wgrad_group=3)),            # up to 5 microbatches in one pass
    (StageShape(2, 384, 3, 200, 2, 4, 1000), 3, 3, dict(grad_accum_fp32=0)),  # ragged tiles, two of one and one of two
    (StageShape(1, 376, 2, 72, 1, 9), 9, 2, dict(grad_accum_fp32=0, wgrad_group=1)),   # masked head dimension, 5 and 4
    (StageShape(1, 1024, 8, 1024, 1, 3), 3, 1, dict()),                       # separate attention backward kernels from 3 on, d 128
    (StageShape(1, 1024, 16, 1000, 1, 2), 2, 1, dict()),                      # from 2 on, d 64, ragged
    (StageShape(1, 1024, 16, 512, 2, 4), 2, 2, dict(qkv_input_split=2)),      # backwards past the forwards between them
    (StageShape(2, 256, 4, 64, 1, 4, 264), 4, 1, dict()),                     # the narrowest MLP: its activations just hold the gradients
], ids=["tiny5", "ragged", "headdim188", "attn_tiles128", "attn_tiles64", "limit2", "narrow_mlp"])
@pytest.mark.parametrize("n_streams", [1, 2])
def test_merged_microbatches_give_the_bits_of_single_ones(sh, limit, passes, opts, n_streams):
    """Messages that run as one pass over all their tokens: every y and dx bit for bit that of direct calls; with a
    done_event per message (nothing merged) and with overlapping result buffers (forwards not merged) too.  `passes`: how
    many forward and backward passes there are, by the library's own count of launches."""
    import torch
    layers, xs, dys = make_stage_inputs(sh, seed=4, perturb=True)
    M = sh.n_microbatches
    X = [dev_bf16(x) for x in xs]; DY = [dev_bf16(d) for d in dys]
    with Stage(sh, pipeline_limit=limit, **opts) as st, Stage(sh, **opts) as whole:
        st.load_params(layers); whole.load_params(layers)
        outs, dxs, grads = run_direct(whole, xs, dys)
        formed = []
        for events, shared in ((False, False), (True, False), (False, True)):
            Y = [torch.zeros_like(X[0]) for _ in range(M)]; DX = [torch.zeros_like(X[0]) for _ in range(M)]
            if shared:
                Y = [Y[0]] * M
            evs = [torch.cuda.Event() for _ in range(2 * M)]
            for e in evs:
                e.record()                                    # torch creates the event behind it at the first record
            torch.cuda.synchronize()
            st.zero_grad()
            order = [(0, i) for i in range(limit)]
            for i in range(M):
                order += [(1, i)] + ([(0, limit + i)] if limit + i < M else [])
            for kind, i in order:
                st.post(kind, i, (X, DY)[kind][i], (Y, DX)[kind][i], **({"done_event": evs[2 * i + kind]} if events else {}))
            made = passes_of(lambda: (st.run(n_streams), st.join()), sh.n_layers)
            assert made == ((M, M) if events else (M, made[1]) if shared else (passes, passes)), (events, shared, made)
            for i in range(M):
                if not shared or i == M - 1:
                    assert np.array_equal(host(Y[i]), outs[i]), (events, shared, i)
                assert np.array_equal(host(DX[i]), dxs[i]), (events, shared, i)
            formed.append(st.grads_numpy())
            for ga, gb, g0 in zip(formed[-1], grads, formed[0]):
                for k in ga:
                    # the same passes over the same microbatches; the LayerNorms' sums go over the rows in another order
                    assert k.startswith("ln") or np.array_equal(ga[k], g0[k]), (events, shared, k)
                    # direct calls, with a slot for every microbatch, close other groups
                    assert rel_fro(ga[k], gb[k]) <= (1e-3 if opts.get("grad_accum_fp32", 1) else 8e-3), (events, shared, k)


@pytest.mark.parametrize("sh,fp32_acc", [
    (StageShape(1, 1024, 16, 256, 1, 1), 1),       # 768 tiles: one launch by direct calls, four beside another stream
    (StageShape(1, 1024, 8, 200, 1, 1, 1000), 0),  # the same, ragged in every dimension
    (StageShape(2, 72, 2, 8, 1, 1, 264), 1),       # one or two ragged tiles per problem, one launch either way
], ids=["tiles768", "ragged", "smallest"])
def test_weight_gradients_of_a_layer_in_one_launch(sh, fp32_acc):
    """A layer's four weight gradients (and bias gradients) as one grid: the oracle's, and bit for bit the same from
    separate launches (other tiles add k in the same order)."""
    import torch
    layers, xs, dys = make_stage_inputs(sh, seed=6, perturb=True)
    ref = oracle.stage_batch(xs, dys, layers, sh.n_heads, EPS)
    with Stage(sh, grad_accum_fp32=fp32_acc) as st:
        st.load_params(layers)
        outs, dxs, grads = run_direct(st, xs, dys)
        check_batch(outs, dxs, grads, ref)
        X, DY = dev_bf16(xs[0]), dev_bf16(dys[0])
        Y, DX = torch.zeros_like(X), torch.zeros_like(X)
        torch.cuda.synchronize()
        st.zero_grad()
        st.post(0, 0, X, Y); st.post(1, 0, DY, DX)
        st.run(2); st.join()
        torch.cuda.synchronize()
        for ga, gb in zip(st.grads_numpy(), grads):
            for k in ga:
                assert np.array_equal(ga[k], gb[k]), k


def test_message_arrival_order_follows_ready_events():
    """A message whose payload has not arrived (event not yet signalled) is passed over for one
    that has: forward vs backward is decided by what is ready, not by posting order."""
    import torch
    sh = StageShape(1, 128, 2, 64, 1, 2)
    layers, xs, dys = make_stage_inputs(sh, seed=2)
    with Stage(sh) as st:
        st.load_params(layers)
        X = [dev_bf16(x) for x in xs]; DY = [dev_bf16(d) for d in dys]
        Y = [torch.zeros_like(X[0]) for _ in range(2)]; DX = [torch.zeros_like(X[0]) for _ in range(2)]
        comm = torch.cuda.Stream()
        late = torch.cuda.Event()
        with torch.cuda.stream(comm):
            torch.cuda._sleep(int(2.4e9 * 0.2))           # ~0.2 s: message 0's payload is "in transit"
            late.record(comm)
        st.zero_grad()
        st.post(0, 0, X[0], Y[0], ready_event=late)
        st.post(0, 1, X[1], Y[1])
        st.post(1, 1, DY[1], DX[1])
        st.post(1, 0, DY[0], DX[0])
        st.run(2)
        st.join()
        torch.cuda.synchronize()
        log = B.axonn_stage_dispatch_log(st.handle)
        assert log[0] == (1, 0) and log[1] == (1, 1)      # microbatch 1 went first, fwd then bwd
        assert log[2:] == [(0, 0), (0, 1)]


def test_state_errors_leave_stage_usable():
    import torch
    sh = StageShape(1, 128, 2, 64, 1, 3)
    layers, xs, dys = make_stage_inputs(sh, seed=2)
    with Stage(sh, pipeline_limit=2) as st:
        st.load_params(layers)
        X = [dev_bf16(x) for x in xs]; Y = torch.zeros_like(X[0]); D = torch.zeros_like(X[0])
        with pytest.raises(B.AxonnError) as e:
            st.backward(0, X[0], D)                       # backward before its forward
        assert e.value.status == B.AXONN_ESTATE
        st.forward(0, X[0], Y)
        with pytest.raises(B.AxonnError) as e:
            st.forward(0, X[0], Y)                        # duplicate microbatch id
        assert e.value.status == B.AXONN_ESTATE
        st.forward(1, X[1], Y)
        with pytest.raises(B.AxonnError) as e:
            st.forward(2, X[2], Y)                        # pipeline_limit overflow
        assert e.value.status == B.AXONN_ESTATE and "pipeline_limit" in str(e.value)
        with pytest.raises(B.AxonnError) as e:
            st.zero_grad()                                # microbatches in flight
        assert e.value.status == B.AXONN_ESTATE
        with pytest.raises(B.AxonnError) as e:
            B.axonn_stage_forward(st.handle, 5, None, Y)  # null pointer
        assert e.value.status == B.AXONN_EINVAL
        st.backward(0, X[0], D)
        st.forward(2, X[2], Y)                            # slot freed: usable again
        st.backward(1, X[1], D)
        st.backward(2, X[2], D)
        # message mode: only backward messages posted and nothing in flight -> cannot progress
        st.zero_grad()
        st.post(1, 0, X[0], D)
        with pytest.raises(B.AxonnError) as e:
            st.run(2)
        assert e.value.status == B.AXONN_ESTATE
        with pytest.raises(B.AxonnError) as e:
            st.post(1, 0, X[0], D)                        # duplicate message
        assert e.value.status == B.AXONN_ESTATE
        torch.cuda.synchronize()


def test_fixed_schedule_is_bit_reproducible():
    sh = CONFIGS["tiny"]
    layers, xs, dys = make_stage_inputs(sh, seed=0, perturb=True)
    with Stage(sh) as st:
        st.load_params(layers)
        a = run_direct(st, xs, dys)
        b = run_direct(st, xs, dys)
    for x, y in zip(a[0] + a[1], b[0] + b[1]):
        assert np.array_equal(x, y)
    for ga, gb in zip(a[2], b[2]):
        for k in ga:
            assert np.array_equal(ga[k], gb[k]), k


def test_device_memory_accounting():
    """Sec. 5.2: parameters and gradients take 4*phi bytes on the device (2 + 2), the optimizer
    n_sets * 12 * bsize (theta, m, v buckets; the bf16 gradient is read in place, so the paper's
    4*bsize descale scratch is not needed)."""
    sh = CONFIGS["tiny"]
    with Stage(sh, grad_accum_fp32=0) as st:
        by = B.axonn_stage_device_bytes(st.handle)
        phi = st.n_params
        assert by[0] + by[1] == 4 * phi and by[2] == 0
        per_layer = 2 * sh.tokens * (13 * sh.hidden + 3 * sh.ffn)   # forward stash + kept output gradients
        assert by[3] >= sh.n_microbatches * sh.n_layers * per_layer
        assert by[3] <= 1.1 * sh.n_microbatches * sh.n_layers * per_layer + (1 << 20)
        bucket = 1 << 16
        n = phi
        hm = [B.axonn_pinned_alloc(4 * n) for _ in range(3)]
        B.axonn_stage_optimizer_attach(st.handle, hm[0], hm[1], hm[2], n, bucket)
        assert B.axonn_stage_device_bytes(st.handle)[5] == 3 * 12 * bucket
    for p in hm:
        B.axonn_pinned_free(p)
    with Stage(sh, grad_accum_fp32=1) as st:
        assert B.axonn_stage_device_bytes(st.handle)[2] == 4 * st.n_params


def _pinned_array(n):
    import ctypes
    p = B.axonn_pinned_alloc(4 * n)
    arr = np.ctypeslib.as_array((ctypes.c_float * n).from_address(p))
    return p, arr


@pytest.mark.parametrize("n,bucket,fresh,wd,step,gs", [
    (1_000_000, 1 << 18, False, 0.0, 100, 1.0),     # 4 buckets, ragged last
    (300_000, 1 << 16, True, 0.01, 1, 0.125),       # 5 buckets, first step, decay, descale
    (5000, 1 << 16, False, 0.0, 7, 1.0),            # single partial bucket, n % 8 == 0
    (12_345, 4096, False, 0.0, 3, 1.0),             # n not a multiple of 8
])
def test_offloaded_adam_matches_oracle(n, bucket, fresh, wd, step, gs):
    import torch
    th, m, v, g16 = make_adam_inputs(n, seed=n, fresh=fresh)
    lr, b1, b2, eps = 1e-4, 0.9, 0.95, 1e-8
    rt, rm, rv, r16 = oracle.adam_step(th, m, v, g16, lr, b1, b2, eps, wd, step, gs, half=B.ELEM)
    ptrs, arrs = zip(*[_pinned_array(n) for _ in range(3)])
    arrs[0][:] = th; arrs[1][:] = m; arrs[2][:] = v
    G = dev_bf16(g16)
    P16 = torch.zeros(n, dtype=B.torch_elem_dtype(), device="cuda")
    opt = B.axonn_offload_adam_create(0, n, bucket, P16, G, ptrs[0], ptrs[1], ptrs[2])
    try:
        assert B.axonn_offload_adam_device_bytes(opt) == 3 * 12 * min(bucket, (n + 7) // 8 * 8)
        B.axonn_offload_adam_step(opt, lr, b1, b2, eps, wd, step, gs)
        torch.cuda.synchronize()
        assert rel_fro(arrs[0], rt) <= ADAM_TOL
        assert rel_fro(arrs[1], rm) <= ADAM_TOL
        assert rel_fro(arrs[2], rv) <= ADAM_TOL
        got16 = host(P16)
        assert np.array_equal(got16, oracle.half_round(arrs[0], B.ELEM).astype(np.float64))   # bf16 of own master, bit exact
        assert np.abs(got16 - r16).max() <= np.abs(r16).max() * 2.0 ** -7             # <= 1 ulp of the oracle's
        # second step continues from the offloaded state
        rt2, rm2, rv2, _ = oracle.adam_step(rt, rm, rv, g16, lr, b1, b2, eps, wd, step + 1, gs, half=B.ELEM)
        B.axonn_offload_adam_step(opt, lr, b1, b2, eps, wd, step + 1, gs)
        torch.cuda.synchronize()
        assert rel_fro(arrs[0], rt2) <= ADAM_TOL and rel_fro(arrs[1], rm2) <= ADAM_TOL
    finally:
        B.axonn_offload_adam_destroy(opt)
        for p in ptrs:
            B.axonn_pinned_free(p)


@pytest.mark.parametrize("n,bucket", [(3, 8), (1027, 1 << 8), (262_147, 1 << 16)])
def test_offloaded_adam_in_place_and_through_buckets_agree(n, bucket):
    """Pinned 16-byte-aligned state is updated in place over the link; pinned state at an odd element and pageable state go
    through the device buckets.  The same elementwise arithmetic: the same bits, and nothing written past the end."""
    import torch
    th, m, v, g16 = make_adam_inputs(n, seed=n)
    G = dev_bf16(g16)
    got = []
    for kind in ("aligned", "odd", "pageable"):
        ptrs, bufs = zip(*[_pinned_array(n + 2) for _ in range(3)])
        arrs = [np.full(n + 2, 7.0, np.float32) for _ in range(3)] if kind == "pageable" else [b for b in bufs]
        lo = 1 if kind == "odd" else 0
        for a, src in zip(arrs, (th, m, v)):
            a[:] = 7.0
            a[lo:lo + n] = src
        P16 = torch.zeros(n, dtype=B.torch_elem_dtype(), device="cuda")
        opt = B.axonn_offload_adam_create(0, n, bucket, P16, G, *[a.ctypes.data + 4 * lo for a in arrs])
        B.axonn_profile_enable(True)
        try:
            for step in (1, 2):
                B.axonn_offload_adam_step(opt, 1e-3, 0.9, 0.95, 1e-8, 0.01, step, 0.5)
            # one launch per step in place, one per bucket otherwise
            assert B.axonn_profile_collect()["adam"][1] == 2 * (1 if kind == "aligned" else -(-n // bucket))
            assert all((a[lo + n:] == 7.0).all() and (a[:lo] == 7.0).all() for a in arrs)
            got.append([a[lo:lo + n].copy() for a in arrs] + [host(P16)])
        finally:
            B.axonn_profile_enable(False)
            B.axonn_offload_adam_destroy(opt)
            for p in ptrs:
                B.axonn_pinned_free(p)
    rt = oracle.adam_step(*oracle.adam_step(th, m, v, g16, 1e-3, 0.9, 0.95, 1e-8, 0.01, 1, 0.5, half=B.ELEM)[:3], g16,
                          1e-3, 0.9, 0.95, 1e-8, 0.01, 2, 0.5, half=B.ELEM)[0]
    assert rel_fro(got[0][0], rt) <= ADAM_TOL
    for other in got[1:]:
        assert all(np.array_equal(a, b) for a, b in zip(got[0], other))


def test_stage_batch_then_optimizer_step():
    """Alg. 1's per-GPU body: all microbatches forward/backward, then "run the optimizer" on the
    stage's own bf16 parameter / gradient buffers with grad_scale = 1/M."""
    import torch
    sh = CONFIGS["tiny"]
    M = sh.n_microbatches
    layers, xs, dys = make_stage_inputs(sh, seed=0, perturb=True)
    with Stage(sh) as st:
        st.load_params(layers)
        n = st.n_params
        ptrs, arrs = zip(*[_pinned_array(n) for _ in range(3)])
        theta0 = st.params.float().cpu().numpy()
        arrs[0][:] = theta0; arrs[1][:] = 0; arrs[2][:] = 0
        run_direct(st, xs, dys)
        g16 = st.grads.float().cpu().numpy()
        B.axonn_stage_optimizer_attach(st.handle, ptrs[0], ptrs[1], ptrs[2], n, 1 << 18)
        with pytest.raises(B.AxonnError):
            B.axonn_stage_optimizer_attach(st.handle, ptrs[0], ptrs[1], ptrs[2], n - 8, 1 << 18)
        B.axonn_stage_optimizer_step(st.handle, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1, 1.0 / M)
        torch.cuda.synchronize()
        rt, rm, rv, r16 = oracle.adam_step(theta0, 0 * theta0, 0 * theta0, g16, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1, 1.0 / M, half=B.ELEM)
        assert rel_fro(arrs[0], rt) <= ADAM_TOL and rel_fro(arrs[1], rm) <= ADAM_TOL and rel_fro(arrs[2], rv) <= ADAM_TOL
        assert np.array_equal(host(st.params), oracle.half_round(arrs[0], B.ELEM).astype(np.float64))
    for p in ptrs:
        B.axonn_pinned_free(p)


@pytest.mark.parametrize("done,opts", [(2, dict(wgrad_group=1)), (2, dict(wgrad_group=2)), (1, dict(ckpt_stride=1)),
                                       (3, dict(ckpt_stride=2)), (1, dict(wgrad_group=1, pipeline_limit=1))])
def test_batch_cut_short_where_no_weight_gradients_are_pending(done, opts):
    """A batch of fewer microbatches than n_microbatches, after a full one: every gradient in the 16-bit buffer, the
    LayerNorms' among them, is that of the short batch, and the optimizer step takes exactly those."""
    import torch
    sh = StageShape(2, 192, 3, 96, 2, 4)
    layers, xs, dys = make_stage_inputs(sh, seed=4, perturb=True)
    pairs = [m for i in range(4) for m in ((0, i), (1, i))]
    with Stage(sh, grad_accum_fp32=0, **opts) as st:
        st.load_params(layers)
        run_direct(st, xs, dys, pairs)
        outs, dxs, grads = run_direct(st, xs[::-1][:done], dys[::-1][:done], pairs[:2 * done])
        check_batch(outs, dxs, grads, oracle.stage_batch(xs[::-1][:done], dys[::-1][:done], layers, sh.n_heads, EPS))
        n = st.n_params
        ptrs, arrs = zip(*[_pinned_array(n) for _ in range(3)])
        try:
            theta0 = st.params.float().cpu().numpy()
            arrs[0][:] = theta0; arrs[1][:] = 0; arrs[2][:] = 0
            B.axonn_stage_optimizer_attach(st.handle, *ptrs, n, 1 << 18)
            assert B.axonn_stage_count_nonfinite_grads(st.handle, None) == 0
            B.axonn_stage_optimizer_step(st.handle, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1, 1.0 / done)
            g16 = np.concatenate([grads[int(k.split(".")[0][5:])][k.split(".")[1]].ravel() for k in st.layout])
            rt = oracle.adam_step(theta0, 0 * theta0, 0 * theta0, g16, 1e-3, 0.9, 0.999, 1e-8, 0.01, 1, 1.0 / done, half=B.ELEM)[0]
            assert rel_fro(arrs[0], rt) <= ADAM_TOL
        finally:
            for p in ptrs:
                B.axonn_pinned_free(p)


@pytest.mark.parametrize("T,h", [(2056, 256), (1032, 512), (1048, 520), (1032, 1024), (520, 1032), (528, 2048), (264, 2056),
                                 (264, 4096), (264, 4104), (264, 6144), (264, 6152), (264, 8192), (264, 8200), (264, 12288),
                                 (264, 12296), (72, 16384)])
def test_layernorm_backward_of_a_layer_at_every_row_width(T, h):
    """The LayerNorm backward a stage runs, on its own: with an identity and a diagonal of powers of two as the MLP's maps, a
    GeLU far in its linear part and nothing else in the layer, dout is dz times the diagonal and the stage's input
    gradient is LayerNorm 2's, residual gradient dz included, all exact but for the kernel's own rounding.  Widths at the
    edges of its variants (1 to 8 waves per row, 1 to 4 chunks per lane), several rounds of rows, two microbatches."""
    import torch
    rng = np.random.default_rng(T + h)
    sh = StageShape(1, h, h // 8, T, 1, 2, h)
    diag = np.float32([1, -2, 0.5, -0.25, 4])[rng.integers(0, 5, h)]
    gamma = round_elem(1 + 0.2 * rng.standard_normal(h)).astype(np.float32)
    with Stage(sh, grad_accum_fp32=0) as st:
        st.tensor("layer0.w_fc1").fill_diagonal_(1.0)
        st.tensor("layer0.w_fc2").copy_(torch.diag(dev_f32(diag)))
        st.tensor("layer0.b_fc1").fill_(64.0)
        st.tensor("layer0.ln2_g").copy_(dev_f32(gamma))
        torch.cuda.synchronize()
        xs, dys = ([round_elem(m + rng.standard_normal((1, T, h))).astype(np.float32) for _ in range(2)] for m in (0.5, 0.0))
        _, dxs, grads = run_direct(st, xs, dys)
    tot_g = tot_b = 0.0
    for x, dy, dx in zip(xs, dys, dxs):
        _, xhat, rstd = OT.layernorm_fwd(x.astype(np.float64), gamma.astype(np.float64), np.zeros(h), EPS)
        ref, dg, db = OT.layernorm_bwd(dy.astype(np.float64) * diag, xhat, rstd, gamma.astype(np.float64))
        parity(dx.reshape(ref.shape), ref + dy, 5e-3, 1.0, label="layernorm_backward_of_a_layer")      # one rounding
        tot_g, tot_b = tot_g + dg, tot_b + db
    parity(grads[0]["ln2_g"], tot_g, 5e-3, 1.0, axis=None, label="layernorm_backward_of_a_layer")
    parity(grads[0]["ln2_b"], tot_b, 5e-3, 1.0, axis=None, label="layernorm_backward_of_a_layer")
