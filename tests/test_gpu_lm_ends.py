"""GPU parity of the pipeline's two ends (Alg. 2's special cases: token + position embedding in front; final
LayerNorm, LM head and the pre-divided cross-entropy behind, Sec. 4.2) against the fp64 oracle, through the
C ABI: the single operations, and stages that are the first, the last, or both."""
import numpy as np
import pytest

from oracle import lm_ends as OE
from oracle import transformer as OT
from paper_2110_13005_amd import binding as B
from paper_2110_13005_amd.inputs import StageShape, make_stage_inputs, make_lm_inputs, snap_elem
from paper_2110_13005_amd.stage import Stage, view_bf16
from helpers import (rel_fro, dev_bf16, host, dev_i32, EmbedHandle, HeadHandle, oracle_model, passes_of, FWD_TOL, GRAD_TOL,
                     EPS)

pytestmark = pytest.mark.gpu


def test_embedding_forward_backward_with_repeated_and_out_of_range_ids():
    import torch
    rng = np.random.default_rng(0)
    V, h, s, b = 40, 136, 24, 3                    # few rows: many repeats; 136 columns: a ragged vector tail
    wte, wpe = snap_elem(rng.standard_normal((V, h), dtype=np.float32)), snap_elem(rng.standard_normal((s, h), dtype=np.float32))
    e = EmbedHandle(V, h, s, b, wte, wpe)
    try:
        tot_te, tot_pe = 0.0, 0.0
        for it in range(3):
            tokens = rng.integers(0, V, (b, s))
            if it == 1:
                tokens[0, 0], tokens[1, 3], tokens[2, 5] = -7, V, V + 1000      # clamped to 0, V-1, V-1
            clamped = np.clip(tokens, 0, V - 1)
            x = torch.zeros(b, s, h, dtype=B.torch_elem_dtype(), device="cuda")
            B.axonn_embed_forward(e.h, dev_i32(tokens), x)
            ref = OE.embedding_forward(clamped, wte, wpe)
            assert rel_fro(host(x), ref) <= 4e-3                               # one bf16 rounding of the sum
            dx = snap_elem(rng.standard_normal((b, s, h), dtype=np.float32))
            B.axonn_embed_backward(e.h, dev_i32(tokens), dev_bf16(dx))
            torch.cuda.synchronize()
            dte, dpe = OE.embedding_backward(dx, clamped, V, s)
            tot_te, tot_pe = tot_te + dte, tot_pe + dpe
            gte, gpe = e.grads_numpy()
            assert rel_fro(gte, tot_te) <= 6e-3 and rel_fro(gpe, tot_pe) <= 6e-3
            unused = np.setdiff1d(np.arange(V), clamped.ravel())
            if it == 0 and len(unused):
                assert not gte[unused].any()                                   # rows nobody used stay exactly zero
        B.axonn_embed_zero_grad(e.h)                                           # the next pass overwrites
        tokens = rng.integers(0, V, (b, s)); dx = snap_elem(rng.standard_normal((b, s, h), dtype=np.float32))
        B.axonn_embed_backward(e.h, dev_i32(tokens), dev_bf16(dx))
        torch.cuda.synchronize()
        dte, dpe = OE.embedding_backward(dx, tokens, V, s)
        gte, gpe = e.grads_numpy()
        assert rel_fro(gte, dte) <= 4e-3 and rel_fro(gpe, dpe) <= 4e-3
    finally:
        e.close()


@pytest.mark.parametrize("T,h,V,M", [(256, 192, 1000, 2), (72, 64, 264, 3), (2056, 256, 4104, 1)])
def test_head_loss_and_backward(T, h, V, M):
    """Several row tiles and ragged tails in every dimension; gradients accumulate over M microbatches."""
    import torch
    rng = np.random.default_rng(T)
    g = snap_elem((1 + 0.1 * rng.standard_normal(h)).astype(np.float32)); bt = snap_elem((0.1 * rng.standard_normal(h)).astype(np.float32))
    W = snap_elem((0.05 * rng.standard_normal((h, V))).astype(np.float32))
    hd = HeadHandle(V, h, T, M, g, bt, W)
    try:
        tot = None
        for it in range(M):
            x = snap_elem(rng.standard_normal((1, T, h), dtype=np.float32)); tg = rng.integers(0, V, (1, T))
            loss = torch.zeros(1, device="cuda"); dx = torch.zeros(T, h, dtype=B.torch_elem_dtype(), device="cuda")
            B.axonn_head_forward_backward(hd.h, dev_bf16(x), dev_i32(tg), loss, dx)
            torch.cuda.synchronize()
            rl, c = OE.head_loss_forward(x, g, bt, W, tg, EPS, M)
            rdx, rg = OE.head_loss_backward(c, g, W, tg, M)
            assert abs(loss.item() - rl) <= 2e-3 * abs(rl), (loss.item(), rl)
            assert rel_fro(host(dx).reshape(rdx.shape), rdx) <= GRAD_TOL
            tot = rg if tot is None else {k: tot[k] + rg[k] for k in rg}
            got = hd.grads_numpy()
            for k in tot:
                assert rel_fro(got[k], tot[k]) <= GRAD_TOL, (k, it)
    finally:
        hd.close()


@pytest.mark.parametrize("T,h", [(8, 8), (2056, 512), (1032, 520), (1048, 1024), (520, 1032), (1032, 2048), (264, 2056),
                                 (264, 4104), (264, 6152), (72, 8200), (264, 16384), (520, 8192), (264, 12288), (264, 12296)])
def test_head_layernorm_backward_at_every_row_width(T, h):
    """The LayerNorm backward kernel splits a row over 1, 2, 4 or 8 waves and holds 1 to 4 chunks per lane, several rows
    per workgroup or several rounds of rows: dx and the parameter gradients of two microbatches at the edges of that."""
    import torch
    rng = np.random.default_rng(T + h)
    V, M = 16, 2
    g = snap_elem((1 + 0.1 * rng.standard_normal(h)).astype(np.float32)); bt = snap_elem((0.1 * rng.standard_normal(h)).astype(np.float32))
    W = snap_elem((rng.standard_normal((h, V)) / np.sqrt(h)).astype(np.float32))
    hd = HeadHandle(V, h, T, M, g, bt, W)
    try:
        tot = None
        for it in range(M):
            x = snap_elem(rng.standard_normal((1, T, h), dtype=np.float32)); tg = rng.integers(0, V, (1, T))
            loss = torch.zeros(1, device="cuda"); dx = torch.zeros(T, h, dtype=B.torch_elem_dtype(), device="cuda")
            B.axonn_head_forward_backward(hd.h, dev_bf16(x), dev_i32(tg), loss, dx)
            torch.cuda.synchronize()
            rl, c = OE.head_loss_forward(x, g, bt, W, tg, EPS, M)
            rdx, rg = OE.head_loss_backward(c, g, W, tg, M)
            assert rel_fro(host(dx).reshape(rdx.shape), rdx) <= GRAD_TOL
            tot = rg if tot is None else {k: tot[k] + rg[k] for k in rg}
            got = hd.grads_numpy()
            for k in ("lnf_g", "lnf_b"):
                assert rel_fro(got[k], tot[k]) <= GRAD_TOL, (k, it)
    finally:
        hd.close()


@pytest.mark.parametrize("T,h", [(8, 8), (16, 520), (8, 2056)])
def test_head_layernorm_backward_of_large_equal_rows(T, h):
    """Rows of one large value (2^120 in bfloat16): xhat is exactly zero and every gradient finite, although -mean * rstd
    would overflow."""
    import torch
    V, rng = 16, np.random.default_rng(h)
    big = 2.0 ** 120 if B.ELEM == "bf16" and h == 8 else 2.0 ** 110 if B.ELEM == "bf16" else 2.0 ** 14
    hd = HeadHandle(V, h, T, 1, np.ones(h, np.float32), np.zeros(h, np.float32), snap_elem(rng.standard_normal((h, V)).astype(np.float32)))
    try:
        x = np.full((1, T, h), big, np.float32)
        loss = torch.zeros(1, device="cuda"); dx = torch.zeros(T, h, dtype=B.torch_elem_dtype(), device="cuda")
        B.axonn_head_forward_backward(hd.h, dev_bf16(x), dev_i32(rng.integers(0, V, (1, T))), loss, dx)
        torch.cuda.synchronize()
        assert np.isfinite(host(dx)).all() and np.isfinite(hd.grads_numpy()["lnf_g"]).all()
        assert not hd.grads_numpy()["lnf_g"].any() and np.abs(host(dx)).max() > 0      # xhat = 0: no gain gradient
    finally:
        hd.close()


@pytest.mark.parametrize("n_streams,ckpt", [(1, 0), (2, 0), (3, 2)])
def test_whole_model_on_one_stage_message_driven(n_streams, ckpt):
    """A stage that is both the first and the last one: token messages in, losses out, every gradient against the
    oracle's plain embedding -> layers -> head -> loss chain."""
    import torch
    sh = StageShape(2, 128, 2, 64, 2, 4)
    V = 520
    layers, _, _ = make_stage_inputs(sh, seed=11, perturb=True)
    tokens, targets, wte, wpe, g, bt, W = make_lm_inputs(sh, V, seed=12)
    ref_losses, ref = oracle_model(tokens, targets, wte, wpe, layers, g, bt, W, sh.n_heads, sh.n_microbatches)
    M = sh.n_microbatches
    e = EmbedHandle(V, sh.hidden, sh.seq_len, sh.microbatch_size, wte, wpe)
    hd = HeadHandle(V, sh.hidden, sh.tokens, M, g, bt, W)
    try:
        with Stage(sh, pipeline_limit=2, ckpt_stride=ckpt) as st:
            st.load_params(layers)
            B.axonn_stage_attach_ends(st.handle, e.h, hd.h)
            TK = [dev_i32(t) for t in tokens]; TG = [dev_i32(t) for t in targets]
            losses = torch.zeros(M, device="cuda")
            for rep in range(2):        # the second batch must start from cleared accumulators at both ends
                st.zero_grad()
                with pytest.raises(B.AxonnError):
                    st.post(1, 0, TK[0], None)                       # a last stage takes no backward messages
                for i in range(M):
                    st.post(0, i, TK[i], None, targets=TG[i], loss=losses[i:i + 1])
                st.run(n_streams)
                st.join()
                torch.cuda.synchronize()
                for i in range(M):
                    assert abs(losses[i].item() - ref_losses[i]) <= 2e-3 * abs(ref_losses[i])
                for li, gl in enumerate(st.grads_numpy()):
                    for k, v in gl.items():
                        assert rel_fro(v, ref["layers"][li][k]) <= GRAD_TOL, (li, k)
                got = hd.grads_numpy()
                for k in got:
                    assert rel_fro(got[k], ref["head"][k]) <= GRAD_TOL, k
                gte, gpe = e.grads_numpy()
                assert rel_fro(gte, ref["wte"]) <= GRAD_TOL and rel_fro(gpe, ref["wpe"]) <= GRAD_TOL
            with pytest.raises(B.AxonnError):
                st.forward(0, TK[0], TK[0])                          # direct calls are refused with ends attached
    finally:
        e.close(); hd.close()


def test_first_stage_and_last_stage_separately():
    """The two special cases of Alg. 2 one at a time: a first stage (tokens in, activations out; gradients in,
    nothing out) and a last stage (activations in, loss and input gradient out at once)."""
    import torch
    sh = StageShape(2, 128, 2, 64, 1, 3)
    V, M = 264, 3
    layers, xs, dys = make_stage_inputs(sh, seed=13, perturb=True)
    tokens, targets, wte, wpe, g, bt, W = make_lm_inputs(sh, V, seed=14)
    l64 = [{k: np.asarray(v, np.float64) for k, v in p.items()} for p in layers]
    # first stage
    e = EmbedHandle(V, sh.hidden, sh.seq_len, sh.microbatch_size, wte, wpe)
    try:
        with Stage(sh) as st:
            st.load_params(layers)
            B.axonn_stage_attach_ends(st.handle, e.h, None)
            Y = [torch.zeros(sh.microbatch_size, sh.seq_len, sh.hidden, dtype=B.torch_elem_dtype(), device="cuda") for _ in range(M)]
            TK = [dev_i32(t) for t in tokens]; DY = [dev_bf16(d) for d in dys]
            st.zero_grad()
            for i in range(M):
                st.post(0, i, TK[i], Y[i])
            for i in range(M):
                st.post(1, i, DY[i], None)
            st.run(2); st.join(); torch.cuda.synchronize()
            tot_te = 0.0
            for i in range(M):
                z, caches = OT.stage_forward(OE.embedding_forward(tokens[i], wte, wpe), l64, sh.n_heads, EPS)
                assert rel_fro(host(Y[i]).reshape(z.shape), z) <= FWD_TOL
                dx, _ = OT.stage_backward(dys[i], caches, l64, sh.n_heads)
                tot_te = tot_te + OE.embedding_backward(dx, tokens[i], V, sh.seq_len)[0]
            assert rel_fro(e.grads_numpy()[0], tot_te) <= GRAD_TOL
    finally:
        e.close()
    # last stage
    hd = HeadHandle(V, sh.hidden, sh.tokens, M, g, bt, W)
    try:
        with Stage(sh) as st:
            st.load_params(layers)
            B.axonn_stage_attach_ends(st.handle, None, hd.h)
            X = [dev_bf16(x) for x in xs]
            DX = [torch.zeros_like(X[0]) for _ in range(M)]
            TG = [dev_i32(t) for t in targets]
            losses = torch.zeros(M, device="cuda")
            st.zero_grad()
            with pytest.raises(B.AxonnError):
                st.post(0, 0, X[0], DX[0])                           # targets and loss are required
            for i in range(M):
                st.post(0, i, X[i], DX[i], targets=TG[i], loss=losses[i:i + 1])
            st.run(2); st.join(); torch.cuda.synchronize()
            log = B.axonn_stage_dispatch_log(st.handle)
            assert log == [(i, k) for i in range(M) for k in (0, 1)]      # Backward follows each Forward at once
            for i in range(M):
                z, caches = OT.stage_forward(xs[i], l64, sh.n_heads, EPS)
                loss, c = OE.head_loss_forward(z, g, bt, W, targets[i], EPS, M)
                dz, _ = OE.head_loss_backward(c, g, W, targets[i], M)
                dx, _ = OT.stage_backward(dz, caches, l64, sh.n_heads)
                assert abs(losses[i].item() - loss) <= 2e-3 * abs(loss)
                assert rel_fro(host(DX[i]).reshape(dx.shape), dx) <= GRAD_TOL
    finally:
        hd.close()


@pytest.mark.parametrize("T,h,V", [(8, 8, 1), (1032, 64, 3), (2056, 8, 3000), (264, 2056, 40), (1288, 4104, 7)])
def test_embedding_table_gradient_repeats_across_windows(T, h, V):
    """Occurrences of an id further apart than one round of match masks (1024 tokens), every token the same id, rows wider
    than one pass of a workgroup: sums in token order in fp32, accumulated over two passes, unused rows untouched."""
    import torch
    rng = np.random.default_rng(T + h + V)
    e = EmbedHandle(V, h, T, 1, np.zeros((V, h), np.float32), np.zeros((T, h), np.float32))
    try:
        tot = 0.0
        for _ in range(2):
            tokens = rng.integers(0, V, (1, T))
            dx = snap_elem(rng.standard_normal((1, T, h), dtype=np.float32))
            B.axonn_embed_backward(e.h, dev_i32(tokens), dev_bf16(dx))
            torch.cuda.synchronize()
            tot = tot + OE.embedding_backward(dx, tokens, V, T)[0]
            assert rel_fro(e.grads_numpy()[0], tot) <= 6e-3     # two 16-bit roundings of an fp32 sum
    finally:
        e.close()


# (T, h, V) of a head -> parts its input gradient is split into (test_host_runtime.py checks them)
SPLIT_PARTS = {(136, 72, 4104): 4, (1032, 264, 10248): 4, (2056, 520, 20488): 4, (256, 1024, 16392): 8, (256, 1024, 2048): 1}


@pytest.mark.parametrize("T,h,V", list(SPLIT_PARTS))
def test_head_input_gradient_split_over_the_vocabulary(T, h, V):
    """The head's input gradient is long for its output (its contraction runs over the vocabulary): the parts' fp32 sums and
    their order, ragged tiles, part boundaries that are no multiple of a stage; twice, and the same bits both times."""
    import torch
    rng = np.random.default_rng(T + V)
    g, bt = np.ones(h, np.float32), np.zeros(h, np.float32)
    W = snap_elem((0.05 * rng.standard_normal((h, V))).astype(np.float32))
    hd = HeadHandle(V, h, T, 1, g, bt, W)
    try:
        x = snap_elem(rng.standard_normal((1, T, h), dtype=np.float32)); tg = rng.integers(0, V, (1, T))
        c = OE.head_loss_forward(x, g, bt, W, tg, EPS, 1)[1]
        rdx = OE.head_loss_backward(c, g, W, tg, 1)[0]
        got = []
        for _ in range(2):
            loss = torch.zeros(1, device="cuda"); dx = torch.zeros(T, h, dtype=B.torch_elem_dtype(), device="cuda")
            B.axonn_head_zero_grad(hd.h)
            B.axonn_head_forward_backward(hd.h, dev_bf16(x), dev_i32(tg), loss, dx)
            torch.cuda.synchronize()
            got.append(host(dx))
        assert rel_fro(got[0].reshape(rdx.shape), rdx) <= GRAD_TOL
        assert np.array_equal(got[0], got[1])
    finally:
        hd.close()


# the last: slots taken again while a large table's gradient is formed, which one layer's weight gradients do not hide
@pytest.mark.parametrize("sh,limit,passes,V", [(StageShape(2, 128, 2, 64, 1, 5), 5, 1, 520),
                                               (StageShape(1, 264, 2, 72, 1, 5, 1000), 4, 2, 520),
                                               (StageShape(1, 256, 4, 64, 1, 8), 4, 2, 51200)],
                         ids=["one_pass", "four_and_one", "large_table"])
@pytest.mark.parametrize("with_embed", [True, False])
def test_merged_microbatches_through_the_head(sh, limit, passes, V, with_embed):
    """Forwards and backwards of several microbatches as one pass with the head between them: losses, input gradients and the
    gradients of both ends bit for bit those of a run that takes them one by one (a done_event each)."""
    import torch
    M = sh.n_microbatches
    layers, xs, _ = make_stage_inputs(sh, seed=31, perturb=True)
    tokens, targets, wte, wpe, g, bt, W = make_lm_inputs(sh, V, seed=32)
    e = EmbedHandle(V, sh.hidden, sh.seq_len, sh.microbatch_size, wte, wpe) if with_embed else None
    hd = HeadHandle(V, sh.hidden, sh.tokens, M, g, bt, W)
    got = []
    try:
        with Stage(sh, pipeline_limit=limit) as st:
            st.load_params(layers)
            B.axonn_stage_attach_ends(st.handle, e.h if e else None, hd.h)
            X = [dev_i32(t) for t in tokens] if e else [dev_bf16(x) for x in xs]
            TG = [dev_i32(t) for t in targets]
            for events in (False, True):
                evs = [torch.cuda.Event() for _ in range(M)]
                for ev in evs:
                    ev.record()
                DX = [None if e else torch.zeros_like(X[0]) for _ in range(M)]
                losses = torch.zeros(M, device="cuda")
                torch.cuda.synchronize()
                st.zero_grad()
                for i in range(M):
                    st.post(0, i, X[i], DX[i], targets=TG[i], loss=losses[i:i + 1], done_event=evs[i] if events else None)
                made = passes_of(lambda: (st.run(2), st.join()), sh.n_layers)
                assert made == ((M, M) if events else (passes, passes)), (events, made)
                # message by message, in whatever order their kernels run
                assert B.axonn_stage_dispatch_log(st.handle) == [(i, k) for i in range(M) for k in (0, 1)]
                got.append((losses.cpu().numpy(), [None if d is None else host(d) for d in DX], st.grads_numpy(),
                            [*hd.grads_numpy().values(), *(e.grads_numpy() if e else ())]))
    finally:
        hd.close()
        if e:
            e.close()
    (la, xa, ga, ea), (lb, xb, gb, eb) = got
    assert np.array_equal(la, lb)
    assert e or all(np.array_equal(a, b) for a, b in zip(xa, xb))
    assert len(ea) == len(eb) == (5 if e else 3) and all(np.array_equal(a, b) and a.any() for a, b in zip(ea, eb))
    for p, q in zip(ga, gb):
        for k in p:
            assert rel_fro(p[k], q[k]) <= 1e-3, k          # sums over the microbatches, in another order
