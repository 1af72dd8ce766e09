"""GPU parity of the single operations against the fp64 oracle, through the C ABI.

Tolerances (relative Frobenius, derived from the arithmetic): every output is one bf16
rounding (2^-9 relative per element, ~2.3e-3 worst case, ~1.1e-3 rms) of an fp32-accumulated
value; fused epilogues add one more rounding of an intermediate.  5e-3 bounds single-op
outputs with margin and is 4x tighter than the stage-level forward bound (2e-2)."""
import itertools

import numpy as np
import pytest

import oracle
from oracle import transformer as OT
from paper_2110_13005_amd import binding as B
from paper_2110_13005_amd.inputs import snap_elem
from helpers import rel_fro, parity, dev_bf16, dev_f32, host

pytestmark = pytest.mark.gpu
TOL = 5e-3
# Element-wise bounds, in roundings of the 16-bit format (helpers.elem_factor: 2^-8 of the element's own magnitude
# plus that of a typical element of its row).
# C_ONE: an fp32-accumulated value rounded once (GEMM with any epilogue, LayerNorm): 1/2 by the arithmetic
#   (2^-9 relative), plus the fp32 summation error and, for GeLU, the 3e-7 of the erf form; 1 with margin.
# C_ATTN: the attention output sums probabilities that were rounded to 16 bits (2^-9 each, independent signs: the
#   sum over a row's keys grows like its root mean square) and is rounded once itself.
# C_ATTN_BWD: dq, dk, dv sum products of two rounded tiles (P and dS) and go through one more rounding; delta comes
#   from the rounded o.  Measured worst over the shapes below: 0.86 (one rounding), 2.2 (attention), 7.9 (its backward).
C_ONE, C_ATTN, C_ATTN_BWD = 1.0, 4.0, 16.0


def _rng_bf16(rng, shape, std=1.0):
    return snap_elem((rng.standard_normal(shape) * std).astype(np.float32))


# ------------------------------------------------------------------------- GEMM
GEMM_SHAPES = [
    # ring kernel, tiles of 64 x 64 but for the third (the large-problem kernels run all of these in
    # test_gemm_both_large_kernels_all_layouts_and_results)
    (256, 256, 64),      # one k-step
    (512, 768, 256),     # several tiles
    (2048, 4096, 512),   # tiles of 128 x 256, an even number of them per XCD
    (200, 136, 72),      # ragged in every dimension (multiples of 8 only)
    (8, 8, 8),           # degenerate minimum
    (264, 2056, 1032),   # ragged tails on a multi-tile problem
    # large-problem kernels, ragged rows and columns, k tail, odd number of k-tiles; the launcher picks
    # block widths 160, 192 and 256 for these three
    (2056, 4104, 264),
    (2056, 4512, 264),
    (2056, 5464, 264),
    (4096, 2048, 448),   # ring kernel, 128 x 256: odd number of k-tiles, no tail
    # whole k-tiles (the kernel that copies tiles without staging registers), ragged rows and columns,
    # block widths 160, 192 and 256
    (2056, 4104, 320),
    (2056, 4512, 320),
    (2056, 5464, 320),
    (4096, 4096, 64),    # a single k-tile: the second stage holds a tile of zeros
]


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_forward_layout_bias_res_gelu(M, N, K):
    import torch
    rng = np.random.default_rng(M + N + K)
    x = _rng_bf16(rng, (M, K)); w = _rng_bf16(rng, (K, N), 0.05); bias = _rng_bf16(rng, (N,), 0.5)
    res = _rng_bf16(rng, (M, N))
    ref = x.astype(np.float64) @ w.astype(np.float64) + bias
    dx, dw, db, dr = dev_bf16(x), dev_bf16(w), dev_bf16(bias), dev_bf16(res)
    out = torch.empty(M, N, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS, M, N, K, dx, K, dw, N, out, N, bias=db)
    parity(host(out), ref, TOL, C_ONE, label="gemm_forward_layout_bias_res_gelu")
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS, M, N, K, dx, K, dw, N, out, N, bias=None)
    parity(host(out), ref - bias, TOL, C_ONE, label="gemm_forward_layout_bias_res_gelu")
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS_RES, M, N, K, dx, K, dw, N, out, N, bias=db, res=dr, ld_res=N)
    parity(host(out), ref + res, TOL, C_ONE, label="gemm_forward_layout_bias_res_gelu")
    pre = torch.empty(M, N, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS_GELU, M, N, K, dx, K, dw, N, out, N, bias=db, aux=pre, ld_aux=N)
    torch.cuda.synchronize()
    assert rel_fro(host(pre), OT.gelu_grad(ref)) < TOL      # the epilogue stores GeLU'(z) in place of z
    parity(host(out), OT.gelu(ref), TOL, C_ONE, label="gemm_forward_layout_bias_res_gelu")


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_dgrad_layout_plain_and_dgelu(M, N, K):
    """dx = dy W^T: A [M,K] k-contiguous, B = W stored [N,K] (rows n, k contiguous)."""
    import torch
    rng = np.random.default_rng(M * 3 + N + K)
    dy = _rng_bf16(rng, (M, K)); w = _rng_bf16(rng, (N, K), 0.05); pre = _rng_bf16(rng, (M, N))
    ref = dy.astype(np.float64) @ w.astype(np.float64).T
    a, b, p = dev_bf16(dy), dev_bf16(w), dev_bf16(pre)
    out = torch.empty(M, N, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_bf16(1, 1, B.EPI_BIAS, M, N, K, a, K, b, K, out, N)
    parity(host(out), ref, TOL, C_ONE, label="gemm_dgrad_layout_plain_and_dgelu")
    B.axonn_gemm_bf16(1, 1, B.EPI_DGELU, M, N, K, a, K, b, K, out, N, aux=p, ld_aux=N)
    assert rel_fro(host(out), ref * pre.astype(np.float64)) < TOL       # aux holds the stored derivative


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_wgrad_layout_accumulate(M, N, K):
    """dW = x^T dy: A = x stored [K,M], B = dy stored [K,N]; fp32 and bf16 accumulators."""
    import torch
    rng = np.random.default_rng(M + N * 5 + K)
    x = _rng_bf16(rng, (K, M)); dy = _rng_bf16(rng, (K, N))
    ref = x.astype(np.float64).T @ dy.astype(np.float64)
    a, b = dev_bf16(x), dev_bf16(dy)
    c32 = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    B.axonn_gemm_bf16(0, 0, B.EPI_ACC_F32, M, N, K, a, M, b, N, c32, N, accumulate=0)   # overwrite
    assert rel_fro(host(c32), ref) < 1e-5
    B.axonn_gemm_bf16(0, 0, B.EPI_ACC_F32, M, N, K, a, M, b, N, c32, N, accumulate=1)
    assert rel_fro(host(c32), 2 * ref) < 1e-5
    c16 = torch.full((M, N), 7.0, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_bf16(0, 0, B.EPI_ACC_BF16, M, N, K, a, M, b, N, c16, N, accumulate=0)
    first = host(c16)
    parity(first, ref, TOL, C_ONE, label="gemm_wgrad_layout_accumulate")
    B.axonn_gemm_bf16(0, 0, B.EPI_ACC_BF16, M, N, K, a, M, b, N, c16, N, accumulate=1)
    parity(host(c16), first + ref, TOL, C_ONE, label="gemm_wgrad_layout_accumulate")


@pytest.mark.parametrize("M,N,K", GEMM_SHAPES)
def test_gemm_wgrad_with_bias_gradient(M, N, K):
    """dW = x^T dy and db = the column sums of dy from one call (formed from the tiles of dy that the kernel
    multiplies): stored, then accumulated, in fp32 and
    in 16-bit accumulators; dy with a leading dimension beyond N, whose padding must stay out of the sums."""
    import torch
    rng = np.random.default_rng(M + N * 7 + K)
    ldb = N + 24
    x = _rng_bf16(rng, (K, M)); dybuf = _rng_bf16(rng, (K, ldb)); dy = dybuf[:, :N]
    ref = x.astype(np.float64).T @ dy.astype(np.float64)
    ref_db = dy.astype(np.float64).sum(axis=0)
    bound32 = 1e-5 * np.abs(dy.astype(np.float64)).sum(axis=0) + 1e-30     # fp32 summation of K terms
    a, b = dev_bf16(x), dev_bf16(dybuf)
    ws = torch.empty(((K + 63) // 64) * N, dtype=torch.float32, device="cuda")
    c32 = torch.full((M, N), 7.0, dtype=torch.float32, device="cuda")
    db32 = torch.full((N + 8,), 3.0, dtype=torch.float32, device="cuda")
    B.axonn_gemm_wgrad_colsum(B.EPI_ACC_F32, M, N, K, a, M, b, ldb, c32, N, db32, ws, accumulate=0)   # overwrite
    assert rel_fro(host(c32), ref) < 1e-5
    assert (np.abs(host(db32)[:N] - ref_db) <= bound32).all()
    B.axonn_gemm_wgrad_colsum(B.EPI_ACC_F32, M, N, K, a, M, b, ldb, c32, N, db32, ws, accumulate=1)
    assert rel_fro(host(c32), 2 * ref) < 1e-5
    assert (np.abs(host(db32)[:N] - 2 * ref_db) <= 2 * bound32).all()
    assert (host(db32)[N:] == 3.0).all()                                   # nothing written past column N
    c16 = torch.full((M, N), 7.0, dtype=B.torch_elem_dtype(), device="cuda")
    db16 = torch.full((N + 8,), 3.0, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_wgrad_colsum(B.EPI_ACC_BF16, M, N, K, a, M, b, ldb, c16, N, db16, ws, accumulate=0)
    first, first_db = host(c16), host(db16)[:N]
    parity(first, ref, TOL, C_ONE, label="gemm_wgrad_with_bias_gradient")
    parity(first_db, ref_db, TOL, C_ONE, label="gemm_wgrad_with_bias_gradient")
    B.axonn_gemm_wgrad_colsum(B.EPI_ACC_BF16, M, N, K, a, M, b, ldb, c16, N, db16, ws, accumulate=1)
    parity(host(c16), first + ref, TOL, C_ONE, label="gemm_wgrad_with_bias_gradient")
    parity(host(db16)[:N], first_db + ref_db, TOL, C_ONE, label="gemm_wgrad_with_bias_gradient")
    assert (host(db16)[N:] == 3.0).all()


# Problems for every tile size of the ring kernel (below the threshold of the large-problem kernels the launcher picks the
# one with the lowest modelled time; test_host_runtime.py checks that it still picks these): ragged rows and columns, a k
# tail, k ranges shorter than the ring and longer.
RING_TILES = {
    (72, 136, 40): "64x64",        # one k-tile with a tail, the rest of the ring beyond the end
    (1000, 1016, 456): "64x64",    # 8 k-tiles, the last one short
    (2040, 1016, 520): "128x64",
    (2008, 2040, 328): "128x128",  # an even number of k-steps, 1032 an odd one
    (1032, 3080, 1032): "128x128", # and the columns of a ninth half-empty tile row
    (2040, 3064, 200): "128x192",  # partial results added in place
    (2040, 4088, 264): "128x256",
}
RING_SHAPES = list(RING_TILES)


@pytest.mark.parametrize("M,N,K", RING_SHAPES)
def test_gemm_ring_tiles(M, N, K):
    test_gemm_forward_layout_bias_res_gelu(M, N, K)
    test_gemm_dgrad_layout_plain_and_dgelu(M, N, K)
    test_gemm_wgrad_layout_accumulate(M, N, K)
    test_gemm_wgrad_with_bias_gradient(M, N, K)


def test_gemm_big_tile_strided_operands():
    """Leading dimensions larger than the logical widths and a k tail, on the ring kernel (128 x 256) and, for the third
    problem and wherever axonn_tuning asks for them, the large-problem kernels: what lies beyond K in a row of a
    k-contiguous operand must not enter the sum."""
    import torch
    rng = np.random.default_rng(6)
    for (M, N, K), (a_kc, b_kc, epi) in itertools.product(
            ((2048, 4096, 200), (2048, 4096, 192), (4096, 4104, 200)),
            ((1, 0, B.EPI_BIAS), (1, 1, B.EPI_BIAS), (0, 0, B.EPI_ACC_BF16))):
        ash, bsh = ((M, K) if a_kc else (K, M)), ((N, K) if b_kc else (K, N))
        lda, ldb, ldc = ash[1] + 72, bsh[1] + 136, N + 8
        abuf = _rng_bf16(rng, (ash[0], lda)); bbuf = _rng_bf16(rng, (bsh[0], ldb), 0.05)
        am, bm = abuf[:, :ash[1]].astype(np.float64), bbuf[:, :bsh[1]].astype(np.float64)
        ref = (am if a_kc else am.T) @ (bm.T if b_kc else bm)
        out = torch.zeros(M, ldc, dtype=B.torch_elem_dtype(), device="cuda")
        B.axonn_gemm_bf16(a_kc, b_kc, epi, M, N, K, dev_bf16(abuf), lda, dev_bf16(bbuf), ldb, out, ldc)
        parity(host(out)[:, :N], ref, TOL, C_ONE, label="gemm_big_tile_strided_operands")
        assert not host(out)[:, N:].any()


@pytest.mark.parametrize("mask,min_tiles", [(15, 1), (0, 1), (15, -1)])
def test_gemm_both_large_kernels_all_layouts_and_results(mask, min_tiles):
    """The large-problem kernel whose tiles are copied by the memory pipeline serves all four (layout, result type) classes
    by default, the register-staged one the fourth where operands are not aligned; axonn_tuning fixes the choice, so every GEMM
    case of this file runs again through the copying kernel (mask 15; its variant with a short last k-tile where K
    is no multiple of 64) and through the register-staged kernel everywhere (mask 0), with the threshold lowered so that the small ragged
    shapes reach the large-problem kernels too (all three block widths)."""
    try:
        B.axonn_tuning(B.TUNE_GEMM_COPY_MASK, mask)
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, min_tiles)
        for width in ((-1,) if min_tiles < 0 else (-1, 160, 192)):
            B.axonn_tuning(B.TUNE_GEMM_TILE_N, width)
            for (M, N, K) in GEMM_SHAPES:
                if width > 0 and M * N > 2048 * 4096:
                    continue                          # the forced widths on the small and the ragged shapes only
                test_gemm_forward_layout_bias_res_gelu(M, N, K)
                test_gemm_dgrad_layout_plain_and_dgelu(M, N, K)
                test_gemm_wgrad_layout_accumulate(M, N, K)
                test_gemm_wgrad_with_bias_gradient(M, N, K)
        B.axonn_tuning(B.TUNE_GEMM_TILE_N, -1)
        test_gemm_big_tile_strided_operands()
        test_gemm_strided_operands_and_run_to_run_determinism()
    finally:
        for knob in (B.TUNE_GEMM_COPY_MASK, B.TUNE_GEMM_BIG_MIN_TILES, B.TUNE_GEMM_TILE_N):
            B.axonn_tuning(knob, -1)
    with pytest.raises(B.AxonnError):
        B.axonn_tuning(B.TUNE_GEMM_TILE_N, 128)
    with pytest.raises(B.AxonnError):
        B.axonn_tuning(7, 0)


def test_gelu_of_every_value_does_not_depend_on_the_kernel():
    """GeLU and GeLU' of every finite 16-bit number (as bias under a product of zeros), from each tile of the ring kernel, in
    this order, and both large-problem kernels: the same bits in every row of every launch."""
    import torch
    bits = torch.arange(1 << 16, dtype=torch.int32).to(torch.int16).cuda()
    values = bits.view(B.torch_elem_dtype())
    values = values[torch.isfinite(values)]
    seen = []
    try:
        for M, N, min_tiles, mask in ((64, 2048, 1 << 20, -1), (1024, 2048, 1 << 20, -1), (1536, 2048, 1 << 20, -1),
                                      (2048, 3072, 1 << 20, -1), (2048, 4096, 1 << 20, -1), (64, 2048, 1, 15), (64, 2048, 1, 0)):
            B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, min_tiles)
            B.axonn_tuning(B.TUNE_GEMM_COPY_MASK, mask)
            K = 64
            a, w = (torch.zeros(n, dtype=values.dtype, device="cuda") for n in (M * K, K * N))
            got = []
            for first in range(0, len(values), N):
                bias = torch.zeros(N, dtype=values.dtype, device="cuda")
                piece = values[first:first + N]
                bias[:len(piece)] = piece
                y, aux = (torch.zeros(M, N, dtype=values.dtype, device="cuda") for _ in range(2))
                B.axonn_gemm_bf16(1, 0, B.EPI_BIAS_GELU, M, N, K, a, K, w, N, y, N, bias=bias, aux=aux, ld_aux=N)
                both = torch.stack([y, aux]).view(torch.int16)[:, :, :len(piece)]
                assert bool((both == both[:, :1]).all()), (M, N, first)
                got.append(both[:, 0])
            seen.append(torch.cat(got, dim=1))
    finally:
        for knob in (B.TUNE_GEMM_COPY_MASK, B.TUNE_GEMM_BIG_MIN_TILES):
            B.axonn_tuning(knob, -1)
    for other in seen[1:]:
        assert torch.equal(seen[0], other)


def _wide(rows, width, ld, offset=0):
    """rows x width random elements with leading dimension ld, `offset` elements into a buffer that is NaN elsewhere near
    them -> (values, tensor that starts at the first element)."""
    import torch
    buf = torch.zeros(rows * ld + offset, dtype=B.torch_elem_dtype(), device="cuda")
    view = buf[offset:].view(rows, ld)
    view[:, width:min(ld, width + 256)] = float("nan")
    vals = _rng_bf16(np.random.default_rng(rows + width), (rows, width))
    view[:, :width] = dev_bf16(vals)
    return vals.astype(np.float64), buf[offset:]


@pytest.mark.parametrize("M,N,K", [(4000, 1544, 72), (8000, 1544, 72), (3976, 1800, 136), (1544, 4000, 72), (7944, 2312, 136)])
def test_gemm_tiles_of_128_x_256_in_narrow_bands(M, N, K):
    """More rows of these tiles than columns: the walk goes in bands of 4 tile columns, the last of 1 to 3 (and, the fourth,
    fewer rows than columns)."""
    import torch
    rng = np.random.default_rng(M + N)
    a, w = _rng_bf16(rng, (M, K)), _rng_bf16(rng, (K, N), 0.05)
    try:
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, 1 << 20)
        out = torch.zeros(M, N, dtype=B.torch_elem_dtype(), device="cuda")
        B.axonn_gemm_bf16(1, 0, B.EPI_BIAS, M, N, K, dev_bf16(a), K, dev_bf16(w), N, out, N)
    finally:
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, -1)
    parity(host(out), a.astype(np.float64) @ w.astype(np.float64), TOL, C_ONE, label="gemm_tiles_of_128_x_256_in_narrow_bands")


@pytest.mark.parametrize("off", [0, 4])
def test_gemm_large_fp32_weight_gradient_by_alignment(off):
    """Large weight gradients with an fp32 result: operands at a multiple of 16 bytes take the copying kernel, others the
    register-staged one; stored and added."""
    import torch
    M, N, K = 4096, 4104, 72
    am, a = _wide(K, M, M + 8, off)
    bm, b = _wide(K, N, N + 8, off)
    ref = am.T @ bm
    out = torch.full((M, N), 7.0, device="cuda")
    for acc in (0, 1):
        B.axonn_gemm_bf16(0, 0, B.EPI_ACC_F32, M, N, K, a, M + 8, b, N + 8, out, N, accumulate=acc)
        assert rel_fro(host(out), (1 + acc) * ref) <= 1e-5        # products are exact, 72 fp32 additions


@pytest.mark.parametrize("min_tiles", [-1, 1])
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (136, 264, 200), (264, 136, 72)])
@pytest.mark.parametrize("wide", ["A", "B", "misaligned"])
def test_gemm_operands_of_the_pointer_kernel(M, N, K, wide, min_tiles):
    """Operands that 32-bit byte offsets do not span (a leading dimension of 2^20) and, for small problems, operands that
    do not start at a multiple of 16 bytes: tiles of 128 x 128, or of 256 x 256 above the threshold, all layouts, the
    column sums in launches of their own where an operand is too large."""
    import torch
    off = 4 if wide == "misaligned" else 0
    lda_of = lambda w: 1 << 20 if wide == "A" else w + 8
    ldb_of = lambda w: 1 << 20 if wide == "B" else w + 8
    ws = torch.empty(((K + 63) // 64) * N, dtype=torch.float32, device="cuda")
    try:
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, min_tiles if not off else -1)
        for a_kc, b_kc, epi in ((1, 0, B.EPI_BIAS), (1, 1, B.EPI_BIAS), (0, 0, B.EPI_ACC_F32), (0, 0, B.EPI_ACC_BF16)):
            ash, bsh = ((M, K) if a_kc else (K, M)), ((N, K) if b_kc else (K, N))
            lda, ldb = lda_of(ash[1]), ldb_of(bsh[1])
            am, a = _wide(*ash, lda, off)
            bm, b = _wide(*bsh, ldb, off)
            ref = (am if a_kc else am.T) @ (bm.T if b_kc else bm)
            if a_kc:
                out = torch.zeros(M, N, dtype=B.torch_elem_dtype(), device="cuda")
                B.axonn_gemm_bf16(a_kc, b_kc, epi, M, N, K, a, lda, b, ldb, out, N)
                parity(host(out), ref, TOL, C_ONE, label="gemm_operands_of_the_pointer_kernel")
                continue
            f32 = epi == B.EPI_ACC_F32
            out = torch.full((M, N), 7.0, dtype=torch.float32 if f32 else B.torch_elem_dtype(), device="cuda")
            db = torch.full((N + 8,), 3.0, dtype=out.dtype, device="cuda")
            for acc in (0, 1):
                B.axonn_gemm_wgrad_colsum(epi, M, N, K, a, lda, b, ldb, out, N, db, ws, accumulate=acc)
            # stored, then added to what was stored: each step one 16-bit rounding, or fp32 sums
            assert rel_fro(host(out), 2 * ref) < (1e-5 if f32 else TOL)
            assert rel_fro(host(db)[:N], 2 * bm.sum(axis=0)) < (1e-5 if f32 else TOL)
            assert (host(db)[N:] == 3.0).all()
    finally:
        B.axonn_tuning(B.TUNE_GEMM_BIG_MIN_TILES, -1)


def test_gemm_strided_operands_and_run_to_run_determinism():
    """Leading dimensions larger than the logical width (the qkv weight-gradient uses slices)."""
    import torch
    rng = np.random.default_rng(5)
    M, N, K, lda, ldb, ldc = 136, 264, 520, 600, 320, 400
    abuf = _rng_bf16(rng, (M, lda)); bbuf = _rng_bf16(rng, (K, ldb), 0.05)
    ref = abuf[:, :K].astype(np.float64) @ bbuf[:, :N].astype(np.float64)
    a, b = dev_bf16(abuf), dev_bf16(bbuf)
    out = torch.zeros(M, ldc, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS, M, N, K, a, lda, b, ldb, out, ldc)
    first = out.clone()
    parity(host(out)[:, :N], ref, TOL, C_ONE, label="gemm_strided_operands_and_run_to_run_determinism")
    assert not host(out)[:, N:].any()                     # nothing written outside the tile
    B.axonn_gemm_bf16(1, 0, B.EPI_BIAS, M, N, K, a, lda, b, ldb, out, ldc)
    torch.cuda.synchronize()
    assert torch.equal(first, out)


# -------------------------------------------------------------------- LayerNorm
@pytest.mark.parametrize("T,h", [(256, 256), (77, 5120), (8, 8), (300, 10240), (64, 1000)])
def test_layernorm_fwd_bwd(T, h):
    import torch
    rng = np.random.default_rng(T + h)
    x = _rng_bf16(rng, (T, h), 2.0) + snap_elem(np.float32(0.5))
    x = snap_elem(x)
    g = _rng_bf16(rng, (h,), 0.2) + 1; g = snap_elem(g)
    bta = _rng_bf16(rng, (h,), 0.2)
    dout = _rng_bf16(rng, (T, h)); resg = _rng_bf16(rng, (T, h))
    eps = 1e-5
    ref, xhat, rstd = OT.layernorm_fwd(x, g.astype(np.float64), bta.astype(np.float64), eps)
    dxr, dgr, dbr = OT.layernorm_bwd(dout.astype(np.float64), xhat, rstd, g.astype(np.float64))
    X, G, Bt, DO, RG = dev_bf16(x), dev_bf16(g), dev_bf16(bta), dev_bf16(dout), dev_bf16(resg)
    out = torch.empty(T, h, dtype=B.torch_elem_dtype(), device="cuda")
    stats = torch.empty(T, 2, dtype=torch.float32, device="cuda")
    B.axonn_layernorm_fwd(T, h, X, G, Bt, eps, out, stats)
    parity(host(out), ref, TOL, C_ONE, label="layernorm_fwd_bwd")
    st = host(stats)
    assert rel_fro(st[:, 0], x.astype(np.float64).mean(-1)) < 1e-4 or np.abs(st[:, 0] - x.mean(-1)).max() < 1e-5
    assert rel_fro(st[:, 1], rstd[:, 0]) < 1e-5
    dx = torch.empty(T, h, dtype=B.torch_elem_dtype(), device="cuda")
    dg = torch.empty(h, dtype=torch.float32, device="cuda")
    db = torch.empty(h, dtype=torch.float32, device="cuda")
    ws = torch.empty(2 * ((T + 63) // 64) * h, dtype=torch.float32, device="cuda")
    B.axonn_layernorm_bwd(T, h, DO, X, stats, G, RG, dx, dg, db, ws)
    parity(host(dx), dxr + resg, TOL, C_ONE, label="layernorm_fwd_bwd")
    assert rel_fro(host(dg), dgr) < 1e-4
    assert rel_fro(host(db), dbr) < 1e-4
    B.axonn_layernorm_bwd(T, h, DO, X, stats, G, None, dx, dg, db, ws)
    parity(host(dx), dxr, TOL, C_ONE, label="layernorm_fwd_bwd")


def test_layernorm_constant_row_gives_beta():
    import torch
    T, h = 8, 512
    x = np.full((T, h), 3.0, np.float32)
    g = snap_elem(np.linspace(0.5, 1.5, h).astype(np.float32)); bta = snap_elem(np.linspace(-1, 1, h).astype(np.float32))
    out = torch.empty(T, h, dtype=B.torch_elem_dtype(), device="cuda")
    stats = torch.empty(T, 2, dtype=torch.float32, device="cuda")
    B.axonn_layernorm_fwd(T, h, dev_bf16(x), dev_bf16(g), dev_bf16(bta), 1e-5, out, stats)
    assert np.array_equal(host(out), np.broadcast_to(bta.astype(np.float64), (T, h)))


@pytest.mark.parametrize("T,N,ld", [(256, 768, 768), (100, 520, 1024), (8, 8, 8), (2048, 1024, 1024)])
def test_colsum(T, N, ld):
    import torch
    rng = np.random.default_rng(T + N)
    y = _rng_bf16(rng, (T, ld))
    out = torch.empty(N, dtype=torch.float32, device="cuda")
    ws = torch.empty(((T + 63) // 64) * N, dtype=torch.float32, device="cuda")
    B.axonn_colsum(T, N, dev_bf16(y), ld, out, ws)
    assert rel_fro(host(out), y[:, :N].astype(np.float64).sum(0)) < 1e-5


# -------------------------------------------------------------------- attention
ATTN_SHAPES = [
    (2, 128, 4, 64),    # tiny-config shape
    (1, 256, 2, 128),   # two query tiles, head dim 128
    (1, 200, 3, 128),   # ragged sequence (not a multiple of any tile)
    (2, 72, 2, 64),     # shorter than one tile
    (1, 8, 1, 64),      # minimum
    (1, 520, 2, 128),   # several tiles + ragged tail
    # head dimensions without a kernel of their own: multiples of 4 up to 192, run with masked columns
    (1, 200, 2, 188),   # the paper's Table 1 head dimension (h = 4512, 24 heads), on the 192 kernel
    (1, 264, 2, 176),   # Table 1: 6336 / 36
    (1, 300, 4, 136),   # Table 1: 6528 / 48
    (1, 520, 2, 156),   # Table 1: 9360 / 60
    (2, 136, 2, 44),    # on the 64 kernel, half of a 16-byte chunk at the end of every head
    # long enough for the tiles below the diagonal, which the backward kernels process in pairs of blocks
    (1, 520, 2, 64),
    (1, 400, 2, 100),   # on the 128 kernel with masked columns
    (1, 400, 2, 44),    # on the 64 kernel with masked columns
    (1, 300, 4, 100),   # on the 128 kernel
    (1, 96, 2, 32),     # less than the smallest kernel
    (1, 130, 6, 36),
    (1, 64, 2, 4),      # minimum: one 8-byte half chunk per head
    (1, 100, 2, 192),   # exactly the largest compiled size
]


def _attn_ref(qkv, dout, b, s, a, d):
    h = a * d
    q3 = qkv.astype(np.float64).reshape(b, s, 3 * h)
    q, k, v = q3[..., :h], q3[..., h:2 * h], q3[..., 2 * h:]
    o, P = OT.causal_attention_fwd(q, k, v, a)
    dq, dk, dv = OT.causal_attention_bwd(dout.astype(np.float64).reshape(b, s, h), q, k, v, P, a)
    # lse from the definition (log of the masked sum of exp scores)
    qh = q.reshape(b, s, a, d).transpose(0, 2, 1, 3); kh = k.reshape(b, s, a, d).transpose(0, 2, 1, 3)
    S = qh @ kh.transpose(0, 1, 3, 2) / np.sqrt(d)
    S = np.where(np.tril(np.ones((s, s), bool)), S, -np.inf)
    mx = S.max(-1, keepdims=True)
    lse = (mx + np.log(np.exp(S - mx).sum(-1, keepdims=True)))[..., 0]
    return o.reshape(b * s, h), lse, np.concatenate([dq, dk, dv], -1).reshape(b * s, 3 * h)


@pytest.mark.parametrize("b,s,a,d", ATTN_SHAPES)
def test_attention_fwd_bwd(b, s, a, d):
    import torch
    rng = np.random.default_rng(b * 1000 + s + a + d)
    h = a * d
    qkv = _rng_bf16(rng, (b * s, 3 * h)); dout = _rng_bf16(rng, (b * s, h))
    o_ref, lse_ref, dqkv_ref = _attn_ref(qkv, dout, b, s, a, d)
    QKV, DO = dev_bf16(qkv), dev_bf16(dout)
    o = torch.zeros(b * s, h, dtype=B.torch_elem_dtype(), device="cuda")
    lse = torch.zeros(b, a, s, dtype=torch.float32, device="cuda")
    B.axonn_attention_fwd(b, s, a, d, QKV, o, lse)
    parity(host(o), o_ref, TOL, C_ATTN, label="attention_fwd_bwd")
    assert np.abs(host(lse) - lse_ref).max() < 2e-3
    dqkv = torch.zeros(b * s, 3 * h, dtype=B.torch_elem_dtype(), device="cuda")
    delta = torch.zeros(b * a * s, dtype=torch.float32, device="cuda")
    B.axonn_attention_bwd(b, s, a, d, QKV, o, lse, DO, dqkv, delta)
    got = host(dqkv)
    # backward consumes the GPU's own bf16 o (one extra rounding in delta): 2x the single-op bound
    for name, sl in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
        parity(got[:, sl], dqkv_ref[:, sl], 2 * TOL, C_ATTN_BWD, label="attention_fwd_bwd_bwd")
    # first token attends only to itself: its output is its value row (bit exact)
    v0 = qkv.reshape(b, s, 3 * h)[:, 0, 2 * h:]
    assert np.array_equal(host(o).reshape(b, s, h)[:, 0], v0.astype(np.float64))


@pytest.mark.parametrize("b,s,a,d", [(2, 200, 32, 64), (2, 200, 33, 64), (1, 264, 44, 128), (3, 130, 22, 44), (1, 130, 66, 188)])
def test_attention_around_the_one_launch_backward(b, s, a, d):
    """Up to 128 tiles of 128 rows the backward runs as one launch for dQ, dK and dV, beyond as two: 128 tiles, and 130 to 132
    with exact and masked head dimensions."""
    test_attention_fwd_bwd(b, s, a, d)


@pytest.mark.parametrize("b,s,a,d", [(1, 200, 2, 64), (2, 136, 33, 128), (1, 72, 4, 44), (1, 264, 2, 188), (1, 130, 66, 124)])
def test_attention_of_matrices_that_are_not_16_byte_aligned(b, s, a, d):
    """Such tiles go through registers instead of the memory pipeline's copies; the arithmetic is the same, so are the bits."""
    import torch
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)
    qkv, dout = (torch.randn(b * s, n, generator=g, device="cuda").to(dt) for n in (3 * h, h))

    def shifted(t, by):
        buf = torch.zeros(t.numel() + 8, dtype=dt, device="cuda")
        buf[by:by + t.numel()] = t.flatten()
        return buf[by:by + t.numel()].view(t.shape)

    def run(by):
        q, do = shifted(qkv, by), shifted(dout, by)
        o, dq = torch.zeros(b * s, h, dtype=dt, device="cuda"), torch.zeros(b * s, 3 * h, dtype=dt, device="cuda")
        lse, ws = (torch.zeros(b, a, s, device="cuda") for _ in range(2))
        B.axonn_attention_fwd(b, s, a, d, q, o, lse)
        B.axonn_attention_bwd(b, s, a, d, q, o, lse, do, dq, ws)
        return o, lse, dq

    for x, y in zip(run(0), run(4)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("s,a,d", [(200, 4, 44), (130, 2, 188), (72, 4, 124), (72, 4, 60)])
def test_attention_head_is_not_reached_by_its_neighbours(s, a, d):
    """Heads of an odd multiple of 4 columns share 16-byte chunks: what the neighbours hold there, infinities and NaN included,
    stays out of a head's results."""
    import torch
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)
    qkv, dout = (torch.randn(s, n, generator=g, device="cuda").to(dt) for n in (3 * h, h))

    def run(q, do):
        o, dq = torch.zeros(s, h, dtype=dt, device="cuda"), torch.zeros(s, 3 * h, dtype=dt, device="cuda")
        lse, ws = (torch.zeros(1, a, s, device="cuda") for _ in range(2))
        B.axonn_attention_fwd(1, s, a, d, q, o, lse)
        B.axonn_attention_bwd(1, s, a, d, q, o, lse, do, dq, ws)
        return torch.cat([o.view(s, 1, a, d), dq.view(s, 3, a, d)], 1)

    clean = run(qkv, dout)
    assert torch.isfinite(clean.float()).all()
    for head in range(a):
        others = [x for x in range(a) if x != head]
        q, do = qkv.clone(), dout.clone()
        q.view(s, 3, a, d)[:, :, others] = float("nan")
        do.view(s, a, d)[:, others] = float("inf")
        assert torch.equal(run(q, do)[:, :, head], clean[:, :, head])


@pytest.mark.parametrize("by", [1, 2, 6])
@pytest.mark.parametrize("b,s,a,d", [(1, 200, 2, 64), (2, 136, 33, 128), (1, 72, 4, 44), (1, 264, 2, 188), (1, 130, 66, 124)])
def test_attention_of_matrices_at_any_element(b, s, a, d, by):
    """Matrices start at any element: the copies into LDS take their addresses as they are.  The bits are the same."""
    import torch
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)
    data = [torch.randn(b * s * n, generator=g, device="cuda").to(dt) for n in (3 * h, h)]

    def run(by):
        q, do = (torch.full((x.numel() + by,), float("nan"), dtype=dt, device="cuda")[by:].copy_(x) for x in data)
        o, dq = torch.zeros(b * s, h, dtype=dt, device="cuda"), torch.zeros(b * s, 3 * h, dtype=dt, device="cuda")
        lse, ws = (torch.zeros(b, a, s, device="cuda") for _ in range(2))
        B.axonn_attention_fwd(b, s, a, d, q, o, lse)
        B.axonn_attention_bwd(b, s, a, d, q, o, lse, do, dq, ws)
        return o, lse, dq

    for x, y in zip(run(0), run(by)):
        assert torch.equal(x, y)


@pytest.mark.parametrize("by", [1, 2, 4])
@pytest.mark.parametrize("b,s,a,d", [(2, 130, 2, 188), (2, 72, 4, 44), (3, 33, 2, 64), (2, 200, 34, 128)])
def test_attention_results_at_any_element(b, s, a, d, by):
    """Results go to any element, and nothing is written in front of them or behind: their descriptors end with the last row's last
    column, and one sequence's rows end where the next one's begin."""
    import torch
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)
    qkv, dout = (torch.randn(b * s, n, generator=g, device="cuda").to(dt) for n in (3 * h, h))
    lse, ws = (torch.zeros(b, a, s, device="cuda") for _ in range(2))

    def run(by, guard=64):
        bufs = [torch.full((guard + by + b * s * n + guard,), 7.0, dtype=dt, device="cuda") for n in (h, 3 * h)]
        o, dq = (x[guard + by:guard + by + b * s * n] for x, n in zip(bufs, (h, 3 * h)))
        B.axonn_attention_fwd(b, s, a, d, qkv, o, lse)
        B.axonn_attention_bwd(b, s, a, d, qkv, o, lse, dout, dq, ws)
        for x in bufs:
            assert (x[:guard + by] == 7).all() and (x[-guard:] == 7).all()
        return o, dq

    whole = run(0)
    for x, y in zip(whole, run(by)):
        assert torch.equal(x, y)
    for i in range(b):
        o = torch.zeros(s * h, dtype=dt, device="cuda")
        B.axonn_attention_fwd(1, s, a, d, qkv[i * s:(i + 1) * s], o, lse)
        assert torch.equal(o, whole[0].view(b, -1)[i])


@pytest.mark.parametrize("d", [188, 64])
def test_attention_rows_beyond_32_bit_offsets(d):
    """128 rows of q, k and v longer than 2^31 bytes go through registers: the bits of a few heads by themselves."""
    import torch
    s, dt = 37, B.torch_elem_dtype()
    a = 2 * ((1 << 31) // (128 * 3 * 2 * 2 * d) + 1)
    h = a * d
    assert 128 * 3 * h * 2 >= 1 << 31
    g = torch.Generator(device="cuda"); g.manual_seed(d)
    pick = [0, 1, 77, a // 2, a - 2, a - 1]
    few = [torch.randn(s, n, len(pick), d, generator=g, device="cuda").to(dt) for n in (3, 1)]
    many = [torch.ones(s, n, a, d, dtype=dt, device="cuda") for n in (3, 1)]
    for x, y in zip(many, few):
        x[:, :, pick] = y

    def run(q, do, a):
        o, dq = torch.zeros(s, 1, a, d, dtype=dt, device="cuda"), torch.zeros(s, 3, a, d, dtype=dt, device="cuda")
        lse, ws = (torch.zeros(a, s, device="cuda") for _ in range(2))
        B.axonn_attention_fwd(1, s, a, d, q, o, lse)
        B.axonn_attention_bwd(1, s, a, d, q, o, lse, do, dq, ws)
        return o, lse, dq

    o, lse, dq = run(*few, len(pick))
    mo, mlse, mdq = run(*many, a)
    assert torch.equal(mo[:, :, pick], o) and torch.equal(mlse[pick], lse)
    # more than 128 tiles: where the dQ kernel forms delta (64 columns), its sums are in the other order
    e = torch.linalg.norm((mdq[:, :, pick].float() - dq.float()).double()) / torch.linalg.norm(dq.double())
    assert e <= (0 if d == 188 else 2.0 ** (-8 if dt == torch.bfloat16 else -11))


@pytest.mark.parametrize("by", [4, 1])
def test_attention_of_unaligned_matrices_takes_no_longer(by):
    """16 heads of 128 x 2048 at a multiple of 16 bytes and elsewhere: up to a third longer at an odd element (three to four times as
    long through registers)."""
    import torch
    s, a, d = 2048, 16, 128
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(1)
    data = [torch.randn(s * n, generator=g, device="cuda").to(dt) for n in (3 * h, h)]
    o, dq = torch.zeros(s, h, dtype=dt, device="cuda"), torch.zeros(s, 3 * h, dtype=dt, device="cuda")
    lse, ws = (torch.zeros(1, a, s, device="cuda") for _ in range(2))

    def times(by):
        q, do = (torch.zeros(x.numel() + by, dtype=dt, device="cuda")[by:].copy_(x) for x in data)
        calls = (lambda: B.axonn_attention_fwd(1, s, a, d, q, o, lse), lambda: B.axonn_attention_bwd(1, s, a, d, q, o, lse, do, dq, ws))
        best = [float("inf")] * 2
        for _ in range(5):
            for i, call in enumerate(calls):
                ev = [torch.cuda.Event(enable_timing=True) for _ in range(2)]
                call()
                ev[0].record()
                for _ in range(20):
                    call()
                ev[1].record()
                torch.cuda.synchronize()
                best[i] = min(best[i], ev[0].elapsed_time(ev[1]))
        return best

    aligned, shifted = times(0), times(by)
    assert shifted[0] < 1.8 * aligned[0] and shifted[1] < 1.8 * aligned[1], (aligned, shifted)


@pytest.mark.parametrize("off", [0, 4])
@pytest.mark.parametrize("s,a,d", [(200, 4, 44), (130, 2, 188), (72, 4, 124), (264, 2, 60)])
def test_attention_head_does_not_depend_on_its_place(s, a, d, off):
    """Heads of an odd multiple of 4 columns, the same numbers in each: a head that starts between two 16-byte boundaries gives the
    bits of one that starts at one.  The matrices end with the last head's last column: nothing is read behind it."""
    import torch
    h, dt = a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)

    def same(n):
        buf = torch.full((off + s * n * h,), float("nan"), dtype=dt, device="cuda")
        buf[off:] = torch.randn(s, n, 1, d, generator=g, device="cuda").to(dt).expand(s, n, a, d).reshape(-1)
        return buf[off:].view(s, n * h)

    qkv, dout = same(3), same(1)
    o, dq = torch.zeros(s, h, dtype=dt, device="cuda"), torch.zeros(s, 3 * h, dtype=dt, device="cuda")
    lse, ws = (torch.zeros(1, a, s, device="cuda") for _ in range(2))
    B.axonn_attention_fwd(1, s, a, d, qkv, o, lse)
    B.axonn_attention_bwd(1, s, a, d, qkv, o, lse, dout, dq, ws)
    assert torch.isfinite(dq.float()).all() and o.any() and dq.any()
    for x in (o.view(s, 1, a, d), dq.view(s, 3, a, d)):
        assert torch.equal(x, x[:, :, :1].expand_as(x))
    assert torch.equal(lse, lse[:, :1].expand_as(lse))


@pytest.mark.parametrize("b,a", [(1, 2), (2, 24)])
@pytest.mark.parametrize("d", [44, 64, 128, 188])
def test_attention_is_not_reached_by_tiles_that_causality_leaves_out(d, b, a):
    """A probability of zero times an infinity is no zero: a wave leaves out the tiles of 64 keys that lie in its queries' future
    (forward, dQ) and, where heads have more than 128 columns, the blocks of 32 queries in front of its keys (dK / dV; tiles of 128
    at fewer columns).  Infinities and NaN there do not reach its results; in one launch and in several."""
    import torch
    s, h, dt = 300, a * d, B.torch_elem_dtype()
    g = torch.Generator(device="cuda"); g.manual_seed(d + a)
    qkv, dout = (torch.randn(b * s, n, generator=g, device="cuda").to(dt) for n in (3 * h, h))

    def run(q, do):
        o, dq = torch.zeros(b * s, h, dtype=dt, device="cuda"), torch.zeros(b * s, 3 * h, dtype=dt, device="cuda")
        lse, ws = (torch.zeros(b, a, s, device="cuda") for _ in range(2))
        B.axonn_attention_fwd(b, s, a, d, q, o, lse)
        B.axonn_attention_bwd(b, s, a, d, q, o, lse, do, dq, ws)
        return o.view(b, s, h), lse, dq.view(b, s, 3, h)

    o, lse, dq = run(qkv, dout)
    assert all(torch.isfinite(x.float()).all() for x in (o, lse, dq))
    for value in (float("inf"), float("nan")):
        for p in range(64, s, 64):                      # keys and values from p on
            q = qkv.clone(); q.view(b, s, 3, h)[:, p:, 1:] = value
            po, plse, pdq = run(q, dout)
            assert torch.equal(po[:, :p], o[:, :p]) and torch.equal(plse[..., :p], lse[..., :p])
            assert torch.equal(pdq[:, :p, 0], dq[:, :p, 0])
        step = 32 if d > 128 else 128
        for p in range(step, s, step):                  # queries and their gradients up to p
            q, do = qkv.clone(), dout.clone()
            q.view(b, s, 3, h)[:, :p, 0] = value
            do.view(b, s, h)[:, :p] = value
            assert torch.equal(run(q, do)[2][:, p:, 1:], dq[:, p:, 1:])


@pytest.mark.parametrize("b,s,a,d", [(1, 2040, 24, 128), (4, 512, 16, 64), (1, 50, 8, 64), (2, 500, 24, 188)])
def test_attention_beside_other_work_gives_the_same_bits(b, s, a, d):
    """Waves of a workgroup fall behind each other when others share their CU: 100 passes on each of two streams at once, every
    one the same bits."""
    import torch
    h, dt, n = a * d, B.torch_elem_dtype(), 100
    g = torch.Generator(device="cuda"); g.manual_seed(s + d)
    qkv, dout = (torch.randn(b * s, w, generator=g, device="cuda").to(dt) for w in (3 * h, h))
    new = lambda: (torch.zeros(b * s, h, dtype=dt, device="cuda"), torch.zeros(b * s, 3 * h, dtype=dt, device="cuda"),
                   torch.zeros(b * a * s, device="cuda"), torch.zeros(b * a * s, device="cuda"))
    runs = [(torch.cuda.Stream(), new(), torch.zeros(2, dtype=torch.int64, device="cuda")) for _ in range(2)]
    first = new()
    B.axonn_attention_fwd(b, s, a, d, qkv, first[0], first[2])
    B.axonn_attention_bwd(b, s, a, d, qkv, first[0], first[2], dout, first[1], first[3])
    torch.cuda.synchronize()
    for _ in range(n):
        for stream, (o, dqkv, lse, ws), differ in runs:
            with torch.cuda.stream(stream):
                B.axonn_attention_fwd(b, s, a, d, qkv, o, lse, stream)
                B.axonn_attention_bwd(b, s, a, d, qkv, o, lse, dout, dqkv, ws, stream)
                differ[0] += (o.view(torch.int16) != first[0].view(torch.int16)).any()
                differ[1] += (dqkv.view(torch.int16) != first[1].view(torch.int16)).any()
    torch.cuda.synchronize()
    assert [differ.tolist() for _, _, differ in runs] == [[0, 0]] * 2


@pytest.mark.parametrize("b,s,a,d", [(2, 72, 66, 64), (4, 72, 33, 128)])
def test_attention_delta_is_the_sum_of_products_in_element_order(b, s, a, d):
    """Where the dQ kernel forms delta = sum_d dO O itself (more than 128 tiles): 8 products per lane one after the other, then
    the lanes' sums in a tree, in 32 bits and in both element types.  A product of two 16-bit numbers is exact in 32 bits, so
    a fused multiply-add is an addition of it: the same bits."""
    import torch
    rng = np.random.default_rng(d)
    h = a * d
    qkv, dout = _rng_bf16(rng, (b * s, 3 * h)), _rng_bf16(rng, (b * s, h))
    o = torch.zeros(b * s, h, dtype=B.torch_elem_dtype(), device="cuda"); dqkv = torch.zeros(b * s, 3 * h, dtype=o.dtype, device="cuda")
    lse, delta = (torch.zeros(b * a * s, dtype=torch.float32, device="cuda") for _ in range(2))
    QKV, DO = dev_bf16(qkv), dev_bf16(dout)
    B.axonn_attention_fwd(b, s, a, d, QKV, o, lse)
    B.axonn_attention_bwd(b, s, a, d, QKV, o, lse, DO, dqkv, delta)
    prod = (host(o).astype(np.float32) * host(DO).astype(np.float32)).reshape(b, s, a, d // 8, 8)
    p = np.zeros(prod.shape[:-1], np.float32)
    for e in range(8):
        p = p + prod[..., e]
    while p.shape[-1] > 1:
        p = p[..., :p.shape[-1] // 2] + p[..., p.shape[-1] // 2:]
    assert np.array_equal(delta.cpu().numpy().reshape(b, a, s), p[..., 0].transpose(0, 2, 1))


def test_attention_large_scores_stay_finite():
    """Scores of order +-100: the running-max subtraction must keep exp in range."""
    import torch
    rng = np.random.default_rng(3)
    b, s, a, d = 1, 192, 2, 64
    h = a * d
    qkv = _rng_bf16(rng, (b * s, 3 * h)); qkv[:, :2 * h] *= 4; qkv = snap_elem(qkv)
    o_ref, lse_ref, _ = _attn_ref(qkv, np.zeros((b * s, h), np.float32), b, s, a, d)
    o = torch.zeros(b * s, h, dtype=B.torch_elem_dtype(), device="cuda")
    lse = torch.zeros(b, a, s, dtype=torch.float32, device="cuda")
    B.axonn_attention_fwd(b, s, a, d, dev_bf16(qkv), o, lse)
    got = host(o)
    assert np.isfinite(got).all()
    parity(got, o_ref, TOL, C_ATTN, label="attention_large_scores_stay_finite")


@pytest.mark.parametrize("slope,spike", [(0.02, 0.0), (0.12, 0.0), (0.02, 40.0)])
def test_attention_growing_row_maxima(slope, spike):
    """The forward kernel moves the reference point of its exponentials only when a row maximum has grown by more
    than a threshold.  Scores that rise with the key index -- slowly (the reference stays behind the maximum for
    many tiles), quickly (it moves in every tile), and with one late key far above the rest (a jump after a long
    quiet stretch) -- must give the oracle's output, log-sum-exp and gradients."""
    import torch
    rng = np.random.default_rng(17)
    b, s, a, d = 1, 640, 2, 64
    h = a * d
    qkv = 0.3 * rng.standard_normal((b * s, 3 * h)).astype(np.float32)
    u = rng.standard_normal(d).astype(np.float32); u /= np.linalg.norm(u)
    ramp = (slope * np.arange(s, dtype=np.float32))[:, None]
    for hd in range(a):
        qkv[:, hd * d:(hd + 1) * d] += np.sqrt(d) * u                       # every query has component sqrt(d) along u
        qkv[:, h + hd * d:h + (hd + 1) * d] += ramp * u                     # key j has component slope * j: score rises by slope per key
    if spike:
        qkv[500, h:h + d] += spike * u                                     # one late key of head 0 stands out
    qkv = snap_elem(qkv); dout = _rng_bf16(rng, (b * s, h))
    o_ref, lse_ref, dqkv_ref = _attn_ref(qkv, dout, b, s, a, d)
    QKV, DO = dev_bf16(qkv), dev_bf16(dout)
    o = torch.zeros(b * s, h, dtype=B.torch_elem_dtype(), device="cuda")
    lse = torch.zeros(b, a, s, dtype=torch.float32, device="cuda")
    B.axonn_attention_fwd(b, s, a, d, QKV, o, lse)
    assert np.isfinite(host(o)).all()
    parity(host(o), o_ref, TOL, C_ATTN, label="attention_growing_row_maxima")
    assert np.abs(host(lse) - lse_ref).max() < 2e-3 * max(1.0, np.abs(lse_ref).max() / 10)
    dqkv = torch.zeros(b * s, 3 * h, dtype=B.torch_elem_dtype(), device="cuda")
    delta = torch.zeros(b * a * s, dtype=torch.float32, device="cuda")
    B.axonn_attention_bwd(b, s, a, d, QKV, o, lse, DO, dqkv, delta)
    got = host(dqkv)
    # dv is a plain contraction with P.  dq = dS K / sqrt(d) and dk = dS^T Q / sqrt(d) contract the 16-bit rounding of dS
    # with keys / queries that here carry a large common component along u, while the rows of dS sum to zero: the
    # roundings do not cancel the way the exact terms do.  The bound follows from the input: roundings of relative
    # size 2^-9 / sqrt(3) (uniform) with independent signs give an error of root mean square
    # 2^-9 / sqrt(3) * sqrt((dS*dS) (K*K)) / sqrt(d) per element of dq.  The rounding of o, through delta = rowsum(dO o),
    # adds a term of the same kind (an error per query times the probability-weighted mean key).  Bound: three times
    # the prediction plus the bound of a well-conditioned input (measured at slope 0.12: 5.0e-2 against 6.7e-2).  (The lazy rescaling is a matter of the forward pass: its o, element by element, and
    # its log-sum-exp are compared above.)
    parity(got[:, 2 * h:], dqkv_ref[:, 2 * h:], 2 * TOL, C_ATTN_BWD, label="attention_growing_row_maxima_bwd")
    q64 = qkv.astype(np.float64).reshape(s, 3, a, d)
    for hd in range(a):
        Q, K, V = q64[:, 0, hd], q64[:, 1, hd], q64[:, 2, hd]
        S = np.where(np.tril(np.ones((s, s), bool)), Q @ K.T / np.sqrt(d), -np.inf)
        P = np.exp(S - S.max(-1, keepdims=True)); P /= P.sum(-1, keepdims=True)
        dO = dout.astype(np.float64).reshape(s, a, d)[:, hd]
        dP = dO @ V.T
        dS = P * (dP - (dP * P).sum(-1, keepdims=True))
        r = 2.0 ** -9 / np.sqrt(3.0) / np.sqrt(d)
        for name, c0, pred in (("dq", 0, r * np.sqrt((dS * dS) @ (K * K))), ("dk", h, r * np.sqrt((dS * dS).T @ (Q * Q)))):
            sl = slice(c0 + hd * d, c0 + (hd + 1) * d)
            ref_t = dqkv_ref[:, sl]
            bound = 2 * TOL + 3 * np.linalg.norm(pred) / np.linalg.norm(ref_t)
            e = rel_fro(got[:, sl], ref_t)
            assert e < bound, (name, hd, e, bound)


# ------------------------------------------------------------------------- Adam
@pytest.mark.parametrize("n", [8, 1000, 65536 + 24, 1 << 20])
@pytest.mark.parametrize("fresh,wd,step,gs", [(False, 0.0, 100, 1.0), (True, 0.01, 1, 0.25)])
def test_adam_bucket_kernel(n, fresh, wd, step, gs):
    import torch
    from paper_2110_13005_amd.inputs import make_adam_inputs
    th, m, v, g16 = make_adam_inputs(n, seed=n, fresh=fresh)
    lr, b1, b2, eps = 1e-4, 0.9, 0.95, 1e-8
    rt, rm, rv, r16 = oracle.adam_step(th, m, v, g16, lr, b1, b2, eps, wd, step, gs, half=B.ELEM)
    TH, Mm, V, G = dev_f32(th), dev_f32(m), dev_f32(v), dev_bf16(g16)
    P16 = torch.zeros(n, dtype=B.torch_elem_dtype(), device="cuda")
    B.axonn_adam_bucket(n, TH, Mm, V, G, P16, lr, b1, b2, eps, wd, step, gs)
    assert rel_fro(host(TH), rt) <= 1e-6
    assert rel_fro(host(Mm), rm) <= 1e-6
    assert rel_fro(host(V), rv) <= 1e-6
    # theta16 is the bf16 rounding of the GPU's own fp32 theta, bit for bit
    assert torch.equal(P16, TH.to(B.torch_elem_dtype()))
    # and within one bf16 ulp of the oracle's
    assert np.abs(host(P16) - r16).max() <= np.abs(r16).max() * 2.0 ** -7
