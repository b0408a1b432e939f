"""GPU parity of the single kernels against the CPU oracle, element by element, through the C ABI."""
import numpy as np
import pytest
import torch

import paper_2405_15362_amd as P
import synth
from oracle import layer as OL
import gpu_util as U
from gpu_util import assert_close, dev, host, mat, rel_l2, tol, tuned

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def ctx():
    c = P.pmc_create(None)
    ws = torch.empty(256 << 20, dtype=torch.uint8, device="cuda")
    P.pmc_workspace_attach(c, ws)
    yield c
    torch.cuda.synchronize()
    P.pmc_destroy(c)


def _nan_past_k(key, rows, K, k_fast, scale):
    """A bf16 operand stored [rows, K] (k_fast) or [K, rows] as a view of a buffer that holds NaN everywhere past K, so that
    a value read from there cannot go unnoticed; and its values as [rows, K] in float64."""
    m = mat(key, (rows, K) if k_fast else (K, rows), "bf16", scale)
    big = torch.full((rows, K + 64) if k_fast else (K + 64, rows), float("nan"), dtype=torch.bfloat16, device="cuda")
    v = big[:, :K] if k_fast else big[:K]
    v.copy_(dev(m, "bf16"))
    return v, (m if k_fast else m.T).astype(np.float64)


def _gemm_views(ctx, ta, tb, M, N, K, a, b, c, epi):
    rc = P.lib.pmc_gemm(ctx, P.PMC_BF16, int(ta), int(tb), M, N, K, a.data_ptr(), a.stride(0), b.data_ptr(), b.stride(0),
                        c.data_ptr(), c.stride(0), epi, None, None, None)
    assert rc == 0


def _gemm_case(ctx, dtype, ta, tb, M, N, K, epi):
    key = (dtype, ta, tb, M, N, K, epi)
    print("gemm case", key, flush=True)
    a = mat(key + ("a",), (K, M) if ta else (M, K), dtype)
    b = mat(key + ("b",), (N, K) if tb else (K, N), dtype, 0.05)
    bias = mat(key + ("bias",), (N,), dtype)
    resid = mat(key + ("r",), (M, N), dtype)
    aux_in = mat(key + ("u",), (M, N), dtype)
    A = a.T.astype(np.float64) if ta else a.astype(np.float64)
    B = b.T.astype(np.float64) if tb else b.astype(np.float64)
    ref = A @ B
    out_dtype = "f32" if epi == P.EPI_ACCUM_F32 else dtype
    c0 = mat(key + ("c0",), (M, N), "f32")
    c = dev(c0, out_dtype)
    aux = dev(aux_in, dtype) if epi in (P.EPI_BIAS_GELU, P.EPI_DGELU, P.EPI_BIAS_GELU_GRAD, P.EPI_MUL) else None
    want_aux = None
    if epi == P.EPI_BIAS:
        ref = ref + bias
    elif epi == P.EPI_BIAS_RESID:
        ref = ref + bias + resid
    elif epi == P.EPI_BIAS_GELU:
        ref = ref + bias
        want_aux = OL.gelu(ref)
    elif epi == P.EPI_DGELU:
        ref = ref * OL.gelu_grad(aux_in.astype(np.float64))
    elif epi == P.EPI_ACCUM_F32:
        ref = ref + c0
    elif epi == P.EPI_BIAS_GELU_GRAD:
        want_aux = OL.gelu(ref + bias)
        ref = OL.gelu_grad(ref + bias)
    elif epi == P.EPI_MUL:
        ref = ref * aux_in.astype(np.float64)
    P.pmc_gemm(ctx, dev(a, dtype), dev(b, dtype), c, ta, tb, epi,
               dev(bias, dtype) if epi in (P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU, P.EPI_BIAS_GELU_GRAD) else None,
               dev(resid, dtype) if epi == P.EPI_BIAS_RESID else None, aux)
    torch.cuda.synchronize()
    assert_close(host(c), ref, dtype, str(key))
    if want_aux is not None:
        assert_close(host(aux), want_aux, dtype, str(key))


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_gemm_f32_layouts_and_epilogues(ctx, ta, tb):
    for epi in range(8):
        _gemm_case(ctx, "f32", ta, tb, 77, 130, 45, epi)
    _gemm_case(ctx, "f32", ta, tb, 128, 256, 1024, P.EPI_NONE)


@pytest.mark.parametrize("tile", [0, 1, 2, 3, 4])
def test_gemm_f32_tile_shapes(ctx, tune, tile):
    """Every tile shape of the fp32 product (128x128 .. 16x16) in every layout: less than one tile, ragged
    edges in M and N, K shorter than one 32-deep tile, past the K groups' last full round, and ragged."""
    tune(gemm_tile=tile)
    for ta in (False, True):
        for tb in (False, True):
            for M, N, K in ((4, 4, 4), (36, 68, 200), (132, 260, 36), (256, 132, 416)):
                for epi in (P.EPI_BIAS_RESID, P.EPI_ACCUM_F32, P.EPI_BIAS_GELU_GRAD):
                    _gemm_case(ctx, "f32", ta, tb, M, N, K, epi)


@pytest.mark.parametrize("M,N,K,shape", [(3084, 1036, 68, U.F32_TILE64X128), (1540, 2044, 100, U.F32_TILE64X128), (516, 1036, 516, U.F32_TILE32_FOUR),
                                         (2060, 520, 40, U.F32_TILE32_FOUR), (1028, 1036, 12, U.F32_TILE32_FOUR)])
def test_gemm_f32_tiles_that_no_switch_forces(ctx, M, N, K, shape):
    for ta, tb in ((False, False), (False, True), (True, False)):
        assert U.gemm_plan("f32", ta, tb, M, N, K)[0] == shape, (ta, tb)
        _gemm_case(ctx, "f32", ta, tb, M, N, K, P.EPI_ACCUM_F32 if ta else P.EPI_BIAS_GELU_GRAD)


@pytest.mark.parametrize("tb,epis", [(False, (P.EPI_BIAS_RESID, P.EPI_BIAS_GELU_GRAD)), (True, (P.EPI_NONE, P.EPI_MUL))])
def test_gemm_bf16_128_tiles_in_two_k_groups(ctx, tune, tb, epis):
    """128x128 tiles of at most one round: eight waves in two K groups, with ragged output tiles; and four waves where K is of less than half a
    tile, of half a tile, of whole ones but short, ragged, or where there is one row of tiles."""
    tune(gemm_tile=2)
    for M, K in [(136, K) for K in (8, 32, 40, 64, 72, 128, 200, 328, 960, 1024, 1032, 1088, 4160)] + [(128, 1024)]:
        assert P.lib.pmc_test_gemm_k_groups(M, 264, K) == (M > 128 and K >= 1024 and K % 64 == 0)
        for epi in epis:
            _gemm_case(ctx, "bf16", False, tb, M, 264, K, epi)


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_gemm_f32_element_loads(ctx, ta, tb):
    """Odd sizes: the 64x64 tiles of plain FMAs (every epilogue; one row, one column, one k past whole tiles, and less
    than a 16-deep step) and the 16x16 tiles on the other side of the rule."""
    for epi in range(8):
        assert U.gemm_plan("f32", ta, tb, 1025, 2113, 33, epi)[0] == U.F32_FMA_ELEMENTS
        _gemm_case(ctx, "f32", ta, tb, 1025, 2113, 33, epi)
    assert U.gemm_plan("f32", ta, tb, 3001, 1031, 7)[0] == U.F32_FMA_ELEMENTS
    _gemm_case(ctx, "f32", ta, tb, 3001, 1031, 7, P.EPI_BIAS_RESID)
    assert U.gemm_plan("f32", ta, tb, 257, 255, 517)[0] == U.F32_DIRECT_ELEMENTS
    _gemm_case(ctx, "f32", ta, tb, 257, 255, 517, P.EPI_BIAS_RESID)


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_gemm_f32_operand_of_two_gigabytes(ctx, ta, tb):
    """131072 tokens of hidden 4096: A is exactly 2^31 bytes, past the reach of a 31-bit offset.  Every element against
    float64."""
    M, N, K = 131072, 68, 4096
    assert U.gemm_plan("f32", ta, tb, M, N, K)[0] == U.F32_FMA_ELEMENTS
    gen = torch.Generator(device="cuda").manual_seed(8)
    a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=gen)
    b = torch.randn((N, K) if tb else (K, N), device="cuda", generator=gen)
    c = torch.empty(M, N, device="cuda")
    print("fp32 operand of 2^31 bytes", ta, tb, flush=True)
    P.pmc_gemm(ctx, a, b, c, ta, tb)
    B = (b.T if tb else b).double().contiguous()
    for r in range(0, M, 32768):
        want = (a[:, r:r + 32768].T if ta else a[r:r + 32768]).double().contiguous() @ B
        assert_close(host(c[r:r + 32768]), want.cpu().numpy(), "f32", f"rows {r}..")


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_gemm_f32_output_of_2_to_the_31_elements(ctx, ta, tb):
    """More output elements than 2^31 (8.6 GB) of odd sizes: 2^23 and more 16x16 tiles of 512 threads would not fit one
    launch dimension.  Every element against the same three products in float64, a band of rows at a time."""
    M, N, K = 46343, 46351, 3
    gen = torch.Generator(device="cuda").manual_seed(7)
    a = torch.randn((K, M) if ta else (M, K), device="cuda", generator=gen)
    b = torch.randn((N, K) if tb else (K, N), device="cuda", generator=gen)
    c = torch.empty(M, N, device="cuda")
    print("fp32 output of 2^31 elements", ta, tb, flush=True)
    P.pmc_gemm(ctx, a, b, c, ta, tb)
    torch.cuda.synchronize()
    A, B = (a.T if ta else a).double(), (b.T if tb else b).double()
    for r in range(0, M, 4096):
        want = sum(A[r:r + 4096, k, None] * B[None, k] for k in range(K))
        # three products and two sums, each rounded to 2^-24 relative
        bound = 4 * 2.0 ** -24 * sum((A[r:r + 4096, k, None] * B[None, k]).abs() for k in range(K))
        assert bool(((c[r:r + 4096].double() - want).abs() <= bound).all()), (r, ta, tb)
    del c


@pytest.mark.parametrize("ta", [False, True])
@pytest.mark.parametrize("tb", [False, True])
def test_gemm_bf16_small_tiles_ragged(ctx, ta, tb):
    # several 128x128 tiles with ragged tails in M, N and K
    for epi in range(8):
        _gemm_case(ctx, "bf16", ta, tb, 200, 328, 136, epi)
    _gemm_case(ctx, "bf16", ta, tb, 8, 8, 8, P.EPI_NONE)
    _gemm_case(ctx, "bf16", ta, tb, 512, 768, 1024, P.EPI_NONE)


@pytest.mark.parametrize("ta,tb,epis", [(False, False, (P.EPI_NONE, P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU, P.EPI_BIAS_GELU_GRAD)),
                                        (False, True, (P.EPI_NONE, P.EPI_DGELU, P.EPI_MUL)),
                                        (True, False, (P.EPI_NONE, P.EPI_ACCUM_F32))])
def test_gemm_bf16_direct_to_lds_path(ctx, ta, tb, epis):
    """K in whole 64-wide tiles takes the direct-to-LDS kernel: each of its three tile shapes, with
    ragged edges in M and N (clamped loads), a single K tile and many K tiles."""
    try:
        for tile in (4, 3, 2, 1, 0):      # 256x320, 64x128, 128x128, 256x128, 256x256 tiles
            P.pmc_tuning_set("gemm_tile", tile)
            for epi in epis:
                _gemm_case(ctx, "bf16", ta, tb, 200, 328, 192, epi)
                _gemm_case(ctx, "bf16", ta, tb, 1000, 1544, 64, epi)
            _gemm_case(ctx, "bf16", ta, tb, 8, 8, 64, epis[0])
            _gemm_case(ctx, "bf16", ta, tb, 264, 136, 2048, epis[-1])
    finally:
        P.pmc_tuning_set("gemm_tile", -1)
    _gemm_case(ctx, "bf16", ta, tb, 3848, 4104, 320, epis[-1])   # heuristic choice, many tiles


@pytest.mark.parametrize("ta,tb,epis", [(False, False, (P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU, P.EPI_BIAS_GELU_GRAD)),
                                        (False, True, (P.EPI_NONE, P.EPI_DGELU, P.EPI_MUL)),
                                        (True, False, (P.EPI_ACCUM_F32,))])
def test_gemm_bf16_split_k(ctx, ta, tb, epis):
    """Long K and few tiles: K is cut into ranges whose fp32 partial products (in 128x128 or 64x64 tiles) a second kernel
    adds in a fixed order; the result must also be identical from run to run, and close to the product in one piece.
    Equal and unequal ranges, the last one ending in a whole or a partial K tile, on operands with NaN past K."""
    for epi in epis:
        _gemm_case(ctx, "bf16", ta, tb, 512, 1024, 1024, epi)      # K too short for a split
        _gemm_case(ctx, "bf16", ta, tb, 136, 264, 4096, epi)       # cut only where both operands are stored [k][rows]
    layout_epi = P.EPI_ACCUM_F32 if ta else epis[0]
    # M, N, K, tile of the partial products, ranges
    for M, N, K, shape, ranges in ((304, 3272, 6816, 2, 4), (392, 2544, 6384, 2, 4), (144, 3272, 11576, 2, 8), (144, 3272, 11584, 2, 8),
                                   (72, 3256, 5328, 5, 2), (72, 2992, 5792, 5, 2), (16, 8, 7880, 5, 8), (64, 8, 8704, 5, 8)):
        for epi in epis:
            plan = U.gemm_plan("bf16", ta, tb, M, N, K, epi, ws_bytes=256 << 20)
            assert plan[:2] == (U.PLAN_SPLIT + shape, ranges), (M, N, K, plan)
        for epi in epis if M * N * K < 3e9 else epis[-1:]:
            _gemm_case(ctx, "bf16", ta, tb, M, N, K, epi)
        key = ("split k", ta, tb, M, N, K)
        a, A = _nan_past_k(key + ("a",), M, K, not ta, 1.0)
        b, B = _nan_past_k(key + ("b",), N, K, tb, 0.05)
        accum = layout_epi == P.EPI_ACCUM_F32
        c0 = mat(key + ("c0",), (M, N), "f32")
        outs = []
        for tile in (None, None, 2):                               # a forced tile is never split
            with tuned(gemm_tile=tile):
                c = dev(c0 if accum else np.zeros((M, N)), "f32" if accum else "bf16")
                _gemm_views(ctx, ta, tb, M, N, K, a, b, c, P.EPI_ACCUM_F32 if accum else P.EPI_NONE)
                outs.append(c)
        torch.cuda.synchronize()
        assert torch.equal(outs[0], outs[1]), key
        assert_close(host(outs[0]), A @ B.T + (c0 if accum else 0.0), "f32" if accum else "bf16", str(key))
        assert rel_l2(host(outs[0]), host(outs[2])) <= (1e-6 if accum else 3e-3), key   # fp32 sums in another order; rounding to bf16


@pytest.mark.parametrize("ta,tb,M,N,K,ranges", [(False, False, 536, 2096, 7680, 4), (False, True, 536, 2096, 7680, 4),
                                                (False, False, 208, 3080, 9088, 8), (True, False, 72, 8440, 3104, 7)])
def test_gemm_bf16_split_k_ranges_on_xcds_of_their_own(ctx, ta, tb, M, N, K, ranges):
    """Large tiles whose number does not divide over the XCDs of a range, and a number of ranges that does not divide the XCDs."""
    epi = P.EPI_ACCUM_F32 if ta else P.EPI_NONE if tb else P.EPI_BIAS_RESID
    assert U.gemm_plan("bf16", ta, tb, M, N, K, epi, ws_bytes=256 << 20)[:2] == (U.PLAN_SPLIT + 2, ranges)
    _gemm_case(ctx, "bf16", ta, tb, M, N, K, epi)


@pytest.mark.parametrize("tb,M,N,K,shape,ranges", [(False, 40, 4104, 8200, 5, 2), (False, 56, 1032, 32840, 5, 8), (False, 40, 3080, 11000, 5, 4),
                                                    (False, 104, 4104, 8200, 2, 8), (True, 104, 6152, 22536, 2, 8)])
def test_gemm_bf16_split_k_of_one_row_of_tiles_dealt_in_turn(ctx, tb, M, N, K, shape, ranges):
    """One row of tiles and operands of 64 MB and more, 256 MB with B stored [N][K]; also numbers of tiles that do not divide over the XCDs, ranges of unequal length."""
    epi = P.EPI_MUL if tb else P.EPI_BIAS_RESID
    assert U.gemm_plan("bf16", False, tb, M, N, K, epi, ws_bytes=256 << 20)[:2] == (U.PLAN_SPLIT + shape, ranges)
    assert not P.lib.pmc_test_gemm_split_own_xcds(tb, 1, M, N, K, ranges)
    _gemm_case(ctx, "bf16", False, tb, M, N, K, epi)


def test_gemm_bf16_weight_gradient_persistent(ctx, tune):
    """The persistent W-pass kernel (fp32 C += A^T B; one workgroup per compute unit walks its
    256x256 tiles, its first tile cut in two along K to put the workgroups out of phase): fewer tiles
    than workgroups, more tiles than workgroups with ragged edges, short and long K; and the same
    result from run to run."""
    tune(gemm_wgrad=1)
    for M, N, K in ((512, 256, 256), (264, 136, 1024), (4104, 4360, 256), (4096, 4608, 576), (3848, 4872, 1280)):
        _gemm_case(ctx, "bf16", True, False, M, N, K, P.EPI_ACCUM_F32)
    a = dev(mat(("wg", "a"), (1024, 4104), "bf16"), "bf16")
    b = dev(mat(("wg", "b"), (1024, 4360), "bf16", 0.05), "bf16")
    c0 = dev(mat(("wg", "c"), (4104, 4360), "f32"), "f32")
    outs = []
    for flag in (1, 1, 0):
        tune(gemm_wgrad=flag)
        c = c0.clone()
        P.pmc_gemm(ctx, a, b, c, True, False, P.EPI_ACCUM_F32)
        outs.append(c)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert rel_l2(host(outs[0]), host(outs[2])) <= 1e-6     # the plain kernel adds K in one piece


def test_gemm_bf16_weight_gradient_two_workgroups_per_unit(ctx, tune):
    """The W-pass kernel with 256x128 tiles and a ring of 32-deep stages (two workgroups share a compute
    unit): fewer tiles than units, many more, ragged edges in both directions, K of one 64-wide tile (two
    ring tiles, fewer than the ring has stages), short and long K; the same bits from run to run; and the
    same sums as the plain kernel up to fp32 summation order."""
    tune(gemm_wgrad=2)
    for M, N, K in ((512, 256, 64), (264, 136, 128), (264, 136, 1024), (4104, 4360, 256), (4096, 4608, 576), (3848, 4872, 1280)):
        _gemm_case(ctx, "bf16", True, False, M, N, K, P.EPI_ACCUM_F32)
    a = dev(mat(("wg", "a"), (1024, 4104), "bf16"), "bf16")
    b = dev(mat(("wg", "b"), (1024, 4360), "bf16", 0.05), "bf16")
    c0 = dev(mat(("wg", "c"), (4104, 4360), "f32"), "f32")
    outs = []
    for flag in (2, 2, 0):
        tune(gemm_wgrad=flag)
        c = c0.clone()
        P.pmc_gemm(ctx, a, b, c, True, False, P.EPI_ACCUM_F32)
        outs.append(c)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert rel_l2(host(outs[0]), host(outs[2])) <= 1e-6


@pytest.mark.parametrize("wgrad", [0, 1, 2])
def test_gemm_bf16_grouped_weight_gradient(ctx, tune, wgrad):
    """Queued weight gradients as one product: C += sum_i A_i^T B_i over pieces that live in separate
    buffers.  Every tile shape of the plain kernel and the persistent one; one piece, several pieces,
    the maximum; pieces of a single 64-wide K tile (a piece boundary at every tile) and of many;
    ragged M and N; and the same bits from run to run.  Against the fp64 sum of the pieces' products;
    the result must also agree with adding the pieces one product at a time."""
    tune(gemm_wgrad=wgrad)
    cases = [(512, 256, 64, 3), (264, 136, 192, 2), (1000, 1544, 128, 8), (2048, 2304, 256, 4), (4104, 4360, 64, 5),
             (128, 128, 1024, 1)]
    for tile in (None, 0, 1, 2):
        tune(gemm_tile=tile)
        for M, N, K, count in (cases if tile is None else cases[:3]):
            key = ("grouped", M, N, K, count)
            print("grouped wgrad case", key, "tile", tile, "persistent", wgrad, flush=True)
            a = [mat(key + ("a", i), (K, M), "bf16") for i in range(count)]
            b = [mat(key + ("b", i), (K, N), "bf16", 0.05) for i in range(count)]
            c0 = mat(key + ("c0",), (M, N), "f32")
            ref = c0.astype(np.float64)
            for x, y in zip(a, b):
                ref = ref + x.T.astype(np.float64) @ y.astype(np.float64)
            da, db = [dev(x, "bf16") for x in a], [dev(y, "bf16") for y in b]
            outs = []
            for _ in range(2):
                c = dev(c0, "f32")
                P.pmc_gemm_grouped_wgrad(ctx, da, db, c)
                outs.append(c)
            one_by_one = dev(c0, "f32")
            for x, y in zip(da, db):
                P.pmc_gemm(ctx, x, y, one_by_one, True, False, P.EPI_ACCUM_F32)
            torch.cuda.synchronize()
            assert torch.equal(outs[0], outs[1]), key
            assert rel_l2(host(outs[0]), ref) <= 1e-5, (key, rel_l2(host(outs[0]), ref))   # fp32 sums of exact bf16 products
            assert rel_l2(host(outs[0]), host(one_by_one)) <= 1e-5, key


@pytest.mark.timeout(600)
def test_gemm_bf16_largest_workload_shapes(ctx):
    """The twelve products of a layer at the largest workload (hidden 5120, FFN 20480, 4096 tokens), at
    full size and in the launch configuration the passes use (heuristic tile choice, persistent W
    kernel).  Operands are drawn on the GPU from a seeded generator (2e8 elements per product);
    EVERY output element is checked against the fp64 product with the epilogue's definition applied
    (whole tensor, every 32 x 128 block, every element)."""
    T, h, f = 4096, 5120, 20480
    gen = torch.Generator(device="cuda").manual_seed(4)
    bf = torch.bfloat16

    def rnd(shape, scale):
        return (torch.randn(shape, device="cuda", generator=gen) * scale).to(bf)

    def f64(t):
        return t.float().cpu().numpy().astype(np.float64)

    cases = [("F qkv", False, False, T, 3 * h, h, P.EPI_BIAS), ("F proj", False, False, T, h, h, P.EPI_BIAS_RESID),
             ("F fc1", False, False, T, f, h, P.EPI_BIAS_GELU_GRAD), ("F fc2", False, False, T, h, f, P.EPI_BIAS_RESID),
             ("B dfc2", False, True, T, f, h, P.EPI_MUL), ("B dfc1", False, True, T, h, f, P.EPI_NONE),
             ("B dproj", False, True, T, h, h, P.EPI_NONE), ("B dqkv", False, True, T, h, 3 * h, P.EPI_NONE),
             ("W fc2", True, False, f, h, T, P.EPI_ACCUM_F32), ("W fc1", True, False, h, f, T, P.EPI_ACCUM_F32),
             ("W proj", True, False, h, h, T, P.EPI_ACCUM_F32), ("W qkv", True, False, h, 3 * h, T, P.EPI_ACCUM_F32)]
    for name, ta, tb, M, N, K, epi in cases:
        print("largest-shape gemm", name, M, N, K, flush=True)
        a = rnd((K, M) if ta else (M, K), 1.0)
        b = rnd((N, K) if tb else (K, N), 0.02)
        bias, extra = rnd((N,), 0.02), rnd((M, N), 1.0)          # extra: residual or GeLU input
        c = (torch.randn((M, N), device="cuda", generator=gen) if epi == P.EPI_ACCUM_F32
             else torch.zeros((M, N), device="cuda", dtype=bf))
        c0 = c.clone() if epi == P.EPI_ACCUM_F32 else None
        aux = extra.clone() if epi == P.EPI_MUL else (torch.zeros_like(extra) if epi == P.EPI_BIAS_GELU_GRAD else None)
        P.pmc_gemm(ctx, a, b, c, ta, tb, epi, bias if epi in (P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU_GRAD) else None,
                   extra if epi == P.EPI_BIAS_RESID else None, aux)
        torch.cuda.synchronize()
        A = f64(a).T if ta else f64(a)
        B = f64(b).T if tb else f64(b)
        ref = A @ B
        del A, B
        if epi in (P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU_GRAD):
            ref += f64(bias)
        if epi == P.EPI_BIAS_RESID:
            ref += f64(extra)
        if epi == P.EPI_MUL:
            ref *= f64(extra)
        if epi == P.EPI_ACCUM_F32:
            ref += f64(c0)
        if epi == P.EPI_BIAS_GELU_GRAD:
            assert_close(f64(aux), OL.gelu(ref), "bf16", name + " gelu")
            ref = OL.gelu_grad(ref)
        # fp32 sums of exact bf16 products: the fp32 accumulate is held to the fp32 bounds
        assert_close(f64(c), ref, "f32" if epi == P.EPI_ACCUM_F32 else "bf16", name,
                     whole_tol=1e-5 if epi == P.EPI_ACCUM_F32 else None)
        del a, b, c, c0, aux, extra, ref


@pytest.mark.parametrize("ta,tb,epis", [(False, False, (P.EPI_NONE, P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU, P.EPI_BIAS_GELU_GRAD)),
                                        (False, True, (P.EPI_NONE, P.EPI_DGELU, P.EPI_MUL)),
                                        (True, False, (P.EPI_NONE, P.EPI_ACCUM_F32))])
def test_gemm_bf16_random_shapes(ctx, ta, tb, epis):
    """Seeded random shapes in the library's own choice of kernel and tile: M and N any multiple of 8
    up to a few tiles (ragged edges in both), K in whole 64-wide tiles or any multiple of 8 (a partial
    last tile), split where the library picks it; the epilogue drawn from those the layout is used with."""
    rng = np.random.default_rng(20240515 + 2 * ta + tb)
    for i in range(14):
        M, N = (int(8 * rng.integers(1, 190)) for _ in range(2))
        K = int(64 * rng.integers(1, 40)) if i % 3 else int(8 * rng.integers(1, 90))
        _gemm_case(ctx, "bf16", ta, tb, M, N, K, epis[int(rng.integers(0, len(epis)))])


@pytest.mark.parametrize("ta,tb,epi", [(False, False, P.EPI_NONE), (False, True, P.EPI_NONE), (True, False, P.EPI_ACCUM_F32)])
@pytest.mark.parametrize("K", [8, 40, 56, 104, 968, 1000])
def test_gemm_bf16_partial_last_k_tile(ctx, tune, ta, tb, epi, K):
    """A K that is no multiple of the K tile's depth (64, or 32 in the ring kernels of the weight gradient): every tile
    shape and weight-gradient kernel, on operands that are views of buffers holding NaN everywhere past K, so a value
    read from there cannot go unnoticed."""
    M, N = 328, 200
    key = ("k tail", ta, tb, K)
    a, A = _nan_past_k(key + ("a",), M, K, not ta, 1.0)
    b, B = _nan_past_k(key + ("b",), N, K, tb, 0.05)
    c0 = mat(key + ("c0",), (M, N), "f32")
    accum = epi == P.EPI_ACCUM_F32
    ref = A @ B.T + (c0 if accum else 0.0)
    for switches in [{"gemm_tile": t} for t in range(5)] + ([{"gemm_wgrad": w} for w in range(3)] if accum else [{}]):
        print("k tail", key, switches, flush=True)
        tune(**switches)
        c = dev(c0, "f32" if accum else "bf16")
        _gemm_views(ctx, ta, tb, M, N, K, a, b, c, epi)
        torch.cuda.synchronize()
        tuned.reset()
        assert_close(host(c), ref, "bf16", f"{key} {switches}")


# sizes of which every layout takes the shape; B adds the 64x128 tile whose waves split K, with odd and even numbers of K tiles
SMALL_TILES = [(7, 376, 8, 8), (6, 1160, 200, 40), (7, 8, 376, 104), (6, 200, 1160, 104), (5, 1160, 392, 200), (7, 376, 8, 584),
               (6, 1160, 200, 1000), (5, 1176, 392, 1000), (7, 8, 376, 2040), (5, 1160, 392, 2040), (6, 200, 1168, 2040)]


@pytest.mark.parametrize("ta,tb,shape,M,N,K", [(ta, tb, *c) for ta, tb in ((False, False), (False, True), (True, False)) for c in SMALL_TILES] +
                         [(False, True, 8, 584, 1712, 4496), (False, True, 8, 424, 2336, 4456)])
def test_gemm_bf16_k_split_tiles_with_a_partial_last_k_tile(ctx, ta, tb, shape, M, N, K):
    """The tiles whose four waves split a K tile (64x64, 32x64, 32x32, 64x128), in the library's own choice: shorter than
    one 16-wide step, than one tile, fewer tiles than ring stages, many, on operands with NaN past K; ragged M and N;
    the same bits from run to run."""
    epi = P.EPI_ACCUM_F32 if ta else P.EPI_NONE
    assert U.gemm_plan("bf16", ta, tb, M, N, K, epi, ws_bytes=256 << 20)[0] == U.PLAN_TILE + shape
    key = ("k-split tile", ta, tb, M, N, K)
    print(key, flush=True)
    a, A = _nan_past_k(key + ("a",), M, K, not ta, 1.0)
    b, B = _nan_past_k(key + ("b",), N, K, tb, 0.05)
    c0 = mat(key + ("c0",), (M, N), "f32")
    outs = [dev(c0, "f32" if ta else "bf16") for _ in range(2)]
    for c in outs:
        _gemm_views(ctx, ta, tb, M, N, K, a, b, c, epi)
    torch.cuda.synchronize()
    assert torch.equal(outs[0], outs[1])
    assert_close(host(outs[0]), A @ B.T + (c0 if ta else 0.0), "f32" if ta else "bf16", str(key))


@pytest.mark.parametrize("ta,tb,epi", [(False, False, P.EPI_BIAS_RESID), (False, False, P.EPI_BIAS_GELU_GRAD), (False, True, P.EPI_MUL)])
@pytest.mark.parametrize("M,N,K", [(72, 200, 104), (264, 520, 1000), (520, 1032, 104)])
def test_gemm_bf16_epilogue_operands_aligned_to_eight_bytes(ctx, ta, tb, epi, M, N, K):
    """Bias, residual and second output need 8-byte alignment and a pitch in whole groups of four elements, no more, also
    on the paths that a partial last K tile takes."""
    key = ("eight bytes", ta, tb, epi, M, N, K)
    print(key, flush=True)
    ldc = N + 4

    def off(m):                                          # rows of pitch N + 4 starting 8 bytes past a 16-byte boundary
        big = torch.zeros(m.shape[0] * ldc + 8, dtype=torch.bfloat16, device="cuda")
        v = torch.as_strided(big, m.shape, (ldc, 1), 4)
        v.copy_(dev(m, "bf16"))
        assert v.data_ptr() % 16 == 8
        return v

    a, b = mat(key + ("a",), (M, K), "bf16"), mat(key + ("b",), (N, K) if tb else (K, N), "bf16", 0.05)
    bias, extra = mat(key + ("bias",), (1, N), "bf16"), mat(key + ("x",), (M, N), "bf16")
    ref = a.astype(np.float64) @ (b.T if tb else b).astype(np.float64)
    c = torch.zeros(M, ldc, dtype=torch.bfloat16, device="cuda")
    bias_d, extra_d = off(bias), off(extra)
    da, db = dev(a, "bf16"), dev(b, "bf16")
    rc = P.lib.pmc_gemm(ctx, P.PMC_BF16, int(ta), int(tb), M, N, K, da.data_ptr(), K, db.data_ptr(), db.stride(0), c.data_ptr(), ldc,
                        epi, bias_d.data_ptr(), extra_d.data_ptr(), extra_d.data_ptr())
    torch.cuda.synchronize()
    assert rc == 0
    if epi == P.EPI_BIAS_RESID:
        want = ref + bias + extra
    elif epi == P.EPI_MUL:
        want = ref * extra
    else:
        want = OL.gelu_grad(ref + bias)
        assert_close(host(extra_d), OL.gelu(ref + bias), "bf16", str(key))
    assert_close(host(c)[:, :N], want, "bf16", str(key))
    assert not bool(c[:, N:].any())                      # nothing past the row


@pytest.mark.parametrize("ta,tb,epis", [(False, False, (P.EPI_BIAS, P.EPI_BIAS_RESID, P.EPI_BIAS_GELU_GRAD)),
                                        (False, True, (P.EPI_NONE, P.EPI_DGELU, P.EPI_MUL)),
                                        (True, False, (P.EPI_NONE, P.EPI_ACCUM_F32))])
# M, N, K: one tile, shorter than a 16-wide step, fewer K tiles than ring stages, odd and even numbers of K tiles with a
# partial last one (32x32, 32x64 and 64x64 tiles whose waves split K); 128x128 tiles with a four-stage ring; long K, cut
# into ranges or not, with a partial last K tile
@pytest.mark.parametrize("M,N,K", [(8, 8, 8), (40, 24, 104), (72, 200, 1000), (192, 256, 1088), (264, 520, 584), (488, 840, 840),
                                   (1032, 1000, 392), (1000, 3080, 456), (72, 136, 16392), (264, 1032, 9160)])
def test_gemm_bf16_library_choice_of_small_tiles(ctx, ta, tb, epis, M, N, K):
    for epi in epis:
        _gemm_case(ctx, "bf16", ta, tb, M, N, K, epi)


def test_gemm_grouped_weight_gradient_rejects_bad_arguments(ctx):
    a = [torch.zeros(64, 128, device="cuda", dtype=torch.bfloat16)]
    b = [torch.zeros(64, 128, device="cuda", dtype=torch.bfloat16)]
    c = torch.zeros(128, 128, device="cuda", dtype=torch.float32)
    with pytest.raises(P.PmcError):
        P.pmc_gemm_grouped_wgrad(ctx, a * 9, b * 9, c)                       # more pieces than PMC_MAX_QUEUED_W
    a32 = [torch.zeros(32, 128, device="cuda", dtype=torch.bfloat16)]
    with pytest.raises(P.PmcError):
        P.pmc_gemm_grouped_wgrad(ctx, a32, a32, c)                           # K not in whole 64-wide tiles


@pytest.mark.parametrize("ta,tb", [(False, False), (False, True), (True, False)])
def test_gemm_bf16_large_tiles(ctx, ta, tb):
    # enough 256x256 tiles to take the large-tile path, ragged edge tiles included
    for epi in ((P.EPI_BIAS_GELU, P.EPI_BIAS_RESID) if not ta and not tb else
                (P.EPI_DGELU, P.EPI_NONE) if not ta else (P.EPI_ACCUM_F32,)):
        _gemm_case(ctx, "bf16", ta, tb, 3848, 3592, 200, epi)


def test_gemm_rejects_bad_arguments(ctx):
    a = torch.zeros(16, 16, device="cuda", dtype=torch.bfloat16)
    c = torch.zeros(16, 12, device="cuda", dtype=torch.bfloat16)
    with pytest.raises(P.PmcError) as e:
        P.pmc_gemm(ctx, a, a[:, :12].contiguous(), c)          # N = 12 is not a multiple of 8
    assert e.value.code == P.PMC_ERR_INVALID
    with pytest.raises(P.PmcError):
        P.pmc_gemm(ctx, a, a, torch.zeros(16, 16, device="cuda", dtype=torch.bfloat16), epilogue=P.EPI_BIAS)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("rows,h", [(37, 16), (64, 256), (5, 320), (1100, 1032), (130, 2048), (2100, 4096), (33, 5120), (9, 8192),
                                    (7, 9000), (17, 10240), (6, 12288), (2, 12296), (4096, 5120)])
def test_layernorm_forward_backward(ctx, dtype, rows, h):
    if h > (6144 if dtype == "f32" else 12288):
        # a wave keeps its row in registers: 24 vectors of 16 bytes per lane at most
        td = torch.float32 if dtype == "f32" else torch.bfloat16
        with pytest.raises(P.PmcError):
            P.pmc_layernorm_forward(ctx, *[torch.zeros(rows, h, device="cuda", dtype=td)] + [torch.zeros(h, device="cuda", dtype=td)] * 2,
                                    1e-5, torch.zeros(rows, h, device="cuda", dtype=td), torch.zeros(rows, device="cuda"),
                                    torch.zeros(rows, device="cuda"))
        return
    key = ("ln", dtype, rows, h)
    print("layernorm case", key, flush=True)
    x = mat(key + ("x",), (rows, h), dtype, 2.0)
    g = mat(key + ("g",), (h,), "f32", 0.1) + 1.0
    if dtype == "bf16":
        g = synth.round_to_bf16(g)
    b = mat(key + ("b",), (h,), dtype, 0.1)
    dy = mat(key + ("dy",), (rows, h), dtype)
    resid = mat(key + ("res",), (rows, h), dtype)
    eps = 1e-5
    y_ref, xhat, rstd = OL.layer_norm(x.astype(np.float64), g.astype(np.float64), b.astype(np.float64), eps)
    dx_ref, dg_ref, db_ref = OL.layer_norm_input_grad(dy.astype(np.float64), xhat, rstd, g.astype(np.float64))
    dx_ref = dx_ref + resid
    xd, y = dev(x, dtype), dev(np.zeros_like(x), dtype)
    xc = dev(np.zeros_like(x), dtype)
    mean = torch.zeros(rows, device="cuda")
    rs = torch.zeros(rows, device="cuda")
    P.pmc_layernorm_forward(ctx, xd, dev(g, dtype), dev(b, dtype), eps, y, mean, rs, xc)
    torch.cuda.synchronize()
    assert_close(host(y), y_ref, dtype, "")
    assert np.abs(host(mean) - x.astype(np.float64).mean(-1)).max() <= 1e-5
    assert rel_l2(host(rs), rstd[:, 0]) <= 1e-5
    assert torch.equal(xc, xd)
    dgain = torch.full((h,), 0.25, device="cuda")
    dbias = torch.full((h,), -0.5, device="cuda")
    dx = xd.clone()                      # in place over x, as the B pass does
    P.pmc_layernorm_backward(ctx, dev(dy, dtype), dx, dev(g, dtype), mean, rs, dev(resid, dtype), dx, dgain, dbias)
    torch.cuda.synchronize()
    assert_close(host(dx), dx_ref, dtype, "")
    assert_close(host(dgain) - 0.25, dg_ref, dtype, "dgain", whole_tol=5e-3 if dtype == "bf16" else 1e-5)
    assert_close(host(dbias) + 0.5, db_ref, "f32", "dbias")


# dtype, batch, seq, heads, head size: one row, one row past a block, and sizes that between them reach every forward shape, both kinds of the
# one-launch backward pass and every family of the two launches, in 64- and 128-wide tiles (a host test says so)
ATTN_SHAPES = [("bf16", 1, 8, 1, 64), ("bf16", 1, 64, 3, 128), ("bf16", 1, 65, 2, 128), ("bf16", 2, 192, 3, 64), ("bf16", 3, 200, 5, 112),
               ("bf16", 1, 264, 8, 128), ("bf16", 2, 520, 14, 40), ("bf16", 1, 1024, 16, 64), ("bf16", 1, 1032, 16, 64), ("bf16", 8, 72, 24, 64),
               ("bf16", 9, 136, 16, 128), ("bf16", 4, 328, 15, 128), ("bf16", 4, 328, 16, 72), ("bf16", 8, 64, 64, 32), ("bf16", 9, 64, 57, 16),
               ("bf16", 1, 704, 50, 16), ("bf16", 1, 1544, 16, 72), ("bf16", 1, 3080, 8, 72), ("bf16", 4, 136, 12, 128), ("bf16", 4, 100, 24, 64),
               ("bf16", 8, 256, 25, 72), ("bf16", 8, 252, 25, 40), ("bf16", 2, 704, 25, 72), ("bf16", 8, 200, 33, 72), ("bf16", 1, 328, 20, 40),
               ("f32", 1, 4, 1, 64), ("f32", 1, 256, 16, 20), ("f32", 1, 260, 16, 20), ("bf16", 1, 264, 8, 20), ("f32", 2, 68, 3, 128)]


@pytest.mark.parametrize("case", ATTN_SHAPES, ids=lambda c: "-".join(map(str, c)))
@pytest.mark.parametrize("causal", [True, False])
def test_attention_picked_launch_shapes(ctx, case, causal):
    """Forward; backward apart from qkv, where few blocks run as one launch, and in place; all against the oracle, and bit for bit the
    same where one launch and two have the same workgroups (kind 1 and family 0, kind 2 and family 3) or both are two."""
    dtype, batch, seq, heads, dh = case
    h = heads * dh
    print("one-launch attention case", case, causal, flush=True)
    qkv = mat(("merged", case, causal, "qkv"), (batch * seq, 3 * h), dtype)
    d_o = mat(("merged", case, causal, "do"), (batch * seq, h), dtype)
    q64 = qkv.astype(np.float64)
    o_ref, probs, _ = OL.attention(q64, heads, causal, batch)
    want = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
    qd, dod = dev(qkv, dtype), dev(d_o, dtype)
    o, lse = dev(np.zeros((batch * seq, h)), dtype), torch.zeros(batch * heads * seq, device="cuda")
    P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
    apart, inplace = torch.full_like(qd, float("nan")), qd.clone()
    P.pmc_attention_backward(ctx, qd, o, lse, dod, apart, batch, seq, heads, dh, causal)
    P.pmc_attention_backward(ctx, inplace, o, lse, dod, inplace, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    assert_close(host(o), o_ref, dtype, "o")
    for got in (apart, inplace):
        assert_close(host(got), want, dtype, "dqkv", scale=np.sqrt(np.mean(want ** 2)))
    kind, family = U.attention_plan(batch, seq, heads, dh, causal)[1:]
    if dtype == "f32" or dh % 8 or (kind, family) != (2, 0):
        assert torch.equal(apart, inplace)


@pytest.mark.parametrize("spread", [0.5, 1.0, 2.0])
@pytest.mark.parametrize("batch,seq,heads,dh,causal", [(8, 128, 16, 64, False), (8, 64, 16, 128, False), (1, 192, 16, 128, True), (4, 147, 16, 64, False),
                                                       (2, 333, 32, 112, False), (8, 520, 8, 64, True), (1, 1024, 33, 128, True), (1, 1100, 40, 40, False)])
def test_attention_forward_error_of_every_shape(ctx, tune, batch, seq, heads, dh, causal, spread):
    """Whatever shape is picked for a call of less than 512 128-row workgroups, its output is as close to 64 bits as that of the eight-wave shape, whose
    four key groups give every query four probabilities that bf16 holds exactly.  The rounding errors themselves differ:
    over n outputs the ratio of two error norms scatters by about 1 / sqrt(n), n >= 10^5 here, so 1 % is three times that."""
    assert -(-seq // 128) * heads * batch < 512
    h = heads * dh
    print("attention forward error", batch, seq, heads, dh, causal, spread, U.attention_plan(batch, seq, heads, dh, causal)[0], flush=True)
    gen = torch.Generator(device="cuda").manual_seed(seq)
    qkv = torch.randn(batch * seq, 3 * h, device="cuda", generator=gen)
    qkv[:, :2 * h] *= spread
    qkv = qkv.bfloat16()
    q, k, v = [t.reshape(batch, seq, heads, dh).permute(0, 2, 1, 3).double().contiguous() for t in qkv.reshape(batch * seq, 3, h).unbind(1)]
    s = q @ k.transpose(-1, -2).contiguous() / dh ** 0.5
    if causal:
        s.masked_fill_(torch.ones(seq, seq, device="cuda", dtype=torch.bool).triu(1), float("-inf"))
    want = (torch.softmax(s, -1) @ v).permute(0, 2, 1, 3).reshape(batch * seq, h)
    want_lse = torch.logsumexp(s, -1).reshape(-1)

    def error():
        o, lse = torch.full_like(qkv[:, :h], float("nan")).contiguous(), torch.full((batch * heads * seq,), float("nan"), device="cuda")
        P.pmc_attention_forward(ctx, qkv, o, lse, batch, seq, heads, dh, causal)
        torch.cuda.synchronize()
        assert float((lse.double() - want_lse).abs().max()) <= 2e-5
        return float((o.double() - want).norm())

    picked = error()
    tune(attn_shape=0)
    assert picked <= 1.01 * error()


@pytest.mark.parametrize("dtype,dh", [("f32", 4), ("f32", 16), ("f32", 64), ("f32", 128), ("bf16", 64), ("bf16", 128),
                                      ("bf16", 8), ("bf16", 40), ("bf16", 96), ("bf16", 112)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_forward_backward(ctx, dtype, dh, causal):
    batch, seq, heads = 2, 88, 3
    if dh == 4:
        seq = 24                                     # vectors of 4 fp32: hidden must be a multiple of 4
    h = heads * dh
    key = ("attn", dtype, dh, causal)
    print("attention case", key, flush=True)
    qkv = mat(key + ("qkv",), (batch * seq, 3 * h), dtype)
    d_o = mat(key + ("do",), (batch * seq, h), dtype)
    q64 = qkv.astype(np.float64)
    o_ref, probs, lse_ref = OL.attention(q64, heads, causal, batch)
    dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
    qd = dev(qkv, dtype)
    o = dev(np.zeros((batch * seq, h)), dtype)
    lse = torch.zeros(batch * heads * seq, device="cuda")
    P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    assert_close(host(o), o_ref, dtype, "")
    assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= (2e-2 if dtype == "bf16" else 2e-5)
    # separate output buffer
    dq = dev(np.zeros_like(qkv), dtype)
    P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, dtype), dq, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
        assert_close(host(dq)[:, cols], dqkv_ref[:, cols], dtype, str(name), scale=np.sqrt(np.mean(dqkv_ref ** 2)))
    # in place over qkv, as the B pass does
    inplace = qd.clone()
    P.pmc_attention_backward(ctx, inplace, o, lse, dev(d_o, dtype), inplace, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    assert torch.equal(inplace, dq)


@pytest.mark.parametrize("dtype,heads,dh", [("f32", 4, 3), ("f32", 2, 66), ("f32", 2, 64), ("bf16", 4, 6), ("bf16", 2, 20),
                                            ("bf16", 8, 101)])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_fp32_matrix_path(ctx, dtype, heads, dh, causal):
    """The kernels of the fp32 matrix instruction: head sizes with and without whole aligned groups of four
    columns, on both sides of the 64-column tile; one row, one row past a 16-row block, and more 16-row
    groups than the eight waves of a workgroup."""
    for seq in (1, 17, 145):
        batch, h = (8 if dtype == "bf16" else 4), heads * dh
        key = ("attn-f32path", dtype, heads, dh, causal, seq)
        print("attention case", key, flush=True)
        qkv = mat(key + ("qkv",), (batch * seq, 3 * h), dtype)
        d_o = mat(key + ("do",), (batch * seq, h), dtype)
        q64 = qkv.astype(np.float64)
        o_ref, probs, lse_ref = OL.attention(q64, heads, causal, batch)
        dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
        qd = dev(qkv, dtype)
        o = dev(np.zeros((batch * seq, h)), dtype)
        lse = torch.zeros(batch * heads * seq, device="cuda")
        P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
        P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, dtype), qd, batch, seq, heads, dh, causal)
        torch.cuda.synchronize()
        assert_close(host(o), o_ref, dtype, str(key))
        assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= (2e-2 if dtype == "bf16" else 2e-5)
        for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
            assert_close(host(qd)[:, cols], dqkv_ref[:, cols], dtype, name, scale=np.sqrt(np.mean(dqkv_ref ** 2)))


def test_attention_fp32_more_workgroups_than_one_dimension_holds(ctx):
    """2^23 (row block, head, sequence) triples and more, 512 threads each, would be 2^32 threads in one launch
    dimension.  One-token sequences: o = v, lse = q k / sqrt(dh), dv = dO, no gradient in q and k, element by element."""
    batch, heads, dh = 65535, 132, 1
    gen = torch.Generator(device="cuda").manual_seed(11)
    qkv = torch.randn(batch, 3 * heads, device="cuda", generator=gen)
    d_o = torch.randn(batch, heads, device="cuda", generator=gen)
    o, lse = torch.full_like(d_o, float("nan")), torch.full((batch * heads,), float("nan"), device="cuda")
    print("fp32 attention, one-token sequences", batch, heads, flush=True)
    P.pmc_attention_forward(ctx, qkv, o, lse, batch, 1, heads, dh, True)
    torch.cuda.synchronize()
    q, k, v = qkv.view(batch, 3, heads).unbind(1)
    assert torch.equal(o, v)
    # one product, and the product with sqrt(1)
    assert bool(((lse.view(batch, heads).double() - q.double() * k.double()).abs() <= 2.0 ** -22 * (q * k).abs().double() + 1e-30).all())
    dqkv = torch.full_like(qkv, float("nan"))
    P.pmc_attention_backward(ctx, qkv, o, lse, d_o, dqkv, batch, 1, heads, dh, True)
    torch.cuda.synchronize()
    dq, dk, dv = dqkv.view(batch, 3, heads).unbind(1)
    # P = exp(s - lse) is 1 up to the rounding of its argument, |s| <= 30 here: 30 * 2^-23
    assert bool(((dv - d_o).abs() <= 4e-6 * d_o.abs()).all())
    assert float(dq.abs().max()) <= 1e-5 and float(dk.abs().max()) <= 1e-5


@pytest.mark.timeout(300)
def test_attention_fp32_more_row_blocks_than_one_launch_takes(ctx):
    """A sequence of more than 65535 blocks of 16 rows goes out in several launches.  With q = 0 the causal
    probabilities of row i are all 1 / (i + 1), so outputs and gradients are running sums (float64)."""
    seq, dh = 65535 * 16 + 21, 4
    gen = torch.Generator(device="cuda").manual_seed(12)
    qkv = torch.randn(seq, 3 * dh, device="cuda", generator=gen)
    qkv[:, :dh] = 0
    qkv[:, 2 * dh:] += 0.5
    d_o = torch.randn(seq, dh, device="cuda", generator=gen)
    o, lse = torch.zeros_like(d_o), torch.zeros(seq, device="cuda")
    print("fp32 attention, one sequence of", seq, flush=True)
    P.pmc_attention_forward(ctx, qkv, o, lse, 1, seq, 1, dh, True)
    torch.cuda.synchronize()
    print("forward done", flush=True)
    P.pmc_attention_backward(ctx, qkv, o, lse, d_o, dqkv := torch.zeros_like(qkv), 1, seq, 1, dh, True)
    torch.cuda.synchronize()
    k, v, g = qkv[:, dh:2 * dh].double(), qkv[:, 2 * dh:].double(), d_o.double()
    n = torch.arange(1, seq + 1, device="cuda", dtype=torch.float64)[:, None]
    want_o = v.cumsum(0) / n
    delta = (g * want_o).sum(1, keepdim=True)
    pairs = (v[:, :, None] * k[:, None, :]).cumsum(0)
    want_dq = ((g[:, :, None] * pairs).sum(1) - delta * k.cumsum(0)) / n / dh ** 0.5
    want_dv = (g / n).flip(0).cumsum(0).flip(0)
    assert float((lse.double() - n[:, 0].log()).abs().max()) <= 2e-5
    assert_close(host(o), want_o.cpu().numpy(), "f32", "o")
    assert_close(host(dqkv)[:, :dh], want_dq.cpu().numpy(), "f32", "dq")
    # a wave adds up to seq / 8 terms one after the other, each time rounded by up to 2^-24 of a partial sum that the
    # terms' absolute values bound: independent roundings grow with the root of their number
    bound = (seq / 8) ** 0.5 * 2.0 ** -24 * (g / n).abs().flip(0).cumsum(0).flip(0)
    assert bool(((dqkv[:, 2 * dh:].double() - want_dv).abs() <= bound).all())
    assert float(dqkv[:, dh:2 * dh].abs().max()) == 0.0


def test_attention_random_shapes(ctx):
    """Seeded random batch, sequence length, head count and head size (every multiple of 8 up to 128),
    causal or not, in the library's own choice of launch shape: ragged last blocks, sequences shorter
    than a block, padded head sizes."""
    rng = np.random.default_rng(1536205)
    for i in range(12):
        batch, heads = int(rng.integers(1, 4)), int(rng.integers(1, 5))
        seq, dh, causal = int(rng.integers(1, 600)), int(8 * rng.integers(1, 17)), bool(rng.integers(0, 2))
        h = heads * dh
        key = ("attn-random", i)
        print("attention random case", batch, seq, heads, dh, causal, flush=True)
        qkv = mat(key + ("qkv",), (batch * seq, 3 * h), "bf16")
        d_o = mat(key + ("do",), (batch * seq, h), "bf16")
        q64 = qkv.astype(np.float64)
        o_ref, probs, lse_ref = OL.attention(q64, heads, causal, batch)
        dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
        qd = dev(qkv, "bf16")
        o = dev(np.zeros((batch * seq, h)), "bf16")
        lse = torch.zeros(batch * heads * seq, device="cuda")
        P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
        dq = dev(np.zeros_like(qkv), "bf16")
        P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, "bf16"), dq, batch, seq, heads, dh, causal)
        torch.cuda.synchronize()
        assert_close(host(o), o_ref, "bf16", f"random {i} o")
        assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= 2e-2, i
        scale = np.sqrt(np.mean(dqkv_ref ** 2))
        for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
            assert_close(host(dq)[:, cols], dqkv_ref[:, cols], "bf16", f"random {i} {name}", scale=scale)


@pytest.mark.parametrize("family", [0, 1, 2])
@pytest.mark.parametrize("dh,causal", [(128, True), (64, True), (128, False), (112, True), (48, False)])
def test_attention_launch_shapes(ctx, tune, family, dh, causal):
    """Every family of workgroup shapes (key/query splits, merges through LDS) on a ragged
    sequence that spans several streamed blocks; the library reads the override at each call.
    Head sizes 112 and 48 run in the 128- and 64-wide tiles with the remaining columns held at zero
    (112 = hidden 7168 over 64 heads, one of the paper's model shapes)."""
    tune(attn_shape=family)
    batch, seq, heads = 2, 333, 2
    h = heads * dh
    key = ("attn-shape", dh, causal)
    print("attention shape case", key, family, flush=True)
    qkv = mat(key + ("qkv",), (batch * seq, 3 * h), "bf16")
    d_o = mat(key + ("do",), (batch * seq, h), "bf16")
    q64 = qkv.astype(np.float64)
    o_ref, probs, lse_ref = OL.attention(q64, heads, causal, batch)
    dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
    qd = dev(qkv, "bf16")
    o = dev(np.zeros((batch * seq, h)), "bf16")
    lse = torch.zeros(batch * heads * seq, device="cuda")
    P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    assert_close(host(o), o_ref, "bf16", "")
    assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= 2e-2
    dq = dev(np.zeros_like(qkv), "bf16")
    P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, "bf16"), dq, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
        assert_close(host(dq)[:, cols], dqkv_ref[:, cols], "bf16", str(name), scale=np.sqrt(np.mean(dqkv_ref ** 2)))


@pytest.mark.parametrize("family", [0, 1])
def test_attention_long_sequence(ctx, tune, family):
    """Sequence length 4096 at head size 128 (the longest workload shape), four heads so that the
    oracle's probabilities fit in host memory: 32 to 64 streamed blocks per query block, the
    heaviest-first block order, both families of launch shapes."""
    tune(attn_shape=family)
    batch, seq, heads, dh = 1, 4096, 4, 128
    h = heads * dh
    key = ("attn-long",)
    print("attention long case", family, flush=True)
    qkv = mat(key + ("qkv",), (seq, 3 * h), "bf16")
    d_o = mat(key + ("do",), (seq, h), "bf16")
    q64 = qkv.astype(np.float64)
    o_ref, probs, lse_ref = OL.attention(q64, heads, True, batch)
    dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
    del probs
    qd = dev(qkv, "bf16")
    o = dev(np.zeros((seq, h)), "bf16")
    lse = torch.zeros(heads * seq, device="cuda")
    P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, True)
    torch.cuda.synchronize()
    assert_close(host(o), o_ref, "bf16", "")
    assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= 2e-2
    dq = dev(np.zeros_like(qkv), "bf16")
    P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, "bf16"), dq, batch, seq, heads, dh, True)
    torch.cuda.synchronize()
    for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
        assert_close(host(dq)[:, cols], dqkv_ref[:, cols], "bf16", str(name), scale=np.sqrt(np.mean(dqkv_ref ** 2)))


@pytest.mark.timeout(600)
@pytest.mark.parametrize("seq,heads", [(4096, 40), (2048, 32), (1024, 16)])
def test_attention_workload_shapes(ctx, seq, heads):
    """Attention at the full size of the three bf16 workloads (head size 128, causal), launched as the
    passes launch it (the library's own choice of workgroup shapes for that many heads and blocks).
    The dense oracle for all heads at once would need heads x seq^2 probabilities, so heads are checked
    one at a time, each as a one-head problem cut out of the packed q|k|v rows: output, log-sum-exp and
    all three input gradients, every element.  At the longest shape (4096 tokens, 40 heads) EVERY head
    is checked; at the two shorter ones the first, the last and one in between."""
    dh = 128
    h = heads * dh
    gen = torch.Generator(device="cuda").manual_seed(seq + heads)
    bf = torch.bfloat16
    qkv = torch.randn((seq, 3 * h), device="cuda", generator=gen).to(bf)
    d_o = torch.randn((seq, h), device="cuda", generator=gen).to(bf)
    o = torch.zeros((seq, h), device="cuda", dtype=bf)
    lse = torch.zeros(heads * seq, device="cuda")
    dq = torch.zeros_like(qkv)
    print("attention workload shape", seq, heads, flush=True)
    P.pmc_attention_forward(ctx, qkv, o, lse, 1, seq, heads, dh, True)
    P.pmc_attention_backward(ctx, qkv, o, lse, d_o, dq, 1, seq, heads, dh, True)
    torch.cuda.synchronize()
    lse_h = host(lse).reshape(heads, seq)
    for hd in (range(heads) if seq == 4096 else (0, heads // 2 + 1, heads - 1)):
        cols = [slice(part * h + hd * dh, part * h + (hd + 1) * dh) for part in range(3)]
        one = np.concatenate([host(qkv[:, c]) for c in cols], axis=1)              # [seq, 3 dh]: a one-head qkv
        o_ref, probs, lse_ref = OL.attention(one, 1, True, 1)
        g_ref = OL.attention_input_grad(host(d_o[:, hd * dh:(hd + 1) * dh]), one, probs, 1, 1)
        del probs
        assert_close(host(o[:, hd * dh:(hd + 1) * dh]), o_ref, "bf16", str(hd))
        assert np.abs(lse_h[hd] - lse_ref.reshape(-1)).max() <= 2e-2, hd
        for part, name in enumerate(("dq", "dk", "dv")):
            assert_close(host(dq[:, cols[part]]), g_ref[:, part * dh:(part + 1) * dh], "bf16", str((hd, name)), scale=np.sqrt(np.mean(g_ref ** 2)))


@pytest.mark.parametrize("family", [0, 1, 2])
@pytest.mark.parametrize("dh", [64, 128])
def test_attention_short_sequences(ctx, tune, family, dh):
    """Sequences shorter than one streamed block (a single query, a few, one 32-row tile plus
    one): every tile row past the end is a clamped copy of the last row and must be masked out."""
    tune(attn_shape=family)
    batch, heads = 2, 2
    h = heads * dh
    for seq in (1, 7, 33):
        key = ("attn-short", dh, seq)
        print("attention short case", key, family, flush=True)
        qkv = mat(key + ("qkv",), (batch * seq, 3 * h), "bf16")
        d_o = mat(key + ("do",), (batch * seq, h), "bf16")
        q64 = qkv.astype(np.float64)
        o_ref, probs, lse_ref = OL.attention(q64, heads, True, batch)
        dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
        qd = dev(qkv, "bf16")
        o = dev(np.zeros((batch * seq, h)), "bf16")
        lse = torch.zeros(batch * heads * seq, device="cuda")
        P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, True)
        torch.cuda.synchronize()
        assert_close(host(o), o_ref, "bf16", str(seq))
        assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= 2e-2, seq
        dq = dev(np.zeros_like(qkv), "bf16")
        P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, "bf16"), dq, batch, seq, heads, dh, True)
        torch.cuda.synchronize()
        for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
            assert_close(host(dq)[:, cols], dqkv_ref[:, cols], "bf16", str((seq, name)), scale=np.sqrt(np.mean(dqkv_ref ** 2)))


@pytest.mark.parametrize("family", [0, 1])
@pytest.mark.parametrize("causal", [True, False])
def test_attention_sharp_softmax(ctx, tune, family, causal):
    """Queries and keys three times larger (scores with a standard deviation of 9, 13 in log2
    units): row maxima keep rising from block to block by more and by less than the slack the
    forward kernel allows before it moves its softmax reference, so both branches of the online
    softmax and their mix inside one wave are exercised."""
    tune(attn_shape=family)
    batch, seq, heads, dh = 1, 700, 2, 128
    h = heads * dh
    key = ("attn-sharp", causal)
    print("attention sharp case", key, family, flush=True)
    qkv = mat(key + ("qkv",), (batch * seq, 3 * h), "bf16").copy()
    qkv[:, :2 * h] *= 3.0
    d_o = mat(key + ("do",), (batch * seq, h), "bf16")
    qkv = host(dev(qkv, "bf16"))                             # exactly what the device holds after rounding
    q64 = qkv.astype(np.float64)
    o_ref, probs, lse_ref = OL.attention(q64, heads, causal, batch)
    dqkv_ref = OL.attention_input_grad(d_o.astype(np.float64), q64, probs, heads, batch)
    qd = dev(qkv, "bf16")
    o = dev(np.zeros((batch * seq, h)), "bf16")
    lse = torch.zeros(batch * heads * seq, device="cuda")
    P.pmc_attention_forward(ctx, qd, o, lse, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    assert_close(host(o), o_ref, "bf16", "")
    assert np.abs(host(lse) - lse_ref.reshape(-1)).max() <= 2e-2
    dq = dev(np.zeros_like(qkv), "bf16")
    P.pmc_attention_backward(ctx, qd, o, lse, dev(d_o, "bf16"), dq, batch, seq, heads, dh, causal)
    torch.cuda.synchronize()
    for name, cols in (("dq", slice(0, h)), ("dk", slice(h, 2 * h)), ("dv", slice(2 * h, 3 * h))):
        assert_close(host(dq)[:, cols], dqkv_ref[:, cols], "bf16", str(name), scale=np.sqrt(np.mean(dqkv_ref ** 2)))


def test_attention_rejects_rows_beyond_the_load_window(ctx):
    """The matrix-core kernels address one sequence's q|k|v rows with 32-bit offsets in a 2 GB
    window: a sequence whose rows exceed it is refused before anything is launched."""
    seq, heads, dh = 32768, 128, 128                    # 32768 rows of 96 KiB = 3 GiB
    small = torch.zeros(1024, device="cuda", dtype=torch.bfloat16)
    lse = torch.zeros(16, device="cuda")
    with pytest.raises(P.PmcError) as e:
        P.pmc_attention_forward(ctx, small, small, lse, 1, seq, heads, dh, True)
    assert "2 GB" in str(e.value)
    with pytest.raises(P.PmcError):
        P.pmc_attention_backward(ctx, small, small, lse, small, small, 1, seq, heads, dh, True)


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
def test_column_sum(ctx, dtype):
    for rows, n in ((1, 8), (50, 264), (1000, 2048), (300, 6144)):
        a = mat(("cs", dtype, rows, n), (rows, n), dtype)
        out = torch.full((n,), 2.0, device="cuda")
        P.pmc_column_sum(ctx, dev(a, dtype), out)
        torch.cuda.synchronize()
        assert np.abs(host(out) - 2.0 - a.astype(np.float64).sum(0)).max() <= 1e-4 * max(1.0, np.sqrt(rows))
