"""GPU parity of tw_gemm_bf16 (the compute stand-in of the other token split,
TokenWeave Fig. 7b) against the fp64 textbook product, and of tw_overlap_launch
against the two calls made one after the other.

Tolerance for C (bf16, fp32 accumulation over K): the rounding to bf16 costs up
to 2^-8 relative; fp32 accumulation of K products of magnitude ~sa*sb adds an
absolute error of about K * 2^-24 * sa * sb in the worst case, far below
1e-3 * sqrt(K) * sa * sb. So: |gpu - ref| <= 1e-2 |ref| + 1e-3 * sqrt(K) * sa * sb."""
import numpy as np
import pytest

import oracle
import tw_workloads as W
from helpers import captured_grids, captured_kernels, to_bits, to_gpu

pytestmark = pytest.mark.gpu


@pytest.fixture(scope="module")
def torch_cuda():
    import torch
    assert torch.cuda.is_available()
    return torch


def gemm_check(got_f64, ref_f64, K, std, what):
    tol = 1e-2 * np.abs(ref_f64) + 1e-3 * np.sqrt(max(K, 1)) * std * std
    bad = np.abs(got_f64 - ref_f64) > tol
    assert not bad.any(), "%s: %d of %d out of tolerance, first %s" % (
        what, bad.sum(), bad.size, np.argwhere(bad)[:1])


SHAPES = [(256, 128, 64), (64, 64, 64), (300, 200, 136), (1, 8, 8), (257, 136, 72), (512, 384, 1024),
          (33, 1000, 264), (700, 24, 4096)]


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,N,K", SHAPES)
def test_gemm_small_shapes_full_compare(tw, torch_cuda, M, N, K, layout):
    g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + N + K, b_layout=layout)
    code = tw.B_NK if layout == "nk" else tw.B_KN
    C = tw.gemm_bf16(to_gpu(g["A"]), to_gpu(g["B"]), b_layout=code)
    torch_cuda.cuda.synchronize()
    ref = oracle.gemm(g["A"], g["B"], layout)
    gemm_check(oracle.bf16_to_f64(to_bits(C)), ref, K, 0.5, "gemm %s %dx%dx%d" % (layout, M, N, K))
    # a budgeted (persistent) launch walks the same tiles: same bits
    C2 = tw.gemm_bf16(to_gpu(g["A"]), to_gpu(g["B"]), b_layout=code, cu_budget=3)
    torch_cuda.cuda.synchronize()
    assert np.array_equal(to_bits(C), to_bits(C2))


def test_gemm_both_layouts_give_the_same_bits(tw, torch_cuda):
    """B(k, n) is the same matrix whichever way it is stored, and both kernels
    multiply and add in the same order."""
    a = W.make_gemm_inputs(520, 1000, 392, 0.3, seed=11, b_layout="nk")
    b = W.make_gemm_inputs(520, 1000, 392, 0.3, seed=11, b_layout="kn")
    C1 = tw.gemm_bf16(to_gpu(a["A"]), to_gpu(a["B"]), b_layout=tw.B_NK)
    C2 = tw.gemm_bf16(to_gpu(b["A"]), to_gpu(b["B"]), b_layout=tw.B_KN)
    torch_cuda.cuda.synchronize()
    assert np.array_equal(to_bits(C1), to_bits(C2))


@pytest.mark.parametrize("M,N,K,budget,tile_nk,tile_kn", [
    (4096, 4096, 2048, 0, (256, 256), (256, 128)), (1000, 1096, 520, 10, (256, 256), (256, 128)),
    (2304, 2048, 4104, 72, (256, 256), (256, 128)), (513, 520, 96, 9, (256, 192), (192, 128)),
    (512, 512, 40, 4, (256, 256), (256, 128)), (768, 1024, 64, 6, (256, 256), (256, 128)),
    (520, 264, 200, 3, (256, 128), (192, 128))])
def test_gemm_large_product_tiles_give_the_same_bits(tw, torch_cuda, M, N, K, budget, tile_nk, tile_kn):
    """The tiles of large products launched on their own: 256 x 256 and 256 x 192 (four waves, K steps of 64,
    three LDS slots for A and two for B), and the 256 x 128 and 192 x 128 ones that the same product takes when
    it is stored [K x N]. Same bits (ragged edges and a K that is no multiple of the K step included),
    checked against the oracle on sampled outputs."""
    a = W.make_gemm_inputs(M, K, N, 0.05, seed=M + K, b_layout="nk")
    b = W.make_gemm_inputs(M, K, N, 0.05, seed=M + K, b_layout="kn")
    use = budget or tw.device_cu_count()
    assert tw.gemm_tile_choice(M, N, K, tw.B_NK, use) == tile_nk, "the case is meant to take other tiles"
    assert tw.gemm_tile_choice(M, N, K, tw.B_KN, use) == tile_kn
    C = torch_cuda.full((M, N), float("nan"), dtype=torch_cuda.bfloat16, device="cuda:0")
    tw.gemm_bf16(to_gpu(a["A"]), to_gpu(a["B"]), C=C, b_layout=tw.B_NK, cu_budget=budget)
    C2 = tw.gemm_bf16(to_gpu(b["A"]), to_gpu(b["B"]), b_layout=tw.B_KN, cu_budget=budget)
    torch_cuda.cuda.synchronize()
    Cb = to_bits(C)
    assert np.array_equal(Cb, to_bits(C2))
    rng = np.random.default_rng(M)
    ms = np.concatenate([rng.integers(0, M, 2040), [0, 0, M - 1, M - 1, min(255, M - 1), min(256, M - 1), M // 2, 1]])
    ns = np.concatenate([rng.integers(0, N, 2040), [0, N - 1, 0, N - 1, min(255, N - 1), min(256, N - 1), N // 2, 1]])
    ref = oracle.gemm_samples(a["A"], a["B"], "nk", ms, ns)
    gemm_check(oracle.bf16_to_f64(Cb[ms, ns]), ref, K, 0.05, "large-tile gemm %dx%dx%d" % (M, N, K))


# Sizes at the edges of the small tile shapes (16 ... 192 rows, 16 ... 128 columns, K steps of 64, 128, 256),
# with outputs enough for each of them to be the one that fills the compute units.
SMALL_TILE_SHAPES = [(1, 4096, 256), (15, 3592, 264), (17, 4104, 520), (33, 8, 2056), (64, 8200, 136), (65, 4104, 72),
                     (129, 1288, 328), (200, 3592, 264), (193, 8, 8), (333, 3600, 392), (335, 8200, 72), (500, 3608, 136),
                     (513, 4104, 264), (700, 8200, 328), (1023, 3592, 136)]


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,N,K", SMALL_TILE_SHAPES)
def test_gemm_of_few_rows_gives_the_bits_of_the_same_rows_of_a_large_product(tw, torch_cuda, M, N, K, layout):
    torch = torch_cuda
    rows = 4096          # enough for 256-row tiles
    g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + N + K, b_layout=layout)
    code = tw.B_NK if layout == "nk" else tw.B_KN
    A, B = to_gpu(g["A"]), to_gpu(g["B"])
    big = torch.cat([A, torch.ones((rows - M, K), dtype=torch.bfloat16, device="cuda:0")])
    want = to_bits(tw.gemm_bf16(big, B, b_layout=code)[:M])
    for budget in (0, 5):
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        tw.gemm_bf16(A, B, C, b_layout=code, cu_budget=budget)
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(C), want), "M=%d N=%d K=%d %s budget %d" % (M, N, K, layout, budget)
    rng = np.random.default_rng(M + N)
    ms, ns = rng.integers(0, M, 64), rng.integers(0, N, 64)
    ref = oracle.gemm_samples(g["A"], g["B"], layout, ms, ns)
    gemm_check(oracle.bf16_to_f64(want)[ms, ns], ref, K, 0.5, "sampled")


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,N", [(5, 4096), (64, 8192), (130, 3592), (500, 3608)])
def test_gemm_from_one_k_step_to_past_the_pipeline(tw, torch_cuda, M, N, layout):
    torch = torch_cuda
    code = tw.B_NK if layout == "nk" else tw.B_KN
    for K in (8, 64, 72, 128, 192, 256, 320, 384, 392, 448, 512, 640, 768, 1024, 1032, 1280, 1536, 1800):
        g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + K, b_layout=layout)
        A, B = to_gpu(g["A"]), to_gpu(g["B"])
        big = torch.cat([A, torch.ones((4096 - M, K), dtype=torch.bfloat16, device="cuda:0")])
        want = to_bits(tw.gemm_bf16(big, B, b_layout=code)[:M])
        for budget in (0, 7):
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
            tw.gemm_bf16(A, B, C, b_layout=code, cu_budget=budget)
            torch.cuda.synchronize()
            assert np.array_equal(to_bits(C), want), "M=%d N=%d K=%d %s budget %d" % (M, N, K, layout, budget)


def test_gemm_k_zero_gives_zeros(tw, torch_cuda):
    torch = torch_cuda
    for (M, N, budget) in ((40, 24, 0), (512, 512, 4)):      # 256 x 128 tiles, and 256 x 256
        assert tw.gemm_tile_choice(M, N, 0, tw.B_NK, budget or 256) == (256, 256 if budget else 128)
        A = torch.empty((M, 0), dtype=torch.bfloat16, device="cuda:0")
        B = torch.empty((N, 0), dtype=torch.bfloat16, device="cuda:0")
        C = torch.full((M, N), 7.0, dtype=torch.bfloat16, device="cuda:0")
        tw.gemm_bf16(A, B, C=C, cu_budget=budget)
        torch.cuda.synchronize()
        assert (to_bits(C) == 0).all()


def test_gemm_at_the_largest_k(tw, torch_cuda):
    """K = 2^22, the deepest product the entry point accepts, on the whole device: 16 x 16 tiles, whose rows
    of A start up to 2 GiB into it. Inputs drawn on the GPU; rows from the first to the last tile against the
    fp64 product of those rows."""
    torch = torch_cuda
    M, N, K, std = 256 + 3, 16, 1 << 22, 0.02
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(22)
    A = torch.empty((M, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    B = torch.empty((N, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    C = tw.gemm_bf16(A, B)
    torch.cuda.synchronize()
    rows = [0, 63, 64, 191, 255, 256, M - 1]
    ref = oracle.gemm(to_bits(A[rows]), to_bits(B), "nk")
    gemm_check(oracle.bf16_to_f64(to_bits(C[rows])), ref, K, std, "gemm at K = 2^22")
    assert np.count_nonzero(to_bits(C)) > 0.99 * M * N
    del A, B, C
    torch.cuda.empty_cache()


def _every_tile_shape():
    for rows, cols in NK_TILES:
        for layout in ("nk", "kn") if (rows, cols) in KN_TILES else ("nk",):
            yield rows, cols, layout


# the tile shapes that are built, by layout of B (and, below, sizes and budgets that take each of them)
KN_TILES = [(16, 32), (32, 32), (64, 32), (64, 64), (96, 64), (96, 128), (192, 64), (128, 128), (192, 128), (256, 128)]
NK_TILES = [(16, 16), (32, 16), (48, 32), (96, 96), (256, 64), (256, 192), (256, 256)] + KN_TILES


@pytest.mark.parametrize("rows,cols,layout", list(_every_tile_shape()))
def test_gemm_full_tile_of_the_largest_k(tw, torch_cuda, rows, cols, layout):
    """One full tile of each shape at K = 2^22: rows of 8 MiB, so that a tile of 256 rows is 2 GiB of A (and
    one of 256 columns 2 GiB of B), and every byte offset inside it still has to fit the 32 bits a buffer
    instruction adds up. On one compute unit, which makes each shape the choice for its own size. The first
    and last rows and columns and some between against the fp64 product, and all of it against the bits of
    the tiles that the whole device takes."""
    torch = torch_cuda
    K, std = 1 << 22, 0.02
    code = tw.B_NK if layout == "nk" else tw.B_KN
    assert tw.gemm_tile_choice(rows, cols, K, code, 1) == (rows, cols)
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(rows + cols)
    A = torch.empty((rows, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    Bnk = torch.empty((cols, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    B = Bnk if layout == "nk" else Bnk.t().contiguous()
    C = torch.full((rows, cols), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    tw.gemm_bf16(A, B, C=C, b_layout=code, cu_budget=1)
    other = tw.gemm_bf16(A, B, b_layout=code)
    torch.cuda.synchronize()
    assert rows * cols <= 1024 or tw.gemm_tile_choice(rows, cols, K, code, tw.device_cu_count()) != (rows, cols)
    assert np.array_equal(to_bits(C), to_bits(other))
    ms, ns = [0, rows // 2, rows - 1], [0, cols // 2 - 1, cols - 1]
    ref = oracle.gemm(to_bits(A[ms]), to_bits(Bnk[ns]), "nk")
    gemm_check(oracle.bf16_to_f64(to_bits(C[ms][:, ns])), ref, K, std, "%d x %d tile at K = 2^22" % (rows, cols))
    del A, B, Bnk, C
    torch.cuda.empty_cache()


# (tile, layouts, M, N, K, budget): ragged, several tiles per workgroup and K past the pipeline's depth where the
# shape is ever chosen for that.
TILE_CASES = [((16, 16), "nk", 17, 24, 1032, 4), ((16, 16), "nk", 1, 8, 200, 1),
              ((32, 16), "nk", 33, 24, 1032, 4), ((32, 16), "nk", 17, 8, 200, 1),
              ((16, 32), "nk", 9, 72, 1032, 4), ((16, 32), "both", 16, 72, 1000, 4), ((16, 32), "both", 1, 24, 200, 1),
              ((32, 32), "both", 33, 40, 1032, 4), ((32, 32), "both", 1, 8, 72, 1),
              ((48, 32), "nk", 33, 72, 2056, 3), ((48, 32), "nk", 48, 8, 2048, 1),
              ((64, 32), "both", 65, 40, 1032, 4), ((64, 32), "both", 33, 8, 72, 1),
              ((64, 64), "both", 65, 72, 1032, 4), ((64, 64), "both", 1, 40, 72, 1),
              ((96, 64), "both", 129, 72, 1032, 4), ((96, 64), "both", 1, 8, 8, 1),
              ((96, 96), "nk", 97, 136, 1032, 4), ((96, 96), "nk", 1, 264, 72, 1),
              ((96, 128), "both", 97, 200, 1032, 4), ((96, 128), "both", 1, 328, 72, 1),
              ((192, 64), "both", 300, 136, 1032, 6), ((192, 64), "both", 257, 8, 72, 1),
              ((128, 128), "both", 193, 136, 1032, 4), ((128, 128), "both", 97, 264, 72, 1),
              ((192, 128), "both", 257, 136, 1032, 4), ((192, 128), "both", 129, 72, 200, 1),
              ((256, 64), "nk", 389, 136, 1032, 6), ((256, 64), "nk", 389, 8, 72, 1),
              ((256, 128), "kn", 389, 136, 1032, 1), ((256, 128), "nk", 389, 136, 1032, 4),
              ((256, 128), "kn", 389, 8, 72, 1), ((256, 128), "nk", 257, 72, 72, 1),
              ((256, 192), "nk", 257, 264, 1032, 4), ((256, 192), "nk", 257, 136, 72, 1),
              ((256, 256), "nk", 257, 712, 1032, 2), ((256, 256), "nk", 257, 200, 72, 1)]


@pytest.mark.parametrize("tile,layouts,M,N,K,budget", TILE_CASES)
def test_gemm_every_tile_shape(tw, torch_cuda, tile, layouts, M, N, K, budget):
    for layout in ("nk", "kn") if layouts == "both" else (layouts,):
        code = tw.B_NK if layout == "nk" else tw.B_KN
        assert tw.gemm_tile_choice(M, N, K, code, budget) == tile
        g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + N + K, b_layout=layout)
        C = torch_cuda.full((M, N), float("nan"), dtype=torch_cuda.bfloat16, device="cuda:0")
        tw.gemm_bf16(to_gpu(g["A"]), to_gpu(g["B"]), C=C, b_layout=code, cu_budget=budget)
        torch_cuda.cuda.synchronize()
        ref = oracle.gemm(g["A"], g["B"], layout)
        gemm_check(oracle.bf16_to_f64(to_bits(C)), ref, K, 0.5, "%s tiles, %s %dx%dx%d" % (tile, layout, M, N, K))


# From which K on a shape has waves that only load where its launch has no helpers (not there: none without)
LOADING_FROM = {("kn", (16, 32)): 2048, ("nk", (16, 16)): 2048, ("nk", (32, 16)): 2048, ("nk", (32, 32)): 2048, ("nk", (64, 32)): 2048, ("nk", (64, 64)): 2048,
                ("nk", (96, 64)): 2048, ("nk", (96, 96)): 320, ("nk", (96, 128)): 512, ("kn", (32, 32)): 2048, ("kn", (64, 32)): 2048,
                ("kn", (96, 64)): 320, ("kn", (96, 128)): 512, ("kn", (192, 64)): 2048, ("kn", (128, 128)): 2048}


def assert_loading_waves(tw, tile, layout, M, N, budget, Ks):
    one_row = layout == "nk" and tile[1] <= 32 and tile[0] <= 32 and M <= tile[0]     # weights that are streamed
    for K in Ks:
        plan = tw.gemm_plan(M, N, K, tw.B_NK if layout == "nk" else tw.B_KN, budget)
        assert (plan.tile_m, plan.tile_n) == tile and plan.helpers == 0
        has = K >= LOADING_FROM.get((layout, tile), 1 << 30) and not one_row
        assert plan.loading_waves == (4 if has else 0), (tile, layout, K)


# (tile, layouts, M, N, budget, K): around each K from which on a shape has waves that only load, and every number of K
# steps from there past a whole round of its LDS stages (three to six steps of 64 to 256)
LOADING_CASES = [(c[0], c[1], c[2], c[3], c[5], (2040, 2048, 2056, 2120, 2184, 2304, 2440, 2568))
                 for c in TILE_CASES if c[0][0] < 256 and c[4] == 1032]
LOADING_CASES += [(tile, layouts, M, N, budget, (312, 320, 328, 384, 392, 448, 512, 576, 584, 640))
                  for tile, layouts, M, N, budget in (((96, 96), "nk", 97, 136, 4), ((96, 96), "nk", 1, 264, 1),
                                                      ((96, 64), "kn", 129, 72, 4))]
LOADING_CASES += [((16, 32), "kn", 9, 72, 4, (1976, 2040, 2048, 2184, 2304, 2440, 2560))]
LOADING_CASES += [((96, 128), "both", M, N, budget, (504, 512, 520, 576, 584, 640))
                  for M, N, budget in ((97, 200, 4), (1, 328, 1))]


@pytest.mark.parametrize("tile,layouts,M,N,budget,Ks", LOADING_CASES)
def test_gemm_tiles_with_loading_waves(tw, torch_cuda, tile, layouts, M, N, budget, Ks):
    """Both sides of the K from which on a shape has waves that only load; a tile to a workgroup and several."""
    for layout in ("nk", "kn") if layouts == "both" else (layouts,):
        code = tw.B_NK if layout == "nk" else tw.B_KN
        assert_loading_waves(tw, tile, layout, M, N, budget, Ks)
        for K in Ks:
            g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + N + K, b_layout=layout)
            C = torch_cuda.full((M, N), float("nan"), dtype=torch_cuda.bfloat16, device="cuda:0")
            tw.gemm_bf16(to_gpu(g["A"]), to_gpu(g["B"]), C=C, b_layout=code, cu_budget=budget)
            torch_cuda.cuda.synchronize()
            rng = np.random.default_rng(K)
            ms, ns = np.append(rng.integers(0, M, 400), [0, M - 1]), np.append(rng.integers(0, N, 400), [0, N - 1])
            ref = oracle.gemm_samples(g["A"], g["B"], layout, ms, ns)
            got = oracle.bf16_to_f64(to_bits(C))
            assert np.isfinite(got).all()
            gemm_check(got[ms, ns], ref, K, 0.5, "%s tiles, %s K = %d" % (tile, layout, K))


@pytest.mark.parametrize("M,N,budget", [(47, 40, 2), (33, 104, 4), (48, 24, 1)])
def test_gemm_tiles_of_48_rows_around_every_stage(tw, torch_cuda, M, N, budget):
    """Every number of K steps past a whole round of the LDS stages, eight elements more and less: the bits of the same rows of a
    large product. The shape is taken from K = 2048 on, and always has waves that only load."""
    torch = torch_cuda
    for K in sorted({2048 + n * 128 + d for n in range(6) for d in (0, 8, 120)}):
        plan = tw.gemm_plan(M, N, K, tw.B_NK, budget)
        assert (plan.tile_m, plan.tile_n, plan.loading_waves) == (48, 32, 4)
        g = W.make_gemm_inputs(M, K, N, 0.5, seed=K, b_layout="nk")
        A, B = to_gpu(g["A"]), to_gpu(g["B"])
        big = torch.cat([A, torch.ones((4096 - M, K), dtype=torch.bfloat16, device="cuda:0")])
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        tw.gemm_bf16(A, B, C, cu_budget=budget)
        assert np.array_equal(to_bits(C), to_bits(tw.gemm_bf16(big, B)[:M])), K


@pytest.mark.parametrize("tile,M,N,step,first", [((16, 16), 17, 24, 256, 1), ((32, 16), 33, 24, 256, 1), ((16, 32), 15, 104, 256, 3),
                                                 ((32, 32), 33, 40, 128, 1)])
def test_gemm_tiles_of_one_block_to_a_wave_around_every_stage(tw, torch_cuda, tile, M, N, step, first):
    """K of one to nine LDS stages (16 x 32: from three on, below it is not taken for every K), and eight elements more and less,
    without and with waves that only load (2048; 16 x 32 has them with helpers only, see STREAMED_AND_HELPED): the bits of the
    same rows of a large product; several tiles to a workgroup."""
    torch = torch_cuda
    Ks = sorted({max(8, n * step + d) for n in range(first, 10) for d in (-8, 0, 8)} | {2048 + n * step + d for n in range(3) for d in (0, 8)})
    for K in Ks:
        assert tw.gemm_tile_choice(M, N, K, tw.B_NK, 4) == tile
        g = W.make_gemm_inputs(M, K, N, 0.5, seed=K, b_layout="nk")
        A, B = to_gpu(g["A"]), to_gpu(g["B"])
        big = torch.cat([A, torch.ones((4096 - M, K), dtype=torch.bfloat16, device="cuda:0")])
        want = to_bits(tw.gemm_bf16(big, B)[:M])
        for budget in (4, 0):
            C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
            tw.gemm_bf16(A, B, C, cu_budget=budget)
            assert np.array_equal(to_bits(C), want), (tile, K, budget)


@pytest.mark.parametrize("tile,M,N,step,short", [((16, 16), 15, 1032, 256, False), ((32, 16), 24, 2568, 256, True), ((32, 32), 20, 5128, 128, True)])
def test_gemm_tiles_of_32_rows_take_another_loop_between_one_stage_and_k_1024(tw, torch_cuda, tile, M, N, step, short):
    """Which kernel each K takes, on both sides of the lines; the bits of the same rows of a large product."""
    torch = torch_cuda
    stream = torch.cuda.Stream()
    kernel = {}
    for K in (step, step + 8, 1016, 1024, 1032, 2040):
        assert tw.gemm_tile_choice(M, N, K, tw.B_NK) == tile, K
        gen = torch.Generator(device="cuda:0")
        gen.manual_seed(K)
        big, B = (torch.empty((n, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.5, generator=gen) for n in (4096, N))
        A, C = big[:M].contiguous(), torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        torch.cuda.synchronize()
        ((kernel[K], _),) = captured_kernels(stream, lambda: tw.gemm_bf16(A, B, C, stream=stream))
        tw.gemm_bf16(A, B, C)
        assert np.array_equal(to_bits(C), to_bits(tw.gemm_bf16(big, B)[:M])), K
    assert kernel[step] == kernel[1032] == kernel[2040] and kernel[step + 8] == kernel[1016] == kernel[1024]
    assert (kernel[step] != kernel[1024]) == short


HELPED = [("nk", 16, 1280, 8192), ("nk", 1, 8, 2048), ("nk", 64, 1280, 4096), ("nk", 40, 1272, 2056), ("nk", 150, 600, 4104),
          ("nk", 333, 1280, 4096), ("nk", 700, 1000, 2560), ("kn", 16, 4096, 2048), ("kn", 5, 4104, 2056), ("kn", 64, 4096, 2112),
          ("kn", 130, 1280, 4096), ("kn", 146, 1288, 4104), ("kn", 300, 1000, 3000), ("kn", 433, 328, 4104), ("kn", 1000, 1000, 2504),
          ("kn", 1200, 2000, 2240), ("kn", 16, 8192, 4096),
          ("nk", 2048, 3584, 2048), ("nk", 1990, 3528, 2056), ("nk", 3001, 4096, 2056), ("nk", 2000, 5000, 2504),
          ("nk", 2048, 3584, 4800), ("nk", 1990, 3528, 4904), ("nk", 3001, 4096, 4104), ("nk", 2000, 5000, 3400)]


# of these the ones on the other side of the rule: without helpers
NOT_HELPED = [("nk", 40, 1272, 2056), ("nk", 150, 600, 4104), ("nk", 333, 1280, 4096), ("nk", 700, 1000, 2560),
              ("kn", 146, 1288, 4104), ("kn", 1000, 1000, 2504), ("kn", 1200, 2000, 2240), ("kn", 16, 8192, 4096),
              ("nk", 2048, 3584, 2048), ("nk", 1990, 3528, 2056), ("nk", 3001, 4096, 2056), ("nk", 2000, 5000, 2504)]
# (layout, tile, tiles to a workgroup, M, N, K): every kernel that has helpers as a call of its own (those that only a boundary
# or a train launches with them: STREAMED_AND_HELPED, and the trains of test_weave_gpu.py), rows and windows of K that are not
# whole, tiles in one and in several blocks of rows, and the depths of a model's down projections
HELPED_TILES = [("kn", (16, 32), 1, 16, 1280, 8192), ("kn", (16, 32), 1, 9, 1048, 2056), ("kn", (16, 32), 1, 1, 520, 14336),
                ("nk", (16, 16), 1, 24, 24, 4864), ("nk", (16, 16), 1, 1207, 8, 2048), ("nk", (16, 16), 1, 16, 1024, 14336),
                ("nk", (16, 16), 1, 16, 1024, 28672), ("nk", (32, 16), 1, 483, 144, 2080), ("nk", (32, 16), 1, 18, 2120, 5832), ("nk", (32, 32), 1, 160, 984, 2064),
                ("nk", (64, 32), 1, 250, 1224, 2224), ("nk", (64, 64), 1, 142, 3448, 2152), ("nk", (96, 64), 1, 259, 3520, 2856),
                ("nk", (96, 96), 1, 356, 4144, 2272), ("nk", (128, 128), 1, 500, 5496, 3232),
                ("nk", (256, 128), 1, 1046, 5392, 3432), ("nk", (256, 192), 1, 1609, 5456, 3560),
                ("nk", (256, 256), 1, 2582, 5032, 4000), ("nk", (256, 128), 1, 1989, 3520, 14336),
                ("kn", (32, 32), 1, 16, 4096, 14336), ("kn", (32, 32), 1, 64, 1024, 28672), ("kn", (32, 32), 1, 128, 1024, 28672),
                ("kn", (64, 32), 1, 34, 4392, 2056), ("kn", (64, 64), 1, 1665, 256, 2056), ("kn", (96, 64), 1, 131, 5472, 2136),
                ("kn", (96, 128), 1, 810, 1936, 2056), ("kn", (128, 128), 1, 481, 5568, 2888),
                ("kn", (192, 64), 1, 3981, 392, 3776), ("kn", (256, 128), 2, 1809, 5232, 2160)]


@pytest.mark.parametrize("layout,tile,tiles,M,N,K", HELPED_TILES)
def test_every_gemm_kernel_with_helper_workgroups(tw, torch_cuda, layout, tile, tiles, M, N, K):
    """The launch has the helpers that the plan says; its bits are those of 8 compute units, which have none to spare;
    samples against the fp64 product."""
    torch = torch_cuda
    code = tw.B_NK if layout == "nk" else tw.B_KN
    plan = tw.gemm_plan(M, N, K, code, tw.device_cu_count())
    assert ((plan.tile_m, plan.tile_n), plan.tiles_per_workgroup) == (tile, tiles) and plan.helpers > 0
    assert plan.loading_waves == (0 if tile[0] == 256 else 4)
    assert plan.helpers_for_all == (tile[0] == 256) and tw.gemm_plan(M, N, K, code, 8).helpers == 0
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M + N + K)
    A, Bnk = (torch.empty((n, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.5, generator=gen) for n in (M, N))
    B = Bnk if layout == "nk" else Bnk.t().contiguous()
    C, D = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
    stream = torch.cuda.Stream()
    torch.cuda.synchronize()
    assert captured_grids(stream, lambda: tw.gemm_bf16(A, B, C=C, b_layout=code, stream=stream)) == [plan.workers + plan.helpers]
    tw.gemm_bf16(A, B, C=D, b_layout=code, cu_budget=8)
    for _ in range(2):
        C.fill_(float("nan"))
        tw.gemm_bf16(A, B, C=C, b_layout=code)
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(C), to_bits(D))
    ms, ns = [0, M // 2, M - 1], [0, N // 2 - 1, N - 1]
    ref = oracle.gemm(to_bits(A[ms]), to_bits(Bnk[ns]), "nk")
    gemm_check(oracle.bf16_to_f64(to_bits(C[ms][:, ns])), ref, K, 0.5, "%s %dx%dx%d" % (layout, M, N, K))


@pytest.mark.parametrize("layout,M,N,K", HELPED)
def test_gemm_with_helper_workgroups(tw, torch_cuda, layout, M, N, K):
    """Products of few tiles and long K, where compute units without a tile fetch operands ahead: tiles in one and in
    two blocks of rows, rows that are not whole lines, windows of K that are not whole; the 256-row tiles. Bits as on 8
    compute units, which leave none to spare, and samples against the fp64 product; launch after launch on other weights."""
    torch = torch_cuda
    code = tw.B_NK if layout == "nk" else tw.B_KN
    helpers = tw.gemm_plan(M, N, K, code, tw.device_cu_count()).helpers
    assert (helpers > 0) == ((layout, M, N, K) not in NOT_HELPED)
    for seed in (0, 1):
        g = W.make_gemm_inputs(M, K, N, 0.5, seed=M + N + K + seed, b_layout=layout)
        A, B = to_gpu(g["A"]), to_gpu(g["B"])
        C, D = (torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(2))
        tw.gemm_bf16(A, B, C=C, b_layout=code)
        tw.gemm_bf16(A, B, C=D, b_layout=code, cu_budget=8)
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(C), to_bits(D))
        rng = np.random.default_rng(K + seed)
        ms, ns = np.append(rng.integers(0, M, 200), [0, M - 1]), np.append(rng.integers(0, N, 200), [0, N - 1])
        gemm_check(oracle.bf16_to_f64(to_bits(C))[ms, ns], oracle.gemm_samples(g["A"], g["B"], layout, ms, ns), K, 0.5,
                   "%s %dx%dx%d" % (layout, M, N, K))


@pytest.mark.parametrize("M,N,K,budget", [(3001, 4096, 4104, 0), (4096, 4096, 2176, 0), (4040, 7944, 2112, 0), (4000, 4072, 2344, 100),
                                          (500, 1000, 4168, 4), (700, 1000, 3200, 3), (256, 200, 2456, 1)])
def test_gemm_pairs_of_tiles_of_weights_stored_k_by_n(tw, torch_cuda, M, N, K, budget):
    """Sizes at which a workgroup takes two 256 x 128 tiles of B stored [K x N] at a time (two LDS slots for A, three for
    B): K steps of every remainder of the two rotations, whole and ragged; an odd number of tiles in a row; one pair
    to a workgroup (with and without helpers) and several. The bits of the other storage order and of the
    small tiles that a part of the rows takes, and samples against the fp64 product."""
    torch = torch_cuda
    a = W.make_gemm_inputs(M, K, N, 0.5, seed=M + K, b_layout="nk")
    b = W.make_gemm_inputs(M, K, N, 0.5, seed=M + K, b_layout="kn")
    assert tw.gemm_tile_choice(M, N, K, tw.B_KN, budget or tw.device_cu_count()) == (256, 128)
    plan = tw.gemm_plan(M, N, K, tw.B_KN, budget or tw.device_cu_count())
    assert plan.tiles_per_workgroup == 2 and (plan.helpers > 0) == (M == 3001)
    A, B = to_gpu(b["A"]), to_gpu(b["B"])
    want = to_bits(tw.gemm_bf16(A, to_gpu(a["B"])))
    for _ in range(2):
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        tw.gemm_bf16(A, B, C=C, b_layout=tw.B_KN, cu_budget=budget)
        torch.cuda.synchronize()
        assert np.array_equal(to_bits(C), want)
    assert tw.gemm_tile_choice(90, N, K, tw.B_KN, tw.device_cu_count())[0] < 256
    assert np.array_equal(to_bits(tw.gemm_bf16(A[:90], B, b_layout=tw.B_KN)), want[:90])
    rng = np.random.default_rng(K)
    ms, ns = np.append(rng.integers(0, M, 400), [0, M - 1]), np.append(rng.integers(0, N, 400), [0, N - 1])
    gemm_check(oracle.bf16_to_f64(want)[ms, ns], oracle.gemm_samples(b["A"], b["B"], "kn", ms, ns), K, 0.5, "kn %dx%dx%d" % (M, N, K))


@pytest.mark.parametrize("T", [33, 64, 100, 200])
def test_layer_whose_gemm_has_helper_workgroups_equals_the_three_calls(tw, torch_cuda, T):
    """A chain's long product with weights of more than 32 MB takes larger tiles and helpers than on its own."""
    torch = torch_cuda
    H, P, K1, N2 = 8192, 2, 512, 3584
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(T)
    rand = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.5, generator=gen)
    X1, W1, W2, parts, res, w = rand(T, K1), rand(H, K1), rand(N2, H), [rand(T, H) for _ in range(P)], rand(T, H), rand(H)
    first, second = (tw.gemm_plan(T, n, k, tw.B_NK, tw.device_cu_count(), tw.GEMM_CHAIN) for n, k in ((H, K1), (N2, H)))
    alone = tw.gemm_plan(T, N2, H, tw.B_NK, tw.device_cu_count())
    assert second.helpers > 0 and alone.helpers == 0 and second.tile_m * second.tile_n > alone.tile_m * alone.tile_n
    a, b = torch.cuda.Stream(), torch.cuda.Stream()
    outputs = dict(out=rand(T, H), residual_out=rand(T, H), Y=rand(T, N2))
    torch.cuda.synchronize()
    assert captured_grids(a, lambda: tw.weave_layer_auto(X1, W1, parts, res, w, 1e-5, W2, a, b, parent=a, **outputs)) == [
        first.workers, sum(tw.fused_workgroups(T, H, P, cus=tw.device_cu_count())), second.workers + second.helpers]
    out, res_out, Y, row = tw.weave_layer_auto(X1, W1, parts, res, w, 1e-5, W2, torch.cuda.current_stream(), torch.cuda.Stream())
    torch.cuda.synchronize()
    assert row == T
    parts[0] = tw.gemm_bf16(X1, W1)
    out2, res2 = tw.reduce_add_rmsnorm(parts, res, w, 1e-5)
    Y2 = tw.gemm_bf16(out2, W2)
    torch.cuda.synchronize()
    for a, b in ((out, out2), (res_out, res2), (Y, Y2)):
        assert np.array_equal(to_bits(a), to_bits(b))


# One row of tiles, waves that only load, and helpers, the weights past the caches: (tile, M, N, K, as a boundary's second
# product), K of every remainder of the five LDS stages and, where the choice allows it, eight elements more and less
STREAMED_AND_HELPED = [((16, 16), 16, 1024, sorted(4096 + n * 256 + d for n in range(6) for d in (-8, 0, 8)), False),
                       ((32, 16), 18, 2120, sorted(5888 + n * 256 + d for n in range(6) for d in (-8, 0, 8)), False),
                       ((16, 32), 16, 2560, range(8192, 8192 + 6 * 256, 64), True),
                       ((16, 32), 10, 2728, range(7680, 7680 + 6 * 256, 64), True),
                       ((32, 32), 19, 2912, range(7744, 7744 + 6 * 128, 64), True)]


@pytest.mark.parametrize("tile,M,N,Ks,in_layer", STREAMED_AND_HELPED)
def test_streamed_weights_with_helper_workgroups_around_every_stage(tw, torch_cuda, tile, M, N, Ks, in_layer):
    """The bits of 8 compute units, which have no helpers, and for one K samples against the fp64 product. The tiles of 32
    columns have helpers here only where a boundary's weights are taken to come from memory."""
    torch = torch_cuda
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(M)
    rand = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.5, generator=gen)
    sx, sc = torch.cuda.current_stream(), torch.cuda.Stream()
    for K in Ks:
        plan = tw.gemm_plan(M, N, K, tw.B_NK, tw.device_cu_count(), tw.GEMM_CHAIN if in_layer else tw.GEMM_ALONE)
        assert (plan.tile_m, plan.tile_n, plan.loading_waves) == tile + (4,) and plan.helpers > 0, K
        A, B = rand(M, K), rand(N, K)
        C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
        if in_layer:
            A, _, _ = tw.weave_layer(rand(M, 64), rand(K, 64), [rand(M, K) for _ in range(2)], rand(M, K), rand(K), 1e-5, B, M, sx, sc, Y=C)
        else:
            tw.gemm_bf16(A, B, C=C)
        assert tw.gemm_plan(M, N, K, tw.B_NK, 8).helpers == 0
        assert np.array_equal(to_bits(C), to_bits(tw.gemm_bf16(A, B, cu_budget=8))), K
        if K == Ks[1]:
            rng = np.random.default_rng(K)
            ms, ns = np.append(rng.integers(0, M, 200), [0, M - 1]), np.append(rng.integers(0, N, 200), [0, N - 1])
            ref = oracle.gemm_samples(to_bits(A), to_bits(B), "nk", ms, ns)
            gemm_check(oracle.bf16_to_f64(to_bits(C))[ms, ns], ref, K, 0.5, "%s tiles, K = %d" % (tile, K))


@pytest.mark.parametrize("layout,K,tile", [("nk", 512, (256, 128)), ("nk", 2048, (256, 256)), ("kn", 512, (256, 128))])
def test_gemm_taller_than_four_gib(tw, torch_cuda, layout, K, tile):
    """M = 1.1 M rows: C is 4.5 GB, so tile base addresses run past 2^32 bytes (row 1048576 of C starts
    there, row 524288 at 2^31; A passes 2^30 at row 1048576, and 2^32 at K = 2048). Rows around those seams,
    the first, the last (a ragged tile) and random ones against the fp64 product of those rows, for the two
    tile shapes that such a product takes."""
    torch = torch_cuda
    M, N, std = 1100000 + 37, 2048, 0.05
    assert tw.gemm_tile_choice(M, N, K, tw.B_NK if layout == "nk" else tw.B_KN, tw.device_cu_count()) == tile
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(5)
    A = torch.empty((M, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    Bnk = torch.empty((N, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, std, generator=gen)
    B = Bnk if layout == "nk" else Bnk.t().contiguous()
    C = torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0")
    tw.gemm_bf16(A, B, C=C, b_layout=tw.B_NK if layout == "nk" else tw.B_KN)
    torch.cuda.synchronize()
    rng = np.random.default_rng(9)
    rows = sorted(set([0, 255, 256, 524287, 524288, 1048575, 1048576, 1048577, M - 38, M - 37, M - 1]
                      + [int(r) for r in rng.integers(0, M, 40)]))
    idx = torch.tensor(rows, device="cuda:0")
    ref = oracle.gemm(to_bits(A[idx]), to_bits(Bnk), "nk")
    gemm_check(oracle.bf16_to_f64(to_bits(C[idx])), ref, K, std, "tall gemm " + layout)
    # every element was written: no NaN is left anywhere
    assert not torch.isnan(C).any().item()
    del A, B, Bnk, C
    torch.cuda.empty_cache()


@pytest.mark.parametrize("layout", ["nk", "kn"])
def test_gemm_demo_shape_sampled(tw, torch_cuda, layout):
    """[2048 x 8192] x [8192 x 3584], N(0, 0.02^2): 4096 sampled outputs, one by one."""
    gc = W.CONFIGS["c5_overlap_tp8"]["gemm"]
    g = W.make_gemm_inputs(gc["M"], gc["K"], gc["N"], gc["std"], seed=0, b_layout=layout)
    C = tw.gemm_bf16(to_gpu(g["A"]), to_gpu(g["B"]), b_layout=tw.B_NK if layout == "nk" else tw.B_KN)
    torch_cuda.cuda.synchronize()
    Cb = to_bits(C)
    rng = np.random.default_rng(0)
    ms = np.concatenate([rng.integers(0, gc["M"], 4088), [0, 0, gc["M"] - 1, gc["M"] - 1, 255, 256, 1023, 1024]])
    ns = np.concatenate([rng.integers(0, gc["N"], 4088), [0, gc["N"] - 1, 0, gc["N"] - 1, 127, 128, 3583, 1792]])
    ref = oracle.gemm_samples(g["A"], g["B"], layout, ms, ns)
    gemm_check(oracle.bf16_to_f64(Cb[ms, ns]), ref, gc["K"], gc["std"], "demo gemm " + layout)
    assert np.count_nonzero(Cb) > 0.99 * Cb.size


def test_overlap_launch_equals_the_two_calls(tw, torch_cuda):
    """Fused kernel on half A next to the GEMM on half B (two streams, fork and
    join on a parent stream): same bits as the plain calls, every replay."""
    torch = torch_cuda
    cfg = W.CONFIGS["c5_overlap_tp8"]
    d = W.make_fused_inputs(cfg, N=512)
    g = dict(partials=[to_gpu(p) for p in d["partials"]], residual=to_gpu(d["residual"]),
             weight=to_gpu(d["weight"]), eps=d["eps"])
    gm = W.make_gemm_inputs(512, 1024, 640, 0.02, seed=0, b_layout="nk")
    A, B = to_gpu(gm["A"]), to_gpu(gm["B"])
    out0, res0 = tw.reduce_add_rmsnorm(g["partials"], g["residual"], g["weight"], g["eps"], cu_budget=32)
    C0 = tw.gemm_bf16(A, B)
    torch.cuda.synchronize()
    comm, comp, parent = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    for _ in range(3):
        with torch.cuda.stream(parent):
            out, res, C = tw.overlap_launch(dict(g, cu_budget=32), dict(A=A, B=B, cu_budget=0), comm, comp,
                                            parent=parent, use_parent=True, join=True)
            oc, rc, cc = out.clone(), res.clone(), C.clone()
        parent.synchronize()
        assert np.array_equal(to_bits(oc), to_bits(out0))
        assert np.array_equal(to_bits(rc), to_bits(res0))
        assert np.array_equal(to_bits(cc), to_bits(C0))


@pytest.mark.parametrize("layout", ["nk", "kn"])
@pytest.mark.parametrize("M,K,N", [(1024, 2048, 1536), (512, 1024, 4096), (2048, 8192, 1280), (2048, 2048, 4096)])
def test_overlap_launch_shared_mode_equals_the_two_calls(tw, torch_cuda, M, K, N, layout):
    """The co-resident mode: small fused workgroups on every compute unit next to
    the GEMM's. Same bits as the plain calls, on every one of many launches: next
    to the fused kernel the GEMM's LDS reads and loads take longer, which is when
    a missing wait shows (C starts as NaNs, so a store that went astray is seen).
    The shapes take 96 x 96 (or 96 x 128) tiles, 96 x 128 and 256 x 128 ones, for both
    storage orders of B (the [K x N] one reads its fragments with the transposing LDS
    read and has waits of its own)."""
    torch = torch_cuda
    cfg = W.CONFIGS["c5_overlap_tp8"]
    d = W.make_fused_inputs(cfg, N=1024)
    g = dict(partials=[to_gpu(p) for p in d["partials"]], residual=to_gpu(d["residual"]),
             weight=to_gpu(d["weight"]), eps=d["eps"])
    gm = W.make_gemm_inputs(M, K, N, 0.02, seed=0, b_layout=layout)
    bl = tw.B_NK if layout == "nk" else tw.B_KN
    A, B = to_gpu(gm["A"]), to_gpu(gm["B"])
    out0, res0 = tw.reduce_add_rmsnorm(g["partials"], g["residual"], g["weight"], g["eps"], cu_budget=32)
    C0 = tw.gemm_bf16(A, B, b_layout=bl, cu_budget=16)      # alone, 256-row tiles
    assert tw.gemm_tile_choice(M, N, K, bl, 16)[0] == 256
    beside = {1536: (96, 96) if layout == "nk" else (96, 128), 1280: (96, 128), 4096: (96, 128) if M == 512 else (256, 128)}
    assert tw.gemm_tile_choice(M, N, K, bl, tw.device_cu_count(), beside_other_kernels=True) == beside[N]
    torch.cuda.synchronize()
    assert np.array_equal(to_bits(tw.gemm_bf16(A, B, b_layout=bl)), to_bits(C0))
    if layout == "kn":      # and the same bits as the other storage order of the same matrix
        nk = W.make_gemm_inputs(M, K, N, 0.02, seed=0, b_layout="nk")
        assert np.array_equal(to_bits(tw.gemm_bf16(A, to_gpu(nk["B"]), cu_budget=16)), to_bits(C0))
    comm, comp, parent = torch.cuda.Stream(), torch.cuda.Stream(), torch.cuda.Stream()
    C = torch.empty((M, N), dtype=torch.bfloat16, device="cuda:0")
    out = torch.empty_like(g["residual"])
    res = torch.empty_like(g["residual"])
    for it in range(30):
        with torch.cuda.stream(parent):
            C.fill_(float("nan"))
            if it % 2 == 0:
                tw.overlap_launch(dict(g, cu_budget=tw.CU_SHARED, out=out, residual_out=res),
                                  dict(A=A, B=B, C=C, b_layout=bl, cu_budget=0), comm, comp, parent=parent,
                                  use_parent=True, join=True)
            else:
                # the two calls made by hand on two streams: tw_gemm_bf16 picks its tiles as for a
                # launch on its own
                comp.wait_stream(parent)
                comm.wait_stream(parent)
                tw.gemm_bf16(A, B, C=C, b_layout=bl, cu_budget=0, stream=comp)
                tw.reduce_add_rmsnorm(g["partials"], g["residual"], g["weight"], g["eps"], cu_budget=tw.CU_SHARED,
                                      out=out, residual_out=res, stream=comm)
                parent.wait_stream(comp)
                parent.wait_stream(comm)
            oc, rc, cc = out.clone(), res.clone(), C.clone()
        parent.synchronize()
        assert np.array_equal(to_bits(oc), to_bits(out0)), it
        assert np.array_equal(to_bits(rc), to_bits(res0)), it
        assert np.array_equal(to_bits(cc), to_bits(C0)), (it, int((to_bits(cc) != to_bits(C0)).sum()))


def test_gemm_random_shapes_both_layouts(tw, torch_cuda):
    """Seeded random M, N, K (N and K multiples of 8): both operand layouts and a
    budgeted launch give the same bits, and those match the oracle."""
    rng = np.random.default_rng(7)
    for case in range(16):
        M = int(rng.integers(1, 600))
        N = 8 * int(rng.integers(1, 60))
        K = 8 * int(rng.integers(1, 90))
        a = W.make_gemm_inputs(M, K, N, 0.3, seed=100 + case, b_layout="nk")
        b = W.make_gemm_inputs(M, K, N, 0.3, seed=100 + case, b_layout="kn")
        C1 = tw.gemm_bf16(to_gpu(a["A"]), to_gpu(a["B"]), b_layout=tw.B_NK)
        C2 = tw.gemm_bf16(to_gpu(b["A"]), to_gpu(b["B"]), b_layout=tw.B_KN)
        C3 = tw.gemm_bf16(to_gpu(a["A"]), to_gpu(a["B"]), b_layout=tw.B_NK, cu_budget=int(rng.integers(1, 9)))
        torch_cuda.cuda.synchronize()
        what = "case %d: %dx%dx%d" % (case, M, N, K)
        assert np.array_equal(to_bits(C1), to_bits(C2)), what
        assert np.array_equal(to_bits(C1), to_bits(C3)), what
        gemm_check(oracle.bf16_to_f64(to_bits(C1)), oracle.gemm(a["A"], a["B"], "nk"), K, 0.3, what)


def test_traced_gemm_counts_phases_and_gives_the_same_product(tw, torch_cuda):
    """The tracing variant of the 256 x 256 kernel: same bits as the plain call; every wave reports the
    tiles it worked on (all of them together: the tile count), phases that add up to no more than its
    total, and at least the matrix work's clocks in the two sub-steps (64 MFMAs of 16 clocks per sub-step
    and K step). Products that would not take those tiles are refused."""
    torch = torch_cuda
    M, N, K = 4096, 4096, 1024
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(7)
    A = torch.empty((M, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.05, generator=gen)
    B = torch.empty((N, K), dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.05, generator=gen)
    want = tw.gemm_bf16(A, B, b_layout=tw.B_NK)
    C, cycles = tw.gemm_bf16_traced(A, B)
    torch.cuda.synchronize()
    assert torch.equal(C.view(torch.int16), want.view(torch.int16))
    c = cycles.cpu().numpy()
    names = tw.GEMM_PHASE_NAMES
    tiles = (M // 256) * (N // 256)
    ran = c[:, names.index("tiles")] > 0
    assert ran.sum() == min(tiles, tw.device_cu_count()) * 4
    assert c[ran, names.index("tiles")].sum() == 4 * tiles
    parts = c[:, :6].sum(axis=1)
    assert (parts[ran] <= c[ran, names.index("kernel")]).all() and (c[ran, names.index("kernel")] < 10 ** 8).all()
    steps = c[ran, names.index("tiles")] * (K // 64)
    assert (c[ran, names.index("sub_step_0")] >= 1024 * steps).all()
    assert (c[ran, names.index("sub_step_1")] >= 1024 * steps).all()
    with pytest.raises(tw.TwError):
        tw.gemm_bf16_traced(A[:256], B[:128])


def test_gemms_with_helper_workgroups_on_several_streams(tw, torch_cuda):
    """Three streams that run side by side, with more launches in all than there are words to tell helpers by (128): launches
    whose helpers find no compute unit until the tiles are done end as well, and every product has the bits it has
    alone. Helpers of an XCD, helpers for all beside 256-row tiles, and beside pairs of tiles of [K x N] weights;
    and none."""
    torch = torch_cuda
    gen = torch.Generator(device="cuda:0")
    gen.manual_seed(3)
    rand = lambda *s: torch.empty(s, dtype=torch.bfloat16, device="cuda:0").normal_(0.0, 0.5, generator=gen)
    streams = [torch.cuda.Stream()]
    for _ in range(32):
        s = torch.cuda.Stream()
        if len(streams) < 3 and all(tw.streams_overlap(s, t) for t in streams):
            streams.append(s)
    assert len(streams) == 3
    for M, N, K, layout, tiles, for_all in ((64, 1280, 4096, "nk", 1, 0), (2048, 3584, 4800, "nk", 1, 1),
                                            (3001, 4096, 4104, "kn", 2, 1), (2048, 3584, 2056, "nk", 1, None)):
        code = tw.B_NK if layout == "nk" else tw.B_KN
        plan = tw.gemm_plan(M, N, K, code, tw.device_cu_count())
        assert plan.tiles_per_workgroup == tiles and (plan.helpers_for_all if plan.helpers else None) == for_all
        A = [rand(M, K) for _ in range(3)]
        B = [rand(*((N, K) if layout == "nk" else (K, N))) for _ in range(3)]
        want = [to_bits(tw.gemm_bf16(a, b, b_layout=code, cu_budget=8)) for a, b in zip(A, B)]
        C = [torch.full((M, N), float("nan"), dtype=torch.bfloat16, device="cuda:0") for _ in range(3)]
        torch.cuda.synchronize()
        for _ in range(50):
            for a, b, c, s in zip(A, B, C, streams):
                tw.gemm_bf16(a, b, C=c, b_layout=code, stream=s)
        torch.cuda.synchronize()
        for c, w in zip(C, want):
            assert np.array_equal(to_bits(c), w)
