"""Networks whose layers end inside the tiles of the matrix kernels, against the oracle with the
harness's tolerances (float32 1e-4 normwise: K <= 1040 products of rounding 6e-8 each).

The first cases are small: their float32 GEMMs run on the direct kernel, on both sides of its
limits, and in 32 x 64 tiles; the live 16-column blocks in their comments are those of the weight
gradients' tiles, which have a copy of the float32 loops for each count.  The gather GEMM's larger
tiles and their counts come further down, with the plan of the launch checked."""
import numpy as np
import pytest

from tests.gpu_harness import Pair, check_structure, check_values, log
from tests.test_gpu_parity import _sparse_case
from workloads import he_params, random_labels

pytestmark = pytest.mark.gpu

# ell, k, c_in, classes, batch, density, seed
CASES = [
    (2, 15, 1, 17, 70, 0.5, 900),   # 1, 2, 3 live blocks; classes one past a block
    (2, 17, 5, 33, 64, 0.4, 901),   # 2, 3, 4 blocks; first layer on the matrix cores
    (2, 33, 2, 65, 40, 0.5, 902),   # 3, 5, 7 blocks: 128-wide tiles with 5 and 7
    (1, 66, 1, 129, 150, 0.5, 903), # 5 and 9 blocks
    (2, 48, 9, 10, 3, 0.3, 904),    # few tiles: the direct kernel, K 432 and below
    (2, 65, 1, 10, 2, 0.3, 905),    # K 260 and 520: on both sides of its limit
    (1, 100, 1, 3, 1, 0.1, 906),    # one sample, one site's windows
]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", CASES, ids=[f"l{c[0]}_k{c[1]}_b{c[4]}" for c in CASES])
def test_layers_ending_inside_tiles(case, dtype):
    ell, k, c_in, ncls, batch, p, seed = case
    coords, feats = _sparse_case(seed, ell, batch, p, c_in)
    log(f"[tile edges] {case} {dtype} n={len(coords)}")
    Ws, bs = he_params(ell, k, c_in, ncls, 100 + seed)
    pair = Pair(ell, k, c_in, ncls, batch, coords, feats, Ws, bs, random_labels(batch, ncls, 200 + seed), dtype).run_gpu()
    check_structure(pair)
    check_values(pair)
    assert np.isfinite(pair.loss)


# batch, density: 64, 128 and 256 bitmap words per workgroup of the window lists (32 in the cases
# above), sparse and with more sites in a workgroup's words than its list holds at a time
@pytest.mark.parametrize("batch,p", [(400, 0.02), (400, 0.9), (900, 0.5), (1024, 0.05), (1600, 0.95), (1600, 0.01)])
def test_window_lists_of_large_batches(batch, p):
    ell, k, ncls = 4, 1, 2
    coords, feats = _sparse_case(950 + batch, ell, batch, p, 1, empty=(0, batch // 2))
    log(f"[lists] batch {batch} density {p} n={len(coords)}")
    Ws, bs = he_params(ell, k, 1, ncls, 7)
    pair = Pair(ell, k, 1, ncls, batch, coords, feats, Ws, bs, random_labels(batch, ncls, 8), "f32")
    pair.run_gpu()
    check_structure(pair)
    # the loss is the sum of every sample's term, several samples to a workgroup above 512
    np.testing.assert_allclose(pair.loss, pair.o.loss, rtol=1e-5)


# depth, side of the sites' box: strided rows of one, two, three and six words
@pytest.mark.parametrize("ell,p", [(1, 0.4), (5, 0.004), (6, 0.001), (7, 0.0003)])
def test_bitmaps_of_wide_grids(ell, p):
    coords, feats = _sparse_case(970 + ell, ell, 3, p, 1)
    log(f"[bitmaps] ell {ell} n={len(coords)}")
    Ws, bs = he_params(ell, 1, 1, 2, 7)
    pair = Pair(ell, 1, 1, 2, 3, coords, feats, Ws, bs, random_labels(3, 2, 8), "f32").run_gpu()
    check_structure(pair)


# tile shapes as launch tags give them (bits 12..15), stage in bits 0..7, role in bits 8..11
T128x128, T128x64, T64x64, T32x64 = 0, 1, 2, 3
FORWARD, INPUT_GRAD = 0, 1


def run_planned(pair, stage, role, plan):
    """Runs the pair and checks that the stage's launch had the tile shape that the case is about."""
    pair.net.timing(["gather_gemm"])
    pair.run_gpu()
    got = [t >> 12 & 15 for t, _ in pair.net.timing_launches("gather_gemm") if t & 255 == stage and t >> 8 & 15 == role]
    assert got == [plan], (got, plan)
    return pair


# Input gradients stored through the rectifier derivative of a 1x1 layer below, with its bias sums
# (stage 4 of a DeepCNiN), float32: every tile shape of the LDS-tiled kernel (128 x 128 reads the layer
# below in place, the others stage its tile), one to seven live blocks, rows ending inside a tile, and K
# split (the sums then have a launch of their own).  (At k = 130 and batch 5480 the harness found one of
# the 1.4 million rectifier branches of the topmost layer differing at 1.03 eps of its sum's magnitudes.
# Its band of 1 eps holds the deciding sum's own rounding; the sum's 260 inputs, each a sum of 520
# products, bring up to 520 eps more, in practice as much again.  So the 128 x 64 case is a narrow one.)
# ell, k, batch, plan
MASKED = [(1, 66, 8185, T128x128), (1, 100, 8190, T128x128), (2, 40, 2650, T128x64), (2, 15, 2650, T64x64),
          (1, 33, 1100, T32x64), (1, 66, 30, T32x64)]


@pytest.mark.parametrize("case", MASKED, ids=[f"l{c[0]}k{c[1]}_b{c[2]}" for c in MASKED])
def test_masked_input_gradients_with_bias_sums(case):
    ell, k, batch, plan = case
    coords, feats = _sparse_case(920 + k, ell, batch, 0.3, 1)
    log(f"[masked] {case} n={len(coords)}")
    Ws, bs = he_params(ell, k, 1, 5, 30 + k, "deepcnin")
    pair = Pair(ell, k, 1, 5, batch, coords, feats, Ws, bs, random_labels(batch, 5, 40 + k), "f32", arch="deepcnin")
    run_planned(pair, 4, INPUT_GRAD, plan)
    check_structure(pair)
    check_values(pair)


# Every count of live blocks that the float32 gather GEMM has a copy of its loops for: five to eight
# of a 128 x 128 tile, one to four of a 128 x 64 and a 64 x 64 one (a first layer's forward, K 144 and,
# for the shapes that take shorter K, 108).  k, features, batch, plan
LIVE = [(70, 16, 2060, T128x128), (90, 16, 2060, T128x128), (100, 16, 2060, T128x128), (120, 16, 2060, T128x128),
        (10, 16, 4100, T128x64), (30, 16, 4100, T128x64), (40, 16, 4100, T128x64), (60, 16, 4100, T128x64),
        (10, 12, 4100, T64x64), (30, 12, 4100, T64x64), (40, 12, 4100, T64x64), (60, 12, 4100, T64x64)]


@pytest.mark.parametrize("case", LIVE, ids=[f"k{c[0]}_m{c[1]}" for c in LIVE])
def test_every_count_of_live_blocks(case):
    k, c_in, batch, plan = case
    coords, feats = _sparse_case(940 + k, 1, batch, 0.3, c_in)
    log(f"[live blocks] {case} n={len(coords)}")
    Ws, bs = he_params(1, k, c_in, 10, 50 + k)
    pair = Pair(1, k, c_in, 10, batch, coords, feats, Ws, bs, random_labels(batch, 10, 60 + k), "f32")
    run_planned(pair, 1, FORWARD, plan)
    check_values(pair)


# Without an input-feature gradient the first layer's final ground pass rides on the weight-gradient
# launch of the other tile width, or runs alone where there is none.  arch, ell, k, classes: the first
# layer among the 128-wide tiles with a 64-wide launch beside them (the softmax layer's; convolutions'),
# all layers 128 wide, the first 64 wide, all 64 wide
FINAL = [("deepcnet", 1, 100, 10), ("deepcnet", 2, 70, 33), ("deepcnin", 1, 100, 10), ("deepcnet", 1, 100, 100),
         ("deepcnin", 1, 100, 100), ("deepcnet", 2, 33, 100), ("deepcnet", 2, 12, 10)]


@pytest.mark.parametrize("dtype", ["f32", "bf16"])
@pytest.mark.parametrize("case", FINAL, ids=[f"{c[0]}_l{c[1]}k{c[2]}_c{c[3]}" for c in FINAL])
def test_first_layers_final_pass_without_dfeats(case, dtype):
    arch, ell, k, ncls = case
    batch = 40
    coords, feats = _sparse_case(960 + k, ell, batch, 0.3, 1, empty=(3,))
    log(f"[final pass] {case} {dtype} n={len(coords)}")
    Ws, bs = he_params(ell, k, 1, ncls, 70 + k, arch)
    pair = Pair(ell, k, 1, ncls, batch, coords, feats, Ws, bs, random_labels(batch, ncls, 80 + k), dtype, arch=arch,
                want_dfeats=False).run_gpu()
    check_values(pair)


# Weight gradients whose pass takes another chunk length than the plan's shortest.  dtype, ell, k, batch,
# density; tiles at a quarter / a half of the standard length and at it: a half of a network planned at
# quarters (612 and 412 tiles), the standard length of one planned at quarters (1324 / 738 / 375) and at
# halves (1324 / 738), the quarter (501)
CHUNKED = [("bf16", 2, 60, 1500, 0.3), ("f32", 2, 60, 500, 0.3), ("bf16", 3, 50, 300, 0.2), ("f32", 3, 50, 300, 0.2),
           ("f32", 2, 60, 300, 0.3)]


@pytest.mark.parametrize("case", CHUNKED, ids=[f"{c[0]}_l{c[1]}k{c[2]}_b{c[3]}" for c in CHUNKED])
def test_weight_gradients_of_every_chunk_length(case):
    dtype, ell, k, batch, p = case
    coords, feats = _sparse_case(970 + k, ell, batch, p, 1)
    log(f"[chunks] {case} n={len(coords)}")
    Ws, bs = he_params(ell, k, 1, 10, 90 + k)
    pair = Pair(ell, k, 1, 10, batch, coords, feats, Ws, bs, random_labels(batch, 10, 95 + k), dtype).run_gpu()
    check_values(pair)
