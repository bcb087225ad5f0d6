"""Networks whose layers end inside the tiles of the matrix kernels: every count of live 16-column
blocks of a tile (each has a copy of the float32 loops), single rows past a tile, float32 launches
on both sides of the direct kernel's limits, and the weight gradients' shorter site chunks; against
the oracle with the harness's tolerances (float32 1e-4 normwise: K <= 800 products of rounding
6e-8 each)."""
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
