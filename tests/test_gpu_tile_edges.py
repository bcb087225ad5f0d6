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
