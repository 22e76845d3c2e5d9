"""The fp64 filter gradient at the sizes where it can go wrong: tiles of 128 rows with remainders, slabs of 32 taps and
of 16 x 16 channels with remainders, samples without rows, one share and many."""
import numpy as np
import pytest

import paper_1801_10585_amd as scnn
from tests.test_gpu_bwd_parity import full_check, say
from workloads import make_filter, random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extent,batch,c_in,c_out,ksize,rows", [
    ((1, 1, 1), 1, 1, 1, (3, 3, 3), 1),
    ((8, 8, 8), 1, 8, 16, (3, 3, 3), 127),
    ((8, 8, 8), 1, 16, 15, (3, 3, 3), 128),
    ((8, 8, 8), 4, 15, 17, (3, 3, 3), 129),       # all rows in two of four samples
    ((30, 31), 2, 17, 33, (3, 11), 300),          # 33 taps: a second slab of one tap
    ((9, 9, 9), 2, 33, 8, (5, 5, 5), 200),        # 125 taps, three blocks of input channels
    ((40, 40, 40), 2, 8, 8, (3, 3, 3), 70000),    # more tiles than shares
])
def test_fp64_filter_gradient_edges(extent, batch, c_in, c_out, ksize, rows):
    rng = np.random.default_rng(rows)
    n = int(np.prod(extent))
    keys = np.sort(rng.choice(min(2, batch) * n, size=rows, replace=False))
    coords = np.stack([keys // n, *np.unravel_index(keys % n, extent)], axis=1).astype(np.int32)
    feats = rng.normal(size=(rows, c_in)).astype(np.float32)
    feats *= rng.random(feats.shape) >= 0.2
    w = make_filter(rng, ksize, c_in, c_out, 0.7, 0.3)
    gc = random_sparse_sites(rng, extent, batch, 0.5) if n > 1 else np.zeros((1, 1 + len(extent)), np.int32)
    gf = rng.normal(size=(gc.shape[0], c_out)).astype(np.float32)
    say(f"bwd filter {extent} B={batch} {c_in}->{c_out} {ksize} rows={rows} g_rows={gc.shape[0]}")
    scnn.set_conv_path(1)
    try:
        _, f1, _ = full_check(extent, batch, coords, feats, ksize, w, gc, gf, f"filter {extent}", matrix_cores=False)
        _, f2, _ = full_check(extent, batch, coords, feats, ksize, w, gc, gf, f"filter {extent}", matrix_cores=False)
    finally:
        scnn.set_conv_path(0)
    assert np.array_equal(f1, f2)
