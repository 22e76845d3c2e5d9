"""The fp64 filter gradient at the sizes where it can go wrong: tiles of 128 rows with remainders, slabs of 32 taps and
of 16 x 16 channels with remainders, slabs of several channel blocks, samples without rows, one share and many, and the
vector kernel for long filters of few channels."""
import numpy as np
import pytest

import paper_1801_10585_amd as scnn
from tests.test_gpu_bwd_parity import ATOL, RTOL, full_check, gpu_bwd, say
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
    ((40, 40, 40), 2, 24, 24, (1, 1, 1), 70000),  # both blocks of output channels in one slab of four waves
    ((40, 40, 40), 2, 17, 130, (1, 1, 1), 20000), # nine blocks: sixteen waves
    ((40, 40, 40), 2, 5, 49, (1, 1, 3), 40000),   # twelve slots, the last block of one channel
    ((40, 40, 40), 2, 20, 70, (3, 3, 1), 20000),  # five blocks three to a slab, the last slab of two
    ((30, 30, 30), 1, 1, 8, (5, 5, 5), 12000),    # long filter, few channels: the vector kernel, four blocks of elements
    ((300, 40), 1, 2, 7, (7, 7), 8300),           # its elements no multiple of a block
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


@pytest.mark.parametrize("c_in,c_out,ksize", [(8, 16, (3, 3, 3)), (17, 5, (3, 3, 1)), (24, 24, (1, 1, 1)), (3, 8, (5, 5, 5))])
def test_infinities_and_nan_reach_only_the_taps_that_see_them(c_in, c_out, ksize):
    """An infinite and a NaN row, in a corner and inside, with about half of the gradient sites around them absent: only
    the filter elements of (row, tap) pairs that have a gradient row may lose their finite values (Algorithm 2 visits no
    others), and those exactly as the sum over the pairs does."""
    rng = np.random.default_rng(c_in)
    ext = (10, 9, 11)
    coords = random_sparse_sites(rng, ext, 1, 0.3)
    coords = np.unique(np.concatenate([coords, np.zeros((1, 4), np.int32)]), axis=0).astype(np.int32)
    n = coords.shape[0]
    feats = rng.normal(size=(n, c_in)).astype(np.float32)
    feats[0, 0], feats[n // 2, c_in - 1] = np.inf, np.nan
    w = rng.normal(size=(int(np.prod(ksize)), c_in, c_out)).astype(np.float32)
    gc = random_sparse_sites(rng, ext, 1, 0.5)
    gc = gc[(gc[:, 1:] != 0).any(1)]                      # (no gradient row on the infinite row's own site)
    gf = rng.normal(size=(gc.shape[0], c_out)).astype(np.float32)
    p = [k // 2 for k in ksize]
    grid = np.full([e + 2 * h for e, h in zip(ext, p)], -1)
    grid[tuple(gc[:, 1 + a] + p[a] for a in range(3))] = np.arange(gc.shape[0])
    ref = np.zeros(w.shape)
    with np.errstate(invalid="ignore"):
        for t, off in enumerate(np.ndindex(*ksize)):
            r = grid[tuple(coords[:, 1 + a] + 2 * p[a] - off[a] for a in range(3))]
            ref[t] = feats[r >= 0].astype(np.float64).T @ gf[r[r >= 0]].astype(np.float64)
    scnn.set_conv_path(1)
    try:
        say(f"bwd filter, non-finite rows {c_in}->{c_out} {ksize}")
        _, got = gpu_bwd(ext, 1, coords, feats, ksize, w, gc, gf)
    finally:
        scnn.set_conv_path(0)
    finite = np.isfinite(ref)
    assert finite.any() and (np.isnan(ref).any() or ksize == (1, 1, 1))
    assert np.array_equal(np.isnan(got), np.isnan(ref)) and np.array_equal(np.isinf(got), np.isinf(ref))
    assert np.array_equal(np.sign(got[np.isinf(ref)]), np.sign(ref[np.isinf(ref)]))
    assert (np.abs(got[finite] - ref[finite]) <= RTOL * np.abs(ref[finite]) + ATOL).all()
