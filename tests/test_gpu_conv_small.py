"""Smallest layers of the vector kernels: items of one and of two 16-channel blocks on either side of where the one becomes the
other (512 items of 32 rows and 16 channels), all widths of a gather, against the oracle on small whole numbers."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("ext,batch", [((8, 9, 10), 1), ((25, 99), 1), ((30, 30), 5), ((30, 30), 6), ((30, 30), 9), ((12, 11, 10), 2), ((21, 22, 23), 5), ((21, 22, 23), 12)])
@pytest.mark.parametrize("c_in,c_out", [(8, 8), (16, 16), (24, 17), (8, 32), (12, 33), (4, 40), (2, 20), (6, 16), (16, 50)])
def test_smallest_layers(ext, batch, c_in, c_out):
    rng = np.random.default_rng(c_in * c_out)
    ksize = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, batch, 0.3 if ext[0] != 21 else 0.03)
    feats = rng.integers(1, 4, size=(len(coords), c_in)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), c_in, c_out)).astype(np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, ksize, w, rho_up=0.2, relu=True)
    scnn.set_conv_path(1)
    try:
        gc, gf, n = scnn.sparse_conv_fwd(ext, batch, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats)), ksize,
                                         torch.from_numpy(w).cuda(), rho_up=0.2, relu=True)
    finally:
        scnn.set_conv_path(0)
    assert scnn.last_conv_kernel() == "k_conv_valu" and int(n[2]) == 0
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)


@pytest.mark.parametrize("ext,batch,ksize", [((20, 21), 2, (5, 7)), ((33, 40), 3, (7, 7)), ((6, 7, 8), 2, (5, 5, 5))])
@pytest.mark.parametrize("c_in,c_out", [(8, 16), (24, 24), (16, 50), (12, 33), (4, 8), (6, 20)])
def test_smallest_layers_of_long_filters(ext, batch, ksize, c_in, c_out):
    """Filters of two and four groups of 32 taps, weights of all 24 bits: the sums are exact in fp64 and rounded once."""
    rng = np.random.default_rng(c_in * c_out)
    coords = random_sparse_sites(rng, ext, batch, 0.2)
    feats = rng.integers(1, 4, size=(len(coords), c_in)).astype(np.float32)
    w = rng.integers(-(2 ** 24) + 1, 2 ** 24, size=(int(np.prod(ksize)), c_in, c_out)).astype(np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, ksize, w, rho_up=0.2, relu=True)
    scnn.set_conv_path(1)
    try:
        gc, gf, n = scnn.sparse_conv_fwd(ext, batch, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats)), ksize,
                                         torch.from_numpy(w).cuda(), rho_up=0.2, relu=True)
    finally:
        scnn.set_conv_path(0)
    assert scnn.last_conv_kernel() == "k_conv_valu" and int(n[2]) == 0
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)
