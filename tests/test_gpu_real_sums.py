"""Layers of real values against sums in 64 bits: the forms of the vector kernels add in different orders, all in fp64, and round
once.  The capacity of the workspace, in tiles of 128 candidate sites, is what the host chooses the form by; each case states
it."""
import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


def reference(ext, batch, coords, feats, k, w):
    """Responses and the sums of the products' magnitudes on the whole grid, [batch, c_out, extent...], fp64."""
    d = len(ext)
    x = torch.zeros((batch, *ext, feats.shape[1]), dtype=torch.float64)
    x[tuple(torch.from_numpy(coords.astype(np.int64)).T)] = torch.from_numpy(feats).double()
    x = x.movedim(-1, 1)
    wt = torch.from_numpy(w).double().view(*k, *w.shape[1:]).permute(d + 1, d, *range(d)).contiguous()
    conv = torch.nn.functional.conv3d if d == 3 else torch.nn.functional.conv2d
    pad = [(s - 1) // 2 for s in k]
    return conv(x, wt, padding=pad), conv(x.abs(), wt.abs(), padding=pad)


@pytest.mark.parametrize("ext,batch,k,c_in,c_out,density,tiles,kernel", [
    # one workgroup a sample
    ((28, 28), 1, (3, 3), 1, 8, 0.2, None, "k_layer_tiny"), ((28, 28), 300, (3, 3), 1, 8, 0.2, None, "k_layer_tiny"),
    ((28, 28), 300, (3, 3), 1, 16, 0.2, None, "k_layer_tiny"), ((10, 9), 300, (3, 3), 8, 16, 0.3, None, "k_layer_tiny"),
    ((20, 21), 3, (3, 3), 8, 8, 0.3, None, "k_layer_tiny"), ((9, 10, 11), 2, (3, 3, 3), 5, 12, 0.05, None, "k_layer_tiny"),
    # eight input channels: a thread a site above 3072 tiles, four lanes a site from 257 (where sites have many neighbours 513) on,
    # the 32-row form below
    ((64, 64, 50), 2, (3, 3, 3), 8, 8, 0.05, 3073, "k_conv_valu"), ((64, 64, 50), 2, (3, 3, 3), 8, 7, 0.05, 3072, "k_conv_valu"),
    ((40, 41, 40), 1, (3, 3, 3), 8, 8, 0.4, 514, "k_conv_valu"), ((36, 42, 43), 1, (3, 3, 3), 8, 8, 0.4, 509, "k_conv_valu"),
    ((30, 40, 41), 1, (3, 3, 3), 8, 8, 0.03, 257, "k_conv_valu"), ((30, 40, 41), 1, (3, 3, 3), 8, 8, 0.03, 256, "k_conv_valu"),
    ((60, 70, 15), 2, (1, 1, 31), 8, 5, 0.1, 800, "k_conv_valu"), ((150, 200), 5, (3, 3), 8, 8, 0.3, 1177, "k_conv_valu"),
    # 32-row items of one 16-channel block up to 1024 tiles where sites have few neighbours, else up to 256; of two blocks
    ((50, 50, 53), 1, (3, 3, 3), 16, 16, 0.05, 1024, "k_conv_valu"), ((50, 50, 53), 1, (3, 3, 3), 16, 16, 0.05, 1025, "k_conv_valu"),
    ((50, 50, 53), 1, (3, 3, 3), 4, 12, 0.05, 1000, "k_conv_valu"),
    ((40, 41, 40), 1, (5, 5, 5), 24, 16, 0.1, 514, "k_conv_valu"), ((40, 41, 40), 1, (5, 3, 3), 24, 16, 0.1, 514, "k_conv_valu"), ((30, 30, 36), 1, (3, 3, 3), 16, 16, 0.6, 255, "k_conv_valu"),
    ((30, 30, 40), 1, (3, 3, 3), 16, 16, 0.6, 283, "k_conv_valu"), ((60, 61), 1, (3, 3), 24, 24, 0.2, 27, "k_conv_valu"),
    ((60, 61), 4, (5, 5), 12, 33, 0.1, 119, "k_conv_valu"), ((60, 61), 4, (5, 5), 16, 24, 0.1, 119, "k_conv_valu"), ((60, 61), 4, (3, 3), 6, 20, 0.2, 119, "k_conv_valu"),
    # one input channel; the general forms
    ((50, 60, 70), 1, (3, 3, 3), 1, 16, 0.02, 800, "k_conv_valu"), ((50, 60, 70), 2, (3, 3, 3), 3, 9, 0.2, 3284, "k_conv_valu"), ((50, 60, 70), 2, (3, 3, 3), 16, 16, 0.2, 3284, "k_conv_valu")])
def test_real_sums(ext, batch, k, c_in, c_out, density, tiles, kernel):
    """The fp64 sum of n products is off by at most n 2^-53 of the sum of their magnitudes and is rounded once, to 24 bits."""
    rng = np.random.default_rng(c_in + c_out)
    coords = random_sparse_sites(rng, ext, batch, density)
    feats = rng.standard_normal((len(coords), c_in)).astype(np.float32)
    w = rng.standard_normal((int(np.prod(k)), c_in, c_out)).astype(np.float32)
    ref, mag = reference(ext, batch, coords, feats, k, w)
    cap = 0
    if tiles is not None:  # the capacity that makes it so many tiles, and the call does have room for it
        cap = (tiles - batch) * 128
        bound = min(batch * int(np.prod(ext)), len(coords) * int(np.prod(k)))
        cap = min(cap, bound)
        assert -(-cap // 128) + batch == tiles
    c, f, t = (torch.from_numpy(a).cuda() for a in (coords, feats, w))
    oc, of, nnz = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=1.0, cand_capacity=cap)
    print(ext, batch, c_in, c_out, len(coords), nnz.tolist(), flush=True)
    assert scnn.last_conv_kernel() == kernel and int(nnz[2]) == 0
    got = torch.zeros((batch, *ext, c_out), dtype=torch.float64)
    got[tuple(oc.cpu().long().T)] = of.cpu().double()
    got = got.movedim(-1, 1)
    bound = 2.0 ** -24 * ref.abs() + (2 * c_in * int(np.prod(k)) * 2.0 ** -53) * mag + 2.0 ** -149
    assert bool(((got - ref).abs() <= bound).all())
