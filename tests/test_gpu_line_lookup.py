"""Neighbour look-ups along filter lines: lines shorter than the filter, of one site, that end on or cross bitmap words,
filters of up to 63 taps a line, pruned taps; forward and backward on the vector and the pair-list kernels."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


def _dev(*arrays):
    return [torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


@pytest.mark.parametrize("ext,ksize,density", [
    ((6, 5, 1), (3, 3, 5), 0.5), ((5, 7, 3), (3, 3, 7), 0.5), ((9, 5, 64), (5, 5, 5), 0.1), ((4, 5, 65), (3, 3, 3), 0.4),
    ((40, 130), (1, 63), 0.2), ((30, 70), (3, 35), 0.3), ((33, 31), (7, 31), 1.0), ((3, 3, 200), (1, 3, 33), 0.3)])
@pytest.mark.parametrize("c_in,c_out,path", [(1, 8, 1), (1, 11, 1), (1, 16, 0), (8, 8, 1), (32, 16, 3), (8, 40, 1)])
def test_neighbours_along_filter_lines(ext, ksize, density, c_in, c_out, path):
    """Small whole numbers: every sum is exact, so results are compared bit for bit."""
    rng = np.random.default_rng(len(ext) * 1000 + ext[-1] + c_in)
    t = int(np.prod(ksize))
    coords = random_sparse_sites(rng, ext, 2, density)
    feats = rng.integers(-3, 4, size=(coords.shape[0], c_in)).astype(np.float32)
    w = (rng.integers(-3, 4, size=(t, c_in, c_out)) * (rng.random((t, 1, 1)) < 0.7)).astype(np.float32)
    gc = random_sparse_sites(rng, ext, 2, density)
    gf = rng.integers(-3, 4, size=(gc.shape[0], c_out)).astype(np.float32)
    print(ext, ksize, c_in, c_out, path, coords.shape[0], gc.shape[0], flush=True)
    bias = rng.integers(-2, 3, size=c_out).astype(np.float32)
    scnn.set_conv_path(path)
    try:
        oc, of, _ = scnn.sparse_conv_fwd(ext, 2, *_dev(coords, feats), ksize, *_dev(w, bias))
        scnn.set_conv_path(path if path == 1 else 0)
        data, filt, info = scnn.sparse_conv_bwd(ext, 2, *_dev(coords, feats), ksize, *_dev(w, gc, gf))
    finally:
        scnn.set_conv_path(0)
    rc, rf = oracle.sparse_conv_fwd(ext, 2, coords, feats, ksize, w, bias, rho_up=1.0)
    assert np.array_equal(oc.cpu().numpy(), rc) and np.array_equal(of.cpu().numpy(), rf)
    rd, rw = oracle.sparse_conv_bwd(ext, 2, coords, feats, ksize, w, gc, gf)
    assert int(info[2]) == 0
    assert np.array_equal(data.cpu().numpy(), rd) and np.array_equal(filt.cpu().numpy(), rw)


@pytest.mark.parametrize("ext,batch", [((20, 21, 75), 2), ((46, 40, 43), 2), ((240, 250), 1)])
@pytest.mark.parametrize("c_out", [5, 8, 9, 16])
@pytest.mark.parametrize("rows_at", [0, 4])
def test_eight_input_channels_by_size_and_alignment(ext, batch, c_out, rows_at):
    """Layers from 257 tiles of capacity on, with rows at a 16-byte boundary and past one: small whole numbers, exact."""
    rng = np.random.default_rng(c_out + ext[0])
    k = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, batch, 0.1)
    feats = rng.integers(-3, 4, size=(coords.shape[0], 8)).astype(np.float32)
    w = (rng.integers(-3, 4, size=(3 ** len(ext), 8, c_out)) * (rng.random((3 ** len(ext), 1, 1)) < 0.8)).astype(np.float32)
    room = torch.zeros(feats.size + 4, device="cuda")
    x = room[rows_at // 4:rows_at // 4 + feats.size].view(feats.shape)
    x.copy_(torch.from_numpy(feats))
    oc, of, _ = scnn.sparse_conv_fwd(ext, batch, _dev(coords)[0], x, k, *_dev(w))
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, rho_up=1.0)
    assert np.array_equal(oc.cpu().numpy(), rc) and np.array_equal(of.cpu().numpy(), rf)


@pytest.mark.parametrize("ext,ksize,density", [
    ((40, 1), (1, 31), 0.6), ((40, 3), (1, 31), 0.5), ((30, 64), (1, 31), 0.3), ((30, 65), (1, 31), 0.3),
    ((6, 5, 3), (1, 1, 9), 0.5), ((6, 5, 64), (1, 1, 9), 0.3), ((6, 5, 65), (1, 1, 9), 0.3),
    ((33, 3), (3, 7), 0.5), ((33, 64), (3, 7), 0.3), ((33, 65), (3, 9), 1.0), ((5, 9, 4), (1, 3, 9), 0.4), ((5, 4, 65), (1, 3, 9), 0.4),
    ((20, 65), (9, 3), 0.3), ((5, 65, 1), (3, 3, 1), 0.4), ((40, 65), (1, 1), 0.5)])
@pytest.mark.parametrize("c_in,c_out,path", [(1, 3, 0), (1, 16, 0), (8, 1, 0), (13, 1, 0)])
def test_one_channel_along_short_filters(ext, ksize, density, c_in, c_out, path):
    """Filters of at most 32 taps in at most nine lines, which one input channel takes site by site: forward from one
    channel, backward of layers with one output channel."""
    test_neighbours_along_filter_lines(ext, ksize, density, c_in, c_out, path)


@pytest.mark.parametrize("ext,ksize,density,g_density", [((47, 49, 48), (3, 3, 3), 0.7, 0.8), ((40, 41, 43), (3, 3, 3), 0.6, 0.02),
                                                         ((301, 260), (3, 3), 0.5, 0.5), ((5, 150, 130), (1, 3, 9), 0.9, 0.5)])
@pytest.mark.parametrize("c_in", [1, 5, 8])
@pytest.mark.parametrize("rows_at", [0, 4])
def test_backward_of_eight_output_channels_by_size(ext, ksize, density, g_density, c_in, rows_at):
    """From 257 tiles of rows on where a row meets few gradients, from 513 elsewhere, and gradient rows past a 16-byte
    boundary: small whole numbers, exact."""
    rng = np.random.default_rng(c_in + ext[0])
    coords, gc = random_sparse_sites(rng, ext, 1, density), random_sparse_sites(rng, ext, 1, g_density)
    few = np.prod(ksize) <= 9 or len(gc) * 6 <= len(coords)
    assert len(coords) > (256 if few else 512) * 128
    feats = rng.integers(-3, 4, size=(len(coords), c_in)).astype(np.float32)
    w = (rng.integers(-3, 4, size=(int(np.prod(ksize)), c_in, 8)) * (rng.random((int(np.prod(ksize)), 1, 1)) < 0.8)).astype(np.float32)
    gf = rng.integers(-3, 4, size=(len(gc), 8)).astype(np.float32)
    room = torch.zeros(gf.size + 4, device="cuda")
    g = room[rows_at // 4:rows_at // 4 + gf.size].view(gf.shape)
    g.copy_(torch.from_numpy(gf))
    print(ext, ksize, c_in, rows_at, len(coords), len(gc), flush=True)
    data, filt, info = scnn.sparse_conv_bwd(ext, 1, *_dev(coords, feats), ksize, *_dev(w, gc), g)
    rd, rw = oracle.sparse_conv_bwd(ext, 1, coords, feats, ksize, w, gc, gf)
    assert int(info[2]) == 0
    assert np.array_equal(data.cpu().numpy(), rd) and np.array_equal(filt.cpu().numpy(), rw)


@pytest.mark.parametrize("ext,batch,ksize,density,cap,tiles", [
    ((37, 40, 65), 1, (3, 3, 3), 0.08, 3071 * 128, 753), ((37, 40, 65), 4, (3, 3, 3), 0.3, 0, 3011), ((44, 47, 61), 4, (3, 3, 3), 0.1, 3068 * 128, 3072),
    ((44, 47, 61), 4, (3, 3, 3), 0.1, 3069 * 128, 3073), ((44, 47, 61), 4, (3, 3, 3), 0.1, 0, 3947),
    ((5, 150, 130), 2, (1, 3, 9), 0.2, 0, 1526), ((60, 70, 15), 3, (1, 1, 31), 0.2, 0, 1480), ((2, 200, 150), 1, (9, 1, 3), 0.9, 0, 470),
    ((11, 12, 13), 150, (3, 3, 3), 0.6, 0, 2161)])
@pytest.mark.parametrize("c_out", [1, 6, 8])
def test_eight_input_channels_four_lanes_a_site(ext, batch, ksize, density, cap, tiles, c_out):
    """More than nine taps on 257 tiles of capacity and more, up to 3072, where four lanes share a site, and past them, where each
    has a thread: few and many tiles in use, the tiles' ends, samples of different sizes: small whole numbers, exact."""
    rng = np.random.default_rng(c_out + ext[1])
    coords = random_sparse_sites(rng, ext, batch, density)
    coords = coords[(coords[:, 0] % 2 == 0) | (rng.random(len(coords)) < 0.2)]
    feats = rng.integers(-3, 4, size=(coords.shape[0], 8)).astype(np.float32)
    t = int(np.prod(ksize))
    bound = min(batch * int(np.prod(ext)), len(coords) * t)
    assert -(-(min(cap, bound) if cap else bound) // 128) + batch == tiles
    w = (rng.integers(-3, 4, size=(t, 8, c_out)) * (rng.random((t, 1, 1)) < 0.8)).astype(np.float32)
    bias = rng.integers(-2, 3, size=c_out).astype(np.float32)
    oc, of, n = scnn.sparse_conv_fwd(ext, batch, *_dev(coords, feats), ksize, *_dev(w, bias), cand_capacity=cap)
    print(ext, batch, c_out, len(coords), n.tolist(), flush=True)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, ksize, w, bias, rho_up=1.0)
    assert int(n[2]) == 0 and np.array_equal(oc.cpu().numpy(), rc) and np.array_equal(of.cpu().numpy(), rf)
