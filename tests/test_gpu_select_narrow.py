"""Compaction of narrow layers: the one-launch and the two-launch form on either side of their border (512 or 1152 tiles of
capacity), few and no rows, samples without rows, odd channel counts, more surviving rows than the output holds."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("mode", [scnn.ABS, scnn.SIGNED])
@pytest.mark.parametrize("cap", [510 * 128, 510 * 128 + 1, 200000])
@pytest.mark.parametrize("ext,c_out,density,rho,relu,pool", [
    ((46, 40, 43), 8, 0.025, 0.1, True, False), ((46, 40, 43), 3, 0.025, 0.2, False, True), ((46, 40, 43), 16, 0.025, 0.05, True, True),
    ((30, 50, 60), 31, 0.022, 0.1, False, False), ((30, 50, 60), 1, 0.022, 0.01, False, False), ((300, 310), 7, 0.07, 1.0, False, False)])
def test_narrow_layers_on_either_side_of_the_launch_rule(ext, c_out, density, rho, relu, pool, cap, mode):
    """Small whole numbers, many of them equal: the oracle's rows, bit for bit."""
    rng = np.random.default_rng(c_out + ext[0])
    ksize = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, 2, density)
    coords = coords[(coords[:, 0] == 1) | (rng.random(len(coords)) < 0.3)]
    feats = rng.integers(1, 4, size=(len(coords), 2)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), 2, c_out)).astype(np.float32)
    c, f, t = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats, w))
    print(ext, c_out, len(coords), cap, mode, flush=True)
    rc, rf = oracle.sparse_conv_fwd(ext, 2, coords, feats, ksize, w, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
    gc, gf, n = scnn.sparse_conv_fwd(ext, 2, c, f, ksize, t, rho_up=rho, topk_mode=mode, relu=relu, pool=pool,
                                     cand_capacity=cap, out_capacity=cap)
    assert len(coords) * 3 ** len(ext) > 511 * 128  # (the capacity asked for is the one that the call has)
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)
    if not pool:  # a small output: its rows are the first ones, the count is the whole, the bit is set
        out = (torch.full((70, 1 + len(ext)), -7, dtype=torch.int32, device="cuda"),
               torch.full((70, c_out), -7.0, device="cuda"), torch.zeros(4, dtype=torch.int64, device="cuda"))
        gc, gf, n = scnn.sparse_conv_fwd(ext, 2, c, f, ksize, t, rho_up=rho, topk_mode=mode, relu=relu, cand_capacity=200000,
                                         out_capacity=64, out=out, sync=False)
        assert int(n[0]) == len(rc) and int(n[2]) == 2
        assert np.array_equal(out[0][:64].cpu().numpy(), rc[:64]) and np.array_equal(out[1][:64].cpu().numpy(), rf[:64])
        assert bool((out[0][64:] == -7).all()) and bool((out[1][64:] == -7).all())


def test_narrow_layers_without_rows():
    for cap in (1000, 100000):
        z = (torch.zeros((0, 4), dtype=torch.int32, device="cuda"), torch.zeros((0, 4), device="cuda"))
        rows = torch.randint(0, 3, (50, 1), device="cuda")
        c = torch.cat([torch.zeros_like(rows), torch.arange(50, device="cuda")[:, None], rows, rows], 1).to(torch.int32)
        w = torch.zeros((27, 4, 8), device="cuda")  # (no tap is active: no candidate sites)
        for coords, feats in (z, (c, torch.ones((50, 4), device="cuda"))):
            oc, of, n = scnn.sparse_conv_fwd((60, 60, 60), 1, coords, feats, (3, 3, 3), w, rho_up=0.1, cand_capacity=cap)
            assert oc.shape[0] == of.shape[0] == 0 and [int(v) for v in n] == [0, 0, 0, 0]


@pytest.mark.parametrize("mode", [scnn.ABS, scnn.SIGNED])
@pytest.mark.parametrize("c_out,relu,pool", [(8, False, False), (40, True, False), (70, False, True)])
@pytest.mark.parametrize("ext,rho,below", [((50, 51, 52), 1.0, 0), ((50, 51, 52), 0.5, 0), ((50, 51, 52), 0.5, 1), ((12, 9), 1.0, 0)])
def test_a_selection_that_keeps_everything(ext, rho, below, c_out, relu, pool, mode):
    """k at the sites of the grid, at the capacity of the workspace, and one below it, where columns are selected."""
    rng = np.random.default_rng(c_out)
    ksize = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, 1, 0.01 if len(ext) == 3 else 0.2)
    feats = rng.integers(1, 4, size=(len(coords), 4)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), 4, c_out)).astype(np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, 1, coords, feats, ksize, w, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
    cap = 0 if rho == 1.0 else scnn.k_from_rho(rho, int(np.prod(ext))) + below
    gc, gf, n = scnn.sparse_conv_fwd(ext, 1, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats)), ksize,
                                     torch.from_numpy(w).cuda(), rho_up=rho, topk_mode=mode, relu=relu, pool=pool,
                                     cand_capacity=cap)
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf) and int(n[2]) == 0


@pytest.mark.parametrize("mode", [scnn.ABS, scnn.SIGNED])
@pytest.mark.parametrize("ext,batch,c_out", [((10, 11), 2, 3), ((16, 16), 1, 1), ((18, 20), 3, 8), ((22, 23), 2, 5), ((25, 25), 300, 4),
                                             ((28, 27), 2, 40), ((31, 33), 1, 70), ((10, 10, 10), 2, 8), ((16, 16, 16), 2, 16),
                                             ((16, 15, 14), 130, 8), ((13, 12, 11), 140, 8)])
@pytest.mark.parametrize("rho", [0.0, 0.004, 0.2, 0.6])
def test_selection_of_short_columns(ext, batch, c_out, rho, mode):
    """One to thirty-two tiles a column, few columns and many, runs of equal scores cut at the k-th."""
    rng = np.random.default_rng(ext[0] + c_out)
    k = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, batch, 0.4)
    coords = coords[(coords[:, 0] != 0) | (rng.random(len(coords)) < 0.1)]  # (columns of different lengths)
    feats = rng.integers(1, 4, size=(len(coords), 1)).astype(np.float32)
    w = rng.integers(-3, 4, size=(3 ** len(ext), 1, c_out)).astype(np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, rho_up=rho, topk_mode=mode)
    gc, gf, n = scnn.sparse_conv_fwd(ext, batch, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats, )), k,
                                     torch.from_numpy(w).cuda(), rho_up=rho, topk_mode=mode)
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf) and int(n[2]) == 0


@pytest.mark.parametrize("c_out,relu", [(17, False), (24, True), (32, False)])
@pytest.mark.parametrize("ext,density,cap", [((60, 60, 60), 0.025, 1151 * 128), ((60, 60, 60), 0.025, 1151 * 128 + 1), ((80, 80, 80), 0.0105, 0),
                                             ((80, 80, 80), 0.0118, 0), ((80, 80, 80), 0.027, 0), ((80, 80, 81), 0.3, 0)])
def test_compaction_of_seventeen_to_thirty_two_channels(ext, density, cap, c_out, relu):
    """Either side of 1152 tiles of capacity, and from 1 k to 4 k tiles in use, one, two, three and four a workgroup: small
    whole numbers, nothing selected."""
    rng = np.random.default_rng(c_out)
    coords = random_sparse_sites(rng, ext, 1, density)
    feats = rng.integers(1, 4, size=(len(coords), 1)).astype(np.float32)
    w = rng.integers(-2, 3, size=(27, 1, c_out)).astype(np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, 1, coords, feats, (3, 3, 3), w, rho_up=1.0, relu=relu)
    gc, gf, n = scnn.sparse_conv_fwd(ext, 1, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats)), (3, 3, 3),
                                     torch.from_numpy(w).cuda(), rho_up=1.0, relu=relu, cand_capacity=cap)
    print(ext, c_out, len(coords), int(n[1]) / 128, cap, flush=True)
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf) and int(n[2]) == 0


@pytest.mark.parametrize("c_out,mode,relu,pool", [(33, scnn.ABS, False, False), (64, scnn.SIGNED, True, False), (50, scnn.ABS, True, True)])
@pytest.mark.parametrize("ext,batch,density,rho,cap", [((20, 21, 22), 17, 0.03, 0.2, 0), ((20, 21, 22), 37, 0.03, 0.2, 0), ((3, 5), 2, 0.5, 1.0, 0),
                                                       ((9, 10, 11), 40, 0.2, 1.0, 0), ((20, 21, 22), 17, 0.0005, 1.0, 0), ((120, 150), 13, 0.2, 0.3, 0)])
def test_compaction_of_wide_layers_without_marks(ext, batch, density, rho, cap, c_out, mode, relu, pool):
    """Counted first, where nothing is selected on more than 256 tiles of capacity, and by look-back: samples without rows, a tile a
    workgroup and none, a small output.  Small whole numbers, the oracle's rows."""
    rng = np.random.default_rng(c_out + batch)
    k = (3,) * len(ext)
    coords = random_sparse_sites(rng, ext, batch, density)
    coords = coords[coords[:, 0] % 5 != 1]
    feats = rng.integers(1, 4, size=(len(coords), 2)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), 2, c_out)).astype(np.float32)
    w[:, :, :6] *= rng.random((3 ** len(ext), 1, 1)) < 0.3  # (rows whose first channels are zero)
    c, f, t = (torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats, w))
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
    gc, gf, n = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=rho, topk_mode=mode, relu=relu, pool=pool, cand_capacity=cap)
    print(ext, c_out, len(coords), n.tolist(), flush=True)
    assert int(n[2]) == 0 and np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)
    if len(rc) > 100:
        out = (torch.full((70, 1 + len(ext)), -7, dtype=torch.int32, device="cuda"), torch.full((70, c_out), -7.0, device="cuda"),
               torch.zeros(4, dtype=torch.int64, device="cuda"))
        scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=rho, topk_mode=mode, relu=relu, pool=pool, cand_capacity=cap, out_capacity=64, out=out,
                             sync=False)
        assert int(out[2][0]) == len(rc) and int(out[2][2]) == 2 and np.array_equal(out[0][:64].cpu().numpy(), rc[:64])
        assert np.array_equal(out[1][:64].cpu().numpy(), rf[:64]) and bool((out[0][64:] == -7).all()) and bool((out[1][64:] == -7).all())


@pytest.mark.parametrize("c_out,mode,relu,pool", [(33, scnn.ABS, False, False), (64, scnn.SIGNED, True, False), (50, scnn.ABS, True, True)])
@pytest.mark.parametrize("ext,batch,density,rho", [((20, 21, 22), 60, 0.03, 0.2), ((20, 21, 22), 60, 0.03, 0.5), ((110, 120), 26, 0.3, 0.3), ((60, 60, 80), 1, 0.03, 1.0),
                                                   ((64, 66, 70), 2, 0.02, 1.0)])
def test_counted_compaction_of_several_tiles_a_workgroup(ext, batch, density, rho, c_out, mode, relu, pool):
    """The same from 1025 tiles in use on, where workgroups own two tiles and more and the last ones fewer: selecting layers of
    more than 2048 tiles of capacity (many equal scores, cut inside a tile) and layers that select nothing."""
    rng = np.random.default_rng(c_out + batch)
    coords = random_sparse_sites(rng, ext, batch, density)
    coords = coords[(coords[:, 0] % 5 != 1) | (batch < 5)]
    n_sites = int(np.prod(ext))
    assert rho == 1.0 or (n_sites <= 32768 and min(batch * n_sites, len(coords) * 3 ** len(ext)) // 128 + batch > 2048)
    feats = rng.integers(1, 4, size=(len(coords), 2)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), 2, c_out)).astype(np.float32)
    w[:, :, :6] *= rng.random((3 ** len(ext), 1, 1)) < 0.3  # (rows whose first channels are zero)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, (3,) * len(ext), w, rho_up=rho, topk_mode=mode, relu=relu, pool=pool, threads=8)
    gc, gf, n = scnn.sparse_conv_fwd(ext, batch, *(torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in (coords, feats)), (3,) * len(ext),
                                     torch.from_numpy(w).cuda(), rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
    print(ext, batch, c_out, len(coords), n.tolist(), flush=True)
    assert int(n[1]) > 1024 * 128 and int(n[2]) == 0
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)
