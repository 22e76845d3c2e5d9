"""Layers of small samples, one workgroup a sample: the shapes at the ends of what it takes, one sample and several, against
the oracle and against the general path (scnn_set_conv_path(1)), bit for bit on small whole numbers."""
import numpy as np
import pytest
import torch

import oracle
import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


def gpu(*arrays):
    return [None if a is None else torch.from_numpy(np.ascontiguousarray(a)).cuda() for a in arrays]


def layer(rng, ext, batch, c_in, c_out, k, density):
    coords = random_sparse_sites(rng, ext, batch, density)
    coords = coords[(coords[:, 0] % 3 != 1) | (rng.random(len(coords)) < 0.1)]  # (samples of different sizes)
    feats = rng.integers(1, 4, size=(len(coords), c_in)).astype(np.float32)
    w = rng.integers(-2, 3, size=(int(np.prod(k)), c_in, c_out)).astype(np.float32)
    w[rng.integers(0, len(w))] = 0.0
    return coords, feats, w


@pytest.mark.parametrize("mode,relu,pool,bias", [(scnn.ABS, True, True, False), (scnn.SIGNED, False, True, True), (scnn.ABS, False, False, True),
                                                 (scnn.SIGNED, True, False, False)])
@pytest.mark.parametrize("ext,k,batch,c_in,c_out,density", [
    ((1, 1), (3, 3), 1, 1, 1, 1.0), ((1, 64), (1, 3), 2, 1, 8, 0.4), ((65, 1), (3, 1), 3, 2, 9, 0.5), ((28, 28), (3, 3), 1, 1, 8, 0.19),
    ((28, 28), (3, 3), 300, 1, 8, 0.19), ((7, 9), (3, 5), 700, 3, 5, 0.3), ((32, 64), (3, 3), 2, 1, 12, 0.3), ((32, 64), (3, 3), 1, 1, 8, 1.0),
    ((23, 89), (5, 5), 2, 1, 7, 0.2), ((31, 30), (3, 3), 2, 8, 16, 0.2), ((10, 10, 10), (3, 3, 3), 3, 1, 16, 0.15), ((9, 11, 13), (3, 3, 3), 1, 5, 8, 0.2),
    ((12, 12, 12), (1, 1, 31), 2, 1, 8, 0.2), ((5, 6, 7), (3, 3, 3), 257, 8, 3, 0.3), ((2, 3, 300), (3, 3, 3), 2, 1, 4, 0.3)])
def test_layers_of_small_samples(ext, k, batch, c_in, c_out, density, mode, relu, pool, bias):
    rng = np.random.default_rng(c_out + ext[0])
    coords, feats, w = layer(rng, ext, batch, c_in, c_out, k, density)
    bv = rng.integers(-2, 3, size=c_out).astype(np.float32) if bias else None
    c, f, t, b = gpu(coords, feats, w, bv)
    print(ext, k, batch, c_in, c_out, len(coords), flush=True)
    for rho in (0.0, 0.1, 0.5, 1.0):
        rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, bias=bv, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
        gc, gf, n = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, b, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
        assert scnn.last_conv_kernel() == "k_layer_tiny"
        assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)
        assert [int(v) for v in n[2:]] == [0, 0]
        scnn.set_conv_path(1)
        try:
            gc1, gf1, n1 = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, b, rho_up=rho, topk_mode=mode, relu=relu, pool=pool)
        finally:
            scnn.set_conv_path(0)
        assert torch.equal(gc, gc1) and torch.equal(gf, gf1) and torch.equal(n, n1)


@pytest.mark.parametrize("ext,batch,c_in,c_out,rows,kernel", [
    ((32, 64), 1, 1, 12, 2048, "k_layer_tiny"), ((32, 65), 1, 1, 8, 100, "k_conv_valu"), ((32, 64), 1, 1, 13, 100, "k_conv_valu"),
    ((20, 20), 2, 9, 8, 40, "k_conv_valu"), ((20, 20), 2, 1, 17, 40, "k_conv_valu"), ((20, 20), 1, 8, 16, 347, "k_layer_tiny"),
    ((20, 20), 1, 8, 16, 348, "k_conv_valu")])
def test_which_layers_it_takes(ext, batch, c_in, c_out, rows, kernel):
    n = ext[0] * ext[1]
    coords = np.array([(b, i // ext[1], i % ext[1]) for b in range(batch) for i in range(min(n, rows // batch))], dtype=np.int32)
    feats, w = np.ones((len(coords), c_in), np.float32), np.ones((9, c_in, c_out), np.float32)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, (3, 3), w, rho_up=0.2)
    gc, gf, _ = scnn.sparse_conv_fwd(ext, batch, *gpu(coords, feats), (3, 3), gpu(w)[0], rho_up=0.2)
    assert scnn.last_conv_kernel() == kernel
    assert np.array_equal(gc.cpu().numpy(), rc) and np.array_equal(gf.cpu().numpy(), rf)


@pytest.mark.parametrize("ext,batch,c_in,c_out,rich,rows,kernel", [
    ((12, 12, 12), 8, 8, 8, 1728, 0, "k_conv_valu"), ((12, 12, 12), 64, 8, 8, 1728, 0, "k_conv_valu"), ((12, 12, 12), 300, 8, 8, 1728, 1, "k_conv_valu"),
    ((20, 20), 8, 8, 16, 324, 0, "k_layer_tiny"), ((20, 20), 8, 8, 16, 325, 0, "k_conv_valu"), ((20, 20), 256, 8, 16, 400, 0, "k_layer_tiny"),
    ((45, 45), 8, 1, 12, 731, 0, "k_layer_tiny"), ((45, 45), 8, 1, 12, 733, 0, "k_conv_valu"), ((45, 45), 64, 1, 12, 2025, 0, "k_layer_tiny"),
    ((45, 45), 1024, 1, 8, 100, 1, "k_layer_tiny"), ((45, 45), 1025, 1, 8, 100, 1, "k_conv_valu"), ((28, 28), 5000, 1, 8, 100, 1, "k_layer_tiny"),
    ((3, 3), 5000, 8, 16, 9, 0, "k_conv_valu"), ((3, 3), 5000, 8, 16, 9, 1, "k_layer_tiny")])
def test_samples_of_unequal_rows(ext, batch, c_in, c_out, rich, rows, kernel):
    """The richest sample is what the launch waits for: one of `rich` rows among others of `rows`, the general path's bits."""
    n = int(np.prod(ext))
    lin = np.concatenate([np.arange(b * n, b * n + (rich if b == batch // 2 else rows)) for b in range(batch)])
    coords = np.stack(np.unravel_index(lin, (batch, *ext)), 1).astype(np.int32)
    rng = np.random.default_rng(rich)
    feats = rng.integers(1, 4, size=(len(coords), c_in)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), c_in, c_out)).astype(np.float32)
    c, f, t = gpu(coords, feats, w)
    print(ext, batch, c_in, c_out, len(coords), flush=True)
    gc, gf, nnz = scnn.sparse_conv_fwd(ext, batch, c, f, (3,) * len(ext), t, rho_up=0.3, relu=True, pool=True)
    assert scnn.last_conv_kernel() == kernel
    scnn.set_conv_path(1)
    try:
        gc1, gf1, nnz1 = scnn.sparse_conv_fwd(ext, batch, c, f, (3,) * len(ext), t, rho_up=0.3, relu=True, pool=True)
    finally:
        scnn.set_conv_path(0)
    assert torch.equal(gc, gc1) and torch.equal(gf, gf1) and torch.equal(nnz, nnz1)


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("batch", [1, 5])
def test_capacities_and_counts(batch, pool):
    """Too many candidates: no rows; too many rows: the first ones; a workspace asked for with more rows; a device count below
    the arrays' rows; no rows at all."""
    ext, k = (19, 21), (3, 3)
    rng = np.random.default_rng(batch)
    coords, feats, w = layer(rng, ext, batch, 1, 6, k, 0.2)
    c, f, t = gpu(coords, feats, w)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, rho_up=0.3, pool=pool)
    cap = batch * 19 * 21
    full = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=0.3, pool=pool)[2]
    for cand_cap, out_cap in ((int(full[1]), len(rc)), (int(full[1]) - 1, len(rc)), (cap, len(rc) - 3), (cap, 0)):
        out = (torch.full((len(rc) + 5, 3), -7, dtype=torch.int32, device="cuda"), torch.full((len(rc) + 5, 6), -7.0, device="cuda"),
               torch.zeros(4, dtype=torch.int64, device="cuda"))
        ws = torch.empty(scnn.sparse_conv_fwd_workspace(ext, batch, batch * 400, 1, 6, k, 2 if pool else 0, cap), dtype=torch.uint8, device="cuda")
        scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=0.3, pool=pool, cand_capacity=cand_cap, out_capacity=out_cap, out=out,
                             workspace=ws, sync=False)
        n = out[2].cpu().tolist()
        over = cand_cap < int(full[1])
        rows = 0 if over else len(rc)
        assert n == [rows, int(full[1]), (1 if over else 0) | (2 if rows > out_cap else 0), 0]
        kept = min(rows, out_cap)
        assert np.array_equal(out[0][:kept].cpu().numpy(), rc[:kept]) and np.array_equal(out[1][:kept].cpu().numpy(), rf[:kept])
        assert bool((out[0][kept:] == -7).all()) and bool((out[1][kept:] == -7).all())
    lay = scnn.ChainedLayer(ext, batch, len(coords), 1, k, t, rho_up=0.3, pool=pool)
    for rows in (len(coords) // 2, 0):
        rc, rf = oracle.sparse_conv_fwd(ext, batch, coords[:rows], feats[:rows], k, w, rho_up=0.3, pool=pool)
        cc, ff, n = lay(c, f, torch.tensor([rows], dtype=torch.int64, device="cuda"))
        assert n.cpu().tolist()[::2] == [len(rc), 0]
        assert np.array_equal(cc[:len(rc)].cpu().numpy(), rc) and np.array_equal(ff[:len(rc)].cpu().numpy(), rf)


@pytest.mark.parametrize("pool", [False, True])
@pytest.mark.parametrize("ext,batch,c_out,rows", [((19, 21), 40, 6, 3), ((45, 45), 9, 8, 40), ((45, 45), 300, 4, 20), ((6, 7, 8), 33, 12, 100)])
def test_staged_rows_lie_within_the_workspace(ext, batch, c_out, rows, pool):
    """Capacities from the candidates in use down to where the staged rows no longer fit and the general path takes the layer:
    samples without a row, with a few and full ones, the bytes past the workspace asked for untouched."""
    k, n = (3,) * len(ext), int(np.prod(ext))
    rng = np.random.default_rng(batch)
    counts = [0 if b % 3 == 0 else n if b == batch - 2 else int(rng.integers(1, rows)) for b in range(batch)]
    lin = np.concatenate([b * n + np.sort(rng.permutation(n)[:m]) for b, m in enumerate(counts)])
    coords = np.stack(np.unravel_index(lin, (batch, *ext)), 1).astype(np.int32)
    feats = rng.integers(1, 4, size=(len(coords), 1)).astype(np.float32)
    w = rng.integers(-2, 3, size=(3 ** len(ext), 1, c_out)).astype(np.float32)
    c, f, t = gpu(coords, feats, w)
    rc, rf = oracle.sparse_conv_fwd(ext, batch, coords, feats, k, w, rho_up=0.3, pool=pool)
    used = int(scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=0.3, pool=pool)[2][1])
    ran = set()
    for cap in (0, used, max(1, used // 2), 1):
        need = scnn.sparse_conv_fwd_workspace(ext, batch, len(coords), 1, c_out, k, 2 if pool else 0, cap)
        room = torch.full((need + 4096,), 0x5A, dtype=torch.uint8, device="cuda")
        print(ext, batch, len(coords), used, cap, need, flush=True)
        gc, gf, nnz = scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=0.3, pool=pool, cand_capacity=cap, workspace=room[:need],
                                           out_capacity=len(rc), sync=False)
        ran.add(scnn.last_conv_kernel())
        assert bool((room[need:] == 0x5A).all())
        if cap == 0 or cap >= used:
            assert nnz.cpu().tolist() == [len(rc), used, 0, 0]
            assert np.array_equal(gc[:len(rc)].cpu().numpy(), rc) and np.array_equal(gf[:len(rc)].cpu().numpy(), rf)
        else:
            assert nnz.cpu().tolist()[::2] == [0, 1]
    assert "k_layer_tiny" in ran


@pytest.mark.parametrize("batch", [1, 4])
def test_bad_rows_are_reported(batch):
    ext, k = (12, 13), (3, 3)
    rng = np.random.default_rng(3)
    coords, feats, w = layer(rng, ext, batch, 1, 4, k, 0.3)
    _, f, t = gpu(coords, feats, w)
    for row, column, value, flag in ((0, 1, 12, 4), (len(coords) - 1, 0, batch, 4), (len(coords) // 2, 2, -1, 4), (len(coords) // 2, 0, -1, 4)):
        bad = coords.copy()
        bad[row, column] = value
        n = scnn.sparse_conv_fwd(ext, batch, gpu(bad)[0], f, k, t, rho_up=0.3, sync=False)[2].cpu()
        assert scnn.last_conv_kernel() == "k_layer_tiny" and int(n[2]) & flag
    swapped = coords.copy()
    swapped[[4, len(coords) - 2]] = swapped[[len(coords) - 2, 4]]
    n = scnn.sparse_conv_fwd(ext, batch, gpu(swapped)[0], f, k, t, rho_up=0.3, sync=False)[2].cpu()
    assert int(n[2]) & 8


@pytest.mark.parametrize("batch", [1, 3])
def test_infinities_reach_the_sums_they_belong_to(batch):
    """An infinite row or weight meets present neighbours only: the bits of the general path, whose kernel for one input
    channel walks the same neighbours."""
    ext, k = (14, 15), (3, 3)
    rng = np.random.default_rng(5)
    coords, feats, w = layer(rng, ext, batch, 1, 5, k, 0.3)
    feats[7, 0], w[4, 0, 3] = np.inf, -np.inf
    c, f, t = gpu(coords, feats, w)
    for pool in (False, True):
        got = []
        for path in (0, 1):
            scnn.set_conv_path(path)
            try:
                got.append(scnn.sparse_conv_fwd(ext, batch, c, f, k, t, rho_up=0.4, pool=pool))
            finally:
                scnn.set_conv_path(0)
        assert torch.equal(got[0][0], got[1][0]) and torch.equal(got[0][2], got[1][2])
        assert torch.equal(got[0][1].nan_to_num(nan=1e30), got[1][1].nan_to_num(nan=1e30))
        assert not bool(torch.isfinite(got[0][1]).all())


@pytest.mark.parametrize("batch", [1, 5])
def test_two_layers_captured_in_a_graph(batch):
    """Chained, with device-resident row counts: every replay against call by call, other rows in the same buffers each time."""
    rng = np.random.default_rng(batch)
    ext, k, cap = (28, 28), (3, 3), batch * 200
    w1 = gpu(rng.integers(-2, 3, size=(9, 1, 8)).astype(np.float32))[0]
    w2 = gpu(rng.integers(-2, 3, size=(9, 8, 16)).astype(np.float32))[0]
    l1 = scnn.ChainedLayer(ext, batch, cap, 1, k, w1, rho_up=0.2, relu=True, pool=True)
    l2 = scnn.ChainedLayer(l1.out_extent, batch, l1.out_capacity, 8, k, w2, rho_up=0.3, relu=True)
    c, f = torch.zeros((cap, 3), dtype=torch.int32, device="cuda"), torch.ones((cap, 1), device="cuda")
    n = torch.zeros(1, dtype=torch.int64, device="cuda")
    graph, side = torch.cuda.CUDAGraph(), torch.cuda.Stream()
    side.wait_stream(torch.cuda.current_stream())
    with torch.cuda.stream(side):
        l2(*l1(c, f, n))
        assert scnn.last_conv_kernel() == "k_layer_tiny"
    torch.cuda.current_stream().wait_stream(side)
    torch.cuda.synchronize()
    with torch.cuda.graph(graph):
        oc, of, nnz = l2(*l1(c, f, n))
    for density in (0.15, 0.02, 0.2, 0.0):
        coords = random_sparse_sites(rng, ext, batch, density)[:cap]
        c[:len(coords)] = gpu(coords)[0]
        n.fill_(len(coords))
        oc.fill_(-1)
        graph.replay()
        torch.cuda.synchronize()
        c1, f1, _ = scnn.sparse_conv_fwd(ext, batch, c[:len(coords)], f[:len(coords)], k, w1, rho_up=0.2, relu=True, pool=True)
        c2, f2, n2 = scnn.sparse_conv_fwd((14, 14), batch, c1, f1, k, w2, rho_up=0.3, relu=True)
        assert nnz.cpu().tolist() == n2.tolist()
        assert torch.equal(oc[:len(c2)], c2) and torch.equal(of[:len(c2)], f2) and bool((oc[len(c2):] == -1).all())
