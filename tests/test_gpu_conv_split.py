"""The split-operand convolution (fp32 operands as three bf16 numbers) at the sizes where it can go wrong: units of 256
candidate sites with remainders, ends of samples, odd channel counts, filters other than 3x3x3, wide magnitudes, and the
kernel that takes over where its 31-bit offsets end."""
import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn
from tests.test_gpu_parity import check_conv_against_oracle, say
from workloads.generators import make_filter, random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extent,batch,c_in,c_out,ksize,density", [
    ((1, 1, 1), 1, 32, 64, (3, 3, 3), 1.0),          # one site
    ((3, 3, 3), 5, 32, 33, (3, 3, 3), 0.2),          # samples of less than a tile, odd number of tiles
    ((6, 7, 6), 1, 32, 17, (3, 3, 3), 0.6),          # 252 sites: just below a unit
    ((8, 8, 4), 1, 64, 64, (3, 3, 3), 0.9),          # exactly one unit, every tap present
    ((7, 37, 1), 1, 32, 1, (3, 3, 3), 0.5),          # 259 sites: just above a unit
    ((9, 9, 9), 3, 24, 65, (3, 3, 3), 0.3),          # a second group of one output channel, padded input chunk
    ((300, 5), 2, 48, 16, (5, 5), 0.2),              # 2-D, 25 taps
    ((40, 70), 1, 96, 48, (3, 9), 0.3),              # three chunks, 27 taps that are no 3x3x3
    ((2, 2, 90), 1, 40, 31, (1, 1, 31), 0.2),        # one filter line over two bitmap words
    ((13, 11, 130), 1, 128, 100, (3, 3, 3), 0.05),   # four chunks, rows longer than a bitmap word
])
def test_split_convolution_edges(extent, batch, c_in, c_out, ksize, density):
    rng = np.random.default_rng(c_in * 1000 + c_out)
    coords = random_sparse_sites(rng, extent, batch, density)
    if coords.shape[0] == 0:
        coords = np.zeros((1, 1 + len(extent)), dtype=np.int32)
    feats = (1.0 - rng.random((coords.shape[0], c_in))).astype(np.float32)
    w = make_filter(rng, ksize, c_in, c_out, 0.8, 0.2)
    bias = rng.normal(size=c_out).astype(np.float32)
    n = int(np.prod(extent))
    scnn.set_conv_path(5)
    try:
        for rho, mode in ((1.0, scnn.ABS), (0.3, scnn.SIGNED)):
            say(f"split {extent} B={batch} {c_in}->{c_out} {ksize} rho={rho}")
            check_conv_against_oracle(extent, batch, coords, feats, ksize, w, bias, scnn.k_from_rho(rho, n), rho, mode,
                                      tag=f"split {extent} {c_in}->{c_out}")
        assert scnn.last_conv_kernel() == "k_conv_quad_split"
    finally:
        scnn.set_conv_path(0)


@pytest.mark.parametrize("path,c_in,c_out,k", [(5, 32, 64, 3), (5, 64, 32, 3), (3, 32, 64, 5), (3, 64, 32, 5)])
def test_split_convolution_over_wide_magnitudes(path, c_in, c_out, k):
    """Rows and weights spread over many binades, on the quad and on the pair-list form.  With A = the sum of a response's
    product magnitudes and u = 2^-24: per (tap, 32-channel chunk) the parts' products left out are below 2 u A together,
    the instructions and the addition of their two sums round by at most 7 u A (the large products' 32 terms make most of
    it); then at most taps fp32 additions where the outer sums are fp32 (32 channels, quad form), else one rounding:
    (10 + taps) u A or 10 u A, whatever the magnitudes.
    (One of the six products left out would give 6.9e-6 A = 115 u A or more on this data.)"""
    rng = np.random.default_rng(c_in)
    ext, batch = (12, 12, 12), 2
    coords = random_sparse_sites(rng, ext, batch, 0.3)
    scale = 2.0 ** rng.integers(-40, 40, size=(coords.shape[0], 1))
    feats = (rng.normal(size=(coords.shape[0], c_in)) * scale * 2.0 ** rng.integers(-12, 12, size=(1, c_in))).astype(np.float32)
    taps, p = k ** 3, k // 2
    w = (rng.normal(size=(taps, c_in, c_out)) * 2.0 ** rng.integers(-10, 10, size=(taps, c_in, c_out))).astype(np.float32)
    d = torch.device("cuda")
    scnn.set_conv_path(path)
    try:
        oc, of, _ = scnn.sparse_conv_fwd(ext, batch, torch.from_numpy(coords).to(d), torch.from_numpy(feats).to(d), (k,) * 3,
                                         torch.from_numpy(w).to(d))
        assert scnn.last_conv_kernel() == ("k_conv_quad_split" if path == 5 else "k_conv_mfma_split")
    finally:
        scnn.set_conv_path(0)
    grid = np.full((batch, *(e + 2 * p for e in ext)), -1)
    grid[tuple(coords[:, 0:1].T) + tuple(coords[:, 1:].T + p)] = np.arange(coords.shape[0])
    oc, of = oc.cpu().numpy(), of.cpu().numpy()
    ref, mag = np.zeros(of.shape), np.zeros(of.shape)
    x64, w64 = np.vstack([feats, np.zeros((1, c_in))]).astype(np.float64), w.astype(np.float64)
    for t, (i, j, l) in enumerate(np.ndindex(k, k, k)):
        r = grid[oc[:, 0], oc[:, 1] + i, oc[:, 2] + j, oc[:, 3] + l]
        ref += x64[r] @ w64[t]
        mag += np.abs(x64[r]) @ np.abs(w64[t])
    worst = float((np.abs(of - ref) / np.maximum(mag, 1e-300)).max())
    say(f"split wide magnitudes {c_in}->{c_out} k={k}: worst |error| / A = {worst:.3g}")
    assert worst <= (10 + (taps if path == 5 and c_in == 32 else 0)) * 2.0 ** -24
    assert oc.shape[0] > 0


@pytest.mark.parametrize("share", [1.0, 1 / 6, 1 / 40])
@pytest.mark.parametrize("path,c_in,c_out,k", [(5, 16, 32, 3), (5, 32, 64, 3), (5, 64, 64, 3), (5, 128, 64, 3), (3, 32, 64, 5),
                                               (3, 64, 64, 5), (3, 128, 64, 5)])
def test_split_convolution_is_no_further_from_64_bits_than_fp32_products(path, c_in, c_out, k, share):
    """Rows with all, a sixth (what a selection and ReLU leave) and a 40th of their entries: relative 2-norm of the error
    over all responses.  Up to 32 taps the fp32 quad kernel's on the same data bounds it.  Where the outer sums are fp64,
    two independent roundings to fp32 (a chunk's and the response's, 2.53e-8 each: u / sqrt(3), averaged over mantissas)
    make 3.6e-8; what the instruction and the products left out add raises it to at most 4.9e-8 on full rows, and with
    the few products of sparse ones to 4.0e-8."""
    rng = np.random.default_rng(c_in + k)
    ext, taps, p = (24, 24, 24), k ** 3, k // 2
    coords = random_sparse_sites(rng, ext, 1, 0.1)
    n = coords.shape[0]
    feats = (np.abs(rng.normal(size=(n, c_in))) * (rng.random((n, c_in)) < share)).astype(np.float32)
    w = (rng.normal(size=(taps, c_in, c_out)) * 0.2).astype(np.float32)
    c, f, wt = (torch.from_numpy(a).cuda() for a in (coords, feats, w))
    err = {}
    for run in (path, 2) if k == 3 else (path,):
        scnn.set_conv_path(run)
        try:
            oc, of, _ = scnn.sparse_conv_fwd(ext, 1, c, f, (k, k, k), wt)
            kernel = scnn.last_conv_kernel()
        finally:
            scnn.set_conv_path(0)
        assert kernel == {5: "k_conv_quad_split", 3: "k_conv_mfma_split", 2: "k_conv_quad"}[run]
        grid = torch.full([e + 2 * p for e in ext], n, device="cuda")
        grid[tuple(c[:, 1 + a].long() + p for a in range(3))] = torch.arange(n, device="cuda")
        x64, ref = torch.cat([f.double(), torch.zeros((1, c_in), device="cuda", dtype=torch.float64)]), 0
        o = oc.long()
        for t, (i, j, l) in enumerate(np.ndindex(k, k, k)):
            ref = ref + x64[grid[o[:, 1] + i, o[:, 2] + j, o[:, 3] + l]] @ wt[t].double()
        err[run] = float((of.double() - ref).norm() / ref.norm())
    say(f"split accuracy {c_in}->{c_out} k={k} share={share:.3f}: {err}")
    if k == 3:
        assert err[5] <= err[2]
    if k == 5 or c_in > 32:
        assert err[path] <= (4.9e-8 if share == 1 else 4.0e-8)


@pytest.mark.parametrize("seed", range(6))
def test_split_and_vector_kernels_agree_over_layer_sizes(seed):
    """Layer sizes from less than one unit of 256 candidate sites per workgroup to several, with one and with eight chunks
    of units per XCD: every response, selection bypassed, against the vector kernels (fp64 sums, compared with the oracle
    elsewhere)."""
    from tests.parity import ATOL, RTOL
    rng = np.random.default_rng(7100 + seed)
    c_in, c_out = [(32, 64), (16, 24), (32, 96), (48, 48), (24, 24), (64, 32)][seed]
    e = [20, 64, 48, 40, 72, 56][seed]
    extent, batch = (e, e, int(rng.integers(8, e + 1))), 1 + seed % 3 * 2
    coords = random_sparse_sites(rng, extent, batch, float(rng.choice([0.02, 0.05, 0.3])))
    feats = rng.normal(size=(coords.shape[0], c_in)).astype(np.float32)
    w = (rng.normal(size=(27, c_in, c_out)) * 0.04).astype(np.float32)
    out = {}
    try:
        for path in (1, 5):
            scnn.set_conv_path(path)
            oc, of, n = scnn.sparse_conv_fwd(extent, batch, *(torch.from_numpy(a).cuda() for a in (coords, feats)),
                                             (3, 3, 3), torch.from_numpy(w).cuda())
            assert int(n[2]) == 0
            out[path] = (oc, of.double(), scnn.last_conv_kernel())
    finally:
        scnn.set_conv_path(0)
    say(f"split sizes seed={seed} extent={extent} B={batch} {c_in}->{c_out} sites out={out[1][0].shape[0]}")
    assert out[1][2] == "k_conv_valu" and out[5][2] == "k_conv_quad_split"
    assert torch.equal(out[1][0], out[5][0])
    assert bool(((out[1][1] - out[5][1]).abs() <= RTOL * out[1][1].abs() + ATOL).all())


def test_inputs_beyond_the_split_kernels_offsets():
    """A layer sized for more than 2^31 / 192 rows of 32 channels runs on the fp32 quad kernel, one of the same grid sized
    for its rows on the split kernel; same responses within the parity tolerance, rows past the device count never read."""
    ext, batch, cap = (40, 40, 40), 1, (1 << 31) // 192 + 1000   # (501 tiles: more than the small layers' 384)
    rng = np.random.default_rng(5)
    coords = random_sparse_sites(rng, ext, batch, 0.1)
    feats = (1.0 - rng.random((coords.shape[0], 32))).astype(np.float32)
    w = torch.from_numpy(make_filter(rng, (3, 3, 3), 32, 64, 1.0, 0.2)).cuda()
    c, f = torch.from_numpy(coords).cuda(), torch.from_numpy(feats).cuda()
    big_c = torch.zeros((cap, 4), dtype=torch.int32, device="cuda")
    big_f = torch.zeros((cap, 32), dtype=torch.float32, device="cuda")
    big_c[:c.shape[0]], big_f[:c.shape[0]] = c, f
    small = scnn.sparse_conv_fwd(ext, batch, c, f, (3, 3, 3), w)
    assert scnn.last_conv_kernel() == "k_conv_quad_split"
    lay = scnn.ChainedLayer(ext, batch, cap, 32, (3, 3, 3), w)
    oc, of, nnz = lay(big_c, big_f, torch.tensor([c.shape[0]], dtype=torch.int64, device="cuda"))
    assert scnn.last_conv_kernel() == "k_conv_quad"
    n = int(nnz.cpu()[0])
    assert n == small[0].shape[0] and torch.equal(oc[:n], small[0])
    a, b = of[:n].double(), small[1].double()
    assert bool(((a - b).abs() <= 1e-5 * b.abs() + 1e-6).all())


@pytest.mark.parametrize("c_in,ksize", [(32, (3, 3, 3)), (24, (3, 3, 3)), (16, (5, 5, 5)), (64, (5, 5, 5))])
def test_infinities_and_nan_stay_what_they_are(c_in, ksize):
    """One row with an infinity, one with a NaN, one with the largest fp32 number: sites that see the infinity get it with
    the sign of the weight, sites that see the NaN get NaN, and no other response stops being finite.  The split and the
    pair-list kernel (the 5x5x5 filters)."""
    rng = np.random.default_rng(c_in)
    ext, c_out = (24, 24, 24), 32
    coords = random_sparse_sites(rng, ext, 1, 0.1)
    feats = (1.0 - rng.random((coords.shape[0], c_in))).astype(np.float32)
    t = int(np.prod(ksize))
    w = rng.normal(size=(t, c_in, c_out)).astype(np.float32) * np.float32(0.1)
    n = coords.shape[0]
    feats[n // 4, c_in - 1], feats[n // 2, 0], feats[3 * n // 4, 3] = np.inf, np.nan, np.finfo(np.float32).max
    d = torch.device("cuda")
    scnn.set_conv_path(5 if ksize == (3, 3, 3) else 3)
    try:
        oc, of, _ = scnn.sparse_conv_fwd(ext, 1, torch.from_numpy(coords).to(d), torch.from_numpy(feats).to(d), ksize,
                                         torch.from_numpy(w).to(d))
        say(f"non-finite rows {c_in} {ksize}: {scnn.last_conv_kernel()}")
        assert scnn.last_conv_kernel() == ("k_conv_quad_split" if ksize == (3, 3, 3) else "k_conv_mfma" if c_in == 16
                                           else "k_conv_mfma_split")
    finally:
        scnn.set_conv_path(0)
    p = ksize[0] // 2
    grid = np.full((24 + 2 * p,) * 3, -1)
    grid[tuple(coords[:, 1:].T + p)] = np.arange(n)
    oc, of = oc.cpu().numpy(), of.cpu().numpy()
    ref = np.zeros(of.shape)
    x64 = np.vstack([feats, np.zeros((1, c_in))]).astype(np.float64)
    with np.errstate(invalid="ignore"):
        for k, (a, b, c) in enumerate(np.ndindex(*ksize)):
            ref += x64[grid[oc[:, 1] + a, oc[:, 2] + b, oc[:, 3] + c]] @ w[k].astype(np.float64)
    assert np.isinf(ref).any() and np.isnan(ref).any()
    assert np.array_equal(np.isnan(of), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(of), of, 0), np.where(np.isinf(ref), ref, 0))


@pytest.mark.parametrize("path,c_in,c_out,ksize", [(5, 16, 32, (3, 3, 3)), (5, 64, 64, (3, 3, 3)), (5, 96, 48, (3, 3, 3)),
                                                   (5, 128, 65, (3, 3, 1)), (3, 64, 64, (3, 3, 3)), (3, 32, 48, (5, 5, 5)),
                                                   (3, 96, 32, (5, 5, 5))])
@pytest.mark.parametrize("kind", ["row", "row_large_weights", "weight", "both", "overflow", "tiny"])
def test_values_that_three_bf16_numbers_do_not_hold(path, c_in, c_out, ksize, kind):
    """Infinite and NaN rows against weights of hundreds (whose middle parts are beyond 1 with either sign), an infinite
    and a NaN weight, an infinite row against an infinite weight, finite values whose products overflow, and values below
    2^-109: each response is what the sum over its own (row, tap) pairs gives - infinities with their sign, NaN, and finite
    values (all but the overflow kind's) to a few roundings of its products' magnitudes."""
    rng = np.random.default_rng(c_in + len(kind))
    ext, t = (16, 15, 17), int(np.prod(ksize))
    coords = random_sparse_sites(rng, ext, 1, 0.1)
    n = coords.shape[0]
    feats = (1.0 - rng.random((n, c_in))).astype(np.float32)
    w = (rng.normal(size=(t, c_in, c_out)) * (700 if kind == "row_large_weights" else 0.1)).astype(np.float32)
    if kind in ("row", "row_large_weights"):
        feats[n // 4, c_in - 1], feats[n // 2, 0], feats[3 * n // 4, 3] = np.inf, np.nan, -np.inf
    elif kind == "weight":
        w[1, 2, 5], w[t - 2, c_in - 1, c_out - 1], w[t // 2, 0, 0] = np.inf, np.nan, -np.inf
    elif kind == "both":
        feats[n // 3, 1], feats[n // 5, c_in - 2], w[0, 1, 3], w[t - 1, c_in - 2, 4] = np.inf, -np.inf, np.inf, -np.inf
    elif kind == "overflow":
        feats[n // 3, 1], feats[n // 2, 2], w[:, 1, :5] = 3e38, -3e38, np.float32(1e10) * rng.normal(size=(t, 5))
    else:
        feats = (feats * np.float32(2.0 ** -122)).astype(np.float32)
        w = (w * np.float32(2.0 ** 60)).astype(np.float32)
    scnn.set_conv_path(path)
    try:
        oc, of, _ = scnn.sparse_conv_fwd(ext, 1, *(torch.from_numpy(a).cuda() for a in (coords, feats)), ksize,
                                         torch.from_numpy(w).cuda())
        assert scnn.last_conv_kernel() == ("k_conv_quad_split" if path == 5 else "k_conv_mfma_split")
    finally:
        scnn.set_conv_path(0)
    p = [k // 2 for k in ksize]
    grid = np.full([e + 2 * h for e, h in zip(ext, p)], -1)
    grid[tuple(coords[:, 1 + a] + p[a] for a in range(3))] = np.arange(n)
    oc, of = oc.cpu().numpy(), of.cpu().numpy()
    ref, mag = np.zeros(of.shape), np.zeros(of.shape)
    with np.errstate(invalid="ignore", over="ignore"):
        for k, off in enumerate(np.ndindex(*ksize)):
            r = grid[tuple(oc[:, 1 + a] + off[a] for a in range(3))]
            at = r >= 0
            ref[at] += feats[r[at]].astype(np.float64) @ w[k].astype(np.float64)
            mag[at] += np.abs(feats[r[at]]).astype(np.float64) @ np.abs(w[k]).astype(np.float64)
        ref = ref.astype(np.float32).astype(np.float64)
    say(f"split special values {kind} {c_in}->{c_out} {ksize} path={path}: {int(np.isinf(ref).sum())} inf, "
        f"{int(np.isnan(ref).sum())} NaN of {ref.size}")
    assert kind == "tiny" or not np.isfinite(ref).all()
    assert np.array_equal(np.isnan(of), np.isnan(ref))
    assert np.array_equal(np.where(np.isinf(of), of, 0), np.where(np.isinf(ref), ref, 0))
    ok = np.isfinite(ref) & np.isfinite(mag)
    # (fp32 chains of at most 32 products: half a rounding of their magnitudes on each; 27 fp32 additions of these)
    assert ok.any() and (np.abs(of[ok] - ref[ok]) <= (32 + 27) * 2.0 ** -24 * mag[ok] + 2.0 ** -149).all()


@pytest.mark.parametrize("extent,tiles,c_in,c_out,k,kernel", [
    ((48, 48, 48), 600, 96, 48, 3, "k_conv_mfma_split"),    # 96 and 128 channels: pair lists where they take the width ..
    ((48, 48, 48), 300, 128, 64, 3, "k_conv_mfma_split"),
    ((48, 48, 48), 600, 96, 40, 3, "k_conv_quad_split"),    # .. else as the narrower ones
    ((48, 48, 48), 383, 64, 64, 3, "k_conv_quad"),          # small layers
    ((48, 48, 48), 384, 64, 64, 3, "k_conv_quad_split"),
    ((48, 48, 48), 511, 16, 32, 3, "k_conv_quad"),
    ((48, 48, 48), 512, 16, 32, 3, "k_conv_quad_split"),
    ((400, 400), 1000, 16, 32, 5, "k_conv_quad"),           # 16 channels in 2-D
    ((48, 48, 48), 600, 16, 48, 5, "k_conv_mfma"),          # more than 32 taps
    ((48, 48, 48), 600, 32, 48, 5, "k_conv_mfma_split"),
    ((400, 400), 575, 32, 32, 5, "k_conv_quad"),
    ((400, 400), 576, 32, 32, 5, "k_conv_quad_split"),
])
def test_the_kernel_by_shape_and_size(extent, tiles, c_in, c_out, k, kernel):
    """The library's choice on both sides of each line of its rule (workspaces of `tiles` tiles; a solid block of sites, so
    that its candidates fit them and rows x taps does not bound them)."""
    rng = np.random.default_rng(tiles)
    edge = 15 if len(extent) == 3 else 72
    coords = np.stack([np.zeros(edge ** len(extent)), *(i.reshape(-1) for i in np.indices((edge,) * len(extent)))], 1)
    coords = np.ascontiguousarray(coords.astype(np.int32))
    args = [torch.from_numpy(a).cuda() for a in (coords, rng.random((coords.shape[0], c_in)).astype(np.float32))]
    w = torch.from_numpy(rng.normal(size=(k ** len(extent), c_in, c_out)).astype(np.float32)).cuda()
    cap = (tiles - 1) * 128
    _, _, n = scnn.sparse_conv_fwd(extent, 1, *args, (k,) * len(extent), w, cand_capacity=cap, out_capacity=cap)
    say(f"kernel choice {extent} {tiles} tiles {c_in}->{c_out}: {scnn.last_conv_kernel()}")
    assert int(n[2]) == 0 and scnn.last_conv_kernel() == kernel
