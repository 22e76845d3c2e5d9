"""A grid line of 2^31 - 1 sites, the longest that the library takes: sites at both of its ends and in the middle, where
32-bit sums of site, extent and offset would wrap.  Few rows, so the expected sums are written out from a table of sites."""
import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn

pytestmark = pytest.mark.gpu

E2 = 2 ** 31 - 1
SITES = [0, 1, 5, 70, 2 ** 30 - 1, 2 ** 30, E2 - 40, E2 - 3, E2 - 1]


def _dev(a):
    return torch.from_numpy(np.ascontiguousarray(a)).cuda()


def _rows(values):
    sites = sorted(values)
    coords = np.array([[0, 0, s] for s in sites], dtype=np.int32)
    return sites, coords, np.stack([values[s] for s in sites]).astype(np.float32)


@pytest.mark.parametrize("taps", [1, 5, 31])
@pytest.mark.parametrize("c_in,c_out,path,kernel", [(1, 8, 0, "k_conv_valu"), (8, 8, 1, "k_conv_valu"),
                                                    (32, 16, 2, "k_conv_quad"), (32, 16, 3, "k_conv_mfma_split"),
                                                    (32, 16, 5, "k_conv_quad_split")])
def test_sites_at_the_ends_of_the_longest_line(taps, c_in, c_out, path, kernel):
    """Small whole numbers: every sum is exact.  Forward, and backward with a gradient on every output row."""
    rng = np.random.default_rng(taps * 100 + c_in)
    w = rng.integers(-3, 4, size=(taps, c_in, c_out)).astype(np.float32)
    x = {s: rng.integers(1, 4, size=c_in) for s in SITES}
    _, coords, feats = _rows(x)
    h = taps // 2
    out = {}
    for s in SITES:
        for t in range(taps):
            if 0 <= s + h - t < E2:
                out[s + h - t] = out.get(s + h - t, 0) + x[s] @ w[t]
    out = {s: v for s, v in out.items() if np.any(v != 0)}
    _, want_c, want_f = _rows(out)
    g = {s: rng.integers(-3, 4, size=c_out) for s in out}
    _, g_coords, g_feats = _rows(g)
    want_data = np.zeros_like(feats)
    want_filter = np.zeros_like(w)
    for r, s in enumerate(SITES):
        for t in range(taps):
            if s + h - t in g:
                want_data[r] += w[t] @ g[s + h - t]
                want_filter[t] += np.outer(x[s], g[s + h - t])
    want_filter *= w != 0
    print(taps, c_in, c_out, path, flush=True)
    scnn.set_conv_path(path)
    try:
        oc, of, nnz = scnn.sparse_conv_fwd((1, E2), 1, _dev(coords), _dev(feats), (1, taps), _dev(w))
        assert scnn.last_conv_kernel() == kernel and int(nnz[2]) == 0
        data, filt, info = scnn.sparse_conv_bwd((1, E2), 1, _dev(coords), _dev(feats), (1, taps), _dev(w), _dev(g_coords),
                                                _dev(g_feats))
    finally:
        scnn.set_conv_path(0)
    assert np.array_equal(oc.cpu().numpy(), want_c) and np.array_equal(of.cpu().numpy(), want_f)
    assert int(info[2]) == 0
    assert np.array_equal(data.cpu().numpy(), want_data) and np.array_equal(filt.cpu().numpy(), want_filter)
