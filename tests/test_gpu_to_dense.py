"""sparseToDense on outputs large enough for the form that writes every plane once, and the attention step's layout
conversion with channel counts that take each of its two load widths."""
import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn
import oracle
from tests.test_gpu_parity import dev, host, say
from workloads.generators import random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("extent,batch,channels,density", [
    ((64, 64, 64), 4, 8, 0.25),      # exactly 32 MiB: the smallest output of this form (at this many rows)
    ((64, 64, 64), 4, 8, 0.05),      # .. and with fewer rows than the form asks for at this size
    ((65, 67, 63), 3, 13, 0.08),     # odd sizes, scalar row loads
    ((900, 1100), 2, 24, 0.001),     # 2-D, nearly empty
    ((50, 40, 70), 5, 64, 0.9),      # nearly full
    ((33, 64, 64), 3, 33, 0.8),      # nearly full, scalar row loads: the two launches
])
def test_large_dense_outputs(extent, batch, channels, density):
    rng = np.random.default_rng(channels)
    coords = random_sparse_sites(rng, extent, batch, density)
    feats = rng.normal(size=(coords.shape[0], channels)).astype(np.float32)
    want = oracle.sparse_to_dense(extent, batch, coords, feats)
    out = torch.full((batch, channels, *extent), 7.0, dtype=torch.float32, device="cuda:0")
    say(f"large dense {extent} B={batch} C={channels} rows={coords.shape[0]}")
    assert np.array_equal(host(scnn.sparse_to_dense(extent, batch, dev(coords), dev(feats), out=out)), want)
    # rows in any order, some outside the grid, the count taken from the device
    order = rng.permutation(coords.shape[0])
    c2 = np.concatenate([coords[order], np.full((3, coords.shape[1]), 10 ** 6, np.int32), coords[:5]])
    f2 = np.concatenate([feats[order], np.ones((3, channels), np.float32), np.full((5, channels), 9.0, np.float32)])
    n = torch.tensor([coords.shape[0] + 3], dtype=torch.int64, device="cuda:0")
    out.fill_(float("nan"))
    assert np.array_equal(host(scnn.sparse_to_dense(extent, batch, dev(c2), dev(f2), rows_dev=n, out=out)), want)


@pytest.mark.parametrize("batch,channels", [(1, 3), (2, 64), (16, 12), (17, 12), (33, 68), (5, 130)])
def test_attention_on_few_and_many_samples(batch, channels):
    """Sample bounds by waves (up to 16 samples) and by threads, row loads of 16 and of 4 bytes; empty samples."""
    rng = np.random.default_rng(batch)
    extent = (9, 8, 7)
    coords = random_sparse_sites(rng, extent, batch, 0.4)
    coords = np.ascontiguousarray(coords[coords[:, 0] % 3 != 1])
    resp = rng.integers(-4, 5, size=(coords.shape[0], channels)).astype(np.float32)
    for rows in (coords.shape[0], 1):
        oc, of = oracle.attention_topk(extent, batch, coords[:rows], resp[:rows], 20, scnn.ABS)
        gc, gf, _ = scnn.attention_topk(extent, batch, dev(coords[:rows]), dev(resp[:rows]), 20, scnn.ABS)
        assert np.array_equal(host(gc), oc) and np.array_equal(host(gf), of)
