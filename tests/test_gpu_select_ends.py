"""Where the selection of a column stops: the k-th strongest key among 1 to 4096 entries that share its leading bits (63 to 66
around the 64 that a wave ranks), one key apart, three, many or equal, the first of them, the last and all, on columns either side
of 1024, 4096, 16384 and 32768 positions."""
import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn

pytestmark = pytest.mark.gpu

APART = (1, 0, 3, 1 << 14)  # keys between neighbours of the cluster, by channel


def column(rng, n, cluster, above, apart):
    """n values in random order: `above` from 4 to 8, `cluster` from 2 upwards `apart` keys apart, the rest from 0.5 to 1."""
    v = rng.uniform(0.5, 1.0, n).astype(np.float32)
    v[:above] = rng.uniform(4.0, 8.0, above)
    v[above:above + cluster] = (np.float32(2.0).view(np.uint32) + apart * np.arange(cluster, dtype=np.uint32)).view(np.float32)
    return rng.permutation(v)


@pytest.mark.parametrize("mode", [scnn.ABS, scnn.SIGNED])
@pytest.mark.parametrize("ext,batch,channels", [
    ((31, 33), 1, 4), ((32, 32), 1, 4), ((1025,), 1, 4), ((64, 64), 1, 4), ((64, 64), 300, 4), ((4097,), 1, 4), ((4097,), 40, 4), ((128, 128), 1, 4),
    ((16385,), 1, 4), ((128, 256), 1, 4), ((32769,), 1, 4), ((400, 500), 1, 4), ((200, 200), 1, 20), ((200, 300), 70, 4)])
def test_entries_that_share_their_leading_bits(ext, batch, channels, mode):
    apart = APART * (channels // len(APART))
    ext = ext if len(ext) > 1 else (1, ext[0])
    n = int(np.prod(ext))
    rng = np.random.default_rng(n + batch)
    coords = np.stack(np.unravel_index(np.arange(batch * n), (batch, *ext)), 1).astype(np.int32)
    c = torch.from_numpy(coords).cuda()
    for cluster in (1, 63, 64, 65, 66, 600) + ((4096,) if n > 8192 else ()):
        above = int(rng.integers(1, n // 4))
        cluster = min(cluster, n // 2)
        values = np.stack([column(rng, n, cluster, above, a) for a in apart], 1)
        sign = np.where(rng.random(values.shape) < 0.3, -1, 1).astype(np.float32) if mode == scnn.ABS else np.float32(1)
        resp = torch.from_numpy(np.tile(values * sign, (batch, 1))).cuda()
        order = [np.argsort(-values[:, j], kind="stable") for j in range(channels)]  # (ties: the lower site)
        for k in sorted({above, above + 1, above + (cluster + 1) // 2, above + cluster - 1, above + cluster, above + cluster + 1}):
            print(ext, batch, mode, cluster, above, k, flush=True)
            kept = np.zeros(values.shape, bool)
            for j in range(channels):
                kept[order[j][:k], j] = True
            want = np.where(kept, values * sign, 0).astype(np.float32)
            rows = kept.any(1)
            oc, of, nnz = scnn.attention_topk(ext, batch, c, resp, k, mode)
            assert nnz.tolist()[:3] == [batch * int(rows.sum()), batch * n, 0]
            assert torch.equal(oc, c[torch.from_numpy(np.tile(rows, batch)).cuda()])
            assert np.array_equal(of.view(batch, -1, channels)[[0, -1]].cpu().numpy(), np.stack([want[rows]] * 2))
