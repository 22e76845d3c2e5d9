"""Two host threads, a stream each, that launch the same kernel with different amounts of LDS: every call runs, with its own
result."""
import threading

import numpy as np
import pytest
import torch

import paper_1801_10585_amd as scnn
from workloads import random_sparse_sites

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("layers,kernel", [
    ((((45, 45), (3, 3), 1, 8, 0.1), ((40, 40), (3, 3), 1, 8, 0.1)), "k_layer_tiny"),
    ((((16, 17, 18), (3, 3, 3), 128, 66, 0.02), ((90, 91), (3, 3), 128, 66, 0.02)), "k_conv_quad"),
    ((((60, 61, 62), (3, 3, 3), 64, 64, 0.02), ((300, 301), (3, 3), 64, 64, 0.08)), "k_conv_quad_split")])
def test_two_threads_with_layers_of_different_lds(layers, kernel):
    calls, want = [], []
    for ext, k, c_in, c_out, density in layers:
        rng = np.random.default_rng(c_in)
        coords = random_sparse_sites(rng, ext, 2, density)
        feats = rng.integers(1, 4, size=(len(coords), c_in)).astype(np.float32)
        w = rng.integers(-2, 3, size=(int(np.prod(k)), c_in, c_out)).astype(np.float32)
        c, f, t = (torch.from_numpy(a).cuda() for a in (coords, feats, w))
        calls.append(lambda ext=ext, k=k, c=c, f=f, t=t, **kw: scnn.sparse_conv_fwd(ext, 2, c, f, k, t, rho_up=0.2, **kw))
        want.append(calls[-1]())
        assert scnn.last_conv_kernel() == kernel
    failed = []

    def work(call, ref):
        try:
            stream, rows = torch.cuda.Stream(), len(ref[0])
            with torch.cuda.stream(stream):
                for _ in range(300):
                    got = call(sync=False)
            stream.synchronize()
            assert torch.equal(got[0][:rows], ref[0]) and torch.equal(got[1][:rows], ref[1]) and torch.equal(got[2].cpu(), ref[2])
        except Exception as e:  # (an assertion of a thread does not reach the test by itself)
            failed.append(repr(e))

    torch.cuda.synchronize()
    threads = [threading.Thread(target=work, args=a) for a in zip(calls, want)]
    for t in threads:
        t.start()
    for t in threads:
        t.join()
    assert not failed
