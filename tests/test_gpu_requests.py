"""GPU tests of how requests share 64-source batches on the host loop: the
remainders that just fit, just miss, or fill a batch, in both orders of
arrival, against each request alone (bit for bit) and the oracle."""
import numpy as np
import pytest

import graphgen as gg
import paper_2401_02472_amd as bcm
from tests.gpu_checks import check_bc, oracle_bc

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("sizes", [
    [1, 63, 64, 65], [32, 33, 31, 32, 1, 0, 63], [130, 62, 2, 1, 65], [1] * 66,
    [64, 128, 7], [40, 40, 24, 24, 1],
], ids=str)
def test_shared_batches(sizes):
    import torch
    g = gg.rmat(15, 8, seed=4)  # above the sizes that run a workgroup per source
    reqs = [gg.sample_sources(g, k, seed=70 + i) if k else np.zeros(0, np.int32)
            for i, k in enumerate(sizes)]
    with bcm.Graph(g.n, g.row_ptr, g.col_idx) as G:
        def run(which):
            outs = [torch.full((g.n,), 3.0, dtype=torch.float64, device="cuda") for _ in which]
            G.run_multi([reqs[i] for i in which], outs)
            torch.cuda.synchronize()
            return [o.cpu().numpy() for o in outs]
        mixed, reverse = run(range(len(reqs))), run(range(len(reqs))[::-1])[::-1]
        for i in range(len(reqs)) if len(reqs) < 20 else (0, 1, 63, 64, 65):
            assert np.array_equal(mixed[i], run([i])[0]), f"request {i} differs in the mix"
            assert np.array_equal(mixed[i], reverse[i])
            check_bc(mixed[i], oracle_bc(g, reqs[i]) if sizes[i] else np.zeros(g.n))
