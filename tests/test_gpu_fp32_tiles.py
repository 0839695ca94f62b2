"""fp32 attention at the edges of its matrix tiles: head sizes that are no multiple of 16 and the largest, 1, 16, 17 and 40 query
rows per kv head, parts of 16-token tiles, rows appended inside the launch and before it."""
import numpy as np
import pytest

import oracle
import workloads as wl

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("D", [4, 20, 32, 64, 100, 128, 132, 256])
@pytest.mark.parametrize("Hq,Hkv,kmax", [(2, 2, 1), (4, 2, 8), (17, 1, 1), (10, 2, 8)])
@pytest.mark.parametrize("fused", [False, True])
def test_head_sizes_and_rows(D, Hq, Hkv, kmax, fused):
    from paper_2404_15778_amd import harness
    ctx, nq = [0, 15, 16, 31, 70, 9], [kmax, kmax, 1, kmax, max(1, kmax - 1), 0]
    w = wl.make_attention("fp32_tiles", 6, Hq, Hkv, D, "fp32", ctx, nq, 3, kmax=kmax, Lcap=80)
    Or, lser = oracle.verify_attention(w.Q, w.K, w.V, w.ctx_len, w.draft_len, w.scale)
    O, lse, status, _ = harness.run_attention_workload(w, poison=True, fused=fused)
    assert status == 0 and np.isfinite(O).all()
    # sums of at most 256 and 79 products in 32 bits, outputs of magnitude up to about 4: 2^-24 of it for each of a few roundings in a row
    assert np.abs(O - Or).max() <= 1e-5 and np.abs(lse - lser).max() <= 1e-5
