"""Table builder at the edges of its kernels' ranges: the smallest hidden and
intermediate sizes (one 32-wide K block, one 64-row tile, lanes with no vector of a
row), expert counts that do not fill the 8 XCDs, odd tile counts, both dtypes.  The
oracle's fp64 tables agree within summation order, about 1e-15 of sums of up to
d m terms: 1e-12 relative."""
import numpy as np
import pytest
import torch

import oracle
import paper_2609_05228_amd as ace
import synth
from gpu_helpers import device_layer

pytestmark = pytest.mark.gpu

SHAPES = [(32, 1, 64), (96, 9, 64), (160, 3, 192), (2080, 2, 128), (64, 17, 832)]


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("d,N,m", SHAPES, ids=[f"d{d}_N{n}_m{m}" for d, n, m in SHAPES])
def test_tables_edges(d, N, m, dtype):
    L = synth.make_layer(synth.config("tiny_f32", T=1, d=d, N=N, k=1, m=m, dtype=dtype, seed=d + N))
    want = oracle.tables.build_tables(L)
    got = ace.build_tables(device_layer(L), want_f64=True)
    torch.cuda.synchronize()
    for key in ("a_gsp", "a_rcr"):
        w = want[key + "64"]
        if N == 1 and key == "a_rcr":
            assert w[0] == 0.0  # one expert: its centred router row, and so the table, is 0
        np.testing.assert_allclose(got[key + "64"].cpu().numpy(), w, rtol=1e-12)
        np.testing.assert_allclose(got[key].cpu().numpy(), w.astype(np.float32), rtol=1.2e-7)
