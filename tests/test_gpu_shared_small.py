"""A shared expert in the small-batch launches, against the fp64 oracle: one and several K
splits of its down GEMM with and without splits of the routed one, row counts around the
passes of 8, 16 and 32 rows, widths above and below the routed experts'."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import device_layer, full_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,d,N,k,m,ms", [
    (1, 256, 4, 2, 64, 64), (1, 2048, 16, 4, 256, 1024), (8, 128, 3, 3, 64, 512), (9, 512, 8, 2, 128, 256),
    (16, 1024, 64, 8, 192, 192), (17, 384, 5, 1, 64, 1024), (33, 256, 2, 2, 512, 64), (64, 1024, 130, 8, 64, 768),
    (64, 128, 1, 1, 64, 320)])
def test_shared_small(T, d, N, k, m, ms, dtype):
    L = synth.make_layer(synth.config("prefill_4096", T=T, d=d, N=N, k=k, m=m, dtype=dtype, n_shared=1, m_shared=ms,
                                      seed=T + d + ms))
    tb = oracle.tables.build_tables(L)
    base = oracle.forward.moe_forward(L, k, tb["a_gsp"], tb["a_rcr"], tau=0.0, tokens=[])
    tau = float(np.float32(oracle.tau.tau_table([base["c"]], 1, [0.4])[0.4]))
    full_check(L, device_layer(L), tb["a_gsp"], tb["a_rcr"], tau)
