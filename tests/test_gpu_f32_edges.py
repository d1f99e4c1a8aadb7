"""fp32 layers at the edges of their tiles, against the fp64 oracle: batches around the
small-batch limit, experts with rows around one and several 64-row tiles, the shortest and
longer K, K splits of the small batches, and a shared expert of the routed width or its own."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import device_layer, full_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("T,d,N,k,m,ms", [
    (1, 128, 1, 1, 64, 0), (1, 1024, 8, 2, 512, 512), (17, 640, 5, 3, 192, 64), (64, 256, 1, 1, 1024, 0),
    (64, 1024, 2, 2, 64, 64), (65, 128, 1, 1, 64, 0), (65, 384, 6, 5, 192, 192), (128, 256, 1, 1, 128, 0),
    (129, 256, 2, 2, 64, 320), (255, 128, 3, 2, 64, 64), (321, 512, 16, 8, 128, 0)])
def test_f32_edges(T, d, N, k, m, ms):
    L = synth.make_layer(synth.config("prefill_4096", T=T, d=d, N=N, k=k, m=m, dtype="f32", n_shared=1 if ms else 0,
                                      m_shared=ms, seed=T + d + N))
    tb = oracle.tables.build_tables(L)
    base = oracle.forward.moe_forward(L, k, tb["a_gsp"], tb["a_rcr"], tau=0.0, tokens=[])
    tau = float(np.float32(oracle.tau.tau_table([base["c"]], 1, [0.4])[0.4]))
    full_check(L, device_layer(L), tb["a_gsp"], tb["a_rcr"], tau)
