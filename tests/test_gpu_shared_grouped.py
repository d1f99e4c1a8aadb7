"""A shared expert wider or narrower than the routed ones in the grouped launches, against the
fp64 oracle: own part of the gate/up grid, its own gate/up launch (tile widths that do not
divide each other), batches around one M tile."""
import numpy as np
import pytest

import oracle
import synth
from gpu_helpers import device_layer, full_check

pytestmark = pytest.mark.gpu


@pytest.mark.parametrize("dtype", ["bf16", "f32"])
@pytest.mark.parametrize("T,d,N,k,m,ms", [
    (65, 256, 4, 2, 64, 256), (65, 128, 200, 1, 128, 64), (130, 384, 6, 3, 256, 128), (256, 128, 3, 3, 128, 640),
    (257, 256, 16, 2, 64, 64), (257, 512, 5, 2, 192, 128), (300, 128, 9, 4, 128, 192)])
def test_shared_grouped(T, d, N, k, m, ms, dtype):
    L = synth.make_layer(synth.config("prefill_4096", T=T, d=d, N=N, k=k, m=m, dtype=dtype, n_shared=1, m_shared=ms,
                                      seed=T + d + ms))
    tb = oracle.tables.build_tables(L)
    base = oracle.forward.moe_forward(L, k, tb["a_gsp"], tb["a_rcr"], tau=0.0, tokens=[])
    tau = float(np.float32(oracle.tau.tau_table([base["c"]], 1, [0.4])[0.4]))
    full_check(L, device_layer(L), tb["a_gsp"], tb["a_rcr"], tau)
