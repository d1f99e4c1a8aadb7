"""The gate/up launch's tile order (every expert within one M tile) where the plan has
fewer workgroups than experts: each wave then places several experts.  A tile that the
order missed or named twice would leave an expert's rows unwritten, so every output row
is checked against the oracle."""
import pytest

import oracle
import synth
from gpu_helpers import device_layer, full_check

pytestmark = pytest.mark.gpu

CASES = [(65, 256, 8), (131, 128, 8), (70, 4, 2), (130, 68, 3), (1000, 256, 8)]


@pytest.mark.parametrize("T,N,k", CASES, ids=[f"T{t}_N{n}_k{k}" for t, n, k in CASES])
def test_tile_order(T, N, k):
    L = synth.make_layer(synth.config("prefill_4096", T=T, d=128, N=N, k=k, m=64, seed=90 + N))
    tb = oracle.tables.build_tables(L)
    base = oracle.forward.moe_forward(L, k, tb["a_gsp"], tb["a_rcr"], tau=0.0, tokens=[])
    tau = float(oracle.tau.tau_table([base["c"]], 1, [0.5])[0.5])
    full_check(L, device_layer(L), tb["a_gsp"], tb["a_rcr"], tau)
