"""The threshold mapping's digit passes at their edges, bit-exact against the oracle: row
counts around one and several rows per thread and around the one-workgroup limit, every k,
and scores that crowd into few bins of the top digit, lie outside its fine range, or tie so
that the next larger score is another bin's."""
import numpy as np
import pytest

from test_gpu_tau import _check

pytestmark = pytest.mark.gpu

QS = [0.02, 0.1, 0.25, 0.4, 0.5, 0.6, 0.7, 0.8]


def _scores(kind, rows, k, seed):
    rng = np.random.default_rng(seed)
    if kind == "shares":  # a token's k shares of one
        return rng.dirichlet(np.ones(k), size=rows)
    if kind == "ties":  # more keys in a selection's bin than the direct ranking takes
        return rng.choice([0.0, 0.003, 0.0625, 0.25, 0.2500001, 1.0], size=(rows, k))
    if kind == "coarse":  # 3 significant bits: every boundary ties, the next score bins away
        return np.exp2(np.floor(np.log2(rng.random((rows, k)) + 1e-9) * 4) / 4)
    # outside the fine range on both sides, both signs
    return rng.standard_normal((rows, k)) * 10.0 ** rng.integers(-30, 30, size=(rows, k))


@pytest.mark.parametrize("kind", ["shares", "ties", "coarse", "wide"])
@pytest.mark.parametrize("rows,k,m_min", [(1, 8, 1), (63, 3, 2), (1024, 8, 1), (1025, 5, 1), (2049, 7, 3), (4096, 8, 8),
                                          (4096, 4, 1), (4097, 8, 1), (4097, 2, 1), (300001, 6, 2)])
def test_tau_digits(kind, rows, k, m_min):
    c = _scores(kind, rows, k, rows + k).astype(np.float32)
    _check([c], m_min, QS[:3] if rows % 2 else QS, f"{kind} rows={rows} k={k} m_min={m_min}")
