"""Layers that fit the static scratch without the partial sums of the down GEMMs' K splits
keep fitting it (the splits are left out there)."""
import pytest

from paper_2609_05228_amd import _lib


def _size(T, d, N, k, m, dtype, ms=0):
    return _lib.workspace_size(_lib.Desc(T, d, N, k, m, 1 if ms else 0, ms, dtype, 1, 0.1, 1e-6, 1e-6, 0))


@pytest.mark.parametrize("dtype,T,d,N,k,m,ms", [
    (_lib.ACE_F32, 64, 2048, 8, 8, 16384, 0),         # 38 MB, the routed partial sums 34 MB
    (_lib.ACE_F32, 64, 2048, 8, 8, 16384, 2048),
    (_lib.ACE_BF16, 64, 2048, 64, 1, 64 * 7900, 2048),  # 65 MB, the shared partial sums 4 MB
])
def test_splits_keep_the_scratch_limit(dtype, T, d, N, k, m, ms):
    assert _size(T, d, N, k, m, dtype, ms) <= _lib.NOALLOC_SCRATCH_BYTES


def test_splits_are_taken_below_it():
    plane = 8 * 64 * 1024 * 4
    assert _size(64, 1024, 64, 1, 64, _lib.ACE_BF16, 1024) > _size(64, 1024, 64, 1, 64, _lib.ACE_BF16, 64) + plane
