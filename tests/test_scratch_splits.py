"""Layers that fit the static scratch without the partial sums of the down GEMMs' K splits
keep fitting it (the splits are left out there), and fp32 layers past the small batches need
no more of it than with M tiles of 256 rows (their lists of 64-row tiles are longer)."""
import pytest
import torch

import paper_2609_05228_amd as ace
from paper_2609_05228_amd import _lib
from paper_2609_05228_amd.layer import _marshal


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


@pytest.mark.parametrize("T,d,N,k,m,ms,size", [  # bytes with 256-row tiles, within 10 KB of the limit
    (51797, 128, 8, 1, 64, 0, 67108864), (6317, 128, 111, 7, 192, 128, 67104256),
    (31693, 128, 138, 2, 64, 0, 67107840), (8075, 128, 251, 3, 512, 0, 67108352),
    (3257, 512, 59, 8, 64, 0, 67107328), (4050, 256, 253, 8, 64, 1024, 67107328)])
def test_f32_tile_lists_keep_the_scratch_limit(T, d, N, k, m, ms, size):
    assert _size(T, d, N, k, m, _lib.ACE_F32, ms) <= size <= _lib.NOALLOC_SCRATCH_BYTES


@pytest.mark.gpu
@pytest.mark.parametrize("T,d,N,k,m", [(51797, 128, 8, 1, 64), (8075, 128, 251, 3, 512)])
def test_f32_at_the_scratch_limit(T, d, N, k, m):
    """The plan in one kernel and in two (251 experts), whose chunk bases lie in H: the same
    bits as half the tokens at a time (a row's sums do not depend on its tile)."""
    gen = torch.Generator(device="cuda").manual_seed(T)

    def normal(std, *shape):
        return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen)

    x = normal(1.0, T, d)
    w = dict(gamma=1 + normal(0.1, d), w_router=normal(0.1, N, d), w_gate=normal(0.05, N, m, d),
             w_up=normal(0.05, N, m, d), w_down=normal(0.05, N, d, m))
    tables = 1 + normal(0.05, N), 1 + normal(0.05, N)
    desc, W, O, o, _ = _marshal(x, w, *tables, k, 0.2, 1, 1e-6, 1e-6, False, False, True, None,
                                torch.empty(256, dtype=torch.uint8, device="cuda"), "max")
    assert _lib.workspace_size(desc) <= _lib.NOALLOC_SCRATCH_BYTES
    assert _lib.forward_noalloc_raw(desc, x.data_ptr(), W, O, torch.cuda.current_stream().cuda_stream) == _lib.ACE_OK
    h = T // 2
    halves = [ace.moe_forward(part, w, *tables, k=k, tau=0.2) for part in (x[:h].contiguous(), x[h:].contiguous())]
    torch.cuda.synchronize()
    for key in ("y", "topk_idx", "keep", "gates"):
        assert torch.equal(o[key], torch.cat([half[key] for half in halves])), key
