"""Launches whose workgroups hold 2^32 threads or more, the most one grid dimension takes."""
import pytest
import torch

import paper_2609_05228_amd as ace
from test_gemm_pipe import _build_and_run


def test_fp32_gemm_grids(tmp_path):
    _build_and_run(tmp_path, "grid_check")


def _normal(gen, std, *shape):
    return torch.empty(shape, device="cuda").normal_(0.0, std, generator=gen)


@pytest.mark.gpu
def test_fp32_gemm_past_one_grid_row():
    """slots * m = 2^34: the same bits as half the tokens at a time (a row's sums do not
    depend on its tile), the shared expert's part of the grid after the routed one."""
    if torch.cuda.mem_get_info()[0] < 120 << 30:
        pytest.skip("needs 120 GiB of free device memory")
    gen = torch.Generator(device="cuda").manual_seed(5)
    T, d, N, k, m, ms = 1 << 20, 128, 8, 8, 2048, 64
    x = _normal(gen, 1.0, T, d)
    w = dict(gamma=1 + _normal(gen, 0.1, d), w_router=_normal(gen, 0.1, N, d), w_gate=_normal(gen, 0.05, N, m, d),
             w_up=_normal(gen, 0.05, N, m, d), w_down=_normal(gen, 0.05, N, d, m), ws_gate=_normal(gen, 0.05, ms, d),
             ws_up=_normal(gen, 0.05, ms, d), ws_down=_normal(gen, 0.05, d, ms))
    tables = 1 + _normal(gen, 0.05, N), 1 + _normal(gen, 0.05, N)

    def run(part):
        desc = ace.make_desc(part.shape[0], d, N, k, m, torch.float32, 0.0, n_shared=1, m_shared=ms)
        ws = torch.empty(ace.workspace_size(desc), dtype=torch.uint8, device="cuda")
        o = ace.moe_forward(part, w, *tables, k=k, tau=0.0, ws=ws)
        torch.cuda.synchronize()
        return o

    whole = run(x)
    for i in range(2):
        rows = slice(i * T // 2, (i + 1) * T // 2)
        half = run(x[rows])
        for key in ("y", "topk_idx", "keep", "gates"):
            assert torch.equal(whole[key][rows], half[key]), key


@pytest.mark.gpu
def test_tables_past_one_grid_row():
    """512 experts of 16384: 2^24 and some tile pairs in all, of 256 threads each.  Against
    the definition in fp64 (summation order: 1e-12 relative, as for the small shapes)."""
    if torch.cuda.mem_get_info()[0] < 24 << 30:
        pytest.skip("needs 24 GiB of free device memory")
    gen = torch.Generator(device="cuda").manual_seed(6)
    d, N, m, eps = 32, 512, 16384, 1e-6
    w = {n: _normal(gen, s, *shape).bfloat16() for n, s, shape in (
        ("gamma", 1.0, (d,)), ("w_router", 0.1, (N, d)), ("w_gate", 0.05, (N, m, d)), ("w_up", 0.05, (N, m, d)),
        ("w_down", 0.05, (N, d, m)))}
    got = ace.build_tables(w, want_f64=True)
    torch.cuda.synchronize()
    gam, wr = w["gamma"].double(), w["w_router"].double()
    wr = wr - wr.mean(dim=0)
    q = wr / (wr.square().mean(dim=1, keepdim=True).sqrt() + eps)
    gsp, rcr = [], []
    for e in range(N):
        wg, wu, wd = (w[n][e].double() for n in ("w_gate", "w_up", "w_down"))
        G, U = wg * gam, wu * gam
        gsp.append((U.norm() * (wd @ G).norm() * G.norm() * (wd @ U).norm()).sqrt())
        h = wg @ q[e]
        rcr.append((wd @ (h * torch.sigmoid(h) * (wu @ q[e]))).norm() / (q[e].norm() + eps))
    for key, raw in (("a_gsp64", torch.stack(gsp)), ("a_rcr64", torch.stack(rcr))):
        torch.testing.assert_close(got[key], raw / (raw.mean() + eps), rtol=1e-12, atol=0.0)
