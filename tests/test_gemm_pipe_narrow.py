"""Wait counts of the fp32 expert GEMMs' narrow tiles, replayed on the host."""
from test_gemm_pipe import _build_and_run


def test_narrow_tile_wait_counts(tmp_path):
    _build_and_run(tmp_path, "pipe_check_narrow")
