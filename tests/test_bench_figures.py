"""What bench.py says about a run, against what the library does (no GPU)."""
import sys

import pytest

import paper_2501_00692_amd as ssm
from paper_2501_00692_amd.synth import WORKLOADS

sys.path.insert(0, str(ssm.LIB_PATH.parent.parent))
import bench  # noqa: E402


@pytest.mark.parametrize("name,chunk", [("small", 32), ("layer", 128), ("long", 128), ("slice", 128), ("vlong", 128)])
def test_chunk_in_use(name, chunk):
    """Chunk 0 is reported as the chunk that the library takes at these sizes."""
    assert bench.chunk_in_use(ssm, WORKLOADS[name]) == chunk
    assert bench.chunk_in_use(ssm, WORKLOADS[name], 256) == 256


def test_input_projection_fix_is_one_launch():
    """The reassociated input-projection gradient multiplies both bf16 parts of its
    2 x d_model rows in one launch; with d_model >= D there is none."""
    M, D, N, dm = 262144, 4096, 16, 2048
    f = bench.layer_gemm_flops(M, D, N, dm)
    assert f["gemm_dwin_fix"] == 2 * (2 * dm) * D * (D + 2 * N)
    assert f["gemm_dw"] == 2 * M * (D * (D + 2 * N) + dm * (3 * D + 2 * N))
    assert "gemm_dwin_fix" not in bench.layer_gemm_flops(M, D, N, D)
