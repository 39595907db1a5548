"""The zeroing of a wave's row in LDS (clear_row) is ordered before later
writes of the same words by other lanes: seen in the code compiled for gfx950,
where a wave barrier stands between the two, since in-order LDS hardware hides
its absence from every run."""
import re
import subprocess

from paper_2008_11326_amd import build

KERNEL = """
#include "gpp_device.h"
__global__ void rows(double *out, const double *in)
{
    __shared__ double row[32];
    const int lane = threadIdx.x;
    gpp::clear_row<32>(row, lane);
    if (lane % 16 == 0) row[lane / 16] = in[lane];  // lane 16 writes a word of lane 1
    __syncthreads();
    if (lane < 32) out[lane] = row[lane];
}
"""


def test_clear_row_is_ordered_before_other_lanes_writes(tmp_path):
    src, asm = tmp_path / "rows.hip", tmp_path / "rows.s"
    src.write_text(KERNEL)
    subprocess.run([build.HIPCC, *build.FLAGS, "--cuda-device-only", "-S", str(src), "-o", str(asm)],
                   check=True, capture_output=True)
    marks = re.findall(r"ds_write|wave barrier|s_barrier", asm.read_text())
    assert marks[:3] == ["ds_write", "wave barrier", "ds_write"], marks
