"""Hand-overs through LDS between the lanes of one wave, in the compiled kernels.

The lanes of a wave run in step, so no barrier instruction is needed, but nothing in one
lane's own addresses tells the compiler that its read depends on another lane's write.
wave_fence() (device_common.hpp) does, and leaves a comment in the assembly; each
hand-over has to show it between the LDS accesses that it orders.
"""
import os
import subprocess

import pytest

from paper_2406_12580_amd import build as hipbuild


def _assembly(tmp_path, source):
    out = os.path.join(tmp_path, "k.s")
    cmd = [hipbuild.HIPCC, "-x", "hip", *hipbuild.FLAGS, "--cuda-device-only", "-S", source,
           "-o", out]
    res = subprocess.run(cmd, capture_output=True, text=True, timeout=300)
    assert res.returncode == 0, res.stderr
    with open(out) as f:
        return f.read().splitlines()


def _lds_runs(lines, kernel):
    """The kernel's LDS accesses (R, W), fences (F) and barriers (B) in listing order, runs
    of one kind as one letter."""
    first = next(i for i, l in enumerate(lines) if l.startswith("_Z") and kernel in l)
    ops = ""
    for l in lines[first:]:
        l = l.strip()
        if l.startswith(".Lfunc_end"):
            break
        op = ("R" if l.startswith("ds_read") else "W" if l.startswith("ds_write") else
              "B" if l.startswith("s_barrier") else "F" if l.startswith("; wave_fence") else "")
        if op and not ops.endswith(op):
            ops += op
    return ops


# The gated layer's one-kernel backward: the staged hx of the steps before a lane's own
# (twice: before the loop and in it), and those steps in the conv's backward (whole tile,
# last tile) before the next tile's are written over them.
def test_gated_backward_conv_window(tmp_path):
    source = os.path.join(hipbuild.CSRC, "fused_bwd.hip")
    ops = _lds_runs(_assembly(tmp_path, source), "fused_bwd_kernelIfffLb1E")
    print(ops)
    assert ops.startswith("WFR"), ops
    assert ops.count("WFR") == 2 and ops.count("RF") == 2, ops


# The D = 64 sub-layers' backward: a wave's block of gradients transposed through its own
# LDS (written by unit, read by row).
@pytest.mark.parametrize("kernel", ["ffn_bwd_kernel", "proj_in_bwd_kernel"])
def test_sublayer_transposed_block(tmp_path, kernel):
    source = os.path.join(hipbuild.CSRC, "ffn.hip")
    ops = _lds_runs(_assembly(tmp_path, source), kernel)
    print(ops)
    loop = ops[ops.index("B"):]  # after the first rows are staged
    assert loop.count("F") == 1, ops
    before, after = loop.split("F")
    assert "W" in before and before.count("B") == 1, ops  # the block, then the fence
    assert after.startswith("RB"), ops


# The tile product of the fused scans: each gate's strip written by accumulator rows and
# read by channel, the second gate's over the first one's.
def test_tile_product_strip(tmp_path):
    source = os.path.join(tmp_path, "probe.hip")
    with open(source, "w") as f:
        f.write("""#include "fused_z.hpp"
using namespace recblr;
__global__ __launch_bounds__(fusedz::NT) void probe_kernel(
    const float* x, const __bf16* pack, const float* br, const float* bi, int64_t L, int64_t D,
    float* out) {
    __shared__ __attribute__((aligned(16))) char smem[fusedz::Tile<float>::kSmem];
    const int tid = threadIdx.x, w = wave_id(), lane = tid & 63;
    float zr[fusedz::C], zi[fusedz::C];
    fusedz::tile_z<float>(x, pack, br, bi, L, D, 0, blockIdx.x, 0, smem, tid, w, lane, zr, zi);
    for (int c = 0; c < fusedz::C; ++c) out[(blockIdx.x * fusedz::NT + tid) * 32 + c] = zr[c];
    for (int c = 0; c < fusedz::C; ++c) out[(blockIdx.x * fusedz::NT + tid) * 32 + 16 + c] = zi[c];
}
""")
    ops = _lds_runs(_assembly(tmp_path, source), "probe_kernel")
    print(ops)
    assert ops.endswith("WFRFWFR"), ops
