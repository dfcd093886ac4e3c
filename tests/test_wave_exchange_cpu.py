"""Exchange of point samples through LDS within a wavefront, checked on the
compiled code (no GPU needed).

A probe kernel in which only some lanes store a sample is compiled for gfx950
down to LLVM IR.  Every lane has to read its cell after the samples are stored:
the value written out must not come from a merge with a constant zero, which is
what the compiler makes of the lanes that store nothing when the accesses are
not ordered across lanes (the test shows that on the same code without it).
"""
import os
import re
import shutil
import subprocess

import pytest

from test_index_logic_cpu import CSRC

HIPCC = os.environ.get("HIPCC", "/opt/rocm/bin/hipcc")

PROBE = r"""
#include "%s/internal.h"
#ifdef UNORDERED
namespace fw {
template <int W, int ROWS, class Put>
__device__ __forceinline__ void unordered(float (*cols)[ROWS], int lane, float (&src)[W], Put put) {
  for (int j = 0; j < W; ++j) cols[j][lane] = 0.f;
  put();
  for (int j = 0; j < W; ++j) src[j] += cols[j][lane];
}
}
#define add_through_lds unordered
#endif
extern "C" __global__ void probe(const int2 *ent, const float *val, int cnt, float *out) {
  __shared__ float tile[4][2][72];
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  float src[2] = {0.f, 0.f};
  int2 en = {0, 0};
  float v = 0.f;
  if (lane < cnt) {
    en = ent[lane];
    v = val[lane];
  }
  float(*own)[72] = tile[w];
  fw::add_through_lds(own, lane, src, [&]() {
    if (lane < cnt) own[en.x >> 6][en.x & 63] = v;
  });
  out[threadIdx.x] = src[0] + 2.f * src[1];
}
"""


def _result_is_merged_with_zero(tmp_path, *flags):
    (tmp_path / "probe.hip").write_text(PROBE % CSRC)
    ir = subprocess.run([HIPCC, "--offload-arch=gfx950", "-O3", "-std=c++17", "-S", "-emit-llvm", "--offload-device-only",
                         *flags, "-o", "-", str(tmp_path / "probe.hip")], check=True, capture_output=True, text=True).stdout
    body = ir[ir.index("@probe("):]
    body = body[:body.index("\n}")]
    stored = re.search(r"store float (%\w+), ptr addrspace\(1\)", body).group(1)
    merge = re.search(re.escape(stored) + r" = phi float (.*)", body)
    return bool(merge and "0.000000e+00" in merge.group(1))


@pytest.mark.skipif(shutil.which(HIPCC) is None, reason="hipcc not available")
def test_lanes_without_a_sample_read_their_cell(tmp_path):
    assert _result_is_merged_with_zero(tmp_path, "-DUNORDERED")
    assert not _result_is_merged_with_zero(tmp_path)
