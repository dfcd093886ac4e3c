"""Source samples read by the multi-job stencil, checked on the CPU.

k_step2_multi is compiled with g++ from the kernel source, with a body that
records what step2_body would fetch: the samples of both steps, ahead of its
early exits.  Over every launch of jobs with even and odd records, started at
even steps as in a batch and in the engine, no sample index leaves the record.
"""
import os

from test_index_logic_cpu import CSRC, _function, _run_cpp

STUB = r"""
#include <algorithm>
#include <cstdio>
#include <vector>
using std::max;
using std::min;
#define __global__
#define __shared__ static
#define __launch_bounds__(...)
struct { int x; } blockIdx;
struct Inject { int t = -1; };
struct StepArgs { const float *prev = nullptr, *cur = nullptr; float *out = nullptr; Inject inj, ext; };
struct Step2Args { StepArgs a; float *out2 = nullptr; Inject inj2; int two = 1; };
struct BatchJob2 { Step2Args p; float *buf[4] = {}; int tile_begin = 0, t0 = 0, nt = 0; };
template <int TX> struct Step2Tile {};
int lowest, highest, launches;
template <int TX, int MODE, bool EARLY2>
void step2_body(const Step2Args &p, int, Step2Tile<TX> &, bool, bool) {
  lowest = min(lowest, min(p.a.inj.t, p.inj2.t));
  highest = max(highest, max(p.a.inj.t, p.inj2.t));
  ++launches;
}
"""

MAIN = r"""
int main() {
  for (int nt = 2; nt <= 41; ++nt)
    for (int t0 = 0; t0 <= 6; t0 += 2) {
      BatchJob2 job;
      job.nt = nt;
      job.t0 = t0;
      lowest = 1 << 30;
      highest = launches = 0;
      for (int step = 0; step < t0 + nt + 8; step += 2) k_step2_multi<32, 0>(&job, nullptr, 1, 1, nullptr, step);
      std::printf("%d %d %d %d\n", nt, lowest, highest, launches);
    }
  return 0;
}
"""


def test_multi_job_launches_read_samples_of_the_record_only(tmp_path):
    src = open(os.path.join(CSRC, "kernels_step2.hip")).read()
    kernel = _function(src, "__global__ void __launch_bounds__(256, step2_multi_blocks<TX>()) k_step2_multi(")
    out = _run_cpp(tmp_path, STUB + "template <int TX, int MODE>\n" + kernel + MAIN)
    rows = [tuple(map(int, line.split())) for line in out.splitlines()]
    assert len(rows) == 160
    for nt, lowest, highest, launches in rows:
        assert launches == (nt + 1) // 2 and lowest == 0 and highest == nt - 1, (nt, lowest, highest, launches)
