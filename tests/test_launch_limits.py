"""What the library asks the runtime to launch, recorded by a hipLaunchKernel of the test's own, on the CPU:
the work-items of a launch fit 32 bits, and the pieces of a gather pass cover every workgroup once."""
import host_check

SOURCE = r"""
#include <cstdio>
#include <cstring>
#include "relax_device.h"
using namespace relax;

static dim3 grid_, block_;
static unsigned long long next_ = 0;
static int failure = 0;

extern "C" {
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t, hipStream_t) {
  grid_ = g;
  block_ = b;
  return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* shared, hipStream_t* st) {
  *g = grid_;
  *b = block_;
  *shared = 0;
  *st = nullptr;
  return hipSuccess;
}
hipError_t hipLaunchKernel(const void*, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
  if ((unsigned long long)g.x * b.x >= 1ull << 32) {
    failure = 1;
    return hipErrorInvalidConfiguration;
  }
  if (*static_cast<unsigned*>(args[3]) != next_) failure = 2;  // the first workgroup of the piece
  next_ += g.x;
  return hipSuccess;
}
hipError_t hipGetLastError() { return hipSuccess; }
}

int main() {
  const int sizes[][3] = {{4, 5, 1 << 23}, {4, 4, 1 << 24}, {65, 5, (1 << 22) + 3}, {4, 4, 4}, {64, 64, 192}};
  const int kinds[][2] = {{0, 2}, {0, 3}, {0, 4}, {0, 5}, {0, 6}, {1, 1}, {2, 1}};
  for (auto& n : sizes)
    for (auto& k : kinds) {
      AdjArgs a;
      std::memset(&a, 0, sizeof a);
      for (int c = 0; c < 3; c++) a.g.n[c] = n[c];
      next_ = 0;
      const hipError_t e = launch_adj_gather(a, k[0], k[1], nullptr);
      const unsigned long long all = (unsigned long long)((n[0] + 63) / 64) * ((n[1] + 3) / 4) * n[2];
      if (e != hipSuccess || failure || next_ != all) {
        std::printf("%d x %d x %d mode %d stage %d: status %d failure %d workgroups %llu of %llu\n", n[0], n[1], n[2], k[0],
                    k[1], (int)e, failure, next_, all);
        return 1;
      }
    }
  return 0;
}
"""


def test_gather_of_long_thin_grids_is_launched_in_pieces(tmp_path):
    host_check.run(SOURCE, tmp_path)
