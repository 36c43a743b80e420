// Shared by the GEMM kernels: which problem and which output tile of it a
// workgroup owns, and the launchers they call in one another.
#pragma once

#include "kernels.h"

namespace fal {

// The problem owning workgroup `tile`, selected with constant indices so the
// descriptor stays in scalar registers (a dynamic index into the by-value
// array would copy it to scratch).
__device__ __forceinline__ GemmProblem find_problem(const GemmGroup& g, int tile) {
  static_assert(kMaxGroup == 4, "update find_problem");
  if (g.n > 3 && tile >= g.p[3].tile_start) return g.p[3];
  if (g.n > 2 && tile >= g.p[2].tile_start) return g.p[2];
  if (g.n > 1 && tile >= g.p[1].tile_start) return g.p[1];
  return g.p[0];
}

constexpr int kXcds = 8, kGroupM = 4;
__device__ __forceinline__ int xcd_remap(int bid, int total) {
  const int q = total / kXcds, r = total % kXcds;
  const int xcd = bid % kXcds, slot = bid / kXcds;
  return xcd < r ? xcd * (q + 1) + slot : r * (q + 1) + (xcd - r) * q + slot;
}
__device__ __forceinline__ void grouped_tile(int t, int tiles_m, int tiles_n, int& tm, int& tn) {
  const int band = kGroupM * tiles_n;
  const int first = (t / band) * kGroupM;
  const int gs = min(kGroupM, tiles_m - first);
  const int in = t % band;
  tm = first + in % gs;
  tn = in / gs;
}


// fp32 operands (gemm_f32.hip); g's per-launch fields are filled in there.
hipError_t gemm_f32(int a_kmaj, int b_kmaj, GemmGroup& g, int gelu_tanh, hipStream_t s, float* splitk_scratch,
                    int64_t splitk_floats);
// out = sum over splits of part, slices in order (+ bf16 biases) (gemm.hip).
hipError_t splitk_sum(const GemmProblem& P, hipStream_t s);

}  // namespace fal
