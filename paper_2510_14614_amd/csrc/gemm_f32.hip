// fp32 GEMMs of the fp32 mode on the gfx950 matrix cores
// (v_mfma_f32_16x16x4_f32: fp32 operands, fp32 accumulation, no narrowing
// anywhere), same problem descriptor, orientations and epilogues as the bf16
// kernels in gemm.hip.
//
// What bounds it: the fp32 MFMA rate, 256 flops per clock and CU (157 TFLOP/s
// at 2.4 GHz), a sixteenth of bf16's.  One 16x16x4 MFMA takes 32 clocks for
// two operand registers, so LDS reads and global loads fit beside it with
// room to spare and the kernel needs no deep pipeline: operands go through
// registers into a two-stage LDS ring, one barrier per K slice, with the
// next slice's global loads issued before the current slice's MFMAs.  Two or
// more workgroups share a CU, so one's barrier and epilogue run beside
// another's MFMAs.
//
// Small problems (a few output tiles, K of 64 to 256) are bound by latency
// instead: they take 32 x 32 tiles with K slices of 128, so that the whole K
// range is one or two load round trips and the output spreads over as many
// CUs as it has tiles.
//
// Measured, launches repeated on three operand sets (in brackets the average
// launch of the FMA kernel of 64 x 64 tiles this replaces, from a kernel trace
// of whole steps at the same widths; there two streams shared the chip):
//  * 64 tokens, d 64, f 256: 5.0 us (1, 0), 5.6 us (1, 1), 4.3 us (0, 0)
//    [27.4, 24.3, 14.3];
//  * 2048 tokens, d 768, f 3072: QKV 87 us (83 TFLOP/s), FFN up with GELU 104
//    (93), down projection 154 (63) [312]; data gradients 116 (83), 108 (89)
//    and 84 (86) [326]; weight gradients 111 (87), 85 (85) and 37 (65) [409];
//  * 4096 x 4096 x 4096: 117 TFLOP/s in every orientation.
// Rounding: one fp32 FMA per product as before, in another order of k; against
// fp64 on normal data the two orders' sums are equally far off (1.5e-7 at
// K = 64, 1.0e-6 at 3072, by emulation of both orders), split ones nearer
// (5.5e-7 at K = 3072 in three).  A whole step of two GPT-2-small-sized blocks
// on the GPU is 1.4e-6 from fp64, 1.7e-6 with the FMA kernel.
#include <algorithm>
#include <cstring>

#include "common.h"
#include "gemm_tiles.h"
#include "kernels.h"

namespace fal {

typedef float f32x4_t __attribute__((ext_vector_type(4)));
// four floats at any 4-byte aligned address (one 16-byte global access)
typedef float f32x4_u __attribute__((ext_vector_type(4), aligned(4)));

namespace {

// One operand's tile: R rows of the output dimension by KS of K, staged from
// global memory through registers into LDS.
//  * k-contiguous: LDS rows of KS elements at a pitch of KS + 4, so the 16
//    rows of a fragment read (16 bytes each) start on 16 different 16-byte
//    bank groups.
//  * MN-major: LDS k-rows of R elements at a pitch of R + 4, so the four k-rows
//    4g + s (g = 0..3) a fragment element reads start 16 banks apart.
template <int R, int KMAJ, int KS>
struct Tile {
  static constexpr int PITCH = KMAJ ? KS + 4 : R + 4;
  static constexpr int FLOATS = KMAJ ? R * PITCH : KS * PITCH;
  static constexpr int CPR = (KMAJ ? KS : R) / 4;  // 16-byte chunks per LDS row
  static constexpr int NL = R * KS / 4 / 256;      // chunks per thread
  static_assert(NL >= 1 && NL * 1024 == R * KS, "tile shape");
  f32x4_t v[NL];

  // Slice k0 .. k0 + KS - 1 of X: elements at k >= Kend are zero, rows or
  // columns past the operand's end repeat its last one (their products land
  // in outputs that are not stored).
  __device__ __forceinline__ void load(const float* X, int64_t ld, int r0, int Rmax, int k0, int Kend, int tid) {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = tid + 256 * i, q = idx / CPR, c = 4 * (idx % CPR);
      if (KMAJ) {
        const int k = k0 + c;
        const float* p = X + (int64_t)min(r0 + q, Rmax - 1) * ld + k;
        if (k + 4 <= Kend) {
          v[i] = *reinterpret_cast<const f32x4_u*>(p);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][e] = k + e < Kend ? p[e] : 0.f;
        }
      } else {
        const int k = k0 + q, r = r0 + c;
        const float* p = X + (int64_t)k * ld;
        if (k >= Kend) {
          v[i] = f32x4_t{0.f, 0.f, 0.f, 0.f};
        } else if (r + 4 <= Rmax) {
          v[i] = *reinterpret_cast<const f32x4_u*>(p + r);
        } else {
#pragma unroll
          for (int e = 0; e < 4; ++e) v[i][e] = p[min(r + e, Rmax - 1)];
        }
      }
    }
  }
  __device__ __forceinline__ void store(float* s, int tid) const {
#pragma unroll
    for (int i = 0; i < NL; ++i) {
      const int idx = tid + 256 * i;
      *reinterpret_cast<f32x4_t*>(s + (idx / CPR) * PITCH + 4 * (idx % CPR)) = v[i];
    }
  }
  // Operand values of one 16-row fragment for the 16 k of group kk: lane l
  // holds row l % 16, k = 16 kk + 4 (l / 16) + s in element s.  Both operands
  // use the same k order, so MFMA s of the group covers k = 4g + s.
  static __device__ __forceinline__ f32x4_t frag(const float* s, int row0, int kk, int lane) {
    const int row = row0 + (lane & 15), g = lane >> 4;
    if (KMAJ) return *reinterpret_cast<const f32x4_t*>(s + row * PITCH + 16 * kk + 4 * g);
    f32x4_t f;
#pragma unroll
    for (int e = 0; e < 4; ++e) f[e] = s[(16 * kk + 4 * g + e) * PITCH + row];
    return f;
  }
};

// Four consecutive columns n .. n + 3 of output row m (m < M; columns past N
// are dropped): bias, epilogue and store.
__device__ __forceinline__ void put4(const GemmProblem& P, int m, int n, f32x4_t v, int gelu_tanh) {
  const float* bias = static_cast<const float*>(P.bias);
  const float* bias2 = static_cast<const float*>(P.bias2);
  float* out = static_cast<float*>(P.out) + (int64_t)m * P.ldo + n;
  const float* in = P.epi == EPI_RESID     ? P.resid + (int64_t)m * P.ldr + n
                    : P.epi == EPI_MUL_AUX ? static_cast<const float*>(P.aux) + (int64_t)m * P.ldaux + n
                                           : nullptr;
  float* out2 = P.epi == EPI_GELU && P.out2 ? static_cast<float*>(P.out2) + (int64_t)m * P.ldo2 + n : nullptr;
  if (n + 4 <= P.N) {
    if (bias) v += *reinterpret_cast<const f32x4_u*>(bias + n);
    if (bias2) v += *reinterpret_cast<const f32x4_u*>(bias2 + n);
    if (P.epi == EPI_GELU) {
      f32x4_t dg;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        float gv, d;
        gelu_and_grad(v[e], gelu_tanh, gv, d);
        v[e] = gv;
        dg[e] = d;
      }
      if (out2) *reinterpret_cast<f32x4_u*>(out2) = dg;
    } else if (P.epi == EPI_RESID) {
      v = *reinterpret_cast<const f32x4_u*>(in) + v;
    } else if (P.epi == EPI_MUL_AUX) {
      v *= *reinterpret_cast<const f32x4_u*>(in);
    }
    *reinterpret_cast<f32x4_u*>(out) = v;
    return;
  }
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (n + e >= P.N) break;
    float x = v[e];
    if (bias) x += bias[n + e];
    if (bias2) x += bias2[n + e];
    if (P.epi == EPI_GELU) {
      float gv, d;
      gelu_and_grad(x, gelu_tanh, gv, d);
      if (out2) out2[e] = d;
      x = gv;
    } else if (P.epi == EPI_RESID) {
      x = in[e] + x;
    } else if (P.epi == EPI_MUL_AUX) {
      x *= in[e];
    }
    out[e] = x;
  }
}

}  // namespace

// Four wavefronts own a BM x BN tile as 2 x 2 wavefront tiles.  The MFMA runs
// as B^T A^T, so lane 16g + c of a 16 x 16 block holds row c, columns 4g .. 4g+3
// and stores them as one 16-byte access.
template <int AK, int BKM, int BM, int BN, int KS>
__global__ __launch_bounds__(256, 2) void gemm_f32_mfma(GemmGroup g, int gelu_tanh) {
  typedef Tile<BM, AK, KS> TA;
  typedef Tile<BN, BKM, KS> TB;
  constexpr int FM = BM / 32, FN = BN / 32;
  __shared__ __attribute__((aligned(16))) float sA[2][TA::FLOATS];
  __shared__ __attribute__((aligned(16))) float sB[2][TB::FLOATS];
  const int bid = xcd_remap(blockIdx.x, g.total_tiles);
  const GemmProblem P = find_problem(g, bid);
  const int per_split = P.tiles_m * P.tiles_n;
  const int local = (bid - P.tile_start) % per_split, split = (bid - P.tile_start) / per_split;
  int tmi, tni;
  grouped_tile(local, P.tiles_m, P.tiles_n, tmi, tni);
  const int m0 = tmi * BM, n0 = tni * BN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int rowA = (wave >> 1) * (BM / 2), rowB = (wave & 1) * (BN / 2);

  // slices of KS: segment 0 is [0, nt1), segment 1 is [nt1, nt)
  const int nt1 = (P.K + KS - 1) / KS;
  int sbeg = 0, send = nt1 + (P.K2 + KS - 1) / KS;
  if (P.splits > 1) {
    const int per = (nt1 + P.splits - 1) / P.splits;
    sbeg = min(nt1, split * per);
    send = min(nt1, sbeg + per);
  }
  TA ta;
  TB tb;
  auto load = [&](int s) {
    const int seg = s >= nt1;
    const int k0 = (seg ? s - nt1 : s) * KS, Kend = seg ? P.K2 : P.K;
    ta.load(static_cast<const float*>(seg ? P.A2 : P.A), seg ? P.lda2 : P.lda, m0, P.M, k0, Kend, tid);
    tb.load(static_cast<const float*>(seg ? P.B2 : P.B), seg ? P.ldb2 : P.ldb, n0, P.N, k0, Kend, tid);
  };
  // 16-wide groups of slice s to multiply: all of a 32-wide slice (zeros past
  // K), and of a wide one only those that hold any k
  auto groups = [&](int s) {
    if (KS <= 32) return KS / 16;
    const int left = s >= nt1 ? P.K2 - (s - nt1) * KS : P.K - s * KS;
    return min(KS / 16, (left + 15) / 16);
  };

  f32x4_t acc[FM][FN];
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  if (sbeg < send) {
    load(sbeg);
    ta.store(sA[0], tid);
    tb.store(sB[0], tid);
    __syncthreads();
  }
  for (int s = sbeg; s < send; ++s) {
    const int cur = (s - sbeg) & 1;
    if (s + 1 < send) load(s + 1);
    const int ng = groups(s);
#pragma unroll
    for (int kk = 0; kk < KS / 16; ++kk) {
      if (kk >= ng) break;
      f32x4_t a[FM], b[FN];
#pragma unroll
      for (int i = 0; i < FM; ++i) a[i] = TA::frag(sA[cur], rowA + 16 * i, kk, lane);
#pragma unroll
      for (int j = 0; j < FN; ++j) b[j] = TB::frag(sB[cur], rowB + 16 * j, kk, lane);
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int i = 0; i < FM; ++i)
#pragma unroll
          for (int j = 0; j < FN; ++j) acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(b[j][e], a[i][e], acc[i][j], 0, 0, 0);
    }
    if (s + 1 < send) {
      // the other stage was last read in step s - 1, before that step's barrier
      ta.store(sA[cur ^ 1], tid);
      tb.store(sB[cur ^ 1], tid);
      __syncthreads();
    }
  }
  const int m1 = m0 + rowA + (lane & 15), n1 = n0 + rowB + 4 * (lane >> 4);
  if (P.splits > 1) {
    GemmProblem Q = P;
    Q.out = P.part + (int64_t)split * P.M * P.N;
    Q.ldo = P.N;
    Q.epi = EPI_STORE;
#pragma unroll
    for (int i = 0; i < FM; ++i)
#pragma unroll
      for (int j = 0; j < FN; ++j)
        if (m1 + 16 * i < P.M && n1 + 16 * j < P.N) put4(Q, m1 + 16 * i, n1 + 16 * j, acc[i][j], gelu_tanh);
    return;
  }
#pragma unroll
  for (int i = 0; i < FM; ++i)
#pragma unroll
    for (int j = 0; j < FN; ++j)
      if (m1 + 16 * i < P.M && n1 + 16 * j < P.N) put4(P, m1 + 16 * i, n1 + 16 * j, acc[i][j], gelu_tanh);
}

namespace {

// Launch time model, as the bf16 launcher's: a K slice of one tile costs t1 us
// when its CU holds that workgroup alone and t2 us when the CU holds all
// per_cu it has LDS for (in between, in proportion), each round of tiles adds
// ovh us (first loads, epilogue) and the launch kLaunchUs; a K split adds the
// reduce launch and its partials, written and read back.
//
// Fitted to the launch times of 325 problems on MI355X (each tile shape, splits
// up to 16 where the scratch holds them; 16 to 8192 tokens, widths 32 to 8192
// and a 50257-wide head, the three orientations of a step): the chosen launch
// is 1% slower on average than the fastest of its problem and 25% at worst
// (with assumed shares of the MFMA rate and rounds of 256 tiles it was 8% and
// 100%), and the estimate is off by 6% in the median, 17% for nine in ten.
// What decides between the shapes is how the tiles fill the CUs: per flop a
// full CU takes t2 / per_cu, 1.38, 1.49 and 2.39 times the MFMA's time, but
// 2048 x 768 x 768 has 96 tiles of 128 x 128 (73 us), 384 of 64 x 64 (43 us)
// and 1536 of 32 x 32 (46 us).  128 x 64 was the fastest by 3% at most and the
// fitted rule never took it, so the kernel has no such shape.
struct Shape { int bm, bn, ks, per_cu; double t1, t2, ovh; };
enum { S128 = 0, S64 = 1, S32 = 2, kShapes = 3 };
constexpr Shape kShape[kShapes] = {{128, 128, 32, 2, 2.8, 4.7, 3.3},
                                   {64, 64, 32, 4, 1.07, 2.55, 1.25},
                                   {32, 32, 128, 2, 1.6, 2.04, 0.9}};
constexpr int kCUs = 256, kMaxSplits = 16;
// shortest K a split may get, two slices of 32 (measured over 154 problems: with
// 256 the choice is 2.6% off the fastest on average, with 128 1.6%, with 64 1.1%)
constexpr int kMinSplitK = 64;
constexpr double kLaunchUs = 3.2, kReduceUs = 1.8, kPartialBytesPerUs = 6.8e6;

int slices(const Shape& t, int K) { return (K + t.ks - 1) / t.ks; }

double estimate(const GemmGroup& g, int c, int sp) {
  const Shape& t = kShape[c];
  int64_t tiles = 0;
  int ns = 0;  // longest tile's slices, whole ones as the kernel hands them out
  for (int i = 0; i < g.n; ++i) {
    const GemmProblem& P = g.p[i];
    tiles += (int64_t)((P.M + t.bm - 1) / t.bm) * ((P.N + t.bn - 1) / t.bn) * sp;
    ns = std::max(ns, (slices(t, P.K) + sp - 1) / sp + slices(t, P.K2));
  }
  const int64_t slots = (int64_t)t.per_cu * kCUs, rem = tiles % slots;
  double us = kLaunchUs + (double)(tiles / slots) * (t.ovh + ns * t.t2);
  if (rem > 0) {
    const int q = (int)((rem + kCUs - 1) / kCUs);  // workgroups per CU in the last round
    us += t.ovh + ns * (t.t1 + (t.t2 - t.t1) * (q - 1) / (t.per_cu - 1));
  }
  if (sp > 1) us += kReduceUs + (2.0 * sp + 1.0) * 4.0 * g.p[0].M * g.p[0].N / kPartialBytesPerUs;
  return us;
}

// (a step has no product with a strided A and a k-contiguous B; gemm() refuses it)
template <int BM, int BN, int KS>
void launch(int a_kmaj, int b_kmaj, const GemmGroup& g, int gelu_tanh, hipStream_t s) {
  const dim3 grid(g.total_tiles), block(256);
  if (a_kmaj && b_kmaj) hipLaunchKernelGGL((gemm_f32_mfma<1, 1, BM, BN, KS>), grid, block, 0, s, g, gelu_tanh);
  else if (a_kmaj) hipLaunchKernelGGL((gemm_f32_mfma<1, 0, BM, BN, KS>), grid, block, 0, s, g, gelu_tanh);
  else hipLaunchKernelGGL((gemm_f32_mfma<0, 0, BM, BN, KS>), grid, block, 0, s, g, gelu_tanh);
}

// The shape (and, for a single plain product, the K split) with the smallest
// estimated time.  A split takes ceil(slices / splits) whole slices, and the
// estimate counts them so: a count that leaves the last splits none (35 slices
// in 16 splits of 3, which 12 cover) never beats the smaller one that does not.
double choose(const GemmGroup& g, bool splittable, int64_t splitk_floats, int& shape, int& splits) {
  const GemmProblem& P0 = g.p[0];
  double best = 0.0;
  shape = -1;
  splits = 1;
  for (int c = 0; c < kShapes; ++c)
    for (int sp = 1; sp <= (splittable ? kMaxSplits : 1); ++sp) {
      if (sp > 1 && (P0.K / sp < kMinSplitK || (int64_t)sp * P0.M * P0.N > splitk_floats)) break;
      const double us = estimate(g, c, sp);
      if (shape < 0 || us < best) { best = us; shape = c; splits = sp; }
    }
  return best;
}

}  // namespace

hipError_t gemm_f32(int a_kmaj, int b_kmaj, GemmGroup& g, int gelu_tanh, hipStream_t s, float* splitk_scratch,
                    int64_t splitk_floats) {
  const GemmProblem& P0 = g.p[0];
  const bool splittable = splitk_scratch && g.n == 1 && P0.K2 == 0 && P0.epi == EPI_STORE && !P0.bias && !P0.bias2;
  int shape, splits;
  choose(g, splittable, splitk_floats, shape, splits);
  const Shape& t = kShape[shape];
  int total = 0;
  for (int i = 0; i < g.n; ++i) {
    GemmProblem& P = g.p[i];
    P.tiles_m = (P.M + t.bm - 1) / t.bm;
    P.tiles_n = (P.N + t.bn - 1) / t.bn;
    P.tile_start = total;
    total += P.tiles_m * P.tiles_n;
  }
  if (splits > 1) {
    g.p[0].splits = splits;
    g.p[0].part = splitk_scratch;
    total *= splits;
  }
  g.total_tiles = total;
  switch (shape) {
    case S128: launch<128, 128, 32>(a_kmaj, b_kmaj, g, gelu_tanh, s); break;
    case S64: launch<64, 64, 32>(a_kmaj, b_kmaj, g, gelu_tanh, s); break;
    default: launch<32, 32, 128>(a_kmaj, b_kmaj, g, gelu_tanh, s); break;
  }
  const hipError_t e = hipGetLastError();
  return e != hipSuccess || splits == 1 ? e : splitk_sum(g.p[0], s);
}

// The launcher's choice for one problem, for host tests (not part of the C
// ABI): out = {tile rows, tile columns, K slice, splits}; returns the
// estimated us.
extern "C" double fal_gemm_f32_choice(int32_t M, int32_t N, int32_t K, int32_t K2, int32_t splittable,
                                      int64_t splitk_floats, int32_t* out) {
  GemmGroup g;
  memset(&g, 0, sizeof(g));
  g.n = 1;
  g.p[0].M = M;
  g.p[0].N = N;
  g.p[0].K = K;
  g.p[0].K2 = K2;
  int shape, splits;
  const double us = choose(g, splittable && K2 == 0, splitk_floats, shape, splits);
  out[0] = kShape[shape].bm;
  out[1] = kShape[shape].bn;
  out[2] = kShape[shape].ks;
  out[3] = splits;
  return us;
}

}  // namespace fal
