// Log-sum-exp combine of the per-block attention results (the combine step of
// Algorithm 1; Sec. 2.3).  The current-block kernel has already written each
// row's normalised current-block result to out and its lse to lse; this kernel
// folds the row's history partials (of out's dtype) into them in place:
//   lse = M + ln(sum_i e^{lse_i - M}),  out = sum_i e^{lse_i - lse} O_i,
// accumulated in fp32 in a fixed order (current block first, then history
// slots ascending) and rounded once to the output dtype.
//
// One 16-byte load per lane and partial (bf16: 16 lanes per row, 8 dims each;
// fp32: 32 lanes, 4 dims); each of the row's first lanes loads one slot's lse
// and the row's lanes share them.  Partials
// are read in groups of kGroup, all loads of a group in flight at once, with
// an online rescale between groups (one group covers top-k up to 13).
#include "moba_internal.h"

#include <math.h>

namespace moba {
namespace {

constexpr int kGroup = 12;
constexpr float kLn2 = 0.69314718055994531f;
constexpr float kLog2e = 1.4426950408889634f;

__device__ __forceinline__ void unpack(uint4 u, float (&f)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; i++) {
    f[2 * i] = __uint_as_float(w[i] << 16);
    f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

__device__ __forceinline__ void unpack(uint4 u, float (&f)[4]) {
  f[0] = __uint_as_float(u.x); f[1] = __uint_as_float(u.y);
  f[2] = __uint_as_float(u.z); f[3] = __uint_as_float(u.w);
}

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x2 __attribute__((ext_vector_type(2)));

// Two fp32 values to a packed bf16 pair, round-to-nearest-even.
__device__ __forceinline__ uint32_t pack2(float a, float b) {
  const f32x2 v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2));
}

__device__ __forceinline__ uint4 pack(const float (&f)[8], float inv) {
  return make_uint4(pack2(f[0] * inv, f[1] * inv), pack2(f[2] * inv, f[3] * inv),
                    pack2(f[4] * inv, f[5] * inv), pack2(f[6] * inv, f[7] * inv));
}
__device__ __forceinline__ uint4 pack(const float (&f)[4], float inv) {
  return make_uint4(__float_as_uint(f[0] * inv), __float_as_uint(f[1] * inv),
                    __float_as_uint(f[2] * inv), __float_as_uint(f[3] * inv));
}

template <typename T>
__global__ __launch_bounds__(256) void merge_kernel(AttnArgs a, Problem p, uint32_t first) {
  constexpr int kDims = 16 / sizeof(T);  // dims per lane
  constexpr int kLanesPerRow = kHeadDim / kDims;
  constexpr int kRowsPerGroup = 256 / kLanesPerRow;
  const int64_t TG = p.T * p.G;
  const int64_t nrow = (int64_t)(a.g1 - a.g0) * TG;
  // r = (g - g0) * T * G + t * G + hl: the chunk-relative row, which is also
  // the row index of the history partials
  const int64_t r = (int64_t)(first + blockIdx.x) * kRowsPerGroup + (threadIdx.x / kLanesPerRow);
  const int lr = threadIdx.x % kLanesPerRow;
  if (r >= nrow) return;
  const int gl = (int)(r / TG);
  const int64_t rem = r - gl * TG;
  const int64_t t = rem / p.G;
  const int h = (a.g0 + gl) * p.G + (int)(rem % p.G);
  const int s = find_seq(a.seqs, p.S, t, [](const SeqInfo& x) { return x.tok_start; });
  const SeqInfo sq = a.seqs[s];
  const int c = ((int)t - sq.tok_start) / p.B;
  const int kh = p.topk - 1;
  const int nh = routed_slots(sq, p, c);
  if (nh <= 0) return;

  uint4* orow = reinterpret_cast<uint4*>(static_cast<T*>(a.out) + t * a.o_st + (int64_t)h * a.o_sh +
                                         kDims * lr);
  float* lrow = a.lse + (int64_t)h * p.T + t;
  const float* lp = a.lse_part + r * kh;
  const uint4* op = reinterpret_cast<const uint4*>(static_cast<const T*>(a.o_part) + r * kh * kHeadDim +
                                                   kDims * lr);

  const float lc = *lrow;
  float acc[kDims];
  unpack(*orow, acc);
  float M = lc, wsum = 1.0f;
  for (int x0 = 0; x0 < nh; x0 += kGroup) {
    uint4 v[kGroup];
    float lv[kGroup];
    // the group's lse values: lane lr of the row loads slot x0 + lr, the
    // others read it from that lane
    const float lmine = x0 + lr < nh ? lp[x0 + lr] : 0.0f;
#pragma unroll
    for (int j = 0; j < kGroup; j++) {
      lv[j] = __shfl(lmine, j, kLanesPerRow);
      if (x0 + j < nh) v[j] = op[(int64_t)(x0 + j) * kLanesPerRow];
    }
    float Mg = M;
#pragma unroll
    for (int j = 0; j < kGroup; j++)
      if (x0 + j < nh) Mg = fmaxf(Mg, lv[j]);
    const float sc = __builtin_amdgcn_exp2f((M - Mg) * kLog2e);
    wsum *= sc;
#pragma unroll
    for (int d = 0; d < kDims; d++) acc[d] *= sc;
    M = Mg;
#pragma unroll
    for (int j = 0; j < kGroup; j++) {
      if (x0 + j < nh) {
        const float w = __builtin_amdgcn_exp2f((lv[j] - M) * kLog2e);
        wsum += w;
        float f[kDims];
        unpack(v[j], f);
#pragma unroll
        for (int d = 0; d < kDims; d++) acc[d] = fmaf(w, f[d], acc[d]);
      }
    }
  }
  const float inv = 1.0f / wsum;
  *orow = pack(acc, inv);
  if (lr == 0) *lrow = M + __builtin_amdgcn_logf(wsum) * kLn2;
}

}  // namespace

hipError_t launch_merge(bool bf16, const AttnArgs& a, const Problem& p, hipStream_t st) {
  const int64_t nrow = (int64_t)(a.g1 - a.g0) * p.T * p.G;
  if (nrow <= 0 || p.topk <= 1) return hipSuccess;
  const int64_t rows_wg = bf16 ? 16 : 8;
  return launch_pieces((nrow + rows_wg - 1) / rows_wg, 256, [&](uint32_t first, unsigned n) {
    if (bf16) merge_kernel<__hip_bfloat16><<<n, 256, 0, st>>>(a, p, first);
    else merge_kernel<float><<<n, 256, 0, st>>>(a, p, first);
  });
}

}  // namespace moba
