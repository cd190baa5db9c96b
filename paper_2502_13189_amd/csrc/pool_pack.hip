// Block mean-pool of the keys and the packed V^T layout of the MFMA kernels.
//
// Both are one pass over memory and independent of each other, so a call that
// needs both makes one launch: pool work-groups first, then pack work-groups.
//
// Pool (Eq. 6; Algorithm 1 mean_pool): one work-group per (global block,
// kv-head), 16 lanes to a token row: each lane owns 8 consecutive dims and walks the
// block's tokens, reading a 256-byte key row per 16 lanes (coalesced).  Sums are kept
// in fp64 and reduced across the rows in a fixed order, so the result is the block
// mean rounded once to fp32 and is bit-reproducible.  Two sizes (pool_threads):
//   256 threads, 16 rows, one load in flight: short blocks, which have no more rows to
//     read, and batches of many blocks, where the other work-groups of a CU hide the
//     latency;
//   1024 threads, 64 rows, four loads in flight: few long blocks, bound by the latency
//     of one block's loads.
//
// V^T pack: four waves per (64-key tile of a sequence, kv-head), each 32 dims and
// without a barrier.  A wave's 64 x 32 values are staged in LDS and written back as
// 32 rows (dims) of 64 keys, with the keys of every 16-key group stored in the order
// 0-3, 8-11, 4-7, 12-15.  That order is the k-slot order in which the
// attention kernel's P^T operand holds keys after the QK^T MFMA (see
// attn_mfma.hip), so each lane reads its 8 keys as one 16-byte LDS load.
// Keys past the end of the sequence are stored as zeros.
#include "moba_internal.h"

#include <algorithm>

namespace moba {
namespace {

template <typename T>
struct Load8;

template <>
struct Load8<__hip_bfloat16> {
  static __device__ __forceinline__ void run(const __hip_bfloat16* p, float* f) {
    uint4 u = *reinterpret_cast<const uint4*>(p);
    uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
    for (int i = 0; i < 4; i++) {
      f[2 * i] = __uint_as_float(w[i] << 16);
      f[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
    }
  }
};

template <>
struct Load8<float> {
  static __device__ __forceinline__ void run(const float* p, float* f) {
    float4 a = *reinterpret_cast<const float4*>(p);
    float4 b = *reinterpret_cast<const float4*>(p + 4);
    f[0] = a.x; f[1] = a.y; f[2] = a.z; f[3] = a.w;
    f[4] = b.x; f[5] = b.y; f[6] = b.z; f[7] = b.w;
  }
};

constexpr int kPackRow = 32 + 2;

constexpr int kPoolSums = 16;  // partial sums of a block: 16 rows, or 16 waves

// kterm (nullable): the block keys split exactly into three bf16 planes,
// kbar = hi + mid + lo, each plane [nblk_total, Hkv, D] (read by the
// matrix-core gate).  THREADS / 16 token rows at a time.
template <typename T, int THREADS>
__device__ __forceinline__ void pool_block(const T* __restrict__ k, int64_t k_st, int64_t k_sh,
                                           const SeqInfo* __restrict__ seqs, const Problem& p, int b,
                                           int g, float* __restrict__ kbar,
                                           __hip_bfloat16* __restrict__ kterm,
                                           double (*red)[kHeadDim]) {
  const int s = find_seq(seqs, p.S, b, [](const SeqInfo& x) { return x.blk_off; });
  const SeqInfo sq = seqs[s];
  const int j = b - sq.blk_off;
  const int64_t t0 = (int64_t)sq.tok_start + (int64_t)j * p.B;
  const int n = (int)min((int64_t)p.B, (int64_t)sq.len - (int64_t)j * p.B);
  constexpr int kPoolRows = THREADS / 16;
  constexpr int kPoolAhead = THREADS > 256 ? 4 : 1;  // loads in flight per thread
  const int row = threadIdx.x >> 4;
  const int d0 = (threadIdx.x & 15) * 8;
  const T* src = k + t0 * k_st + (int64_t)g * k_sh + d0;
  double acc[8];
#pragma unroll
  for (int i = 0; i < 8; i++) acc[i] = 0.0;
  int t = row;
  for (; t + (kPoolAhead - 1) * kPoolRows < n; t += kPoolAhead * kPoolRows) {
    float f[kPoolAhead][8];
#pragma unroll
    for (int e = 0; e < kPoolAhead; e++)
      Load8<T>::run(src + (int64_t)(t + e * kPoolRows) * k_st, f[e]);
#pragma unroll
    for (int e = 0; e < kPoolAhead; e++)
#pragma unroll
      for (int i = 0; i < 8; i++) acc[i] += (double)f[e][i];
  }
  for (; t < n; t += kPoolRows) {
    float f[8];
    Load8<T>::run(src + (int64_t)t * k_st, f);
#pragma unroll
    for (int i = 0; i < 8; i++) acc[i] += (double)f[i];
  }
  if constexpr (THREADS == 256) {
#pragma unroll
    for (int i = 0; i < 8; i++) red[row][d0 + i] = acc[i];
  } else {
    // the wave's four rows, then the waves
#pragma unroll
    for (int i = 0; i < 8; i++) {
      acc[i] += __shfl_xor(acc[i], 16, 64);
      acc[i] += __shfl_xor(acc[i], 32, 64);
    }
    const int wave = threadIdx.x >> 6;
    if ((threadIdx.x & 63) < 16) {
#pragma unroll
      for (int i = 0; i < 8; i++) red[wave][d0 + i] = acc[i];
    }
  }
  __syncthreads();
  if (threadIdx.x < kHeadDim) {
    double sum = 0.0;
#pragma unroll
    for (int r = 0; r < kPoolSums; r++) sum += red[r][threadIdx.x];
    const float m = (float)(sum / (double)n);
    const int64_t o = ((int64_t)b * p.Hkv + g) * kHeadDim + threadIdx.x;
    kbar[o] = m;
    if (kterm) {
      const int64_t plane = (int64_t)p.nblk_total * p.Hkv * kHeadDim;
      const __hip_bfloat16 hi = __float2bfloat16(m);
      const float r1 = m - __bfloat162float(hi);
      const __hip_bfloat16 mid = __float2bfloat16(r1);
      kterm[o] = hi;
      kterm[o + plane] = mid;
      kterm[o + 2 * plane] = __float2bfloat16(r1 - __bfloat162float(mid));
    }
  }
}

// Position p (0..63) of a packed tile holds key perm(p) of the tile.
__device__ __forceinline__ int packed_key(int p) {
  const int grp = p & ~15, w = p & 15;
  const int half = w >> 3, jj = w & 7;
  return grp + 8 * (jj >> 2) + 4 * half + (jj & 3);
}

// Dims 32 quarter .. + 31 of tile idx (< vt_tiles) of kv-head g, by one wave.
__device__ __forceinline__ void pack_tile(const __hip_bfloat16* __restrict__ v, int64_t v_st,
                                          int64_t v_sh, const SeqInfo* __restrict__ seqs,
                                          int S, int64_t vt_tiles, int64_t idx, int g,
                                          int quarter, __hip_bfloat16* __restrict__ vt,
                                          uint16_t (*tile)[kPackRow]) {
  const int lane = threadIdx.x & 63;
  const int s = find_seq(seqs, S, idx, [](const SeqInfo& x) { return x.vt_tile_off; });
  const SeqInfo sq = seqs[s];
  const int i = (int)(idx - sq.vt_tile_off);
  // stage 64 keys x 32 dims: 4 lanes per key, 16 keys per load
  uint4 u[4];
#pragma unroll
  for (int x = 0; x < 4; x++) {
    const int local = i * kKeyTile + 16 * x + (lane >> 2);
    u[x] = make_uint4(0, 0, 0, 0);
    if (local < sq.len)
      u[x] = *reinterpret_cast<const uint4*>(v + ((int64_t)sq.tok_start + local) * v_st +
                                             (int64_t)g * v_sh + 32 * quarter + 8 * (lane & 3));
  }
#pragma unroll
  for (int x = 0; x < 4; x++) {
    uint32_t* dst = reinterpret_cast<uint32_t*>(&tile[16 * x + (lane >> 2)][8 * (lane & 3)]);
    dst[0] = u[x].x;
    dst[1] = u[x].y;
    dst[2] = u[x].z;
    dst[3] = u[x].w;
  }
  asm volatile("s_waitcnt lgkmcnt(0)" : : : "memory");  // the wave's own writes, no barrier
  __hip_bfloat16* dst = vt + ((int64_t)g * vt_tiles + idx) * (kKeyTile * kHeadDim) +
                        32 * quarter * kKeyTile;
#pragma unroll
  for (int x = 0; x < 4; x++) {
    const int c = lane + 64 * x;
    const int d = c >> 3, p0 = (c & 7) * 8;
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; e++) {
      const uint32_t lo = tile[packed_key(p0 + 2 * e)][d];
      const uint32_t hi = tile[packed_key(p0 + 2 * e + 1)][d];
      w[e] = lo | (hi << 16);
    }
    *reinterpret_cast<uint4*>(dst + d * kKeyTile + p0) = make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// The pack by itself (dense attention): one tile per work-group (small dense calls ran 0.5-1.3 us
// slower with 1024-thread ones).  It takes the two counts it needs, not the whole Problem: the
// smallest dense calls wait for the host, and the launch costs them 0.15 of 22 us less.
__global__ __launch_bounds__(256) void pack_kernel(const __hip_bfloat16* __restrict__ v,
                                                   int64_t v_st, int64_t v_sh,
                                                   const SeqInfo* __restrict__ seqs, int S,
                                                   int64_t vt_tiles,
                                                   __hip_bfloat16* __restrict__ vt) {
  __shared__ __attribute__((aligned(16))) uint16_t tile[4][kKeyTile][kPackRow];
  const int wave = threadIdx.x >> 6;
  pack_tile(v, v_st, v_sh, seqs, S, vt_tiles, blockIdx.x, blockIdx.y, wave, vt, tile[wave]);
}

// Work-groups [0, npool): pool (block, kv-head); then pack (a tile per four waves, kv-head).
// first: this launch's first work-group.
template <typename T, bool PACK, int THREADS>
__global__ __launch_bounds__(THREADS) __attribute__((amdgpu_waves_per_eu(8)))
void pool_pack_kernel(
    const T* __restrict__ k, int64_t k_st, int64_t k_sh, const __hip_bfloat16* __restrict__ v,
    int64_t v_st, int64_t v_sh, const SeqInfo* __restrict__ seqs, Problem p, uint32_t first,
    uint32_t npool, float* __restrict__ kbar, __hip_bfloat16* __restrict__ kterm, __hip_bfloat16* __restrict__ vt) {
  constexpr int kPackTiles = THREADS / 256;
  constexpr size_t kPoolLds = sizeof(double) * kPoolSums * kHeadDim;
  constexpr size_t kPackLds = sizeof(uint16_t) * (THREADS / 64) * kKeyTile * kPackRow;
  __shared__ __attribute__((aligned(16))) char lds[PACK && kPackLds > kPoolLds ? kPackLds : kPoolLds];
  const uint32_t x = first + blockIdx.x;
  if (x < npool) {
    pool_block<T, THREADS>(k, k_st, k_sh, seqs, p, (int)(x % (uint32_t)p.nblk_total),
                           (int)(x / (uint32_t)p.nblk_total), kbar, kterm,
                           reinterpret_cast<double(*)[kHeadDim]>(lds));
    return;
  }
  if constexpr (PACK) {
    const uint32_t per = (uint32_t)((p.vt_tiles + kPackTiles - 1) / kPackTiles);
    const uint32_t y = x - npool;
    const int wave = threadIdx.x >> 6;
    const int64_t idx = (int64_t)(y % per) * kPackTiles + (wave >> 2);
    if (idx < p.vt_tiles)
      pack_tile(v, v_st, v_sh, seqs, p.S, p.vt_tiles, idx, (int)(y / per), wave & 3, vt,
                reinterpret_cast<uint16_t(*)[kPackRow]>(lds) + wave * kKeyTile);
  }
}

template <typename T, bool PACK, int THREADS>
hipError_t launch_threads(const T* k, int64_t k_st, int64_t k_sh, const __hip_bfloat16* v,
                          int64_t v_st, int64_t v_sh, const SeqInfo* seqs, const Problem& p,
                          float* kbar, __hip_bfloat16* kterm, __hip_bfloat16* vt, hipStream_t st) {
  constexpr int kPackTiles = THREADS / 256;
  const int64_t npool = (int64_t)p.nblk_total * p.Hkv;
  const int64_t npack = PACK ? (p.vt_tiles + kPackTiles - 1) / kPackTiles * p.Hkv : 0;
  return launch_pieces(npool + npack, THREADS, [&](uint32_t first, unsigned n) {
    pool_pack_kernel<T, PACK, THREADS><<<n, THREADS, 0, st>>>(
        k, k_st, k_sh, v, v_st, v_sh, seqs, p, first, (uint32_t)npool, kbar, kterm, vt);
  });
}

// Threads per pool work-group: 256 where a block has no more than 128 rows, or where
// there are so many (kv-head, block) pairs that 1024 threads have nothing left to hide
// (2048: eight work-groups of 256 on every CU).  Block means alone, with 1024 -> 256
// threads: B = 64: 32768 pairs 239 -> 132 us, 2048 pairs 18.8 -> 8.5, 128 pairs 6.6 ->
// 6.2; B = 256: 512 pairs 9.0 -> 8.8, 128 pairs 6.7 -> 7.6; B = 512: 4096 pairs 120 -> 96,
// 1024 pairs 23.6 -> 22.8, 256 pairs 7.7 -> 11.8; B = 1024: 2048 pairs 123 -> 98, 512 pairs
// 24 -> 30; B = 4096: 512 pairs 105 -> 155.  With the pack beside them the line is the
// same (65536 tokens, 32 kv-heads, B = 64: 455 -> 371 us; B = 512: 361 -> 338).
int pool_threads(const Problem& p) {
  const int64_t pairs = (int64_t)p.nblk_total * p.Hkv;
  return p.B <= 128 || pairs >= std::min<int64_t>(2 * (int64_t)p.B, 2048) ? 256 : 1024;
}

template <typename T, bool PACK>
hipError_t launch_typed(const T* k, int64_t k_st, int64_t k_sh, const __hip_bfloat16* v,
                        int64_t v_st, int64_t v_sh, const SeqInfo* seqs, const Problem& p,
                        float* kbar, __hip_bfloat16* kterm, __hip_bfloat16* vt, hipStream_t st) {
  if (pool_threads(p) == 256)
    return launch_threads<T, PACK, 256>(k, k_st, k_sh, v, v_st, v_sh, seqs, p, kbar, kterm, vt, st);
  return launch_threads<T, PACK, 1024>(k, k_st, k_sh, v, v_st, v_sh, seqs, p, kbar, kterm, vt, st);
}

}  // namespace

hipError_t launch_pool(const void* k, bool bf16, int64_t k_st, int64_t k_sh, const SeqInfo* seqs,
                       const Problem& p, float* kbar, __hip_bfloat16* kterm, hipStream_t st) {
  if (p.nblk_total == 0) return hipSuccess;
  if (bf16)
    return launch_typed<__hip_bfloat16, false>(static_cast<const __hip_bfloat16*>(k), k_st, k_sh,
                                               nullptr, 0, 0, seqs, p, kbar, kterm, nullptr, st);
  return launch_typed<float, false>(static_cast<const float*>(k), k_st, k_sh, nullptr, 0, 0, seqs,
                                    p, kbar, kterm, nullptr, st);
}

hipError_t launch_pack(const __hip_bfloat16* v, int64_t v_st, int64_t v_sh, const SeqInfo* seqs,
                       const Problem& p, __hip_bfloat16* vt, hipStream_t st) {
  if (p.vt_tiles == 0) return hipSuccess;
  pack_kernel<<<dim3((unsigned)p.vt_tiles, p.Hkv), 256, 0, st>>>(v, v_st, v_sh, seqs, p.S, p.vt_tiles,
                                                                      vt);
  return hipGetLastError();
}

hipError_t launch_pool_pack(const __hip_bfloat16* k, int64_t k_st, int64_t k_sh,
                            const __hip_bfloat16* v, int64_t v_st, int64_t v_sh,
                            const SeqInfo* seqs, const Problem& p, float* kbar,
                            __hip_bfloat16* kterm, __hip_bfloat16* vt, hipStream_t st) {
  if (p.vt_tiles == 0) return hipSuccess;
  return launch_typed<__hip_bfloat16, true>(k, k_st, k_sh, v, v_st, v_sh, seqs, p, kbar, kterm, vt,
                                            st);
}

}  // namespace moba
