// fp32 attention on the fp32 matrix cores (v_mfma_f32_32x32x2_f32: fp32
// products and sums, no narrower split), for fp32 inputs.  History-block
// tiles (partials), causal current-block tiles and dense causal tiles, from
// one kernel; the history and current-block tiles of a chunk go in one launch,
// as neither waits for the other (the merge kernel folds the partials into the
// current-block result).
//
// Work-group = 4 waves = 32 query rows; its keys are cut into subtiles of 32
// and wave w takes subtiles w, w + 4, ...: no barrier in the key loop, short
// blocks still keep four SIMDs busy, and each wave's sums cover a quarter of
// the keys.  The four partial results meet in LDS at the end, in wave order.
// The plan's 128-row tiles are four such work-groups each.
//
// Per subtile and wave:
//   S^T (keys x rows) = K . Q^T: 64 MFMAs in two chains.  Lane (key, half) reads
//   its key's dims 8c + 4 half .. + 3 (c = 0..15) straight from global memory
//   as A operands; Q waits in LDS (rows padded by 16 bytes: conflict-free).
//   softmax: a lane holds 16 keys of one row, its partner (lane ^ 32) the others.
//   O^T (dims x rows) += V^T . P^T: the accumulator layout of S^T (lane half,
//   register i: key 8 (i / 4) + 4 half + i % 4) is the B operand of step i, so
//   P never leaves its registers; A operand dt of lane j is dim 4 j + dt, so
//   one 16-byte load of V row feeds four MFMAs and a half-wave reads whole rows.
// Loads land beside matrix work: half of V is requested before S^T, the other
// half after it (in K's registers), the wave's next K before O^T.  That order,
// pinned by scheduling barriers, holds the kernel at 256 registers without
// spills, so two waves share a SIMD and one's softmax runs beside the other's
// MFMAs.
//
// Bound: the fp32 matrix cores (256 FLOP/clk/CU); a subtile's 128 MFMAs of 64
// cycles outweigh its 32 KB of loads (16 B/clk/CU, mostly L2) and its softmax.
// Against one row per thread on the vector ALUs (128-row work-groups, K and V
// broadcast from LDS), the whole moba_forward: 1024 tokens, one head, B = 128,
// top-3: 620 -> 47 us; 6373 ragged tokens, 8/2 heads, B = 256, top-4: 1865 ->
// 304 us.  Error against fp64 unchanged (2.7e-7 of the norm).
#include "mfma_tile.h"

#include <math.h>

namespace moba {
namespace {

constexpr int kSub = 32;                         // keys per subtile
constexpr int kWaves = 4;
constexpr int kRowsWg = 32;                      // query rows per work-group
constexpr int kSubTiles = kTileRowsF32 / kRowsWg;  // work-groups per plan tile
constexpr int kQRow = kHeadDim / 4 + 1;          // float4 per padded LDS row
constexpr float kLn2 = 0.69314718055994531f;

__device__ __forceinline__ f32x16 mfma_f32(float a, float b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, c, 0, 0, 0);
}

// nhist: work-groups of history tiles (a multiple of 8), first in the grid; first:
// the first work-group of this piece of it.
__global__ __launch_bounds__(64 * kWaves) __attribute__((amdgpu_waves_per_eu(2)))
void attn_f32_kernel(AttnArgs a, Problem p, uint32_t nhist, uint32_t first) {
  // the four waves' results; the query rows live in the first part until then
  __shared__ float4 lds[kWaves * kRowsWg * kQRow];
  __shared__ float sm[kWaves][kRowsWg], sl[kWaves][kRowsWg];
  __shared__ int64_t sdst[kRowsWg];  // output row (float4 units), -1: none
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int qc = lane & 31, hh = lane >> 5;

  // ------------------------------------------------------------ tile setup
  const uint32_t bx = first + blockIdx.x;
  const bool hist = bx < nhist;
  int g, h;
  int64_t kbeg, kend, dst, tmin;
  int t;  // (T is below 2^31)
  bool valid;
  if (hist) {
    // tiles of one bin share its K/V block: a contiguous run of tiles per XCD
    const int64_t nb = p.nblk_total;
    const int64_t tbeg = a.bin_tile_start[a.g0 * nb];
    const int64_t tend = a.bin_tile_start[a.g1 * nb];
    const uint32_t per = (uint32_t)((tend - tbeg) * kSubTiles + 7) / 8;
    const uint32_t w = (bx % 8) * per + bx / 8;
    const int64_t tile = tbeg + w / kSubTiles;
    if (bx / 8 >= per || tile >= tend) return;
    const int bin = a.tile_bin[tile];
    g = bin / p.nblk_total;
    const int b = bin % p.nblk_total;
    const int64_t e0 = a.bin_start[bin] + (tile - a.bin_tile_start[bin]) * kTileRowsF32 +
                       (w % kSubTiles) * kRowsWg;
    const int n = (int)min((int64_t)kRowsWg, a.bin_start[bin] + a.bin_count[bin] - e0);
    if (n <= 0) return;
    const int s = find_seq(a.seqs, p.S, b, [](const SeqInfo& x) { return x.blk_off; });
    kbeg = (int64_t)a.seqs[s].tok_start + (int64_t)(b - a.seqs[s].blk_off) * p.B;
    kend = kbeg + p.B;
    tmin = kend;  // every key precedes every routed query
    const uint32_t kh = (uint32_t)(p.topk - 1);
    const uint32_t ev = a.entries[e0 + min(qc, n - 1)];
    const uint64_t TG = (uint64_t)p.T * p.G;
    const uint64_t rem = ev / kh - (uint64_t)g * TG;
    const bool ok = rem < TG;  // (T * G is below 2^32)
    valid = qc < n && ok;
    t = ok ? (int)((uint32_t)rem / (uint32_t)p.G) : (int)kbeg;
    h = g * p.G + (ok ? (int)((uint32_t)rem % (uint32_t)p.G) : 0);
    dst = (int64_t)(ev - (uint64_t)a.g0 * TG * kh);
  } else {
    // 8 consecutive tiles of the list sit on the 8 XCDs; the sub-tiles of a
    // tile follow on its XCD
    const uint32_t x = bx - nhist;
    const uint32_t per = (uint32_t)((a.ntiles + 7) / 8 * 8 * kSubTiles);
    g = a.g0 + (int)(x / per);
    const uint32_t y = x % per;
    const uint32_t tile = y / (8 * kSubTiles) * 8 + y % 8;
    if (tile >= a.ntiles) return;
    const CausalTile ct = a.tiles[tile];
    const int r0 = (int)(y / 8 % kSubTiles) * kRowsWg;
    const int n = min(kRowsWg, (ct.t1 - ct.t0) * p.G - r0);
    if (n <= 0) return;  // also the padding of the tile list
    kbeg = ct.kbeg;
    tmin = ct.t0 + r0 / p.G;
    kend = ct.t0 + (r0 + n - 1) / p.G + 1;
    valid = qc < n;
    const int rr = r0 + (valid ? qc : 0);
    t = ct.t0 + rr / p.G;
    h = g * p.G + rr % p.G;
    dst = 0;
  }
  g = __builtin_amdgcn_readfirstlane(g);
  kbeg = uniform64(kbeg);
  kend = uniform64(kend);
  tmin = uniform64(tmin);

  // query rows to LDS: thread -> row tid / 8, 4 of its 32 chunks
  if (tid < kRowsWg) sdst[tid] = (int64_t)t * a.q_st + (int64_t)h * a.q_sh;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const int row = tid >> 3, c = (tid & 7) + 8 * j;
    lds[row * kQRow + c] = reinterpret_cast<const float4*>(static_cast<const float*>(a.q) + sdst[row])[c];
  }

  const float* kb = static_cast<const float*>(a.k) + (int64_t)g * a.k_sh;
  const float* vb = static_cast<const float*>(a.v) + (int64_t)g * a.v_sh;
  const float c2 = a.scale_log2;
  const int nsub = (int)((kend - kbeg + kSub - 1) / kSub);
  f32x16 o[4];
#pragma unroll
  for (int dt = 0; dt < 4; dt++)
#pragma unroll
    for (int r = 0; r < 16; r++) o[dt][r] = 0.0f;
  float m = -INFINITY, l = 0.0f;
  float4 kf[16], vf[16];
  // rows past the key range repeat its last key; they are always masked
  auto load_k = [&](int i) {
    const int64_t u = min(kbeg + (int64_t)i * kSub + qc, kend - 1);
    const float4* kr = reinterpret_cast<const float4*>(kb + u * a.k_st) + hh;
#pragma unroll
    for (int c = 0; c < 16; c++) kf[c] = kr[2 * c];
  };
  auto load_v = [&](int i, int r0) {
#pragma unroll
    for (int r = r0; r < r0 + 8; r++) {
      const int64_t u = min(kbeg + (int64_t)i * kSub + 8 * (r >> 2) + 4 * hh + (r & 3), kend - 1);
      vf[r] = reinterpret_cast<const float4*>(vb + u * a.v_st)[qc];
    }
  };
  if (wave < nsub) load_k(wave);
  __syncthreads();
  const float4* qrow = lds + qc * kQRow + hh;
  for (int i = wave; i < nsub; i += kWaves) {
    load_v(i, 0);
    __builtin_amdgcn_sched_barrier(0);
    f32x16 s0, s1;
#pragma unroll
    for (int r = 0; r < 16; r++) s0[r] = s1[r] = 0.0f;
#pragma unroll
    for (int c = 0; c < 16; c += 2) {
      const float4 qa = qrow[2 * c], qb = qrow[2 * c + 2];
      s0 = mfma_f32(kf[c].x, qa.x, s0);
      s1 = mfma_f32(kf[c + 1].x, qb.x, s1);
      s0 = mfma_f32(kf[c].y, qa.y, s0);
      s1 = mfma_f32(kf[c + 1].y, qb.y, s1);
      s0 = mfma_f32(kf[c].z, qa.z, s0);
      s1 = mfma_f32(kf[c + 1].z, qb.z, s1);
      s0 = mfma_f32(kf[c].w, qa.w, s0);
      s1 = mfma_f32(kf[c + 1].w, qb.w, s1);
      if (c % 4 == 2) __builtin_amdgcn_sched_barrier(0);
    }
    load_v(i, 8);
    __builtin_amdgcn_sched_barrier(0);
    const int64_t u0 = kbeg + (int64_t)i * kSub;
    float z[16];
#pragma unroll
    for (int r = 0; r < 16; r++) z[r] = (s0[r] + s1[r]) * c2;
    if (u0 + kSub > kend || u0 + kSub - 1 > tmin) {
      // keys of this lane: u0 + 4 hh + 8 (r / 4) + r % 4, kept below lim
      const int lim = (int)(min(hist ? kend : (int64_t)t + 1, kend) - u0) - 4 * hh;
#pragma unroll
      for (int r = 0; r < 16; r++) z[r] = 8 * (r >> 2) + (r & 3) < lim ? z[r] : -INFINITY;
    }
    float mx = z[0];
#pragma unroll
    for (int r = 1; r < 16; r++) mx = fmaxf(mx, z[r]);
    mx = fmaxf(mx, xor32(mx));
    const float m_new = fmaxf(m, mx);
    const float m_use = m_new == -INFINITY ? 0.0f : m_new;
    const float alpha = __builtin_amdgcn_exp2f(m - m_use);
    l *= alpha;
#pragma unroll
    for (int dt = 0; dt < 4; dt++)
#pragma unroll
      for (int r = 0; r < 16; r++) o[dt][r] *= alpha;
    m = m_new;
#pragma unroll
    for (int r = 0; r < 16; r++) {
      z[r] = __builtin_amdgcn_exp2f(z[r] - m_use);
      l += z[r];
    }
    if (i + kWaves < nsub) load_k(i + kWaves);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int r = 0; r < 16; r++) {
      o[0] = mfma_f32(vf[r].x, z[r], o[0]);
      o[1] = mfma_f32(vf[r].y, z[r], o[1]);
      o[2] = mfma_f32(vf[r].z, z[r], o[2]);
      o[3] = mfma_f32(vf[r].w, z[r], o[3]);
    }
  }

  // -------------------------------------------------------------- epilogue
  // each wave scales its sums to the row's overall max and leaves them in LDS
  const float lw = l + xor32(l);
  if (hh == 0) {
    sm[wave][qc] = m;
    sl[wave][qc] = lw;
  }
  __syncthreads();  // every wave is done with the query rows too
  float M = sm[0][qc];
#pragma unroll
  for (int w = 1; w < kWaves; w++) M = fmaxf(M, sm[w][qc]);
  float L = 0.0f;
#pragma unroll
  for (int w = 0; w < kWaves; w++) L += sl[w][qc] * __builtin_amdgcn_exp2f(sm[w][qc] - M);
  const float scl = __builtin_amdgcn_exp2f(m - M) / L;
  float4* mine = lds + (wave * kRowsWg + qc) * kQRow;
#pragma unroll
  for (int r = 0; r < 16; r++)
    mine[8 * (r >> 2) + 4 * hh + (r & 3)] =
        make_float4(o[0][r] * scl, o[1][r] * scl, o[2][r] * scl, o[3][r] * scl);
  if (tid < kRowsWg) {
    sdst[qc] = !valid ? -1 : hist ? dst * kHeadDim : (int64_t)t * a.o_st + (int64_t)h * a.o_sh;
    if (valid) {
      const float lse = (M + __builtin_amdgcn_logf(L)) * kLn2;
      if (hist) a.lse_part[dst] = lse;
      else a.lse[(int64_t)h * p.T + t] = lse;
    }
  }
  __syncthreads();
  float* outp = static_cast<float*>(hist ? a.o_part : a.out);
#pragma unroll
  for (int j = 0; j < 4; j++) {
    const int row = (tid >> 5) + 8 * j, c = tid & 31;
    float4 x = lds[row * kQRow + c];
#pragma unroll
    for (int w = 1; w < kWaves; w++) {
      const float4 y = lds[(w * kRowsWg + row) * kQRow + c];
      x.x += y.x;
      x.y += y.y;
      x.z += y.z;
      x.w += y.w;
    }
    if (sdst[row] >= 0) reinterpret_cast<float4*>(outp + sdst[row])[c] = x;
  }
}

}  // namespace

hipError_t launch_attn_f32(const AttnArgs& a, const Problem& p, int64_t hist_tiles, bool in_place,
                           hipStream_t st) {
  if (a.g1 <= a.g0) return hipSuccess;
  const int64_t nhist = (hist_tiles * kSubTiles + 7) / 8 * 8;
  const int64_t ncur = (a.ntiles + 7) / 8 * 8 * kSubTiles * (a.g1 - a.g0);
  const auto run = [&](int64_t begin, int64_t groups) {
    return launch_pieces(groups, 64 * kWaves, [&](uint32_t first, unsigned n) {
      attn_f32_kernel<<<n, 64 * kWaves, 0, st>>>(a, p, (uint32_t)nhist, (uint32_t)begin + first);
    });
  };
  if (!in_place) return run(0, nhist + ncur);
  const hipError_t e = run(0, nhist);
  return e != hipSuccess ? e : run(nhist, ncur);
}

}  // namespace moba
