// Decode: one new query per sequence against its key/value cache.  Query s
// sits at the last position L_s - 1 of sequence s (its key and value are the
// cache's last entries), so its result is the last row of the prefill over
// the cache: MoBA (the gate of Eq. 5 / Eq. 6 with the causal rules of
// Sec. 2.2, attention of Eq. 2 over the key set of Eq. 4) or causal full
// attention (Eq. 1), which is what the paper uses for generation (Sec. 3.3).
//
// Decode reads each attended key once per kv-head and does ~2 FLOP per byte,
// far below the ridge of either the matrix cores or the vector ALUs, so it is
// bound by HBM and the loads decide: a probe of the bare loads ran at 4.6-5.0
// TB/s with one key row per lane and at 5.8-6.1 TB/s with K as matrix operands (16
// rows x 64 bytes per load) and V by whole rows, the layouts used here; so S
// comes from the matrix cores, P V from packed bf16 dot products.  In MoBA
// mode only the selected blocks are touched.
//
//   gate     one work-group per (sequence, query head): fp32 scores of the
//            query against the block means of the sequence's complete past
//            blocks (four partial sums over dim quarters, added in order), then top-(k-1) (ties:
//            lower block index): up to 1024 candidates by rank, each thread
//            counting the candidates that precede its own; beyond, by k-1
//            rounds of a wave-wide argmax.  The selection is written
//            ascending with the current block last.
//   attend   one work-group per (sequence, kv-head, 256-key chunk; chunks
//            never cross a block boundary; in MoBA mode only the chunks of
//            the blocks the group's query heads selected, which each
//            work-group finds from the selections itself: its slot's block
//            in the ascending union), all query heads of the group:
//            S (64 keys x up to 16 heads per wave) on 16x16x32 MFMAs, a per-head
//            softmax over the chunk (a lane holds 16 keys of one head), P V with
//            8 dims and 16 of the wave's 64 keys per lane (dot2 over key
//            pairs: weights rounded once to bf16, as the prefill's P V, fp32
//            sums); the value rows are all requested before the softmax; the
//            normalised partial and its lse go to the workspace; a head that
//            did not select the chunk's block skips it.
//   combine  log-sum-exp merge of each row's partials: nsplit work-groups
//            per row each fold a share of up to kCombineShare consecutive
//            partial slots (16 interleaved groups, eight partial loads in
//            flight per group, then the groups in order); with one share
//            the work-group writes the row, otherwise a second kernel folds
//            the shares in order.  Rounded once to the output dtype.
#include "decode_internal.h"

#include <math.h>

#include <type_traits>

namespace moba {
namespace {

constexpr float kLn2 = 0.69314718055994531f;
constexpr float kLog2e = 1.4426950408889634f;

typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef float f32x4_t __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4_t __attribute__((ext_vector_type(4)));
__device__ __forceinline__ bf16x2_t as_bf16x2(uint32_t w) { return __builtin_bit_cast(bf16x2_t, w); }
__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
// Two fp32 values to a packed bf16 pair, round-to-nearest-even.
__device__ __forceinline__ uint32_t pack_bf16(float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  const f32x2_t v = {a, b};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, bf16x2_t));
}
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xffff0000u); }

// Key range of chunk x of sequence length L: block j = x / nsub, piece
// i = x % nsub of kDecodeChunk keys, cut at the block end and at L.
__device__ __forceinline__ void chunk_range(int x, int nsub, int B, int64_t L, int64_t& u0,
                                            int64_t& u1) {
  const int64_t j = x / nsub, i = x % nsub;
  u0 = j * B + i * kDecodeChunk;
  u1 = min(min(u0 + kDecodeChunk, (j + 1) * (int64_t)B), L);
}

// ================================================================== gate
// One work-group per (sequence, query head).  Four lanes per block mean, each
// a quarter of its dims straight into registers (a quarter is one 128-byte line),
// all of a pass's loads in flight at once; a quarter is summed in dim order and the
// four are added in order across the lanes.  (Staged through LDS 64 blocks at a
// time, with three barriers each, the kernel took 16.3 us at 255 blocks, 32 heads; this
// way 14.9 us.)
constexpr int kGateAhead = 4;               // blocks per thread and pass
constexpr int kGatePass = 64 * kGateAhead;  // blocks per pass
constexpr int kRankMax = 1024;              // candidates ranked in parallel (4 per thread)

__global__ __launch_bounds__(256) void decode_gate_kernel(DecodeArgs a, Problem p,
                                                          const SeqInfo* __restrict__ seqs) {
  __shared__ __attribute__((aligned(16))) float sc[kMaxBlocksPerSeq + 4];
  const int tid = threadIdx.x, lane = tid & 63;
  const int64_t row = blockIdx.x;  // s * Hq + h
  const int s = (int)(row / p.Hq), h = (int)(row % p.Hq);
  const int g = h / p.G;
  const SeqInfo sq = seqs[s];
  const int quarter = tid & 3;
  const int c = (int)((sq.len - 1) / p.B);  // current block; candidates j < c
  uint4 qw[4];  // this quarter of the query
  {
    const __hip_bfloat16* qr = a.q + (int64_t)s * a.q_ss + (int64_t)h * a.q_sh + 32 * quarter;
#pragma unroll
    for (int i = 0; i < 4; i++) qw[i] = reinterpret_cast<const uint4*>(qr)[i];
  }
  // one pass from block j0: AHEAD x 64 blocks
  const auto pass = [&](int j0, auto ahead) {
    constexpr int kAhead = decltype(ahead)::value;
    float4 kv[kAhead][8];
#pragma unroll
    for (int e = 0; e < kAhead; e++) {
      const int j = min(j0 + 64 * e + (tid >> 2), c - 1);  // past the candidates: re-read, unused
      const float4* kr = reinterpret_cast<const float4*>(
          a.kbar + ((int64_t)(sq.blk_off + j) * p.Hkv + g) * kHeadDim + 32 * quarter);
#pragma unroll
      for (int i = 0; i < 8; i++) kv[e][i] = kr[i];
    }
#pragma unroll
    for (int e = 0; e < kAhead; e++) {
      float acc = 0.0f;
#pragma unroll
      for (int i = 0; i < 8; i++) {
        const uint32_t w0 = i & 1 ? qw[i >> 1].z : qw[i >> 1].x, w1 = i & 1 ? qw[i >> 1].w : qw[i >> 1].y;
        acc = fmaf(bf16_lo(w0), kv[e][i].x, acc);
        acc = fmaf(bf16_hi(w0), kv[e][i].y, acc);
        acc = fmaf(bf16_lo(w1), kv[e][i].z, acc);
        acc = fmaf(bf16_hi(w1), kv[e][i].w, acc);
      }
      const float p1 = __shfl_down(acc, 1, 4), p2 = __shfl_down(acc, 2, 4), p3 = __shfl_down(acc, 3, 4);
      const int j = j0 + 64 * e + (tid >> 2);
      // NaN counts as -inf, so that the order is total and exactly nh blocks are kept
      if (quarter == 0 && j < c) sc[j] = fmaxf(((acc + p1) + p2) + p3, -INFINITY);
    }
  };
  for (int j0 = 0; j0 < c; j0 += kGatePass) {
    // (a row of few blocks would otherwise read its last one over and over)
    if (c - j0 > 128) pass(j0, std::integral_constant<int, kGateAhead>{});
    else if (c - j0 > 64) pass(j0, std::integral_constant<int, 2>{});
    else pass(j0, std::integral_constant<int, 1>{});
  }
  if (tid < 4) sc[c + tid] = -INFINITY;  // the rank loop reads whole groups of four
  __syncthreads();
  const int kh = p.topk - 1;
  const int nh = min(kh, c);
  if (c <= kRankMax) {
    // top-(k-1) by rank: candidate j is kept iff fewer than nh candidates
    // precede it in (score desc, index asc) order — the same set as the
    // argmax rounds below.  Thread t ranks candidates t + 256 i against all
    // (every lane reads the same score: broadcast), then the kept ones are
    // written ascending: a kept candidate's place is the number of kept ones
    // in the earlier 64-candidate groups plus those below it in its own.
    __shared__ int gcnt[kRankMax / 64];
    const int wave = tid >> 6;
    uint64_t bal[kRankMax / 256];
#pragma unroll
    for (int i = 0; i < kRankMax / 256; i++) {
      const int j = tid + 256 * i;
      bool keep = false;
      if (j < c) {
        const float sj = sc[j];
        int above = 0;
#pragma unroll 4
        for (int u = 0; u < c; u += 4) {  // (padded with -inf past c)
          const float4 su = *reinterpret_cast<const float4*>(&sc[u]);
          above += (su.x > sj || (su.x == sj && u < j)) ? 1 : 0;
          above += (su.y > sj || (su.y == sj && u + 1 < j)) ? 1 : 0;
          above += (su.z > sj || (su.z == sj && u + 2 < j)) ? 1 : 0;
          above += (su.w > sj || (su.w == sj && u + 3 < j)) ? 1 : 0;
        }
        keep = above < nh;
      }
      bal[i] = __ballot(keep);
      if (lane == 0) gcnt[4 * i + wave] = __popcll(bal[i]);
    }
    __syncthreads();
    int32_t* out = a.sel + row * p.topk;
#pragma unroll
    for (int i = 0; i < kRankMax / 256; i++) {
      if ((bal[i] >> lane) & 1) {
        int pos = __popcll(bal[i] & ((uint64_t(1) << lane) - 1));
        for (int x = 0; x < 4 * i + wave; x++) pos += gcnt[x];
        out[pos] = tid + 256 * i;
      }
    }
    if (tid == 0) out[nh] = c;
    for (int x = nh + 1 + tid; x < p.topk; x += 256) out[x] = -1;
    return;
  }
  if (tid >= 64) return;
  // top-(k-1) for longer sequences: rounds of a wave-wide argmax over (score
  // desc, index asc); lane L owns candidates L, L + 64, ... and marks its
  // taken ones in a mask
  uint64_t taken = 0;
  for (int r = 0; r < nh; r++) {
    float best = -INFINITY;
    int bj = INT32_MAX;
    for (int j = lane, x = 0; j < c; j += 64, x++) {
      if ((taken >> x) & 1) continue;
      const float v = sc[j];
      if (v > best || (v == best && j < bj)) { best = v; bj = j; }
    }
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) {
      const float ob = __shfl_xor(best, m, 64);
      const int oj = __shfl_xor(bj, m, 64);
      if (ob > best || (ob == best && oj < bj)) { best = ob; bj = oj; }
    }
    if (bj < c && bj % 64 == lane) taken |= uint64_t(1) << (bj / 64);
  }
  // ascending: round x covers candidates 64x .. 64x+63, one per lane
  int32_t* out = a.sel + row * p.topk;
  int pos = 0;
  for (int x = 0; 64 * x < c; x++) {
    const bool mine = (taken >> x) & 1;
    const uint64_t bal = __ballot(mine);
    if (mine) out[pos + __popcll(bal & ((uint64_t(1) << lane) - 1))] = 64 * x + lane;
    pos += __popcll(bal);
  }
  if (lane == 0) out[nh] = c;
  for (int x = nh + 1 + lane; x < p.topk; x += 64) out[x] = -1;
}

// ================================================================ attend
// GM: the group size rounded up to a power of two (sizes the LDS arrays, so
// small groups leave room for more resident work-groups).  near, first: full attention's
// order (see full_heads_near) and the launch's first eight chunks.
template <int GM>
__global__ __launch_bounds__(256) void decode_attend_kernel(DecodeArgs a, Problem p, bool near,
                                                            uint32_t first,
                                                            const SeqInfo* __restrict__ seqs) {
  __shared__ __attribute__((aligned(16))) uint32_t pw[GM][kDecodeChunk / 2];
  __shared__ float red[4][GM][2];
  // per-wave P V sums of each head (dims 2*lane, 2*lane+1)
  __shared__ __attribute__((aligned(16))) float2 accs[4][GM][64];
  __shared__ int use_head[GM];
  __shared__ unsigned long long umask[kMaxBlocksPerSeq / 64];
  __shared__ int ublock;
  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int G = p.G;
  int s, g, x;  // x: chunk id, block * nsub + piece
  if (a.full) {
    // the grid runs over every sequence's chunks
    const uint32_t c = near ? 8 * (first + blockIdx.y) + blockIdx.x % 8 : blockIdx.x;
    if (c >= (uint32_t)p.nblk_total) return;
    s = find_seq(seqs, p.S, c, [](const SeqInfo& y) { return y.blk_off; });
    g = (int)(near ? blockIdx.x / 8 : blockIdx.y);
    x = (int)c - seqs[s].blk_off;
  } else {
    s = blockIdx.y / p.Hkv;
    g = blockIdx.y % p.Hkv;
    // MoBA: the grid runs over the group's selected blocks only.  Work-group
    // slot blockIdx.x / nsub takes the slot-th smallest block any head of
    // the group selected: the selections as a bitmask (lane w: blocks
    // 64w .. 64w+63), a prefix count over the lanes, then the block.
    const int slot = blockIdx.x / a.nsub;
    if (tid < 64) umask[tid] = 0;
    __syncthreads();
    const int32_t* gs = a.sel + ((int64_t)s * p.Hq + (int64_t)g * G) * p.topk;
    for (int i = tid; i < G * p.topk; i += 256) {
      const int j = gs[i];
      if (j >= 0) atomicOr(&umask[j >> 6], 1ull << (j & 63));
    }
    __syncthreads();
    if (tid < 64) {
      const unsigned long long w = umask[tid];
      const int n = __popcll(w);
      int incl = n;
#pragma unroll
      for (int d = 1; d < 64; d <<= 1) {
        const int o = __shfl_up(incl, d, 64);
        if (lane >= d) incl += o;
      }
      if (slot >= incl - n && slot < incl) {
        unsigned long long r = w;
        for (int k = slot - (incl - n); k > 0; k--) r &= r - 1;
        ublock = 64 * tid + __ffsll((long long)r) - 1;
      }
      if (tid == 63 && slot >= incl) ublock = -1;  // fewer distinct blocks than slots
    }
    __syncthreads();
    const int j = ublock;
    if (j < 0) return;
    x = j * a.nsub + blockIdx.x % a.nsub;
  }
  const SeqInfo sq = seqs[s];
  int64_t u0, u1;
  chunk_range(x, a.nsub, a.chunk_block, sq.len, u0, u1);
  if (u0 >= u1) return;
  // heads of the group that attend this chunk
  if (tid < G) {
    const int h = g * G + tid;
    int use = 1;
    if (!a.full) {
      const int j = (int)(u0 / p.B);
      const int32_t* sl = a.sel + ((int64_t)s * p.Hq + h) * p.topk;
      use = 0;
      for (int y = 0; y < p.topk; y++) use |= sl[y] == j;
    }
    use_head[tid] = use;
  }
  __syncthreads();
  int any = 0;
  for (int hl = 0; hl < G; hl++) any |= use_head[hl];
  if (!any) return;

  // S: keys 64 wave .. + 63 in four 16-key tiles.  A operands: lane -> key row
  // lane % 16 of the tile, 16 bytes at dims 32 ks + 8 (lane / 16); rows past the
  // chunk end load the chunk's first row (their scores are discarded).  B
  // operands: head lane % 16 of the group, the same dims.
  const int kend = (int)min((int64_t)64, u1 - (u0 + 64 * wave));  // may be <= 0
  const int hc = lane & 15, kq = lane >> 4;
  bf16x8_t kf[4][4], qb[4];
  {
    const __hip_bfloat16* kp = a.k + (int64_t)g * a.k_sh + 8 * kq;
#pragma unroll
    for (int t = 0; t < 4; t++) {
      const int kl = 16 * t + hc;
      const __hip_bfloat16* row = kp + (sq.tok_start + u0 + (kl < kend ? 64 * wave + kl : 0)) * a.k_st;
#pragma unroll
      for (int ks = 0; ks < 4; ks++)
        kf[t][ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(row + 32 * ks));
    }
    const __hip_bfloat16* qp = a.q + (int64_t)s * a.q_ss +
                               (int64_t)(g * G + min(hc, G - 1)) * a.q_sh + 8 * kq;
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
      qb[ks] = __builtin_bit_cast(bf16x8_t, *reinterpret_cast<const u32x4_t*>(qp + 32 * ks));
  }
  // a lane's values: head hc, keys 16 t + 4 kq + i
  float z[16];
  float m = -INFINITY;
#pragma unroll
  for (int t = 0; t < 4; t++) {
    f32x4_t acc = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
    for (int ks = 0; ks < 4; ks++)
      acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[t][ks], qb[ks], acc, 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; i++) {
      z[4 * t + i] = 16 * t + 4 * kq + i < kend ? acc[i] * a.scale_log2 : -INFINITY;
      m = fmaxf(m, z[4 * t + i]);
    }
  }
  m = fmaxf(m, __shfl_xor(m, 16, 64));
  m = fmaxf(m, __shfl_xor(m, 32, 64));
  if (lane < G) red[wave][lane][0] = m;
  // this wave's 64 value rows, 16 lanes x 16 bytes per row and four rows per load
  // (keys 4 i + kq at dims 8 hc .. + 7), all in flight across the softmax below
  // (requested with the keys they would cost a quarter of the resident waves: 146 vs
  // 135 us in MoBA mode at 1M tokens); slots past the chunk end load the chunk's first
  // row, which exists, and get weight 0
  uint4 wv[16];
  {
    const __hip_bfloat16* vp = a.v + (sq.tok_start + u0) * a.v_st + (int64_t)g * a.v_sh + 8 * hc;
#pragma unroll
    for (int i = 0; i < 16; i++) {
      const int kl = 4 * i + kq;
      wv[i] = *reinterpret_cast<const uint4*>(vp + (int64_t)(kl < kend ? 64 * wave + kl : 0) * a.v_st);
    }
  }
  __syncthreads();
  // per head: chunk max, weights (keys 8 j + e and 8 j + 4 + e as one bf16 pair, word 4
  // j + e: the keys a lane holds in two value loads), sum
  if (hc < G) {
    m = fmaxf(fmaxf(red[0][hc][0], red[1][hc][0]), fmaxf(red[2][hc][0], red[3][hc][0]));
    float l = 0.0f;
#pragma unroll
    for (int t = 0; t < 4; t++) {
      float pv[4];
#pragma unroll
      for (int i = 0; i < 4; i++) {
        pv[i] = 16 * t + 4 * kq + i < kend ? __builtin_amdgcn_exp2f(z[4 * t + i] - m) : 0.0f;
        l += pv[i];
      }
      float po[4];  // the weights four keys on (or before)
#pragma unroll
      for (int i = 0; i < 4; i++) po[i] = __shfl_xor(pv[i], 16, 64);
      if ((kq & 1) == 0)
        *reinterpret_cast<uint4*>(&pw[hc][32 * wave + 4 * (2 * t + (kq >> 1))]) =
            make_uint4(pack_bf16(pv[0], po[0]), pack_bf16(pv[1], po[1]), pack_bf16(pv[2], po[2]),
                       pack_bf16(pv[3], po[3]));
    }
    l += __shfl_xor(l, 16, 64);  // (the four lanes of a head take this branch together)
    l += __shfl_xor(l, 32, 64);
    if (kq == 0) red[wave][hc][1] = l;
  }
  __syncthreads();
  // P V: a lane sums its keys of the wave's 64 for dims 8 hc .. + 7, a key pair per
  // dot2 (weights rounded once to bf16, fp32 accumulation; slots past the chunk end
  // carry weight 0); the four lanes of a dim group are added, kq order fixed.
  // Four heads at a time share the value pairs.
  for (int h0 = 0; h0 < GM; h0 += 4) {
    if (h0 >= G) break;
    constexpr int kH = GM < 4 ? GM : 4;
    float acc[kH][8];
#pragma unroll
    for (int e = 0; e < kH; e++)
#pragma unroll
      for (int d = 0; d < 8; d++) acc[e][d] = 0.0f;
#pragma unroll
    for (int j = 0; j < 8; j++) {
      const uint32_t lo[4] = {wv[2 * j].x, wv[2 * j].y, wv[2 * j].z, wv[2 * j].w};
      const uint32_t hi[4] = {wv[2 * j + 1].x, wv[2 * j + 1].y, wv[2 * j + 1].z, wv[2 * j + 1].w};
      bf16x2_t vv[8];
#pragma unroll
      for (int c = 0; c < 4; c++) {
        vv[2 * c] = as_bf16x2(__builtin_amdgcn_perm(hi[c], lo[c], 0x05040100u));
        vv[2 * c + 1] = as_bf16x2(__builtin_amdgcn_perm(hi[c], lo[c], 0x07060302u));
      }
#pragma unroll
      for (int e = 0; e < kH; e++) {
        const bf16x2_t pp = as_bf16x2(pw[h0 + e][32 * wave + 4 * j + kq]);
#pragma unroll
        for (int d = 0; d < 8; d++)
          acc[e][d] = __builtin_amdgcn_fdot2_f32_bf16(pp, vv[d], acc[e][d], false);
      }
    }
#pragma unroll
    for (int e = 0; e < kH; e++) {
#pragma unroll
      for (int d = 0; d < 8; d++) {
        acc[e][d] += __shfl_xor(acc[e][d], 16, 64);
        acc[e][d] += __shfl_xor(acc[e][d], 32, 64);
      }
      if (kq == 0 && h0 + e < G) {
        float4* dst = reinterpret_cast<float4*>(&accs[wave][h0 + e][4 * hc]);
        dst[0] = make_float4(acc[e][0], acc[e][1], acc[e][2], acc[e][3]);
        dst[1] = make_float4(acc[e][4], acc[e][5], acc[e][6], acc[e][7]);
      }
    }
  }
  __syncthreads();
  // normalised partial and lse per attending head; wave w handles heads w, w+4, ...
  for (int hl = wave; hl < G; hl += 4) {
    if (!use_head[hl]) continue;
    const float m = fmaxf(fmaxf(red[0][hl][0], red[1][hl][0]), fmaxf(red[2][hl][0], red[3][hl][0]));
    const float l = red[0][hl][1] + red[1][hl][1] + red[2][hl][1] + red[3][hl][1];
    const float inv = 1.0f / l;
    float2 o = accs[0][hl][lane];
#pragma unroll
    for (int w = 1; w < 4; w++) {
      o.x += accs[w][hl][lane].x;
      o.y += accs[w][hl][lane].y;
    }
    const int64_t pr = ((int64_t)s * p.Hq + g * G + hl) * a.nchunk + x;
    reinterpret_cast<float2*>(a.part_o + pr * kHeadDim)[lane] = make_float2(o.x * inv, o.y * inv);
    if (lane == 0) a.part_lse[pr] = (m + __builtin_amdgcn_logf(l)) * kLn2;
  }
}

// =============================================================== combine
// One work-group per row: 16 groups of 16 lanes each fold every 16th of the
// row's partials (8 dims per lane, online rescale), then the 16 group results
// are merged in group order.
__global__ __launch_bounds__(256) void decode_combine_kernel(DecodeArgs a, Problem p) {
  __shared__ float gm[16], gw[16];
  __shared__ float go[16][kHeadDim];
  const int64_t row = blockIdx.x / a.nsplit;  // s * Hq + h
  const int share = (int)(blockIdx.x % a.nsplit);
  const int xb = share * a.split_len;  // this work-group's partial slots start here
  const int grp = threadIdx.x / 16, l16 = threadIdx.x % 16;
  const int s = (int)(row / p.Hq), h = (int)(row % p.Hq);
  const SeqInfo sq = a.seqs[s];
  float M = -INFINITY, wsum = 0.0f, acc[8];
#pragma unroll
  for (int d = 0; d < 8; d++) acc[d] = 0.0f;
  auto fold_loaded = [&](float lv, float4 o0, float4 o1) {
    const float Mn = fmaxf(M, lv);
    const float sc = __builtin_amdgcn_exp2f((M - Mn) * kLog2e);
    const float w = __builtin_amdgcn_exp2f((lv - Mn) * kLog2e);
    const float f[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
    for (int d = 0; d < 8; d++) acc[d] = fmaf(w, f[d], acc[d] * sc);
    wsum = wsum * sc + w;
    M = Mn;
  };
  if (a.full) {
    // the group's partials x = grp + 16 i, eight loads in flight per round
    constexpr int kAhead = 8;
    const int n = min((int)((sq.len + kDecodeChunk - 1) / kDecodeChunk), xb + a.split_len);
    for (int x0 = xb + grp; x0 < n; x0 += 16 * kAhead) {
      float lv[kAhead];
      float4 o0[kAhead], o1[kAhead];
#pragma unroll
      for (int e = 0; e < kAhead; e++) {
        const int x = min(x0 + 16 * e, n - 1);
        const int64_t pr = row * a.nchunk + x;
        const float4* op = reinterpret_cast<const float4*>(a.part_o + pr * kHeadDim + 8 * l16);
        lv[e] = a.part_lse[pr];
        o0[e] = op[0];
        o1[e] = op[1];
      }
#pragma unroll
      for (int e = 0; e < kAhead; e++)
        if (x0 + 16 * e < n) fold_loaded(lv[e], o0[e], o1[e]);
    }
  } else {
    // the row's chunks: z = y * nsub + i for selection entry y, piece i;
    // the group's z = grp + 16 i, eight loads in flight per round
    constexpr int kAhead = 8;
    const int32_t* sl = a.sel + row * p.topk;
    const int zend = min(p.topk * a.nsub, xb + a.split_len);
    for (int z0 = xb + grp; z0 < zend; z0 += 16 * kAhead) {
      // selections, then partials, each without a branch so that all are in
      // flight (slots without a partial read the row's first one, unused)
      int js[kAhead];
#pragma unroll
      for (int e = 0; e < kAhead; e++) js[e] = sl[min(z0 + 16 * e, zend - 1) / a.nsub];
      float lv[kAhead];
      float4 o0[kAhead], o1[kAhead];
      bool ok[kAhead];
#pragma unroll
      for (int e = 0; e < kAhead; e++) {
        const int z = z0 + 16 * e, i = z % a.nsub, j = js[e];
        const int64_t u0 = (int64_t)j * p.B + (int64_t)i * kDecodeChunk;
        ok[e] = z < zend && j >= 0 && u0 < min((int64_t)(j + 1) * p.B, (int64_t)sq.len);
        const int64_t pr = row * a.nchunk + (ok[e] ? j * a.nsub + i : 0);
        const float4* op = reinterpret_cast<const float4*>(a.part_o + pr * kHeadDim + 8 * l16);
        lv[e] = a.part_lse[pr];
        o0[e] = op[0];
        o1[e] = op[1];
      }
#pragma unroll
      for (int e = 0; e < kAhead; e++)
        if (ok[e]) fold_loaded(lv[e], o0[e], o1[e]);
    }
  }
#pragma unroll
  for (int d = 0; d < 8; d++) go[grp][8 * l16 + d] = acc[d];
  if (l16 == 0) {
    gm[grp] = M;
    gw[grp] = wsum;
  }
  __syncthreads();
  if (threadIdx.x >= kHeadDim) return;
  const int d = threadIdx.x;
  float Mt = -INFINITY;
#pragma unroll
  for (int x = 0; x < 16; x++) Mt = fmaxf(Mt, gm[x]);
  float o = 0.0f, wt = 0.0f;
#pragma unroll
  for (int x = 0; x < 16; x++) {
    if (gw[x] == 0.0f) continue;  // a group without partials
    const float sc = __builtin_amdgcn_exp2f((gm[x] - Mt) * kLog2e);
    o = fmaf(sc, go[x][d], o);
    wt = fmaf(sc, gw[x], wt);
  }
  if (a.nsplit == 1) {
    a.out[(int64_t)s * a.o_ss + (int64_t)h * a.o_sh + d] = __float2bfloat16(o / wt);
    if (d == 0) a.lse[(int64_t)h * p.S + s] = Mt + __builtin_amdgcn_logf(wt) * kLn2;
    return;
  }
  // a share without partials leaves weight sum 0, which the second pass skips
  float* m = a.mid + (int64_t)blockIdx.x * (kHeadDim + 2);
  m[d] = o;
  if (d == 0) {
    m[kHeadDim] = Mt;
    m[kHeadDim + 1] = wt;
  }
}

// Second pass: one work-group per row folds its shares in order (every row
// has at least the partial of the chunk holding its own key).
__global__ __launch_bounds__(kHeadDim) void decode_fold_kernel(DecodeArgs a, Problem p) {
  static_assert(kCombineMaxSplit <= kHeadDim, "one thread per share loads its max and sum");
  __shared__ float sm[kCombineMaxSplit], sw[kCombineMaxSplit];
  const int64_t row = blockIdx.x;
  const int s = (int)(row / p.Hq), h = (int)(row % p.Hq);
  const int d = threadIdx.x;
  const float* m = a.mid + row * a.nsplit * (kHeadDim + 2);
  if (d < a.nsplit) {
    sm[d] = m[(int64_t)d * (kHeadDim + 2) + kHeadDim];
    sw[d] = m[(int64_t)d * (kHeadDim + 2) + kHeadDim + 1];
  }
  __syncthreads();
  float Mt = -INFINITY;
  for (int x = 0; x < a.nsplit; x++)
    if (sw[x] != 0.0f) Mt = fmaxf(Mt, sm[x]);
  // every share's value in flight at once (slots past the last share
  // re-read it and are not used)
  float v[kCombineMaxSplit];
#pragma unroll
  for (int x = 0; x < kCombineMaxSplit; x++)
    v[x] = m[(int64_t)min(x, a.nsplit - 1) * (kHeadDim + 2) + d];
  float o = 0.0f, wt = 0.0f;
#pragma unroll
  for (int x = 0; x < kCombineMaxSplit; x++) {
    if (x >= a.nsplit || sw[x] == 0.0f) continue;
    const float sc = __builtin_amdgcn_exp2f((sm[x] - Mt) * kLog2e);
    o = fmaf(sc, v[x], o);
    wt = fmaf(sc, sw[x], wt);
  }
  a.out[(int64_t)s * a.o_ss + (int64_t)h * a.o_sh + d] = __float2bfloat16(o / wt);
  if (d == 0) a.lse[(int64_t)h * p.S + s] = Mt + __builtin_amdgcn_logf(wt) * kLn2;
}

}  // namespace

hipError_t launch_decode_gate(const DecodeArgs& a, const Problem& p, hipStream_t st) {
  const int64_t rows = (int64_t)p.S * p.Hq;
  if (rows <= 0 || a.full) return hipSuccess;
  decode_gate_kernel<<<(unsigned)rows, 256, 0, st>>>(a, p, a.seqs);
  return hipGetLastError();
}

// Full attention: the kv-heads of eight chunks (one on each XCD) before the next eight.
// A token's rows of all kv-heads lie side by side, so memory, and each XCD's address
// translation, then go through the cache once; one kv-head after the other they go
// through it Hkv times.  Calls, one after the other -> this way: 1M tokens, 8 kv-heads 850 ->
// 802 us; 300K, 4 kv-heads 123 -> 118; 65536, 32 kv-heads 251 -> 187; 200 sequences of 130
// tokens, 32 kv-heads 105 -> 89.  A cache of up to about the 256 MB last-level cache, read
// again by the next call, was the faster one the other way: 127K tokens, 4 kv-heads (260 MB)
// 45.5 and 48.7; 65536, 8 kv-heads (268 MB) 49.1 and 51.4; 20000, 32 kv-heads (327 MB) 61.6
// and 60.7.  The line lies between (counted in whole chunks).
bool full_heads_near(const Problem& p) {
  constexpr int64_t kChunkBytes = 2 * 2 * kHeadDim * kDecodeChunk;
  return (int64_t)p.nblk_total * p.Hkv * kChunkBytes > (int64_t(300) << 20);
}

hipError_t launch_decode_attend(const DecodeArgs& a, const Problem& p, hipStream_t st) {
  if (p.S <= 0 || a.nchunk <= 0) return hipSuccess;
  const bool near = a.full && full_heads_near(p);
  const auto run = [&](dim3 grid, uint32_t first) {
    if (p.G <= 1) decode_attend_kernel<1><<<grid, 256, 0, st>>>(a, p, near, first, a.seqs);
    else if (p.G <= 2) decode_attend_kernel<2><<<grid, 256, 0, st>>>(a, p, near, first, a.seqs);
    else if (p.G <= 4) decode_attend_kernel<4><<<grid, 256, 0, st>>>(a, p, near, first, a.seqs);
    else if (p.G <= 8) decode_attend_kernel<8><<<grid, 256, 0, st>>>(a, p, near, first, a.seqs);
    else decode_attend_kernel<kDecodeMaxGroup><<<grid, 256, 0, st>>>(a, p, near, first, a.seqs);
  };
  // full: every sequence's chunks (the plan's blocks are chunks then); MoBA: slots
  if (near) {
    constexpr int64_t kMost = 65535;  // of a grid's second dimension
    const int64_t eights = ((int64_t)p.nblk_total + 7) / 8;
    for (int64_t first = 0; first < eights; first += kMost) {
      run(dim3(8 * (unsigned)p.Hkv, (unsigned)std::min(kMost, eights - first)), (uint32_t)first);
      const hipError_t e = hipGetLastError();
      if (e != hipSuccess) return e;
    }
    return hipSuccess;
  }
  run(a.full ? dim3((unsigned)p.nblk_total, (unsigned)p.Hkv)
             : dim3((unsigned)(a.nunion * a.nsub), (unsigned)(p.S * p.Hkv)), 0);
  return hipGetLastError();
}

hipError_t launch_decode_combine(const DecodeArgs& a, const Problem& p, hipStream_t st) {
  const int64_t rows = (int64_t)p.S * p.Hq;
  if (rows <= 0) return hipSuccess;
  decode_combine_kernel<<<(unsigned)(rows * a.nsplit), 256, 0, st>>>(a, p);
  if (a.nsplit == 1) return hipGetLastError();
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  decode_fold_kernel<<<(unsigned)rows, kHeadDim, 0, st>>>(a, p);
  return hipGetLastError();
}

}  // namespace moba
