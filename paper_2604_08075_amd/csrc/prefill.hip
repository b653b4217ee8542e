// Chunked-prefill attention over the block-paged KV cache, for gfx950.
//
// What it computes: each pool runs chunked prefill internally (Sec. 1.2): a
// long prompt is attended in fixed-size chunks (2,048 tokens by default)
// whose K and V are written into the paged cache first.  For sequence s with
// T = context_lens[s] cached tokens and n = q_start[s+1] - q_start[s] query
// tokens, query row r = q_start[s] + i sits at position p = T - n + i and
// attends causally over the cache:
//     out[r,h] = sum_{t <= p} softmax_t(scale * q[r,h] . K_t) V_t,  g = h / G,
// with K_t, V_t gathered through the block table exactly as for decode
// (token-major K tiles, dims-major V tiles, per-head fp8 scales).
//
// Unlike decode, a chunk reuses every K/V tile for many query rows, so the
// work is a dense contraction and belongs on the matrix cores.  The (token,
// head) pairs of one sequence and KV head form one list of columns, token by
// token, and an item is the next COLS of them, whatever the GQA group: no
// column of a full item is idle.  Workgroups are persistent and take items in
// turn, the ones with the most KV steps first.
//
// A workgroup's waves share the K and V of 32 tokens (a sub-tile, two blocks)
// through LDS; each wave owns 16 NC columns and keeps their queries and
// outputs in registers.  A wave computes up to the tile of its own last token
// and only takes part in the copies of the item's later steps.  Per step:
//   * S^T = K Q^T with v_mfma_f32_16x16x32_bf16 (rows: KV tokens, columns:
//     16 (token, head) pairs), the K rows read from LDS in a token order
//     chosen so that each lane's eight scores are the eight tokens its
//     operand of O^T += V^T P^T needs (no cross-lane movement of
//     probabilities);
//   * online softmax in base 2 (scale * log2 e folded into one fused
//     multiply-add in the exponent); the reference max of a column moves
//     only when a score passes it by 2^kSlack, so the common path has no
//     cross-lane reduction, no rescale and no branch;
//   * the denominator is one more product against ones: it sums the rounded
//     probabilities the output product uses.
// The three parts of a step belong to three tiles: the scores of tile j + 1,
// the probabilities of tile j and the output products of tile j - 1.  They
// do not depend on each other, and the code orders them by hand, a few vector
// instructions behind every matrix product (sched_barrier keeps the order):
// left to itself the compiler sinks the softmax to its use, one step later,
// and matrix and vector work take turns.
//
// What bounds it: power.  The card lowers its clock under this load (2.1 GHz
// of 2.4 on the four 2,048-token bf16 chunks at contexts of 2 K to 32 K), so
// energy per product counts as much as cycles.  On normal data a loop of
// nothing but 16x16x32 products reaches 1,996 TFLOP/s, one of 32x32x16
// products 1,825 (2,443 and 2,458 on zeros), so the 32x32 shape, which needs
// half the operand reads, still lost here: 1,120 TFLOP/s at 2.0 GHz.  Waves of
// 64 columns (four of them, half the LDS reads per product) came to 1,114 to
// 1,198: one wave on a SIMD has nothing to fill its own stalls with.  Measured,
// same card in turn, before (eight heads by 32 tokens an item; scores, softmax
// and output products of one tile in sequence) and now: the bf16 chunks 3.26
// -> 3.13 ms (1,184 TFLOP/s), four fp8 chunks at 2 K to 8 K 1.05 -> 0.95 ms,
// eleven fresh prompts of 179 to 3,372 tokens 471 -> 424 us, 381 tokens at
// context 20,861 571 -> 298 us, three prompts of up to 493 tokens with GQA 4
// 18.5 -> 13.3 us.
//
// LDS tiles: K rows are 320 bytes apart with 32 more in every second group of
// eight, V rows 64 with 32 after every eight, so that the sixteen lanes one
// pass of a 16-byte LDS read serves (0-3, 12-15, 20-23, 24-27 and the rest)
// start in distinct banks, and every operand is a constant away from one base.
// Tokens at or past T inside the last tile are zero in LDS (their V could be
// stale or poisoned; zero keeps 0 * V finite) and masked by causality.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <mutex>
#include <type_traits>

#include "common.h"

namespace dpool_prefill {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
typedef unsigned short u16x8 __attribute__((ext_vector_type(8)));

constexpr int kD = 128;
constexpr int kBS = 16;
constexpr int kKT = 32;               // KV tokens of a sub-tile: one wave's step
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kSlack = 8.0f;        // probabilities may reach 2^8 before the reference max moves
constexpr float kMinusBig = -3.0e38f; // the reference max of a column with no score yet (finite: no inf - inf)
constexpr int kMaxBatch = 4096;
constexpr int kIdCap = 4096;          // block ids staged in LDS: contexts up to 65,536 tokens
constexpr int kList = 64;             // rounds of items looked up at once
// LDS layout of a sub-tile (byte offsets; a chunk is 16 bytes)
constexpr int kKPitch = 320, kKSlot = 32 * kKPitch + 32;
constexpr int kVPitch = 64, kVSlot = 128 * kVPitch + 512;
__device__ __forceinline__ int kaddr(int row, int chunk) { return row * kKPitch + ((row >> 3) & 1) * 32 + chunk * 16; }
__device__ __forceinline__ int vaddr(int row, int chunk) { return row * kVPitch + (row >> 3) * 32 + chunk * 16; }

struct PrefillArgs {
  const uint16_t* q;            // [total_q, Hq, 128] bf16
  const char* k;                // [num_blocks, Hkv, 16, 128]
  const char* v;                // [num_blocks, Hkv, 128, 16]
  const int32_t* block_tables;  // [B, max_blocks_per_seq]
  const int32_t* context_lens;  // [B]
  const int32_t* q_start;       // [B + 1]
  const float* k_scale;
  const float* v_scale;
  void* out;                    // [total_q, Hq, 128] bf16 or fp32
  float scale_log2;             // scale * log2(e)
  int32_t batch, hq, hkv, group;
  int32_t max_blocks_per_seq, max_ctx, num_blocks_m1, out_fp32;
  int32_t total_q;
};

// Max over the four lanes li, li + 16, li + 32, li + 48
__device__ __forceinline__ float xor_max(float x) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto a = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  x = fmaxf(__builtin_bit_cast(float, (unsigned)a[0]), __builtin_bit_cast(float, (unsigned)a[1]));
  const unsigned v = __builtin_bit_cast(unsigned, x);
  const auto b = __builtin_amdgcn_permlane32_swap(v, v, false, false);
  return fmaxf(__builtin_bit_cast(float, (unsigned)b[0]), __builtin_bit_cast(float, (unsigned)b[1]));
}

// Inclusive prefix sum over the 64 lanes of a wave, in the vector ALU (no
// LDS round trips): data-parallel-primitive moves shift each 16-lane row
// right by 1, 2, 4 and 8 lanes (a lane with no source adds 0), then lane 15
// of rows 0 and 2 is added into rows 1 and 3, and lane 31 into rows 2 and 3.
__device__ __forceinline__ int wave_incl_scan(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
  return x;
}

// Largest of non-negative values over the 64 lanes, by the same moves.
__device__ __forceinline__ int wave_max(int x) {
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false));
  x = max(x, __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false));
  return __builtin_amdgcn_readlane(x, 63);
}

__device__ __forceinline__ i32x4 fp8x8_to_bf16(int lo, int hi) {
  bf16x2 a = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, false);
  bf16x2 b = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(lo, 1.0f, true);
  bf16x2 c = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, false);
  bf16x2 d = __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(hi, 1.0f, true);
  return i32x4{__builtin_bit_cast(int, a), __builtin_bit_cast(int, b), __builtin_bit_cast(int, c),
               __builtin_bit_cast(int, d)};
}

__device__ __forceinline__ i32x4 zero_tokens_from(i32x4 x, int first, int lim) {
#pragma unroll
  for (int wd = 0; wd < 4; ++wd) {
    unsigned m = 0;
    if (first + 2 * wd < lim) m |= 0xffffu;
    if (first + 2 * wd + 1 < lim) m |= 0xffff0000u;
    x[wd] &= (int)m;
  }
  return x;
}

__device__ __forceinline__ uint16_t f32_to_bf16_bits(float x) { return __builtin_bit_cast(uint16_t, (__bf16)x); }

__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// A workgroup of kWaves waves, each with NC blocks of 16 columns.  S: the
// waves are S to a column group and take turns at its sub-tiles; their sums
// are folded through LDS at the end of the item.
template <bool FP8, int kWaves, int NC, int S>
__global__ __launch_bounds__(kWaves * 64, 2) void prefill_kernel(PrefillArgs a) {
  constexpr int kThreads = kWaves * 64;
  constexpr int kWaveCols = 16 * NC;            // (token, head) columns of a wave
  constexpr int COLS = kWaveCols * kWaves / S;  // columns per item
  constexpr int ST = kKT * S;                   // tokens per step
  constexpr int NL = 8 / kWaves;                // pieces per thread of a sub-tile, K or V
  using Piece = std::conditional_t<FP8, i32x2, i32x4>;  // eight values
  struct Tiles {
    char k[2][S][kKSlot], v[2][S][kVSlot];
  };
  __shared__ __attribute__((aligned(16))) Tiles tiles;
  __shared__ int ids_lds[kIdCap];
  __shared__ int wsum[kWaves];
  __shared__ int list[kList][2];  // (sequence, tile) of this workgroup's next rounds
  __shared__ float first_max[kWaves / S][NC][16];  // S > 1: the columns' first reference maxima
  extern __shared__ int tile_pre[];  // [B + 1] items per KV head of sequences 0..s-1, then r0[B], r1[B], T[B]

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int w = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lj = lane >> 4;
  const int ks = w % S, cg = w / S;
  const int B = a.batch, G = a.group;
  int* const row0 = tile_pre + B + 1;
  int* const row1 = row0 + B;
  int* const ctx = row1 + B;

  if (tid == 0) tile_pre[0] = 0;
  for (int base = 0; base < B; base += kThreads) {
    __syncthreads();
    const int s = base + tid;
    int cnt = 0;
    if (s < B) {
      const int r0 = min(max(a.q_start[s], 0), a.total_q);
      const int r1 = min(max(a.q_start[s + 1], r0), a.total_q);
      const int T = min(max(a.context_lens[s], 0), a.max_ctx);
      cnt = (min(r1 - r0, T) * G + COLS - 1) / COLS;
      row0[s] = r0;
      row1[s] = r1;
      ctx[s] = T;
    }
    int incl = cnt;
    for (int off = 1; off < 64; off <<= 1) {
      const int v = __shfl_up(incl, off);
      if (lane >= off) incl += v;
    }
    if (lane == 63) wsum[w] = incl;
    __syncthreads();
    int carry = tile_pre[base];
    for (int k = 0; k < w; ++k) carry += wsum[k];
    if (s < B) tile_pre[s + 1] = carry + incl;
  }
  __syncthreads();
  const int total_tiles = tile_pre[B];
  const int per_tile = a.hkv;
  const int total_items = total_tiles * per_tile;

  // Copy geometry of a 32-token sub-tile: piece y of wave w is part
  // (w NL + y) % 4 of block (w NL + y) / 4 (4 tokens of K, 32 dims of V).
  constexpr int EB = FP8 ? 1 : 2;
  const int cb = w * NL >> 2, cp = w * NL & 3;
  const int koff_g = ((4 * cp + (lane >> 4)) * 128 + (lane & 15) * 8) * EB;  // + 512 EB y
  const int voff_g = ((32 * cp + (lane >> 1)) * 16 + (lane & 1) * 8) * EB;   // + 512 EB y
  const int kdst = kaddr(16 * cb + 4 * cp + (lane >> 4), lane & 15);         // + 4 kKPitch y
  const int vdst = vaddr(32 * cp + (lane >> 1), 2 * cb + (lane & 1));        // + (32 kVPitch + 128) y
  // LDS operand offsets.  K: row li of MFMA m is token 8 (li / 4) + 4 m + li % 4, dims 32 c + 8 lj .. + 8;
  // V: row li of MFMA nn is dim 32 (nn / 2) + 8 (li / 4) + 4 (nn % 2) + li % 4, tokens 8 lj .. + 8.
  const int kro = kaddr(8 * (li >> 2) + (li & 3), lj);
  const int vro = vaddr(8 * (li >> 2) + (li & 3), lj);

  // Tiles are handed out by the number of steps they take, most first: round
  // r hands the next gridDim.x items of that order out forwards (r even) or
  // backwards (r odd), so every workgroup's items sum to about the same work.
  // A workgroup's tiles of up to kList rounds are found at once, each by one
  // wave.  Up to 64 sequences (one a lane): the tile of rank k by a search for
  // the step count that just over k tiles exceed.  With more, the tiles are
  // numbered from the end of the batch backwards, and the sums even out with
  // their number only (replayed on the CPU for fresh prompts of median 600
  // tokens on 32/4 heads, the busiest workgroup is 19% above the mean at 65
  // sequences, 13% at 100, 6% at 400; 1% were they ranked).
  const int nwg = gridDim.x, wg = blockIdx.x;
  auto item_of = [&](int round) __attribute__((always_inline)) {
    return round * nwg + ((round & 1) ? nwg - 1 - wg : wg);
  };
  auto fill_list = [&](int round0) __attribute__((always_inline)) {
    int cnt = 0, n = 0, pre = 0;
    if (lane < B) {
      cnt = tile_pre[lane + 1] - tile_pre[lane];
      n = min(row1[lane] - row0[lane], ctx[lane]);
      pre = ctx[lane] - n;
    }
    const int t_max = (wave_max(pre + n) + kKT - 1) / kKT;  // no tile takes more steps
    auto above = [&](int t) __attribute__((always_inline)) {  // this lane's tiles that attend more than 32 t tokens
      const int x = kKT * t - pre;  // the tile's last token reaches index x of the chunk
      return x <= 0 ? cnt : x > n - 1 ? 0 : cnt - x * G / COLS;
    };
    for (int r = w; r < kList && (round0 + r) * nwg < total_items; r += kWaves) {
      const int item = item_of(round0 + r);
      if (item >= total_items) continue;
      const int k = item / per_tile;
      int s, q;
      if (B > 64) {
        const int idx = total_tiles - 1 - k;
        int lo = 0, hi = B - 1;  // largest s with tile_pre[s] <= idx
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (tile_pre[mid] <= idx) lo = mid;
          else hi = mid - 1;
        }
        s = lo;
        q = idx - tile_pre[lo];
      } else {
        int lo = 0, hi = t_max;  // largest t that more than k tiles exceed
        while (lo < hi) {
          const int mid = (lo + hi + 1) >> 1;
          if (__builtin_amdgcn_readlane(wave_incl_scan(above(mid)), 63) > k) lo = mid;
          else hi = mid - 1;
        }
        const int more = above(lo + 1), d = above(lo) - more;  // d: this lane's tiles of lo + 1 steps
        const int rank = k - __builtin_amdgcn_readlane(wave_incl_scan(more), 63);  // among all of those
        const int incl = wave_incl_scan(d);
        s = __ffsll(__ballot(incl > rank)) - 1;
        q = __builtin_amdgcn_readlane(cnt - more - incl, s) + rank;
      }
      if (lane == 0) {
        list[r][0] = s;
        list[r][1] = q;
      }
    }
  };
  for (int round = 0; round * nwg < total_items; ++round) {
    const int r = round % kList;
    if (r == 0) {
      lds_barrier();  // the previous list is done with
      fill_list(round);
    }
    const int item = item_of(round);
    if (item >= total_items) continue;  // uniform over the workgroup
    __syncthreads();  // the list is complete; the previous item's LDS is done with
    const int g = item % per_tile;
    const int s = __builtin_amdgcn_readfirstlane(list[r][0]);
    const int qt = __builtin_amdgcn_readfirstlane(list[r][1]);
    const int r0 = __builtin_amdgcn_readfirstlane(row0[s]);
    const int T = __builtin_amdgcn_readfirstlane(ctx[s]);
    const int n = min(__builtin_amdgcn_readfirstlane(row1[s]) - r0, T);
    const int ncols = n * G;
    const int c0 = qt * COLS;
    const int tok_last = (min(c0 + COLS, ncols) - 1) / G;
    const int n_kv = T - n + tok_last + 1;
    const int nt = (n_kv + ST - 1) / ST;
    const int nb = (T + kBS - 1) / kBS;
    const int32_t* bt = a.block_tables + (size_t)s * a.max_blocks_per_seq;
    const int pmin = T - n + min(c0 + cg * kWaveCols, ncols - 1) / G;  // first position of this wave's columns
    // Steps this wave computes: up to the sub-tile of its own last position,
    // not of the item's, and none without a column.  Past them every one of
    // its probabilities is 0, and 0 times a value that is not finite is not.
    const int p_end = T - n + (min(c0 + (cg + 1) * kWaveCols, ncols) - 1) / G;
    const int nt_w = c0 + cg * kWaveCols >= ncols || p_end < kKT * ks ? 0 : (p_end - kKT * ks) / ST + 1;

    float cmul = a.scale_log2, vsc = 1.0f;
    if constexpr (FP8) {
      cmul *= a.k_scale[g];
      vsc = a.v_scale[g];
    }
    const int n_ids = min(min(2 * S * nt, nb), kIdCap);
    const int id0 = bt[min(tid, n_ids - 1)];  // the first ids' loads go out before the queries'
    // token of the chunk and row (token, head) of this lane's column in block b; idle columns repeat the last one
    auto column = [&](int b, int& tok, size_t& row) __attribute__((always_inline)) {
      const int cc = min(c0 + cg * kWaveCols + 16 * b + li, ncols - 1);
      tok = cc / G;
      row = (size_t)(r0 + tok) * a.hq + (g * G + (cc - tok * G));
    };
    int pcol[NC];  // position of this lane's columns
    i32x4 qf[NC][4];
#pragma unroll
    for (int b = 0; b < NC; ++b) {
      int tok;
      size_t row;
      column(b, tok, row);
      pcol[b] = T - n + tok;
      const uint16_t* qp = a.q + row * kD + 8 * lj;
#pragma unroll
      for (int c = 0; c < 4; ++c) qf[b][c] = *(const i32x4*)(qp + 32 * c);
    }
    if (tid < n_ids) ids_lds[tid] = min(max(id0, 0), a.num_blocks_m1);
    for (int i = tid + kThreads; i < n_ids; i += kThreads) ids_lds[i] = min(max(bt[i], 0), a.num_blocks_m1);
    lds_barrier();

    constexpr int TB = FP8 ? 2048 : 4096;
    struct Ids { int x[S]; };
    struct Chunk { Piece x[S * NL]; };
    auto read_ids = [&](int j, Ids& id) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < S; ++x) id.x[x] = ids_lds[min(2 * (S * j + x) + cb, n_ids - 1)];
    };
    auto bases = [&](const Ids& id, Ids& t) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < S; ++x) t.x[x] = __builtin_amdgcn_readfirstlane(id.x[x]) * a.hkv + g;
    };
    auto load = [&](const char* base, int off, const Ids& t, Chunk& r) __attribute__((always_inline)) {
#pragma unroll
      for (int x = 0; x < S; ++x) {
        const char* p = base + (size_t)t.x[x] * TB + off;
#pragma unroll
        for (int y = 0; y < NL; ++y) r.x[x * NL + y] = *(const Piece*)(p + 512 * EB * y);
      }
    };
    auto widen = [&](const Piece& p) __attribute__((always_inline)) {
      if constexpr (FP8) return fp8x8_to_bf16(p[0], p[1]);
      else return p;
    };
    auto store_k = [&](int slot, int x, const Chunk& r) __attribute__((always_inline)) {
      *(i32x4*)(tiles.k[slot][x / NL] + kdst + 4 * kKPitch * (x % NL)) = widen(r.x[x]);
    };
    auto store_v = [&](int slot, int x, const Chunk& r) __attribute__((always_inline)) {
      *(i32x4*)(tiles.v[slot][x / NL] + vdst + (32 * kVPitch + 128) * (x % NL)) = widen(r.x[x]);
    };
    // zero the tokens of V tile j past the sequence's end
    auto clip_v = [&](int j, Chunk& r) __attribute__((always_inline)) {
      if (ST * j + ST > T) {
#pragma unroll
        for (int x = 0; x < S * NL; ++x) {
          const int t0 = ST * j + kKT * (x / NL) + 16 * cb + 8 * (lane & 1);
          if constexpr (FP8) {
#pragma unroll
            for (int wd = 0; wd < 2; ++wd) {
              const int k = min(max(T - t0 - 4 * wd, 0), 4);
              r.x[x][wd] &= k == 4 ? -1 : (1 << (8 * k)) - 1;
            }
          } else {
            r.x[x] = zero_tokens_from(r.x[x], t0, T);
          }
        }
      }
    };

    f32x4 acc[NC][8];
    f32x4 lsum[NC];  // column sums of the rounded probabilities
    float mc[NC], mlim[NC], lmax[NC], over = 0.f;  // scaled reference max; the scaled score that moves it
#pragma unroll
    for (int b = 0; b < NC; ++b) {
      mc[b] = kMinusBig;
      mlim[b] = kMinusBig;
      lsum[b] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int nn = 0; nn < 8; ++nn) acc[b][nn] = f32x4{0.f, 0.f, 0.f, 0.f};
    }
    bf16x8 ones;
#pragma unroll
    for (int x = 0; x < 8; ++x) ones[x] = (__bf16)1.0f;

    // K tiles 0 and 1 to LDS; K tiles 2, 3 and V tiles 0, 1 in registers
    Chunk kA, vA, kB, vB;
    Ids idn, tb[2];  // ids of K tile j + 4; bases of tiles j + 2, j + 3
    {
      Ids id[5], t[4];
#pragma unroll
      for (int x = 0; x < 5; ++x) read_ids(x, id[x]);
#pragma unroll
      for (int x = 0; x < 4; ++x) bases(id[x], t[x]);
      idn = id[4];
      tb[0] = t[2];
      tb[1] = t[3];
      Chunk k0, k1;
      load(a.k, koff_g, t[0], k0);
      load(a.k, koff_g, t[1], k1);
      load(a.k, koff_g, t[2], kA);
      load(a.v, voff_g, t[0], vA);
      load(a.k, koff_g, t[3], kB);
      load(a.v, voff_g, t[1], vB);
#pragma unroll
      for (int y = 0; y < S * NL; ++y) {
        store_k(0, y, k0);
        store_k(1, y, k1);
        store_v(1, y, Chunk{});  // V tile -1, which step 0 multiplies by zero
      }
    }

    auto kfrag = [&](int slot, int f) __attribute__((always_inline)) {  // f = 4 m + c
      return *(const i32x4*)(tiles.k[slot][ks] + kro + 4 * kKPitch * (f >> 2) + 64 * (f & 3));
    };
    auto vfrag = [&](int slot, int nn) __attribute__((always_inline)) {
      return *(const i32x4*)(tiles.v[slot][ks] + vro + (32 * kVPitch + 128) * (nn >> 1) + 4 * kVPitch * (nn & 1));
    };
    struct Scores { f32x4 z[NC][2]; };       // [column block][m]: tokens 8 lj + 4 m + e
    struct Probs { i32x4 p[NC]; };
    // S^T += K Q^T: row group and 32-dim chunk f, column block b
    auto qkmm = [&](Scores& sc, const i32x4& kf, int f, int b) __attribute__((always_inline)) {
      sc.z[b][f >> 2] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
          __builtin_bit_cast(bf16x8, kf), __builtin_bit_cast(bf16x8, qf[b][f & 3]),
          (f & 3) == 0 ? f32x4{0.f, 0.f, 0.f, 0.f} : sc.z[b][f >> 2], 0, 0, 0);
    };
    auto pvmm = [&](const i32x4& vf, const Probs& pp, int nn, int b) __attribute__((always_inline)) {
      acc[b][nn] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, vf),
                                                           __builtin_bit_cast(bf16x8, pp.p[b]), acc[b][nn], 0, 0, 0);
    };
    auto summm = [&](const Probs& pp, int b) __attribute__((always_inline)) {
      lsum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, __builtin_bit_cast(bf16x8, pp.p[b]), lsum[b], 0, 0, 0);
    };
    // maximum of a column's scores, four at a time: y = 0 .. 3
    auto colmax = [&](const Scores& sc, int b, int y) __attribute__((always_inline)) {
      const float u = sc.z[b][y >> 1][2 * (y & 1)], v = sc.z[b][y >> 1][2 * (y & 1) + 1];
      lmax[b] = y == 0 ? fmaxf(u, v) : fmaxf(fmaxf(lmax[b], u), v);
    };
    // > 0 if some column's score would raise its probability above 2^kSlack
    auto excess = [&]() __attribute__((always_inline)) {
      over = __builtin_fmaf(lmax[0], cmul, -mlim[0]);
#pragma unroll
      for (int b = 1; b < NC; ++b) over = fmaxf(over, __builtin_fmaf(lmax[b], cmul, -mlim[b]));
    };
    float alpha[NC];
#pragma unroll
    for (int b = 0; b < NC; ++b) alpha[b] = 1.0f;
    // the rare work ahead of step j: causal masking, and moving the reference
    // maxima; true if the sums so far must be rescaled by alpha
    auto prepare = [&](int j, Scores& sc) __attribute__((always_inline)) {
      const int t0 = ST * j + kKT * ks;
      if (t0 + kKT - 1 > pmin) {
#pragma unroll
        for (int b = 0; b < NC; ++b) {
#pragma unroll
          for (int x = 0; x < 8; ++x)
            if (t0 + 8 * lj + x > pcol[b]) sc.z[b][x >> 2][x & 3] = -INFINITY;
#pragma unroll
          for (int y = 0; y < 4; ++y) colmax(sc, b, y);
        }
        excess();
      }
      if (__builtin_amdgcn_ballot_w64(over > 0.f) == 0) return false;
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        const float m_new = fmaxf(mc[b], xor_max(lmax[b]) * cmul);
        const bool up = m_new > mlim[b];
        alpha[b] = up ? __builtin_amdgcn_exp2f(mc[b] - m_new) : 1.0f;
        if (up) {
          mc[b] = m_new;
          mlim[b] = m_new + kSlack;
        }
      }
      return true;
    };
    auto rescale = [&]() __attribute__((always_inline)) {
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        lsum[b] *= alpha[b];
#pragma unroll
        for (int nn = 0; nn < 8; ++nn) acc[b][nn] *= alpha[b];
      }
    };

    lds_barrier();
    Scores sA, sB;
    i32x4 kf[8], vf[8];
#pragma unroll
    for (int f = 0; f < 8; ++f) kf[f] = kfrag(0, f);
#pragma unroll
    for (int f = 0; f < 8; ++f)
#pragma unroll
      for (int b = 0; b < NC; ++b) qkmm(sA, kf[f], f, b);
#pragma unroll
    for (int b = 0; b < NC; ++b)
#pragma unroll
      for (int y = 0; y < 4; ++y) colmax(sA, b, y);
    excess();
    // Both waves of a pair start from the reference maxima of the first 32
    // tokens, so that a column's probabilities are rounded as in the variants
    // without pairs: the variant changes the order of sums only.
    if (S > 1 && ks == 0) {
      prepare(0, sA);
      if (lj == 0)
#pragma unroll
        for (int b = 0; b < NC; ++b) first_max[cg][b][li] = mc[b];
    }
    lds_barrier();  // K tile 0 is read before tile 2 takes its place
    if (S > 1 && ks > 0) {
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        mc[b] = first_max[cg][b][li];
        mlim[b] = mc[b] + kSlack;
      }
    }
    if constexpr (S > 1) excess();

    Probs pA, pB;
#pragma unroll
    for (int b = 0; b < NC; ++b) pB.p[b] = i32x4{0, 0, 0, 0};
    // first step with a token past some column's position in its scores, or
    // past the sequence's end in the V tile it writes
    const int j_rare = min((pmin + 1 - kKT * ks) / ST, T / ST);
    // One step: scores of tile j+1, output products of tile j-1 and
    // probabilities of tile j, independent of one another, in sixteen slots
    // of four matrix products each.
    auto step = [&](int j, int par, Scores& cur, Scores& nxt, Probs& pn, Probs& pp, Chunk& kr, Chunk& vr)
                    __attribute__((always_inline)) {
#pragma unroll
      for (int f = 0; f < 4; ++f) kf[f] = kfrag(par ^ 1, f);
      bool grown = false;
      if (j >= j_rare || __builtin_amdgcn_ballot_w64(over > 0.f) != 0) {
        grown = prepare(j, cur);
        clip_v(j, vr);
      }
      Ids t4;
      float z0 = __builtin_fmaf(cur.z[0][0][0], cmul, -mc[0]), z1 = __builtin_fmaf(cur.z[0][0][1], cmul, -mc[0]);
      float e0 = 0.f, e1 = 0.f;
      auto round_pair = [&](int y, float u0, float u1) __attribute__((always_inline)) {
        const bf16x2 p2 = {(__bf16)u0, (__bf16)u1};
        int v = __builtin_bit_cast(int, p2);
        asm volatile("" : "+v"(v));
        pn.p[y >> 2][y & 3] = v;
      };
      float x0 = 0.f, x1 = 0.f;
      // Work between the matrix products of a slot: gap(i, b) follows product
      // b.  A product occupies the matrix core for four issue cycles; one
      // exponential or two other vector instructions fit behind it without
      // delaying the next.
      auto gap = [&](int i, int b) __attribute__((always_inline)) {
        // probabilities, three stages apart so that no instruction waits for
        // the one before it: exponentials of pair y, rounding of pair y - 1,
        // scaled scores of pair y + 1
        const int u = i * NC + b, y = u >> 2, part = u & 3;
        constexpr int NP = 4 * NC;  // pairs
        const int nb_ = (y + 1) >> 2, nm = ((y + 1) >> 1) & 1, ne = 2 * ((y + 1) & 1);
        if (part == 0) {
          x0 = __builtin_amdgcn_exp2f(z0);
          asm volatile("" : "+v"(x0));
        } else if (part == 1) {
          x1 = __builtin_amdgcn_exp2f(z1);
          asm volatile("" : "+v"(x1));
        } else if (part == 2) {
          if (y > 0) round_pair(y - 1, e0, e1);
          if (y < NP - 1) {
            z0 = __builtin_fmaf(cur.z[nb_][nm][ne], cmul, -mc[nb_]);
            asm volatile("" : "+v"(z0));
          }
        } else {
          if (y < NP - 1) {
            z1 = __builtin_fmaf(cur.z[nb_][nm][ne + 1], cmul, -mc[nb_]);
            asm volatile("" : "+v"(z1));
          }
          e0 = x0;
          e1 = x1;
        }
        // operand reads, four slots ahead
        if (b == NC - 1) {
          if (i < 4) kf[i + 4] = kfrag(par ^ 1, i + 4);
          else if (i < 12) vf[i - 4] = vfrag(par ^ 1, i - 4);
        }
        // column maxima of the next scores, well after the products that made them
#pragma unroll
        for (int c = 0; c < 4 * NC; ++c)
          if (i == 6 + c * 2 / NC && b == 0) {
            colmax(nxt, c % NC, c / NC);
            asm volatile("" : "+v"(lmax[c % NC]));
          }
        // copies: K tile j + 2 and V tile j to LDS; the loads of K tile j + 4 and V tile j + 2
        constexpr int NS = S * NL;
        if (b == NC / 2) {
          if (i == 0) bases(idn, t4);
          if (i < NS) store_k(par, i, kr);
          else if (i < 2 * NS) store_v(par, i - NS, vr);
          else if (i == 2 * NS) load(a.k, koff_g, t4, kr);
          else if (i == 2 * NS + 1) load(a.v, voff_g, tb[0], vr);
          else if (i == 10) {
            tb[0] = tb[1];
            tb[1] = t4;
            read_ids(j + 5, idn);
          }
        }
        if (i == 15 && b == NC - 1) {
          round_pair(NP - 1, e0, e1);
          excess();
          asm volatile("" : "+v"(over));
        }
        __builtin_amdgcn_sched_barrier(0);
      };
#pragma unroll
      for (int i = 0; i < 16; ++i) {
#pragma unroll
        for (int b = 0; b < NC; ++b) {
          if (i < 8) qkmm(nxt, kf[i], i, b);
          else pvmm(vf[i - 8], pp, i - 8, b);
          if (i >= 8 && (i & 1) && ((i - 8) >> 1) < NC && b == NC - 1) summm(pp, (i - 8) >> 1);
          gap(i, b);
        }
      }
      if (grown) rescale();
      // every wave's copies are in LDS, and its operands of this step are read
      lds_barrier();
      __builtin_amdgcn_sched_barrier(0);
    };
    int j = 0;
    for (; j + 1 < nt_w; j += 2) {
      step(j, 0, sA, sB, pA, pB, kA, vA);
      step(j + 1, 1, sB, sA, pB, pA, kB, vB);
    }
    if (j < nt_w) {
      step(j, 0, sA, sB, pA, pB, kA, vA);
#pragma unroll
      for (int b = 0; b < NC; ++b) pB.p[b] = pA.p[b];
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) vf[i] = (nt_w & 1) ? vfrag(0, i) : vfrag(1, i);
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
      for (int b = 0; b < NC; ++b) pvmm(vf[i], pB, i, b);
#pragma unroll
    for (int b = 0; b < NC; ++b) summm(pB, b);

    // the item's remaining steps: only this wave's part of the copies, for the
    // waves that still compute (its last V tile, read above, lies in the slot
    // that step nt_w leaves alone)
    auto copy_step = [&](int j, int par, Chunk& kr, Chunk& vr) __attribute__((always_inline)) {
      Ids t4;
      bases(idn, t4);
      clip_v(j, vr);
#pragma unroll
      for (int x = 0; x < S * NL; ++x) {
        store_k(par, x, kr);
        store_v(par, x, vr);
      }
      load(a.k, koff_g, t4, kr);
      load(a.v, voff_g, tb[0], vr);
      tb[0] = tb[1];
      tb[1] = t4;
      read_ids(j + 5, idn);
      lds_barrier();
    };
    j = nt_w;
    if (j < nt) {
      // The loads in flight are waited for here, once: which register set was
      // loaded last depends on the parity of nt_w, and without this the
      // compiler would wait for every load in every step below.
      __builtin_amdgcn_s_waitcnt(0xf70);  // vmcnt(0)
      if (j & 1) copy_step(j++, 1, kB, vB);
      for (; j + 1 < nt; j += 2) {
        copy_step(j, 0, kA, vA);
        copy_step(j + 1, 1, kB, vB);
      }
      if (j < nt) copy_step(j, 0, kA, vA);
    }

    // This lane holds dims 32 (nn / 2) + 8 lj + 4 (nn % 2) + e of its columns.
    // Idle columns are not stored: the last column's own lane writes its row.
    auto store_row = [&](int b, int n0, auto n_c, float inv, auto at) __attribute__((always_inline)) {
      constexpr int N = decltype(n_c)::value;
      if (c0 + cg * kWaveCols + 16 * b + li >= ncols) return;
      int tok;
      size_t row;
      column(b, tok, row);
      const size_t off = row * kD + 8 * lj + 16 * n0;
      if (a.out_fp32) {
#pragma unroll
        for (int nn = 0; nn < N; ++nn) *(f32x4*)((float*)a.out + off + 32 * (nn >> 1) + 4 * (nn & 1)) = at(nn) * inv;
      } else {
#pragma unroll
        for (int nn = 0; nn < N; nn += 2) {
          const f32x4 x = at(nn) * inv, y = at(nn + 1) * inv;
          u16x8 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            o[e] = f32_to_bf16_bits(x[e]);
            o[4 + e] = f32_to_bf16_bits(y[e]);
          }
          *(u16x8*)((uint16_t*)a.out + off + 16 * nn) = o;
        }
      }
    };
    if constexpr (S == 1) {
#pragma unroll
      for (int b = 0; b < NC; ++b)
        store_row(b, 0, std::integral_constant<int, 8>{}, vsc / lsum[b][0],
                    [&](int nn) __attribute__((always_inline)) { return acc[b][nn]; });
    } else {
      // Fold the two halves of the KV range: each wave of a pair hands the
      // other half of its dims over through LDS and finishes its own.
      static_assert(S == 2, "pairs of waves");
      auto pick = [&](f32x4 u, f32x4 v) __attribute__((always_inline)) {  // u for the first wave of a pair, else v
        f32x4 r;
#pragma unroll
        for (int e = 0; e < 4; ++e) r[e] = ks == 0 ? u[e] : v[e];
        return r;
      };
      lds_barrier();  // every wave is done with the tiles
      f32x4* const part = (f32x4*)&tiles;                      // [wave][b][4][lane]
      float* const ml = (float*)(part + kWaves * NC * 4 * 64);  // [wave][b][lane][2]
      static_assert(kWaves * NC * 64 * (4 * 16 + 8) <= (int)sizeof(Tiles), "partials fit over the tiles");
#pragma unroll
      for (int b = 0; b < NC; ++b) {
#pragma unroll
        for (int nn = 0; nn < 4; ++nn)
          part[((w * NC + b) * 4 + nn) * 64 + lane] = pick(acc[b][4 + nn], acc[b][nn]);
        ml[((w * NC + b) * 64 + lane) * 2] = mc[b];
        ml[((w * NC + b) * 64 + lane) * 2 + 1] = lsum[b][0];
      }
      lds_barrier();
      const int ow = w ^ 1;
#pragma unroll
      for (int b = 0; b < NC; ++b) {
        const float om = ml[((ow * NC + b) * 64 + lane) * 2], ol = ml[((ow * NC + b) * 64 + lane) * 2 + 1];
        const float mx = fmaxf(mc[b], om);
        const float w0 = __builtin_amdgcn_exp2f(mc[b] - mx), w1 = __builtin_amdgcn_exp2f(om - mx);
        const float inv = vsc / __builtin_fmaf(ol, w1, lsum[b][0] * w0);
        store_row(b, 4 * ks, std::integral_constant<int, 4>{}, inv, [&](int nn) __attribute__((always_inline)) {
            const f32x4 x = part[((ow * NC + b) * 4 + nn) * 64 + lane];
            const f32x4 y = pick(acc[b][nn], acc[b][4 + nn]);
            f32x4 r;
#pragma unroll
            for (int e = 0; e < 4; ++e) r[e] = __builtin_fmaf(x[e], w1, y[e] * w0);
            return r;
          });
      }
    }
  }
}

}  // namespace dpool_prefill

using namespace dpool_prefill;

namespace {

// Compute units of the current device (cached per device); 256 without one.
int compute_units() {
  static std::mutex mu;
  static int cached[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) {
    (void)hipGetLastError();
    return 256;
  }
  std::lock_guard<std::mutex> lock(mu);
  if (!cached[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) {
      (void)hipGetLastError();
      n = 256;
    }
    cached[dev] = n;
  }
  return cached[dev];
}

// Enqueue one variant: as many persistent workgroups as the device holds, or
// one per item (an upper bound; the kernel counts them exactly).
template <int kWaves, int NC, int S>
void launch(const PrefillArgs& a, bool fp8, int64_t workgroups, hipStream_t st) {
  constexpr int cols = 16 * NC * kWaves / S;
  const int64_t items = (((int64_t)a.total_q * a.group + cols - 1) / cols + a.batch) * a.hkv;
  const dim3 grid((unsigned)std::min(items, workgroups)), block(kWaves * 64);
  const size_t dyn = (size_t)(4 * a.batch + 1) * sizeof(int);  // tile prefix, rows, contexts
  if (fp8) hipLaunchKernelGGL((prefill_kernel<true, kWaves, NC, S>), grid, block, dyn, st, a);
  else hipLaunchKernelGGL((prefill_kernel<false, kWaves, NC, S>), grid, block, dyn, st, a);
}

}  // namespace

extern "C" int chunked_prefill_attention(const void* q, const void* k_blocks, const void* v_blocks,
                                         const int32_t* block_tables, const int32_t* context_lens,
                                         const int32_t* q_start, float scale, const float* k_scale,
                                         const float* v_scale, void* out, const dp_prefill_shape* sh, void* stream) {
  using dpool::fail;
  if (!sh) return fail(DP_EINVAL, "chunked_prefill_attention: null shape");
  if (sh->head_dim != kD) return fail(DP_ENOTSUP, "chunked_prefill_attention: head_dim %d (only 128)", sh->head_dim);
  if (sh->block_size != kBS)
    return fail(DP_ENOTSUP, "chunked_prefill_attention: block_size %d (only 16)", sh->block_size);
  if (sh->kv_dtype != DP_KV_BF16 && sh->kv_dtype != DP_KV_FP8_E4M3)
    return fail(DP_ENOTSUP, "chunked_prefill_attention: kv_dtype %d", sh->kv_dtype);
  if (sh->out_dtype != DP_OUT_BF16 && sh->out_dtype != DP_OUT_FP32)
    return fail(DP_ENOTSUP, "chunked_prefill_attention: out_dtype %d", sh->out_dtype);
  if (sh->query_tile != 0 && sh->query_tile != 32)
    return fail(DP_EINVAL, "chunked_prefill_attention: query_tile must be 0 or 32");
  if (sh->reserved != 0) return fail(DP_EINVAL, "chunked_prefill_attention: reserved must be 0");
  if (sh->batch < 0) return fail(DP_EINVAL, "chunked_prefill_attention: batch < 0");
  if (sh->batch > kMaxBatch) return fail(DP_ENOTSUP, "chunked_prefill_attention: batch above 4096");
  if (sh->n_kv_heads <= 0 || sh->n_q_heads <= 0 || sh->n_q_heads % sh->n_kv_heads != 0)
    return fail(DP_EINVAL, "chunked_prefill_attention: n_q_heads must be a positive multiple of n_kv_heads");
  if (sh->max_blocks_per_seq <= 0 || sh->max_context_len < 0 ||
      (int64_t)sh->max_blocks_per_seq * kBS < sh->max_context_len || sh->num_blocks <= 0 ||
      sh->num_blocks > INT32_MAX)
    return fail(DP_EINVAL, "chunked_prefill_attention: need max_blocks_per_seq * 16 >= max_context_len and "
                           "0 < num_blocks <= INT32_MAX");
  if (sh->max_context_len > kIdCap * kBS)
    return fail(DP_ENOTSUP, "chunked_prefill_attention: max_context_len above %d", kIdCap * kBS);
  if (sh->total_q < 0 || sh->total_q > INT32_MAX / 2)
    return fail(DP_EINVAL, "chunked_prefill_attention: total_q out of range");
  if (sh->batch == 0 || sh->total_q == 0) return DP_OK;
  if (!q || !k_blocks || !v_blocks || !block_tables || !context_lens || !q_start || !out)
    return fail(DP_EINVAL, "chunked_prefill_attention: null tensor pointer");
  if (((uintptr_t)q | (uintptr_t)k_blocks | (uintptr_t)v_blocks | (uintptr_t)out) & 15)
    return fail(DP_EINVAL, "chunked_prefill_attention: q, k_blocks, v_blocks and out must be 16-byte aligned");
  const bool fp8 = sh->kv_dtype == DP_KV_FP8_E4M3;
  if (fp8 && (!k_scale || !v_scale))
    return fail(DP_EINVAL, "chunked_prefill_attention: e4m3 cache needs k_scale and v_scale");
  if (!fp8 && (k_scale || v_scale))
    return fail(DP_EINVAL, "chunked_prefill_attention: k_scale/v_scale must be NULL for a bf16 cache");
  if (!(scale > 0.0f) || !std::isfinite(scale))
    return fail(DP_EINVAL, "chunked_prefill_attention: scale must be finite and > 0");

  const int group = sh->n_q_heads / sh->n_kv_heads;
  // The kernel counts items in 32 bits.  The bound is on tiles of 32 query
  // tokens of eight heads: items of 256 columns are never more than those, and
  // the variants with smaller items are taken only where the columns make
  // fewer items of 256 than there are compute units.
  const int64_t tiles = (sh->total_q + 31) / 32 + sh->batch;
  if (tiles * sh->n_kv_heads * (((int64_t)group + 7) / 8) > INT32_MAX / 2)
    return fail(DP_EINVAL, "chunked_prefill_attention: too many query tiles");

  PrefillArgs a;
  a.q = (const uint16_t*)q;
  a.k = (const char*)k_blocks;
  a.v = (const char*)v_blocks;
  a.block_tables = block_tables;
  a.context_lens = context_lens;
  a.q_start = q_start;
  a.k_scale = k_scale;
  a.v_scale = v_scale;
  a.out = out;
  a.scale_log2 = scale * kLog2e;
  a.batch = sh->batch;
  a.hq = sh->n_q_heads;
  a.hkv = sh->n_kv_heads;
  a.group = group;
  a.max_blocks_per_seq = sh->max_blocks_per_seq;
  a.max_ctx = sh->max_context_len;
  a.num_blocks_m1 = (int32_t)(sh->num_blocks - 1);
  a.out_fp32 = sh->out_dtype == DP_OUT_FP32;
  a.total_q = (int32_t)sh->total_q;
  (void)hipGetLastError();
  hipStream_t st = (hipStream_t)stream;
  // The variant.  full(c): items of c columns, were the chunks one list;
  // items(c): the same, were they all of one length.  (Times: one call from a
  // replayed graph.)
  //  - full(256) covers every compute unit: eight waves of 32 columns, whose 256
  //    columns share each K and V tile they copy.  That holds for sequences of
  //    few columns too, as some may be long: 2,048 tokens at 8,192 beside 500
  //    decodes at about 2,000 on 64/8 heads 1,115 us, 1,413 with 64-column
  //    items (1,000 decodes alone, at about 200: 247 and 181).
  //  - full(128) still does: four-wave workgroups of 128 columns, two to a unit,
  //    which overlap each other's set-up and epilogue.
  //  - Contexts may be long (max_context_len > 2048): an item is a chain of KV
  //    steps, so waves work in pairs, each of a pair on half of them.  64
  //    columns to eight waves if these items do not outnumber the compute
  //    units, or no sequence (on average) has more columns (100 tokens at
  //    context 8,000 on 64/8 heads: 95 us, 120 with 128 columns); else 128
  //    columns to eight waves while those items fit one round (381 tokens at
  //    context 20,861: 297 us; 400 with 64 columns to four waves without
  //    pairs), or where a few long chunks among sequences of few columns hide
  //    in the average (381 tokens at 20,861 beside 63 decodes at 1,000: 356 us,
  //    504 with 64).  Where the contexts are short all the same, the pairs' fold
  //    costs up to 5 us (nine fresh prompts below 400 tokens on 16/4 heads: 18.3
  //    us, 13.1 with 64 columns to four waves); the host does not know them.
  //  - Otherwise two four-wave workgroups to a unit again: of 64 columns where
  //    contexts are at most 2,048 and these items all run at once, or sequences
  //    have no more columns (ten chunks of 200 tokens at context 1,000 on 16/2
  //    heads: 28 us; 32 with 128 columns), else of 128 (five chunks of 100
  //    tokens at 500 on 64/8 heads, 280 items of 128: 22 us; 26 with 64 columns,
  //    29 with pairs, which take a second round; but 381 tokens at 20,861 beside
  //    20 decodes at 1,000, 352 items of 128: 373 us, 334 with pairs).
  const int64_t cus = compute_units();
  const int64_t per_seq = (sh->total_q * group + sh->batch - 1) / sh->batch;
  const auto full = [&](int c) { return (sh->total_q * group + c - 1) / c * sh->n_kv_heads; };
  const auto items = [&](int c) { return (per_seq + c - 1) / c * sh->batch * sh->n_kv_heads; };
  const bool may_be_long = sh->max_context_len > 2048;
  if (full(256) >= cus)
    launch<8, 2, 1>(a, fp8, cus, st);
  else if (full(128) > cus)
    launch<4, 2, 1>(a, fp8, 2 * cus, st);
  else if (may_be_long && full(64) <= cus && (per_seq <= 64 || items(64) <= cus))
    launch<8, 1, 2>(a, fp8, cus, st);
  else if (may_be_long && (per_seq <= 64 || items(128) <= cus))
    launch<8, 2, 2>(a, fp8, cus, st);
  else if (!may_be_long && (per_seq <= 64 || items(64) <= 2 * cus))
    launch<4, 1, 1>(a, fp8, 2 * cus, st);
  else
    launch<4, 2, 1>(a, fp8, 2 * cus, st);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return fail(DP_EIO, "chunked_prefill_attention: kernel launch failed: %s", hipGetErrorString(e));
  return DP_OK;
}
