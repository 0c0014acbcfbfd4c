// K2: fused cosine-similarity contraction with two masked row max / argmax reductions.
//
// For every problem (head, sequence) and token i it computes, without materialising the
// N x N matrix (Sec. 3.2 Eq. 1 and the twin window; Sec. 3.4 Eq. 4):
//   best over all j with |i-j| > w of sim(i, j)        -> best_all / arg_all
//   best over j in S0 with |i-j| > w of sim(i, j)      -> best_ret / arg_ret  (= b_i(S0))
// In count mode (Sec. 3.2 Eq. 2) the same sweep counts, per token, the j with |i-j| > w and
// sim(i, j) > tau.
//
// sim(i, j) = sim(j, i), so every unordered pair is computed once and reduced into both of its
// tokens.  Tokens are addressed by their slot in the partitioned order [S0 | evicted] of the
// column copy; keys there are scaled by an exact power of two to a norm in (0.5, 1], and
// r' = 1 / ||scaled key|| lies in [1, 2).
//
// Mapping onto gfx950:
//  * A workgroup owns RB = 4 * NSUB * 32 consecutive slots (its stationary rows) and sweeps the
//    columns from its own slots on to the end: the upper triangle of the pair matrix.  Each
//    wave holds NSUB 32-row blocks as MFMA A operands in registers for the whole sweep (d <= 128
//    makes this a short-K contraction); columns stream through double-buffered LDS tiles of
//    TN = 32 * CPT slots, moved by direct global -> LDS loads, as MFMA B operands.
//  * v_mfma_f32_32x32x16_bf16 gives each lane one column j (lane % 32) and 16 rows: register v
//    holds row 8*(v/4) + 4*(lane/32) + v%4.
//  * Both reductions work on x = dot * r' + 3 in [2, 4), where the fp32 bit pattern is monotone
//    and the low bits can carry an index: for token t and candidate u, x = dot * r'_u + 3 (the
//    similarity is (x - 3) * r'_t), whichever of the two is the row, so a pair's value has the
//    same bits on both sides and the same pair is found whatever its place in the sweep.
//     - column direction: max over a lane's 16 * NSUB rows, index = the register; one LDS
//       64-bit max per 32 columns merges the waves, one global 64-bit max per column and tile
//       merges the workgroups;
//     - row direction: a running maximum per register (never reduced across lanes in the
//       sweep), index = the 32-column chunk inside a window of 2^BITS chunks; at the end of a
//       window the 32 lanes of a row are reduced and merged by one global 64-bit max per row.
//    The 64-bit candidates order by value, then by the smaller slot (the smaller position inside
//    its group), so results do not depend on the order of the merges.
//  * Cost per pair of tokens: 5 VALU instructions per lane element (two v_fma, two v_and_or, two
//    halves of a v_max3) beside half the MFMA work of a full square.  The sweep is bound by VALU
//    issue (VALU busy 69% of the cycles and MFMA 46% at d = 128, 32k tokens; 78% and 23% at d = 64, 8k;
//    63% and 35% on 1k-4k ragged sequences); with every ordered pair on its own it was bound by the
//    MFMA (1313 of the 1340 TFLOP/s a large matrix product reaches).
//  * Measured, full square -> upper triangle, whole calls: 288 heads x 32k, d = 128 59.6 -> 43.1 ms
//    (this kernel 41.8); 288 heads x 64 ragged sequences of 1k-4k 34.4 -> 29.4 ms (this kernel 23.7, the
//    key preparation 4.8, finishing 0.7); 8 heads x 4001 123 -> 62 us; 128 heads x 8k, d = 64 1186 -> 1100 us (half the MFMA work per pair,
//    the same VALU work); counting and eviction, 288 x 16k 14.8 -> 9.3 ms.  Two waves per SIMD: with one, nothing hides
//    the row direction's serial maxima (NSUB 2 and 4, both slower); with three the 2 x 16 running
//    maxima per row block do not fit.
//  * Products of bf16 values are exact in fp32; accumulation is fp32.  fp32 keys use the
//    split k = hi + lo (bf16 each).  The cross sums lo.hi and hi.lo have accumulators of their own:
//    swapping the two tokens swaps them, and their sum, from which the hi.hi chain goes on, is the same.
//  * Chunks that hold pairs inside the window, the rows' own chunks and padding are dropped by
//    scalar masks in the sweep (their r' and the bias become 0, so x stays below any candidate);
//    a masked pass after the sweep redoes those that hold real pairs, with the window tested per
//    element (a kernel of its own for them was bound by load latency: 5.6 ms of the ragged batch).
//  * Few row blocks leave the chip idle: a row block's columns are then cut into up to 16 segments,
//    one workgroup each, until 1024 workgroups are in flight (4 per CU: the segments near the end
//    of the triangle are short).  The candidates merge them like any other workgroups.
//  * The S0 columns alone (no best_all) are swept by the kernel in sim_rect.hip: the lower half
//    of a rectangle of S0 x all cannot be shared.  So are all columns of many short sequences.
//  * The candidates become results in finish_kernel, or in the repair kernel of short sequences.
#include <hip/hip_runtime.h>

#include <type_traits>

#include "finish.h"
#include "sim_common.h"

namespace twinkv {
namespace {

typedef unsigned long long u64;

constexpr uint32_t kBias = 0x40400000u;  // 3.0f

// Count mode: a lane keeps a row's count in 8 bits.  The sweep writes them out after kCountChunks chunks,
// looked at every 32.  The pass after the sweep does after kMaskedCountChunks of a range of chunks, then
// after kMaskedCountMore further ones; a range can leave all but one of those to the next range's first.
constexpr int kCountChunks = 192, kMaskedCountChunks = 32, kMaskedCountMore = 224;
static_assert(kCountChunks + 32 <= 255 && kMaskedCountMore - 1 + kMaskedCountChunks <= 255, "8 bits");

template <int D, bool SPLIT, int NSUB, int CPT, int BITS, int OCC_>
struct Cfg {
  static constexpr int OCC = OCC_;  // workgroups per CU (waves per SIMD)
  // registers of the last row block whose even chunks' candidates wait for the odd chunk's
  static constexpr int HOLD_LAST = D != 128 ? 16 : (SPLIT ? 0 : 8);
  static constexpr int DCOL = SPLIT ? 2 * D : D;      // bf16 elements per column in LDS
  static constexpr int UF = DCOL / 16;                // fragments of one key
  static constexpr int MFMAS = SPLIT ? 3 * D / 16 : D / 16;
  static constexpr int PPC = DCOL / 8;                // 16-byte pieces per column
  static constexpr int TN = CPT * kChunk;             // columns per LDS tile
  static constexpr int NT = kWaves * 64;
  static constexpr int WR = NSUB * 32;                // rows per wave
  static constexpr int RB = kWaves * WR;              // rows per workgroup
  static constexpr int CHUNK_BYTES = kChunk * DCOL * 2;  // keys of one 32-column chunk
  static constexpr int KEY_BYTES = TN * DCOL * 2;
  static constexpr int STAGE = KEY_BYTES + TN * 4;    // keys + r'
  static constexpr int COL_BYTES = 3 * 2 * TN * 8;    // column candidates of three tiles
  static constexpr int LDS_BYTES = 2 * STAGE + COL_BYTES + RB * 4;
  static constexpr int LOADS_PER_WAVE = TN * PPC / (kWaves * 64);  // 1-KB direct loads
  static constexpr uint32_t LOW = (1u << BITS) - 1u;
  static constexpr int WIN = 1 << BITS;               // chunks per window of the row direction
  static_assert(WIN % CPT == 0 && (CPT % 2) == 0, "whole tiles per window, chunks in pairs");
  static_assert(RB % TN == 0, "a workgroup's rows start on a tile boundary");
  static_assert(kGroupAlign % TN == 0, "the evicted group must start on a tile boundary");
  static_assert(kGroupAlign % WR == 0, "a wave's rows lie in one group");
  static_assert((TN * PPC) % (kWaves * 64) == 0, "tile copy must divide evenly");
  static_assert(TN % 64 == 0 && TN <= 128, "the r' table moves in 64-column pieces");
  static_assert(LDS_BYTES * OCC <= 160 * 1024, "LDS of OCC workgroups must fit one CU");
};

__device__ inline void max_global(u64* p, u64 v) {
  (void)__hip_atomic_fetch_max(p, v, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}
// LDS maximum / sum without a result, as instructions of their own: the compiler would wait for
// every direct global -> LDS load in flight before an LDS atomic of its own.  The waits before
// the barriers that publish them are explicit (finish_tile).
__device__ inline uint32_t lds_offset(const void* p) {
  return (uint32_t)(uintptr_t)(const __attribute__((address_space(3))) void*)p;
}
__device__ inline void max_lds(uint32_t off, u64 v) {
  asm volatile("ds_max_u64 %0, %1" : : "v"(off), "v"(v) : "memory");
}
__device__ inline void add_lds(uint32_t off, uint32_t v) {
  asm volatile("ds_add_u32 %0, %1" : : "v"(off), "v"(v) : "memory");
}

// x of the lane whose index differs by the DPP control: quad_perm xor 1 / xor 2, mirror inside
// 8 lanes (xor 7), rotate by 8 inside 16 lanes (xor 8).
template <int CTRL>
__device__ inline uint32_t dpp(uint32_t x) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)x, CTRL, 0xF, 0xF, true);
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor7 = 0x141, kXor8 = 0x128;

// One step of the row reduction over lanes: each lane keeps one of two registers (bit clear:
// a, set: b) and merges its partner's copy of it.
template <int CTRL>
__device__ inline u64 max_step(u64 a, u64 b, bool bit) {
  const u64 keep = bit ? b : a, send = bit ? a : b;
  const u64 got = ((u64)dpp<CTRL>((uint32_t)(send >> 32)) << 32) | dpp<CTRL>((uint32_t)send);
  return keep > got ? keep : got;
}
template <int CTRL>
__device__ inline uint32_t sum_step(uint32_t a, uint32_t b, bool bit) {
  const uint32_t keep = bit ? b : a, send = bit ? a : b;
  return keep + dpp<CTRL>(send);
}

// Which register's row a lane holds after the lane reductions below.
__device__ inline int reduced_reg(int l32) {
  return ((l32 >> 4) << 3) | (((l32 >> 3) & 1) << 2) | (((l32 >> 2) & 1) << 1) | ((l32 >> 1) & 1);
}

// The largest (value, then smaller lane) of each of 16 registers over the 32 lanes of a half:
// the lane pair 2m, 2m + 1 ends with register reduced_reg's result as value << 32 | 31 - lane.
__device__ inline u64 reduce_rows_max(const uint32_t (&run)[16], int l32) {
  u64 k8[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    // lanes 0-15 take register i, lanes 16-31 register i + 8
    const auto sw = __builtin_amdgcn_permlane16_swap(run[i], run[i + 8], false, false);
    const uint32_t lo = sw[0], hi = sw[1];  // from lanes 0-15 / 16-31 of the half
    const bool up = hi > lo;
    k8[i] = ((u64)(up ? hi : lo) << 32) | (uint32_t)(31 - ((l32 & 15) + (up ? 16 : 0)));
  }
  u64 k4[4], k2[2];
#pragma unroll
  for (int i = 0; i < 4; ++i) k4[i] = max_step<kXor8>(k8[i], k8[i + 4], (l32 & 8) != 0);
#pragma unroll
  for (int i = 0; i < 2; ++i) k2[i] = max_step<kXor7>(k4[i], k4[i + 2], (l32 & 4) != 0);
  const u64 k1 = max_step<kXor2>(k2[0], k2[1], (l32 & 2) != 0);
  const u64 got = ((u64)dpp<kXor1>((uint32_t)(k1 >> 32)) << 32) | dpp<kXor1>((uint32_t)k1);
  return k1 > got ? k1 : got;
}
// The sums of 16 registers over the 32 lanes of a half, in the same places.
__device__ inline uint32_t reduce_rows_sum(const uint32_t (&c)[16], int l32) {
  uint32_t k8[8], k4[4], k2[2];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const auto sw = __builtin_amdgcn_permlane16_swap(c[i], c[i + 8], false, false);
    k8[i] = sw[0] + sw[1];
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) k4[i] = sum_step<kXor8>(k8[i], k8[i + 4], (l32 & 8) != 0);
#pragma unroll
  for (int i = 0; i < 2; ++i) k2[i] = sum_step<kXor7>(k4[i], k4[i + 2], (l32 & 4) != 0);
  const uint32_t k1 = sum_step<kXor2>(k2[0], k2[1], (l32 & 2) != 0);
  return k1 + dpp<kXor1>(k1);
}

// Column chunks with pairs inside the window of a wave's rows (slots [row0, row0 + rows) of group
// grp, at least one of them real): in the rows' own group up to a_hi, in the other group [b_lo, b_hi].  The columns at positions x0 <= j < x1 are one contiguous range of slots
// per group, read off the S0 prefix counts.
struct Band {
  int a_hi, b_lo, b_hi;
};
__device__ inline Band window_band(const SimArgs& a, const Place& pl, int row0, int rows, int grp) {
  const int32_t* pc = a.pcol + pl.colbase;
  const int32_t* prk = a.prank + pl.colbase;
  const int ret_pad = pl.ret_chunks * kChunk;
  const int end = grp == 0 ? pl.n_ret : ret_pad + (pl.len - pl.n_ret);  // of the group's real slots
  Band bd{-1, 1, 0};
  const int x0 = max(pc[row0] - a.w, 0), x1 = min(pc[min(row0 + rows, end) - 1] + a.w + 1, pl.len);
  const int r0 = prk[x0], r1 = prk[x1];
  const int e0 = ret_pad + (x0 - r0), e1 = ret_pad + (x1 - r1);
  if (grp == 0) {
    bd.a_hi = (r1 - 1) / kChunk;
    if (e1 > e0) {
      bd.b_lo = e0 / kChunk;
      bd.b_hi = (e1 - 1) / kChunk;
    }
  } else {
    bd.a_hi = (e1 - 1) / kChunk;
  }
  bd.a_hi = __builtin_amdgcn_readfirstlane(bd.a_hi);
  bd.b_lo = __builtin_amdgcn_readfirstlane(bd.b_lo);
  bd.b_hi = __builtin_amdgcn_readfirstlane(bd.b_hi);
  return bd;
}

// Position of a slot of group grp; padding (copies of the group's last token) has that token's, so
// that it stays an exact tie of it.
__device__ inline int slot_position(const SimArgs& a, const Place& pl, int slot, int grp) {
  const int last = grp == 0 ? pl.n_ret - 1 : pl.ret_chunks * kChunk + (pl.len - pl.n_ret) - 1;
  return a.pcol[pl.colbase + min(slot, last)];
}

// The window test of a pair with the row at pi: base - pi >= thr as unsigned numbers.  In the rows'
// own group (SAME) the column has to lie more than w after the row, so that each pair counts once
// and the lower half of the triangle not at all; in the other group more than w away on either side.
struct Window {
  uint32_t base, thr;
};
__device__ inline Window window_of(int pj, int w, bool same) {
  return same ? Window{(uint32_t)(pj - w - 1) + 0x80000000u, 0x80000000u}
              : Window{(uint32_t)(pj + w), 2u * (uint32_t)w + 1u};
}

// A 32-row block's MFMA A operands and r' (count mode: thresholds) of a lane's 16 rows.  A block
// past the last slot reads the last one; its results are never used.
template <bool COUNT, int D, bool SPLIT, int UF>
__device__ inline void load_rows(const SimArgs& a, const Place& pl, int row0, int l32, int half,
                                 bf16x8 (&af)[UF], float (&rs)[16]) {
  constexpr int DCOL = SPLIT ? 2 * D : D;
  const int r0 = min(row0, pl.total_chunks * kChunk - 32);
  const uint16_t* src = a.pkeys + (pl.colbase + r0) * DCOL + 8 * (l32 + 32 * half);
#pragma unroll
  for (int t = 0; t < UF; ++t) af[t] = *reinterpret_cast<const bf16x8*>(src + 512 * t);
  const float* rc = a.rcol + pl.colbase + r0 + 4 * half;
#pragma unroll
  for (int v4 = 0; v4 < 4; ++v4) {
    const float4 x = *reinterpret_cast<const float4*>(rc + 8 * v4);
    rs[4 * v4 + 0] = x.x;
    rs[4 * v4 + 1] = x.y;
    rs[4 * v4 + 2] = x.z;
    rs[4 * v4 + 3] = x.w;
  }
  if constexpr (COUNT) {
    // sim(i, j) > tau  <=>  dot * r'_j - tau / r'_i > 0.  A zero key has similarity 0 to every
    // key: it counts every candidate exactly when tau < 0 (the smallest normal number stands
    // for tau = 0, so that a similarity of exactly 0 is not above it).  Rows that are padding
    // count nothing.
    const float t = a.tau == 0.0f ? 1.17549435e-38f : a.tau;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const float r = rs[v];
      const bool real = row0 + slot_row(v, half) < pl.len;
      rs[v] = !real ? -INFINITY : (r > 0.0f ? -t / r : (a.tau < 0.0f ? INFINITY : -INFINITY));
    }
  }
}

template <bool COUNT, int D, bool SPLIT, int NSUB, int CPT, int BITS, int OCC>
__global__ __launch_bounds__(kWaves * 64, OCC) void sim_reduce_kernel(SimArgs a, int nseg) {
  using C = Cfg<D, SPLIT, NSUB, CPT, BITS, OCC>;
  constexpr uint32_t LOW = C::LOW;
  constexpr int G = D / 16;
  __shared__ __attribute__((aligned(1024))) char smem[C::LDS_BYTES];
  // column candidates (counts in count mode) of three tiles in turn, one plane per group of
  // the rows they came from: [tile % 3][group][column]
  u64* const s_col = reinterpret_cast<u64*>(smem + 2 * C::STAGE);
  int* const s_pos = reinterpret_cast<int*>(smem + 2 * C::STAGE + C::COL_BYTES);  // the rows' positions

  Place pl;
  int seg;  // segment of the row block's columns
  if (!find_place(a, (int)blockIdx.x, pl, seg)) return;
  const int nslots = pl.total_chunks * kChunk;
  const int ret_chunks = pl.ret_chunks;                      // a multiple of kGroupAlign / 32
  const int ret_pad = ret_chunks * kChunk;
  // (the row blocks are counted for the largest padding)
  if (pl.rb * C::RB >= nslots) return;
  const int ret_real = (pl.n_ret + kChunk - 1) / kChunk;     // S0 chunks with a real column
  const int nchunks = pl.total_chunks;
  const int ncols = nchunks * kChunk;                        // columns swept
  const int ntiles = (nchunks + CPT - 1) / CPT;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int half = lane >> 5;
  const int l32 = lane & 31;
  const int row0 = pl.rb * C::RB + wave * C::WR;  // this wave's first slot
  const int grp = row0 >= ret_pad ? 1 : 0;        // ... and its group (0: S0, 1: evicted)

  const uint16_t* pk = a.pkeys + pl.colbase * C::DCOL;
  const float* rc = a.rcol + pl.colbase;
  const int64_t plane = (int64_t)a.n_heads * a.PT;
  u64* const best0 = COUNT ? nullptr : reinterpret_cast<u64*>(a.best) + pl.colbase;
  int32_t* const counts = COUNT ? a.counts + pl.rowbase : nullptr;

  // A wave without rows of its own here only takes its share of the tile loads.
  const bool active = row0 < nslots && !(row0 >= pl.n_ret && row0 < ret_pad);

  // ---- chunks the sweep drops for this wave: up to bd.a_hi (its own, their window band and the
  // other half of the triangle) and the band in the other group, which the pass after the sweep
  // redoes, and padding.  Count mode: copies of the last column must not be counted, so the
  // partly filled last chunk is redone too (there is no S0 group then).
  Band bd{-1, 1, 0};
  if (active) bd = window_band(a, pl, row0, C::WR, grp);
  const int pad_c = COUNT && (pl.len % kChunk) ? pl.total_chunks - 1 : -1;
  // Result bits of a tile in the sweep (bit k: chunk c0 + k counts).
  auto keep_bits = [&](int c0) -> uint32_t {
    // most tiles drop nothing: one range test over the whole tile
    const int c1 = c0 + CPT - 1;
    if (c0 > bd.a_hi && c1 < nchunks && !(c1 >= ret_real && c0 < ret_chunks) &&
        !(c1 >= bd.b_lo && c0 <= bd.b_hi) && !(pad_c >= c0 && pad_c <= c1))
      return (1u << CPT) - 1u;
    uint32_t bits = 0u;
#pragma unroll
    for (int kc = 0; kc < CPT; ++kc) {
      const int gc = c0 + kc;
      const int drop = (int)(gc <= bd.a_hi) | (int)(gc >= nchunks) |
                       ((int)(gc >= ret_real) & (int)(gc < ret_chunks)) |
                       ((int)(gc >= bd.b_lo) & (int)(gc <= bd.b_hi)) | (int)(gc == pad_c);
      bits |= (uint32_t)(drop ^ 1) << kc;
    }
    return bits;
  };

  // ---- this workgroup's tiles: from its own rows on, cut into nseg segments ----
  int ta, tb;
  {
    const int t0 = pl.rb * C::RB / C::TN;
    const int per = (max(ntiles - t0, 0) + nseg - 1) / nseg;
    ta = t0 + seg * per;
    tb = min(ta + per, ntiles);
  }

  // ---- row keys: MFMA A operands, resident for the whole sweep --------------------------
  // rs: r' of the lane's 16 * NSUB rows (count mode: their thresholds)
  bf16x8 afrag[NSUB][C::UF];
  float rs[NSUB][16];
  if (active) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s)
      load_rows<COUNT, D, SPLIT, C::UF>(a, pl, row0 + 32 * s, l32, half, afrag[s], rs[s]);
  } else {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
#pragma unroll
      for (int t = 0; t < C::UF; ++t) afrag[s][t] = bf16x8{};
#pragma unroll
      for (int v = 0; v < 16; ++v) rs[s][v] = 0.0f;
    }
  }

  // Row direction.  run: the running maximum of each register over the chunks of the current
  // window, as value bits with LOW - (chunk - window) in the low bits; hold: the even chunk's
  // candidates, merged with the odd chunk's by one v_max3 (where registers allow).  Count mode:
  // run holds the sign bits of the last 32 chunks (newest in bit 0), kept which of those chunks
  // count, and cnt the counts of the windows before, four rows of 8 bits a register (a lane
  // counts at most one column per chunk, and they are written out every kCountChunks).
  uint32_t run[NSUB][16], hold[NSUB][16];
  uint32_t cnt[NSUB][4];
  uint32_t kept[NSUB];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    kept[s] = 0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      run[s][v] = hold[s][v] = 0u;
      cnt[s][v / 4] = 0u;
    }
  }

  // ---- column tiles: global -> LDS by direct (asynchronous) loads, double buffered ------
  // The copy stores each 32-slot chunk piece by piece (16-byte piece p of the chunk's column c at
  // p * 512 + 16 c), so a tile is one plain stream, a fragment read takes 64 consecutive 16-byte
  // words (no bank conflicts) and every fragment lies at a constant offset from one lane address.
  // Each wave moves LOADS_PER_WAVE blocks of 1 KB.  The buffer resource of a tile ends at the
  // problem's last column, so the hardware range check turns loads past it into zeros instead of
  // reads (those columns are dropped).
  const uint32_t lane_base = lds_offset(smem) + 16 * lane;
  auto read_frag = [&](uint32_t base, int t, int chunk) -> bf16x8 {
    return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(
        (uintptr_t)(base + (uint32_t)(t * 1024 + chunk * C::CHUNK_BYTES)));
  };
  auto issue_tile = [&](int tile, int buf) {
    // one resource per tile (the range check sees a lane's offset and the instruction's; the
    // instruction's offset also moves the LDS address, four 1-KB blocks per base)
    char* st = smem + buf * C::STAGE;
    const int64_t first = (int64_t)tile * C::TN;
    const int left = ncols - (int)first;                // > 0 for every issued tile
    const int ncol = left < C::TN ? left : C::TN;
    const __amdgpu_buffer_rsrc_t rk = tile_rsrc(pk + first * C::DCOL, ncol * C::DCOL * 2);
    const int base = wave * C::LOADS_PER_WAVE * 1024;
    int ln = lane;
    asm("" : "+v"(ln));  // (the offsets are made here: held over the sweep, they would be spilled)
#pragma unroll
    for (int kk = 0; kk < C::LOADS_PER_WAVE; kk += 4) {
      char* lds = st + base + kk * 1024;
      const int off = 16 * ln + base + kk * 1024;
      load_lds16<0>(rk, lds, off);
      if constexpr (C::LOADS_PER_WAVE > 1) load_lds16<1024>(rk, lds, off);
      if constexpr (C::LOADS_PER_WAVE > 2) load_lds16<2048>(rk, lds, off);
      if constexpr (C::LOADS_PER_WAVE > 3) load_lds16<3072>(rk, lds, off);
    }
    // The r' table in 256-byte pieces, 4 bytes a lane.
    if (wave < C::TN / 64)
      load_lds4(tile_rsrc(rc + first, ncol * 4), st + C::KEY_BYTES + wave * 256,
                4 * ln + wave * 256);
  };
  auto finish_tile = [&]() {  // wait for this wave's direct loads and its LDS maxima
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  };

  // ---- reductions of one 32 x 32 block (rows of block s, one chunk's columns) ------------
  // Row direction with the chunk's code; column direction into cb (one best per row block).
  struct ColBest {
    uint32_t b[NSUB];
  };
  auto reduce_block = [&](const f32x16& acc, int s, bool odd, float rl, uint32_t m,
                          uint32_t code, ColBest& cb) {
    // a dropped block (m = 0): r' and the bias become 0, below any candidate
    const float bias = __uint_as_float(m & kBias);
    rl = __uint_as_float(__float_as_uint(rl) & m);
    if constexpr (COUNT) {
      uint32_t neg = 0u;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t y = __float_as_uint(fmaf(acc[v], rl, rs[s][v]));
        run[s][v] = __builtin_amdgcn_alignbit(run[s][v], y, 31);
        neg = __builtin_amdgcn_alignbit(neg, y, 31);
      }
      cb.b[s] = (16u - (uint32_t)__builtin_popcount(neg)) & m;
    } else {
      uint32_t b = 0u;
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const uint32_t us = (__float_as_uint(fmaf(acc[v], rl, bias)) & ~LOW) | code;
        if (s == NSUB - 1 && v >= C::HOLD_LAST) {
          run[s][v] = max(run[s][v], us);
          asm("" : "+v"(run[s][v]));  // (kept from merging with the next chunk's candidates)
        } else if (odd) {
          run[s][v] = max(max(run[s][v], hold[s][v]), us);
        } else {
          hold[s][v] = us;
        }
        b = max(b, (__float_as_uint(fmaf(acc[v], rs[s][v], 3.0f)) & ~LOW) | (uint32_t)(15 - v));
      }
      cb.b[s] = b & m;
    }
  };
  // The column candidate of a chunk over the wave's row blocks: value bits and ~slot (zero value:
  // none); equal values keep the earlier row block, and inside it the earlier register.
  const uint32_t nrow = ~(uint32_t)(row0 + 4 * half);
  auto col_key = [&](const ColBest& cb) -> u64 {
    uint32_t b = cb.b[0], off = 0u;
#pragma unroll
    for (int s = 1; s < NSUB; ++s) {
      const bool up = (cb.b[s] >> BITS) > (b >> BITS);
      b = up ? cb.b[s] : b;
      off = up ? 32u * s : off;
    }
    const uint32_t q = 15u - (b & 15u);
    return ((u64)(b & ~LOW) << 32) | (nrow - off - q - (q & ~3u));
  };
  // A chunk's column result (count mode: the count), and its merge into the tile's entries.
  auto col_result = [&](const ColBest& cb) -> u64 {
    if constexpr (COUNT) {
      uint32_t c = 0u;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) c += cb.b[s];
      return c;
    } else {
      return col_key(cb);
    }
  };
  const uint32_t col_lane = lds_offset(s_col) + 8 * (l32 + (COUNT ? 0 : grp * C::TN));
  auto col_emit = [&](u64 r, int buf3, int kc) {
    const uint32_t off = col_lane + 8 * (buf3 * 2 * C::TN + kc * kChunk);
    if constexpr (COUNT) add_lds(off, (uint32_t)r);
    else max_lds(off, r);
  };
  // A complete tile's column results to global memory; the LDS entries start over.
  auto cols_out = [&](int tile, int buf3) {
    constexpr int WPG = C::TN / 64;  // waves per group's entries
    const int g = wave / WPG;
    if (g < 2) {
      int ln = lane;
      asm("" : "+v"(ln));
      const int c0 = (wave % WPG) * 64;
      u64* p = s_col + (buf3 * 2 + g) * C::TN + c0 + ln;
      const u64 v = *p;
      *p = 0ull;
      const int col0 = tile * C::TN + c0;
      if constexpr (COUNT) {
        if ((uint32_t)v != 0u && col0 + ln < pl.len) atomicAdd(&counts[col0 + ln], (int)(uint32_t)v);
      } else {
        u64* dst = best0 + (g ? plane : 0) + col0;
        if ((uint32_t)(v >> 32) >= kValidMin && col0 + ln < ncols) max_global(dst + ln, v);
      }
    }
  };
  // End of a window of the row direction: chunk base + i * stride is coded LOW - i; dst is the
  // candidates' plane (by the group of the columns).
  auto rows_out = [&](int base, int stride, u64* dst) {
    if constexpr (!COUNT) {
      u64 key[NSUB];
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        key[s] = reduce_rows_max(run[s], l32);
#pragma unroll
        for (int v = 0; v < 16; ++v) run[s][v] = 0u;
      }
      // even lanes write the rows of block s0, odd lanes those of block s0 + 1 (if there is one)
#pragma unroll
      for (int s0 = 0; s0 < NSUB; s0 += 2) {
        constexpr int kOne = NSUB > 1 ? 1 : 0;
        const bool second = s0 + 1 < NSUB && (lane & 1);
        const u64 ka = key[s0], kb2 = key[s0 + 1 < NSUB ? s0 + kOne : s0];
        const u64 kx = second ? kb2 : ka;
        const uint32_t val = (uint32_t)(kx >> 32);
        const int chunk = base + (int)(LOW - (val & LOW)) * stride;
        const uint32_t slot = (uint32_t)(chunk * kChunk + 31 - (int)(kx & 31u));
        const int row = row0 + 32 * (s0 + second) + slot_row(reduced_reg(l32), half);
        if (val >= kValidMin && row < nslots && (s0 + 1 < NSUB || !(lane & 1)))
          max_global(dst + row, ((u64)(val & ~LOW) << 32) | (uint32_t)~slot);
      }
    }
  };
  auto counts_fold = [&]() {  // count mode: a window's sign bits into the counts
    if constexpr (COUNT) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          cnt[s][v / 4] += (uint32_t)__builtin_popcount(~run[s][v] & kept[s]) << (8 * (v & 3));
          run[s][v] = 0u;
        }
        kept[s] = 0u;
      }
    }
  };
  auto counts_out = [&]() {  // count mode: the rows' counts so far
    if constexpr (COUNT) {
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        uint32_t cs[16];
#pragma unroll
        for (int v = 0; v < 16; ++v) cs[v] = (cnt[s][v / 4] >> (8 * (v & 3))) & 0xFFu;
#pragma unroll
        for (int v = 0; v < 4; ++v) cnt[s][v] = 0u;
        const uint32_t c = reduce_rows_sum(cs, l32);
        const int row = row0 + 32 * s + slot_row(reduced_reg(l32), half);
        if (c != 0u && row < pl.len && !(lane & 1))
          atomicAdd(&counts[row], (int)c);
      }
    }
  };

  // ---- the pending reduction: the last row block of the previous chunk is reduced while the
  // first MFMA chain of the next chunk runs (software pipelining across chunks).
  f32x16 pacc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float prl = 0.0f;
  uint32_t pcode = 0u, pm_mask = 0u;
  ColBest pcb;
#pragma unroll
  for (int s = 0; s < NSUB; ++s) pcb.b[s] = 0u;

  // One tile: each chain's reductions run beside the following chain's MFMAs, and the last
  // chain's are left pending for the next chunk.  During the last chain, fragment t of the next
  // chunk is read into the registers that MFMA t has just consumed.
  auto sweep_tile = [&](uint32_t stage, int c0, uint32_t keep, int wbase,
                        int buf3, int pbuf3) {
    // VALU instructions placed beside each MFMA: one block's reductions over its MFMAs
    constexpr int VALU_PER_MFMA =
        ((COUNT ? 54 : 86) + (SPLIT ? 16 : 0) + C::MFMAS - 1) / C::MFMAS;
    const uint32_t fbase = lane_base + stage;
    const char* st = smem + stage;
    bf16x8 fb[C::UF];
    u64 cres = 0ull;  // the pending chunk's column result
#pragma unroll
    for (int t = 0; t < C::UF; ++t) fb[t] = read_frag(fbase, t, 0);
#pragma unroll
    for (int kc = 0; kc < CPT; ++kc) {
      const uint32_t mask = 0u - ((keep >> kc) & 1u);
      const float rl = *reinterpret_cast<const float*>(st + C::KEY_BYTES + (kc * kChunk + l32) * 4);
      // (in a vector register: the value mask takes the one scalar operand of v_and_or)
      uint32_t code = LOW - (uint32_t)(c0 + kc - wbase);
      asm("" : "+v"(code));
      ColBest cb;
      f32x16 x;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        f32x16 y = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        f32x16 yq = y;
        const bool pre = (s == NSUB - 1) && (kc + 1 < CPT);
#pragma unroll
        for (int t = 0; t < C::UF; ++t) {
          if constexpr (!SPLIT) {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t], fb[t], y, 0, 0, 0);
          } else if (t < G) {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][G + t], fb[t], y, 0, 0, 0);
            yq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t], fb[G + t], yq, 0, 0, 0);
            if (t == G - 1) {
#pragma unroll
              for (int v = 0; v < 16; ++v) y[v] += yq[v];
            }
          } else {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t - G], fb[t - G], y, 0, 0, 0);
          }
          const int done = !SPLIT ? t : t < G ? G + t : t - G;
          if (pre) fb[done] = read_frag(fbase, done, kc + 1);
        }
        if (s == 0) {
          // the pending chunk: the previous chunk of this tile, or the last of the previous tile
          kept[NSUB - 1] = (kept[NSUB - 1] << 1) | (pm_mask & 1u);
          reduce_block(pacc, NSUB - 1, kc == 0 ? true : ((kc - 1) & 1) != 0, prl, pm_mask, pcode, pcb);
          cres = col_result(pcb);
        } else {
          kept[s - 1] = (kept[s - 1] << 1) | (mask & 1u);
          reduce_block(x, s - 1, (kc & 1) != 0, rl, mask, code, cb);
        }
#pragma unroll
        for (int i = 0; i < C::MFMAS; ++i) {
          __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          if (pre) __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedValu, VALU_PER_MFMA, 0);
        }
        __builtin_amdgcn_sched_barrier(0);
        if (s == 0) {
          col_emit(cres, kc == 0 ? pbuf3 : buf3, kc == 0 ? CPT - 1 : kc - 1);
          __builtin_amdgcn_sched_barrier(0);
        }
        x = y;
      }
      pacc = x;
      prl = rl;
      pcode = code;
      pm_mask = mask;
      pcb = cb;
    }
  };
  // Reduce the pending block now, with nothing left pending.
  auto drain = [&](int pbuf3) {
    // The opaque copy keeps the compiler from moving the tile body's own pending reduction out of
    // the body to share it with this rare path.
    f32x16 pa = pacc;
    asm volatile("" : "+v"(pa));
    kept[NSUB - 1] = (kept[NSUB - 1] << 1) | (pm_mask & 1u);
    reduce_block(pa, NSUB - 1, true, prl, pm_mask, pcode, pcb);
    col_emit(col_result(pcb), pbuf3, CPT - 1);
    prl = 0.0f;
    pm_mask = 0u;
#pragma unroll
    for (int s = 0; s < NSUB; ++s) pcb.b[s] = 0u;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      pacc[v] = 0.0f;
      hold[NSUB - 1][v] = 0u;
    }
  };

#ifdef TWINKV_DEBUG
  // Debug build: both stages start as poison.
  {
    uint4* all = reinterpret_cast<uint4*>(smem);
    for (int i = threadIdx.x; i < 2 * C::STAGE / 16; i += C::NT)
      all[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
  }
  __syncthreads();
#endif
  for (int e = threadIdx.x; e < 3 * 2 * C::TN; e += C::NT) s_col[e] = 0ull;
  for (int e = threadIdx.x; e < C::RB; e += C::NT) {
    const int slot = pl.rb * C::RB + e, g = slot >= ret_pad ? 1 : 0;
    s_pos[e] = g == 0 && pl.n_ret == 0 ? 0 : slot_position(a, pl, slot, g);
  }
  // Tiles from the last down to the rows' own: the row blocks of a problem that run at the same
  // time start on the same tile and stay near each other, so a tile is read from HBM about once
  // (sweeping up from each block's own rows spreads them over the whole problem).
  if (ta < tb) issue_tile(tb - 1, 0);
  bool open = false;     // a window of the row direction is open
  bool pending = false;  // ... and its last block is pending
  int wbase = 0;         // ... its first chunk
  int nacc = 0;          // (count mode) chunks counted since the counts were written out
  int buf3 = 0;          // candidates' buffer of this tile: iteration % 3
#pragma unroll 1
  for (int tile = tb - 1; tile >= ta; --tile) {
    const int buf = (tb - 1 - tile) & 1;
    const int pbuf3 = buf3 == 0 ? 2 : buf3 - 1;
    finish_tile();
    __syncthreads();
    if (tile > ta) issue_tile(tile - 1, buf ^ 1);
    // every wave has finished the tile before the previous one (its last block is reduced in the
    // tile after it)
    if (tile + 2 < tb) cols_out(tile + 2, buf3 == 2 ? 0 : buf3 + 1);
    const int c0 = tile * CPT;
    const uint32_t keep = active ? __builtin_amdgcn_readfirstlane(keep_bits(c0)) : 0u;
    const bool work = keep != 0u;  // (tiles of dropped chunks only are skipped)
    // the window ends after its last chunk, at the end of a group of columns and with the sweep
    const bool close = open && (c0 < wbase || (!COUNT && c0 + CPT == ret_chunks));
    if (pending && (close || !work)) {
      drain(pbuf3);
      pending = false;
      if constexpr (COUNT) counts_fold();
    }
    if (close) {
      if constexpr (COUNT) {
        nacc += 32;
        if (nacc >= kCountChunks) {  // a lane's counts still fit 8 bits, with 32 chunks more at the end
          counts_out();
          nacc = 0;
        }
      } else {
        rows_out(wbase, 1, best0 + (c0 + CPT >= ret_chunks ? plane : 0));
      }
      open = false;
    }
    if (work) {
      if (!open) wbase = c0 + CPT - (COUNT ? 32 : C::WIN);
      open = true;
      sweep_tile((uint32_t)(buf * C::STAGE), c0, keep, wbase, buf3, pbuf3);
      pending = true;
    }
    buf3 = buf3 == 2 ? 0 : buf3 + 1;
#ifdef TWINKV_DEBUG
    // Debug build: once every wave has swept this stage, fill it with 0xFF bytes (NaN keys
    // and inverse norms) before the next tile's loads refill it.  A read of a stage outside its
    // tile's lifetime then sees the poison, and the results differ from the normal build's.
    __syncthreads();
    {
      uint4* stg = reinterpret_cast<uint4*>(smem + buf * C::STAGE);
      for (int i = threadIdx.x; i < C::STAGE / 16; i += C::NT)
        stg[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    }
    __syncthreads();
#endif
  }
  if (pending) {
    drain(buf3 == 0 ? 2 : buf3 - 1);
    if constexpr (COUNT) counts_fold();
  }
  if constexpr (!COUNT) {
    if (open) rows_out(wbase, 1, best0 + (ta * CPT >= ret_chunks ? plane : 0));
  }
  finish_tile();
  __syncthreads();
  if (tb - ta >= 2) cols_out(ta + 1, buf3 == 2 ? 0 : buf3 + 1);
  if (tb - ta >= 1) cols_out(ta, buf3 == 0 ? 2 : buf3 - 1);

  // ---- the dropped chunks that hold real pairs, read straight from the column copy, every element
  // tested (the other workgroup of the CU sweeps meanwhile).  Segment k takes every nseg-th.
  auto masked_range = [&](int l, int h, int cgrp) {
    u64* const dst_rows = best0 + (cgrp ? plane : 0);
    u64* const dst_cols = best0 + (grp ? plane : 0);
    int n = 0;
#pragma unroll 1
    for (int gc = l + seg; gc <= h; gc += nseg) {
      const int col = gc * kChunk + l32;
      bf16x8 fb[C::UF];
      const uint16_t* src = pk + (int64_t)gc * (kChunk * C::DCOL) + 8 * lane;
#pragma unroll
      for (int t = 0; t < C::UF; ++t) fb[t] = *reinterpret_cast<const bf16x8*>(src + 512 * t);
      const float rl = rc[col];
      // (counting, columns of padding are excluded: position -1)
      const int pj = COUNT ? a.pcol[pl.colbase + col] : slot_position(a, pl, col, cgrp);
      const Window win = window_of(pj, a.w, cgrp == grp);
      const uint32_t code = LOW - (uint32_t)n;
      ColBest cb;
#pragma unroll
      for (int s = 0; s < NSUB; ++s) {
        cb.b[s] = 0u;
        if (cgrp == grp && gc < row0 / kChunk + s) continue;  // the other half of the triangle
        f32x16 y = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        f32x16 yq = y;
#pragma unroll
        for (int t = 0; t < C::UF; ++t) {
          if constexpr (!SPLIT) {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t], fb[t], y, 0, 0, 0);
          } else if (t < G) {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][G + t], fb[t], y, 0, 0, 0);
            yq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t], fb[G + t], yq, 0, 0, 0);
            if (t == G - 1) {
#pragma unroll
              for (int v = 0; v < 16; ++v) y[v] += yq[v];
            }
          } else {
            y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(afrag[s][t - G], fb[t - G], y, 0, 0, 0);
          }
        }
#pragma unroll
        for (int v4 = 0; v4 < 4; ++v4) {
          const int4 p4 = *reinterpret_cast<const int4*>(s_pos + wave * C::WR + 32 * s + 8 * v4 + 4 * half);
          const int pi[4] = {p4.x, p4.y, p4.z, p4.w};
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int v = 4 * v4 + e;
            const bool ok = win.base - (uint32_t)pi[e] >= win.thr;
            if constexpr (COUNT) {
              const uint32_t c = (uint32_t)ok & ((~__float_as_uint(fmaf(y[v], rl, rs[s][v]))) >> 31);
              cnt[s][v / 4] += c << (8 * (v & 3));
              cb.b[s] += c;
            } else {
              const uint32_t us = (__float_as_uint(fmaf(y[v], rl, 3.0f)) & ~LOW) | code;
              const uint32_t ut = (__float_as_uint(fmaf(y[v], rs[s][v], 3.0f)) & ~LOW) | (uint32_t)(15 - v);
              run[s][v] = max(run[s][v], ok ? us : 0u);
              cb.b[s] = max(cb.b[s], ok ? ut : 0u);
            }
          }
        }
      }
      if constexpr (COUNT) {
        const uint32_t c = (uint32_t)col_result(cb);
        if (c != 0u) atomicAdd(&counts[col], (int)c);
        if (++n == kMaskedCountChunks) {  // a lane's counts still fit 8 bits
          counts_out();
          n -= kMaskedCountMore;
        }
      } else {
        const u64 key = col_key(cb);  // the better of the two halves' rows
        const auto sh = __builtin_amdgcn_permlane32_swap((uint32_t)(key >> 32), (uint32_t)(key >> 32), false, false);
        const auto sl = __builtin_amdgcn_permlane32_swap((uint32_t)key, (uint32_t)key, false, false);
        const u64 k0 = ((u64)sh[0] << 32) | sl[0], k1 = ((u64)sh[1] << 32) | sl[1];
        const u64 kx = k0 > k1 ? k0 : k1;
        if (half == 0 && (uint32_t)(kx >> 32) >= kValidMin) max_global(dst_cols + col, kx);
        ++n;
        if (n == C::WIN || gc + nseg > h) {
          rows_out(gc - (n - 1) * nseg, nseg, dst_rows);
          n = 0;
        }
      }
    }
  };
  if constexpr (COUNT) counts_out();  // (an inactive wave has counted nothing)
#pragma unroll 1
  for (int r = active ? 0 : 3; r < 3; ++r) {  // (one copy of the code)
    const int l = r == 0 ? row0 / kChunk : (r == 1 ? bd.b_lo : pad_c);
    const int h = r == 0 ? bd.a_hi : (r == 1 ? bd.b_hi : (pad_c > bd.a_hi ? pad_c : -1));
    masked_range(l, h, r == 1 ? grp ^ 1 : grp);
  }
  if constexpr (COUNT) counts_out();
}

constexpr int kFlatThreads = 256;

// The candidates of every token to its results.
__global__ __launch_bounds__(kFlatThreads) void finish_kernel(SimArgs a, int h0) {
  const int64_t t = (int64_t)blockIdx.x * kFlatThreads + threadIdx.x;
  if (t >= a.T) return;
  const int head = h0 + (int)blockIdx.y;
  int lo = 0, hi = a.n_seqs - 1;  // the last sequence that starts at or before t
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.seqtab[mid].start <= t) lo = mid; else hi = mid - 1;
  }
  const SeqInfo si = a.seqtab[lo];
  const ProblemMeta pm = a.pmeta[head * a.n_seqs + lo];
  finish_tokens<1>(a, finish_place(a, head, si, pm), si.len, (int)(t - si.start), 0);
}

template <int D, bool SPLIT, int NSUB, int CPT, int BITS, int OCC>
hipError_t run(const SimArgs& a, hipStream_t st) {
  using C = Cfg<D, SPLIT, NSUB, CPT, BITS, OCC>;
  const int64_t groups = a.n_heads >= 8 ? 8LL * ((a.n_heads + 7) / 8) : (int64_t)a.n_heads;
  const int64_t rows = groups * a.total_tiles;
  if (rows == 0) return hipSuccess;
  int nseg = 1;
  while (nseg < 16 && rows * nseg < 1024) ++nseg;
  const dim3 block(C::NT), sweep((unsigned)(rows * nseg));
  if (a.counts != nullptr) {
    hipLaunchKernelGGL((sim_reduce_kernel<true, D, SPLIT, NSUB, CPT, BITS, OCC>), sweep, block, 0, st, a, nseg);
    return hipGetLastError();
  }
  hipLaunchKernelGGL((sim_reduce_kernel<false, D, SPLIT, NSUB, CPT, BITS, OCC>), sweep, block, 0, st, a, nseg);
  hipError_t e = hipGetLastError();
  if (a.finish_later) return e;
  for (int h0 = 0; e == hipSuccess && h0 < a.n_heads; h0 += 65535) {
    const int by = a.n_heads - h0 < 65535 ? a.n_heads - h0 : 65535;
    hipLaunchKernelGGL(finish_kernel, dim3((unsigned)((a.T + kFlatThreads - 1) / kFlatThreads), (unsigned)by),
                       dim3(kFlatThreads), 0, st, a, h0);
    e = hipGetLastError();
  }
  return e;
}

}  // namespace

// Tile shapes: (d, fp32 split, 32-row blocks per wave, 32-column chunks per LDS tile, index bits
// in the packed values).
#ifndef TWINKV_CFG_BF16_128
#define TWINKV_CFG_BF16_128 128, false, 2, 4, 6, 2
#endif
#ifndef TWINKV_CFG_BF16_64
#define TWINKV_CFG_BF16_64 64, false, 2, 4, 4, 2
#endif
#ifndef TWINKV_CFG_F32_64
#define TWINKV_CFG_F32_64 64, true, 1, 4, 4, 2
#endif
#ifndef TWINKV_CFG_F32_128
#define TWINKV_CFG_F32_128 128, true, 1, 2, 4, 2
#endif

int sim_rows_per_block(Sweep sweep, int dtype, int d) {
  if (sweep != kSweepPairs) return sim_rect_rows_per_block(dtype, d);
  if (d != 64 && d != 128) return 0;
  if (dtype == 0) return 4 * 2 * 32;
  if (dtype == 1) return 4 * 1 * 32;
  return 0;
}

int launch_sim_reduce(const SimArgs& a, int dtype, int d, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (a.sweep != kSweepPairs) return launch_sim_rect(a, dtype, d, st);
  if (dtype == 0 && d == 128) return run<TWINKV_CFG_BF16_128>(a, st);
  if (dtype == 0 && d == 64) return run<TWINKV_CFG_BF16_64>(a, st);
  if (dtype == 1 && d == 64) return run<TWINKV_CFG_F32_64>(a, st);
  if (dtype == 1 && d == 128) return run<TWINKV_CFG_F32_128>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace twinkv
