// K2 over a full rectangle of rows x columns, each value reduced into its row only:
//  * over the S0 columns alone (kSweepRetained): b_i(S0), the best similarity of every token to a key of
//    S0 more than w positions away, and that key's position.  Only one direction is wanted here, so
//    nothing is gained by computing a pair once for both of its tokens (the sweep of all pairs was slower:
//    288 heads x 16k in three levels 12.0 -> 12.4 ms, 96 problems of 150-3000 tokens at d = 64 98 -> 101 us);
//  * over all columns (kSweepAll), the best over all and over S0, or the twin counts: every pair is
//    computed twice, but a row's result stays in registers, nothing has to be merged, padded or finished.
//    That is the faster sweep for many short sequences (sweep_for in api.cpp).
// Bound by the MFMA.  Mapping onto gfx950:
//  * One workgroup owns RB = kWaves * NSUB * 32 consecutive rows of one problem; each wave holds NSUB
//    32-row blocks of its row keys (scaled by an exact power of two g_i so that ||g_i k_i|| is in
//    (0.5, 1]) as MFMA B operands in registers for the whole sweep.
//  * The columns stream through LDS in double-buffered tiles of TN = 32 * CPT columns from the
//    contiguous copy [slot][DCOL] that the key preparation writes, S0 columns first.
//  * v_mfma_f32_32x32x16_bf16 with A = 32 column keys, B = 32 row keys gives each lane one
//    row i (lane % 32) and 16 columns: register v holds column 8*(v/4) + 4*(lane/32) + v%4.
//  * x = dot * r_j + 3 lies in [2, 4), where the fp32 bit pattern is monotone and the low mantissa
//    bits can carry a column code: one v_max_u32 reduces value and argmax together.  With a running
//    update per chunk the code is the register (4 bits, quantum 2^-18 of the scaled similarity); with
//    one per tile of 4 chunks it also holds the chunk's place in the tile (6 bits, quantum 2^-16), so
//    the compare-and-select of the running update runs once per 128 columns.  Counting, the sign bits of
//    dot * r_j - tau * g_i / r_i are collected and counted 16 at a time.
//  * fp32 keys use the bf16 split k = hi + lo and three products (lo.hi, hi.lo, hi.hi).
//  * A pair's value has the bits of the all-pairs sweep's (scaling a column by a power of two changes
//    no bit), so both sweeps report the same.
#include <type_traits>

#include "sim_common.h"

namespace twinkv {
namespace {

template <int D, bool SPLIT, int NSUB, int CPT, int OCC, int FG>
struct Cfg {
  static_assert(FG == 1 || FG == CPT, "results merge per chunk or per tile");
  static constexpr int WG_PER_CU = OCC * 4 / kWaves;  // OCC waves per SIMD
  // count mode's epilogue holds more registers: at most 2 waves per SIMD
  static constexpr int WG_PER_CU_COUNT = (OCC < 2 ? OCC : 2) * 4 / kWaves;
  static constexpr int DCOL = SPLIT ? 2 * D : D;      // bf16 elements per column in LDS
  static constexpr int UF = DCOL / 16;                // fragments of one key
  static constexpr int MFMAS = SPLIT ? 3 * D / 16 : D / 16;
  static constexpr int PPC = DCOL / 8;                // 16-byte pieces per column
  static constexpr int SWZ = (PPC < 16 ? PPC : 16) - 1;  // piece-index XOR swizzle mask
  // columns sharing one 256-byte LDS bank row (2 at d = 64 bf16), and the period in
  // columns of the swizzle ((column / CPR) & SWZ)
  static constexpr int CPR = DCOL * 2 < 256 ? 256 / (DCOL * 2) : 1;
  static constexpr int SWZ_PERIOD = (SWZ + 1) * CPR;
  static_assert(kChunk % SWZ_PERIOD == 0, "a chunk's columns repeat the swizzle");
  static constexpr int TN = CPT * kChunk;             // columns per LDS tile
  static constexpr int NT = kWaves * 64;
  static constexpr int RB = kWaves * NSUB * 32;       // rows per workgroup
  static constexpr int CHUNK_BYTES = kChunk * DCOL * 2;  // keys of one 32-column chunk
  static constexpr int KEY_BYTES = TN * DCOL * 2;
  static constexpr int STAGE = KEY_BYTES + TN * 4;    // keys + inverse norms
  static constexpr int RETIRED = kWaves * NSUB * 64 * 8;  // S0 results parked in LDS
  static constexpr int LOADS_PER_WAVE = TN * PPC / (kWaves * 64);  // 1-KB direct loads
  // VALU instructions the schedule places beside each MFMA: one chunk's epilogue (about 40
  // with the tile merge, 48 with a running update per chunk) over its MFMAs
  static constexpr int VALU_PER_MFMA = ((FG > 1 ? 40 : 48) + (SPLIT ? 16 : 0) + MFMAS - 1) / MFMAS;
  static_assert((TN * PPC) % (kWaves * 64) == 0, "tile copy must divide evenly");
  static_assert(TN % 64 == 0 && TN <= kWaves * 64, "the inverse norms move in 64-column pieces");
  static_assert(2 * STAGE + RETIRED <= 160 * 1024 / WG_PER_CU,
                "LDS of WG_PER_CU workgroups must fit one CU");
};

// The products of one 32 x 32 block.  fp32 keys hold fragments [hi | lo] on both sides; the two cross
// sums have accumulators of their own and their sum starts the hi.hi chain, as in the all-pairs sweep:
// the same bits for a pair, whichever of its tokens is the row.  (Summed after the chains, twice the
// adds: 64 heads x 16k 5.66 ms at d = 128 and 3.10 at d = 64, against 5.46 and 2.95 here; all products
// in one chain take 5.33 and 2.80, but their bits depend on the order of the two tokens.)
template <int D, bool SPLIT>
struct Block {
  static constexpr int G = D / 16;
  f32x16 y, yq;
  __device__ Block() {
#pragma unroll
    for (int v = 0; v < 16; ++v) y[v] = yq[v] = 0.0f;
  }
  // step t of UF (one fragment of the column is done after it: done(t))
  static __device__ constexpr int done(int t) { return !SPLIT ? t : t < G ? G + t : t - G; }
  template <int UF>
  __device__ void step(const bf16x8 (&col)[UF], const bf16x8 (&row)[UF], int t) {
    if constexpr (!SPLIT) {
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col[t], row[t], y, 0, 0, 0);
    } else if (t < G) {
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col[t], row[G + t], y, 0, 0, 0);
      yq = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col[G + t], row[t], yq, 0, 0, 0);
      if (t == G - 1) {
#pragma unroll
        for (int v = 0; v < 16; ++v) y[v] += yq[v];
      }
    } else {
      y = __builtin_amdgcn_mfma_f32_32x32x16_bf16(col[t - G], row[t - G], y, 0, 0, 0);
    }
  }
};

// Low bits of a packed candidate when the chunks of a group of FG chunks are merged before
// the running update: register slot v (4 bits) and the chunk's place kc in the group,
// coded as LOW - (16 kc + v), so that among equal values the smaller column has the larger
// code.  FG = 1 leaves the plain slot code 15 - v.
template <int FG>
struct Slots {
  static_assert(FG == 1 || FG == 2 || FG == 4, "1, 2 or 4 chunks per group");
  static constexpr int BITS = 4 + (FG >= 2) + (FG >= 4);
  static constexpr uint32_t LOW = (1u << BITS) - 1u;
};

// Value + code of the best column of one lane's 16 accumulators of chunk kc of its group.
template <int FG>
__device__ inline uint32_t chunk_best(const f32x16& acc, const float (&rv)[16], int kc) {
  constexpr uint32_t LOW = Slots<FG>::LOW;
  uint32_t b = 0u;
#pragma unroll
  for (int v = 0; v < 16; ++v) {
    const float x = fmaf(acc[v], rv[v], 3.0f);
    b = max(b, (__float_as_uint(x) & ~LOW) | (LOW - (uint32_t)(16 * kc + v)));
  }
  return b;
}

// Number of a lane's 16 similarities above the row's threshold (count mode, Eq. 2):
// y = dot * r_j + c_i with c_i = -tau * g_i / r_i is positive exactly when sim(i, j) > tau
// (a y of exactly +0, sim equal to tau up to fp32 rounding, counts as above).  Each sign
// bit is shifted into a mask with one v_alignbit (a serial chain the compiler cannot
// reassociate into a wide tree), and one v_bcnt counts them.
__device__ inline uint32_t chunk_count(const f32x16& acc, const float (&rv)[16], float c_row) {
  uint32_t neg = 0u;
#pragma unroll
  for (int v = 0; v < 16; ++v)
    neg = __builtin_amdgcn_alignbit(neg, __float_as_uint(fmaf(acc[v], rv[v], c_row)), 31);
  return 16u - (uint32_t)__builtin_popcount(neg);
}

// Branch-free running update: a strictly larger value (code bits ignored) replaces the
// running best, so an earlier chunk (group) keeps exact ties.  c: its first chunk.
template <int FG>
__device__ inline void run_update(uint32_t best, int c, uint32_t& run, int& cid) {
  constexpr int B = Slots<FG>::BITS;
  const bool upd = (best >> B) > (run >> B);
  run = upd ? best : run;
  cid = upd ? c : cid;
}

// A running best in the per-chunk form: value, slot code 15 - v, chunk index.
template <int FG>
__device__ inline void to_chunk_form(uint32_t& run, int& cid) {
  constexpr uint32_t LOW = Slots<FG>::LOW;
  const uint32_t q = LOW - (run & LOW);
  cid += (int)(q >> 4);
  run = (run & ~LOW) | (15u - (q & 15u));
}

// ALL: over all columns, S0 columns first (else over the S0 columns alone); COUNT (with ALL, without
// an S0 group): the twin counts.
template <int D, bool SPLIT, int NSUB, int CPT, int OCC, int FG, bool ALL, bool COUNT>
__global__ __launch_bounds__(kWaves * 64, (COUNT ? Cfg<D, SPLIT, NSUB, CPT, OCC, FG>::WG_PER_CU_COUNT
                                                 : Cfg<D, SPLIT, NSUB, CPT, OCC, FG>::WG_PER_CU))
void sim_rect_kernel(SimArgs a) {
  using C = Cfg<D, SPLIT, NSUB, CPT, OCC, FG>;
  constexpr uint32_t LOW = Slots<FG>::LOW;
  constexpr bool PARK = ALL && !COUNT;  // two results per row
  static_assert(kGroupAlign % C::TN == 0, "the evicted group must start on a tile boundary");
  __shared__ __attribute__((aligned(1024))) char smem[2 * C::STAGE + (PARK ? C::RETIRED : 0)];

  // ---- which (head, sequence, row block) this workgroup owns --------------------------
  Place pl;
  int part;
  if (!find_place(a, (int)blockIdx.x, pl, part)) return;
  const int len = pl.len, n_ret = pl.n_ret;
  const int ret_chunks = pl.ret_chunks;                // a multiple of CPT
  const int ret_pad = ret_chunks * kChunk;
  const int n_ev = len - n_ret;
  const int nchunks = ALL ? pl.total_chunks : ret_chunks;
  const int ret_real = (n_ret + kChunk - 1) / kChunk;  // S0 chunks with a real column
  const int ncols = nchunks * kChunk;
  const int ntiles = (nchunks + CPT - 1) / CPT;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63;
  const int half = lane >> 5;
  const int l32 = lane & 31;
  const int wrow0 = pl.rb * C::RB + wave * NSUB * 32;

  const uint16_t* pk = a.pkeys + pl.colbase * C::DCOL;
  const int32_t* pc = a.pcol + pl.colbase;
  const int32_t* prk = a.prank + pl.colbase;
  const float* rc = a.rcol + pl.colbase;
  const float* rinv = a.rinv + pl.rowbase;

  // ---- chunks that need the masked epilogue: the window band of this wave's rows and partly
  // padded last chunks.  The columns j with x0 <= j < x1 are one contiguous range per group, read off
  // the S0 prefix counts.
  struct Band {
    int r_lo, r_hi, e_lo, e_hi;  // chunks in the S0 group and (ALL) among the evicted columns
  };
  auto band = [&](int row, int rows) -> Band {
    const int x0 = min(max(row - a.w, 0), len);
    const int x1 = min(max(row + rows + a.w, 0), len);
    const int r0 = prk[x0], r1 = prk[x1];
    Band bd{1, 0, 1, 0};
    bd.r_lo = __builtin_amdgcn_readfirstlane(r0 < r1 ? r0 / kChunk : 1);
    bd.r_hi = __builtin_amdgcn_readfirstlane(r0 < r1 ? (r1 - 1) / kChunk : 0);
    if constexpr (ALL) {
      const int e0 = ret_pad + (x0 - r0), e1 = ret_pad + (x1 - r1);
      bd.e_lo = __builtin_amdgcn_readfirstlane(e0 < e1 ? e0 / kChunk : 1);
      bd.e_hi = __builtin_amdgcn_readfirstlane(e0 < e1 ? (e1 - 1) / kChunk : 0);
    }
    return bd;
  };
  const Band bd = band(wrow0, NSUB * 32);
  // The key preparation fills a group's partial last chunk with copies of its last column (exact ties),
  // so with the tile merge the maximum needs no padding test there; counting does, and the per-chunk
  // configurations keep the test (the masked pass skips the copies by their position -1).
  constexpr bool PAD_TEST = COUNT || FG == 1;
  const int pad_r = PAD_TEST && (n_ret % kChunk) ? n_ret / kChunk : -1;
  const int pad_e = ALL && PAD_TEST && (n_ev % kChunk) ? (ret_pad + n_ev) / kChunk : -1;
  // With the tile merge, the band is also kept per 32-row block: a chunk is dropped and
  // redone only for the row blocks whose own band holds it (the sweep's chunk mask is one
  // scalar operand per chunk and row block either way).
  constexpr bool SUB_BANDS = FG > 1;
  Band sb[NSUB];
  if constexpr (SUB_BANDS) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) sb[s] = band(wrow0 + 32 * s, 32);
  }
  auto in_band = [&](const Band& q, int gc) -> int {
    int in = (int)(gc >= q.r_lo) & (int)(gc <= q.r_hi);
    if constexpr (ALL) in |= (int)(gc >= q.e_lo) & (int)(gc <= q.e_hi);
    return in;
  };
  // Result bits of the CPT chunks of a tile in the main sweep (bit k: keep chunk c0 + k).
  // Dropped: chunks the masked pass redoes, the padding-only chunks that align the S0 group and chunks
  // past the last one.  Branch-free scalar arithmetic, so the tile body stays one straight-line block.
  auto keep_bits = [&](int c0) -> uint32_t {
    // most tiles drop nothing: one range test over the whole tile
    const int c1 = c0 + CPT - 1;
    bool clean = !(c1 >= bd.r_lo && c0 <= bd.r_hi) && !(pad_r >= c0 && pad_r <= c1);
    if constexpr (ALL)
      clean = clean && c1 < nchunks && !(c1 >= ret_real && c0 < ret_chunks) &&
              !(c1 >= bd.e_lo && c0 <= bd.e_hi) && !(pad_e >= c0 && pad_e <= c1);
    else
      clean = clean && c1 < ret_real;
    if (clean) return SUB_BANDS ? (1u << (CPT * NSUB)) - 1u : (1u << CPT) - 1u;
    uint32_t bits = 0u;
#pragma unroll
    for (int kc = 0; kc < CPT; ++kc) {
      const int gc = c0 + kc;
      int common = (int)(gc == pad_r);
      if constexpr (ALL)
        common |= (int)(gc >= nchunks) | ((int)(gc >= ret_real) & (int)(gc < ret_chunks)) | (int)(gc == pad_e);
      else
        common |= (int)(gc >= ret_real);
      if constexpr (SUB_BANDS) {
#pragma unroll
        for (int s = 0; s < NSUB; ++s)
          bits |= (uint32_t)((common | in_band(sb[s], gc)) ^ 1) << (kc * NSUB + s);
      } else {
        bits |= (uint32_t)((common | in_band(bd, gc)) ^ 1) << kc;
      }
    }
    return bits;
  };

  // ---- row keys: MFMA B operands, resident for the whole sweep ------------------------
  bf16x8 bfrag[NSUB][C::UF];
  // Count mode: sim(i, j) > tau  <=>  dot * r_j - tau * g_i / r_i > 0  (per row; a zero key
  // has similarity 0 to every key, so it counts every candidate exactly when tau < 0).
  float thr[NSUB];
  {
    // All of a wave's row loads are issued before any of them is used (one memory round
    // trip).  A row past the end of the sequence reads the last row instead: the results of
    // its lane are never written.  With every column copied, row i is read from its own column in the
    // partitioned copy, which the problem's other row blocks are streaming through this XCD's L2, rather
    // than from the key rows: the same bits, and no fresh lines pushed into L2 (measured about 1% faster
    // on 1k-4k-token sequences).
    float ri[NSUB];
    const uint16_t* src[NSUB];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = min(wrow0 + s * 32 + l32, len - 1);
      if constexpr (ALL) {
        const int r0 = prk[i], r1 = prk[i + 1];
        src[s] = pk + (int64_t)(r1 > r0 ? r0 : ret_pad + (i - r0)) * C::DCOL;
      } else {
        src[s] = (const uint16_t*)a.keys + pl.keybase + (int64_t)i * a.token_stride;
      }
    }
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = min(wrow0 + s * 32 + l32, len - 1);
      ri[s] = rinv[i];
#pragma unroll
      for (int t = 0; t < C::UF; ++t)
        bfrag[s][t] = *reinterpret_cast<const bf16x8*>(src[s] + 16 * t + half * 8);
    }
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const float g = row_scale(ri[s]);
      thr[s] = ri[s] > 0.0f ? -a.tau * g / ri[s] : (a.tau < 0.0f ? INFINITY : -INFINITY);
#pragma unroll
      for (int t = 0; t < C::UF; ++t)
        bfrag[s][t] = __builtin_bit_cast(bf16x8, scale_bf16x8(__builtin_bit_cast(uint4, bfrag[s][t]), g));
    }
  }

  // One running maximum (count) per row block; tb: with FG = CPT, the best of the current tile's chunks
  // so far.  The S0 columns come first; their results are parked in LDS when the sweep reaches the
  // evicted columns.
  uint32_t run[NSUB], tb[NSUB];
  int cid[NSUB];
#pragma unroll
  for (int s = 0; s < NSUB; ++s) {
    run[s] = 0u;
    tb[s] = 0u;
    cid[s] = 0;
  }
  uint2* const parked = reinterpret_cast<uint2*>(smem + 2 * C::STAGE) + wave * NSUB * 64;
  bool park_done = false;
  auto park = [&]() {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      to_chunk_form<FG>(run[s], cid[s]);
      parked[s * 64 + lane] = make_uint2(run[s], (uint32_t)cid[s]);
      run[s] = 0u;
      cid[s] = 0;
    }
    park_done = true;
  };
  // ---- LDS addressing ------------------------------------------------------------------
  // A column's 16-byte piece p is stored in slot p ^ ((column / CPR) & SWZ) of its row, so
  // the lanes that read one piece of consecutive columns in one LDS pass hit distinct banks
  // (with two 128-byte columns per 256-byte bank row at d = 64, the even and the odd columns
  // take the two halves of the row and the swizzle changes every second column).  The
  // swizzle repeats every SWZ_PERIOD columns, which divides 32, so for column c*32 + l32 it
  // only depends on l32: the byte offset of k-step t of a lane's column is a lane constant
  // plus c * (chunk bytes) plus the stage offset.
  int aoff[C::UF];
#pragma unroll
  for (int t = 0; t < C::UF; ++t) {
    const int part = 2 * t + half;
    aoff[t] = l32 * (C::DCOL * 2) + ((part ^ ((l32 / C::CPR) & C::SWZ)) << 4);
  }
  const int roff = C::KEY_BYTES + 16 * half;  // this lane's inverse norms inside a chunk

  auto load_rv = [&](const char* st, int c, float (&rv)[16]) {
#pragma unroll
    for (int g4 = 0; g4 < 4; ++g4) {
      const float4 x = *reinterpret_cast<const float4*>(st + roff + c * kChunk * 4 + 32 * g4);
      rv[4 * g4 + 0] = x.x;
      rv[4 * g4 + 1] = x.y;
      rv[4 * g4 + 2] = x.z;
      rv[4 * g4 + 3] = x.w;
    }
  };

  // ---- column tiles: global -> LDS by direct (asynchronous) loads, double buffered ------
  // Each wave moves LOADS_PER_WAVE blocks of 1 KB with buffer loads; lane l of a block lands
  // at byte 16*l.  Block blk holds columns blk*B .. blk*B+B-1 (B = 64 / PPC), lane l piece
  // l % PPC of column blk*B + l / PPC, stored in slot piece ^ ((column / CPR) & SWZ).  The S0 tiles
  // are whole (the group is padded to kGroupAlign columns); the buffer resource of a tile ends at the
  // problem's last column, so the hardware range check turns loads past it into zeros instead of reads
  // (those columns are dropped).
  constexpr int B = 64 / C::PPC;
  constexpr int NV = C::SWZ_PERIOD / B;  // distinct lane offsets over a wave's blocks
  static_assert(C::SWZ_PERIOD % B == 0 && ((C::LOADS_PER_WAVE * B) % C::SWZ_PERIOD) == 0,
                "the swizzle of a block's columns must repeat with the block index");
  const int lcol = lane / C::PPC;
  int vlane[NV];
#pragma unroll
  for (int r = 0; r < NV; ++r)
    vlane[r] = lcol * (C::DCOL * 2) + 16 * ((lane % C::PPC) ^ (((r * B + lcol) / C::CPR) & C::SWZ));
  auto issue_tile = [&](int tile, int buf) {
    char* st = smem + buf * C::STAGE;
    const int64_t first = (int64_t)tile * C::TN;
    const int cols = ALL ? min(ncols - (int)first, C::TN) : C::TN;  // > 0 for every issued tile
#pragma unroll
    for (int kk = 0; kk < C::LOADS_PER_WAVE; ++kk) {
      // one resource per 1-KB block, based at the block: the range check sees the whole
      // offset of every lane
      const int blk = wave * C::LOADS_PER_WAVE + kk;
      const int bytes = ALL ? min(max(cols * C::DCOL * 2 - blk * 1024, 0), 1024) : 1024;
      load_lds16<0>(tile_rsrc(pk + (first * C::DCOL + blk * 512), bytes), st + blk * 1024, vlane[kk % NV]);
    }
    // The inverse norms in 256-byte pieces, 4 bytes a lane.
    if (wave < C::TN / 64) {
      const int bytes = ALL ? min(max(cols * 4 - wave * 256, 0), 256) : 256;
      load_lds4(tile_rsrc(rc + first + wave * 64, bytes), st + C::KEY_BYTES + wave * 256, 4 * lane);
    }
  };
  auto finish_tile = [&]() {  // wait for this wave's direct loads of the issued tile
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };

  // ---- the pending reduction: the last 32-row block of the previous chunk is reduced
  // while the first MFMA chain of the next chunk runs (software pipelining across chunks).
  f32x16 pacc = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float prv[16];
#pragma unroll
  for (int v = 0; v < 16; ++v) prv[v] = 0.0f;
  int pgc = 0;
  uint32_t pmask = 0u;  // result mask of the pending chunk (zero: dropped)

  // Chunk gc (chunk kc of its tile) into row block s.  With FG = CPT the chunks of a tile
  // are merged in tb first and the tile enters the running best at ``flush``.
  auto reduce_into = [&](const f32x16& acc, const float (&rv)[16], int gc, int kc, int s,
                         uint32_t m) {
    if constexpr (COUNT) {
      run[s] += chunk_count(acc, rv, thr[s]) & m;
    } else if constexpr (FG == 1) {
      const uint32_t best = chunk_best<1>(acc, rv, 0) & m;
      run_update<1>(best, gc, run[s], cid[s]);
    } else {
      tb[s] = max(tb[s], chunk_best<FG>(acc, rv, kc) & m);
    }
  };
  auto flush = [&](int s, int c0) {
    if constexpr (!COUNT && FG > 1) {
      run_update<FG>(tb[s], c0, run[s], cid[s]);
      tb[s] = 0u;
    }
  };

  // One tile: each chain's epilogue runs beside the following chain's MFMAs, and the last
  // chain's epilogue is left pending for the next chunk.  During the last chain, k-step t of
  // the next chunk's A fragments is read into the registers that MFMA t has just consumed.
  auto sweep_tile = [&](auto buf_tag, int c0, uint32_t keep) {
    constexpr int BUF = decltype(buf_tag)::value;
    const char* st = smem + BUF * C::STAGE;
    bf16x8 fc[C::UF];
#pragma unroll
    for (int t = 0; t < C::UF; ++t)
      fc[t] = *reinterpret_cast<const bf16x8*>(st + aoff[t]);
#pragma unroll
    for (int kc = 0; kc < CPT; ++kc) {
      const int gc = c0 + kc;
      const uint32_t m = 0u - ((keep >> kc) & 1u);
      // with bands per row block, the result mask of row block sb for this chunk
      auto mask_of = [&](int sb) -> uint32_t {
        if constexpr (SUB_BANDS) return 0u - ((keep >> (kc * NSUB + sb)) & 1u);
        else return m;
      };
      float rcur[16];
      // with a single row block, chain 0 is also the last chain and carries the prefetch
      const bool pre0 = (NSUB == 1) && (kc + 1 < CPT);
      Block<D, SPLIT> b0;
#pragma unroll
      for (int t = 0; t < C::UF; ++t) {
        b0.step(fc, bfrag[0], t);
        if (pre0)
          fc[Block<D, SPLIT>::done(t)] = *reinterpret_cast<const bf16x8*>(
              st + (kc + 1) * C::CHUNK_BYTES + aoff[Block<D, SPLIT>::done(t)]);
      }
      // the pending chunk: the previous chunk of this tile, or the last of the previous tile
      reduce_into(pacc, prv, pgc, kc == 0 ? CPT - 1 : kc - 1, NSUB - 1, pmask);
      if (kc == 0) flush(NSUB - 1, c0 - CPT);
      load_rv(st, kc, rcur);
#pragma unroll
      for (int i = 0; i < C::MFMAS; ++i) {
        __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
        if (i < 4 || pre0) __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
        __builtin_amdgcn_sched_group_barrier(kSchedValu, C::VALU_PER_MFMA, 0);
      }
      f32x16 x = b0.y;
#pragma unroll
      for (int s = 1; s < NSUB; ++s) {
        Block<D, SPLIT> bs;
        const bool pre = (s == NSUB - 1) && (kc + 1 < CPT);
#pragma unroll
        for (int t = 0; t < C::UF; ++t) {
          bs.step(fc, bfrag[s], t);
          if (pre)
            fc[Block<D, SPLIT>::done(t)] = *reinterpret_cast<const bf16x8*>(
              st + (kc + 1) * C::CHUNK_BYTES + aoff[Block<D, SPLIT>::done(t)]);
        }
        reduce_into(x, rcur, gc, kc, s - 1, mask_of(s - 1));
        if (kc == CPT - 1) flush(s - 1, c0);
#pragma unroll
        for (int i = 0; i < C::MFMAS; ++i) {
          __builtin_amdgcn_sched_group_barrier(kSchedMfma, 1, 0);
          if (pre) __builtin_amdgcn_sched_group_barrier(kSchedDsRead, 1, 0);
          __builtin_amdgcn_sched_group_barrier(kSchedValu, C::VALU_PER_MFMA, 0);
        }
        x = bs.y;
      }
      pacc = x;
#pragma unroll
      for (int v = 0; v < 16; ++v) prv[v] = rcur[v];
      pgc = gc;
      pmask = mask_of(NSUB - 1);
    }
  };

  // A wave whose rows all lie past the end of the sequence (in the last row block of a
  // sequence) only takes its share of the tile loads; its SIMD's MFMA pipe is left to the
  // other workgroup's wave.
  const bool active = wrow0 < len;
#ifdef TWINKV_DEBUG
  // Debug build: both stages and the parked results start as poison.
  {
    uint4* all = reinterpret_cast<uint4*>(smem);
    for (int i = threadIdx.x; i < (int)sizeof(smem) / 16; i += C::NT) all[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
  }
  __syncthreads();
#endif
  if (ntiles > 0) issue_tile(0, 0);
#pragma unroll 1
  for (int tile = 0; tile < ntiles; ++tile) {
    const int buf = tile & 1;
    finish_tile();
    __syncthreads();
    if (tile + 1 < ntiles) issue_tile(tile + 1, buf ^ 1);
    const int c0 = tile * CPT;
    if (PARK && c0 == ret_chunks) {
      // First evicted chunk: finish the pending S0 reduction here and park the S0 results.
      // The opaque copy keeps the compiler from moving the tile body's own pending
      // reduction out of the body to share it with this rare path.
      f32x16 pa = pacc;
      asm volatile("" : "+v"(pa));
      reduce_into(pa, prv, pgc, CPT - 1, NSUB - 1, pmask);
      flush(NSUB - 1, c0 - CPT);
      pmask = 0u;
      park();
    }
    const uint32_t keep = __builtin_amdgcn_readfirstlane(keep_bits(c0));
    if (active) {
      if (buf == 0) sweep_tile(std::integral_constant<int, 0>{}, c0, keep);
      else sweep_tile(std::integral_constant<int, 1>{}, c0, keep);
    }
#ifdef TWINKV_DEBUG
    // Debug build: once every wave has swept this stage, fill it with 0xFF bytes (NaN keys
    // and inverse norms) before the next tile's loads refill it.  A read of a
    // stage outside its tile's lifetime then sees the poison, and the results differ from
    // the normal build's.
    __syncthreads();
    {
      uint4* stg = reinterpret_cast<uint4*>(smem + buf * C::STAGE);
      for (int i = threadIdx.x; i < C::STAGE / 16; i += C::NT)
        stg[i] = make_uint4(~0u, ~0u, ~0u, ~0u);
    }
    __syncthreads();
#endif
  }
  reduce_into(pacc, prv, pgc, CPT - 1, NSUB - 1, pmask);
  flush(NSUB - 1, (ntiles - 1) * CPT);
  if (PARK && !park_done) park();  // no evicted columns were swept
  if constexpr (!COUNT) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) to_chunk_form<FG>(run[s], cid[s]);
  }
  if (!active) return;

  // ---- masked pass: the chunks holding window pairs or padding next to real columns, read
  // straight from the column copy, with the window / padding test per element.  Chunks are
  // visited out of order here, so equal values keep the smaller chunk index explicitly.
  //
  // Maximum with the tile merge: in each group the columns whose positions lie within w of a
  // lane's row form one contiguous range of column indices, read off the S0 prefix counts,
  // so the test per element is one unsigned range compare and the position list is not read.
  // The copies of a group's last column in its partly filled last chunk are excluded with
  // that column (and otherwise only tie with it).
  constexpr bool RANGE_TEST = !COUNT && FG > 1;
  // S0 prefix counts at the two ends of each row's window (loaded here, used once the first
  // chunks' loads are in flight)
  int wrx[NSUB], wry[NSUB];
  if constexpr (RANGE_TEST) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = min(wrow0 + s * 32 + l32, len - 1);
      wrx[s] = prk[max(i - a.w, 0)];
      wry[s] = prk[min(i + a.w + 1, len)];
    }
  }
  // First excluded column and number of excluded columns of row block s's lane row in group grp.
  auto excluded_range = [&](int grp, int s, int& lo, int& num) {
    // opaque copies: computed here, in each chunk's step, not hoisted ahead of the chunk loads
    int rx = wrx[s], ry = wry[s];
    asm volatile("" : "+v"(rx), "+v"(ry));
    if (grp == 0) {
      lo = rx;
      num = (ry == n_ret ? ret_pad : ry) - lo;
    } else {
      const int i = min(wrow0 + s * 32 + l32, len - 1);
      lo = ret_pad + max(i - a.w, 0) - rx;
      const int e = ret_pad + min(i + a.w + 1, len) - ry;
      num = (e == ret_pad + n_ev ? ncols : e) - lo;
    }
  };
  struct MaskedChunk {  // one chunk's A fragments and column tables, in registers (two
                        // chunks per memory round trip measured slower)
    bf16x8 af[C::UF];
    float rv[16];
    int jv[16];
  };
  auto masked_load = [&](int gc, MaskedChunk& mc) {
    const int col = gc * kChunk + l32;
#pragma unroll
    for (int t = 0; t < C::UF; ++t)
      mc.af[t] = *reinterpret_cast<const bf16x8*>(pk + (int64_t)col * C::DCOL + 16 * t + 8 * half);
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int cc = gc * kChunk + slot_row(v, half);
      mc.rv[v] = rc[cc];
      mc.jv[v] = RANGE_TEST ? 0 : pc[cc];
    }
  };
  auto masked_compute = [&](int gc, int grp, const MaskedChunk& mc, uint32_t (&rs)[NSUB], int (&cs)[NSUB]) {
    const bf16x8 (&af)[C::UF] = mc.af;
    const float (&rv)[16] = mc.rv;
    const int (&jv)[16] = mc.jv;
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      if constexpr (SUB_BANDS) {
        // only the row blocks that dropped this chunk in the sweep
        const bool need = grp == 0 ? (gc == pad_r || (gc >= sb[s].r_lo && gc <= sb[s].r_hi))
                                   : (gc == pad_e || (gc >= sb[s].e_lo && gc <= sb[s].e_hi));
        if (!need) continue;
      }
      Block<D, SPLIT> b;
#pragma unroll
      for (int t = 0; t < C::UF; ++t) b.step(af, bfrag[s], t);
      const f32x16 x = b.y;
      const int i = wrow0 + s * 32 + l32;
      if constexpr (COUNT) {
        uint32_t c = 0u;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const uint32_t ok = (uint32_t)(jv[v] >= 0) & (uint32_t)(abs(i - jv[v]) > a.w);
          c += ok & ((~__float_as_uint(fmaf(x[v], rv[v], thr[s]))) >> 31);
        }
        rs[s] += c;
      } else {
        uint32_t best = 0u;
        // column of slot v, relative to the first excluded column of this row's range
        int xlo = 0, xnum = 0;
        if constexpr (RANGE_TEST) excluded_range(grp, s, xlo, xnum);
        const uint32_t rel = (uint32_t)(gc * kChunk + 4 * half - xlo);
        const uint32_t nex = (uint32_t)xnum;
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const float y = fmaf(x[v], rv[v], 3.0f);
          const uint32_t u = (__float_as_uint(y) & ~LOW) | (uint32_t)(15 - v);
          bool ok;
          if constexpr (RANGE_TEST) ok = rel + (uint32_t)(8 * (v >> 2) + (v & 3)) >= nex;
          else ok = (jv[v] >= 0) & (abs(i - jv[v]) > a.w);
          best = max(best, ok ? u : 0u);
        }
        const bool upd = (best >> 4) > (rs[s] >> 4) ||
                         ((best >> 4) == (rs[s] >> 4) && best >= kValidMin && gc < cs[s]);
        rs[s] = upd ? best : rs[s];
        cs[s] = upd ? gc : cs[s];
      }
    }
  };
  // The band's chunks [lo, hi] of a group, then its padded last chunk unless the band holds it.
  auto masked_range = [&](int lo, int hi, int pad, int grp, uint32_t (&rs)[NSUB], int (&cs)[NSUB]) {
    const int nband = max(hi - lo + 1, 0);
    const int nmask = nband + (int)(pad >= 0 && !(pad >= lo && pad <= hi));
#pragma unroll 1
    for (int k = 0; k < nmask; ++k) {
      const int gc = k < nband ? lo + k : pad;
      MaskedChunk mc;
      masked_load(gc, mc);
      masked_compute(gc, grp, mc, rs, cs);
    }
  };
  // the live registers: the evicted columns, or the S0 columns when they are the only ones
  if constexpr (ALL) masked_range(bd.e_lo, bd.e_hi, pad_e, 1, run, cid);
  else masked_range(bd.r_lo, bd.r_hi, pad_r, 0, run, cid);

  // ---- resolve: lanes l and l+32 hold the same row over disjoint column halves ----------
  if constexpr (COUNT) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = wrow0 + s * 32 + l32;
      const uint32_t total = run[s] + __shfl_xor(run[s], 32);
      if (half == 0 && i < len) a.counts[pl.rowbase + i] = (int32_t)total;
    }
    return;
  }
  // value (0: no candidate) and slot of a running best of group grp
  auto resolve = [&](uint32_t r, int c, int grp, uint32_t& v, int& p) {
    v = r & ~LOW;
    p = c * kChunk + slot_row(15 - (int)(r & 15u), half);
    // a slot past the group's last column holds a copy of that column
    if constexpr (FG > 1) p = min(p, grp == 0 ? n_ret - 1 : ret_pad + n_ev - 1);
    const uint32_t v2 = __shfl_xor(v, 32);
    const int p2 = __shfl_xor(p, 32);
    if (v2 > v || (v2 == v && p2 < p)) { v = v2; p = p2; }
  };
  if constexpr (!ALL) {
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = wrow0 + s * 32 + l32;
      uint32_t v;
      int p;
      resolve(run[s], cid[s], 0, v, p);
      if (half == 0 && i < len) {
        const int64_t o = pl.rowbase + i;
        const bool any = v >= kValidMin;
        if (a.best_ret) a.best_ret[o] = any ? similarity(v, rinv[i]) : -1.0f;
        if (a.arg_ret) a.arg_ret[o] = any ? pc[p] : -1;
      }
    }
  } else {
    uint32_t rr[NSUB];
    int rcid[NSUB];
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const uint2 v = parked[s * 64 + lane];
      rr[s] = v.x;
      rcid[s] = (int)v.y;
    }
    masked_range(bd.r_lo, bd.r_hi, pad_r, 0, rr, rcid);
#pragma unroll
    for (int s = 0; s < NSUB; ++s) {
      const int i = wrow0 + s * 32 + l32;
      uint32_t vr, ve;
      int pr, pe;
      resolve(rr[s], rcid[s], 0, vr, pr);
      resolve(run[s], cid[s], 1, ve, pe);
      if (half == 0 && i < len) {
        const int64_t o = pl.rowbase + i;
        const float ri = rinv[i];
        const int jr = vr >= kValidMin ? pc[pr] : -1;
        const int je = ve >= kValidMin ? pc[pe] : -1;
        if (a.best_ret) a.best_ret[o] = jr >= 0 ? similarity(vr, ri) : -1.0f;
        if (a.arg_ret) a.arg_ret[o] = jr;
        const bool take_r = jr >= 0 && (je < 0 || vr > ve || (vr == ve && jr < je));
        const int j = take_r ? jr : je;
        if (a.best_all) a.best_all[o] = j >= 0 ? similarity(take_r ? vr : ve, ri) : -1.0f;
        if (a.arg_all) a.arg_all[o] = j;
      }
    }
  }
}

template <int D, bool SPLIT, int NSUB, int CPT, int OCC, int FG>
hipError_t run(const SimArgs& a, hipStream_t st) {
  using C = Cfg<D, SPLIT, NSUB, CPT, OCC, FG>;
  const int64_t groups = a.n_heads >= 8 ? 8LL * ((a.n_heads + 7) / 8) : (int64_t)a.n_heads;
  const int64_t blocks = groups * a.total_tiles;
  if (blocks == 0) return hipSuccess;
  const dim3 grid((unsigned)blocks), block(C::NT);
  if (a.sweep == kSweepRetained)
    hipLaunchKernelGGL((sim_rect_kernel<D, SPLIT, NSUB, CPT, OCC, FG, false, false>), grid, block, 0, st, a);
  else if (a.counts == nullptr)
    hipLaunchKernelGGL((sim_rect_kernel<D, SPLIT, NSUB, CPT, OCC, FG, true, false>), grid, block, 0, st, a);
  else if constexpr (!SPLIT)  // (sweep_for counts fp32 keys over the pairs only)
    hipLaunchKernelGGL((sim_rect_kernel<D, SPLIT, NSUB, CPT, OCC, FG, true, true>), grid, block, 0, st, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Tile shapes: (d, fp32 split, NSUB 32-row blocks per wave, 32-column chunks per LDS tile, waves per
// SIMD, chunks merged before each running update: 1 or the chunks per tile).  Overridable at build
// time for tuning sweeps.
#ifndef TWINKV_RECT_BF16_128
#define TWINKV_RECT_BF16_128 128, false, 3, 4, 2, 4
#endif
#ifndef TWINKV_RECT_BF16_64
#define TWINKV_RECT_BF16_64 64, false, 4, 2, 3, 1
#endif
#ifndef TWINKV_RECT_F32_64
#define TWINKV_RECT_F32_64 64, true, 1, 4, 2, 1
#endif
#ifndef TWINKV_RECT_F32_128
#define TWINKV_RECT_F32_128 128, true, 1, 2, 2, 1
#endif
static_assert(Cfg<TWINKV_RECT_BF16_128>::RB == sim_rect_rows_per_block(0, 128) &&
                  Cfg<TWINKV_RECT_BF16_64>::RB == sim_rect_rows_per_block(0, 64) &&
                  Cfg<TWINKV_RECT_F32_64>::RB == sim_rect_rows_per_block(1, 64) &&
                  Cfg<TWINKV_RECT_F32_128>::RB == sim_rect_rows_per_block(1, 128),
              "the sequence table counts these row blocks");

}  // namespace

int launch_sim_rect(const SimArgs& a, int dtype, int d, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (dtype == 0 && d == 128) return run<TWINKV_RECT_BF16_128>(a, st);
  if (dtype == 0 && d == 64) return run<TWINKV_RECT_BF16_64>(a, st);
  if (dtype == 1 && d == 64) return run<TWINKV_RECT_F32_64>(a, st);
  if (dtype == 1 && d == 128) return run<TWINKV_RECT_F32_128>(a, st);
  return hipErrorInvalidValue;
}

}  // namespace twinkv
