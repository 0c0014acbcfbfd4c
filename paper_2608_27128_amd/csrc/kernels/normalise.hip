// K1a: per-problem stable partition of the positions into [S0 | evicted] column lists (the
//      S0 list padded to a multiple of kGroupAlign columns, the evicted list to whole
//      32-column chunks), from the retained mask alone.
// K1b: one pass over the keys: per-key inverse l2 norm (Sec. 3.2: k_hat = k / ||k||_2), and
//      the key itself copied to its slot of the partitioned column list (bf16; for fp32 keys
//      the bf16 hi/lo split that the similarity sweeps multiply on bf16 MFMA).
//
// K1a reads 1 byte and writes 8 bytes per key.  K1b is an HBM stream: it reads d*esize bytes
// (+5 bytes of mask and rank) and writes d*2 (d*4 for fp32) + 8 bytes per key; for the pair sweep
// 16 bytes of cleared candidates more (4 of cleared counts), for the S0 sweep only the S0 keys (and fp32
// keys' row plane).
#include <hip/hip_runtime.h>

#include <algorithm>
#include <type_traits>

#include "../twinkv_internal.h"
#include "key_scale.h"

namespace twinkv {
namespace {

__device__ inline uint16_t bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ inline float bf16_to_f32(uint16_t h) { return __uint_as_float((uint32_t)h << 16); }

template <int NT>
__device__ inline int block_sum(int v, int* s_red) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) v += __shfl_xor(v, off);
  const int wv = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) s_red[wv] = v;
  __syncthreads();
  int tot = 0;
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) tot += s_red[k];
  __syncthreads();
  return tot;
}

// The sequence table reaches the device with the partition: up to kTableArgs sequences as an argument of
// the kernel (ARGS), whose workgroups of head 0 write it to the workspace for the kernels that follow, which
// saves a launch (a call on one short sequence is bound by its launches: repair of 1 head x 512 tokens,
// fp32 keys, 39.4 -> 35.9 us); a longer table is uploaded first.
constexpr int kTableArgs = 16;
struct TableArgs {
  SeqInfo s[kTableArgs];
};
struct TableUploaded {};
template <bool ARGS>
using Table = typename std::conditional<ARGS, TableArgs, TableUploaded>::type;
template <bool ARGS>
__device__ inline SeqInfo sequence_of(const Table<ARGS>& table, SeqInfo* seqtab, int h, int s) {
  if constexpr (ARGS) {
    const SeqInfo si = table.s[s];
    if (h == 0 && threadIdx.x == 0) seqtab[s] = si;
    return si;
  } else {
    return seqtab[s];
  }
}

// One workgroup of kLongThreads threads per (head, sequence) problem, for batches with long sequences.
constexpr int kLongThreads = 1024;
template <bool ARGS>
__global__ __launch_bounds__(kLongThreads) void partition_kernel(
    const uint8_t* __restrict__ retained, const Table<ARGS> table, SeqInfo* __restrict__ seqtab, int n_seqs,
    int64_t T, int64_t PT, int32_t* __restrict__ pcol, float* __restrict__ rcol,
    int32_t* __restrict__ prank, ProblemMeta* __restrict__ pmeta, int32_t* __restrict__ status) {
  constexpr int NT = kLongThreads;
  __shared__ int s_red[NT / 64];
  __shared__ int s_wave[NT / 64];
  const int q = blockIdx.x;
  const int h = q / n_seqs;
  const int s = q - h * n_seqs;
  const SeqInfo si = sequence_of<ARGS>(table, seqtab, h, s);
  const int len = si.len;
  const uint8_t* ret = retained ? retained + h * T + si.start : nullptr;
  int32_t* pc = pcol + h * PT + si.perm_off;
  float* rc = rcol + h * PT + si.perm_off;
  int32_t* pr = prank + h * PT + si.perm_off;

  int cnt = 0;
  if (ret != nullptr)
    for (int t = threadIdx.x; t < len; t += NT) cnt += (ret[t] != 0);
  const int n_ret = block_sum<NT>(cnt, s_red);
  const int ret_pad = (n_ret + kGroupAlign - 1) / kGroupAlign * kGroupAlign;
  const int n_ev = len - n_ret;
  const int ev_pad = (n_ev + kChunk - 1) / kChunk * kChunk;

  const int lane = threadIdx.x & 63;
  const int wv = threadIdx.x >> 6;
  int ret_before_round = 0;
  for (int t0 = 0; t0 < len; t0 += NT) {
    const int t = t0 + threadIdx.x;
    const bool in = t < len;
    const bool r = in && ret != nullptr && ret[t] != 0;
    const unsigned long long bal = __ballot(r);
    const int pre = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) s_wave[wv] = __popcll(bal);
    __syncthreads();
    int wbase = 0, tot = 0;
#pragma unroll
    for (int k = 0; k < NT / 64; ++k) {
      const int c = s_wave[k];
      wbase += (k < wv) ? c : 0;
      tot += c;
    }
    if (in) {
      const int ret_before = ret_before_round + wbase + pre;
      pc[r ? ret_before : ret_pad + (t - ret_before)] = t;
      pr[t] = ret_before;
    }
    ret_before_round += tot;
    __syncthreads();
  }
  // padding columns: no position, inverse norm 0 (their keys are never used)
  for (int k = n_ret + (int)threadIdx.x; k < ret_pad; k += NT) {
    pc[k] = -1;
    rc[k] = 0.0f;
  }
  for (int k = ret_pad + n_ev + (int)threadIdx.x; k < ret_pad + ev_pad; k += NT) {
    pc[k] = -1;
    rc[k] = 0.0f;
  }
  if (threadIdx.x == 0) {
    pr[len] = n_ret;
    ProblemMeta m;
    m.n_ret = n_ret;
    m.ret_chunks = ret_pad / kChunk;
    m.total_chunks = (ret_pad + ev_pad) / kChunk;
    m.flags = 0;
    pmeta[q] = m;
    if (status) status[q] = 0;
  }
}

// Sequences of at most kShortLen tokens: all of a thread's mask bytes in one round of loads, the
// waves' ballot counts scanned by one wave, two barriers in all (the slab-by-slab kernel takes two
// per 256 tokens: 9.0 against 5.5 us for 12 x 8 problems of 150 to 3000 tokens, where it is one
// of few short kernels in a row).  ROUNDS of 256 tokens each: 16, or 4 where no sequence is longer, so
// that many short problems don't pay for empty rounds (2048 problems of 240-300 tokens: 6.4 us with 16,
// 5.6 with 4, 5.7 slab by slab).
constexpr int kShortLen = 4096;
template <int ROUNDS, bool ARGS>
__global__ __launch_bounds__(256) void partition_short_kernel(
    const uint8_t* __restrict__ retained, const Table<ARGS> table, SeqInfo* __restrict__ seqtab, int n_seqs,
    int64_t T, int64_t PT, int32_t* __restrict__ pcol, float* __restrict__ rcol,
    int32_t* __restrict__ prank, ProblemMeta* __restrict__ pmeta, int32_t* __restrict__ status) {
  constexpr int U = ROUNDS;
  static_assert(U * 4 <= 64, "one count per lane of the scanning wave");
  __shared__ int s_cnt[U * 4], s_pre[U * 4], s_total;
  const int q = blockIdx.x;
  const int h = q / n_seqs;
  const int s = q - h * n_seqs;
  const SeqInfo si = sequence_of<ARGS>(table, seqtab, h, s);
  const int len = si.len;
  const int lane = threadIdx.x & 63, wv = threadIdx.x >> 6;
  const uint8_t* ret = retained ? retained + h * T + si.start : nullptr;
  int32_t* pc = pcol + h * PT + si.perm_off;
  float* rc = rcol + h * PT + si.perm_off;
  int32_t* pr = prank + h * PT + si.perm_off;
  uint8_t m[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * 256 + (int)threadIdx.x;
    m[u] = ret != nullptr && t < len ? ret[t] : 0;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int c = __popcll(__ballot(m[u] != 0));
    if (lane == 0) s_cnt[u * 4 + wv] = c;
  }
  __syncthreads();
  if (wv == 0) {
    const int v = lane < U * 4 ? s_cnt[lane] : 0;
    int inc = v;
#pragma unroll
    for (int off = 1; off < 64; off <<= 1) {
      const int y = __shfl_up(inc, off);
      if (lane >= off) inc += y;
    }
    if (lane < U * 4) s_pre[lane] = inc - v;
    if (lane == 63) s_total = inc;
  }
  __syncthreads();
  const int n_ret = s_total;
  const int ret_pad = (n_ret + kGroupAlign - 1) / kGroupAlign * kGroupAlign;
  const int n_ev = len - n_ret;
  const int ev_pad = (n_ev + kChunk - 1) / kChunk * kChunk;
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int t = u * 256 + (int)threadIdx.x;
    if (u * 256 >= len) break;  // uniform over the block
    const unsigned long long bal = __ballot(m[u] != 0);
    const int before = s_pre[u * 4 + wv] + __popcll(bal & ((1ull << lane) - 1ull));
    if (t < len) {
      pc[m[u] != 0 ? before : ret_pad + (t - before)] = t;
      pr[t] = before;
    }
  }
  // padding columns: no position, r' 0 until the key preparation copies the last column there
  for (int k = n_ret + (int)threadIdx.x; k < ret_pad; k += 256) {
    pc[k] = -1;
    rc[k] = 0.0f;
  }
  for (int k = ret_pad + n_ev + (int)threadIdx.x; k < ret_pad + ev_pad; k += 256) {
    pc[k] = -1;
    rc[k] = 0.0f;
  }
  if (threadIdx.x == 0) {
    pr[len] = n_ret;
    ProblemMeta mt;
    mt.n_ret = n_ret;
    mt.ret_chunks = ret_pad / kChunk;
    mt.total_chunks = (ret_pad + ev_pad) / kChunk;
    mt.flags = 0;
    pmeta[q] = mt;
    if (status) status[q] = 0;
  }
}

// LPT lanes cooperate on one key; each lane owns 16 contiguous bytes of it.  A workgroup
// takes kPrepIter groups of TPB consecutive tokens of one (head, sequence) problem, all their
// loads issued before any is used.  blockIdx.y is the head; blockIdx.x runs over the
// workgroups of all sequences (seqtab[s].prep_blk0 = the first one of sequence s), so no
// workgroup is launched past the end of a short sequence.  Key reads are nontemporal (each byte is
// touched once here).  So are the writes of whole bf16 rows, issued before the norms are summed (8 heads x
// 16 sequences of 400-512 tokens, d = 128: 14.9 -> 10.4 us; three levels of 64 heads x 16k: 105 ->
// 95 us).  The writes for kSweepPairs are not, as neighbouring workgroups complete each other's lines
// in L2 (ragged batch of 64 sequences of 1k-4k tokens, 288 heads: 5.3 ms with nontemporal writes, 5.0
// ms without; 4.3 ms with the rows written whole, which the sweep then pays for with swizzled, slower
// tile loads and uncoalesced row loads).
constexpr int kPrepIter = 4;

typedef unsigned int prep_u32x4 __attribute__((ext_vector_type(4)));

// p moved by a byte offset (one level group's array from group 0's)
template <typename T>
__device__ inline T* byte_offset(T* p, int64_t bytes) {
  using C = typename std::conditional<std::is_const<T>::value, const char, char>::type;
  return reinterpret_cast<T*>(reinterpret_cast<C*>(p) + bytes);
}

__device__ inline uint4 prep_load16(const uint8_t* p) {
  const prep_u32x4 v = __builtin_nontemporal_load(reinterpret_cast<const prep_u32x4*>(p));
  return make_uint4(v.x, v.y, v.z, v.w);
}
__device__ inline void prep_store16(char* p, uint4 x) {
  *reinterpret_cast<uint4*>(p) = x;
}
__device__ inline void prep_store16_nt(char* p, uint4 x) {
  const prep_u32x4 v = {x.x, x.y, x.z, x.w};
  __builtin_nontemporal_store(v, reinterpret_cast<prep_u32x4*>(p));
}

// LEVELS: the groups of nested retained sets in one pass (PrepLevels): each token goes to
// the column list of its own group, whose arrays lie group_stride bytes after the previous
// group's; rinv (and the fp32 row plane) is written once for all groups.  Without LEVELS,
// `retained` splits the positions into the one S0 list and the evicted list.  ALL: the copy of
// kSweepPairs; without it, evicted columns are copied as copy_evicted says.
template <int D, bool F32, bool LEVELS, bool ALL>
__global__ __launch_bounds__(256) void prepare_keys_kernel(
    const uint8_t* __restrict__ keys, int64_t T, int64_t hs_bytes, int64_t ts_bytes, int64_t PT,
    const uint8_t* __restrict__ retained, const int32_t* __restrict__ prank,
    ProblemMeta* __restrict__ pmeta, const SeqInfo* __restrict__ seqtab, int n_seqs,
    float* __restrict__ rinv, float* __restrict__ rcol, uint16_t* __restrict__ hilo,
    uint16_t* __restrict__ pkeys, int32_t* __restrict__ status, int h0, int copy_evicted,
    unsigned long long* __restrict__ best, int32_t* __restrict__ counts, int64_t plane, int total_blocks,
    PrepLevels lv) {
  constexpr int ESZ = F32 ? 4 : 2;
  constexpr int LPT = D * ESZ / 16;
  constexpr int TPB = 256 / LPT;
  constexpr int DCOL = F32 ? 2 * D : D;
  static_assert(LPT <= 64 && (64 % LPT) == 0, "a key must fit inside one wave");
  const int64_t h = h0 + (int64_t)blockIdx.y;
  const int bx = prep_block((int)blockIdx.x, (int)blockIdx.y, (int)gridDim.x, total_blocks);
  if (bx >= total_blocks) return;
  int lo = 0, hi = n_seqs - 1;  // the last sequence whose first workgroup is <= bx
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (seqtab[mid].prep_blk0 <= bx) lo = mid; else hi = mid - 1;
  }
  const int s = lo;
  const int q = (int)h * n_seqs + s;
  const SeqInfo si = seqtab[s];
  const int sub = threadIdx.x % LPT;
  const int tfirst = (bx - si.prep_blk0) * (TPB * kPrepIter) + threadIdx.x / LPT;
  const int64_t base = h * PT + si.perm_off;
  const int ret_cols = LEVELS ? 0 : pmeta[q].ret_chunks * kChunk;
  const int n_ret0 = LEVELS ? 0 : pmeta[q].n_ret;
  // With ALL the scaled keys pass through LDS ([row][piece], pieces swizzled by the row so that a
  // piece of 16 consecutive rows lies in distinct banks), with the workgroup's tokens of one column
  // list on neighbouring rows, and leave piece by piece, lanes along the rows: they are neighbours
  // in the copy's layout too, so a wave writes runs of up to 1 KB (written token by token, the
  // 16-byte pieces of a key lie 512 bytes apart: ragged batch of 64 sequences of 1k-4k tokens, this
  // kernel 5.7 ms).  The S0 columns alone are too few for runs and leave token by token.
  constexpr int TOK = TPB * kPrepIter;
  constexpr int PPC = DCOL / 8;
  constexpr int SWZ = (PPC < 16 ? PPC : 16) - 1;
  constexpr int CPR = DCOL * 2 < 256 ? 256 / (DCOL * 2) : 1;
  __shared__ __attribute__((aligned(16))) char s_keys[ALL ? TOK * DCOL * 2 : 16];
  __shared__ int64_t s_dst[ALL ? TOK : 1];  // byte offset of the row's slot from the problem's copy
  const int t_first = (bx - si.prep_blk0) * TOK, t_end = min(t_first + TOK, si.len);
  const int rank0 = prank[base + t_first], n_here = prank[base + t_end] - rank0;
  auto lds_piece = [&](int row, int piece) -> char* {
    return s_keys + row * (DCOL * 2) + ((piece ^ ((row / CPR) & SWZ)) << 4);
  };
  auto slot_bytes = [](int slot) -> int64_t {
    return (int64_t)(slot / kChunk) * (kChunk * DCOL * 2) + (slot % kChunk) * 16;
  };

  uint4 raw[kPrepIter];
#pragma unroll
  for (int it = 0; it < kPrepIter; ++it) {
    const int tl = tfirst + it * TPB;
    raw[it] = make_uint4(0, 0, 0, 0);
    if (tl < si.len)
      raw[it] = prep_load16(keys + h * hs_bytes + (si.start + tl) * ts_bytes + sub * 16);
  }
#pragma unroll
  for (int it = 0; it < kPrepIter; ++it) {
    const int tl = tfirst + it * TPB;
    const bool valid = tl < si.len;
    const int64_t tt = si.start + (valid ? tl : 0);
    // this token's column list: its group's (LEVELS) or the single split's
    int64_t goff = 0;
    bool r;
    int n_ret = n_ret0;
    if constexpr (LEVELS) {
      const int l = lv.level[h * T + tt];
      const int g = (l >= 1 && l <= lv.n_levels) ? l - 1
                    : (lv.n_groups > lv.n_levels ? lv.n_levels : -1);
      r = g >= 0;                      // a member of its group's list; else copied nowhere
      goff = (int64_t)(r ? g : 0) * lv.group_stride;
      n_ret = byte_offset(pmeta, goff)[q].n_ret;
    } else {
      r = retained != nullptr && retained[h * T + tt] != 0;
    }
    const int pr = byte_offset(prank, goff)[base + (valid ? tl : 0)];
    const int p = r ? pr : ret_cols + ((valid ? tl : 0) - pr);
    const bool copy = valid && (r || ALL || copy_evicted);  // evicted columns only for all-keys sweeps
    // The last column of a group fills the rest of the group's padding (S0: up to kGroupAlign
    // columns, evicted: its 32-column chunk) with copies of itself (key and r'; the position
    // list keeps -1 there), so the padding holds only exact ties of a real column.
    const int last = r ? n_ret - 1 : ret_cols + (si.len - n_ret) - 1;
    const int unit = ALL && r ? kGroupAlign : kChunk;
    const int fill_end = (p == last && copy) ? (p / unit + 1) * unit : p + 1;
    const int row = r ? pr - rank0 : n_here + (tl - t_first) - (pr - rank0);  // the token's row
    float* const grcol = byte_offset(rcol, goff);
    uint16_t* const gkeys = byte_offset(pkeys, goff);

    if constexpr (!ALL && !F32) {
      for (int k = p; copy && k < fill_end; ++k)
        prep_store16_nt(reinterpret_cast<char*>(gkeys + (base + k) * DCOL + sub * 8), raw[it]);
    }
    double ss = 0.0;
    if constexpr (F32) {
      const float v[4] = {__uint_as_float(raw[it].x), __uint_as_float(raw[it].y),
                          __uint_as_float(raw[it].z), __uint_as_float(raw[it].w)};
#pragma unroll
      for (int e = 0; e < 4; ++e) ss += (double)v[e] * (double)v[e];
    } else {
      const uint32_t wds[4] = {raw[it].x, raw[it].y, raw[it].z, raw[it].w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const double x0 = (double)__uint_as_float(wds[e] << 16);
        const double x1 = (double)__uint_as_float(wds[e] & 0xFFFF0000u);
        ss += x0 * x0 + x1 * x1;
      }
    }
#pragma unroll
    for (int off = LPT / 2; off > 0; off >>= 1) ss += __shfl_xor(ss, off, LPT);
    const bool bad = !(ss < 1.0e300);  // NaN or Inf in the key
    float rv;
    if (bad) rv = __uint_as_float(0x7FC00000u);
    else if (ss > 0.0) rv = (float)(1.0 / sqrt(ss));
    else rv = 0.0f;                    // zero key: similarity 0 to all
    const float g = ALL ? row_scale(rv) : 1.0f;  // (ALL) the copy's norm lies in (0.5, 1]

    if constexpr (F32) {
      const float v[4] = {__uint_as_float(raw[it].x) * g, __uint_as_float(raw[it].y) * g,
                          __uint_as_float(raw[it].z) * g, __uint_as_float(raw[it].w) * g};
      uint16_t hs[4], ls[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        hs[e] = bf16_rne(v[e]);
        ls[e] = bf16_rne(v[e] - bf16_to_f32(hs[e]));  // v - hi is exact in fp32
      }
      if (valid) {
        uint2 phi, plo;
        phi.x = hs[0] | ((uint32_t)hs[1] << 16);
        phi.y = hs[2] | ((uint32_t)hs[3] << 16);
        plo.x = ls[0] | ((uint32_t)ls[1] << 16);
        plo.y = ls[2] | ((uint32_t)ls[3] << 16);
        if constexpr (!ALL) {
          if (!copy_evicted) {  // (else the rows are read from the copy)
            uint16_t* plane_row = hilo + (h * T + tt) * (2 * D) + sub * 4;
            *reinterpret_cast<uint2*>(plane_row) = phi;
            *reinterpret_cast<uint2*>(plane_row + D) = plo;
          }
          for (int k = p; copy && k < fill_end; ++k) {
            uint16_t* dk = gkeys + (base + k) * DCOL + sub * 4;
            *reinterpret_cast<uint2*>(dk) = phi;
            *reinterpret_cast<uint2*>(dk + D) = plo;
          }
        } else {
          *reinterpret_cast<uint2*>(lds_piece(row, sub / 2) + 8 * (sub & 1)) = phi;
          *reinterpret_cast<uint2*>(lds_piece(row, D / 8 + sub / 2) + 8 * (sub & 1)) = plo;
        }
      }
    } else {
      if constexpr (ALL) {
        if (valid) *reinterpret_cast<uint4*>(lds_piece(row, sub)) = scale_bf16x8(raw[it], g);
      }
    }
    if (ALL && valid && sub == 0) s_dst[row] = slot_bytes(p);
    if (valid && sub == 0) {
      rinv[h * T + tt] = rv;
      // (a token in no group of the LEVELS pass has no column anywhere)
      for (int k = p; (copy || !LEVELS) && k < fill_end; ++k) grcol[base + k] = rv / g;
      if (bad) {
        for (int g = 0; g < (LEVELS ? lv.n_groups : 1); ++g)  // every list of the problem
          atomicOr(&byte_offset(pmeta, (int64_t)g * lv.group_stride)[q].flags, kFlagNonfinite);
        if (status) status[q] = 2;  // TWINKV_PROBLEM_NONFINITE
      }
    }
  }
  if constexpr (ALL) {
    __syncthreads();
    char* const out = reinterpret_cast<char*>(pkeys + base * DCOL);
    const int n_all = t_end - t_first;
    for (int e = threadIdx.x; e < TOK * PPC; e += 256) {
      const int row = e % TOK, piece = e / TOK;
      if (row < n_all)
        prep_store16(out + s_dst[row] + piece * (kChunk * 16),
                     *reinterpret_cast<const uint4*>(lds_piece(row, piece)));
    }
    // the last token of a list, if it is here, fills the list's padding
    for (int f = 0; f < 2; ++f) {
      const int n = f == 0 ? n_here : n_all - n_here;                               // its tokens here
      const int last = f == 0 ? n_ret0 - 1 : ret_cols + (si.len - n_ret0) - 1;      // its last slot
      const int next = f == 0 ? rank0 + n_here : ret_cols + (t_end - rank0 - n_here);
      const int row = f == 0 ? n_here - 1 : n_all - 1;
      const int unit = f == 0 ? kGroupAlign : kChunk;
      const int fill = n > 0 && next == last + 1 ? (unit - next % unit) % unit : 0;
      for (int e = threadIdx.x; e < fill * PPC; e += 256) {
        const int k = next + e % fill, piece = e / fill;
        prep_store16(out + slot_bytes(k) + piece * (kChunk * 16),
                     *reinterpret_cast<const uint4*>(lds_piece(row, piece)));
      }
    }
    // the sweep's candidates of these tokens' slots start empty (padding slots are never read), or
    // the tokens' counts
    if ((int)threadIdx.x < n_all) {
      const int i = threadIdx.x;
      if (counts != nullptr) {
        counts[h * T + si.start + t_first + i] = 0;
        return;
      }
      const int slot = i < n_here ? rank0 + i : ret_cols + (t_first - rank0) + (i - n_here);
      best[base + slot] = 0ull;
      best[plane + base + slot] = 0ull;
    }
  }
}

template <bool ARGS>
int run_partition(const uint8_t* retained, const Table<ARGS>& table, SeqInfo* seqtab, int n_heads, int n_seqs,
                  int64_t T, int64_t PT, int max_len, int32_t* pcol, float* rcol, int32_t* prank,
                  ProblemMeta* pmeta, int32_t* status, hipStream_t st) {
  const dim3 grid((unsigned)((int64_t)n_heads * n_seqs));
  if (max_len > kShortLen)
    hipLaunchKernelGGL(partition_kernel<ARGS>, grid, dim3(kLongThreads), 0, st, retained, table, seqtab,
                       n_seqs, T, PT, pcol, rcol, prank, pmeta, status);
  else if (max_len > kShortLen / 4)
    hipLaunchKernelGGL((partition_short_kernel<kShortLen / 256, ARGS>), grid, dim3(256), 0, st, retained,
                       table, seqtab, n_seqs, T, PT, pcol, rcol, prank, pmeta, status);
  else
    hipLaunchKernelGGL((partition_short_kernel<kShortLen / 1024, ARGS>), grid, dim3(256), 0, st, retained,
                       table, seqtab, n_seqs, T, PT, pcol, rcol, prank, pmeta, status);
  return hipGetLastError();
}

template <int D, bool F32>
constexpr int prep_tokens_per_block() {
  return 256 / (D * (F32 ? 4 : 2) / 16) * kPrepIter;
}

template <int D, bool F32, bool LEVELS, bool ALL>
hipError_t run_prepare(const void* keys, int n_heads, int64_t T, int64_t hs, int64_t ts,
                       int64_t PT, int total_blocks, const uint8_t* retained, const int32_t* prank,
                       ProblemMeta* pmeta, const SeqInfo* seqtab, int n_seqs, float* rinv,
                       float* rcol, uint16_t* hilo, uint16_t* pkeys, int32_t* status,
                       int copy_evicted, unsigned long long* best, int32_t* counts,
                       const PrepLevels& lv, hipStream_t st) {
  constexpr int ESZ = F32 ? 4 : 2;
  if (total_blocks == 0 || n_heads == 0) return hipSuccess;
  for (int h0 = 0; h0 < n_heads; h0 += 65535) {  // heads along y, in slices the grid holds
    const int by = n_heads - h0 < 65535 ? n_heads - h0 : 65535;
    hipLaunchKernelGGL((prepare_keys_kernel<D, F32, LEVELS, ALL>),
                       dim3((unsigned)prep_grid(total_blocks), (unsigned)by), dim3(256), 0, st,
                       (const uint8_t*)keys, T, hs * ESZ, ts * ESZ, PT, retained, prank, pmeta,
                       seqtab, n_seqs, rinv, rcol, hilo, pkeys, status, h0, copy_evicted,
                       best, counts, (int64_t)n_heads * PT, total_blocks, lv);
    const hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

template <bool LEVELS, bool ALL>
int prepare_dispatch(const void* keys, int dtype, int d, int n_heads, int64_t T,
                     int64_t head_stride, int64_t token_stride, int64_t PT, int total_blocks,
                     const uint8_t* retained, const int32_t* prank, ProblemMeta* pmeta,
                     const SeqInfo* seqtab, int n_seqs, float* rinv, float* rcol, uint16_t* hilo,
                     uint16_t* pkeys, int32_t* status, int copy_evicted, unsigned long long* best,
                     int32_t* counts, const PrepLevels& lv, void* stream) {
  hipStream_t st = (hipStream_t)stream;
  if (dtype == 0 && d == 64)
    return run_prepare<64, false, LEVELS, ALL>(keys, n_heads, T, head_stride, token_stride, PT,
                                          total_blocks, retained, prank, pmeta, seqtab, n_seqs,
                                          rinv, rcol, hilo, pkeys, status, copy_evicted, best, counts, lv, st);
  if (dtype == 0 && d == 128)
    return run_prepare<128, false, LEVELS, ALL>(keys, n_heads, T, head_stride, token_stride, PT,
                                           total_blocks, retained, prank, pmeta, seqtab, n_seqs,
                                           rinv, rcol, hilo, pkeys, status, copy_evicted, best, counts, lv, st);
  if (dtype == 1 && d == 64)
    return run_prepare<64, true, LEVELS, ALL>(keys, n_heads, T, head_stride, token_stride, PT,
                                         total_blocks, retained, prank, pmeta, seqtab, n_seqs,
                                         rinv, rcol, hilo, pkeys, status, copy_evicted, best, counts, lv, st);
  if (dtype == 1 && d == 128)
    return run_prepare<128, true, LEVELS, ALL>(keys, n_heads, T, head_stride, token_stride, PT,
                                          total_blocks, retained, prank, pmeta, seqtab, n_seqs,
                                          rinv, rcol, hilo, pkeys, status, copy_evicted, best, counts, lv, st);
  return hipErrorInvalidValue;
}

}  // namespace

int launch_partition(const uint8_t* retained, const SeqInfo* table, SeqInfo* seqtab, int n_heads, int n_seqs,
                     int64_t T, int64_t PT, int max_len, int32_t* pcol, float* rcol,
                     int32_t* prank, ProblemMeta* pmeta, int32_t* status, void* stream) {
  if (n_seqs <= kTableArgs) {
    TableArgs args{};
    std::copy(table, table + n_seqs, args.s);
    return run_partition<true>(retained, args, seqtab, n_heads, n_seqs, T, PT, max_len, pcol, rcol, prank,
                               pmeta, status, (hipStream_t)stream);
  }
  const int e = launch_upload(table, sizeof(SeqInfo) * (size_t)n_seqs, seqtab, stream);
  if (e != 0) return e;
  return run_partition<false>(retained, TableUploaded{}, seqtab, n_heads, n_seqs, T, PT, max_len, pcol, rcol,
                              prank, pmeta, status, (hipStream_t)stream);
}

int prepare_tokens_per_block(int dtype, int d) {
  if (dtype == 0 && d == 64) return prep_tokens_per_block<64, false>();
  if (dtype == 0 && d == 128) return prep_tokens_per_block<128, false>();
  if (dtype == 1 && d == 64) return prep_tokens_per_block<64, true>();
  if (dtype == 1 && d == 128) return prep_tokens_per_block<128, true>();
  return 0;
}

int launch_prepare_keys(const void* keys, int dtype, int d, int n_heads, int64_t T,
                        int64_t head_stride, int64_t token_stride, int64_t PT, int total_blocks,
                        const uint8_t* retained, const int32_t* prank, ProblemMeta* pmeta,
                        const SeqInfo* seqtab, int n_seqs, float* rinv, float* rcol,
                        uint16_t* hilo, uint16_t* pkeys, int32_t* status, Sweep sweep,
                        unsigned long long* best, int32_t* counts, void* stream) {
  const PrepLevels none{nullptr, 0, 1, 0};
  const auto dispatch =
      sweep == kSweepPairs ? prepare_dispatch<false, true> : prepare_dispatch<false, false>;
  return dispatch(keys, dtype, d, n_heads, T, head_stride, token_stride, PT, total_blocks, retained,
                  prank, pmeta, seqtab, n_seqs, rinv, rcol, hilo, pkeys, status,
                  sweep == kSweepAll ? 1 : 0, best, counts, none, stream);
}

int launch_prepare_keys_levels(const void* keys, int dtype, int d, int n_heads, int64_t T,
                               int64_t head_stride, int64_t token_stride, int64_t PT,
                               int total_blocks, const PrepLevels& lv, const int32_t* prank,
                               ProblemMeta* pmeta, const SeqInfo* seqtab, int n_seqs, float* rinv,
                               float* rcol, uint16_t* hilo, uint16_t* pkeys, int32_t* status,
                               void* stream) {
  return prepare_dispatch<true, false>(keys, dtype, d, n_heads, T, head_stride, token_stride, PT,
                                       total_blocks, nullptr, prank, pmeta, seqtab, n_seqs, rinv,
                                       rcol, hilo, pkeys, status, 0, nullptr, nullptr, lv, stream);
}

}  // namespace twinkv
