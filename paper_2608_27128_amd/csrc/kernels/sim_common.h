// Device pieces shared by the similarity sweeps: operand types, LDS loads, and the mapping from
// workgroups to row blocks.
#pragma once
#include <hip/hip_runtime.h>

#include "../twinkv_internal.h"
#include "key_scale.h"

namespace twinkv {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kWaves = 4;

// Row (0..31 inside a block) held by register v of a lane in half `half`.
__device__ inline constexpr int slot_row(int v, int half) {
  return 8 * (v >> 2) + 4 * half + (v & 3);
}

// Fourth dword of a raw buffer resource on gfx9-family parts (32-bit data format).
constexpr int kBufferFlags = 0x00020000;

// Raw buffer resource of nbytes; direct loads of 16 (4) bytes per lane at voff + IMM into LDS at
// lds + IMM + 16 (4) * lane.  Lanes whose offset is past the end read nothing (zeros).
__device__ inline __amdgpu_buffer_rsrc_t tile_rsrc(const void* base, int nbytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, nbytes, kBufferFlags);
}
template <int IMM>
__device__ inline void load_lds16(__amdgpu_buffer_rsrc_t rs, char* lds, int voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (void __attribute__((address_space(3)))*)lds, 16,
                                           voff, 0, IMM, 0);
}
__device__ inline void load_lds4(__amdgpu_buffer_rsrc_t rs, char* lds, int voff) {
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rs, (void __attribute__((address_space(3)))*)lds, 4,
                                           voff, 0, 0, 0);
}

// Scheduling-group masks for __builtin_amdgcn_sched_group_barrier.
constexpr int kSchedValu = 0x002;
constexpr int kSchedMfma = 0x008;
constexpr int kSchedDsRead = 0x100;

// A row block's place in the batch.
struct Place {
  int head, rb, len, n_ret, ret_chunks, total_chunks;
  int64_t colbase, rowbase;  // first slot in the column arrays, first token in the row arrays
  int problem;               // head * n_seqs + sequence
  int64_t keybase;           // element offset of the sequence's first row key
};
// Workgroup k (of those of XCD x when there are >= 8 heads: heads h = x (mod 8) go to the XCD the
// hardware dispatches block b = x (mod 8) to, so one problem's row blocks share that XCD's L2;
// inside an XCD the sequences run longest first, and a sequence's longest sweeps first, up to
// spread_row_block).  part
// receives the index beyond the row blocks.  False: no such row block.
__device__ inline bool find_place(const SimArgs& a, int block, Place& pl, int& part) {
  int k, hx, hmax, h0, hstep;
  if (a.n_heads >= 8) {
    const int x = block & 7;
    k = block >> 3;
    hx = (a.n_heads - x + 7) >> 3;
    hmax = (a.n_heads + 7) >> 3;
    h0 = x;
    hstep = 8;
  } else {
    k = block;
    hx = hmax = a.n_heads;
    h0 = 0;
    hstep = 1;
  }
  part = k / (hmax * a.total_tiles);
  k -= part * hmax * a.total_tiles;
  if (k >= hx * a.total_tiles) return false;
  int lo = 0, hi = a.n_seqs - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (hx * a.seqtab[mid].tile_cum <= k) lo = mid; else hi = mid - 1;
  }
  const int nb = a.seqtab[lo].nb;
  const int local = k - hx * a.seqtab[lo].tile_cum;
  pl.head = h0 + hstep * (local / nb);
  pl.rb = spread_row_block(local - (local / nb) * nb, nb, lo * hx + local / nb, a.n_heads >= 8);
  const int seq = a.seqtab[lo].sorted_seq;
  const SeqInfo si = a.seqtab[seq];
  pl.problem = pl.head * a.n_seqs + seq;
  const ProblemMeta pm = a.pmeta[pl.problem];
  pl.len = si.len;
  pl.n_ret = pm.n_ret;
  pl.ret_chunks = pm.ret_chunks;
  pl.total_chunks = pm.total_chunks;
  pl.colbase = (int64_t)pl.head * a.PT + si.perm_off;
  pl.rowbase = (int64_t)pl.head * a.T + si.start;
  pl.keybase = (int64_t)pl.head * a.head_stride + (int64_t)si.start * a.token_stride;
  return true;
}

}  // namespace
}  // namespace twinkv
