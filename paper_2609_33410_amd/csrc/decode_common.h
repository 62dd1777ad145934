// Pieces shared by the decode scan kernels: buffer resources over 16-key
// chunks, query-row lookup, and the chunk schedule of a split.
#pragma once

#include "fold_device.h"
#include "fold_internal.h"

namespace fold {

constexpr int kScanWaves = 4;
constexpr int kScanThreads = 64 * kScanWaves;
constexpr uint32_t kRsrcWord3 = 0x00020000u;  // raw buffer, 32-bit data (gfx9 family)
constexpr uint32_t kOutOfRange = 0x80000000u;  // an offset past any chunk resource

typedef __amdgpu_buffer_rsrc_t rsrc_t;

// A buffer resource over `bytes` bytes at `base`: loads at offsets past the
// end return zero and touch no memory.
__device__ __forceinline__ rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), static_cast<short>(0),
                                           static_cast<int>(bytes), static_cast<int>(kRsrcWord3));
}

// Cache policy of the cache-row stream: non-temporal (the NT bit of the gfx950
// cache-policy field).  A call reads each cached key and value row once; with
// this bit, randomly placed 4 KiB page slabs stream from HBM at about 6.6 TB/s
// against 5.9 TB/s with the default policy (measured on MI355X).
constexpr int kStreamPolicy = 2;

template <int POLICY = kStreamPolicy>
__device__ __forceinline__ u32x4 buf_load(rsrc_t r, uint32_t off) {
  return __builtin_amdgcn_raw_buffer_load_b128(r, off, 0, POLICY);
}

struct RowInfo {
  int req;
  int head;
  bool ok;
};

// Query row rho of the rows attending (kv sequence seq, kv head kvh):
// rho = (position of the request in the sequence's row list) * G + (h mod G).
__device__ __forceinline__ RowInfo row_info(const ScanGeometry& g, int seq, int kvh, int rho,
                                            int nrows, int req0) {
  RowInfo ri;
  ri.ok = rho < nrows;
  const int rr = ri.ok ? rho : 0;
  ri.req = g.row_indptr ? ld_uniform(g.row_req, req0 + rr / g.group) : seq;
  ri.head = kvh * g.group + rr % g.group;
  ri.ok = ri.ok && ri.req >= 0 && ri.req < g.batch;
  return ri;
}

// Where one workgroup works: kv sequence, kv head, split, read group; the
// sequence's length and rows.  Block index order: sequence fastest, then kv
// head, split, read group.
struct ScanPlace {
  int seq, kvh, split, rg;
  int req0, nrows;
  int n, nchunks;
};

__device__ __forceinline__ ScanPlace scan_place(const DecodeArgs& a) {
  const ScanGeometry& g = a.geo;
  ScanPlace p;
  int bid = blockIdx.x;
  p.seq = bid % g.num_seqs;
  bid /= g.num_seqs;
  p.kvh = bid % g.hkv;
  bid /= g.hkv;
  p.split = bid % a.num_splits;
  p.rg = bid / a.num_splits;
  p.req0 = p.seq;
  int nreq = 1;
  if (g.row_indptr) {
    p.req0 = ld_uniform(g.row_indptr, p.seq);
    nreq = ld_uniform(g.row_indptr, p.seq + 1) - p.req0;
  }
  p.nrows = nreq * g.group;
  p.n = clamp_len(ld_uniform(g.seq_lens, p.seq), view_capacity(g));
  p.nchunks = (p.n + kChunk - 1) / kChunk;
  return p;
}

// Longest sequences first.  For a per-request view of at most kOrderMax
// sequences the block index runs over kv heads fastest, then splits, then the
// sequences by decreasing length, then read groups.  Blocks
// are dispatched in index order as slots free up, so the workgroups of the
// longest sequences start first and the last to start are the shortest ones:
// a ragged batch drains with less of the call left to a half-empty chip.
// Which workgroup scans which keys changes nothing else (same sums, same
// bits), so the order need not be exact: lengths that agree in the kLenBits
// leading bits of the view's capacity, and equal ones, come by index.  Every
// wave finds its sequence itself, lane i holding sequence i's length: a radix
// selection by ballots, seven instructions a bit whatever the count of
// sequences, no LDS and no barrier.  Ranking every lane by num_seqs readlanes
// took six instructions a sequence before the first key load, and short scans
// of many sequences felt it: 64 requests of 1-2K keys, 8 kv heads, groups of 2,
// two-plane scan at T = 16: 36.1 us ranked, 32.5 selected, 30.9 in natural order;
// 32 ragged ones of 8-16K keys, groups of 8: 61.3, 59.9 and 73.9.
constexpr int kLenBits = 7;

__device__ __forceinline__ ScanPlace scan_place_by_length(const DecodeArgs& a) {
  static_assert(kOrderMax <= 64, "a lane per sequence");
  const ScanGeometry& g = a.geo;
  const int cap = view_capacity(g);
  const int lane = threadIdx.x & 63;
  const bool mine = lane < g.num_seqs;
  const int li = mine ? clamp_len(g.seq_lens[lane], cap) : 0;
  ScanPlace p;
  int bid = blockIdx.x;
  p.kvh = bid % g.hkv;
  bid /= g.hkv;
  p.split = bid % a.num_splits;
  bid /= a.num_splits;
  int rank = bid % g.num_seqs;  // among the candidates below
  p.rg = bid / g.num_seqs;
  uint64_t cand = __builtin_amdgcn_ballot_w64(mine);
  const int top = 31 - __builtin_clz(static_cast<unsigned>(cap) | 1u);
#pragma unroll
  for (int i = 0; i < kLenBits; ++i) {
    const uint64_t hi = cand & __builtin_amdgcn_ballot_w64(((li >> max(top - i, 0)) & 1) != 0);
    const int longer = __builtin_popcountll(hi);
    const bool up = rank < longer;
    cand = up ? hi : cand & ~hi;
    rank = up ? rank : rank - longer;
  }
  // the candidate with `rank` candidates below it: one lane
  const int below = __builtin_amdgcn_mbcnt_hi(static_cast<uint32_t>(cand >> 32),
                                              __builtin_amdgcn_mbcnt_lo(static_cast<uint32_t>(cand), 0));
  const uint64_t hit = __builtin_amdgcn_ballot_w64(((cand >> lane) & 1) != 0 && below == rank);
  p.seq = hit ? __builtin_ctzll(hit) : 0;
  p.req0 = p.seq;
  p.nrows = g.group;
  p.n = __builtin_amdgcn_readlane(li, p.seq);
  p.nchunks = (p.n + kChunk - 1) / kChunk;
  return p;
}

// Element-row index of (sequence, position, kv head) in the view's layout, or
// -1 when the view cannot address it.  UNIFORM: the wave asks for one token (the
// block-table entry is a scalar load); else each lane for its own.
template <bool UNIFORM>
__device__ __forceinline__ long long row_of(const ScanGeometry& g, int seq, int pos, int kvh) {
  if (seq < 0 || seq >= g.num_seqs || pos < 0 || pos >= view_capacity(g)) return -1;
  if (g.page_size > 0) {
    const uint32_t page = static_cast<uint32_t>(pos) / static_cast<uint32_t>(g.page_size);
    const size_t at = static_cast<size_t>(seq) * g.max_pages + page;
    const int phys = UNIFORM ? ld_uniform(g.block_table, at) : g.block_table[at];
    if (phys < 0 || phys >= g.num_pages) return -1;
    return (static_cast<long long>(phys) * g.hkv + kvh) * g.page_size +
           (pos - static_cast<int>(page) * g.page_size);
  }
  return (static_cast<long long>(seq) * g.hkv + kvh) * g.max_seq_len + pos;
}

// Block-table entry of the page holding 16-key chunk c of the sequence (0 for
// a contiguous view or past the sequence end).  A scalar load: issuing it well
// before chunk_rsrc_at() hides its latency.
__device__ __forceinline__ int chunk_page(const ScanGeometry& g, const ScanPlace& p, int c) {
  if (g.page_size <= 0 || c >= p.nchunks) return 0;
  return ld_uniform(g.block_table,
                    static_cast<size_t>(p.seq) * g.max_pages + (c * kChunk) / g.page_size);
}

// Buffer resources over the valid keys of 16-key chunk c of (seq, kvh), given
// the chunk's block-table entry: empty past the sequence end or for a page id
// outside [0, num_pages).
template <int D>
__device__ __forceinline__ void chunk_rsrc_at(const ScanGeometry& g, const ScanPlace& p, int c,
                                              int phys, rsrc_t* rk, rsrc_t* rv) {
  const uint16_t* kb = g.k;
  const uint16_t* vb = g.v;
  uint32_t bytes = 0;
  if (c < p.nchunks) {
    const int key0 = c * kChunk;
    const int nk = min(kChunk, p.n - key0);
    size_t off;
    bool ok = true;
    if (g.page_size > 0) {
      const int page = key0 / g.page_size;
      ok = phys >= 0 && phys < g.num_pages;
      off = ((static_cast<size_t>(ok ? phys : 0) * g.hkv + p.kvh) * g.page_size +
             (key0 - page * g.page_size)) * D;
    } else {
      off = ((static_cast<size_t>(p.seq) * g.hkv + p.kvh) * g.max_seq_len + key0) * D;
    }
    if (ok) {
      kb += off;
      vb += off;
      bytes = static_cast<uint32_t>(nk) * D * 2;
    }
  }
  *rk = make_rsrc(kb, bytes);
  *rv = make_rsrc(vb, bytes);
}

template <int D>
__device__ __forceinline__ void chunk_rsrc(const ScanGeometry& g, const ScanPlace& p, int c,
                                           rsrc_t* rk, rsrc_t* rv) {
  chunk_rsrc_at<D>(g, p, c, chunk_page(g, p, c), rk, rv);
}

}  // namespace fold
