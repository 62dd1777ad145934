// Split-KV decode over a two-plane INT8 key cache for read groups of 2 to 16
// query rows, at any depth (Section 4, "Cache format", "Weight-gated reads",
// "Value product", "Depth as a dial"; Algorithm 1 with BF16 or 8-bit values).
//
// The arithmetic is Algorithm 1's: coarse scores from plane A and the key
// scales, per-GQA-group live / refine-K / refine-V verdicts on them, plane B
// only for refined keys, value rows only for live keys, the weight 2^x with
// every key's weight in L.  The work is laid out so that the key stream waits
// for no verdict:
//
//   step      two of the wave's 16-key chunks.  Plane A and the scales of the
//             next two steps are in flight.  Dense decode: and their value
//             rows (or the first E4M3 plane).  Finite depth: a step's value
//             rows are requested when it is scored and multiplied one step
//             later; every load is issued, those of cut keys past their
//             resource (no bytes), so that the number in flight is known.
//   list      a refined key (a few in a thousand at the default thresholds)
//             leaves the stream with weight 0 and joins a list in the wave's
//             LDS: cache row, scale, coarse scores.  Sixteen listed keys at a
//             time (and the rest at the end) are gathered: verdicts, plane B
//             and value rows, refined scores, weights, value product.
//   in place  a step with more than kListMost refined keys (raised thresholds),
//             or a wave's only one, fetches plane B, and the second value plane,
//             for both chunks at once and waits.
//   packing   with at most eight rows (PK = 2) each chunk takes eight of the 16
//             row lanes: the integer products 256 a.qa + a.qb of the second
//             move there by a DPP shift, so scores and weights cost one pass
//             per step; with 9 to 16 rows (PK = 1) one pass per chunk.
//   product   v_mfma_f32_16x16x32_bf16 over the step's 32 keys (bf16 hi and
//             residual weights): the score tile's register layout is the
//             operand layout.  E4M3 rows stay bytes in LDS and are widened
//             after the transposing read.
//   loads     whole 128-byte lines (lane l, load c: bytes 1024 c + 16 l of the
//             chunk); a plane chunk reaches the i8 operand layout (lane l: 16
//             bytes of key l%16) through the wave's LDS tile.  Loaded in the
//             operand layout directly, 16 half lines an instruction, the scan
//             below took 72.6 us and not 65.0 with 37 % of the wave time spent
//             waiting to issue.  Where chunks live comes from a window of 64
//             in a register (v_readlane), not from a scalar load each.
//
// What bounds it: memory latency at two waves per SIMD (D = 128: the registers
// of two steps in flight; three waves spill and are three times slower), then
// HBM.  Whole kernel, 32 requests of 8-16K keys, before (verdict, plane B and
// values fetched inside the step) and now:
//   D = 128, G = 8,  BF16 values, T = 16    90.4 -> 58.6 us (4.5 TB/s; 14 % of
//                                           the keys are live for some row)
//   D = 128, G = 16, BF16 values, T = 16    74.8 -> 63.7 us (4.7 TB/s; 92 % live)
//   D = 64,  G = 8,  8-bit values, dense   133.5 -> 77.4 us (5.7 TB/s)
// Short scans, warm: 64 x 512 keys, G = 8, 4 splits, dense 7.1 -> 6.2 us; 64 x
// 1024, G = 16, 8 splits, T = 16 21.6 -> 19.1; 32 x 1024, G = 4, 4 splits, dense
// 25.7 -> 25.6.
// Steps refined in place wait their round trip; where all are (kappa = inf,
// groups of 4) some shapes take up to 3 % longer than with the kernel before:
// 8 x 32768 keys, G = 4, dense 165.9 -> 169.6 us, 15 x 3-9K, D = 64, G = 4,
// T = 16 43.3 -> 44.5; others less (32 x 5-16K, G = 8, dense 131.8 -> 122.9,
// T = 16 155.3 -> 121.2).
// Listing every live key, and not the refined ones only, was slower where
// many are live (G = 16: 84 us).
#include "q8_common.h"

namespace fold {
namespace {

typedef int i32x2 __attribute__((ext_vector_type(2)));
typedef __attribute__((address_space(3))) i32x2 lds_i32x2;

constexpr int kListMost = 8;   // keys a step may list; more are refined in place
constexpr int kListKeys = 32;  // list slots per wave: 15 keys left over and two steps' keys
constexpr uint32_t kNoRow = 0xFFFFFFFFu;

// Keeps the vector-memory loads on their side, in program order (every other
// instruction may cross): loads retire in issue order, so a wait for one
// leaves in flight what the program issued after it, and no less.
__device__ __forceinline__ void load_fence() { __builtin_amdgcn_sched_barrier(0x78F); }

template <int CTRL>
__device__ __forceinline__ uint32_t dpp_or(uint32_t v) {
  return v | static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), CTRL, 0xF, 0xF, true));
}

// The value of lane I of the lane's quad.
template <int I>
__device__ __forceinline__ float quad_lane(float v) {
  return __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), 0x55 * I, 0xF, 0xF, true));
}

// Where a chunk lives: its first key row in the cache (kNoRow for a page
// outside the pool; a key takes at least 130 bytes of cache, so rows are fewer
// than 2^32) and the keys it holds.
struct RowLoc {
  uint32_t row;
  uint32_t nk;
};

template <int D, int PK, bool DENSE, bool DBG, bool V8>
struct Q8Rows {
  static constexpr int NKI = D / 64;                // plane loads per lane per chunk
  static constexpr int NKV = V8 ? D / 64 : D / 32;  // value loads per lane per chunk
  static constexpr int NB = D / 16;                 // 16-channel blocks of the value product
  static constexpr int CH = 2;                      // chunks per step
  static constexpr int NSET = CH / PK;              // score passes per step
  static constexpr int BW = 16 / PK;                // row lanes per chunk
  static constexpr int PSTRIDE = D + 16;            // bytes per row of a byte-plane tile
  static constexpr int VSTRIDE = 2 * D + 16;        // bytes per row of a BF16 value tile
  static constexpr int kValueTile = CH * 16 * (V8 ? PSTRIDE : VSTRIDE);
  static constexpr int kStage = 16 * VSTRIDE;       // a gathered group's value rows
  static constexpr int kPlaneTile = CH * 16 * PSTRIDE;
  static constexpr int kTile0 = kValueTile > kStage ? kValueTile : kStage;
  static constexpr int kTile = kTile0 > kPlaneTile ? kTile0 : kPlaneTile;
  // The dense scan of BF16 values at D = 128 keeps two steps of values in
  // registers and its query planes in LDS (16 registers that would spill).
  static constexpr bool kQueryLds = DENSE && !V8 && D == 128;
  static constexpr int QSTRIDE = 2 * D + 16;        // bytes per query row in LDS
  static constexpr int kListBytes = kListKeys * (BW + 2 + (DBG ? 1 : 0)) * 4;
  static constexpr int kWaveBytes = kTile + kListBytes + (kQueryLds ? 16 * QSTRIDE : 0);
  static constexpr int kGatherKeys = 16;            // keys of one gather
  static_assert(kGatherKeys - 1 + 2 * kListMost <= kListKeys && kListKeys % 16 == 0, "list space");

  struct Step {
    RowLoc loc[CH];
    u32x4 a[CH][NKI];
    uint16_t sc[CH];
    u32x4 v[DENSE ? CH : 1][NKV];
  };

  // A scored step waiting for its value rows (finite depth).
  struct Pending {
    u32x4 v[CH][NKV];
    u32x4 hi, lo;    // its weights, the product's operand
    uint32_t mask;   // its live keys: chunk 0 in the low half, chunk 1 in the high
  };

  const Q8DecodeArgs& a;
  const ScanGeometry& g;
  ScanPlace p;
  int lane, n16, grp, slot, cstride, c0, m, pshift, gspan;
  size_t gate_row;
  unsigned char* tile;
  float* list_x;      // [kListKeys][BW] coarse x
  uint32_t* list_row; // cache row, or kNoRow
  float* list_e;      // key scale / 256
  int* list_key;      // key index (debug)
  int head, count;    // the list: slots head .. head + count - 1 (mod kListKeys)

  u32x4 qa[kQueryLds ? 1 : NKI], qb[kQueryLds ? 1 : NKI];  // query planes of row n16 (the operand layout)
  unsigned char* qrow;     // kQueryLds: the lane's 16 bytes of row n16
  bool rok;                // row n16 exists
  // Of row n16 % BW: the row a lane weighs, and in the lanes of a row of its
  // own (n16 < BW, the only ones with rok) that row.
  bool pok;
  float zp, etap;          // Z (+inf for no row), eta
  float ntau, ntau_v;      // -tau
  float thr;               // the score from which a key is refined
  size_t xrow, prow;       // query rows of n16 and n16 % BW (debug)
  f32x4 acc[NB];
  float lsum, lcut;
  uint32_t win_row, win_nk;  // RowLoc of local chunks win_base .. win_base + 63, one per lane
  int win_base;
  bool cut_out;              // the caller wants the cut masses
  int list_most;             // keys a step may list

  __device__ Q8Rows(const Q8DecodeArgs& a_) : a(a_), g(a_.d.geo) {}

  // Where local chunks base .. base + 63 live, one per lane: one vector load of
  // block-table entries, and no address arithmetic per chunk but two readlanes.
  __device__ __forceinline__ void window(int base) {
    win_base = base;
    const int k = base + lane;
    const int c = c0 + k * cstride;
    win_row = kNoRow;
    win_nk = 0;
    if (k < m) {
      const int key0 = c * kChunk;
      win_nk = static_cast<uint32_t>(min(kChunk, p.n - key0));
      if (g.page_size > 0) {
        const int page = chunk_page_of(g, c, pshift);
        const int phys = g.block_table[static_cast<size_t>(p.seq) * g.max_pages + page];
        if (phys >= 0 && phys < g.num_pages)
          win_row = (static_cast<uint32_t>(phys) * static_cast<uint32_t>(g.hkv) +
                     static_cast<uint32_t>(p.kvh)) * static_cast<uint32_t>(g.page_size) +
                    static_cast<uint32_t>(key0 - page * g.page_size);
      } else {
        win_row = (static_cast<uint32_t>(p.seq) * static_cast<uint32_t>(g.hkv) +
                   static_cast<uint32_t>(p.kvh)) * static_cast<uint32_t>(g.max_seq_len) +
                  static_cast<uint32_t>(key0);
      }
    }
  }

  // A chunk's rows of ROW bytes in a plane: empty for a page outside the pool.
  template <int ROW>
  static __device__ __forceinline__ rsrc_t rows_at(const void* base, const RowLoc& l) {
    return make_rsrc(static_cast<const unsigned char*>(base) + static_cast<size_t>(l.row) * ROW,
                     l.row == kNoRow ? 0u : l.nk * ROW);
  }

  // Plane A as whole lines (lane l, load c: bytes 1024 c + 16 l of the chunk),
  // and the scales.
  __device__ __forceinline__ void issue_a(int step, Step& s) {
    const int k0 = step * CH;
    if (k0 >= win_base + 64 && k0 < m) window(k0 & ~63);  // uniform
    load_fence();
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const int at = (k0 + q) & 63;
      RowLoc l;
      l.row = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(win_row), at));
      l.nk = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(win_nk), at));
      if (k0 >= m) l.nk = 0;  // past the split: nothing is read
      s.loc[q] = l;
      // the scale of key 4(l/16) + l%4, in the lanes that weigh the chunk
      s.sc[q] = __builtin_amdgcn_raw_buffer_load_b16(
          rows_at<2>(a.keys.ks, l),
          PK == 1 || slot == q ? 2u * (4 * grp + (lane & 3)) : kOutOfRange, 0, kStreamPolicy);
      const rsrc_t ra = rows_at<D>(a.keys.ka, l);
#pragma unroll
      for (int c = 0; c < NKI; ++c) s.a[q][c] = buf_load(ra, 1024u * c + 16u * lane);
    }
    load_fence();
  }

  __device__ __forceinline__ void issue_v(Step& s) const {
    if constexpr (DENSE) {
#pragma unroll
      for (int q = 0; q < CH; ++q) {
        const rsrc_t rv = V8 ? rows_at<D>(a.vp, s.loc[q]) : rows_at<2 * D>(g.v, s.loc[q]);
#pragma unroll
        for (int i = 0; i < NKV; ++i) s.v[q][i] = buf_load(rv, 1024u * i + 16u * lane);
      }
      load_fence();
    }
  }

  // 16-byte loads of one chunk into rows of STRIDE bytes, ROW bytes each.
  template <int ROW, int STRIDE, int NL>
  __device__ __forceinline__ void put(const u32x4 (&ld)[NL], unsigned char* to) const {
#pragma unroll
    for (int c = 0; c < NL; ++c) {
      const uint32_t off = 1024u * c + 16u * lane;
      const uint32_t key = off / ROW;
      *reinterpret_cast<u32x4*>(to + key * STRIDE + (off - key * ROW)) = ld[c];
    }
  }

  // 256 (p . qa) + p . qb of a plane chunk in the operand layout: exact in
  // int32 (each product sum is below 2^21).
  __device__ __forceinline__ i32x4 plane_product(const u32x4 (&op)[NKI]) const {
    i32x4 ta = {0, 0, 0, 0}, tb = {0, 0, 0, 0};
#pragma unroll
    for (int c = 0; c < NKI; ++c) {
      u32x4 a4, b4;
      if constexpr (kQueryLds) {
        a4 = *reinterpret_cast<const u32x4*>(qrow + 64 * c);
        b4 = *reinterpret_cast<const u32x4*>(qrow + D + 64 * c);
      } else {
        a4 = qa[c];
        b4 = qb[c];
      }
      ta = mfma_i8(op[c], a4, ta);
      tb = mfma_i8(op[c], b4, tb);
    }
    i32x4 t;
#pragma unroll
    for (int i = 0; i < 4; ++i) t[i] = (ta[i] << 8) + tb[i];
    return t;
  }

  // Weight halves of four keys: bf16 truncated, bf16 residual.
  __device__ __forceinline__ void halves(const float (&w)[4], u32x2* hi, u32x2* lo) const {
    uint32_t h[4];
    float r[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      h[i] = __float_as_uint(w[i]) & 0xffff0000u;
      r[i] = w[i] - __uint_as_float(h[i]);
    }
    *hi = u32x2{(h[0] >> 16) | h[1], (h[2] >> 16) | h[3]};
    *lo = u32x2{pack_bf16_rne(r[0], r[1]), pack_bf16_rne(r[2], r[3])};
  }

  // acc += V^T P^T over the step's 32 keys staged in the tile (16 rows per
  // chunk).  k slots 8 (l/16) .. +7 are keys 4 (l/16) .. +3 of chunk 0, then
  // of chunk 1.
  __device__ __forceinline__ void product32(const u32x4& hi, const u32x4& lo, float scale = 1.0f) {
    if constexpr (V8) {
      // lanes 2i and 2i + 1 of each 16-lane group point at 8 channels each of
      // the i-th of the eight keys; lane l receives channel 16 blk + l%16
      const int i = n16 >> 1;
      const unsigned char* src = tile + ((i >> 2) * 16 + 4 * grp + (i & 3)) * PSTRIDE + 8 * (n16 & 1);
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) {
        const i32x2 b = __builtin_amdgcn_ds_read_tr8_b64_v2i32((lds_i32x2*)(src + 16 * blk));
        u32x4 va;
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          va[2 * j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(
                                                       j ? b.y : b.x, scale, false));
          va[2 * j + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(
                                                           j ? b.y : b.x, scale, true));
        }
        acc[blk] = mfma_16x16x32(va, hi, acc[blk]);
        acc[blk] = mfma_16x16x32(va, lo, acc[blk]);
      }
    } else {
      const unsigned char* src = tile + (4 * grp + (n16 >> 2)) * VSTRIDE + 8 * (n16 & 3);
#pragma unroll
      for (int blk = 0; blk < NB; ++blk) {
        const u32x2 v0 = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(src + 32 * blk)));
        const u32x2 v1 = __builtin_bit_cast(
            u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16(
                       (lds_s16x4*)(src + 16 * VSTRIDE + 32 * blk)));
        const u32x4 va = {v0.x, v0.y, v1.x, v1.y};
        acc[blk] = mfma_16x16x32(va, hi, acc[blk]);
        acc[blk] = mfma_16x16x32(va, lo, acc[blk]);
      }
    }
  }

  // acc += V^T P^T over one gathered 16-key group staged as BF16 rows.
  __device__ __forceinline__ void product16(const u32x2& hi, const u32x2& lo) {
    const unsigned char* src = tile + (4 * grp + (n16 >> 2)) * VSTRIDE + 8 * (n16 & 3);
#pragma unroll
    for (int blk = 0; blk < NB; ++blk) {
      const u32x2 va = __builtin_bit_cast(
          u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4*)(src + 32 * blk)));
      acc[blk] = mfma_16x16x16(va, hi, acc[blk]);
      acc[blk] = mfma_16x16x16(va, lo, acc[blk]);
    }
  }

  // Sixteen gathered rows as BF16 in the tile; E4M3 codes are widened exactly.
  template <int NL>
  __device__ __forceinline__ void stage(const u32x4 (&vv)[NL], float scale) const {
    if constexpr (V8) {
#pragma unroll
      for (int i = 0; i < NL; ++i) {
        const uint32_t off = 1024u * i + 16u * lane;
        const uint32_t key = off / D;
        uint32_t w[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          w[2 * j] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(
                                                      static_cast<int>(vv[i][j]), scale, false));
          w[2 * j + 1] = __builtin_bit_cast(uint32_t, __builtin_amdgcn_cvt_scalef32_pk_bf16_fp8(
                                                          static_cast<int>(vv[i][j]), scale, true));
        }
        unsigned char* dst = tile + key * VSTRIDE + 2 * (off - key * D);
        *reinterpret_cast<u32x4*>(dst) = u32x4{w[0], w[1], w[2], w[3]};
        *reinterpret_cast<u32x4*>(dst + 16) = u32x4{w[4], w[5], w[6], w[7]};
      }
    } else {
      put<2 * D, VSTRIDE, NL>(vv, tile);
    }
  }

  // Moves the keys of the row-ORed fields u (key 4(l/16)+i of the lane's chunk;
  // both: their key_mask) to the list.
  __device__ __forceinline__ void append(const Step& s, const float (&x)[4], const float (&e)[4],
                                         uint32_t u, uint32_t both, int set) {
    const uint32_t m0 = both & 0xFFFFu;
    const uint32_t mask = PK == 2 && slot ? both >> 16 : m0;
    const int before = count + (PK == 2 && slot ? __builtin_popcount(m0) : 0);
    const RowLoc l = PK == 2 ? (slot ? s.loc[1] : s.loc[0]) : s.loc[set];
    const int row = n16 % BW;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int k = 4 * grp + i;
      if ((u >> i) & 1u) {
        int at = head + before + __builtin_popcount(mask & ((1u << k) - 1u));
        if (at >= kListKeys) at -= kListKeys;
        list_x[at * BW + row] = x[i];
        if (row == 0) {
          list_row[at] = l.row == kNoRow ? kNoRow : l.row + k;
          list_e[at] = e[i];
          if (DBG) list_key[at] = debug_key0(set) + k;
        }
      }
    }
    count += __builtin_popcount(both);
  }

  int dbg_key0[DBG ? CH : 1];  // first keys of the step's chunks (debug)

  // OR of the lanes' four-bit fields (key 4(l/16)+i of the lane's chunk) over
  // the chunk's row lanes.
  __device__ __forceinline__ uint32_t rows_or(uint32_t bits) const {
    uint32_t u = dpp_or<0x141>(dpp_or<0x4E>(dpp_or<0xB1>(bits)));
    if constexpr (BW == 16) u = dpp_or<0x140>(u);
    return u;
  }

  // The 16-key masks of row-ORed fields: PK == 2: chunk 0 in the low half,
  // chunk 1 in the high; else the pass's chunk.
  __device__ __forceinline__ uint32_t key_mask(uint32_t u) const {
    uint32_t w = u << (4 * grp);
    const auto r = __builtin_amdgcn_permlane16_swap(w, w, false, false);
    w = r[0] | r[1];
    const auto t = __builtin_amdgcn_permlane32_swap(w, w, false, false);
    w = t[0] | t[1];
    uint32_t m = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w), 0));
    if constexpr (PK == 2)
      m |= static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(w), 8)) << 16;
    return m;
  }

  // Clears the values of the step's keys in mask (dense: they came with the
  // stream).  Bit 16 q + 1024 i / (2 D) of the lane's copy is its key of load i.
  __device__ __forceinline__ void clear_values(Step& s, uint32_t mask) const {
    const uint32_t own = mask >> (16u * lane / (2 * D));
#pragma unroll
    for (int q = 0; q < CH; ++q)
#pragma unroll
      for (int i = 0; i < NKV; ++i)
        if ((own >> (16 * q + 1024 * i / (2 * D))) & 1u) s.v[DENSE ? q : 0][i] = u32x4{0, 0, 0, 0};
  }

  // Scores and weights of step j from its plane A: listed keys go to the list;
  // hi and lo receive the weights that enter A, mask the live keys left in
  // the stream (finite depth).
  // LIST: keys may be listed; else a refined key is refined in place.
  template <bool LIST = true>
  __device__ __forceinline__ void score(int j, Step& s, u32x4* h4, u32x4* l4, uint32_t* mask) {
    if (DBG) {
#pragma unroll
      for (int q = 0; q < CH; ++q) dbg_key0[DBG ? q : 0] = (c0 + (j * CH + q) * cstride) * kChunk;
    }
    i32x4 t[CH];
    step_product(s.a, t);
    const bool whole = s.loc[0].nk == kChunk && s.loc[1].nk == kChunk;  // uniform
    float x[NSET][4], scale[NSET];
    bool any = false;
#pragma unroll
    for (int b = 0; b < NSET; ++b) {
      // pinned here: widened or ORed where they are requested, the scales
      // would be waited for there
      uint16_t sc0 = s.sc[PK == 2 ? 0 : b], sc1 = s.sc[PK == 2 ? 1 : b];
      asm volatile("" : "+v"(sc0), "+v"(sc1));
      // 1/256 for the products' unit goes to the key scale: its eight significant
      // bits stay exact down to the smallest BF16, where eta's 24 would not
      const float sc = bf16_lo(PK == 2 ? static_cast<uint32_t>(sc0) | sc1 : sc0) * (1.0f / 256.0f);
      // the scale of key 4(l/16)+i sits in lane i of the quad; -inf in the lanes
      // of no row (zp = +inf there)
      x[b][0] = __builtin_fmaf(etap * quad_lane<0>(sc), static_cast<float>(t[b][0]), -zp);
      x[b][1] = __builtin_fmaf(etap * quad_lane<1>(sc), static_cast<float>(t[b][1]), -zp);
      x[b][2] = __builtin_fmaf(etap * quad_lane<2>(sc), static_cast<float>(t[b][2]), -zp);
      x[b][3] = __builtin_fmaf(etap * quad_lane<3>(sc), static_cast<float>(t[b][3]), -zp);
      scale[b] = sc;
      if (!whole) {
        const int nkl = keys_of(s, b);
#pragma unroll
        for (int i = 0; i < 4; ++i) x[b][i] = 4 * grp + i < nkl ? x[b][i] : -INFINITY;
      }
      any = any || fmaxf(fmaxf(x[b][0], x[b][1]), fmaxf(x[b][2], x[b][3])) >= thr;
    }
    uint32_t refv[NSET] = {}, rvmask = 0;
    u32x4 R[V8 ? CH : 1][V8 ? D / 64 : 1];
    if (__builtin_expect(__builtin_amdgcn_ballot_w64(any) != 0, 0)) {  // uniform: some key is refined
      uint32_t u[NSET], sets[NSET], both = 0;
#pragma unroll
      for (int b = 0; b < NSET; ++b) {
        const int nkl = keys_of(s, b);
        uint32_t bits = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i)
          if (x[b][i] >= thr && pok && 4 * grp + i < nkl) bits |= 1u << i;
        u[b] = rows_or(bits);
        sets[b] = key_mask(u[b]);
        both |= sets[b] << (16 * b);
      }
      if (LIST && __builtin_expect(__builtin_popcount(both) <= list_most, 1)) {  // uniform
#pragma unroll
        for (int b = 0; b < NSET; ++b) {
          float sl = scale[b];
          asm volatile("" : "+v"(sl));  // the scales above stay operands of the multiplies
          const float e[4] = {quad_lane<0>(sl), quad_lane<1>(sl), quad_lane<2>(sl), quad_lane<3>(sl)};
          append(s, x[b], e, u[b], sets[b], b);
          if (DBG) debug_stream(b, x[b], u[b], keys_of(s, b));
#pragma unroll
          for (int i = 0; i < 4; ++i)  // listed keys leave the stream, in every row
            if ((u[b] >> i) & 1u) x[b][i] = -INFINITY;
        }
        // their weight in the stream is 0, but 0 times an infinite value is not
        // (E4M3 has no infinity); cleared here, where few steps come, and not in
        // the staged tile, whose extra branch cost the dense scans 2.5 to 4 %
        if constexpr (DENSE && !V8) clear_values(s, both);
      } else {
        refine(s, scale, x, refv, &rvmask, R);
      }
    } else if (DBG) {
#pragma unroll
      for (int b = 0; b < NSET; ++b) debug_stream(b, x[b], 0u, keys_of(s, b));
    }
    u32x2 hi[NSET], lo[NSET];
    *mask = 0;
#pragma unroll
    for (int b = 0; b < NSET; ++b) {
      float w[4];
      uint32_t live = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w[i] = exp2_fast(x[b][i]);
        lsum += w[i];
        if constexpr (!DENSE) {
          const bool lv = x[b][i] >= a.d.neg_T;
          if (cut_out) lcut += lv ? 0.0f : w[i];
          w[i] = lv ? w[i] : 0.0f;
          if (lv) live |= 1u << i;
        }
      }
      if constexpr (!DENSE) *mask |= key_mask(rows_or(live)) << (16 * b);
      halves(w, &hi[b], &lo[b]);
    }
    operand(hi, h4);
    operand(lo, l4);
    if constexpr (V8) {
      if (__builtin_expect(rvmask != 0, 0)) {  // uniform: second plane of the keys refined here
#pragma unroll
        for (int b = 0; b < NSET; ++b) {
          // it counts only where this row's own group read it
          const uint32_t r = refv[b];
          const u32x2 mk = {((r & 1u) ? 0x0000FFFFu : 0u) | ((r & 2u) ? 0xFFFF0000u : 0u),
                            ((r & 4u) ? 0x0000FFFFu : 0u) | ((r & 8u) ? 0xFFFF0000u : 0u)};
          hi[b] = u32x2{hi[b].x & mk.x, hi[b].y & mk.y};
          lo[b] = u32x2{lo[b].x & mk.x, lo[b].y & mk.y};
        }
        u32x4 h2, l2;
        operand(hi, &h2);
        operand(lo, &l2);
#pragma unroll
        for (int q = 0; q < CH; ++q) put<D, PSTRIDE, D / 64>(R[q], tile + q * 16 * PSTRIDE);
        product32(h2, l2, 0.0625f);
        // the last sums' wait states, kept on this side of the branch back
        asm volatile("s_nop 7" : "+v"(acc[NB - 1]));
      }
    }
  }

  // The product's operand (32 keys) of a step's weight halves.
  __device__ __forceinline__ void operand(const u32x2 (&h)[NSET], u32x4* o) const {
    if constexpr (PK == 2)  // chunk 1's weights back to row lanes 0-7 (row_shl:8)
      *o = u32x4{h[0].x, h[0].y, shl8(h[0].x), shl8(h[0].y)};
    else
      *o = u32x4{h[0].x, h[0].y, h[NSET - 1].x, h[NSET - 1].y};
  }

  // Keys of the chunk a score pass weighs in this lane.
  __device__ __forceinline__ int keys_of(const Step& s, int set) const {
    return static_cast<int>(PK == 2 ? (slot ? s.loc[1].nk : s.loc[0].nk) : s.loc[set].nk);
  }

  // Refines a step in place: verdicts, plane B (and second value plane) rows
  // of both chunks as whole lines, refined scores in x.  Waits a round trip,
  // for up to 32 keys at once.
  __device__ __forceinline__ void refine(const Step& s, const float (&scale)[NSET],
                                         float (&x)[NSET][4], uint32_t (&refv)[NSET],
                                         uint32_t* rvmask,
                                         u32x4 (&R)[V8 ? CH : 1][V8 ? D / 64 : 1]) {
    uint32_t ref[NSET], bmask = 0;
#pragma unroll
    for (int b = 0; b < NSET; ++b) {
      const int nkl = keys_of(s, b);
      uint32_t lv = 0, rf = 0, rv = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const bool ok = pok && 4 * grp + i < nkl;
        if (ok && (DENSE || x[b][i] >= a.d.neg_T)) lv |= 1u << i;
        if (ok && x[b][i] >= ntau) rf |= 1u << i;
        if (V8 && ok && x[b][i] >= ntau_v) rv |= 1u << i;
      }
      const uint32_t bits = group_verdicts(lv | (rv << 8) | (rf << 16));
      ref[b] = (bits >> 16) & 0xFu;
      refv[b] = (bits >> 8) & 0xFu;
      const uint32_t u = rows_or(bits);
      bmask |= key_mask((u >> 16) & 0xFu) << (16 * b);
      if (V8) *rvmask |= key_mask((u >> 8) & 0xFu) << (16 * b);
      if (DBG) debug_refine(b, x[b], u, nkl);
    }
    u32x4 B[CH][NKI];
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const rsrc_t rb = rows_at<D>(a.keys.kb, s.loc[q]);
#pragma unroll
      for (int c = 0; c < NKI; ++c) {
        const uint32_t off = 1024u * c + 16u * lane;
        B[q][c] = buf_load(rb, (bmask >> (16 * q + off / D)) & 1u ? off : kOutOfRange);
      }
      if constexpr (V8) {
        const rsrc_t rr = rows_at<D>(a.vr, s.loc[q]);
#pragma unroll
        for (int c = 0; c < D / 64; ++c) {
          const uint32_t off = 1024u * c + 16u * lane;
          R[q][c] = buf_load(rr, (*rvmask >> (16 * q + off / D)) & 1u ? off : kOutOfRange);
        }
      }
    }
    i32x4 t[CH];
    step_product(B, t);
    if constexpr (V8) {
      // landed here, on every path out: a load in flight on one path only would
      // be waited for by all that reuse its registers
#pragma unroll
      for (int q = 0; q < CH; ++q)
#pragma unroll
        for (int c = 0; c < D / 64; ++c) asm volatile("" : "+v"(R[q][c]));
    }
#pragma unroll
    for (int b = 0; b < NSET; ++b) {
      const float e[4] = {quad_lane<0>(scale[b]), quad_lane<1>(scale[b]), quad_lane<2>(scale[b]),
                          quad_lane<3>(scale[b])};
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((ref[b] >> i) & 1u)
          x[b][i] = x[b][i] + (etap * e[i]) * (static_cast<float>(t[b][i]) * (1.0f / 256.0f));
      if (DBG) debug_x(b, x[b], keys_of(s, b));
    }
  }

  // OR over the rows of one GQA group (aligned groups of lanes) of the fields
  // live, refine-V (<< 8) and refine-K (<< 16); refine only live keys.
  __device__ __forceinline__ uint32_t group_verdicts(uint32_t bits) const {
    if (gspan >= 1) bits = dpp_or<0xB1>(bits);    // quad_perm [1, 0, 3, 2]
    if (gspan >= 3) bits = dpp_or<0x4E>(bits);    // quad_perm [2, 3, 0, 1]
    if (gspan >= 7) bits = dpp_or<0x141>(bits);   // row_half_mirror
    if (gspan >= 15) bits = dpp_or<0x140>(bits);  // row_mirror
    return bits & (((bits & 0xFFu) << 16) | ((bits & 0xFFu) << 8) | 0xFFu);
  }

  // 256 (p . qa) + p . qb of a step's two plane chunks (whole-line loads),
  // through the tile; PK == 2: both packed in t[0].
  __device__ __forceinline__ void step_product(const u32x4 (&pl)[CH][NKI], i32x4 (&t)[CH]) const {
#pragma unroll
    for (int q = 0; q < CH; ++q) put<D, PSTRIDE, NKI>(pl[q], tile + q * 16 * PSTRIDE);
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      u32x4 op[NKI];
#pragma unroll
      for (int c = 0; c < NKI; ++c)
        op[c] = *reinterpret_cast<const u32x4*>(tile + (q * 16 + n16) * PSTRIDE + 64 * c + 16 * grp);
      t[q] = plane_product(op);
    }
    if constexpr (PK == 2) {
#pragma unroll
      for (int i = 0; i < 4; ++i)  // row_shr:8 into the upper half of each row
        t[0][i] = __builtin_amdgcn_update_dpp(t[0][i], t[1][i], 0x118, 0xF, 0xC, false);
    } else {
      // Taken here, before any branch: the compiler sank the second chunk's sums
      // into the block after one, where on the taken path it left 5 to 7 wait
      // states, and not the 8 a vector read of these products needs.
      asm volatile("" : "+v"(t[0]), "+v"(t[1]));
    }
  }

  // A step's value rows (V8: first plane) into the tile, and its product.
  __device__ __forceinline__ void put_values(const u32x4 (&v)[CH][NKV]) const {
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      if constexpr (V8) put<D, PSTRIDE, NKV>(v[q], tile + q * 16 * PSTRIDE);
      else put<2 * D, VSTRIDE, NKV>(v[q], tile + q * 16 * VSTRIDE);
    }
  }

  // Dense decode, step j: plane A in s.a, values in s.v; those of step `next`
  // are requested into the same registers.
  __device__ __forceinline__ void step_dense(int j, Step& s, int next) {
    u32x4 hi = {0, 0, 0, 0}, lo = {0, 0, 0, 0};
    uint32_t mask;
    const bool some = s.loc[0].nk != 0;  // uniform; the loads are issued all the same
    if (some) score(j, s, &hi, &lo, &mask);
    issue_a(next, s);
    if (some) put_values(s.v);
    issue_v(s);
    if (some) product32(hi, lo);
  }

  // Finite depth, step j: plane A in s.a; plane A of step `next` is requested
  // into the same registers.  d holds the step before, whose value rows were
  // requested when it was scored: its product, then this step takes its place.
  __device__ __forceinline__ void step_gated(int j, Step& s, int next, Pending& d) {
    u32x4 hi = {0, 0, 0, 0}, lo = {0, 0, 0, 0};
    uint32_t mask = 0;
    if (s.loc[0].nk != 0) score(j, s, &hi, &lo, &mask);  // uniform; the loads are issued all the same
    const RowLoc l0 = s.loc[0], l1 = s.loc[1];
    issue_a(next, s);
    settle(d);
    d.hi = hi;
    d.lo = lo;
    d.mask = mask;
    issue_gated(d, l0, l1);
  }

  // The scan of a wave of one step, requested in s: nothing to request ahead,
  // and nothing to hide a gather behind.
  __device__ __forceinline__ void step_only(Step& s, Pending& d) {
    u32x4 hi, lo;
    uint32_t mask;
    score<false>(0, s, &hi, &lo, &mask);
    if constexpr (DENSE) {
      put_values(s.v);
      product32(hi, lo);
    } else {
      d.hi = hi;
      d.lo = lo;
      d.mask = mask;
      issue_gated(d, s.loc[0], s.loc[1]);
      settle(d);
    }
  }

  // Requests the value rows of d's live keys (chunks at l0 and l1).
  __device__ __forceinline__ void issue_gated(Pending& d, const RowLoc& l0, const RowLoc& l1) const {
    // every load is issued, those of cut keys with an offset that moves no
    // bytes: the count of loads in flight stays known (an offset each: equal
    // ones would be merged, and a copy waits)
    constexpr uint32_t kRowBytes = V8 ? D : 2 * D;
    const unsigned char* base = V8 ? a.vp : reinterpret_cast<const unsigned char*>(g.v);
    // bit 16 q + 1024 i / row bytes of the lane's copy is its key of load i
    const int own = static_cast<int>(d.mask >> (16u * lane / kRowBytes));
#pragma unroll
    for (int q = 0; q < CH; ++q) {
      const rsrc_t rv = rows_at<kRowBytes>(base, q ? l1 : l0);
#pragma unroll
      for (int i = 0; i < NKV; ++i) {
        const int bit = 16 * q + 1024 * i / static_cast<int>(kRowBytes);
        const uint32_t all = static_cast<uint32_t>((own << (31 - bit)) >> 31);  // 0 or ~0
        d.v[q][i] = buf_load(rv, (all & (1024u * i + 16u * lane)) | (~all & (kOutOfRange + 16u * i)));
      }
    }
    load_fence();
  }

  __device__ __forceinline__ void settle(Pending& d) {
    if (d.mask == 0) return;  // uniform: no live key
    put_values(d.v);
    product32(d.hi, d.lo);
  }

  static __device__ __forceinline__ uint32_t shl8(uint32_t v) {
    return static_cast<uint32_t>(__builtin_amdgcn_mov_dpp(static_cast<int>(v), 0x108, 0xF, 0xF, true));
  }

  // Debug exports of a score pass: coarse x of every key, x and read bits of
  // the keys that stay in the stream unrefined (u: the lane's listed keys).
  __device__ __forceinline__ void debug_stream(int set, const float (&x)[4], uint32_t u, int nkl) {
    if constexpr (DBG) {
      uint32_t lv = 0;
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (pok && 4 * grp + i < nkl && (DENSE || x[i] >= a.d.neg_T)) lv |= 1u << i;
      debug_gates(set, rows_or(lv), u, nkl);
      const int key0 = debug_key0(set);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (pok && 4 * grp + i < nkl && a.xc_out)
          a.xc_out[prow * g.max_seq_len + key0 + 4 * grp + i] = x[i];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (pok && 4 * grp + i < nkl && a.d.x_out && !((u >> i) & 1u))
          a.d.x_out[prow * g.max_seq_len + key0 + 4 * grp + i] = x[i];
    }
  }

  // ... of a step refined in place: coarse x and read bits (bits: verdict
  // fields ORed over the rows), then the final x.
  __device__ __forceinline__ void debug_refine(int set, const float (&x)[4], uint32_t bits, int nkl) {
    if constexpr (DBG) {
      debug_gates(set, bits, 0u, nkl);
      const int key0 = debug_key0(set);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (pok && 4 * grp + i < nkl && a.xc_out)
          a.xc_out[prow * g.max_seq_len + key0 + 4 * grp + i] = x[i];
    }
  }
  __device__ __forceinline__ void debug_x(int set, const float (&x)[4], int nkl) {
    if constexpr (DBG) {
      const int key0 = debug_key0(set);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (pok && 4 * grp + i < nkl && a.d.x_out)
          a.d.x_out[prow * g.max_seq_len + key0 + 4 * grp + i] = x[i];
    }
  }
  __device__ __forceinline__ int debug_key0(int set) const {
    if constexpr (DBG) return (PK == 2 ? slot : set) ? dbg_key0[1] : dbg_key0[0];
    return 0;
  }
  // Read bits of the lane's keys that are not listed (u), and the page's.
  __device__ __forceinline__ void debug_gates(int set, uint32_t bits, uint32_t u, int nkl) {
    if constexpr (DBG) {
      const int key0 = debug_key0(set);
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int k = 4 * grp + i;
        if (k >= nkl || n16 % BW != 0 || ((u >> i) & 1u)) continue;
        const size_t kr = gate_row * g.max_seq_len + key0 + k;
        if (a.d.key_gate_out) a.d.key_gate_out[kr] = (bits >> i) & 1u;
        if (a.refine_gate_out) a.refine_gate_out[kr] = (bits >> (16 + i)) & 1u;
        if (V8 && a.refine_v_gate_out) a.refine_v_gate_out[kr] = (bits >> (8 + i)) & 1u;
      }
      uint32_t any = bits & 0xFu;
      any |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(any), 16, 64));
      any |= static_cast<uint32_t>(__shfl_xor(static_cast<int>(any), 32, 64));
      if (a.d.page_gate_out && n16 % BW == 0 && grp == 0 && nkl > 0)
        a.d.page_gate_out[gate_row * ((g.max_seq_len + kChunk - 1) / kChunk) + key0 / kChunk] =
            any ? 1 : 0;
    }
  }

  // The first `keys` (at most 16) keys of the list: verdicts, reads, refined
  // scores, weights, products.
  __device__ __forceinline__ void gather(int keys) {
    const int at = head;  // a multiple of 16
    float x[4];
    uint32_t lv = 0, rf = 0, rv = 0;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float xc = list_x[(at + 4 * grp + i) * BW + n16 % BW];
      const bool ok = rok && 4 * grp + i < keys;
      x[i] = ok ? xc : -INFINITY;
      if (ok && (DENSE || xc >= a.d.neg_T)) lv |= 1u << i;
      if (ok && xc >= ntau) rf |= 1u << i;
      if (V8 && ok && xc >= ntau_v) rv |= 1u << i;
    }
    const uint32_t bits = group_verdicts(lv | (rv << 8) | (rf << 16));
    const uint32_t u = group_or16(bits);
    uint32_t vm = 0, bm = 0, rvm = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      const uint32_t r = static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(u), 16 * q));
      vm |= (r & 0xFu) << (4 * q);
      rvm |= ((r >> 8) & 0xFu) << (4 * q);
      bm |= ((r >> 16) & 0xFu) << (4 * q);
    }
    if (DBG && lane < keys) {
      const size_t kr = gate_row * g.max_seq_len + list_key[at + lane];
      if (a.d.key_gate_out) a.d.key_gate_out[kr] = (vm >> lane) & 1u;
      if (a.refine_gate_out) a.refine_gate_out[kr] = (bm >> lane) & 1u;
      if (V8 && a.refine_v_gate_out) a.refine_v_gate_out[kr] = (rvm >> lane) & 1u;
    }
    u32x4 B[NKI], V[NKV], R[V8 ? D / 64 : 1];
    {
      const uint32_t row = list_row[at + n16];
      const bool want = ((bm >> n16) & 1u) && row != kNoRow;
#pragma unroll
      for (int c = 0; c < NKI; ++c)
        B[c] = want ? *reinterpret_cast<const u32x4*>(a.keys.kb + static_cast<size_t>(row) * D +
                                                      64 * c + 16 * grp)
                    : u32x4{0, 0, 0, 0};
    }
    constexpr uint32_t kRowBytes = V8 ? D : 2 * D;
    const unsigned char* vbase = V8 ? a.vp : reinterpret_cast<const unsigned char*>(g.v);
#pragma unroll
    for (int i = 0; i < NKV; ++i) {
      const uint32_t off = 1024u * i + 16u * lane;
      const uint32_t key = off / kRowBytes;
      const uint32_t row = list_row[at + key];
      const bool want = ((vm >> key) & 1u) && row != kNoRow;
      V[i] = want ? *reinterpret_cast<const u32x4*>(
                        vbase + static_cast<size_t>(row) * kRowBytes + (off - key * kRowBytes))
                  : u32x4{0, 0, 0, 0};
    }
    if constexpr (V8) {
#pragma unroll
      for (int i = 0; i < D / 64; ++i) {
        const uint32_t off = 1024u * i + 16u * lane;
        const uint32_t key = off / D;
        const uint32_t row = list_row[at + key];
        const bool want = ((rvm >> key) & 1u) && row != kNoRow;
        R[i] = want ? *reinterpret_cast<const u32x4*>(a.vr + static_cast<size_t>(row) * D +
                                                      (off - key * D))
                    : u32x4{0, 0, 0, 0};
      }
    }
    if (bm) {  // uniform: some key is refined
      const uint32_t refl = (bits >> 16) & 0xFu;
      const i32x4 t = plane_product(B);
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if ((refl >> i) & 1u)
          x[i] = x[i] + (etap * list_e[at + 4 * grp + i]) * (static_cast<float>(t[i]) * (1.0f / 256.0f));
    }
    float w[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      w[i] = exp2_fast(x[i]);
      const bool live = DENSE || x[i] >= a.d.neg_T;
      lsum += w[i];
      if (!DENSE) lcut += live ? 0.0f : w[i];
      w[i] = live ? w[i] : 0.0f;
      if (DBG && a.d.x_out && rok && 4 * grp + i < keys)
        a.d.x_out[xrow * g.max_seq_len + list_key[at + 4 * grp + i]] = x[i];
    }
    u32x2 hi, lo;
    halves(w, &hi, &lo);
    stage(V, 1.0f);
    product16(hi, lo);
    if constexpr (V8) {
      if (rvm) {
        // the second plane counts only where this row's own group read it
        const uint32_t r = (bits >> 8) & 0xFu;
        const u32x2 mk = {((r & 1u) ? 0x0000FFFFu : 0u) | ((r & 2u) ? 0xFFFF0000u : 0u),
                          ((r & 4u) ? 0x0000FFFFu : 0u) | ((r & 8u) ? 0xFFFF0000u : 0u)};
        stage(R, 0.0625f);
        product16(u32x2{hi.x & mk.x, hi.y & mk.y}, u32x2{lo.x & mk.x, lo.y & mk.y});
      }
    }
    head = head + 16 < kListKeys ? head + 16 : 0;
    count -= keys;
  }
};

// ONE: no wave has more than one step (launch_q8_decode_rows).  A step requests
// two ahead, and where there are none, its loads that move no bytes, and their
// resources, are most of what a wave issues: 64 x 1024 keys, 8 splits, dense,
// groups of 8 10.6 us without this form and 8.6 with it, of 16 24.8 and 20.4.
// A branch in one kernel spills in the loop (groups of 8, 8-16K keys 94 -> 131 us).
template <int D, int PK, bool DENSE, bool DBG, bool V8, bool ONE>
__global__ __launch_bounds__(kScanThreads)
__attribute__((amdgpu_waves_per_eu(D == 128 ? 2 : 3)))
void decode_q8_rows_kernel(const Q8DecodeArgs a) {
  using S = Q8Rows<D, PK, DENSE, DBG, V8>;
  constexpr int kWaveFloats = S::NB * 4 * 64 + 64;  // one wave's accumulators, L and cut mass
  constexpr int kRedBytes = kScanWaves * kWaveFloats * 4;
  constexpr int kScanBytes = kScanWaves * S::kWaveBytes;
  __shared__ __attribute__((aligned(16))) unsigned char smem[kScanBytes > kRedBytes ? kScanBytes : kRedBytes];

  const ScanGeometry& g = a.d.geo;
  S sc(a);
  sc.p = a.d.by_length ? scan_place_by_length(a.d) : scan_place(a.d);
  sc.lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  sc.n16 = sc.lane & 15;
  sc.grp = sc.lane >> 4;
  sc.slot = sc.n16 / S::BW;
  sc.tile = smem + wave * S::kWaveBytes;
  sc.list_x = reinterpret_cast<float*>(sc.tile + S::kTile);
  sc.list_row = reinterpret_cast<uint32_t*>(sc.list_x + S::BW * kListKeys);
  sc.list_e = reinterpret_cast<float*>(sc.list_row + kListKeys);
  sc.list_key = reinterpret_cast<int*>(sc.list_e + kListKeys);
  sc.head = sc.count = 0;
  sc.gate_row = static_cast<size_t>(sc.p.seq) * g.hkv + sc.p.kvh;
  sc.gspan = (g.group < 16 ? g.group : 16) - 1;
  sc.pshift = q8_page_shift(g);
  sc.cstride = kScanWaves * a.d.num_splits;
  sc.c0 = kScanWaves * sc.p.split + wave;
  sc.m = sc.p.nchunks > sc.c0 ? (sc.p.nchunks - sc.c0 + sc.cstride - 1) / sc.cstride : 0;
  const int steps = (sc.m + S::CH - 1) / S::CH;
  sc.window(0);
  sc.cut_out = a.d.part_Lcut != nullptr;
  // a wave of one step has nothing to hide a gather behind: refined in place,
  // its keys wait for one round trip and not two
  sc.list_most = steps > 1 ? kListMost : 0;

  // The rows' query planes, Z, eta and thresholds are requested before the
  // stream's first loads and taken after them: one round trip less in a short
  // scan.  A lane of no row reads request 0's (there is one) and drops them.
  const RowInfo ri = row_info(g, sc.p.seq, sc.p.kvh, sc.n16, sc.p.nrows, sc.p.req0);
  sc.rok = ri.ok;
  const size_t row = static_cast<size_t>(ri.ok ? ri.req : 0) * g.heads + (ri.ok ? ri.head : 0);
  u32x4 qa[S::NKI], qb[S::NKI];
#pragma unroll
  for (int c = 0; c < S::NKI; ++c) {
    const int8_t* src = a.qp + row * 2 * D + 64 * c + 16 * sc.grp;
    qa[c] = *reinterpret_cast<const u32x4*>(src);
    qb[c] = *reinterpret_cast<const u32x4*>(src + D);
  }
  float z = a.d.z[row];
  float eta = a.eta[row];
  float nt = -a.tau[ri.ok ? ri.req : 0];
  float ntv = V8 ? -a.tau_v[ri.ok ? ri.req : 0] : 0.0f;
  sc.lsum = sc.lcut = 0.0f;
#pragma unroll
  for (int blk = 0; blk < S::NB; ++blk) sc.acc[blk] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};

  // two steps in flight, each in registers of its own
  typename S::Step s0, s1;
  typename S::Pending pend;
  sc.issue_a(0, s0);
  sc.issue_v(s0);
  if constexpr (!ONE) {
    sc.issue_a(1, s1);
    sc.issue_v(s1);
    pend.mask = 0;
    if constexpr (!DENSE) sc.issue_gated(pend, s0.loc[0], s0.loc[1]);  // no bytes: as the loop leaves it
  }

  {
    sc.qrow = sc.tile + S::kTile + S::kListBytes + sc.n16 * S::QSTRIDE + 16 * sc.grp;
#pragma unroll
    for (int c = 0; c < S::NKI; ++c) {
      qa[c] = ri.ok ? qa[c] : u32x4{0, 0, 0, 0};
      qb[c] = ri.ok ? qb[c] : u32x4{0, 0, 0, 0};
      if constexpr (S::kQueryLds) {
        *reinterpret_cast<u32x4*>(sc.qrow + 64 * c) = qa[c];
        *reinterpret_cast<u32x4*>(sc.qrow + D + 64 * c) = qb[c];
      } else {
        sc.qa[c] = qa[c];
        sc.qb[c] = qb[c];
      }
    }
    z = ri.ok ? z : INFINITY;
    eta = ri.ok ? eta : 0.0f;
    nt = ri.ok ? nt : 0.0f;
    ntv = V8 && ri.ok ? ntv : 0.0f;
    // the packed row's values sit in lane n16 % BW of the same 16 lanes
    const int src = (sc.lane & ~15) | (sc.n16 % S::BW);
    sc.pok = __shfl(static_cast<int>(sc.rok), src, 64) != 0;
    sc.zp = __shfl(z, src, 64);
    sc.etap = __shfl(eta, src, 64);
    sc.ntau = __shfl(nt, src, 64);
    sc.ntau_v = __shfl(ntv, src, 64);
    // a key is refined when some row reaches a threshold and some row is live
    sc.thr = V8 ? fminf(sc.ntau, sc.ntau_v) : sc.ntau;
    if (!DENSE) sc.thr = fmaxf(sc.thr, a.d.neg_T);
    if (DBG) {
      const RowInfo rp = row_info(g, sc.p.seq, sc.p.kvh, sc.n16 % S::BW, sc.p.nrows, sc.p.req0);
      sc.xrow = row;
      sc.prow = static_cast<size_t>(rp.req) * g.heads + rp.head;
    }
  }
  if constexpr (ONE) {
    if (steps > 0) sc.step_only(s0, pend);  // uniform
  } else {
    auto step = [&](int j, typename S::Step& st) {
      if constexpr (DENSE)
        sc.step_dense(j, st, j + 2);
      else
        sc.step_gated(j, st, j + 2, pend);
    };
    // an odd last step is followed by an empty one: a way out between the two
    // would be a path on which fewer loads follow those of the next step, and the
    // waits would be set for it
    for (int j = 0;; j += 2) {
      const bool last = j + 2 >= steps;  // uniform
      if (j < steps) {
        step(j, s0);
        step(j + 1, s1);
      }
      // one copy of the gather (short scans wait for its instructions): the list
      // holds two steps' keys beside the 15 left over
      while (sc.count >= (last ? 1 : S::kGatherKeys))  // uniform
        sc.gather(min(sc.count, S::kGatherKeys));
      if (last) break;
    }
    if constexpr (!DENSE) sc.settle(pend);
  }

  // L and cut mass: the lanes of a row hold different keys; add them.
#pragma unroll
  for (int sh = S::BW; sh < 64; sh <<= 1) {
    sc.lsum += __shfl_xor(sc.lsum, sh, 64);
    sc.lcut += __shfl_xor(sc.lcut, sh, 64);
  }

  // Add the four waves through LDS (the tiles are dead now): each wave stores
  // its accumulators in its own region (in their lane order, so that no two
  // lanes share a bank), one barrier, then every thread adds four channels of
  // one row over the waves in wave order and stores them as one 16-byte group.
  // Row n16's accumulator sits at (blk * 4 + i) * 64 + l with l % 16 = n16 and
  // channel 16 blk + 4 (l / 16) + i; lanes 0-15 of a region hold L, lanes
  // 16-31 the cut mass (lane n16 < BW holds packed row n16).
  __shared__ long long out_row[16];  // query row of row n16, or -1
  __syncthreads();
  float* red = reinterpret_cast<float*>(smem);
  {
    float* mine = red + wave * kWaveFloats;
#pragma unroll
    for (int blk = 0; blk < S::NB; ++blk)
#pragma unroll
      for (int i = 0; i < 4; ++i) mine[(blk * 4 + i) * 64 + sc.lane] = sc.acc[blk][i];
    if (sc.lane < 32) mine[S::NB * 4 * 64 + sc.lane] = sc.lane < 16 ? sc.lsum : sc.lcut;
    if (wave == 0 && sc.lane < 16) {
      const RowInfo ri = row_info(g, sc.p.seq, sc.p.kvh, sc.n16, sc.p.nrows, sc.p.req0);
      out_row[sc.lane] = ri.ok ? static_cast<long long>(ri.req) * g.heads + ri.head : -1;
    }
  }
  __syncthreads();
  const size_t slot_rows = (static_cast<size_t>(a.d.slot_offset) + sc.p.split) * g.batch * g.heads;
  const bool vec_ok = (reinterpret_cast<uintptr_t>(a.d.part_A) & 15u) == 0;
  for (int f = threadIdx.x; f < 16 * (D / 4); f += kScanThreads) {
    const int r = f / (D / 4);
    const int d = 4 * (f % (D / 4));
    const long long xr = out_row[r];
    if (xr < 0) continue;
    const int base = (d / 16) * 4 * 64 + 16 * ((d % 16) / 4) + r;
    float v[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int e = base + i * 64;
      v[i] = ((red[e] + red[kWaveFloats + e]) + red[2 * kWaveFloats + e]) + red[3 * kWaveFloats + e];
      if (V8) v[i] *= a.v_scale;  // 2^e: exact
    }
    float* dst = a.d.part_A + (slot_rows + static_cast<size_t>(xr)) * D + d;
    if (vec_ok) {
      *reinterpret_cast<f32x4*>(dst) = f32x4{v[0], v[1], v[2], v[3]};
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) dst[i] = v[i];
    }
  }
  if (threadIdx.x < 32) {
    const int r = threadIdx.x & 15;
    const long long xr = out_row[r];
    const int e = S::NB * 4 * 64 + threadIdx.x;
    const float v = ((red[e] + red[kWaveFloats + e]) + red[2 * kWaveFloats + e]) + red[3 * kWaveFloats + e];
    if (xr >= 0) {
      if (threadIdx.x < 16)
        a.d.part_L[slot_rows + static_cast<size_t>(xr)] = v;
      else if (a.d.part_Lcut)
        a.d.part_Lcut[slot_rows + static_cast<size_t>(xr)] = v;
    }
  }
}

template <int D, int PK, bool DENSE, bool V8>
hipError_t launch_rows(const Q8DecodeArgs& a, bool dbg, unsigned blocks, hipStream_t stream) {
  // the longest sequence the view holds gives a wave at most two chunks
  const bool one = a.d.geo.max_seq_len <= 2LL * kScanWaves * kChunk * a.d.num_splits;
  const dim3 grid(blocks), block(kScanThreads);
  if (dbg)
    hipLaunchKernelGGL((decode_q8_rows_kernel<D, PK, DENSE, true, V8, false>), grid, block, 0,
                       stream, a);
  else if (one)
    hipLaunchKernelGGL((decode_q8_rows_kernel<D, PK, DENSE, false, V8, true>), grid, block, 0,
                       stream, a);
  else
    hipLaunchKernelGGL((decode_q8_rows_kernel<D, PK, DENSE, false, V8, false>), grid, block, 0,
                       stream, a);
  return hipGetLastError();
}

template <int D, int PK>
hipError_t launch_rows_v(const Q8DecodeArgs& a, bool dbg, unsigned blocks, hipStream_t stream) {
  if (a.d.dense)
    return a.vp ? launch_rows<D, PK, true, true>(a, dbg, blocks, stream)
                : launch_rows<D, PK, true, false>(a, dbg, blocks, stream);
  return a.vp ? launch_rows<D, PK, false, true>(a, dbg, blocks, stream)
              : launch_rows<D, PK, false, false>(a, dbg, blocks, stream);
}

}  // namespace

// Two-plane scan of read groups of 2 to 16 rows (one read group per kv
// sequence and head), at any depth.
hipError_t launch_q8_decode_rows(const Q8DecodeArgs& a, int head_dim, hipStream_t stream) {
  const long long blocks = static_cast<long long>(a.d.geo.num_seqs) * a.d.geo.hkv * a.d.num_splits;
  if (blocks == 0 || a.d.geo.batch == 0) return hipSuccess;  // no row to read or write
  const unsigned nb = static_cast<unsigned>(blocks);
  const bool dbg = a.d.x_out || a.d.key_gate_out || a.d.page_gate_out || a.xc_out ||
                   a.refine_gate_out || a.refine_v_gate_out;
  const bool pack = a.d.rows_per_seq <= 8;
  if (head_dim == 128) return pack ? launch_rows_v<128, 2>(a, dbg, nb, stream)
                                   : launch_rows_v<128, 1>(a, dbg, nb, stream);
  if (head_dim == 64) return pack ? launch_rows_v<64, 2>(a, dbg, nb, stream)
                                  : launch_rows_v<64, 1>(a, dbg, nb, stream);
  return hipErrorInvalidValue;
}

}  // namespace fold
 