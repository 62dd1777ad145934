// Front of a two-plane INT8 key cache (Section 4, "Cache format"): the key
// writer, the per-step query split and the writer of 8-bit values; and the
// stacked level's FP16 keys (Appendix E, tile layouts: a level past 64
// stacked rows runs laid out as prefill is, with one FP16 product per logit
// of each key's code rounded once per prefix): q8_stack_kernel writes
// fp16(e (a + b/256)) per element, the product being exact in FP32 (a 16-bit
// code times an 8-bit scale) and rounded once, to nearest even.
//
// Both rotate a D-vector by the Sylvester Hadamard matrix H_D (entries +-1;
// the paper's orthonormal rotation is H_D / sqrt(D), and its 1/D on a dot
// product is folded into the query scale) and split the result into two INT8
// planes under one scale:
//   key   k'' = e (a + b/256), e = the smallest BF16 value >= max|k''| / 127
//         (rounded up: plane A never saturates); a key whose scale would fall
//         below 2^-126 is stored as zero;
//   query q'' = f (qa + qb/256), f = max|q''| / 127, with the base-2 score
//         scale eta = log2(e) sm_scale f / D rounded once to FP32;
//   a = rint(x / s), b = rint(256 (x / s - a)) clamped to [-128, 127].
// The query split and the writer of a step's few keys give one wave64 to a
// vector; lane l holds elements 64 i + hadamard_lane(l).  The other writers
// give D/16 lanes to a row, 16 consecutive elements each (16-byte loads and
// stores).  The transform is a radix-2 butterfly in FP64, strides 1, 2, 4, ...:
// every partial sum of +-BF16 inputs is exact while the inputs of one vector
// span at most 38 binades, so the codes do not depend on the order of the
// butterflies.  Division, rint and the rounded-up scale are exact IEEE FP64
// operations.
#include "decode_common.h"
#include "q8_split.h"

namespace fold {
namespace {

constexpr int kFrontThreads = 256;
constexpr int kWavesPerBlock = kFrontThreads / 64;

// Smallest value with 8 significant bits (a BF16 significand) >= t, t > 0 normal.
__device__ __forceinline__ double ceil_to_bf16(double t) {
  constexpr unsigned long long kLow = (1ull << 45) - 1;
  const unsigned long long u = static_cast<unsigned long long>(__double_as_longlong(t));
  return __longlong_as_double(static_cast<long long>((u + kLow) & ~kLow));
}

// The token row a group of lanes writes, and where it goes.
struct WriteRow {
  size_t src;     // row of the source [n_tok][hkv]
  long long dst;  // element row of the cache, or -1: nothing is written
};

// Row `local` of the workgroup's first row item0 of n_tok * hkv.
__device__ __forceinline__ WriteRow write_row(const ScanGeometry& g, const int32_t* tok_seq,
                                              const int32_t* tok_pos, int n_tok, long long item0,
                                              uint32_t local) {
  const int tok0 = static_cast<int>(item0 / g.hkv);  // uniform
  const uint32_t h = static_cast<uint32_t>(item0 % g.hkv) + local;
  const bool in = item0 + local < static_cast<long long>(n_tok) * g.hkv;
  const int tok = in ? tok0 + static_cast<int>(h / static_cast<uint32_t>(g.hkv)) : 0;
  WriteRow w;
  w.src = in ? static_cast<size_t>(item0 + local) : 0;
  w.dst = row_of<false>(g, in ? tok_seq[tok] : -1, tok_pos[tok],
                      static_cast<int>(h % static_cast<uint32_t>(g.hkv)));
  return w;
}

// E (4 or 16) consecutive BF16 elements, as the E/2 words that hold them.
template <int E, bool WIDE>
__device__ __forceinline__ void load_bf16(const uint16_t* src, uint32_t (&w)[E / 2]) {
  if constexpr (WIDE && E == 4) {
    const u32x2 a = *reinterpret_cast<const u32x2*>(src);
    w[0] = a.x;
    w[1] = a.y;
  } else if constexpr (WIDE) {
#pragma unroll
    for (int j = 0; j < E / 8; ++j) {
      const u32x4 a = reinterpret_cast<const u32x4*>(src)[j];
#pragma unroll
      for (int i = 0; i < 4; ++i) w[4 * j + i] = a[i];
    }
  } else {
#pragma unroll
    for (int i = 0; i < E / 2; ++i)
      w[i] = src[2 * i] | (static_cast<uint32_t>(src[2 * i + 1]) << 16);
  }
}

// E bytes, four to a word.
template <int E, bool WIDE>
__device__ __forceinline__ void store_bytes(uint8_t* dst, const uint32_t (&w)[E / 4]) {
  if constexpr (WIDE && E == 4) {
    *reinterpret_cast<uint32_t*>(dst) = w[0];
  } else if constexpr (WIDE) {
#pragma unroll
    for (int j = 0; j < E / 16; ++j)
      reinterpret_cast<u32x4*>(dst)[j] = u32x4{w[4 * j], w[4 * j + 1], w[4 * j + 2], w[4 * j + 3]};
  } else {
#pragma unroll
    for (int i = 0; i < E; ++i) dst[i] = static_cast<uint8_t>(w[i / 4] >> (8 * (i % 4)));
  }
}

// A butterfly stage across lanes: the partner's element is o, and the lane
// whose index bit is set keeps o - x.
template <int CTRL>
__device__ __forceinline__ void lane_stage(double (&x)[16], bool upper) {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const double o = dpp_f64<CTRL>(x[i]);
    x[i] = upper ? o - x[i] : x[i] + o;
  }
}

// Planes of x / s for a finite scale s > 0, without a division per element:
// with r = 1/s rounded, q = x r and two corrections q += (x - q s) r give the
// correctly rounded quotient (Markstein's theorem: the residual of a faithful
// q is exact, and r is the rounded reciprocal; s has eight significant bits
// and nothing here comes near the ends of the FP64 range).  Adding and taking
// away 1.5 2^52 rounds to an integer, ties to even, and leaves that integer in
// the low word.
__device__ __forceinline__ void split_value_rcp(double x, double s, double r, uint32_t* a,
                                                uint32_t* b) {
  constexpr double kRint = 0x1.8p52;
  double q = x * r;
  q = __builtin_fma(__builtin_fma(-q, s, x), r, q);
  q = __builtin_fma(__builtin_fma(-q, s, x), r, q);
  const double ta = q + kRint;
  const double tb = __builtin_fma(256.0, q - (ta - kRint), kRint);
  *a = static_cast<uint32_t>(__double_as_longlong(ta));
  *b = static_cast<uint32_t>(min(static_cast<int>(__double_as_longlong(tb)), 127));
}

// A vector per wave: the writer of a decode step's tokens.  Its chain is
// shorter than the row groups' below (two elements per lane and not 16), and
// there are enough waves for every row.
template <int D>
__global__ __launch_bounds__(kFrontThreads) void q8_write_wave_kernel(const Q8WriteArgs a) {
  const int lane = threadIdx.x & 63;
  const int el = hadamard_lane(lane);
  const WriteRow row = write_row(a.geo, a.tok_seq, a.tok_pos, a.n_tok,
                                 static_cast<long long>(blockIdx.x) * kWavesPerBlock,
                                 __builtin_amdgcn_readfirstlane(threadIdx.x >> 6));
  const uint16_t* src = a.k_src + row.src * D;
  double x[D / 64];
#pragma unroll
  for (int i = 0; i < D / 64; ++i) x[i] = static_cast<double>(bf16_lo(src[64 * i + el]));
  if (row.dst < 0) return;  // uniform per wave
  hadamard_wave<D>(x, lane);
  const double m = wave_absmax_f64<D>(x);
  const double e = m >= 127.0 * 0x1p-126 ? ceil_to_bf16(m / 127.0) : 0.0;
#pragma unroll
  for (int i = 0; i < D / 64; ++i) {
    int8_t qa, qb;
    split_value(x[i], e, &qa, &qb);
    a.ka[row.dst * D + 64 * i + el] = qa;
    a.kb[row.dst * D + 64 * i + el] = qb;
  }
  if (lane == 0)
    a.ks[row.dst] = static_cast<uint16_t>(__float_as_uint(static_cast<float>(e)) >> 16);
}

// D/16 lanes per row; lane p of a row holds the 16 elements from 16 b on, b =
// p below four and b = 11 - p above (D = 128), so that the partner for index
// bit 6 is the half-row mirror.  Bound by instruction issue before HBM
// bandwidth: 9 FP64 operations per element for the codes, 7 butterfly steps, and
// the exchanges' register moves (each FP64 exchange is two moves and two that
// set its destination to zero).
// 4 x 8192 tokens, 8 kv heads, D = 128 (134 MB): 54 us; 118 us with a vector
// per wave (2-byte loads, 1-byte stores, every stride through LDS shuffles).
// WIDE: source and planes are 16-byte aligned.
template <int D, bool WIDE>
__global__ __launch_bounds__(kFrontThreads) void q8_write_kernel(const Q8WriteArgs a) {
  constexpr uint32_t LPR = D / 16;
  const uint32_t p = threadIdx.x % LPR;
  const uint32_t blk = D == 128 && p >= 4 ? 11 - p : p;
  const WriteRow row = write_row(a.geo, a.tok_seq, a.tok_pos, a.n_tok,
                                 static_cast<long long>(blockIdx.x) * (kFrontThreads / LPR),
                                 threadIdx.x / LPR);
  uint32_t w[8];
  load_bf16<16, WIDE>(a.k_src + row.src * D + 16 * blk, w);
  double x[16];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    x[2 * i] = static_cast<double>(bf16_lo(w[i]));
    x[2 * i + 1] = static_cast<double>(bf16_hi(w[i]));
  }
#pragma unroll
  for (int s = 1; s < 16; s <<= 1) {
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      if (i & s) continue;
      const double u = x[i], v = x[i + s];
      x[i] = u + v;
      x[i + s] = u - v;
    }
  }
  lane_stage<0xB1>(x, blk & 1);                         // quad_perm [1, 0, 3, 2]
  lane_stage<0x4E>(x, blk & 2);                         // quad_perm [2, 3, 0, 1]
  if constexpr (D == 128) lane_stage<0x141>(x, blk & 4);  // row_half_mirror
  double m = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) m = fmax(m, fabs(x[i]));
  m = fmax(m, dpp_f64<0xB1>(m));
  m = fmax(m, dpp_f64<0x4E>(m));
  if constexpr (D == 128) m = fmax(m, dpp_f64<0x141>(m));
  if (row.dst < 0) return;
  const double e = m >= 127.0 * 0x1p-126 ? ceil_to_bf16(m / 127.0) : 0.0;
  uint32_t ca[4] = {0, 0, 0, 0}, cb[4] = {0, 0, 0, 0};
  if (e > 0.0 && e < static_cast<double>(INFINITY)) {
    const double r = 1.0 / e;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      uint32_t qa, qb;
      split_value_rcp(x[i], e, r, &qa, &qb);
      ca[i / 4] |= (qa & 0xFFu) << (8 * (i % 4));
      cb[i / 4] |= (qb & 0xFFu) << (8 * (i % 4));
    }
  } else if (e > 0.0) {  // a key with an infinity
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      int8_t qa, qb;
      split_value(x[i], e, &qa, &qb);
      ca[i / 4] |= static_cast<uint32_t>(static_cast<uint8_t>(qa)) << (8 * (i % 4));
      cb[i / 4] |= static_cast<uint32_t>(static_cast<uint8_t>(qb)) << (8 * (i % 4));
    }
  }
  const size_t at = static_cast<size_t>(row.dst) * D + 16 * blk;
  store_bytes<16, WIDE>(reinterpret_cast<uint8_t*>(a.ka) + at, ca);
  store_bytes<16, WIDE>(reinterpret_cast<uint8_t*>(a.kb) + at, cb);
  if (p == 0)
    a.ks[row.dst] = static_cast<uint16_t>(__float_as_uint(static_cast<float>(e)) >> 16);
}

template <int D>
__global__ __launch_bounds__(kFrontThreads) void q8_split_kernel(const Q8SplitArgs a) {
  const int lane = threadIdx.x & 63;
  const int el = hadamard_lane(lane);
  if (blockIdx.x == 0 && a.tau) {
    for (int r = threadIdx.x; r < a.batch; r += kFrontThreads) {
      const int n = a.req_lens[r];
      const int c = n > 1 ? 32 - __builtin_clz(static_cast<unsigned>(n - 1)) : 0;
      a.tau[r] = a.kappa + static_cast<float>(c);
      if (a.tau_v) a.tau_v[r] = a.kappa_v + static_cast<float>(c);
    }
  }
  const long long row = static_cast<long long>(blockIdx.x) * kWavesPerBlock +
                        __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (row >= a.rows) return;  // uniform per wave
  const uint16_t* src = a.q + row * D;
  double x[D / 64];
#pragma unroll
  for (int i = 0; i < D / 64; ++i) x[i] = static_cast<double>(bf16_lo(src[64 * i + el]));
  hadamard_wave<D>(x, lane);
  const double f = wave_absmax_f64<D>(x) / 127.0;
  int8_t* dst = a.qp + row * 2 * D;
#pragma unroll
  for (int i = 0; i < D / 64; ++i) {
    int8_t qa, qb;
    split_value(x[i], f, &qa, &qb);
    dst[64 * i + el] = qa;
    dst[D + 64 * i + el] = qb;
  }
  if (lane == 0)
    a.eta[row] = static_cast<float>(((kLog2eF64 * static_cast<double>(a.sm_scale)) * f) / D);
}

// E4M3 codes (OCP E4M3FN: bias 7, subnormals m 2^-9, largest finite 448) of
// four values, first in the low byte: rounded to nearest even
// (v_cvt_pk_fp8_f32) after magnitudes of 448 and above (and NaN) are set to
// 448 and those that round to zero to +0, whose code is 0.  val receives the
// codes' values.
__device__ __forceinline__ uint32_t e4m3_rne_sat4(const float (&y)[4], float (&val)[4]) {
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  float c[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    c[i] = fabsf(y[i]) < 448.0f ? y[i] : copysignf(448.0f, y[i]);
    c[i] = fabsf(c[i]) <= 0x1p-10f ? 0.0f : c[i];
  }
  int w = __builtin_amdgcn_cvt_pk_fp8_f32(c[0], c[1], 0, false);
  w = __builtin_amdgcn_cvt_pk_fp8_f32(c[2], c[3], w, true);
  const f32x2 lo = __builtin_amdgcn_cvt_pk_f32_fp8(w, false);
  const f32x2 hi = __builtin_amdgcn_cvt_pk_f32_fp8(w, true);
  val[0] = lo.x;
  val[1] = lo.y;
  val[2] = hi.x;
  val[3] = hi.y;
  return static_cast<uint32_t>(w);
}

// D/E lanes per row, E elements each: 16 for a prompt, 4 for a decode step's
// tokens (a shorter chain on more waves).  Bound by HBM bandwidth; 4 x 8192
// tokens, 8 kv heads, D = 128 (134 MB): 30 us (4.5 TB/s; a large device copy
// makes 4.9); 102 us with a row per wave (2-byte loads, 1-byte stores, the
// codes by ilogb, ldexp and rint).
// WIDE: source and planes are 16-byte aligned.
template <int D, int E, bool WIDE>
__global__ __launch_bounds__(kFrontThreads) void v8_write_kernel(const V8WriteArgs a) {
  constexpr uint32_t LPR = D / E;
  const uint32_t p = threadIdx.x % LPR;
  const WriteRow row = write_row(a.geo, a.tok_seq, a.tok_pos, a.n_tok,
                                 static_cast<long long>(blockIdx.x) * (kFrontThreads / LPR),
                                 threadIdx.x / LPR);
  uint32_t w[E / 2];
  load_bf16<E, WIDE>(a.v_src + row.src * D + E * p, w);
  if (row.dst < 0) return;
  uint32_t cp[E / 4], cr[E / 4];
#pragma unroll
  for (int i = 0; i < E / 4; ++i) {
    const float y[4] = {ldexpf(bf16_lo(w[2 * i]), -a.scale_exp),  // exact
                        ldexpf(bf16_hi(w[2 * i]), -a.scale_exp),
                        ldexpf(bf16_lo(w[2 * i + 1]), -a.scale_exp),
                        ldexpf(bf16_hi(w[2 * i + 1]), -a.scale_exp)};
    float pv[4], rest[4], rv[4];
    cp[i] = e4m3_rne_sat4(y, pv);
#pragma unroll
    for (int j = 0; j < 4; ++j) rest[j] = 16.0f * (y[j] - pv[j]);  // both exact
    cr[i] = e4m3_rne_sat4(rest, rv);
  }
  const size_t at = static_cast<size_t>(row.dst) * D + E * p;
  store_bytes<E, WIDE>(a.vp + at, cp);
  store_bytes<E, WIDE>(a.vr + at, cr);
}

// One thread per 8 elements of a key: D/8 threads per key, 256/(D/8) keys per
// workgroup.  Grid: (kv sequence, kv head, key block).
template <int D>
__global__ __launch_bounds__(kFrontThreads) void q8_stack_kernel(const Q8StackArgs a, int blocks_per_seq) {
  constexpr int TPK = D / 8;
  constexpr int KPB = kFrontThreads / TPK;
  const ScanGeometry& g = a.geo;
  int bid = blockIdx.x;
  const int kb = bid % blocks_per_seq;
  bid /= blocks_per_seq;
  const int kvh = bid % g.hkv;
  const int seq = bid / g.hkv;
  const int j = kb * KPB + static_cast<int>(threadIdx.x) / TPK;
  const int part = threadIdx.x % TPK;
  const int n = clamp_len(ld_uniform(g.seq_lens, seq), view_capacity(g));
  if (j >= n) return;
  size_t row;
  if (g.page_size > 0) {
    const int phys = g.block_table[static_cast<size_t>(seq) * g.max_pages + j / g.page_size];
    if (phys < 0 || phys >= g.num_pages) return;
    row = (static_cast<size_t>(phys) * g.hkv + kvh) * g.page_size + j % g.page_size;
  } else {
    row = (static_cast<size_t>(seq) * g.hkv + kvh) * g.max_seq_len + j;
  }
  const size_t el = row * D + 8 * part;
  const uint2 pa = *reinterpret_cast<const uint2*>(a.ka + el);
  const uint2 pb = *reinterpret_cast<const uint2*>(a.kb + el);
  const float e = bf16_lo(a.ks[row]);
  uint32_t h[8];
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const uint32_t wa = i < 4 ? pa.x : pa.y;
    const uint32_t wb = i < 4 ? pb.x : pb.y;
    const int ca = static_cast<int8_t>((wa >> (8 * (i & 3))) & 0xffu);
    const int cb = static_cast<int8_t>((wb >> (8 * (i & 3))) & 0xffu);
    // a + b/256 is exact in FP32, and so is its product with an 8-bit scale
    const float code = static_cast<float>(ca) + static_cast<float>(cb) * (1.0f / 256.0f);
    h[i] = f32_to_f16_bits(e * code);
  }
  *reinterpret_cast<u32x4*>(a.out + el) =
      u32x4{h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
}

bool all_aligned16(const void* a, const void* b, const void* c) {
  return ((reinterpret_cast<uintptr_t>(a) | reinterpret_cast<uintptr_t>(b) |
           reinterpret_cast<uintptr_t>(c)) & 15u) == 0;
}

// Workgroups of a writer with `lanes` lanes per row.
dim3 write_grid(long long items, int lanes) {
  const long long rows = kFrontThreads / lanes;
  return dim3(static_cast<unsigned>((items + rows - 1) / rows));
}

// Up to these counts a writer takes its step form, whose shorter chain is
// what counts there.  Back-to-back calls in a graph, step form / prompt form:
// keys, D = 128: 64 rows 2.67 / 3.57 us, 2048 rows 3.24 / 3.78, 4096 rows 4.09
// / 3.85, 65536 rows 30.9 / 13.7 (D = 64 crosses between the same two counts);
// values, D = 128: 64 rows 2.36 / 2.79 us, 4096 rows 2.63 / 3.04, 8192 rows
// 3.24 / 3.16, 65536 rows 12.5 / 8.1 (D = 64: at 16384 rows 3.22 / 3.14).
constexpr long long kStepKeyRows = 2048;
constexpr long long kStepValueElements = 1 << 19;

template <int D>
hipError_t launch_q8w(const Q8WriteArgs& a, long long items, hipStream_t stream) {
  const dim3 block(kFrontThreads);
  if (items <= kStepKeyRows)
    hipLaunchKernelGGL((q8_write_wave_kernel<D>), write_grid(items, 64), block, 0, stream, a);
  else if (all_aligned16(a.k_src, a.ka, a.kb))
    hipLaunchKernelGGL((q8_write_kernel<D, true>), write_grid(items, D / 16), block, 0, stream, a);
  else
    hipLaunchKernelGGL((q8_write_kernel<D, false>), write_grid(items, D / 16), block, 0, stream, a);
  return hipGetLastError();
}

template <int D, int E>
hipError_t launch_v8(const V8WriteArgs& a, long long items, hipStream_t stream) {
  const dim3 grid = write_grid(items, D / E), block(kFrontThreads);
  if (all_aligned16(a.v_src, a.vp, a.vr))
    hipLaunchKernelGGL((v8_write_kernel<D, E, true>), grid, block, 0, stream, a);
  else
    hipLaunchKernelGGL((v8_write_kernel<D, E, false>), grid, block, 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_q8_stack_keys(const Q8StackArgs& a, int head_dim, hipStream_t stream) {
  const int cap = view_capacity(a.geo);
  const int kpb = kFrontThreads / (head_dim / 8);
  const int per_seq = (cap + kpb - 1) / kpb;
  const long long blocks = static_cast<long long>(a.geo.num_seqs) * a.geo.hkv * per_seq;
  if (blocks == 0) return hipSuccess;
  if (head_dim == 128)
    hipLaunchKernelGGL(q8_stack_kernel<128>, dim3(static_cast<unsigned>(blocks)),
                       dim3(kFrontThreads), 0, stream, a, per_seq);
  else if (head_dim == 64)
    hipLaunchKernelGGL(q8_stack_kernel<64>, dim3(static_cast<unsigned>(blocks)),
                       dim3(kFrontThreads), 0, stream, a, per_seq);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t launch_v8_write(const V8WriteArgs& a, int head_dim, hipStream_t stream) {
  const long long items = static_cast<long long>(a.n_tok) * a.geo.hkv;
  if (items == 0) return hipSuccess;
  const bool step = items * head_dim <= kStepValueElements;
  if (head_dim == 128)
    return step ? launch_v8<128, 4>(a, items, stream) : launch_v8<128, 16>(a, items, stream);
  if (head_dim == 64)
    return step ? launch_v8<64, 4>(a, items, stream) : launch_v8<64, 16>(a, items, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_q8_write(const Q8WriteArgs& a, int head_dim, hipStream_t stream) {
  const long long items = static_cast<long long>(a.n_tok) * a.geo.hkv;
  if (items == 0) return hipSuccess;
  if (head_dim == 128) return launch_q8w<128>(a, items, stream);
  if (head_dim == 64) return launch_q8w<64>(a, items, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_q8_split(const Q8SplitArgs& a, int head_dim, hipStream_t stream) {
  const long long waves = a.rows > 0 ? a.rows : 1;  // block 0 also writes tau
  if (a.rows == 0 && !a.tau) return hipSuccess;
  const unsigned blocks = static_cast<unsigned>((waves + kWavesPerBlock - 1) / kWavesPerBlock);
  if (head_dim == 128)
    hipLaunchKernelGGL(q8_split_kernel<128>, dim3(blocks), dim3(kFrontThreads), 0, stream, a);
  else if (head_dim == 64)
    hipLaunchKernelGGL(q8_split_kernel<64>, dim3(blocks), dim3(kFrontThreads), 0, stream, a);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace fold
