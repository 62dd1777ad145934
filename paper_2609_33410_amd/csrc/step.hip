// The decode step around the scan: BF16 token append, the certificate's
// reference update, and the row gather that lays out draft columns.
//
// * append: the front writes each step's new token into the paged cache
//   (Section 4, "Weight-gated reads").
// * certificate update (Section 3, certificate paragraph): a flagged row is
//   decoded again with Z = its base-2 log-sum-exp; where that is not finite
//   (L formed as 0 or infinity) Z moves 64 binades towards it.
// * draft gather (Section 4, "Value product": drafts are query columns masked
//   to their ancestors): each column's ancestor keys are copied into spare
//   pages, so that the column's visible keys are the committed keys (shared
//   by every column of the request) plus a private level of its own.
//
// The certificate update is one block and the gather a wave per (column, kv
// head) moving rows of at most a few hundred bytes: both latency-bound.  The
// append is latency-bound for a step's tokens and HBM-bound for a prompt's.

#include "decode_common.h"

namespace fold {
namespace {

constexpr int kStepThreads = 256;
constexpr int kStepWaves = kStepThreads / 64;
constexpr float kCertStep = 64.0f;

// Copy one row with the widest unit its size allows; both rows start at a
// multiple of row_bytes from a 16-byte aligned base.
__device__ __forceinline__ void copy_row(uint8_t* dst, const uint8_t* src, int row_bytes,
                                         int lane) {
  if ((row_bytes & 15) == 0) {
    for (int i = lane; i < (row_bytes >> 4); i += 64)
      reinterpret_cast<uint4*>(dst)[i] = reinterpret_cast<const uint4*>(src)[i];
  } else if ((row_bytes & 1) == 0) {
    for (int i = lane; i < (row_bytes >> 1); i += 64)
      reinterpret_cast<uint16_t*>(dst)[i] = reinterpret_cast<const uint16_t*>(src)[i];
  } else {
    for (int i = lane; i < row_bytes; i += 64) dst[i] = src[i];
  }
}

// Rows of 2^LPR 16-byte pieces, one piece per lane: a wave moves 64 >> LPR
// rows per step, U steps with their loads in flight together.  U = 1 is the
// decode step's append (a few rows: as many workgroups as there are), U = 4 a
// prompt's.  A prompt of 4 x 8192 tokens, 8 kv heads, D = 128 (268 MB moved)
// took 107 us with one wave per row (16 of 64 lanes at work) and takes 56 us
// now, 4.8 TB/s, the rate of a large device copy (4.9); non-temporal stores
// are slower (60 us) and only hand the difference to the next reader.
template <int LPR, int U>
__global__ __launch_bounds__(kStepThreads) void append_rows_kernel(const AppendArgs a) {
  constexpr int kRows = kStepThreads >> LPR;  // rows per step of the workgroup
  const ScanGeometry& g = a.geo;
  const long long items = static_cast<long long>(a.n_tok) * g.hkv;
  const long long item0 = static_cast<long long>(blockIdx.x) * (kRows * U);
  const int tok0 = static_cast<int>(item0 / g.hkv);  // uniform
  const uint32_t kvh0 = static_cast<uint32_t>(item0 % g.hkv);
  const uint32_t local = threadIdx.x >> LPR;
  const uint32_t piece = threadIdx.x & ((1u << LPR) - 1);
  int seq[U], pos[U], kvh[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const uint32_t r = local + u * kRows;
    const uint32_t h = kvh0 + r;
    const bool in = item0 + r < items;
    const int tok = in ? tok0 + static_cast<int>(h / static_cast<uint32_t>(g.hkv)) : 0;
    kvh[u] = static_cast<int>(h % static_cast<uint32_t>(g.hkv));
    seq[u] = in ? a.tok_seq[tok] : -1;
    pos[u] = a.tok_pos[tok];
  }
  long long row[U];
  u32x4 k[U] = {}, v[U] = {};
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t src = static_cast<size_t>(item0 + local + u * kRows) << LPR;
    const bool in = item0 + local + u * kRows < items;
    if (a.k_dst && in) k[u] = reinterpret_cast<const u32x4*>(a.k_src)[src + piece];
    if (a.v_dst && in) v[u] = reinterpret_cast<const u32x4*>(a.v_src)[src + piece];
    row[u] = row_of<false>(g, seq[u], pos[u], kvh[u]);
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    if (row[u] < 0) continue;
    const size_t dst = (static_cast<size_t>(row[u]) << LPR) + piece;
    if (a.k_dst) reinterpret_cast<u32x4*>(a.k_dst)[dst] = k[u];
    if (a.v_dst) reinterpret_cast<u32x4*>(a.v_dst)[dst] = v[u];
  }
}

__global__ __launch_bounds__(kStepThreads) void cert_update_kernel(const CertArgs a) {
  __shared__ int partial[kStepWaves];
  int flagged = 0;
  for (int i = threadIdx.x; i < a.n; i += kStepThreads) {
    if (a.cert[i] == 0) continue;
    const float l = a.lse[i];
    const float z = a.z[i];
    float nz = z;  // NaN: no better reference is known
    if (isfinite(l))
      nz = l;
    else if (l < 0.0f)
      nz = z - kCertStep;
    else if (l > 0.0f)
      nz = z + kCertStep;
    a.z[i] = nz;
    if (a.reruns) a.reruns[i] += 1;
    ++flagged;
  }
  for (int off = 32; off > 0; off >>= 1) flagged += __shfl_xor(flagged, off);
  if ((threadIdx.x & 63) == 0) partial[threadIdx.x >> 6] = flagged;
  __syncthreads();
  if (threadIdx.x == 0) {
    int total = 0;
    for (int w = 0; w < kStepWaves; ++w) total += partial[w];
    a.count[0] = total;
  }
}

// One wave per (column, kv head): copy the column's ancestor rows into its
// spare pages; the kv head 0 wave also copies the request's block-table row
// into the column's table when one is requested.
__global__ __launch_bounds__(kStepThreads) void draft_gather_kernel(const DraftGatherArgs a) {
  const int lane = threadIdx.x & 63;
  const long long item = static_cast<long long>(blockIdx.x) * kStepWaves +
                         __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  if (item >= static_cast<long long>(a.num_cols) * a.geo.hkv) return;  // uniform per wave
  const int col = static_cast<int>(item / a.geo.hkv);
  const int kvh = static_cast<int>(item % a.geo.hkv);
  const int req = ld_uniform(a.col_req, col);
  const int cap = a.pages_per_col * a.geo.page_size;
  int n = ld_uniform(a.anc_lens, col);
  n = n < 0 ? 0 : (n > cap ? cap : n);
  if (a.col_block_table && kvh == 0 && req >= 0 && req < a.geo.num_seqs) {
    for (int p = lane; p < a.geo.max_pages; p += 64)
      a.col_block_table[static_cast<size_t>(col) * a.geo.max_pages + p] =
          a.geo.block_table[static_cast<size_t>(req) * a.geo.max_pages + p];
  }
  if (!a.src || !a.dst) return;
  for (int i = 0; i < n; ++i) {
    const int pos = ld_uniform(a.anc_pos, static_cast<size_t>(col) * cap + i);
    const long long src = row_of<true>(a.geo, req, pos, kvh);
    const int spare =
        ld_uniform(a.spare_pages, static_cast<size_t>(col) * a.pages_per_col + i / a.geo.page_size);
    if (src < 0 || spare < 0 || spare >= a.geo.num_pages) continue;
    const long long dst =
        (static_cast<long long>(spare) * a.geo.hkv + kvh) * a.geo.page_size + i % a.geo.page_size;
    copy_row(a.dst + static_cast<size_t>(dst) * a.row_bytes,
             a.src + static_cast<size_t>(src) * a.row_bytes, a.row_bytes, lane);
  }
}

// Four steps per thread once a single step would give more than four
// workgroups per compute unit (256 of them); below, latency counts and not the
// rate.
template <int LPR>
hipError_t launch_append(const AppendArgs& a, long long items, hipStream_t stream) {
  constexpr int kRows = kStepThreads >> LPR;
  const long long blocks = (items + kRows - 1) / kRows;
  if (blocks > 1024)
    hipLaunchKernelGGL((append_rows_kernel<LPR, 4>), dim3(static_cast<unsigned>((blocks + 3) / 4)),
                       dim3(kStepThreads), 0, stream, a);
  else
    hipLaunchKernelGGL((append_rows_kernel<LPR, 1>), dim3(static_cast<unsigned>(blocks)),
                       dim3(kStepThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_append_rows(const AppendArgs& a, hipStream_t stream) {
  const long long items = static_cast<long long>(a.n_tok) * a.geo.hkv;
  if (items == 0) return hipSuccess;
  if (a.row_bytes == 256) return launch_append<4>(a, items, stream);
  if (a.row_bytes == 128) return launch_append<3>(a, items, stream);
  return hipErrorInvalidValue;
}

hipError_t launch_cert_update(const CertArgs& a, hipStream_t stream) {
  hipLaunchKernelGGL(cert_update_kernel, dim3(1), dim3(kStepThreads), 0, stream, a);
  return hipGetLastError();
}

hipError_t launch_draft_gather(const DraftGatherArgs& a, hipStream_t stream) {
  const long long items = static_cast<long long>(a.num_cols) * a.geo.hkv;
  if (items == 0) return hipSuccess;
  const unsigned blocks = static_cast<unsigned>((items + kStepWaves - 1) / kStepWaves);
  hipLaunchKernelGGL(draft_gather_kernel, dim3(blocks), dim3(kStepThreads), 0, stream, a);
  return hipGetLastError();
}

}  // namespace fold
