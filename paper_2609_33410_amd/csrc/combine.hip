// Additive combine for gfx950 (Algorithm 1, last step; Section 4; the range
// certificate of Section 3).
//
// Four channels a lane, D / 4 lanes a query row, one wave a workgroup.  A lane
// adds the slots' A in increasing slot order; every lane forms its row's L sum
// in the same order.  o = A / L with no maximum and no rescale.  Optional outputs: the
// base-2 log-sum-exp Z + log2 L and the certificate bits.  With the cut-key
// value model (Section 4, depth paragraph) the slots' cut masses, summed in
// slot order, multiply the request's mean value row and join A: a virtual row
// standing in for every cut key.
//
// Latency bounds it, not its bytes (512 rows of 32 slots: 8 MB): up to sixteen
// slots' loads and what the last lines need are in flight together, a short
// remainder too, and the certificate's vote is a ballot, no barrier.  Against
// a thread per channel in batches of eight (combine_kernel below): 512 rows x
// 32 slots 4.7 -> 4.0 us, 4096 x 5 5.3 -> 5.1, 1024 x 8 4.7 -> 4.6, 4 x 1
// 2.2 -> 1.9, all at D = 128 but the last (64).  Workgroups of 128 or 256
// threads: 4.2 and 4.3 us for the first, the others alike.
#include "fold_device.h"
#include "fold_internal.h"

namespace fold {
namespace {

constexpr int kCombineThreads = 64;

// For arrays without the 16-byte alignment of the kernel below: one workgroup
// of head_dim threads per row, one channel each.
__global__ __launch_bounds__(128) void combine_kernel(const CombineArgs a) {
  const int row = blockIdx.x;
  const int d = threadIdx.x;
  const int D = a.head_dim;
  float acc = 0.0f;
  float l = 0.0f;
  // Slots are added in increasing order; loads are batched eight at a time so
  // they are in flight together.
  int s = 0;
  for (; s + 8 <= a.num_slots; s += 8) {
    float av[8], lv[8];
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      const size_t sr = static_cast<size_t>(s + u) * a.num_rows + row;
      av[u] = a.part_A[sr * D + d];
      lv[u] = a.part_L[sr];
    }
#pragma unroll
    for (int u = 0; u < 8; ++u) {
      acc += av[u];
      l += lv[u];
    }
  }
  for (; s < a.num_slots; ++s) {
    const size_t sr = static_cast<size_t>(s) * a.num_rows + row;
    acc += a.part_A[sr * D + d];
    l += a.part_L[sr];
  }
  if (a.part_Lcut) {
    float c = 0.0f;
    for (int t = 0; t < a.num_slots; ++t) c += a.part_Lcut[static_cast<size_t>(t) * a.num_rows + row];
    const int req = row / a.heads;
    const int kvh = (row - req * a.heads) / (a.heads / a.hkv);
    acc = __builtin_fmaf(c, a.mean[(static_cast<size_t>(req) * a.hkv + kvh) * D + d], acc);
  }
  const float o = acc / l;
  const size_t oi = static_cast<size_t>(row) * D + d;
  if (a.out_bf16)
    static_cast<uint16_t*>(a.out)[oi] = f32_to_bf16_rne(o);
  else
    static_cast<float*>(a.out)[oi] = o;
  const int bad = __syncthreads_or(!isfinite(o) ? 1 : 0);
  if (d == 0) {
    if (a.lse_out) a.lse_out[row] = a.z[row] + log2f(l);
    if (a.cert_out) {
      uint8_t c = 0;
      if (l < 0.5f) c |= 1;
      if (l > 0x1p100f) c |= 2;
      if (bad) c |= 4;
      a.cert_out[row] = c;
    }
  }
}

// U slots of a lane's four channels and of its row's L (and cut mass): every
// load is issued before the first add, which run in slot order; a slot past
// the last repeats the last one's address and is left out.
template <int D, int U, bool CUT>
__device__ __forceinline__ void add_slots(const CombineArgs& a, int row, int d, int s0, f32x4& acc,
                                          float& l, float& c) {
  f32x4 v[U];
  float lv[U], cv[U];
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const size_t sr = static_cast<size_t>(min(s0 + u, a.num_slots - 1)) * a.num_rows + row;
    v[u] = *reinterpret_cast<const f32x4*>(a.part_A + sr * D + d);
    lv[u] = a.part_L[sr];
    cv[u] = CUT ? a.part_Lcut[sr] : 0.0f;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const bool in = s0 + u < a.num_slots;  // uniform
    acc = in ? acc + v[u] : acc;
    l = in ? l + lv[u] : l;
    if (CUT) c = in ? c + cv[u] : c;
  }
}

template <int D, bool CUT>
__global__ __launch_bounds__(kCombineThreads) void combine_wide_kernel(const CombineArgs a) {
  constexpr int kLanes = D / 4;  // lanes of a row
  const long long row0 =
      static_cast<long long>(blockIdx.x) * (blockDim.x / kLanes) + threadIdx.x / kLanes;
  const bool have = row0 < a.num_rows;
  const int row = have ? static_cast<int>(row0) : a.num_rows - 1;
  const int d = 4 * (threadIdx.x % kLanes);
  const float z = a.lse_out ? a.z[row] : 0.0f;
  f32x4 mean = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (CUT) {
    const int req = row / a.heads;
    const int kvh = (row - req * a.heads) / (a.heads / a.hkv);
    mean = *reinterpret_cast<const f32x4*>(a.mean + (static_cast<size_t>(req) * a.hkv + kvh) * D + d);
  }
  f32x4 acc = {0.0f, 0.0f, 0.0f, 0.0f};
  float l = 0.0f, c = 0.0f;
  for (int s = 0; s < a.num_slots; s += 16) {
    const int k = a.num_slots - s;
    if (k > 8) add_slots<D, 16, CUT>(a, row, d, s, acc, l, c);
    else if (k > 4) add_slots<D, 8, CUT>(a, row, d, s, acc, l, c);
    else add_slots<D, 4, CUT>(a, row, d, s, acc, l, c);
  }
  float o[4];
  bool nf = false;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float v = CUT ? __builtin_fmaf(c, mean[i], acc[i]) : acc[i];
    o[i] = v / l;
    nf = nf || !isfinite(o[i]);
  }
  const uint64_t bad = __ballot(nf);
  if (!have) return;
  const size_t oi = static_cast<size_t>(row) * D + d;
  if (a.out_bf16) {
    const u32x2 ob = {f32_to_bf16_rne(o[0]) | (static_cast<uint32_t>(f32_to_bf16_rne(o[1])) << 16),
                      f32_to_bf16_rne(o[2]) | (static_cast<uint32_t>(f32_to_bf16_rne(o[3])) << 16)};
    *reinterpret_cast<u32x2*>(static_cast<uint16_t*>(a.out) + oi) = ob;
  } else {
    *reinterpret_cast<f32x4*>(static_cast<float*>(a.out) + oi) = f32x4{o[0], o[1], o[2], o[3]};
  }
  if (d == 0) {
    if (a.lse_out) a.lse_out[row] = z + log2f(l);
    if (a.cert_out) {
      const int base = (threadIdx.x & 63) / kLanes * kLanes;
      uint8_t b = 0;
      if (l < 0.5f) b |= 1;
      if (l > 0x1p100f) b |= 2;
      if ((bad >> base) & ((1ull << kLanes) - 1)) b |= 4;
      a.cert_out[row] = b;
    }
  }
}

template <int D>
void launch_wide(const CombineArgs& a, hipStream_t stream) {
  const long long lanes = static_cast<long long>(a.num_rows) * (D / 4);
  const int threads = kCombineThreads;
  const unsigned blocks = static_cast<unsigned>((lanes + threads - 1) / threads);
  if (a.part_Lcut)
    hipLaunchKernelGGL((combine_wide_kernel<D, true>), dim3(blocks), dim3(threads), 0, stream, a);
  else
    hipLaunchKernelGGL((combine_wide_kernel<D, false>), dim3(blocks), dim3(threads), 0, stream, a);
}

}  // namespace

hipError_t launch_combine(const CombineArgs& a, hipStream_t stream) {
  if (a.num_rows == 0) return hipSuccess;
  // 16-byte lines of the slots, means and output (a bf16 output needs 8); rows
  // start at multiples of D elements, so the bases decide.
  auto aligned = [](const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15) == 0; };
  if (aligned(a.part_A) && aligned(a.mean) && aligned(a.out)) {
    if (a.head_dim == 128) launch_wide<128>(a, stream);
    else launch_wide<64>(a, stream);
    return hipGetLastError();
  }
  hipLaunchKernelGGL(combine_kernel, dim3(a.num_rows), dim3(a.head_dim), 0, stream, a);
  return hipGetLastError();
}

}  // namespace fold
