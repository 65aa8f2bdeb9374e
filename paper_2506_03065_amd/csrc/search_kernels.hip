// gfx950 kernels of the offline search step (Section 4.2, Eq. 2, Algorithm 1).
// Both are streaming kernels bound by HBM: the reduction reads two tensors
// once, the selection reads one and writes one.
#include <hip/hip_runtime.h>

#include "search_kernels.h"

namespace svd {
namespace {

typedef unsigned u32x4 __attribute__((ext_vector_type(4)));

constexpr int kMseThreads = 256;
constexpr int kMseChunkBytes = 1 << 18;   // of one tensor, per work-group

__device__ __forceinline__ float bf16_lo(unsigned w) { return __builtin_bit_cast(float, w << 16); }
__device__ __forceinline__ float bf16_hi(unsigned w) { return __builtin_bit_cast(float, w & 0xffff0000u); }

template <int N>
struct MseSources {
  const __bf16* a[N];   // nullptr: zeros
};

// Pass 1: work-group (chunk, b * H + h) sums (a - ref)^2 over its share of the
// head's L * D elements, 16 bytes per thread, tensor and step.  N = 4: the modes of the
// search step against the dense output, which is read once for all of them, the zeros of skipped heads not at all
// (with the lists copied ahead, 24 heads x 11,880, D = 64: the step 1,725 -> 1,670 us).
template <int N>
__global__ void __launch_bounds__(kMseThreads) head_mse_partial_kernel(const MseSources<N> src,
                                                                       const __bf16* __restrict__ ref,
                                                                       const TensorView t, const int n_chunks,
                                                                       float* __restrict__ partial) {
  const int bh = blockIdx.y, b = bh / t.H, h = bh % t.H;
  const int64_t base = (int64_t)b * t.stride_b + (int64_t)h * t.stride_h;
  const int cpr = t.D / 8;                                  // 16-byte pieces per row
  const int64_t total = (int64_t)t.L * cpr;
  const int64_t per = (total + n_chunks - 1) / n_chunks;
  const int64_t g0 = (int64_t)blockIdx.x * per;
  const int64_t g1 = g0 + per < total ? g0 + per : total;
  float acc[N];
#pragma unroll
  for (int m = 0; m < N; ++m) acc[m] = 0.f;
  struct Piece {
    u32x4 x[N], y;
  };
  auto piece = [&](const int64_t g) {
    Piece p;
    const int64_t off = base + (g / cpr) * t.stride_l + (g % cpr) * 8;
    p.y = *reinterpret_cast<const u32x4*>(ref + off);
#pragma unroll
    for (int m = 0; m < N; ++m) {
      p.x[m] = u32x4{0u, 0u, 0u, 0u};
      if (src.a[m]) p.x[m] = *reinterpret_cast<const u32x4*>(src.a[m] + off);
    }
    return p;
  };
  auto add = [&](const Piece& p) {
#pragma unroll
    for (int m = 0; m < N; ++m)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const float d0 = bf16_lo(p.x[m][i]) - bf16_lo(p.y[i]), d1 = bf16_hi(p.x[m][i]) - bf16_hi(p.y[i]);
        acc[m] = __builtin_fmaf(d0, d0, acc[m]);
        acc[m] = __builtin_fmaf(d1, d1, acc[m]);
      }
  };
  constexpr int U = N == 1 ? 4 : 2;   // eight to ten loads in flight per thread
  int64_t g = g0 + threadIdx.x;
  for (; g + (U - 1) * kMseThreads < g1; g += U * kMseThreads) {
    Piece p[U];
#pragma unroll
    for (int u = 0; u < U; ++u) p[u] = piece(g + u * kMseThreads);
#pragma unroll
    for (int u = 0; u < U; ++u) add(p[u]);
  }
  for (; g < g1; g += kMseThreads) add(piece(g));
  // wave reduction, then the four waves through LDS, always in the same order
  __shared__ float wave_sum[N][kMseThreads / 64];
#pragma unroll
  for (int m = 0; m < N; ++m) {
#pragma unroll
    for (int s = 32; s > 0; s >>= 1) acc[m] += __shfl_down(acc[m], s, 64);
    if ((threadIdx.x & 63) == 0) wave_sum[m][threadIdx.x >> 6] = acc[m];
  }
  __syncthreads();
  if (threadIdx.x < N) {
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kMseThreads / 64; ++w) s += wave_sum[threadIdx.x][w];
    partial[((int64_t)threadIdx.x * gridDim.y + bh) * n_chunks + blockIdx.x] = s;
  }
}

// Pass 2: one thread per (tensor, head) adds the partial sums of all batch entries and
// chunks in double, in index order.
__global__ void head_mse_final_kernel(const float* __restrict__ partial, const TensorView t, const int n_chunks,
                                      const int n_tensors, float* __restrict__ mse) {
  const int i = blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= t.H * n_tensors) return;
  const int h = i % t.H, m = i / t.H;
  double s = 0.0;
  for (int b = 0; b < t.B; ++b)
    for (int c = 0; c < n_chunks; ++c) s += (double)partial[(((int64_t)m * t.B + b) * t.H + h) * n_chunks + c];
  mse[i] = (float)(s / ((double)t.B * t.L * t.D));
}

template <int N>
hipError_t launch_mse(const MseSources<N>& src, const __bf16* ref, const TensorView& t, float* mse, float* scratch,
                      hipStream_t stream) {
  const int n_chunks = mse_chunks(t);
  hipLaunchKernelGGL(head_mse_partial_kernel<N>, dim3(n_chunks, t.B * t.H), dim3(kMseThreads), 0, stream, src, ref, t,
                     n_chunks, scratch);
  if (hipError_t e = hipGetLastError(); e != hipSuccess) return e;
  hipLaunchKernelGGL(head_mse_final_kernel, dim3((t.H * N + 63) / 64), dim3(64), 0, stream, scratch, t, n_chunks, N, mse);
  return hipGetLastError();
}

struct SelectArgs {
  const __bf16* src[5];
  unsigned char mode[kMaxSelectHeads];
};

// out[:, h] = src[mode[h]][:, h], 16 bytes per thread and step.
__global__ void __launch_bounds__(256) select_heads_kernel(const SelectArgs args, const TensorView sv,
                                                           __bf16* __restrict__ out, const TensorView ov) {
  const int bh = blockIdx.y, b = bh / sv.H, h = bh % sv.H;
  const __bf16* __restrict__ src = args.src[args.mode[h]] + (int64_t)b * sv.stride_b + (int64_t)h * sv.stride_h;
  __bf16* __restrict__ dst = out + (int64_t)b * ov.stride_b + (int64_t)h * ov.stride_h;
  const int cpr = sv.D / 8;
  const int64_t total = (int64_t)sv.L * cpr;
  for (int64_t g = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; g < total; g += (int64_t)gridDim.x * blockDim.x) {
    const int64_t row = g / cpr;
    const int c = (int)(g % cpr) * 8;
    *reinterpret_cast<u32x4*>(dst + row * ov.stride_l + c) = *reinterpret_cast<const u32x4*>(src + row * sv.stride_l + c);
  }
}

}  // namespace

int mse_chunks(const TensorView& t) {
  const int64_t bytes = (int64_t)t.L * t.D * 2;
  const int64_t n = (bytes + kMseChunkBytes - 1) / kMseChunkBytes;
  return (int)(n < 1 ? 1 : n);
}

size_t mse_scratch_floats(const TensorView& t) { return (size_t)t.B * t.H * mse_chunks(t); }

hipError_t launch_head_mse(const __bf16* a, const __bf16* ref, const TensorView& t, float* mse, float* scratch,
                           hipStream_t stream) {
  return launch_mse<1>(MseSources<1>{{a}}, ref, t, mse, scratch, stream);
}

hipError_t launch_head_mse4(const __bf16* const a[4], const __bf16* ref, const TensorView& t, float* mse, float* scratch,
                            hipStream_t stream) {
  return launch_mse<4>(MseSources<4>{{a[0], a[1], a[2], a[3]}}, ref, t, mse, scratch, stream);
}

hipError_t launch_select_heads(const __bf16* const src[5], const TensorView& src_view, const int32_t* mode_of_head,
                               __bf16* out, const TensorView& out_view, hipStream_t stream) {
  if (src_view.H > kMaxSelectHeads) return hipErrorInvalidValue;
  SelectArgs args{};
  for (int m = 0; m < 5; ++m) args.src[m] = src[m];
  for (int h = 0; h < src_view.H; ++h) args.mode[h] = (unsigned char)mode_of_head[h];
  const int64_t total = (int64_t)src_view.L * (src_view.D / 8);
  int bx = (int)((total + 255) / 256);
  if (bx > 1024) bx = 1024;
  hipLaunchKernelGGL(select_heads_kernel, dim3(bx, src_view.B * src_view.H), dim3(256), 0, stream, args, src_view, out,
                     out_view);
  return hipGetLastError();
}

}  // namespace svd
