// Fill kernels and FP64 wavefront-reduction l2 norms (power iterations, diagnostics).
// The sum of squares is deterministic: fixed-size per-workgroup partials, then one
// workgroup sums them in a fixed order.
#include "plan.hpp"

namespace ri {

namespace {

constexpr int RT = 256;
constexpr int RPART = SUMSQ_SCRATCH - 1;  // partial sums (first pass workgroups)

__global__ void k_zero_f32(float* __restrict__ p, size_t n) {
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    p[i] = 0.f;
}

// Copies of the solver state (ri_pd_get / ri_pd_set): 16-byte words, four in flight per thread.
// Bound by HBM (36 MiB in 14 us, 5.4 TB/s read and written).  hipMemcpyAsync between device
// buffers is as fast once it runs, but each call costs about 10 us more of the stream's time
// than a launch: four iterations at 64^2 and three such copies took 378 us, with this kernel 347.
template <class W>
__global__ __launch_bounds__(RT) void k_copy(const W* __restrict__ src, W* __restrict__ dst, size_t n) {
  const size_t stride = size_t(gridDim.x) * RT;
  size_t i = blockIdx.x * size_t(RT) + threadIdx.x;
  for (; i + 3 * stride < n; i += 4 * stride) {
    const W a = src[i], b = src[i + stride], c = src[i + 2 * stride], d = src[i + 3 * stride];
    dst[i] = a;
    dst[i + stride] = b;
    dst[i + 2 * stride] = c;
    dst[i + 3 * stride] = d;
  }
  for (; i < n; i += stride) dst[i] = src[i];
}

__global__ __launch_bounds__(RT) void k_sumsq_part(const float* __restrict__ x, size_t n, double* __restrict__ part) {
  __shared__ double red[RT / 64];
  double acc = 0.0;
  for (size_t i = blockIdx.x * size_t(RT) + threadIdx.x; i < n; i += size_t(gridDim.x) * RT) {
    const double v = x[i];
    acc += v * v;
  }
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < RT / 64; ++k) t += red[k];
    part[blockIdx.x] = t;
  }
}

__global__ __launch_bounds__(RT) void k_sum_parts(const double* __restrict__ part, int np, double* __restrict__ out) {
  __shared__ double red[RT / 64];
  double acc = 0.0;
  for (int i = threadIdx.x; i < np; i += RT) acc += part[i];
  acc = wave_sum(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x / 64] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double t = 0.0;
    for (int k = 0; k < RT / 64; ++k) t += red[k];
    *out = t;
  }
}

__global__ void k_scale_rsqrt(float* __restrict__ x, size_t n, const double* __restrict__ sq) {
  const double s = *sq;
  const float f = s > 0.0 ? float(1.0 / sqrt(s)) : 0.f;
  for (size_t i = blockIdx.x * size_t(blockDim.x) + threadIdx.x; i < n; i += size_t(gridDim.x) * blockDim.x)
    x[i] *= f;
}

unsigned blocks_for(size_t n) {
  const size_t b = (n + RT - 1) / RT;
  return unsigned(b < 4096 ? (b > 0 ? b : 1) : 4096);
}

}  // namespace

int zero_f32(float* p, size_t n, hipStream_t s) {
  if (n == 0) return RI_OK;
  hipLaunchKernelGGL(k_zero_f32, dim3(blocks_for(n)), dim3(RT), 0, s, p, n);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

// Device memory of the current GPU at a float's alignment, which k_copy can reach.
static bool kernel_can_copy(const void* p) {
  hipPointerAttribute_t a{};
  int dev = -1;
  if (hipPointerGetAttributes(&a, p) != hipSuccess || hipGetDevice(&dev) != hipSuccess) {
    (void)hipGetLastError();  // memory the runtime does not know
    return false;
  }
  return a.type == hipMemoryTypeDevice && a.device == dev && reinterpret_cast<uintptr_t>(p) % sizeof(float) == 0;
}

// A caller's buffer may be any memory hipMemcpyAsync takes: host memory (a kernel would fault on pages
// the GPU does not map), another GPU's, bytes without alignment.
int copy_user(void* dst, const void* src, size_t bytes, const void* user, hipStream_t s) {
  if (kernel_can_copy(user)) return copy_f32(static_cast<float*>(dst), static_cast<const float*>(src), bytes / 4, s);
  RI_HIP(hipMemcpyAsync(dst, src, bytes, hipMemcpyDefault, s));
  return RI_OK;
}

// Sixteen-byte words need both pointers and the length aligned to them; any other view of a
// caller's buffer is copied by single floats.
int copy_f32(float* dst, const float* src, size_t n, hipStream_t s) {
  if (n == 0) return RI_OK;
  const bool wide = (reinterpret_cast<uintptr_t>(dst) | reinterpret_cast<uintptr_t>(src) | (n * 4)) % 16 == 0;
  const size_t words = wide ? n / 4 : n, per = size_t(RT) * 4;
  const size_t g = (words + per - 1) / per;
  const dim3 grid(unsigned(g < 8192 ? g : 8192));
  if (wide)
    hipLaunchKernelGGL(k_copy<float4>, grid, dim3(RT), 0, s, reinterpret_cast<const float4*>(src),
                       reinterpret_cast<float4*>(dst), words);
  else
    hipLaunchKernelGGL(k_copy<float>, grid, dim3(RT), 0, s, src, dst, words);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

int zero_c64(float2* p, size_t n, hipStream_t s) { return zero_f32(reinterpret_cast<float*>(p), 2 * n, s); }

// out points at SUMSQ_SCRATCH doubles: the result goes to out[0], the partials to out[1..].
int sumsq_f32(const float* x, size_t n, double* out, hipStream_t s) {
  double* part = out + 1;
  hipLaunchKernelGGL(k_sumsq_part, dim3(RPART), dim3(RT), 0, s, x, n, part);
  RI_LAUNCH_CHECK();
  hipLaunchKernelGGL(k_sum_parts, dim3(1), dim3(RT), 0, s, part, RPART, out);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

int scale_by_rsqrt(float* x, size_t n, const double* sq, hipStream_t s) {
  hipLaunchKernelGGL(k_scale_rsqrt, dim3(blocks_for(n)), dim3(RT), 0, s, x, n, sq);
  RI_LAUNCH_CHECK();
  return RI_OK;
}

}  // namespace ri
