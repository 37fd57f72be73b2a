// Element-wise and reduction kernels around the operator: buffer clearing,
// float64 dot products (traces and the adjoint check), the float32 products
// and normalisation of the power iteration, and the fused FISTA update
// (proximal step of Sec. 2.3 plus the momentum extrapolation).
#include "pat_internal.hpp"

namespace pat {

__global__ void k_fill_zero(uint4* p, size_t n16, unsigned char* tail, size_t ntail) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride)
    p[i] = make_uint4(0, 0, 0, 0);
  if (blockIdx.x == 0 && threadIdx.x < ntail) tail[threadIdx.x] = 0;
}

pat_status fill_zero(void* p, size_t bytes, hipStream_t st) {
  if (bytes == 0) return PAT_OK;
  const size_t n16 = bytes / 16;
  int blocks = (int)((n16 + 255) / 256);
  if (blocks > 4096) blocks = 4096;
  if (blocks < 1) blocks = 1;
  k_fill_zero<<<blocks, 256, 0, st>>>(reinterpret_cast<uint4*>(p), n16,
                                      reinterpret_cast<unsigned char*>(p) + n16 * 16, bytes % 16);
  PAT_LAUNCHED("fill");
  return PAT_OK;
}

__device__ __forceinline__ double block_sum(double v, double* sh) {
  sh[threadIdx.x] = v;
  __syncthreads();
  for (int s = blockDim.x / 2; s > 0; s >>= 1) {
    if ((int)threadIdx.x < s) sh[threadIdx.x] += sh[threadIdx.x + s];
    __syncthreads();
  }
  return sh[0];
}

__global__ __launch_bounds__(256) void k_dot_part(const float* __restrict__ a,
                                                  const float* __restrict__ b, long long n,
                                                  double* __restrict__ part) {
  __shared__ double sh[256];
  double s = 0;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += stride)
    s += (double)a[i] * (double)b[i];
  const double tot = block_sum(s, sh);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_dot_final(const double* __restrict__ part, int np,
                                                   double* __restrict__ result) {
  __shared__ double sh[256];
  double s = 0;
  for (int i = threadIdx.x; i < np; i += blockDim.x) s += part[i];
  const double tot = block_sum(s, sh);
  if (threadIdx.x == 0) result[0] = tot;
}

pat_status dot_f64(const float* a, const float* b, long long n, double* part, double* result,
                   hipStream_t st) {
  k_dot_part<<<kRedBlocks, 256, 0, st>>>(a, b, n, part);
  PAT_LAUNCHED("dot64 partials");
  k_dot_final<<<1, 256, 0, st>>>(part, kRedBlocks, result);
  PAT_LAUNCHED("dot64 final");
  return PAT_OK;
}

// Power iteration: <a, b> and <b, b> in one pass, then b / sqrt(<b, b>).  Both
// passes are launch and memory bound (n floats read twice, then read and
// written once), so they are two kernels instead of two dot products of two
// kernels each and a scaling: partial sums of both products per block here,
// and every block of k_power_scale adds the kRedBlocks partials itself
// (4 KB from the cache) rather than wait for a kernel that does.  16-byte
// accesses; 4 running sums per product and thread, then trees: float32
// throughout.  128x128x96, a device trace: 4.2 + 4.3 us per
// iteration (20.0 us in five kernels before); 30 iterations 1.86 -> 1.48 ms.
__device__ __forceinline__ float2 block_sum2(float2 v, float2* sh) {
#pragma unroll
  for (int m = 32; m > 0; m >>= 1) {
    v.x += __shfl_xor(v.x, m);
    v.y += __shfl_xor(v.y, m);
  }
  if ((threadIdx.x & 63) == 0) sh[threadIdx.x >> 6] = v;
  __syncthreads();
  const float2 p = sh[0], q = sh[1], r = sh[2], t = sh[3];
  return make_float2((p.x + q.x) + (r.x + t.x), (p.y + q.y) + (r.y + t.y));
}

__global__ __launch_bounds__(256) void k_power_dots(const float* a, const float* b, long long n,
                                                    float2* __restrict__ part) {
  __shared__ float2 sh[4];
  const float4* a4 = reinterpret_cast<const float4*>(a);
  const float4* b4 = reinterpret_cast<const float4*>(b);
  const long long n4 = n >> 2, stride = (long long)gridDim.x * blockDim.x;
  const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  float4 ab = make_float4(0, 0, 0, 0), bb = ab;
#pragma unroll 4
  for (long long i = i0; i < n4; i += stride) {
    const float4 u = a4[i], v = b4[i];
    ab.x += u.x * v.x; ab.y += u.y * v.y; ab.z += u.z * v.z; ab.w += u.w * v.w;
    bb.x += v.x * v.x; bb.y += v.y * v.y; bb.z += v.z * v.z; bb.w += v.w * v.w;
  }
  if (i0 < (n & 3)) {  // the last n % 4 values
    const float u = a[4 * n4 + i0], v = b[4 * n4 + i0];
    ab.x += u * v;
    bb.x += v * v;
  }
  const float2 tot = block_sum2(
      make_float2((ab.x + ab.y) + (ab.z + ab.w), (bb.x + bb.y) + (bb.z + bb.w)), sh);
  if (threadIdx.x == 0) part[blockIdx.x] = tot;
}

__global__ __launch_bounds__(256) void k_power_scale(float* __restrict__ dst,
                                                     const float* __restrict__ src, long long n,
                                                     const float2* __restrict__ part,
                                                     float* __restrict__ ab) {
  static_assert(kRedBlocks == 512, "two partials per thread");
  __shared__ float2 sh[4];
  const float2 p = part[threadIdx.x], q = part[threadIdx.x + 256];
  const float2 tot = block_sum2(make_float2(p.x + q.x, p.y + q.y), sh);
  const float s = 1.0f / sqrtf(tot.y);
  const float4* s4 = reinterpret_cast<const float4*>(src);
  float4* d4 = reinterpret_cast<float4*>(dst);
  const long long n4 = n >> 2, stride = (long long)gridDim.x * blockDim.x;
  const long long i0 = (long long)blockIdx.x * blockDim.x + threadIdx.x;
  for (long long i = i0; i < n4; i += stride) {
    const float4 v = s4[i];
    d4[i] = make_float4(v.x * s, v.y * s, v.z * s, v.w * s);
  }
  if (i0 < (n & 3)) dst[4 * n4 + i0] = src[4 * n4 + i0] * s;
  if (i0 == 0 && ab) ab[0] = tot.x;
}

pat_status power_normalise(float* dst, const float* v, const float* u, long long n, float2* part,
                           float* vu, hipStream_t st) {
  k_power_dots<<<kRedBlocks, 256, 0, st>>>(v, u, n, part);
  PAT_LAUNCHED("power iteration dots");
  long long blocks = (n / 4 + 255) / 256;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  k_power_scale<<<(int)blocks, 256, 0, st>>>(dst, u, n, part, vu);
  PAT_LAUNCHED("power iteration normalise");
  return PAT_OK;
}

__global__ void k_trace_combine(float* out, const double* s) {
  out[0] = (float)(0.5 * (s[0] - s[1] + s[2]));
}

pat_status trace_combine(float* out, const double* s, hipStream_t st) {
  k_trace_combine<<<1, 1, 0, st>>>(out, s);
  PAT_LAUNCHED("trace");
  return PAT_OK;
}

// x_old = x; v = z - tau g; x = prox(v); z = x + beta (x - x_old)
__global__ __launch_bounds__(256) void k_fista_update(float* __restrict__ x, float* __restrict__ z,
                                                      const float* __restrict__ g,
                                                      long long n_per_obj, FistaBatch p,
                                                      int32_t* __restrict__ nonfinite) {
  const int b = blockIdx.y;
  const FistaObj o = p.o[b];
  float* xb = x + (size_t)b * n_per_obj;
  float* zb = z + (size_t)b * n_per_obj;
  const float* gb = g + (size_t)b * n_per_obj;
  bool bad = false;
  const long long stride = (long long)gridDim.x * blockDim.x;
  for (long long i = (long long)blockIdx.x * blockDim.x + threadIdx.x; i < n_per_obj; i += stride) {
    const float xo = xb[i];
    const float v = zb[i] - o.tau * gb[i];
    float xn;
    if (o.nonneg) {
      xn = fmaxf(v - o.thr, 0.f);
    } else {
      const float m = fmaxf(fabsf(v) - o.thr, 0.f);
      xn = copysignf(m, v);
    }
    bad |= !isfinite(xn);
    xb[i] = xn;
    zb[i] = xn + o.beta * (xn - xo);
  }
  if (bad && nonfinite) nonfinite[b] = 1;
}

pat_status fista_update(float* x, float* z, const float* g, long long n_per_obj, int B,
                        const FistaBatch& p, int32_t* nonfinite, hipStream_t st) {
  long long blocks = (n_per_obj + 1023) / 1024;
  if (blocks > 2048) blocks = 2048;
  if (blocks < 1) blocks = 1;
  dim3 grid((unsigned)blocks, B);
  k_fista_update<<<grid, 256, 0, st>>>(x, z, g, n_per_obj, p, nonfinite);
  PAT_LAUNCHED("fista update");
  return PAT_OK;
}

}  // namespace pat
