// 2D transforms of small grids in one kernel (included by fft.hip, after its
// twiddle tables): a workgroup holds two real slices as one complex grid in
// LDS and runs both axes there.
//
// What bounds the two-pass transforms on such grids is latency: a pass of a
// few MB lasts as long as its launch, its loads and its stores take one after
// the other (4 to 5 us), and the host needs as long to enqueue it.  One kernel
// pays that once.  It writes 16 bytes per spectrum row (two slices), so eight
// workgroups share a 128-byte line; they are placed on one XCD, whose L2 puts
// the pieces together.
//
// Each axis is the four-step split N = N1 * N2 of the two-pass kernels, in
// place: the thread of column t of the split reads and writes positions
// t + N2 n1, the thread of k1 positions n2 + N2 k1, so output k1 + N1 k2 ends
// at position N2 k1 + k2 and one barrier per stage is enough.  Rows of the
// grid are PX (odd) values apart and the threads of a wave take adjacent rows
// in the x stages and adjacent columns in the y stages: no bank conflicts.
// Four values per thread (up to 1,024 threads): with 512 threads an A + A^T
// pair at 48 x 48 x 48, 200 samples took 52 us, with 576 41 us (two passes 49).
#pragma once

namespace pat {

constexpr int small_threads(int nx, int ny) { return nx * ny >= 2048 ? nx * ny / 4 : 256; }

template <int NX, int NY>
struct SmallGrid {
  static constexpr int X1 = Split<NX>::N1, X2 = Split<NX>::N2;
  static constexpr int Y1 = Split<NY>::N1, Y2 = Split<NY>::N2;
  static constexpr int NT = small_threads(NX, NY);
  static_assert(NX * NY % NT == 0, "whole rounds of loads");
  // N2 positions per group of N2 + 1 along x, two more columns for c2r
  static constexpr int EXTRA = NX + X1;
  static constexpr int PX = (EXTRA + 2) | 1;
  static constexpr int LDS = NY * PX;
  static __device__ __forceinline__ int xin(int x) { return (x / X2) * (X2 + 1) + x % X2; }
  static __device__ __forceinline__ int xout(int m) { return (m % X1) * (X2 + 1) + m / X1; }
  static __device__ __forceinline__ int yout(int p) { return (p % Y1) * Y2 + p / Y1; }

  template <int DIR>
  static __device__ __forceinline__ void along_x(float2* z, const float2* tw, int tid) {
    for (int u = tid; u < NY * X2; u += NT) {
      const int t = u / NY;
      float2* p = z + (u % NY) * PX + t;
      float2 v[X1];
#pragma unroll
      for (int i = 0; i < X1; ++i) v[i] = p[(X2 + 1) * i];
      dft<X1, DIR>(v);
#pragma unroll
      for (int i = 0; i < X1; ++i) p[(X2 + 1) * i] = cmul(v[i], tw[t * i]);
    }
    __syncthreads();
    for (int u = tid; u < NY * X1; u += NT) {
      float2* p = z + (u % NY) * PX + (u / NY) * (X2 + 1);
      float2 v[X2];
#pragma unroll
      for (int i = 0; i < X2; ++i) v[i] = p[i];
      dft<X2, DIR>(v);
#pragma unroll
      for (int i = 0; i < X2; ++i) p[i] = v[i];
    }
    __syncthreads();
  }
  // first stage along y of ncol columns
  template <int DIR>
  static __device__ __forceinline__ void first_y(float2* z, const float2* tw, int tid, int ncol) {
    for (int u = tid; u < ncol * Y2; u += NT) {
      const int t = u / ncol, c = u % ncol;
      float2* p = z + t * PX + (c < NX ? xin(c) : EXTRA + c - NX);
      float2 v[Y1];
#pragma unroll
      for (int i = 0; i < Y1; ++i) v[i] = p[Y2 * PX * i];
      dft<Y1, DIR>(v);
#pragma unroll
      for (int i = 0; i < Y1; ++i) p[Y2 * PX * i] = cmul(v[i], tw[t * i]);
    }
    __syncthreads();
  }
};

// block -> pair of slices: eight neighbours (a line of 16 slices) per XCD
__device__ __forceinline__ int small_pair() {
  const int x = blockIdx.x & 7, l = blockIdx.x >> 3;
  return (l >> 3) * 64 + x * 8 + (l & 7);
}

// X[row(p * nh + m) * rs + s] of slices f[s][nyc][nxc] (zeros outside)
template <int NX, int NY>
__global__ __launch_bounds__(small_threads(NX, NY)) void k_fft_small_r2c(const float* __restrict__ f, float2* __restrict__ X,
                                                       int nyc, int nxc, int S, int rs,
                                                       const int32_t* __restrict__ rowmap) {
  using G = SmallGrid<NX, NY>;
  constexpr int NH = NX / 2 + 1;
  __shared__ float2 z[G::LDS], twx[NX], twy[NY];
  const int tid = threadIdx.x, s0 = 2 * small_pair();
  if (s0 >= S) return;
  const bool two = s0 + 1 < S;
  const float* fa = f + (size_t)s0 * nyc * nxc;
  const float* fb = fa + (size_t)nyc * nxc;
  constexpr int IT = NX * NY / G::NT;
  float2 ld[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int u = tid + i * G::NT, y = u / NX, x = u % NX;
    const bool in = y < nyc && x < nxc;
    ld[i] = make_float2(in ? fa[y * nxc + x] : 0.f, in && two ? fb[y * nxc + x] : 0.f);
  }
  // spectrum rows of this thread's results: read here, the stores wait for nothing
  constexpr int OT = (NY * NH + G::NT - 1) / G::NT;
  int rows[OT];
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    const int u = tid + i * G::NT;
    rows[i] = u >= NY * NH ? -1 : rowmap ? rowmap[u] : u;
  }
  for (int e = tid; e < NX; e += G::NT) twx[e] = g_tw[tw_offset(NX) + e];
  for (int e = tid; e < NY; e += G::NT) twy[e] = g_tw[tw_offset(NY) + e];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int u = tid + i * G::NT;
    z[(u / NX) * G::PX + G::xin(u % NX)] = ld[i];
  }
  __syncthreads();
  G::template along_x<-1>(z, twx, tid);
  // positions of x hold frequencies in another order: each is a column all the same
  G::template first_y<-1>(z, twy, tid, NX);
  for (int u = tid; u < NX * G::Y1; u += G::NT) {
    float2* p = z + (u / NX) * G::Y2 * G::PX + G::xin(u % NX);
    float2 v[G::Y2];
#pragma unroll
    for (int i = 0; i < G::Y2; ++i) v[i] = p[i * G::PX];
    dft<G::Y2, -1>(v);
#pragma unroll
    for (int i = 0; i < G::Y2; ++i) p[i * G::PX] = v[i];
  }
  __syncthreads();
  // separate the two slices' half spectra
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    if (rows[i] < 0) continue;
    const int u = tid + i * G::NT, p = u / NH, m = u % NH;
    const float2 a = z[G::yout(p) * G::PX + G::xout(m)];
    const float2 b = z[G::yout(p ? NY - p : 0) * G::PX + G::xout(m ? NX - m : 0)];
    float2* dst = X + (size_t)rows[i] * rs + s0;
    const float4 r = make_float4(0.5f * (a.x + b.x), 0.5f * (a.y - b.y), 0.5f * (a.y + b.y), 0.5f * (b.x - a.x));
    if (two)
      *reinterpret_cast<float4*>(dst) = r;
    else
      *dst = make_float2(r.x, r.y);
  }
}

// f[s][y][x] = scale * inverse transform - sub, the window nyc x nxc of it;
// imaginary parts of m = 0 and NX / 2 are dropped after the y axis
template <int NX, int NY>
__global__ __launch_bounds__(small_threads(NX, NY)) void k_fft_small_c2r(const float2* __restrict__ X, float* __restrict__ f,
                                                       int nyc, int nxc, int S, int rs, float scale,
                                                       const float* __restrict__ sub,
                                                       const int32_t* __restrict__ rowmap) {
  using G = SmallGrid<NX, NY>;
  constexpr int NH = NX / 2 + 1;
  __shared__ float2 z[G::LDS], twx[NX], twy[NY];
  const int tid = threadIdx.x, s0 = 2 * small_pair();
  if (s0 >= S) return;
  const bool two = s0 + 1 < S;
  // column m of slice s0 at position m, of slice s0 + 1 at NX - m (or extra)
  auto col_b = [](int m) { return m == 0 ? G::EXTRA : m == NX / 2 ? G::EXTRA + 1 : G::xin(NX - m); };
  constexpr int IT = (NY * NH + G::NT - 1) / G::NT;
  float4 ld[IT];
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int u = min(tid + i * G::NT, NY * NH - 1);
    const int row = rowmap ? rowmap[u] : u;
    ld[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (row >= 0) {  // rows are padded to even lengths: the pair is there, its second half may be no slice
      ld[i] = *reinterpret_cast<const float4*>(X + (size_t)row * rs + s0);
      if (!two) ld[i].z = ld[i].w = 0.f;
    }
  }
  for (int e = tid; e < NX; e += G::NT) twx[e] = cconj(g_tw[tw_offset(NX) + e]);
  for (int e = tid; e < NY; e += G::NT) twy[e] = cconj(g_tw[tw_offset(NY) + e]);
#pragma unroll
  for (int i = 0; i < IT; ++i) {
    const int u = tid + i * G::NT;
    if (u >= NY * NH) break;
    float2* zr = z + (u / NH) * G::PX;
    zr[G::xin(u % NH)] = make_float2(ld[i].x, ld[i].y);
    zr[col_b(u % NH)] = make_float2(ld[i].z, ld[i].w);
  }
  __syncthreads();
  G::template first_y<+1>(z, twy, tid, NX + 2);
  // second stage of both slices' columns, packed into rows of A + i B
  for (int u = tid; u < NH * G::Y1; u += G::NT) {
    const int m = u % NH;
    float2* pr = z + (u / NH) * G::Y2 * G::PX;
    float2* pa = pr + G::xin(m);
    float2* pb = pr + col_b(m);
    float2 a[G::Y2], b[G::Y2];
#pragma unroll
    for (int i = 0; i < G::Y2; ++i) {
      a[i] = pa[i * G::PX];
      b[i] = pb[i * G::PX];
    }
    dft<G::Y2, +1>(a);
    dft<G::Y2, +1>(b);
    const bool self = m == 0 || m == NX / 2;
#pragma unroll
    for (int i = 0; i < G::Y2; ++i) {
      pa[i * G::PX] = self ? make_float2(a[i].x, b[i].x) : make_float2(a[i].x - b[i].y, a[i].y + b[i].x);
      if (!self) pb[i * G::PX] = make_float2(a[i].x + b[i].y, b[i].x - a[i].y);
    }
  }
  __syncthreads();
  G::template along_x<+1>(z, twx, tid);
  float* fa = f + (size_t)s0 * nyc * nxc;
  const size_t next = (size_t)nyc * nxc;
  constexpr int OT = NX * NY / G::NT;
#pragma unroll
  for (int i = 0; i < OT; ++i) {
    const int u = tid + i * G::NT, y = u / NX, x = u % NX;
    if (y >= nyc || x >= nxc) continue;
    const float2 v = z[G::yout(y) * G::PX + G::xout(x)];
    const size_t o = (size_t)y * nxc + x, g = (size_t)s0 * next + o;
    fa[o] = v.x * scale - (sub ? sub[g] : 0.f);
    if (two) fa[next + o] = v.y * scale - (sub ? sub[g + next] : 0.f);
  }
}

}  // namespace pat
