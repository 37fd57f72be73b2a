// Transverse transforms along an axis whose length N is not a fast FFT size
// (even, 16 .. 512; the 202 and 326 points of the experimental grids): dense
// DFTs on the float32 matrix instruction v_mfma_f32_16x16x4_f32.
//
// With K = N/2 + 1, even and odd parts e_n = x_n + x_{N-n}, o_n = x_n - x_{N-n}
// turn the N x N complex matrix into two real K x K ones,
//     sum_n x_n exp(-+ 2 pi i k n / N) = C_k -+ i S_k,   C = cos . e,  S = sin . o,
// and the output at N - k is the other sign.  The columns of the product are
// 16 slices (the layout's fastest index); the cosines and sines come from one
// table of the N-th roots in LDS, indexed k n mod N by a running sum, each read
// serving four products.  Sums of 32 terms are kept apart before they join the
// total (the instruction adds its products one after the other).
//
// N^2 work, but at the matrix rate it costs less than the chirp-z transforms
// (Bluestein: two FFTs of at least 2N - 1 points through LDS) that it
// replaced, at any length here.  256 slices of 202 x 202, row passes 81 and
// 97 us, now 44 and 51; column passes 60, now 47.  One A + one A^T: 202 x 202
// x 37 x 256, 439 us, now 311; 326 x 326 x 20 x 100, 719, now 473; 510 x 510 x
// 8 x 64 (the worst of lengths just below a power of two), 764, now 727.
// A workgroup loads, multiplies and stores in turn: with the matrix work (17
// us of a 202-point pass) and the bytes (17 us at the copy rate) overlapping
// only across workgroups.
#include "pat_internal.hpp"

namespace pat {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v4f4 __attribute__((ext_vector_type(4), aligned(4)));

constexpr int kDS = 16;      // slices per block
constexpr int kES = 33;      // LDS row stride of the row pass's folded rows (2 x 16 columns)
constexpr int kFlush = 8;    // steps of 4 terms between additions to the total

__host__ __device__ __forceinline__ int dense_k4(int N) { return (N / 2 + 4) & ~3; }  // N/2 + 1 up to whole steps

// four products per step and tile, cos with x0, x2 and sin with x1, x3, over
// all K4 / 4 steps: acc[u][0..3] of output tiles mt .. mt + NT - 1 (rows 16 mt
// ..).  Two tiles share the operand reads: LDS (table reads hit few of the
// same banks together) is otherwise as busy as the matrix cores.
template <int NT, typename Load>
__device__ __forceinline__ void dense_tiles(const float2* tab, int N, int K4, int mt, int lane, Load load,
                                            v4f (&acc)[NT][4]) {
  constexpr int RUN = NT == 1 ? kFlush : kFlush / 2;  // steps whose reads are in flight together
  const int k0 = lane >> 4;
  int idx[NT], stp[NT];
  v4f part[NT][4];
#pragma unroll
  for (int u = 0; u < NT; ++u) {
    const int m = 16 * (mt + u) + (lane & 15);
    idx[u] = m * k0 % N;
    stp[u] = 4 * m % N;
#pragma unroll
    for (int i = 0; i < 4; ++i) acc[u][i] = v4f(0.f);
  }
  for (int k = 0; k < K4; k += 4 * kFlush) {
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) part[u][i] = v4f(0.f);
#pragma unroll
    for (int h = 0; h < kFlush; h += RUN) {
      const int n = min(RUN, ((K4 - k) >> 2) - h);
      auto steps = [&](int cnt) {
        // table and operand reads of all steps go out before the first product
        float2 t[RUN][NT];
        float x[RUN][4];
#pragma unroll
        for (int q = 0; q < RUN; ++q) {
          if (q >= cnt) break;
#pragma unroll
          for (int u = 0; u < NT; ++u) {
            t[q][u] = tab[idx[u]];
            idx[u] += stp[u];
            if (idx[u] >= N) idx[u] -= N;
          }
          load(k + 4 * (h + q) + k0, x[q]);
        }
#pragma unroll
        for (int q = 0; q < RUN; ++q) {
          if (q >= cnt) break;
#pragma unroll
          for (int u = 0; u < NT; ++u) {
            part[u][0] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[q][u].x, x[q][0], part[u][0], 0, 0, 0);
            part[u][1] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[q][u].y, x[q][1], part[u][1], 0, 0, 0);
            part[u][2] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[q][u].x, x[q][2], part[u][2], 0, 0, 0);
            part[u][3] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[q][u].y, x[q][3], part[u][3], 0, 0, 0);
          }
        }
      };
      if (n == RUN)
        steps(RUN);  // (inlined with a constant count)
      else if (n > 0)
        steps(n);
    }
#pragma unroll
    for (int u = 0; u < NT; ++u)
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[u][i] += part[u][i];
  }
}

// T[(j*NH + m)*rs + s] = sum_i f[s][j][i] exp(-2 pi i m i / N), rows j0, j0 + 1
// of 16 slices per workgroup
template <int NT>
__global__ __launch_bounds__(256) void k_dense_rows_r2c(const float* __restrict__ f, float2* __restrict__ T, int ny,
                                                        int N, int S, int rs, const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float* E = reinterpret_cast<float*>(tab + N);
  float* O = E + K4 * kES;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j0 = 2 * blockIdx.x, s0 = kDS * blockIdx.y;
  for (int e = tid; e < N; e += 256) tab[e] = tw[e];
  // rows w, w + 4, .. of the 32 (row j0 + r/16, slice s0 + r%16), lanes along i
  for (int i = lane; i < K4; i += 64) {
    float a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = w + 4 * q, j = j0 + (r >> 4), s = s0 + (r & 15);
      a[q] = b[q] = 0.f;
      if (i < K && j < ny && s < S) {
        const float* row = f + ((size_t)s * ny + j) * N;
        a[q] = row[i];
        if (i > 0 && i < N / 2) b[q] = row[N - i];
      }
    }
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = w + 4 * q;
      E[i * kES + r] = a[q] + b[q];
      O[i * kES + r] = (i > 0 && i < N / 2) ? a[q] - b[q] : 0.f;
    }
  }
  __syncthreads();
  const int c = lane >> 4, s = s0 + (lane & 15);
  for (int mt = NT * w; 16 * mt < K; mt += 4 * NT) {
    v4f acc[NT][4];  // row j0: re, -im; row j0 + 1: re, -im
    dense_tiles<NT>(tab, N, K4, mt, lane, [&](int k, float (&x)[4]) {
      const int o = k * kES + (lane & 15);
      x[0] = E[o];
      x[1] = O[o];
      x[2] = E[o + 16];
      x[3] = O[o + 16];
    }, acc);
    if (s >= S) continue;
#pragma unroll
    for (int e = 0; e < 4 * NT; ++e) {
      const int u = e >> 2, r = e & 3, m = 16 * (mt + u) + 4 * c + r;
      if (m >= K) continue;
      T[(size_t)(j0 * K + m) * rs + s] = make_float2(acc[u][0][r], -acc[u][1][r]);
      if (j0 + 1 < ny) T[(size_t)((j0 + 1) * K + m) * rs + s] = make_float2(acc[u][2][r], -acc[u][3][r]);
    }
  }
}

// f[s][j][i] = scale * (real rows of the Hermitian half spectra in T) - sub
template <int NT>
__global__ __launch_bounds__(256) void k_dense_rows_c2r(const float2* __restrict__ T, float* __restrict__ f, int ny,
                                                        int N, int S, int rs, float scale,
                                                        const float* __restrict__ sub, const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float2* W = tab + N;  // [row][m][slice]: both parts times 2 (m = 0, N/2: the real part alone)
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int j0 = 2 * blockIdx.x, s0 = kDS * blockIdx.y;
  const int ls = tid & 15, lm = tid >> 4;
  for (int e = tid; e < N; e += 256) tab[e] = tw[e];
  constexpr int kRun = 4;
  for (int q0 = lm; q0 < 2 * K4; q0 += 16 * kRun) {
    float2 v[kRun];
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int e = q0 + 16 * q, jj = e >= K4, m = e - jj * K4;
      v[q] = make_float2(0.f, 0.f);
      if (jj < 2 && m < K && j0 + jj < ny && s0 + ls < S) v[q] = T[(size_t)((j0 + jj) * K + m) * rs + s0 + ls];
    }
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int e = q0 + 16 * q, m = e >= K4 ? e - K4 : e;
      if (e >= 2 * K4) break;
      W[e * 16 + ls] = (m == 0 || m == N / 2) ? make_float2(v[q].x, 0.f) : make_float2(2.f * v[q].x, 2.f * v[q].y);
    }
  }
  __syncthreads();
  const int c = lane >> 4, s = s0 + (lane & 15);
  for (int it = NT * w; 16 * it < K; it += 4 * NT) {
    v4f acc[NT][4];  // row j0: cos, sin sums; row j0 + 1
    dense_tiles<NT>(tab, N, K4, it, lane, [&](int k, float (&x)[4]) {
      const float2 a = W[k * 16 + (lane & 15)], b = W[(K4 + k) * 16 + (lane & 15)];
      x[0] = a.x;
      x[1] = a.y;
      x[2] = b.x;
      x[3] = b.y;
    }, acc);
    if (s >= S) continue;
#pragma unroll
    for (int e = 0; e < 2 * NT; ++e) {
      const int u = e >> 1, jj = e & 1;
      const int i0 = 16 * (it + u) + 4 * c;  // this lane's outputs i0 .. i0 + 3 and N - i0 - 3 .. N - i0
      if (j0 + jj >= ny) continue;
      const size_t row = ((size_t)s * ny + j0 + jj) * N;
      v4f lo, hi;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        lo[r] = scale * (acc[u][2 * jj][r] - acc[u][2 * jj + 1][r]);
        hi[3 - r] = scale * (acc[u][2 * jj][r] + acc[u][2 * jj + 1][r]);
      }
      if (i0 > 0 && i0 + 3 < N / 2) {
        v4f4* pl = reinterpret_cast<v4f4*>(f + row + i0);
        v4f4* ph = reinterpret_cast<v4f4*>(f + row + N - i0 - 3);
        if (sub) {
          lo -= (v4f)*reinterpret_cast<const v4f4*>(sub + row + i0);
          hi -= (v4f)*reinterpret_cast<const v4f4*>(sub + row + N - i0 - 3);
        }
        *pl = lo;
        *ph = hi;
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int i = i0 + r;
          if (i > N / 2) continue;
          f[row + i] = lo[r] - (sub ? sub[row + i] : 0.f);
          if (i > 0 && i < N / 2) f[row + N - i] = hi[3 - r] - (sub ? sub[row + N - i] : 0.f);
        }
      }
    }
  }
}

// out[orow(p)*rs + s] = sum_y exp(DIR 2 pi i p y / N) in[irow(y)*rs + s] for
// frequency column m; the spectrum side's rows by the map, the other's y*nh + m
template <int DIR, int NT>
__global__ __launch_bounds__(256) void k_dense_cols(const float2* __restrict__ in, float2* __restrict__ out, int nh,
                                                    int N, int S, int rs, const int32_t* __restrict__ imap,
                                                    const int32_t* __restrict__ omap, int sfast,
                                                    const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float2* E = tab + N;
  float2* O = E + K4 * 16;
  int* rin = reinterpret_cast<int*>(O + K4 * 16);
  int* rout = rin + N;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int m = sfast ? blockIdx.y : blockIdx.x;
  const int s0 = (sfast ? blockIdx.x : blockIdx.y) * kDS;
  const int ls = tid & 15, ly = tid >> 4;
  for (int y = tid; y < N; y += 256) {
    tab[y] = tw[y];
    rin[y] = imap ? imap[y * nh + m] : y * nh + m;
    rout[y] = omap ? omap[y * nh + m] : y * nh + m;
  }
  __syncthreads();
  constexpr int kRun = 4;
  for (int y0 = ly; y0 < K4; y0 += 16 * kRun) {
    float2 a[kRun], b[kRun];
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int y = y0 + 16 * q;
      a[q] = b[q] = make_float2(0.f, 0.f);
      if (y < K && s0 + ls < S) {
        if (rin[y] >= 0) a[q] = in[(size_t)rin[y] * rs + s0 + ls];
        if (y > 0 && y < N / 2 && rin[N - y] >= 0) b[q] = in[(size_t)rin[N - y] * rs + s0 + ls];
      }
    }
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int y = y0 + 16 * q;
      if (y >= K4) break;
      E[y * 16 + ls] = make_float2(a[q].x + b[q].x, a[q].y + b[q].y);
      O[y * 16 + ls] = (y > 0 && y < N / 2) ? make_float2(a[q].x - b[q].x, a[q].y - b[q].y) : make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
  const int c = lane >> 4, s = s0 + (lane & 15);
  for (int pt = NT * w; 16 * pt < K; pt += 4 * NT) {
    v4f acc[NT][4];  // C re, S re, C im, S im
    dense_tiles<NT>(tab, N, K4, pt, lane, [&](int k, float (&x)[4]) {
      const float2 e = E[k * 16 + (lane & 15)], o = O[k * 16 + (lane & 15)];
      x[0] = e.x;
      x[1] = o.x;
      x[2] = e.y;
      x[3] = o.y;
    }, acc);
    if (s >= S) continue;
#pragma unroll
    for (int e = 0; e < 4 * NT; ++e) {
      const int u = e >> 2, r = e & 3, p = 16 * (pt + u) + 4 * c + r;
      if (p >= K) continue;
      const float2 minus = make_float2(acc[u][0][r] + acc[u][3][r], acc[u][2][r] - acc[u][1][r]);  // C - i S
      const float2 plus = make_float2(acc[u][0][r] - acc[u][3][r], acc[u][2][r] + acc[u][1][r]);   // C + i S
      if (rout[p] >= 0) out[(size_t)rout[p] * rs + s] = DIR < 0 ? minus : plus;
      if (p > 0 && p < N / 2 && rout[N - p] >= 0) out[(size_t)rout[N - p] * rs + s] = DIR < 0 ? plus : minus;
    }
  }
}

static pat_status check_dense(int N) {
  if (N < 16 || N > 512 || N % 2) return fail(PAT_EUNSUPPORTED, "dense transforms: an even length in [16, 512]");
  return PAT_OK;
}

// Tiles of 16 outputs a wave takes together: two for long axes, where the
// waves then have no more rounds than with one (one A + one A^T: 510 x 510 x 8
// x 64, 727 us with two and 758 with one; 202 x 202 x 37 x 256, whose seven
// tiles make the fourth wave work for nothing, 330 and 311)
static bool two_tiles(int N) {
  const int tiles = (N / 2 + 16) / 16;
  return tiles > 8 && 2 * ((tiles + 7) / 8) <= (tiles + 3) / 4;
}

pat_status dense_rows_r2c(const float* f, float2* T, int ny, int N, int S, int rs, const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 8 + (size_t)2 * dense_k4(N) * kES * 4;
  const dim3 grid((ny + 1) / 2, (S + kDS - 1) / kDS);
  if (two_tiles(N))
    k_dense_rows_r2c<2><<<grid, 256, lds, st>>>(f, T, ny, N, S, rs, tw);
  else
    k_dense_rows_r2c<1><<<grid, 256, lds, st>>>(f, T, ny, N, S, rs, tw);
  PAT_LAUNCHED("dense rows r2c");
  return PAT_OK;
}

pat_status dense_rows_c2r(const float2* T, float* f, int ny, int N, int S, int rs, float scale, const float* sub,
                          const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 8 + (size_t)2 * dense_k4(N) * 16 * 8;
  const dim3 grid((ny + 1) / 2, (S + kDS - 1) / kDS);
  if (two_tiles(N))
    k_dense_rows_c2r<2><<<grid, 256, lds, st>>>(T, f, ny, N, S, rs, scale, sub, tw);
  else
    k_dense_rows_c2r<1><<<grid, 256, lds, st>>>(T, f, ny, N, S, rs, scale, sub, tw);
  PAT_LAUNCHED("dense rows c2r");
  return PAT_OK;
}

pat_status dense_cols(int dir, const float2* in, float2* out, int nh, int N, int S, int rs, const int32_t* imap,
                      const int32_t* omap, const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 16 + (size_t)2 * dense_k4(N) * 16 * 8;
  const int sfast = S >= 2048, nsb = (S + kDS - 1) / kDS;
  const dim3 grid = sfast ? dim3(nsb, nh) : dim3(nh, nsb);
  auto go = [&](auto kernel) { kernel<<<grid, 256, lds, st>>>(in, out, nh, N, S, rs, imap, omap, sfast, tw); };
  if (two_tiles(N))
    dir < 0 ? go(k_dense_cols<-1, 2>) : go(k_dense_cols<+1, 2>);
  else
    dir < 0 ? go(k_dense_cols<-1, 1>) : go(k_dense_cols<+1, 1>);
  PAT_LAUNCHED("dense columns");
  return PAT_OK;
}

}  // namespace pat
