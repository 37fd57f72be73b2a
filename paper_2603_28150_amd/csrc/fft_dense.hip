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
#include <algorithm>

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

// T[(j*NH + m)*rs + s] = sum_i f[s][j][i] exp(-2 pi i m i / N), two rows of 16
// slices per workgroup, or (PACK) 2^(5 - lsp) rows of 2^lsp slices
template <int NT, bool PACK>
__global__ __launch_bounds__(256) void k_dense_rows_r2c(const float* __restrict__ f, float2* __restrict__ T, int ny,
                                                        int N, int S, int rs, int lsp, int parts,
                                                        const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float* E = reinterpret_cast<float*>(tab + N);
  float* O = E + K4 * kES;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ls = PACK ? lsp : 4;
  const int j0 = (2 * kDS >> ls) * blockIdx.x, s0 = blockIdx.y << ls, sm = (1 << ls) - 1;
  for (int e = tid; e < N; e += 256) tab[e] = tw[e];
  // rows w, w + 4, .. of the 32 (row j0 + (r >> ls), slice s0 + (r & sm)), lanes along i
  for (int i = lane; i < K4; i += 64) {
    float a[8], b[8];
#pragma unroll
    for (int q = 0; q < 8; ++q) {
      const int r = w + 4 * q, j = j0 + (r >> ls), s = s0 + (r & sm);
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
  const int c = lane >> 4, l16 = lane & 15, s = s0 + (l16 & sm), ja = j0 + (l16 >> ls), jb = j0 + ((l16 + 16) >> ls);
  for (int mt = NT * (w + 4 * blockIdx.z); 16 * mt < K; mt += 4 * NT * parts) {
    v4f acc[NT][4];  // columns 0..15: re, -im; columns 16..31: re, -im
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
      if (ja < ny) T[(size_t)(ja * K + m) * rs + s] = make_float2(acc[u][0][r], -acc[u][1][r]);
      if (jb < ny) T[(size_t)(jb * K + m) * rs + s] = make_float2(acc[u][2][r], -acc[u][3][r]);
    }
  }
}

// f[s][j][i] = scale * (real rows of the Hermitian half spectra in T) - sub, rows
// as above
template <int NT, bool PACK>
__global__ __launch_bounds__(256) void k_dense_rows_c2r(const float2* __restrict__ T, float* __restrict__ f, int ny,
                                                        int N, int S, int rs, int lsp, int parts, float scale,
                                                        const float* __restrict__ sub, const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float2* W = tab + N;  // [half][m][column]: both parts times 2 (m = 0, N/2: the real part alone)
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ls = PACK ? lsp : 4;
  const int j0 = (2 * kDS >> ls) * blockIdx.x, s0 = blockIdx.y << ls, sm = (1 << ls) - 1;
  const int col = tid & 15, lm = tid >> 4;
  for (int e = tid; e < N; e += 256) tab[e] = tw[e];
  constexpr int kRun = 4;
  for (int q0 = lm; q0 < 2 * K4; q0 += 16 * kRun) {
    float2 v[kRun];
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int e = q0 + 16 * q, jj = e >= K4, m = e - jj * K4;
      v[q] = make_float2(0.f, 0.f);
      const int r = 16 * jj + col, j = j0 + (r >> ls), s = s0 + (r & sm);
      if (jj < 2 && m < K && j < ny && s < S) v[q] = T[(size_t)(j * K + m) * rs + s];
    }
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int e = q0 + 16 * q, m = e >= K4 ? e - K4 : e;
      if (e >= 2 * K4) break;
      W[e * 16 + col] = (m == 0 || m == N / 2) ? make_float2(v[q].x, 0.f) : make_float2(2.f * v[q].x, 2.f * v[q].y);
    }
  }
  __syncthreads();
  const int c = lane >> 4, l16 = lane & 15, s = s0 + (l16 & sm);
  for (int it = NT * (w + 4 * blockIdx.z); 16 * it < K; it += 4 * NT * parts) {
    v4f acc[NT][4];  // columns 0..15: cos, sin sums; columns 16..31
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
      const int j = j0 + ((16 * jj + l16) >> ls);
      if (j >= ny) continue;
      const size_t row = ((size_t)s * ny + j) * N;
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
// frequency column m; the spectrum side's rows by the map, the other's y*nh + m;
// 16 slices of one column per workgroup, or (PACK) 2^lsp of 2^(4 - lsp) columns
template <int DIR, int NT, bool PACK>
__global__ __launch_bounds__(256) void k_dense_cols(const float2* __restrict__ in, float2* __restrict__ out, int nh,
                                                    int N, int S, int rs, const int32_t* __restrict__ imap,
                                                    const int32_t* __restrict__ omap, int sfast, int lsp, int parts,
                                                    const float2* __restrict__ tw) {
  extern __shared__ float2 dlds[];
  const int K = N / 2 + 1, K4 = dense_k4(N);
  float2* tab = dlds;
  float2* E = tab + N;
  float2* O = E + K4 * 16;
  int* rin = reinterpret_cast<int*>(O + K4 * 16);
  int* rout = rin + N;
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int ls = PACK ? lsp : 4;
  const int m0 = (sfast ? blockIdx.y : blockIdx.x) * (kDS >> ls), sm = (1 << ls) - 1;
  const int s0 = (sfast ? blockIdx.x : blockIdx.y) << ls;
  const int col = tid & 15, ly = tid >> 4;  // column of 16: frequency m0 + (col >> ls), slice s0 + (col & sm)
  const int m = m0 + (col >> ls), s = s0 + (col & sm);
  const bool live = m < nh && s < S;
  for (int y = tid; y < N; y += 256) {
    tab[y] = tw[y];
    if (!PACK) {  // one frequency: its rows once for all threads
      rin[y] = imap ? imap[y * nh + m0] : y * nh + m0;
      rout[y] = omap ? omap[y * nh + m0] : y * nh + m0;
    }
  }
  auto row = [&](const int32_t* map, const int* rows, int y) {
    return !PACK ? rows[y] : map ? map[y * nh + m] : y * nh + m;
  };
  __syncthreads();
  constexpr int kRun = 4;
  for (int y0 = ly; y0 < K4; y0 += 16 * kRun) {
    float2 a[kRun], b[kRun];
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int y = y0 + 16 * q;
      a[q] = b[q] = make_float2(0.f, 0.f);
      if (y < K && live) {
        const int ra = row(imap, rin, y), rb = y > 0 && y < N / 2 ? row(imap, rin, N - y) : -1;
        if (ra >= 0) a[q] = in[(size_t)ra * rs + s];
        if (rb >= 0) b[q] = in[(size_t)rb * rs + s];
      }
    }
#pragma unroll
    for (int q = 0; q < kRun; ++q) {
      const int y = y0 + 16 * q;
      if (y >= K4) break;
      E[y * 16 + col] = make_float2(a[q].x + b[q].x, a[q].y + b[q].y);
      O[y * 16 + col] = (y > 0 && y < N / 2) ? make_float2(a[q].x - b[q].x, a[q].y - b[q].y) : make_float2(0.f, 0.f);
    }
  }
  __syncthreads();
  const int c = lane >> 4;  // (the lane's column of the results is col: tid and lane agree in the last four bits)
  for (int pt = NT * (w + 4 * blockIdx.z); 16 * pt < K; pt += 4 * NT * parts) {
    v4f acc[NT][4];  // C re, S re, C im, S im
    dense_tiles<NT>(tab, N, K4, pt, lane, [&](int k, float (&x)[4]) {
      const float2 e = E[k * 16 + (lane & 15)], o = O[k * 16 + (lane & 15)];
      x[0] = e.x;
      x[1] = o.x;
      x[2] = e.y;
      x[3] = o.y;
    }, acc);
    if (!live) continue;
#pragma unroll
    for (int e = 0; e < 4 * NT; ++e) {
      const int u = e >> 2, r = e & 3, p = 16 * (pt + u) + 4 * c + r;
      if (p >= K) continue;
      const float2 minus = make_float2(acc[u][0][r] + acc[u][3][r], acc[u][2][r] - acc[u][1][r]);  // C - i S
      const float2 plus = make_float2(acc[u][0][r] - acc[u][3][r], acc[u][2][r] + acc[u][1][r]);   // C + i S
      const int ra = row(omap, rout, p), rb = p > 0 && p < N / 2 ? row(omap, rout, N - p) : -1;
      if (ra >= 0) out[(size_t)ra * rs + s] = DIR < 0 ? minus : plus;
      if (rb >= 0) out[(size_t)rb * rs + s] = DIR < 0 ? plus : minus;
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

// A workgroup's loads and products take turns, and a few workgroups cannot fill
// the chip: up to kShareBlocks of them, the output tiles of a workgroup's slices
// are dealt to several (grid.z), each with one round of tiles; more would repeat
// the loads for nothing (one forward / inverse transform, one workgroup each and
// shared: 510 x 18, 16 slices, 32 / 45 us, 17 / 27; 202 x 202, 16 slices, 22 / 27, 17 /
// 22; 510 x 510, 16 slices, 74 / 82, 68 / 75, and with up to 1,024 workgroups 80 / 94).
constexpr int kShareBlocks = 512;
static int tile_rounds(int N) { return ((N / 2 + 16) / 16 + 3) / 4; }
static int tile_shares(int N, const dim3& grid) {
  return (int)std::max(1LL, std::min((long long)tile_rounds(N), kShareBlocks / ((long long)grid.x * grid.y)));
}

// log2 of the slices among a product's 16 columns.  Fewer than nine slices leave
// room for further rows (or frequencies; `lines` in all, 2^lines16 per workgroup
// of 16 slices) beside them, taken where the workgroups are too many to share
// their tiles (510 x 510, one slice: 69 / 77 us, 44 / 53 so; not for 100 x 100, 50
// workgroups of one round: A 30.5 us, 35.4 if packed).
static int slice_bits(int S, int N, int lines, int lines16) {
  int ls = 4;
  while (ls > 0 && S <= 1 << (ls - 1) && ((lines << ls) >> (4 + lines16)) * tile_rounds(N) > kShareBlocks) --ls;
  return ls;
}

pat_status dense_rows_r2c(const float* f, float2* T, int ny, int N, int S, int rs, const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 8 + (size_t)2 * dense_k4(N) * kES * 4;
  const int ls = slice_bits(S, N, ny, 1), rows = 2 * kDS >> ls;
  dim3 grid((ny + rows - 1) / rows, (S + (1 << ls) - 1) >> ls);
  grid.z = tile_shares(N, grid);
  auto go = [&](auto kernel) { kernel<<<grid, 256, lds, st>>>(f, T, ny, N, S, rs, ls, (int)grid.z, tw); };
  if (ls < 4)
    go(k_dense_rows_r2c<1, true>);
  else if (grid.z == 1 && two_tiles(N))
    go(k_dense_rows_r2c<2, false>);
  else
    go(k_dense_rows_r2c<1, false>);
  PAT_LAUNCHED("dense rows r2c");
  return PAT_OK;
}

pat_status dense_rows_c2r(const float2* T, float* f, int ny, int N, int S, int rs, float scale, const float* sub,
                          const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 8 + (size_t)2 * dense_k4(N) * 16 * 8;
  const int ls = slice_bits(S, N, ny, 1), rows = 2 * kDS >> ls;
  dim3 grid((ny + rows - 1) / rows, (S + (1 << ls) - 1) >> ls);
  grid.z = tile_shares(N, grid);
  auto go = [&](auto kernel) { kernel<<<grid, 256, lds, st>>>(T, f, ny, N, S, rs, ls, (int)grid.z, scale, sub, tw); };
  if (ls < 4)
    go(k_dense_rows_c2r<1, true>);
  else if (grid.z == 1 && two_tiles(N))
    go(k_dense_rows_c2r<2, false>);
  else
    go(k_dense_rows_c2r<1, false>);
  PAT_LAUNCHED("dense rows c2r");
  return PAT_OK;
}

pat_status dense_cols(int dir, const float2* in, float2* out, int nh, int N, int S, int rs, const int32_t* imap,
                      const int32_t* omap, const float2* tw, hipStream_t st) {
  PAT_TRY(check_dense(N));
  const size_t lds = (size_t)N * 16 + (size_t)2 * dense_k4(N) * 16 * 8;
  const int ls = slice_bits(S, N, nh, 0), per = kDS >> ls;
  const int sfast = S >= 2048, nsb = (S + (1 << ls) - 1) >> ls, nmb = (nh + per - 1) / per;
  dim3 grid = sfast ? dim3(nsb, nmb) : dim3(nmb, nsb);
  grid.z = tile_shares(N, grid);
  auto go = [&](auto kernel) { kernel<<<grid, 256, lds, st>>>(in, out, nh, N, S, rs, imap, omap, sfast, ls, (int)grid.z, tw); };
  if (ls < 4)
    dir < 0 ? go(k_dense_cols<-1, 1, true>) : go(k_dense_cols<+1, 1, true>);
  else if (grid.z == 1 && two_tiles(N))
    dir < 0 ? go(k_dense_cols<-1, 2, false>) : go(k_dense_cols<+1, 2, false>);
  else
    dir < 0 ? go(k_dense_cols<-1, 1, false>) : go(k_dense_cols<+1, 1, false>);
  PAT_LAUNCHED("dense columns");
  return PAT_OK;
}

}  // namespace pat
