// Kernel library build: the sensor-plane response of a unit point absorber at
// each depth, in the transverse Fourier domain (the depth-indexed impulse
// responses of Sec. 2.1, built once and reused by every apply, Sec. 3.2).
//
// On the grid that is periodic in x, y and z (z-period nq = nz_sim) the exact
// semi-discrete solution of the wave equation with zero initial velocity is
// cos(c t |k|) times the initial spectrum.  Restricted to the sensor plane:
//
//   H^[l, n] = (1/nq) sum_{q} cos(n c dt |k(q)|) cos(2 pi q l / nq)
//            = sum_{q=0}^{floor(nq/2)} w_q/nq cos(n theta_q) cos(2 pi q l / nq),
//
// with theta_q = c dt sqrt(kx^2 + ky^2 + kz(q)^2), w_q = 2 for the pairs
// {q, -q} and 1 for q = 0 and the Nyquist plane; the imaginary parts cancel
// in pairs, so H^ is real.  Phases reach several hundred radians, so the
// whole build runs in float64 and rounds once (to float32, then to 16 bits
// for the reduced-precision forms).  A sensor response r (causal FIR) is
// folded in along t: H^'[l, n] = sum_j r_j H^[l, n - j].
//
// Two ways to obtain the time factor: evaluated directly (closed form), or
// by one k-space time-stepping run from a unit point source at the origin,
// P^0 = 1, P^1 = cos(theta) P^0, P^{n+1} = 2 cos(theta) P^n - P^{n-1} (the
// exact propagator with zero initial velocity, float64), whose field on depth
// plane l at step n is the inverse z-DFT sum above: by reciprocity the field
// at depth l due to a source on the sensor plane is the sensor-plane
// response to a source at depth l (the single-simulation library of
// Sec. 3.2).  The stepper records the field of a block of classes in build
// scratch; the depth sum then reads the record instead of the cosines.
#include <algorithm>
#include <cmath>

#include "pat_internal.hpp"

namespace pat {

constexpr int kNT = 64;   // time samples per workgroup
constexpr int kLP = 128;  // depths per pass
constexpr int kQB = 32;   // q values per LDS chunk
constexpr int kPS = 80;   // LDS row stride of a chunk: its four rows of a product fall into different banks
constexpr int kTS = kLP + 1;  // LDS row stride of the finished tile
constexpr int kMaxNq = 4096;

typedef double v4d __attribute__((ext_vector_type(4)));

__device__ __forceinline__ int ceil_log2_d(double v) {
  int e;
  const double f = frexp(v, &e);  // v = f 2^e, 0.5 <= f < 1
  return f == 0.5 ? e - 1 : e;
}

__device__ __forceinline__ double depth_scale(const unsigned long long* amax, int l, int hdtype) {
  if (hdtype == PAT_H_F32) return 1.0;
  const double m = __longlong_as_double((long long)amax[l]);
  if (!(m > 0.0)) return 1.0;
  const int e = hdtype == PAT_H_BF16 ? 0 : 15;
  return ldexp(1.0, e - ceil_log2_d(m));
}

__device__ __forceinline__ unsigned short to_bf16(float f) {
  unsigned u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (unsigned short)(u >> 16);
}

__device__ __forceinline__ unsigned short to_f16(float f) {
  _Float16 h = (_Float16)f;
  unsigned short b;
  __builtin_memcpy(&b, &h, 2);
  return b;
}

// Stepped time factor of class a.c0 + blockIdx.y for the wavenumbers
// q = 0 .. nq/2 (one thread each): P^n(q) for n < nt, weighted by w_q / nq,
// into ptab[(blockIdx.y * nt + n) * (nq/2 + 1) + q].
__global__ __launch_bounds__(256) void k_hstep(HBuildArgs a) {
  const int Qn = a.nq / 2 + 1;
  const int q = blockIdx.x * blockDim.x + threadIdx.x;
  if (q >= Qn) return;
  const int c = a.c0 + blockIdx.y;
  const double two_pi = 6.283185307179586476925286766559;
  const double kx = two_pi * a.cls_freq[2 * c] / (a.nx * a.dx);
  const double ky = two_pi * a.cls_freq[2 * c + 1] / (a.ny * a.dy);
  const double kz = two_pi * q / (a.nq * a.dz);
  const double theta = a.c * a.dt * sqrt(kx * kx + ky * ky + kz * kz);
  const double two_cos = 2.0 * cos(theta);
  const double w = ((q == 0 || 2 * q == a.nq) ? 1.0 : 2.0) / a.nq;
  double* rec = a.ptab + (size_t)blockIdx.y * a.nt * Qn + q;
  double prev = 1.0;             // P^0: unit point source (flat spectrum)
  double cur = 0.5 * two_cos;    // P^1 = cos(theta) P^0: zero initial velocity
  rec[0] = w * prev;
  for (int n = 1; n < a.nt; ++n) {
    rec[(size_t)n * Qn] = w * cur;
    const double next = fma(two_cos, cur, -prev);
    prev = cur;
    cur = next;
  }
}

// LDS of k_hbuild: cos(2 pi r / nq), the time factors of a q chunk and (in
// their place) the finished tile, then theta, cos theta and sin theta of every
// q (closed form) and the sensor response with the unfiltered time factors
struct BuildLds {
  int o_p, o_th, o_raw, o_ir, total;
  __host__ __device__ BuildLds(int nq, bool fir, bool step) {
    const int qn = nq / 2 + 1;
    o_p = nq * 8;
    const int p = kQB * kPS * 8, t = kNT * kTS * 4;
    o_th = o_p + (p > t ? p : t);
    o_raw = o_th + (step ? 0 : 3 * qn * 8);
    o_ir = o_raw + (fir ? kQB * (kNT + kMaxIr - 1) * 8 : 0);
    total = o_ir + (fir ? kMaxIr * 8 : 0);
  }
};

// MODE 0: per-depth max |H^| only, 1: write the slabs.  FIR: fold the sensor
// response into the time axis.  The library is linear in the time factor
// cos(n theta_q), so the filter acts on that factor: each q-chunk also
// evaluates it at the n_ir - 1 earlier samples (zero before t = 0) and
// filters in LDS before the depth sum.
//
// The depth sum is the product of the constant matrix cos(2 pi q l / nq) with
// the class's time factors, on the float64 matrix instruction: workgroup =
// (class, 64 samples), wave = half of the samples and every other 16 depths
// of a pass of 128, so that a time factor is evaluated once per pass and a
// cosine read from LDS serves two products.  Bound by the matrix rate (45 TF
// measured for this instruction) and the evaluation of the time factors, one
// sincos and seven rotations by theta for eight samples.  The vector form it
// replaced (one multiply-add per cosine read, a cosine per sample, passes of
// 64 depths) took 24.3 ms at 256 x 256 x 128 x 512 and 2.59 ms at
// 128 x 128 x 96 x 384; now 5.4 and 0.51.
template <int MODE, bool FIR, bool STEP>
__global__ __launch_bounds__(256, 3) void k_hbuild(HBuildArgs a) {
  extern __shared__ double hb_lds[];
  const int nq = a.nq, Qn = nq / 2 + 1;
  char* base = reinterpret_cast<char*>(hb_lds);
  const BuildLds at(nq, FIR, STEP);
  double* ctab = hb_lds;
  double* P = reinterpret_cast<double*>(base + at.o_p);
  float* tile = reinterpret_cast<float*>(base + at.o_p);
  double* th = reinterpret_cast<double*>(base + at.o_th);
  double* Praw = reinterpret_cast<double*>(base + at.o_raw);
  double* irs = reinterpret_cast<double*>(base + at.o_ir);
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  const int c = a.c0 + blockIdx.y;
  const int n0 = blockIdx.x * kNT;
  const double* rec = STEP ? a.ptab + (size_t)blockIdx.y * a.nt * Qn : nullptr;
  const double two_pi = 6.283185307179586476925286766559;
  const double inv_nq = 1.0 / nq;

  for (int r = tid; r < nq; r += 256) ctab[r] = cos(two_pi * (double)r / (double)nq);
  if constexpr (FIR)
    for (int j = tid; j < a.n_ir; j += 256) irs[j] = a.ir[j];
  if constexpr (!STEP) {
    const double kx = two_pi * a.cls_freq[2 * c] / (a.nx * a.dx);
    const double ky = two_pi * a.cls_freq[2 * c + 1] / (a.ny * a.dy);
    const double kperp2 = kx * kx + ky * ky;
    const double cdt = a.c * a.dt;
    for (int q = tid; q < Qn; q += 256) {
      const double kz = two_pi * q / (nq * a.dz);
      const double theta = cdt * sqrt(kperp2 + kz * kz);
      double sn, cs;
      sincos(theta, &sn, &cs);
      th[q] = theta;
      th[Qn + q] = cs;
      th[2 * Qn + q] = sn;
    }
  }

  // weighted time factors of samples ng .. ng + 7 at wavenumber q: one sincos,
  // then rotations by theta (seven, a few 1e-16)
  auto factors8 = [&](int q, int ng, double (&v)[8]) {
    const double wq = (q == 0 || 2 * q == nq) ? inv_nq : 2.0 * inv_nq;
    const double cs = th[Qn + q], sn = th[2 * Qn + q];
    double C, S;
    sincos((double)ng * th[q], &S, &C);
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      v[j] = wq * C;
      const double C1 = C * cs - S * sn;
      S = S * cs + C * sn;
      C = C1;
    }
  };

  for (int l0 = 0; l0 < a.nz; l0 += kLP) {
    // depth tile u of this wave: depths l0 + 16 (2u + w/2) + ..; samples
    // 32 (w & 1) + 16 s + .. of the tile
    const int nlt = (min(a.nz - l0, kLP) + 15) >> 4;
    v4d acc[4][2];
    int idx[4], stp[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      acc[u][0] = acc[u][1] = v4d{0.0, 0.0, 0.0, 0.0};
      const int l = (l0 + 16 * (2 * u + (w >> 1)) + li) % nq;
      idx[u] = (int)((long long)lk * l % nq);
      stp[u] = (int)(4LL * l % nq);
    }
    for (int q0 = 0; q0 < Qn; q0 += kQB) {
      __syncthreads();
      if constexpr (!FIR && !STEP) {
        const int qq = tid >> 3, nb = 8 * (tid & 7), q = q0 + qq;
        double v[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) v[j] = 0.0;
        if (q < Qn) factors8(q, n0 + nb, v);
#pragma unroll
        for (int j = 0; j < 8; ++j) P[qq * kPS + nb + j] = n0 + nb + j < a.nt ? v[j] : 0.0;
      } else if constexpr (!FIR) {
        for (int e = tid; e < kQB * kNT; e += 256) {
          const int qq = e / kNT, nn = e % kNT;
          const int q = q0 + qq, ng = n0 + nn;
          P[qq * kPS + nn] = (q < Qn && ng < a.nt) ? rec[(size_t)ng * Qn + q] : 0.0;
        }
      } else {
        const int L = a.n_ir, W = kNT + L - 1;
        const int nbase = n0 - (L - 1);
        if constexpr (STEP) {
          for (int e = tid; e < kQB * W; e += 256) {
            const int qq = e / W, nr = e % W;
            const int q = q0 + qq, ng = nbase + nr;
            Praw[qq * W + nr] = (q < Qn && ng >= 0 && ng < a.nt) ? rec[(size_t)ng * Qn + q] : 0.0;
          }
        } else {
          const int nblk = (W + 7) >> 3;
          for (int e = tid; e < kQB * nblk; e += 256) {
            const int qq = e / nblk, nb = 8 * (e - qq * nblk), q = q0 + qq;
            double v[8];
#pragma unroll
            for (int j = 0; j < 8; ++j) v[j] = 0.0;
            if (q < Qn) factors8(q, nbase + nb, v);
#pragma unroll
            for (int j = 0; j < 8; ++j) {
              const int ng = nbase + nb + j;
              if (nb + j < W) Praw[qq * W + nb + j] = (ng >= 0 && ng < a.nt) ? v[j] : 0.0;
            }
          }
        }
        __syncthreads();
        for (int e = tid; e < kQB * kNT; e += 256) {
          const int qq = e / kNT, nn = e % kNT;
          const double* pr = Praw + qq * W + nn + (L - 1);
          double v = 0.0;
          for (int j = 0; j < L; ++j) v = fma(irs[j], pr[-j], v);
          P[qq * kPS + nn] = v;
        }
      }
      __syncthreads();
      // four q per product; rows of P past the last q are zeros
      const int steps = min(kQB / 4, (Qn - q0 + 3) >> 2);
      for (int k = 0; k < steps; ++k) {
        const double* pr = P + (4 * k + lk) * kPS + 32 * (w & 1) + li;
        const double b0 = pr[0], b1 = pr[16];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          if (2 * u + (w >> 1) >= nlt) break;
          const double x = ctab[idx[u]];
          idx[u] += stp[u];
          if (idx[u] >= nq) idx[u] -= nq;
          acc[u][0] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b0, acc[u][0], 0, 0, 0);
          acc[u][1] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, b1, acc[u][1], 0, 0, 0);
        }
      }
    }

    // accumulator register r of a lane: depth lk + 4 r, sample li of its tile
    if (MODE == 0) {
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int l = l0 + 16 * (2 * u + (w >> 1)) + lk + 4 * r;
          double m = 0.0;
#pragma unroll
          for (int s = 0; s < 2; ++s)
            if (n0 + 32 * (w & 1) + 16 * s + li < a.nt) m = fmax(m, fabs(acc[u][s][r]));
          for (int off = 8; off >= 1; off >>= 1) m = fmax(m, __shfl_xor(m, off));
          if (li == 0 && l < a.nz) atomicMax(&a.amax[l], (unsigned long long)__double_as_longlong(m));
        }
    } else {
      // the scaled values through LDS (in place of the last chunk), so that
      // every layout is written in runs
      __syncthreads();
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const int ll = 16 * (2 * u + (w >> 1)) + lk + 4 * r, l = l0 + ll;
          const double sc = l < a.nz ? depth_scale(a.amax, l, a.hdtype) : 0.0;
#pragma unroll
          for (int s = 0; s < 2; ++s)
            tile[(32 * (w & 1) + 16 * s + li) * kTS + ll] = (float)(acc[u][s][r] * sc);
        }
      __syncthreads();
      // [l][n] rows: lanes along n
      const int nl = min(a.nz - l0, kLP);
      for (int e = tid; e < kNT * nl; e += 256) {
        const int ll = e / kNT, nn = e % kNT;
        const int n = n0 + nn, l = l0 + ll;
        if (n >= a.nt) continue;
        const float f = tile[nn * kTS + ll];
        const size_t o = ((size_t)c * a.nz + l) * a.sA_row + n;
        if (a.hdtype == PAT_H_F32) reinterpret_cast<float*>(a.rowA)[o] = f;
        else if (a.hdtype == PAT_H_BF16) reinterpret_cast<unsigned short*>(a.rowA)[o] = to_bf16(f);
        else reinterpret_cast<unsigned short*>(a.rowA)[o] = to_f16(f);
      }
      // [n][l] rows: lanes along l
      for (int e = tid; e < kNT * kLP; e += 256) {
        const int nn = e / kLP, ll = e % kLP;
        const int ng = n0 + nn, l = l0 + ll;
        if (ng >= a.nt || l >= a.nz) continue;
        const float f = tile[nn * kTS + ll];
        const size_t o = ((size_t)c * a.nt + ng) * a.sT_row + l;
        if (a.hdtype == PAT_H_F32) reinterpret_cast<float*>(a.rowT)[o] = f;
        else if (a.hdtype == PAT_H_BF16) reinterpret_cast<unsigned short*>(a.rowT)[o] = to_bf16(f);
        else reinterpret_cast<unsigned short*>(a.rowT)[o] = to_f16(f);
      }
      if (a.hdtype != PAT_H_F32) {
        // 16-bit library: MFMA fragments for both directions, from the tile
        for (int dir = 0; dir < 2; ++dir) {
          // dir 0: rows n, k = l (forward);  dir 1: rows l, k = n (adjoint)
          const int nt = dir == 0 ? a.ntA : a.ntT, ks = dir == 0 ? a.ksA : a.ksT;
          const int rt0 = (dir == 0 ? n0 : l0) / 32, kt0 = (dir == 0 ? l0 : n0) / 16;
          const int kts = dir == 0 ? kLP / 16 : kNT / 16;  // k tiles of the LDS tile
          unsigned short* dst = reinterpret_cast<unsigned short*>(dir == 0 ? a.slabA : a.slabT);
          for (int unit = tid; unit < (kNT / 32) * (kLP / 16) * 64; unit += 256) {
            const int f = unit >> 6, L = unit & 63;
            const int rt = f / kts, kt = f % kts;
            if (rt0 + rt >= nt || kt0 + kt >= ks) continue;
            const int r = rt * 32 + (L & 31), k = kt * 16 + 8 * (L >> 5);
            unsigned short v[8];
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = dir == 0 ? tile[r * kTS + k + e] : tile[(k + e) * kTS + r];
              v[e] = a.hdtype == PAT_H_BF16 ? to_bf16(x) : to_f16(x);
            }
            uint4 pk;
            pk.x = v[0] | ((unsigned)v[1] << 16);
            pk.y = v[2] | ((unsigned)v[3] << 16);
            pk.z = v[4] | ((unsigned)v[5] << 16);
            pk.w = v[6] | ((unsigned)v[7] << 16);
            const size_t o = (((size_t)c * nt + rt0 + rt) * ks + kt0 + kt) * 64 + L;
            reinterpret_cast<uint4*>(dst)[o] = pk;
          }
        }
      }
    }
  }
}

__global__ void k_scales(const unsigned long long* amax, float* inv_scale, int nz, int hdtype) {
  const int l = blockIdx.x * blockDim.x + threadIdx.x;
  if (l < nz) inv_scale[l] = (float)(1.0 / depth_scale(amax, l, hdtype));
}

template <int MODE>
static pat_status launch_depth_sum(const HBuildArgs& a, int ncls, hipStream_t st) {
  dim3 grid((a.nt + kNT - 1) / kNT, ncls);
  const bool fir = a.n_ir > 0, step = a.ptab != nullptr;
  const size_t lds = (size_t)BuildLds(a.nq, fir, step).total;
  if (step && fir) k_hbuild<MODE, true, true><<<grid, 256, lds, st>>>(a);
  else if (step) k_hbuild<MODE, false, true><<<grid, 256, lds, st>>>(a);
  else if (fir) k_hbuild<MODE, true, false><<<grid, 256, lds, st>>>(a);
  else k_hbuild<MODE, false, false><<<grid, 256, lds, st>>>(a);
  PAT_LAUNCHED(MODE == 0 ? "H build (max pass)" : "H build");
  return PAT_OK;
}

// one pass over all classes (MODE 0: per-depth maxima, 1: the slabs); the
// stepped build records and sums one block of classes at a time
template <int MODE>
static pat_status build_pass(const HBuildArgs& a, hipStream_t st) {
  if (!a.ptab) return launch_depth_sum<MODE>(a, a.nclass, st);
  const size_t per = step_class_bytes(a.nt, a.nq);
  const int block = (int)std::min<size_t>((size_t)a.nclass, a.ptab_bytes / per);
  if (block < 1) return fail(PAT_EINVAL, "build scratch holds less than one class's record");
  const int Qn = a.nq / 2 + 1;
  for (int c0 = 0; c0 < a.nclass; c0 += block) {
    HBuildArgs b = a;
    b.c0 = c0;
    const int ncls = std::min(block, a.nclass - c0);
    k_hstep<<<dim3((Qn + 255) / 256, ncls), 256, 0, st>>>(b);
    PAT_LAUNCHED("H build (k-space stepper)");
    PAT_TRY(launch_depth_sum<MODE>(b, ncls, st));
  }
  return PAT_OK;
}

pat_status hbuild(const HBuildArgs& a, hipStream_t st) {
  if (a.nq > kMaxNq) return fail(PAT_EUNSUPPORTED, "nz_sim above 4096 is not supported");
  if (a.n_ir < 0 || a.n_ir > kMaxIr || (a.n_ir > 0 && !a.ir))
    return fail(PAT_EINVAL, "sensor response: 0..64 taps");
  if (a.hdtype != PAT_H_F32) PAT_TRY(build_pass<0>(a, st));
  k_scales<<<(a.nz + 127) / 128, 128, 0, st>>>(a.amax, a.inv_scale, a.nz, a.hdtype);
  PAT_LAUNCHED("H build (scales)");
  return build_pass<1>(a, st);
}

// ------------------------------------------------------------ export
__global__ void k_hexport(const void* slabA, int hdtype, const int32_t* kclass,
                          const float* inv_scale, int k0, int nz, int nt, int sA_row, int ntA,
                          int ksA, float* out) {
  const int kk = blockIdx.x;
  const int c = kclass[k0 + kk];
  for (int e = threadIdx.x; e < nz * nt; e += blockDim.x) {
    const int l = e / nt, n = e % nt;
    float f;
    if (hdtype == PAT_H_F32) {
      f = reinterpret_cast<const float*>(slabA)[((size_t)c * nz + l) * sA_row + n];
    } else {
      // fragment (n/32, l/16), lane n%32 + 32*((l%16)/8), element l%8
      const size_t o = ((((size_t)c * ntA + n / 32) * ksA + l / 16) * 64 + (n & 31) + 32 * ((l >> 3) & 1)) * 8 + (l & 7);
      const unsigned short b = reinterpret_cast<const unsigned short*>(slabA)[o];
      if (hdtype == PAT_H_BF16) {
        f = __uint_as_float((unsigned)b << 16);
      } else {
        _Float16 h;
        __builtin_memcpy(&h, &b, 2);
        f = (float)h;
      }
    }
    out[(size_t)kk * nz * nt + e] = f * inv_scale[l];
  }
}

pat_status hexport(const void* slabA, int hdtype, const int32_t* kclass, const float* inv_scale,
                   int k0, int nk, int nz, int nt, int sA_row, int ntA, int ksA, float* out,
                   hipStream_t st) {
  if (nk <= 0) return PAT_OK;
  k_hexport<<<nk, 256, 0, st>>>(slabA, hdtype, kclass, inv_scale, k0, nz, nt, sA_row, ntA, ksA,
                                out);
  PAT_LAUNCHED("H export");
  return PAT_OK;
}


// ------------------------------------------------------- normal operator
// Gram blocks of the stored (dequantised) library: G_s[l][l'] =
// sum_n H^_s[l][n] H^_s[l'][n], accumulated in float64 and rounded once.  A^T A
// is block diagonal in the transverse Fourier basis with these blocks, so the
// gradient of the data term, A^T (A z - d) = A^T A z - A^T d (eq. 15), can be
// formed per frequency from the spectrum of z alone.
//
// Blocks of 128 x 128 outputs on and above the diagonal (the rest is their
// mirror image), in 16 x 16 tiles dealt to the four waves: the float64 matrix
// instruction takes both operands in the same lane order (16 depths x 4
// samples), read from one LDS chunk of the slab's rows.  Bound by the matrix
// rate; the vector form it replaced (every block, 4 x 4 outputs per thread)
// took 6.2 ms at 256 x 256 x 128 x 512, 1.17 at 128 x 128 x 96 x 384; now
// 1.6 and 0.24.
constexpr int kGN = 32;    // time samples per LDS chunk
constexpr int kGB = 128;   // depths per block
constexpr int kGS = kGN + 1;
constexpr int kGP = 16;    // tile products per wave, at most (64 tiles, 4 waves)

// 4 consecutive library values of row l from sample n (a multiple of 4; rows
// are padded with zeros to whole 16-byte units)
__device__ __forceinline__ float4 lib_values(const GramArgs& a, int s, int l, int n) {
  if (l >= a.nz || n >= a.sA_row) return make_float4(0.f, 0.f, 0.f, 0.f);
  const size_t o = ((size_t)s * a.nz + l) * a.sA_row + n;
  if (a.hdtype == PAT_H_F32) return *reinterpret_cast<const float4*>(reinterpret_cast<const float*>(a.rowA) + o);
  const ushort4 b = *reinterpret_cast<const ushort4*>(reinterpret_cast<const unsigned short*>(a.rowA) + o);
  const unsigned short u[4] = {b.x, b.y, b.z, b.w};
  float f[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    if (a.hdtype == PAT_H_BF16) {
      f[e] = __uint_as_float((unsigned)u[e] << 16);
    } else {
      _Float16 h;
      __builtin_memcpy(&h, &u[e], 2);
      f[e] = (float)h;
    }
    f[e] *= a.inv_scale[l];
  }
  return make_float4(f[0], f[1], f[2], f[3]);
}

__global__ __launch_bounds__(256, 2) void k_gram(GramArgs a, int nb) {
  __shared__ float hi[kGB * kGS], hj[kGB * kGS];
  const int nblk = nb * (nb + 1) / 2;
  const int s = blockIdx.x / nblk, tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int li = lane & 15, lk = lane >> 4;
  int bi = 0, bj = blockIdx.x - s * nblk;  // block (bi, bj), bi <= bj, rows of nb, nb - 1, ... blocks
  while (bj >= nb - bi) {
    bj -= nb - bi;
    ++bi;
  }
  bj += bi;
  const int i0 = bi * kGB, j0 = bj * kGB;
  const bool diag = bi == bj;
  const int nti = (min(a.nz - i0, kGB) + 15) >> 4, ntj = (min(a.nz - j0, kGB) + 15) >> 4;
  // tile products p = w, w + 4, ... of this wave: (ti, tj), ti <= tj on the diagonal
  const int np = diag ? nti * (nti + 1) / 2 : nti * ntj;
  int ti[kGP], tj[kGP];
#pragma unroll
  for (int m = 0; m < kGP; ++m) {
    int p = w + 4 * m;
    ti[m] = tj[m] = 0;
    if (p < np) {
      if (diag) {
        while (p >= nti - ti[m]) {
          p -= nti - ti[m];
          ++ti[m];
        }
        tj[m] = ti[m] + p;
      } else {
        ti[m] = p / ntj;
        tj[m] = p - ti[m] * ntj;
      }
    }
    ti[m] = __builtin_amdgcn_readfirstlane(ti[m]);
    tj[m] = __builtin_amdgcn_readfirstlane(tj[m]);
  }
  v4d acc[kGP];
#pragma unroll
  for (int m = 0; m < kGP; ++m) acc[m] = v4d{0.0, 0.0, 0.0, 0.0};
  const float* hb = diag ? hi : hj;
  const int lr = tid >> 3, lc = 4 * (tid & 7);  // rows lr + 32 r, samples lc .. lc + 3 of a chunk
  float4 vi[4], vj[4];
  auto fetch = [&](int n0) {
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      vi[r] = lib_values(a, s, i0 + lr + 32 * r, n0 + lc);
      if (!diag) vj[r] = lib_values(a, s, j0 + lr + 32 * r, n0 + lc);
    }
  };
  fetch(0);
  for (int n0 = 0; n0 < a.nt; n0 += kGN) {
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      float* d = hi + (lr + 32 * r) * kGS + lc;
      d[0] = vi[r].x;
      d[1] = vi[r].y;
      d[2] = vi[r].z;
      d[3] = vi[r].w;
      if (!diag) {
        float* e = hj + (lr + 32 * r) * kGS + lc;
        e[0] = vj[r].x;
        e[1] = vj[r].y;
        e[2] = vj[r].z;
        e[3] = vj[r].w;
      }
    }
    __syncthreads();
    if (n0 + kGN < a.nt) fetch(n0 + kGN);  // travels while this chunk is multiplied
    for (int k = 0; k < kGN / 4; ++k) {
      const int o = li * kGS + 4 * k + lk;
#pragma unroll
      for (int m = 0; m < kGP; ++m) {
        if (w + 4 * m >= np) break;
        const double x = hi[ti[m] * 16 * kGS + o], y = hb[tj[m] * 16 * kGS + o];
        acc[m] = __builtin_amdgcn_mfma_f64_16x16x4f64(x, y, acc[m], 0, 0, 0);
      }
    }
  }
  float* g = a.gram + (size_t)s * a.nz * a.sG_row;
#pragma unroll
  for (int m = 0; m < kGP; ++m) {
    if (w + 4 * m >= np) break;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int i = i0 + 16 * ti[m] + lk + 4 * r, j = j0 + 16 * tj[m] + li;
      if (i >= a.nz || j >= a.nz) continue;
      const float v = (float)acc[m][r];
      g[(size_t)i * a.sG_row + j] = v;
      if (!diag || ti[m] != tj[m]) g[(size_t)j * a.sG_row + i] = v;
    }
  }
}

pat_status gram_build(const GramArgs& a, hipStream_t st) {
  if (a.nslab == 0) return PAT_OK;
  const int nb = (a.nz + kGB - 1) / kGB;
  const long long grid = (long long)a.nslab * (nb * (nb + 1) / 2);
  if (grid > 0x7fffffffLL) return fail(PAT_EUNSUPPORTED, "Gram blocks: grid too large");
  k_gram<<<dim3((unsigned)grid), 256, 0, st>>>(a, nb);
  PAT_LAUNCHED("Gram blocks");
  return PAT_OK;
}

}  // namespace pat
