// Gram products from half of every block (G is symmetric).
//
// FISTA and the power iteration multiply each class's nz x nz Gram block with
// the spectra of its member frequencies once per step; for one object reading
// the blocks is the cost.  A wave takes a whole group (up to 8 members: 16
// columns of real and imaginary parts) and reads, of each 16 rows, the columns
// from the diagonal tile on: tile (I, J) serves y_I += G_IJ x_J as it is and,
// off the diagonal, y_J += G_IJ^T x_I.  The matrix instruction
// v_mfma_f32_16x16x4_f32 wants the two uses in different lanes (row lane % 16,
// or column lane % 16), so tiles go through 2.3 KB of LDS that only their wave
// uses (no barrier: a wave's LDS accesses are in order).  x and y of all rows
// stay in registers: in both uses lane group q = lane / 16 holds rows 4 q ..
// 4 q + 3 of a tile, which is also how the instruction leaves its sums.
//
// Loads take 16 rows x 32 columns, whole 128-byte lines: loaded as 16 x 16
// tiles, in pieces of 64 bytes, half the bytes took as long as all of them
// (256 x 256 x 128: 79 us against 85 for the whole blocks and 66 with whole
// lines, 5.0 TB/s; loading each tile a second time from the cache instead of
// turning it, 86).  Three to seven units in flight made no difference.
//
// A step of FISTA, whole blocks and this: 256 x 256 x 128, 158 us, now 142;
// 256 x 256 x 30, 62 and 46; 128 x 128 x 96, 43.2 and 40.8; 256 x 192 x 96 (two
// members), 143 and 118.  Of 4 objects: 256 x 256 x 32, 157 and 106; 128 x 128 x
// 96, 96.8 and 88.5 (there the general kernel reads a value once for all
// pairs: 4 times fewer loads, but one wave per tile and half the workgroups).
//
// Each tile's four instructions form a sum of 16 products of their own, added
// to y once: no longer a chain of roundings than the general kernel's.
#include "contract_slab.hpp"
#include "pat_internal.hpp"

namespace pat {

// orders a wave's own LDS accesses (no other wave touches them)
__device__ __forceinline__ void wave_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

typedef float v4f8 __attribute__((ext_vector_type(4), aligned(8)));  // two complex values, 8-byte aligned

constexpr int kUnits = 4;  // units in flight

// T tiles of 16 rows; NT: non-temporal loads; WT: lines written through
template <int T, bool NT, bool WT>
__global__ __launch_bounds__(256, 3) void k_contract_sym(ContractArgs a, int per_xcd, int pgroups) {
  constexpr int T2 = (T + 1) / 2;  // units of 16 rows x 32 columns (whole lines) from the diagonal on
  constexpr int N = T2 * (T2 + 1) - T % 2;
  constexpr int D = kUnits < N ? kUnits : N;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // units (group, 8 pairs) in order, one contiguous range per XCD (workgroups
  // go round-robin): the units of a group read its block at about the same time
  const int in_range = (blockIdx.x >> 3) * 4 + w, u = (blockIdx.x & 7) * per_xcd + in_range;
  if (in_range >= per_xcd || u >= a.ngroup * pgroups) return;
  const int t = u / pgroups, pg0 = 8 * (u - t * pgroups);
  const int4 grp = a.groups[t];  // first spectrum row, members, slab
  const int np = grp.y * a.B;    // pairs: members times objects
  if (pg0 >= np) return;
  const int lane = threadIdx.x & 63, q = lane >> 4, c = lane & 15;
  const int nz = a.ni, sr = a.s_row;
  constexpr int last = 16 * (T - 1);
  // byte offsets of a lane within a unit (8 lanes take the 128 bytes of a row,
  // a unit is two loads of 8 rows); the last rows and columns stop at the
  // block's end (values read there once more meet zeros of x or are not stored)
  const int lr = lane >> 3, lc = 4 * (lane & 7), lastc = 32 * (T2 - 1);
  const int ce = min(lastc + lc, sr - 4) - lastc;
  const int r0 = min(last + lr, nz - 1) - last, r1 = min(last + 8 + lr, nz - 1) - last;
  const unsigned o_f = (lr * sr + lc) * 4, o_c = (lr * sr + ce) * 4;
  const unsigned o_r0 = (r0 * sr + ce) * 4, o_r1 = (r1 * sr + ce) * 4;
  const char* hb = reinterpret_cast<const char*>(reinterpret_cast<const float*>(a.slab) + (size_t)grp.z * a.slab_elems);
  auto here = [](unsigned o) {  // a 32-bit lane offset beside a scalar base
    asm("" : "+v"(o));
    return o;
  };
  struct Unit {
    v4f h[2];
  };
  Unit buf[D];
  auto load = [&](Unit& b, int I, int P) {
    const char* p = hb + (size_t)(16 * I * sr + 32 * P) * 4;
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      const bool lastrow = I == T - 1;  // then P is the last pair as well
      const char* ph = lastrow ? p : p + (size_t)8 * h * sr * 4;
      const unsigned o = lastrow ? (h ? o_r1 : o_r0) : P < T2 - 1 ? o_f : o_c;
      const v4f* pd = reinterpret_cast<const v4f*>(ph + here(o));
      b.h[h] = NT ? __builtin_nontemporal_load(pd) : *pd;
    }
  };
  __shared__ float turn[4][16 * 36];  // rows 144 bytes apart: no bank conflicts in any of the accesses
  float* wr = turn[w] + lr * 36 + lc;
  const float* rd = turn[w] + c * 36 + 4 * q;
  const float* rt = turn[w] + 4 * q * 36 + c;
  // x: lane holds rows 4 q + e of tile J for column c (pair pg0 + c / 2, part c % 2)
  const int pr = min(pg0 + (c >> 1), np - 1), mem = a.B == 1 ? pr : pr / a.B, ob = pr - mem * a.B;
  const float* xrow =
      reinterpret_cast<const float*>(a.in + (size_t)(grp.x + mem) * a.in_rs + (size_t)ob * nz + 4 * q) + (c & 1);
  v4f x[T], y[T];
#pragma unroll
  for (int J = 0; J < T; ++J) {
    y[J] = v4f(0.f);
#pragma unroll
    for (int e = 0; e < 4; ++e) x[J][e] = xrow[2 * (16 * J + e)];
  }
  int li = 0, lj = 0;  // unit to load next
#pragma unroll
  for (int n = 0; n < D - 1; ++n) {
    load(buf[n], li, lj);
    if (++lj == T2) lj = ++li / 2;
  }
  __builtin_amdgcn_sched_barrier(0);
  const bool im = c & 1;
#pragma unroll
  for (int e = 0; e < 4; ++e)
    if (last + 4 * q + e >= nz) x[T - 1][e] = 0.f;
  auto add = [](v4f& sum, const v4f& part) {
    sum += part;
    asm("" : "+v"(sum));  // here and not at the end, where all parts would have to be kept
  };
  int I = 0, P = 0;
#pragma unroll
  for (int n = 0; n < N; ++n) {
    if (n + D - 1 < N) {
      load(buf[(n + D - 1) % D], li, lj);
      if (++lj == T2) lj = ++li / 2;
    }
    __builtin_amdgcn_sched_barrier(0);
    *reinterpret_cast<v4f*>(wr) = buf[n % D].h[0];
    *reinterpret_cast<v4f*>(wr + 8 * 36) = buf[n % D].h[1];
    wave_order();
    v4f d[2], t[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int J = 2 * P + k;
      if (J < I || J >= T) continue;
      d[k] = *reinterpret_cast<const v4f*>(rd + 16 * k);
#pragma unroll
      for (int e = 0; e < 4; ++e)
        if (J > I) t[k][e] = rt[36 * e + 16 * k];
    }
    wave_order();
    v4f pd[2] = {v4f(0.f), v4f(0.f)}, pt[2] = {v4f(0.f), v4f(0.f)};
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int k = 0; k < 2; ++k) {
        const int J = 2 * P + k;
        if (J < I || J >= T) continue;
        pd[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(d[k][e], x[J][e], pd[k], 0, 0, 0);
        if (J > I) pt[k] = __builtin_amdgcn_mfma_f32_16x16x4f32(t[k][e], x[I][e], pt[k], 0, 0, 0);
      }
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int J = 2 * P + k;
      if (J < I || J >= T) continue;
      add(y[I], pd[k]);
      if (J > I) add(y[J], pt[k]);
    }
    if (++P == T2) P = ++I / 2;
    __builtin_amdgcn_sched_barrier(0);
  }
  // rows 16 I + 4 q + r of column c: the lanes of a member's real and imaginary
  // parts exchange two values, then each stores two complex values; four lane
  // groups complete the 128 bytes of a tile in the member's row
  const size_t o0 = (size_t)(grp.x + mem) * a.out_rs + (size_t)ob * nz + 4 * q + 2 * (c & 1);
  const bool live = pg0 + (c >> 1) < np;
  v4f sub[T];
#pragma unroll
  for (int I = 0; I < T; ++I) {
    const int left = live ? nz - (16 * I + 4 * q + 2 * (c & 1)) : 0;
    sub[I] = v4f(0.f);
    if (a.out_sub && left >= 2) sub[I] = *reinterpret_cast<const v4f8*>(a.out_sub + o0 + 16 * I);
    if (a.out_sub && left == 1) {
      const float2 s1 = a.out_sub[o0 + 16 * I];
      sub[I][0] = s1.x;
      sub[I][1] = s1.y;
    }
  }
  const auto orow = __builtin_amdgcn_make_buffer_rsrc(a.out + (size_t)grp.x * a.out_rs, (short)0, 8 * a.out_rs * 8, 0x00020000);
#pragma unroll
  for (int I = 0; I < T; ++I) {
    const int left = live ? nz - (16 * I + 4 * q + 2 * (c & 1)) : 0;
    const float r0 = __shfl_xor(im ? y[I][0] : y[I][2], 1), r1 = __shfl_xor(im ? y[I][1] : y[I][3], 1);
    v4f v = im ? v4f{r0, y[I][2], r1, y[I][3]} : v4f{y[I][0], r0, y[I][1], r1};
    v -= sub[I];
    if (WT) {
      if (left > 0) {  // nz % 16 == 0: whole lines, written through
        v4u bits;
        __builtin_memcpy(&bits, &v, 16);
        __builtin_amdgcn_raw_buffer_store_b128(
            bits, orow, (int)((unsigned)(o0 + 16 * I - (size_t)grp.x * a.out_rs) * 8u), 0, 16);  // sc1
      }
    } else if (left >= 2) {
      *reinterpret_cast<v4f8*>(a.out + o0 + 16 * I) = v;
    } else if (left == 1) {
      a.out[o0 + 16 * I] = make_float2(v[0], v[1]);
    }
  }
}

template <int T>
static void launch_sym(const ContractArgs& a, bool nt, hipStream_t st) {
  const int pgroups = (a.members * a.B + 7) / 8;
  const int per_xcd = (a.ngroup * pgroups + 7) / 8;
  const int grid = 8 * ((per_xcd + 3) / 4);
  const bool wt = a.nj % 16 == 0;
  auto go = [&](auto kernel) { kernel<<<grid, 256, 0, st>>>(a, per_xcd, pgroups); };
  if (nt && wt) return go(k_contract_sym<T, true, true>);
  if (nt) return go(k_contract_sym<T, true, false>);
  if (wt) return go(k_contract_sym<T, false, true>);
  go(k_contract_sym<T, false, false>);
}

pat_status contract_sym(const ContractArgs& a, bool nt, hipStream_t st) {
  switch ((a.ni + 15) / 16) {
    case 1: launch_sym<1>(a, nt, st); break;
    case 2: launch_sym<2>(a, nt, st); break;
    case 3: launch_sym<3>(a, nt, st); break;
    case 4: launch_sym<4>(a, nt, st); break;
    case 5: launch_sym<5>(a, nt, st); break;
    case 6: launch_sym<6>(a, nt, st); break;
    case 7: launch_sym<7>(a, nt, st); break;
    case 8: launch_sym<8>(a, nt, st); break;
    default: return fail(PAT_EUNSUPPORTED, "symmetric product: more than 128 rows");
  }
  PAT_LAUNCHED("symmetric contraction");
  return PAT_OK;
}

}  // namespace pat
