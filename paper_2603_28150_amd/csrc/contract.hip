// Per-frequency multiply-accumulate of the operator (step (ii) of Sec. 3.2).
//
// For every transverse frequency k:
//   A   :  D^[k, n] = sum_l H^[k, l, n] X^[k, l]          (sum over depth)
//   A^T :  G^[k, l] = sum_n conj(H^[k, l, n]) R^[k, n]    (sum over time)
// H^ is real and identical for all frequencies of one symmetry class, so the
// library keeps one slab per class in two layouts, [l][n] for A and [n][l] for
// A^T.  Both products then have the same shape: the summed index i runs over
// slab rows, the kept index j runs along a row, and the slab serves every
// (member frequency, object) pair of its work item.  For one object streaming
// the slab is the whole cost (>95 % of the bytes an apply moves).
//
// The product runs on the float32 matrix instruction v_mfma_f32_16x16x4_f32:
// its 16 rows are the real and imaginary parts of 8 pairs, its 16 columns are
// outputs, 4 slab rows are summed per instruction, all in float32.  A wave owns
// a tile of 16 VEC outputs (VEC values per load, 16 bytes of them as a rule) and streams its slab
// rows straight into the operand registers, VEC instructions per load: no
// barrier and no sum across lanes, so that a wave only ever waits for its own
// loads, and no vector arithmetic beside the matrix instructions (a load costs
// one issue slot: scalar block base plus a fixed lane offset).
//
// Bound by HBM at full size, by latency below.  The vector kernel this replaced
// (one workgroup per slab, spectra in LDS, an LDS tree over the row groups), per
// launch of A / A^T under the profiler, and this: 32 x 32 x 16 x 64, 9.9 / 12.7 us,
// now 4.3 / 4.6 (the tree was six levels deep); 128 x 128 x 96 x 384, 55 / 59, now
// 55 / 52; 202 x 202 x 37 x 256 on 432 x 432, 171 / 243, now 146 / 194; 256 x 256 x
// 128 x 512, 308 / 307, now 308 / 311 (5.6 TB/s of slabs and spectra); with bf16
// slabs 186 / 204, now 182 / 181 (groups of 8 members read a slab once that two
// items of 4 read twice).  contract() says which products go to the half-block
// kernel (contract_sym.hip) and the vector units (contract_pair.hip) instead.
#include <algorithm>
#include <type_traits>

#include "contract_slab.hpp"
#include "pat_internal.hpp"

namespace pat {

typedef float v4f8 __attribute__((ext_vector_type(4), aligned(8)));  // two complex values, 8-byte aligned

// orders a wave's own LDS accesses (no other wave touches them)
__device__ __forceinline__ void wave_sync() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront", "local");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront", "local");
}

// workgroup barrier that orders LDS accesses only (global loads stay in flight)
__device__ __forceinline__ void lds_barrier() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}
// bytes of a staged pair: the rows of four lane groups and eight pairs that a
// wave reads together fall into different banks
__host__ __device__ __forceinline__ int xl_stride(int ni) { return (ni * 8 + 255) / 256 * 256 + 64; }

// Rows are taken in blocks of 8: lane group c = lane / 16 holds rows 2c and
// 2c + 1 of a block (two 16-byte slab loads), so that one 16-byte load brings
// both rows' spectrum values of a pair.  Two register buffers of U blocks
// keep up to 4 U slab loads of a wave in flight.

// One wave: outputs [tile * 16 VEC, ...) of the CT * 8 pairs from pg0 on,
// summed over the wave's share (kpart of KP) of the row blocks; the shares
// are added in a fixed order by share 0, which stores the result.  np: pairs
// of the group (members times objects).
//
// Short rows (at most half or a quarter of a tile) with few pairs leave lanes
// and instruction rows idle: then S = 2 or 4 sets of 16/S lanes take different
// row blocks of the slab, set i's pairs in the instruction rows 16 i/S .., and
// only the diagonal (set, set) part of the product is used and summed.
//
// XL: the pairs' spectra go through LDS first, whole runs of a row per load
// (where they are long and come from memory, reading them piecewise between
// the slab loads costs more than the barrier).  NT: non-temporal slab loads.
// WT: output lines are written through.
template <typename HT, int V, int CT, int U, bool NT, bool WT, bool XL>
__device__ __forceinline__ void stream_tile(const ContractArgs& a, int row0, int slab_id, int tile, int kpart, int KP,
                                            int pg0, int np, float* red) {
  typedef Slab<HT, V> SL;
  typedef typename SL::raw_t raw_t;
  constexpr int VEC = V;
  constexpr unsigned ESZ = sizeof(HT);
  constexpr bool SCALED = ESZ == 2;  // 16-bit libraries have scales
  const int lane = threadIdx.x & 63;
  const int c = lane >> 4, l16 = lane & 15;
  int ls = 0;  // log2 S
  if (CT == 1 && !XL && a.nj <= 8 * VEC) ls = (a.nj <= 4 * VEC && np - pg0 <= 2) ? 2 : np - pg0 <= 4 ? 1 : 0;
  const int pmask = (8 >> ls) - 1;  // pairs of a set of lanes
  const int set = l16 >> (4 - ls);
  const int lb = 3 + ls;         // log2 rows per block
  const int nfull = a.ni >> lb;  // whole blocks; a partial one is the last share's
  const int b0 = nfull * kpart / KP, b1 = nfull * (kpart + 1) / KP;

  // Addresses: a wave-uniform base that advances by blocks (scalar
  // arithmetic) plus a fixed 32-bit byte offset per lane, so that a load costs
  // no vector instruction besides itself (the launcher checks the range).
  constexpr int tn = 16 * VEC;  // outputs of a tile
  const int n = tile * tn + VEC * (l16 & ((16 >> ls) - 1));  // first output of this lane
  const unsigned col = min(n, a.s_row - VEC);  // clamped: always a valid address
  const char* hb = reinterpret_cast<const char*>(reinterpret_cast<const HT*>(a.slab) + (size_t)slab_id * a.slab_elems);
  const unsigned rl = 8 * set + 2 * c;  // this lane's first row in a block
  const unsigned hv[2] = {(rl * a.s_row + col) * ESZ, ((rl + 1) * a.s_row + col) * ESZ};
  const unsigned hstep = (unsigned)(a.s_row << lb) * ESZ;
  const int xstep = 8 << lb;
  // spectrum rows of this lane's pairs (a pair past the end reads pair pg0's)
  const char* xb = reinterpret_cast<const char*>(a.in + (size_t)row0 * a.in_rs);
  unsigned xv[CT];
#pragma unroll
  for (int m = 0; m < CT; ++m) {
    const int pr = pg0 + 8 * m + ((l16 >> 1) & pmask);
    const int p = pr < np ? pr : pg0;
    const int g = a.B == 1 ? p : p / a.B, b = p - g * a.B;
    xv[m] = (unsigned)(g * a.in_rs + b * a.ni) * 8u + rl * 8u;
  }
  const bool im = lane & 1;
  unsigned xl[XL ? CT : 1];  // the same in LDS
  const int xstride = xl_stride(a.ni);  // bytes per pair
  if constexpr (XL) {
#pragma unroll
    for (int m = 0; m < CT; ++m) {
      const int pl = 8 * m + ((l16 >> 1) & pmask);
      xl[m] = (pg0 + pl < np ? pl : 0) * xstride + rl * 8;
    }
  }

  struct Buf {
    raw_t h[U][2];
    v4f x[U][CT];
    float2 sc[SCALED ? U : 1];
  };
  // keeps a 32-bit offset next to its load (widened in advance, it would take
  // two registers and a 64-bit addition per load)
  auto here = [](unsigned o) {
    asm("" : "+v"(o));
    return o;
  };
  auto slab_load = [&](const char* q) {
    const raw_t* p = reinterpret_cast<const raw_t*>(q);
    return NT ? __builtin_nontemporal_load(p) : *p;
  };
  // Loads of row blocks b .. b + U - 1, unconditional (past the last whole
  // block it is read again and not used) so that no branch hides them from
  // the wait counter.
  auto load = [&](Buf& o, int b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int bb = min(b + u, nfull - 1);
      const char* ph = hb + (unsigned)bb * hstep;
      const char* px = xb + (size_t)bb * xstep;
#pragma unroll
      for (int s = 0; s < 2; ++s) o.h[u][s] = slab_load(ph + here(hv[s]));
      if constexpr (!XL) {
#pragma unroll
        for (int m = 0; m < CT; ++m) o.x[u][m] = *reinterpret_cast<const v4f8*>(px + here(xv[m]));
      }
      if constexpr (SCALED)
        o.sc[u] = a.in_scale ? *reinterpret_cast<const float2*>(a.in_scale + ((size_t)bb << lb) + rl)
                             : make_float2(1.f, 1.f);
    }
    __builtin_amdgcn_sched_barrier(0);  // the products that follow stay behind these loads
  };
  // spectrum values of row blocks b .. b + U - 1 from LDS
  auto load_x = [&](Buf& o, int b) {
    if constexpr (XL) {
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int m = 0; m < CT; ++m)
          o.x[u][m] = *reinterpret_cast<const v4f*>(reinterpret_cast<const char*>(red) + xl[m] + min(b + u, nfull - 1) * xstep);
    }
  };
  // The matrix instruction adds its four products to the accumulator one after
  // the other: sums of 8 or 16 rows are kept apart (part) and added to the
  // total, which shortens the chain of roundings from the share's length to
  // that of a group plus the number of groups.
  v4f acc[CT][VEC], part[CT][VEC];
#pragma unroll
  for (int m = 0; m < CT; ++m)
#pragma unroll
    for (int v = 0; v < VEC; ++v) acc[m][v] = part[m][v] = v4f(0.f);
  auto flush = [&]() {
#pragma unroll
    for (int m = 0; m < CT; ++m)
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        acc[m][v] += part[m][v];
        part[m][v] = v4f(0.f);
      }
  };
  auto mma_block = [&](const raw_t (&h)[2], const v4f (&x)[CT], float2 sc) {
#pragma unroll
    for (int s = 0; s < 2; ++s) {
      float xs[CT];
#pragma unroll
      for (int m = 0; m < CT; ++m) {
        xs[m] = im ? x[m][2 * s + 1] : x[m][2 * s];
        if constexpr (SCALED) xs[m] *= s ? sc.y : sc.x;
      }
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const float hval = SL::get(h[s], v);
#pragma unroll
        for (int m = 0; m < CT; ++m)
          part[m][v] = __builtin_amdgcn_mfma_f32_16x16x4f32(xs[m], hval, part[m][v], 0, 0, 0);
      }
    }
  };
  auto mma = [&](const Buf& o, int b) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      if (b + u >= b1) break;
      mma_block(o.h[u], o.x[u], o.sc[SCALED ? u : 0]);
      if (u % 2 == 1 || (ESZ == 4 && CT == 1 && U == 2)) flush();
    }
    __builtin_amdgcn_sched_barrier(0);
  };

  // the rows after the last whole block: loaded first (clamped into the slab
  // and, in pairs, into the spectrum row), multiplied last
  const bool tail = (nfull << lb) < a.ni && kpart == KP - 1;
  const int r0 = (nfull << lb) + rl;
  raw_t th[2];
  v4f tx[CT];
  float2 tsc = make_float2(1.f, 1.f);
  if (tail) {
    const int x0 = min(r0, (a.ni - 1) & ~1);
#pragma unroll
    for (int s = 0; s < 2; ++s)
      th[s] = slab_load(hb + (unsigned)(min(r0 + s, a.ni - 1) * a.s_row + col) * ESZ);
#pragma unroll
    for (int m = 0; m < CT; ++m)
      tx[m] = *reinterpret_cast<const v4f8*>(xb + (xv[m] - rl * 8u) + (unsigned)x0 * 8u);
    if (SCALED && a.in_scale)
      tsc = make_float2(a.in_scale[min(r0, a.ni - 1)], a.in_scale[min(r0 + 1, a.ni - 1)]);
  }
  Buf ba, bb;
  if (b0 < b1) load(ba, b0);
  if constexpr (XL) {
    // the pairs' spectra into LDS, whole runs of a row per wave instruction
    constexpr int kRun = 4;
    const int nw = blockDim.x >> 6, wv = threadIdx.x >> 6, h = (a.ni + 1) >> 1;
    const int npl = min(8 * CT, np - pg0);
    for (int p = wv; p < npl; p += nw) {
      const int pr = pg0 + p;
      const int g = a.B == 1 ? pr : pr / a.B, ob = pr - g * a.B;
      const char* src = xb + (size_t)(g * a.in_rs + ob * a.ni) * 8;
      char* dst = reinterpret_cast<char*>(red) + p * xstride;
      for (int q0 = lane; q0 < h; q0 += 64 * kRun) {
        v4f v[kRun];
#pragma unroll
        for (int r = 0; r < kRun; ++r) v[r] = *reinterpret_cast<const v4f8*>(src + min(q0 + 64 * r, h - 1) * 16);
#pragma unroll
        for (int r = 0; r < kRun; ++r)
          if (q0 + 64 * r < h) *reinterpret_cast<v4f*>(dst + (q0 + 64 * r) * 16) = v[r];
      }
    }
    lds_barrier();
  }
  if (b0 < b1) {
    // the loads of the next blocks go out before the products of the current ones
    int b = b0;
    load_x(ba, b);
    for (; b + 2 * U < b1; b += 2 * U) {
      load(bb, b + U);
      load_x(bb, b + U);
      mma(ba, b);
      load(ba, b + 2 * U);
      load_x(ba, b + 2 * U);
      mma(bb, b + U);
      if (U == 1) flush();
    }
    if (b + U < b1) {
      load(bb, b + U);
      load_x(bb, b + U);
      mma(ba, b);
      mma(bb, b + U);
    } else {
      mma(ba, b);
    }
  }
  if (tail) {
#pragma unroll
    for (int s = 0; s < 2; ++s)
      if (r0 + s >= a.ni) {  // past the end: zeros
        th[s] = raw_t(0);
#pragma unroll
        for (int m = 0; m < CT; ++m) tx[m][2 * s] = tx[m][2 * s + 1] = 0.f;
      }
    if (U > 1) flush();
    mma_block(th, tx, tsc);
  }
  flush();

  const int w = threadIdx.x >> 6;
  if (XL) lds_barrier();  // every wave is done with the staged spectra
  if (KP > 1) {  // shares 1 .. KP-1 pass their sums through LDS (workgroup-uniform)
    constexpr int NA = CT * VEC * 4;
    float* mine = red + (size_t)w * NA * 64 + lane;
    if (kpart > 0) {
#pragma unroll
      for (int m = 0; m < CT; ++m)
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int r = 0; r < 4; ++r) mine[((m * VEC + v) * 4 + r) * 64] = acc[m][v][r];
    }
    lds_barrier();
    if (kpart > 0) return;
    for (int p = 1; p < KP; ++p) {
#pragma unroll
      for (int m = 0; m < CT; ++m)
#pragma unroll
        for (int v = 0; v < VEC; ++v)
#pragma unroll
          for (int r = 0; r < 4; ++r)
            acc[m][v][r] += mine[(size_t)p * NA * 64 + ((m * VEC + v) * 4 + r) * 64];
    }
  }

  // Accumulator row r of lane group c holds a part of pair 2c + r/2 (re, im), at output n + v for instruction v.  The tile goes
  // through the wave's own part of LDS so that each store instruction writes
  // whole runs of a spectrum row instead of half of every 32 bytes.
  constexpr int NU = VEC;                              // 16-byte units per lane
  constexpr int lu = VEC == 8 ? 6 : VEC == 4 ? 5 : 4;  // log2 units of a row (tn / 2)
  float* tr = red + (size_t)w * (KP > 1 ? CT : 1) * VEC * 256;
  const size_t obase = (size_t)row0 * a.out_rs;
  const auto orow = __builtin_amdgcn_make_buffer_rsrc(a.out + obase, (short)0, 8 * a.out_rs * 8, 0x00020000);
  float osc[VEC];
#pragma unroll
  for (int v = 0; v < VEC; ++v) osc[v] = a.out_scale ? a.out_scale[min(n + v, a.nj - 1)] : 1.f;
#pragma unroll
  for (int m = 0; m < CT; ++m) {
    if (pg0 + 8 * m >= np) break;
    if ((2 * c) >> (3 - ls) == set) {  // S > 1: only the set's own pairs
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int v = 0; v < VEC; v += 2)
          *reinterpret_cast<v4f*>(tr + (2 * c + e) * 2 * tn + 2 * (n - tile * tn + v)) =
              v4f{acc[m][v][2 * e] * osc[v], acc[m][v][2 * e + 1] * osc[v],
                  acc[m][v + 1][2 * e] * osc[v + 1], acc[m][v + 1][2 * e + 1] * osc[v + 1]};
    }
    wave_sync();
    v4f d[NU];
    size_t off[NU];
    int left[NU];  // outputs of the unit to store: 2, 1 or (<= 0) none
#pragma unroll
    for (int j = 0; j < NU; ++j) {
      const int idx = j * 64 + lane, q = idx & ((1 << lu) - 1);
      const int pr = pg0 + 8 * m + (idx >> lu);
      const int g = a.B == 1 ? pr : pr / a.B, ob = pr - g * a.B;
      const int nq = tile * tn + 2 * q;
      off[j] = (size_t)(row0 + g) * a.out_rs + (size_t)ob * a.nj + nq;
      left[j] = pr < np ? a.nj - nq : 0;
      d[j] = v4f(0.f);
      if (left[j] > 0) {
        d[j] = *reinterpret_cast<const v4f*>(tr + 4 * idx);
        for (int k = 1; k < (1 << ls); ++k) d[j] += *reinterpret_cast<const v4f*>(tr + 4 * idx + k * (8 >> ls) * 2 * tn);
      }
    }
    if (a.out_sub) {
      v4f sub[NU];
#pragma unroll
      for (int j = 0; j < NU; ++j) {
        sub[j] = v4f(0.f);
        if (left[j] >= 2) {
          sub[j] = *reinterpret_cast<const v4f8*>(a.out_sub + off[j]);
        } else if (left[j] == 1) {
          const float2 w1 = a.out_sub[off[j]];
          sub[j][0] = w1.x;
          sub[j][1] = w1.y;
        }
      }
#pragma unroll
      for (int j = 0; j < NU; ++j) d[j] -= sub[j];
    }
#pragma unroll
    for (int j = 0; j < NU; ++j) {
      if (WT) {
        if (left[j] > 0) {
          v4u bits;
          __builtin_memcpy(&bits, &d[j], 16);
          __builtin_amdgcn_raw_buffer_store_b128(bits, orow, (int)((unsigned)(off[j] - obase) * 8u), 0, 16);  // sc1
        }
      } else if (left[j] >= 2) {
        __builtin_nontemporal_store((v4f8)d[j], reinterpret_cast<v4f8*>(a.out + off[j]));
      } else if (left[j] == 1) {
        a.out[off[j]] = make_float2(d[j][0], d[j][1]);
      }
    }
    wave_sync();
  }
}

// Slabs that come round again before this much else has been read stay in the
// memory-side cache (256 MB) with plain loads; a larger working set streams,
// and non-temporal loads stream faster (7.1 against 6.2 TB/s on a plain read
// of 1.55 GB).  One A + one A^T: 128 x 128 x 64 x 256 (210 MB in both layouts)
// 108 us plain, 111 non-temporal; 128 x 128 x 96 x 384 (470 MB) 187 and 174.
// Long float32 products of rows that do not start at whole 64-byte pieces take
// plain loads at any size: neighbouring tiles share a line there, and a line
// loaded as non-temporal is often gone from the L2 when the second tile asks for
// it (1.2 times the slab's bytes fetched at 600 values per row, 1.0 plain).  One A +
// one A^T (medians over ten placements in memory), non-temporal and plain: 128 x
// 128 x 130 x 402, 258 and 247 us; 144 x 144 x 200 x 200, 240 and 231; 128 x 128 x 67 x
// 1643, 571 and 526; short sums and short rows lose, as the plain loads push the
// spectra out of that cache: 128 x 128 x 33 x 700, 187 and 192; 192 x 192 x 100 x 229,
// 260 and 264 with A^T plain; 384 x 384 x 100 x 101, 512 and 522.  16-bit slabs, half as
// long, lose throughout (144 x 144 x 217 x 333, 254 and 266).
constexpr long long kCacheBytes = 256LL << 20;

// Rows from which the spectra are staged in LDS (XL; float32 slabs: with 16-bit
// ones, busier on the matrix cores, the barrier costs more than it saves: one A +
// one A^T at 256 x 256 x 128 x 208, bf16, 363 us staged and 342 direct; 192 x 192 x 96 x
// 384, 282 and 275).  Shorter products gain
// nothing from it (A^T of 128 x 128 x 64 x 256: 22.5 us direct, 25.4 staged);
// longer ones 1 to 4 % (one A + one A^T at 256 x 256 x 128 x 512: 898 us staged and
// 908; contractions at 96 x 96 x 320 x 512, 241 and 244; a step at 64 x 64 x 512, 115
// and 120).  Rows of less than a tile are short runs of a slab with as many
// spectrum bytes: staged, 202 x 202 x 37 x 256 (linear) took 640 instead of
// 612 us.
constexpr int kXlRows = 192;
constexpr size_t kMaxLds = 160 * 1024;  // of a CU

// Workgroup = TW tiles x KP row shares of one (group, tile group, pair group).
// Workgroups are dealt to the eight XCDs round-robin by index, so the units,
// in group order, are cut into eight contiguous ranges, one per XCD, each taken
// in order: the pair groups of a group, and the groups a large class is split
// into (adjacent, reading the same slab), run on one XCD at about the same
// time, and every read of a slab after the first comes from that XCD's L2
// instead of HBM.
//
// LD: how slabs are loaded.  A slab that two or three groups read: non-temporal,
// most of its lines are gone before the next group asks for them.  A in float32
// takes plain loads there, kStreamOnce (read at 256 x 256 x 128 x 512: 1.632 GB, now
// 1.588; one A + one A^T 904 us, now 901; 128 x 128 x 192 x 224, 191 and 186).  Short
// sums, A^T's result and 16-bit slabs, at more spectra per slab byte, lose as
// much in the transforms, whose lines the slabs then displace (256 x 256 x 32 x
// 512, 436 and 438; A^T, 906 and 914; 202 x 202 x 37 x 256 linear, A^T 179 and 180).
enum Loads { kPlain, kStream, kStreamOnce };
template <typename HT, int V, int CT, int U, int LD, bool WT, bool XL>
__global__ __launch_bounds__((XL ? 512 : 256), (CT > 1 ? 2 : 3)) void k_contract(ContractArgs a, int TW, int KP, int tgroups,
                                                                     int pgroups, int ntile) {
  extern __shared__ float red[];
  constexpr bool NT = LD != kPlain;
  const int units = a.ngroup * tgroups * pgroups;
  const int per_xcd = (units + 7) >> 3;
  const int u = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (u >= units) return;  // whole workgroup: padding of the grid
  const int pg = u % pgroups, tg = (u / pgroups) % tgroups, t = u / (pgroups * tgroups);
  const int4 grp = a.groups[t];  // first spectrum row, members, slab, whether other groups read it
  const int np = grp.y * a.B, pg0 = pg * 8 * CT;
  if (pg0 >= np) return;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int kpart = w % KP, tile = min(tg * TW + w / KP, ntile);  // tile ntile: no outputs (idle wave)
  if (!XL && KP == 1 && tile == ntile) return;
  if constexpr (CT == 4) {  // few pairs left: the cheaper bodies
    if (np - pg0 <= 8) return stream_tile<HT, V, 1, 2, NT, WT, XL>(a, grp.x, grp.z, tile, kpart, KP, pg0, np, red);
    if (np - pg0 <= 16) return stream_tile<HT, V, 2, 2, NT, WT, XL>(a, grp.x, grp.z, tile, kpart, KP, pg0, np, red);
  }
  if constexpr (CT == 2) {
    if (np - pg0 <= 8) return stream_tile<HT, V, 1, 2, NT, WT, XL>(a, grp.x, grp.z, tile, kpart, KP, pg0, np, red);
  }
  if constexpr (LD == kStreamOnce) {
    if (grp.w) return stream_tile<HT, V, CT, U, false, WT, XL>(a, grp.x, grp.z, tile, kpart, KP, pg0, np, red);
  }
  stream_tile<HT, V, CT, U, NT, WT, XL>(a, grp.x, grp.z, tile, kpart, KP, pg0, np, red);
}

template <typename HT, int V, int CT, int U>
static pat_status launch_u(const ContractArgs& a, dim3 grid, int TW, int KP, int tgroups, int pgroups, int ntile, bool nt,
                     bool xl, hipStream_t st) {
  // Written-through lines (whole 128-byte lines only: parts of lines made the
  // launch up to twice as slow) where little is written per slab byte: mixing
  // writes into the slab stream costs more than their bytes (1.55 GB read in
  // 0.23 ms without stores, 0.29 with 135 MB of them), written through a
  // little less: Gram products (whole blocks) 157 against 160 us a step at
  // 256 x 256 x 128; one A + one A^T with A^T's lines written through and not:
  // 128 x 128 x 256 x 256, 244 and 250 us, 64 x 64 x 512 x 512, 218 and 223.  A's
  // spectra stay cached for the transform that follows (written through as
  // well: 256 x 256 x 128 x 512, 902 and 901; 202 x 202 x 32 x 256 linear, 551 and 555).
  const bool wt = a.nj % 16 == 0 && (a.gram || a.ni >= 256);
  const dim3 block(64 * TW * KP);
  // the sums that waves of a workgroup pass on and, in the kernels that stage
  // them, the spectra.  CT = 1 alone stages: the spectra of 32 pairs would
  // leave room for one workgroup per CU from 289 rows on (a step of 4 and 16
  // objects at 64 x 64 x 512: 222 and 986 us with that much LDS, 216 and 881
  // without) and for none beyond 608
  const size_t lds = std::max((size_t)TW * KP * (KP > 1 ? CT : 1) * V * 256 * sizeof(float),
                              xl ? (size_t)8 * xl_stride(a.ni) : 0);
  if (lds > kMaxLds) return fail(PAT_EUNSUPPORTED, "contraction: sums and spectra do not fit in LDS");
  auto kernel = nt && wt ? k_contract<HT, V, CT, U, kStream, true, false>
                : nt     ? k_contract<HT, V, CT, U, kStream, false, false>
                : wt     ? k_contract<HT, V, CT, U, kPlain, true, false>
                         : k_contract<HT, V, CT, U, kPlain, false, false>;
  if constexpr (CT == 1 && sizeof(HT) == 4) {
    const bool once = nt && !wt && !a.gram && a.ni > 64 && a.nj >= a.ni;
    if (xl)  // (rows of whole 16 values are whole 64 bytes: no written-through form with plain loads)
      kernel = !nt    ? k_contract<HT, V, CT, U, kPlain, false, true>
               : wt   ? k_contract<HT, V, CT, U, kStream, true, true>
               : once ? k_contract<HT, V, CT, U, kStreamOnce, false, true>
                      : k_contract<HT, V, CT, U, kStream, false, true>;
    else if (once)
      kernel = k_contract<HT, V, CT, U, kStreamOnce, false, false>;
  }
  kernel<<<grid, block, lds, st>>>(a, TW, KP, tgroups, pgroups, ntile);
  PAT_LAUNCHED("contraction");
  return PAT_OK;
}

constexpr int kFewGroups = 3 * 256;  // three workgroups per CU

template <typename HT, int V, int CT>
static pat_status launch_t(const ContractArgs& a, hipStream_t st) {
  // four waves per workgroup: one per tile up to four tiles; with one or two
  // tiles, four or two waves share the rows of each
  constexpr int tn = 16 * V;
  const int ntile = (a.nj + tn - 1) / tn;
  int tgroups = (ntile + 3) / 4, TW = (ntile + tgroups - 1) / tgroups;
  int KP = TW == 1 ? 4 : TW == 2 ? 2 : 1;
  const int pgroups = (a.members * a.B + 8 * CT - 1) / (8 * CT);
  // 16-bit slabs keep the matrix cores as busy as the loads: with fewer than
  // three workgroups per CU some CUs would have half of the others' work.  One
  // tile per workgroup, its rows shared by the four waves, evens that out (A,
  // bf16: 32 x 32 x 1024 x 1024, 90 us and 65 so; 48 x 48 x 700 x 700, 91 and 69;
  // float32, bound by the loads, is better left: A^T at 64 x 64 x 256 x 1024, 82
  // and 86)
  if (sizeof(HT) == 2 && (KP == 1 || V == 4) && (long long)a.ngroup * tgroups < kFewGroups && a.ni >= 256) {
    KP = 4;
    TW = 1;
    tgroups = ntile;
  }
  const bool big = a.reuse_bytes > kCacheBytes;
  const bool broken = sizeof(HT) == 4 && a.s_row % 16 != 0 && a.ni >= 128 && (a.nj >= 128 || (a.nj > tn && a.ni >= 256));
  const bool nt = big && !broken;
  const bool xl = CT == 1 && sizeof(HT) == 4 && big && a.members > 2 && a.ni >= kXlRows && a.nj >= 64 &&
                  (size_t)8 * xl_stride(a.ni) <= 64 * 1024;
  // Staged products of more than four tiles: up to eight of them share one
  // staging and read whole rows, where the groups are one and a half per CU or more
  // (a step at 96 x 96 x 400, 185 us and 171 so; one A + one A^T at 96 x 96 x 320 x 512,
  // 310 and 298; 64 x 64 x 512 x 512, 215 and 206; of 275 groups, 48 x 48 x 768, 146 and
  // 158; rows of broken pieces no better: 72 x 72 x 500, 164 and 172)
  if (xl && nt && KP == 1 && ntile > 4 && a.ngroup >= 384) {
    tgroups = (ntile + 7) / 8;
    TW = (ntile + tgroups - 1) / tgroups;
  }
  const long long nblk = ((long long)a.ngroup * tgroups * pgroups + 7) / 8 * 8;
  if (nblk > 0x7fffffffLL) return fail(PAT_EUNSUPPORTED, "contraction grid too large");
  const dim3 grid((unsigned)nblk);
  // Row blocks per register buffer: four where a wave's blocks come in fours, so
  // that no load is wasted, else two (one A + one A^T with two instead: 256 x 256 x
  // 128 x 512, contractions 604 and 610 us; a step at 96 x 96 x 320, 121 and 124; on the
  // other side 202 x 202 x 32 x 256 linear, 285 and 272; four at any length: A^T at
  // 256 x 256 x 24 x 300, 55 and 62 us)
  const int share = (a.ni >> 3) / KP;  // row blocks of a wave
  constexpr int U4 = CT == 1 && V <= 4 ? 4 : 2;
  if (CT == 1 && V <= 4 && share % 4 == 0)
    return launch_u<HT, V, CT, U4>(a, grid, TW, KP, tgroups, pgroups, ntile, nt, xl, st);
  return launch_u<HT, V, CT, (CT == 4 ? 1 : 2)>(a, grid, TW, KP, tgroups, pgroups, ntile, nt, xl, st);
}

// 16-bit rows: a tile of 16-byte loads is 128 outputs, and a matrix instruction
// is issued per value of a load whether its columns are outputs or not.  Rows
// of up to a half or a quarter of that take 8- or 4-byte loads (A^T, bf16, 16-
// byte loads and these: 216 x 216 x 5 x 1670, 250 and 92 us; 64 x 64 x 1100 x 48 (A),
// 29 and 20), and one tile's rows two tiles of 8-byte loads where the groups
// are few (72 x 72 x 127 x 992, A^T: 47 and 35).
template <typename HT>
static pat_status launch_16(const ContractArgs& a, hipStream_t st) {
  if (a.nj <= 32) return launch_t<HT, 2, 1>(a, st);
  if (a.nj <= 64 || (a.nj <= 128 && a.ngroup < kFewGroups)) return launch_t<HT, 4, 1>(a, st);
  return launch_t<HT, 8, 1>(a, st);
}

// Gram products that the vector units' kernel takes: of one object with two
// members per class, from HBM, of more than 128 rows that are not whole 128-byte
// lines, where the groups are many (a step, vector / matrix: 256 x 192 x 140,
// 254 / 287 us; 96 x 64 x 400, 207 / 236; 48 x 32 x 1050, 348 / 395; of whole lines, 256 x
// 192 x 192, 418 / 411; 153 groups: 32 x 16 x 1601, 374 / 333).
static bool pair_gram(const ContractArgs& a) {
  return a.gram && a.B == 1 && a.members <= 2 && a.ni > 128 && a.s_row % 32 != 0 && a.reuse_bytes > kCacheBytes &&
         a.ngroup >= 200;
}

pat_status contract(const ContractArgs& a, int hdtype, hipStream_t st) {
  if (a.ngroup == 0 || a.B == 0) return PAT_OK;
  if (a.slab_elems > (1LL << 28) || (long long)kGroup * a.in_rs > (1LL << 27) ||
      (long long)kGroup * a.out_rs > (1LL << 27))
    return fail(PAT_EUNSUPPORTED, "contraction slab or spectrum rows beyond 32-bit offsets");
  // one object on the two-member fold: the vector units' kernel
  if ((a.members <= 2 && a.B == 1 && !a.gram) || pair_gram(a)) return contract_pair(a, hdtype, st);
  // Gram products from half of each block, where the units (a group's 8 pairs,
  // a wave each) fill the CUs and, for one object, rows start at whole 64-byte
  // pieces (a step of one object at 108 x 108 x 100, 400-byte rows: 42.0 us
  // whole, 44.5 half; of 2 and 16 at 144 x 144 x 105: 92.9 and 85.8, 600 and 563;
  // one at 64 x 64 x 96, 561 units: 25.4 and 27.2; at 96 x 96 x 128, 1,225 units:
  // 39.7 and 38.4); up to 64 rows always (one object at 64 x 64 x 64: 24.4 and 24.5;
  // 128 x 128 x 52: 35.5 and 34.2; 16 objects at 96 x 96 x 13: 92.8 and 44.0)
  const long long units = (long long)a.ngroup * ((a.members * a.B + 7) / 8);
  if (a.gram && (a.ni <= 64 || (a.ni <= 128 && (a.B > 1 || a.s_row % 16 == 0) && units >= 1024)))
    return contract_sym(a, a.reuse_bytes > kCacheBytes, st);
  if (hdtype == PAT_H_BF16) return launch_16<bf16_t>(a, st);
  if (hdtype == PAT_H_F16) return launch_16<f16_t>(a, st);
  const int pairs = a.members * a.B;
  if (pairs <= 8) return launch_t<float, 4, 1>(a, st);
  if (pairs <= 16) return launch_t<float, 4, 2>(a, st);
  return launch_t<float, 4, 4>(a, st);
}

}  // namespace pat
