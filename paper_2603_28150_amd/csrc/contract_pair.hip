// The per-frequency contraction (step (ii) of Sec. 3.2) of one object on grids
// that are not square, whose classes hold at most two frequencies (m, +-p).
//
// With two members a slab value meets four spectrum parts: the matrix kernel
// (contract.hip) would fill a quarter of its instructions, while the vector
// units do the same products in the time the slab takes to arrive.  A slab
// (or, for long rows, half of every row) belongs to one workgroup: lanes of a
// row group cover one row with 16-byte non-temporal loads, row groups take
// interleaved rows, the member spectra sit in LDS, and an LDS tree adds the
// row groups' sums in a fixed order.  Measured against the matrix kernel on this
// fold (one A + one A^T, float32): 192 x 32 transforms x 54 x 476, 118 and 126 us;
// 96 x 108 x 95 x 167, 127 and 130 us; 192 x 96 x 50 x 301, 197 and 205 us.
//
// Gram products beyond 128 depths come here where contract() says so: a workgroup
// reads whole rows, so that rows of broken lines meet no line twice.  Their
// sums of 16 rows are kept apart before they join the total, as in the matrix
// kernel, whose error they would otherwise pass (700 rows: 4.6e-7, 1.4e-7 so); the
// loads of the long rows hide it (a step at 256 x 192 x 140, 256 us without, 254
// with), those of short ones do not (144 x 192 x 21 x 162, bf16: 162 and 166).
#include <algorithm>
#include <type_traits>

#include "contract_slab.hpp"
#include "dft.hpp"
#include "pat_internal.hpp"

namespace pat {

constexpr int kRowParts = 2;  // workgroups per slab for long rows
template <typename HT> constexpr int kRows = std::is_same<HT, float>::value ? 2 : 4;  // rows per register buffer

// float32: two rows per register buffer instead of four, so that the kernel
// fits 128 registers and four waves per SIMD (measured faster on short rows,
// neutral on long ones)
template <typename HT, bool GRAM>
__global__ __launch_bounds__(256, (std::is_same<HT, float>::value ? 4 : 1)) void k_contract_pair(ContractArgs a,
                                                                                                int lr_log2, int JS,
                                                                                                int chpart) {
  extern __shared__ float4 smem_raw[];
  // workgroups are dealt to the eight XCDs round-robin by index: the units
  // (class, row part) are cut into eight contiguous ranges, one per XCD
  const int units = a.ngroup * JS;
  const int per_xcd = (units + 7) >> 3;
  const int unit = (blockIdx.x & 7) * per_xcd + (blockIdx.x >> 3);
  if (unit >= units) return;  // whole workgroup: padding of the grid
  const int t = unit / JS, part = unit - t * JS;
  const int4 grp = a.groups[t];  // first spectrum row, members (1 or 2), slab
  constexpr int GG = 2;
  typedef Slab<HT> SL;
  typedef typename SL::raw_t raw_t;
  constexpr int VEC = SL::VEC;
  constexpr int U = kRows<HT>;      // rows per register buffer
  constexpr int NS = VEC * GG * 2;  // accumulators per thread
  const int j0 = part * chpart * VEC;
  const int njl = min(a.nj - j0, chpart * VEC);
  float2* xin = reinterpret_cast<float2*>(smem_raw);
  float* red = reinterpret_cast<float*>(smem_raw);
  const int tid = threadIdx.x;
  const int Lr = 1 << lr_log2, R = 256 >> lr_log2;
  const int lr = tid & (Lr - 1), rg = tid >> lr_log2;

  // this workgroup's part of the rows: elements j0 .. j0 + njl - 1
  const HT* slab = reinterpret_cast<const HT*>(a.slab) + (size_t)grp.z * a.slab_elems + j0;
  const int nchunks = (njl + VEC - 1) / VEC;
  const bool cl = lr < nchunks;
  const HT* colp = slab + (size_t)min(lr, nchunks - 1) * VEC;  // clamped: always a valid address

  // Rows in flight: the loads of the next U rows are issued before the FMAs
  // of the current ones (two register buffers), so that every wave keeps
  // memory requests outstanding while it computes.  Loads are unconditional
  // (rows and chunks clamped into the slab, the value zeroed by a select) so
  // that no branch hides them from the wait counter.
  auto load_rows = [&](raw_t (&raw)[U], int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * R;
      const int ic = min(i, a.ni - 1);
      const raw_t v = __builtin_nontemporal_load(reinterpret_cast<const raw_t*>(colp + (size_t)ic * a.s_row));
      raw[u] = (i < a.ni && cl) ? v : raw_t(0);
    }
  };
  raw_t ra[U], rb[U];
  load_rows(ra, rg);  // the first rows travel while the member vectors are staged

  // member input vectors -> LDS xin[i][g], with the optional per-row scale;
  // 16-byte loads along each member row when the row length is even
  if ((a.ni & 1) == 0) {
    // batches of kStage loads per thread, all issued before their LDS stores
    // (one memory latency per batch instead of one per load); consecutive
    // lanes take consecutive members of one k pair, so that the LDS stores
    // are contiguous (the loads still cover whole 128-byte lines per wave)
    constexpr int kStage = 8;
    const int h = a.ni >> 1;
    const int total = GG * h;
    for (int base = tid; base < total; base += 256 * kStage) {
      float4 v[kStage];
      float2 sv[kStage];  // the per-row scales of the pair, loaded with it
#pragma unroll
      for (int q = 0; q < kStage; ++q) {
        const int idx = base + q * 256;
        v[q] = make_float4(0.f, 0.f, 0.f, 0.f);
        sv[q] = make_float2(1.f, 1.f);
        if (idx < total) {
          const int g = idx % GG, i = 2 * (idx / GG);
          if (g < grp.y) v[q] = *reinterpret_cast<const float4*>(a.in + (size_t)(grp.x + g) * a.in_rs + i);
          if (a.in_scale) sv[q] = *reinterpret_cast<const float2*>(a.in_scale + i);
        }
      }
#pragma unroll
      for (int q = 0; q < kStage; ++q) {
        const int idx = base + q * 256;
        if (idx >= total) break;
        const int g = idx % GG, i = 2 * (idx / GG);
        float4 w = v[q];
        if (a.in_scale) w = make_float4(w.x * sv[q].x, w.y * sv[q].x, w.z * sv[q].y, w.w * sv[q].y);
        xin[i * GG + g] = make_float2(w.x, w.y);
        xin[(i + 1) * GG + g] = make_float2(w.z, w.w);
      }
    }
  } else {
    for (int idx = tid; idx < a.ni * GG; idx += 256) {
      const int i = idx / GG, g = idx % GG;
      float2 v = make_float2(0.f, 0.f);
      if (g < grp.y) {
        v = a.in[(size_t)(grp.x + g) * a.in_rs + i];
        if (a.in_scale) v = cscale(v, a.in_scale[i]);
      }
      xin[idx] = v;
    }
  }
  __syncthreads();

  float acc[NS], sum16[GRAM ? NS : 1];
#pragma unroll
  for (int s = 0; s < NS; ++s) acc[s] = 0.f;
  auto flush = [&]() {
#pragma unroll
    for (int s = 0; s < (GRAM ? NS : 0); ++s) {
      acc[s] += sum16[s];
      sum16[s] = 0.f;
    }
  };
  if constexpr (GRAM) {
#pragma unroll
    for (int s = 0; s < NS; ++s) sum16[s] = 0.f;
  }

  auto fma_rows = [&](const raw_t (&raw)[U], int i0) {
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int i = i0 + u * R;
      if (i >= a.ni) break;
      float2 xv[GG];
#pragma unroll
      for (int g = 0; g < GG; ++g) xv[g] = xin[i * GG + g];
#pragma unroll
      for (int v = 0; v < VEC; ++v) {
        const float h = SL::get(raw[u], v);
#pragma unroll
        for (int g = 0; g < GG; ++g) {
          float* p = GRAM ? &sum16[(v * GG + g) * 2] : &acc[(v * GG + g) * 2];
          p[0] = fmaf(h, xv[g].x, p[0]);
          p[1] = fmaf(h, xv[g].y, p[1]);
        }
      }
    }
  };
  int left = 16;  // rows to the next addition to the total
  for (int i0 = rg; i0 < a.ni; i0 += 2 * R * U) {
    load_rows(rb, i0 + R * U);
    fma_rows(ra, i0);
    if (i0 + R * U >= a.ni) break;
    load_rows(ra, i0 + 2 * R * U);
    fma_rows(rb, i0 + R * U);
    if (GRAM && (left -= 2 * U) <= 0) {
      flush();
      left = 16;
    }
  }
  flush();

  // add the partial sums of the R row groups (fixed order: deterministic)
  for (int half = R >> 1; half >= 1; half >>= 1) {
    __syncthreads();
    const int span = half * Lr;
    if (rg >= half && rg < 2 * half) {
      const int w = (rg - half) * Lr + lr;
#pragma unroll
      for (int s = 0; s < NS; ++s) red[s * span + w] = acc[s];
    }
    __syncthreads();
    if (rg < half) {
      const int w = rg * Lr + lr;
#pragma unroll
      for (int s = 0; s < NS; ++s) acc[s] += red[s * span + w];
    }
  }

  // float32 (no scales), whole 16-byte pairs per lane and nothing to subtract:
  // row group 0 stores its sums directly (each lane four consecutive outputs
  // per member, the lanes of a member row contiguous), without a pass through
  // LDS (A and A^T 1.5 % faster; the 16-bit kernels, eight outputs per lane,
  // measured 4 % slower that way and keep the pass through LDS)
  if (std::is_same<HT, float>::value && a.out_sub == nullptr && (a.nj & 1) == 0 && njl % VEC == 0) {
    const int cj = lr * VEC;
    if (rg != 0 || cj >= njl) return;
#pragma unroll
    for (int g = 0; g < GG; ++g) {
      if (g >= grp.y) continue;
      v4f* dst = reinterpret_cast<v4f*>(a.out + (size_t)(grp.x + g) * a.out_rs + j0 + cj);
#pragma unroll
      for (int v = 0; v < VEC; v += 2) {
        const float* q0 = &acc[(v * GG + g) * 2];
        const float* q1 = &acc[((v + 1) * GG + g) * 2];
        __builtin_nontemporal_store(v4f{q0[0], q0[1], q1[0], q1[1]}, dst + v / 2);
      }
    }
    return;
  }

  // stage the member rows in LDS, then store each row contiguously (whole
  // cache lines per store instruction)
  __syncthreads();
  float2* ob = reinterpret_cast<float2*>(smem_raw);
  if (rg == 0) {
    // per-row output scales: every load issued before the first is used
    float scv[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) scv[v] = a.out_scale ? a.out_scale[j0 + min(lr * VEC + v, njl - 1)] : 1.f;
#pragma unroll
    for (int v = 0; v < VEC; ++v) {
      const int j = lr * VEC + v;
      if (j >= njl) continue;
#pragma unroll
      for (int g = 0; g < GG; ++g) {
        const float* p = &acc[(v * GG + g) * 2];
        ob[g * njl + j] = make_float2(p[0] * scv[v], p[1] * scv[v]);
      }
    }
  }
  __syncthreads();
  const size_t o0 = (size_t)grp.x * a.out_rs + j0;
  if ((njl & 1) == 0 && (a.nj & 1) == 0) {
    // two complex values (16 bytes) per store, non-temporal: the rows are
    // not read again by this kernel
    const int h = njl >> 1;
    for (int e = tid; e < GG * h; e += 256) {
      const int g = e >= h, j = 2 * (e - g * h);
      if (g >= grp.y) continue;
      v4f d = *reinterpret_cast<const v4f*>(ob + g * njl + j);
      const size_t o = o0 + (size_t)g * a.out_rs + j;
      if (GRAM && a.out_sub) d -= *reinterpret_cast<const v4f*>(a.out_sub + o);
      __builtin_nontemporal_store(d, reinterpret_cast<v4f*>(a.out + o));
    }
  } else {
    for (int e = tid; e < GG * njl; e += 256) {
      const int g = e >= njl, j = e - g * njl;
      if (g >= grp.y) continue;
      const size_t o = o0 + (size_t)g * a.out_rs + j;
      a.out[o] = GRAM && a.out_sub ? csub(ob[e], a.out_sub[o]) : ob[e];
    }
  }
}

template <typename HT, bool GRAM>
static pat_status launch_pair(const ContractArgs& a, hipStream_t st) {
  constexpr int VEC = Slab<HT>::VEC;
  // rows of 128 or more 16-byte chunks are split over kRowParts workgroups
  // per slab (halves of 1 KB and more still stream well; shorter parts
  // measured slower)
  const int chunks = (a.nj + VEC - 1) / VEC;
  const int JS = chunks >= 128 ? kRowParts : 1;
  const int chpart = (chunks + JS - 1) / JS;  // 16-byte chunks per part
  if (chpart > 256) return fail(PAT_EUNSUPPORTED, "contraction row longer than 512 vectors");
  int lr_log2 = 0;
  while ((1 << lr_log2) < chpart) ++lr_log2;
  const int Lr = 1 << lr_log2, R = 256 / Lr;
  const size_t red_bytes = R > 1 ? (size_t)(R / 2) * Lr * VEC * 4 * sizeof(float) : 0;
  const size_t in_bytes = (size_t)a.ni * 2 * sizeof(float2);
  const size_t out_bytes = (size_t)chpart * VEC * 2 * sizeof(float2);
  const size_t lds = std::max(red_bytes, std::max(in_bytes, out_bytes));
  if (lds > 160 * 1024) return fail(PAT_EUNSUPPORTED, "contraction input vector does not fit in LDS");
  const long long nblk = ((long long)a.ngroup * JS + 7) / 8 * 8;
  if (nblk > 0x7fffffffLL) return fail(PAT_EUNSUPPORTED, "contraction grid too large");
  k_contract_pair<HT, GRAM><<<dim3((unsigned)nblk), 256, lds, st>>>(a, lr_log2, JS, chpart);
  PAT_LAUNCHED("contraction (two members)");
  return PAT_OK;
}

pat_status contract_pair(const ContractArgs& a, int hdtype, hipStream_t st) {
  if (a.members > 2 || a.B != 1) return fail(PAT_EINVAL, "the two-member contraction takes one object");
  if (a.gram) return launch_pair<float, true>(a, st);
  if (hdtype == PAT_H_F32) return launch_pair<float, false>(a, st);
  if (hdtype == PAT_H_BF16) return launch_pair<bf16_t, false>(a, st);
  return launch_pair<f16_t, false>(a, st);
}

}  // namespace pat
