// The exact merge of one row's partial results where many workgroups share a row block (calls of
// few queries), by a whole workgroup.
#pragma once
#include "vmla_device.h"

namespace vmla {

// dst[0 .. width) = sum_s 2^(m_s - M) O_s / sum_s 2^(m_s - M) l_s over the ns partial results s of
// partial row `prow`, by the 256 threads of a workgroup: thread (slice, 8 columns) takes the splits
// slice, slice + SL, .. with the loads of eight in flight together, under its own running max; the
// SL slices are then combined through LDS. Rows split 63 ways are bound by the latency of their
// loads: one thread per 8 columns walks them in 16 dependent groups of four.
__device__ __forceinline__ void merge_row_split(const AttendArgs& a, size_t prow, size_t total_rows,
                                                int width, int ns, uint16_t* dst) {
  constexpr float kNone = -__builtin_huge_valf();
  constexpr int kMaxSlices = 16;
  __shared__ f32x4 part[2][256];
  __shared__ float sm[kMaxSlices], sl[kMaxSlices];
  const int gpr = width / 8, SL = min(256 / gpr, kMaxSlices);
  const int slice = threadIdx.x / gpr, grp = threadIdx.x % gpr;
  float M = kNone, L = 0.f;
  f32x4 lo = {0.f, 0.f, 0.f, 0.f}, hi = {0.f, 0.f, 0.f, 0.f};
  if (slice < SL) {
    for (int s0 = slice; s0 < ns; s0 += 8 * SL) {
      f32x2 ml[8];
      f32x4 vlo[8], vhi[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int s = s0 + j * SL;
        if (s < ns) {
          const size_t base = (size_t)s * total_rows + prow;
          ml[j] = *reinterpret_cast<const f32x2*>(a.ml_part + base * 2);
          const f32x4* src = reinterpret_cast<const f32x4*>(a.o_part + base * width + grp * 8);
          vlo[j] = src[0];
          vhi[j] = src[1];
        } else {
          ml[j] = f32x2{kNone, 0.f};
        }
      }
      float m = M;
#pragma unroll
      for (int j = 0; j < 8; ++j) m = fmaxf(m, ml[j][0]);
      const float keep = fast_exp2(M - m);  // 0 for the first group
      L *= keep;
      lo *= keep;
      hi *= keep;
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        if (s0 + j * SL < ns) {
          const float coef = fast_exp2(ml[j][0] - m);
          L += coef * ml[j][1];
          lo += coef * vlo[j];
          hi += coef * vhi[j];
        }
      }
      M = m;
    }
    part[0][threadIdx.x] = lo;
    part[1][threadIdx.x] = hi;
    if (grp == 0) {
      sm[slice] = M;
      sl[slice] = L;
    }
  }
  __syncthreads();
  if (slice > 0) return;
  const int used = min(SL, ns);
  for (int s = 1; s < used; ++s) M = fmaxf(M, sm[s]);
  L = 0.f;
  lo = f32x4{0.f, 0.f, 0.f, 0.f};
  hi = lo;
  for (int s = 0; s < used; ++s) {
    const float coef = fast_exp2(sm[s] - M);
    L += coef * sl[s];
    lo += coef * part[0][s * gpr + grp];
    hi += coef * part[1][s * gpr + grp];
  }
  const float il = 1.f / L;
  const f32x8 v = {lo[0] * il, lo[1] * il, lo[2] * il, lo[3] * il,
                   hi[0] * il, hi[1] * il, hi[2] * il, hi[3] * il};
  *reinterpret_cast<bf16x8*>(dst + grp * 8) = to_bf16x8(v);
}

}  // namespace vmla
