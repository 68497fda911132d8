// The verifier-derived update signal (Sec. 3.4, Eq. 8) and the drafter row it
// is read from, shared by the acceptance kernels (whose last step it is) and
// the commit's planning.
#pragma once
#include "common.h"
#include "kernels.h"
#include "specblock.h"

namespace sb {

// The drafter row at position pos(cur) + 1 on a path through node cur: the
// next row of cur's block when cur is a chain node short of K, else row 1 of
// a block started at cur; -1 when the tree has none.  Called by a whole wave
// (the rows are searched 64 at a time, the first candidates' loads issued
// before the chain of dependent ones).
__device__ __forceinline__ int continuing_row(const TreeDims& td,
                                              const sb_tree& t, int s, int cur) {
  const int lane = threadIdx.x & 63;
  const size_t nb = (size_t)s * td.budget;
  const size_t rb = (size_t)s * td.row_cap;
  const int nrows = t.n_rows[s];
  if (cur == 0) return nrows > 0 ? 0 : -1;
  const int j = min(lane, td.row_cap - 1);
  const int st0 = t.row_start[rb + j], k0 = t.row_k[rb + j];
  const int r = t.row[nb + cur];
  if (t.rank[nb + cur] == 1 && t.row_k[rb + r] < td.K && r + 1 < nrows)
    return r + 1;
  uint64_t m = __ballot(lane < nrows && st0 == cur && k0 == 1);
  if (m != 0) return __builtin_ctzll(m);
  for (int j0 = 64; j0 < nrows; j0 += 64) {
    const int q = j0 + lane;
    m = __ballot(q < nrows && t.row_start[rb + q] == cur && t.row_k[rb + q] == 1);
    if (m != 0) return j0 + __builtin_ctzll(m);
  }
  return -1;
}

// At the rejected position (the one after the last accepted node cur, where
// the bonus token stands), the drafter's probability r of the target's token,
// from the row that predicted that position: r = exp(z[bonus] - lse) with
// z[bonus] = W_lm[bonus] . norm(h^(L)) recomputed from the row's cached
// h^(L) (the final RMSNorm and the LM-head operand rounding of the drafter
// forward), lse the row's log-sum-exp.  -1 when no drafter row predicts that
// position; 0 when the bonus token is outside a reduced drafter vocabulary.
// Called by a workgroup of 256 threads (d <= 8192): a thread owns eight
// columns of every 2048, and the hidden row, the gains and the LM-head row
// are loaded in one round trip.
template <typename T>
__device__ __forceinline__ void reject_signal_block(const TreeDims& td,
                                                    const sb_tree& t, int s,
                                                    int cur, int bonus,
                                                    const SignalArgs& g) {
  constexpr int MAXQ = 4;
  __shared__ float red[2][4];
  const int tid = threadIdx.x, lane = tid & 63, w = tid >> 6;
  const int cont = continuing_row(td, t, s, cur);
  int id = -1;
  if (g.d2t == nullptr) {
    id = (bonus >= 0 && bonus < g.Vd) ? bonus : -1;
  } else {   // d2t is strictly increasing: binary search
    int lo = 0, hi = g.Vd - 1;
    while (lo <= hi) {
      const int mid = (lo + hi) >> 1;
      const int v = g.d2t[mid];
      if (v == bonus) {
        id = mid;
        break;
      }
      if (v < bonus) lo = mid + 1;
      else hi = mid - 1;
    }
  }
  if (cont < 0 || id < 0) {   // uniform
    if (tid == 0) g.r[s] = cont < 0 ? -1.f : 0.f;
    return;
  }
  const int d = td.d;
  const size_t o = (size_t)s * td.row_cap + cont;
  const float lse = g.row_lse[o];
  const float* h = t.h_last + o * d;
  const T* lm = static_cast<const T*>(g.lm_head);
  float4 hv[MAXQ][2], gv[MAXQ][2];
  T wv[MAXQ][8];
  float ss = 0.f;
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    const int k0 = 8 * tid + 2048 * q;
    if (k0 >= d) break;
    size_t wi;
    if constexpr (sizeof(T) == 2) {
      // fragment-packed LM head (32-row x 64-column blocks)
      const int c = k0 & 63;
      const int l = (id & 31) + 32 * (c >> 5);
      wi = ((((size_t)(k0 >> 6) * (g.Vd >> 5) + (id >> 5)) * 4 + ((c & 31) >> 3)) *
            512) + (size_t)l * 8;
    } else {
      wi = (size_t)id * d + k0;
    }
#pragma unroll
    for (int e = 0; e < 8 * (int)sizeof(T) / 16; ++e)
      reinterpret_cast<uint4*>(wv[q])[e] =
          reinterpret_cast<const uint4*>(lm + wi)[e];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      hv[q][e] = reinterpret_cast<const float4*>(h + k0)[e];
      gv[q][e] = reinterpret_cast<const float4*>(g.gain + k0)[e];
      ss += hv[q][e].x * hv[q][e].x + hv[q][e].y * hv[q][e].y +
            hv[q][e].z * hv[q][e].z + hv[q][e].w * hv[q][e].w;
    }
  }
  ss = wave_sum(ss);
  if (lane == 0) red[0][w] = ss;
  __syncthreads();
  const float rs = 1.0f / sqrtf((red[0][0] + red[0][1] + red[0][2] + red[0][3]) /
                                    (float)d + g.eps);
  float z = 0.f;
#pragma unroll
  for (int q = 0; q < MAXQ; ++q) {
    if (8 * tid + 2048 * q >= d) break;
    const float hx[8] = {hv[q][0].x, hv[q][0].y, hv[q][0].z, hv[q][0].w,
                         hv[q][1].x, hv[q][1].y, hv[q][1].z, hv[q][1].w};
    const float gx[8] = {gv[q][0].x, gv[q][0].y, gv[q][0].z, gv[q][0].w,
                         gv[q][1].x, gv[q][1].y, gv[q][1].z, gv[q][1].w};
#pragma unroll
    for (int e = 0; e < 8; ++e)
      z += Elem<T>::to_f32(wv[q][e]) *
           Elem<T>::to_f32(Elem<T>::from_f32(hx[e] * rs * gx[e]));
  }
  z = wave_sum(z);
  if (lane == 0) red[1][w] = z;
  __syncthreads();
  if (tid == 0)
    g.r[s] = __expf((red[1][0] + red[1][1] + red[1][2] + red[1][3]) - lse);
}

}  // namespace sb
