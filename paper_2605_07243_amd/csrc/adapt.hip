// Head-only serving-time update of the drafter (Sec. 3.4; the per-query
// adaptation procedure of App. A.3): buffered rejected positions step the
// drafter's LM head and rank head on their cross-entropy against the
// verifier's token plus a KL penalty towards the pre-deployment head, one
// SGD step on a training copy of the weights.  The decoder trunk and the
// final norm stay frozen.  The logit statistics and gradients of each
// position are computed by adapt_kl_kernel and adapt_grad_kernel
// (vocab.hip); here are the operand preparation and the two weight updates.
#include <float.h>

#include "common.h"
#include "kernels.h"

namespace sb {

namespace {

constexpr int kStripeRows = 64;      // LM-head rows per update workgroup

}  // namespace

// a_i = RMSNorm(h_i) * g in the weights' element type (the LM head's operand
// in the drafter forward), for i < n = min(count, cap); n_eff = n.
template <typename T>
__global__ __launch_bounds__(1024) void adapt_prep_kernel(
    const float* __restrict__ h, const int* __restrict__ count, int cap,
    const float* __restrict__ g, float eps, int d, T* __restrict__ A,
    int* __restrict__ n_eff) {
  __shared__ float red[16];
  const int i = blockIdx.x;
  const int n = min(*count, cap);
  if (i == 0 && threadIdx.x == 0) *n_eff = n;
  if (i >= n) return;
  const float* hr = h + (size_t)i * d;
  float ss = 0.f;
#pragma unroll 4
  for (int k = threadIdx.x; k < d; k += 1024) ss += hr[k] * hr[k];
  ss = block_sum(ss, red);
  const float rs = 1.0f / sqrtf(ss / (float)d + eps);
#pragma unroll 4
  for (int k = threadIdx.x; k < d; k += 1024)
    A[(size_t)i * d + k] = Elem<T>::from_f32(hr[k] * rs * g[k]);
}

// f32: W -= lr * G^T A over a stripe of 64 LM-head rows x CW columns, with
// G [n][Vd] the (already 1/n-scaled) logit gradients and A [n][d] the
// operands, n <= 64.  A thread owns 8 consecutive columns of one row.
template <int CW>
__global__ __launch_bounds__(256) void lm_update_f32_kernel(
    float* __restrict__ W, int Vd, int d, const float* __restrict__ G,
    const float* __restrict__ A, const int* __restrict__ n_eff, float lr) {
  __shared__ float gs[64][kStripeRows];
  __shared__ float as[64][CW];
  const int n = *n_eff;
  if (n <= 0) return;
  const int r0 = blockIdx.x * kStripeRows, c0 = blockIdx.y * CW;
  for (int e = threadIdx.x; e < n * kStripeRows; e += 256) {
    const int i = e / kStripeRows, r = e % kStripeRows;
    gs[i][r] = G[(size_t)i * Vd + r0 + r];
  }
  for (int e = threadIdx.x; e < n * CW; e += 256) {
    const int i = e / CW, c = e % CW;
    as[i][c] = A[(size_t)i * d + c0 + c];
  }
  __syncthreads();
  constexpr int kChunks = kStripeRows * CW / 8;
  for (int q = threadIdx.x; q < kChunks; q += 256) {
    const int r = q / (CW / 8), c = 8 * (q % (CW / 8));
    const size_t addr = (size_t)(r0 + r) * d + c0 + c;
    float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (int i = 0; i < n; ++i) {
      const float gv = gs[i][r];
#pragma unroll
      for (int e = 0; e < 8; ++e) acc[e] += gv * as[i][c + e];
    }
#pragma unroll
    for (int e = 0; e < 8; ++e) W[addr + e] -= lr * acc[e];
  }
}

typedef float upd_f32x16_t __attribute__((ext_vector_type(16)));
typedef unsigned int upd_u32x4_t __attribute__((ext_vector_type(4)));

// Contraction index i (a buffered position) of a 16-position step held by
// lane group l / 32 of an MFMA operand: 16 j + 8 (l / 32) + e, e = 0..7.
// Weight column that row m (= l % 32) of the operand of half f stands for:
// with output register r of lane half h being row 8 (r / 4) + 4 h + r % 4,
// this order leaves lane half h with columns 32 h + 16 f + r, r = 0..15, i.e.
// with the packed layout's sub-steps 2 f and 2 f + 1 of its own chunk.
__device__ __forceinline__ int upd_column(int m, int f) {
  return 32 * ((m >> 2) & 1) + 16 * f + 4 * (m >> 3) + (m & 3);
}

// The operands of 64 columns as MFMA operands, At[kb][f][j][lane][8]; zero
// past the n positions.  One workgroup per 64 columns.
__global__ __launch_bounds__(256) void lm_operand_kernel(
    const bf16_t* __restrict__ A, int d, const int* __restrict__ n_eff,
    bf16_t* __restrict__ At) {
  __shared__ bf16_t as[64][64 + 8];
  const int n = *n_eff, kb = blockIdx.x, tid = threadIdx.x;
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int i = (tid >> 3) + 32 * q, c = 8 * (tid & 7);
    uint4 v = make_uint4(0, 0, 0, 0);
    if (i < n) v = *reinterpret_cast<const uint4*>(A + (size_t)i * d + 64 * kb + c);
    *reinterpret_cast<uint4*>(&as[i][c]) = v;
  }
  __syncthreads();
#pragma unroll
  for (int q = 0; q < 2; ++q) {
    const int chunk = tid + 256 * q, l = chunk & 63;
    const int j = (chunk >> 6) & 3, f = chunk >> 8;
    const int c = upd_column(l & 31, f), i0 = 16 * j + 8 * (l >> 5);
    uint32_t w[4];
#pragma unroll
    for (int e = 0; e < 4; ++e)
      w[e] = (uint32_t)as[i0 + 2 * e][c] | ((uint32_t)as[i0 + 2 * e + 1][c] << 16);
    *reinterpret_cast<uint4*>(At + ((size_t)kb * 512 + chunk) * 8) =
        make_uint4(w[0], w[1], w[2], w[3]);
  }
}

// bf16: W -= lr * G^T A over the fragment-packed LM head, n <= 64 positions.
// A wave owns one 32-row block and walks over its 64-column blocks: each
// 4 KiB of weights is read once, stepped and written back where it changed
// (a step is far below the spacing of most weights, so most 16-byte chunks
// keep their bits).  The contraction runs on the matrix cores: G (fp32) is
// split once per wave into three bf16 parts that sum to it exactly, the
// operands are bf16 already, so all products are exact and only the fp32
// accumulation rounds, as it does with fp32 FMAs.  Bound by HBM (the head
// read, and written back where it changes); the VALU form took one LDS
// operand per FMA: 64 positions x 128256 x 4096 2270 -> 330 us.
__global__ __launch_bounds__(256, 2) void lm_update_kernel(
    bf16_t* __restrict__ W, int Vd, int d, const float* __restrict__ G,
    const bf16_t* __restrict__ At, const int* __restrict__ n_eff, float lr,
    int kb_per) {
  const int n = *n_eff;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int lr32 = lane & 31, h = lane >> 5;
  const int rb = blockIdx.x * 4 + wave, n_rb = Vd >> 5;
  if (n <= 0 || rb >= n_rb) return;
  const int kb0 = blockIdx.y * kb_per, kb1 = min(d >> 6, kb0 + kb_per);
  upd_u32x4_t gf[3][4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    float g[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int i = 16 * j + 8 * h + e;
      g[e] = i < n ? G[(size_t)i * Vd + 32 * rb + lr32] : 0.f;
    }
#pragma unroll
    for (int s = 0; s < 3; ++s)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const uint32_t w = pack_bf16x2(g[2 * e], g[2 * e + 1]);
        gf[s][j][e] = w;
        // what the part leaves (nothing where it is not finite)
        const float lo = __uint_as_float(w << 16);
        const float hi = __uint_as_float(w & 0xFFFF0000u);
        g[2 * e] = fabsf(lo) <= FLT_MAX ? g[2 * e] - lo : 0.f;
        g[2 * e + 1] = fabsf(hi) <= FLT_MAX ? g[2 * e + 1] - hi : 0.f;
      }
  }
  bf16_t* wp = W + (size_t)rb * 2048 + lane * 8;
  const size_t kstride = (size_t)n_rb * 2048;
  const bf16_t* ap = At + lane * 8;
  upd_u32x4_t w[4], wn[4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
    w[i] = *reinterpret_cast<const upd_u32x4_t*>(wp + kb0 * kstride + 512 * i);
  for (int kb = kb0; kb < kb1; ++kb) {
    upd_u32x4_t a[2][4];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int j = 0; j < 4; ++j)
        a[f][j] = *reinterpret_cast<const upd_u32x4_t*>(
            ap + ((size_t)kb * 8 + f * 4 + j) * 512);
    const size_t nx = (size_t)min(kb + 1, kb1 - 1) * kstride;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      wn[i] = *reinterpret_cast<const upd_u32x4_t*>(wp + nx + 512 * i);
    upd_f32x16_t acc[2];
#pragma unroll
    for (int f = 0; f < 2; ++f)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[f][r] = 0.f;
#pragma unroll
    for (int s = 2; s >= 0; --s)       // the small parts first
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int f = 0; f < 2; ++f)
          acc[f] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
              __builtin_bit_cast(bf16x8_t, a[f][j]),
              __builtin_bit_cast(bf16x8_t, gf[s][j]), acc[f], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      upd_u32x4_t o;
      uint32_t diff = 0u;
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = 8 * (i & 1) + 2 * e;
        o[e] = pack_bf16x2(
            __uint_as_float(w[i][e] << 16) - lr * acc[i >> 1][r],
            __uint_as_float(w[i][e] & 0xFFFF0000u) - lr * acc[i >> 1][r + 1]);
        diff |= o[e] ^ w[i][e];
      }
      if (diff != 0u)
        *reinterpret_cast<upd_u32x4_t*>(wp + kb * kstride + 512 * i) = o;
      w[i] = wn[i];
    }
  }
}

// Rank head: W_r[b][j] -= lr * sum_i ds[i][b] x_i[j], x_i = [h_i, psi_i];
// b_r[b] -= lr * sum_i ds[i][b]; the mean loss; the buffer is emptied.  A
// thread owns one column of the four rows; sixteen of its loads are in flight
// at once.
__global__ __launch_bounds__(64) void rank_update_kernel(
    float* __restrict__ rank_w, float* __restrict__ rank_b,
    const float* __restrict__ ds, const float* __restrict__ h,
    const float* __restrict__ psi, int d, const int* __restrict__ n_eff,
    float lr, const float* __restrict__ loss, float* __restrict__ loss_out,
    int* __restrict__ count) {
  __shared__ float4 dsh[64];
  const int n = *n_eff, tid = threadIdx.x;
  const int ld = d + SB_PSI;
  const int j = blockIdx.x * 64 + tid;
  dsh[tid] = tid < n ? reinterpret_cast<const float4*>(ds)[tid]
                     : make_float4(0.f, 0.f, 0.f, 0.f);
  __syncthreads();
  if (j < ld) {
    float g[4] = {0.f, 0.f, 0.f, 0.f};
    const float* x = j < d ? h + j : psi + (j - d);
    const size_t ldx = j < d ? d : SB_PSI;
    for (int i0 = 0; i0 < n; i0 += 16) {
      float v[16];
#pragma unroll
      for (int u = 0; u < 16; ++u) v[u] = x[(size_t)min(i0 + u, n - 1) * ldx];
#pragma unroll
      for (int u = 0; u < 16; ++u) {
        const float4 s = dsh[i0 + u];   // zero past the n positions
        g[0] += s.x * v[u];
        g[1] += s.y * v[u];
        g[2] += s.z * v[u];
        g[3] += s.w * v[u];
      }
    }
#pragma unroll
    for (int b = 0; b < 4; ++b) rank_w[(size_t)b * ld + j] -= lr * g[b];
  }
  if (blockIdx.x == 0) {   // one wave: lane i holds position i
    const float4 s = dsh[tid];
    const float gb[4] = {wave_sum(s.x), wave_sum(s.y), wave_sum(s.z),
                         wave_sum(s.w)};
    const float t = wave_sum(tid < n ? loss[tid] : 0.f);
    if (tid == 0) {
#pragma unroll
      for (int b = 0; b < 4; ++b) rank_b[b] -= lr * gb[b];
      if (loss_out) *loss_out = n > 0 ? t / (float)n : 0.f;
      *count = 0;
    }
  }
}

template <typename T>
void launch_adapt_prep(const float* h, const int* count, int cap,
                       const float* g, float eps, int d, T* A, int* n_eff,
                       hipStream_t st) {
  adapt_prep_kernel<T><<<cap, 1024, 0, st>>>(h, count, cap, g, eps, d, A,
                                            n_eff);
}

template <typename T>
void launch_lm_update(T* W, int Vd, int d, const float* G, const T* A, T* At,
                      const int* n_eff, float lr, hipStream_t st) {
  if constexpr (sizeof(T) == 2) {
    lm_operand_kernel<<<d / 64, 256, 0, st>>>(A, d, n_eff, At);
    // two workgroups fit a CU: halves of the columns, for rounds of 512 even
    // enough with a full vocabulary's 1002 groups of row blocks (2004
    // workgroups).  A reduced vocabulary fills less of the chip: 500
    // workgroups at 32000 tokens, 126 at 8000; finer splits are not measured
    const int kb_per = (d / 64 + 1) / 2;
    lm_update_kernel<<<dim3((Vd / 32 + 3) / 4, 2), 256, 0, st>>>(
        W, Vd, d, G, At, n_eff, lr, kb_per);
  } else {
    constexpr int CW = 128;
    lm_update_f32_kernel<CW><<<dim3(Vd / kStripeRows, d / CW), 256, 0, st>>>(
        W, Vd, d, G, A, n_eff, lr);
  }
}

void launch_rank_update(float* rank_w, float* rank_b, const float* ds,
                        const float* h, const float* psi, int d,
                        const int* n_eff, float lr, const float* loss,
                        float* loss_out, int* count, hipStream_t st) {
  rank_update_kernel<<<(d + SB_PSI + 63) / 64, 64, 0, st>>>(
      rank_w, rank_b, ds, h, psi, d, n_eff, lr, loss, loss_out, count);
}

// Granularity of d_model that a head update accepts.  For fp32 the columns of
// a workgroup; the bf16 kernels work in 64 columns, the interface's 256 stands.
int adapt_column_width(int elem_bytes) { return elem_bytes == 2 ? 256 : 128; }
int adapt_stripe_rows() { return kStripeRows; }

template void launch_adapt_prep<float>(const float*, const int*, int,
                                       const float*, float, int, float*, int*,
                                       hipStream_t);
template void launch_adapt_prep<bf16_t>(const float*, const int*, int,
                                        const float*, float, int, bf16_t*,
                                        int*, hipStream_t);
template void launch_lm_update<float>(float*, int, int, const float*,
                                      const float*, float*, const int*,
                                      float, hipStream_t);
template void launch_lm_update<bf16_t>(bf16_t*, int, int, const float*,
                                       const bf16_t*, bf16_t*, const int*,
                                       float, hipStream_t);

}  // namespace sb
