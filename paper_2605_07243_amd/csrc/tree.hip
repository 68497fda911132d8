// Tree bookkeeping on the device: row plans for each forward call, rank-
// guided sibling attachment and next-block starts (Sec. 3.2, Alg. 2), the
// greedy acceptance walk and the commit copies.  Small single-workgroup or
// one-wave-per-sequence kernels; nothing here synchronises with the host.
#include <float.h>

#include "bounds.h"
#include "common.h"
#include "kernels.h"
#include "signal.h"
#include "specblock.h"

namespace sb {

// ---------------------------------------------------------------------------
// Block 1: reset the tree to the root (node 0, one start) and count the
// W_cond rows (one per sequence).
__global__ void block1_reset_kernel(TreeDims td, sb_tree t,
                                    const int* __restrict__ root,
                                    int* __restrict__ n_aux) {
  for (int s = threadIdx.x; s < td.S; s += blockDim.x) {
    const size_t b = (size_t)s * td.budget;
    t.n_nodes[s] = 1;
    t.token[b] = checked_index(root[s], td.V, td.err, kDevToken);
    t.parent[b] = -1;
    t.depth[b] = 0;
    t.row[b] = -1;
    t.rank[b] = 0;
    t.logp[b] = 0.f;
    t.cum_logp[b] = 0.f;
    for (int w = 0; w < td.bw; ++w) t.anc[b * td.bw + w] = (w == 0) ? 1u : 0u;
    t.n_rows[s] = 0;
    t.n_starts[s] = 1;
    t.starts[(size_t)s * td.B_max] = 0;
  }
  if (threadIdx.x == 0) *n_aux = td.S;
}

// Rows of one block expansion: start b of sequence s gets rows k = 1..K at
// positions pos(start) + k; they see the rows visible to the row that
// proposed the start plus their own block's rows <= k.
// The call rows are also exported (call_seq / call_row [out_cap], -1 past
// the rows, n_call).
__global__ void plan_block_kernel(TreeDims td, int m, sb_tree t,
                                  const int* __restrict__ T, CallPlan p,
                                  int* __restrict__ blk_row0,
                                  int* __restrict__ blk_nst, int out_cap,
                                  int* __restrict__ call_seq,
                                  int* __restrict__ call_row,
                                  int* __restrict__ n_call) {
  __shared__ int cnt[SB_MAX_SEQS], old[SB_MAX_SEQS], off[SB_MAX_SEQS + 1];
  __shared__ int Ts[SB_MAX_SEQS];
  const int K = td.K, rw = td.rw;
  const int tid = threadIdx.x;
  // every sequence's counts loaded at once (one thread each), offsets by a
  // scan in LDS, then one pass over all rows: no chain of dependent global
  // round trips per sequence
  if (tid < td.S) {
    const int s = tid;
    const int n_old = t.n_rows[s];
    int nst = min(t.n_starts[s], td.B_max);
    nst = max(0, min(nst, (td.row_cap - n_old) / K));
    cnt[s] = nst * K;
    old[s] = n_old;
    Ts[s] = T[s];
    p.prefix_len[s] = Ts[s];
    p.seg_len[s] = n_old + nst * K;
    blk_row0[s] = n_old;
    blk_nst[s] = nst;
  }
  __syncthreads();
  if (tid == 0) {
    int o = 0;
    for (int s = 0; s < td.S; ++s) {
      off[s] = o;
      o += cnt[s];
    }
    off[td.S] = o;
  }
  __syncthreads();
  const int total = off[td.S];
  if (tid <= td.S) p.seq_off[tid] = off[tid];
  if (tid == 0) {
    *p.n = total;
    *n_call = total;
  }
  for (int i = total + tid; i < out_cap; i += blockDim.x) {
    call_seq[i] = -1;
    call_row[i] = -1;
  }
  for (int i = tid; i < total; i += blockDim.x) {
    int s = 0;
    while (off[s + 1] <= i) ++s;
    const int j = i - off[s];
    const int b = j / K, k = j % K + 1;
    const int lr = old[s] + j;
    call_seq[i] = s;
    call_row[i] = lr;
    const int sn = t.starts[(size_t)s * td.B_max + b];
    const size_t nidx = (size_t)s * td.budget + sn;
    const int srow = t.row[nidx];
    const int pos = Ts[s] + t.depth[nidx] + k;
    p.seq[i] = s;
    p.slot[i] = lr;
    p.pos[i] = pos;
    p.token[i] = t.token[nidx];
    p.k[i] = k;
    p.pred[i] = k > 1 ? i - 1 : i;
    p.cond[i] = (m == 1 || srow < 0) ? s : s * td.row_cap + srow;
    p.out_row[i] = s * td.row_cap + lr;
    p.kv_dst[i] = -1;
    const size_t rbase = (size_t)s * td.row_cap;
    for (int w = 0; w < rw; ++w) {
      uint32_t bits = (m > 1 && srow >= 0) ? t.row_vis[(rbase + srow) * rw + w] : 0u;
      // own block rows lr-k+1 .. lr
      for (int q = lr - k + 1; q <= lr; ++q)
        if ((q >> 5) == w) bits |= 1u << (q & 31);
      t.row_vis[(rbase + lr) * rw + w] = bits;
      p.vis[(size_t)i * p.vis_words + w] = bits;
    }
    t.row_block[rbase + lr] = m;
    t.row_start[rbase + lr] = sn;
    t.row_k[rbase + lr] = k;
    t.row_pos[rbase + lr] = pos;
  }
  __syncthreads();
  if (tid < td.S) t.n_rows[tid] = old[tid] + cnt[tid];
}

// Sibling attachment of one block in (k, start, rank) order within the
// budget, then the next block's starts.  One wave per sequence; lane b owns
// start b of the block.  The block's row results (branch, bucket, lse,
// top-10 ids and logits: rows row0 .. row0 + nst K - 1, at most 512) are
// staged in LDS with coalesced loads before the attachment loop, and the
// cumulative log-probability of every new node that qualifies as a next
// start is kept in LDS, so that the loop and the start selection read no
// global memory.
constexpr int kAttachRows = 512;
__global__ __launch_bounds__(64) void attach_kernel(
    TreeDims td, sb_tree t, const int* __restrict__ topk_id,
    const float* __restrict__ topk_logit, const float* __restrict__ lse,
    const int* __restrict__ bucket, const int* __restrict__ branch,
    const int* __restrict__ blk_row0, const int* __restrict__ blk_nst) {
  __shared__ int ids_s[kAttachRows * SB_TOPK_K];
  __shared__ float lg_s[kAttachRows * SB_TOPK_K];
  __shared__ float lse_s[kAttachRows];
  __shared__ int br_s[kAttachRows];
  __shared__ int bk_s[kAttachRows];
  __shared__ float cand_s[kAttachRows];   // new node id - first_new
  __shared__ uint32_t anc_s[SB_MAX_ANC_WORDS][64];   // a lane's chain node
  const int s = blockIdx.x;
  const int lane = threadIdx.x;
  const int K = td.K, budget = td.budget, bw = td.bw;
  const int nst = blk_nst[s];
  const int row0 = blk_row0[s];
  const size_t nb = (size_t)s * budget;
  const size_t rb = (size_t)s * td.row_cap;
  const int nrows = min(nst * K, kAttachRows);
  const bool mine = lane < nst;
  // independent loads first: the block's rows, the start nodes
  for (int e = lane; e < nrows * SB_TOPK_K; e += 64) {
    ids_s[e] = topk_id[(rb + row0) * SB_TOPK_K + e];
    lg_s[e] = topk_logit[(rb + row0) * SB_TOPK_K + e];
  }
  for (int j = lane; j < nrows; j += 64) {
    lse_s[j] = lse[rb + row0 + j];
    br_s[j] = branch[rb + row0 + j];
    bk_s[j] = bucket[rb + row0 + j];
  }
  for (int j = lane; j < budget; j += 64) cand_s[j] = -FLT_MAX;
  int chain = mine ? t.starts[(size_t)s * td.B_max + lane] : 0;
  bool alive = mine;
  int chain_depth = 0;
  float chain_cum = 0.f;
  if (mine) {
    chain_depth = t.depth[nb + chain];
    chain_cum = t.cum_logp[nb + chain];
#pragma unroll 2
    for (int w = 0; w < bw; ++w) anc_s[w][lane] = t.anc[(nb + chain) * bw + w];
  }
  int nn = t.n_nodes[s];
  const int first_new = nn;
  __syncthreads();
  for (int k = 1; k <= K; ++k) {
    const int j = lane * K + (k - 1);          // block-local row
    const int r = row0 + j;
    const bool live = mine && alive && j < nrows;
    const int want = live ? br_s[j] : 0;   // 0..10
    int total;
    const int excl = wave_excl_scan_small<4>(want, total);
    const int id0 = nn + excl;
    if (live) {
      const float l0 = lse_s[j];
      const int bk = bk_s[j];
      const bool cand_row = bk == 1 || bk == 2;
#pragma unroll 1
      for (int rank = 1; rank <= want; ++rank) {
        const int id = id0 + rank - 1;
        if (id >= budget) break;
        const int q = j * SB_TOPK_K + (rank - 1);
        const float lp = lg_s[q] - l0;
        t.token[nb + id] = ids_s[q];
        t.parent[nb + id] = chain;
        t.depth[nb + id] = chain_depth + 1;
        t.row[nb + id] = r;
        t.rank[nb + id] = rank;
        t.logp[nb + id] = lp;
        t.cum_logp[nb + id] = chain_cum + lp;
        if (rank >= 2 && cand_row) cand_s[id - first_new] = chain_cum + lp;
#pragma unroll 2
        for (int w = 0; w < bw; ++w)
          t.anc[(nb + id) * bw + w] =
              anc_s[w][lane] | ((id >> 5) == w ? (1u << (id & 31)) : 0u);
      }
      if (want >= 1 && id0 < budget) {
        chain = id0;
        chain_depth += 1;
        chain_cum += lg_s[j * SB_TOPK_K] - l0;
        anc_s[id0 >> 5][lane] |= 1u << (id0 & 31);
      } else {
        alive = false;
      }
    }
    nn = min(budget, nn + total);
  }
  if (lane == 0) t.n_nodes[s] = nn;
  __syncthreads();   // candidate values of all lanes visible below
  // next-block starts: chain ends first, then rank >= 2 siblings of b1/b2
  // rows by cumulative log-probability (ties: lower node id)
  int* out = t.starts + (size_t)s * td.B_max;
  if (nn >= budget) {
    if (lane == 0) t.n_starts[s] = 0;
    return;
  }
  int n_ends;
  const int is_end = (mine && alive) ? 1 : 0;
  const int e_excl = wave_excl_scan_small<1>(is_end, n_ends);
  if (is_end && e_excl < td.B_max) out[e_excl] = chain;
  int taken = min(n_ends, td.B_max);
  // candidates of a lane: nodes first_new + lane + 64 q (values in registers;
  // most blocks add at most 64 nodes, and then one round of q is all); a NaN
  // is no candidate and must not hide the lane's others below
  const int nq = (nn - first_new + 63) >> 6;
  float cand[8];
#pragma unroll
  for (int q = 0; q < 8; ++q) {
    const int j = lane + 64 * q;
    cand[q] = q < nq && first_new + j < nn ? fmaxf(cand_s[j], -FLT_MAX) : -FLT_MAX;
  }
#pragma unroll 1
  while (taken < td.B_max) {
    float v = cand[0];
    int q0 = 0;
    if (nq > 1) {
#pragma unroll
      for (int q = 1; q < 8; ++q)
        if (cand[q] > v) {          // equal values: the lower id stays
          v = cand[q];
          q0 = q;
        }
    }
    int id = v > -FLT_MAX ? first_new + lane + 64 * q0 : 0x7FFFFFFF;
    wave_best_pair(v, id);
    if (id == 0x7FFFFFFF) break;
    if (lane == 0) out[taken] = id;
    const int j = id - first_new;
    if ((j & 63) == lane) {
#pragma unroll
      for (int q = 0; q < 8; ++q)
        if (q == (j >> 6)) cand[q] = -FLT_MAX;
    }
    ++taken;
  }
  if (lane == 0) t.n_starts[s] = taken;
}

// Verification rows: every node of every tree at T + depth, seeing its
// ancestors-or-self.
__global__ void plan_verify_kernel(TreeDims td, sb_tree t,
                                   const int* __restrict__ T, CallPlan p) {
  __shared__ int off[SB_MAX_SEQS + 1];
  __shared__ int Ts[SB_MAX_SEQS];
  const int tid = threadIdx.x;
  // counts loaded at once, offsets by a scan in LDS, one pass over all rows
  if (tid < td.S) {
    off[tid + 1] = min(t.n_nodes[tid], td.budget);
    Ts[tid] = T[tid];
  }
  __syncthreads();
  if (tid == 0) {
    off[0] = 0;
    for (int s = 0; s < td.S; ++s) off[s + 1] += off[s];
  }
  __syncthreads();
  const int total = off[td.S];
  if (tid < td.S) {
    p.prefix_len[tid] = Ts[tid];
    p.seg_len[tid] = off[tid + 1] - off[tid];
  }
  if (tid <= td.S) p.seq_off[tid] = off[tid];
  if (tid == 0) *p.n = total;
  for (int i = tid; i < total; i += blockDim.x) {
    int s = 0;
    while (off[s + 1] <= i) ++s;
    const int j = i - off[s];
    const size_t nidx = (size_t)s * td.budget + j;
    p.seq[i] = s;
    p.slot[i] = j;
    p.pos[i] = Ts[s] + t.depth[nidx];
    p.token[i] = t.token[nidx];
    p.k[i] = 1;
    p.pred[i] = i;
    p.cond[i] = -1;
    p.out_row[i] = s * td.budget + j;
    p.kv_dst[i] = -1;
    for (int w = 0; w < p.vis_words; ++w)
      p.vis[(size_t)i * p.vis_words + w] = w < td.bw ? t.anc[nidx * td.bw + w] : 0u;
  }
}

// Greedy acceptance walk, one workgroup per sequence: the tree is staged in
// LDS, wave 0 walks, and the whole workgroup computes the verifier-derived
// signal when it is asked for (g.r).
template <typename T>
__global__ __launch_bounds__(256) void accept_kernel(TreeDims td, sb_tree t,
                                                     const int* __restrict__ argmax,
                                                     sb_accept_out out,
                                                     SignalArgs g) {
  __shared__ int par[512], tok[512], am[512];
  __shared__ int sh_cur, sh_bonus;
  const int s = blockIdx.x;
  const int lane = threadIdx.x & 63;
  const size_t nb = (size_t)s * td.budget;
  const int nn = min(t.n_nodes[s], td.budget);
  const int path_cap = td.M * td.K;
  // (node 0's argmax is read whatever n_nodes says)
  for (int j = threadIdx.x; j < td.budget; j += 256) {
    par[j] = t.parent[nb + j];
    tok[j] = t.token[nb + j];
    am[j] = argmax[nb + j];
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    int cur = 0, a = 0;
    while (a < path_cap) {
      const int gr = am[cur];
      int best = 0x7FFFFFFF;
      for (int j = 1 + lane; j < nn; j += 64)
        if (par[j] == cur && tok[j] == gr) best = min(best, j);
      best = wave_min_i(best);
      if (best == 0x7FFFFFFF) break;
      if (lane == 0) out.path[(size_t)s * path_cap + a] = best;
      cur = best;
      ++a;
    }
    if (lane == 0) {
      out.n_accepted[s] = a;
      out.bonus[s] = am[cur];
      sh_cur = cur;
      sh_bonus = am[cur];
    }
  }
  if (g.r == nullptr) return;
  __syncthreads();
  reject_signal_block<T>(td, t, s, sh_cur, sh_bonus, g);
}

// Commit planning: last accepted node, the drafter row continuing it (or a
// catch-up row when the tree has none) and the catch-up call plan.  One
// workgroup: a wave per sequence, then lane s of wave 0 plans sequence s's
// catch-up row (a serial walk over the sequences took 18 us for 16).
__global__ __launch_bounds__(1024) void commit_plan_kernel(
    TreeDims td, sb_tree t, sb_accept_out acc, const int* __restrict__ T,
    CommitInfo ci, CallPlan fb, int* __restrict__ taps_idx,
    int* __restrict__ n_aux) {
  __shared__ int a_s[SB_MAX_SEQS], cur_s[SB_MAX_SEQS], cont_s[SB_MAX_SEQS];
  __shared__ int T_s[SB_MAX_SEQS];
  const int path_cap = td.M * td.K;
  const int lane = threadIdx.x & 63;
  for (int s = threadIdx.x >> 6; s < td.S; s += 16) {
    const int a = acc.n_accepted[s];
    const int cur = a > 0 ? acc.path[(size_t)s * path_cap + a - 1] : 0;
    const int Ts = T[s];
    const int cont = continuing_row(td, t, s, cur);
    if (lane == 0) {
      ci.T_old[s] = T_s[s] = Ts;
      ci.a[s] = a_s[s] = a;
      ci.cur[s] = cur_s[s] = cur;
      ci.cont[s] = cont_s[s] = cont;
    }
  }
  __syncthreads();
  const int s = threadIdx.x;
  if (s >= 64) return;
  const bool mine = s < td.S;
  const uint64_t need = __ballot(mine && cont_s[s] < 0);
  if (!mine) return;
  const int o = __popcll(need & ((1ull << s) - 1ull));
  fb.seq_off[s] = o;
  fb.prefix_len[s] = T_s[s] + a_s[s];   // drafter entries 1..T+a
  fb.seg_len[s] = cont_s[s] < 0 ? 1 : 0;
  if (cont_s[s] < 0) {
    const size_t nidx = (size_t)s * td.budget + cur_s[s];
    fb.seq[o] = s;
    fb.slot[o] = 0;
    fb.pos[o] = T_s[s] + a_s[s] + 1;
    fb.token[o] = t.token[nidx];
    fb.k[o] = 1;
    fb.pred[o] = o;
    fb.cond[o] = o;
    fb.out_row[o] = -1;
    fb.kv_dst[o] = T_s[s] + a_s[s];
    for (int w = 0; w < fb.vis_words; ++w)
      fb.vis[(size_t)o * fb.vis_words + w] = (w == 0) ? 1u : 0u;
    taps_idx[o] = s * td.budget + max(t.parent[nidx], 0);
  }
  if (s == 0) {
    const int n = __popcll(need);
    fb.seq_off[td.S] = n;
    *fb.n = n;
    *n_aux = n;
  }
}

// Copy committed K/V entries.  Target: the root and accepted nodes (verify
// scratch slot = node id) to entries T .. T+a.  Drafter: the rows that
// proposed the accepted nodes to entries T .. T+a-1 (positions T+1 ..
// T+a), and the continuing row, if any, to entry T+a.  Grid (sequence, entry,
// (layer, KV head)): the target's layers, then the drafter's, four heads per
// workgroup, then one slice that sets the new sequence state.
template <typename T>
__global__ __launch_bounds__(512) void commit_apply_kernel(
    TreeDims td, sb_tree t, sb_accept_out acc, CommitInfo ci, KVPools tkv,
    int tl, KVPools dkv, int dl, int pool_seqs, int Hkv, int hd, sb_seqs sq,
    const float* __restrict__ taps) {
  const int s = blockIdx.x;
  const int j = blockIdx.y;               // 0 .. M K
  const int a = ci.a[s];
  const int T0 = ci.T_old[s];
  const int z = 4 * blockIdx.z + (threadIdx.x >> 7);
  if (blockIdx.z == gridDim.z - 1) {
    if (j != 0) return;
    // cond_taps = taps of the last accepted node: 3 d floats (d % 32 == 0);
    // the destination cannot alias the taps
    const float4* __restrict__ src = reinterpret_cast<const float4*>(
        taps + ((size_t)s * td.budget + ci.cur[s]) * 3 * td.d);
    float4* __restrict__ dst =
        reinterpret_cast<float4*>(sq.cond_taps + (size_t)s * 3 * td.d);
#pragma unroll 4
    for (int e = threadIdx.x; e < 3 * td.d / 4; e += 512) dst[e] = src[e];
    if (threadIdx.x == 0) {
      sq.T[s] = T0 + a + 1;
      sq.root[s] = acc.bonus[s];
    }
    return;
  }
  if (z >= (tl + dl) * Hkv) return;
  const bool drafter = z >= tl * Hkv;
  const KVPools& kv = drafter ? dkv : tkv;
  const int lz = z - (drafter ? tl * Hkv : 0);
  const int l = lz / Hkv, kh = lz % Hkv;
  const int path_cap = td.M * td.K;
  int src_slot, dst;
  if (!drafter) {
    if (j > a) return;
    src_slot = j == 0 ? 0 : acc.path[(size_t)s * path_cap + j - 1];
    dst = T0 + j;
  } else {
    if (j < a) {
      const int node = acc.path[(size_t)s * path_cap + j];
      src_slot = t.row[(size_t)s * td.budget + node];
      dst = T0 + j;
    } else if (j == a && ci.cont[s] >= 0) {
      src_slot = ci.cont[s];
      dst = T0 + a;
    } else {
      return;
    }
  }
  // entries outside the page table (a negative T included) are not written
  if (dst < 0 || (dst >> 4) >= kv.max_pages) return;
  const int page_i = dst >> 4;
  const int page = checked_index(kv.page_table[(size_t)s * kv.max_pages + page_i],
                                 kv.n_pages, kv.err, kDevPage);
  const int sl = dst & 15;
  const int sp = src_slot >> 4, ss = src_slot & 15;
  if (sp >= kv.seg_pages) return;
  const size_t lay = (size_t)l;
  const size_t src_page = ((lay * pool_seqs + s) * kv.seg_pages + sp) * Hkv + kh;
  const size_t dst_page = (lay * kv.n_pages + page) * Hkv + kh;
  const T* sk = static_cast<const T*>(kv.seg_k) + src_page * 16 * hd;
  const T* sv = static_cast<const T*>(kv.seg_v) + src_page * 16 * hd;
  T* dk = static_cast<T*>(kv.k) + dst_page * 16 * hd;
  T* dv = static_cast<T*>(kv.v) + dst_page * 16 * hd;
  for (int e = threadIdx.x & 127; e < hd; e += 128) {
    dk[sl * hd + e] = sk[ss * hd + e];
    dv[e * 16 + sl] = sv[e * 16 + ss];
  }
}

// Call plan of a prefill pass, one wave per piece: prompt position a + t of
// the piece's sequence.  Target rows run token x_{a+t} at that position and
// leave their taps in row 1 + i of the tap buffer (row 0: the position before
// the pass).  Drafter catch-up rows are K = 1 blocks started at position
// a + t with token x_{a+t}, at position a + t + 1, conditioned on the taps of
// position a + t - 1, row i of the tap buffer (none for position 0).
__global__ __launch_bounds__(kPieceRows) void plan_prefill_kernel(
    PrefillPass pass, int drafter, const int* __restrict__ prompt, int ld,
    CallPlan p, int* __restrict__ n_aux, int V, int* __restrict__ err) {
  const int j = blockIdx.x, t = threadIdx.x;
  const int i0 = pass.row0[j], n = pass.row0[j + 1] - i0;
  const int a = pass.a[j], s = pass.seq[j];
  if (t == 0) {
    p.seq_off[j] = i0;
    p.prefix_len[j] = a + n;
    p.seg_len[j] = 0;
    p.kv_row[j] = s;
    if (j == 0) {
      p.seq_off[pass.n_pieces] = pass.n_rows;
      *p.n = pass.n_rows;
      *n_aux = pass.n_rows;
    }
  }
  if (t >= n) return;
  const int i = i0 + t;
  p.seq[i] = s;
  p.slot[i] = 0;
  p.pos[i] = a + t + drafter;
  p.token[i] = checked_index(prompt[(size_t)s * ld + a + t], V, err, kDevToken);
  p.k[i] = 1;
  p.pred[i] = i;
  p.cond[i] = drafter && a + t >= 1 ? i : -1;
  p.out_row[i] = drafter ? -1 : 1 + i;
  p.kv_dst[i] = a + t;
}

// Prompts that end in a pass, one workgroup each: T = len, cond_taps = the
// taps of position len - 1, and the LM-head operand of that row (the next
// row of `out`) with its sequence, for one LM head after the last pass.
template <typename T>
__global__ __launch_bounds__(1024) void prefill_ends_kernel(
    PrefillEnds ends, sb_seqs sq, int d, const float* __restrict__ taps_pf,
    const T* __restrict__ src, T* __restrict__ out, int* __restrict__ n,
    int* __restrict__ out_seq) {
  const int j = blockIdx.x, s = ends.seq[j];
  constexpr int V = 16 / sizeof(T);       // d % 32 == 0
  const uint4* __restrict__ a =
      reinterpret_cast<const uint4*>(src + (size_t)ends.row[j] * d);
  uint4* __restrict__ o =
      reinterpret_cast<uint4*>(out + (size_t)(ends.first + j) * d);
  for (int e = threadIdx.x; e < d / V; e += 1024) o[e] = a[e];
  float4* __restrict__ ct =
      reinterpret_cast<float4*>(sq.cond_taps + (size_t)s * 3 * d);
  const float4* __restrict__ tp = reinterpret_cast<const float4*>(
      taps_pf + (size_t)(1 + ends.row[j]) * 3 * d);
  for (int e = threadIdx.x; e < 3 * d / 4; e += 1024) ct[e] = tp[e];
  if (threadIdx.x == 0) {
    sq.T[s] = ends.len[j];
    out_seq[ends.first + j] = s;
    if (j == 0) *n = ends.first + ends.n;
  }
}

__global__ void copy_f32_kernel(float* __restrict__ dst, const float* __restrict__ src,
                                int n) {
  for (int e = blockIdx.x * blockDim.x + threadIdx.x; e < n; e += gridDim.x * blockDim.x)
    dst[e] = src[e];
}

__global__ void set_int_kernel(int* __restrict__ p, int v) { *p = v; }

__global__ void copy_int_kernel(int* __restrict__ dst,
                                const int* __restrict__ src) {
  *dst = *src;
}

// ---------------------------------------------------------------------------
// launchers

void launch_block1_reset(const TreeDims& td, const sb_tree& t, const int* root,
                         int* n_aux, hipStream_t st) {
  block1_reset_kernel<<<1, 64, 0, st>>>(td, t, root, n_aux);
}
void launch_plan_block(const TreeDims& td, int m, const sb_tree& t,
                       const int* T, const CallPlan& p, int* blk_row0,
                       int* blk_nst, int out_cap, int* call_seq,
                       int* call_row, int* n_call, hipStream_t st) {
  plan_block_kernel<<<1, 256, 0, st>>>(td, m, t, T, p, blk_row0, blk_nst,
                                       out_cap, call_seq, call_row, n_call);
}
void launch_attach(const TreeDims& td, const sb_tree& t, const sb_draft_out& o,
                   const int* blk_row0, const int* blk_nst, hipStream_t st) {
  attach_kernel<<<td.S, 64, 0, st>>>(td, t, o.topk_id, o.topk_logit, o.lse,
                                     o.bucket, o.branch, blk_row0, blk_nst);
}
void launch_plan_verify(const TreeDims& td, const sb_tree& t, const int* T,
                        const CallPlan& p, hipStream_t st) {
  plan_verify_kernel<<<1, 256, 0, st>>>(td, t, T, p);
}
void launch_accept(const TreeDims& td, const sb_tree& t, const int* argmax,
                   const sb_accept_out& o, const SignalArgs& g, bool bf16,
                   hipStream_t st) {
  if (bf16)
    accept_kernel<bf16_t><<<td.S, 256, 0, st>>>(td, t, argmax, o, g);
  else
    accept_kernel<float><<<td.S, 256, 0, st>>>(td, t, argmax, o, g);
}
// Adaptation buffer push (Sec. 3.4): each sequence's rejected position
// (the one after its last accepted node) whose drafter row exists appends
// (that row's cached h^(L), the bonus token) to the buffer, in sequence
// order, while room is left.  One workgroup.
__global__ __launch_bounds__(1024) void adapt_push_kernel(
    TreeDims td, sb_tree t, sb_accept_out acc, float* __restrict__ buf_h,
    int* __restrict__ buf_y, int* __restrict__ count, int cap) {
  __shared__ int slot[SB_MAX_SEQS], src[SB_MAX_SEQS];
  const int path_cap = td.M * td.K;
  for (int s = threadIdx.x >> 6; s < td.S; s += 16) {
    const int a = acc.n_accepted[s];
    const int cur = a > 0 ? acc.path[(size_t)s * path_cap + a - 1] : 0;
    const int r = continuing_row(td, t, s, cur);
    if ((threadIdx.x & 63) == 0) src[s] = r;
  }
  __syncthreads();
  if (threadIdx.x == 0) {
    int c = *count;
    for (int s = 0; s < td.S; ++s) {
      slot[s] = (src[s] >= 0 && c < cap) ? c : -1;
      if (slot[s] >= 0) {
        buf_y[slot[s]] = acc.bonus[s];
        ++c;
      }
    }
    *count = c;
  }
  __syncthreads();
  const int d = td.d;
  for (int s = 0; s < td.S; ++s) {
    if (slot[s] < 0) continue;
    const float* hs = t.h_last + ((size_t)s * td.row_cap + src[s]) * d;
    float* hd = buf_h + (size_t)slot[s] * d;
    for (int k = threadIdx.x; k < d; k += 1024) hd[k] = hs[k];
  }
}

void launch_adapt_push(const TreeDims& td, const sb_tree& t,
                       const sb_accept_out& acc, float* buf_h, int* buf_y,
                       int* count, int cap, hipStream_t st) {
  adapt_push_kernel<<<1, 1024, 0, st>>>(td, t, acc, buf_h, buf_y, count, cap);
}

void launch_commit_plan(const TreeDims& td, const sb_tree& t,
                        const sb_accept_out& acc, const int* T,
                        const CommitInfo& ci, const CallPlan& fb,
                        int* taps_idx, int* n_aux, hipStream_t st) {
  commit_plan_kernel<<<1, 1024, 0, st>>>(td, t, acc, T, ci, fb, taps_idx, n_aux);
}
template <typename T>
void launch_commit_apply(const TreeDims& td, const sb_tree& t,
                         const sb_accept_out& acc, const CommitInfo& ci,
                         const KVPools& tkv, int tl, const KVPools& dkv,
                         int dl, int pool_seqs, int Hkv, int hd,
                         const sb_seqs& sq, const float* taps, hipStream_t st) {
  dim3 grid(td.S, td.M * td.K + 1, ((tl + dl) * Hkv + 3) / 4 + 1);
  commit_apply_kernel<T><<<grid, 512, 0, st>>>(td, t, acc, ci, tkv, tl, dkv,
                                               dl, pool_seqs, Hkv, hd, sq, taps);
}
void launch_plan_prefill(const PrefillPass& pass, bool drafter,
                         const int* prompt, int ld, const CallPlan& p,
                         int* n_aux, int V, int* err, hipStream_t st) {
  plan_prefill_kernel<<<pass.n_pieces, kPieceRows, 0, st>>>(
      pass, drafter ? 1 : 0, prompt, ld, p, n_aux, V, err);
}
template <typename T>
void launch_prefill_ends(const PrefillEnds& ends, const sb_seqs& sq, int d,
                         const float* taps_pf, const T* src, T* out, int* n,
                         int* out_seq, hipStream_t st) {
  prefill_ends_kernel<T><<<ends.n, 1024, 0, st>>>(ends, sq, d, taps_pf, src,
                                                  out, n, out_seq);
}
template void launch_prefill_ends<float>(const PrefillEnds&, const sb_seqs&,
                                         int, const float*, const float*,
                                         float*, int*, int*, hipStream_t);
template void launch_prefill_ends<bf16_t>(const PrefillEnds&, const sb_seqs&,
                                          int, const float*, const bf16_t*,
                                          bf16_t*, int*, int*, hipStream_t);
void launch_copy_f32(float* dst, const float* src, int n, hipStream_t st) {
  copy_f32_kernel<<<(n + 255) / 256 < 1024 ? (n + 255) / 256 : 1024, 256, 0,
                    st>>>(dst, src, n);
}
void launch_set_int(int* p, int v, hipStream_t st) {
  set_int_kernel<<<1, 1, 0, st>>>(p, v);
}
void launch_copy_int(int* dst, const int* src, hipStream_t st) {
  copy_int_kernel<<<1, 1, 0, st>>>(dst, src);
}

#define SB_APPLY(T)                                                           \
  template void launch_commit_apply<T>(                                       \
      const TreeDims&, const sb_tree&, const sb_accept_out&,                  \
      const CommitInfo&, const KVPools&, int, const KVPools&, int, int, int,  \
      int, const sb_seqs&, const float*, hipStream_t);
SB_APPLY(float)
SB_APPLY(bf16_t)
#undef SB_APPLY
}  // namespace sb
