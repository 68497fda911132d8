// Stochastic tree verification at temperature T > 0 (the paper's T = 1.0
// decoding setting, Sec. 4).  At node n with target distribution
// p_n = softmax(z_n / T) the children are tested in node-id order as
// point-mass drafts against the residual distribution (p_n with the tokens
// rejected so far removed and renormalised): child c with token x is taken
// when u_acc[c] < r(x), else x leaves the residual.  A child whose token was
// already rejected has residual probability zero and is skipped.  When no
// child is taken, the bonus token is drawn from the residual by inverse
// transform over increasing token ids with u_bonus[n].  A row with a logit
// that is NaN or +inf has no distribution: no child is taken there, and the
// bonus is token 0.  Every emitted token
// is then distributed as the target's (speculative sampling applied
// recursively over a node's candidates).
//
// Two launches.  The first reads every verified node's row once and leaves,
// per block of 1024 tokens, the maximum x and the sum of exp(x - maximum) of
// x = z / T, the sum in float64 (bound by HBM: 613 rows of 128256 logits in
// 53 us, 5.9 TB/s; reading only the rows that the walk visits, one workgroup
// per sequence, took 123 us for the longest of 16 walks, as a CU reads a cold
// row in about 12 us).  The second is one wave per sequence: a node's
// log-sum-exp is a merge of its blocks, and the bonus draw scans the block
// masses for the block that the target falls into, so that it reads 1024
// logits of the row and not all of it (blocks that hold a rejected token are
// summed again without it): 44 -> 12 us without the signal.
#include <float.h>

#include "common.h"
#include "kernels.h"
#include "signal.h"
#include "specblock.h"

namespace sb {

namespace {

constexpr int kThreads = 256;
constexpr int kTileBlocks = 16;       // blocks per workgroup of the first pass
constexpr int kMaxBlocks = 256;       // V <= 262144
constexpr int kLaneBlocks = kMaxBlocks / 64;
constexpr int kMaxKids = 64;          // children tested per node (a node has
                                      // at most 2 * SB_TOPK: its continuing
                                      // row and the first row of a block
                                      // started at it)

__device__ __forceinline__ double wave_sum_d(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o, SB_WAVE);
  return v;
}

// Rows of sequences before s in call-row order (sequence-major, node order);
// called by a whole wave.
__device__ __forceinline__ int row_offset(const int* __restrict__ n_nodes,
                                          int s, int budget) {
  const int lane = threadIdx.x & 63;
  return wave_sum_i(lane < s ? min(n_nodes[lane], budget) : 0);
}

// A wave's 1024 tokens of a block, four float4 a lane; -inf (exp = 0) past
// the vocabulary.  QS: token stride between a lane's float4 (256: one
// contiguous KiB per load; 4: sixteen consecutive tokens per lane).
template <int QS>
__device__ __forceinline__ void load_block(const float* __restrict__ z, int V,
                                           int b, int lane, float4 (&v)[4]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const int e = kSampleBlock * b + QS * q + (QS == 256 ? 4 : 16) * lane;
    v[q] = e < V ? *reinterpret_cast<const float4*>(z + e)
                 : make_float4(-INFINITY, -INFINITY, -INFINITY, -INFINITY);
  }
}

// exp(x - ref) of a lane's sixteen consecutive tokens of a block, without the
// rejected ones.
__device__ __forceinline__ void block_probs(const float4 (&v)[4], float inv_t,
                                            float ref, int x0, const int* rej,
                                            int nrej, float (&p)[16]) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    p[4 * q] = __expf(v[q].x * inv_t - ref);
    p[4 * q + 1] = __expf(v[q].y * inv_t - ref);
    p[4 * q + 2] = __expf(v[q].z * inv_t - ref);
    p[4 * q + 3] = __expf(v[q].w * inv_t - ref);
  }
#pragma unroll 1
  for (int r = 0; r < nrej; ++r) {
    const int x = rej[r] - x0;
#pragma unroll
    for (int i = 0; i < 16; ++i)
      if (x == i) p[i] = 0.f;
  }
}

}  // namespace

// stats[(s * budget + n) * n_blk + b]: block b of node n's row.  One wave per
// block, sixteen blocks per workgroup, all loads of a wave in flight.
// ROWS: every node; the nodes that have children; or the one that the walk
// ended at, if it has none.
enum StatRows { kAllNodes, kInnerNodes, kLastLeaf };
template <StatRows ROWS>
__global__ __launch_bounds__(kThreads) void node_stats_kernel(
    const float* __restrict__ logits, int V, float inv_t,
    const int* __restrict__ n_nodes, const int* __restrict__ parent, int budget,
    int n_blk, const SampleWalk* __restrict__ walk,
    SampleStat* __restrict__ stats) {
  const int s = blockIdx.z;
  const int nn = min(n_nodes[s], budget);
  int n = blockIdx.y;
  if constexpr (ROWS == kLastLeaf) {
    if (!walk[s].leaf) return;
    n = walk[s].cur;
  }
  if (n >= nn) return;
  if constexpr (ROWS == kInnerNodes) {
    bool kids = false;
    for (int j = threadIdx.x; j < nn; j += kThreads)
      kids |= parent[(size_t)s * budget + j] == n;
    if (!__syncthreads_or(kids ? 1 : 0)) return;
  }
  const float* z = logits + (size_t)(row_offset(n_nodes, s, budget) + n) * V;
  const int lane = threadIdx.x & 63;
  const int b0 = blockIdx.x * kTileBlocks + (threadIdx.x >> 6);
  float4 v[4][4];
#pragma unroll
  for (int k = 0; k < 4; ++k)
    load_block<256>(z, b0 + 4 * k < n_blk ? V : 0, b0 + 4 * k, lane, v[k]);
#pragma unroll
  for (int k = 0; k < 4; ++k) {
    const int b = b0 + 4 * k;
    if (b >= n_blk) break;
    float m = -INFINITY;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      m = fmaxf(m, fmaxf(fmaxf(v[k][q].x, v[k][q].y), fmaxf(v[k][q].z, v[k][q].w)));
    m = wave_max(m);
    const float ref = m * inv_t;
    double sum = 0.0;
    if (ref > -INFINITY) {      // (a logit of the type's lowest value counts)
#pragma unroll
      for (int q = 0; q < 4; ++q)
        sum += ((double)__expf(v[k][q].x * inv_t - ref) +
                (double)__expf(v[k][q].y * inv_t - ref)) +
               ((double)__expf(v[k][q].z * inv_t - ref) +
                (double)__expf(v[k][q].w * inv_t - ref));
    }
    sum = wave_sum_d(sum);
    if (lane == 0)
      stats[((size_t)s * budget + n) * n_blk + b] = SampleStat{sum, ref, 0.f};
  }
}

// A node's blocks, kLaneBlocks consecutive ones a lane, and its log-sum-exp.
__device__ __forceinline__ void load_stats(const SampleStat* __restrict__ row,
                                           int n_blk, int lane,
                                           float (&bm)[kLaneBlocks],
                                           double (&bs)[kLaneBlocks]) {
#pragma unroll
  for (int k = 0; k < kLaneBlocks; ++k) {
    const int b = kLaneBlocks * lane + k;
    SampleStat e{0.0, -FLT_MAX, 0.f};
    if (b < n_blk) e = row[b];
    bm[k] = e.m;
    bs[k] = e.s;
  }
}
__device__ __forceinline__ float merge_stats(const float (&bm)[kLaneBlocks],
                                             const double (&bs)[kLaneBlocks]) {
  float m = bm[0];
#pragma unroll
  for (int k = 1; k < kLaneBlocks; ++k) m = fmaxf(m, bm[k]);
  m = wave_max(m);
  float sum = 0.f;
#pragma unroll
  for (int k = 0; k < kLaneBlocks; ++k)
    if (bs[k] != 0.0) sum += (float)bs[k] * __expf(bm[k] - m);   // NaN stays
  return m + logf(wave_sum(sum));
}

// Nodes of a sequence's tree in LDS.
struct SampleTree {
  int par[512], tok[512];
  float ua[512];
};

// The walk (one wave of the workgroup; the tests are lane 0's).
__device__ __forceinline__ void sample_walk(
    const TreeDims& td, const sb_tree& t, const SampleTree& tr, int s,
    const float* __restrict__ logits, int V, float inv_t,
    const SampleStat* __restrict__ stats, int n_blk, const sb_accept_out& out,
    SampleWalk& wk) {
  __shared__ int kid[kMaxKids];
  __shared__ float kp[kMaxKids];
  __shared__ int sh_next, sh_nrej;
  const int lane = threadIdx.x & 63;
  const size_t nb = (size_t)s * td.budget;
  const int nn = min(t.n_nodes[s], td.budget);
  const int off = row_offset(t.n_nodes, s, td.budget);
  const int path_cap = td.M * td.K;
  int cur = 0, a = 0, nk = 0;
#pragma unroll 1
  while (true) {
    const float* z = logits + (size_t)(off + cur) * V;
    float bm[kLaneBlocks];
    double bs[kLaneBlocks];
    load_stats(stats + (nb + cur) * n_blk, n_blk, lane, bm, bs);
    // children of cur in node-id order (ballot compaction), their logits on
    // the way while the statistics are merged
    nk = 0;
    for (int j0 = 1; j0 < nn; j0 += 64) {
      const int j = j0 + lane;
      const bool f = j < nn && tr.par[j] == cur;
      const uint64_t mk = __ballot(f);
      const int pos = nk + __popcll(mk & ((1ull << lane) - 1ull));
      if (f && pos < kMaxKids) kid[pos] = j;
      nk += __popcll(mk);
    }
    nk = min(nk, kMaxKids);
    wave_lds_sync();
    float zk = -INFINITY;
    if (lane < nk) {
      const int x = tr.tok[kid[lane]];
      // a token outside the vocabulary has no target mass
      if (x >= 0 && x < V) zk = z[x];
    }
    // (a leaf's statistics may not be there yet: it has no tests)
    if (nk == 0) {
      if (lane == 0) sh_nrej = 0;
      break;
    }
    const float l = merge_stats(bm, bs);
    if (lane < nk) kp[lane] = zk > -INFINITY ? __expf(zk * inv_t - l) : 0.f;
    wave_lds_sync();
    // sequential tests (lane 0), result broadcast through LDS
    if (lane == 0) {
      int next = -1, n_rej = 0;
      float mass = 1.f;
#pragma unroll 1
      for (int i = 0; i < nk; ++i) {
        const int x = tr.tok[kid[i]];
        bool seen = false;
        for (int r = 0; r < n_rej; ++r) seen |= wk.rej[r] == x;
        if (seen) continue;
        if (tr.ua[kid[i]] < kp[i] / mass) {
          next = kid[i];
          break;
        }
        wk.rej[n_rej++] = x;
        mass -= kp[i];
      }
      sh_next = next;
      sh_nrej = n_rej;
    }
    wave_lds_sync();
    const int next = sh_next;
    if (next < 0 || a >= path_cap) break;
    if (lane == 0) out.path[(size_t)s * path_cap + a] = next;
    cur = next;
    ++a;
  }
  if (lane == 0) {
    out.n_accepted[s] = a;
    wk.cur = cur;
    wk.leaf = nk == 0;
    wk.nrej = sh_nrej;
  }
}

// The residual draw at the node that the walk ended at (one wave); the bonus
// token, in every lane.
__device__ __forceinline__ int sample_draw(
    const TreeDims& td, const sb_tree& t, int s, const float* __restrict__ logits,
    int V, float inv_t, const SampleStat* __restrict__ stats, int n_blk,
    const float* __restrict__ u_bonus, int cur, int nrej, const int* rej) {
  const int lane = threadIdx.x & 63;
  const size_t nb = (size_t)s * td.budget;
  const float* z =
      logits + (size_t)(row_offset(t.n_nodes, s, td.budget) + cur) * V;
  float bm[kLaneBlocks];
  double bs[kLaneBlocks];
  load_stats(stats + (nb + cur) * n_blk, n_blk, lane, bm, bs);
  const float l = merge_stats(bm, bs);
  // block masses relative to l; those that hold a rejected token again,
  // without the rejected ones
#pragma unroll
  for (int k = 0; k < kLaneBlocks; ++k)
    bs[k] = bs[k] != 0.0 ? bs[k] * (double)__expf(bm[k] - l) : 0.0;
#pragma unroll 1
  for (int r = 0; r < nrej; ++r) {
    const int b = rej[r] / kSampleBlock;
    if (rej[r] < 0 || b >= n_blk) continue;
    float4 v[4];
    load_block<4>(z, V, b, lane, v);
    float p[16];
    block_probs(v, inv_t, l, kSampleBlock * b + 16 * lane, rej, nrej, p);
    double g = 0.0;
#pragma unroll
    for (int i = 0; i < 16; ++i) g += (double)p[i];
    g = wave_sum_d(g);
#pragma unroll
    for (int k = 0; k < kLaneBlocks; ++k)
      if (kLaneBlocks * lane + k == b) bs[k] = g;
  }
  double incl = 0.0;
#pragma unroll
  for (int k = 0; k < kLaneBlocks; ++k) incl += bs[k];
  const double mine = incl;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double x = __shfl_up(incl, o, SB_WAVE);
    if (lane >= o) incl += x;
  }
  const double total = __shfl(incl, 63, SB_WAVE);
  const double target = (double)u_bonus[nb + cur] * total;
  // the first block whose cumulative mass passes the target, and the mass
  // before it; none (rounding): the last block with mass
  int first = kMaxBlocks, last = -1;
  double before = 0.0, lo = incl - mine;
#pragma unroll
  for (int k = 0; k < kLaneBlocks; ++k) {
    const double hi = lo + bs[k];
    if (bs[k] > 0.0) {
      last = kLaneBlocks * lane + k;
      if (first == kMaxBlocks && hi > target) {
        first = kLaneBlocks * lane + k;
        before = lo;
      }
    }
    lo = hi;
  }
  const int b_first = wave_min_i(first);
  const int b_last = -wave_min_i(-last);
  const bool past = b_first == kMaxBlocks;
  const int b = past ? b_last : b_first;
  if (b < 0) return 0;   // no mass at all
  before = __shfl(before, b / kLaneBlocks, SB_WAVE);
  // the token: lane i takes sixteen consecutive ones
  const int x0 = kSampleBlock * b + 16 * lane;
  float4 v[4];
  load_block<4>(z, V, b, lane, v);
  float p[16];
  block_probs(v, inv_t, l, x0, rej, nrej, p);
  double sum16 = 0.0;
#pragma unroll
  for (int i = 0; i < 16; ++i) sum16 += (double)p[i];
  double in16 = sum16;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const double x = __shfl_up(in16, o, SB_WAVE);
    if (lane >= o) in16 += x;
  }
  double acc = before + (in16 - sum16);
  int pick = 0x7FFFFFFF, pos = -1;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    if (p[i] > 0.f) pos = x0 + i;
    acc += (double)p[i];
    if (p[i] > 0.f && acc > target && pick == 0x7FFFFFFF) pick = x0 + i;
  }
  // (rounding can leave the running sum short of the block's end: the
  // block's last token with mass is then the draw)
  const int t_first = wave_min_i(pick);
  const int t_last = -wave_min_i(-pos);
  return !past && t_first != 0x7FFFFFFF ? t_first : max(t_last, 0);
}

// One workgroup per sequence: wave 0 walks (WALK) and draws (DRAW), then all
// four waves compute the verifier-derived signal when it is asked for.  With
// the two phases in separate launches, walk[s] carries the state between.
template <typename T, bool WALK, bool DRAW>
__global__ __launch_bounds__(256) void accept_sample_kernel(
    TreeDims td, sb_tree t, const float* __restrict__ logits, int V,
    float inv_t, const SampleStat* __restrict__ stats, int n_blk,
    const float* __restrict__ u_acc, const float* __restrict__ u_bonus,
    sb_accept_out out, SampleWalk* __restrict__ walk, SignalArgs g) {
  __shared__ SampleWalk wk;
  __shared__ int sh_bonus;
  const int s = blockIdx.x, tid = threadIdx.x;
  __shared__ SampleTree tr;
  if constexpr (WALK) {
    const size_t nb = (size_t)s * td.budget;
    for (int j = tid; j < min(t.n_nodes[s], td.budget); j += 256) {
      tr.par[j] = t.parent[nb + j];
      tr.tok[j] = t.token[nb + j];
      tr.ua[j] = u_acc[nb + j];
    }
    __syncthreads();
  }
  if (tid < 64) {
    if constexpr (WALK) {
      sample_walk(td, t, tr, s, logits, V, inv_t, stats, n_blk, out, wk);
    } else {
      wk.rej[tid] = walk[s].rej[tid];
      if (tid == 0) {
        wk.cur = walk[s].cur;
        wk.nrej = walk[s].nrej;
      }
    }
    wave_lds_sync();
    if constexpr (DRAW) {
      const int b = sample_draw(td, t, s, logits, V, inv_t, stats, n_blk,
                                u_bonus, wk.cur, wk.nrej, wk.rej);
      if (tid == 0) {
        out.bonus[s] = b;
        sh_bonus = b;
      }
    } else {
      walk[s].rej[tid] = tid < wk.nrej ? wk.rej[tid] : 0;
      if (tid == 0) {
        walk[s].cur = wk.cur;
        walk[s].leaf = wk.leaf;
        walk[s].nrej = wk.nrej;
      }
    }
  }
  if constexpr (DRAW) {
    if (g.r == nullptr) return;
    __syncthreads();
    reject_signal_block<T>(td, t, s, wk.cur, sh_bonus, g);
  }
}

int sample_blocks(int V) { return (V + kSampleBlock - 1) / kSampleBlock; }
int sample_max_vocab() { return kSampleBlock * kMaxBlocks; }

size_t sample_scratch(int n_seqs, int budget, int n_blk) {
  return (size_t)n_seqs * budget * n_blk +
         (n_seqs * sizeof(SampleWalk) + sizeof(SampleStat) - 1) / sizeof(SampleStat);
}

namespace {

template <typename T>
void launch_sample(const TreeDims& td, const sb_tree& t, const float* logits,
                   int V, float inv_t, SampleStat* stats, const float* u_acc,
                   const float* u_bonus, const sb_accept_out& o,
                   const SignalArgs& g, hipStream_t st) {
  const int n_blk = sample_blocks(V);
  const int tiles = (n_blk + kTileBlocks - 1) / kTileBlocks;
  SampleWalk* walk =
      reinterpret_cast<SampleWalk*>(stats + (size_t)td.S * td.budget * n_blk);
  const dim3 all(tiles, td.budget, td.S);
  // Most nodes of a tree are leaves, whose statistics matter only where the
  // walk ends at one.  With many rows, the inner nodes' statistics alone, the
  // walk, those of the last nodes that are leaves and the draw take less than
  // a pass over all rows: 65 against 86 us for 16 trees of at most 64 nodes
  // (38 on average), 8 us less for four of 96.  With few rows the two more
  // launches cost more than the rows that are not read (one tree of 60, 31 MB
  // of logits: 2 to 5 us more); the line lies between the two.
  if ((size_t)td.S * td.budget * V * 4 < ((size_t)96 << 20)) {
    node_stats_kernel<kAllNodes><<<all, kThreads, 0, st>>>(
        logits, V, inv_t, t.n_nodes, t.parent, td.budget, n_blk, walk, stats);
    accept_sample_kernel<T, true, true><<<td.S, 256, 0, st>>>(
        td, t, logits, V, inv_t, stats, n_blk, u_acc, u_bonus, o, walk, g);
    return;
  }
  node_stats_kernel<kInnerNodes><<<all, kThreads, 0, st>>>(
      logits, V, inv_t, t.n_nodes, t.parent, td.budget, n_blk, walk, stats);
  accept_sample_kernel<T, true, false><<<td.S, 256, 0, st>>>(
      td, t, logits, V, inv_t, stats, n_blk, u_acc, u_bonus, o, walk, g);
  node_stats_kernel<kLastLeaf><<<dim3(tiles, 1, td.S), kThreads, 0, st>>>(
      logits, V, inv_t, t.n_nodes, t.parent, td.budget, n_blk, walk, stats);
  accept_sample_kernel<T, false, true><<<td.S, 256, 0, st>>>(
      td, t, logits, V, inv_t, stats, n_blk, u_acc, u_bonus, o, walk, g);
}

}  // namespace

void launch_accept_sample(const TreeDims& td, const sb_tree& t,
                          const float* logits, int V, float inv_t,
                          SampleStat* stats, const float* u_acc,
                          const float* u_bonus, const sb_accept_out& o,
                          const SignalArgs& g, bool bf16, hipStream_t st) {
  if (bf16)
    launch_sample<bf16_t>(td, t, logits, V, inv_t, stats, u_acc, u_bonus, o, g,
                          st);
  else
    launch_sample<float>(td, t, logits, V, inv_t, stats, u_acc, u_bonus, o, g,
                         st);
}

}  // namespace sb
