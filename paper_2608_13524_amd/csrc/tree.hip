// Selection and tree kernels of one round:
//  * select_level (Algorithm 1, scoring the children, keeping the global
//    top-W and updating their states): per request, the n_parent * k
//    candidates get s = (s_parent + log q~) + beta (eq. (5) one depth at a
//    time), the best n_keep by (s desc, parent slot asc, token asc) become
//    S_d in that order, and every kept child gets r = act(tanh(t_parent +
//    e U[token])).  The kernel also finishes the softmax pass when that pass
//    split its rows into segments.
//  * prune_emit   (Sec. 3.3, deferred best-first pruning): top-B of the whole
//    supertree by (s desc, depth asc, slot asc) - prefix-closed by Lemma 1 -
//    flattened in canonical breadth-first order (depth, parent's output index,
//    token) with parent indices and the ancestor-or-self mask.
// Every selection packs its order into one 64-bit key (score mapped to an
// ascending key in the high word, the tie-break fields in the low word) and
// ranks the keys by counting or sorts them with a bitonic network in LDS, one
// block per request, so the result does not depend on thread timing; the
// prune, which needs a set and not an order, finds the score at its edge.
#include <float.h>

#include <algorithm>
#include <type_traits>

#include "reduce.hpp"

namespace dartree {
namespace {

constexpr int kSortMax = DARTREE_MAX_SORT;

// grid: batch * S, block (q, sl): request q, state slice sl.  Three steps of
// one depth in one launch:
//  1. the candidate log-probabilities of request q's parent rows: read as
//     written by the softmax pass, or merged here from its per-segment
//     records, or (shared candidate set) computed here from the row's logits
//     over C_d (one wave per row; block 0 of the request also stores them);
//  2. s = (s_parent + log q~) + beta for every candidate and the best n_keep
//     by (s desc, parent slot asc, token asc), from one bitonic sort of 64-bit
//     keys (low word: parent slot (12 bits) << 20 | token (20 bits)); block 0
//     of the request writes the level;
//  3. the states r = act(tanh(t_parent + e U[token])) of kept children sl,
//     sl + S, ... (child i of request q is row q * n_keep + i).
// Steps 1-2 run in each of the S blocks of a request, which then need no
// further synchronisation.
template <int K>
constexpr int select_threads() { return K >= 32 ? 256 : K >= 16 ? 512 : 1024; }  // registers per lane for wide lists

template <int K>
__global__ __launch_bounds__(select_threads<K>()) void select_level(LevelArgs a, int S) {
  __shared__ __attribute__((aligned(16))) uint64_t keys[kSortMax];
  __shared__ float c_logp[kSortMax];
  __shared__ int32_t c_ids[kSortMax];
  __shared__ float ps[kSortMax];   // parent scores (n_parent <= n_parent k <= kSortMax), fetched early
  const int q = blockIdx.x / S, sl = blockIdx.x - q * S;
  const int np = a.n_parent, k = a.k;
  int n = np * k;
  const int64_t rbase = int64_t(q) * np;
  if (a.stamp && blockIdx.x == 0 && threadIdx.x == 0) {   // the workspace's depth record
    a.stamp[0] = a.stamp_key_lo;
    a.stamp[1] = a.stamp_key_hi;
    a.stamp[2] = uint32_t(a.stamp_depth);
  }
  for (int j = threadIdx.x; j < np; j += blockDim.x)
    ps[j] = a.parent_score ? a.parent_score[int64_t(q) * a.parent_stride + j] : 0.f;
  if (a.shared_k > 0) {
    // shared candidate set: row j's K corrected logits over C_d -> log q~
    // normalised over C_d, and its k best by (z desc, id asc), ranked by
    // counting over the row (staged in this wave's LDS row)
    __shared__ __attribute__((aligned(16))) float rz[16][DARTREE_MAX_CANDIDATES];
    __shared__ __attribute__((aligned(16))) int32_t rid[16][DARTREE_MAX_CANDIDATES];
    const int nk = a.shared_k;
    const float scale = kLog2e / a.tau;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    const int32_t* set = a.cset + q * a.cset_stride;
    for (int j = wave; j < np; j += nwaves) {
      const float* zr = a.zsh + (rbase + j) * nk;
      float m = -INFINITY;
      for (int c = lane; c < nk; c += 64) {
        const float v = zr[c];
        rz[wave][c] = v;
        rid[wave][c] = min(max(set[c], 0), a.vocab - 1);   // workspace ids, clamped into U
        m = fmaxf(m, v);
      }
      m = wave_max(m);
      float sum = 0.f;
      for (int c = lane; c < nk; c += 64) sum += __builtin_amdgcn_exp2f((rz[wave][c] - m) * scale);
      const float log_s = logf(wave_sum(sum));
      __builtin_amdgcn_wave_barrier();
      auto place = [&](auto Rc) {
        constexpr int R = decltype(Rc)::value;
        int rank[R];
        wave_rank_row<R>(rz[wave], rid[wave], nk, rank);
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const int c = lane + 64 * i;
          if (c >= nk || rank[i] >= k) continue;
          const float lp = (rz[wave][c] - m) / a.tau - log_s;
          const int id = rid[wave][c];
          c_logp[j * k + rank[i]] = lp;
          c_ids[j * k + rank[i]] = id;
          if (sl == 0) {
            a.cand_logp[(rbase + j) * k + rank[i]] = lp;
            a.cand_ids[(rbase + j) * k + rank[i]] = id;
          }
        }
      };
      if (nk <= 64) place(std::integral_constant<int, 1>{});
      else place(std::integral_constant<int, DARTREE_MAX_CANDIDATES / 64>{});
      if (sl == 0 && lane == 0) a.lse[rbase + j] = m / a.tau + log_s;
      __builtin_amdgcn_wave_barrier();   // the LDS row is rewritten for the next row
    }
  } else if (a.nseg > 1) {
    constexpr int RF = record_floats<K>();
    const float scale = kLog2e / a.tau;
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), nwaves = blockDim.x >> 6;
    for (int j = wave; j < np; j += nwaves) {
      uint64_t out[K];
      const Partial p = wave_merge_records<K>(a.part + (rbase + j) * a.nseg * RF, a.nseg, k, scale, out);
      const float log_s = logf(p.s);
#pragma unroll
      for (int r = 0; r < K; ++r) {
        if (r < k && lane == r) {
          const float lp = (key_value(out[r]) - p.m) / a.tau - log_s;
          const int id = key_id(out[r]);
          c_logp[j * k + r] = lp;
          c_ids[j * k + r] = id;
          if (sl == 0) {
            a.cand_logp[(rbase + j) * k + r] = lp;
            a.cand_ids[(rbase + j) * k + r] = id;
          }
        }
      }
      if (sl == 0 && lane == 0) a.lse[rbase + j] = p.m / a.tau + log_s;
    }
  } else {
    for (int c = threadIdx.x; c < n; c += blockDim.x) {
      c_logp[c] = a.cand_logp[rbase * k + c];
      c_ids[c] = a.cand_ids[rbase * k + c];
    }
  }
  __syncthreads();
  auto score_at = [&](int j, int r) {   // s of row j's candidate r, as in the keys below
    return (ps[j] + c_logp[j * k + r]) + a.beta;
  };
  // With rows in rank order, a row's candidates from position n_keep on have
  // scores <= its candidate n_keep's; if that is strictly below its candidate
  // n_keep - 1's in every row, each of them is beaten by n_keep children of its
  // own parent and can never be kept, so only the first n_keep of each row
  // compete.  (Equal fp32 scores order by token, not by rank, so a row with
  // such a tie keeps every candidate in play.)
  int kk = k;
  if (a.rows_ranked && a.n_keep < k) {
    __shared__ int tie;
    if (threadIdx.x == 0) tie = 0;
    __syncthreads();
    for (int j = threadIdx.x; j < np; j += blockDim.x)
      if (!(score_at(j, a.n_keep - 1) > score_at(j, a.n_keep))) tie = 1;
    __syncthreads();
    if (!tie) kk = a.n_keep;
  }
  n = np * kk;
  auto key_of = [&](int c) {
    const int j = c / kk;
    const int r = c - j * kk;
    const float sc = score_at(j, r);
    // ids < 2^20; the mask keeps a malformed id out of the parent-slot field
    return (uint64_t(score_desc_key(sc)) << 32) | (uint32_t(j) << 20) | (uint32_t(c_ids[j * k + r]) & 0xFFFFFu);
  };
  const uint64_t* kept = keys;   // the n_keep best, in order
  if (n <= int(blockDim.x)) {
    // few candidates: rank by counting (keys are distinct: (slot, token)
    // pairs are), one barrier instead of a sorting network.  Sixteen lanes
    // share a key (12 parents x 64 of C_d: 8.4 us a launch with one lane per
    // key and ids compared with every value of a row, 6.9 with both changes).
    uint64_t mine = ~0ull;
    if (int(threadIdx.x) < n) mine = key_of(threadIdx.x);
    keys[threadIdx.x] = mine;
    __syncthreads();
    // 16 lanes per key, each comparing a sixteenth of them by 16-byte reads of
    // key pairs (the keys past n are ~0); n <= 1024 and n_keep <= n: the ranked
    // copy sits above the keys
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const u64x2* kp = reinterpret_cast<const u64x2*>(keys) + (threadIdx.x & 15);
    const int pairs = ((n + 31) & ~31) >> 1;
    for (int i0 = 0; i0 < n; i0 += int(blockDim.x >> 4)) {
      const int i = i0 + int(threadIdx.x >> 4);
      const uint64_t key = keys[min(i, n - 1)];
      int rank = 0;
#pragma unroll 4
      for (int j = 0; j < pairs; j += 16) {
        const u64x2 kk = kp[j];
        rank += int(kk.x < key) + int(kk.y < key);
      }
      rank = row16_sum(rank);
      if ((threadIdx.x & 15) == 0 && i < n && rank < a.n_keep) keys[kSortMax / 2 + rank] = key;
    }
    kept = keys + kSortMax / 2;
    __syncthreads();
  } else {
    const int npad = next_pow2(n);
    for (int c = threadIdx.x; c < npad; c += blockDim.x) keys[c] = c < n ? key_of(c) : ~0ull;
    __syncthreads();
    bitonic_sort(keys, npad);
  }
  if (sl == 0) {
    for (int i = threadIdx.x; i < a.n_keep; i += blockDim.x) {
      const uint64_t key = kept[i];
      const uint32_t lo = uint32_t(key);
      const int64_t o = int64_t(q) * a.out_stride + i;
      a.out_tok[o] = int32_t(lo & 0xFFFFFu);
      a.out_par[o] = int32_t(lo >> 20);
      a.out_score[o] = score_from_desc_key(uint32_t(key >> 32));
    }
  }
  if (!a.state) return;
  const int h = a.hidden;
  for (int i = sl; i < a.n_keep; i += S) {
    const uint32_t lo = uint32_t(kept[i]);
    // an empty candidate (a row without finite values) is clamped into U
    const int64_t prow = rbase + (lo >> 20), tok = min(int(lo & 0xFFFFFu), a.vocab - 1);
    const int64_t c = int64_t(q) * a.n_keep + i;
    const float* tp = a.t + prow * h;
    if (a.precision == DARTREE_BF16) {
      typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
      const uint16_t* up = static_cast<const uint16_t*>(a.U) + tok * h;
      uint16_t* rp = static_cast<uint16_t*>(a.r_out) + c * h;
      for (int x = threadIdx.x * 8; x < h; x += blockDim.x * 8) {
        const f32x4 t0 = *reinterpret_cast<const f32x4*>(tp + x);
        const f32x4 t1 = *reinterpret_cast<const f32x4*>(tp + x + 4);
        const u16x8 u = *reinterpret_cast<const u16x8*>(up + x);
        u16x8 r;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          const float e0 = a.e * bf16_to_f32(u[j]), e1 = a.e * bf16_to_f32(u[j + 4]);
          r[j] = f32_to_bf16(a.markov ? e0 : tanhf(t0[j] + e0));
          r[j + 4] = f32_to_bf16(a.markov ? e1 : tanhf(t1[j] + e1));
        }
        *reinterpret_cast<u16x8*>(rp + x) = r;
      }
    } else {
      const float* up = static_cast<const float*>(a.U) + tok * h;
      float* rp = static_cast<float*>(a.r_out) + c * h;
      for (int x = threadIdx.x; x < h; x += blockDim.x) rp[x] = a.markov ? a.e * up[x] : tanhf(tp[x] + a.e * up[x]);
    }
  }
}

// grid: batch.  Level arrays are [L][batch][W]; node g of request q is slot
// g - off[d-1] of depth d, so ascending g is (depth asc, slot asc).
//
// One block per request and latency throughout: what counts is the chain of
// dependent steps, so
//  * the top-B is a threshold, not a sort: the B-th best score key is found
//    four bits at a time, wave w counting the keys below the w-th of 15
//    candidates from registers (8 rounds of one barrier; a bitonic sort of
//    1024 keys is 55 of them), and ties at the threshold go by g;
//  * levels of at most 16 nodes are ordered by one wave without barriers (B =
//    64, width 12: 16.9 us, 18.0 with the other way; at width 64, where every
//    node is compared with 64 scalars in turn, 32 against 22); in wider ones 16
//    lanes count a node's rank, each comparing a few keys, so that a depth
//    costs one LDS round trip per barrier;
//  * a mask thread walks its node's path once for four words.
// Measured at 16 requests x 16 levels of 64, B = 512: 60.8 -> 22.0 us
// (threshold 14000, order 21000, mask 1500, all else 4500 clocks).
constexpr int kPruneWaves = 16;
constexpr int kPruneRounds = kSortMax / (64 * kPruneWaves);   // nodes per thread
static_assert(kPruneRounds * kPruneWaves == 64, "one count of equal keys per lane");
constexpr int kPruneRegs = 16;   // keys per lane held in registers (1024 nodes; the rest is read from LDS)

__global__ __launch_bounds__(64 * kPruneWaves) void prune_emit(LevelShape shape, int budget, int batch,
                                                              const int32_t* __restrict__ lvl_tok,
                                                              const int32_t* __restrict__ lvl_par,
                                                              const float* __restrict__ lvl_score, dartree_tree out) {
  // per supertree node: score key, token, parent slot, score, depth, output index (-1 if pruned)
  __shared__ uint32_t key[kSortMax];
  __shared__ int32_t s_tok[kSortMax], s_par[kSortMax];
  __shared__ float s_score[kSortMax];
  __shared__ uint8_t s_dep[kSortMax];
  __shared__ int32_t out_idx[kSortMax];
  __shared__ int32_t par_out[kSortMax];   // per output index: parent's output index
  __shared__ __attribute__((aligned(16))) uint32_t rank_key[DARTREE_MAX_WIDTH + 64];
  __shared__ int32_t kept[DARTREE_MAX_DEPTH];
  __shared__ int32_t cnt[2][kPruneWaves];
  __shared__ int32_t eq_at[64];

  const int q = blockIdx.x, tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int L = shape.depth, W = shape.width;
  // lane l holds off[l + 1]: a depth's offset is one lane read away
  const int voff = shape.off[min(lane + 1, L)];
  auto off_of = [&](int d) { return d == 0 ? 0 : __builtin_amdgcn_readlane(voff, d - 1); };
  const int total = off_of(L);
  const int n_out = min(budget, total);
  const int words = (budget + 63) / 64;

  // 0. stage the levels in LDS (one pass of independent loads)
  for (int g = tid; g < total; g += blockDim.x) {
    int lo = 0, first = 0;   // depth - 1 of node g and that depth's first node 
    for (int d = 1; d < L; ++d) {
      const int o = off_of(d);
      lo += int(g >= o);
      first = g >= o ? o : first;
    }
    const int64_t li = (int64_t(lo) * batch + q) * W + (g - first);
    const float sc = lvl_score[li];
    s_tok[g] = lvl_tok[li];
    s_par[g] = lvl_par[li];
    s_score[g] = sc;
    s_dep[g] = uint8_t(lo + 1);
    key[g] = score_desc_key(sc);
  }
  __syncthreads();

  // 1. T = the n_out-th smallest key; `need` of the keys equal to it are kept
  uint32_t T = ~0u;
  int need = total, eq = total;
  if (n_out < total) {
    uint32_t kr[kPruneRegs];
#pragma unroll
    for (int j = 0; j < kPruneRegs; ++j) kr[j] = lane + 64 * j < total ? key[lane + 64 * j] : ~0u;
    // keys below th; keys past the last node count only against th = 0 .. (never below ~0)
    auto below = [&](uint32_t th) {
      int c = 0;
#pragma unroll
      for (int j = 0; j < kPruneRegs; ++j) c += int(kr[j] < th);
      for (int g = 64 * kPruneRegs + lane; g < total; g += 64) c += int(key[g] < th);
      return wave_sum_int(c);
    };
    T = 0;
#pragma unroll 1
    for (int r = 0; r < 8; ++r) {
      const int shift = 28 - 4 * r;
      if (wave < 15) {
        const int c = below(T | (uint32_t(wave + 1) << shift));
        if (lane == 0) cnt[r & 1][wave] = c;
      }
      __syncthreads();
      T |= uint32_t(__popcll(__ballot(lane < 15 && cnt[r & 1][lane & 15] < n_out))) << shift;
    }
    if (wave == 0) {
      const int c = below(T);
      if (lane == 0) cnt[0][0] = c;
    } else if (wave == 1) {   // keys equal to T among the nodes
      int c = 0;
      for (int g = lane; g < total; g += 64) c += int(key[g] == T);
      c = wave_sum_int(c);
      if (lane == 0) cnt[0][1] = c;
    }
    __syncthreads();
    need = n_out - cnt[0][0];
    eq = cnt[0][1];
  }
  // Where only some of the equal keys are kept, they are the first in g order:
  // the counts of every 64 nodes in eq_at, then a lane's place among its own (64
  // levels of 64, one score: 86 us; 276 with each node counting those before it).
  const bool some = n_out < total && need < eq;
  if (some) {
    for (int j = 0; j < kPruneRounds; ++j) {
      const int g = tid + 64 * kPruneWaves * j;
      const uint64_t tied = __ballot(g < total && key[min(g, total - 1)] == T);
      if (lane == 0) eq_at[kPruneWaves * j + wave] = __popcll(tied);
    }
    __syncthreads();
  }
  for (int j = 0; 64 * kPruneWaves * j < total; ++j) {
    const int g = tid + 64 * kPruneWaves * j;
    const bool in = g < total;
    const uint32_t kg = key[min(g, total - 1)];
    bool keep = kg < T || n_out == total;
    const bool tied = in && !keep && kg == T;
    if (some) {
      const uint64_t bal = __ballot(tied);
      const int before = wave_sum_int(lane < kPruneWaves * j + wave ? eq_at[lane] : 0) +
                         int(__builtin_amdgcn_mbcnt_hi(uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0)));
      keep |= tied && before < need;
    } else {
      keep |= tied;
    }
    if (in) out_idx[g] = keep ? 0 : -1;
  }
  __syncthreads();
  // 2. canonical order, one depth at a time: rank kept nodes of depth d by
  //    (parent's output index, token); siblings have distinct tokens.
  int base = 0, pd = 0, od = 0;   // first output of depth d, first nodes of depths d - 1 and d
  // slots outside S_{d-1} are clamped: malformed levels cannot index out of
  // bounds.  A parent that was pruned (scores that rise along an edge) is -1:
  // as an index its 12 bits would be the last node's, which has no children.
  auto parent_of = [](uint32_t k, int d) {
    const int pi = int(k >> 20);
    return d == 1 || pi == 0xFFF ? -1 : pi;
  };
  if (W <= 16) {
    // one wave, a node per lane: no barriers, the parent's output index by a
    // lane exchange and the keys compared as scalars
    if (wave == 0) {
      int prev = 0;   // this lane's output index in the depth before
      int nx_par = 0, nx_tok = 0, nx_keep = -1;
      auto fetch = [&](int first, int n) {   // the next depth's nodes, while this one is ranked
        nx_keep = -1;
        if (lane < n) {
          nx_par = s_par[first + lane];
          nx_tok = s_tok[first + lane];
          nx_keep = out_idx[first + lane];
        }
      };
      fetch(0, off_of(1));
      for (int d = 1; d <= L; ++d) {
        const int nd = off_of(d) - od;
        const uint32_t pidx = d > 1 ? uint32_t(__shfl(prev, min(max(nx_par, 0), od - pd - 1))) : 0u;
        const bool keep = nx_keep >= 0;
        const uint32_t mine = keep ? (pidx << 20) | (uint32_t(nx_tok) & 0xFFFFFu) : ~0u;
        if (d < L) fetch(od + nd, off_of(d + 1) - od - nd);
        int r = 0;
        for (int j = 0; j < nd; j += 8)
#pragma unroll
          for (int e = 0; e < 8; ++e) r += int(uint32_t(__builtin_amdgcn_readlane(mine, j + e)) < mine);
        const int n_kept = __popcll(__ballot(keep));
        // ranks of distinct keys are 0 .. n_kept - 1; equal keys (malformed levels) go by slot
        if (wave_sum_int(keep ? r : 0) != n_kept * (n_kept - 1) / 2)
          for (int j = 0; j < nd; ++j) r += int(uint32_t(__builtin_amdgcn_readlane(mine, j)) == mine && j < lane);
        prev = keep ? base + r : -1;
        if (keep && mine != ~0u) {
          out_idx[od + lane] = prev;
          par_out[prev] = parent_of(mine, d);
        }
        base += n_kept;
        pd = od;
        od += nd;
      }
    }
    __syncthreads();
  } else {
    for (int d = wave; d < L; d += kPruneWaves) {   // kept nodes of depth d + 1
      const int end = off_of(d + 1);
      int c = 0;
      for (int g = off_of(d); g < end; g += 64) c += __popcll(__ballot(g + lane < end && out_idx[min(g + lane, end - 1)] >= 0));
      if (lane == 0) kept[d] = c;
    }
    // the 16 lanes of a row count one node's rank
    const int row = tid >> 4, sub = tid & 15;
    for (int d = 1; d <= L; ++d) {
      const int nd = off_of(d) - od;
      const int padded = (nd + 63) & ~63;
      for (int i = tid; i < padded; i += blockDim.x) {
        uint32_t rk = ~0u;
        if (i < nd && out_idx[od + i] >= 0) {
          const uint32_t pidx = d > 1 ? uint32_t(out_idx[pd + min(max(s_par[od + i], 0), od - pd - 1)]) : 0u;
          rk = (pidx << 20) | (uint32_t(s_tok[od + i]) & 0xFFFFFu);
        }
        rank_key[i] = rk;
      }
      __syncthreads();
      for (int i0 = 0; i0 < nd; i0 += 64) {   // whole waves: the row sums need every lane
        const int i = i0 + row;
        const uint32_t mine = rank_key[i];
        typedef uint32_t u32x4v __attribute__((ext_vector_type(4)));
        const u32x4v* rk4 = reinterpret_cast<const u32x4v*>(rank_key) + sub;
        int r = 0;
        for (int j = 0; j < padded; j += 64) {
          const u32x4v kv = rk4[j >> 2];
#pragma unroll
          for (int e = 0; e < 4; ++e) r += int(kv[e] < mine) | int((kv[e] == mine) & (j + 4 * sub + e < i));
        }
        r = row16_sum(r);
        if (sub == 0 && mine != ~0u) {
          out_idx[od + i] = base + r;
          par_out[base + r] = parent_of(mine, d);
        }
      }
      base += kept[d - 1];
      pd = od;
      od += nd;
      __syncthreads();
    }
  }

  // 3. emit node arrays (pad slots past n_out)
  const int64_t ob = int64_t(q) * budget;
  for (int o = n_out + tid; o < budget; o += blockDim.x) {
    out.tokens[ob + o] = -1;
    out.parents[ob + o] = -1;
    out.depths[ob + o] = 0;
    out.scores[ob + o] = -INFINITY;
  }
  for (int g = tid; g < total; g += blockDim.x) {
    const int o = out_idx[g];
    if (o < 0) continue;
    out.tokens[ob + o] = s_tok[g];
    out.parents[ob + o] = par_out[o];
    out.depths[ob + o] = s_dep[g];
    out.scores[ob + o] = s_score[g];
  }
  // 4. ancestor-or-self mask, four 64-bit words of a row per thread
  const int64_t mb = int64_t(q) * budget * words;
  const int wg = (words + 3) / 4;
  for (int t = tid; t < budget * wg; t += blockDim.x) {
    const int o = t / wg, w0 = (t - o * wg) * 4;
    uint64_t bits[4] = {0, 0, 0, 0};
    if (o < n_out) {
      // parents precede children in the output order, so the walk strictly
      // decreases and ends at -1 after at most L steps
      for (int j = o; j >= 0;) {
        const uint64_t bit = 1ull << (j & 63);
        const int w = (j >> 6) - w0;
#pragma unroll
        for (int e = 0; e < 4; ++e) bits[e] |= w == e ? bit : 0ull;
        const int nx = par_out[j];
        j = nx < j ? nx : -1;
      }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (w0 + e < words) out.mask[mb + int64_t(o) * words + w0 + e] = bits[e];
  }
  if (tid == 0) out.num_nodes[q] = n_out;
}

}  // namespace

int select_level_waves(int k) {
  switch (topk_bucket(k)) {
    case 1: return select_threads<1>() / 64;
    case 2: return select_threads<2>() / 64;
    case 4: return select_threads<4>() / 64;
    case 8: return select_threads<8>() / 64;
    case 16: return select_threads<16>() / 64;
    default: return select_threads<32>() / 64;
  }
}

hipError_t launch_select_level(const LevelArgs& a, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  // state slices: enough blocks to spread the state rows over the chip
  const int S = a.state ? std::max(1, std::min(a.n_keep, (256 + a.batch - 1) / a.batch)) : 1;
  const dim3 grid(unsigned(a.batch) * unsigned(S));
  // the top-k bucket only sizes the segment merge; without one the widest block serves
  switch ((a.shared_k > 0 || a.nseg <= 1) ? 1 : topk_bucket(a.k)) {
    case 1: hipLaunchKernelGGL((select_level<1>), grid, dim3(select_threads<1>()), 0, s, a, S); break;
    case 2: hipLaunchKernelGGL((select_level<2>), grid, dim3(select_threads<2>()), 0, s, a, S); break;
    case 4: hipLaunchKernelGGL((select_level<4>), grid, dim3(select_threads<4>()), 0, s, a, S); break;
    case 8: hipLaunchKernelGGL((select_level<8>), grid, dim3(select_threads<8>()), 0, s, a, S); break;
    case 16: hipLaunchKernelGGL((select_level<16>), grid, dim3(select_threads<16>()), 0, s, a, S); break;
    default: hipLaunchKernelGGL((select_level<32>), grid, dim3(select_threads<32>()), 0, s, a, S); break;
  }
  return hipGetLastError();
}

hipError_t launch_prune_emit(int batch, const LevelShape& shape, int budget, const int32_t* lvl_tok,
                             const int32_t* lvl_par, const float* lvl_score, const dartree_tree& out,
                             hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  hipLaunchKernelGGL(prune_emit, dim3(batch), dim3(64 * kPruneWaves), 0, s, shape, budget, batch, lvl_tok, lvl_par,
                     lvl_score, out);
  return hipGetLastError();
}

}  // namespace dartree
