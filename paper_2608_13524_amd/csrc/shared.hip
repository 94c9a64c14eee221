// Shared candidate sets (Algorithm 1 as printed): C_d = TopK(L_d^base, K) for
// every request and depth, and the corrected logits of every node of a depth
// over C_d only, z_j[c] = L_d^base[C_d[c]] + U[C_d[c]] . a_j.
//  * cset_group_max / cset_select: theta = the K-th largest of the maxima of up
//    to 4 K disjoint groups of a row bounds the K-th largest value from below;
//    the elements >= theta, all in groups whose maximum is, are compacted and
//    ranked as 64-bit keys (score key << 32 | id, ascending = (value desc, id
//    asc)), with an exact radix select when too many qualify (heavy ties).
//  * shared_logits_bf16: a gather-product on MFMA.  Block (request, 16
//    candidates, up to 64 node rows); the A operand is 16 rows of U picked by
//    the set, the B operand 16 node rows of a; 16 waves split h and are
//    summed through LDS in wave order.  fp32 mode: one thread per (node,
//    candidate).
#include <algorithm>
#include <type_traits>

#include "reduce.hpp"

namespace dartree {
namespace {

// Orderable 32-bit key of a logit: larger key = larger value (-0 taken as +0).
__device__ __forceinline__ uint32_t ord_key(float x) {
  const uint32_t b = __float_as_uint(x + 0.0f);
  return (b & 0x80000000u) ? ~b : (b | 0x80000000u);
}

// The 16 leading bits of a value's orderable key: never above the key, so K
// groups with codes >= c hold K elements whose keys are >= c << 16.
__device__ __forceinline__ uint32_t ord_code(float x) { return ord_key(x) >> 16; }
// The least value with this code.  Of -inf's code that is -inf itself, the
// greatest key with it (the ones below are bit patterns of NaNs).
constexpr uint32_t kCodeNegInf = 0x007F;
__device__ __forceinline__ float code_value(uint32_t c) {
  if (c <= kCodeNegInf) return -INFINITY;
  const uint32_t k = c << 16;
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7FFFFFFFu) : ~k);
}

// Groups of a row: 4 K where that leaves 16 values a group, at least K.  Their
// codes take 2 bytes each: the first 2 K live in the scratch (K words a row),
// the others in the row's output, which cset_select overwrites last.  A group's
// maximum is taken by 16 lanes, from 193 values on by a wave, past 1024 by a
// block (four 16-byte loads a lane go out together).
constexpr int kMaxGroups = 4 * DARTREE_MAX_CANDIDATES;
int cset_groups(int64_t vocab, int K) {
  return int(std::min<int64_t>(4 * int64_t(K), std::max<int64_t>(K, vocab / 16)));
}
__host__ __device__ __forceinline__ int group_lanes(int vocab, int G) {
  const int len = (vocab + G - 1) / G;
  return len <= 192 ? 16 : len <= 1024 ? 64 : 256;
}
__device__ __forceinline__ uint16_t* group_code(void* scratch, int32_t* ids, int64_t row, int K, int g) {
  return g < 2 * K ? static_cast<uint16_t*>(scratch) + row * 2 * K + g
                   : reinterpret_cast<uint16_t*>(ids + row * K) + (g - 2 * K);
}
// Group g of a row is [group_start(g), group_start(g + 1)).  Whole float4s of
// the row where it has enough of them, so that only its last group is ragged (a
// ragged end costs a round trip of its own).
__device__ __forceinline__ int group_start(int g, int vocab, int G) {
  const int quads = (vocab + 3) / 4;
  return quads >= G ? min(vocab, 4 * int(int64_t(g) * quads / G)) : int(int64_t(g) * vocab / G);
}

// Four values from v on, -inf past v1 (rows and groups start at any multiple of 4 bytes).
__device__ __forceinline__ f32x4 load4(const float* x, int v, int v1) {
  f32x4 r{-INFINITY, -INFINITY, -INFINITY, -INFINITY};
  if (v + 4 <= v1) {
    r = *reinterpret_cast<const f32x4u*>(x + v);
  } else {
#pragma unroll
    for (int i = 0; i < 3; ++i)
      if (v + i < v1) r[i] = x[v + i];
  }
  return r;
}

// group_lanes per group, 256 lanes a block; grid: rows * gpb.
__global__ __launch_bounds__(256) void cset_group_max(const float* __restrict__ logits, int vocab, int K, int G, int gpb,
                                                      void* scratch, int32_t* ids) {
  __shared__ float red[4];
  const int64_t row = blockIdx.x / gpb;
  const int LPG = group_lanes(vocab, G);
  const int g = (blockIdx.x % gpb) * (256 / LPG) + int(threadIdx.x) / LPG;
  const int lane = threadIdx.x & (LPG - 1);
  const int gc = min(g, G - 1);   // surplus lanes repeat the last group
  const int v0 = group_start(gc, vocab, G), v1 = group_start(gc + 1, vocab, G);
  const float* x = logits + row * int64_t(vocab);
  float m = -INFINITY;
#pragma unroll 4
  for (int v = v0 + 4 * lane; v < v1; v += 4 * LPG) {
    const f32x4 q = load4(x, v, v1);
    m = fmaxf(m, fmaxf(fmaxf(q[0], q[1]), fmaxf(q[2], q[3])));
  }
  m = LPG == 16 ? row16_max(m) : wave_max(m);
  if (LPG == 256) {   // the same for the block
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = m;
    __syncthreads();
    m = fmaxf(fmaxf(red[0], red[1]), fmaxf(red[2], red[3]));
  }
  if (lane == 0 && g < G) *group_code(scratch, ids, row, K, g) = uint16_t(ord_code(m));
}

constexpr int kSelCap = 4096;   // candidates above the threshold kept in LDS

// One row per block (1024 threads).  theta, the value of the K-th largest group
// code, is <= the K-th largest value of the row, and everything >= theta lies
// in the groups whose code is no smaller: about a quarter of them (with 4 K
// groups), so the row is not read a second time.  The elements >= theta (at
// least K, about 1.2 K on smooth data) are compacted and ranked.  When more
// than kSelCap qualify (heavy ties), an exact radix select finds the K-th
// largest key T instead: the elements above T (fewer than K) are sorted, and
// the elements equal to T follow in id order.
// Latency-bound (one block per row).  With K groups, whose least maximum let
// 4.7 K elements of all groups through, a block read its whole row again:
// 64 rows x 151936, K = 64: 23.0 us, 11.3 here (both launches 34 and 19 us); 4
// rows x 16000, K = 256: 34 and 19.5 us.
__global__ __launch_bounds__(1024) void cset_select(const float* __restrict__ logits, int vocab, int K, int G,
                                                    void* scratch, int32_t* ids) {
  __shared__ __attribute__((aligned(16))) uint64_t cand[kSelCap];
  __shared__ uint32_t hist[16][256];
  __shared__ int count, nflag, remaining_s, taken_s;
  __shared__ uint32_t prefix_s, theta_s;
  __shared__ uint16_t flagged[kMaxGroups];
  __shared__ int wave_tot[16];
  const int64_t row = blockIdx.x;
  const float* x = logits + row * int64_t(vocab);
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  int32_t* out = ids + row * K;

  const int code = tid < G ? int(*group_code(scratch, ids, row, K, tid)) : -1;
  if (tid == 0) count = nflag = 0;
  if (wave == 0) {
    // the K-th largest code, one bit at a time: R codes per lane
    auto kth = [&](auto Rc) {
      constexpr int R = decltype(Rc)::value;
      int c[R];
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const int g = lane + 64 * j;
        c[j] = g < G ? int(*group_code(scratch, ids, row, K, g)) : -1;
      }
      // the bits all codes share need no search (small whole numbers: exact as floats)
      float lo = 65536.f, hi = -1.f;
#pragma unroll
      for (int j = 0; j < R; ++j) {
        if (c[j] >= 0) lo = fminf(lo, float(c[j]));
        hi = fmaxf(hi, float(c[j]));
      }
      const int top = int(wave_max(hi)), diff = top ^ int(-wave_max(-lo));
      if (G == K) return uint32_t(top ^ diff);   // the least
      const int bits = diff ? 32 - __builtin_clz(diff) : 0;
      int t = top & ~((1 << bits) - 1);
#pragma unroll 1
      for (int bit = bits ? 1 << (bits - 1) : 0; bit > 0; bit >>= 1) {
        int n = 0;
#pragma unroll
        for (int j = 0; j < R; ++j) n += __popcll(__ballot(c[j] >= (t | bit)));
        if (n >= K) t |= bit;
      }
      return uint32_t(t);
    };
    const uint32_t t = G <= 256 ? kth(std::integral_constant<int, 4>{}) : kth(std::integral_constant<int, kMaxGroups / 64>{});
    if (lane == 0) theta_s = t;
  }
  __syncthreads();
  const float theta = code_value(theta_s);
  {   // one atomic per wave
    const uint64_t bal = __ballot(code >= int(theta_s));
    int first = 0;
    if (lane == 0 && bal) first = atomicAdd(&nflag, __popcll(bal));
    first = __builtin_amdgcn_readfirstlane(first);
    if ((bal >> lane) & 1)
      flagged[first + __builtin_amdgcn_mbcnt_hi(uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0))] = uint16_t(tid);
  }
  __syncthreads();
  auto keep = [&](const f32x4& q, int v, int end) __attribute__((always_inline)) {   // values v .. v + 3 of the row
    if (!(fmaxf(fmaxf(q[0], q[1]), fmaxf(q[2], q[3])) >= theta)) return;
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (v + i < end && q[i] >= theta) {
        const int pos = atomicAdd(&count, 1);
        if (pos < kSelCap) cand[pos] = (uint64_t(score_desc_key(q[i])) << 32) | uint32_t(v + i);
      }
  };
  const int nf = nflag;
  if (2 * nf > G) {
    // Most groups are flagged (few values a group, ties, masked rows): the row in
    // sequence, a float4 per lane.  By groups of 16 values a quarter of the lanes
    // took four times the atomics (5000 values, K = 256: 29.1 -> 26.6 us).
    constexpr int kSeq = 8;
    for (int at = 4 * tid; at - 4 * tid < vocab; at += 4 * 1024 * kSeq) {
      f32x4 xv[kSeq];
#pragma unroll
      for (int u = 0; u < kSeq; ++u) xv[u] = load4(x, at + 4 * 1024 * u, vocab);
#pragma unroll
      for (int u = 0; u < kSeq; ++u) keep(xv[u], at + 4 * 1024 * u, vocab);
    }
  } else {
    // LPG lanes per flagged group, kBatch groups and kChunk float4 of each per lane
    // and pass, whose loads go out before any check (the atomics would otherwise
    // keep them from overlapping): enough lanes to read a group in one pass, as
    // long as the about K flagged groups still do too (K = 1 x 151936: 146 us with
    // 64 lanes, 20 so; K = 16 x 16384 values a group: 64, 24).
    constexpr int kBatch = 5, kChunk = 3;
    const int len = (vocab + G - 1) / G;
    const int LPG = len <= 192 ? 16 : len <= 768 || K > 16 ? 64 : len <= 3072 || K > 8 ? 256 : 1024;
    const int slots = 1024 / LPG, gl = tid & (LPG - 1), longest = len + 4;
    for (int f0 = tid / LPG; f0 - tid / LPG < nf; f0 += slots * kBatch) {
      int v0[kBatch], v1[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int f = f0 + slots * u;
        const int g = f < nf ? int(flagged[f]) : -1;
        v0[u] = g < 0 ? 0 : group_start(g, vocab, G);
        v1[u] = g < 0 ? 0 : group_start(g + 1, vocab, G);
      }
      for (int at = 0; at < longest; at += 4 * kChunk * LPG) {
        f32x4 xv[kBatch][kChunk];
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
          for (int e = 0; e < kChunk; ++e) xv[u][e] = load4(x, v0[u] + at + 4 * (LPG * e + gl), v1[u]);
#pragma unroll
        for (int u = 0; u < kBatch; ++u)
#pragma unroll
          for (int e = 0; e < kChunk; ++e) keep(xv[u][e], v0[u] + at + 4 * (LPG * e + gl), v1[u]);
      }
    }
  }
  __syncthreads();
  const int n = count;
  if (n <= 512) {
    // ranked by counting, 16 lanes per key (keys are distinct: ids are);
    // positions past n hold -1
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const int padded = (n + 31) & ~31;
    for (int i = n + tid; i < padded; i += blockDim.x) cand[i] = ~0ull;
    __syncthreads();
    const u64x2* cp = reinterpret_cast<const u64x2*>(cand) + (tid & 15);
    for (int i0 = 0; i0 < n; i0 += int(blockDim.x >> 4)) {
      const int i = i0 + (tid >> 4);
      const uint64_t mine = cand[min(i, n - 1)];
      int rank = 0;
      for (int j = 0; j < padded >> 1; j += 16) {
        const u64x2 k = cp[j];
        rank += int(k.x < mine) + int(k.y < mine);
      }
      rank = row16_sum(rank);
      if ((tid & 15) == 0 && i < n && rank < K) out[rank] = int32_t(uint32_t(mine));
    }
    for (int r = n + tid; r < K; r += blockDim.x) out[r] = -1;
    return;
  }
  if (n <= kSelCap) {
    const int npad = next_pow2(n);
    for (int i = n + tid; i < npad; i += blockDim.x) cand[i] = ~0ull;
    __syncthreads();
    bitonic_sort(cand, npad);
    for (int r = tid; r < K; r += blockDim.x) out[r] = int32_t(uint32_t(cand[r]));
    return;
  }

  // exact radix select of the K-th largest orderable key, 8 bits at a time
  uint32_t prefix = 0, mask = 0;
  if (tid == 0) remaining_s = K;
  for (int pass = 3; pass >= 0; --pass) {
    for (int i = tid; i < 16 * 256; i += blockDim.x) (&hist[0][0])[i] = 0;
    __syncthreads();
    const int shift = 8 * pass;
    for (int v = tid; v < vocab; v += blockDim.x) {
      const uint32_t u = ord_key(x[v]);
      if ((u & mask) == prefix) atomicAdd(&hist[wave][(u >> shift) & 0xFF], 1u);
    }
    __syncthreads();
    if (tid == 0) {
      int rem = remaining_s;
      int bsel = 0;
      for (int bin = 255; bin >= 0; --bin) {
        int c = 0;
        for (int w = 0; w < int(blockDim.x >> 6); ++w) c += int(hist[w][bin]);
        if (c >= rem) { bsel = bin; break; }
        rem -= c;
      }
      remaining_s = rem;
      prefix_s = prefix | (uint32_t(bsel) << shift);
    }
    __syncthreads();
    prefix = prefix_s;
    mask |= 0xFFu << shift;
  }
  const uint32_t T = prefix;
  const int need_eq = remaining_s;   // elements equal to T to take, lowest ids first
  // elements above T: fewer than K, sorted
  if (tid == 0) count = 0;
  __syncthreads();
  for (int v = tid; v < vocab; v += blockDim.x) {
    const float xv = x[v];
    if (ord_key(xv) > T) cand[atomicAdd(&count, 1)] = (uint64_t(score_desc_key(xv)) << 32) | uint32_t(v);
  }
  __syncthreads();
  const int n_gt = count;   // = K - need_eq
  {
    const int npad = next_pow2(n_gt);
    for (int i = n_gt + tid; i < npad; i += blockDim.x) cand[i] = ~0ull;
    __syncthreads();
    bitonic_sort(cand, npad);
    for (int r = tid; r < n_gt; r += blockDim.x) out[r] = int32_t(uint32_t(cand[r]));
  }
  // elements equal to T in id order: block-wide prefix counts over tiles
  if (tid == 0) taken_s = 0;
  __syncthreads();
  for (int base = 0; base < vocab; base += blockDim.x) {
    const int v = base + tid;
    const bool eq = v < vocab && ord_key(x[v]) == T;
    const uint64_t bal = __ballot(eq);
    const int before_in_wave = __builtin_amdgcn_mbcnt_hi(uint32_t(bal >> 32), __builtin_amdgcn_mbcnt_lo(uint32_t(bal), 0));
    if (lane == 0) wave_tot[wave] = __popcll(bal);
    __syncthreads();
    int before = taken_s + before_in_wave;
    for (int w = 0; w < wave; ++w) before += wave_tot[w];
    if (eq && before < need_eq) out[n_gt + before] = v;
    __syncthreads();
    if (tid == 0) {
      int t = 0;
      for (int w = 0; w < int(blockDim.x >> 6); ++w) t += wave_tot[w];
      taken_s += t;
    }
    __syncthreads();
    if (taken_s >= need_eq) break;
  }
}

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

constexpr int kRowTiles = 4;  // node-row tiles of 16 per block

// grid: batch * ncb * nrb; block (q, cb, rb): candidates 16 cb .. 16 cb + 15,
// node rows 64 rb .. 64 rb + 63 of request q.  Rows past K or n_parent are
// clamped (computed, never stored).
__global__ __launch_bounds__(1024) void shared_logits_bf16(int np, int K, int hidden, int vocab, int ncb, int nrb,
                                                          const uint16_t* __restrict__ a,
                                                          const uint16_t* __restrict__ U,
                                                          const float* __restrict__ lb, int64_t lb_stride,
                                                          const int32_t* __restrict__ cset, int64_t cset_stride,
                                                          const int32_t* __restrict__ group_index, float* z) {
  constexpr int kWaves = 16;   // split h
  __shared__ f32x4 red[kWaves][kRowTiles][64];
  const int q = blockIdx.x / (ncb * nrb);
  const int rest = blockIdx.x - q * ncb * nrb;
  const int cb = rest / nrb, rb = rest % nrb;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, kg = lane >> 4;
  const int64_t g = group_index ? group_index[q] : q;   // L^base / C_d row of request q
  const int32_t* set = cset + g * cset_stride;
  const int c = min(16 * cb + r16, K - 1);
  // set ids come from the workspace: clamped into the vocabulary, so a set
  // that was never built (depths enqueued out of order) cannot index past U
  auto id_at = [&](int i) { return min(max(set[i], 0), vocab - 1); };
  const uint16_t* urow = U + int64_t(id_at(c)) * hidden + kg * 8;
  const uint16_t* arow[kRowTiles];
#pragma unroll
  for (int t = 0; t < kRowTiles; ++t) {
    const int j = min(64 * rb + 16 * t + r16, np - 1);
    arow[t] = a + (int64_t(q) * np + j) * hidden + kg * 8;
  }
  // node-row tiles this block needs (block-uniform)
  const int ntile = min(kRowTiles, (np - 64 * rb + 15) / 16);
  // wave 0 adds L^base at its lanes' four candidates: fetch them now, while
  // the products run, rather than after the reduction
  float lbv[4] = {0.f, 0.f, 0.f, 0.f};
  if (wave == 0) {
    const float* lbq = lb + g * lb_stride;
#pragma unroll
    for (int i = 0; i < 4; ++i) lbv[i] = lbq[id_at(min(16 * cb + 4 * kg + i, K - 1))];
  }
  f32x4 acc[kRowTiles];
#pragma unroll
  for (int t = 0; t < kRowTiles; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int k = wave * 32; k < hidden; k += kWaves * 32) {
    const bf16x8 av = __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(urow + k));
#pragma unroll
    for (int t = 0; t < kRowTiles; ++t) {
      if (t < ntile) {
        const bf16x8 bv = __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(arow[t] + k));
        acc[t] = mfma16(av, bv, acc[t]);
      }
    }
  }
#pragma unroll
  for (int t = 0; t < kRowTiles; ++t) red[wave][t][lane] = acc[t];
  __syncthreads();
  if (wave != 0) return;
  // lane holds D[candidate 4 kg + i][node row r16] of each tile; waves summed in order
#pragma unroll
  for (int t = 0; t < kRowTiles; ++t) {
    if (t >= ntile) continue;
    f32x4 v = red[0][t][lane];
#pragma unroll
    for (int w = 1; w < kWaves; ++w) v += red[w][t][lane];
    const int j = 64 * rb + 16 * t + r16;
    if (j >= np) continue;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int cc = 16 * cb + 4 * kg + i;
      if (cc < K) z[(int64_t(q) * np + j) * K + cc] = v[i] + lbv[i];
    }
  }
}

// fp32: grid batch * ceil(np K / 256); thread (q, j, c) computes one dot product.
__global__ __launch_bounds__(256) void shared_logits_f32(int np, int K, int hidden, int vocab, int nblk,
                                                         const float* __restrict__ a,
                                                         const float* __restrict__ U, const float* __restrict__ lb,
                                                         int64_t lb_stride, const int32_t* __restrict__ cset,
                                                         int64_t cset_stride, const int32_t* __restrict__ group_index,
                                                         float* z) {
  const int q = blockIdx.x / nblk;
  const int e = (blockIdx.x % nblk) * blockDim.x + threadIdx.x;
  if (e >= np * K) return;
  const int j = e / K, cc = e % K;
  const int64_t g = group_index ? group_index[q] : q;
  const int tok = min(max(cset[g * cset_stride + cc], 0), vocab - 1);   // clamped as above
  const float* ar = a + (int64_t(q) * np + j) * hidden;
  const float* ur = U + int64_t(tok) * hidden;
  float acc = 0.f;
  for (int k = 0; k < hidden; ++k) acc = fmaf(ar[k], ur[k], acc);
  z[(int64_t(q) * np + j) * K + cc] = acc + lb[g * lb_stride + tok];
}

}  // namespace

size_t candidate_sets_scratch_bytes(int64_t rows, int64_t vocab, int K) {
  (void)vocab;
  return size_t(rows) * K * sizeof(float);   // the codes of the first 2 K groups
}

bool candidate_sets_supported(int64_t vocab, int K) { return K >= 1 && K <= vocab && K <= DARTREE_MAX_CANDIDATES; }

hipError_t launch_candidate_sets(const float* logits, int64_t rows, int64_t vocab, int K, int32_t* ids,
                                 void* scratch, hipStream_t s) {
  if (rows <= 0) return hipSuccess;
  const int G = cset_groups(vocab, K), per = 256 / group_lanes(int(vocab), G), gpb = (G + per - 1) / per;
  hipLaunchKernelGGL(cset_group_max, dim3(unsigned(rows * gpb)), dim3(256), 0, s, logits, int(vocab), K, G, gpb, scratch,
                     ids);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(cset_select, dim3(unsigned(rows)), dim3(1024), 0, s, logits, int(vocab), K, G, scratch, ids);
  return hipGetLastError();
}

hipError_t launch_shared_logits(int precision, int batch, int np, int K, int hidden, int vocab, const void* a,
                                const void* U, const float* lb, int64_t lb_stride, const int32_t* cset,
                                int64_t cset_stride, const int32_t* group_index, float* z, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  if (precision == DARTREE_BF16) {
    const int ncb = (K + 15) / 16, nrb = (np + 16 * kRowTiles - 1) / (16 * kRowTiles);
    hipLaunchKernelGGL(shared_logits_bf16, dim3(unsigned(batch * ncb * nrb)), dim3(1024), 0, s, np, K, hidden, vocab,
                       ncb, nrb, static_cast<const uint16_t*>(a), static_cast<const uint16_t*>(U), lb, lb_stride, cset,
                       cset_stride, group_index, z);
  } else {
    const int nblk = (np * K + 255) / 256;
    hipLaunchKernelGGL(shared_logits_f32, dim3(unsigned(batch * nblk)), dim3(256), 0, s, np, K, hidden, vocab, nblk,
                       static_cast<const float*>(a), static_cast<const float*>(U), lb, lb_stride, cset, cset_stride,
                       group_index, z);
  }
  return hipGetLastError();
}

}  // namespace dartree
