// The consumer of the emitted tree (Sec. 2.1, Sec. 2.3, Sec. 4.1):
//
//  * accept_walk: from the root, move to the child whose token equals the
//    target's token at the current position (its greedy prediction at T = 0,
//    its sample at T = 1) and stop at the first position without one; the
//    target's token there is the bonus.  One wavefront per request, the tree
//    staged in LDS; the loop is bounded by the path capacity and the node
//    count, so it ends on any input.
//  * tree_attention: one attention layer over the flattened tree.  Node i's
//    query attends to the verified context and to the nodes of mask row i.
//    On MFMA: a block owns 64 query rows of one key/value head (16 nodes x 4
//    query heads of a group share every K/V block it loads).  With few rows
//    (one request of a few dozen nodes: too few blocks for the chip) it is
//    flash-decoding: the keys are spread over the waves of a block and over
//    several blocks, partial (max, sum, unnormalised output) go to the
//    workspace and a second kernel merges them.  With many blocks a block
//    sweeps the whole context and then the tree keys with one online softmax
//    and writes the normalised output itself.  S = K Q^T leaves lane l with
//    query row l % 16 and keys 4 (l / 16) + i of every 16-key tile, which is
//    exactly the B operand layout of the P V product when the keys of each
//    32-key chunk are taken in the order {4g..4g+3, 16+4g..16+4g+3} for lane
//    group g = l / 16, so P never leaves the registers.  The sweep transposes
//    V in registers (4 keys x 8 dims per thread) and stores it to LDS with its
//    keys already in that order: one 16-byte read gives a lane its operand.
//    The spread kernel's waves read V once, transposed on the way from LDS.
#include <algorithm>

#include "internal.hpp"

namespace dartree {
namespace {

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// ---------------------------------------------------------------------------
// Acceptance walk
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(64) void accept_walk(int budget, int max_len, const int32_t* __restrict__ tokens,
                                                  const int32_t* __restrict__ parents,
                                                  const int32_t* __restrict__ num_nodes,
                                                  const int32_t* __restrict__ target, int32_t* accepted,
                                                  int32_t* n_accepted, int32_t* bonus) {
  __shared__ int32_t tok[DARTREE_MAX_SORT], par[DARTREE_MAX_SORT];
  const int q = blockIdx.x, lane = threadIdx.x;
  const int n = min(max(num_nodes[q], 0), budget);
  const int64_t tb = int64_t(q) * budget;
  for (int j = lane; j < n; j += 64) {
    tok[j] = tokens[tb + j];
    par[j] = parents[tb + j];
  }
  __syncthreads();
  const int32_t* tgt = target + int64_t(q) * (budget + 1);
  int cur = -1, count = 0;
  const int steps = min(max_len, n);
  while (count < steps) {
    const int want = tgt[cur + 1];
    int found = INT32_MAX;
    for (int j = lane; j < n; j += 64)
      if (par[j] == cur && tok[j] == want) found = min(found, j);
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) found = min(found, __shfl_xor(found, off));
    if (found == INT32_MAX) break;
    if (lane == 0) accepted[int64_t(q) * max_len + count] = found;
    cur = found;
    ++count;
  }
  for (int j = count + lane; j < max_len; j += 64) accepted[int64_t(q) * max_len + j] = -1;
  if (lane == 0) {
    n_accepted[q] = count;
    bonus[q] = tgt[cur + 1];
  }
}

// ---------------------------------------------------------------------------
// Tree attention (head_dim 128)
// ---------------------------------------------------------------------------
constexpr int kD = 128;
constexpr int kKeys = 64;                  // keys per block step
constexpr int kKS = kD + 8;                // padded LDS row of K (bf16)
constexpr int kRows = 64;                  // query rows per block of the spread kernel
constexpr int kVS = kKeys + 8;             // padded LDS row of V^T (bf16)
constexpr int kSegLen = 4 * kKeys;         // context keys per segment, and per share of the workspace
// Spread, sweep or segments, by the number of 64-row blocks.  A spread block
// fills a compute unit's LDS, so past 256 its blocks take a second round and the
// sweep, whose blocks cover all keys with no merge, is the faster one.  Spread /
// sweep, 2048 positions, 32 / 8 heads, 64 nodes: 8 requests (256 blocks) 43.8 /
// 63.8 us, 14 (448) 79.5 / 65.3; 128 nodes, 4 x 500 positions (256) 18.8 / 25.2,
// 7 x 1000 (448) 52.3 / 41.4, 15 x 2048 (960) 150 / 94.  Few rows leave most of a
// tile idle and the layer is bound by the keys' bytes: below 512 blocks those
// take small blocks, one per 256 positions.  Up to 48 rows past 256 blocks (33
// requests x 8 nodes, 2048 positions, 8 / 8 heads: segments 56 us, spread 75, sweep
// 90; 33 x 40 nodes: 85, -, 90; 33 x 60: 101, 92, 93), and up to 24 rows from 81
// on: a spread call's shares are cut for the longest context and wait for it
// (contexts of up to 2048, 12 requests x 1 node 21 / 27 us, 24 x 4 29 / 40; all of
// 2048, 17 x 4 33 / 38, 24 x 16 44 / 42; 40 rows, 12 x 40 27 / 27, 20 x 40 39 / 36),
// unless they may be longer than 4096 (16 x 4 nodes, 8192 positions: 142 / 109;
// where a request has 500 of them, 38 / 16: most segments are empty).
constexpr int kSpreadMaxBlocks = 256, kSegMaxBlocks = 511, kSegMaxRows = 48;
constexpr int kFewRows = 24, kFewRowsBlocks = 80, kFewRowsCtx = 4096;
bool attention_in_segments(int64_t blocks, int rows, int max_ctx) {
  const int above = rows <= kFewRows && max_ctx <= kFewRowsCtx ? kFewRowsBlocks : kSpreadMaxBlocks;
  return rows <= kSegMaxRows && blocks > above && blocks <= kSegMaxBlocks;
}

// Position of key group kg4 (keys 4 kg4 .. 4 kg4 + 3 of a 64-key step) in a
// V^T row: 32-key chunk c = kg4 / 8, lane group g = kg4 % 4, half
// (kg4 / 4) % 2; the chunk holds, per lane group, its 4 keys of the first
// 16-key tile and then its 4 of the second.
__device__ __forceinline__ int vt_pos(int kg4) { return (kg4 >> 3) * 32 + (kg4 & 3) * 8 + ((kg4 >> 2) & 1) * 4; }

// grid: batch * Hkv * row tiles (SEG: * segments), the row tiles of one (request,
// key/value head), which read the same keys and values, on one XCD.  A block has 4 waves, each
// with RG groups of 16 query rows (a row tile is 64 RG), and covers the context
// keys [0, ctx_len) and then the tree keys.  SEG: segment s < nseg_ctx covers
// kSegLen context keys (clipped to the request's length), segment nseg_ctx the
// tree's, and the partial results go to tree_attention_merge.
template <bool SEG, int RG>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2))) void tree_attention_sweep(AttnArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t Ks[kKeys][kKS];
  __shared__ __attribute__((aligned(16))) uint16_t Vt[kD][kVS];
  constexpr int kTileRows = 64 * RG;
  const int nseg = SEG ? a.nseg_ctx + 1 : 1;
  const int rows = a.budget * a.group;
  const int ntile = (rows + kTileRows - 1) / kTileRows;
  int bid = SEG ? int(blockIdx.x) : xcd_order(blockIdx.x, gridDim.x);
  const int seg = bid % nseg;
  bid /= nseg;
  const int rt = bid % ntile;
  bid /= ntile;
  const int kvh = bid % a.heads_kv;
  const int q = bid / a.heads_kv;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int r16 = lane & 15, g = lane >> 4;
  const int clen = a.ctx_len ? min(max(a.ctx_len[q], 0), a.max_ctx) : a.max_ctx;
  const int words = (a.budget + 63) / 64;

  // this lane's query rows (rows past the end are computed on the last row, never stored)
  int row[RG], node[RG], head[RG];
  bf16x8 qf[RG][kD / 32];
  const uint64_t* mrow[RG];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    row[rg] = rt * kTileRows + (wave * RG + rg) * 16 + r16;
    const int rowc = min(row[rg], rows - 1);
    node[rg] = rowc / a.group;
    head[rg] = kvh * a.group + rowc % a.group;
    const uint16_t* qp = a.q + ((int64_t(q) * a.budget + node[rg]) * a.heads_q + head[rg]) * kD + g * 8;
#pragma unroll
    for (int ks = 0; ks < kD / 32; ++ks)
      qf[rg][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(qp + ks * 32));
    mrow[rg] = a.mask + (int64_t(q) * a.budget + node[rg]) * words;
  }

  float m_run[RG], l_run[RG];
  f32x4 o[RG][kD / 16];
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    m_run[rg] = -INFINITY;
    l_run[rg] = 0.f;
#pragma unroll
    for (int dt = 0; dt < kD / 16; ++dt) o[rg][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }

  typedef uint16_t u16x8 __attribute__((ext_vector_type(8)));
  typedef uint16_t u16x4 __attribute__((ext_vector_type(4)));
  // this thread's share of a 64-key step: 4 chunks of K (chunk c = tid + 256 i:
  // key c / 16, dims 8 (c % 16)), and of V the 8 dims 8 (tid / 16) of the 4
  // keys 4 (tid % 16) .. +3.  They are read with buffer loads whose range ends
  // at the step's last valid key (k1), so keys past it read as zero with no
  // per-lane test; the byte offsets within a step are fixed per thread.  The
  // next step's share is loaded while the current one is multiplied.
  const int vkg = threadIdx.x & 15, vdc = threadIdx.x >> 4;
  constexpr int kChunks = kKeys * kD / 8 / 256;
  const int key_bytes = a.heads_kv * kD * 2;
  int koff[kChunks], voff[4];
#pragma unroll
  for (int i = 0; i < kChunks; ++i) {
    const int c = threadIdx.x + 256 * i;
    koff[i] = (c / (kD / 8)) * key_bytes + kvh * kD * 2 + (c % (kD / 8)) * 16;
    voff[i] = (4 * vkg + i) * key_bytes + kvh * kD * 2 + 16 * vdc;
  }
  // keys [k0, k1) of one source (the context, or the tree under the mask)
  auto sweep = [&](const bool tree, const int k0, const int k1) {
    const uint16_t* kbase = tree ? a.k_tree + int64_t(q) * a.budget * a.heads_kv * kD
                                 : a.k_ctx + int64_t(q) * a.max_ctx * a.heads_kv * kD;
    const uint16_t* vbase = tree ? a.v_tree + int64_t(q) * a.budget * a.heads_kv * kD
                                 : a.v_ctx + int64_t(q) * a.max_ctx * a.heads_kv * kD;
    u16x8 kn[kChunks], vn[4];
    auto load_step = [&](int kb) {
      const int bytes = min(k1 - kb, kKeys) * key_bytes;
      const int64_t first = int64_t(kb) * a.heads_kv * kD;
      const __amdgpu_buffer_rsrc_t rk =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(kbase + first), (short)0, bytes, 0x00020000);
      const __amdgpu_buffer_rsrc_t rv =
          __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(vbase + first), (short)0, bytes, 0x00020000);
#pragma unroll
      for (int i = 0; i < kChunks; ++i) kn[i] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, koff[i], 0, 0));
#pragma unroll
      for (int i = 0; i < 4; ++i) vn[i] = __builtin_bit_cast(u16x8, __builtin_amdgcn_raw_buffer_load_b128(rv, voff[i], 0, 0));
    };
    if (k0 < k1) load_step(k0);

    for (int kb = k0; kb < k1; kb += kKeys) {
      __syncthreads();   // every wave is done with the previous step's tiles
#pragma unroll
      for (int i = 0; i < kChunks; ++i) {
        const int c = threadIdx.x + 256 * i;
        *reinterpret_cast<u16x8*>(&Ks[c / (kD / 8)][(c % (kD / 8)) * 8]) = kn[i];
      }
#pragma unroll
      for (int e = 0; e < 8; ++e)
        *reinterpret_cast<u16x4*>(&Vt[8 * vdc + e][vt_pos(vkg)]) = u16x4{vn[0][e], vn[1][e], vn[2][e], vn[3][e]};
      __syncthreads();
      if (kb + kKeys < k1) load_step(kb + kKeys);

      // S[key][query] for the 4 key tiles of 16, every row group
      f32x4 s[RG][4];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) s[rg][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < kD / 32; ++ks) {
          const bf16x8 kf =
              __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(&Ks[t * 16 + r16][ks * 32 + g * 8]));
#pragma unroll
          for (int rg = 0; rg < RG; ++rg) s[rg][t] = mfma16(kf, qf[rg][ks], s[rg][t]);
        }
      }
      // visibility: a context step wholly inside [k0, k1) needs no test
      if (tree || kb + kKeys > k1) {
#pragma unroll
        for (int rg = 0; rg < RG; ++rg) {
          const uint64_t mw = tree ? mrow[rg][kb / 64] : ~0ull;
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int kl = t * 16 + g * 4 + i;   // key within the 64-key step
              if (!(kb + kl < k1 && ((mw >> kl) & 1ull))) s[rg][t][i] = -INFINITY;
            }
        }
      }
      // online softmax on the unscaled scores (scale > 0 keeps the order);
      // p = exp2(scale log2(e) (s - m)).  The running maximum m moves only when
      // a row's new maximum exceeds it by more than 8 / (scale log2(e)), so
      // p <= 2^8 and the rescaling of l and O is skipped for most steps.  A
      // row that has seen no visible key keeps m = -inf, l = 0, O = 0; the
      // arithmetic handles it (exp2(-inf) = 0), so control flow stays uniform
      // around the matrix-core instructions.
      const float c2 = a.scale_log2;
      bf16x8 pb[RG][2];
#pragma unroll
      for (int rg = 0; rg < RG; ++rg) {
        float bmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) bmax = fmaxf(bmax, s[rg][t][i]);
        bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
        bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
        const bool grow = bmax * c2 > m_run[rg] * c2 + 8.f;
        if (__any(grow)) {
          const float m_new = grow ? bmax : m_run[rg];
          const float alpha = __builtin_amdgcn_exp2f((m_run[rg] - (m_new == -INFINITY ? 0.f : m_new)) * c2);
          l_run[rg] *= alpha;
#pragma unroll
          for (int dt = 0; dt < kD / 16; ++dt) o[rg][dt] *= alpha;
          m_run[rg] = m_new;
        }
        const float nmc = -(m_run[rg] == -INFINITY ? 0.f : m_run[rg]) * c2;
        float psum = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[rg][t][i] = __builtin_amdgcn_exp2f(fmaf(s[rg][t][i], c2, nmc));
            psum += s[rg][t][i];
          }
        psum += __shfl_xor(psum, 16);
        psum += __shfl_xor(psum, 32);
        l_run[rg] += psum;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            pb[rg][c][i] = __bf16(s[rg][2 * c][i]);
            pb[rg][c][4 + i] = __bf16(s[rg][2 * c + 1][i]);
          }
      }
      // O[dim][query] += V^T[dim][key] P[query][key] over the two 32-key chunks
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int dt = 0; dt < kD / 16; ++dt) {
          const bf16x8 vv =
              __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(&Vt[dt * 16 + r16][c * 32 + g * 8]));
#pragma unroll
          for (int rg = 0; rg < RG; ++rg) o[rg][dt] = mfma16(vv, pb[rg][c], o[rg][dt]);
        }
    }
  };

  if (SEG) {
    if (seg == a.nseg_ctx) sweep(true, 0, a.budget);
    else sweep(false, seg * kSegLen, min(clen, seg * kSegLen + kSegLen));
#pragma unroll
    for (int rg = 0; rg < RG; ++rg) {
      if (row[rg] >= rows) continue;
      const int64_t pr = ((int64_t(seg) * a.batch + q) * a.heads_kv + kvh) * a.rows_pad + row[rg];
      if (g == 0) {
        a.part_ml[pr * 2] = m_run[rg];
        a.part_ml[pr * 2 + 1] = l_run[rg];
      }
      float* op = a.part_o + pr * kD;
#pragma unroll
      for (int dt = 0; dt < kD / 16; ++dt) *reinterpret_cast<f32x4*>(op + dt * 16 + g * 4) = o[rg][dt];
    }
    return;
  }
  sweep(false, 0, clen);
  sweep(true, 0, a.budget);
#pragma unroll
  for (int rg = 0; rg < RG; ++rg) {
    if (row[rg] >= rows) continue;
    const float inv = l_run[rg] > 0.f ? 1.f / l_run[rg] : 0.f;   // a row that sees nothing is zero
    float* op = a.out + ((int64_t(q) * a.budget + node[rg]) * a.heads_q + head[rg]) * kD;
#pragma unroll
    for (int dt = 0; dt < kD / 16; ++dt) *reinterpret_cast<f32x4*>(op + dt * 16 + g * 4) = o[rg][dt] * inv;
  }
}

// ---------------------------------------------------------------------------
// Few rows: the keys are spread over the waves.  A block owns 64 query rows of
// one key/value head and one of S shares of the 64-key steps (the context's
// ceil(ctx_len / 64), then the tree's); its 8 waves are 4 pairs, step i of a
// request goes to pair i mod 4 S (pair i % 4 of share i / 4 mod S), and each
// wave of a pair holds half of the rows (2 groups of 16).  With enough shares
// every pair has one or two steps, and all keys and values of the block are in
// flight at once: the layer of one request is bound by that one round trip, the
// launches and the fetch of the code itself (hence the rolled loops), not by
// bytes.  Keys and values go to the pair's 32 KB of LDS by buffer loads: rows of
// 256 bytes, 16-byte chunk c of row r at c ^ (r % 16).  V is read transposed
// (ds_read_b64_tr_b16: lane l gets dim l % 16 of keys 4 (l / 16) .. + 3), which
// is the operand order described above.  The pairs' (max, sum, output) meet in
// LDS in pair order; with one share the block writes the output itself,
// otherwise its partial result for tree_attention_merge.
// Measured (both launches): 1 request x 64 nodes, 32 / 8 heads, 2048 positions
// 16.8 + 4.0 us (18.5 + 7.4 with a block per 256 positions); 3 x 100 nodes, 16 / 4
// heads, ragged up to 1500, 18.0 + 4.2 (28.6 together -> 22.0); 1 x 512 nodes x
// 2048 97 -> 45 us, 4 x 128 x 2048 91 -> 41.
// ---------------------------------------------------------------------------
constexpr int kPairLds = 2 * kKeys * kD;     // elements: K, then V
#define LDS_AS __attribute__((address_space(3)))
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
constexpr int vmcnt_imm(int n) { return ((n >> 4) << 14) | (n & 15) | 0x0F70; }

__global__ __launch_bounds__(512, 2) void tree_attention_share(AttnArgs a, int S) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[4 * kPairLds];
  __shared__ float ml[4][64][2];
  const int rows = a.budget * a.group;
  const int ntile = (rows + 63) / 64;
  int bid = xcd_order(blockIdx.x, gridDim.x);
  const int rt = bid % ntile;
  bid /= ntile;
  const int share = bid % S;
  bid /= S;
  const int kvh = bid % a.heads_kv, q = bid / a.heads_kv;
  const int lane = threadIdx.x & 63, r16 = lane & 15, g = lane >> 4;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int pair = wave >> 1, half = wave & 1;
  const int clen = __builtin_amdgcn_readfirstlane(a.ctx_len ? min(max(a.ctx_len[q], 0), a.max_ctx) : a.max_ctx);
  const int nctx = (clen + kKeys - 1) / kKeys, nsteps = nctx + (a.budget + kKeys - 1) / kKeys;
  const int first = 4 * share + pair, stride = 4 * S;
  const int iters = (nsteps - 4 * share + stride - 1) / stride;   // of the block's first pair, which has the most (<= 0: none)

  LDS_AS uint16_t* const lk = (LDS_AS uint16_t*)smem + pair * kPairLds;
  LDS_AS uint16_t* const lv = lk + kKeys * kD;
  const int key_bytes = a.heads_kv * kD * 2;
  auto keys_of = [&](int step, bool& tree, int& kb, int& n) {
    tree = step >= nctx;
    kb = (tree ? step - nctx : step) * kKeys;
    n = min(kKeys, (tree ? a.budget : clen) - kb);
  };
  // this wave's half of a step's rows; fill i: rows 4 i + l / 16, chunk
  // (l % 16) ^ row at position l % 16; the range ends at the step's last key,
  // and rows past it are filled with zeros
  auto fill = [&](int step, bool v) __attribute__((always_inline)) {
    bool tree;
    int kb, n;
    keys_of(step, tree, kb, n);
    const uint16_t* base = tree ? (v ? a.v_tree : a.k_tree) + (int64_t(q) * a.budget + kb) * a.heads_kv * kD
                                : (v ? a.v_ctx : a.k_ctx) + (int64_t(q) * a.max_ctx + kb) * a.heads_kv * kD;
    const __amdgpu_buffer_rsrc_t rs =
        __builtin_amdgcn_make_buffer_rsrc(const_cast<uint16_t*>(base), (short)0, n * key_bytes, 0x00020000);
    LDS_AS uint16_t* const dst = v ? lv : lk;
#pragma unroll 2
    for (int j = 0; j < 8; ++j) {
      const int i = 8 * half + j;
      __builtin_amdgcn_raw_ptr_buffer_load_lds(
          rs, (LDS_AS void*)(dst + i * 4 * kD), 16,
          (4 * i + g) * key_bytes + kvh * kD * 2 + ((r16 ^ ((4 * i + g) & 15)) * 16), 0, 0, 0);
    }
  };
  auto barrier = [] {
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("s_barrier" ::: "memory");
    __builtin_amdgcn_sched_barrier(0);
  };
  // the first step's keys and values go out before anything else is worked out
  if (first < nsteps) {
    fill(first, false);
    fill(first, true);
  }
  __builtin_amdgcn_sched_barrier(0);

  // the pair's first tree step, whose mask words are fetched with the queries
  int tree0 = first;
  if (tree0 < nctx) tree0 += (nctx - tree0 + stride - 1) / stride * stride;
  const int words = (a.budget + 63) / 64;
  int row[2];
  bf16x8 qf[2][kD / 32];
  const uint64_t* mrow[2];
  uint64_t mw0[2];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    row[r] = rt * 64 + half * 32 + r * 16 + r16;
    const int rowc = min(row[r], rows - 1);   // rows past the end: computed on the last row, never stored
    const int node = rowc / a.group, head = kvh * a.group + (rowc - node * a.group);
    const uint16_t* qp = a.q + ((int64_t(q) * a.budget + node) * a.heads_q + head) * kD + g * 8;
#pragma unroll
    for (int ks = 0; ks < kD / 32; ++ks)
      qf[r][ks] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const f32x4*>(qp + ks * 32));
    mrow[r] = a.mask + (int64_t(q) * a.budget + node) * words;
    mw0[r] = mrow[r][min(max(tree0 - nctx, 0), words - 1)];
  }
  float m_run[2], l_run[2];
  f32x4 o[2][kD / 16];
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    m_run[r] = -INFINITY;
    l_run[r] = 0.f;
#pragma unroll
    for (int dt = 0; dt < kD / 16; ++dt) o[r][dt] = f32x4{0.f, 0.f, 0.f, 0.f};
  }
  const int vr = 4 * g + (r16 >> 2);   // V row (mod 16) this lane addresses in a transposed read
  const float c2 = a.scale_log2;
  // From here on the waits count fills, and register loads need not finish in
  // order with them: none may be in flight.
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
  barrier();   // the first step's keys and values landed
#pragma unroll 1
  for (int it = 0; it < iters; ++it) {
    const int step = first + it * stride;
    const bool act = step < nsteps, next = step + stride < nsteps, more = it + 1 < iters;   // more: block-uniform
    bool tree;
    int kb, n;
    keys_of(step, tree, kb, n);
    if (it > 0) {   // K landed (V's 8 fills may be in flight)
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
      barrier();
    }
    f32x4 s[2][4];
    if (act) {
#pragma unroll
      for (int t = 0; t < 4; ++t) {
#pragma unroll
        for (int r = 0; r < 2; ++r) s[r][t] = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int ks = 0; ks < 4; ++ks) {
          const bf16x8 kf = __builtin_bit_cast(
              bf16x8, *reinterpret_cast<const LDS_AS u32x4*>(lk + t * 16 * kD + r16 * kD + (((4 * ks + g) ^ r16) * 8)));
#pragma unroll
          for (int r = 0; r < 2; ++r) s[r][t] = mfma16(kf, qf[r][ks], s[r][t]);
        }
      }
    }
    uint64_t mw[2];
#pragma unroll
    for (int r = 0; r < 2; ++r) mw[r] = tree ? mw0[r] : ~0ull;
    if (act && tree && step != tree0) {   // no fill may be in flight with these loads
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
#pragma unroll
      for (int r = 0; r < 2; ++r) mw[r] = mrow[r][step - nctx];
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __builtin_amdgcn_sched_barrier(0);
    }
    if (more) {   // both waves have K in registers: its LDS may be refilled
      __builtin_amdgcn_s_waitcnt(0xC07F);
      barrier();
      if (next) fill(step + stride, false);
    }
    bf16x8 pb[2][2];
    if (act) {
#pragma unroll
      for (int r = 0; r < 2; ++r) {
        if (tree || n < kKeys) {
#pragma unroll
          for (int t = 0; t < 4; ++t)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const int kl = t * 16 + g * 4 + i;
              if (!(kl < n && ((mw[r] >> kl) & 1ull))) s[r][t][i] = -INFINITY;
            }
        }
        // online softmax as in tree_attention_sweep
        float bmax = -INFINITY;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) bmax = fmaxf(bmax, s[r][t][i]);
        bmax = fmaxf(bmax, __shfl_xor(bmax, 16));
        bmax = fmaxf(bmax, __shfl_xor(bmax, 32));
        const bool grow = bmax * c2 > m_run[r] * c2 + 8.f;
        if (__any(grow)) {
          const float m_new = grow ? bmax : m_run[r];
          const float alpha = __builtin_amdgcn_exp2f((m_run[r] - (m_new == -INFINITY ? 0.f : m_new)) * c2);
          l_run[r] *= alpha;
#pragma unroll
          for (int dt = 0; dt < kD / 16; ++dt) o[r][dt] *= alpha;
          m_run[r] = m_new;
        }
        const float nmc = -(m_run[r] == -INFINITY ? 0.f : m_run[r]) * c2;
        float psum = 0.f;
#pragma unroll
        for (int t = 0; t < 4; ++t)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            s[r][t][i] = __builtin_amdgcn_exp2f(fmaf(s[r][t][i], c2, nmc));
            psum += s[r][t][i];
          }
        psum += __shfl_xor(psum, 16);
        psum += __shfl_xor(psum, 32);
        l_run[r] += psum;
#pragma unroll
        for (int c = 0; c < 2; ++c)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            pb[r][c][i] = __bf16(s[r][2 * c][i]);
            pb[r][c][4 + i] = __bf16(s[r][2 * c + 1][i]);
          }
      }
    }
    if (it > 0) {   // V landed (the next K's fills may be in flight)
      __builtin_amdgcn_sched_barrier(0);
      if (next) __builtin_amdgcn_s_waitcnt(vmcnt_imm(8));
      else __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      barrier();
    }
    if (act) {
#pragma unroll
      for (int c = 0; c < 2; ++c)
#pragma unroll
        for (int dt = 0; dt < kD / 16; ++dt) {
          const int va = (32 * c + vr) * kD + (((2 * dt + ((r16 & 3) >> 1)) ^ vr) * 8) + (r16 & 1) * 4;
          const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(lv + va));
          const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((LDS_AS s16x4*)(lv + va + 16 * kD));
          const bf16x8 vv = __builtin_bit_cast(bf16x8, s16x8{lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], hi[2], hi[3]});
#pragma unroll
          for (int r = 0; r < 2; ++r) o[r][dt] = mfma16(vv, pb[r][c], o[r][dt]);
        }
    }
    if (more) {   // both waves have V in registers
      __builtin_amdgcn_s_waitcnt(0xC07F);
      barrier();
      if (next) fill(step + stride, true);
    }
  }

  // The pairs' results in pair order: each wave scales its rows to the block's
  // maximum and hands them over through LDS; wave w adds up and stores dims
  // 64 (w % 2) .. of row group w / 2.
  if (g == 0) {
#pragma unroll
    for (int r = 0; r < 2; ++r) {
      ml[pair][half * 32 + r * 16 + r16][0] = m_run[r];
      ml[pair][half * 32 + r * 16 + r16][1] = l_run[r];
    }
  }
  __syncthreads();   // every wave is done with its keys and values
  f32x4* const red = reinterpret_cast<f32x4*>(smem);   // [pair][group][dt][lane]
#pragma unroll
  for (int r = 0; r < 2; ++r) {
    const int lr = half * 32 + r * 16 + r16;
    float M = ml[0][lr][0];
#pragma unroll
    for (int p = 1; p < 4; ++p) M = fmaxf(M, ml[p][lr][0]);
    const float f = m_run[r] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((m_run[r] - M) * c2);
#pragma unroll
    for (int dt = 0; dt < kD / 16; ++dt) red[((pair * 4 + 2 * half + r) * (kD / 16) + dt) * 64 + lane] = o[r][dt] * f;
  }
  __syncthreads();
  const int rg = wave >> 1, lr = rg * 16 + r16, rw = rt * 64 + lr;
  if (rw >= rows) return;
  float M = ml[0][lr][0], L = 0.f;
#pragma unroll
  for (int p = 1; p < 4; ++p) M = fmaxf(M, ml[p][lr][0]);
#pragma unroll
  for (int p = 0; p < 4; ++p) {
    const float mp = ml[p][lr][0];
    L += (mp == -INFINITY ? 0.f : __builtin_amdgcn_exp2f((mp - M) * c2)) * ml[p][lr][1];
  }
  const int64_t pr = ((int64_t(share) * a.batch + q) * a.heads_kv + kvh) * a.rows_pad + rw;
  const int node = rw / a.group, head = kvh * a.group + (rw - node * a.group);
  float* op = S == 1 ? a.out + ((int64_t(q) * a.budget + node) * a.heads_q + head) * kD : a.part_o + pr * kD;
  const float inv = S > 1 ? 1.f : L > 0.f ? 1.f / L : 0.f;   // a row that sees nothing is zero
  if (S > 1 && g == 0 && (wave & 1) == 0) {
    a.part_ml[pr * 2] = M;
    a.part_ml[pr * 2 + 1] = L;
  }
#pragma unroll
  for (int e = 0; e < kD / 32; ++e) {
    const int dt = (wave & 1) * (kD / 32) + e;
    f32x4 v = red[(rg * (kD / 16) + dt) * 64 + lane];
#pragma unroll
    for (int p = 1; p < 4; ++p) v += red[((p * 4 + rg) * (kD / 16) + dt) * 64 + lane];
    *reinterpret_cast<f32x4*>(op + dt * 16 + g * 4) = v * inv;
  }
}

// Merge the S shares: 32 lanes per (request, node, query head), four dims each.
// Weights w_s = exp2(scale log2(e) (m_s - M)) / L (m_s the share's unscaled row
// maximum, M their maximum).  A share's maximum, sum and output are loaded
// together, eight shares at a time, and folded online, so a row waits one round
// trip per eight shares.
__global__ __launch_bounds__(256) void tree_attention_merge(AttnArgs a, int S) {
  const int64_t t = int64_t(blockIdx.x) * 8 + (threadIdx.x >> 5);   // (request, node, query head)
  if (t >= int64_t(a.batch) * a.budget * a.heads_q) return;
  const int head = int(t % a.heads_q), node = int(t / a.heads_q % a.budget), q = int(t / a.heads_q / a.budget);
  const int d = 4 * (threadIdx.x & 31);
  const int kvh = head / a.group, row = node * a.group + head % a.group;
  const int64_t step = int64_t(a.batch) * a.heads_kv * a.rows_pad;
  const int64_t p0 = (int64_t(q) * a.heads_kv + kvh) * a.rows_pad + row;
  float M = -INFINITY, L = 0.f;
  f32x4 acc{0.f, 0.f, 0.f, 0.f};
  constexpr int B = 8;
  typedef float f32x2 __attribute__((ext_vector_type(2)));
  for (int s0 = 0; s0 < S; s0 += B) {
    f32x2 ml[B];
    f32x4 o[B];
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const int64_t p = p0 + min(s0 + i, S - 1) * step;
      ml[i] = *reinterpret_cast<const f32x2*>(a.part_ml + 2 * p);
      o[i] = *reinterpret_cast<const f32x4*>(a.part_o + p * kD + d);
    }
    float m = M;
#pragma unroll
    for (int i = 0; i < B; ++i) m = fmaxf(m, ml[i][0]);
    if (m == -INFINITY) continue;
    const float f = __builtin_amdgcn_exp2f((M - m) * a.scale_log2);
    L *= f;
    acc *= f;
    M = m;
#pragma unroll
    for (int i = 0; i < B; ++i) {
      const float w = s0 + i < S ? __builtin_amdgcn_exp2f((ml[i][0] - m) * a.scale_log2) : 0.f;
      L += w * ml[i][1];
      acc += o[i] * w;
    }
  }
  const float inv = L > 0.f ? 1.f / L : 0.f;   // a row that sees nothing is zero
  *reinterpret_cast<f32x4*>(a.out + ((int64_t(q) * a.budget + node) * a.heads_q + head) * kD + d) = acc * inv;
}

// Shares of the key steps: one block of tree_attention_share per compute unit
// is resident (128 KB of LDS), so a choice costs rounds over 256 units times
// steps per wave, plus about two steps a round for the queries and the merging
// of the waves.  The workspace holds one share per 256 context positions and one
// for the tree.
int attention_shares(const AttnArgs& a) {
  const int64_t blocks = int64_t(a.batch) * a.heads_kv * ((a.budget * a.group + 63) / 64);
  const int steps = (a.max_ctx + kKeys - 1) / kKeys + (a.budget + kKeys - 1) / kKeys;
  int best = 1;
  int64_t cost = INT64_MAX;
  for (int S = 1; S <= std::min<int64_t>(std::min(a.nseg_ctx + 1, 256), std::max<int64_t>(1, 1024 / blocks)); ++S) {
    const int64_t c = (blocks * S + 255) / 256 * ((steps + 4 * S - 1) / (4 * S) + 2);
    if (c < cost) {
      cost = c;
      best = S;
    }
  }
  return best;
}

}  // namespace

constexpr int kMaxSegments = 1024;   // workspace limit: context segments of 256 and the tree

int attention_segment_len() { return kSegLen; }
int attention_max_segments() { return kMaxSegments; }
bool attention_needs_workspace(int batch, int budget, int heads_q, int heads_kv) {
  const int64_t rows = int64_t(budget) * (heads_q / heads_kv);
  return int64_t(batch) * heads_kv * ((rows + kRows - 1) / kRows) <= kSegMaxBlocks;
}

hipError_t launch_accept_walk(int batch, int budget, int max_len, const int32_t* tokens, const int32_t* parents,
                              const int32_t* num_nodes, const int32_t* target, int32_t* accepted,
                              int32_t* n_accepted, int32_t* bonus, hipStream_t s) {
  if (batch <= 0) return hipSuccess;
  hipLaunchKernelGGL(accept_walk, dim3(unsigned(batch)), dim3(64), 0, s, budget, max_len, tokens, parents,
                     num_nodes, target, accepted, n_accepted, bonus);
  return hipGetLastError();
}

hipError_t launch_tree_attention(const AttnArgs& a, hipStream_t s) {
  if (a.batch <= 0) return hipSuccess;
  const int rows = a.budget * a.group;
  const int ntile = (rows + kRows - 1) / kRows;
  const int64_t blocks = int64_t(a.batch) * a.heads_kv * ntile;
  const bool seg = attention_in_segments(blocks, rows, a.max_ctx);
  if (!seg && blocks > kSpreadMaxBlocks) {
    const int ntile2 = (rows + 2 * kRows - 1) / (2 * kRows);   // 128-row tiles
    hipLaunchKernelGGL((tree_attention_sweep<false, 2>), dim3(unsigned(a.batch) * a.heads_kv * ntile2), dim3(256), 0, s, a);
    return hipGetLastError();
  }
  const int S = seg ? a.nseg_ctx + 1 : attention_shares(a);
  if (seg) hipLaunchKernelGGL((tree_attention_sweep<true, 1>), dim3(unsigned(blocks * S)), dim3(256), 0, s, a);
  else hipLaunchKernelGGL(tree_attention_share, dim3(unsigned(blocks * S)), dim3(512), 0, s, a, S);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || (S == 1 && !seg)) return e;
  const int64_t out_rows = int64_t(a.batch) * a.budget * a.heads_q;
  hipLaunchKernelGGL(tree_attention_merge, dim3(unsigned((out_rows + 7) / 8)), dim3(256), 0, s, a, S);
  return hipGetLastError();
}

}  // namespace dartree
