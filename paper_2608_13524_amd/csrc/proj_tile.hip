// Products of more than 64 node rows (the batched workloads' depths), and of
// 17..64 rows against matrices of middle length:
//   out[m][n] = epilogue(bias, sum_k x[m][k] w[n][k]),  w = A or U [N][K].
//
// A block of 8 waves owns a tile of BM = 32 RT node rows x BN = 64 NT weight
// rows (RT 2..8 by the number of rows, NT 4 or, for the last columns, less; short
// matrices both by cost);
// wave (g, q) owns 16 RT node rows x 16 NT weight rows of it, accumulated on
// v_mfma_f32_16x16x32_bf16 over the whole K loop (no sums across waves or
// blocks: every output is one chain over K, with 64-row tiles up to 16).
//
// Bound: up to about 200 rows the stream of w from HBM; above, the matrix
// cores at a power-limited clock and the waits around the LDS (1024 rows x 151936
// x 5120, by counters: matrix cores busy 64% of the cycles, operand reads 25%, no
// bank conflicts, 3.07 GB moved).  Hence the schedule:
//  * both operands go memory -> LDS by buffer loads, rows of 64 k (128 bytes)
//    with 16-byte chunk c of row r at c ^ (r % 8) (conflict-free reads), S
//    steps in a ring;
//  * a step is four clusters of RT/2 x NT/2 products per wave (node half 0/1 x
//    weight half 0/1 in the order 00, 01, 11, 10), each preceded by a memory
//    part that reads the operands of the next clusters (at most 8 16-byte
//    reads a wave) and refills the ring's halves just read, S steps ahead;
//  * the two groups of waves run half a cluster apart, so on every SIMD one
//    wave multiplies while the other reads; a barrier ends every part.  The
//    waits are explicit: a read is waited for at the end of the part before
//    its use, and a fill (vmcnt counts only fills: nothing else is loaded in
//    the loop) before the barrier that precedes its first read in any wave.
// A tile past a whole number of rounds over the compute units would leave
// most of them idle, so the last columns are cut into narrower tiles.
// Measured on one MI355X (dartree_project, product only, against 128 x 128
// tiles up to 511 rows, split 512 x 128 / 256 x 256 tiles above): 128 x 151936
// x 4096 421 -> 228 us, 256 rows 577 -> 295 us, 300 x 50257 x 2560 223 -> 118
// us, 1024 x 151936 x 5120 1500-1540 -> 1250-1275 us in a loop of its own
// (1.25-1.27 PFLOP/s; 1240-1375 us in a round and next to the softmax pass), 1024
// x 5120 x 5120 115 -> 71 us.
// No faster: four waves of 128 x 128 (one per SIMD, 1480-1560 us at the 1024
// rows), ten 16 KB ring slots instead of two whole stages (1275 us), the
// operands of a cluster all read in the part before it (1311 us).
#include <algorithm>
#include <type_traits>

#include "internal.hpp"

namespace dartree {
namespace {

typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
#define LDS_AS __attribute__((address_space(3)))

struct TileArgs {
  const uint16_t* x;
  const uint16_t* w;
  int M, N, K;
  int rows_per_group;
  int64_t bias_stride;
  const float* bias_f32;
  const uint16_t* bias_act;
  const int32_t* group_index;
  float* out;
  uint16_t* act_out;
  // tiles [0, full) cover weight rows [0, 256 nf) with NT = 4; the others
  // cover the rest with NT = tail
  int full, nf, tail;
  int nt_out;   // logits stored non-temporally
};

__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
constexpr int vmcnt_imm(int n) { return ((n >> 4) << 14) | (n & 15) | 0x0F70; }
constexpr int lgkm_imm(int n) { return 0xC07F | (n << 8); }
constexpr int kAuxNT = 2;   // cache policy: non-temporal

__device__ __forceinline__ int64_t group_row(const TileArgs& a, int g) {
  return int64_t(a.group_index ? a.group_index[g] : g) * a.bias_stride;
}

template <int EPI>
__device__ __forceinline__ float bias_at(const TileArgs& a, int64_t row, int n) {
  if constexpr (EPI == EPI_LOGITS) return a.bias_f32[row + n];
  else return bf16_to_f32(a.bias_act[row + n]);
}

// Stages of the ring: as many as fit 160 KB with BN = 256.
constexpr int tile_stages(int RT) {
  return (32 * RT + 256) * 128 * 4 <= 160 * 1024 ? 4 : (32 * RT + 256) * 128 * 3 <= 160 * 1024 ? 3 : 2;
}

// One tile at (m0, n0).  WAUX: cache policy of the weight fills.
template <int RT, int NT, int EPI, int WAUX>
struct Tile {
  static constexpr int S = tile_stages(RT);
  static constexpr int RT0 = (RT + 1) / 2, RT1 = RT - RT0;   // node tiles of the two halves
  static constexpr int NT0 = (NT + 1) / 2, NT1 = NT - NT0;   // weight tiles
  static constexpr int BM = 32 * RT, BN = 64 * NT;
  // fills (8 rows each) per wave and step of the halves of x; NT of w
  static constexpr int I0 = (4 * RT0 + 7) / 8, I1 = (4 * RT1 + 7) / 8;
  static constexpr int P = I0 + I1 + NT;
  static constexpr int kStage = (BM + BN) * 64;   // elements
  // a stage: x half 0 [2][16 RT0] rows, x half 1 [2][16 RT1], w half 0 [4][16 NT0], w half 1 [4][16 NT1]
  static constexpr int oX1 = 32 * RT0 * 64, oW0 = BM * 64, oW1 = oW0 + 64 * NT0 * 64;
  static_assert((S - 1) * P <= 63, "vmcnt range");
  // 64-row tiles (17..64 rows) add K up in kPieces partial sums, as the stream
  // kernels do with their waves: one chain over K is 2 to 3 times as far from the
  // exact sum (20 rows x 16000 x 4096: 1.6e-7 of the norm, 5e-8 so), and these have
  // the registers for a second set.
  static constexpr bool kSums = RT == 2;
  static constexpr int kPieces = 16;

  static __device__ __forceinline__ void run(const TileArgs& a, int m0, int n0, uint16_t* smem) {
    LDS_AS uint16_t* const lds = (LDS_AS uint16_t*)smem;
    const int lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = wave >> 2, q = wave & 3;
    const int M = a.M, N = a.N, K = a.K, nk = K >> 6;
    const unsigned rowb = unsigned(K) * 2u;
    const int mrows = min(BM, M - m0), nrows = min(BN, N - n0);
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.x + int64_t(m0) * K), (short)0, mrows * K * 2, 0x00020000);
    const __amdgpu_buffer_rsrc_t rw = __builtin_amdgcn_make_buffer_rsrc(
        const_cast<uint16_t*>(a.w + int64_t(n0) * K), (short)0, nrows * K * 2, 0x00020000);
    // Fill f of a half: LDS rows 8 f .. 8 f + 7, lane l row 8 f + l / 8, chunk
    // (l % 8) ^ (row % 8) at position l % 8.  Rows past M or N repeat the last
    // one (computed, never stored); where a half has fewer fills than waves
    // the surplus waves repeat one (the same bytes to the same place).
    const unsigned pc = unsigned(((lane & 7) ^ (lane >> 3)) * 16);
    unsigned vx0[I0], vx1[I1], vw0[NT0], vw1[NT1 ? NT1 : 1];
    int lx0[I0], lx1[I1], lw0[NT0], lw1[NT1 ? NT1 : 1];
#pragma unroll
    for (int i = 0; i < I0; ++i) {
      const int f = (wave + 8 * i) % (4 * RT0), r = 8 * f + (lane >> 3);
      const int m = (r / (16 * RT0)) * 16 * RT + r % (16 * RT0);
      vx0[i] = unsigned(min(m, mrows - 1)) * rowb + pc;
      lx0[i] = 8 * f * 64;
    }
#pragma unroll
    for (int i = 0; i < I1; ++i) {
      const int f = (wave + 8 * i) % (4 * RT1), r = 8 * f + (lane >> 3);
      const int m = (r / (16 * RT1)) * 16 * RT + 16 * RT0 + r % (16 * RT1);
      vx1[i] = unsigned(min(m, mrows - 1)) * rowb + pc;
      lx1[i] = oX1 + 8 * f * 64;
    }
#pragma unroll
    for (int i = 0; i < NT0; ++i) {
      const int f = wave + 8 * i, r = 8 * f + (lane >> 3);
      const int n = (r / (16 * NT0)) * 16 * NT + r % (16 * NT0);
      vw0[i] = unsigned(min(n, nrows - 1)) * rowb + pc;
      lw0[i] = oW0 + 8 * f * 64;
    }
#pragma unroll
    for (int i = 0; i < NT1; ++i) {
      const int f = wave + 8 * i, r = 8 * f + (lane >> 3);
      constexpr int R1 = 16 * (NT1 ? NT1 : 1);
      const int n = (r / R1) * 16 * NT + 16 * NT0 + r % R1;
      vw1[i] = unsigned(min(n, nrows - 1)) * rowb + pc;
      lw1[i] = oW1 + 8 * f * 64;
    }
    // Fills past the last step repeat it (into stages nothing reads any
    // more), so that every step issues the same number and the waits can count.
    auto kbytes = [&](int kt) __attribute__((always_inline)) { return unsigned(min(kt, nk - 1)) * 128u; };
    auto fill_x = [&](int dst, unsigned vo, unsigned so) __attribute__((always_inline)) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rx, (LDS_AS void*)(lds + dst), 16, vo, so, 0, 0);
    };
    auto fill_w = [&](int dst, unsigned vo, unsigned so) __attribute__((always_inline)) {
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rw, (LDS_AS void*)(lds + dst), 16, vo, so, 0, WAUX);
    };
    auto fill_h0 = [&](int kt, int st) __attribute__((always_inline)) {   // halves 0 of x and w
#pragma unroll
      for (int i = 0; i < I0; ++i) fill_x(st * kStage + lx0[i], vx0[i], kbytes(kt));
#pragma unroll
      for (int i = 0; i < NT0; ++i) fill_w(st * kStage + lw0[i], vw0[i], kbytes(kt));
    };
    auto fill_w1 = [&](int kt, int st) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < NT1; ++i) fill_w(st * kStage + lw1[i], vw1[i], kbytes(kt));
    };
    auto fill_x1 = [&](int kt, int st) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < I1; ++i) fill_x(st * kStage + lx1[i], vx1[i], kbytes(kt));
    };
    // A bare barrier: the workgroup fence of __syncthreads would also wait for
    // the fills in flight.
    auto barrier = [] {
      __builtin_amdgcn_sched_barrier(0);
      asm volatile("s_barrier" ::: "memory");
      __builtin_amdgcn_sched_barrier(0);
    };
    auto lgkm = [](auto Nc) {
      __builtin_amdgcn_sched_barrier(0);
      __builtin_amdgcn_s_waitcnt(lgkm_imm(decltype(Nc)::value));
    };
    auto vm = [](auto Nc) { __builtin_amdgcn_s_waitcnt(vmcnt_imm(decltype(Nc)::value)); };

    f32x4 acc[RT][NT], sum[kSums ? RT : 1][kSums ? NT : 1];
#pragma unroll
    for (int i = 0; i < RT; ++i)
#pragma unroll
      for (int j = 0; j < NT; ++j) {
        acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
        if constexpr (kSums) sum[i][j] = acc[i][j];
      }
    // steps of a partial sum (at most kPieces of them, of two steps and more: a
    // sum waits for the products)
    const int piece = kSums ? max(2, (nk + kPieces - 1) / kPieces) : nk;
    int left = piece;
    // operand fragments of a 64-deep step, [tile][32-deep sub-step]: lane l
    // row l % 16, chunk 4 u + l / 16
    bf16x8 x0[RT0][2], x1[RT1][2], w0[NT0][2], w1[NT1 ? NT1 : 1][2];
    constexpr int RA = (RT0 + 1) / 2;   // tiles of x half 0 read before cluster 11, the rest before cluster 10
    const int px0 = (g * 16 * RT0 + r16) * 64, px1 = oX1 + (g * 16 * RT1 + r16) * 64;
    const int pw0 = oW0 + (q * 16 * NT0 + r16) * 64, pw1 = oW1 + (q * 16 * NT1 + r16) * 64;
    const int cs[2] = {(kg ^ (r16 & 7)) * 8, ((4 + kg) ^ (r16 & 7)) * 8};
    auto read = [&](bf16x8 (&f)[2], int p, int i) __attribute__((always_inline)) {
#pragma unroll
      for (int u = 0; u < 2; ++u)
        f[u] = __builtin_bit_cast(bf16x8, *reinterpret_cast<const LDS_AS u32x4*>(lds + p + i * 1024 + cs[u]));
    };
    // cluster: node tiles xb .. of fragments xf, weight tiles wb .. of wf
    auto multiply = [&](auto& xf, auto XN, auto XB, auto& wf, auto WN, auto WB) __attribute__((always_inline)) {
      constexpr int xn = decltype(XN)::value, xb = decltype(XB)::value, wn = decltype(WN)::value, wb = decltype(WB)::value;
      __builtin_amdgcn_s_setprio(1);
#pragma unroll
      for (int u = 0; u < 2; ++u)
#pragma unroll
        for (int i = 0; i < xn; ++i)
#pragma unroll
          for (int j = 0; j < wn; ++j) acc[xb + i][wb + j] = mfma16(xf[i][u], wf[j][u], acc[xb + i][wb + j]);
      __builtin_amdgcn_s_setprio(0);
    };
    constexpr std::integral_constant<int, 0> c0{};
    constexpr std::integral_constant<int, RT0> cRT0{};
    constexpr std::integral_constant<int, RT1> cRT1{};
    constexpr std::integral_constant<int, NT0> cNT0{};
    constexpr std::integral_constant<int, NT1> cNT1{};

    for (int s = 0; s < S; ++s) {
      fill_h0(s, s);
      fill_w1(s, s);
      fill_x1(s, s);
    }
    vm(std::integral_constant<int, (S - 1) * P>{});   // step 0 landed
    barrier();
#pragma unroll
    for (int i = 0; i < RT0; ++i) read(x0[i], px0, i);
    if (g == 1) barrier();   // group 1 runs one part behind
    int st = 0;
#pragma unroll 1
    for (int s = 0; s < nk; ++s) {
      const int stn = st == S - 1 ? 0 : st + 1;
      const int b = st * kStage, bn = stn * kStage;
      // Landed at the loop's top, in every wave: x half 0 of step s (in
      // registers), w of step s.
      // cluster 00 (x half 0, w half 0); reads all of w
#pragma unroll
      for (int j = 0; j < NT0; ++j) read(w0[j], b + pw0, j);
#pragma unroll
      for (int j = 0; j < NT1; ++j) read(w1[j], b + pw1, j);
      vm(std::integral_constant<int, (S - 1) * P>{});        // x half 1 of step s
      lgkm(std::integral_constant<int, 2 * NT1>{});          // x half 0, w half 0
      barrier();
      multiply(x0, cRT0, c0, w0, cNT0, c0);
      barrier();
      // cluster 01; reads x half 1; both groups have read halves 0 of step s
#pragma unroll
      for (int i = 0; i < RT1; ++i) read(x1[i], b + px1, i);
      vm(std::integral_constant<int, (S - 1) * P - I0>{});   // x half 0 of step s + 1
      fill_h0(s + S, st);
      lgkm(std::integral_constant<int, 2 * RT1>{});          // w half 1
      barrier();
      if constexpr (NT1 > 0) multiply(x0, cRT0, c0, w1, cNT1, cNT0);
      barrier();
      // cluster 11; reads the first of the next step's x half 0; w half 1 was read
#pragma unroll
      for (int i = 0; i < RA; ++i) read(x0[i], bn + px0, i);
      fill_w1(s + S, st);
      lgkm(std::integral_constant<int, 2 * RA>{});           // x half 1
      barrier();
      if constexpr (NT1 > 0) multiply(x1, cRT1, cRT0, w1, cNT1, cNT0);
      barrier();
      // cluster 10; reads the rest of it; x half 1 was read
#pragma unroll
      for (int i = RA; i < RT0; ++i) read(x0[i], bn + px0, i);
      vm(std::integral_constant<int, (S - 1) * P>{});        // w of step s + 1
      fill_x1(s + S, st);
      barrier();
      multiply(x1, cRT1, cRT0, w0, cNT0, c0);
      if constexpr (kSums) {
        if (--left == 0) {
          left = piece;
#pragma unroll
          for (int i = 0; i < RT; ++i)
#pragma unroll
            for (int j = 0; j < NT; ++j) {
              sum[i][j] += acc[i][j];
              acc[i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            }
        }
      }
      barrier();
      st = stn;
    }
    if constexpr (kSums) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] += sum[i][j];
    }
    if (g == 0) barrier();
    vm(std::integral_constant<int, 0>{});   // the repeated fills land before the block's LDS goes

    if (a.rows_per_group >= 16) {
      if (EPI == EPI_LOGITS && a.nt_out) store<true, true>(a, acc, m0, n0, mrows);
      else store<true, false>(a, acc, m0, n0, mrows);
    } else {
      store<false, false>(a, acc, m0, n0, mrows);
    }
  }

  // Lane l of acc[i][j][v] holds node row 16 RT g + 16 i + 4 (l / 16) + v and
  // weight row 16 NT q + 16 j + l % 16.  Swapping 16-lane rows between the
  // registers of two neighbouring weight tiles gives each store instruction
  // two whole 128-byte lines (32 consecutive n of rows mt + 8 (l / 32) + v and
  // of + 4).  The buffer's range ends at row M; columns past N get an offset
  // beyond it.  GROUP16: 16 rows meet at most two bias groups.
  template <bool GROUP16, bool NTS>
  static __device__ __forceinline__ void store(const TileArgs& a, f32x4 (&acc)[RT][NT], int m0, int n0, int mrows) {
    const int lane = threadIdx.x & 63, r16 = lane & 15, kg = lane >> 4, h2 = lane >> 5, l5 = lane & 31;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int g = wave >> 2, q = wave & 3;
    const int M = a.M, N = a.N;
    const __amdgpu_buffer_rsrc_t ro = __builtin_amdgcn_make_buffer_rsrc(
        a.out + int64_t(m0) * N, (short)0, unsigned(mrows) * unsigned(N) * 4u, 0x00020000);
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(
        EPI == EPI_HEAD ? a.act_out + int64_t(m0) * N : nullptr, (short)0,
        EPI == EPI_HEAD ? unsigned(mrows) * unsigned(N) * 2u : 0u, 0x00020000);
#pragma unroll
    for (int i = 0; i < RT; ++i) {
      const int mt = 16 * RT * g + 16 * i;   // first row of the 16, within the tile
      if (mt >= mrows) break;
      // the group of the first row, the row where the next one begins and the two groups' bias rows
      const int g0 = (m0 + mt) / a.rows_per_group;
      const int next = (g0 + 1) * a.rows_per_group - m0;
      int64_t row0 = 0, row1 = 0;
      if constexpr (GROUP16) {
        row0 = group_row(a, g0);
        row1 = group_row(a, min(g0 + 1, (M - 1) / a.rows_per_group));
      }
#pragma unroll
      for (int j = 0; j < NT; j += 2) {
        constexpr int NTv = NT;
        const bool pair = j + 1 < NTv;
        const int nl = 16 * NT * q + 16 * j + (pair ? l5 : r16);
        const int n = min(n0 + nl, N - 1);
        auto row_of = [&](int v) { return mt + (pair ? 8 * h2 + v : 4 * kg + v); };   // v < 8 (pair) or < 4
        float bv[8];
        if constexpr (GROUP16) {
          const float b0 = bias_at<EPI>(a, row0, n), b1 = bias_at<EPI>(a, row1, n);
#pragma unroll
          for (int v = 0; v < 8; ++v) bv[v] = row_of(v) < next ? b0 : b1;
        } else {
#pragma unroll
          for (int v = 0; v < 8; ++v)
            if (pair || v < 4) bv[v] = bias_at<EPI>(a, group_row(a, min(m0 + row_of(v), M - 1) / a.rows_per_group), n);
        }
        const bool ok = n0 + nl < N;
        auto put = [&](float s, float b, int ml) __attribute__((always_inline)) {
          const unsigned e = unsigned(ml) * unsigned(N) + unsigned(n0 + nl);
          if constexpr (EPI == EPI_LOGITS) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s + b), ro, ok ? e * 4u : 0xFFFFFFF0u, 0, NTS ? kAuxNT : 0);
          } else {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(s), ro, ok ? e * 4u : 0xFFFFFFF0u, 0, 0);
            __builtin_amdgcn_raw_buffer_store_b16(f32_to_bf16(tanhf(s + b)), ra, ok ? e * 2u : 0xFFFFFFF0u, 0, 0);
          }
        };
        if (pair) {
#pragma unroll
          for (int v = 0; v < 4; ++v) {
            const auto p = __builtin_amdgcn_permlane16_swap(__float_as_uint(acc[i][j][v]),
                                                            __float_as_uint(acc[i][j + 1 < NT ? j + 1 : j][v]), false, false);
            put(__uint_as_float(p[0]), bv[v], row_of(v));
            put(__uint_as_float(p[1]), bv[4 + v], row_of(4 + v));
          }
        } else {
#pragma unroll
          for (int v = 0; v < 4; ++v) put(acc[i][j][v], bv[v], row_of(v));
        }
        __builtin_amdgcn_sched_barrier(0);   // keep the tiles' epilogues apart (registers)
      }
    }
  }
};

// The node-row tiles of one weight tile run on one XCD and share it in its L2.
template <int RT, int EPI, int WAUX>
__global__ __launch_bounds__(512, 2) void proj_bf16_tile(TileArgs a) {
  __shared__ __attribute__((aligned(16))) uint16_t smem[(32 * RT + 256) * 64 * tile_stages(RT)];
  const int ntm = (a.M + 32 * RT - 1) / (32 * RT);
  if (int(blockIdx.x) < a.full) {
    const int t = xcd_order(blockIdx.x, a.full);
    Tile<RT, 4, EPI, WAUX>::run(a, (t % ntm) * 32 * RT, (t / ntm) * 256, smem);
    return;
  }
  const int t = xcd_order(int(blockIdx.x) - a.full, int(gridDim.x) - a.full);
  const int m0 = (t % ntm) * 32 * RT, n0 = a.nf * 256 + (t / ntm) * 64 * a.tail;
  if (a.tail == 1) Tile<RT, 1, EPI, WAUX>::run(a, m0, n0, smem);
  else if (a.tail == 2) Tile<RT, 2, EPI, WAUX>::run(a, m0, n0, smem);
  else if (a.tail == 3) Tile<RT, 3, EPI, WAUX>::run(a, m0, n0, smem);
}

// Whole rounds of NT = 4 tiles (one block per compute unit is resident), then
// the remaining columns in the tiles of NT = 1..4 whose rounds cost least.  A
// tile of NT weight tiles per wave takes about 0.4, 0.6, 0.8, 1 of the widest
// one's time (measured at RT = 4..8: the node rows' share of a step and the
// barriers do not shrink with NT).
void plan(TileArgs& a, int RT) {
  const int ntm = (a.M + 32 * RT - 1) / (32 * RT), ntn = (a.N + 255) / 256;
  const int cus = device_cus();
  a.nf = int(int64_t(ntm) * ntn / cus * cus / ntm);
  const int rest = a.N - std::min<int64_t>(int64_t(a.nf) * 256, a.N);
  int best = 4;
  int64_t cost = INT64_MAX;
  for (int t = 4; t >= 1; --t) {
    const int64_t tiles = int64_t(ntm) * ((rest + 64 * t - 1) / (64 * t));
    const int64_t c = (tiles + cus - 1) / cus * (1 + t);
    if (c < cost) {
      cost = c;
      best = t;
    }
  }
  a.tail = best;
  if (best == 4) a.nf = ntn;
  a.full = a.nf * ntm;
}

// Less than one round of 256-column tiles (heads, short matrices): one size for
// all tiles, the one whose rounds cost least.  A round of RT x NT tiles takes
// about 30 + 8 RT + 20 NT + RT NT units of 6.3 ns a step, 8 more where the ring
// holds two stages only, and 460 once (fitted to 15 shapes x 28 sizes, 128 to 2048
// rows, K 2560 to 5120, 9% off; the size it picks is the fastest measured one for
// all 13 short shapes).  The largest tile of the rows with the plan above / the
// pick, weights not in the caches: 1024 x 5120 x 5120 95 / 74 us, 512 rows 80 / 52,
// 256 rows 82 / 44, 512 x 4096 x 4096 56 / 38, 128 x 5120 x 5120 55 / 42, 1024 x
// 2560 x 2560 39 / 30.
int short_plan(TileArgs& a) {
  const int64_t nk = a.K >> 6, cus = device_cus();
  int rt = 8, nt = 4;
  int64_t cost = INT64_MAX;
  for (int r = 3; r <= 8; ++r)
    for (int t = 1; t <= 4; ++t) {
      const int64_t tiles = ((int64_t(a.M) + 32 * r - 1) / (32 * r)) * ((int64_t(a.N) + 64 * t - 1) / (64 * t));
      const int64_t c = (tiles + cus - 1) / cus * (nk * (30 + 8 * r + 20 * t + r * t + (tile_stages(r) == 2 ? 8 : 0)) + 460);
      if (c < cost) {
        cost = c;
        rt = r;
        nt = t;
      }
    }
  a.tail = nt;
  a.nf = nt == 4 ? (a.N + 255) / 256 : 0;
  a.full = a.nf * ((a.M + 32 * rt - 1) / (32 * rt));
  return rt;
}

template <int RT>
hipError_t launch_rt(TileArgs& a, int epi, bool nt_weights, bool planned, hipStream_t s) {
  if (!planned) plan(a, RT);
  const int ntm = (a.M + 32 * RT - 1) / (32 * RT);
  const int rest = std::max(0, a.N - a.nf * 256);
  const dim3 grid(unsigned(a.full + (a.tail < 4 ? ntm * ((rest + 64 * a.tail - 1) / (64 * a.tail)) : 0)));
  if (epi == EPI_HEAD) hipLaunchKernelGGL((proj_bf16_tile<RT, EPI_HEAD, 0>), grid, dim3(512), 0, s, a);
  else if (nt_weights) hipLaunchKernelGGL((proj_bf16_tile<RT, EPI_LOGITS, kAuxNT>), grid, dim3(512), 0, s, a);
  else hipLaunchKernelGGL((proj_bf16_tile<RT, EPI_LOGITS, 0>), grid, dim3(512), 0, s, a);
  return hipGetLastError();
}

}  // namespace

// A tile's operand bytes and the bytes of its rows of the output fit 32-bit
// buffer ranges, the latter below the offset 0xFFFFFFF0 that drops a store (256
// rows: up to 4194303 columns).
bool proj_tile_shape(int64_t M, int64_t N, int64_t K) {
  return K % 64 == 0 && K <= (int64_t(1) << 20) && std::min<int64_t>(M, 256) * N * 4 <= int64_t(0xFFFFFFF0u);
}

hipError_t launch_project_tile(const ProjArgs& p, hipStream_t s) {
  TileArgs a{};
  a.x = static_cast<const uint16_t*>(p.x);
  a.w = static_cast<const uint16_t*>(p.w);
  a.M = int(p.M);
  a.N = int(p.N);
  a.K = int(p.K);
  a.rows_per_group = int(p.rows_per_group);
  a.bias_stride = p.bias_stride;
  a.bias_f32 = p.bias_f32;
  a.bias_act = static_cast<const uint16_t*>(p.bias_act);
  a.group_index = p.group_index;
  a.out = p.out;
  a.act_out = static_cast<uint16_t*>(p.act_out);
  // Beyond the 256 MB Infinity Cache: weights read and logits written around
  // it (128 x 151936 x 4096: 242 us with ordinary weight loads, 225 without;
  // 300 x 50257 x 2560, whose 257 MB fit: 118 with, 138 without).
  constexpr int64_t kCache = int64_t(256) << 20;
  const bool nt_weights = p.N * p.K * 2 > kCache;
  a.nt_out = p.M * p.N * 4 > kCache;
  // the fewest node tiles of at most 256 rows, and the least tile that covers them
  const int ntm = (a.M + 255) / 256;
  int rt = std::max(2, ((a.M + ntm - 1) / ntm + 31) / 32);
  const bool planned = rt > 2 && int64_t(ntm) * ((a.N + 255) / 256) < device_cus();
  if (planned) rt = short_plan(a);
  switch (rt) {
    case 2: return launch_rt<2>(a, p.epilogue, nt_weights, planned, s);
    case 3: return launch_rt<3>(a, p.epilogue, nt_weights, planned, s);
    case 4: return launch_rt<4>(a, p.epilogue, nt_weights, planned, s);
    case 5: return launch_rt<5>(a, p.epilogue, nt_weights, planned, s);
    case 6: return launch_rt<6>(a, p.epilogue, nt_weights, planned, s);
    case 7: return launch_rt<7>(a, p.epilogue, nt_weights, planned, s);
    default: return launch_rt<8>(a, p.epilogue, nt_weights, planned, s);
  }
}

}  // namespace dartree
