// Output projection fused with the streaming log-sum-exp, for gfx950 (CDNA4).
//
//   fopd_k7_lm_head_lse   z[t, v] = sum_k H[t, k] * W[v, k] on the matrix cores, reduced on the fly to
//                         a running (reference, sum) pair per token; the [T, V] logits never exist
//                         in memory.
//   fopd_k7_finish        the sampled token's logit as one dot product per token, the merge of the
//                         per-strip pairs: lse_t, lp_t = z_{t,y_t} - lse_t.
//
// This is the step in front of the loss pass (pi_theta^t(y | x) of Eq. "kl-diagnostics" is the softmax of
// the projected hidden state), and the only dense contraction near it.
//
// Tiling.  A workgroup of eight wavefronts (2 along the vocabulary x 4 along the tokens, two per SIMD)
// owns 256 tokens and walks a strip of the vocabulary in tiles of 256 rows; each wavefront holds a
// 128 x 64 block of the tile as 8 x 4 accumulators of v_mfma_f32_16x16x32_bf16.  The vocabulary is the
// M side of the instruction and the tokens the N side, because a lane of the 16 x 16 result holds four
// rows of ONE column: the reduction over the vocabulary then runs inside a lane and needs two
// cross-lane steps at the very end (the four groups of 16 lanes).  Both operands are k-contiguous in memory (hidden [T, d],
// weight [V, d]), so a lane's 8-element fragment is one 16-byte LDS read.
//
// The loop over the hidden elements (matrix_step below) is shared with the contraction kernels.  Bound by power: the matrix
// cores are 0.75 busy at the 1.83 GHz that the part then holds (logits of 8192 rows; with the 32 x 32 x 16 instruction 0.74 at
// 1.68 GHz).  The 16 x 16 x 32 instruction has the other's rate but goes over its accumulators half as often per product;
// log-probs of 16,384 rows x
// 151,936, d = 4096: 15.4 - 16.0 -> 14.7 - 15.1 ms, of 2048 rows 1.92 - 1.98 -> 1.86 ms.  With the vocabulary tiles of a strip as
// one stream (matrix_tiles), whose loads have offsets that stay from step to step, 14.15 - 14.4 and 1.73 ms, and without a wave
// priority 13.9 - 14.4 and 1.70 - 1.75 ms.

#ifndef FOPD_LM_HEAD_HIP_
#define FOPD_LM_HEAD_HIP_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>
#include <type_traits>

#include "fopd_kernels.hip"

namespace fopd {

constexpr int kLmTile = 256;                              // vocabulary rows and token rows of a workgroup tile
constexpr int kLmK = 64;                                  // hidden elements of a step
constexpr int kLmStrips = 32;                             // vocabulary strips = partial pairs per token: room for 32 of all
constexpr int kLmPairsExtra = 57344;                      // tokens and this many pairs more (256 strips of one token tile)
constexpr int kLmThreads = 512;                           // 8 wavefronts: 2 (vocabulary) x 4 (tokens)
constexpr int kHalfBytes = 128 * kLmK * 2;                // half an operand tile of a step: 16 KB
constexpr int kStepBytes = 4 * kHalfBytes;                // both operand tiles of a step
constexpr int kLoopLdsBytes = 2 * kStepBytes;             // two steps: 128 KB of the compute unit's 160
constexpr int kNarrowBytes = 3 * kHalfBytes;              // a step with half a B tile, of which the LDS holds three
constexpr int kLmLdsBytes = 3 * kNarrowBytes;             // 144 KB; the other forms of the loop take 128 of it, and the exchange
                                                          // between wavefronts at the end the first few again
constexpr float kLmNone = -__builtin_inff();              // "no value yet": the reference of an empty pair

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

// A wavefront's block of the result tile: [A half][SIDE-row block of its 64][B half][SIDE-row block of its 32].  SIDE is that of
// the matrix instruction's result, 16 (v_mfma_f32_16x16x32_bf16) or 32 (v_mfma_f32_32x32x16_bf16).
template <int A_HALVES, int B_HALVES, int SIDE = 16>
using BlockAcc = typename std::conditional<SIDE == 16, f32x4, f32x16>::type[A_HALVES][64 / SIDE][B_HALVES][32 / SIDE];

namespace {

// (m, s) <- merge of two running pairs, s in units of exp(. - m).  An empty pair is (-inf, 0); the
// equality tests keep (-inf) - (-inf) out of the arithmetic.
__device__ __forceinline__ void lm_merge(float& m, float& s, float m2, float s2) {
  const float mx = fmaxf(m, m2);
  const float a = (m == mx) ? 1.f : fast_exp2((m - mx) * kLog2e);
  const float b = (m2 == mx) ? 1.f : fast_exp2((m2 - mx) * kLog2e);
  s = s * a + s2 * b;
  m = mx;
}

// Which tile a workgroup owns.  A launch is a list of groups of 32 workgroups; workgroups go to the eight XCDs in turn
// (id mod 8), so group g runs on XCD g mod 8 and its 32 tiles share that XCD's L2.  A group is up to 4 tiles along n
// (the side with few tiles when the batch is small) x the 8 (16, 32) along m that fill it: with one or two tiles along n
// the group takes 16 or 32 tiles along m instead of leaving workgroups without work.  That matters because an idle
// workgroup is not free: it asks for the same 128 or 144 KB of LDS, so it queues for a compute unit like a working one.
// Logits of 512 rows x 151,936 entries, d = 4096 (1188 tiles): 4 x 8 groups always, 2560 workgroups, 836 us; 2 x 16, 1280,
// 558 us.  Idle workgroups remain where the last group along n has 1 to 3 tiles and another one stands beside it, or the only
// one has 3, and where the groups are rounded up to eight: 594 tiles take 768 workgroups for 256 rows, 1782 take 2560 for 768
// rows (0.52 us a tile, 0.46 with the 2376 of 1024 rows), 2970 take 4864 for 1280 rows (0.55).  (Launches whose workgroups walk
// the tiles, TileWalk in fopd_gemm.hip, have none.  The figures are from the 32 x 32 x 16 instruction.)
// Consecutive groups, and with them the XCDs, go along n first (N_FIRST) or along m first.  Along m first there are few
// groups in a line, and the last of it may be a small one: where the line's length has a factor in common with 8 the same
// XCDs would get it in every line, so the order in a line moves on by one each time the XCDs have come round to its start
// (weight gradient of 4096 rows x 151,936, lines of 8 + 2 tiles, d = 2560: 3971 -> 2711 us).
struct TilePlace {
  int m, n;
};

__host__ __device__ __forceinline__ int tile_group_n(int tiles_n) { return tiles_n >= 3 ? 4 : (tiles_n == 2 ? 2 : 1); }

// Groups of a launch.  For fewer tiles along n never more groups than for more of them, so a launch sized for all rows
// covers any smaller count that the device finds.
__host__ __device__ __forceinline__ int64_t tile_groups(int tiles_m, int tiles_n) {
  const int gn = tile_group_n(tiles_n), gm = 32 / gn;
  return static_cast<int64_t>((tiles_n + gn - 1) / gn) * ((tiles_m + gm - 1) / gm);
}

// Rounds of a launch of `runs` times the groups, along n first: the most that one XCD, 32 compute units of one workgroup
// each, has to go through.  Groups that do not fill it run side by side where whole ones fit (16 tiles: two, 24 tiles: one;
// measured on 768 rows, whose groups hold 24: a round takes as long for 24 tiles as for 32, whatever follows).
__host__ inline int64_t tile_rounds(int tiles_m, int tiles_n, int runs) {
  const int gn = tile_group_n(tiles_n), gm = 32 / gn;
  const int groups_n = (tiles_n + gn - 1) / gn, groups_m = (tiles_m + gm - 1) / gm;
  int64_t one[8] = {}, load[8] = {};                       // parts of 32 of a round, by XCD
  for (int m = 0; m < groups_m; ++m)
    for (int n = 0; n < groups_n; ++n) {
      const int m_left = tiles_m - m * gm, n_left = tiles_n - n * gn;
      const int tiles = (m_left < gm ? m_left : gm) * (n_left < gn ? n_left : gn);
      one[(static_cast<int64_t>(m) * groups_n + n) % 8] += 32 / (32 / tiles);
    }
  const int64_t groups = static_cast<int64_t>(groups_m) * groups_n;
  int64_t most = 0;
  for (int r = 0; r < runs; ++r)
    for (int x = 0; x < 8; ++x) {
      int64_t& l = load[(x + r * groups) % 8];
      l += one[x];
      if (l > most) most = l;
    }
  return (most + 31) / 32;
}

// Strips of the vocabulary for fopd_k7_lm_head_lse: the launch takes its rounds (tile_rounds) one after the other, a
// round as long as its longest strip has tiles (plus a little for the item itself: first loads, last merge), and the
// number of strips with the least total is taken. Few token tiles give many short strips, so that one short rollout fills
// the chip too: 200 rows x 151,936 entries, d = 4096, 32 strips 1408 us, 64 848, 128 448, 224 297; 512 rows 32 strips 1613, 64
// 865, 128 525.  What counts is the fullest XCD, not the number of items: 1280 rows (groups of 32 and of 8 items in turn) 32
// strips 1389 us, 48 strips, 240 items, 1835; 768 rows (24 items a group) 64 strips 882 us, 80 strips 1181.  Whole groups
// only (tile_place): strips that leave part of a group empty share the weight's L2 copies worse.
__host__ inline int lm_strips(int n_token_tiles, int n_vocab_tiles) {
  const int group_strips = 32 / tile_group_n(n_token_tiles);
  const int strips_max = kLmStrips + kLmPairsExtra / (n_token_tiles * kLmTile);
  int n_strips = group_strips;
  double best = 0.0;
  for (int cand = group_strips; cand <= strips_max && (cand == group_strips || cand <= n_vocab_tiles);
       cand += group_strips) {
    const double rounds = static_cast<double>(tile_rounds(cand, n_token_tiles, 1));
    const double cost = rounds * (static_cast<double>((n_vocab_tiles + cand - 1) / cand) + 0.15);
    if (cand == group_strips || cost < best) {
      best = cost;
      n_strips = cand;
    }
  }
  return n_strips;
}

// Token tiles of fopd_k7_lm_head_lse: `whole` of them in `strips` strips each, and a last one of at most 128 tokens in
// `tail_strips` (0: none).  whole = tail_strips = 0: all tokens in one tile of at most 384 (wide).
struct LmSplit {
  int whole, strips, tail_strips;
  __host__ __device__ bool wide() const { return whole == 0 && tail_strips == 0; }
};

// A last tile of up to 128 tokens goes through a step in kNarrowCost of the time of a whole one, so few whole tiles and that one
// share the chip best with strips of their own: all of them in one round, a group for each XCD, as long as the longer of the
// two strips.  With more tiles the tail is one tile of many and has the strips of the others.  151,936 x 4096, us, all tiles whole /
// so: 64 rows 318 / 260, 600 rows 847 / 680, 1100 rows 1480 / 1075, 1600 rows (a tail among seven) 1770 / 1620.
constexpr double kNarrowCost = 0.6;
__host__ inline LmSplit lm_split(int64_t T, int64_t V) {
  const int n_vocab_tiles = static_cast<int>((V + kLmTile - 1) / kLmTile);
  const int tiles = static_cast<int>((T + kLmTile - 1) / kLmTile);
  const int tail = static_cast<int>(T - static_cast<int64_t>(tiles - 1) * kLmTile);
  LmSplit best = {tiles, lm_strips(tiles, n_vocab_tiles), 0};
  if (tail > kLmTile / 2) return best;
  auto steps = [&](int strips) { return (n_vocab_tiles + strips - 1) / strips; };
  if (tiles == 1) return {0, 0, std::min(256, (n_vocab_tiles + 31) / 32 * 32)};
  const int whole = tiles - 1, group_strips = 32 / tile_group_n(whole), groups_n = (whole + 3) / 4;
  double least = static_cast<double>(tile_rounds(best.strips, tiles, 1)) * steps(best.strips);
  if (tiles == 2) {
    // 257 to 384 tokens: as two tiles with strips of their own the projection matrix is read twice, at different times (2.5 GB at
    // 5.4 TB/s).  In one tile of 128 x 384 a step has three products of four, for half the vocabulary rows.  As many strips as
    // the pairs have room for, at most one a compute unit, in whole rounds.  151,936 x 4096, two tiles / one, us: 257 - 300 rows
    // 462 / 412 (five rounds), 310 - 372 rows 470 - 485 / 450 (six), 384 rows 493 / 506 (seven, so two tiles).  How far one
    // tile goes follows from the rounds: 376 rows at 50,000 entries, all 384 at 32,000 and 70,000.
    const int vocab_tiles = static_cast<int>((V + kLmTile / 2 - 1) / (kLmTile / 2));
    const int64_t most = std::min<int64_t>(256, (static_cast<int64_t>(kLmStrips) * tiles * kLmTile + kLmPairsExtra) / T);
    const int rounds = static_cast<int>((vocab_tiles + most - 1) / most);
    if (3.0 * rounds < 4.0 * least) return {0, (vocab_tiles + rounds - 1) / rounds, 0};
  }
  for (int tail_groups = 1; tail_groups < 8; ++tail_groups) {
    const int strips = (8 - tail_groups) / groups_n * group_strips, tail_strips = 32 * tail_groups;
    if (strips <= 0 || strips > n_vocab_tiles || tail_strips > n_vocab_tiles) continue;
    const double cost = std::max<double>(steps(strips), kNarrowCost * steps(tail_strips));
    if (cost < least) {
      least = cost;
      best = {whole, strips, tail_strips};
    }
  }
  return best;
}

template <bool N_FIRST>
__host__ __device__ __forceinline__ TilePlace tile_place(unsigned group, unsigned slot, int tiles_m, int tiles_n) {
  const int gn = tile_group_n(tiles_n), gm = 32 / gn;
  const int groups_n = (tiles_n + gn - 1) / gn, groups_m = (tiles_m + gm - 1) / gm;
  const int g = static_cast<int>(group), sl = static_cast<int>(slot);
  const int common = min(groups_m & -groups_m, 8);         // largest common divisor of 8 and the length of a line
  const int at_n = N_FIRST ? g % groups_n : g / groups_m;
  const int at_m = N_FIRST ? g / groups_n : (g + g / (8 / common * groups_m)) % groups_m;
  return TilePlace{at_m * gm + sl / gn, at_n * gn + sl % gn};
}

// ---- the loop of the matrix kernels -------------------------------------------------------------------------------
// A workgroup of eight wavefronts multiplies a 256-row tile A by a 256-row tile B, 64 elements of the contraction index a
// step.  Each tile is two halves of 128 rows (A0, A1, B0, B1: 16 KB each); the LDS holds two steps.  Wavefront (wm, wn),
// wm = wave / 4, wn = wave % 4, owns rows 64 wm .. + 63 of both A halves and 32 wn .. + 31 of both B halves: four
// products of 64 x 32, acc[A half][.][B half][.], one a phase.
//
// A phase is two slots between barriers: LDS reads and requests of one half tile, then the sixteen matrix instructions of
// a product.  The wavefronts of wm = 1 pass one barrier more at the start, so they are always one slot behind: on each
// SIMD, which holds one wavefront of either kind, one multiplies while the other reads.  A half tile goes from memory
// straight to the LDS (16 bytes a lane) as soon as both kinds have read what it replaces, five to seven phases before it
// is read, and nothing ever waits for all requests:
//
//   phase   reads      multiplies   requests              waits for (besides its own LDS reads)
//     1     B0, A0     A0 x B0      A1 of the next step
//     2     B1         A0 x B1      B0 of the next but one   A1 of this step       (5 half tiles stay in flight)
//     3     A1         A1 x B1      A0 of the next but one
//     4                A1 x B0      B1 of the next but one   B0, A0, B1 of the next step   (4 stay in flight)
//
// What replaces what: a half tile is requested in the slot after the one in which the later kind's reads of its
// predecessor have returned (each reading slot ends with a wait for the LDS, then the barrier).  A wavefront's two loads a
// phase are followed by its wait count one barrier before the earlier kind reads.
//
// Measured on the log-probs of 16,384 rows x 151,936 entries, d = 4096, against the loop before (tiles through vector
// registers, a quarter of 64 elements per 16, one barrier per 64): 16.40 - 16.73 -> 15.91 - 15.95 ms on one box, 0 - 4 % on
// others.  Contractions of two steps a tile (d = 128) are up to 25 % slower with it.  Variants of an experiment: with the
// operands loaded once and not again 14.07 of 16.70 ms (another box 12.8 of 15.9), with every step reading the same 64
// elements, lines just used, 16.02 (14.3).  Slower: the loads of a slot before its LDS reads (+ 14 %), inside the run of
// matrix instructions (+ 10 - 16 %): requests wait at the L1, and hold up what follows them; non-temporal loads (+ 14 %); B0
// read a phase earlier to even out the reads (+ 1 %).  A higher wave priority for the multiplying slots held up the other kind's
// LDS reads once the instructions came twice as often: with / without, dL/dhidden of 256 rows x 4096 over 151,936 entries 2895 /
// 2850 us, of 512 rows of 1024 over 32,000 155.4 / 153.5; loss and gradients of 4096 rows 12.60 / 12.49 ms, of 16,384 rows 49.5 /
// 49.0; log-probs of 16,384 rows 14.63 / 14.42 ms.

struct MatrixPlace {
  int wm, wn;
  uint32_t lds;        // LDS address of the wavefront's share of half tile A0 of step buffer 0
};

__device__ __forceinline__ MatrixPlace matrix_place(const unsigned char* smem) {
  typedef __attribute__((address_space(3))) const unsigned char lds_byte;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  return MatrixPlace{wave >> 2, wave & 3, static_cast<uint32_t>(reinterpret_cast<uintptr_t>((lds_byte*)smem)) + wave * 2048u};
}

// 16 bytes a lane from (uniform base) + (32-bit offset of the lane) to LDS bytes lds + 16 lane.  Has no result register;
// whoever reads the LDS bytes waits for the wavefront's count of loads first.  M0, which holds the LDS address of such a
// load, is named as written, so that the compiler does not take an M0 of its own for still there behind it (hipcc warns of
// any reserved register in that list; it does write M0 again).  M0 as an input of the statement, written by the
// compiler, is 1 - 3 % slower: log-probs of 300 / 2048 / 16,384 rows x 151,936, d = 4096, 528 / 2006 / 16,100 -> 533 /
// 2028 / 16,640 us.
__device__ __forceinline__ void load_to_lds(const char* base, uint32_t offset, uint32_t lds) {
#pragma clang diagnostic push
#pragma clang diagnostic ignored "-Winline-asm"
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(offset), "s"(base)
               : "memory", "m0");
#pragma clang diagnostic pop
}

// Barrier of the workgroup that no instruction passes in either direction (nothing else is waited for).
__device__ __forceinline__ void slot_end() {
  __builtin_amdgcn_sched_barrier(0);
  __builtin_amdgcn_s_barrier();
  __builtin_amdgcn_sched_barrier(0);
}

enum { kHalfA0 = 0, kHalfA1 = 1, kHalfB0 = 2, kHalfB1 = 3, kHalfB2 = 1 };          // (places in a step's buffer)

// B_FIRST: the B fragment is the matrix instruction's first operand (a lane then holds four B rows of one A row), else the A
// fragment is.
template <bool B_FIRST, int SIDE, typename Acc, typename FragsA, typename FragsB>
__device__ __forceinline__ void multiply_phase(Acc& acc, int a, int b, const FragsA& fa, const FragsB& fb) {
#pragma unroll
  for (int ks = 0; ks < SIDE / 8; ++ks)
#pragma unroll
    for (int i = 0; i < 64 / SIDE; ++i)
#pragma unroll
      for (int j = 0; j < 32 / SIDE; ++j) {
        const bf16x8 first = B_FIRST ? fb[j][ks] : fa[i][ks], second = B_FIRST ? fa[i][ks] : fb[j][ks];
        if constexpr (SIDE == 16)
          acc[a][i][b][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(first, second, acc[a][i][b][j], 0, 0, 0);
        else
          acc[a][i][b][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(first, second, acc[a][i][b][j], 0, 0, 0);
      }
}

// One step.  read_a(half, i, ks) / read_b(half, j, ks): the fragment of SIDE-row block i / j, elements (512 / SIDE) ks on, from
// this step's buffer.  request(half): the wavefront's two loads of that half tile of a later step (any readable one past the last:
// never read).  STORED: at least 63 stores have been issued since the requests that this
// step waits for, which are done when 63 later ones are all that is left (loads and stores count and end in order).
template <bool B_FIRST, bool STORED, int SIDE, typename ReadA, typename ReadB, typename Request>
__device__ __forceinline__ void matrix_step(BlockAcc<2, 2, SIDE>& acc, ReadA read_a, ReadB read_b, Request request) {
  constexpr int I = 64 / SIDE, J = 32 / SIDE, KS = SIDE / 8;
  bf16x8 fa[I][KS], fb0[J][KS], fb1[J][KS];
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fb0[j][ks] = read_b(0, j, ks);
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[i][ks] = read_a(0, i, ks);
  request(kHalfA1);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  slot_end();
  multiply_phase<B_FIRST, SIDE>(acc, 0, 0, fa, fb0);
  slot_end();
#pragma unroll
  for (int j = 0; j < J; ++j)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fb1[j][ks] = read_b(1, j, ks);
  request(kHalfB0);
  if constexpr (STORED) asm volatile("s_waitcnt vmcnt(63) lgkmcnt(0)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)" ::: "memory");
  slot_end();
  multiply_phase<B_FIRST, SIDE>(acc, 0, 1, fa, fb1);
  slot_end();
#pragma unroll
  for (int i = 0; i < I; ++i)
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) fa[i][ks] = read_a(1, i, ks);
  request(kHalfA0);
  asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
  slot_end();
  multiply_phase<B_FIRST, SIDE>(acc, 1, 1, fa, fb1);
  slot_end();
  request(kHalfB1);
  if constexpr (STORED) asm volatile("s_waitcnt vmcnt(63)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  slot_end();
  multiply_phase<B_FIRST, SIDE>(acc, 1, 0, fa, fb0);
  slot_end();
}

// Before the first step: the seven half tiles that precede its own requests, in the order of the steps, and the extra
// barrier of wm = 1.
template <typename Request>
__device__ __forceinline__ void matrix_begin(const MatrixPlace& place, Request request) {
  request(kHalfB0, 0);
  request(kHalfA0, 0);
  request(kHalfB1, 0);
  request(kHalfA1, 0);
  request(kHalfB0, 1);
  request(kHalfA0, 1);
  request(kHalfB1, 1);
  asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
  slot_end();
  if (place.wm == 1) slot_end();
}

// The same for a tile with at most 128 rows of B: without B1 a step is two phases, and the LDS holds three steps of 48 KB.
//
//   phase   reads      multiplies   requests                        waits for (besides its own LDS reads)
//     1     B0, A0     A0 x B0      A1 of the next step but one     A1 of this step          (6 half tiles stay in flight)
//     2     A1         A1 x B0      B0, A0 of the next but two      B0, A0 of the next step  (6 stay in flight)
//
template <bool B_FIRST, typename ReadA, typename ReadB, typename Request>
__device__ __forceinline__ void matrix_step_narrow(BlockAcc<2, 1>& acc, ReadA read_a, ReadB read_b, Request request) {
  bf16x8 fa[4][2], fb[2][2];
#pragma unroll
  for (int j = 0; j < 2; ++j)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fb[j][ks] = read_b(0, j, ks);
#pragma unroll
  for (int a = 0; a < 2; ++a) {
#pragma unroll
    for (int i = 0; i < 4; ++i)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fa[i][ks] = read_a(a, i, ks);
    if (a == 0) {
      request(kHalfA1);
    } else {
      request(kHalfB0);
      request(kHalfA0);
    }
    asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
    slot_end();
    multiply_phase<B_FIRST, 16>(acc, a, 0, fa, fb);
    slot_end();
  }
}

template <typename Request>
__device__ __forceinline__ void matrix_begin_narrow(const MatrixPlace& place, Request request) {
#pragma unroll
  for (int buf = 0; buf < 3; ++buf) {
    request(kHalfB0, buf);
    request(kHalfA0, buf);
    if (buf < 2) request(kHalfA1, buf);
  }
  asm volatile("s_waitcnt vmcnt(12)" ::: "memory");
  slot_end();
  if (place.wm == 1) slot_end();
}

// The same for a tile of 128 rows of A and up to 384 of B (B2 in the place of A1), three phases a step:
//
//   phase   reads      multiplies   requests                     waits for (besides its own LDS reads)
//     1     A0, B0     A0 x B0      B2 of the next step          B1 of this step           (5 half tiles stay in flight)
//     2     B1         A0 x B1      A0, B0 of the next but one   B2 of this step           (6 stay in flight)
//     3     B2         A0 x B2      B1 of the next but one       A0, B0 of the next step   (5 stay in flight)
//
template <bool B_FIRST, typename ReadA, typename ReadB, typename Request>
__device__ __forceinline__ void matrix_step_wide(BlockAcc<1, 3>& acc, ReadA read_a, ReadB read_b, Request request) {
  bf16x8 fa[4][2], fb[2][2];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) fa[i][ks] = read_a(0, i, ks);
#pragma unroll
  for (int b = 0; b < 3; ++b) {
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int ks = 0; ks < 2; ++ks) fb[j][ks] = read_b(b < 2 ? b : -1, j, ks);
    if (b == 0) {
      request(kHalfB2);
      asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)" ::: "memory");
    } else if (b == 1) {
      request(kHalfA0);
      request(kHalfB0);
      asm volatile("s_waitcnt vmcnt(12) lgkmcnt(0)" ::: "memory");
    } else {
      request(kHalfB1);
      asm volatile("s_waitcnt vmcnt(10) lgkmcnt(0)" ::: "memory");
    }
    slot_end();
    multiply_phase<B_FIRST, 16>(acc, 0, b, fa, fb);
    slot_end();
  }
}

template <typename Request>
__device__ __forceinline__ void matrix_begin_wide(const MatrixPlace& place, Request request) {
#pragma unroll
  for (int buf = 0; buf < 2; ++buf) {
    request(kHalfA0, buf);
    request(kHalfB0, buf);
    request(kHalfB1, buf);
    if (buf == 0) request(kHalfB2, buf);
  }
  asm volatile("s_waitcnt vmcnt(10)" ::: "memory");
  slot_end();
  if (place.wm == 1) slot_end();
}

// After the last step: every wavefront has passed the same number of barriers, and no request is left in flight (they
// write to the LDS).
__device__ __forceinline__ void matrix_end(const MatrixPlace& place) {
  if (place.wm == 0) slot_end();
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();
}

// Operands with the contraction index contiguous.  A row of a half tile is 128 bytes in the LDS; its eight 16-byte chunks
// are permuted by bits 1 .. 3 of the row, so that the sixteen rows that a quarter of a wavefront reads at one chunk lie in
// all 64 banks.  Wavefront w fills rows 16 w .. + 15 in two loads of eight rows: lane i writes chunk i % 8 of row i / 8
// and so fetches chunk (i % 8) ^ (row / 2 % 8).
struct RowMajorHalf {
  int row, chunk[2];           // row of the wavefront's first load (the second: + 8), bytes of the chunk in the row
  __device__ __forceinline__ explicit RowMajorHalf(const MatrixPlace& p) {
    const int lane = threadIdx.x & 63;
    row = 16 * (p.wm * 4 + p.wn) + (lane >> 3);
    chunk[0] = ((lane & 7) ^ (lane >> 4)) * 16;
    chunk[1] = chunk[0] ^ 64;
  }
};

template <int SIDE = 16>
struct RowMajorFragments {
  static constexpr int KS = SIDE / 8;
  uint32_t a_off, b_off, xk[KS];
  __device__ __forceinline__ explicit RowMajorFragments(const MatrixPlace& p) {
    const int lane = threadIdx.x & 63;
    a_off = (p.wm * 64 + (lane & (SIDE - 1))) * 128;
    b_off = 2 * kHalfBytes + (p.wn * 32 + (lane & (SIDE - 1))) * 128;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) xk[ks] = (((64 / SIDE) * ks + lane / SIDE) ^ ((lane >> 1) & 7)) << 4;
  }
  __device__ __forceinline__ bf16x8 a(const unsigned char* step, int half, int i, int ks) const {
    return *reinterpret_cast<const bf16x8*>(step + half * kHalfBytes + a_off + i * (SIDE * 128) + xk[ks]);
  }
  __device__ __forceinline__ bf16x8 b(const unsigned char* step, int half, int j, int ks) const {
    return *reinterpret_cast<const bf16x8*>(step + half * kHalfBytes + b_off + j * (SIDE * 128) + xk[ks]);
  }
};

// A tile of the result and the steps of the contraction index that go into it: all of them, or those of one run (split).
struct GemmTile {
  int m0, n0, first, steps, split;
};

// Where the loads of a tile come from.  Operands with the contraction index contiguous: rows past the last are clamped, so the
// loop has no branch.
struct RowMajorSource {
  const char* base;
  int64_t ld;
  int rows;
  const char* src;
  uint32_t off[2][2];
  __device__ __forceinline__ void locate(const RowMajorHalf& at, int r0, int64_t k0) {
    src = base + (static_cast<int64_t>(r0) * ld + k0) * 2;
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int e = 0; e < 2; ++e)
        off[h][e] = static_cast<uint32_t>(min(h * 128 + at.row + 8 * e, rows - 1 - r0)) * (static_cast<uint32_t>(ld) * 2u) + at.chunk[e];
  }
  __device__ __forceinline__ void step(bool on = true) { src += on ? 2 * kLmK : 0; }
  __device__ __forceinline__ void request(int half, uint32_t dst) {
#pragma unroll
    for (int e = 0; e < 2; ++e) load_to_lds(src, off[half][e], dst + e * 1024);
  }
};

template <typename A, typename B, typename AtA, typename AtB, int STEP_BYTES = kStepBytes, bool WIDE = false>
struct TileLoader {
  A a;
  B b;
  const AtA& at_a;
  const AtB& at_b;
  uint32_t lds;
  __device__ __forceinline__ void locate(const GemmTile& t) {
    const int64_t k0 = static_cast<int64_t>(t.first) * kLmK;
    a.locate(at_a, t.m0, k0);
    b.locate(at_b, t.n0, k0);
  }
  __device__ __forceinline__ void step(bool on = true) {                          // (not on: stays where it is)
    a.step(on);
    b.step(on);
  }
  __device__ __forceinline__ void request(int half, int buf) {
    const uint32_t dst = lds + buf * STEP_BYTES + half * kHalfBytes;
    if (half < (WIDE ? 1 : 2)) a.request(half, dst);
    else b.request(half == kHalfB2 ? 2 : half - 2, dst);
  }
};

// The loop over a workgroup's tiles: their steps are one stream.  The requests run ahead of the products into the next tile
// (past the last step of all: that one again, never read), so a tile has no first loads to wait for.  A step in which the
// requests pass from one tile to the next, or which follows a tile's stores, is code of its own: branches in the others cost
// 10 % (16,384 rows 14.1 -> 15.7 ms).
//   load.locate(tile)        the requests go on at the tile's first step
//   load.step()              ... at the next step
//   load.request(half, buf)  the wavefront's two loads of a half tile into a step buffer
//   store(tile, acc)         what to do with a finished tile; returns whether it left at least 63 stores behind the requests and
//                            waited for none
// A Walk without kWalks has one tile: its steps have one form, in which the requests stop at the last one without a branch, and
// the tile is stored after the end of the loop.  A_HALVES x B_HALVES: 2 x 2, 2 x 1 (matrix_step_narrow) or 1 x 3
// (matrix_step_wide); SIDE other than 16 with 2 x 2 only.
template <bool B_FIRST, int A_HALVES, int B_HALVES, int SIDE = 16, typename Walk, typename Loader, typename ReadA, typename ReadB,
          typename Store>
__device__ __forceinline__ void matrix_tiles(const MatrixPlace& mine, const unsigned char* smem, GemmTile tile, Walk walk,
                                             Loader& load, ReadA read_a, ReadB read_b, Store store) {
  GemmTile ahead_tile = tile;
  Walk ahead = walk;
  int left = tile.steps;
  load.locate(tile);
  auto advance = [&]() {
    if constexpr (!Walk::kWalks) {
      const bool more = left > 1;
      left -= more ? 1 : 0;
      load.step(more);
    } else if (--left > 0) {
      load.step();
    } else if (ahead.next(ahead_tile)) {
      left = ahead_tile.steps;
      load.locate(ahead_tile);
    } else {
      left = 1;                                            // the last step again, never read
    }
  };
  constexpr bool kNarrow = B_HALVES == 1, kWide = B_HALVES == 3;
  constexpr int kLast = 1;                                 // A1, or with three B halves B2: the last half tile of a step
  auto request_from = [&](int half, int buf) {
    load.request(half, buf);
    if (half == kLast) advance();
  };
  if constexpr (kNarrow) matrix_begin_narrow(mine, request_from);
  else if constexpr (kWide) matrix_begin_wide(mine, request_from);
  else matrix_begin(mine, request_from);
  int cur = 0;                                             // the step's buffer
  bool stored = false;
  BlockAcc<A_HALVES, B_HALVES, SIDE> acc;
  while (true) {
#pragma unroll
    for (int h = 0; h < A_HALVES; ++h)
#pragma unroll
      for (int i = 0; i < 64 / SIDE; ++i)
#pragma unroll
        for (int b = 0; b < B_HALVES; ++b)
#pragma unroll
          for (int j = 0; j < 32 / SIDE; ++j)
#pragma unroll
            for (int r = 0; r < SIDE * SIDE / 64; ++r) acc[h][i][b][j][r] = 0.f;
    auto run = [&](auto stored_tag, auto switch_tag) {
      constexpr int kBufs = kNarrow ? 3 : 2;
      const unsigned char* here = smem + cur * (kNarrow ? kNarrowBytes : kStepBytes);
      const int before = cur == 0 ? kBufs - 1 : cur - 1;
      auto a = [&](int half, int i, int ks) { return read_a(here, half, i, ks); };
      auto b = [&](int half, int j, int ks) { return read_b(here, half, j, ks); };
      auto request = [&](int half) {                       // a step's last half tile is a buffer behind the others
        load.request(half, half == kLast ? before : cur);
        if (half == kLast) {
          if constexpr (decltype(switch_tag)::value) {
            advance();
          } else {
            --left;
            load.step();
          }
        }
      };
      if constexpr (kNarrow) matrix_step_narrow<B_FIRST>(acc, a, b, request);
      else if constexpr (kWide) matrix_step_wide<B_FIRST>(acc, a, b, request);
      else matrix_step<B_FIRST, decltype(stored_tag)::value, SIDE>(acc, a, b, request);
      cur = cur == kBufs - 1 ? 0 : cur + 1;
    };
    int kt = tile.steps;
    if constexpr (!Walk::kWalks) {
      for (; kt > 0; --kt) run(std::false_type(), std::true_type());
      matrix_end(mine);
      store(tile, acc);
      return;
    }
    if (stored) {
      if (left > 1) run(std::true_type(), std::false_type());
      else run(std::true_type(), std::true_type());
      --kt;
    }
    while (kt > 0) {
      const int plain = min(kt, left - 1);
      for (int i = 0; i < plain; ++i) run(std::false_type(), std::false_type());
      kt -= plain;
      if (kt > 0) {
        run(std::false_type(), std::true_type());
        --kt;
      }
    }
    stored = store(tile, acc);
    if (!walk.next(tile)) break;
  }
  matrix_end(mine);
}

}  // namespace

namespace {

// The vocabulary tiles of a strip, one after the other.
struct StripWalk {
  static constexpr bool kWalks = true;
  int end, tile;               // first vocabulary row past the strip; rows of a tile
  __device__ __forceinline__ bool next(GemmTile& t) const {
    if (t.m0 + tile >= end) return false;
    t.m0 += tile;
    return true;
  }
};

// The tokens of a workgroup, the same for every vocabulary tile: rows of the hidden states, perhaps through a row map.
struct HiddenSource {
  const char* base;
  const char* src;
  uint32_t off[3][2];
  __device__ __forceinline__ void locate(const RowMajorHalf&, int, int64_t) { src = base; }
  __device__ __forceinline__ void step(bool on = true) { src += on ? 2 * kLmK : 0; }
  __device__ __forceinline__ void request(int half, uint32_t dst) {
#pragma unroll
    for (int e = 0; e < 2; ++e) load_to_lds(src, off[half][e], dst + e * 1024);
  }
};

// One strip of the vocabulary for the up to 128 B_HALVES tokens of a tile: pair (reference, sum) of token i to pairs[i].  The
// strip's vocabulary tiles have 128 A_HALVES rows.
template <int A_HALVES, int B_HALVES>
__device__ __forceinline__ void lm_strip(unsigned char* smem, const __bf16* __restrict__ W, int64_t ldw,
                                         const __bf16* __restrict__ H, int64_t ldh, int tokens, int V, int d, int t0,
                                         int vt_begin, int vt_end, const int* __restrict__ row_map,
                                         float2* __restrict__ pairs) {
  constexpr int J = 2 * B_HALVES;                          // 16-token blocks of a wavefront
  constexpr int kTile = 128 * A_HALVES;
  const int tid = threadIdx.x, lane = tid & 63;
  const MatrixPlace mine = matrix_place(smem);
  const RowMajorHalf at(mine);
  const RowMajorFragments<> frags(mine);
  // Rows past the end of a matrix re-read its last row (they are discarded later).  All offsets fit 32 bits (checked on the host).
  TileLoader<RowMajorSource, HiddenSource, RowMajorHalf, RowMajorHalf, B_HALVES == 1 ? kNarrowBytes : kStepBytes, B_HALVES == 3>
      load = {
      {}, {}, at, at, mine.lds};
  load.a.base = reinterpret_cast<const char*>(W);
  load.a.ld = ldw;
  load.a.rows = V;
  load.b.base = reinterpret_cast<const char*>(H) + (row_map != nullptr ? 0 : static_cast<int64_t>(t0) * ldh * 2);
#pragma unroll
  for (int h = 0; h < J / 2; ++h)
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      const int r = min(h * 128 + at.row + 8 * e, tokens - 1);
      const uint32_t row = (row_map != nullptr) ? static_cast<uint32_t>(row_map[t0 + r]) : static_cast<uint32_t>(r);
      load.b.off[h][e] = row * static_cast<uint32_t>(ldh) * 2u + at.chunk[e];
    }

  float run_ref[J], run_sum[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    run_ref[j] = kLmNone;
    run_sum[j] = 0.f;
  }
  // One finished tile.  Result register r of block i = 4 (half of the tile) + 16-row block, token block j = 2 (half) + block, is
  // vocabulary row 128 (i / 4) + 16 (i % 4) + 4 (lane / 16) + r from the wavefront's first, token 128 (j / 2) + 32 wn +
  // 16 (j % 2) + lane % 16.  RAGGED (the last vocabulary tile only): rows at or past V count as "no value".
  auto epilogue = [&](auto ragged_tag, const BlockAcc<A_HALVES, B_HALVES>& acc, int vlane) {
    constexpr bool RAGGED = decltype(ragged_tag)::value;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      auto value = [&](int i, int r) -> float {
        if (RAGGED && vlane + (i >> 2) * 128 + (i & 3) * 16 + r >= V) return kLmNone;
        return acc[i >> 2][i & 3][j >> 1][j & 1][r];
      };
      float mx = run_ref[j];
#pragma unroll
      for (int i = 0; i < 4 * A_HALVES; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) mx = fmaxf(mx, value(i, r));
      // a lane that has seen no value yet (only in a tile that hangs over the vocabulary's end) keeps
      // a finite reference, so that every term below is exp2(-inf) = 0 rather than a NaN
      const float mref = (mx == kLmNone) ? 0.f : mx * kLog2e;
      const float carried = run_sum[j] * fast_exp2(fmaf(run_ref[j], kLog2e, -mref));
      __builtin_amdgcn_sched_barrier(0);
      float part[4] = {0.f, 0.f, 0.f, 0.f};            // four short chains, added as a tree
#pragma unroll
      for (int i = 0; i < 4 * A_HALVES; ++i)
#pragma unroll
        for (int r = 0; r < 4; ++r) part[i & 3] += fast_exp2(fmaf(value(i, r), kLog2e, -mref));
      run_ref[j] = mx;
      run_sum[j] = carried + ((part[0] + part[1]) + (part[2] + part[3]));
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  const GemmTile first = {vt_begin * kTile, t0, 0, d / kLmK, 0};
  matrix_tiles<false, A_HALVES, B_HALVES>(
      mine, smem, first, StripWalk{min(vt_end * kTile, V), kTile}, load,
      [&](const unsigned char* here, int half, int i, int ks) { return frags.a(here, half, i, ks); },
      [&](const unsigned char* here, int half, int j, int ks) { return frags.b(here, half, j, ks); },
      [&](const GemmTile& t, const BlockAcc<A_HALVES, B_HALVES>& acc) {
        const int vlane = t.m0 + mine.wm * 64 + ((lane >> 4) << 2);
        if (t.m0 + kTile > V) epilogue(std::true_type(), acc, vlane);
        else epilogue(std::false_type(), acc, vlane);
        return false;
      });

  // the four groups of 16 lanes, then the two wavefronts that share these tokens, then one pair per token and strip
  float2* ex = reinterpret_cast<float2*>(smem);
#pragma unroll
  for (int j = 0; j < J; ++j) {
    float m = run_ref[j], s = run_sum[j];
    const float m2 = __shfl_xor(m, 32), s2 = __shfl_xor(s, 32);
    lm_merge(m, s, m2, s2);
    const float m3 = __shfl_xor(m, 16), s3 = __shfl_xor(s, 16);
    if (lane < 16) {
      lm_merge(m, s, m3, s3);
      ex[mine.wm * 64 * J + (j >> 1) * 128 + mine.wn * 32 + (j & 1) * 16 + lane] = make_float2(m, s);
    }
  }
  __syncthreads();
  if (tid < min(tokens, J * 64)) {
    const float2 e0 = ex[tid], e1 = ex[64 * J + tid];
    float m = e0.x, s = e0.y;
    lm_merge(m, s, e1.x, e1.y);
    pairs[tid] = make_float2(m, s);
  }
}

}  // namespace

// The launch: `whole` token tiles of 256 in `strips` strips each, then, if tail_strips > 0, one more tile of at most 128 tokens
// in strips of its own.  partial[strip * pitch + token] with pitch = 256 whole, behind them [strip * 128 + token] of the tail.
// WIDE (no whole tiles, no tail; a kernel of its own, the code of the others is 2 % slower with it): all tokens in one tile of at
// most 384, strips of 128-row vocabulary tiles, pitch T of the call.
template <bool WIDE>
__global__ void __launch_bounds__(kLmThreads)
fopd_k7_lm_head_lse(const __bf16* __restrict__ W, int64_t ldw, const __bf16* __restrict__ H, int64_t ldh,
                    int T, int V, int d, float2* __restrict__ partial, LmSplit split, int n_vocab_tiles,
                    const int* __restrict__ row_map, const int* __restrict__ n_live) {
  extern __shared__ __align__(16) unsigned char lm_smem[];
  const int pitch = WIDE ? T : split.whole * kLmTile;
  // Only the rows row_map[0 .. *n_live - 1] of H take part when a count is given (masked rows left out; the count stays
  // on the device and the launch covers all T): token tile c holds compact rows 256 c .. 256 c + 255, gathered by the
  // loads.  (A row map without a count holds all T rows.)
  if (n_live != nullptr) {
    T = *n_live;
    if (T <= 0) return;
  }
  // m: vocabulary strips, n: token tiles; each L2 serves up to 4 hidden tiles and 8 strips of the weight to 32 users
  const unsigned group = ((blockIdx.x >> 8) << 3) + (blockIdx.x & 7), slot = (blockIdx.x >> 3) & 31;
  if constexpr (WIDE) {
    const int strip = static_cast<int>(group * 32 + slot);
    if (strip >= split.strips) return;                     // whole workgroup, before any barrier
    const int vt_begin = static_cast<int>(static_cast<int64_t>(strip) * n_vocab_tiles / split.strips);
    const int vt_end = static_cast<int>(static_cast<int64_t>(strip + 1) * n_vocab_tiles / split.strips);
    lm_strip<1, 3>(lm_smem, W, ldw, H, ldh, T, V, d, 0, vt_begin, vt_end, row_map, partial + static_cast<int64_t>(strip) * pitch);
    return;
  }
  const unsigned whole_groups = static_cast<unsigned>(tile_groups(split.strips, split.whole));
  int strip, token_tile, strips = split.strips;
  float2* pairs = partial;
  if (group < whole_groups) {
    // (tiles past the count are left out, and the others packed as if there were no more)
    const int tiles = min(split.whole, (T + kLmTile - 1) / kLmTile);
    const TilePlace place = tile_place<true>(group, slot, strips, tiles);
    strip = place.m;
    token_tile = place.n;
    if (token_tile >= tiles) return;                       // whole workgroup, before any barrier
    pairs += static_cast<int64_t>(strip) * pitch + token_tile * kLmTile;
  } else {
    strip = static_cast<int>((group - whole_groups) * 32 + slot);
    strips = split.tail_strips;
    token_tile = split.whole;
    pairs += static_cast<int64_t>(split.strips) * (split.whole * kLmTile) + strip * 128;
  }
  const int t0 = token_tile * kLmTile, tokens = T - t0;
  if (strip >= strips || tokens <= 0) return;
  const int vt_begin = static_cast<int>(static_cast<int64_t>(strip) * n_vocab_tiles / strips);
  const int vt_end = static_cast<int>(static_cast<int64_t>(strip + 1) * n_vocab_tiles / strips);
  if (vt_begin == vt_end) {                                // more strips than vocabulary tiles: pairs of nothing
    if (static_cast<int>(threadIdx.x) < min(tokens, kLmTile)) pairs[threadIdx.x] = make_float2(kLmNone, 0.f);
    return;
  }
  if (tokens > 128)
    lm_strip<2, 2>(lm_smem, W, ldw, H, ldh, tokens, V, d, t0, vt_begin, vt_end, row_map, pairs);
  else
    lm_strip<2, 1>(lm_smem, W, ldw, H, ldh, tokens, V, d, t0, vt_begin, vt_end, row_map, pairs);
}

// One wavefront per token: the sampled token's logit as a dot product of two rows (fp32 products of
// bf16 are exact, the sum is fp32), then the merge of the strip pairs.  lp is clamped at 0 because
// this dot product and the matrix cores sum the same products in different orders.  ex != NULL: the unmasked rows were
// projected first or alone, row t as compact row ex[t] (ex[t] = unmasked rows before row t).
__global__ void __launch_bounds__(256)
fopd_k7_finish(const __bf16* __restrict__ W, int64_t ldw, const __bf16* __restrict__ H, int64_t ldh,
               const float2* __restrict__ partial, LmSplit split, int T, int V, int d,
               const int32_t* __restrict__ token_ids, const uint8_t* __restrict__ mask,
               float* __restrict__ logp, float* __restrict__ lse, int32_t* flags, const int* __restrict__ ex) {
  const int lane = threadIdx.x & 63;
  const int t = blockIdx.x * 4 + (threadIdx.x >> 6);
  if (t >= T) return;
  const int y = token_ids[t];
  bool live = (mask == nullptr) || (mask[t] != 0);
  if (live && (y < 0 || y >= V)) {
    if (lane == 0) atomicOr(flags, kFlagToken);
    live = false;
  }
  if (!live) {
    if (lane == 0) {
      logp[t] = 0.f;
      lse[t] = 0.f;
    }
    return;
  }
  const __bf16* h = H + static_cast<int64_t>(t) * ldh;
  const __bf16* w = W + static_cast<int64_t>(y) * ldw;
  float dot = 0.f;
  for (int k = lane * 8; k < d; k += 512) {
    const u32x4 hv = *reinterpret_cast<const u32x4*>(h + k);
    const u32x4 wv = *reinterpret_cast<const u32x4*>(w + k);
    float hx[8], wx[8];
    unpack<FOPD_BF16>(hv, hx);
    unpack<FOPD_BF16>(wv, wx);
#pragma unroll
    for (int e = 0; e < 8; ++e) dot = fmaf(hx[e], wx[e], dot);
  }
  dot = wave_sum(dot);
  // the strips' pairs: one per lane (up to 256 of them, a token's at a distance of the tokens), then across the wavefront
  const int c = (ex != nullptr) ? ex[t] : t;             // the token's place among the rows that were projected
  const bool in_tail = split.tail_strips > 0 && c >= split.whole * kLmTile;
  const int n_strips = in_tail ? split.tail_strips : split.strips, pitch = in_tail ? 128 : (split.whole > 0 ? split.whole * kLmTile : T);
  const float2* pairs = partial + (in_tail ? static_cast<int64_t>(split.strips - 1) * (split.whole * kLmTile) : 0) + c;
  float m = kLmNone, s = 0.f;
  for (int k = lane; k < n_strips; k += 64) {
    const float2 e = pairs[static_cast<int64_t>(k) * pitch];
    lm_merge(m, s, e.x, e.y);
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    const float m2 = __shfl_xor(m, off, 64), s2 = __shfl_xor(s, off, 64);
    lm_merge(m, s, m2, s2);
  }
  if (lane == 0) {
    const double l = static_cast<double>(m) + log(static_cast<double>(s));
    lse[t] = static_cast<float>(l);
    logp[t] = static_cast<float>(fmin(static_cast<double>(dot) - l, 0.0));
  }
}

}  // namespace fopd

#endif  // FOPD_LM_HEAD_HIP_
