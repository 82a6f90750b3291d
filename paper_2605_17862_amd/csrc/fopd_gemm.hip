// Dense bf16 contractions on the matrix cores of gfx950 (CDNA4), and the small kernels around them, for the
// loss pass whose logits are the output projection of the hidden states and are made chunk by chunk:
//
//   fopd_gemm_nt            Out[n, m] = sum_k Bn[n, k] * Am[m, k]         bf16 in, fp32 accumulate, fp32 out; Am as it
//                                                                        is written or stored [k, m]
//   fopd_gemm_tn            Out[n, m] (+)= sum_k Bk[k, n] * Am[m, k]     the same with B k-major
//   fopd_transpose_bf16     out[c, r] = in[r, c], zero-padded along r    (brings an operand into k-contiguous form)
//   fopd_k4_grad_wide       gradient rows from fp32 logits to bf16        c_t (softmax(z_t) - onehot)
//
// The three contractions of one chunk of R rows (d hidden size, V vocabulary):
//   logits      Z[R, V]   = H[R, d]  . W[V, d]^T          nt: n = row, m = vocabulary entry, k = hidden element
//   dL/dhidden  dH[R, d]  = dZ[R, V] . W[V, d]            nt: n = row, m = hidden element, k = vocabulary entry; W as it
//                                                         is (k-major), or for many rows W^T, formed once per call
//   dL/dweight  dW[V, d] += dZ[R, V]^T . H[R, d]          tn: n = vocabulary entry, m = hidden element, k = row; H^T is
//                                                         formed once per chunk
//
// Tiling and loop are those of the projection kernel fused with the log-sum-exp (fopd_lm_head.hip, matrix_step): a
// workgroup of eight wavefronts owns a 256 x 256 tile of the result.  The n-side fragment is the instruction's first
// operand: sixteen lanes then hold consecutive m of one output row, the contiguous side of the output.

#ifndef FOPD_GEMM_HIP_
#define FOPD_GEMM_HIP_

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "fopd_kernels.hip"
#include "fopd_lm_head.hip"

namespace fopd {

constexpr int kGemmTile = kLmTile;          // 256 x 256 result tile
constexpr int kGemmThreads = kLmThreads;

// Into how many runs of the contraction index Out[N, M] = sum over K is cut, at most `most`.  A product with few result
// tiles leaves most of the 256 compute units idle while the others walk a long contraction index; each run is a result of
// its own that is summed afterwards.  Estimate in microseconds: the rounds of the launch (tile_rounds) follow each other, an
// item takes 1.6 a step of 64 (with all compute units at work; 1.2 with sixteen) plus 13 for its first loads and its stores,
// and the partial results are read at 4.5 TB/s when they are summed.  151,936 x 4096, the contraction alone, us by number of
// runs: 256 rows 1: 2728, 8: 420, 16: 265; 512 rows 1: 2882, 4: 905, 8: 474, 16: 477; 768 rows 1: 3022, 4: 902, 8: 834, 16: 846
// (5, which 240 items on 256 compute units seem to ask for: 1289); 2048 rows 1: 3637, 2: 1863, 4: 1871; 3072 rows 1: 3602, 4:
// 2838, 8: 2887.
inline int gemm_splits(int64_t M, int64_t N, int64_t K, int64_t most) {
  const int tiles_m = static_cast<int>((M + kGemmTile - 1) / kGemmTile);
  const int tiles_n = static_cast<int>((N + kGemmTile - 1) / kGemmTile);
  const int64_t steps = K / kLmK;
  most = std::min<int64_t>(std::min<int64_t>(most, 32), steps / 8);
  int best = 1;
  double least = 0.0;
  for (int splits = 1; splits == 1 || splits <= most; ++splits) {
    const double rounds = static_cast<double>(tile_rounds(tiles_m, tiles_n, splits));
    double cost = rounds * (1.6 * static_cast<double>((steps + splits - 1) / splits) + 13.0);
    if (splits > 1) cost += static_cast<double>(splits) * static_cast<double>(M) * static_cast<double>(N) * 4.0 / 4.5e6;
    if (splits == 1 || cost < least) {
      least = cost;
      best = splits;
    }
  }
  return best;
}

// A value that is the same in every lane, for a scalar register.
__host__ __device__ __forceinline__ int uniform(int x) {
#ifdef __HIP_DEVICE_COMPILE__
  return __builtin_amdgcn_readfirstlane(x);
#else
  return x;
#endif
}

// The wavefront's part of a finished tile, rows n0 .. , columns m0 .. of Out.  The n-side fragment is the matrix
// instruction's first operand, so register r of acc[a][i][b][j] is output row n = 128 b + 32 wn + 16 j + 4 (lane / 16) + r of
// the tile and column m = 128 a + 64 wm + 16 i + lane % 16: a store of it would write half a 128-byte line to each of four
// rows.  The second and fourth 16 lanes of one register change places with the first and third of the next block's, and a store
// writes whole lines of two rows (rows n and n + 8 of one block, n + 4 and n + 12).  Weight gradient of 512 / 2048 rows x
// 151,936, d = 4096: half lines 1170 / 2647 us, whole lines 967 / 2458; four consecutive m in a lane (the m side first), 16
// bytes to each of 16 rows four times, 1251 / 2829.  The results are not read by this kernel and are far larger than the L2,
// whose lines the operand tiles need: non-temporal stores, loss and gradients of 16,384 rows 52.7 -> 51.8 ms, of 4096 rows
// 13.42 -> 13.33 ms, fewer rows unchanged (with the 32 x 32 x 16 instruction).
template <bool ACCUMULATE, bool WHOLE>
__device__ __forceinline__ void store_entry(float* to, float v, bool exists) {
  if (WHOLE || exists) {
    // (every entry of Out belongs to one lane of one workgroup, so the hardware add, which does not wait for the
    // old value to come back, gives the same sums as load - add - store, in the same order)
    if (ACCUMULATE) unsafeAtomicAdd(to, v);
    else __builtin_nontemporal_store(v, to);
  }
}

template <bool ACCUMULATE, bool WHOLE>
__device__ __forceinline__ void store_block(const BlockAcc<2, 2, 16>& acc, const MatrixPlace& place, int m0, int n0, int M,
                                            int N, float* __restrict__ Out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int m = m0 + place.wm * 64 + (lane & 31);
#pragma unroll
  for (int b = 0; b < 4; ++b) {
    const int block_n = n0 + (b >> 1) * 128 + place.wn * 32 + (b & 1) * 16;
    if (!WHOLE && uniform(block_n) >= N) continue;           // sixteen rows past the end
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int n = block_n + ((lane >> 5) << 3) + r;
      float* orow = Out + static_cast<int64_t>(n) * ldo;
#pragma unroll
      for (int i = 0; i < 8; i += 2) {
        const int mi = m + (i >> 2) * 128 + (i & 3) * 16;
        const float e0 = acc[i >> 2][i & 3][b >> 1][b & 1][r], e1 = acc[(i + 1) >> 2][(i + 1) & 3][b >> 1][b & 1][r];
        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(e0), __float_as_uint(e1), false, false);
        const float v[2] = {__uint_as_float(sw[0]), __uint_as_float(sw[1])};
#pragma unroll
        for (int h = 0; h < 2; ++h)
          store_entry<ACCUMULATE, WHOLE>(orow + 4 * h * ldo + mi, v[h], mi < M && n + 4 * h < N);
      }
    }
  }
}

// With the 32 x 32 result register r is row n = 128 b + 32 wn + 8 (r / 4) + 4 (lane / 32) + r % 4, column m = 128 a + 64 wm +
// 32 i + lane % 32: whole lines of two rows.
template <bool ACCUMULATE, bool WHOLE>
__device__ __forceinline__ void store_block(const BlockAcc<2, 2, 32>& acc, const MatrixPlace& place, int m0, int n0, int M,
                                            int N, float* __restrict__ Out, int64_t ldo) {
  const int lane = threadIdx.x & 63;
  const int m = m0 + place.wm * 64 + (lane & 31);
#pragma unroll
  for (int b = 0; b < 2; ++b)
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      const int rows_n = n0 + b * 128 + place.wn * 32 + ((r >> 2) << 3);
      if (!WHOLE && uniform(rows_n) >= N) continue;          // eight rows past the end
      const int n = rows_n + ((lane >> 5) << 2) + (r & 3);
      float* orow = Out + static_cast<int64_t>(n) * ldo;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        const int mi = m + (i >> 1) * 128 + (i & 1) * 32;
        store_entry<ACCUMULATE, WHOLE>(orow + mi, acc[i >> 1][i & 1][b][0][r], mi < M && n < N);
      }
    }
}

// A whole tile: 128 stores a wavefront, none waited for (true); else, where a tile follows, they are waited for, their number
// being unknown.  Of a tile
// with few rows only the blocks that have some are gone through: logits of 64 rows x 8192 / 32,000 / 128,000, d = 1024, 31.6 /
// 32.2 / 66 us with every store tested, 28.3 / 29.2 / 61.6 so.
template <bool ACCUMULATE, bool WALK, int SIDE>
__device__ __forceinline__ bool store_tile(const BlockAcc<2, 2, SIDE>& acc, const MatrixPlace& place, int m0, int n0, int M, int N,
                                           float* __restrict__ Out, int64_t ldo) {
  if (m0 + kGemmTile <= M && n0 + kGemmTile <= N) {
    store_block<ACCUMULATE, true>(acc, place, m0, n0, M, N, Out, ldo);
    return true;
  }
  store_block<ACCUMULATE, false>(acc, place, m0, n0, M, N, Out, ldo);
  if (WALK) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  return false;
}

// The tiles of a workgroup.  Launched with a workgroup for every place of every group (tile_place), each has one tile or none.
// Launched with kGemmGrid, one a compute unit (WALK), workgroup 8 s + x is the s-th of XCD x and takes every 32nd tile of that
// XCD's groups x, x + 8, .. in their order, only tiles that exist being counted.  The next tile's first steps are then requested
// before this one's results are stored, and no workgroup waits for its place: workgroups are started in the order of their
// ids, which keeps the compute units at the same point of their tiles.  Weight gradient of 151,936 x 4096, a workgroup a
// tile / walking, us: 256 rows 738 / 640 - 700, 512 rows 947 / 861, 1024 rows 1357 / 1286, 2048 rows 2257 / 2226, 8192 rows
// 7408 / 7334, 16,384 rows 14,804 / 14,852; logits (64 steps a tile) 512 rows 516 / 513 - 519, 16,384 rows 14,550 / 14,380;
// dL/dhidden (2374 steps) 16,384 rows 13,885 / 13,894.  So tiles of up to kWalkSteps steps are walked.  (Workgroups started a
// fraction of a tile apart: no difference; results stored 16 bytes a lane: 1 % on the logits.)  With no more tiles than workgroups there
// is nothing to walk, and the walk's code (four forms of a step, twice the instructions to fetch before the first one) is 4 - 6
// us a launch: walking / not, us: weight gradient of 3000 rows x 8192, d = 64, 65.6 / 60.3, x 1000, d = 1024, 65.4 / 60.1; loss
// and gradients of 64 rows x 8192, d = 1024, 110 / 102.  Nor where a result is added to after a single step: the memory's
// adds are all there is (weight gradient of 64 more rows, 32,000 x 1024 / 128,000 x 1024, walking 105 / 408, not 102 / 404).
constexpr unsigned kGemmGrid = 256;
constexpr int64_t kWalkSteps = 128;

inline bool gemm_walks(int64_t tiles, int64_t steps, bool accumulate) {
  return tiles > kGemmGrid && steps <= kWalkSteps && !(accumulate && steps == 1);
}

// dL/dhidden from the matrix as it is stored, where it has few tiles (a chunk of few rows of a call of many, whose sums take the
// order of the whole call): with the 32 x 32 x 16 instruction.  The multiplying slots issue half as many instructions, which
// leaves the transposing reads of the other kind their way to the LDS, and with this many compute units at work there is no
// power to be saved.  16 x 16 x 32 / 32 x 32 x 16, us by number of tiles of all runs: 151,936 entries x 4096, one run, 16: 2850
// / 2707, 32: 2986 / 2784, 48: 2910 / 2940, 64: 3374 / 3655, 128: 3570 / 3750; 32,000 x 1024, four runs, 16: 153 / 141, 32: 154
// / 143, 64: 159 / 150, 128: 170 / 161, 256: 206 / 222.  (Past 32 the larger one loses where the tiles fill their XCDs and gains
// where they fill half.  Both operands k-contiguous, 4 tiles: 1 %.)
inline bool gemm_tall(int64_t tiles) { return tiles <= 32; }

// Workgroups: walking ones, else one for every place of every group of tiles (rounds of eight groups).
inline unsigned gemm_grid(int64_t rounds, bool walk) { return walk ? kGemmGrid : static_cast<unsigned>(rounds * 256); }

// (Places are moved on by additions: a division is some thirty vector instructions in every wavefront.)
template <bool N_FIRST, bool WALK>
struct TileWalk {
  static constexpr bool kWalks = WALK;
  int tiles_m, tiles_n, all_steps, splits;
  int gn, gm, groups_n, groups_m;                // tiles and groups either way
  int split, line, pos;                          // the group: pos-th of a line of groups along n (N_FIRST) or m
  int slot;                                      // place from the group's first tile on

  __host__ __device__ __forceinline__ bool first(GemmTile& t, unsigned block) {
    gn = tile_group_n(tiles_n);
    gm = 32 / gn;
    groups_n = (tiles_n + gn - 1) / gn;
    groups_m = (tiles_m + gm - 1) / gm;
    const int per_split = groups_n * groups_m, group = static_cast<int>((block >> 8) << 3) + static_cast<int>(block & 7);
    slot = static_cast<int>(block >> 3) & 31;
    split = WALK || splits > 1 ? uniform(group / per_split) : 0;
    if (split >= splits) return false;
    const int in_split = group - split * per_split;
    if constexpr (WALK) {
      line = uniform(in_split / (N_FIRST ? groups_n : groups_m));
      pos = in_split - line * (N_FIRST ? groups_n : groups_m);
      return find(t);
    }
    const TilePlace place = tile_place<N_FIRST>(static_cast<unsigned>(in_split), static_cast<unsigned>(slot), tiles_m, tiles_n);
    if (place.m >= tiles_m || place.n >= tiles_n) return false;
    set(t, place.m, place.n);
    return true;
  }
  // (asked again after the last tile, the answer stays)
  __host__ __device__ __forceinline__ bool next(GemmTile& t) {
    if (!WALK || split >= splits) return false;
    slot += 32;
    return find(t);
  }

 private:
  __host__ __device__ __forceinline__ bool find(GemmTile& t) {
    const int length = N_FIRST ? groups_n : groups_m, lines = N_FIRST ? groups_m : groups_n;
    while (split < splits) {
      int at_m = line, at_n = pos;
      if (!N_FIRST) {                            // as tile_place: the order in a line moves on
        const int common = min(groups_m & -groups_m, 8);
        at_n = line;
        at_m = uniform((pos + (line >> (common == 1 ? 3 : common == 2 ? 2 : common == 4 ? 1 : 0))) % groups_m);
      }
      const int m = at_m * gm, n = at_n * gn;
      const int here_m = min(gm, tiles_m - m), here_n = min(gn, tiles_n - n);
      if (slot < here_m * here_n) {
        const int row = here_n == 3 ? slot / 3 : slot >> (here_n >> 1);          // here_n is 1 to 4
        set(t, m + row, n + slot - row * here_n);
        return true;
      }
      slot -= here_m * here_n;
      pos += 8;                                  // the XCD's next group
      while (pos >= length) {
        pos -= length;
        if (++line == lines) {
          line = 0;
          ++split;
        }
      }
    }
    return false;
  }
  __host__ __device__ __forceinline__ void set(GemmTile& t, int m, int n) {
    int from = 0, to = all_steps;
    if (splits > 1) {
      from = static_cast<int>(static_cast<int64_t>(all_steps) * split / splits);
      to = static_cast<int>(static_cast<int64_t>(all_steps) * (split + 1) / splits);
    }
    t = GemmTile{uniform(m * kGemmTile), uniform(n * kGemmTile), uniform(from), uniform(to - from), uniform(split)};
  }
};

// Operands with the contraction index as their row index (k-major).  A half tile of a step holds 64 k-rows of 128
// consecutive m or n as they are in memory, 256 bytes per row, the eight 32-byte blocks of a row permuted by bits 0, 1 and 3 of
// the row.  A fragment of the matrix instruction (lane = one m, eight consecutive k) is two LDS transpose reads
// (ds_read_b64_tr_b16): within a group of 16 lanes, lane 4 e + q supplies the address of four consecutive 16-bit entries and
// lane i receives entry i % 4 of the lanes 4 e + i / 4, e = 0..3 (measured with an in-bounds probe); with lane 4 e + q
// pointing at row k + e, entries m + 4 q .. 4 q + 3, lane i gets rows k .. k + 3 of entry m + i.  The 32 lanes of a pass read
// 32 bytes of rows k .. k + 3 and k + 8 .. + 11, by the permutation in eight different blocks: all 64 banks once.
//
// Wavefront w fills k-rows 8 w .. + 7 of a half tile in two loads of four rows: lane i writes 16-byte piece i % 16 of row
// i / 16 and so fetches piece (i % 16) ^ 4 (row % 4) ^ 2 (row / 8 % 2) of the 128 entries.
typedef short tn_i16x4 __attribute__((ext_vector_type(4)));
typedef short tn_i16x8 __attribute__((ext_vector_type(8)));

struct KMajorHalf {
  int krow, piece;             // row of the wavefront's first load (the second: + 4), 16-byte piece of the row
  __device__ __forceinline__ explicit KMajorHalf(const MatrixPlace& p) {
    const int lane = threadIdx.x & 63;
    const int wave = p.wm * 4 + p.wn;
    krow = 8 * wave + (lane >> 4);
    piece = (lane & 15) ^ ((lane >> 4) << 2) ^ ((wave & 1) << 1);
  }
};

template <int SIDE = 16>
struct KMajorFragments {
  static constexpr int kBlocks = SIDE / 16;      // 16-entry blocks of a fragment; the other groups of 16 lanes: rows 8 on
  int a_off[64 / SIDE], b_off[32 / SIDE];
  __device__ __forceinline__ explicit KMajorFragments(const MatrixPlace& p) {
    // lane 16 g + 4 e + q: row 8 (g / kBlocks) + e (+ 4) of those of a slice, entries 4 q .. + 3 of 16-entry block g % kBlocks
    const int lane = threadIdx.x & 63;
    const int g = (lane >> 4) / kBlocks, block = (lane >> 4) % kBlocks, e = (lane >> 2) & 3, q = lane & 3;
    const int rows = (8 * g + e) * 256 + q * 8;
#pragma unroll
    for (int i = 0; i < 64 / SIDE; ++i) a_off[i] = rows + (((4 * p.wm + i * kBlocks + block) * 32) ^ (e << 6) ^ ((g & 1) << 5));
#pragma unroll
    for (int j = 0; j < 32 / SIDE; ++j)
      b_off[j] = 2 * kHalfBytes + rows + (((2 * p.wn + j * kBlocks + block) * 32) ^ (e << 6) ^ ((g & 1) << 5));
  }
  __device__ __forceinline__ bf16x8 fragment(const unsigned char* p) const {
    typedef __attribute__((address_space(3))) tn_i16x4* lds_ptr;
    const tn_i16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p));
    const tn_i16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr)(p + 4 * 256));
    const tn_i16x8 both = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
    return __builtin_bit_cast(bf16x8, both);
  }
  __device__ __forceinline__ bf16x8 a(const unsigned char* step, int half, int i, int ks) const {
    return fragment(step + half * kHalfBytes + a_off[i] + ks * (512 / SIDE * 256));
  }
  __device__ __forceinline__ bf16x8 b(const unsigned char* step, int half, int j, int ks) const {
    return fragment(step + half * kHalfBytes + b_off[j] + ks * (512 / SIDE * 256));
  }
};

// k-major operands: pieces past the last of a row are clamped; with ROW_END there may be fewer rows than the steps have, and
// those past the last are taken from it.  By a minimum: a test for the last step, asked in every request, cuts the loop's steps
// into blocks that are scheduled apart.  In a launch with a workgroup a tile, test / minimum: dL/dhidden of 256 rows x 4096 over
// 151,936 entries 3055 / 2900 us, of 4096 rows 3900 / 3755; weight gradient of 300 - 16,384 rows 0 - 1 %.
template <bool ROW_END>
struct KMajorSource {
  const char* base;
  int64_t ld;
  int cols, rows;              // 16-byte pieces of a row, readable rows
  const char* src;
  int left;                    // rows from this step's first on
  uint32_t off[2][2], piece[2];
  __device__ __forceinline__ void locate(const KMajorHalf& at, int c0, int64_t k0) {
    src = base + k0 * ld * 2;
    left = rows - static_cast<int>(k0);
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      piece[h] = 16u * static_cast<uint32_t>(min((c0 >> 3) + 16 * h + at.piece, cols - 1));
#pragma unroll
      for (int e = 0; e < 2; ++e) off[h][e] = piece[h] + static_cast<uint32_t>(at.krow + 4 * e) * (static_cast<uint32_t>(ld) * 2u);
    }
  }
  __device__ __forceinline__ void step(bool on = true) {
    src += on ? 2 * kLmK * ld : 0;
    left -= on ? kLmK : 0;
  }
  __device__ __forceinline__ void request(int half, uint32_t dst) {
    const uint32_t last = piece[half] + static_cast<uint32_t>(min(left, kLmK) - 1) * (static_cast<uint32_t>(ld) * 2u);
#pragma unroll
    for (int e = 0; e < 2; ++e) load_to_lds(src, ROW_END ? min(off[half][e], last) : off[half][e], dst + e * 1024);
  }
};

// K must be a positive multiple of 64 (at least 64 for every split); rows of Bn, and with A_K_MAJOR = false of Am, past the
// end of an operand are clamped (re-read) and their results discarded.  Byte offsets inside one 256-row operand tile must
// fit 32 bits (checked on the host).
//
// A_K_MAJOR: Am is stored [k, m] and has rows_a (K - 64 < rows_a <= K) readable rows; rows rows_a .. K - 1 are taken from
// row rows_a - 1, so Bn must hold zeros in those columns; pieces past entry M - 1 of a row are clamped.  M % 8 == 0, lda % 8
// == 0.  This is dL/dhidden with the projection matrix as it is stored, for few rows.
template <bool A_K_MAJOR, bool WALK, int SIDE = 16>
__global__ void __launch_bounds__(kGemmThreads)
fopd_gemm_nt(const __bf16* __restrict__ Am, int64_t lda, int M, int rows_a, const __bf16* __restrict__ Bn, int64_t ldb,
             int N, int K, float* __restrict__ Out, int64_t ldo, int tiles_m, int tiles_n,
             const int* __restrict__ n_live, int splits, int64_t split_stride) {
  extern __shared__ __align__(16) unsigned char gemm_smem[];
  // Only the first *n_live rows of Bn count when a count is given (it stays on the device, the launch covers all N):
  // tiles past them are left out, and as the groups of tiles are dealt to the XCDs in turn, these stay evenly loaded
  // whatever the count is.
  if (n_live != nullptr) {
    const int live = *n_live;
    if (live <= 0) return;
    tiles_n = min(tiles_n, (live + kGemmTile - 1) / kGemmTile);
  }
  // With splits > 1 the contraction index is cut into that many runs of whole steps, each with a result of its
  // own, split_stride floats apart, which the caller sums; the groups of a run follow each other.
  TileWalk<true, WALK> walk = {tiles_m, tiles_n, K / kLmK, splits};
  GemmTile tile;
  if (!walk.first(tile, blockIdx.x)) return;               // whole workgroup, before any barrier

  const MatrixPlace mine = matrix_place(gemm_smem);
  typedef typename std::conditional<A_K_MAJOR, KMajorHalf, RowMajorHalf>::type HalfA;
  const HalfA at_a(mine);
  const RowMajorHalf at_b(mine);
  const typename std::conditional<A_K_MAJOR, KMajorFragments<SIDE>, RowMajorFragments<SIDE>>::type frags_a(mine);
  const RowMajorFragments<SIDE> frags_b(mine);
  typedef typename std::conditional<A_K_MAJOR, KMajorSource<true>, RowMajorSource>::type SourceA;
  TileLoader<SourceA, RowMajorSource, HalfA, RowMajorHalf> load = {{}, {}, at_a, at_b, mine.lds};
  load.a.base = reinterpret_cast<const char*>(Am);
  load.a.ld = lda;
  load.a.rows = A_K_MAJOR ? rows_a : M;
  if constexpr (A_K_MAJOR) load.a.cols = M >> 3;
  load.b.base = reinterpret_cast<const char*>(Bn);
  load.b.ld = ldb;
  load.b.rows = N;
  matrix_tiles<true, 2, 2, SIDE>(
      mine, gemm_smem, tile, walk, load,
      [&](const unsigned char* here, int half, int i, int ks) { return frags_a.a(here, half, i, ks); },
      [&](const unsigned char* here, int half, int j, int ks) { return frags_b.b(here, half, j, ks); },
      [&](const GemmTile& t, const BlockAcc<2, 2, SIDE>& acc) {
        return store_tile<false, WALK, SIDE>(acc, mine, t.m0, t.n0, M, N, Out + t.split * split_stride, ldo);
      });
}

// The same contraction with B k-major (the contraction index is its row index):
//
//   fopd_gemm_tn            Out[n, m] (+)= sum_{k < K} Bk[k, n] * Am[m, k]
//
// which is the weight gradient, dW[v, j] += sum_t dZ[t, v] H[t, j], with the gradient rows as they are stored and the hidden
// rows transposed (fopd_transpose_bf16: 41 - 49 us for 16,384 rows of 4096).  Loop and result stores are those of fopd_gemm_nt;
// B leaves the LDS as KMajorHalf says.  With the hidden rows k-major too, two thirds of the fragments take two transposing
// reads each, 48 LDS reads a step instead of 32, and the reading slots are longer than the multiplying ones (matrix cores
// 0.59 busy, 0.65 so): 151,936 x 4096 from 512 / 2048 / 16,384 rows 970 / 2455 / 16,300 us, so 950 / 2285 / 14,720 (a workgroup
// a tile; as it is now, 0.69 busy, 860 / 2200 / 14,800).
//
// K must be a positive multiple of 64, and Am and Bk finite up to it; what is not to count is zero in one of them.  M and N need
// not be multiples of the tile: rows of Am past M - 1 and 16-byte pieces past entry N - 1 of a row of Bk are clamped (re-read)
// and their results discarded; lda % 8 == 0, ldb % 8 == 0, and every row of Bk is readable up to N rounded up to 8 (ldb is at
// least that).  Byte offsets inside 256 rows of Am and inside 64 of Bk must fit 32 bits.
template <bool ACCUMULATE, bool WALK>
__global__ void __launch_bounds__(kGemmThreads)
fopd_gemm_tn(const __bf16* __restrict__ Am, int64_t lda, int M, const __bf16* __restrict__ Bk, int64_t ldb,
             int N, int K, float* __restrict__ Out, int64_t ldo, int tiles_m, int tiles_n,
             const int* __restrict__ k_live) {
  extern __shared__ __align__(16) unsigned char gemm_smem[];
  if (k_live != nullptr) {
    // only the first *k_live entries of the contraction index count (a device-side count; up to the next multiple of 64
    // both operands hold zeros behind them)
    const int live = *k_live;
    if (ACCUMULATE && live <= 0) return;
    K = min(K, max(64, (live + 63) & ~63));
  }
  // the groups of one set of tiles along n follow each other on neighbouring XCDs: they read the same columns of Bk, by
  // far the larger operand
  TileWalk<false, WALK> walk = {tiles_m, tiles_n, K / kLmK, 1};
  GemmTile tile;
  if (!walk.first(tile, blockIdx.x)) return;               // whole workgroup, before any barrier

  const MatrixPlace mine = matrix_place(gemm_smem);
  const RowMajorHalf at_a(mine);
  const KMajorHalf at_b(mine);
  const RowMajorFragments<> frags_a(mine);
  const KMajorFragments<> frags_b(mine);
  TileLoader<RowMajorSource, KMajorSource<false>, RowMajorHalf, KMajorHalf> load = {{}, {}, at_a, at_b, mine.lds};
  load.a.base = reinterpret_cast<const char*>(Am);
  load.a.ld = lda;
  load.a.rows = M;
  load.b.base = reinterpret_cast<const char*>(Bk);
  load.b.ld = ldb;
  load.b.rows = K;
  load.b.cols = (N + 7) >> 3;
  matrix_tiles<true, 2, 2>(
      mine, gemm_smem, tile, walk, load,
      [&](const unsigned char* here, int half, int i, int ks) { return frags_a.a(here, half, i, ks); },
      [&](const unsigned char* here, int half, int j, int ks) { return frags_b.b(here, half, j, ks); },
      [&](const GemmTile& t, const BlockAcc<2, 2>& acc) {
        return store_tile<ACCUMULATE, WALK, 16>(acc, mine, t.m0, t.n0, M, N, Out, ldo);
      });
}

// out[c, r] = in[r, c] for r < rows, c < cols; out[c, r] = 0 for rows <= r < rows_pad.  GATHER: out[c, r] = in[row_map[r], c] for
// r < n_rows[0] <= rows instead, zeros from there up to the next multiple of 64 (at least 64), and nothing is written behind
// that (what fopd_gemm_tn reads of the hidden rows that have a gradient).  128 x 128 tiles through the LDS;
// grid (ceil(rows_pad / 128), ceil(cols / 128)), 256 lanes.  cols, rows_pad, ld_in and ld_out multiples of 8, both
// matrices 16-byte aligned.  Bound by HBM (one read, one write): both sides move 16 bytes a lane in whole 128-byte lines.
// The LDS pitch of 65 words spreads the writes (four rows of sixteen lanes, four words apart) and the reads (rows eight
// apart, 8 x 65 = 8 modulo 64 words) over all banks.  151,936 x 4096: 1020 us with two bytes a lane, 453 us so (5.5 TB/s).
constexpr int kTrTile = 128;
constexpr int kTrPitch = 65;              // words

template <bool GATHER>
__global__ void __launch_bounds__(256)
fopd_transpose_bf16(const uint16_t* __restrict__ in, int64_t ld_in, int rows, int cols, uint16_t* __restrict__ out,
                    int64_t ld_out, int rows_pad, const int* __restrict__ row_map, const int* __restrict__ n_rows) {
  __shared__ uint32_t tile[kTrTile * kTrPitch];
  const int r0 = blockIdx.x * kTrTile, c0 = blockIdx.y * kTrTile;
  const int tid = threadIdx.x;
  int from[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {           // (map and count asked for together; entries behind the count are not used)
    from[u] = r0 + 16 * u + (tid >> 4);
    if (GATHER) from[u] = row_map[min(from[u], rows - 1)];
  }
  if constexpr (GATHER) {
    rows = min(rows, n_rows[0]);
    rows_pad = min(rows_pad, max(64, (rows + 63) & ~63));
    if (r0 >= rows_pad) return;
  }
  u32x4 q[8];
#pragma unroll
  for (int u = 0; u < 8; ++u) {           // sixteen rows of sixteen 16-byte pieces at a time
    const int r = r0 + 16 * u + (tid >> 4), c = c0 + 8 * (tid & 15);
    q[u] = u32x4{0u, 0u, 0u, 0u};
    if (r < rows && c < cols) q[u] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(in + from[u] * ld_in + c));
  }
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    uint32_t* dst = tile + (16 * u + (tid >> 4)) * kTrPitch + 4 * (tid & 15);
    dst[0] = q[u].x;
    dst[1] = q[u].y;
    dst[2] = q[u].z;
    dst[3] = q[u].w;
  }
  __syncthreads();
  // a wavefront writes eight output rows of eight pieces: lane = piece (rows of `in` 8 p .. 8 p + 7) + 8 x output row
  const uint16_t* half = reinterpret_cast<const uint16_t*>(tile);
#pragma unroll
  for (int u = 0; u < 8; ++u) {
    const int p = (tid & 7) + 8 * (u & 1), cc = (tid >> 3) + 32 * (u >> 1);
    const int c = c0 + cc, r = r0 + 8 * p;
    const uint16_t* src = half + 8 * p * (2 * kTrPitch) + cc;
    uint32_t e[8];
#pragma unroll
    for (int k = 0; k < 8; ++k) e[k] = src[k * (2 * kTrPitch)];
    if (c < cols && r < rows_pad)
      *reinterpret_cast<u32x4*>(out + static_cast<int64_t>(c) * ld_out + r) =
          u32x4{e[0] | (e[1] << 16), e[2] | (e[3] << 16), e[4] | (e[5] << 16), e[6] | (e[7] << 16)};
  }
}

// Gradient rows of one chunk from fp32 logits (ldz floats per row) to bf16 (ldg entries per row):
//   g[t, v] = c_t (exp(z[t, v] - lse_t) - [v == y_t]),  columns V .. ldg - 1 written as zeros
// (they are the zero padding of the contraction that follows).  One workgroup per row; rows with c_t == 0 or
// an out-of-range token id are zero-filled without reading the logits.  With grad_ex (grad_ex[t] = rows that have
// a gradient row before row t, t = 0 .. rows) the rows that have one (grad_ex[t + 1] > grad_ex[t]) are written
// densely, row t to row grad_ex[t] of G, and the others not at all.
__global__ void __launch_bounds__(kGradThreads)
fopd_k4_grad_wide(const float* __restrict__ Z, int64_t ldz, uint16_t* __restrict__ G, int64_t ldg, int V,
                  const int32_t* __restrict__ token_ids, const float* __restrict__ lse,
                  const float* __restrict__ logp, const float* __restrict__ coef,
                  const int* __restrict__ grad_ex) {
  const int64_t t = blockIdx.x;
  const int tid = threadIdx.x;
  const float c = coef[t];
  const int y = token_ids[t];
  int64_t out = t;
  if (grad_ex != nullptr) {
    out = grad_ex[t];
    if (grad_ex[t + 1] == out) return;
  }
  uint16_t* orow = G + out * ldg;
  u32x4* ov = reinterpret_cast<u32x4*>(orow);
  const int nvec_out = static_cast<int>(ldg / 8);
  if (c == 0.f || y < 0 || y >= V) {
    const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
    for (int j = tid; j < nvec_out; j += kGradThreads) __builtin_nontemporal_store(zero, ov + j);
    return;
  }
  const float lseL = lse[t] * kLog2e;
  const float gy = c * expm1f(logp[t]);
  const float* zrow = Z + t * ldz;
  const u32x4* zv = reinterpret_cast<const u32x4*>(zrow);
  const int nfull = V / 8;                       // output vectors made of eight existing logits
  for (int j = tid; j < nfull; j += kGradThreads) {
    const u32x4 q0 = __builtin_nontemporal_load(zv + 2 * j);
    const u32x4 q1 = __builtin_nontemporal_load(zv + 2 * j + 1);
    float x[8];
    unpack<FOPD_F32>(q0, x);
    unpack<FOPD_F32>(q1, x + 4);
#pragma unroll
    for (int e = 0; e < 8; ++e) x[e] = c * fast_exp2(fmaf(x[e], kLog2e, -lseL));
    if (j == (y >> 3)) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        if (e == (y & 7)) x[e] = gy;
    }
    __builtin_nontemporal_store(pack<FOPD_BF16>(x), ov + j);
  }
  for (int v = nfull * 8 + tid; v < static_cast<int>(ldg); v += kGradThreads) {    // ragged tail, then the padding
    float g = 0.f;
    if (v < V) {
      g = c * fast_exp2(fmaf(zrow[v], kLog2e, -lseL));
      if (v == y) g = gy;
    }
    store_elem<FOPD_BF16>(orow, v, g);
  }
}

// Zeroes the first `cols` entries of every row (one workgroup per row) of an fp32 matrix.
__global__ void __launch_bounds__(256) fopd_fill_zero_f32(float* out, int64_t ld, int cols) {
  float* row = out + static_cast<int64_t>(blockIdx.x) * ld;
  for (int c = threadIdx.x; c < cols; c += 256) row[c] = 0.f;
}

// ---- rows that take part moved to the front of a chunk, so that the contractions skip the others ----
// Masked rows (observations, prompts) have no log-prob and no gradient row: the chunk's per-row inputs and hidden
// states are gathered into dense arrays of the live rows (mask != 0), every kernel of the chunk runs on those, and
// the per-row outputs are scattered back (zeros at masked rows).  With scores supplied the live rows of the whole
// call are numbered once and the chunks are runs of that numbering, so that every chunk but the last is full; with
// the scores formed inside, the chunks are whole samples and each is numbered by itself.  Once the coefficients are known the same is done
// again for the gradient side: only the rows with c_t != 0 (not those of samples the freshness weight gates out)
// get a gradient row, written densely, and the two gradient contractions run on those.  The counts stay on the
// device: the launches cover the whole chunk, the contraction kernels read the count and leave out the rest.

constexpr int kLiveScanThreads = 1024;

// keep[i] = 1 if sample i has a positive weight under the scores given (float64 ones if fresh64 != NULL, else the
// float32 ones), else 0.
__global__ void __launch_bounds__(256)
fopd_sample_keep(const double* __restrict__ fresh64, const float* __restrict__ fresh32,
                 const int32_t* __restrict__ n_train, const int32_t* __restrict__ n_roll,
                 const int32_t* __restrict__ lag, int B, float xi, int* __restrict__ keep) {
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= B) return;
  const int32_t n = n_train[i];
  const double f = (fresh64 != nullptr) ? fresh64[i] : static_cast<double>(fresh32[i]);
  keep[i] = weight_of(f, n, (n_roll != nullptr) ? n_roll[i] : n, lag[i], xi) > 0.0 ? 1 : 0;
}

// One workgroup.  A row is live if coef != NULL ? (coef[j] != 0 or, with coef2, coef2[j] != 0) : (mask == NULL ||
// mask[j] != 0) and, with keep, keep[sample of row row_begin + j] != 0; mask / coef / coef2 point at the chunk's
// first row.  ex[j] = live rows before chunk row j, j = 0 .. R; row_map[c] = chunk row of compact row c
// (row_map may be NULL; with rest_too the other rows follow in it, the last first); n_live[0] = ex[R]; cu_c[i] =
// ex[clamp(cu[i] - row_begin, 0, R)], i = 0 .. B: the samples' offsets among the chunk's live rows (B < 0: none wanted).
__global__ void __launch_bounds__(kLiveScanThreads)
fopd_live_scan(const uint8_t* __restrict__ mask, const float* __restrict__ coef, const float* __restrict__ coef2, int R,
               const int64_t* __restrict__ cu,
               int B, int64_t row_begin, int* __restrict__ ex, int* __restrict__ row_map, int* __restrict__ n_live,
               int64_t* __restrict__ cu_c, const int* __restrict__ keep, bool rest_too) {
  __shared__ int wave_total[kLiveScanThreads / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto is_live = [&](int j) {
    if (coef != nullptr) return coef[j] != 0.f || (coef2 != nullptr && coef2[j] != 0.f);
    if (mask != nullptr && mask[j] == 0) return false;
    return keep == nullptr || keep[sample_of_row(cu, B, row_begin + j)] != 0;
  };
  // 1024 rows at a time, row base + tid to lane tid (reads and writes of consecutive lanes are consecutive): a
  // wavefront's ballot gives each lane its place among the wavefront's live rows, the sixteen totals give the rest
  int run = 0;
  for (int64_t base = 0; base < R; base += kLiveScanThreads) {
    const int64_t j = base + tid;
    const bool live = j < R && is_live(static_cast<int>(j));
    const unsigned long long votes = __ballot(live);
    const int before_lane = __popcll(votes & ((1ull << lane) - 1ull));
    if (lane == 0) wave_total[wave] = __popcll(votes);
    __syncthreads();
    int before_wave = 0, all = 0;
#pragma unroll
    for (int w = 0; w < kLiveScanThreads / 64; ++w) {
      const int n = wave_total[w];
      before_wave += (w < wave) ? n : 0;
      all += n;
    }
    if (j < R) {
      const int at = run + before_wave + before_lane;
      ex[j] = at;
      if (live && row_map != nullptr) row_map[at] = static_cast<int>(j);
      if (!live && rest_too) row_map[R - 1 - (j - at)] = static_cast<int>(j);
    }
    run += all;
    __syncthreads();                                         // before the totals are overwritten
  }
  if (tid == 0) {
    ex[R] = run;
    n_live[0] = run;
  }
  __syncthreads();                                           // ex[] of the other lanes is visible from here on
  for (int i = tid; i <= B; i += kLiveScanThreads) {
    int64_t j = cu[i] - row_begin;
    j = j < 0 ? 0 : (j > R ? R : j);
    cu_c[i] = ex[j];
  }
}

// Dense row c = blockIdx.x of a chunk (c < gridDim.x) is live row map_off + c of the scan: row row_base +
// row_map[map_off + c] of the caller's arrays if map_off + c < n_live[0], else a masked row of zeros.  Gathers the
// per-row inputs, the listed teacher and the hidden row; the arrays are the caller's (first row), not the chunk's;
// teacher_logp, teacher_stale and the list may be NULL.  n_chunk[0] = the chunk's live rows (what the contraction
// kernels read).  d % 8 == 0.
__global__ void __launch_bounds__(256)
fopd_live_gather(const int* __restrict__ row_map, const int* __restrict__ n_live, int64_t map_off, int64_t row_base,
                 int* __restrict__ n_chunk, const int32_t* __restrict__ token_ids, const uint8_t* __restrict__ mask,
                 const float* __restrict__ behav_logp, const float* __restrict__ teacher_logp,
                 const float* __restrict__ teacher_stale, const int32_t* __restrict__ list_ids,
                 const float* __restrict__ list_logp, int k, const uint16_t* __restrict__ hidden, int64_t ldh, int d,
                 int32_t* __restrict__ token_ids_c, uint8_t* __restrict__ mask_c, float* __restrict__ behav_c,
                 float* __restrict__ teacher_c, float* __restrict__ stale_c, int32_t* __restrict__ list_ids_c,
                 float* __restrict__ list_logp_c, uint16_t* __restrict__ hidden_c) {
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  const int64_t total = n_live[0];
  const bool live = map_off + c < total;
  const int64_t j = live ? row_base + row_map[map_off + c] : 0;
  if (tid == 0) {
    if (c == 0) {
      const int64_t here = total - map_off;
      n_chunk[0] = static_cast<int>(here < 0 ? 0 : (here > gridDim.x ? gridDim.x : here));
    }
    token_ids_c[c] = live ? token_ids[j] : 0;
    mask_c[c] = live ? (mask != nullptr ? mask[j] : static_cast<uint8_t>(1)) : static_cast<uint8_t>(0);
    behav_c[c] = live ? behav_logp[j] : 0.f;
    if (teacher_logp != nullptr) teacher_c[c] = live ? teacher_logp[j] : 0.f;
    if (teacher_stale != nullptr) stale_c[c] = live ? teacher_stale[j] : 0.f;
  }
  if (list_ids != nullptr) {
    for (int q = tid; q < k; q += 256) {
      list_ids_c[c * k + q] = live ? list_ids[j * k + q] : -1;
      list_logp_c[c * k + q] = live ? list_logp[j * k + q] : 0.f;
    }
  }
  const u32x4* src = reinterpret_cast<const u32x4*>(hidden + j * ldh);
  u32x4* dst = reinterpret_cast<u32x4*>(hidden_c + c * d);
  const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
  for (int v = tid; v < d / 8; v += 256) dst[v] = live ? src[v] : zero;
}

// Zeros behind the gradient rows, up to the next multiple of 64 (at least 64 rows in all): the contraction over rows reads that
// far.  Row n_grad[0] + blockIdx.x of G (ldg entries, ldg % 8 == 0); grid: 64 workgroups.
__global__ void __launch_bounds__(256)
fopd_grad_tail_zero(const int* __restrict__ n_grad, uint16_t* __restrict__ G, int64_t ldg) {
  const int n = n_grad[0];
  const int64_t row = static_cast<int64_t>(n) + blockIdx.x;
  if (row >= max(64, (n + 63) & ~63)) return;
  const u32x4 zero = u32x4{0u, 0u, 0u, 0u};
  u32x4* g = reinterpret_cast<u32x4*>(G + row * ldg);
  for (int v = threadIdx.x; v < static_cast<int>(ldg / 8); v += 256) g[v] = zero;
}

// dst[0 .. d) = sum over k < splits, in that order, of src[k split_stride ..], by 256 lanes.  src 16-byte aligned,
// split_stride and d multiples of 4; dst 16-byte aligned where its pitch lddst is a multiple of 4.
__device__ __forceinline__ void sum_splits_row(const float* __restrict__ src, int splits, int64_t split_stride, int d,
                                               float* __restrict__ dst, int64_t lddst) {
  const bool wide = (lddst & 3) == 0;
  for (int v = threadIdx.x * 4; v < d; v += 1024) {
    f32x4 sum = *reinterpret_cast<const f32x4*>(src + v);
    for (int k = 1; k < splits; ++k) sum += *reinterpret_cast<const f32x4*>(src + k * split_stride + v);
    if (wide) {
      *reinterpret_cast<f32x4*>(dst + v) = sum;
    } else {
#pragma unroll
      for (int e = 0; e < 4; ++e) dst[v + e] = sum[e];
    }
  }
}

// Dense row c = blockIdx.x of a chunk hands its outputs to the caller's row row_base + row_map[map_off + c] (nothing
// if map_off + c >= n_live[0]): log-prob and log-sum-exp (logp, lse: NULL together), token loss, and as dL/dhidden row the dense gradient row
// grad_ex[c] of dhidden_g if the row has one (grad_ex[c + 1] > grad_ex[c]), zeros if not.  token_loss / token_loss_c
// and dhidden / dhidden_g / grad_ex may be NULL.
__global__ void __launch_bounds__(256)
fopd_live_scatter(const int* __restrict__ row_map, const int* __restrict__ n_live, int64_t map_off, int64_t row_base,
                  const float* __restrict__ logp_c, const float* __restrict__ lse_c,
                  const float* __restrict__ token_loss_c, const int* __restrict__ grad_ex,
                  const float* __restrict__ dhidden_g, int splits, int64_t split_stride, int d,
                  float* __restrict__ logp, float* __restrict__ lse, float* __restrict__ token_loss,
                  float* __restrict__ dhidden, int64_t lddh) {
  const int64_t c = blockIdx.x;
  const int tid = threadIdx.x;
  if (map_off + c >= n_live[0]) return;
  const int64_t t = row_base + row_map[map_off + c];
  if (tid == 0) {
    if (logp != nullptr) {
      logp[t] = logp_c[c];
      lse[t] = lse_c[c];
    }
    if (token_loss != nullptr) token_loss[t] = token_loss_c[c];
  }
  if (dhidden != nullptr) {
    const int g = grad_ex[c];
    const bool has = grad_ex[c + 1] > g;
    const float* src = dhidden_g + static_cast<int64_t>(g) * d;
    float* dst = dhidden + t * lddh;
    if (has) {
      sum_splits_row(src, splits, split_stride, d, dst, lddh);
    } else {
      for (int v = tid; v < d; v += 256) dst[v] = 0.f;
    }
  }
}

// Row blockIdx.x of dhidden = the sum of the partial results of fopd_gemm_nt (R rows of d floats each).
__global__ void __launch_bounds__(256)
fopd_sum_splits(const float* __restrict__ partial, int splits, int64_t split_stride, int d, float* __restrict__ dhidden,
                int64_t lddh) {
  const int64_t r = blockIdx.x;
  sum_splits_row(partial + r * d, splits, split_stride, d, dhidden + r * lddh, lddh);
}

// Zeros in the outputs of the rows first .. first + gridDim.x - 1 that take no part: masked ones (mask != NULL and mask[r] == 0)
// and, with keep, those of samples with keep[i] == 0 (cu: the samples' offsets).  Log-prob and log-sum-exp (NULL
// together), token loss (may be NULL), dL/dhidden row (may be NULL).
__global__ void __launch_bounds__(256)
fopd_masked_rows_zero(int64_t first, const uint8_t* __restrict__ mask, const int64_t* __restrict__ cu, int B,
                      const int* __restrict__ keep, float* __restrict__ logp, float* __restrict__ lse,
                      float* __restrict__ token_loss, float* __restrict__ dhidden, int64_t lddh, int d) {
  const int64_t r = first + blockIdx.x;
  const bool masked = (mask != nullptr && mask[r] == 0);
  if (!masked && (keep == nullptr || keep[sample_of_row(cu, B, r)] != 0)) return;
  if (threadIdx.x == 0) {
    if (logp != nullptr) {
      logp[r] = 0.f;
      lse[r] = 0.f;
    }
    if (token_loss != nullptr) token_loss[r] = 0.f;
  }
  if (dhidden != nullptr) {
    float* dst = dhidden + r * lddh;
    for (int v = threadIdx.x; v < d; v += 256) dst[v] = 0.f;
  }
}

// loss = sum of the per-chunk shares, in chunk order.
__global__ void fopd_sum_chunks(const float* chunk_loss, int n, float* loss) {
  if (threadIdx.x == 0 && blockIdx.x == 0) {
    double s = 0.0;
    for (int i = 0; i < n; ++i) s += static_cast<double>(chunk_loss[i]);
    loss[0] = static_cast<float>(s);
  }
}

}  // namespace fopd

#endif  // FOPD_GEMM_HIP_
