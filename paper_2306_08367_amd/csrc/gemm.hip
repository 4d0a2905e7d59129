// Dense C = act(A * B + bias) on the matrix cores, fp32 accumulate.
//
// Used for the pre-fusion products P_k = D_k * (rows of L owned by dimension k) (underlined terms
// of Eq. 1) and for the layer-by-layer model evaluation of the non-fused pipeline (T * L, second
// line of Eq. 1).  Five kernels:
//   gemm_tiled_kernel  - 128 x BN tiles (BN = 64 or 128) staged through LDS, 4 wavefronts in a
//                        2 x 2 arrangement, each owning 64 x BN/2 as 32x32 MFMA accumulators.
//                        bf16 inputs stay bf16 in LDS and use the 32x32x16 bf16 MFMA, the next
//                        k-tile fetched into registers while the current one is multiplied; fp32
//                        inputs of up to 16 k, which are one k-tile, use the 32x32x2 f32 MFMA.
//   gemm_split_kernel  - fp32, more than 16 k: every operand as the sum of three bf16 numbers, six of
//                        their nine products on the 32x32x16 bf16 MFMA.
//   gemm_rowsplit_kernel - fp32, N <= 8, 32 <= K: the shape of projecting a wide dimension table
//                        onto a handful of outputs, bound by reading A once.  The lanes of a
//                        wavefront read A as contiguous 16-byte pieces (a row is split over 8..64
//                        neighbouring lanes), multiply with the weights held in LDS and sum over
//                        the lanes of a row with DPP adds: no matrix cores, every load a full
//                        coalesced run.
//   gemm_skinny_kernel - N <= 16 (linear models with a handful of outputs).  Bandwidth-shaped:
//                        no LDS, every wavefront streams 16 rows of A at a time straight into
//                        16x16 MFMA operands; B is tiny and comes from cache.
//   gemm_short_kernel  - fp32, k <= 16, 17 to 128 columns: weights in registers, no LDS, the result
//                        is nearly all of the traffic.
#include "lq_common.h"

namespace lq {
namespace {

typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));

struct GemmArgs {
  const void* A; int64_t lda;
  const void* B; int64_t ldb;
  void* C; int64_t ldc;
  const void* bias;
  int64_t M; int32_t N; int32_t Kd;
  int32_t relu;
  int32_t a_vec_ok, b_vec_ok;   // 16-byte loads of A / B rows are legal
  int32_t tiles_n;
};

// Up to LQ_MAX_DIMS independent products of the same type in one launch (the projections of all
// dimension tables): workgroup b works on problem p where first_tile[p] <= b < first_tile[p + 1].
// A launch of one problem (MOST = 1) passes and looks up that one only: the arguments of eight and the search among
// them cost a small launch about half a microsecond (one table of 15,338 x 8 onto 4 outputs with the join of 1.6e6 rows: 18.2 us,
// 17.6 so).
template <int MOST>
struct GemmBatchOf {
  GemmArgs g[MOST];
  int32_t first_tile[MOST + 1];
  int32_t count;
};
typedef GemmBatchOf<LQ_MAX_DIMS> GemmBatch;
inline GemmBatchOf<1> only_problem(const GemmBatch& b) { return {{b.g[0]}, {b.first_tile[0], b.first_tile[1]}, 1}; }

// The problem this workgroup works on.
template <int MOST>
__device__ __forceinline__ int problem_of(const GemmBatchOf<MOST>& b) {
  int p = 0;
  if constexpr (MOST == 1) return p;
  while (p + 1 < b.count && static_cast<int>(blockIdx.x) >= b.first_tile[p + 1]) ++p;
  return p;
}

// ------------------------------------------------------------------ tiled --------------

constexpr int BM = 128;
constexpr int TILED_THREADS = 256;

template <typename T> struct Tile;
template <> struct Tile<float> {
  static constexpr int BK = 16;        // k per LDS tile
  static constexpr int VEC = 4;        // elements per 16-byte chunk
};
template <> struct Tile<bf16_t> {
  static constexpr int BK = 64;
  static constexpr int VEC = 8;
};

struct __attribute__((packed, aligned(4))) Words4 { unsigned int x, y, z, w; };

// 16 bytes starting at p, of which only the first `valid` elements exist (others read as zero).
template <typename T>
__device__ __forceinline__ v4u load_chunk(const T* p, int valid, bool vec_ok) {
  constexpr int VEC = Tile<T>::VEC;
  if (valid >= VEC && vec_ok) return *reinterpret_cast<const v4u*>(p);
  if constexpr (sizeof(T) == 4) {
    // Rows whose stride is not a multiple of four floats (a table with 683 columns): still one 16-byte
    // load, declared with the 4-byte alignment the pointer has.
    if (valid >= VEC) {
      const Words4 t = *reinterpret_cast<const Words4*>(p);
      return v4u{t.x, t.y, t.z, t.w};
    }
  }
  v4u r = {0u, 0u, 0u, 0u};
  if (valid <= 0) return r;
  if constexpr (sizeof(T) == 4) {
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < valid) r[q] = reinterpret_cast<const unsigned int*>(p)[q];
  } else {
#pragma unroll
    for (int q = 0; q < 8; ++q)
      if (q < valid) r[q >> 1] |= static_cast<unsigned int>(p[q]) << (16 * (q & 1));
  }
  return r;
}

// Three (128 columns) and four (64) workgroups a compute unit, as many as the accumulators leave room for.
template <typename TA, typename TC, int BN>
__global__ __launch_bounds__(TILED_THREADS, BN == 64 ? 4 : 3) void gemm_tiled_kernel(GemmBatch batch) {
  int problem = 0;
  while (problem + 1 < batch.count && static_cast<int32_t>(blockIdx.x) >= batch.first_tile[problem + 1]) ++problem;
  const GemmArgs g = batch.g[problem];
  const int64_t tile = static_cast<int64_t>(blockIdx.x) - batch.first_tile[problem];
  constexpr int BK = Tile<TA>::BK, VEC = Tile<TA>::VEC;
  constexpr bool F32 = sizeof(TA) == 4;
  constexpr int WN = BN / 2;              // columns per wavefront
  constexpr int TN = WN / 32;             // 32-wide MFMA tiles per wavefront along n (1 or 2)
  constexpr int A_CHUNKS = BM * BK / VEC / TILED_THREADS;   // 16-byte chunks per thread
  constexpr int B_CHUNKS = BK * BN / VEC / TILED_THREADS;
  constexpr int A_CPR = BK / VEC;         // chunks per A row
  constexpr int B_CPR = BN / VEC;         // chunks per B row
  // fp32: k-major tiles  As[k][m], Bs[k][n] (one word per MFMA operand read).
  // bf16: As[m][k], Bs[n][k] with k contiguous (eight consecutive k per MFMA operand read).
  constexpr int PADF = 4, PADH = 8;
  constexpr int A_WORDS = F32 ? BK * (BM + PADF) : BM * (BK + PADH) / 2;
  constexpr int B_WORDS = F32 ? BK * (BN + PADF) : BN * (BK + PADH) / 2;
  __shared__ __align__(16) unsigned int smemA[A_WORDS];
  __shared__ __align__(16) unsigned int smemB[B_WORDS];

  const TA* __restrict__ A = static_cast<const TA*>(g.A);
  const TA* __restrict__ B = static_cast<const TA*>(g.B);
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int64_t tile_m = tile / g.tiles_n;
  const int tile_n = static_cast<int>(tile % g.tiles_n);
  const int64_t m0 = tile_m * BM;
  const int n0 = tile_n * BN;

  v16f acc[2][TN];
#pragma unroll
  for (int i = 0; i < 2; ++i)
#pragma unroll
    for (int j = 0; j < TN; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[i][j][v] = 0.f;

  v4u ra[A_CHUNKS], rb[B_CHUNKS];
  auto fetch = [&](int k0) {
#pragma unroll
    for (int c = 0; c < A_CHUNKS; ++c) {
      const int id = tid + c * TILED_THREADS;
      const int r = id / A_CPR, kc = (id % A_CPR) * VEC;
      const int64_t row = min(m0 + r, g.M - 1);            // rows past the end repeat the last row
      ra[c] = load_chunk<TA>(A + row * g.lda + k0 + kc, g.Kd - (k0 + kc), g.a_vec_ok);
    }
#pragma unroll
    for (int c = 0; c < B_CHUNKS; ++c) {
      const int id = tid + c * TILED_THREADS;
      const int kk = id / B_CPR, nc = (id % B_CPR) * VEC;
      const int k = k0 + kk;
      rb[c] = load_chunk<TA>(B + static_cast<int64_t>(min(k, g.Kd - 1)) * g.ldb + n0 + nc,
                             k < g.Kd ? g.N - (n0 + nc) : 0, g.b_vec_ok);
    }
  };
  auto stage = [&]() {
#pragma unroll
    for (int c = 0; c < A_CHUNKS; ++c) {
      const int id = tid + c * TILED_THREADS;
      const int r = id / A_CPR, kc = (id % A_CPR) * VEC;
      if constexpr (F32) {
#pragma unroll
        for (int q = 0; q < 4; ++q) smemA[(kc + q) * (BM + PADF) + r] = ra[c][q];
      } else {
        *reinterpret_cast<v4u*>(&smemA[(r * (BK + PADH) + kc) / 2]) = ra[c];
      }
    }
#pragma unroll
    for (int c = 0; c < B_CHUNKS; ++c) {
      const int id = tid + c * TILED_THREADS;
      const int kk = id / B_CPR, nc = (id % B_CPR) * VEC;
      if constexpr (F32) {
        *reinterpret_cast<v4u*>(&smemB[kk * (BN + PADF) + nc]) = rb[c];
      } else {
        unsigned short* sb = reinterpret_cast<unsigned short*>(smemB);
#pragma unroll
        for (int q = 0; q < 8; ++q)
          sb[(nc + q) * (BK + PADH) + kk] = static_cast<unsigned short>(rb[c][q >> 1] >> (16 * (q & 1)));
      }
    }
  };

  auto multiply = [&](int k0) {
    if constexpr (F32) {
      const float* As = reinterpret_cast<const float*>(smemA);
      const float* Bs = reinterpret_cast<const float*>(smemB);
      // Steps past k hold nothing but zeros and are left out, eight columns at a time.
      const int steps = min(BK, (g.Kd - k0 + 7) & ~7);
      for (int k8 = 0; k8 < steps; k8 += 8) {
#pragma unroll
        for (int kk = k8; kk < k8 + 8; kk += 2) {
          const int k = kk + (lane >> 5);
          float a[2], b[TN];
#pragma unroll
          for (int i = 0; i < 2; ++i) a[i] = As[k * (BM + PADF) + wm * 64 + i * 32 + (lane & 31)];
#pragma unroll
          for (int j = 0; j < TN; ++j) b[j] = Bs[k * (BN + PADF) + wn * WN + j * 32 + (lane & 31)];
#pragma unroll
          for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j)
              acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(a[i], b[j], acc[i][j], 0, 0, 0);
        }
      }
    } else {
#pragma unroll
      for (int kk = 0; kk < BK; kk += 16) {
        const int k = kk + 8 * (lane >> 5);
        v4u a[2], b[TN];
#pragma unroll
        for (int i = 0; i < 2; ++i)
          a[i] = *reinterpret_cast<const v4u*>(&smemA[((wm * 64 + i * 32 + (lane & 31)) * (BK + PADH) + k) / 2]);
#pragma unroll
        for (int j = 0; j < TN; ++j)
          b[j] = *reinterpret_cast<const v4u*>(&smemB[((wn * WN + j * 32 + (lane & 31)) * (BK + PADH) + k) / 2]);
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
          for (int j = 0; j < TN; ++j)
            acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[i]),
                                                                __builtin_bit_cast(bf16x8, b[j]), acc[i][j], 0, 0, 0);
      }
    }
  };

  fetch(0);
  for (int k0 = 0; k0 < g.Kd; k0 += BK) {
    __syncthreads();            // previous tile fully consumed
    stage();
    __syncthreads();
    if (k0 + BK < g.Kd) fetch(k0 + BK);
    multiply(k0);
  }

  // 32x32 accumulator: register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.  The bias goes in before the
  // row tests: used inside them it would be waited for again in each, and such a wait is for every store before it
  // too (rows written one after the other: 5,000 x 32 -> 128 columns 13.9 us with the waits, 7.7 without).
  TC* __restrict__ C = static_cast<TC*>(g.C);
  const TA* bias = static_cast<const TA*>(g.bias);
  const int64_t row0 = m0 + wm * 64 + 4 * (lane >> 5);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    const int col = n0 + wn * WN + j * 32 + (lane & 31);
    if (col >= g.N) continue;
    const float bv = bias ? Elem<TA>::load(bias + col) : 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float x = acc[i][j][v] + bv;
        acc[i][j][v] = g.relu ? fmaxf(x, 0.f) : x;
      }
    TC* p = C + row0 * g.ldc + col;
    if (m0 + BM <= g.M) {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) Elem<TC>::store(p + (i * 32 + 8 * (v >> 2) + (v & 3)) * g.ldc, acc[i][j][v]);
    } else {
#pragma unroll
      for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int at = i * 32 + 8 * (v >> 2) + (v & 3);
          if (row0 + at < g.M) Elem<TC>::store(p + at * g.ldc, acc[i][j][v]);
        }
    }
  }
}

// ------------------------------------------------------------------ split --------------

// fp32, more than 16 k and 16 columns.  An fp32 number is exactly the sum of three bf16 numbers: each piece is rounded to nearest at 8 bits,
// so the second one is at most 2^-8 of the number and the third one at most 2^-17.  Of the nine products of two such sums the six
// largest go through the bf16 matrix instruction, whose products are exact and whose sums are fp32.  The other three are at most 2^-24 of the
// product (both operands next to 1.0039) and 2^-28 of it on average over all mantissas, of either sign.  Six bf16 instructions take 3/8 of the
// time of the fp32 instructions for the same tile.
// The products of the two first pieces and the five small ones have sums of their own, added at the end: a sum is rounded with every
// instruction that adds to it, so the large one is rounded once per 16 k, and the rounding of the small ones does not show.  (All six in
// one sum: 277 us instead of 289 at 16,555 x 683 -> 2,048 in three problems, 2,110 instead of 2,220 at 200,000 x 1,024 -> 1,024, but
// farther off than fp32 instructions where operands are zero, which round nothing there, and a little biased.)
// Relative error in the 2-norm against float64 with fp32 instructions / one sum / so, for k = 64 and 683: normal values 1.4e-7, 1.1e-7,
// 5.0e-8 and 4.7e-7, 4.0e-7, 1.5e-7; values in [0, 1] 1.2e-7, 8.5e-8, 4.9e-8 and 4.0e-7, 2.9e-7, 1.5e-7; normal values cut off at zero
// 1.0e-7, 1.05e-7, 4.2e-8 and 3.3e-7, 3.8e-7, 1.2e-7; one operand of 20 not zero 4.1e-8, 6.5e-8, 2.7e-8 and 1.1e-7, 2.1e-7, 4.2e-8; a single
// product of two 24-bit numbers, where the products left out do show, 2.53e-8, 3.3e-8, 2.58e-8.
// What the pieces cannot hold is computed again with fp32 instructions before it is stored:
//  * an infinity or a value that rounds to a bf16 infinity leaves a NaN in its row or column, since the second piece is then inf - inf or an
//    infinity of the other sign (a NaN leaves one too, which stands);
//  * an operand below 2^-100 other than zero has pieces among the subnormal numbers and may lose up to 2^-126.  A result whose row or
//    column holds one is computed again if it is below 2^-30, or if its column or row holds an operand of 2^64 or more.  What
//    stands is then at least 2^-30 and has lost less than 2^-62 a term.  (Not where the row or the column is all zeros.)
// Which results these are depends on their own row and column only, and the order of the sums on k only: a row computed alone equals
// the same row computed as part of a table, whichever of the instances below computes it.
// A wavefront with such an operand, or with a NaN, reads its rows once more, and its rows and the columns of a tile of 32 again for
// a tile with results to compute again.  16,555 x 683 -> 2,048, 289 us without any and 411 with fp32 instructions: a NaN in one row 290, in a row
// of a hundred 318, in all rows 349, in one column 288; operands below 2^-100 in one row 292, in one of a hundred 323, in all 363; an infinity in one
// row 383, in one of a hundred 710, in all 1,003, in one column 342.  10,000 x 32 -> 64, 4.0 us: 7.2 to 9.6 in rows, 11.1 with a column of infinities.
//
// A wavefront owns 32 rows and all 32 TN columns of the tile.  Its rows of A go from memory straight into operand layout
// (lane: row l % 32, eight consecutive k) and are split once, in registers; only B passes through LDS, split by the workgroup,
// in two buffers with one barrier per 16 k.  With 128 columns the two sums leave room for two wavefronts a SIMD, in two workgroups or in
// one of eight wavefronts, which splits B half as often.  (Both operands through LDS, 64 x 64 a wavefront, in one sum: 278 instead of 271 us
// for the former shape, 2,200 instead of 2,000 for the latter; 64 rows a wavefront and 64 columns in two sums: 309 and 2,410, 64 rows
// and 128 columns, one wavefront a SIMD: 350 and 2,520; with fp32 instructions, one word of either operand a lane from LDS, 412 and 3,250.)
// Large tables are bound by the matrix instructions and the splitting beside them: 1.1 PFLOP/s in bf16 operations, 1.26 in a bf16 product of
// 8,192^3 from the vendor's library, 1.6 to 1.8 in these instructions alone on registers with random operands (2.0 to 2.5 on zeros);
// short tables by the chain of a step: load, split, LDS, products.

// Floats as sums of three bf16 numbers each, packed in pairs.
template <int N>
__device__ __forceinline__ void split_pairs(const float (&x)[N], unsigned int (&p)[3][N / 2]) {
#pragma unroll
  for (int q = 0; q < N / 2; ++q) {
    const unsigned int h = f32x2_to_bf16x2(x[2 * q], x[2 * q + 1]);
    const float r0 = x[2 * q] - __uint_as_float(h << 16), r1 = x[2 * q + 1] - __uint_as_float(h & 0xffff0000u);
    const unsigned int m = f32x2_to_bf16x2(r0, r1);
    p[0][q] = h;
    p[1][q] = m;
    p[2][q] = f32x2_to_bf16x2(r0 - __uint_as_float(m << 16), r1 - __uint_as_float(m & 0xffff0000u));
  }
}

// The smaller of `least` and |x| as a number without its sign bit, shifted left; zero counts as the largest.
template <int N>
__device__ __forceinline__ uint32_t least_of(const float (&x)[N], uint32_t least) {
#pragma unroll
  for (int q = 0; q < N; ++q) least = min(least, (__float_as_uint(x[q]) << 1) - 1u);
  return least;
}

// The larger of `most` and |x|; a NaN stays one.
template <int N>
__device__ __forceinline__ float most_of(const float (&x)[N], float most) {
#pragma unroll
  for (int q = 0; q < N; q += 2)
    most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(__builtin_fabsf(x[q]), __builtin_fabsf(x[q + 1])), most);
  return most;
}

template <int TN, int WAVES>
__global__ __launch_bounds__(64 * WAVES, TN > 2 ? 2 : 4) void gemm_split_kernel(GemmBatch batch) {
  int problem = 0;
  while (problem + 1 < batch.count && static_cast<int32_t>(blockIdx.x) >= batch.first_tile[problem + 1]) ++problem;
  const GemmArgs g = batch.g[problem];
  // Tiles are dealt to the eight XCDs in runs, columns first, so that an XCD's L2 sees an eighth of A's rows only (200,000 x 1,024 ->
  // 1,024 1,973 us so, 2,026 dealt in turn).
  const int32_t at = static_cast<int32_t>(blockIdx.x) - batch.first_tile[problem];
  const int32_t tiles = batch.first_tile[problem + 1] - batch.first_tile[problem];
  const int32_t tile = at % 8 * (tiles / 8) + min(at % 8, tiles % 8) + at / 8;
  constexpr int BK = 16, BN = 32 * TN;
  constexpr int THREADS = 64 * WAVES, BP = BN * BK / THREADS;  // consecutive k of B in a thread
  static_assert(THREADS % BN == 0 && BP * (THREADS / BN) == BK, "B's tile must be dealt out evenly");
  constexpr int PLANE = BN * 2;                                // 16-byte pieces of a part: [column / 32][half of k][column % 32]
  __shared__ __align__(16) v4u smem[2][3 * PLANE];
  __shared__ int range_b[THREADS], tiny_b[WAVES];              // of a thread's part of its column, of a wavefront
  const float* __restrict__ A = static_cast<const float*>(g.A);
  const float* __restrict__ B = static_cast<const float*>(g.B);
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), half = lane >> 5;
  const int64_t m0 = (static_cast<int64_t>(tile / g.tiles_n) * WAVES + wave) * 32;
  const int n0 = tile % g.tiles_n * BN;

  v16f acc[TN], low[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) { acc[j][v] = 0.f; low[j][v] = 0.f; }

  // Rows past the end repeat the last row and columns past the end the last column; both are never stored.
  float ra[8], rb[BP];
  const float* row_a = A + min(m0 + (lane & 31), g.M - 1) * g.lda;
  const int bk = tid / BN * BP, bc = tid % BN;
  const uint32_t col_b = min(n0 + bc, g.N - 1);
  uint32_t least_a = 0xffffffffu, least_b = 0xffffffffu;
  float most_b = 0.f;

  auto fetch_a = [&](int k0) {
#pragma unroll
    for (int h = 0; h < 8; h += 4) {
      const Words4 t = *reinterpret_cast<const Words4*>(row_a + k0 + 8 * half + h);
      ra[h] = __uint_as_float(t.x); ra[h + 1] = __uint_as_float(t.y);
      ra[h + 2] = __uint_as_float(t.z); ra[h + 3] = __uint_as_float(t.w);
    }
  };
  auto fetch = [&](int k0) {
    fetch_a(k0);
    const float* base = B + static_cast<int64_t>(k0 + (BN >= 64 ? __builtin_amdgcn_readfirstlane(bk) : bk)) * g.ldb;
#pragma unroll
    for (int q = 0; q < BP; ++q) rb[q] = (base + q * g.ldb)[col_b];
  };
  // The last step takes the last 16 k there are; those of them that the step before has had are cleared.
  const int steps = (g.Kd + BK - 1) / BK, last_k = g.Kd - BK, had = steps * BK - g.Kd;
  auto clear_a = [&]() {
#pragma unroll
    for (int q = 0; q < 8; ++q) ra[q] = 8 * half + q >= had ? ra[q] : 0.f;
  };
  auto clear_b = [&]() {
#pragma unroll
    for (int q = 0; q < BP; ++q) rb[q] = bk + q >= had ? rb[q] : 0.f;
  };
  auto stage_b = [&](int buf) {
    unsigned int pb[3][BP / 2];
    split_pairs<BP>(rb, pb);
    least_b = least_of<BP>(rb, least_b);
    most_b = most_of<BP>(rb, most_b);
#pragma unroll
    for (int p = 0; p < 3; ++p) {
      v4u* to = &smem[buf][p * PLANE + (bc / 32 * 2 + bk / 8) * 32 + bc % 32];
      if constexpr (BP == 8) *to = v4u{pb[p][0], pb[p][1], pb[p][2], pb[p][3]};
      else if constexpr (BP == 4) reinterpret_cast<uint2*>(to)[bk / 4 % 2] = make_uint2(pb[p][0], pb[p][1]);
      else reinterpret_cast<unsigned int*>(to)[bk / 2 % 4] = pb[p][0];
    }
  };
  auto is_tiny = [](uint32_t least) { return least < (27u << 24) - 1u; };           // (27 << 24: 2^-100 shifted left)
  constexpr int TINY = 1, VAST = 2, NANS = 4, SOME = 8;        // an operand below 2^-100, one of 2^64 or more, a NaN, one that is not zero
  auto range_of = [&](uint32_t least, float most) {
    return (is_tiny(least) ? TINY : 0) | (most < 0x1p64f ? 0 : VAST) | (most != most ? NANS : 0) | (least != 0xffffffffu ? SOME : 0);
  };
  v4u a[3];
  auto split_a = [&]() {
    unsigned int pa[3][4];
    split_pairs<8>(ra, pa);
    least_a = least_of<8>(ra, least_a);
#pragma unroll
    for (int p = 0; p < 3; ++p) a[p] = v4u{pa[p][0], pa[p][1], pa[p][2], pa[p][3]};
  };
  auto multiply = [&](int buf) {
    const v4u* from = &smem[buf][half * 32 + lane % 32];
    // Two column tiles at a time: their sums are independent of each other, and no more of B's operands fit beside the sums of four.
    constexpr int JB = TN > 2 ? 2 : 1;
#pragma unroll
    for (int j0 = 0; j0 < TN; j0 += JB) {
      constexpr int PA[6] = {2, 0, 1, 0, 1, 0}, PB[6] = {0, 2, 1, 0, 0, 1}, READ[3] = {0, 2, 1};
      v4u b[JB][3];
#pragma unroll
      for (int t = 0; t < 3; ++t)
#pragma unroll
        for (int j = 0; j < JB; ++j) b[j][READ[t]] = from[READ[t] * PLANE + (j0 + j) * 64];
      if constexpr (TN == 4) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = 0; t < 6; ++t)
#pragma unroll
        for (int j = 0; j < JB; ++j) {
          v16f& sum = PA[t] + PB[t] == 0 ? acc[j0 + j] : low[j0 + j];
          sum = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a[PA[t]]), __builtin_bit_cast(bf16x8, b[j][PB[t]]), sum, 0, 0, 0);
        }
    }
  };

  // Step st: A's operands are in ra, B's in LDS since the step before; both of the next step are fetched ahead of the products.
  // The buffer that B's next part goes to was read in the step before, which every wavefront has left at the barrier.
  // The last two steps stand apart: next to a branch the loads would be waited for before the products.
  int st = 0;
  fetch(0);
  stage_b(0);
  for (; st + 2 < steps; ++st) {
    split_a();
    fetch((st + 1) * BK);
    __syncthreads();
    multiply(st & 1);
    stage_b(~st & 1);
  }
  split_a();
  fetch(last_k);
  __syncthreads();
  multiply(st & 1);
  clear_b();
  stage_b(~st & 1);
  const int tiny_here = __any(is_tiny(least_b));
  if (lane == 0) tiny_b[wave] = tiny_here;
  range_b[tid] = range_of(least_b, most_b);
  clear_a();
  split_a();
  __syncthreads();
  multiply(~st & 1);
  bool tiny = __any(is_tiny(least_a)) != 0;                    // an operand below 2^-100, not zero, in these rows or columns
#pragma unroll
  for (int w = 0; w < WAVES; ++w) tiny = tiny || tiny_b[w] != 0;

  // 32x32 accumulator: register v of lane l is row 8*(v/4) + 4*(l/32) + v%4, column l%32.
  // Zero times an infinity or a NaN is a NaN: one instruction an element where nothing is to be computed again.
  float zeros[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int j = 0; j < TN; ++j)
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      acc[j][v] += low[j][v];
      zeros[v % 4] = __builtin_fmaf(acc[j][v], 0.f, zeros[v % 4]);
    }
  const bool stands = !tiny && !__any(zeros[0] + zeros[1] + zeros[2] + zeros[3] != 0.f);

  // The bias goes in before the row tests: used inside them it would be waited for again in each, and such a wait is for every
  // store before it too (rows written one after the other: 5,000 x 32 -> 128 columns 13.9 us with the waits, 7.7 without).
  float* __restrict__ C = static_cast<float*>(g.C);
  const float* bias = static_cast<const float*>(g.bias);
  const int64_t row0 = m0 + 4 * half;
  float bv[TN];
#pragma unroll
  for (int j = 0; j < TN; ++j) bv[j] = bias ? bias[min(n0 + j * 32 + (lane & 31), g.N - 1)] : 0.f;
  auto value = [&](float x, int j) {
    x += bv[j];
    return g.relu ? fmaxf(x, 0.f) : x;
  };
  if (stands && m0 + 32 <= g.M) {
#pragma unroll
    for (int j = 0; j < TN; ++j) {
      const int col = n0 + j * 32 + (lane & 31);
      if (col >= g.N) continue;
      float* p = C + row0 * g.ldc + col;
#pragma unroll
      for (int v = 0; v < 16; ++v) p[(8 * (v >> 2) + (v & 3)) * g.ldc] = value(acc[j][v], j);
    }
    return;
  }

  auto store = [&](const v16f& x, int j, uint32_t which) {
    const int col = n0 + j * 32 + (lane & 31);
    float* p = C + row0 * g.ldc + col;
#pragma unroll
    for (int v = 0; v < 16; ++v) {
      const int r = 8 * (v >> 2) + (v & 3);
      if ((which >> v & 1u) && row0 + r < g.M && col < g.N) p[r * g.ldc] = value(x[v], j);
    }
  };
  if (stands) {
#pragma unroll
    for (int j = 0; j < TN; ++j) store(acc[j], j, 0xffffu);
    return;
  }

  // Something is to be computed again, or may be.  The rows are read once more, for what they hold; a lane reads half of one.
  // (Kept up in the loop above, their largest operands took 3 % of every product.)
  least_a = 0xffffffffu;
  float most_a = 0.f;
#pragma unroll 4
  for (int st = 0; st < steps; ++st) {
    fetch_a(min(st * BK, last_k));
    least_a = least_of<8>(ra, least_a);
    most_a = most_of<8>(ra, most_a);
  }
  int of_a = range_of(least_a, most_a);
  of_a |= __shfl_xor(of_a, 32);
  auto rows_with = [&](int what) { return static_cast<uint32_t>(__ballot((of_a & what) != 0)) >> 4 * half; };      // a bit a row, from row0 on
  const uint32_t tiny_rows = rows_with(TINY), vast_rows = rows_with(VAST), nan_rows = rows_with(NANS), some_rows = rows_with(SOME);
#pragma unroll
  for (int j = 0; j < TN; ++j) {
    float zero = 0.f;
#pragma unroll
    for (int v = 0; v < 16; ++v) zero = __builtin_fmaf(acc[j][v], 0.f, zero);
    uint32_t redo = 0;                                         // a bit an element
    const int c = n0 + j * 32 + (lane & 31);
    const float* col = B + min(c, g.N - 1);
    auto load_b = [&](int k0, float (&x)[8]) {
      const float* p = col + static_cast<int64_t>(k0 + 8 * half) * g.ldb;
#pragma unroll
      for (int q = 0; q < 8; ++q) x[q] = p[q * g.ldb];
    };
    if (tiny || __any(zero != 0.f)) {
      int of_b = 0;
#pragma unroll
      for (int q = 0; q < THREADS; q += BN) of_b |= range_b[q + j * 32 + (lane & 31)];
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int r = 8 * (v >> 2) + (v & 3);
        const uint32_t u = __float_as_uint(acc[j][v]) & 0x7fffffffu;
        const bool small = u < (97u << 23);                    // (2^-30)
        const bool lost = ((tiny_rows >> r & 1u) && (small || (of_b & VAST))) || ((of_b & TINY) && (small || (vast_rows >> r & 1u)));
        const bool again = u >= 0x7f800000u ? !((nan_rows >> r & 1u) || (of_b & NANS)) : lost && (some_rows >> r & 1u) && (of_b & SOME);
        redo |= again && row0 + r < g.M && c < g.N ? 1u << v : 0u;
      }
    }
    store(acc[j], j, ~redo);
    if (!__any(redo != 0)) continue;
    // With fp32 instructions, the operands straight from memory (lane: row or column l % 32, eight consecutive k), those of the next step ahead of
    // the products.  The last step as above.
    v16f x;
#pragma unroll
    for (int v = 0; v < 16; ++v) x[v] = 0.f;
    float xb[8];
    fetch_a(0);
    load_b(0, xb);
#pragma unroll 1
    for (int st = 0; st < steps; ++st) {
      const int skip = st + 1 < steps ? 0 : had, next = min((st + 1) * BK, last_k);
      float ya[8], yb[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) {
        ya[q] = 8 * half + q >= skip ? ra[q] : 0.f;
        yb[q] = 8 * half + q >= skip ? xb[q] : 0.f;
      }
      fetch_a(next);
      load_b(next, xb);
#pragma unroll
      for (int q = 0; q < 8; ++q) x = __builtin_amdgcn_mfma_f32_32x32x2f32(ya[q], yb[q], x, 0, 0, 0);
    }
    store(x, j, redo);
  }
}

// ------------------------------------------------------------------ skinny -------------

constexpr int SKINNY_THREADS = 256;

// N <= 16.  A wavefront takes 16 rows per pass; lane (g = lane / 16, i = lane % 16) loads 16-byte
// pieces of row i at k = kc + VEC*g and feeds them element by element as the K-slices of 16x16
// MFMAs whose B operand holds the matching rows of the weight matrix (which rows of k a slot
// means is irrelevant as long as A and B agree, and they are built from the same index).
template <typename TA, typename TC, int MOST>
__global__ __launch_bounds__(SKINNY_THREADS) void gemm_skinny_kernel(GemmBatchOf<MOST> batch) {
  const int p = problem_of(batch);
  const GemmArgs g = batch.g[p];             // (a copy: through a reference the loop has fewer loads in flight, three bf16
                                             // tables of 200,000 x 256 onto 4 outputs 141.8 us instead of 128.4)
  constexpr int VEC = Tile<TA>::VEC;
  constexpr bool F32 = sizeof(TA) == 4;
  constexpr int KSTEP = 4 * VEC;             // k covered by one 16-byte load per lane
  const TA* __restrict__ A = static_cast<const TA*>(g.A);
  const TA* __restrict__ B = static_cast<const TA*>(g.B);
  const int lane = threadIdx.x & 63, grp = lane >> 4, i = lane & 15;
  const int64_t wave = static_cast<int64_t>(blockIdx.x - batch.first_tile[p]) * (SKINNY_THREADS / 64) + (threadIdx.x >> 6);
  const int64_t nwaves = static_cast<int64_t>(batch.first_tile[p + 1] - batch.first_tile[p]) * (SKINNY_THREADS / 64);
  const int64_t npass = (g.M + 15) / 16;
  const float bv = (g.bias && i < g.N) ? Elem<TA>::load(static_cast<const TA*>(g.bias) + i) : 0.f;

  for (int64_t pass = wave; pass < npass; pass += nwaves) {
    const int64_t row = min(pass * 16 + i, g.M - 1);
    const TA* ar = A + row * g.lda;
    v4f acc = {0.f, 0.f, 0.f, 0.f};
    for (int kc = 0; kc < g.Kd; kc += KSTEP) {
      const int k = kc + VEC * grp;
      const v4u a = load_chunk<TA>(ar + k, g.Kd - k, g.a_vec_ok);
      // B operand: lane (grp, n = i) needs W[k + t][n] for t = 0..VEC-1
      if constexpr (F32) {
#pragma unroll
        for (int t = 0; t < 4; ++t) {
          const float b = (k + t < g.Kd && i < g.N) ? B[static_cast<int64_t>(k + t) * g.ldb + i] : 0.f;
          acc = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(a[t]), b, acc, 0, 0, 0);
        }
      } else {
        v4u b = {0u, 0u, 0u, 0u};
#pragma unroll
        for (int t = 0; t < 8; ++t)
          if (k + t < g.Kd && i < g.N)
            b[t >> 1] |= static_cast<unsigned int>(B[static_cast<int64_t>(k + t) * g.ldb + i]) << (16 * (t & 1));
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b),
                                                      acc, 0, 0, 0);
      }
    }
    // register v of lane (grp, n) is row 4*grp + v of the pass, column n
    if (i < g.N) {
      TC* __restrict__ C = static_cast<TC*>(g.C);
#pragma unroll
      for (int v = 0; v < 4; ++v) {
        const int64_t r = pass * 16 + 4 * grp + v;
        if (r >= g.M) continue;
        float x = acc[v] + bv;
        if (g.relu) x = fmaxf(x, 0.f);
        Elem<TC>::store(C + r * g.ldc + i, x);
      }
    }
  }
}

// ------------------------------------------------------------------ short k ------------

// fp32, at most 16 rows of weights and 17 to 128 columns (a narrow star under a wide first layer).  The result is most of
// the traffic, so what bounds the product is how soon and how steadily it is written; a tile of the kernel above has one
// k-step, and its barriers and the way through LDS are then a good part of a workgroup's time.  Here a wavefront keeps 64
// columns of the weights in registers and walks over its row blocks without LDS or barriers: A goes from memory into
// the operand (both halves of the wavefront read the same 16 bytes, which costs an L1 hit), the next block's rows are
// requested before the products of this one.  Order of the additions as in the tiled kernel: the same bits.
// Over k = 1, 4, 8, 11, 16, 17 to 128 columns and 1,000 to 2,400,000 rows it takes 0.87 times the tiled kernel's time (0.56 to
// 1.15).  k = 4 / 16: 5,000 rows, 128 columns 7.0 -> 4.9 / 7.4 -> 5.0 us; 100,000 rows, 64 columns 9.4 -> 9.7 / 10.2 -> 10.7;
// 200,000 rows, 128 columns 21.2 -> 24.3 / 24.4 -> 25.9 (its worst); 2,400,000 rows, 64 columns 143 -> 122 / 145 -> 147,
// 128 columns 223 -> 235 / 275 -> 266 (4.6 TB/s written).  With a second instance for 17 to 32 rows of weights the tiled kernel
// was the faster one from 20,000 rows on (64 columns, k = 17: 6.5 against 7.0 us, 600,000 rows 38 against 47).
constexpr int SHORT_THREADS = 256, SHORT_K = 16, SHORT_ROWS = 32, SHORT_COLS = 64;

__global__ __launch_bounds__(SHORT_THREADS) void gemm_short_kernel(GemmArgs g, int per_wave /*row blocks*/) {
  const float* __restrict__ A = static_cast<const float*>(g.A);
  const float* __restrict__ B = static_cast<const float*>(g.B);
  float* __restrict__ C = static_cast<float*>(g.C);
  const float* bias = static_cast<const float*>(g.bias);
  const int lane = threadIdx.x & 63, r = lane & 31, h = lane >> 5;
  const int64_t wave = static_cast<int64_t>(blockIdx.x) * (SHORT_THREADS / 64) + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int col_groups = (g.N + SHORT_COLS - 1) / SHORT_COLS;       // neighbouring wavefronts share the rows
  const int64_t blocks = (g.M + SHORT_ROWS - 1) / SHORT_ROWS;
  const int64_t first = wave / col_groups * per_wave, last = min(first + per_wave, blocks);
  const int n0 = static_cast<int>(wave % col_groups) * SHORT_COLS;
  if (first >= blocks) return;

  // (loaded with clamped indexes and cleared afterwards: loads under a test each are waited for one by one)
  float b[SHORT_K / 2][2], bv[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int col = min(n0 + j * 32 + r, g.N - 1);
    bv[j] = bias ? bias[col] : 0.f;
#pragma unroll
    for (int s = 0; s < SHORT_K / 2; ++s) b[s][j] = B[min(2 * s + h, g.Kd - 1) * g.ldb + col];
  }
#pragma unroll
  for (int s = 0; s < SHORT_K / 2; ++s)
#pragma unroll
    for (int j = 0; j < 2; ++j) b[s][j] = 2 * s + h < g.Kd ? b[s][j] : 0.f;
  v4u a[SHORT_K / 4], next[SHORT_K / 4];
  // (16 bytes at a time whatever the alignment: 600,000 x 16 -> 128 79.8 to 80.4 us so, 80.2 to 80.9 with aligned loads)
  auto fetch = [&](int64_t block) {
    const float* row = A + min(block * SHORT_ROWS + r, g.M - 1) * g.lda;      // rows past the end repeat the last row
#pragma unroll
    for (int q = 0; q < SHORT_K / 4; ++q) next[q] = load_chunk<float>(row + 4 * q, g.Kd - 4 * q, false);
  };
  fetch(first);
  for (int64_t block = first; block < last; ++block) {
#pragma unroll
    for (int q = 0; q < SHORT_K / 4; ++q) a[q] = next[q];
    if (block + 1 < last) fetch(block + 1);
    v16f acc[2];
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) acc[j][v] = 0.f;
#pragma unroll
    for (int s = 0; s < SHORT_K / 2; ++s) {
      if (s >= SHORT_K / 4 && 2 * s >= g.Kd) break;               // nothing but zeros from here
      const float x = __uint_as_float(h ? a[s / 2][2 * (s & 1) + 1] : a[s / 2][2 * (s & 1)]);
#pragma unroll
      for (int j = 0; j < 2; ++j) acc[j] = __builtin_amdgcn_mfma_f32_32x32x2f32(x, b[s][j], acc[j], 0, 0, 0);
    }
    // the bias before the row and column tests, as in the tiled kernel
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const float x = acc[j][v] + bv[j];
        acc[j][v] = g.relu ? fmaxf(x, 0.f) : x;
      }
    const int64_t row0 = block * SHORT_ROWS + 4 * h;
    const bool in0 = n0 + r < g.N, in1 = n0 + 32 + r < g.N;
    float* p = C + row0 * g.ldc + n0 + r;
    if (block * SHORT_ROWS + SHORT_ROWS <= g.M) {
      if (in0) {
#pragma unroll
        for (int v = 0; v < 16; ++v) p[(8 * (v >> 2) + (v & 3)) * g.ldc] = acc[0][v];
      }
      if (in1) {
#pragma unroll
        for (int v = 0; v < 16; ++v) p[(8 * (v >> 2) + (v & 3)) * g.ldc + 32] = acc[1][v];
      }
    } else {
#pragma unroll
      for (int v = 0; v < 16; ++v) {
        const int at = 8 * (v >> 2) + (v & 3);
        if (row0 + at >= g.M) continue;
        if (in0) p[at * g.ldc] = acc[0][v];
        if (in1) p[at * g.ldc + 32] = acc[1][v];
      }
    }
  }
}

int launch_short(const GemmArgs& g, hipStream_t s) {
  const int64_t col_groups = (g.N + SHORT_COLS - 1) / SHORT_COLS, blocks = (g.M + SHORT_ROWS - 1) / SHORT_ROWS;
  // up to four row blocks a wavefront once there are three wavefronts a SIMD without that (5,000 rows with four blocks
  // each: 11 us, with one 5; 2,400,000 rows with up to eight 5 to 10 % slower than with four)
  const int per_wave = static_cast<int>(std::max<int64_t>(1, std::min<int64_t>(4, blocks * col_groups / (int64_t{num_cus()} * 12))));
  const int64_t waves = (blocks + per_wave - 1) / per_wave * col_groups, wgs = (waves + 3) / 4;
  if (wgs > 0x7fffff) return -1;             // (a grid's threads stay below 2^32)
  hipLaunchKernelGGL(gemm_short_kernel, dim3(static_cast<unsigned>(wgs)), dim3(SHORT_THREADS), 0, s, g, per_wave);
  LQ_LAUNCH_CHECK("gemm_short_kernel");
  return LQ_OK;
}

// Deals the tiles of bm x bn out to the workgroups of one launch; all problems of the batch share N.  `blocks`: their number.
int deal_tiles(GemmBatch& b, int bm, int bn, int64_t* blocks) {
  *blocks = 0;
  for (int p = 0; p < b.count; ++p) {
    GemmArgs& g = b.g[p];
    g.tiles_n = (g.N + bn - 1) / bn;
    b.first_tile[p] = static_cast<int32_t>(*blocks);
    *blocks += (g.M + bm - 1) / bm * g.tiles_n;
    if (*blocks > 0x7fffffffLL) return fail(LQ_ERR_UNSUPPORTED, "gemm: %lld tiles exceed one grid", (long long)*blocks);
  }
  b.first_tile[b.count] = static_cast<int32_t>(*blocks);
  return LQ_OK;
}

// All problems of the batch share N (hence the tile width) and the element types.
template <typename TA, typename TC>
int launch_tiled_batch(GemmBatch& b, hipStream_t s) {
  const bool wide = b.g[0].N > 64;
  for (int p = 0; p < b.count; ++p) {
    GemmArgs& g = b.g[p];
    g.a_vec_ok = aligned(g.A, 16) && (g.lda * sizeof(TA)) % 16 == 0;
    g.b_vec_ok = aligned(g.B, 16) && (g.ldb * sizeof(TA)) % 16 == 0;
  }
  int64_t blocks;
  const int rc = deal_tiles(b, BM, wide ? 128 : 64, &blocks);
  if (rc || blocks == 0) return rc;
  if (wide)
    hipLaunchKernelGGL((gemm_tiled_kernel<TA, TC, 128>), dim3(static_cast<unsigned>(blocks)), dim3(TILED_THREADS), 0, s, b);
  else
    hipLaunchKernelGGL((gemm_tiled_kernel<TA, TC, 64>), dim3(static_cast<unsigned>(blocks)), dim3(TILED_THREADS), 0, s, b);
  LQ_LAUNCH_CHECK("gemm_tiled_kernel");
  return LQ_OK;
}

// All problems of the batch share N.  The narrowest tiles keep the most loads in flight and the shortest chain of a step, the widest
// read A and split it the fewest times: 32 columns up to two and a half tiles of 128 x 32 a compute unit, 128 columns from four
// tiles of 128 x 128 on, and those in workgroups of eight wavefronts from eight tiles of 256 x 128 on (eight rounds) unless k is short, when
// filling and emptying a tile is most of it.  Time in us with 32 / 64 / 128 columns / eight wavefronts for k = 32, 128 and 512:
// 16,384 rows -> 128 columns (512 narrow tiles) 5.2 / 5.4 / 6.7 / 7.6, 8.0 / 9.0 / 11 / 14 and 23 / 26 / 31 / 39; 41,600 -> 128 (1,300; 325 wide ones)
// 9.4 / 8.5 / 9.3 / 9.3, 18 / 15 / 17 / 16 and 54 / 42 / 43 / 42; 28,000 -> 512 (3,500; 876) 18 / 15 / 16 / 17, 39 / 31 / 31 / 31 and 128 / 95 / 89 / 93;
// 40,000 -> 512 (1,252 wide) 23 / 20 / 20 / 23, 54 / 43 / 41 / 43 and 182 / 132 / 123 / 127; 96,000 -> 512 (3,000; 1,500 large ones) 51 / 42 / 42 / 45,
// 128 / 101 / 94 / 93 and 444 / 326 / 302 / 294; 160,000 -> 512 (2,500 large) 117 / 90 / 86 / 85, 238 / 185 / 175 / 162 and 746 / 540 / 504 / 480; 600,000 x 33 ->
// 128 (2,344) 123 / 94 / 87 / 96; 16,555 x 683 -> 2,048 (1,040) 404 / 306 / 291 / 294; 200,000 x 1,024 -> 1,024 (6,256) 3,610 / 2,530 / 2,320 / 2,210.
int launch_split_batch(GemmBatch& b, hipStream_t s) {
  const int N = b.g[0].N;
  const int64_t cus = num_cus();
  int64_t large, wide, narrow, blocks;
  if (int rc = deal_tiles(b, 128, 32, &narrow)) return rc;
  if (narrow == 0) return LQ_OK;
  if (int rc = deal_tiles(b, 256, 128, &large)) return rc;
  if (int rc = deal_tiles(b, 128, 128, &wide)) return rc;
#define LQ_SPLIT(TN_, WAVES_)                                                                                                 \
  do {                                                                                                                        \
    if (int rc = deal_tiles(b, 32 * WAVES_, 32 * TN_, &blocks)) return rc;                                                    \
    hipLaunchKernelGGL((gemm_split_kernel<TN_, WAVES_>), dim3(static_cast<unsigned>(blocks)), dim3(64 * WAVES_), 0, s, b);    \
  } while (0)
  if (N <= 32 || 2 * narrow <= 5 * cus) LQ_SPLIT(1, 4);
  else if (N <= 64 || wide < 4 * cus) LQ_SPLIT(2, 4);
  else if (large < 8 * cus || b.g[0].Kd < 64) LQ_SPLIT(4, 4);
  else LQ_SPLIT(4, 8);
#undef LQ_SPLIT
  LQ_LAUNCH_CHECK("gemm_split_kernel");
  return LQ_OK;
}

// fp32 problems of one N, more than 16 columns: each by its k alone, so that a row does not depend on the table it is part of.
int launch_wide_f32(const GemmBatch& all, hipStream_t s) {
  for (const bool split : {false, true}) {
    GemmBatch b{};
    for (int p = 0; p < all.count; ++p)
      if ((all.g[p].Kd > 16) == split) b.g[b.count++] = all.g[p];
    if (b.count == 0) continue;
    const int rc = split ? launch_split_batch(b, s) : launch_tiled_batch<float, float>(b, s);
    if (rc) return rc;
  }
  return LQ_OK;
}

// All problems of the batch have up to 16 columns and the same element types.
template <typename TA, typename TC>
int launch_skinny_batch(GemmBatch& b, hipStream_t s) {
  int64_t blocks = 0;
  for (int p = 0; p < b.count; ++p) {
    GemmArgs& g = b.g[p];
    g.a_vec_ok = aligned(g.A, 16) && (g.lda * sizeof(TA)) % 16 == 0;
    b.first_tile[p] = static_cast<int32_t>(blocks);
    blocks += std::min<int64_t>(((g.M + 15) / 16 + 3) / 4, static_cast<int64_t>(num_cus()) * 8);
  }
  b.first_tile[b.count] = static_cast<int32_t>(blocks);
  if (blocks == 0) return LQ_OK;
  const dim3 grid(static_cast<unsigned>(blocks)), block(SKINNY_THREADS);
  if (b.count == 1) hipLaunchKernelGGL((gemm_skinny_kernel<TA, TC, 1>), grid, block, 0, s, only_problem(b));
  else hipLaunchKernelGGL((gemm_skinny_kernel<TA, TC, LQ_MAX_DIMS>), grid, block, 0, s, b);
  LQ_LAUNCH_CHECK("gemm_skinny_kernel");
  return LQ_OK;
}

template <typename TA, typename TC>
int launch_typed(GemmArgs g, hipStream_t s) {
  if (g.M <= 0 || g.N <= 0) return LQ_OK;
  if (g.N <= 16) {
    GemmBatch b{};
    b.g[0] = g;
    b.count = 1;
    return launch_skinny_batch<TA, TC>(b, s);
  }
  if constexpr (sizeof(TA) == 4 && sizeof(TC) == 4) {
    if (g.Kd >= 1 && g.Kd <= SHORT_K && g.N <= 128) {     // (17 to 128 columns: see gemm_short_kernel)
      const int rc = launch_short(g, s);
      if (rc >= 0) return rc;
    }
  }
  GemmBatch b{};
  b.g[0] = g;
  b.count = 1;
  if constexpr (sizeof(TA) == 4) return launch_wide_f32(b, s);
  else return launch_tiled_batch<TA, TC>(b, s);
}

// ------------------------------------------------------------------ row split ----------

constexpr int RS_THREADS = 256;

template <int CTRL> __device__ __forceinline__ float rs_dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, false));
}
// One step of a sum over lanes that scatters its results: the lane keeps the half of its V values that its bit selects and
// gets the other lane's share of that half; a single value is just summed.  `other` fetches from the lane that differs in that bit.
template <int V, typename F> __device__ __forceinline__ void rs_halve(float* y, bool upper, F other) {
  if constexpr (V == 1) y[0] += other(y[0]);
#pragma unroll
  for (int i = 0; i < V / 2; ++i) {
    const float keep = upper ? y[V / 2 + i] : y[i], send = upper ? y[i] : y[V / 2 + i];
    y[i] = keep + other(send);
  }
}
constexpr int rs_half(int v) { return v > 1 ? v / 2 : 1; }
// Sums of V values (a power of two) over the LPR lanes of a group, V / LPR of them or one in every lane: lane c ends with
// number rs_first(c) and the ones behind it.  (The mirrored exchanges also flip the lower lane bits, so they come before
// those have selected anything.)
template <int V, int LPR> __device__ __forceinline__ void rs_reduce(float (&y)[V], int lane) {
  constexpr int V1 = LPR >= 16 ? rs_half(V) : V, V2 = rs_half(V1), V3 = rs_half(V2), V4 = rs_half(V3);
  if constexpr (LPR >= 16) rs_halve<V>(y, lane & 8, [](float v) { return rs_dpp<0x140>(v); });    // row_mirror
  rs_halve<V1>(y, lane & 4, [](float v) { return rs_dpp<0x141>(v); });                            // row_half_mirror
  rs_halve<V2>(y, lane & 2, [](float v) { return rs_dpp<0x4E>(v); });                             // quad_perm [2,3,0,1]
  rs_halve<V3>(y, lane & 1, [](float v) { return rs_dpp<0xB1>(v); });                             // quad_perm [1,0,3,2]
  if constexpr (LPR >= 32) rs_halve<V4>(y, lane & 16, [](float v) { return __shfl_xor(v, 16, 64); });
  if constexpr (LPR >= 64) rs_halve<rs_half(V4)>(y, lane & 32, [](float v) { return __shfl_xor(v, 32, 64); });
}
template <int V, int LPR> __device__ __forceinline__ int rs_first(int c) {
  int v = V, at = 0;                        // the selecting bits in the order of the steps
#pragma unroll
  for (int bit = LPR >= 16 ? 8 : 4; bit; bit >>= 1)
    if (v > 1) { v /= 2; at += c & bit ? v : 0; }
  if (LPR >= 32 && v > 1) { v /= 2; at += c & 16 ? v : 0; }
  return at;
}
// Is c the first of the lanes that end with the same outputs?
template <int V, int LPR> __device__ __forceinline__ bool rs_stores(int c) {
  int v = V, twins = 0;
#pragma unroll
  for (int bit = LPR >= 16 ? 8 : 4; bit; bit >>= 1)
    if (v > 1) v /= 2; else twins |= bit;
  if (LPR >= 32) { if (v > 1) v /= 2; else twins |= 16; }
  if (LPR >= 64) twins |= 32;
  return (c & twins) == 0;
}

// LPR lanes share a row (piece c, c + LPR, ... of its K / 4 pieces); a wavefront works on
// U x (64 / LPR) rows per step, all loads of a step issued before the first is used.
// NN = N rounded up to a power of two; the weights sit in LDS as [K][NN] with zero padding.  (With more
// outputs the products and the per-row sums outweigh the loads and the matrix-core kernel wins.)
// Bound by reading A, 5.8 TB/s over two tables of 1e6 x 128.  The sums of a step's U x NN outputs are scattered over the
// lanes of a row and stored by one instruction; summed into every lane and stored an output at a time by the first lane of each row
// the same took 210 us instead of 183 with 4 outputs, 307 instead of 200 with 7, and 100,000 x 64 26 instead of 19 (with the
// join of 100,000 rows in each).
template <int LPR, int NN, int MOST>
__global__ __launch_bounds__(RS_THREADS) void gemm_rowsplit_kernel(GemmBatchOf<MOST> batch) {
  constexpr int RPW = 64 / LPR;             // rows per wavefront and sub-step
  constexpr int U = 4;                      // sub-steps in flight
  constexpr int V = U * NN, LEFT = V > LPR ? V / LPR : 1;
  extern __shared__ __align__(16) float Bs[];
  const int prob = problem_of(batch);
  const GemmArgs& g = batch.g[prob];
  const float* __restrict__ A = static_cast<const float*>(g.A);
  const float* __restrict__ B = static_cast<const float*>(g.B);
  for (int idx = threadIdx.x; idx < g.Kd * NN; idx += RS_THREADS) {
    const int k = idx / NN, n = idx - k * NN;
    Bs[idx] = n < g.N ? B[static_cast<int64_t>(k) * g.ldb + n] : 0.f;
  }
  __syncthreads();
  const int lane = threadIdx.x & 63, c = lane % LPR, sub = lane / LPR;
  const int ppr = g.Kd / 4;                 // 16-byte pieces per row
  const int64_t wave = static_cast<int64_t>(blockIdx.x - batch.first_tile[prob]) * (RS_THREADS / 64) + (threadIdx.x >> 6);
  const int64_t nwaves = static_cast<int64_t>(batch.first_tile[prob + 1] - batch.first_tile[prob]) * (RS_THREADS / 64);
  const int64_t nsteps = (g.M + RPW * U - 1) / (RPW * U);
  const int first = rs_first<V, LPR>(c);    // this lane's outputs of a step: sub-step first / NN, column first % NN and on
  float bv[LEFT];
#pragma unroll
  for (int i = 0; i < LEFT; ++i) bv[i] = (g.bias && first % NN + i < g.N) ? static_cast<const float*>(g.bias)[first % NN + i] : 0.f;

  for (int64_t step = wave; step < nsteps; step += nwaves) {
    float acc[V];
#pragma unroll
    for (int i = 0; i < V; ++i) acc[i] = 0.f;
    for (int p = c; p < ppr; p += LPR) {
      v4f a[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int64_t row = (step * U + u) * RPW + sub;
        a[u] = v4f{0.f, 0.f, 0.f, 0.f};
        if (row < g.M) a[u] = __builtin_nontemporal_load(reinterpret_cast<const v4f*>(A + row * g.lda) + p);
      }
      v4f w[NN];                              // the piece's four rows of B
#pragma unroll
      for (int q = 0; q < NN; ++q) w[q] = *reinterpret_cast<const v4f*>(Bs + 4 * (p * NN + q));
#pragma unroll
      for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int u = 0; u < U; ++u)
#pragma unroll
          for (int n = 0; n < NN; ++n) acc[u * NN + n] = fmaf(a[u][t], w[(t * NN + n) / 4][(t * NN + n) % 4], acc[u * NN + n]);
    }
    rs_reduce<V, LPR>(acc, lane);
    const int64_t row = (step * U + first / NN) * RPW + sub;
    if (row < g.M && rs_stores<V, LPR>(c)) {
      float* cr = static_cast<float*>(g.C) + row * g.ldc + first % NN;
#pragma unroll
      for (int i = 0; i < LEFT; ++i)
        if (first % NN + i < g.N) {
          float x = acc[i] + bv[i];
          if (g.relu) x = fmaxf(x, 0.f);
          cr[i] = x;
        }
    }
  }
}

// The lanes a row is split over, or 0 when the kernel does not cover the shape.  The choice depends on N, K, the row
// stride and the alignment only, never on M, so a row computed alone equals the same row computed
// as part of the whole table.
int rowsplit_lanes(const GemmArgs& g) {
  if (g.N > 8 || g.Kd < 32 || g.Kd % 4 || g.lda % 4 || !aligned(g.A, 16) || !aligned(g.C, 4)) return 0;
  if (static_cast<size_t>(g.Kd) * 8 * sizeof(float) > 64 * 1024) return 0;
  const int ppr = g.Kd / 4;
  return ppr <= 8 ? 8 : ppr <= 16 ? 16 : ppr <= 32 ? 32 : 64;
}

// All problems of the batch have the same number of columns and lanes a row.
template <int LPR>
int launch_rowsplit_batch(GemmBatch& b, hipStream_t s) {
  const int N = b.g[0].N, nn = N <= 2 ? N : N <= 4 ? 4 : 8;
  size_t lds = 0;
  const int rows_per_step = (64 / LPR) * 4;
  int64_t blocks = 0;
  for (int p = 0; p < b.count; ++p) {
    const GemmArgs& g = b.g[p];
    lds = std::max(lds, static_cast<size_t>(g.Kd) * nn * sizeof(float));
    b.first_tile[p] = static_cast<int32_t>(blocks);
    blocks += std::min<int64_t>(((g.M + rows_per_step - 1) / rows_per_step + 3) / 4, static_cast<int64_t>(num_cus()) * 16);
  }
  b.first_tile[b.count] = static_cast<int32_t>(blocks);
  const dim3 grid(static_cast<unsigned>(blocks)), block(RS_THREADS);
#define LQ_ROWSPLIT(NN_)                                                                                          \
  do {                                                                                                           \
    if (b.count == 1) hipLaunchKernelGGL((gemm_rowsplit_kernel<LPR, NN_, 1>), grid, block, lds, s, only_problem(b)); \
    else hipLaunchKernelGGL((gemm_rowsplit_kernel<LPR, NN_, LQ_MAX_DIMS>), grid, block, lds, s, b);              \
  } while (0)
  if (nn == 1) LQ_ROWSPLIT(1); else if (nn == 2) LQ_ROWSPLIT(2); else if (nn == 4) LQ_ROWSPLIT(4); else LQ_ROWSPLIT(8);
#undef LQ_ROWSPLIT
  LQ_LAUNCH_CHECK("gemm_rowsplit_kernel");
  return LQ_OK;
}
int launch_rowsplit(int lanes, GemmBatch& b, hipStream_t s) {
  switch (lanes) {
    case 8: return launch_rowsplit_batch<8>(b, s);
    case 16: return launch_rowsplit_batch<16>(b, s);
    case 32: return launch_rowsplit_batch<32>(b, s);
    default: return launch_rowsplit_batch<64>(b, s);
  }
}

}  // namespace

// C[M x N] = act(A[M x Kd] * B[Kd x N] + bias).  A, B, bias share `in_dtype`.
int launch_gemm(const void* A, int64_t lda, const void* B, int64_t ldb, void* C, int64_t ldc,
                const void* bias, int64_t M, int32_t N, int32_t Kd, int relu, int32_t in_dtype,
                int32_t out_dtype, hipStream_t s) {
  GemmArgs g{};
  g.A = A; g.lda = lda; g.B = B; g.ldb = ldb; g.C = C; g.ldc = ldc; g.bias = bias;
  g.M = M; g.N = N; g.Kd = Kd; g.relu = relu;
  if (in_dtype == LQ_F32 && out_dtype == LQ_F32) {
    const int lanes = M > 0 && N > 0 ? rowsplit_lanes(g) : 0;
    if (lanes) {
      GemmBatch b{};
      b.g[0] = g;
      b.count = 1;
      return launch_rowsplit(lanes, b, s);
    }
    return launch_typed<float, float>(g, s);
  }
  if (in_dtype == LQ_BF16 && out_dtype == LQ_F32) return launch_typed<bf16_t, float>(g, s);
  if (in_dtype == LQ_BF16 && out_dtype == LQ_BF16) return launch_typed<bf16_t, bf16_t>(g, s);
  return fail(LQ_ERR_DTYPE, "gemm: f32 inputs cannot produce a bf16 result");
}

int launch_project_dims(const lq_mat& D, const lq_mat& W, int32_t row_off, const lq_mat& P, hipStream_t s);

// P_k = D_k W[off_k .. off_k + c_k) for all K dimensions: one launch for all tables that the same kernel serves (a launch
// on a small table is 2 to 3 us whatever it does).
int launch_project_dims_all(int32_t K, const lq_mat* D, const lq_mat& W, int32_t first_off, const lq_mat* P,
                            hipStream_t s) {
  const size_t es = dtype_size(W.dtype);
  bool same_types = K > 1;
  for (int k = 0; k < K; ++k) same_types = same_types && D[k].dtype == D[0].dtype && P[k].dtype == P[0].dtype;
  if (!same_types) {
    int32_t off = first_off;
    for (int k = 0; k < K; ++k) {
      const int rc = launch_project_dims(D[k], W, off, P[k], s);
      if (rc) return rc;
      off += D[k].cols;
    }
    return LQ_OK;
  }
  const int32_t in = D[0].dtype, out = P[0].dtype;
  GemmBatch all{};
  int32_t off = first_off;
  for (int k = 0; k < K; ++k) {
    GemmArgs& g = all.g[all.count];
    g.A = D[k].data; g.lda = D[k].ld;
    g.B = static_cast<const char*>(W.data) + static_cast<size_t>(off) * W.ld * es; g.ldb = W.ld;
    g.C = P[k].data; g.ldc = P[k].ld;
    g.M = D[k].rows; g.N = W.cols; g.Kd = D[k].cols;
    off += D[k].cols;
    if (g.M > 0) ++all.count;
  }
  if (all.count == 0 || W.cols < 1) return LQ_OK;
  const bool f32 = in == LQ_F32 && out == LQ_F32, mixed = in == LQ_BF16 && out == LQ_F32, bf16 = in == LQ_BF16 && out == LQ_BF16;
  if (!f32 && !mixed && !bf16) return fail(LQ_ERR_DTYPE, "gemm: f32 inputs cannot produce a bf16 result");
  if (W.cols <= 16) {
    int lanes[LQ_MAX_DIMS];
    for (int p = 0; p < all.count; ++p) lanes[p] = f32 ? rowsplit_lanes(all.g[p]) : 0;
    for (const int l : {0, 8, 16, 32, 64}) {
      GemmBatch b{};
      for (int p = 0; p < all.count; ++p)
        if (lanes[p] == l) b.g[b.count++] = all.g[p];
      if (b.count == 0) continue;
      const int rc = l ? launch_rowsplit(l, b, s) : f32 ? launch_skinny_batch<float, float>(b, s)
                     : mixed ? launch_skinny_batch<bf16_t, float>(b, s) : launch_skinny_batch<bf16_t, bf16_t>(b, s);
      if (rc) return rc;
    }
    return LQ_OK;
  }
  if (f32) return launch_wide_f32(all, s);
  if (mixed) return launch_tiled_batch<bf16_t, float>(all, s);
  return launch_tiled_batch<bf16_t, bf16_t>(all, s);
}

int launch_project_dims(const lq_mat& D, const lq_mat& W, int32_t row_off, const lq_mat& P,
                        hipStream_t s) {
  const size_t es = dtype_size(W.dtype);
  const void* Wk = static_cast<const char*>(W.data) + static_cast<size_t>(row_off) * W.ld * es;
  return launch_gemm(D.data, D.ld, Wk, W.ld, P.data, P.ld, nullptr, D.rows, W.cols, D.cols, 0,
                     D.dtype, P.dtype, s);
}

}  // namespace lq
