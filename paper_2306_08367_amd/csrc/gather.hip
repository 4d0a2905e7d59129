// Materialisation of the joined table (first line of Eq. 1, T = X_f M_f + sum_k I_k D_k M_k),
// foreign-key validation, and the plain stream-copy yardstick.
#include "lq_common.h"

namespace lq {
namespace {

struct MatArgs {
  int64_t row0, rows;
  const void* X; int64_t ldx; int32_t c_f;
  int32_t K;
  const void* D[LQ_MAX_DIMS]; int64_t ldd[LQ_MAX_DIMS]; int32_t c[LQ_MAX_DIMS];
  int32_t off[LQ_MAX_DIMS];          // first column of dimension k in T
  const int32_t* fk[LQ_MAX_DIMS];
  void* T; int64_t ldt; int32_t kw;  // joined width
};

// Any column counts and strides, one element a thread, columns fastest: for joins of so few rows that the kernel below
// leaves compute units idle and its way through LDS shows: 1,000 / 6,000 rows of 22 + 21 + 21 columns, with the layer behind
// the join, 9.9 / 10.1 us through the kernel below, 6.8 / 7.7 so (smaller workgroups there: 7.8 / 9.7).
template <typename E>
__global__ __launch_bounds__(256) void materialize_each_kernel(MatArgs a, uint32_t total, uint32_t magic /*ceil(2^32 / kw), kw > 1*/) {
  const uint32_t e = blockIdx.x * 256u + threadIdx.x, kw = static_cast<uint32_t>(a.kw);
  if (e >= total) return;
  uint32_t r = kw > 1 ? __umulhi(e, magic) : e;       // at most one too large (e < 2^31)
  r -= r * kw > e;
  const int32_t col = static_cast<int32_t>(e - r * kw);
  const int64_t row = a.row0 + r;
  E v;
  if (col < a.c_f) {
    v = static_cast<const E*>(a.X)[row * a.ldx + col];
  } else {
    const int32_t* fk = a.fk[0];
    const void* D = a.D[0];
    int64_t ld = a.ldd[0];
    int32_t off = a.off[0];
#pragma unroll
    for (int q = 1; q < LQ_MAX_DIMS; ++q)
      if (q < a.K && col >= a.off[q]) { fk = a.fk[q]; D = a.D[q]; ld = a.ldd[q]; off = a.off[q]; }
    v = static_cast<const E*>(D)[fk[row] * ld + (col - off)];
  }
  static_cast<E*>(a.T)[r * a.ldt + col] = v;
}

// The same for more rows.  A workgroup takes `rb` rows, columns fastest: the writes to T are coalesced and the
// reads of one dimension row are contiguous across lanes.  The row's keys and the segments (fact columns, dimension
// 0, ..) come from LDS and the row of an element from a 32-bit product; U elements of a thread are in flight, since
// what bounds the kernel is the latency of key, then element.
constexpr int MAT_ROWS = 256;
template <typename E>
__global__ __launch_bounds__(256) void materialize_kernel(MatArgs a, int rb, uint32_t magic /*ceil(2^32 / kw), kw > 1*/) {
  constexpr int U = 4;
  struct Segment { const E* base; int64_t ld; };      // base: where column 0 of the joined row would be
  __shared__ Segment seg[LQ_MAX_DIMS + 1];
  __shared__ int32_t key[LQ_MAX_DIMS + 1][MAT_ROWS];
  const int tid = threadIdx.x;
  const int64_t r0 = static_cast<int64_t>(blockIdx.x) * rb;
  const int n = static_cast<int>(min(static_cast<int64_t>(rb), a.rows - r0));
  if (tid == 0) {
    seg[0].base = static_cast<const E*>(a.X) + (a.c_f > 0 ? (a.row0 + r0) * a.ldx : 0);
    seg[0].ld = a.ldx;
  }
  for (int r = tid; r < n; r += 256) key[0][r] = r;
#pragma unroll
  for (int k = 0; k < LQ_MAX_DIMS; ++k) {
    if (k >= a.K) break;
    if (tid == 0) { seg[k + 1].base = static_cast<const E*>(a.D[k]); seg[k + 1].ld = a.ldd[k]; }
    if (tid < n) key[k + 1][tid] = a.fk[k][a.row0 + r0 + tid];
  }
  __syncthreads();
  E* T = static_cast<E*>(a.T) + r0 * a.ldt;
  const uint32_t kw = static_cast<uint32_t>(a.kw), total = static_cast<uint32_t>(n) * kw;
  for (uint32_t e0 = tid; e0 < total; e0 += 256 * U) {
    E v[U];
    int64_t at[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const uint32_t e = min(e0 + 256u * u, total - 1);
      uint32_t r = kw > 1 ? __umulhi(e, magic) : e;   // at most one too large (e < 2^31)
      r -= r * kw > e;
      const int32_t col = static_cast<int32_t>(e - r * kw);
      int k = 0, off = 0;
#pragma unroll
      for (int q = 0; q < LQ_MAX_DIMS; ++q)
        if (q < a.K && col >= a.off[q]) { k = q + 1; off = a.off[q]; }
      v[u] = seg[k].base[key[k][r] * seg[k].ld + (col - off)];
      at[u] = static_cast<int64_t>(r) * a.ldt + col;
    }
#pragma unroll
    for (int u = 0; u < U; ++u)
      if (e0 + 256u * u < total) T[at[u]] = v[u];
  }
}

// 16-byte version: every segment of the joined row (fact columns, each dimension's columns) is a
// whole number of 16-byte chunks and every row start is 16-byte aligned.  A group of GROUP lanes
// copies one joined row, chunk by chunk; a dimension row is read as one contiguous run.
template <int GROUP>
__global__ __launch_bounds__(256) void materialize_vec_kernel(MatArgs a, int vec /*elements per chunk*/,
                                                              int chunks_per_row) {
  const int sub = threadIdx.x / GROUP, c0 = threadIdx.x % GROUP;
  constexpr int ROWS_PER_BLOCK = 256 / GROUP;
  const size_t es = 16 / vec;
  for (int64_t r = static_cast<int64_t>(blockIdx.x) * ROWS_PER_BLOCK + sub; r < a.rows;
       r += static_cast<int64_t>(gridDim.x) * ROWS_PER_BLOCK) {
    const int64_t row = a.row0 + r;
    for (int ch = c0; ch < chunks_per_row; ch += GROUP) {
      const int col = ch * vec;
      const char* src;
      if (col < a.c_f) {
        src = static_cast<const char*>(a.X) + (row * a.ldx + col) * es;
      } else {
        int k = 0;
#pragma unroll
        for (int q = 1; q < LQ_MAX_DIMS; ++q)
          if (q < a.K && col >= a.off[q]) k = q;
        const int64_t j = a.fk[k][row];
        src = static_cast<const char*>(a.D[k]) + (j * a.ldd[k] + (col - a.off[k])) * es;
      }
      const uint4 v = *reinterpret_cast<const uint4*>(src);
      *reinterpret_cast<uint4*>(static_cast<char*>(a.T) + (r * a.ldt + col) * es) = v;
    }
  }
}

struct CheckArgs {
  int64_t n; int32_t K;
  const int32_t* fk[LQ_MAX_DIMS];
  int64_t rows[LQ_MAX_DIMS];
  int negative_ok;
};

__global__ __launch_bounds__(256) void check_fks_kernel(CheckArgs a, int32_t* flag) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  int bad = 0;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; i < a.n; i += stride)
    for (int k = 0; k < a.K; ++k) {
      const int64_t j = a.fk[k][i];
      if (j >= a.rows[k] || (j < 0 && !a.negative_ok)) bad = 1;
    }
  if (bad) atomicOr(flag, 1);
}

// Group codes of the dimension side: bit 1 of the flag is raised for a code outside [0, card) on a
// dimension row whose mask lets it through (rows that are filtered out are never looked up).
struct CodeCheckArgs {
  int32_t K;
  const uint8_t* mask[LQ_MAX_DIMS];
  const int32_t* code[LQ_MAX_DIMS];
  int64_t rows[LQ_MAX_DIMS];
  int32_t card[LQ_MAX_DIMS];
};

__global__ __launch_bounds__(256) void check_codes_kernel(CodeCheckArgs a, int32_t* flag) {
  const int64_t stride = static_cast<int64_t>(gridDim.x) * blockDim.x;
  int bad = 0;
  for (int k = 0; k < a.K; ++k) {
    if (!a.code[k]) continue;
    for (int64_t j = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x; j < a.rows[k]; j += stride) {
      const int32_t v = a.code[k][j];
      if ((v < 0 || v >= a.card[k]) && (!a.mask[k] || a.mask[k][j])) bad = 1;
    }
  }
  if (bad) atomicOr(flag, 2);
}

__global__ __launch_bounds__(256) void zero_flag_kernel(int32_t* flag) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *flag = 0;
}

// One 16-byte element per thread: workgroups sweep memory in launch order, which keeps the
// set of open DRAM pages compact (measurably faster here than a grid-stride loop).
__global__ __launch_bounds__(256) void copy_kernel(uint4* __restrict__ dst,
                                                   const uint4* __restrict__ src, int64_t n16) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * blockDim.x + threadIdx.x;
  if (i < n16) dst[i] = src[i];
}

}  // namespace

int launch_materialize(const lq_star& star, void* T, int64_t ldt, int64_t row0, int64_t rows,
                       hipStream_t s) {
  MatArgs a{};
  a.row0 = row0; a.rows = rows;
  a.X = star.fact.data; a.ldx = star.fact.ld; a.c_f = star.fact.cols;
  a.K = star.n_dims;
  int32_t off = a.c_f;
  for (int k = 0; k < a.K; ++k) {
    a.D[k] = star.dims[k].data; a.ldd[k] = star.dims[k].ld; a.c[k] = star.dims[k].cols;
    a.off[k] = off; off += a.c[k];
    a.fk[k] = star.fks[k];
  }
  a.T = T; a.ldt = ldt; a.kw = off;
  const int64_t total = rows * off;
  if (total <= 0) return LQ_OK;
  {
    const int32_t dt0 = a.c_f > 0 ? star.fact.dtype : star.dims[0].dtype;
    const int vec = dt0 == LQ_BF16 ? 8 : 4;
    const size_t es = dtype_size(dt0);
    bool ok = aligned(T, 16) && ldt % vec == 0 && a.c_f % vec == 0 &&
              (a.c_f == 0 || (aligned(a.X, 16) && a.ldx % vec == 0));
    for (int k = 0; k < a.K && ok; ++k)
      ok = a.c[k] % vec == 0 && a.ldd[k] % vec == 0 && aligned(a.D[k], 16);
    (void)es;
    if (ok) {
      const int cpr = off / vec;
      int group = 1;
      while (group < cpr && group < 64) group <<= 1;
      const int rpb = 256 / group;
      const int64_t blocks = std::min<int64_t>((rows + rpb - 1) / rpb, 0x7fffffffLL);
      switch (group) {
#define LQ_MAT_CASE(G) case G: hipLaunchKernelGGL(materialize_vec_kernel<G>, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a, vec, cpr); break;
        LQ_MAT_CASE(1) LQ_MAT_CASE(2) LQ_MAT_CASE(4) LQ_MAT_CASE(8) LQ_MAT_CASE(16) LQ_MAT_CASE(32) LQ_MAT_CASE(64)
#undef LQ_MAT_CASE
      }
      LQ_LAUNCH_CHECK("materialize_vec_kernel");
      return LQ_OK;
    }
  }
  // Rows a workgroup: 64, of wide rows as many as make 4,096 elements, of rows of up to 5 columns 1,024 elements (64 of those
  // leave threads without work: 2,400,000 rows of 3 columns 109 us with 64 rows, 73 with 256).
  const int rb = off <= 5 ? std::min(MAT_ROWS, 1024 / off) : std::max(1, std::min(64, 4096 / off));
  const uint32_t magic = off > 1 ? static_cast<uint32_t>(((uint64_t{1} << 32) + off - 1) / off) : 0u;
  const int32_t dt = a.c_f > 0 ? star.fact.dtype : star.dims[0].dtype;
  // Few rows: one element a thread.  The lines lie where the two kernels meet (with the layer behind the join): 16, 64 and 100
  // columns between 20,000 rows (7.1 against 7.3 us, 11.1 / 11.9, 13.7 / 16.0) and 40,000 (8.8 / 8.2, 15.0 / 14.5, 22.1 / 22.4);
  // 3 and 5 columns at 200,000 (11.5 / 12.0, 12.6 / 13.0); 2,048 columns between 1,000 rows (21.7 / 24.4) and 6,000 (51.6 / 49.8).
  if (rows < int64_t{num_cus()} * (off <= 5 ? 768 : 96) && total < (1 << 23)) {
    const dim3 grid(static_cast<unsigned>((total + 255) / 256));
    if (dt == LQ_BF16) hipLaunchKernelGGL(materialize_each_kernel<uint16_t>, grid, dim3(256), 0, s, a, static_cast<uint32_t>(total), magic);
    else hipLaunchKernelGGL(materialize_each_kernel<float>, grid, dim3(256), 0, s, a, static_cast<uint32_t>(total), magic);
    LQ_LAUNCH_CHECK("materialize_each_kernel");
    return LQ_OK;
  }
  const int64_t most = int64_t{0x7fffff} * rb;  // rows of one grid (its threads stay below 2^32)
  for (; a.rows > 0; a.row0 += most, a.T = static_cast<char*>(a.T) + most * a.ldt * dtype_size(dt), a.rows -= most) {
    const dim3 grid(static_cast<unsigned>((std::min(a.rows, most) + rb - 1) / rb));
    if (dt == LQ_BF16) hipLaunchKernelGGL(materialize_kernel<uint16_t>, grid, dim3(256), 0, s, a, rb, magic);
    else hipLaunchKernelGGL(materialize_kernel<float>, grid, dim3(256), 0, s, a, rb, magic);
    LQ_LAUNCH_CHECK("materialize_kernel");
  }
  return LQ_OK;
}

int launch_check_fks(int64_t n, int32_t K, const int32_t* const* fks, const int64_t* rows,
                     bool negative_ok, int32_t* d_flag, hipStream_t s) {
  CheckArgs a{};
  a.n = n; a.K = K; a.negative_ok = negative_ok ? 1 : 0;
  for (int k = 0; k < K; ++k) { a.fk[k] = fks[k]; a.rows[k] = rows[k]; }
  hipLaunchKernelGGL(zero_flag_kernel, dim3(1), dim3(64), 0, s, d_flag);
  LQ_LAUNCH_CHECK("zero_flag_kernel");
  if (n > 0 && K > 0) {
    const int64_t blocks = std::min<int64_t>((n + 255) / 256, static_cast<int64_t>(num_cus()) * 8);
    hipLaunchKernelGGL(check_fks_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a, d_flag);
    LQ_LAUNCH_CHECK("check_fks_kernel");
  }
  return LQ_OK;
}

// Must follow launch_check_fks on the same stream (which clears the flag word).
int launch_check_codes(int32_t K, const int64_t* rows, const uint8_t* const* mask, const int32_t* const* code,
                       const int32_t* card, int32_t* d_flag, hipStream_t s) {
  CodeCheckArgs a{};
  a.K = K;
  int64_t most = 0;
  for (int k = 0; k < K; ++k) {
    a.mask[k] = mask ? mask[k] : nullptr;
    a.code[k] = code ? code[k] : nullptr;
    a.rows[k] = rows[k];
    a.card[k] = (code && code[k] && card) ? card[k] : 1;
    if (a.code[k]) most = std::max(most, rows[k]);
  }
  if (most == 0) return LQ_OK;
  const int64_t blocks = std::min<int64_t>((most + 255) / 256, static_cast<int64_t>(num_cus()) * 8);
  hipLaunchKernelGGL(check_codes_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, a, d_flag);
  LQ_LAUNCH_CHECK("check_codes_kernel");
  return LQ_OK;
}

int launch_copy(void* dst, const void* src, size_t bytes, hipStream_t s) {
  int64_t n16 = static_cast<int64_t>(bytes / 16);
  const uint4* sp = static_cast<const uint4*>(src);
  uint4* dp = static_cast<uint4*>(dst);
  const int64_t per_launch = static_cast<int64_t>(1) << 37 >> 4;   // 128 GiB per launch keeps the grid below 2^31
  while (n16 > 0) {
    const int64_t m = std::min<int64_t>(n16, per_launch);
    hipLaunchKernelGGL(copy_kernel, dim3(static_cast<unsigned>((m + 255) / 256)), dim3(256), 0, s, dp, sp, m);
    LQ_LAUNCH_CHECK("copy_kernel");
    sp += m; dp += m; n16 -= m;
  }
  return LQ_OK;
}

}  // namespace lq
