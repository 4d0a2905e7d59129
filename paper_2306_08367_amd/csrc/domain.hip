// Group discovery (Sections 2.4.1-2.4.2) and ordering of an aggregate's result (Section 2.5).
//
// The paper finds the groups of a table with a numerical unique (one attribute) or with a
// sort-unique over tuples (several attributes), i.e. by sorting every row.  Grouping attributes of
// a star schema have few distinct values next to the number of rows (the group-by keeps at most
// 65,535 per dimension), so the rows are not sorted here: they are deduplicated through an
// open-addressing hash set whose slots name a representative row, and only the distinct tuples are
// ordered (rank = number of smaller distinct tuples, tiles of them staged in LDS).  A row's code is
// the rank of its tuple, so codes number the distinct tuples in ascending lexicographic order, as
// the sorted domain of the paper does; a dense group-by result indexed by such codes is therefore
// already ordered by the grouping attributes (the way Section 2.5 folds sorting into the matrix
// form).  Ordering by an aggregate (ORDER BY revenue DESC) counts, for each of the at most 8,192 groups,
// the groups that come before it.
#include "lq_common.h"

namespace lq {
namespace {

constexpr int MAX_COLS = 4;
constexpr int32_t MAX_DISTINCT = 65535;
constexpr size_t HEADER = 256;            // [0] number of distinct tuples (u32)

struct Cols {
  const int32_t* c[MAX_COLS];
  int32_t n_cols;
};

__device__ __forceinline__ uint32_t hash_row(const Cols& t, int64_t i, uint32_t shift) {
  uint32_t h = 0x811C9DC5u;
  for (int q = 0; q < t.n_cols; ++q) {
    h ^= static_cast<uint32_t>(t.c[q][i]);
    h *= 0x9E3779B1u;
    h ^= h >> 15;
  }
  return (h * 0x85EBCA6Bu) >> shift;
}
__device__ __forceinline__ bool same_tuple(const Cols& t, int64_t i, int64_t j) {
  bool eq = true;
  for (int q = 0; q < t.n_cols; ++q) eq = eq && t.c[q][i] == t.c[q][j];
  return eq;
}

__global__ __launch_bounds__(256) void domain_clear_kernel(int32_t* slots, uint32_t capacity, uint32_t* header) {
  const uint32_t i = blockIdx.x * 256u + threadIdx.x;
  if (i < capacity) slots[i] = -1;
  if (i == 0) header[0] = 0u;
}

// Every row either finds a slot whose representative row holds the same tuple or claims an empty
// slot for itself.  Claimed slots are listed in `reps` (the first MAX_DISTINCT + 1 of them).
__global__ __launch_bounds__(256) void domain_insert_kernel(Cols t, int64_t first, int64_t rows, int32_t* slots,
                                                            uint32_t mask, uint32_t shift, uint32_t* header,
                                                            uint32_t* reps) {
  const int64_t i = first + static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= rows) return;
  uint32_t s = hash_row(t, i, shift) & mask;
  for (uint32_t probes = 0; probes <= mask; ++probes) {           // bounded: at most one sweep of the table
    int32_t v = slots[s];
    if (v < 0) {
      v = atomicCAS(&slots[s], -1, static_cast<int32_t>(i));
      if (v < 0) {
        const uint32_t idx = atomicAdd(&header[0], 1u);
        if (idx <= static_cast<uint32_t>(MAX_DISTINCT)) reps[idx] = s;
        return;
      }
    }
    if (same_tuple(t, i, v)) return;
    s = (s + 1) & mask;
  }
}

__device__ __forceinline__ bool tuple_less(const int32_t* a, const int32_t* b, int n_cols) {
  for (int q = 0; q < n_cols; ++q) {
    if (a[q] != b[q]) return a[q] < b[q];
  }
  return false;
}

// rank of distinct tuple t = number of distinct tuples below it; writes the sorted value table.
constexpr int RANK_THREADS = 256;
__global__ __launch_bounds__(RANK_THREADS) void domain_rank_kernel(Cols t, int32_t d, const int32_t* __restrict__ slots,
                                                                  const uint32_t* __restrict__ reps,
                                                                  int32_t* __restrict__ slot_rank,
                                                                  int32_t* __restrict__ values) {
  __shared__ int32_t tile[RANK_THREADS][MAX_COLS];
  const int me = blockIdx.x * RANK_THREADS + threadIdx.x;
  int32_t mine[MAX_COLS] = {0, 0, 0, 0};
  if (me < d) {
    const int64_t row = slots[reps[me]];
    for (int q = 0; q < t.n_cols; ++q) mine[q] = t.c[q][row];
  }
  int rank = 0;
  for (int base = 0; base < d; base += RANK_THREADS) {
    const int j = base + threadIdx.x;
    if (j < d) {
      const int64_t row = slots[reps[j]];
      for (int q = 0; q < t.n_cols; ++q) tile[threadIdx.x][q] = t.c[q][row];
    }
    __syncthreads();
    const int cnt = min(RANK_THREADS, d - base);
    for (int u = 0; u < cnt; ++u) rank += tuple_less(tile[u], mine, t.n_cols) ? 1 : 0;
    __syncthreads();
  }
  if (me < d) {
    slot_rank[reps[me]] = rank;
    for (int q = 0; q < t.n_cols; ++q) values[static_cast<int64_t>(rank) * t.n_cols + q] = mine[q];
  }
}

__global__ __launch_bounds__(256) void domain_encode_kernel(Cols t, int64_t rows, const int32_t* __restrict__ slots,
                                                            uint32_t mask, uint32_t shift,
                                                            const int32_t* __restrict__ slot_rank,
                                                            int32_t* __restrict__ code) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= rows) return;
  uint32_t s = hash_row(t, i, shift) & mask;
  int32_t out = -1;
  for (uint32_t probes = 0; probes <= mask; ++probes) {           // bounded; every row was inserted, so it is found
    const int32_t v = slots[s];
    if (v < 0) break;
    if (same_tuple(t, i, v)) { out = slot_rank[s]; break; }
    s = (s + 1) & mask;
  }
  code[i] = out;
}

uint32_t domain_capacity(int64_t rows) {
  uint64_t c = 1024;
  while (c < 2 * static_cast<uint64_t>(rows)) c <<= 1;
  return static_cast<uint32_t>(c);
}

// ---- ordering of the populated groups -----------------------------------------------------------
// The place of a group in the result is the number of groups that come before it, so the order is counted, not sorted:
// every workgroup takes 32 groups, stages the keys of all groups in LDS, 1,024 at a time, and counts.  At most 8,192^2
// comparisons, spread over the whole chip in one launch without a workspace; a sort inside one workgroup's LDS leaves
// the other 255 compute units idle and pays a barrier for each of its 91 steps (a call in a graph, bitonic sort ->
// counted: 4,375 groups by a column and a sum 112 -> 14 us, 8,192 groups 111 -> 20, by four wide keys 117 -> 100).
// The keys are packed into one 64-bit number where they fit: each needs only the bits of its range over the
// populated groups (a year and a sum of a few billion: 3 + 33 bits), and 13 more for the group index make the
// numbers distinct; a comparison is then one of 64-bit numbers.  Keys of a wider range (more than 50 bits together)
// are compared one after the other.
constexpr int MAX_GROUPS = 8192;
constexpr int ORDER_THREADS = 1024;
constexpr int ORDER_TILE = 32;                              // groups placed by a workgroup
constexpr int INDEX_BITS = 13;

typedef unsigned long long u64;

struct OrderArgs {
  int32_t G;
  int32_t n_keys;
  int32_t kind[4], desc[4];
  uint32_t by_stride[4], by_card[4], card[4];   // a grouping column: ceil(2^32 / stride) and / card (g < 8,192: exact), card
  const long long* sums[4];                     // a SUM: its row
  const long long* counts;                      // [G]
};

__device__ __forceinline__ uint32_t divided(uint32_t g, uint32_t by) { return by ? __umulhi(g, by) : g; }   // by == 0: divisor 1

// Key q of group g, as an unsigned number in ascending order.
__device__ __forceinline__ u64 key_value(const OrderArgs& a, int q, int32_t g, long long count) {
  u64 u;
  if (a.kind[q] == LQ_KEY_GROUP_COLUMN) {
    const uint32_t v = divided(static_cast<uint32_t>(g), a.by_stride[q]);
    u = v - a.card[q] * divided(v, a.by_card[q]);
    return a.desc[q] ? a.card[q] - 1 - u : u;
  }
  u = static_cast<u64>(a.kind[q] == LQ_KEY_SUM ? a.sums[q][g] : count) ^ 0x8000000000000000ull;
  return a.desc[q] ? ~u : u;
}

// Few groups: one workgroup, keys compared one after the other by 16 threads a group (at least a wavefront, at most 1,024
// threads).  What such a call costs is the way from the arguments to the result, and the kernel below, with its range
// pass and its unrolled code, takes twice as long: 7 groups by one sum 7.0 -> 3.4 us, by four wide keys 20.8 -> 3.9, 64
// groups 7.1 -> 4.2 and 21.0 -> 5.6.  From 65 groups on the kernel below packs one or two keys in less time (128 groups by a
// column and a sum 6.9 us, here 8.0), with three or four keys from 129 on (128 groups by four 11.2 here, 175 groups 33
// against 15 there).
constexpr int SMALL_GROUPS = 128;
__global__ __launch_bounds__(ORDER_THREADS) void order_few_groups_kernel(OrderArgs a, int log2_g /*of the next power of two*/,
                                                                         int32_t* __restrict__ order, int32_t* __restrict__ n_out) {
  __shared__ u64 key[4][SMALL_GROUPS];
  __shared__ int32_t state[SMALL_GROUPS], before[SMALL_GROUPS];       // state: 0 populated, 1 not, 2 past the last group
  const int tid = threadIdx.x, size = 1 << log2_g;
  int populated = 0;
  if (tid < size) {
    const long long c = tid < a.G ? a.counts[tid] : 0;
    populated = c > 0;
    state[tid] = tid >= a.G ? 2 : populated ? 0 : 1;
    before[tid] = 0;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < a.n_keys) key[q][tid] = populated ? key_value(a, q, tid, c) : 0;
  }
  const int total = __syncthreads_count(populated);
  const int g = tid & (size - 1), shares = blockDim.x >> log2_g;
  const int mine = state[g];
  u64 own[4];
#pragma unroll
  for (int q = 0; q < 4; ++q) own[q] = q < a.n_keys ? key[q][g] : 0;
  int count = 0;
  for (int j = tid >> log2_g; j < size; j += shares) {
    bool less = state[j] < mine, equal = state[j] == mine;
#pragma unroll
    for (int q = 0; q < 4; ++q)
      if (q < a.n_keys) {
        const u64 k = key[q][j];
        less = less || (equal && k < own[q]);
        equal = equal && k == own[q];
      }
    count += less || (equal && j < g) ? 1 : 0;
  }
  atomicAdd(&before[g], count);
  __syncthreads();
  if (tid < a.G) order[before[tid]] = populated ? tid : -1;
  if (tid == 0) *n_out = total;
}

template <int NK>
__global__ __launch_bounds__(ORDER_THREADS) void order_groups_kernel(OrderArgs a, int32_t* __restrict__ order,
                                                                     int32_t* __restrict__ n_out) {
  __shared__ __align__(16) u64 tile[NK][ORDER_THREADS];
  __shared__ int32_t tile_state[ORDER_THREADS];             // 0 populated, 1 not, 2 past the last group
  __shared__ u64 lo_of[NK][ORDER_THREADS / 64], hi_of[NK][ORDER_THREADS / 64];
  __shared__ int mine_of[ORDER_THREADS / 64];
  __shared__ int before[ORDER_TILE];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  if (tid < ORDER_TILE) before[tid] = 0;
  // range of the keys over the populated groups (known beforehand for grouping columns)
  u64 lo[NK], hi[NK];
  int mine = 0;
  auto ranged = [&](int q) { return q < a.n_keys && a.kind[q] != LQ_KEY_GROUP_COLUMN; };
#pragma unroll
  for (int q = 0; q < NK; ++q) { lo[q] = ~0ull; hi[q] = 0; }
#pragma unroll NK == 4 ? 1 : 2
  for (int g = tid; g < a.G; g += ORDER_THREADS) {
    const long long c = a.counts[g];
#pragma unroll
    for (int q = 0; q < NK; ++q)
      if (ranged(q)) {
        const u64 k = key_value(a, q, g, c);
        if (c > 0) { lo[q] = min(lo[q], k); hi[q] = max(hi[q], k); }
      }
    mine += c > 0 ? 1 : 0;
  }
  // the group this thread counts for (32 groups times 32 shares of the comparisons)
  const int gi = blockIdx.x * ORDER_TILE + (tid & (ORDER_TILE - 1)), share = tid / ORDER_TILE;
  const long long ci = gi < a.G ? a.counts[gi] : 0;
  const int si = gi >= a.G ? 2 : ci > 0 ? 0 : 1;
  u64 own[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q) own[q] = (q < a.n_keys && si == 0) ? key_value(a, q, gi, ci) : 0;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) mine += __shfl_xor(mine, off, 64);
  if (lane == 0) mine_of[wave] = mine;
#pragma unroll
  for (int q = 0; q < NK; ++q)
    if (ranged(q)) {
      for (int off = 32; off > 0; off >>= 1) {
        lo[q] = min(lo[q], static_cast<u64>(__shfl_xor(static_cast<long long>(lo[q]), off, 64)));
        hi[q] = max(hi[q], static_cast<u64>(__shfl_xor(static_cast<long long>(hi[q]), off, 64)));
      }
      if (lane == 0) { lo_of[q][wave] = lo[q]; hi_of[q][wave] = hi[q]; }
    }
  __syncthreads();
  int bits = INDEX_BITS, width[NK];
#pragma unroll
  for (int q = 0; q < NK; ++q) {
    if (ranged(q)) {
      for (int w = 0; w < ORDER_THREADS / 64; ++w) { lo[q] = min(lo[q], lo_of[q][w]); hi[q] = max(hi[q], hi_of[q][w]); }
    } else {
      lo[q] = 0;
      hi[q] = q < a.n_keys ? a.card[q] - 1 : 0;
    }
    width[q] = hi[q] > lo[q] ? 64 - __clzll(static_cast<long long>(hi[q] - lo[q])) : 0;
    bits += width[q];
  }
  int count = 0;
  const bool packed = bits <= 63;                           // (the same for every thread)
  auto pack = [&](const u64 (&k)[NK], int st, int g) {
    if (st != 0) return st == 1 ? (0x8000000000000000ull | static_cast<u64>(g)) : ~0ull;
    u64 v = 0;
#pragma unroll
    for (int q = 0; q < NK; ++q) v = width[q] ? (v << width[q]) | (k[q] - lo[q]) : v;
    return (v << INDEX_BITS) | static_cast<u64>(g);
  };
  const u64 mykey = packed ? pack(own, si, gi) : 0;
  for (int t = 0; t < a.G; t += ORDER_THREADS) {
    const int g = t + tid;
    const long long c = g < a.G ? a.counts[g] : 0;
    const int st = g >= a.G ? 2 : c > 0 ? 0 : 1;
    u64 k[NK];
#pragma unroll
    for (int q = 0; q < NK; ++q) k[q] = (q < a.n_keys && st == 0) ? key_value(a, q, g, c) : 0;
    __syncthreads();
    if (packed) {
      tile[0][tid] = pack(k, st, g);
    } else {
#pragma unroll
      for (int q = 0; q < NK; ++q) tile[q][tid] = k[q];
      tile_state[tid] = st;
    }
    __syncthreads();
    if (packed) {
#pragma unroll
      for (int u = 0; u < ORDER_THREADS / 64; ++u) {        // the two shares of a wavefront read neighbouring pieces
        const ulonglong2 two = *reinterpret_cast<const ulonglong2*>(&tile[0][u * 64 + 2 * share]);
        count += (two.x < mykey ? 1 : 0) + (two.y < mykey ? 1 : 0);
      }
    } else {
      const int pieces = min(ORDER_THREADS, a.G - t + ORDER_TILE - 1) / ORDER_TILE;      // past the last group nothing counts
      for (int u = 0; u < pieces; ++u) {
        const int j = u * ORDER_TILE + share;
        bool less = tile_state[j] < si, equal = tile_state[j] == si;
#pragma unroll
        for (int q = 0; q < NK; ++q) {
          const u64 kj = tile[q][j];
          less = less || (equal && kj < own[q]);
          equal = equal && kj == own[q];
        }
        count += (less || (equal && t + j < gi)) ? 1 : 0;
      }
    }
  }
  count += __shfl_xor(count, ORDER_TILE, 64);
  if (lane < ORDER_TILE) atomicAdd(&before[lane], count);
  __syncthreads();
  if (tid < ORDER_TILE && gi < a.G) order[before[tid]] = si == 0 ? gi : -1;
  if (blockIdx.x == 0 && tid == 0) {
    int populated = 0;
    for (int w = 0; w < ORDER_THREADS / 64; ++w) populated += mine_of[w];
    *n_out = populated;
  }
}

}  // namespace
}  // namespace lq

using namespace lq;

extern "C" {

size_t lq_group_domain_workspace_bytes(int64_t rows) {
  if (rows < 0 || rows > 0x3fffffffLL) return 0;
  const size_t cap = domain_capacity(rows);
  return HEADER + 2 * cap * sizeof(int32_t) + round_up((static_cast<size_t>(MAX_DISTINCT) + 1) * sizeof(uint32_t), 256);
}

int lq_group_domain(int64_t rows, int32_t n_cols, const int32_t* const* cols, int32_t max_card, int32_t* code,
                    int32_t* values, int32_t* card, void* ws, size_t ws_bytes, void* hip_stream) {
  clear_error();
  if (rows < 0 || rows > 0x3fffffffLL) return fail(LQ_ERR_SHAPE, "rows out of range");
  if (n_cols < 1 || n_cols > MAX_COLS) return fail(LQ_ERR_SHAPE, "n_cols %d outside 1..%d", n_cols, MAX_COLS);
  if (max_card < 1 || max_card > MAX_DISTINCT) return fail(LQ_ERR_SHAPE, "max_card %d outside 1..%d", max_card, MAX_DISTINCT);
  if (!cols || !card) return fail(LQ_ERR_NULL, "cols or card is NULL");
  if (rows > 0 && (!code || !values)) return fail(LQ_ERR_NULL, "code or values is NULL");
  Cols t{};
  t.n_cols = n_cols;
  for (int q = 0; q < n_cols; ++q) {
    if (rows > 0 && !cols[q]) return fail(LQ_ERR_NULL, "cols[%d] is NULL", q);
    if (!aligned(cols[q], 4)) return fail(LQ_ERR_SHAPE, "cols[%d] is not 4-byte aligned", q);
    t.c[q] = cols[q];
  }
  if (!aligned(code, 4) || !aligned(values, 4)) return fail(LQ_ERR_SHAPE, "code / values are not 4-byte aligned");
  const size_t need = lq_group_domain_workspace_bytes(rows);
  if (!ws || !aligned(ws, 256) || ws_bytes < need)
    return fail(LQ_ERR_WORKSPACE, "group discovery needs a 256-byte aligned workspace of %zu bytes", need);
  *card = 0;
  if (rows == 0) return LQ_OK;
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const uint32_t cap = domain_capacity(rows);
  uint32_t shift = 32;
  for (uint32_t c = cap; c > 1; c >>= 1) --shift;
  uint32_t* header = static_cast<uint32_t*>(ws);
  int32_t* slots = reinterpret_cast<int32_t*>(static_cast<uint8_t*>(ws) + HEADER);
  int32_t* slot_rank = slots + cap;
  uint32_t* reps = reinterpret_cast<uint32_t*>(slot_rank + cap);
  const unsigned row_blocks = static_cast<unsigned>((rows + 255) / 256);
  hipLaunchKernelGGL(domain_clear_kernel, dim3((cap + 255) / 256), dim3(256), 0, s, slots, cap, header);
  LQ_LAUNCH_CHECK("domain_clear_kernel");
  // A small first slice claims the slots of the frequent tuples, so that the bulk of the rows only reads
  // them: with few distinct tuples, half a million lanes racing for the same empty slots cost 20x more.
  const int64_t head = std::min<int64_t>(rows, 8192);
  hipLaunchKernelGGL(domain_insert_kernel, dim3(static_cast<unsigned>((head + 255) / 256)), dim3(256), 0, s, t,
                     static_cast<int64_t>(0), head, slots, cap - 1, shift, header, reps);
  LQ_LAUNCH_CHECK("domain_insert_kernel");
  if (rows > head) {
    hipLaunchKernelGGL(domain_insert_kernel, dim3(static_cast<unsigned>((rows - head + 255) / 256)), dim3(256), 0, s, t,
                       head, rows, slots, cap - 1, shift, header, reps);
    LQ_LAUNCH_CHECK("domain_insert_kernel");
  }
  uint32_t d = 0;
  LQ_HIP_TRY(hipMemcpyAsync(&d, header, sizeof(d), hipMemcpyDeviceToHost, s));
  LQ_HIP_TRY(hipStreamSynchronize(s));
  if (d > static_cast<uint32_t>(max_card))
    return fail(LQ_ERR_UNSUPPORTED, "more than max_card = %d distinct tuples", max_card);
  hipLaunchKernelGGL(domain_rank_kernel, dim3((d + RANK_THREADS - 1) / RANK_THREADS), dim3(RANK_THREADS), 0, s, t,
                     static_cast<int32_t>(d), slots, reps, slot_rank, values);
  LQ_LAUNCH_CHECK("domain_rank_kernel");
  hipLaunchKernelGGL(domain_encode_kernel, dim3(row_blocks), dim3(256), 0, s, t, rows, slots, cap - 1, shift, slot_rank, code);
  LQ_LAUNCH_CHECK("domain_encode_kernel");
  *card = static_cast<int32_t>(d);
  return LQ_OK;
}

int lq_order_groups(int32_t n_group_cols, const int32_t* group_card, int32_t n_measures, const int64_t* sums,
                    const int64_t* counts, int32_t n_keys, const lq_sort_key* keys, int32_t* order, int32_t* n_out,
                    void* hip_stream) {
  clear_error();
  if (n_group_cols < 0 || n_group_cols > LQ_MAX_DIMS) return fail(LQ_ERR_SHAPE, "n_group_cols %d outside 0..%d", n_group_cols, LQ_MAX_DIMS);
  if (n_keys < 0 || n_keys > 4) return fail(LQ_ERR_SHAPE, "n_keys %d outside 0..4", n_keys);
  if (n_measures < 0 || n_measures > LQ_MAX_MEASURES) return fail(LQ_ERR_SHAPE, "n_measures %d outside 0..%d", n_measures, LQ_MAX_MEASURES);
  if ((n_group_cols > 0 && !group_card) || !counts || !order || !n_out || (n_keys > 0 && !keys))
    return fail(LQ_ERR_NULL, "group_card, counts, order, n_out or keys is NULL");
  if (!aligned(counts, 8) || !aligned(sums, 8) || !aligned(order, 4) || !aligned(n_out, 4))
    return fail(LQ_ERR_SHAPE, "an array is misaligned");
  OrderArgs a{};
  int64_t G = 1;
  for (int k = 0; k < n_group_cols; ++k) {
    if (group_card[k] < 1) return fail(LQ_ERR_SHAPE, "group_card[%d] < 1", k);
    G *= group_card[k];
    if (G > MAX_GROUPS) return fail(LQ_ERR_UNSUPPORTED, "more than %d groups", MAX_GROUPS);
  }
  int32_t stride[LQ_MAX_DIMS];
  for (int k = n_group_cols - 1, below = 1; k >= 0; --k) { stride[k] = below; below *= group_card[k]; }
  auto reciprocal = [](int32_t d) { return d == 1 ? 0u : static_cast<uint32_t>(((1ull << 32) + d - 1) / d); };
  for (int q = 0; q < n_keys; ++q) {
    const lq_sort_key& key = keys[q];
    if (key.kind == LQ_KEY_GROUP_COLUMN) {
      if (key.index < 0 || key.index >= n_group_cols) return fail(LQ_ERR_SHAPE, "keys[%d]: no grouping column %d", q, key.index);
      a.by_stride[q] = reciprocal(stride[key.index]);
      a.by_card[q] = reciprocal(group_card[key.index]);
      a.card[q] = static_cast<uint32_t>(group_card[key.index]);
    } else if (key.kind == LQ_KEY_SUM) {
      if (key.index < 0 || key.index >= n_measures || !sums) return fail(LQ_ERR_SHAPE, "keys[%d]: no measure %d", q, key.index);
      a.sums[q] = reinterpret_cast<const long long*>(sums) + static_cast<int64_t>(key.index) * G;
    } else if (key.kind != LQ_KEY_COUNT) {
      return fail(LQ_ERR_SHAPE, "keys[%d].kind is unknown", q);
    }
    a.kind[q] = key.kind; a.desc[q] = key.descending ? 1 : 0;
  }
  a.G = static_cast<int32_t>(G);
  a.n_keys = n_keys;
  a.counts = reinterpret_cast<const long long*>(counts);
  const dim3 grid(static_cast<unsigned>((a.G + ORDER_TILE - 1) / ORDER_TILE)), threads(ORDER_THREADS);
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  if (a.G <= (n_keys <= 2 ? SMALL_GROUPS / 2 : SMALL_GROUPS)) {      // (the lines: see order_few_groups_kernel)
    int log2_g = 0;
    while ((1 << log2_g) < a.G) ++log2_g;
    const unsigned few = static_cast<unsigned>(std::max(64, std::min(ORDER_THREADS, 16 << log2_g)));
    hipLaunchKernelGGL(order_few_groups_kernel, dim3(1), dim3(few), 0, s, a, log2_g, order, n_out);
    LQ_LAUNCH_CHECK("order_few_groups_kernel");
    return LQ_OK;
  }
  if (n_keys <= 1) hipLaunchKernelGGL(order_groups_kernel<1>, grid, threads, 0, s, a, order, n_out);
  else if (n_keys == 2) hipLaunchKernelGGL(order_groups_kernel<2>, grid, threads, 0, s, a, order, n_out);
  else hipLaunchKernelGGL(order_groups_kernel<4>, grid, threads, 0, s, a, order, n_out);
  LQ_LAUNCH_CHECK("order_groups_kernel");
  return LQ_OK;
}

}  // extern "C"
