// Key -> row mapping for 64-bit key values: the same cached key domain as for 32-bit keys
// (Algorithm 1's domain generation), for tables whose keys do not fit an int32.
//
// Buffer: [256-byte header | capacity / 2 buckets of 24 bytes: two keys, their two row numbers].  Two
// forms, chosen when the map is built: direct, when largest - smallest key is below 2 x capacity (the
// buffer then holds 4-byte cells "row of key base + i, or -1"), else an open-addressing hash table
// (a slot is claimed with a compare-and-swap on its key; the row number is written into the same
// bucket, so that a lookup asks for keys and rows at once and, mostly, of one line).  The smallest
// int64 marks an empty slot and is therefore not a legal key.
#include "lq_common.h"

namespace lq {
namespace {

typedef unsigned long long u64;
typedef long long i64;
constexpr i64 EMPTY_KEY = static_cast<i64>(0x8000000000000000ull);
constexpr size_t HEADER = 256;
constexpr unsigned FLAG_DUPLICATE = 1u, FLAG_FULL = 2u, FLAG_WINDOW = 4u, FLAG_RESERVED = 8u;

struct Header64 {
  u64 capacity;
  unsigned flags;
  int32_t direct;
  i64 base;
  i64 min_key, max_key;      // of the keys given to the build
};

// The key is folded into one half, and that twice into itself, before the product.  One product alone lays evenly spaced
// keys out in a lattice: mostly an even one, but some spacings fill a few buckets over and over, and with a second product of
// the key as the distance to the next bucket the paths of such keys run into each other (400,000 keys 8 apart: map built in
// 30 ms, 3e6 lookups 13.2 ms; folded 46 and 48 us.  8,192 keys 101 apart, spread in LDS: 925 -> 17 and 630 -> 27 us.
// 2,500,000 scattered keys of 500 and 2,000 rows in LDS 2 % slower, of 4,096 rows 17.2 -> 13.3 us).  Over 48 spacings of 8 to
// 2^44 the longest path of 500 to 200,000 keys has 12 buckets, as with a 64-bit product between folds, which costs
// lookups in LDS up to a sixth.
__device__ __forceinline__ uint32_t mixed(i64 key) {
  uint32_t h = static_cast<uint32_t>(key) ^ static_cast<uint32_t>(key >> 32) * 0x85EBCA6Bu;
  h ^= h >> 9;
  return (h ^ (h >> 4)) * 0x9E3779B1u;
}
__device__ __forceinline__ uint32_t slot_of(i64 key, uint32_t shift) { return mixed(key) >> shift; }

// Distance to the next bucket on a key's path, in slots: an odd number of buckets that depends on the key (with a
// fixed distance full buckets grow into runs).
__device__ __forceinline__ uint32_t step_of(i64 key) {
  const uint32_t h = mixed(key);
  return 2u * (((h ^ (h >> 15)) * 0x85EBCA6Bu >> 8) | 1u);
}

// Slot s of the table: its bucket is s / 2.
__device__ __forceinline__ i64* key_at(char* buckets, uint32_t s) {
  return reinterpret_cast<i64*>(buckets + 24 * static_cast<size_t>(s >> 1) + 8 * (s & 1u));
}
__device__ __forceinline__ int32_t* row_at(char* buckets, uint32_t s) {
  return reinterpret_cast<int32_t*>(buckets + 24 * static_cast<size_t>(s >> 1) + 16 + 4 * (s & 1u));
}

__global__ void keymap64_init_kernel(Header64* header, u64 capacity) {
  header->capacity = capacity; header->flags = 0u; header->direct = 0; header->base = 0;
  header->min_key = 0x7fffffffffffffffll; header->max_key = EMPTY_KEY;
}

__global__ __launch_bounds__(256) void keymap64_minmax_kernel(const i64* __restrict__ keys, int64_t r, Header64* header) {
  i64 lo = 0x7fffffffffffffffll, hi = EMPTY_KEY;
  for (int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x; i < r; i += static_cast<int64_t>(gridDim.x) * 256) {
    const i64 k = keys[i];
    lo = min(lo, k); hi = max(hi, k);
  }
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, __shfl_xor(lo, off, 64));
    hi = max(hi, __shfl_xor(hi, off, 64));
  }
  __shared__ i64 wlo[4], whi[4];
  if ((threadIdx.x & 63) == 0) { wlo[threadIdx.x >> 6] = lo; whi[threadIdx.x >> 6] = hi; }
  __syncthreads();
  if (threadIdx.x == 0) {
    atomicMin(&header->min_key, min(min(wlo[0], wlo[1]), min(wlo[2], wlo[3])));
    atomicMax(&header->max_key, max(max(whi[0], whi[1]), max(whi[2], whi[3])));
  }
}

// Decides the form from the key range (every thread alike, the first one records it) and empties
// the buffer accordingly: cells of -1, or slots holding the empty key.  One thread per bucket.
__global__ __launch_bounds__(256) void keymap64_clear_kernel(char* buckets, u64 n_buckets, Header64* header) {
  const i64 lo = header->min_key, hi = header->max_key;
  const bool direct = hi >= lo && static_cast<u64>(hi) - static_cast<u64>(lo) < 4 * n_buckets;
  const u64 i = static_cast<u64>(blockIdx.x) * 256 + threadIdx.x;
  if (i < n_buckets) {
    i64* two = reinterpret_cast<i64*>(buckets + (direct ? 16 : 24) * i);
    two[0] = two[1] = direct ? -1ll : EMPTY_KEY;
  }
  if (i == 0) { header->direct = direct ? 1 : 0; header->base = direct ? lo : 0; }
}

__global__ __launch_bounds__(256) void keymap64_insert_kernel(char* buckets, uint32_t mask, uint32_t shift,
                                                              const i64* __restrict__ keys, int64_t r, int64_t row0,
                                                              Header64* header) {
  const int64_t i = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  if (i >= r) return;
  const i64 key = keys[i];
  if (header->direct) {
    const i64 base = header->base;
    const u64 cell = static_cast<u64>(key) - static_cast<u64>(base);
    if (key < base || cell >= 2 * (static_cast<u64>(mask) + 1)) { atomicOr(&header->flags, FLAG_WINDOW); return; }
    const int old = atomicCAS(reinterpret_cast<int*>(buckets) + cell, -1, static_cast<int>(row0 + i));
    if (old != -1) atomicOr(&header->flags, FLAG_DUPLICATE);
    atomicMax(&header->max_key, key);
    return;
  }
  if (key == EMPTY_KEY) { atomicOr(&header->flags, FLAG_RESERVED); return; }
  // first slot of the bucket, second slot, next bucket: a bucket's second slot is only taken when its first one is
  uint32_t s = slot_of(key, shift) & mask & ~1u;
  for (uint32_t probes = 0; probes <= mask; ++probes) {           // bounded: at most one sweep of the table
    const i64 old = static_cast<i64>(atomicCAS(reinterpret_cast<u64*>(key_at(buckets, s)), static_cast<u64>(EMPTY_KEY),
                                               static_cast<u64>(key)));
    if (old == EMPTY_KEY) { *row_at(buckets, s) = static_cast<int32_t>(row0 + i); return; }
    if (old == key) { atomicOr(&header->flags, FLAG_DUPLICATE); return; }
    s = (probes & 1) ? ((s & ~1u) + step_of(key)) & mask : s + 1;
  }
  atomicOr(&header->flags, FLAG_FULL);
}

typedef long long v2l __attribute__((ext_vector_type(2)));
typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v4i __attribute__((ext_vector_type(4)));
typedef v2l __attribute__((aligned(8))) v2l_a8;

struct Bucket { v2l key; v2i row; };

// Rows of N keys: all first probes together, then only the keys whose bucket is full of other keys (see keymap.hip).
// `at(slot)` fetches the bucket of an even slot.
template <int N, typename AT>
__device__ __forceinline__ void find64(AT&& at, uint32_t mask, uint32_t shift, const i64 (&key)[N], int32_t (&row)[N]) {
  uint32_t s[N];
  Bucket b[N];
  bool open = false, more[N];
#pragma unroll
  for (int q = 0; q < N; ++q) {
    s[q] = slot_of(key[q], shift) & mask & ~1u;
    b[q] = at(s[q]);
  }
  auto resolve = [&](int q) {
    const i64 k = key[q];
    const bool e0 = b[q].key[0] == k, e1 = b[q].key[1] == k, none = k == EMPTY_KEY;
    row[q] = none ? -1 : e0 ? b[q].row[0] : e1 ? b[q].row[1] : -1;
    more[q] = !e0 && !e1 && !none && b[q].key[1] != EMPTY_KEY;
    open = open || more[q];
  };
#pragma unroll
  for (int q = 0; q < N; ++q) resolve(q);
  for (uint32_t probes = 2; open && probes <= mask; probes += 2) {   // bounded: at most one sweep of the table
    open = false;
#pragma unroll
    for (int q = 0; q < N; ++q)
      if (more[q]) {
        s[q] = (s[q] + step_of(key[q])) & mask;
        b[q] = at(s[q]);
      }
#pragma unroll
    for (int q = 0; q < N; ++q)
      if (more[q]) resolve(q);
  }
}

template <int N>
__device__ __forceinline__ void find64_in_buffer(const char* buckets, bool direct, i64 base, uint32_t mask, uint32_t shift,
                                                 const i64 (&key)[N], int32_t (&row)[N]) {
  if (direct) {
    const int32_t* cells = reinterpret_cast<const int32_t*>(buckets);
    int32_t v[N];
    bool in[N];
#pragma unroll
    for (int q = 0; q < N; ++q) {
      const u64 cell = static_cast<u64>(key[q]) - static_cast<u64>(base);
      in[q] = key[q] >= base && cell < 2 * (static_cast<u64>(mask) + 1);
      v[q] = cells[in[q] ? cell : 0];
    }
#pragma unroll
    for (int q = 0; q < N; ++q) row[q] = in[q] ? v[q] : -1;
    return;
  }
  find64<N>([&](uint32_t s) {
    const char* p = buckets + 24 * static_cast<size_t>(s >> 1);
    return Bucket{*reinterpret_cast<const v2l_a8*>(p), *reinterpret_cast<const v2i*>(p + 16)};
  }, mask, shift, key, row);
}

// Two keys per thread (one 16-byte load) when the columns allow it; the odd last key one by one.  With four keys a thread
// direct maps past LDS took 4 to 12 % longer from 2.5e6 keys on (less than that up to 2^20), hashed ones 2 to 10 %.
__global__ __launch_bounds__(256) void keymap64_lookup_kernel(const Header64* __restrict__ header, const char* __restrict__ buckets,
                                                              uint32_t mask, uint32_t shift, const i64* __restrict__ keys,
                                                              int64_t n, int32_t* __restrict__ fk, int vec_ok) {
  const bool direct = header->direct != 0;
  const i64 base = header->base;
  const int64_t t = static_cast<int64_t>(blockIdx.x) * 256 + threadIdx.x;
  const int64_t n2 = vec_ok ? n / 2 : 0;
  if (t < n2) {
    const v2l a = __builtin_nontemporal_load(reinterpret_cast<const v2l*>(keys) + t);
    const i64 k[2] = {a[0], a[1]};
    int32_t r[2];
    find64_in_buffer<2>(buckets, direct, base, mask, shift, k, r);
    const v2i out = {r[0], r[1]};
    __builtin_nontemporal_store(out, reinterpret_cast<v2i*>(fk) + t);
  } else if (t - n2 < n - 2 * n2) {
    const int64_t i = 2 * n2 + (t - n2);
    const i64 k[1] = {keys[i]};
    int32_t r[1];
    find64_in_buffer<1>(buckets, direct, base, mask, shift, k, r);
    fk[i] = r[0];
  }
}

// Small maps, as in keymap.hip: every workgroup spreads the hash table over LDS64_SLOTS slots of LDS (SPREAD; a table of that
// many slots is copied as it is) or copies the cells of a direct map there, and serves a slice of the fact keys from
// it, four at a time, the first ones in flight meanwhile.
constexpr int LDS64_THREADS = 1024;
constexpr uint32_t LDS64_SLOTS = 8192;              // 96 KB; a direct map of as many slots has 64 KB of cells
template <bool SPREAD>
__global__ __launch_bounds__(LDS64_THREADS) void keymap64_lookup_lds_kernel(const Header64* __restrict__ header,
                                                                            const char* __restrict__ buckets, uint32_t slots,
                                                                            uint32_t lds_shift, const i64* __restrict__ keys,
                                                                            int64_t n, int32_t* __restrict__ fk,
                                                                            int64_t per_block) {
  extern __shared__ __align__(16) i64 lds64[];
  i64* lkey = lds64;                                                 // [LDS64_SLOTS]
  int32_t* lrow = reinterpret_cast<int32_t*>(lds64 + LDS64_SLOTS);   // [LDS64_SLOTS]
  const int64_t n4 = n / 4;
  const int64_t lo = static_cast<int64_t>(blockIdx.x) * per_block, hi = min(n4, lo + per_block);
  const v2l* kp = reinterpret_cast<const v2l*>(keys);
  int64_t t = lo + threadIdx.x;
  v2l ka = {0, 0}, kb = {0, 0};
  if (t < hi) { ka = __builtin_nontemporal_load(kp + 2 * t); kb = __builtin_nontemporal_load(kp + 2 * t + 1); }
  const bool direct = header->direct != 0;
  const i64 base = header->base;
  const uint32_t mask = LDS64_SLOTS - 1;
  const uint32_t direct_mask = slots - 1;
  if (direct) {
    for (uint32_t i = threadIdx.x; i < slots; i += LDS64_THREADS) lkey[i] = reinterpret_cast<const i64*>(buckets)[i];   // two cells
  } else if constexpr (SPREAD) {
    for (uint32_t i = threadIdx.x; i < LDS64_SLOTS; i += LDS64_THREADS) lkey[i] = EMPTY_KEY;
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < slots; i += LDS64_THREADS) {
      const char* p = buckets + 24 * static_cast<size_t>(i >> 1);
      const i64 key = *reinterpret_cast<const i64*>(p + 8 * (i & 1u));
      if (key == EMPTY_KEY) continue;
      const int32_t row = *reinterpret_cast<const int32_t*>(p + 16 + 4 * (i & 1u));
      uint32_t s = slot_of(key, lds_shift) & mask & ~1u;
      for (uint32_t probes = 0; probes <= mask; ++probes) {          // (there is room: at most `slots` keys)
        if (atomicCAS(reinterpret_cast<u64*>(&lkey[s]), static_cast<u64>(EMPTY_KEY), static_cast<u64>(key)) ==
            static_cast<u64>(EMPTY_KEY)) {
          lrow[s] = row;
          break;
        }
        s = (probes & 1) ? ((s & ~1u) + step_of(key)) & mask : s + 1;
      }
    }
  } else {
    for (uint32_t i = threadIdx.x; i < LDS64_SLOTS / 2; i += LDS64_THREADS) {
      const char* p = buckets + 24 * static_cast<size_t>(i);
      *reinterpret_cast<v2l*>(&lkey[2 * i]) = *reinterpret_cast<const v2l_a8*>(p);
      *reinterpret_cast<v2i*>(&lrow[2 * i]) = *reinterpret_cast<const v2i*>(p + 16);
    }
  }
  __syncthreads();
  auto rows_of = [&](auto& k, auto& r) {
    constexpr int N = sizeof(k) / sizeof(i64);
    if (direct)
      find64_in_buffer<N>(reinterpret_cast<const char*>(lkey), true, base, direct_mask, 0, k, r);
    else
      find64<N>([&](uint32_t s) {
        return Bucket{*reinterpret_cast<const v2l*>(&lkey[s]), *reinterpret_cast<const v2i*>(&lrow[s])};
      }, mask, lds_shift, k, r);
  };
  while (t < hi) {
    const i64 k[4] = {ka[0], ka[1], kb[0], kb[1]};
    const int64_t next = t + LDS64_THREADS;
    if (next < hi) { ka = __builtin_nontemporal_load(kp + 2 * next); kb = __builtin_nontemporal_load(kp + 2 * next + 1); }
    int32_t r[4];
    rows_of(k, r);
    const v4i out = {r[0], r[1], r[2], r[3]};
    __builtin_nontemporal_store(out, reinterpret_cast<v4i*>(fk) + t);
    t = next;
  }
  if (blockIdx.x == 0) {
    const int64_t i = 4 * n4 + threadIdx.x;
    if (i < n) {
      const i64 k[1] = {keys[i]};
      int32_t r[1];
      rows_of(k, r);
      fk[i] = r[0];
    }
  }
}

struct Geometry64 { u64 capacity; uint32_t mask, shift; };
bool geometry64(size_t table_bytes, Geometry64* g) {
  if (table_bytes < HEADER + 2 * 12) return false;
  u64 cap = 2;
  while (HEADER + cap * 2 * 12 <= table_bytes && cap < (1ull << 31)) cap <<= 1;
  int log2 = 0;
  while ((1ull << log2) < cap) ++log2;
  g->capacity = cap; g->mask = static_cast<uint32_t>(cap - 1); g->shift = static_cast<uint32_t>(32 - log2);
  return true;
}

int check_flags64(const Header64* header, hipStream_t s) {
  unsigned h = 0;
  LQ_HIP_TRY(hipMemcpyAsync(&h, &header->flags, sizeof(h), hipMemcpyDeviceToHost, s));
  LQ_HIP_TRY(hipStreamSynchronize(s));
  if (h & FLAG_DUPLICATE) return fail(LQ_ERR_DUPLICATE_KEY, "the dimension key column holds a value twice");
  if (h & FLAG_FULL) return fail(LQ_ERR_WORKSPACE, "key map is full");
  if (h & FLAG_WINDOW) return fail(LQ_ERR_WORKSPACE, "a key lies outside the window of this direct-address map: rebuild the map with all keys");
  if (h & FLAG_RESERVED) return fail(LQ_ERR_UNSUPPORTED, "the smallest int64 is not a legal key");
  return LQ_OK;
}

}  // namespace
}  // namespace lq

using namespace lq;

extern "C" {

size_t lq_keymap64_bytes(int64_t max_keys) {
  if (max_keys < 0 || max_keys > (1ll << 29)) return 0;
  u64 cap = 2;
  while (cap < static_cast<u64>(max_keys) * 2) cap <<= 1;
  return HEADER + cap * 12;
}

int lq_keymap64_insert(void* table, size_t table_bytes, const int64_t* keys, int64_t n_keys, int64_t first_row,
                       uint32_t flags, void* hip_stream) {
  clear_error();
  Geometry64 g;
  if (!table || !aligned(table, 256) || !geometry64(table_bytes, &g)) return fail(LQ_ERR_WORKSPACE, "key map buffer is NULL, misaligned or too small");
  if (n_keys < 0 || first_row < 0 || first_row + n_keys > 0x7fffffffLL) return fail(LQ_ERR_SHAPE, "row numbers do not fit int32");
  if (n_keys > 0 && (!keys || !aligned(keys, 8))) return fail(LQ_ERR_NULL, "keys is NULL or misaligned");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  Header64* header = static_cast<Header64*>(table);
  char* buckets = static_cast<char*>(table) + HEADER;
  if (n_keys > 0) {
    hipLaunchKernelGGL(keymap64_insert_kernel, dim3(static_cast<unsigned>((n_keys + 255) / 256)), dim3(256), 0, s,
                       buckets, g.mask, g.shift, reinterpret_cast<const i64*>(keys), n_keys, first_row, header);
    LQ_LAUNCH_CHECK("keymap64_insert_kernel");
  }
  if (flags & LQ_CHECK_KEYS) return check_flags64(header, s);
  return LQ_OK;
}

int lq_keymap64_build(void* table, size_t table_bytes, const int64_t* keys, int64_t n_keys, uint32_t flags,
                      void* hip_stream) {
  clear_error();
  Geometry64 g;
  if (!table || !aligned(table, 256) || !geometry64(table_bytes, &g)) return fail(LQ_ERR_WORKSPACE, "key map buffer is NULL, misaligned or too small");
  if (n_keys < 0 || static_cast<u64>(n_keys) * 2 > g.capacity) return fail(LQ_ERR_WORKSPACE, "key map buffer holds %llu slots, %lld keys need twice as many", (unsigned long long)g.capacity, (long long)n_keys);
  if (n_keys > 0 && (!keys || !aligned(keys, 8))) return fail(LQ_ERR_NULL, "keys is NULL or misaligned");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  Header64* header = static_cast<Header64*>(table);
  char* buckets = static_cast<char*>(table) + HEADER;
  hipLaunchKernelGGL(keymap64_init_kernel, dim3(1), dim3(1), 0, s, header, g.capacity);
  LQ_LAUNCH_CHECK("keymap64_init_kernel");
  if (n_keys > 0) {
    const unsigned mm_blocks = static_cast<unsigned>(std::min<int64_t>((n_keys + 1023) / 1024, 256));
    hipLaunchKernelGGL(keymap64_minmax_kernel, dim3(mm_blocks), dim3(256), 0, s, reinterpret_cast<const i64*>(keys), n_keys, header);
    LQ_LAUNCH_CHECK("keymap64_minmax_kernel");
  }
  hipLaunchKernelGGL(keymap64_clear_kernel, dim3(static_cast<unsigned>((g.capacity / 2 + 255) / 256)), dim3(256), 0, s,
                     buckets, g.capacity / 2, header);
  LQ_LAUNCH_CHECK("keymap64_clear_kernel");
  return lq_keymap64_insert(table, table_bytes, keys, n_keys, 0, flags, hip_stream);
}

int lq_keymap64_lookup(const void* table, size_t table_bytes, const int64_t* fact_keys, int64_t n, int32_t* fk,
                       void* hip_stream) {
  clear_error();
  Geometry64 g;
  if (!table || !aligned(table, 256) || !geometry64(table_bytes, &g)) return fail(LQ_ERR_WORKSPACE, "key map buffer is NULL, misaligned or too small");
  if (n < 0) return fail(LQ_ERR_SHAPE, "n < 0");
  if (n == 0) return LQ_OK;
  if (!fact_keys || !fk || !aligned(fact_keys, 8) || !aligned(fk, 4)) return fail(LQ_ERR_NULL, "fact_keys or fk is NULL or misaligned");
  hipStream_t s = static_cast<hipStream_t>(hip_stream);
  const Header64* header = static_cast<const Header64*>(table);
  const char* buckets = static_cast<const char*>(table) + HEADER;
  if (aligned(fact_keys, 16) && aligned(fk, 16) && g.capacity <= LDS64_SLOTS && n >= (1 << 20)) {
    constexpr int lds_bytes = static_cast<int>(LDS64_SLOTS) * 12;
    const int64_t n4 = n / 4;
    const int64_t blocks = std::max<int64_t>(1, std::min<int64_t>((n4 + LDS64_THREADS - 1) / LDS64_THREADS, num_cus()));
    const auto kernel = g.capacity == LDS64_SLOTS ? keymap64_lookup_lds_kernel<false> : keymap64_lookup_lds_kernel<true>;
    LQ_HIP_TRY(hipFuncSetAttribute(reinterpret_cast<const void*>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes));
    hipLaunchKernelGGL(kernel, dim3(static_cast<unsigned>(blocks)), dim3(LDS64_THREADS), lds_bytes, s, header, buckets,
                       static_cast<uint32_t>(g.capacity), 32u - 13u, reinterpret_cast<const i64*>(fact_keys), n, fk,
                       (n4 + blocks - 1) / blocks);
    LQ_LAUNCH_CHECK("keymap64_lookup_lds_kernel");
    return LQ_OK;
  }
  const int vec_ok = aligned(fact_keys, 16) && aligned(fk, 8);
  const int64_t threads = vec_ok ? n / 2 + n % 2 : n;
  const int64_t blocks = (threads + 255) / 256;
  if (blocks > 0x7fffffffLL) return fail(LQ_ERR_UNSUPPORTED, "too many rows for one launch");
  hipLaunchKernelGGL(keymap64_lookup_kernel, dim3(static_cast<unsigned>(blocks)), dim3(256), 0, s, header, buckets, g.mask, g.shift,
                     reinterpret_cast<const i64*>(fact_keys), n, fk, vec_ok);
  LQ_LAUNCH_CHECK("keymap64_lookup_kernel");
  return LQ_OK;
}

}  // extern "C"
