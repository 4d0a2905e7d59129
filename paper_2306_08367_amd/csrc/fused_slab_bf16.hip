// Join-computation stage (last line of Eq. 1) for wide bf16 models on many fact rows: hidden width a multiple of 8 up
// to 256, one to four dimensions, no fact columns or four, a second layer of up to 64 outputs on the matrix cores and
// one more layer of up to 16 behind it.
//
// What bounds it is the way of the projected rows to the compute units, and it is laid out for that twice over:
//   * A load instruction is taken apart into pieces that lie side by side in one cache line.  The layout the matrix
//     instruction asks for (lane (g, j): row j, 16-byte piece g) has no two such pieces in neighbouring lanes, and the
//     gathers then run at one 16-byte piece a cycle and compute unit, 9.3 TB/s, wherever the tables are.  Here eight
//     neighbouring lanes fetch 128 bytes of one row (28 TB/s out of L2), the sum over the tables is made where it
//     arrives, and the rectified bf16 values cross over to the matrix layout through 2 KB of LDS a wavefront.
//   * The hidden units are taken in slabs of 64 (128 bytes of a row, a cache line).  A wavefront keeps the second
//     layer's sums of up to 512 rows in registers and goes over the rows once for each slab, so that at any time the
//     chip reads one slab of every table: four tables of 10,000 x 256 are 20 MB, which every one of the eight 4 MB L2s
//     would have to fetch over the fabric, but 5 MB a slab.  That only works while the workgroups of an XCD are in the
//     same slab: a counter for each XCD counts the workgroups that are nearly through a slab, and one that is through
//     waits for the others before it goes on.  The wait is bounded and nothing depends on it but the time.
// 50e6 rows, four such tables, 256 -> 16: 11.5 ms row by row in the matrix layout, here 5.56, 18.4 TB/s gathered (bare gathers:
// whole rows of 512 bytes 9.6 TB/s, 128-byte rows of one slab 22); 5e6 rows 256 -> 64 -> 16 2.58 -> 1.08; 256 -> 16 with four
// fact columns and three tables of 2,000 rows 1.87 -> 0.81 ms.  What is left besides the gathers is vector instructions, the sums
// over the tables above all.
#include <atomic>

#include "lq_common.h"

namespace lq {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float v4f __attribute__((ext_vector_type(4)));
typedef float v16f __attribute__((ext_vector_type(16)));
typedef float v32f __attribute__((ext_vector_type(32)));
typedef unsigned int v4u __attribute__((ext_vector_type(4)));
typedef unsigned int v2u __attribute__((ext_vector_type(2)));

constexpr int SLAB_WAVES = 8;                     // one workgroup a compute unit, two wavefronts a SIMD
constexpr int SLAB_THREADS = 64 * SLAB_WAVES;
constexpr int SLAB_XCDS = 8;                      // workgroups are dealt to the XCDs in turn
constexpr int SLAB_PACE_STRIDE = 32;              // counters 128 bytes apart
constexpr int SLAB_PACE_POLLS = 128;              // about 100 us
constexpr int SLAB_PACE_SLOTS = 64;

// The counters of the paced calls in flight, 1 KB a call, in the library image (a caller's workspace may hold what another
// call of it still needs).  Calls take the slots in turn; more than 64 at once share some and wait longer or less, no more.
__device__ unsigned slab_pace[SLAB_PACE_SLOTS * SLAB_XCDS * SLAB_PACE_STRIDE];
__device__ __forceinline__ unsigned* pace_counter(int slot, int xcd) { return slab_pace + (slot * SLAB_XCDS + xcd) * SLAB_PACE_STRIDE; }

struct SlabArgs {
  int32_t slabs;        // slabs of 64 hidden units
  int32_t pairs;        // pairs of 16-row tiles a wavefront takes at a time
  int32_t keys_cap;     // rows of a wavefront's key buffer, pairs * 32 rounded up to 64
  int32_t vec_y;        // four outputs of a row can be stored at once
  int64_t batches;      // of 8 x 32 x pairs rows
  int32_t pace_slot;    // of the call's counters, or -1
  int32_t xch, keys, w2, b2, w3, b3, b1;   // byte offsets in LDS
};

__device__ __forceinline__ void wave_lds_order() {
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}
__device__ __forceinline__ float lo16(unsigned int w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float hi16(unsigned int w) { return __uint_as_float(w & 0xffff0000u); }

// Weights as A operands, zero-padded, [chunk of 32 inputs][tile of 16 outputs][64 lanes].  slab: inputs are hidden units
// of layer 1 in their order; otherwise the outputs of two tiles side by side, as the tiles' registers hold them.
__device__ __forceinline__ void stage_operand(const PredictArgs& a, int layer, bool slab, int chunks, int tout, v4u* dst, float* bias) {
  const bf16_t* W = static_cast<const bf16_t*>(a.W[layer]);
  for (int i = threadIdx.x; i < chunks * tout * 64; i += SLAB_THREADS) {
    const int ln = i & 63, tile = i >> 6, c = tile / tout, ot = tile - c * tout, g = ln >> 4, col = 16 * ot + (ln & 15);
    unsigned int h[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      const int unit = slab ? 32 * c + 8 * g + e : 32 * c + (e < 4 ? 4 * g + e : 16 + 4 * g + e - 4);
      h[e] = (unit < a.win[layer] && col < a.wout[layer]) ? W[static_cast<int64_t>(unit) * a.ldw[layer] + col] : 0u;
    }
    dst[i] = (v4u){h[0] | (h[1] << 16), h[2] | (h[3] << 16), h[4] | (h[5] << 16), h[6] | (h[7] << 16)};
  }
  for (int i = threadIdx.x; i < 16 * tout; i += SLAB_THREADS)
    bias[i] = (i < a.wout[layer] && a.bias[layer]) ? bf16_to_f32(static_cast<const bf16_t*>(a.bias[layer])[i]) : 0.f;
}

// 16 x 16 tiles of second-layer sums a wavefront keeps, four registers each.
template <int CF> struct SlabSums { static constexpr int TILES = 32; typedef v32f vec; };
template <> struct SlabSums<4> { static constexpr int TILES = 16; typedef v16f vec; };

// K tables, TH tiles of 16 second-layer outputs, the fact table's four columns (CF = 4) or none (0), a first bias or none.
template <int K, int TH, int CF, bool BIAS>
__global__ __launch_bounds__(SLAB_THREADS) void fused_slab_bf16_kernel(PredictArgs a, SlabArgs sa) {
  constexpr int KP = K == 3 ? 4 : K;
  extern __shared__ __align__(16) unsigned char smem[];
  const int w = threadIdx.x >> 6, lane = threadIdx.x & 63, c = lane & 7, sub = lane >> 3, g = lane >> 4, j = lane & 15;
  const int l1 = a.wout[0], l2 = a.wout[1];

  stage_operand(a, 1, true, 2 * sa.slabs, TH, reinterpret_cast<v4u*>(smem + sa.w2), reinterpret_cast<float*>(smem + sa.b2));
  if (a.n_layers == 3)
    stage_operand(a, 2, false, (TH + 1) / 2, 1, reinterpret_cast<v4u*>(smem + sa.w3), reinterpret_cast<float*>(smem + sa.b3));
  if constexpr (BIAS || CF > 0) {          // first bias (fp32) and the fact columns' rows of W_0 (bf16), zeros past l_1
    float* b1 = reinterpret_cast<float*>(smem + sa.b1);
    bf16_t* wf = reinterpret_cast<bf16_t*>(b1 + 64 * sa.slabs);
    for (int i = threadIdx.x; i < 64 * sa.slabs; i += SLAB_THREADS) {
      b1[i] = (BIAS && i < l1) ? bf16_to_f32(static_cast<const bf16_t*>(a.bias[0])[i]) : 0.f;
      for (int q = 0; q < CF; ++q) wf[q * 64 * sa.slabs + i] = i < l1 ? static_cast<const bf16_t*>(a.W[0])[q * a.ldw[0] + i] : bf16_t{0};
    }
  }
  __syncthreads();

  const bool paced = sa.pace_slot >= 0;
  unsigned* const pace = pace_counter(paced ? sa.pace_slot : 0, blockIdx.x % SLAB_XCDS);
  const int pairs = sa.pairs, rows = 32 * pairs;
  unsigned char* const xch = smem + sa.xch + w * 2048;
  uint32_t* const keys0 = reinterpret_cast<uint32_t*>(smem + sa.keys) + w * (2 * KP) * sa.keys_cap;   // two buffers
  const int key_chunks = (rows + 63) / 64;

  // One 64-row chunk of key column k of batch b, as byte offsets of the table's rows.
  auto key_load = [&](int64_t b, int k, int chunk) -> int {
    int64_t r = (b * SLAB_WAVES + w) * rows + chunk * 64 + lane;
    if (r >= a.n) r = a.n - 1;
    return __builtin_nontemporal_load(a.fk[k] + r);
  };
  auto key_store = [&](uint32_t* buf, int k, int chunk, int key) {
    buf[(chunk * 64 + lane) * KP + k] = static_cast<uint32_t>(key) * static_cast<uint32_t>(a.ldp[k] * 2);
  };
  // The offsets of row i (within the wavefront's rows).
  auto key_read = [&](const uint32_t* buf, int i, uint32_t (&f)[K]) {
    if constexpr (KP == 4) {
      const v4u q = *reinterpret_cast<const v4u*>(buf + i * 4);
#pragma unroll
      for (int k = 0; k < K; ++k) f[k] = q[k];
    } else if constexpr (KP == 2) {
      const v2u q = *reinterpret_cast<const v2u*>(buf + i * 2);
      f[0] = q[0]; f[1] = q[1];
    } else {
      f[0] = buf[i];
    }
  };

  int64_t b = blockIdx.x;
  if (b < sa.batches)
    for (int k = 0; k < K; ++k)
      for (int ch = 0; ch < key_chunks; ++ch) key_store(keys0, k, ch, key_load(b, k, ch));
  wave_lds_order();

  // Requests of step s (8 rows) of pair p in slab sl; a lane whose units lie past l_1 fetches the row's first piece.
  struct Step { v4u t[K]; v2u x; };
  auto request = [&](const uint32_t* buf, int64_t row0, int sl, int p, int s, Step& st) {
    const int i = 32 * p + 8 * s + sub;
    uint32_t f[K];
    key_read(buf, i, f);
    const uint32_t piece = 64 * sl + 8 * c < l1 ? 128u * sl + 16u * c : 0u;
#pragma unroll
    for (int k = 0; k < K; ++k)
      st.t[k] = *reinterpret_cast<const v4u*>(static_cast<const char*>(a.P[k]) + (f[k] + piece));
    if constexpr (CF > 0) {
      int64_t r = row0 + i;
      if (r >= a.n) r = a.n - 1;
      st.x = *reinterpret_cast<const v2u*>(static_cast<const bf16_t*>(a.X) + r * a.ldx);
    }
  };

  // Register v of tile (pair p, half h, outputs ot) is element (2 p + h) TH + ot of acc[v]: output 16 ot + 4 g + v of row j.
  typename SlabSums<CF>::vec acc[4];
  int parity = 0, phase = 0, polls = SLAB_PACE_POLLS;
  float zero = 0.f;
  asm volatile("" : "+s"(zero));
  Step st[4];
  if (b < sa.batches)
#pragma unroll
    for (int s = 0; s < 4; ++s) request(keys0, (b * SLAB_WAVES + w) * rows, 0, 0, s, st[s]);

  for (; b < sa.batches; b += gridDim.x) {
    const int64_t row0 = (b * SLAB_WAVES + w) * rows;
    const int64_t bn = b + gridDim.x < sa.batches ? b + gridDim.x : b;
    uint32_t* const cur = keys0 + parity * (KP * sa.keys_cap);
    uint32_t* const nxt = keys0 + (parity ^ 1) * (KP * sa.keys_cap);
    parity ^= 1;
    int it = 0;
    for (int sl = 0; sl < sa.slabs; ++sl) {
      if (paced && phase) {                // wait until the XCD's workgroups are nearly through the slab before
        __syncthreads();
        if (threadIdx.x == 0) {
          const unsigned peers = (gridDim.x - blockIdx.x % SLAB_XCDS + SLAB_XCDS - 1) / SLAB_XCDS;
          int i = 0;
          while (i < polls && __hip_atomic_load(pace, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) < peers * phase) {
            __builtin_amdgcn_s_sleep(2);
            ++i;
          }
          if (i == polls) polls = 0;       // others are not running (another kernel has their place): no more waiting
        }
        __syncthreads();
      }
      ++phase;
      const v4u* w2 = reinterpret_cast<const v4u*>(smem + sa.w2) + sl * (2 * TH * 64) + lane;
      v4u w2r[TH == 1 ? 2 : 1];
      if constexpr (TH == 1) { w2r[0] = w2[0]; w2r[1] = w2[64]; }
      const float* b1 = reinterpret_cast<const float*>(smem + sa.b1) + 64 * sl + 8 * c;
      const bf16_t* wf = reinterpret_cast<const bf16_t*>(smem + sa.b1 + 256 * sa.slabs) + 64 * sl + 8 * c;
      const bool partial = 64 * (sl + 1) > l1, dead = 64 * sl + 8 * c >= l1;

      for (int p = 0; p < pairs; ++p, ++it) {
        asm volatile("" ::: "memory");       // the staged model is read where it is used: held in registers it would not fit
        if (paced && p == pairs - 1 - (pairs >> 3) && threadIdx.x == 0)
          __hip_atomic_fetch_add(pace, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        // keys of the next batch, 64 rows at a time (the request for its first pair comes in the batch's last iteration,
        // so there are at least two)
        int fresh[K];
        const bool stage = it < key_chunks;
        if (stage)
#pragma unroll
          for (int k = 0; k < K; ++k) fresh[k] = key_load(bn, k, it);
        // the next pair: of this slab, of the next slab, or of the next batch
        const bool last_p = p + 1 == pairs, last_s = last_p && sl + 1 == sa.slabs;
        const int np = last_p ? 0 : p + 1, ns = last_p ? (last_s ? 0 : sl + 1) : sl;
        const uint32_t* nkeys = last_s ? nxt : cur;
        const int64_t nrow0 = last_s ? (bn * SLAB_WAVES + w) * rows : row0;
        if (last_s) wave_lds_order();
#pragma unroll
        for (int h = 0; h < 2; ++h) {
#pragma unroll
          for (int s = 2 * h; s < 2 * h + 2; ++s) {
            float z[8];
            int k1 = 0;
            if constexpr (BIAS || CF > 0) {
              const v4f ba = *reinterpret_cast<const v4f*>(b1), bb = *reinterpret_cast<const v4f*>(b1 + 4);
#pragma unroll
              for (int e = 0; e < 4; ++e) { z[e] = ba[e]; z[4 + e] = bb[e]; }
              if constexpr (CF > 0) {
#pragma unroll
                for (int q = 0; q < CF; ++q) {
                  const float x = q & 1 ? hi16(st[s].x[q >> 1]) : lo16(st[s].x[q >> 1]);
                  const v4u wq = *reinterpret_cast<const v4u*>(wf + q * 64 * sa.slabs);
#pragma unroll
                  for (int e = 0; e < 4; ++e) {
                    z[2 * e] = fmaf(x, lo16(wq[e]), z[2 * e]);
                    z[2 * e + 1] = fmaf(x, hi16(wq[e]), z[2 * e + 1]);
                  }
                }
              }
            } else {
#pragma unroll
              for (int e = 0; e < 4; ++e) { z[2 * e] = lo16(st[s].t[0][e]); z[2 * e + 1] = hi16(st[s].t[0][e]); }
              k1 = 1;
            }
#pragma unroll
            for (int k = k1; k < K; ++k)
#pragma unroll
              for (int e = 0; e < 4; ++e) { z[2 * e] += lo16(st[s].t[k][e]); z[2 * e + 1] += hi16(st[s].t[k][e]); }
            v4u hv = {f32x2_to_bf16x2(fmaxf(z[0], 0.f), fmaxf(z[1], 0.f)), f32x2_to_bf16x2(fmaxf(z[2], 0.f), fmaxf(z[3], 0.f)),
                      f32x2_to_bf16x2(fmaxf(z[4], 0.f), fmaxf(z[5], 0.f)), f32x2_to_bf16x2(fmaxf(z[6], 0.f), fmaxf(z[7], 0.f))};
            if (partial && dead) hv = (v4u){0u, 0u, 0u, 0u};
            request(nkeys, nrow0, ns, np, s, st[s]);
            // row r = 8 (s & 1) + sub of the tile, piece c at place c ^ (r / 2): both directions touch every bank once
            const int r = 8 * (s & 1) + sub;
            *reinterpret_cast<v4u*>(xch + r * 128 + ((c ^ (r >> 1)) << 4)) = hv;
          }
          wave_lds_order();
          const v4u h0 = *reinterpret_cast<const v4u*>(xch + j * 128 + ((g ^ (j >> 1)) << 4));
          const v4u h1 = *reinterpret_cast<const v4u*>(xch + j * 128 + (((4 + g) ^ (j >> 1)) << 4));
          wave_lds_order();
          const int t0 = (2 * p + h) * TH;
#pragma unroll
          for (int ot = 0; ot < TH; ++ot) {
            v4f y = {0.f, 0.f, 0.f, 0.f};
            if (sl > 0) y = (v4f){acc[0][t0 + ot], acc[1][t0 + ot], acc[2][t0 + ot], acc[3][t0 + ot]};
            const v4u wa = TH == 1 ? w2r[0] : w2[ot * 64], wb = TH == 1 ? w2r[TH == 1 ? 1 : 0] : w2[(TH + ot) * 64];
            y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wa), __builtin_bit_cast(bf16x8, h0), y, 0, 0, 0);
            y = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wb), __builtin_bit_cast(bf16x8, h1), y, 0, 0, 0);
            // The sums are put away from the result of a vector addition, never straight from the matrix instruction: the
            // compiler counts the s_set_gpr_idx_on ahead of an indexed move as one of the 8 wait states that the move has to
            // keep, and the first move was then seen to take the register's old value.  The addend is zero, but only the
            // program knows, so that no optimisation drops the addition.
#pragma unroll
            for (int v = 0; v < 4; ++v) acc[v][t0 + ot] = y[v] + zero;
          }
        }
        if (stage)
#pragma unroll
          for (int k = 0; k < K; ++k) key_store(nxt, k, it, fresh[k]);
      }
    }

    // ---- the batch's rows: second bias, then stored or through the last layer
    const float* b2 = reinterpret_cast<const float*>(smem + sa.b2) + 4 * g;
    for (int t = 0; t < 2 * pairs; ++t) {
      const int64_t row = row0 + 16 * t + j;
      v4f y[TH];
#pragma unroll
      for (int ot = 0; ot < TH; ++ot) {
        const int at = t * TH + ot;
        y[ot] = (v4f){acc[0][at], acc[1][at], acc[2][at], acc[3][at]} + *reinterpret_cast<const v4f*>(b2 + 16 * ot);
      }
      int l_out = l2;
      if (a.n_layers == 3) {
        // the few activations of this layer go to the matrix cores as their bf16 rounding and the rounding of the rest
        const v4u* w3 = reinterpret_cast<const v4u*>(smem + sa.w3) + lane;
        v4f o = *reinterpret_cast<const v4f*>(reinterpret_cast<const float*>(smem + sa.b3) + 4 * g);
#pragma unroll
        for (int m = 0; m < (TH + 1) / 2; ++m) {
          v4u head = {0u, 0u, 0u, 0u}, tail = {0u, 0u, 0u, 0u};
#pragma unroll
          for (int e = 0; e < 4; ++e)
            if (2 * m + (e >> 1) < TH) {
              const float x0 = fmaxf(y[(2 * m + (e >> 1)) % TH][2 * (e & 1)], 0.f), x1 = fmaxf(y[(2 * m + (e >> 1)) % TH][2 * (e & 1) + 1], 0.f);
              head[e] = f32x2_to_bf16x2(x0, x1);
              tail[e] = f32x2_to_bf16x2(x0 - lo16(head[e]), x1 - hi16(head[e]));
            }
          const bf16x8 wv = __builtin_bit_cast(bf16x8, w3[m * 64]);
          o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8, head), o, 0, 0, 0);
          o = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wv, __builtin_bit_cast(bf16x8, tail), o, 0, 0, 0);
        }
        y[0] = o;
        l_out = a.wout[2];
      }
      if (row < a.n) {
#pragma unroll
        for (int ot = 0; ot < TH; ++ot) {
          if (ot > 0 && a.n_layers == 3) break;
          const int col = 16 * ot + 4 * g;
          const int64_t at = row * a.ldy + col;
          if (sa.vec_y) {
            if (col < l_out) {
              if (a.y_dtype == LQ_BF16)
                __builtin_nontemporal_store((v2u){f32x2_to_bf16x2(y[ot][0], y[ot][1]), f32x2_to_bf16x2(y[ot][2], y[ot][3])},
                                            reinterpret_cast<v2u*>(static_cast<bf16_t*>(a.Y) + at));
              else
                __builtin_nontemporal_store(y[ot], reinterpret_cast<v4f*>(static_cast<float*>(a.Y) + at));
            }
          } else {
#pragma unroll
            for (int v = 0; v < 4; ++v)
              if (col + v < l_out) store_from_f32(a.Y, at + v, a.y_dtype, y[ot][v]);
          }
        }
      }
    }
  }
  // a workgroup with fewer batches than others counts as through for the rest
  if (paced && threadIdx.x == 0) {
    const int64_t rounds = (sa.batches + gridDim.x - 1) / gridDim.x;
    const unsigned missing = static_cast<unsigned>(rounds * sa.slabs - phase);
    if (missing)
      __hip_atomic_fetch_add(pace, missing, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  }
}

__global__ void slab_pace_clear_kernel(int slot) {
  if (threadIdx.x < SLAB_XCDS) *pace_counter(slot, threadIdx.x) = 0u;
}

template <int K, int TH, int CF, bool BIAS>
int launch_inst(const PredictArgs& a, SlabArgs sa, size_t lds, int grid, hipStream_t s) {
  const void* fn = reinterpret_cast<const void*>(&fused_slab_bf16_kernel<K, TH, CF, BIAS>);
  if (lds > 64 * 1024)
    LQ_HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds)));
  if (sa.pace_slot >= 0) {
    hipLaunchKernelGGL(slab_pace_clear_kernel, dim3(1), dim3(64), 0, s, sa.pace_slot);
    LQ_LAUNCH_CHECK("slab_pace_clear_kernel");
  }
  hipLaunchKernelGGL((fused_slab_bf16_kernel<K, TH, CF, BIAS>), dim3(static_cast<unsigned>(grid)), dim3(SLAB_THREADS), lds, s, a, sa);
  LQ_LAUNCH_CHECK("fused_slab_bf16_kernel");
  return LQ_OK;
}
template <int K, int TH>
int pick(const PredictArgs& a, const SlabArgs& sa, size_t lds, int grid, hipStream_t s) {
  if (a.c_f) return a.bias[0] ? launch_inst<K, TH, 4, true>(a, sa, lds, grid, s) : launch_inst<K, TH, 4, false>(a, sa, lds, grid, s);
  return a.bias[0] ? launch_inst<K, TH, 0, true>(a, sa, lds, grid, s) : launch_inst<K, TH, 0, false>(a, sa, lds, grid, s);
}
template <int K>
int pick_th(int TH, const PredictArgs& a, const SlabArgs& sa, size_t lds, int grid, hipStream_t s) {
  return TH == 1 ? pick<K, 1>(a, sa, lds, grid, s) : TH == 2 ? pick<K, 2>(a, sa, lds, grid, s) : pick<K, 4>(a, sa, lds, grid, s);
}

}  // namespace

// Microseconds of a call in this kernel and in the ones it would take otherwise, from about 2,400 shapes of 65,536 to 6e6 rows over
// tables of 100 to 1e6 rows, each timed in both (half of the estimates are within 5 % here and 9 % there).  A unit is the
// 65,536 rows that fill the chip with a pair of tiles a wavefront; this kernel works in whole units (131,149 rows take it as
// long as 196,608) and whole slabs, which is what it loses on some calls:
//   131,149 rows 128 -> 40 -> 8, one table of 40,000 rows and four fact columns 29 us here, 17 there; 65,536 rows 96 -> 64 -> 16, four
//   tables of 10,000 rows 23 and 15; 2.5e6 rows 104 -> 64 -> 1, one table of 700 rows 179 and 124; against
//   500,003 rows 256 -> 16 -> 1 with a bias, two tables of 20,000 rows, 53 and 161; 1e6 rows 128 -> 16, one table of 700 rows, 40 and 60.
// Taken on all of these shapes this kernel is 1.42 times as fast as the others in the geometric mean and 3 % or more behind on
// 331 of them; taken where its estimate is the smaller one, 1.45 times and on 73 (the best choice for each: 1.46).
struct SlabCost { double here, there; };
SlabCost slab_cost(const PredictArgs& a, int TH, int slabs, int64_t whole_units, double units) {
  const int l1 = a.wout[0], l_out = a.wout[a.n_layers - 1];
  const bool fact = a.c_f > 0, bias = a.bias[0] != nullptr;
  const double stored = l_out * static_cast<double>(dtype_size(a.y_dtype)) / 64;
  int64_t rows = 0;
  for (int k = 0; k < a.K; ++k) rows += a.prows[k];
  const double beyond_l2 = std::min(10.0, std::max(0.0, rows * 128.0 / (1 << 20) - 3));      // MB of a slab
  double slab = 0.3 * a.K + 0.012 * a.K * a.K * beyond_l2 + (fact ? 1.0 : 0) + 0.35 * TH;
  double rest = 0.9 + 0.2 * stored + (a.n_layers == 2 && l_out % 4 ? 0.2 * TH : 0);
  SlabCost c;
  c.here = 4.5 + 0.3 * slabs + whole_units * (rest + slabs * slab);
  if (a.K == 4 && TH == 4 && !fact) c.here += 4.5;           // (these instances keep registers in scratch memory)
  // there: the one-tile kernel, or the one for deeper models, whose first layer is padded to a power of two
  const bool one_tile = a.n_layers == 2 && l_out <= 16 && !fact && (l1 == 64 || l1 == 128 || l1 == 256);
  const int padded = l1 <= 64 ? 1 : (l1 <= 128 ? 2 : 4);
  c.there = 2.5 + 1.25 * padded + units * (l1 / 64.0 * (0.86 * a.K + (fact ? 1.0 : 0)) + (one_tile ? 2.5 : 1.55) * stored +
                                           padded * (0.25 + 0.17 * TH + (bias && !one_tile ? 1.7 : 0)));
  return c;
}

// Returns -1 when the shape is not one this kernel covers.
int try_fused_slab_bf16(const PredictArgs& a, hipStream_t s) {
  if (a.x_dtype != LQ_BF16 || a.p_dtype != LQ_BF16) return -1;
  if (a.n_layers < 2 || a.n_layers > 3 || a.K < 1 || a.K > 4) return -1;
  const int l1 = a.wout[0], l2 = a.wout[1];
  if (l1 % 8 || l1 < 40 || l1 > 256 || l2 > 64 || (a.n_layers == 3 && a.wout[2] > 16)) return -1;
  // Two layers with up to four outputs belong to the kernel that keeps the hidden units in fp32.
  if (a.n_layers == 2 && l2 <= 4) return -1;
  if (a.c_f != 0 && (a.c_f != 4 || a.ldx % 4 || !aligned(a.X, 8))) return -1;
  int64_t bytes = 0;
  for (int k = 0; k < a.K; ++k) {
    // whole cache lines: a slab of rows that straddle them takes two of them a row (200 -> 16: 0.7 times as fast as the
    // kernels below)
    if (!aligned(a.P[k], 128) || a.ldp[k] % 64 || a.prows[k] * a.ldp[k] * 2 > 0xffffffffLL) return -1;
    bytes += a.prows[k] * l1 * 2;
  }
  const int64_t cus = num_cus();
  // A pair of tiles for every wavefront of the chip, two where there is one slab; below that the kernels below, which spread
  // 16 rows at a time: 32,000 rows 128 -> 16 8.4 us, here 8.8, 50,000 11.3 and 9.4; 64 -> 16 8.0 and 10.4, 100,000 11.3 and 10.6.
  if (a.n < cus * SLAB_WAVES * 32 * (l1 <= 64 ? 2 : 1)) return -1;

  const int TH = l2 <= 16 ? 1 : (l2 <= 32 ? 2 : 4);
  const int l_out = a.n_layers == 3 ? a.wout[2] : l2;
  const int KP = a.K == 3 ? 4 : a.K;
  SlabArgs sa{};
  sa.slabs = (l1 + 63) / 64;
  sa.vec_y = l_out % 4 == 0 && a.ldy % 4 == 0 && aligned(a.Y, 4 * dtype_size(a.y_dtype));
  const int max_pairs = (a.c_f ? SlabSums<4>::TILES : SlabSums<0>::TILES) / (2 * TH);
  const int64_t per_pair = cus * SLAB_WAVES * 32;           // rows of one pair on every wavefront of the chip
  const int64_t rounds = (a.n + per_pair * max_pairs - 1) / (per_pair * max_pairs);
  sa.pairs = static_cast<int32_t>((a.n + per_pair * rounds - 1) / (per_pair * rounds));
  if (sa.slabs == 1) sa.pairs = (sa.pairs + 1) / 2 * 2;     // two iterations a batch at the least
  const SlabCost cost = slab_cost(a, TH, sa.slabs, rounds * sa.pairs, static_cast<double>(a.n) / per_pair);
  if (cost.here >= cost.there) return -1;
  if (a.probe) return LQ_OK;
  sa.keys_cap = (sa.pairs * 32 + 63) / 64 * 64;
  sa.batches = (a.n + SLAB_WAVES * 32 * sa.pairs - 1) / (SLAB_WAVES * 32 * sa.pairs);
  int off = 0;
  sa.w2 = off; off += 2 * sa.slabs * TH * 1024;
  sa.b2 = off; off += 64 * TH;
  sa.w3 = off; if (a.n_layers == 3) off += (TH + 1) / 2 * 1024;
  sa.b3 = off; off += 64;
  sa.b1 = off; if (a.c_f || a.bias[0]) off += 64 * sa.slabs * (4 + 2 * a.c_f);
  sa.xch = off; off += SLAB_WAVES * 2048;
  sa.keys = off; off += SLAB_WAVES * 2 * KP * sa.keys_cap * 4;
  const int grid = static_cast<int>(std::min<int64_t>(cus, sa.batches));
  // Pacing pays where the tables are several L2s large, a pass reads a quarter or a third of a row and the gathers, not the
  // later layers, take the time.  Unpaced -> paced in us: 4 x 10,000 rows of 256, 256 -> 16, 300,000 fact rows 62.5 -> 59.3
  // (the launch that clears the counters among it), 1e6 168 -> 142, 3e6 496 -> 400; 4 x 20,000 3e6 650 -> 595; 4 x 6,000 (11.7 MB)
  // 394 -> 356; 9,000 rows (4.4 MB) 300 -> 301; rows of 128 265 -> 250 and, in tables of 2 x 20,000, 183 -> 183;
  // 256 -> 64 -> 16 4 x 10,000 649 -> 576, 2 x 20,000 382 -> 404, 4 x 6,000 542 -> 552.
  const bool paced = sa.slabs >= 3 && a.n >= 1000000 && bytes > (TH == 1 ? 10 << 20 : 16 << 20) && (TH == 1 || a.K >= 3);
  static std::atomic<unsigned> next_slot{0};
  sa.pace_slot = paced ? static_cast<int32_t>(next_slot.fetch_add(1, std::memory_order_relaxed) % SLAB_PACE_SLOTS) : -1;
  switch (a.K) {
    case 1: return pick_th<1>(TH, a, sa, static_cast<size_t>(off), grid, s);
    case 2: return pick_th<2>(TH, a, sa, static_cast<size_t>(off), grid, s);
    case 3: return pick_th<3>(TH, a, sa, static_cast<size_t>(off), grid, s);
    default: return pick_th<4>(TH, a, sa, static_cast<size_t>(off), grid, s);
  }
}

}  // namespace lq
