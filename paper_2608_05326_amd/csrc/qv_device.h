// Device-side helpers shared by the gfx950 kernels: vector types, exact
// fp16 / bf16 conversions and the launch argument blocks.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "qv_layout.h"

namespace qv {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

struct AttnArgs {
  Geometry g;
  UnitLayout L;
  uint8_t* base;            // unit block of (layer, seq 0)
  const uint16_t* q;        // [B][H_q][d]
  const uint16_t* k_new;    // [B][H_kv][d]
  const uint16_t* v_new;
  void* out;                // [B][H_q][d]
  int32_t T;                // sequence length after appending this step's token
  int32_t ring_w0;          // first window not routed yet
  int32_t n_ring;           // windows in [ring_w0, ring_w0 + n_ring) are attended from the ring
  int32_t n_sink_items;     // sink slots holding sink tokens
  float decay;              // factor on every updated window score before this step's mass
  int32_t key_norm;         // 1: key-norm scores (no attention masses; the new token's key norm)
  float pnorm_p;            // > 0: attention p-norm scores with this p
  int32_t period_start;     // 1: first step after a routing event (or prefill)
};

// Routing events of up to kRouteBatch layers go to one launch (one workgroup row
// per layer): the per-layer part of an event.
constexpr int kRouteBatch = 8;
// polls of the routing stream's wait for the cache stream before it gives up even
// if the wall clock has not passed its limit (each poll sleeps about 1024 clocks)
constexpr int64_t kGateMaxPolls = 40000000;
struct RetierUnit {
  uint8_t* base;            // the layer's first unit (sequence 0)
  int32_t aged_w0, aged_w1; // aged windows entering the candidate pool
  // split plans for the decode steps up to the next routing event, one per slot:
  // the sequence lengths [plan_t0, plan_t1] it serves (plan_t0 <= 0: none) and the
  // recent-region + sink windows those steps attend after the live list
  int32_t plan_t0[kPlanSlots], plan_t1[kPlanSlots];
  int32_t plan_extra[kPlanSlots];
};

struct RetierArgs {
  Geometry g;
  UnitLayout L;
  int32_t prefill;          // 1: candidates are the prompt's historical windows
  const float* init_scores; // prefill: [B][n_init]
  int32_t n_init;
  int32_t n_units;          // layers of this launch: workgroup row y serves unit[y]
  RetierUnit unit[kRouteBatch];
  const int32_t* gate_fail; // routing stream: nonzero when its wait for the cache stream timed out
};

struct MigrateArgs {
  Geometry g;
  UnitLayout L;
  int32_t n_units;          // layers of this launch: workgroup layer z serves base[z]
  uint8_t* base[kRouteBatch];
  const uint16_t* src_k;    // prompt keys [B][H_kv][T][d] (prefill only)
  const uint16_t* src_v;
  int32_t src_T;
  const int32_t* gate_fail; // as RetierArgs::gate_fail
  int32_t n_quant_blocks;   // workgroups (of a grid row) that take quantizations; the others take promotions
  int32_t n_promote_blocks;
};

struct KeyNormArgs {        // key-norm scores of the prompt windows
  Geometry g;
  const uint16_t* k;        // [B][H_kv][T][d] bf16 prompt keys
  int32_t T, n_init;
  float* out;               // [B][n_init]
};

// max / sum over the four 16-lane rows: lanes i, i^16, i^32, i^48 (gfx950 permlane
// swaps; every lane of the four gets the same value)
__device__ __forceinline__ float rows_max(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t a0 = a[0], a1 = a[1];
  const float y = fmaxf(__uint_as_float(a0), __uint_as_float(a1));
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const uint32_t b0 = b[0], b1 = b[1];
  return fmaxf(__uint_as_float(b0), __uint_as_float(b1));
}
__device__ __forceinline__ float rows_sum(float x) {
  const uint32_t u = __float_as_uint(x);
  const auto a = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const uint32_t a0 = a[0], a1 = a[1];
  const float y = __uint_as_float(a0) + __uint_as_float(a1);
  const uint32_t v = __float_as_uint(y);
  const auto b = __builtin_amdgcn_permlane16_swap(v, v, false, false);
  const uint32_t b0 = b[0], b1 = b[1];
  return __uint_as_float(b0) + __uint_as_float(b1);
}

// Reads one word of every 64-byte line of the kernel's argument block (a struct of
// BYTES bytes) and waits for them once; returns 0, to be added to a value the kernel
// needs first.  The compiler loads arguments where it first needs them, so a kernel
// whose arguments span eight lines meets a miss of the scalar cache (several hundred
// ns: the block lies in device memory) in each of the few dependent steps of its
// prologue; after this they hit.  (Not a volatile asm: after one the compiler no
// longer reads uniform memory with scalar loads.)
template <int BYTES>
__device__ __forceinline__ int touch_kernargs() {
  typedef __attribute__((address_space(4))) const uint32_t word;
  word* p = (word*)__builtin_amdgcn_kernarg_segment_ptr();
  uint32_t x = 0;
#pragma unroll
  for (int i = 0; i < (BYTES + 63) / 64; ++i) x |= p[16 * i];
  int zero;
  asm("s_mov_b32 %0, 0" : "=s"(zero) : "s"(x));
  return zero;
}

struct ObsArgs {            // initial window scores from the observation queries' attention
  const uint16_t* q;        // [B][H_q][n_obs][d] bf16
  const uint16_t* k;        // [B][H_kv][T][d] bf16
  int32_t B, H_q, H_kv, gqa, T, n_obs, n_rows, W, sink, n_w;
  int32_t cbase;            // first key of chunk 0 (sink - 64 n_pre, <= 0)
  int32_t n_pre;            // chunks before the first window (sink keys)
  int32_t n_chunks;         // chunks of 64 keys
  float scale_log2;
  float* cm;                // [B][H_kv][n_chunks][n_rows] logit max (log2 units) per chunk and row
  float* cl;                // the same layout: exp-sum relative to it
  float* wl;                // [B][H_kv][n_w][n_rows] window exp-sum relative to its chunk's max
  float2* row_ml;           // [B][H_kv][n_rows] (M, 1 / L)
  float* scores;            // [B][n_w]
};

struct ScorePowArgs {       // p-norm ranking: prompt scores raised to the power p
  const float* in;
  float* out;
  int32_t n;
  float p;
};

struct PackArgs {           // copy the prompt's sink tokens and tail into sink / ring slots
  Geometry g;
  UnitLayout L;
  uint8_t* base;
  const uint16_t* src_k;
  const uint16_t* src_v;
  int32_t src_T;
  int32_t n_sink;           // tokens [0, n_sink) and [tail0, src_T) are copied
  int32_t tail0;
};

__device__ inline float bf16_to_f32(uint16_t b) { return __uint_as_float((uint32_t)b << 16); }

__device__ inline uint16_t f32_to_bf16_rne(float f) {
  uint32_t u = __float_as_uint(f);
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}

__device__ inline double fp16_bits_to_f64(uint16_t h) {
  return (double)(float)__builtin_bit_cast(_Float16, h);
}

// next fp16 value toward -inf / +inf (finite inputs)
__device__ inline uint16_t fp16_next_down(uint16_t h) {
  if ((h & 0x7FFFu) == 0) return 0x8001u;
  return (h & 0x8000u) ? (uint16_t)(h + 1) : (uint16_t)(h - 1);
}
__device__ inline uint16_t fp16_next_up(uint16_t h) {
  if ((h & 0x7FFFu) == 0) return 0x0001u;
  return (h & 0x8000u) ? (uint16_t)(h - 1) : (uint16_t)(h + 1);
}

// largest fp16 <= x (x finite, |x| <= 65504)
__device__ inline uint16_t fp16_round_down(float x) {
  uint16_t h = __builtin_bit_cast(uint16_t, (_Float16)x);
  if ((float)__builtin_bit_cast(_Float16, h) > x) h = fp16_next_down(h);
  return h;
}

__device__ inline void set_error(int32_t* counts, int32_t bits) {
  __hip_atomic_fetch_or(counts + CNT_ERROR, bits, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace qv
