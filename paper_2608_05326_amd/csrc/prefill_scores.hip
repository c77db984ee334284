// Initial window scores from prompt attention (Sec. 4.2: prompt attention
// initialises the window scores before the first tier assignment).
//
// The observation queries are the last n_obs prompt positions.  For KV head g
// of sequence b their rows are r = h_local * n_obs + j (h_local < H_q / H_kv,
// j < n_obs; query position T - n_obs + j), a contiguous [rows][d] slab of the
// [B][H_q][n_obs][d] query tensor.  Row r attends causally to keys 0 .. its
// position.  The window score is the mass the window's keys receive, summed
// over rows and KV heads and divided by H_q.
//
// The keys are cut into chunks of 64 aligned with the windows: chunk c holds
// keys cbase + 64 c .. + 63, cbase = sink - 64 * ceil(sink / 64) <= 0, so a
// chunk is either all sink (and keys < 0) or exactly 64 / W whole windows.
// Three launches, every reduction in a fixed order (bitwise repeatable):
//   k_obs_chunks   one pass over the keys: per (row, chunk) the logit max m
//                  and the exp-sum l relative to it, and per (row, window) the
//                  window's exp-sum relative to the same m
//   k_obs_rows     per row: global max M and 1 / L from its chunks
//   k_obs_windows  per window: sum over KV heads and rows of
//                  l_window * exp(m - M) / L, divided by H_q
// Logits come from bf16 MFMAs with the keys as the A operand (rows = keys) and the
// query rows as the B operand (columns = query rows): a lane holds several keys of
// one query row, so per-row sums fold in-lane and then over the lanes that share the
// row.  A wave holds one chunk's A operands in registers for every row; the query
// rows are staged in LDS.
#include <algorithm>
#include <mutex>

#include "qv_device.h"

namespace qv {

// Fixed scratch of the allocation-free entry point (qevict_prefill_scores_noalloc):
// every device the library runs on holds one copy for the life of the process.
// Host code never uses this name as an address: the per-device address comes
// from static_obs_scratch(), looked up once per device at cache creation.
static __device__ __align__(256) uint8_t scratch[kStaticObsScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex g_scratch_mu;
void* g_scratch_ptr[kMaxDevices] = {};
}  // namespace

// Device address of `scratch` on the current device (looked up on the first
// call for that device, with it current).  *what names the HIP call that failed.
hipError_t static_obs_scratch(void** ptr, const char** what) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) {
    *what = "hipGetDevice";
    return e;
  }
  if (dev < 0 || dev >= kMaxDevices) {
    *what = "device index";
    return hipErrorInvalidDevice;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) {
      *what = "hipGetSymbolAddress";
      return e;
    }
    g_scratch_ptr[dev] = p;
  }
  *ptr = g_scratch_ptr[dev];
  return hipSuccess;
}

constexpr int kObsChunkKeys = 64;      // keys per wave
constexpr int kObsRows = 512;          // query rows staged in LDS at once (139 KB)
constexpr int kObsThreads = 512;
constexpr int kObsRowBytes = 272;      // 256 B of a row + 16 B pad (conflict-free B reads)

typedef float f32x16 __attribute__((ext_vector_type(16)));
__device__ __forceinline__ f32x16 mfma_obs(bf16x8 a, bf16x8 b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}
// Sums over the lane pair l, l ^ 32 of two values at once: lanes below 32 get x's
// sum, the others y's.
__device__ __forceinline__ float pair_sums(float x, float y) {
  const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  const uint32_t s0 = s[0], s1 = s[1];
  return __uint_as_float(s0) + __uint_as_float(s1);
}

// One chunk against the staged rows [r0, r0 + nr): its keys in kop (tile kt, k-step
// ks: channels 16 ks + 8 lh .. + 7 of key kbase + 32 kt + lr).
template <bool W8>
__device__ __forceinline__ void obs_chunk(const ObsArgs& a, const u32x4 (&kop)[2][8], const uint8_t* sq, int c,
                                          int64_t bg, int r0, int nr, int lane) {
  const int lr = lane & 31, lh = lane >> 5, n_rows = a.n_rows;
  const int kbase = a.cbase + kObsChunkKeys * c;
  const int pos0 = a.T - a.n_obs;   // position of observation row j = pos0 + j
  // only a chunk reaching below key 0 or past the first observation position masks keys
  const bool edge = kbase < 0 || kbase + kObsChunkKeys - 1 > pos0;
  const int wpc = kObsChunkKeys / a.W;          // windows per chunk: 8 (W = 8), 2 (W = 32) or 1 (W = 64)
  const int w0 = (c - a.n_pre) * wpc;           // first window of the chunk (< 0: sink chunk)
  const float sc = a.scale_log2;
  // outputs of this lane: the chunk's max (lanes lh = 0) or exp-sum (lh = 1), and the
  // sum of window lh of the chunk (W = 32) or of the one window (W = 64, lh = 0)
  float* const ml_out = (lh ? a.cl : a.cm) + (bg * a.n_chunks + c) * n_rows + r0;
  float* const wl_c = a.wl + (bg * a.n_w + w0) * n_rows + r0;
  float* const wl_out = wl_c + (wpc == 2 && lh ? n_rows : 0);
  const bool has_w = w0 >= 0 && (wpc == 2 ? w0 + lh < a.n_w : lh == 0 && w0 < a.n_w);
  // the query operands of a row tile are read while the tile before is reduced
  u32x4 q[8];
  auto read_q = [&](int row) {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) q[ks] = *(const u32x4*)(sq + row * kObsRowBytes + 32 * ks + 16 * lh);
  };
  read_q(lr);
  for (int row = lr; row - lr < nr; row += 32) {
    f32x16 acc[2];
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[kt][i] = 0.f;
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
        acc[kt] = mfma_obs(__builtin_bit_cast(bf16x8, kop[kt][ks]), __builtin_bit_cast(bf16x8, q[ks]), acc[kt]);
    __builtin_amdgcn_sched_barrier(0);
    read_q(row - lr + 32 < nr ? row + 32 : lr);
    // acc[kt][i]: raw logit of key kbase + 32 kt + 8 (i / 4) + 4 lh + i % 4 for this row
    if (edge) {
      // (the first key goes through an opaque register: the compiler would keep all 32
      // key numbers and their signs across the loop)
      int k0 = kbase + 4 * lh;
      asm volatile("" : "+v"(k0));
      const uint32_t last = (uint32_t)(pos0 + ((r0 + row) % a.n_obs));   // this row's query position
#pragma unroll
      for (int kt = 0; kt < 2; ++kt)
#pragma unroll
        for (int i = 0; i < 16; ++i)   // key numbers below 0 are above every position unsigned
          acc[kt][i] = (uint32_t)(k0 + 32 * kt + 8 * (i >> 2) + (i & 3)) <= last ? acc[kt][i] : -INFINITY;
    }
    float mr = -INFINITY;
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int i = 0; i < 16; ++i) mr = fmaxf(mr, acc[kt][i]);
    {
      const auto s = __builtin_amdgcn_permlane32_swap(__float_as_uint(mr), __float_as_uint(mr), false, false);
      const uint32_t s0 = s[0], s1 = s[1];
      mr = fmaxf(__uint_as_float(s0), __uint_as_float(s1));
    }
    const float m = mr * sc;                      // the chunk's max for this row, log2 units
    const float mu = mr > -INFINITY ? m : 0.f;    // all keys masked: every term is exp2(-inf) = 0
    float l8[8];                                  // in-lane sums of the chunk's eight 8-key groups
#pragma unroll
    for (int kt = 0; kt < 2; ++kt)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        float e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) e[i] = __builtin_amdgcn_exp2f(fmaf(acc[kt][4 * j + i], sc, -mu));
        l8[4 * kt + j] = (e[0] + e[1]) + (e[2] + e[3]);
      }
    // lanes below 32: keys of tile 0, the others: tile 1
    const float lw = pair_sums((l8[0] + l8[1]) + (l8[2] + l8[3]), (l8[4] + l8[5]) + (l8[6] + l8[7]));
    const auto t = __builtin_amdgcn_permlane32_swap(__float_as_uint(lw), __float_as_uint(lw), false, false);
    const uint32_t t0 = t[0], t1 = t[1];
    const float lt = __uint_as_float(t0) + __uint_as_float(t1);   // the chunk's sum
    if (row < nr) {
      ml_out[row] = lh ? lt : m;
      if constexpr (!W8) {
        if (has_w) wl_out[row] = wpc == 2 ? lw : lt;
      }
    }
    if constexpr (W8) {   // lanes below 32: windows 0, 2, 4, 6; the others: 1, 3, 5, 7
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const float s = pair_sums(l8[2 * j], l8[2 * j + 1]);
        const int w = 2 * j + lh;   // of the chunk's eight
        if (row < nr && w0 >= 0 && w0 + w < a.n_w) wl_c[(uint32_t)(w * n_rows + row)] = s;
      }
    }
  }
}

// One workgroup of eight waves per compute unit: it stages up to 512 query rows of a
// (sequence, KV head) once and its waves go through the chunks in turn; while a wave
// computes one the keys of its next are on their way into a second set of registers.  With a workgroup per four chunks (keys loaded, then used) all
// workgroups of the chip loaded at once and then computed at once: 213 -> 194 us at
// 8 x 512 rows x 2048 chunks (128K; 268 MB of keys, 137 GFLOP), 226 -> 184 us at
// 32 x 256 rows x 1024 chunks (four 64K prompts, 537 MB), 40.6 -> 38.6 us at 8 x 128
// rows x 1024 chunks (64K).
// Where whole workgroups per (sequence, KV head) pair fill the chip, a pair's chunks go
// round its `share` workgroups (their reads then follow one another through the keys;
// parts of 1 MB each, a power of two apart, took 2% longer).  Otherwise (share 0) the
// chunks of all pairs are one list of which every workgroup takes an equal contiguous
// part, staging the next pair's rows where it crosses one: whole workgroups left compute
// units without work (136 pairs on 256) or ran a second, nearly empty wave of workgroups
// (264).  Parts of whole rounds of eight chunks are not equal enough: 78 -> 82 us at 8
// pairs x 625 chunks.
// 32x32 tiles halve the cross-lane work of 16x16 ones: a row's 64 logits lie in two
// lanes instead of four, one lane exchange serves both window sums, and a tile's
// masks, addresses and stores serve 32 rows.
// Bound by issue at many rows: vector and matrix instructions of a SIMD do not
// overlap here (measured: their times add), per logit one FMA, one exp (3.8 ns a wave
// against 1.2), one add and half a max beside the MFMAs.  Interleaving the products of
// one tile with the exponentials of the other within a wave changed nothing.
// W8: 8-token windows (eight per chunk), a separate instantiation so the other window
// sizes carry none of it
constexpr int kObsWaves = kObsThreads / 64;
constexpr int kObsUnits = 256;         // compute units (and resident workgroups)
template <bool W8>
__global__ __launch_bounds__(kObsThreads, 1) void k_obs_chunks(ObsArgs a, int share) {
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  __shared__ __attribute__((aligned(16))) uint8_t sq[kObsRows * kObsRowBytes];
  // this workgroup's part [begin, end) of all pairs' chunks (2^31 chunks of keys exceed
  // any memory); with a share, the whole pair, of which it takes every share-th chunk
  const int64_t total = (int64_t)a.n_chunks * a.B * a.H_kv;
  const int parts = share ? gridDim.x / share : gridDim.x, part = share ? blockIdx.x / share : blockIdx.x;
  const int begin = (int)(total * part / parts), end = (int)(total * (part + 1) / parts);
  const int step = kObsWaves * max(share, 1);
  for (int at = begin; at < end;) {
    const int pair = __builtin_amdgcn_readfirstlane(at / a.n_chunks);
    const int64_t bg = pair;
    // the pair's chunks [c0, c_end) of the part; the wave after the one that took the
    // part's last chunk so far takes the first
    const int c0 = at - pair * a.n_chunks, c_end = min(c0 + end - at, a.n_chunks);
    const int c_first = share ? wave * share + (int)blockIdx.x % share : c0 + ((wave - (at - begin)) & (kObsWaves - 1));
    at += c_end - c0;
    const uint16_t* kb = a.k + bg * a.T * kHeadDim;
    const uint16_t* qb = a.q + bg * a.gqa * a.n_obs * kHeadDim;   // (H_q = H_kv * gqa)
    auto load = [&](int c, u32x4 (&kop)[2][8]) {
#pragma unroll
      for (int kt = 0; kt < 2; ++kt) {
        const int key = a.cbase + kObsChunkKeys * c + 32 * kt + (lane & 31);
        // (keys outside the prompt are masked: any key in their place)
        const uint16_t* p = kb + (int64_t)max(min(key, a.T - 1), 0) * kHeadDim + 8 * (lane >> 5);
#pragma unroll
        for (int ks = 0; ks < 8; ++ks) kop[kt][ks] = *(const u32x4*)(p + 16 * ks);
      }
    };
    u32x4 k0[2][8], k1[2][8];
    for (int r0 = 0; r0 < a.n_rows; r0 += kObsRows) {
      const int nr = min(kObsRows, a.n_rows - r0), nr32 = (nr + 31) & ~31;
      int c = c_first;
      if (c < c_end) load(c, k0);
      __syncthreads();   // the previous rows are consumed
#pragma unroll 4
      for (int e = tid; e < nr32 * 16; e += kObsThreads) {
        const int row = e >> 4, part = e & 15;
        const u32x4 x = row < nr ? *(const u32x4*)(qb + (int64_t)(r0 + row) * kHeadDim + 8 * part)
                                 : (u32x4){0, 0, 0, 0};
        *(u32x4*)(sq + row * kObsRowBytes + 16 * part) = x;
      }
      __syncthreads();
      for (; c < c_end; c += 2 * step) {
        const int c1 = c + step, c2 = c1 + step;
        if (c1 < c_end) load(c1, k1);
        obs_chunk<W8>(a, k0, sq, c, bg, r0, nr, lane);
        if (c1 < c_end) {
          if (c2 < c_end) load(c2, k0);
          obs_chunk<W8>(a, k1, sq, c1, bg, r0, nr, lane);
        }
      }
    }
  }
}

constexpr int kOnceRows = 128;         // query rows staged in LDS at once
__device__ __forceinline__ f32x4 mfma_obs16(bf16x8 a, bf16x8 b, f32x4 c) {
  return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}

// The same for prompts whose chunks all fit the chip at once (at most 16 waves a
// compute unit), for few rows and for prompts of at most eight chunks: one chunk per
// wave, four to a workgroup, logits by 16x16x32 MFMAs.  With nothing to overlap across
// chunks, or little to compute for one, more and shorter waves hide more latency: 25.7
// against 29.1 us at 8 x 128 rows x 512 chunks (32K), 6.2 against 7.4 at 8 x 32 rows x
// 33 chunks (2K); all three launches 42.7 against 45.0 at 8 x 32 rows x 1024 chunks
// (64K), 53.6 against 57.3 at 1024 x 128 rows x 6 chunks.
// Four workgroups per compute unit (at most 128 VGPRs); W8: 8-token windows (eight
// per chunk), a separate instantiation so the other window sizes carry none of it.
// That one holds its chunk's addresses in scalar registers (a scalar wave number) and
// each exponential once: with 9 spilled registers it took 32.4 us at 8 x 128 rows x 512
// chunks, without 28.2.  (The other spills with a scalar wave number.)
template <bool W8>
__global__ __launch_bounds__(256, 4) void k_obs_chunks_once(ObsArgs a) {
  const int g = blockIdx.y, b = blockIdx.z;
  const int tid = threadIdx.x, lane = tid & 63, wave = W8 ? __builtin_amdgcn_readfirstlane(tid >> 6) : tid >> 6;
  const int T = a.T, n_rows = a.n_rows;
  const int lr = lane & 15, lq = lane >> 4;
  const int c = blockIdx.x * 4 + wave;           // this wave's chunk
  const bool live = c < a.n_chunks;             // uniform per wave
  const int kbase = a.cbase + kObsChunkKeys * c;
  __shared__ __attribute__((aligned(16))) uint8_t sq[kOnceRows * kObsRowBytes];

  // A operands: tile kt, k-step kc covers channels 32 kc + 8 lq .. + 7 of key
  // kbase + 16 kt + lr
  const uint16_t* kb = a.k + ((int64_t)b * a.H_kv + g) * T * kHeadDim;
  u32x4 kop[4][4];
#pragma unroll
  for (int kt = 0; kt < 4; ++kt) {
    const int key = kbase + 16 * kt + lr;
    const bool ok = live && key >= 0 && key < T;
#pragma unroll
    for (int kc = 0; kc < 4; ++kc)
      kop[kt][kc] = ok ? *(const u32x4*)(kb + (int64_t)key * kHeadDim + 32 * kc + 8 * lq)
                       : (u32x4){0, 0, 0, 0};
  }
  const uint16_t* qb = a.q + ((int64_t)b * a.H_q + (int64_t)g * a.gqa) * a.n_obs * kHeadDim;
  const int pos0 = T - a.n_obs;   // position of observation row j = pos0 + j
  // only a chunk reaching below key 0 or past the first observation position masks keys
  const bool edge = kbase < 0 || kbase + kObsChunkKeys - 1 > pos0;
  const int wpc = kObsChunkKeys / a.W;          // windows per chunk: 8 (W = 8), 2 (W = 32) or 1 (W = 64)
  const int w0 = (c - a.n_pre) * wpc;           // first window of the chunk (< 0: sink chunk)
  const int64_t bg = (int64_t)b * a.H_kv + g;
  const float sc = a.scale_log2;
  // outputs of this chunk (uniform pointers): statistics, and the sums of its windows
  float* const cm_out = a.cm + (bg * a.n_chunks + c) * n_rows;
  float* const cl_out = a.cl + (bg * a.n_chunks + c) * n_rows;
  float* const wl_a = a.wl + (bg * a.n_w + w0) * n_rows;
  const bool has_a = w0 >= 0 && w0 < a.n_w;
  const bool has_b = wpc == 2 && w0 >= 0 && w0 + 1 < a.n_w;

  for (int r0 = 0; r0 < n_rows; r0 += kOnceRows) {
    const int nr = min(kOnceRows, n_rows - r0);
    __syncthreads();   // the previous rows are consumed
#pragma unroll 2
    for (int i = 0; i < kOnceRows * 16 / 256; ++i) {
      const int e = tid + 256 * i, row = e >> 4, part = e & 15;
      const u32x4 v = row < nr ? *(const u32x4*)(qb + (int64_t)(r0 + row) * kHeadDim + 8 * part)
                               : (u32x4){0, 0, 0, 0};
      *(u32x4*)(sq + row * kObsRowBytes + 16 * part) = v;
    }
    __syncthreads();
    if (!live) continue;
    for (int rt = 0; rt < (nr + 15) / 16; ++rt) {
      const int row = rt * 16 + lr;   // this lane's query row inside the staged rows
      const int rg = r0 + row;
      f32x4 acc[4];
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) acc[kt] = (f32x4){0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int kc = 0; kc < 4; ++kc) {
        const u32x4 qv = *(const u32x4*)(sq + row * kObsRowBytes + 64 * kc + 16 * lq);
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
          acc[kt] = mfma_obs16(__builtin_bit_cast(bf16x8, kop[kt][kc]), __builtin_bit_cast(bf16x8, qv),
                             acc[kt]);
      }
      // acc[kt][i]: raw logit of key kbase + 16 kt + 4 lq + i for this row
      if (edge) {
        const int pos = pos0 + (rg % a.n_obs);   // this row's query position
#pragma unroll
        for (int kt = 0; kt < 4; ++kt)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            const int key = kbase + 16 * kt + 4 * lq + i;
            if (key < 0 || key > pos) acc[kt][i] = -INFINITY;
          }
      }
      float mr = -INFINITY;
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) mr = fmaxf(mr, acc[kt][i]);
      mr = rows_max(mr);
      const float m = mr * sc;                      // the chunk's max for this row, log2 units
      const float mu = mr > -INFINITY ? m : 0.f;    // all keys masked: every term is exp2(-inf) = 0
      float lA = 0.f, lB = 0.f;                     // keys of tiles 0-1 and 2-3
#pragma unroll
      for (int kt = 0; kt < 4; ++kt)
#pragma unroll
        for (int i = 0; i < 4; ++i) acc[kt][i] = __builtin_amdgcn_exp2f(fmaf(acc[kt][i], sc, -mu));
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        lA += acc[0][i];
        lA += acc[1][i];
        lB += acc[2][i];
        lB += acc[3][i];
      }
      if constexpr (W8) {
        // 8-token windows: tile kt holds windows 2 kt (lanes lq 0, 1) and 2 kt + 1
        // (lq 2, 3); the pair sums land in lanes lq 0 and 2
#pragma unroll
        for (int kt = 0; kt < 4; ++kt) {
          float lt = ((acc[kt][0] + acc[kt][1]) + acc[kt][2]) + acc[kt][3];
          lt += __shfl_xor(lt, 16, 64);
          const int w = 2 * kt + (lq >> 1);          // of the chunk's eight
          if (row < nr && (lq & 1) == 0 && w0 >= 0 && w0 + w < a.n_w) wl_a[w * n_rows + rg] = lt;
        }
      }
      lA = rows_sum(lA);
      lB = rows_sum(lB);
      if (row < nr) {
        if (lq == 0) cm_out[rg] = m;
        if (lq == 3) cl_out[rg] = lA + lB;
        if constexpr (!W8) {
          if (lq == 1 && has_a) wl_a[rg] = wpc == 2 ? lA : lA + lB;
          if (lq == 2 && has_b) wl_a[n_rows + rg] = lB;
        }
      }
    }
  }
}

// (M, 1 / L) of every row from its chunks' maxima and exp-sums: 32 rows per
// workgroup (a chunk's maxima of 32 consecutive rows are a whole cache line), P
// threads per row; thread (p, r) folds chunks p, p + P, ... of row r, eight to a
// round whose loads are issued together, and the P results of a row are folded by a
// pairwise tree (a fixed order).  Bound by the latency of its rounds, so P is 32
// (1024 threads) where a row has more than 64 chunks: 35.6 -> 15.5 us at 8 x 512
// rows x 2048 chunks against 16 threads per row and a separate pass for the maximum.
__device__ __forceinline__ float2 ml_combine(float2 x, float2 y) {
  const float mm = fmaxf(x.x, y.x);
  float ls = 0.f;
  if (x.x > -INFINITY) ls += x.y * __builtin_amdgcn_exp2f(x.x - mm);
  if (y.x > -INFINITY) ls += y.y * __builtin_amdgcn_exp2f(y.x - mm);
  return make_float2(mm, ls);
}

constexpr int kRowsPerBlock = 32;
template <int P>
__global__ __launch_bounds__(P * kRowsPerBlock) void k_obs_rows(ObsArgs a) {
  constexpr int RPB = kRowsPerBlock, ROUND = 8;
  const int g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const int rl = tid % RPB, p = tid / RPB, r = blockIdx.x * RPB + rl;
  const int64_t bg = (int64_t)b * a.H_kv + g;
  __shared__ float2 part[P][RPB];
  float m = -INFINITY, l = 0.f;
  if (r < a.n_rows) {
    const int64_t o = bg * a.n_chunks * a.n_rows + r;
    for (int c0 = p; c0 < a.n_chunks; c0 += P * ROUND) {
      float cm[ROUND], cl[ROUND];
#pragma unroll
      for (int i = 0; i < ROUND; ++i) {
        const int64_t at = o + (int64_t)min(c0 + P * i, a.n_chunks - 1) * a.n_rows;
        cm[i] = a.cm[at];
        cl[i] = a.cl[at];
      }
      float mn = m;
#pragma unroll
      for (int i = 0; i < ROUND; ++i) {
        cm[i] = c0 + P * i < a.n_chunks ? cm[i] : -INFINITY;
        mn = fmaxf(mn, cm[i]);
      }
      if (mn > -INFINITY) {
        l *= __builtin_amdgcn_exp2f(m - mn);   // (0 before the first chunk with a visible key)
#pragma unroll
        for (int i = 0; i < ROUND; ++i) l += cl[i] * __builtin_amdgcn_exp2f(cm[i] - mn);
        m = mn;
      }
    }
  }
  part[p][rl] = make_float2(m, l);
  __syncthreads();
  for (int h = P / 2; h > 0; h >>= 1) {
    if (p < h) part[p][rl] = ml_combine(part[p][rl], part[p + h][rl]);
    __syncthreads();
  }
  if (p == 0 && r < a.n_rows) {
    const float2 t = part[0][rl];
    a.row_ml[bg * a.n_rows + r] = make_float2(t.x, t.y > 0.f ? 1.f / t.y : 0.f);
  }
}

// score[b][w] = (1 / H_q) * sum over KV heads and rows of l_w * exp2(m_c - M) / L.
// A workgroup of 256 threads serves wpw windows (1, 2 or 4: enough workgroups
// for the chip whatever the window count), 256 / wpw threads each: thread t of
// a window takes rows t, t + 256 / wpw, ... of every KV head; the window's sum
// is folded by a butterfly per wave, then its waves in order.
__global__ __launch_bounds__(256) void k_obs_windows(ObsArgs a, int wpw) {
  const int b = blockIdx.y, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int tpw = 256 / wpw;                      // threads per window
  const int w = blockIdx.x * wpw + tid / tpw, t = tid % tpw;
  __shared__ float red[4];
  float s = 0.f;
  if (w < a.n_w) {
    const int c = a.n_pre + w / (kObsChunkKeys / a.W);
    // entries (g, r) = t, t + tpw, ... of the KV head x row list, stepped without division
    const int nr = a.n_rows, dg = tpw / nr, dr = tpw % nr;
    int g = t / nr, r = t % nr;
#pragma unroll 4
    while (g < a.H_kv) {
      const int64_t bg = (int64_t)b * a.H_kv + g;
      // M is finite for every row; a chunk with no visible key has m = -inf and l = 0
      const float2 rm = a.row_ml[bg * nr + r];
      const float m = a.cm[(bg * a.n_chunks + c) * nr + r];
      s += a.wl[(bg * a.n_w + w) * nr + r] * __builtin_amdgcn_exp2f(m - rm.x) * rm.y;
      r += dr;
      g += dg;
      if (r >= nr) {
        r -= nr;
        ++g;
      }
    }
  }
  for (int o = 1; o < 64; o <<= 1) s += __shfl_xor(s, o, 64);
  if (lane == 0) red[wave] = s;
  __syncthreads();
  const int wpwv = tpw / 64;                      // waves per window
  if (t == 0 && w < a.n_w) {
    const int w0 = wave;                          // this window's first wave
    float v = red[w0];
    for (int k = 1; k < wpwv; ++k) v += red[w0 + k];
    a.scores[(int64_t)b * a.n_w + w] = v / (float)a.H_q;
  }
}

hipError_t launch_prefill_scores(const ObsArgs& a, hipStream_t st) {
  if (a.n_w <= 0) return hipSuccess;
  constexpr int kOnceWaves = 16 * kObsUnits, kOnceMaxRows = 64, kOnceMaxChunks = 8;
  if ((int64_t)a.n_chunks * a.H_kv * a.B <= kOnceWaves || a.n_rows <= kOnceMaxRows || a.n_chunks <= kOnceMaxChunks) {
    const dim3 grid((a.n_chunks + 3) / 4, a.H_kv, a.B);
    if (a.W == 8) hipLaunchKernelGGL(k_obs_chunks_once<true>, grid, dim3(256), 0, st, a);
    else hipLaunchKernelGGL(k_obs_chunks_once<false>, grid, dim3(256), 0, st, a);
  } else {   // (more than 4096 chunks: two or more a wave)
    // whole workgroups per pair where they fill 15 of 16 units (12 pairs x 384 rows x 625
    // chunks: 87 against 92 us with equal parts)
    const int64_t pairs = (int64_t)a.H_kv * a.B;
    int share = (int)(kObsUnits / pairs);
    if (16 * share * pairs < 15 * kObsUnits) share = 0;
    const dim3 grid((unsigned)(share ? share * pairs : kObsUnits));
    if (a.W == 8) hipLaunchKernelGGL(k_obs_chunks<true>, grid, dim3(kObsThreads), 0, st, a, share);
    else hipLaunchKernelGGL(k_obs_chunks<false>, grid, dim3(kObsThreads), 0, st, a, share);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const dim3 rgrid((a.n_rows + kRowsPerBlock - 1) / kRowsPerBlock, a.H_kv, a.B);
  if (a.n_chunks > 64) hipLaunchKernelGGL(k_obs_rows<32>, rgrid, dim3(1024), 0, st, a);
  else hipLaunchKernelGGL(k_obs_rows<8>, rgrid, dim3(256), 0, st, a);
  if ((e = hipGetLastError()) != hipSuccess) return e;
  const int64_t nwin = (int64_t)a.n_w * a.B;
  const int wpw = nwin >= 4096 ? 4 : nwin >= 2048 ? 2 : 1;   // windows per workgroup
  hipLaunchKernelGGL(k_obs_windows, dim3((a.n_w + wpw - 1) / wpw, a.B), dim3(256), 0, st, a, wpw);
  return hipGetLastError();
}

}  // namespace qv
