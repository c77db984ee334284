// Window migrations between the tier pools (QEvict Sec. 4.3, migration-stable
// quantization; Algorithm 1 promote / quantize-once steps), driven by the work
// lists the re-tier kernel wrote; grids are sized for the worst case and idle
// workgroups exit at once, so no host synchronisation is needed.
//
// Quantization of one group x (asymmetric, b bits, n = 2^b - 1 levels):
//   z = largest fp16 <= min(x); s = smallest fp16 >= 0 with z + n s >= max(x);
//   c = round-half-even((x - z) / s)   (all codes 0 when s = 0).
// z + k s / 2 is exact in float64 for the integers k involved (fp16 operands),
// so the comparisons that decide s are exact; a code comes from an fp32 quotient
// where that decides as the exact one (see entry_codes) and from those boundaries
// elsewhere.  The result is bit-identical to the definition.  Keys form one group per
// channel across the window's tokens, values one group per token across G channels.
// Promotion writes RNE_bf16(z + s c), one rounding of the exact value.
//
// One wave takes one part of one (window, KV head): the keys or the values of one
// half of the channels, 64 lanes on W x 64 values, so no step of a task waits for
// another wave.  A wave's key lanes read the window in the chunk order of the bf16
// slots straight into registers (also from the prompt's rows), reduce each channel
// over its tokens with lane exchanges and form whole code words; value rows pass
// through LDS, which turns the prompt's rows into the columns the chunks and code
// words hold.  Routing events of few windows take half a part per wave (k_migrate_few).
#include <algorithm>

#include "qv_device.h"

namespace qv {

__device__ __forceinline__ bool quant_params(float lo, float hi, int nbits, uint16_t* zb, uint16_t* sb) {
  if (!(lo >= -65504.f && hi <= 65504.f)) return false;   // also rejects NaN
  const uint16_t zh = fp16_round_down(lo);
  const double z = fp16_bits_to_f64(zh);
  const double n = (double)((1 << nbits) - 1);
  const double hid = hi;
  // an fp32 estimate of (hi - z) / n, then the exact condition decides
  const float zf = (float)__builtin_bit_cast(_Float16, zh);
  const float t = (hi - zf) * (nbits == 4 ? 1.f / 15.f : 1.f / 3.f);
  uint16_t sh = __builtin_bit_cast(uint16_t, (_Float16)t);
  for (int k = 0; k < 8 && z + fp16_bits_to_f64(sh) * n < hid; ++k) sh = fp16_next_up(sh);
  for (int k = 0; k < 8 && sh != 0 && z + fp16_bits_to_f64(fp16_next_down(sh)) * n >= hid; ++k)
    sh = fp16_next_down(sh);
  *zb = zh;
  *sb = sh;
  return true;
}

// A (window, KV head) migration has four parts, one per wave: part = 2 area + h,
// area 0 the keys and 1 the values, h the channel half.  Key half h holds the
// channel blocks 32 kb of kb = 2h, 2h + 1; with RoPE, whose un-rotation pairs
// channels i and i + 64, of kb = h, h + 2.  Value half h holds channels
// 64 h .. 64 h + 63 (blocks cb = 4h .. 4h + 3).
constexpr int kParts = 4;
constexpr int kMigrateThreads = 256;   // the four parts of one (window, KV head)
static_assert(kMigrateThreads == 64 * kParts, "one wave per part");
// value group (channels) of a window length: G = W, except 32 for 8-token windows
template <int W>
constexpr int value_group() { return W == 8 ? 32 : W; }
// LDS row of one token's 64 channels: the padding puts the rows 4 q + j that the
// four lane groups read together in different banks
constexpr int kLdsRow = 64 + 8;

// A group's parameters as the code pass uses them, one 16-byte LDS entry: zero
// point, scale and its reciprocal in fp32, and the magnitude below which a value's
// code is decided in float64 (see entry_codes).
struct GroupParams {
  float z, s, inv, thr;
};
template <int W>
struct PartLds {   // a value part: rows and the 64 groups' parameters
  uint16_t rows[W * kLdsRow];
  GroupParams gp[64];
};
struct KeyLds {    // a key part: entry 32 i + 8 q + j for channel 32 kb(i) + 8 q + j
  GroupParams gp[64];
};
template <int W>
struct MigrateLds {
  KeyLds k[2];
  PartLds<W> v[2];
};

// Orders this wave's LDS traffic (a wave's LDS operations execute in order; the
// memory clobber keeps the compiler from moving accesses across).
__device__ __forceinline__ void lds_order() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

__device__ __forceinline__ u32x4 gld16(const void* p) { return *(const u32x4*)p; }
__device__ __forceinline__ float elem_f32(const u32x4& v, int j) {
  const uint32_t w = v[j >> 1];
  return __uint_as_float((j & 1) ? (w & 0xFFFF0000u) : (w << 16));
}

// value of x in the lane that the DPP control names
template <int CTRL>
__device__ __forceinline__ float dpp(float x) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(x), CTRL, 0xF, 0xF, false));
}
constexpr int kXor1 = 0xB1, kXor2 = 0x4E, kXor7 = 0x141, kXor8 = 0x128;   // partner lane ^ 1, 2, 7, 8 (in its row)

// One step of a reduce-scatter: of 2 N running (min, max) pairs a lane keeps the
// upper N if `up` and the lower N otherwise, combined with its partner's.
template <int N, int CTRL>
__device__ __forceinline__ void scatter_minmax(float* mn, float* mx, bool up) {
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const float keep_n = up ? mn[N + i] : mn[i], send_n = up ? mn[i] : mn[N + i];
    const float keep_x = up ? mx[N + i] : mx[i], send_x = up ? mx[i] : mx[N + i];
    mn[i] = fminf(keep_n, dpp<CTRL>(send_n));
    mx[i] = fmaxf(keep_x, dpp<CTRL>(send_x));
  }
}

// Scale and zero point of one group from its extremes; latches ERR_RANGE (and
// gives zeros) when they are outside fp16.
__device__ __forceinline__ void group_params(float lo, float hi, int nb, GroupParams* gp, uint16_t* zb,
                                             uint16_t* sb, int32_t* counts) {
  *zb = *sb = 0;
  if (!quant_params(lo, hi, nb, zb, sb)) set_error(counts, ERR_RANGE);
  GroupParams p;
  p.z = (float)__builtin_bit_cast(_Float16, *zb);
  p.s = (float)__builtin_bit_cast(_Float16, *sb);
  p.inv = p.s > 0.f ? 1.f / p.s : 0.f;
  const float span = (float)(1 << nb) * p.s;   // more than any x - z
  p.thr = p.z != 0.f && fabsf(p.z) < span * 0x1p-11f ? INFINITY : span * 0x1p-14f;
  *gp = p;
}

// Round-half-even code of x in its group, decided exactly: an fp32
// estimate of floor((x - z) / s), off by one at most where the quotient is next to
// an integer, then the half-step boundary z + (c + 1/2) s above it, formed in
// float64 where it is exact (fp16 operands, c <= 15).
__device__ __forceinline__ uint32_t quant_code_exact(float x, const GroupParams& p, int nmax) {
  float z = p.z, s = p.s;
  asm volatile("" : "+v"(z), "+v"(s));   // (formed here, not kept in float64 from entry to entry)
  float c = floorf((x - z) * p.inv);
  c = fminf(fmaxf(c, 0.f), (float)nmax);
  const double b = fma((double)(c + 0.5f), (double)s, (double)z), xd = x;
  const int up = ((xd > b) | ((xd == b) & ((int)c & 1))) & (c < (float)nmax);
  return s == 0.f ? 0u : (uint32_t)((int)c + up);
}

// bit of code j of a word's first entry (an int2 word's second entry: 8 bits higher)
__device__ __forceinline__ int code_bit(int nb, int j) { return (j & 1) * 16 + nb * (j >> 1); }

// The 8 codes of an entry, nb bits each: round-half-even of q = (x - z) / s in
// fp32, which decides as the exact quotient does:
//  - |x| >= 2^-14 2^nb s and |z| >= 2^-11 2^nb s (or z = 0) put x - z, less than
//    2^nb s, on a grid of at least 2^-22 of it: d = x - z is exact;
//  - q is d / s correctly rounded (one residual step on d * (1 / s); the quotient
//    of a 22-bit by an 11-bit number is nowhere nearer a rounding boundary than
//    the step's error);
//  - d / s is either k + 1/2 exactly, and then q is, or at least 2^-23 q away from
//    it, more than half an ulp, and q lies on the same side.
// An entry with a value below the threshold (one wave entry in about ten) is
// decided with float64 boundaries.  Nine VALU operations a value; deciding every
// value in float64 took 29 and bound the prompt's migrations.  Adding 1.5 * 2^23
// rounds half to even into the low bits of the sum.
// val(j): value j; prm(j): its group's parameters.
constexpr float kRoundBias = 12582912.f;      // 1.5 * 2^23
constexpr uint32_t kRoundBits = 0x4B400000u;
template <class V, class P>
__device__ __forceinline__ uint32_t entry_codes(int nb, V&& val, P&& prm) {
  const int nmax = (1 << nb) - 1;
  uint32_t wd = 0;
  bool small = false;
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const GroupParams p = prm(j);
    const float x = val(j), d = x - p.z;
    const float q0 = d * p.inv;
    const float q = fmaf(fmaf(-q0, p.s, d), p.inv, q0);
    small |= fabsf(x) < p.thr;
    // (a NaN becomes 0, as in the exact decision)
    wd += (__float_as_uint(__builtin_amdgcn_fmed3f(q, 0.f, (float)nmax) + kRoundBias) - kRoundBits) << code_bit(nb, j);
  }
  if (__builtin_amdgcn_ballot_w64(small) != 0) {
    wd = 0;
#pragma unroll
    for (int j = 0; j < 8; ++j) wd |= quant_code_exact(val(j), prm(j), nmax) << code_bit(nb, j);
  }
  return wd;
}
// One work-list entry (win, src_kind, src_idx, dst, bits, dep), held in registers.
struct WorkEntry {
  int32_t v[kQEntry];
};
__device__ __forceinline__ WorkEntry load_entry(const int32_t* list, int e) {
  WorkEntry x;
#pragma unroll
  for (int i = 0; i < kQEntry; ++i) x.v[i] = __builtin_amdgcn_readfirstlane(list[e * kQEntry + i]);
  return x;
}

// One (window, KV head) of a routing event: where it lies.
struct Task {
  const MigrateArgs& a;
  uint8_t* ub;
  int b, g;
  __device__ __forceinline__ const uint16_t* prompt_rows(int area, int w) const {
    const int64_t row0 = ((int64_t)b * a.g.H_kv + g) * a.src_T + a.g.sink + (int64_t)w * a.g.W;
    return (area == 0 ? a.src_k : a.src_v) + row0 * kHeadDim;
  }
  __device__ __forceinline__ uint8_t* slot(int src_kind, int idx) const {
    return ub + (src_kind == SRC_FSLOT ? a.L.fpool : a.L.ring) + (int64_t)idx * a.g.fslot_bytes +
           g * a.g.fhead_bytes;
  }
  __device__ __forceinline__ uint8_t* record(int idx) const {
    return ub + a.L.qpool + (int64_t)idx * a.g.qslot_bytes + g * a.g.qrec_bytes;
  }
};

// ---- keys ------------------------------------------------------------------
// Pieces of 16 bytes in chunk order: 32- and 64-token windows, lane (q, r) holds
// token 16 tb + r, channels 32 kb(i) + 8 q .. + 7 in x[2 tb + i]; 8-token windows,
// lane (i, q, r < 8) token r, channels 32 (2h + i) + 8 q .. + 7 in x[0].
template <int W>
constexpr int key_pieces() { return W == 8 ? 1 : W / 8; }
template <bool ROPE>
__device__ __forceinline__ constexpr int key_block(int h, int i) { return ROPE ? h + 2 * i : 2 * h + i; }

template <int W, bool ROPE>
__device__ __forceinline__ int key_piece_off(int h, int pc, int lane) {   // byte offset in a bf16 slot
  if constexpr (W == 8) return (2 * h * 4 * 8 + lane) * 16;
  else return (((pc >> 1) * 4 + key_block<ROPE>(h, pc & 1)) * 64 + lane) * 16;
}
template <int W, bool ROPE>
__device__ __forceinline__ void load_keys(const Task& t, int w, int src_kind, int src_idx, int h, int lane,
                                          u32x4 (&x)[key_pieces<W>()]) {
  if (src_kind == SRC_PROMPT) {
    const uint16_t* src = t.prompt_rows(0, w);
#pragma unroll
    for (int pc = 0; pc < key_pieces<W>(); ++pc) {
      if constexpr (W == 8)
        x[pc] = gld16(src + (lane & 7) * kHeadDim + 64 * h + 8 * (lane >> 3));
      else
        x[pc] = gld16(src + (16 * (pc >> 1) + (lane & 15)) * kHeadDim + 32 * key_block<ROPE>(h, pc & 1) +
                      8 * (lane >> 4));
    }
  } else {
    const uint8_t* p = t.slot(src_kind, src_idx);
#pragma unroll
    for (int pc = 0; pc < key_pieces<W>(); ++pc) x[pc] = gld16(p + key_piece_off<W, ROPE>(h, pc, lane));
  }
}

// RoPE (cos, sin) of position p, channel pair i
__device__ __forceinline__ float2 rope_cs(const Geometry& G, int p, int i) {
  return *(const float2*)(G.rope + 2 * ((int64_t)p * (kHeadDim / 2) + i));
}

// Pre-RoPE keys of a part's pieces (absolute position of token t = p0 + t): channel
// i < 64 becomes x_i cos + x_{i+64} sin, channel i + 64 becomes x_{i+64} cos - x_i
// sin, each product and sum rounded to float32 (no fused multiply-add), then RNE to
// bf16.  Pieces 2 tb and 2 tb + 1 of a lane hold the two channels of each pair.
template <int W>
__device__ __forceinline__ void unrotate_keys(const Geometry& G, u32x4 (&x)[key_pieces<W>()], int p0, int h,
                                              int lane) {
#pragma clang fp contract(off)
#pragma unroll
  for (int tb = 0; tb < W / 16; ++tb) {
    const int p = p0 + 16 * tb + (lane & 15), i0 = 32 * h + 8 * (lane >> 4);
    u32x4 lo = x[2 * tb], hi = x[2 * tb + 1];
#pragma unroll
    for (int d = 0; d < 4; ++d) {
      uint32_t lw = 0, hw = 0;
#pragma unroll
      for (int o = 0; o < 2; ++o) {
        const int j = 2 * d + o;
        const float a = elem_f32(x[2 * tb], j), bb = elem_f32(x[2 * tb + 1], j);
        const float2 cs = rope_cs(G, p, i0 + j);
        const float ac = a * cs.x, bs = bb * cs.y, bc = bb * cs.x, as = a * cs.y;
        lw |= (uint32_t)f32_to_bf16_rne(ac + bs) << (16 * o);
        hw |= (uint32_t)f32_to_bf16_rne(bc - as) << (16 * o);
      }
      lo[d] = lw;
      hi[d] = hw;
    }
    x[2 * tb] = lo;
    x[2 * tb + 1] = hi;
  }
}

// Code words of a key part.
template <int W, bool ROPE>
__device__ __forceinline__ void store_key_codes(const u32x4 (&x)[key_pieces<W>()], const KeyLds& sm, uint8_t* rec,
                                                int nb, int h, int lane) {
  GroupParams p[8];     // parameters of the 8 channels of a piece
  auto params = [&](int first) {
#pragma unroll
    for (int j = 0; j < 8; ++j) p[j] = sm.gp[first + j];
  };
  auto codes = [&](const u32x4& y) {
    return entry_codes(nb, [&](int j) { return elem_f32(y, j); }, [&](int j) { return p[j]; });
  };
  if constexpr (W == 8) {
    const int i = lane >> 5, ln = lane & 31;
    params(8 * (lane >> 3));
    const uint32_t wd = codes(x[0]);
    // int2: the half's word holds entry i = 0 in bytes 0 and 2, i = 1 in bytes 1 and 3
    const uint32_t other = (uint32_t)__shfl_xor((int)wd, 32, 64);
    if (nb == 4) *(uint32_t*)(rec + ln * 16 + 4 * (2 * h + i)) = wd;
    else if (i == 0) *(uint32_t*)(rec + ln * 8 + 4 * h) = wd | (other << 8);
  } else {
    uint32_t wd[W / 8];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      params(32 * i + 8 * (lane >> 4));
#pragma unroll
      for (int tb = 0; tb < W / 16; ++tb) wd[2 * tb + i] = codes(x[2 * tb + i]);
      if constexpr (W == 64) asm volatile("" ::: "memory");
    }
    if (nb == 4) {
#pragma unroll
      for (int tb = 0; tb < W / 16; ++tb) {
        uint8_t* d = rec + (tb * 64 + lane) * 16;
        if constexpr (ROPE) {
          *(uint32_t*)(d + 4 * h) = wd[2 * tb];
          *(uint32_t*)(d + 4 * h + 8) = wd[2 * tb + 1];
        } else {
          *(uint2*)(d + 8 * h) = make_uint2(wd[2 * tb], wd[2 * tb + 1]);
        }
      }
    } else {
#pragma unroll
      for (int tb = 0; tb < W / 16; ++tb) {
        if constexpr (ROPE) {   // word 2 tb + i, entry h: its bytes h and h + 2
#pragma unroll
          for (int i = 0; i < 2; ++i) {
            uint8_t* d = rec + ((tb >> 1) * 64 + lane) * 16 + (2 * (tb & 1) + i) * 4 + h;
            d[0] = (uint8_t)wd[2 * tb + i];
            d[2] = (uint8_t)(wd[2 * tb + i] >> 16);
          }
        } else {                // word 2 tb + h, both entries
          *(uint32_t*)(rec + ((tb >> 1) * 64 + lane) * 16 + (2 * (tb & 1) + h) * 4) = wd[2 * tb] | (wd[2 * tb + 1] << 8);
        }
      }
    }
  }
}

template <int W, bool ROPE>
__device__ __forceinline__ void quantize_keys(const Task& t, const WorkEntry& ent, KeyLds& sm, int32_t* counts,
                                              int h, int lane) {
  const Geometry& G = t.a.g;
  const int w = ent.v[0], nb = ent.v[4];
  constexpr int NP = key_pieces<W>();
  u32x4 x[NP];
  load_keys<W, ROPE>(t, w, ent.v[1], ent.v[2], h, lane, x);
  if constexpr (ROPE) unrotate_keys<W>(G, x, G.sink + w * W, h, lane);
  uint8_t* rec = t.record(ent.v[3]);
  // extremes of every channel over the window's tokens: in the lane over its row
  // tiles, then over the 16 (8) lanes of a row, each step halving the channels a
  // lane keeps; a lane ends with one channel of the part
  float lo, hi;
  int idx;   // parameter entry: 32 i + 8 q + j
  if constexpr (W == 8) {
    float mn[8], mx[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) mn[j] = mx[j] = elem_f32(x[0], j);
    scatter_minmax<4, kXor7>(mn, mx, (lane & 4) != 0);
    scatter_minmax<2, kXor2>(mn, mx, (lane & 2) != 0);
    scatter_minmax<1, kXor1>(mn, mx, (lane & 1) != 0);
    lo = mn[0];
    hi = mx[0];
    idx = (lane >> 3) * 8 + (lane & 7);
  } else {
    float l2[2], h2[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      float mn[8], mx[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) mn[j] = mx[j] = elem_f32(x[i], j);
#pragma unroll
      for (int tb = 1; tb < W / 16; ++tb)
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float v = elem_f32(x[2 * tb + i], j);
          mn[j] = fminf(mn[j], v);
          mx[j] = fmaxf(mx[j], v);
        }
      scatter_minmax<4, kXor8>(mn, mx, (lane & 8) != 0);
      scatter_minmax<2, kXor7>(mn, mx, (lane & 4) != 0);
      scatter_minmax<1, kXor2>(mn, mx, (lane & 2) != 0);
      l2[i] = fminf(mn[0], dpp<kXor1>(mn[0]));
      h2[i] = fmaxf(mx[0], dpp<kXor1>(mx[0]));
    }
    lo = (lane & 1) ? l2[1] : l2[0];
    hi = (lane & 1) ? h2[1] : h2[0];
    idx = 32 * (lane & 1) + 8 * (lane >> 4) + ((lane & 15) >> 1);
  }
  {
    uint16_t zb, sb;
    group_params(lo, hi, nb, &sm.gp[idx], &zb, &sb, counts);
    uint16_t* mk = (uint16_t*)(rec + meta_k_off(G)) + 32 * key_block<ROPE>(h, idx >> 5) + (idx & 31);
    mk[0] = sb;
    mk[kHeadDim] = zb;
  }
  lds_order();
  store_key_codes<W, ROPE>(x, sm, rec, nb, h, lane);
}

// ---- values ----------------------------------------------------------------
// One half's value rows into LDS, [token][64 channels].
template <int W>
__device__ __forceinline__ void stage_values(const Task& t, int w, int src_kind, int src_idx, int h, int lane,
                                             uint16_t* rows) {
  if (src_kind == SRC_PROMPT) {
    const uint16_t* src = t.prompt_rows(1, w) + 64 * h + 8 * (lane & 7);
    u32x4 x[W / 8];
#pragma unroll
    for (int k = 0; k < W / 8; ++k) x[k] = gld16(src + (8 * k + (lane >> 3)) * kHeadDim);
#pragma unroll
    for (int k = 0; k < W / 8; ++k) *(u32x4*)(rows + (8 * k + (lane >> 3)) * kLdsRow + 8 * (lane & 7)) = x[k];
  } else {
    const uint8_t* p = t.slot(src_kind, src_idx) + (int64_t)W * kHeadDim * 2;
    const int r = lane & 15, q = lane >> 4;
    if constexpr (W == 8) {   // piece (cp, q < 2, r): tokens 4 q + j, channels 16 (2 cp + e) + r
      const u32x4 x = gld16(p + (2 * h * 32 + lane) * 16);
      const int cpl = lane >> 5, qq = q & 1;
#pragma unroll
      for (int e = 0; e < 2; ++e)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          rows[(4 * qq + j) * kLdsRow + 16 * (2 * cpl + e) + r] = (uint16_t)(x[2 * e + (j >> 1)] >> (16 * (j & 1)));
    } else {                  // chunk (kt, cb): tokens tok(kt, q, 0..7), channel 16 cb + r
      u32x4 x[W / 8];
#pragma unroll
      for (int c = 0; c < W / 8; ++c) x[c] = gld16(p + (((c >> 2) * 8 + 4 * h + (c & 3)) * 64 + lane) * 16);
#pragma unroll
      for (int c = 0; c < W / 8; ++c)
#pragma unroll
        for (int j = 0; j < 8; ++j)
          rows[v_tok(c >> 2, q, j) * kLdsRow + 16 * (c & 3) + r] = (uint16_t)(x[c][j >> 1] >> (16 * (j & 1)));
    }
  }
}

// Column piece of a value part: lane (q, r) of block c (8-token windows: lane (cp,
// q < 2, r), element 4 e + j: token 4 q + j, channel 16 (2 cp + e) + r).
template <int W>
__device__ __forceinline__ uint16_t row_value(const uint16_t* rows, int c, int lane, int j) {
  const int r = lane & 15, q = lane >> 4;
  if constexpr (W == 8)
    return rows[(4 * (q & 1) + (j & 3)) * kLdsRow + 16 * (2 * (lane >> 5) + (j >> 2)) + r];
  else
    return rows[v_tok(c >> 2, q, j) * kLdsRow + 16 * (c & 3) + r];
}

template <int W>
__device__ __forceinline__ void store_value_codes(const Geometry& G, const PartLds<W>& sm, uint8_t* rec, int nb,
                                                  int h, int lane) {
  constexpr int NGH = 64 / value_group<W>();   // value groups of a token in one half
  uint8_t* vc = rec + G.qcodes_bytes;
  const int q = lane >> 4;
  if constexpr (W == 8) {
    const int cpl = lane >> 5, ln = lane & 31, p0 = 8 * cpl + 4 * (q & 1);   // entries (group, token)
    GroupParams p[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) p[j] = sm.gp[p0 + j];
    const uint32_t wd = entry_codes(
        nb, [&](int j) { return bf16_to_f32(row_value<8>(sm.rows, 0, lane, j)); }, [&](int j) { return p[j & 3]; });
    const uint32_t other = (uint32_t)__shfl_xor((int)wd, 32, 64);
    if (nb == 4) *(uint32_t*)(vc + ln * 16 + 4 * (2 * h + cpl)) = wd;
    else if (cpl == 0) *(uint32_t*)(vc + ln * 8 + 4 * h) = wd | (other << 8);
  } else {
#pragma unroll
    for (int kt = 0; kt < W / 32; ++kt) {
      uint32_t wds[4];
#pragma unroll
      for (int vgl = 0; vgl < NGH; ++vgl) {
        // parameters of the lane's 8 tokens tok(kt, q, j): two runs of four
        const int t0 = W * vgl + 32 * kt + 4 * q;
        GroupParams p[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) p[j] = sm.gp[t0 + 16 * (j >> 2) + (j & 3)];
#pragma unroll
        for (int c = 0; c < 4 / NGH; ++c) {
          const int cl = vgl * (4 / NGH) + c;
          if constexpr (W == 64) asm volatile("" ::: "memory");   // one entry's values at a time (registers)
          wds[cl] = entry_codes(
              nb, [&](int j) { return bf16_to_f32(row_value<W>(sm.rows, 4 * kt + cl, lane, j)); },
              [&](int j) { return p[j]; });
        }
      }
      if (nb == 4)
        *(u32x4*)(vc + ((2 * kt + h) * 64 + lane) * 16) = (u32x4){wds[0], wds[1], wds[2], wds[3]};
      else
        *(uint2*)(vc + (kt * 64 + lane) * 16 + 8 * h) = make_uint2(wds[0] | (wds[1] << 8), wds[2] | (wds[3] << 8));
    }
  }
}

template <int W>
__device__ __forceinline__ void quantize_values(const Task& t, const WorkEntry& ent, PartLds<W>& sm,
                                                int32_t* counts, int h, int lane) {
  const Geometry& G = t.a.g;
  constexpr int GV = value_group<W>();
  constexpr int NGH = 64 / GV;
  constexpr int K = W / 8;          // rows a lane reads: token 8 k + (lane >> 3), channels 8 (lane & 7) .. + 7
  constexpr int LG = GV / 8;        // lanes of a group (4 or 8)
  const int nb = ent.v[4];
  stage_values<W>(t, ent.v[0], ent.v[1], ent.v[2], h, lane, sm.rows);
  lds_order();
  uint8_t* rec = t.record(ent.v[3]);
  // extremes of every (token, group): in the lane over its 8 channels, then over
  // the group's lanes; lane l of a group keeps row k = l % LG
  float lo = 0.f, hi = 0.f;
#pragma unroll
  for (int k = 0; k < K; ++k) {
    const u32x4 v = *(const u32x4*)(sm.rows + (8 * k + (lane >> 3)) * kLdsRow + 8 * (lane & 7));
    float mn = elem_f32(v, 0), mx = mn;
#pragma unroll
    for (int j = 1; j < 8; ++j) {
      const float f = elem_f32(v, j);
      mn = fminf(mn, f);
      mx = fmaxf(mx, f);
    }
    mn = fminf(mn, dpp<kXor1>(mn));
    mx = fmaxf(mx, dpp<kXor1>(mx));
    mn = fminf(mn, dpp<kXor2>(mn));
    mx = fmaxf(mx, dpp<kXor2>(mx));
    if constexpr (LG == 8) {
      mn = fminf(mn, dpp<kXor7>(mn));
      mx = fmaxf(mx, dpp<kXor7>(mx));
    }
    const bool mine = (lane & (LG - 1)) == k;
    lo = mine ? mn : lo;
    hi = mine ? mx : hi;
  }
  static_assert(K <= LG, "one group per lane at most");
  const int k = lane & (LG - 1);
  if (k < K) {
    const int tok = 8 * k + (lane >> 3), vgl = LG == 8 ? 0 : (lane >> 2) & 1;
    uint16_t zb, sb;
    group_params(lo, hi, nb, &sm.gp[W * vgl + tok], &zb, &sb, counts);
    uint8_t* mv = rec + meta_v_elem(G, tok, NGH * h + vgl);
    *(uint16_t*)mv = sb;
    *(uint16_t*)(mv + meta_v_zero_delta(G)) = zb;
  }
  lds_order();
  store_value_codes<W>(G, sm, rec, nb, h, lane);
  lds_order();   // the rows are read before a task that follows stages its own
}

// ---- promotions and admissions ---------------------------------------------

// RNE_bf16 of a value whose fp32 rounding is f (off: f differs from it, above: it lies
// above f): f is on the value's side of every bf16 tie unless f is that tie itself.
__device__ __forceinline__ uint32_t bf16_of(float f, bool off, bool above) {
  uint32_t u = __float_as_uint(f);
  const bool tie = (u & 0xFFFFu) == 0x8000u && off;
  u += tie ? (above == (f > 0.f) ? 1u : ~0u) : 0u;
  return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// RNE_bf16(z + s c): s c is exact in fp32 (11-bit scale, 4-bit code); the sum is
// rounded to fp32 with its error e (two-sum), so the result is that of one rounding of
// the exact value.  (Sums are multiples of 2^-24.)
__device__ __forceinline__ uint32_t dequant_bf16(uint16_t zb, uint16_t sb, uint32_t code) {
  const float z = (float)__builtin_bit_cast(_Float16, zb), s = (float)__builtin_bit_cast(_Float16, sb);
  const float p = s * (float)code;
  const float f = z + p;
  const float pp = f - z;
  const float e = (z - (f - pp)) + (p - pp);
  return bf16_of(f, e != 0.f, e > 0.f);
}

// 8 bf16 values z_j + s_j c_j (one rounding each) packed for a 16-byte store
template <int NB>
__device__ __forceinline__ u32x4 dequant8(uint32_t wd, int ee, u32x4 s8, u32x4 z8) {
  constexpr uint32_t mask = (1u << NB) - 1u;
  u32x4 out;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t sw = s8[i], zw = z8[i];
    const uint32_t c = wd >> (NB * (4 * ee + i));
    out[i] = dequant_bf16((uint16_t)zw, (uint16_t)sw, c & mask) |
             (dequant_bf16((uint16_t)(zw >> 16), (uint16_t)(sw >> 16), (c >> 16) & mask) << 16);
  }
  return out;
}

// z + s c (exact in float64) of key entry e (channels 32 (e & 3) + 8 q .. + 7 of
// token 16 (e >> 2) + r) for lane L = 16 q + r
template <int NB>
__device__ __forceinline__ void key_entry_f64(const Geometry& G, const uint8_t* rec, int e, int L,
                                              double (&x)[8]) {
  constexpr int PER = 4 / NB;
  constexpr uint32_t mask = (1u << NB) - 1u;
  const int q = L >> 4, word = e / PER, ee = e % PER;
  const uint32_t wd = *(const uint32_t*)(rec + ((int64_t)(word >> 2) * 64 + L) * 16 + (word & 3) * 4);
  const uint8_t* ps = rec + meta_k_off(G) + 2 * (32 * (e & 3) + 8 * q);
  const u32x4 s8 = *(const u32x4*)ps, z8 = *(const u32x4*)(ps + 2 * kHeadDim);
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const uint32_t code = (wd >> (o * 16 + NB * (4 * ee + i))) & mask;
      const double sj = fp16_bits_to_f64((uint16_t)(s8[i] >> (16 * o)));
      const double zj = fp16_bits_to_f64((uint16_t)(z8[i] >> (16 * o)));
      x[2 * i + o] = zj + sj * (double)code;
    }
}

// Promoted bf16 keys of entry e with RoPE: the dequantized pre-RoPE keys of the
// entry and of its partner entry e ^ 2 (channels +- 64) rotated to position
// p0 + token: channel i < 64 takes x_i cos - x_{i+64} sin, channel i + 64 takes
// x_{i+64} cos + x_i sin, products and sums rounded in float64, then RNE to bf16.
template <int NB>
__device__ __forceinline__ u32x4 rope_key8(const Geometry& G, const uint8_t* rec, int e, int L, int p0) {
#pragma clang fp contract(off)
  double x[8], y[8];
  key_entry_f64<NB>(G, rec, e, L, x);
  key_entry_f64<NB>(G, rec, e ^ 2, L, y);
  const int kb = e & 3, q = L >> 4, r = L & 15;
  const int p = p0 + 16 * (e >> 2) + r;
  uint32_t outw[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    uint32_t pair = 0;
#pragma unroll
    for (int o = 0; o < 2; ++o) {
      const int j = 2 * i + o;
      const float2 cs = rope_cs(G, p, (32 * kb + 8 * q + j) & 63);
      const double t1 = x[j] * (double)cs.x, t2 = y[j] * (double)cs.y;
      const double v = kb < 2 ? t1 - t2 : t1 + t2;
      const float f = (float)v;
      pair |= bf16_of(f, (double)f != v, v > (double)f) << (16 * o);
    }
    outw[i] = pair;
  }
  return (u32x4){outw[0], outw[1], outw[2], outw[3]};
}

// Promotion of entry ei (of area's W / 4) of a (window, KV head) from its quantized
// record: lane L takes its code word, 8 scales and 8 zeros and writes 8 bf16 values to
// the same (entry, lane) position of the bf16 slot.
template <int W, int NB, bool ROPE>
__device__ __forceinline__ void promote_entry(const Geometry& G, const uint8_t* rec, uint8_t* dp, int area, int ei,
                                              int L, int p0) {
  constexpr int PER = 4 / NB;
  if (ROPE && area == 0) {
    *(u32x4*)(dp + ((int64_t)ei * 64 + L) * 16) = rope_key8<NB>(G, rec, ei, L, p0);
    return;
  }
  const int ng = kHeadDim / G.G;
  const int q = L >> 4, r = L & 15;
  const int word = ei / PER;
  const uint32_t wd = *(const uint32_t*)(rec + area * G.qcodes_bytes +
                                         ((int64_t)(word >> 2) * 64 + L) * 16 + (word & 3) * 4);
  const uint8_t* ps;
  u32x4 s8, z8;
  if (area == 0) {   // key entry (tb, kb): channels 32 kb + 8 q .. + 7
    ps = rec + meta_k_off(G) + 2 * (32 * (ei & 3) + 8 * q);
    s8 = *(const u32x4*)ps;
    z8 = *(const u32x4*)(ps + 2 * kHeadDim);
  } else {           // value entry (kt, cb): tokens tok(kt, q, 0..7), channel 16 cb + r
    const int c = 16 * (ei & 7) + r;
    ps = rec + meta_v_off(G) + (((ei >> 3) * 4 + q) * ng + c / G.G) * 32;
    s8 = *(const u32x4*)ps;
    z8 = *(const u32x4*)(ps + 16);
  }
  const int64_t off = (area == 0 ? 0 : (int64_t)W * kHeadDim * 2) + ((int64_t)ei * 64 + L) * 16;
  *(u32x4*)(dp + off) = dequant8<NB>(wd, ei % PER, s8, z8);
}

// Promotion of one part of a (window, KV head).
template <int W, int NB, bool ROPE>
__device__ __forceinline__ void promote_record(const Geometry& G, const uint8_t* rec, uint8_t* dp, int area, int h,
                                               int L, int p0) {
#pragma unroll 4   // the loads of four entries in one round
  for (int o = 0; o < W / 8; ++o) {
    const int ei = area == 0 ? 4 * (o >> 1) + key_block<ROPE>(h, o & 1) : 8 * (o >> 2) + 4 * h + (o & 3);
    promote_entry<W, NB, ROPE>(G, rec, dp, area, ei, L, p0);
  }
}

// Promotion of one part of an 8-token window from its record: a lane writes one
// 16-byte piece (keys: block kb, lane (q, r < 8); values: block pair cp, lane
// (q < 2, r), elements 4 e + j).
template <int NB>
__device__ __forceinline__ void promote_record8(const Geometry& G, const uint8_t* rec, uint8_t* dp, int area, int h,
                                                int lane) {
  constexpr int LB = NB == 4 ? 16 : 8;
  if (area == 0) {
    const int kb = 2 * h + (lane >> 5), q = (lane >> 3) & 3, r = lane & 7;
    const int word = NB == 4 ? kb : kb >> 1, ee = NB == 4 ? 0 : kb & 1;
    const uint32_t wd = *(const uint32_t*)(rec + (q * 8 + r) * LB + 4 * word);
    const uint8_t* ps = rec + meta_k_off(G) + 2 * (32 * kb + 8 * q);
    const u32x4 s8 = *(const u32x4*)ps, z8 = *(const u32x4*)(ps + 2 * kHeadDim);
    *(u32x4*)(dp + ((kb * 4 + q) * 8 + r) * 16) = dequant8<NB>(wd, ee, s8, z8);
  } else {
    const int cp = 2 * h + (lane >> 5), q = (lane >> 4) & 1, r = lane & 15;
    const int word = NB == 4 ? cp : cp >> 1, ee = NB == 4 ? 0 : cp & 1;
    const uint32_t wd = *(const uint32_t*)(rec + G.qcodes_bytes + (q * 16 + r) * LB + 4 * word);
    // value group cp: scales then zero points of tokens 4 q .. 4 q + 3
    const u32x4 m = *(const u32x4*)(rec + meta_v_off(G) + (q * 4 + cp) * 16);
    const uint32_t s01 = m[0], s23 = m[1], z01 = m[2], z23 = m[3];
    *(u32x4*)(dp + (int64_t)8 * kHeadDim * 2 + ((cp * 2 + q) * 16 + r) * 16) =
        dequant8<NB>(wd, ee, (u32x4){s01, s23, s01, s23}, (u32x4){z01, z23, z01, z23});
  }
}

template <int W, bool ROPE>
__device__ __forceinline__ void promote_part(const Task& t, const WorkEntry& ent, MigrateLds<W>& sm, int area, int h,
                                             int lane) {
  const Geometry& G = t.a.g;
  const int w = ent.v[0], src_kind = ent.v[1], src_idx = ent.v[2], nb = ent.v[4];
  uint8_t* dp = t.slot(SRC_FSLOT, ent.v[3]);
  constexpr int64_t VB = (int64_t)W * kHeadDim * 2;   // value part of a slot
  if (src_kind == SRC_QSLOT) {
    const uint8_t* rec = t.record(src_idx);
    if constexpr (W == 8) {
      if (nb == 4) promote_record8<4>(G, rec, dp, area, h, lane);
      else promote_record8<2>(G, rec, dp, area, h, lane);
    } else {
      const int p0 = G.sink + w * W;   // position of the window's first token
      if (nb == 4) promote_record<W, 4, ROPE>(G, rec, dp, area, h, lane, p0);
      else promote_record<W, 2, ROPE>(G, rec, dp, area, h, lane, p0);
    }
  } else if (area == 0) {
    u32x4 x[key_pieces<W>()];
    load_keys<W, ROPE>(t, w, src_kind, src_idx, h, lane, x);
#pragma unroll
    for (int pc = 0; pc < key_pieces<W>(); ++pc) *(u32x4*)(dp + key_piece_off<W, ROPE>(h, pc, lane)) = x[pc];
  } else {
    constexpr int NP = W == 8 ? 1 : W / 8;
    auto off = [&](int c) {
      return W == 8 ? (int64_t)(2 * h * 32 + lane) * 16
                    : (int64_t)(((c >> 2) * 8 + 4 * h + (c & 3)) * 64 + lane) * 16;
    };
    if (src_kind == SRC_RING) {
      const uint8_t* sp = t.slot(SRC_RING, src_idx) + VB;
      u32x4 x[NP];
#pragma unroll
      for (int c = 0; c < NP; ++c) x[c] = gld16(sp + off(c));
#pragma unroll
      for (int c = 0; c < NP; ++c) *(u32x4*)(dp + VB + off(c)) = x[c];
    } else {   // the prompt's rows become columns through LDS
      uint16_t* rows = sm.v[h].rows;
      stage_values<W>(t, w, src_kind, src_idx, h, lane, rows);
      lds_order();
#pragma unroll
      for (int c = 0; c < NP; ++c) {
        uint32_t d[4];
#pragma unroll
        for (int i = 0; i < 4; ++i)
          d[i] = (uint32_t)row_value<W>(rows, c, lane, 2 * i) | ((uint32_t)row_value<W>(rows, c, lane, 2 * i + 1) << 16);
        *(u32x4*)(dp + VB + off(c)) = (u32x4){d[0], d[1], d[2], d[3]};
      }
      lds_order();
    }
  }
}

// Migrations of one routing event, one (window, KV head) per workgroup pass and one
// part per wave.  The first a.n_quant_blocks workgroups take the quantizations, the
// others the promotions / admissions, so a workgroup knows its list before the
// counts arrive and reads the counts and its first entry in one round.  A
// promotion whose bf16 slot is being vacated by a quantization in the same event
// (dep >= 0) runs in that quantization's waves right after it, part by part, so
// the slot is read before it is overwritten without any ordering across waves.
// Bound by memory for a prompt and by the latency of one task for a routing event.
// Admission of a 32K prompt (8 KV heads, 204 windows copied, 307 quantized to int4;
// 106 MB moved): 78.7 -> 24.8 us; four 64K prompts (964 MB): 582 -> 192 us, 5.0 TB/s,
// against one looping workgroup per part with every code decided in float64.  (Events of
// few windows, where one wave would do what four did: k_migrate_few.)
// At most 80 VGPRs without RoPE and with windows of 8 or 32 tokens (six waves per
// SIMD): a migration workgroup then fits on a compute unit beside two attention
// workgroups of up to 216, so routing on its own stream does not hold back the
// attention of the next layers.
template <int W, bool ROPE>
constexpr int migrate_waves_per_simd() { return W == 64 ? (ROPE ? 3 : 4) : (ROPE ? 5 : 6); }

template <int W, bool ROPE>
__global__ __launch_bounds__(kMigrateThreads, (migrate_waves_per_simd<W, ROPE>())) void k_migrate(MigrateArgs a) {
  const Geometry& G = a.g;
  const int b = blockIdx.y + touch_kernargs<sizeof(MigrateArgs)>();
  __shared__ __attribute__((aligned(16))) MigrateLds<W> sm;
  // Everything up to the first task in two rounds of loads without a branch between
  // them: the arguments; then the count, the first entry and the gate word.  (A
  // routing batch whose wait for the cache stream timed out moves nothing.)
  uint8_t* ub = a.base[blockIdx.z] + (int64_t)b * a.L.unit_bytes;
  int32_t* counts = (int32_t*)(ub + a.L.counts);
  const int32_t* plist = (const int32_t*)(ub + a.L.plist);
  const bool quant = (int)blockIdx.x < a.n_quant_blocks;
  const int stride = quant ? a.n_quant_blocks : a.n_promote_blocks;
  const int x0 = quant ? blockIdx.x : blockIdx.x - a.n_quant_blocks;
  const int32_t* list = (const int32_t*)(ub + (quant ? a.L.qlist : a.L.plist));
  const int32_t* gate = a.gate_fail ? a.gate_fail : counts;
  const int e0 = x0 / G.H_kv;
  const int n_entries = counts[quant ? CNT_QUANT : CNT_PROMOTE];
  const WorkEntry first = load_entry(list, e0 <= G.max_fq ? e0 : 0);   // lists hold max_fq + 1 entries
  const int gate_word = __hip_atomic_load(gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int n_tasks = a.gate_fail && gate_word ? 0 : n_entries * G.H_kv;
  int lane = threadIdx.x & 63;
  const int part = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int area = part >> 1, h = part & 1;
  for (int task = x0; task < n_tasks; task += stride) {
    // (keeps the lane's many addresses out of the registers that live across the
    // loop, which otherwise spill; it rarely runs twice)
    asm volatile("" : "+v"(lane));
    const WorkEntry ent = task == x0 ? first : load_entry(list, task / G.H_kv);
    const Task t{a, ub, b, task % G.H_kv};
    WorkEntry pe = ent;
    bool promote = !quant && ent.v[5] < 0;
    if (quant) {
      if (area == 0) quantize_keys<W, ROPE>(t, ent, sm.k[h], counts, h, lane);
      else quantize_values<W>(t, ent, sm.v[h], counts, h, lane);
      promote = ent.v[5] >= 0;
      if (promote) pe = load_entry(plist, ent.v[5]);
    }
    if (promote) promote_part<W, ROPE>(t, pe, sm, area, h, lane);
  }
}

// ---- routing events of a few windows ---------------------------------------
// The same migrations with half a part per wave (32- and 64-token windows, no prompt
// source): a workgroup takes the keys or the values of one (window, KV head), wave
// (h, sub) of it the key block key_block(h, sub), or of channel half h the values of
// value group sub (32-token windows) or of token block sub (64).
// Bound by latency: one task's chain of loads, reductions and codes (a task of
// k_migrate's waves is twice as long), and the float64 rotation with RoPE.  One layer's
// event after a decode step, 8 KV heads, 5 to 6 promotions and as many windows quantized
// at first, medians: 10.4 -> 5.2 us (32K, int4), 9.8 -> 5.8 (128K, 64-token windows),
// 22.9 -> 6.6 with RoPE; with four workgroups per (window, KV head) whose waves shared a
// part in barrier-separated phases 7.9, 7.1 and 15.8.
template <int W>
constexpr int few_channels() { return W == 32 ? 32 : 64; }   // of a wave's value rows (32 tokens)
template <int W>
constexpr int few_row() { return few_channels<W>() + 8; }
template <int W>
struct FewLds {    // of one wave
  uint16_t rows[32 * few_row<W>()];
  GroupParams gp[32];   // keys: channel of the block; values: token
};

template <int W, bool ROPE>
__device__ __forceinline__ void quantize_key_block(const Task& t, const WorkEntry& ent, GroupParams* gp,
                                                   int32_t* counts, int h, int sub, int lane) {
  const Geometry& G = t.a.g;
  constexpr int TB = W / 16;
  const int w = ent.v[0], nb = ent.v[4], kb = key_block<ROPE>(h, sub);
  const uint8_t* src = t.slot(ent.v[1], ent.v[2]);
  u32x4 x[TB];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) x[tb] = gld16(src + ((tb * 4 + kb) * 64 + lane) * 16);
  if constexpr (ROPE) {   // as unrotate_keys, for this block's channels of the pairs
#pragma clang fp contract(off)
    const int pb = key_block<ROPE>(h, 1 - sub), i0 = 32 * h + 8 * (lane >> 4);
    u32x4 y[TB];
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) y[tb] = gld16(src + ((tb * 4 + pb) * 64 + lane) * 16);
#pragma unroll
    for (int tb = 0; tb < TB; ++tb) {
      const int p = G.sink + w * W + 16 * tb + (lane & 15);
      u32x4 z = x[tb];
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        uint32_t zw = 0;
#pragma unroll
        for (int o = 0; o < 2; ++o) {
          const float2 cs = rope_cs(G, p, i0 + 2 * d + o);
          const float c = elem_f32(x[tb], 2 * d + o) * cs.x, s = elem_f32(y[tb], 2 * d + o) * cs.y;
          zw |= (uint32_t)f32_to_bf16_rne(sub ? c - s : c + s) << (16 * o);
        }
        z[d] = zw;
      }
      x[tb] = z;
    }
  }
  // extremes of the block's channels: lanes 2 c, 2 c + 1 of a row end with channel c
  float mn[8], mx[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) mn[j] = mx[j] = elem_f32(x[0], j);
#pragma unroll
  for (int tb = 1; tb < TB; ++tb)
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const float v = elem_f32(x[tb], j);
      mn[j] = fminf(mn[j], v);
      mx[j] = fmaxf(mx[j], v);
    }
  scatter_minmax<4, kXor8>(mn, mx, (lane & 8) != 0);
  scatter_minmax<2, kXor7>(mn, mx, (lane & 4) != 0);
  scatter_minmax<1, kXor2>(mn, mx, (lane & 2) != 0);
  const float lo = fminf(mn[0], dpp<kXor1>(mn[0])), hi = fmaxf(mx[0], dpp<kXor1>(mx[0]));
  uint8_t* rec = t.record(ent.v[3]);
  if ((lane & 1) == 0) {
    const int c = lane >> 1;   // channel of the block: 8 (lane >> 4) + (lane & 15) / 2
    uint16_t zb, sb;
    group_params(lo, hi, nb, &gp[c], &zb, &sb, counts);
    uint16_t* mk = (uint16_t*)(rec + meta_k_off(G)) + 32 * kb + c;
    mk[0] = sb;
    mk[kHeadDim] = zb;
  }
  lds_order();
  GroupParams p[8];
#pragma unroll
  for (int j = 0; j < 8; ++j) p[j] = gp[8 * (lane >> 4) + j];
#pragma unroll
  for (int tb = 0; tb < TB; ++tb) {
    const uint32_t wd =
        entry_codes(nb, [&](int j) { return elem_f32(x[tb], j); }, [&](int j) { return p[j]; });
    if (nb == 4) {
      *(uint32_t*)(rec + (tb * 64 + lane) * 16 + 4 * kb) = wd;
    } else {   // entry kb & 1 of word 2 tb + kb / 2: its bytes kb & 1 and + 2
      uint8_t* d = rec + ((tb >> 1) * 64 + lane) * 16 + (2 * (tb & 1) + (kb >> 1)) * 4 + (kb & 1);
      d[0] = (uint8_t)wd;
      d[2] = (uint8_t)(wd >> 16);
    }
  }
}

template <int W>
__device__ __forceinline__ void quantize_value_block(const Task& t, const WorkEntry& ent, FewLds<W>& sm,
                                                     int32_t* counts, int h, int sub, int lane) {
  const Geometry& G = t.a.g;
  constexpr int NC = W == 32 ? 2 : 4;              // 16-channel blocks
  constexpr int RS = few_row<W>();
  constexpr int CL = few_channels<W>() / 2;        // channels a lane reduces
  const int nb = ent.v[4], r = lane & 15, q = lane >> 4;
  const int kt = W == 32 ? 0 : sub, cl0 = W == 32 ? 2 * sub : 0;   // token block, first block of the half
  const uint8_t* src = t.slot(ent.v[1], ent.v[2]) + (int64_t)W * kHeadDim * 2;
  u32x4 x[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c) x[c] = gld16(src + ((kt * 8 + 4 * h + cl0 + c) * 64 + lane) * 16);
#pragma unroll
  for (int c = 0; c < NC; ++c)
#pragma unroll
    for (int j = 0; j < 8; ++j)
      sm.rows[v_tok(0, q, j) * RS + 16 * c + r] = (uint16_t)(x[c][j >> 1] >> (16 * (j & 1)));
  lds_order();
  uint8_t* rec = t.record(ent.v[3]);
  {   // extremes of token lane / 2: half its channels in the lane, then the two halves
    float mn = 0.f, mx = 0.f;
#pragma unroll
    for (int k = 0; k < CL / 8; ++k) {
      const u32x4 v = *(const u32x4*)(sm.rows + (lane >> 1) * RS + CL * (lane & 1) + 8 * k);
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const float f = elem_f32(v, j);
        mn = k + j == 0 ? f : fminf(mn, f);
        mx = k + j == 0 ? f : fmaxf(mx, f);
      }
    }
    mn = fminf(mn, dpp<kXor1>(mn));
    mx = fmaxf(mx, dpp<kXor1>(mx));
    if ((lane & 1) == 0) {
      uint16_t zb, sb;
      group_params(mn, mx, nb, &sm.gp[lane >> 1], &zb, &sb, counts);
      uint8_t* mv = rec + meta_v_elem(G, 32 * kt + (lane >> 1), W == 32 ? 2 * h + sub : h);
      *(uint16_t*)mv = sb;
      *(uint16_t*)(mv + meta_v_zero_delta(G)) = zb;
    }
  }
  lds_order();
  GroupParams p[8];   // of the lane's 8 tokens tok(kt, q, j): two runs of four
#pragma unroll
  for (int j = 0; j < 8; ++j) p[j] = sm.gp[v_tok(0, q, j)];
  uint32_t wds[NC];
#pragma unroll
  for (int c = 0; c < NC; ++c)
    wds[c] = entry_codes(
        nb, [&](int j) { return elem_f32(x[c], j); }, [&](int j) { return p[j]; });
  uint8_t* vc = rec + G.qcodes_bytes;
  if constexpr (W == 32) {
    if (nb == 4) *(uint2*)(vc + (h * 64 + lane) * 16 + 8 * sub) = make_uint2(wds[0], wds[1]);
    else *(uint32_t*)(vc + lane * 16 + 8 * h + 4 * sub) = wds[0] | (wds[1] << 8);
  } else {
    if (nb == 4)
      *(u32x4*)(vc + ((2 * kt + h) * 64 + lane) * 16) = (u32x4){wds[0], wds[1], wds[2], wds[3]};
    else
      *(uint2*)(vc + (kt * 64 + lane) * 16 + 8 * h) = make_uint2(wds[0] | (wds[1] << 8), wds[2] | (wds[3] << 8));
  }
  lds_order();   // the rows are read before a task that follows stages its own
}

template <int W, bool ROPE>
__device__ __forceinline__ void promote_half_part(const Task& t, const WorkEntry& ent, int area, int h, int sub,
                                                  int lane) {
  const Geometry& G = t.a.g;
  const int w = ent.v[0], src_kind = ent.v[1], src_idx = ent.v[2], nb = ent.v[4];
  uint8_t* dp = t.slot(SRC_FSLOT, ent.v[3]);
  constexpr int NE = W / 16;   // entries (chunks) of half a part
  auto entry = [&](int o) {
    return area == 0 ? 4 * o + key_block<ROPE>(h, sub) : W == 32 ? 4 * h + 2 * sub + o : 8 * sub + 4 * h + o;
  };
  if (src_kind == SRC_QSLOT) {
    const uint8_t* rec = t.record(src_idx);
    const int p0 = G.sink + w * W;   // position of the window's first token
#pragma unroll
    for (int o = 0; o < NE; ++o) {
      if (nb == 4) promote_entry<W, 4, ROPE>(G, rec, dp, area, entry(o), lane, p0);
      else promote_entry<W, 2, ROPE>(G, rec, dp, area, entry(o), lane, p0);
    }
  } else {
    const uint8_t* sp = t.slot(SRC_RING, src_idx);
    const int64_t base = area == 0 ? 0 : (int64_t)W * kHeadDim * 2;
    u32x4 x[NE];
#pragma unroll
    for (int o = 0; o < NE; ++o) x[o] = gld16(sp + base + ((int64_t)entry(o) * 64 + lane) * 16);
#pragma unroll
    for (int o = 0; o < NE; ++o) *(u32x4*)(dp + base + ((int64_t)entry(o) * 64 + lane) * 16) = x[o];
  }
}

template <int W, bool ROPE>
__global__ __launch_bounds__(kMigrateThreads, (migrate_waves_per_simd<W, ROPE>())) void k_migrate_few(MigrateArgs a) {
  const Geometry& G = a.g;
  const int b = blockIdx.y + touch_kernargs<sizeof(MigrateArgs)>();
  __shared__ __attribute__((aligned(16))) FewLds<W> sm[4];
  uint8_t* ub = a.base[blockIdx.z] + (int64_t)b * a.L.unit_bytes;   // (the rounds of loads: as k_migrate)
  int32_t* counts = (int32_t*)(ub + a.L.counts);
  const int32_t* plist = (const int32_t*)(ub + a.L.plist);
  const bool quant = (int)blockIdx.x < a.n_quant_blocks;
  const int stride = quant ? a.n_quant_blocks : a.n_promote_blocks;
  const int x0 = quant ? blockIdx.x : blockIdx.x - a.n_quant_blocks;
  const int32_t* list = (const int32_t*)(ub + (quant ? a.L.qlist : a.L.plist));
  const int32_t* gate = a.gate_fail ? a.gate_fail : counts;
  const int per = 2 * G.H_kv;   // tasks of an entry
  const int e0 = x0 / per;
  const int n_entries = counts[quant ? CNT_QUANT : CNT_PROMOTE];
  const WorkEntry first = load_entry(list, e0 <= G.max_fq ? e0 : 0);
  const int gate_word = __hip_atomic_load(gate, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  const int n_tasks = a.gate_fail && gate_word ? 0 : n_entries * per;
  int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int h = wave >> 1, sub = wave & 1;
  for (int task = x0; task < n_tasks; task += stride) {
    asm volatile("" : "+v"(lane));   // (as in k_migrate)
    const WorkEntry ent = task == x0 ? first : load_entry(list, task / per);
    const int rest = task % per, area = rest / G.H_kv;
    const Task t{a, ub, b, rest - area * G.H_kv};
    WorkEntry pe = ent;
    bool promote = !quant && ent.v[5] < 0;
    if (quant) {
      if (area == 0) quantize_key_block<W, ROPE>(t, ent, sm[wave].gp, counts, h, sub, lane);
      else quantize_value_block<W>(t, ent, sm[wave], counts, h, sub, lane);
      promote = ent.v[5] >= 0;
      if (promote) {
        pe = load_entry(plist, ent.v[5]);
        // with RoPE a wave also read the block that its partner overwrites (the task is
        // the workgroup's: all four waves come here)
        if constexpr (ROPE) __syncthreads();
      }
    }
    if (promote) promote_half_part<W, ROPE>(t, pe, area, h, sub, lane);
  }
}

// Copy the prompt's sink tokens [0, n_sink) and its tail [tail0, src_T) into the
// sink slots and the recent ring: one thread per (token, 8 channels, keys or
// values), 8 tokens a workgroup, so that a copy is one round of loads.
__global__ __launch_bounds__(256) void k_pack_tokens(PackArgs a) {
  const Geometry& G = a.g;
  const int g = blockIdx.y, b = blockIdx.z, tid = threadIdx.x;
  const int i = blockIdx.x * 8 + (tid & 127) / 16, c = 8 * (tid & 15);
  const bool value = tid >= 128;
  const int t = i < a.n_sink ? i : a.tail0 + (i - a.n_sink);
  if (t >= a.src_T) return;
  uint8_t* ub = a.base + (int64_t)b * a.L.unit_bytes;
  const int64_t row = ((int64_t)b * G.H_kv + g) * a.src_T + t;
  const int s = t < G.sink ? t : t - G.sink;            // token within its region
  const int w = s / G.W, tt = s % G.W;
  uint8_t* dp = ub + (t < G.sink ? a.L.sinkp + (int64_t)w * G.fslot_bytes
                                 : a.L.ring + (int64_t)(w % G.NR) * G.fslot_bytes) + g * G.fhead_bytes;
  const u32x4 x = gld16((value ? a.src_v : a.src_k) + row * kHeadDim + c);
  if (!value) {
    *(u32x4*)(dp + k_elem_off(G.W, tt, c)) = x;         // 8 channels of a token lie together
  } else {
#pragma unroll
    for (int j = 0; j < 8; ++j)
      *(uint16_t*)(dp + v_elem_off(G.W, tt, c + j)) = (uint16_t)(x[j >> 1] >> (16 * (j & 1)));
  }
}

// The form with half a part per wave: two workgroups per (window, KV head) of the event's
// windows or of a sixteenth of the kept ones, at most eight, which most events after a
// single step stay below (511 windows kept: with four the mean event took 7.0 instead of
// 5.5 us; 40 kept: eight cost 0.04 us an event in idle workgroups).  For launches of a
// wave of workgroups on the chip (six a compute unit) and some; larger ones are mostly
// idle workgroups, whose number then counts, and take the form with fewer.  So does a
// batch that runs beside attention, which its work delays and its latency does not,
// except with RoPE (32K int4, eight layers, tiers turning over after every step: 21.5 us a
// step against 22.4 with half a part per wave; with RoPE, under the queue-level wait, 43.6
// and 31.6.  On one stream 68.5 and 42.4, with RoPE 153 and 57.5).
constexpr int kFewBlocks = 2048, kFewWindows = 8;
static int few_blocks(const Geometry& g, int entries) {
  return 2 * g.H_kv * std::max({entries, std::min(g.max_fq / 16, kFewWindows), 1});
}

// Workgroups for `entries` windows: one per (window, KV head), at most 16384
// (larger events loop).  A prompt's migrations (2456 quantizations and 1632
// admissions at 32K with 8 KV heads) then run without a serial chain of tasks in
// a workgroup: 1024 looping workgroups took 79 us there, ten tasks each.
static int migrate_blocks(const Geometry& g, int entries) {
  const int64_t n = (int64_t)entries * g.H_kv;
  return n < 1 ? 1 : (n > 16384 ? 16384 : (int)n);
}

// beside: on the routing stream beside attention (the device-side gate)
hipError_t launch_migrate(MigrateArgs a, int max_quant, int max_promote, bool beside, hipStream_t st) {
  const Geometry& g = a.g;
  const int fq = few_blocks(g, max_quant), fp = few_blocks(g, max_promote);
  if (!a.src_k && g.W != 8 && (!beside || g.rope) && (int64_t)(fq + fp) * g.B * a.n_units <= kFewBlocks) {
    a.n_quant_blocks = fq;
    a.n_promote_blocks = fp;
    const dim3 grid(fq + fp, g.B, a.n_units);
    if (g.rope && g.W == 32) hipLaunchKernelGGL((k_migrate_few<32, true>), grid, dim3(kMigrateThreads), 0, st, a);
    else if (g.rope) hipLaunchKernelGGL((k_migrate_few<64, true>), grid, dim3(kMigrateThreads), 0, st, a);
    else if (g.W == 32) hipLaunchKernelGGL((k_migrate_few<32, false>), grid, dim3(kMigrateThreads), 0, st, a);
    else hipLaunchKernelGGL((k_migrate_few<64, false>), grid, dim3(kMigrateThreads), 0, st, a);
    return hipGetLastError();
  }
  a.n_quant_blocks = migrate_blocks(g, max_quant);
  a.n_promote_blocks = migrate_blocks(g, max_promote);
  const dim3 grid(a.n_quant_blocks + a.n_promote_blocks, g.B, a.n_units);
  if (g.rope) {
    if (g.W == 32) hipLaunchKernelGGL((k_migrate<32, true>), grid, dim3(kMigrateThreads), 0, st, a);
    else hipLaunchKernelGGL((k_migrate<64, true>), grid, dim3(kMigrateThreads), 0, st, a);
  } else {
    if (g.W == 8) hipLaunchKernelGGL((k_migrate<8, false>), grid, dim3(kMigrateThreads), 0, st, a);
    else if (g.W == 32) hipLaunchKernelGGL((k_migrate<32, false>), grid, dim3(kMigrateThreads), 0, st, a);
    else hipLaunchKernelGGL((k_migrate<64, false>), grid, dim3(kMigrateThreads), 0, st, a);
  }
  return hipGetLastError();
}
// Registers per lane and LDS bytes per workgroup of the migration kernels a geometry
// launches (the larger of its forms).
hipError_t migrate_footprint(const Geometry& g, int* vgprs, size_t* lds) {
  auto ptr = [](auto* k) { return reinterpret_cast<const void*>(k); };
  const void* ks[2] = {nullptr, nullptr};
  if (g.W == 8) ks[0] = ptr(&k_migrate<8, false>);
  else if (g.W == 32 && g.rope) ks[0] = ptr(&k_migrate<32, true>), ks[1] = ptr(&k_migrate_few<32, true>);
  else if (g.W == 32) ks[0] = ptr(&k_migrate<32, false>), ks[1] = ptr(&k_migrate_few<32, false>);
  else if (g.rope) ks[0] = ptr(&k_migrate<64, true>), ks[1] = ptr(&k_migrate_few<64, true>);
  else ks[0] = ptr(&k_migrate<64, false>), ks[1] = ptr(&k_migrate_few<64, false>);
  *vgprs = 0;
  *lds = 0;
  for (const void* k : ks) {
    if (!k) continue;
    hipFuncAttributes fa;
    hipError_t e = hipFuncGetAttributes(&fa, k);
    if (e != hipSuccess) return e;
    *vgprs = std::max(*vgprs, fa.numRegs);
    *lds = std::max(*lds, (size_t)fa.sharedSizeBytes);
  }
  return hipSuccess;
}
hipError_t launch_pack_tokens(const PackArgs& a, hipStream_t st) {
  const int n = a.n_sink + (a.src_T - a.tail0);
  if (n <= 0) return hipSuccess;
  hipLaunchKernelGGL(k_pack_tokens, dim3((n + 7) / 8, a.g.H_kv, a.g.B), dim3(256), 0, st, a);
  return hipGetLastError();
}

}  // namespace qv
