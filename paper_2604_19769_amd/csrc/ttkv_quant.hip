// Row conversion kernels: append (Sec. 4.1), Q_8bit / Q_4bit (Sec. 4.2), the eviction path's decompress ->
// re-quantize, and the running key sums behind block identification.  Compiled with -ffp-contract=off: every fp32
// step of the recipes is one IEEE operation (round to nearest even), so codes, scales and zeros are reproducible
// bit for bit.
//
// Work unit of the row kernel: up to 64 consecutive rows of ONE destination block, one KV head, K or V.  A 16-lane
// group converts one row at a time (8 channels per lane).  Block and record look-ups happen once per unit on the scalar
// unit, without a division (entry and KV head are the grid's, ring blocks come by a multiplication: a unit of 64 rows is
// short, and its look-ups took 1.5 of its 3 us; 2 x 32 heads x 8192 tokens into fp16 + int4 75.6 -> 73.2 us, 8 x 32768 into
// bf16 + K int8 / V int4 channel-major 43.3 -> 42.1, three tiers deep with sums 162.0 -> 158.7); source and destination
// formats are compile-time inside the unit; all of a unit's loads are in flight before the first conversion.  Where keys
// also feed block summaries a unit is a whole destination block (see sum_rows).  Bound: memory for the plain copies (5.3 TB/s of read + write), fp16 -> int8
// (5.2) and fp16 -> int4 (4.8; a copy of 2 GiB reaches 4.9); a second recipe in front (int4 through int8) issues 139
// vector instructions per four rows, as long as their bytes take: 88 us for 430 MB (4.9 TB/s; 103 with 176 instructions),
// with key sums about 100 (153).  The one generic body before -- a 64-bit address and a division by the block
// size per row, a near-tie branch per element, exchanges through LDS -- reached 3.0 for int4: tiering 2 x 32 heads x
// 8192 tokens into fp16 + int4 105.6 -> 77.4 us; 8 heads x 32768 tokens into fp16 + K int8 / V int4 channel-major, one
// launch instead of two, 60 -> 43.5 us.
#include "ttkv_internal.h"

#include <hip/hip_fp16.h>

#include <algorithm>

namespace ttkv {

namespace {

constexpr int CHUNK = 64;             // rows of a unit; block sizes are multiples of it
constexpr int SUM_THREADS = 512;      // workgroup of small launches that also keep key sums (256 threads in large ones);
                                      // between two barriers it converts a row per 16 threads
constexpr int NO_STORE = -1;          // destination "format" of a unit that only feeds the key sums

__device__ __forceinline__ float h2f(uint16_t h) { return __half2float(__ushort_as_half(h)); }
__device__ __forceinline__ uint16_t f2h(float f) { return __half_as_ushort(__float2half_rn(f)); }

// ---------------------------------------------------------------- the recipes, eight channels per lane
// The codes of Sec. 4.2 are rint(RN(y / s)), one IEEE division per element.  The divisor is an fp16 number common to
// the group, so its correctly rounded reciprocal r is formed once, and q = y r, q + (y - q s) r (two fused steps,
// Markstein's correction) IS the correctly rounded quotient: equal to the division for every fp16 mantissa of s with
// every fp32 mantissa of y (a test takes all 2^33 pairs).  Three operations per element where a division takes ten; a
// rounded product with an exact fallback near half-integers, used here before, cost as much and sent a tenth of the rows
// through the divisions (keys and scales are both fp16, so exact ties are common).  Adding 1.5 x 2^23 rounds to nearest
// even and leaves the integer in the low mantissa bits, from where the codes are packed without conversions.
constexpr float kMagic = 12582912.0f;
__device__ __forceinline__ float clamped(float t, float lo, float hi) {
  return __builtin_amdgcn_fmed3f(t, lo, hi);   // NaN: the lower bound, as fmin(fmax(NaN, lo), hi)
}

// d / D rounded to nearest even, in three operations for a constant D: the product with the rounded reciprocal is
// within 1 ulp and one residual step corrects it (checked against the division for every fp32 mantissa); the fixup
// restores infinities and NaN.
template <int D>
__device__ __forceinline__ float div_const(float d) {
  constexpr float c = 1.0f / (float)D;
  const float y = d * c;
  const float e = __builtin_fmaf(-(float)D, y, d);
  return __builtin_amdgcn_div_fixupf(__builtin_fmaf(e, c, y), (float)D, d);
}

// A group's scale as divisor: r = 1 / s rounded to nearest even (the approximate reciprocal is within 1 ulp; one
// step corrects it, checked for every fp16 mantissa and 1 ulp either way).  A scale of zero or infinity divides
// everything to zero.
struct Divisor {
  float s, r;
  __device__ __forceinline__ explicit Divisor(float scale) {
    const float r0 = __builtin_amdgcn_rcpf(scale);
    const bool none = scale == 0.0f || r0 == 0.0f;
    s = none ? 0.0f : scale;
    r = none ? 0.0f : __builtin_fmaf(__builtin_fmaf(-scale, r0, 1.0f), r0, r0);
  }
  // 1.5 x 2^23 + rint(y / s) clamped to [lo, hi]
  __device__ __forceinline__ float code(float y, float lo, float hi) const {
    const float q = y * r;
    return clamped(__builtin_fmaf(__builtin_fmaf(-q, s, y), r, q), lo, hi) + kMagic;
  }
};

// The zero point to subtract.  One of minus infinity (a minimum below fp16's range) would make every quotient infinite,
// which the correction step turns into NaN; the codes are then the top one, and any finite number far below the values
// gives them: with a finite scale above 0 the group spans less than 2^20, so its values lie above -2^44.
__device__ __forceinline__ float zero_of(float z) { return fmaxf(z, -1152921504606846976.0f); }

template <int CTRL>
__device__ __forceinline__ uint32_t lanes_max(uint32_t v) {
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, 0xf, 0xf, true));
}

// Nearly every group is ordinary: no NaN, a scale that is a normal fp16 number, and (Q2) a zero point within 3/8 of a
// scale of the minimum.  Its quotients then round to codes inside the range by themselves (d / s is at most
// 127 (1 + 2^-10), 15 (1 + 2^-10) + 3/8), so clamps, fixups and the treatment of scales of zero drop out; a wave with any
// other group takes the general recipe for its codes, and looks for its range again only where a NaN or an infinity is
// in it (zeros into fp16 + int4, 2 x 32 heads x 8192 tokens: 80.3 us with all of the general recipe behind the quick one,
// 77.4 so, 76.3 with the general recipe alone, which takes 217 us instead of 163 for ordinary values three tiers deep).
// The quotient of an ordinary group costs two steps, q = y r + RN(y r'), where
// r' = RN((1 - s r) r) is what r lacks: off by 2^-46 before its one rounding, and a 24-bit y over an 11-bit s lies at
// least 2^-12 ulp from any midpoint, so this is the correctly rounded quotient as well.
__device__ __forceinline__ bool normal_half(float s) { return s >= 6.103515625e-05f && s <= 65504.0f; }   // false for NaN
__device__ __forceinline__ bool every_lane(bool ok) { return __builtin_amdgcn_ballot_w64(!ok) == 0; }
__device__ __forceinline__ float reciprocal(float s) {   // RN(1 / s) of a normal fp16 number
  const float r0 = __builtin_amdgcn_rcpf(s);
  return __builtin_fmaf(__builtin_fmaf(-s, r0, 1.0f), r0, r0);
}
template <int D>
__device__ __forceinline__ float div_const_finite(float d) {
  constexpr float c = 1.0f / (float)D;
  const float y = d * c;
  float q = __builtin_fmaf(__builtin_fmaf(-(float)D, y, d), c, y);
  asm("" : "+v"(q));   // rounded to fp32 before it is rounded to fp16, not in one mixed instruction
  return q;
}
// Largest magnitude, smallest value: NaN if any of the eight is one.
__device__ __forceinline__ float max_abs(const float (&x)[8]) {
  float m = __builtin_elementwise_maximum(fabsf(x[0]), fabsf(x[1]));
#pragma unroll
  for (int i = 2; i < 8; ++i) m = __builtin_elementwise_maximum(m, fabsf(x[i]));
  return m;
}

// Q1: n[i] = 1.5 x 2^23 + code as a float; the group is 4 lanes.  Returns the fp16 scale bits.
__device__ __forceinline__ uint32_t q1_over_group(uint32_t bits) {   // non-negative floats: ordered like the integers
  bits = lanes_max<0xB1>(bits);                                      // quad_perm [1,0,3,2]
  return lanes_max<0x4E>(bits);                                      // quad_perm [2,3,0,1]
}
// HALF: the values have at most 11 significant bits (fp16, bf16).  Quotients of two such numbers are half-integers or
// at least 2^-12 away from one, so y r (off by 2^-17) rounded to multiples of 2^-13 by adding 1536 decides every code and
// keeps every tie, and the second addition rounds to even: two steps per code.
template <bool HALF>
__device__ __forceinline__ uint16_t q1_codes(const float (&x)[8], float (&n)[8], float *s_out) {
  uint32_t bits = q1_over_group(__float_as_uint(max_abs(x)));   // NaN lies above infinity and passes to the whole group
  uint16_t sh = f2h(div_const_finite<127>(__uint_as_float(bits)));
  float s = h2f(sh);
  if (__builtin_expect(!every_lane(normal_half(s)), 0)) {
    if (__builtin_expect(!every_lane(bits < 0x7f800000u), 0)) {
      float amax = 0.0f;   // a group's NaNs do not count
#pragma unroll
      for (int i = 0; i < 8; ++i) amax = fmaxf(amax, fabsf(x[i]));
      sh = f2h(div_const<127>(__uint_as_float(q1_over_group(__float_as_uint(amax)))));
      s = h2f(sh);
    }
    const Divisor d(s);
#pragma unroll
    for (int i = 0; i < 8; ++i) n[i] = d.code(x[i], -127.0f, 127.0f);
    *s_out = s;
    return sh;
  }
  const float r = reciprocal(s);
  if constexpr (HALF) {
#pragma unroll
    for (int i = 0; i < 8; ++i) n[i] = __builtin_fmaf(x[i], r, 1536.0f) + (kMagic - 1536.0f);
  } else {
    const float rest = __builtin_fmaf(-s, r, 1.0f) * r;
#pragma unroll
    for (int i = 0; i < 8; ++i) n[i] = __builtin_fmaf(x[i], r, x[i] * rest) + kMagic;
  }
  *s_out = s;
  return sh;
}

__device__ __forceinline__ void q2_range(float *lo_out, float *hi_out) {
  float lo = *lo_out, hi = *hi_out;
  // over the group's eight lanes; as one block because the compiler would quiet every exchanged value first (18
  // instructions instead of 6).  A lane exchange reads a register two issue slots after it is written at the earliest.
  asm("s_nop 1\n\t"
      "v_min_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_min_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\t"
      "s_nop 0\n\t"
      "v_min_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\t"
      "v_max_f32_dpp %1, %1, %1 row_half_mirror row_mask:0xf bank_mask:0xf"
      : "+v"(lo), "+v"(hi));
  if (lo == 0.0f) lo = 0.0f;  // a zero minimum is stored as +0 whatever its sign
  *lo_out = lo;
  *hi_out = hi;
}
// Q2: the same for 4-bit codes; the group is 8 lanes.
struct Q2Scale {
  uint32_t word;   // fp16 {scale, zero} as stored
  float s, z;
};
__device__ __forceinline__ Q2Scale q2_codes(const float (&x)[8], float (&n)[8]) {
  float lo = x[0], hi = x[0];   // NaN if one of the eight is
#pragma unroll
  for (int i = 1; i < 8; ++i) {
    lo = __builtin_elementwise_minimum(lo, x[i]);
    hi = __builtin_elementwise_maximum(hi, x[i]);
  }
  const float own = lo;
  q2_range(&lo, &hi);
  uint16_t sh = f2h(div_const_finite<15>(hi - lo)), zh = f2h(lo);
  float s = h2f(sh), z = h2f(zh);
  if (__builtin_expect(!every_lane(normal_half(s) && fabsf(own - own) == 0.0f && fabsf(lo - z) <= 0.375f * s), 0)) {
    if (__builtin_expect(!every_lane(fabsf(own - own) == 0.0f && hi - lo < INFINITY), 0)) {
      lo = x[0];
      hi = x[0];
#pragma unroll
      for (int i = 1; i < 8; ++i) {   // NaNs do not count
        lo = fminf(lo, x[i]);
        hi = fmaxf(hi, x[i]);
      }
      q2_range(&lo, &hi);
      zh = f2h(lo);
      z = h2f(zh);
    }
    sh = f2h(div_const<15>(hi - lo));   // infinities, and the sign of zero
    s = h2f(sh);
    const Divisor d(s);
#pragma unroll
    for (int i = 0; i < 8; ++i) n[i] = d.code(x[i] - zero_of(z), 0.0f, 15.0f);
    return Q2Scale{(uint32_t)sh | ((uint32_t)zh << 16), s, z};
  }
  const float r = reciprocal(s), rest = __builtin_fmaf(-s, r, 1.0f) * r;
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const float y = x[i] - z;
    n[i] = __builtin_fmaf(y, r, y * rest) + kMagic;
  }
  return Q2Scale{(uint32_t)sh | ((uint32_t)zh << 16), s, z};
}

__device__ __forceinline__ uint32_t pack_bytes(const float *n) {   // low bytes of four codes
  const uint32_t a = __builtin_amdgcn_perm(__float_as_uint(n[1]), __float_as_uint(n[0]), 0x0c0c0400u);
  const uint32_t b = __builtin_amdgcn_perm(__float_as_uint(n[3]), __float_as_uint(n[2]), 0x04000c0cu);
  return a | b;
}
__device__ __forceinline__ uint32_t pack_nibbles(const float (&n)[8]) {
  // every n is 0x4B400000 + code: a chain of shift-adds, less what the constants add up to modulo 2^32
  uint32_t w = __float_as_uint(n[7]);
#pragma unroll
  for (int i = 6; i >= 0; --i) w = (w << 4) + __float_as_uint(n[i]);
  uint32_t c = 0x4B400000u;
#pragma unroll
  for (int i = 6; i >= 0; --i) c = (c << 4) + 0x4B400000u;
  return w - c;
}

// The values a format decompresses to (a token that passed through a tier).  code x scale is exact in fp32 (at most
// 7 + 11 bits), so the offset of the codes leaves in the same fused step.
template <bool HALF>
__device__ __forceinline__ void roundtrip_q1(float (&x)[8]) {
  float n[8], s;
  q1_codes<HALF>(x, n, &s);
  const float off = -kMagic * s;
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(n[i], s, off);
}
__device__ __forceinline__ void roundtrip_q2(float (&x)[8]) {
  float n[8];
  const Q2Scale q = q2_codes(x, n);
#pragma unroll
  for (int i = 0; i < 8; ++i) x[i] = __builtin_fmaf(n[i] - kMagic, q.s, q.z);
}

// ---------------------------------------------------------------- sources
// What a lane loads of one row: its eight channels in the source's format, with the group's scale words.
struct Raw {
  uint4 a, b;
};
// Rows are read once and written once: both with the streaming hint.  Tiering 2 x 32 heads x 8192 tokens into fp16 +
// int4, the stores' part of it: 83.5 -> 77.2 us; scales and zeros, a few bytes per row, go through the caches.  Not so
// for a tier in pinned memory, whose writes over PCIe the caches gather: 8 heads x 16384 tokens stored there directly,
// int4 365 us with the hint, 351 without; int8 682 and 644; K int8 / V int4 channel-major 524 and 500.
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 ld16(const uint8_t *p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
  return uint4{v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ u32x4 as_vec(const uint4 &v) { return u32x4{v.x, v.y, v.z, v.w}; }
__device__ __forceinline__ u32x2 as_vec(const uint2 &v) { return u32x2{v.x, v.y}; }
__device__ __forceinline__ uint32_t as_vec(uint32_t v) { return v; }
template <bool STREAM, typename T>
__device__ __forceinline__ void st_row(uint8_t *p, const T &v) {
  const auto x = as_vec(v);
  typedef decltype(as_vec(v)) V;
  if constexpr (STREAM) __builtin_nontemporal_store(x, (V *)p);
  else *(V *)p = x;
}
template <int F>
__device__ __forceinline__ void load_row(Raw &w, const uint8_t *code, const uint8_t *meta, int l16) {
  if constexpr (F == TTKV_F32) {
    w.a = ld16(code + l16 * 32);
    w.b = ld16(code + l16 * 32 + 16);
  } else if constexpr (F == TTKV_F16 || F == TTKV_BF16) {
    w.a = ld16(code + l16 * 16);
  } else if constexpr (F == TTKV_I8_SYM_G32) {
    const uint2 c = *(const uint2 *)(code + l16 * 8);
    w.a.x = c.x;
    w.a.y = c.y;
    w.a.z = *(const uint16_t *)(meta + (l16 >> 2) * 2);
  } else {
    w.a.x = *(const uint32_t *)(code + l16 * 4);
    w.a.y = *(const uint32_t *)(meta + (l16 >> 3) * 4);
  }
}
template <int F>
__device__ __forceinline__ void expand(const Raw &w, float (&x)[8]) {
  if constexpr (F == TTKV_F32) {
    const uint32_t u[8] = {w.a.x, w.a.y, w.a.z, w.a.w, w.b.x, w.b.y, w.b.z, w.b.w};
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = __uint_as_float(u[i]);
  } else if constexpr (F == TTKV_F16 || F == TTKV_BF16) {
    const uint32_t u[4] = {w.a.x, w.a.y, w.a.z, w.a.w};
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      x[2 * i] = F == TTKV_F16 ? h2f((uint16_t)(u[i] & 0xffff)) : __uint_as_float(u[i] << 16);
      x[2 * i + 1] = F == TTKV_F16 ? h2f((uint16_t)(u[i] >> 16)) : __uint_as_float(u[i] & 0xffff0000u);
    }
  } else if constexpr (F == TTKV_I8_SYM_G32) {
    const uint32_t u[2] = {w.a.x, w.a.y};
    const float s = h2f((uint16_t)w.a.z);
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = (float)(int)(int8_t)((u[i >> 2] >> (8 * (i & 3))) & 0xff) * s;
  } else {
    const float s = h2f((uint16_t)(w.a.y & 0xffff)), z = h2f((uint16_t)(w.a.y >> 16));
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float p = (float)(int)((w.a.x >> (4 * i)) & 0xf) * s;
      x[i] = p + z;
    }
  }
}
// Bytes of one row's codes in a source format.
template <int F>
constexpr int row_bytes() {
  return F == TTKV_F32 ? 512 : F == TTKV_I8_SYM_G32 ? 128 : F == TTKV_I4_ASYM_G64 ? 64 : 256;
}

__device__ __forceinline__ int wrap(int tok, const TierView &v) {
  const int ring = v.ring_blocks * v.bt;
  return tok >= ring ? tok - ring : tok;
}
// One KV head of ring block r of sequence seq.
__device__ __forceinline__ uint8_t *block_head(const TierView &v, int seq, int rec_base, int r, int h) {
  const int64_t rec = v.table ? (int64_t)v.table[(int64_t)seq * v.ring_blocks + r] : (int64_t)rec_base + r;
  return v.base + rec * v.rec_bytes + (int64_t)h * v.head_bytes;
}

// Rows t_first .. of one (entry, KV head, K / V) of the source: a flat array, or rows of a source tier that lie in
// at most two of its blocks (a unit has at most 64 rows, a block at least 64).
struct RowSource {
  const uint8_t *code, *meta;         // first row of the unit
  const uint8_t *code1, *meta1;       // first row of the block after
  int split;                          // rows of the unit in the first block
};
// The source of one (entry, KV head, K / V), gathered from the launch arguments once per workgroup: everything below
// works on these scalars (a reference to the arguments, indexed from many places, would put them into scratch).
struct Source {
  const uint8_t *flat;                // row 0, or null: the rows of `tier` from ring token `tok`
  TierView tier;
  int tok, rec_base, code_off, meta_off, seq, h;
  int n_via;
  uint32_t via;                       // formats passed through first, 8 bits each
};
__device__ __forceinline__ Source make_source(const ConvArgs &a, int which, int j, int h, int seq) {
  Source s;
  s.flat = nullptr;
  s.tier = a.s.src;
  if (!a.s.from_tier) {
    const int64_t rows = ((int64_t)j * a.Hkv + h) * a.n_tokens;
    const int bytes = a.s.flat_fmt == TTKV_F32 ? 512 : 256;
    const uint8_t *k = (const uint8_t *)a.s.k_flat, *v = (const uint8_t *)a.s.v_flat;
    s.flat = (which ? v : k) + rows * bytes;
  }
  s.tok = a.s.src_first_tok[j];
  s.rec_base = a.s.src_rec_base[j];
  s.code_off = which ? s.tier.v_off : 0;
  s.meta_off = which ? s.tier.v_meta_off : s.tier.k_meta_off;
  s.seq = seq;
  s.h = h;
  s.n_via = a.n_via;
  const uint32_t via_k = a.via_k, via_v = a.via_v;
  s.via = which ? via_v : via_k;
  return s;
}
template <int F>
__device__ __forceinline__ RowSource row_source(const Source &c, int t_first) {
  RowSource s;
  if (c.flat) {
    s.code = s.code1 = c.flat + (int64_t)t_first * row_bytes<F>();
    s.meta = s.meta1 = nullptr;
    s.split = 1 << 30;
    return s;
  }
  const int tok = wrap(c.tok + t_first, c.tier);
  const int r = div_bt(tok, c.tier.bt, c.tier.bt_magic), row = tok - r * c.tier.bt;
  const uint8_t *h0 = block_head(c.tier, c.seq, c.rec_base, r, c.h);
  s.code = s.code1 = h0 + c.code_off + row * row_bytes<F>();
  s.meta = s.meta1 = h0 + c.meta_off + row * 8;
  s.split = c.tier.bt - row;
  if (s.split < CHUNK) {
    const uint8_t *h1 = block_head(c.tier, c.seq, c.rec_base, r + 1 == c.tier.ring_blocks ? 0 : r + 1, c.h);
    s.code1 = h1 + c.code_off;
    s.meta1 = h1 + c.meta_off;
  }
  return s;
}
template <int F>
__device__ __forceinline__ void load_from(const RowSource &s, int i, int l16, Raw &w) {   // row i of the unit
  const bool next = i >= s.split;
  const int o = next ? i - s.split : i;
  load_row<F>(w, (next ? s.code1 : s.code) + o * row_bytes<F>(), (next ? s.meta1 : s.meta) + o * 8, l16);
}
// The formats a token has passed through before this one (Sec. 4.2's recipes, applied and taken back): at most two,
// the fp formats change nothing.  Written out because a loop over them would copy the eight values in every turn.
template <int SRC>
__device__ __forceinline__ void pass_through(const Source &c, float (&x)[8]) {
  static_assert(TTKV_MAX_TIERS == 4, "tiers 1 and 2 lie above the last one");
  if (c.n_via > 0) {
    const uint32_t f = c.via & 0xff;
    if (f == TTKV_I8_SYM_G32) roundtrip_q1<SRC == TTKV_F16 || SRC == TTKV_BF16>(x);
    if (f == TTKV_I4_ASYM_G64) roundtrip_q2(x);
  }
  if (c.n_via > 1) {
    const uint32_t f = c.via >> 8;
    if (f == TTKV_I8_SYM_G32) roundtrip_q1<false>(x);
    if (f == TTKV_I4_ASYM_G64) roundtrip_q2(x);
  }
}

// ---------------------------------------------------------------- one unit
// Where a unit's rows land: `head` is the KV head's part of the destination block, `row0` the block row of the
// unit's row 0; rows [lo, hi) of the unit are live and row lo is token t_lo of the call.
// S: rows stored with the streaming hint.
template <bool S>
struct Unit {
  static constexpr bool STREAM = S;
  uint8_t *head;
  int code_off, meta_off, row0;
  int lo, hi, t_lo;
};

// A thread's number inside its unit (workgroups of SUM_THREADS may take two units side by side).
template <int THREADS>
__device__ __forceinline__ int unit_thread() { return threadIdx.x & (THREADS - 1); }
template <int SRC, int THREADS, int ROWS, typename U>
__device__ __forceinline__ void load_unit(const Source &c, const U &u, Raw (&raw)[ROWS * 16 / THREADS]) {
  const RowSource s = row_source<SRC>(c, u.t_lo);
  const int t = unit_thread<THREADS>(), l16 = t & 15, r = t >> 4;
  if (u.lo == 0 && u.hi == ROWS && s.split >= ROWS) {   // every row live and in one block: one base, constant offsets
#pragma unroll
    for (int p = 0; p < ROWS * 16 / THREADS; ++p) {
      const uint32_t i = p * (THREADS / 16) + r;
      load_row<SRC>(raw[p], s.code + i * row_bytes<SRC>(), s.meta + i * 8, l16);
    }
  } else {
#pragma unroll
    for (int p = 0; p < ROWS * 16 / THREADS; ++p)
      load_from<SRC>(s, min(max(p * (THREADS / 16) + r, u.lo), u.hi - 1) - u.lo, l16, raw[p]);   // dead rows repeat a live one
  }
}

// Row i of the unit from its values x: quantized to DST, stored if live.  Channel-major values leave their codes in
// s_t32 instead.
constexpr int kT32Stride = 20;   // words per row of codes: rows 4 apart fall 16 banks apart
constexpr int kT32Bytes = CHUNK * kT32Stride * 4 + 2 * 2048;
template <int DST, typename U>
__device__ __forceinline__ void put_row(const U &u, int i, int l16, const float (&x)[8], uint32_t *s_t32) {
  uint8_t *const code = u.head + u.code_off, *const meta = u.head + u.meta_off;
  const bool live = i >= u.lo && i < u.hi;
  const uint32_t row = u.row0 + i;
  float n[8];
  if constexpr (DST == TTKV_F16 || DST == TTKV_BF16) {
    uint32_t w[4];
#pragma unroll
    for (int k = 0; k < 4; ++k) {
      uint32_t lo16, hi16;
      if constexpr (DST == TTKV_F16) {
        lo16 = f2h(x[2 * k]);
        hi16 = f2h(x[2 * k + 1]);
      } else {  // the upper halves (exact for values that come from bf16)
        lo16 = __float_as_uint(x[2 * k]) >> 16;
        hi16 = __float_as_uint(x[2 * k + 1]) >> 16;
      }
      w[k] = lo16 | (hi16 << 16);
    }
    if (live) st_row<U::STREAM>(code + row * 256 + l16 * 16, uint4{w[0], w[1], w[2], w[3]});
  } else if constexpr (DST == TTKV_I8_SYM_G32) {
    float s;
    const uint16_t sh = q1_codes<false>(x, n, &s);
    const bool zero = s == 0.0f;
    const uint2 w = {zero ? 0u : pack_bytes(n), zero ? 0u : pack_bytes(n + 4)};
    if (live) {
      st_row<U::STREAM>(code + row * 128 + l16 * 8, w);
      if ((l16 & 3) == 0) *(uint16_t *)(meta + row * 8 + (l16 >> 2) * 2) = sh;
    }
  } else if constexpr (DST == TTKV_I4_ASYM_G64 || DST == TTKV_I4_ASYM_G64_T32) {
    const Q2Scale q = q2_codes(x, n);
    const uint32_t w = pack_nibbles(n);
    if constexpr (DST == TTKV_I4_ASYM_G64) {
      if (live) st_row<U::STREAM>(code + row * 64 + l16 * 4, w);
    } else {
      s_t32[i * kT32Stride + l16] = w;
    }
    if (live && (l16 & 7) == 0) *(uint32_t *)(meta + row * 8 + (l16 >> 3) * 4) = q.word;
  }
}
__device__ __forceinline__ void keep_values(float (*s_x)[128], int i, int l16, const float (&x)[8]) {
  float4 *o = (float4 *)(s_x[i] + l16 * 8);
  o[0] = float4{x[0], x[1], x[2], x[3]};
  o[1] = float4{x[4], x[5], x[6], x[7]};
}

// The unit's loaded rows.  SUM: the arriving values also go to s_x.
template <int SRC, int DST, int THREADS, int ROWS, bool SUM, typename U>
__device__ __forceinline__ void convert_unit(const Source &c, const U &u, const Raw (&raw)[ROWS * 16 / THREADS],
                                             float (*s_x)[128], uint32_t *s_t32) {
  const int t = unit_thread<THREADS>(), l16 = t & 15;
#pragma unroll
  for (int p = 0; p < ROWS * 16 / THREADS; ++p) {
    const int i = p * (THREADS / 16) + (t >> 4);
    constexpr bool COPY = SRC == DST && (DST == TTKV_F16 || DST == TTKV_BF16);
    if (COPY && !SUM && c.n_via == 0) {   // bytes as they are
      if (i >= u.lo && i < u.hi) st_row<U::STREAM>(u.head + u.code_off + (u.row0 + i) * 256 + l16 * 16, raw[p].a);
      continue;
    }
    float x[8];
    expand<SRC>(raw[p], x);
    pass_through<SRC>(c, x);
    if constexpr (SUM) keep_values(s_x, i, l16, x);
    put_row<DST>(u, i, l16, x, s_t32);
  }
}

#define TTKV_FOR_SOURCES(DST, CALL)                                       \
  switch (src_fmt) {                                                      \
    case TTKV_F16: CALL(TTKV_F16, DST); break;                            \
    case TTKV_BF16: CALL(TTKV_BF16, DST); break;                          \
    case TTKV_F32: CALL(TTKV_F32, DST); break;                            \
    case TTKV_I8_SYM_G32: CALL(TTKV_I8_SYM_G32, DST); break;              \
    default: CALL(TTKV_I4_ASYM_G64, DST); break;                          \
  }

// Channel-major values: the unit's two groups of 32 tokens leave as 2 KiB each in the operand order of the
// matrix-core kernel: piece p = 64 hh + 16 kg + c, word w: channel 16 (4 hh + w) + c, nibble q: token kTok[q] + 4 kg.
// A thread takes the words of eight such tokens (eight channels each) and turns them by 8 x 8 nibbles in registers --
// nibbles by masks, then bytes by v_perm, 32 operations for 8 words instead of 24 per word gathered one by one -- and
// the words meet in LDS in the group's order, pieces permuted inside eights to spread them over the banks.
template <int THREADS, typename U>
__device__ __forceinline__ void store_t32(const U &u, uint32_t *s_t32) {   // (a unit without live rows takes part in the barriers)
  const int t = unit_thread<THREADS>();
  const bool live = u.lo < u.hi;
  uint4 *const s_out = (uint4 *)(s_t32 + CHUNK * kT32Stride);
  __syncthreads();
  if (live && t < 128) {
    const int g = t >> 6, kg = (t >> 4) & 3, cw = t & 15;
    const int kTok[8] = {0, 2, 16, 18, 1, 3, 17, 19};
    uint32_t in[8], even[4], odd[4];
#pragma unroll
    for (int q = 0; q < 8; ++q) in[q] = s_t32[(g * 32 + kTok[q] + 4 * kg) * kT32Stride + cw];
#pragma unroll
    for (int q = 0; q < 4; ++q) {   // byte k of even (odd): channel 2 k (2 k + 1) of tokens 2 q, 2 q + 1
      even[q] = (in[2 * q] & 0x0F0F0F0Fu) | ((in[2 * q + 1] << 4) & 0xF0F0F0F0u);
      odd[q] = ((in[2 * q] >> 4) & 0x0F0F0F0Fu) | (in[2 * q + 1] & 0xF0F0F0F0u);
    }
    uint32_t *const out = (uint32_t *)(s_out + g * 128);
    const int hh = cw >> 3, w = (cw >> 1) & 3, base = 64 * hh + 16 * kg + 8 * (cw & 1), turn = 2 * kg + hh;
    auto turned = [&](const uint32_t (&m)[4], int odd_channel) {
      const uint32_t lo01 = __builtin_amdgcn_perm(m[1], m[0], 0x05010400u), lo23 = __builtin_amdgcn_perm(m[3], m[2], 0x05010400u);
      const uint32_t hi01 = __builtin_amdgcn_perm(m[1], m[0], 0x07030602u), hi23 = __builtin_amdgcn_perm(m[3], m[2], 0x07030602u);
      const uint32_t turned4[4] = {__builtin_amdgcn_perm(lo23, lo01, 0x05040100u), __builtin_amdgcn_perm(lo23, lo01, 0x07060302u),
                             __builtin_amdgcn_perm(hi23, hi01, 0x05040100u), __builtin_amdgcn_perm(hi23, hi01, 0x07060302u)};
#pragma unroll
      for (int k = 0; k < 4; ++k) out[4 * ((base + 2 * k + odd_channel) ^ turn) + w] = turned4[k];
    };
    turned(even, 0);
    turned(odd, 1);
  }
  __syncthreads();
  for (int idx = t; idx < 256; idx += THREADS) {
    const int g = idx >> 7, p = idx & 127, turn = 2 * ((p >> 4) & 3) + (p >> 6);
    if (g * 32 >= u.lo && g * 32 < u.hi) st_row<U::STREAM>(u.head + u.code_off + (u.row0 + g * 32) * 64 + p * 16, s_out[g * 128 + (p ^ turn)]);
  }
}

// Keys of one destination block, converted like any other unit and summed per channel in token order (fp32) for the
// block's mean key: a block that was partly filled before continues from its stored sum.  The arriving values of 16 rows
// (32 with 512 threads) go to LDS, where the two waves whose turn it is add them up (one channel per lane) while the other
// waves convert the next rows; the running sums pass from turn to turn through LDS.  The order of the additions is the
// token order, so the sums are reproducible bit for bit; what made the former kernel (one thread per channel,
// reading and re-quantizing one row after the other from memory) 331 us of the 572 us tiering of 4 x 32768 tokens
// was the chain of loads, not the additions.
// One loop per pair of formats: with the formats looked up in every turn, the waves whose turn it was waited for their next
// rows before they began to add (tiering 4 x 32768 tokens three deep 180 us, now 162) and the kernel took 74 registers
// instead of 56.
template <int SRC, int DST, int THREADS, typename U>
__device__ __forceinline__ void sum_rows(const Source &src, U u, int rows_lo, int rows_hi, float *k_sum, uint16_t *k_summary,
                                         float inv_bt, char *s_buf) {
  constexpr int ROWS = THREADS / 16;
  float (*s_x)[ROWS][128] = (float (*)[ROWS][128])s_buf;            // two buffers
  float *s_sum = (float *)(s_buf + 2 * ROWS * 128 * sizeof(float));
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int t0 = u.t_lo;
  auto place = [&](int row0) {
    u.row0 = row0;
    u.lo = max(rows_lo - row0, 0);
    u.hi = min(rows_hi - row0, ROWS);
    u.t_lo = t0 + row0 + u.lo - rows_lo;
  };
  Raw raw[1];
  place(rows_lo / ROWS * ROWS);
  load_unit<SRC, THREADS, ROWS>(src, u, raw);
  if (threadIdx.x < 128) s_sum[threadIdx.x] = rows_lo ? k_sum[threadIdx.x] : 0.0f;   // the threads that add first
  for (int c = 0;; ++c) {
    convert_unit<SRC, DST, THREADS, ROWS, true>(src, u, raw, s_x[c & 1], nullptr);
    const int lo = u.lo, hi = u.hi, next = u.row0 + ROWS;
    const bool more = next < rows_hi;
    if (more) {
      place(next);
      load_unit<SRC, THREADS, ROWS>(src, u, raw);
    }
    __syncthreads();
    const int turn = wave - 2 * (c % (THREADS / 128));
    if (turn == 0 || turn == 1) {
      const int ch = turn * 64 + lane;
      float sum = s_sum[ch];
      const float *x = &s_x[c & 1][0][ch];
      if (lo == 0 && hi == ROWS) {
#pragma unroll 16
        for (int r = 0; r < ROWS; ++r) sum = sum + x[r * 128];
      } else {
        for (int r = lo; r < hi; ++r) sum = sum + x[r * 128];
      }
      if (more) {
        s_sum[ch] = sum;
      } else {
        k_sum[ch] = sum;
        k_summary[ch] = f2h(sum * inv_bt);
      }
    }
    if (!more) break;
  }
}
template <int THREADS, typename U>
__device__ __forceinline__ void sum_unit(const Source &src, const U &u, int src_fmt, int dst_fmt, int rows_lo, int rows_hi, float *k_sum,
                                         uint16_t *k_summary, float inv_bt, char *s_buf) {
  // k_sum, k_summary: the block's; rows [rows_lo, rows_hi) of the block arrive, row rows_lo is token u.t_lo
#define TTKV_SUM_ROWS(S, D) sum_rows<S, D, THREADS>(src, u, rows_lo, rows_hi, k_sum, k_summary, inv_bt, s_buf)
  switch (dst_fmt) {
    case TTKV_F16: TTKV_SUM_ROWS(TTKV_F16, TTKV_F16); break;
    case TTKV_BF16: TTKV_SUM_ROWS(TTKV_BF16, TTKV_BF16); break;
    case TTKV_I8_SYM_G32: TTKV_FOR_SOURCES(TTKV_I8_SYM_G32, TTKV_SUM_ROWS) break;
    case TTKV_I4_ASYM_G64: TTKV_FOR_SOURCES(TTKV_I4_ASYM_G64, TTKV_SUM_ROWS) break;
    default: TTKV_FOR_SOURCES(NO_STORE, TTKV_SUM_ROWS) break;
  }
#undef TTKV_SUM_ROWS
}

// Grid: x = K units then V units of one (entry, KV head), y = KV head, z = entry.  SUM: K units are whole destination
// blocks and keep the key sums (dst_fmt of K may be NO_STORE: sums only); otherwise every unit is 64 rows.
// With SUM a conversion that keeps no sums (beside one that does) has units of 64 rows for K and V.  UT: threads of such a
// unit; a workgroup takes THREADS / UT of them.
template <bool SUM, bool STREAM, int THREADS, int UT>
__device__ __forceinline__ void convert_rows(const ConvArgs &a, int k_units, int k_dst_fmt, bool sums, int j) {
  constexpr int SUM_BYTES = 2 * (THREADS / 16) * 128 * 4 + 512;
  constexpr int PER = THREADS / UT;
  __shared__ __align__(16) char s_buf[SUM && SUM_BYTES > PER * kT32Bytes ? SUM_BYTES : PER * kT32Bytes];
  const int h = blockIdx.y, seq = a.seq_id[j];
  const int which = (int)blockIdx.x >= k_units;
  int unit = which ? blockIdx.x - k_units : blockIdx.x;
  const int first = a.dst_first_tok[j];                   // ring token the call's first row lands on
  const int dst_rec_base = a.dst_rec_base[j], n_tokens = a.n_tokens;
  const TierView dst = a.dst;
  const Source src = make_source(a, which, j, h, seq);
  const int src_fmt = src.flat ? a.s.flat_fmt : which ? src.tier.v_fmt : src.tier.k_fmt;
  Unit<STREAM> u;
  u.code_off = which ? dst.v_off : 0;
  u.meta_off = which ? dst.v_meta_off : dst.k_meta_off;

  if (SUM && !which && sums) {
    const int r = div_bt(first, dst.bt, dst.bt_magic), r0 = first - r * dst.bt;
    const int t_lo = max(0, unit * dst.bt - r0), t_hi = min(n_tokens, (unit + 1) * dst.bt - r0);
    if (t_lo >= t_hi) return;
    int rb = r + unit;
    if (rb >= dst.ring_blocks) rb -= dst.ring_blocks;
    u.head = k_dst_fmt == NO_STORE ? nullptr : block_head(dst, seq, dst_rec_base, rb, h);
    int sb = a.sum_first_block[j] + unit;
    if (sb >= a.sum_ring_blocks) sb -= a.sum_ring_blocks;
    const int64_t rec = a.sum_table ? (int64_t)a.sum_table[(int64_t)seq * a.sum_ring_blocks + sb] : (int64_t)seq * a.sum_ring_blocks + sb;
    const int64_t sum_at = (rec * a.Hkv + h) * 128;
    const int rows_lo = t_lo + r0 - unit * dst.bt, rows_hi = t_hi + r0 - unit * dst.bt;
    u.t_lo = t_lo;
    float *const k_sum = a.k_sum + sum_at;
    uint16_t *const k_summary = a.k_summary + sum_at;
    const float inv_bt = a.inv_bt;
    sum_unit<THREADS>(src, u, src_fmt, k_dst_fmt, rows_lo, rows_hi, k_sum, k_summary, inv_bt, s_buf);
    return;
  }

  const int side = PER > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x / UT) : 0;
  unit = unit * PER + side;
  int tok = first / CHUNK * CHUNK + unit * CHUNK;         // ring token of the unit's row 0
  const int t0 = tok - first;                             // its token of the call (the first unit may start before it)
  u.lo = max(0, -t0);
  u.hi = min(CHUNK, n_tokens - t0);
  u.t_lo = t0 + u.lo;
  const int dst_fmt = which ? dst.v_fmt : k_dst_fmt;
  // A unit without rows leaves; beside another one whose values meet in LDS it takes part in the workgroup's barriers.
  const bool live = u.lo < u.hi;
  if (!live && (PER == 1 || dst_fmt != TTKV_I4_ASYM_G64_T32)) return;
  uint32_t *const s_t32 = (uint32_t *)(s_buf + side * kT32Bytes);
  if (live) {
    tok = wrap(tok, dst);
    const int r = div_bt(tok, dst.bt, dst.bt_magic);
    u.row0 = tok - r * dst.bt;
    u.head = block_head(dst, seq, dst_rec_base, r, h);
    Raw raw[CHUNK * 16 / UT];
#define TTKV_ROW_UNIT(S, D) load_unit<S, UT, CHUNK>(src, u, raw), convert_unit<S, D, UT, CHUNK, false>(src, u, raw, nullptr, s_t32)
    switch (dst_fmt) {
      case TTKV_F16: TTKV_ROW_UNIT(TTKV_F16, TTKV_F16); break;
      case TTKV_BF16: TTKV_ROW_UNIT(TTKV_BF16, TTKV_BF16); break;
      case TTKV_I8_SYM_G32: TTKV_FOR_SOURCES(TTKV_I8_SYM_G32, TTKV_ROW_UNIT) break;
      case TTKV_I4_ASYM_G64_T32: TTKV_FOR_SOURCES(TTKV_I4_ASYM_G64_T32, TTKV_ROW_UNIT) break;
      default: TTKV_FOR_SOURCES(TTKV_I4_ASYM_G64, TTKV_ROW_UNIT) break;
    }
#undef TTKV_ROW_UNIT
  }
  if (dst_fmt == TTKV_I4_ASYM_G64_T32) store_t32<UT>(u, s_t32);
}
template <bool SUM, bool STREAM, int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == 256 ? 8 : 6) void convert_rows_kernel(const ConvArgs a, int k_units, int k_dst_fmt) {
  convert_rows<SUM, STREAM, THREADS, THREADS>(a, k_units, k_dst_fmt, true, blockIdx.z);
}

// Two conversions side by side (two boundaries of an eviction): the entries of the second follow those of the first.
struct ConvPair {
  ConvArgs a[2];
  int32_t k_units[2], units[2];   // workgroups of K, of K and V
  int32_t n_first;                // entries of the first one
};
template <bool SUM, int THREADS>
__global__ __launch_bounds__(THREADS, THREADS == 256 ? 8 : 6) void convert_pair_kernel(const ConvPair c) {
  const int i = (int)blockIdx.z >= c.n_first;
  const ConvArgs &a = c.a[i];
  if ((int)blockIdx.x >= c.units[i]) return;
  convert_rows<SUM, true, THREADS, 256>(a, c.k_units[i], a.dst.k_fmt, a.k_sum != nullptr, (int)blockIdx.z - (i ? c.n_first : 0));
}

// Keys of a tier whose int4 groups run over 128 consecutive tokens of one channel (Q_4bit's arithmetic with the
// group turned by 90 degrees): one workgroup per (token group, KV head, entry).  The group's 128 arriving rows are
// read once and stay in registers (a 16-lane group holds rows r, r + 16, ..; 8 channels per lane); the ranges meet
// over the lanes and waves, one thread per channel forms the scale, and the rows are coded from the registers.
template <int SRC, bool STREAM>
__device__ __forceinline__ void keys_t128(const Source &src, int g, uint8_t *head, int k_meta_off, int row0, float (*s_lo)[128],
                                          float (*s_hi)[128], float (*s_q)[128]) {
  const int l16 = threadIdx.x & 15, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  float x[8][8];
  {
    Raw raw[8];
#pragma unroll
    for (int half = 0; half < 2; ++half) {
      const RowSource s = row_source<SRC>(src, g * 128 + half * 64);
#pragma unroll
      for (int p = 0; p < 4; ++p) load_from<SRC>(s, p * 16 + (threadIdx.x >> 4), l16, raw[half * 4 + p]);
    }
#pragma unroll
    for (int p = 0; p < 8; ++p) {
      expand<SRC>(raw[p], x[p]);
      pass_through<SRC>(src, x[p]);
    }
  }
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    float lo = x[0][i], hi = x[0][i];
#pragma unroll
    for (int p = 1; p < 8; ++p) {
      lo = fminf(lo, x[p][i]);
      hi = fmaxf(hi, x[p][i]);
    }
    lo = fminf(lo, __shfl_xor(lo, 16));
    hi = fmaxf(hi, __shfl_xor(hi, 16));
    lo = fminf(lo, __shfl_xor(lo, 32));
    hi = fmaxf(hi, __shfl_xor(hi, 32));
    if (lane < 16) {
      s_lo[wave][l16 * 8 + i] = lo;
      s_hi[wave][l16 * 8 + i] = hi;
    }
  }
  __syncthreads();
  if (threadIdx.x < 128) {
    const int i = threadIdx.x;
    float lo = fminf(fminf(s_lo[0][i], s_lo[1][i]), fminf(s_lo[2][i], s_lo[3][i]));
    const float hi = fmaxf(fmaxf(s_hi[0][i], s_hi[1][i]), fmaxf(s_hi[2][i], s_hi[3][i]));
    if (lo == 0.0f) lo = 0.0f;  // a zero minimum is stored as +0 whatever its sign
    const uint16_t sh = f2h(div_const<15>(hi - lo)), zh = f2h(lo);
    s_q[0][i] = h2f(sh);
    s_q[1][i] = h2f(zh);
    // the group's 128 meta rows of 4 bytes hold {scale, zero} of the 128 channels
    *(uint32_t *)(head + k_meta_off + row0 * 4 + i * 4) = (uint32_t)sh | ((uint32_t)zh << 16);
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 8; ++i) {
    const Divisor d(s_q[0][l16 * 8 + i]);
    const float z = zero_of(s_q[1][l16 * 8 + i]);
#pragma unroll
    for (int p = 0; p < 8; ++p) x[p][i] = d.code(x[p][i] - z, 0.0f, 15.0f);
  }
#pragma unroll
  for (int p = 0; p < 8; ++p)
    st_row<STREAM>(head + (row0 + p * 16 + (threadIdx.x >> 4)) * 64 + l16 * 4, pack_nibbles(x[p]));
}
template <bool STREAM>
__global__ __launch_bounds__(256) void convert_keys_t128_kernel(const ConvArgs a) {
  __shared__ float s_lo[4][128], s_hi[4][128], s_q[2][128];
  const int g = blockIdx.x, h = blockIdx.y, j = blockIdx.z;
  const int seq = a.seq_id[j], dst_rec_base = a.dst_rec_base[j];
  const TierView dst = a.dst;
  const Source src = make_source(a, 0, j, h, seq);
  const int src_fmt = src.flat ? a.s.flat_fmt : src.tier.k_fmt;
  const int tok = wrap(a.dst_first_tok[j] + g * 128, dst);
  const int r = div_bt(tok, dst.bt, dst.bt_magic), row0 = tok - r * dst.bt;
  uint8_t *const head = block_head(dst, seq, dst_rec_base, r, h);
#define TTKV_T128(S, D) keys_t128<S, STREAM>(src, g, head, dst.k_meta_off, row0, s_lo, s_hi, s_q)
  TTKV_FOR_SOURCES(0, TTKV_T128)
#undef TTKV_T128
}

}  // namespace

namespace {
// How a conversion is cut: units of the entry that needs most.
struct Units {
  int chunks, blocks;   // of 64 rows; whole destination blocks
};
Units units_of(const ConvArgs &a) {
  Units u{0, 0};
  for (int j = 0; j < a.n_seq; ++j) {
    u.chunks = std::max(u.chunks, (a.dst_first_tok[j] % CHUNK + a.n_tokens + CHUNK - 1) / CHUNK);
    u.blocks = std::max(u.blocks, (a.dst_first_tok[j] % a.dst.bt + a.n_tokens + a.dst.bt - 1) / a.dst.bt);
  }
  return u;
}
template <bool STREAM>
hipError_t launch(const ConvArgs &a, hipStream_t s, int *n_kernels) {
  if ((int64_t)a.n_seq * a.Hkv * a.n_tokens <= 0) return hipSuccess;
  const Units u = units_of(a);
  const bool t128 = a.dst.k_fmt == TTKV_I4_ASYM_T128;   // whole aligned groups (the caller has checked)
  if (t128) {
    hipLaunchKernelGGL(convert_keys_t128_kernel<STREAM>, dim3(a.n_tokens / 128, a.Hkv, a.n_seq), dim3(256), 0, s, a);
    ++*n_kernels;
  }
  if (a.k_sum) {
    const int k_dst = t128 ? NO_STORE : a.dst.k_fmt;
    // A block's keys are one workgroup's work from end to end.  With four blocks per CU and more, eight small workgroups
    // per CU keep it busy across each other's barriers (2560 blocks of 256 tokens: step 166 us, 187 with 512 threads); with
    // fewer the time is that of one block, which more threads shorten (640 blocks 59.5 and 56.8 us; evictions of 128 rows:
    // 256 blocks 22.2 and 18.5, 384 27.0 and 25.3, 512 29.7 and 30.3).
    if ((int64_t)u.blocks * a.n_seq * a.Hkv >= 1024)
      hipLaunchKernelGGL((convert_rows_kernel<true, STREAM, 256>), dim3(u.blocks + u.chunks, a.Hkv, a.n_seq), dim3(256), 0, s, a, u.blocks, k_dst);
    else
      hipLaunchKernelGGL((convert_rows_kernel<true, STREAM, SUM_THREADS>), dim3(u.blocks + u.chunks, a.Hkv, a.n_seq), dim3(SUM_THREADS), 0, s, a, u.blocks, k_dst);
  } else {
    const int k_units = t128 ? 0 : u.chunks;
    hipLaunchKernelGGL((convert_rows_kernel<false, STREAM, 256>), dim3(k_units + u.chunks, a.Hkv, a.n_seq), dim3(256), 0, s, a, k_units, a.dst.k_fmt);
  }
  ++*n_kernels;
  return hipGetLastError();
}
}  // namespace

// Converts the rows and, where the destination keeps block summaries (a.k_sum), their key sums.
hipError_t launch_convert(const ConvArgs &a, hipStream_t s, int *n_kernels) {
  return a.to_host ? launch<false>(a, s, n_kernels) : launch<true>(a, s, n_kernels);
}

// One launch takes as long as the slower of the two, where two launches take their sum and the gap between them: 39 x 16 heads,
// 128 rows of fp16 into int8 and of int8 into int4, 27.2 -> 23.1 us, 39 x 2 heads 14.4 -> 8.4.  With sums all its workgroups
// have the 512 threads and 33 KB of LDS of those that add, three on a CU; they take two 64-row units, or 16 x 8 heads were 1024
// of them for 768 places: two launches 15.8, with one unit 12.6, with two 9.1 (24 x 8 heads 14.3, 18.0, 11.4; 56 x 16 heads 43.0,
// 65.7, 39.0; 40 x 32 heads 55.6 and 53.2).  64 x 32 heads, 2048 summed blocks, are faster apart, with 256 threads each (78.8, 81.2).
hipError_t launch_convert_pair(const ConvArgs &a, const ConvArgs &b, hipStream_t s, int *n_kernels) {
  const bool turned = b.k_sum && !a.k_sum;   // the one with sums first: its workgroups take longest
  ConvPair c{{turned ? b : a, turned ? a : b}, {}, {}, turned ? b.n_seq : a.n_seq};
  const bool sums = a.k_sum || b.k_sum;
  bool apart = a.to_host || b.to_host;
  for (int i = 0; i < 2; ++i) {
    const Units u = units_of(c.a[i]);
    const int groups = sums ? (u.chunks + SUM_THREADS / 256 - 1) / (SUM_THREADS / 256) : u.chunks;   // of 64-row units
    c.k_units[i] = c.a[i].k_sum ? u.blocks : groups;
    c.units[i] = c.k_units[i] + groups;
    apart |= c.a[i].dst.k_fmt == TTKV_I4_ASYM_T128 || (c.a[i].k_sum && (int64_t)u.blocks * c.a[i].n_seq * c.a[i].Hkv > 1536);
  }
  const dim3 grid(std::max(c.units[0], c.units[1]), a.Hkv, a.n_seq + b.n_seq);   // (one cache: as many KV heads in both)
  if (apart) {
    const hipError_t e = launch_convert(a, s, n_kernels);
    return e != hipSuccess ? e : launch_convert(b, s, n_kernels);
  }
  if (sums)
    hipLaunchKernelGGL((convert_pair_kernel<true, SUM_THREADS>), grid, dim3(SUM_THREADS), 0, s, c);
  else
    hipLaunchKernelGGL((convert_pair_kernel<false, 256>), grid, dim3(256), 0, s, c);
  ++*n_kernels;
  return hipGetLastError();
}

}  // namespace ttkv
