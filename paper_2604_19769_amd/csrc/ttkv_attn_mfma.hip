// Grouped-query variant of the split-K decode attention partials (Alg. 1: Attn on the
// fast tier, Decompress + Attn per slow-tier block): all query heads that share a KV
// head are served by ONE pass over that head's K/V bytes, with the two contractions on
// the matrix cores (v_mfma_f32_16x16x32 f16 / bf16 for q.k and p.v, v_mfma_f32_16x16x16 for
// the layout changes).  Same work items, same partials and same record layout as the vector
// kernel; only the lane mapping differs.
//
// One 16-token tile, lane = (c = lane % 16, kg = lane / 16):
//   K rows reach the MFMA A layout as 32 channels of token c per lane, spliced into packed 16-bit pairs as in the vector
//   kernel.  Four 32-deep steps give
//       S[token][head] = sum_d K[token][d] * Q[d][head]
//   Quantized keys: the lane's channels are 8 bytes of each 32-byte stretch of the row, so a step (or two, int4) stays
//   inside one channel group and every group has a product chain of its own; up to 16 heads are the columns, whatever
//   the format, and no product is spent on zeros.  The splice offsets leave through the initial accumulator value.  In
//   the MFMA result layout lane (c, kg) holds head c of tokens 4 kg .. 4 kg + 3; those tokens' meta words (scale, zero
//   point per group) are read from LDS in that layout (the lanes of one kg read the same 16 bytes) and enter as fp16
//   operands of fused multiply-adds.
//   The softmax is per column (lane-local over 4 tokens, two lane exchanges over kg); its scale is applied inside the
//   exponent.
//   Quantized V: gfx950's transposing LDS reads (ds_read_b64_tr_b4 / _b8) hand lane (c, kg) the codes of ONE channel of
//   eight tokens of a 32-token pair of tiles -- after the splice, whose offset (and the centre 8 of int4 codes) leaves
//   exactly, the A operand of
//       O[channel][head] += sum_token V^T[channel][token] * P_g[token][head],
//   and the token's scale rides on the other operand: P_g = fp16(p_t * s_{t,g}), one per channel group g, the one
//   rounding of the product; the weights p carry a power of two that keeps it in fp16's normal range whatever the size
//   of the values (wexp below).  The int4 zero points and the centre come back as sum_t p_t (z_{t,g} + 8 s_{t,g}) in fp32 on
//   the vector units.  Values stored channel-major per 32 tokens (TTKV_I4_ASYM_G64_T32) are those operand words as they
//   lie.
//   fp16 / bf16 V, and int4 V beside keys grouped over tokens: rows like K's (the latter dequantized in packed fp16);
//   a product with the identity matrix brings the tile from [token][channel] to [channel][token]: the fp32 result
//   (exact) has lane (c, kg) holding channel-row c for tokens 4 kg .. 4 kg + 3, the A layout.  Two 16-token tiles feed
//   one 32-deep product.  The zero points and scales ride along as a 4-channel V.  P is rounded to fp16 once and that
//   rounded value is used for the row sum as well.
//   Keys grouped over 128 tokens per channel have no channel groups; the token group's scales fold into the q operand,
//   carried as fp16 rounded product + exact remainder (two products per step), rebuilt for every 64 tokens in flight.
//
// Bound: the memory system.  With every product taken out (same copies, same LDS reads) 8 x 64K tokens of K int8 / V int4
// take the same 81 us for 64 / 4 heads, 16 ragged sequences of K int4 / V4c 182 us (187 with them).  What matters is
// what keeps the copies fed and how the work is cut: 64 q / 4 kv heads, K int8 / V int4 110.3 -> 83.7 us per step
// (before: four score passes against zero-padded operands, one per group, 228 registers), 32 / 8 at 128K tokens
// 48.3 -> 44.6, block-sparse recall 129.5 -> 123.2.  Error against 64 bits, 4096 tokens, 2-norm: int8 values of standard
// deviation 1 to 0.005 1.8e-4 (rounding dequantized values: 2.8e-4), beside a token 7 above the rest 1e-6 (1.8e-4); int4
// 2.0e-4 (2.7e-4) and 1e-6 (1.4e-4).  More heads per KV head than 16 are cut into blocks of 16, one workgroup and one pass over the bytes per
// block.
#include "ttkv_attn_dev.h"

#include <algorithm>
#include <type_traits>

namespace ttkv {

namespace {

using namespace dev;

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));

template <bool BF>
__device__ __forceinline__ f4 mma(uint32_t a0, uint32_t a1, uint32_t b0, uint32_t b1, f4 c) {
  const uint2 A = {a0, a1}, B = {b0, b1};
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_16x16x16bf16_1k(__builtin_bit_cast(s4, A), __builtin_bit_cast(s4, B), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x16f16(__builtin_bit_cast(h4, A), __builtin_bit_cast(h4, B), c, 0, 0, 0);
}

typedef _Float16 h8 __attribute__((ext_vector_type(8)));
typedef __bf16 b8 __attribute__((ext_vector_type(8)));
// 32-deep step (v_mfma_f32_16x16x32): lane (c, kg) supplies eight k-values; which eight is free as long as
// the A and the B lane of the same kg agree, so two 16-deep steps simply concatenate.
template <bool BF>
__device__ __forceinline__ f4 mma32(const uint32_t *a, const uint32_t *b, f4 c) {
  const uint4 A = {a[0], a[1], a[2], a[3]}, B = {b[0], b[1], b[2], b[3]};
  if constexpr (BF)
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(b8, A), __builtin_bit_cast(b8, B), c, 0, 0, 0);
  else
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(h8, A), __builtin_bit_cast(h8, B), c, 0, 0, 0);
}

// two fp32 values -> packed fp16, round to nearest even (v_cvt_pk_f16_f32)
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint32_t pk(float x, float y) {
  const f2 v = {x, y};
  return __builtin_bit_cast(uint32_t, __builtin_convertvector(v, h2));
}

template <int F>
constexpr int n_groups() {
  return (F == TTKV_I4_ASYM_G64 || F == TTKV_I4_ASYM_G64_T32) ? 2 : (F == TTKV_I8_SYM_G32 ? 4 : 1);
}
// Channel, relative to the lane's 32-channel slice, of k-value i of step s: step s takes
// the packed registers 2s and 2s+1 that unpack16 produced (int4 pairs are (0,4) (1,5) | (2,6) (3,7)).
template <int F>
constexpr int chan(int s, int i) {
  if (is_i4<F>())
    return 8 * (s / 2) + ((s % 2) ? (i < 2 ? 2 + 4 * i : 3 + 4 * (i - 2)) : (i < 2 ? 4 * i : 1 + 4 * (i - 2)));
  return 4 * s + i;
}
// A lane's 32 channels of a value row are the 16-byte pieces kg, kg + 4, ... of it (piece x of the lane = bytes
// [64 x + 16 kg, + 16) of the row), so that every load instruction of a tile reads 64 contiguous bytes per row
// (measured on a load-only kernel: 6.3 TB/s, against 5.3 TB/s when a lane's pieces are adjacent).  Element j
// of the lane's slice (j = 4 s + i in unpack order for fp16 / bf16 / int8) is therefore row channel:
template <int F>
__device__ __forceinline__ constexpr int slice_channel(int kg, int j) {
  if (is_i4<F>()) return 32 * kg + j;                                     // one piece of 32 channels
  if (F == TTKV_I8_SYM_G32) return 64 * (j / 16) + 16 * kg + j % 16;      // two pieces of 16
  return 32 * (j / 8) + 8 * kg + j % 8;                                   // four pieces of 8
}
// Key rows with channel groups are sliced so that a 32-deep step stays inside one group: the lane takes 8 bytes of
// each 32-byte stretch, bytes [32 x + 8 kg, + 8): int8 channels 32 x + 8 kg .. (group x, step x), int4 channels
// 64 x + 16 kg .. (group x, steps 2 x and 2 x + 1).
template <int F>
__device__ __forceinline__ constexpr int key_channel(int kg, int j) {
  if (F == TTKV_I4_ASYM_G64) return 64 * (j / 16) + 16 * kg + j % 16;
  if (F == TTKV_I8_SYM_G32) return 32 * (j / 8) + 8 * kg + j % 8;
  return slice_channel<F>(kg, j);
}
// Splice offset carried by k-value i of a step.
template <int F>
constexpr float k_offset(int i) {
  return is_i4<F>() ? (i < 2 ? 1024.0f : 64.0f) : (F == TTKV_I8_SYM_G32 ? 1152.0f : 0.0f);
}

// ---- tiles of quantized rows prefetched through LDS
// The rows of a batch of tiles are copied global -> LDS asynchronously (no registers in between), the K half and
// the V half separately, while the batch before is being computed; the copy instructions read whole rows (whole
// 128-byte lines, so they carry the streaming hint), and the lanes then read their 16-byte pieces from LDS in the
// operand layout.  Inside LDS row r keeps its pieces in the order p ^ swz(r), which makes the 16 rows that the
// lanes of one piece read at a time fall into 16 different bank groups; the copy realises the order by choosing
// which piece each lane fetches.
// Per wave: K rows, V rows, and two buffers of four planes of meta words (K words 0 and 1 of the batch's tokens, V words
// 0 and 1), used in turn: a batch's meta words stay readable while the next batch arrives.
constexpr int kMetaLds = 4 * 256, kTileRowsLds = 8 * 1024, kTileLds = kTileRowsLds + 2 * kMetaLds;
typedef const __attribute__((address_space(1))) void *gas_ptr;
typedef __attribute__((address_space(3))) void *las_ptr;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
// lane L's 16 (4) bytes land at dst + 16 L (4 L); dst is wave-uniform; OFF is added to both addresses.
template <int OFF = 0>
__device__ __forceinline__ void dma16(const uint8_t *src, char *dst) {
  __builtin_amdgcn_global_load_lds((gas_ptr)src, (las_ptr)dst, 16, OFF, 2);   // 2: non-temporal
}
__device__ __forceinline__ void dma4(const uint8_t *src, char *dst) {
  __builtin_amdgcn_global_load_lds((gas_ptr)src, (las_ptr)dst, 4, 0, 2);
}
// At most N of the wave's vector-memory loads are still outstanding (they complete in order).
template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory");
}
// LDS reads of a landed half and the wait for them as one block (no use of a result can be scheduled in between;
// the reads are opaque to the compiler, which would otherwise wait for every copy in flight before an LDS read).
// fp16 / bf16: w[4 tt + x] = piece x of the lane of tile tt, from ax (tile 1: 4 KiB further); no meta words.
__device__ __forceinline__ void lds_half_fp(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x4 *w) {
  asm volatile("ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
               "ds_read_b128 %4, %8 offset:4096\n\tds_read_b128 %5, %9 offset:4096\n\t"
               "ds_read_b128 %6, %10 offset:4096\n\tds_read_b128 %7, %11 offset:4096\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// int8 key rows: w[4 tt + x] = the lane's 8 bytes of group x of tile tt, from ax (tile 1: 2 KiB further).
__device__ __forceinline__ void lds_keys_i8(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 *w) {
  asm volatile("ds_read_b64 %0, %8\n\tds_read_b64 %1, %9\n\tds_read_b64 %2, %10\n\tds_read_b64 %3, %11\n\t"
               "ds_read_b64 %4, %8 offset:2048\n\tds_read_b64 %5, %9 offset:2048\n\t"
               "ds_read_b64 %6, %10 offset:2048\n\tds_read_b64 %7, %11 offset:2048\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// int4 key rows: w[2 tt + x] = the lane's 8 bytes of group x of tile tt, from ax (tiles 1 KiB apart).
__device__ __forceinline__ void lds_keys_i4(uint32_t a0, uint32_t a1, u32x2 *w) {
  asm volatile("ds_read_b64 %0, %8\n\tds_read_b64 %1, %9\n\tds_read_b64 %2, %8 offset:1024\n\tds_read_b64 %3, %9 offset:1024\n\t"
               "ds_read_b64 %4, %8 offset:2048\n\tds_read_b64 %5, %9 offset:2048\n\t"
               "ds_read_b64 %6, %8 offset:3072\n\tds_read_b64 %7, %9 offset:3072\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(a0), "v"(a1) : "memory");
}
// Value rows, transposed on the way out of LDS (ds_read_b64_tr_*: the 16 lanes of one kg give the addresses of 16
// stretches of 8 bytes, i.e. of 16 rows x 16 nibbles or 8 rows x 16 bytes, and lane c receives column c of that block).
// int4, 64 tokens: lane L of the 16 names token 32 (L / 8) + kTok[L % 8] + 4 kg; block s of 16 channels is 8 bytes of
// the row; w[s] = the lane's channel, x: tokens of tiles 0 and 1, y: of tiles 2 and 3.
__device__ __forceinline__ void lds_values_i4x4(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 *w) {
  asm volatile("ds_read_b64_tr_b4 %0, %8\n\tds_read_b64_tr_b4 %1, %8 offset:8\n\tds_read_b64_tr_b4 %2, %9\n\t"
               "ds_read_b64_tr_b4 %3, %9 offset:8\n\tds_read_b64_tr_b4 %4, %10\n\tds_read_b64_tr_b4 %5, %10 offset:8\n\t"
               "ds_read_b64_tr_b4 %6, %11\n\tds_read_b64_tr_b4 %7, %11 offset:8\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// int4, 32 tokens: lane L names token kTok[L % 8] + 4 kg and block 2 q + L / 8; w[q] = blocks 2 q (x) and 2 q + 1 (y).
__device__ __forceinline__ void lds_values_i4x2(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 *w) {
  asm volatile("ds_read_b64_tr_b4 %0, %4\n\tds_read_b64_tr_b4 %1, %5\n\tds_read_b64_tr_b4 %2, %6\n\t"
               "ds_read_b64_tr_b4 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// int8, 32 tokens: lane L names token (L / 2) % 4 + 16 (L / 8) + 4 kg, bytes 8 (L % 2) of block s; w[s] = the lane's
// channel of block s, tokens 4 kg .. of tile 0 (x) and of tile 1 (y).  Four blocks.
__device__ __forceinline__ void lds_values_i8(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x2 *w) {
  asm volatile("ds_read_b64_tr_b8 %0, %4\n\tds_read_b64_tr_b8 %1, %5\n\tds_read_b64_tr_b8 %2, %6\n\t"
               "ds_read_b64_tr_b8 %3, %7\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
// channel-major values: the lane's pieces, 1 KiB apart
template <int NT>
__device__ __forceinline__ void lds_pieces(uint32_t a0, u32x4 *w) {
  if constexpr (NT == 4)
    asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:1024\n\tds_read_b128 %2, %4 offset:2048\n\t"
                 "ds_read_b128 %3, %4 offset:3072\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]) : "v"(a0) : "memory");
  else
    asm volatile("ds_read_b128 %0, %2\n\tds_read_b128 %1, %2 offset:1024\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]) : "v"(a0) : "memory");
}
// The two meta words of four consecutive tokens of two tiles: m[2 u + w] = words w of tile u, from a0 (tile 1: 64
// bytes further, words 1 one plane further); lanes of one kg read the same addresses.
__device__ __forceinline__ void lds_meta(uint32_t a0, u32x4 *m) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %4 offset:256\n\tds_read_b128 %2, %4 offset:64\n\t"
               "ds_read_b128 %3, %4 offset:320\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=&v"(m[3]) : "v"(a0) : "memory");
}
// The same with the two words of the lane's own token (one lane per token, from t0), for what is decided per batch.
__device__ __forceinline__ void lds_meta_own(uint32_t a0, uint32_t t0, u32x4 *m, u32x2 *t) {
  asm volatile("ds_read2_b32 %4, %6 offset1:64\n\t"
               "ds_read_b128 %0, %5\n\tds_read_b128 %1, %5 offset:256\n\tds_read_b128 %2, %5 offset:64\n\t"
               "ds_read_b128 %3, %5 offset:320\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(m[0]), "=&v"(m[1]), "=&v"(m[2]), "=&v"(m[3]), "=&v"(*t) : "v"(a0), "v"(t0) : "memory");
}
typedef unsigned short us2 __attribute__((ext_vector_type(2)));
// the larger halves of two words, as unsigned numbers
__device__ __forceinline__ uint32_t halves_max(uint32_t a, uint32_t b) {
  return __builtin_bit_cast(uint32_t, __builtin_elementwise_max(__builtin_bit_cast(us2, a), __builtin_bit_cast(us2, b)));
}
// the largest value of the wave's lanes (16-bit numbers)
__device__ __forceinline__ uint32_t wave_max16(uint32_t v) {
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true));    // quad_perm [1,0,3,2]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true));    // quad_perm [2,3,0,1]
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x141, 0xf, 0xf, true));   // row_half_mirror
  v = max(v, (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x140, 0xf, 0xf, true));   // row_mirror
  return max(max((uint32_t)__builtin_amdgcn_readlane((int)v, 0), (uint32_t)__builtin_amdgcn_readlane((int)v, 16)),
             max((uint32_t)__builtin_amdgcn_readlane((int)v, 32), (uint32_t)__builtin_amdgcn_readlane((int)v, 48)));
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }   // |e| < 127
// fp16 halves of a meta word
__device__ __forceinline__ float half0(uint32_t w) { return (float)as_h2(w).x; }
__device__ __forceinline__ float half1(uint32_t w) { return (float)as_h2(w).y; }

// Any number of query heads up to 16 (the columns of both products).
template <int KF, int VF>
__device__ __forceinline__ void process_mfma(const FusedArgs &a, const TierView &tv, const RunView &en, const int32_t *sel,
                                             int chunk_tokens, int chunk, int seq, int hq0, int Gr, int hkv, char *s_buf,
                                             float (*s_m)[16], float (*s_l)[16]) {
  // sel: null, or the block ids behind a run made of selected blocks (ring block of token i: sel[i / bt])
  // hq0, Gr: first query head and number of heads of this workgroup's block of heads (all heads of the KV head,
  // or a block of up to 16 of them)
  using FK = Fmt<KF>;
  using FV = Fmt<VF>;
  constexpr int NLK = FK::ROWB / 64, NLV = FV::ROWB / 64;   // 16-byte loads per lane per 16-token tile
  // Quantized keys: rows prefetched through LDS (asynchronous global -> LDS copies with the streaming hint, the batch
  // after next in flight while one is computed).  Measured per format against register loads: K8/V8 5.2 -> 6.0-6.2
  // TB/s, K8/V4 4.9-5.1 -> 5.7-5.8 (batches of 32 tokens); int4 keys in batches of 64 tokens: with channel-major
  // values 5.2 -> 5.97 (of which 32 -> 64 tokens per batch 5.85 -> 5.97), with token-major values 5.09 -> 5.27 (in
  // batches of 32 they gained nothing: their unpack / dequantize / transpose arithmetic fills the issue slots).
  // fp16 / bf16 rows take the one-region variant further down.
  constexpr bool PF = (KF == TTKV_I8_SYM_G32 && (VF == TTKV_I8_SYM_G32 || VF == TTKV_I4_ASYM_G64 || VF == TTKV_I4_ASYM_G64_T32)) ||
                      (KF == TTKV_I4_ASYM_G64 && (VF == TTKV_I4_ASYM_G64_T32 || VF == TTKV_I4_ASYM_G64));
  // tiles in flight per wave (int4 on register loads: 4; with 2 that kernel is 10 % slower)
  constexpr bool PF64 = KF == TTKV_I4_ASYM_G64 && (VF == TTKV_I4_ASYM_G64_T32 || VF == TTKV_I4_ASYM_G64);   // prefetched in batches of 64 tokens
  constexpr int NT = PF64 ? 4 : (NLK == 4 || PF) ? 2 : 4 / NLK;
  constexpr int TT = 16 * NT;
  constexpr int NGK = n_groups<KF>(), NGV = n_groups<VF>();
  constexpr bool KQ = NGK > 1, VQ = NGV > 1;
  constexpr bool KT = KF == TTKV_I4_ASYM_T128;   // keys grouped over 128 tokens per channel: the scales fold into q
  constexpr bool KBF = KF == TTKV_BF16, VBF = VF == TTKV_BF16;
  constexpr bool VT = VF == TTKV_I4_ASYM_G64_T32;   // values stored channel-major per 32 tokens
  constexpr bool V4 = PF && VF != TTKV_I8_SYM_G32;  // 4-bit codes as operand words (VT: as they lie; else transposed out of LDS)
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kg = lane >> 4;
  char *const wbuf = s_buf + wave * kTileLds;   // the wave's LDS: a batch of tiles in flight, at the end its result
  const int c0 = chunk * chunk_tokens;
  const int c1 = min(en.len, c0 + chunk_tokens);
  const int ring_tokens = tv.ring_blocks * tv.bt;
  const float cs = a.scale * kLog2e;       // scores are kept in the log2 domain

  const bool col_on = n < Gr;   // column = query head

  // ---- q operand: 16 packed registers (step s: 4 s .. 4 s + 3); per channel group of the keys the sum that the
  // splice offsets add to the products (it leaves with their initial value) and the plain sum (for the zero points).
  uint32_t qB[16];
  float off[NGK], qs[NGK];
  {
    const uint4 *qrow = (const uint4 *)((const uint16_t *)a.q + ((int64_t)seq * a.Hq + hq0 + min(n, Gr - 1)) * 128);
    uint32_t qw[16];
#pragma unroll
    for (int i = 0; i < 4; ++i) {     // 8 channels per 16-byte load
      const uint4 w = qrow[key_channel<KF>(kg, 8 * i) / 8];
      qw[4 * i] = w.x; qw[4 * i + 1] = w.y; qw[4 * i + 2] = w.z; qw[4 * i + 3] = w.w;
    }
    if constexpr (!KBF) {
      if (a.q_fmt == TTKV_BF16) {   // bf16 -> fp16 (exact inside the fp16 normal range, clamped outside)
#pragma unroll
        for (int i = 0; i < 16; ++i) {
          const float lo = fminf(fmaxf(__uint_as_float(qw[i] << 16), -65504.0f), 65504.0f);
          const float hi = fminf(fmaxf(__uint_as_float(qw[i] & 0xffff0000u), -65504.0f), 65504.0f);
          qw[i] = (uint32_t)__half_as_ushort(__float2half_rn(lo)) | ((uint32_t)__half_as_ushort(__float2half_rn(hi)) << 16);
        }
      }
    }
    // Register r of the operand pairs with register r of unpack16: elements (2r, 2r+1) of the slice, or for int4
    // (r = 4d + e) elements (8d + e, 8d + e + 4).
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};
    float se[NGK], so[NGK];   // sums over the registers that carry splice offset 1024 / 64 (int4: even / odd)
#pragma unroll
    for (int gr = 0; gr < NGK; ++gr) se[gr] = so[gr] = 0.0f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      uint32_t w = qw[r];
      if constexpr (is_i4<KF>()) {
        const int dd = r / 4, e = r % 4;
        w = __builtin_amdgcn_perm(qw[4 * dd + 2 + e / 2], qw[4 * dd + e / 2], (e & 1) ? 0x07060302u : 0x05040100u);
      }
      qB[r] = col_on ? w : 0u;
      if constexpr (KQ) {   // quantized keys are dotted with fp16 queries
        const int gr = r / (16 / NGK);
        if ((r & 1) && KF == TTKV_I4_ASYM_G64) so[gr] = __builtin_amdgcn_fdot2(as_h2(qB[r]), ones, so[gr], false);
        else se[gr] = __builtin_amdgcn_fdot2(as_h2(qB[r]), ones, se[gr], false);
      }
    }
#pragma unroll
    for (int gr = 0; gr < NGK; ++gr) {   // over the four channel slices
      qs[gr] = se[gr] + so[gr];
      off[gr] = KF == TTKV_I4_ASYM_G64 ? fmaf(1024.0f, se[gr], 64.0f * so[gr]) : k_offset<KF>(0) * se[gr];
      off[gr] += __shfl_xor(off[gr], 16); off[gr] += __shfl_xor(off[gr], 32);
      qs[gr] += __shfl_xor(qs[gr], 16);   qs[gr] += __shfl_xor(qs[gr], 32);
    }
  }

  // identity operand of the transposing product: k-value i of this lane is row 4 kg + i
  const uint32_t one = VBF ? 0x3F80u : 0x3C00u;
  const uint32_t id0 = (n == 4 * kg ? one : 0u) | (n == 4 * kg + 1 ? one << 16 : 0u);
  const uint32_t id1 = (n == 4 * kg + 2 ? one : 0u) | (n == 4 * kg + 3 ? one << 16 : 0u);
  // byte selector that duplicates the fp16 scale of group kg / 2 of this lane's piece out of the V meta words
  // (s0, z0, s1, z1): the values beside keys grouped over tokens are dequantized row by row
  const uint32_t vh = (kg >> 1) * 2;
  const uint32_t vsel = (2 * vh) | ((2 * vh + 1) << 8) | ((2 * vh) << 16) | ((2 * vh + 1) << 24);
  // minus (splice offset + centre) as packed fp16 pairs: int4 -(1024 + 8), -(64 + 8); int8 -(1024 + 128)
  uint32_t no_a = 0xE408E408u, no_b = 0xD480D480u, no_c = 0xE480E480u;
  asm volatile("" : "+s"(no_a), "+s"(no_b), "+s"(no_c));

  const f4 zero4 = f4{0.0f, 0.0f, 0.0f, 0.0f};
  f4 acc[8], accz = zero4;
  float zs[2] = {0.0f, 0.0f};     // V4: sum_t p_t (z_{t,g} + 8 s_{t,g})
#pragma unroll
  for (int s = 0; s < 8; ++s) acc[s] = zero4;
  float m = -INFINITY, l = 0.0f, mcs = INFINITY;   // a token's weight: exp2(score cs + mcs)
  // PF: the value operand is fp16(p s), and with p <= 1 that falls into fp16's subnormals or to zero for value scales
  // well below 1 (std 0.02 beside a token 7 above the rest: an error of 1.7e-2 of the output).  So the weights carry a
  // power of two that brings the largest value scale the wave has met to [2^14, 2^15): mcs = wexp - m cs, in l,
  // zs and acc alike; it leaves them at the end.  s_top: the largest fp16 number (as bits, ordered
  // like the numbers) of that scale's binade, so that only a scale of another binade takes the branch below.
  uint32_t s_top = 0;
  int wexp = 0;
  // (a maximum beyond 4 million has no bits left for it: such a column keeps weights up to 1)
  // Product and difference rounded one after the other: wexp - mcs, the reference of the item's result, is then exact.
  auto shift_of = [&](float mx) {
#pragma clang fp contract(off)
    const float r = mx * cs;
    return PF ? (fabsf(r) < 4194304.0f ? (float)wexp : 0.0f) - r : -r;
  };

  Splice sp;
  sp.init();

  struct TileRegs {
    uint4 kw[NT][NLK], vw[NT][NLV];
    uint32_t vop[NT / 2][8][VF == TTKV_I8_SYM_G32 ? 2 : 1];   // PF: codes of channel 16 s + n, the pair's 8 tokens of this kg
    uint2 vmeta[NT];
    uint4 gm[KT ? 8 : 1];   // KT: {scale, zero} of the lane's 32 channels for the token group of these tiles
  };
  const uint32_t kdoff = n * FK::ROWB + kg * 16, vdoff = n * FV::ROWB + kg * 16;

  // Plain loads here, not the non-temporal ones of the vector kernel: the load instructions of a tile share
  // cache lines (each reads 64 of a line's 128 bytes), and lines fetched with the streaming hint do not
  // survive until the next instruction.
  // Head section and row inside it of the chunk's token i.  The block table does not change during the launch and
  // the index is wave-uniform: it is read through the constant address space (a scalar load).
  auto locate = [&](int i, int &row0) -> const uint8_t * {
    int tok0 = en.first_tok + i;
    if (tok0 >= ring_tokens) tok0 -= ring_tokens;
    int rb = tok0 / tv.bt;
    row0 = tok0 - rb * tv.bt;
    typedef const __attribute__((address_space(4))) int32_t *const_i32;
    if (sel) rb = ((const_i32)(uintptr_t)sel)[rb] % tv.ring_blocks;   // written by the launch before this one: a scalar load
    const int64_t rec = tv.table ? (int64_t)((const_i32)(uintptr_t)tv.table)[(int64_t)seq * tv.ring_blocks + rb]
                                 : (int64_t)en.rec_base + rb;
    return tv.base + rec * tv.rec_bytes + (int64_t)hkv * tv.head_bytes;
  };
  auto load_tiles = [&](TileRegs &t, int i0, int nv, auto full_tag) {
    constexpr bool FULL = decltype(full_tag)::value;
    int row0;
    const uint8_t *head = locate(i0, row0);
    const uint8_t *kb = head + row0 * FK::ROWB;
    const uint8_t *vb = head + tv.v_off + row0 * FV::ROWB, *vmb = head + tv.v_meta_off + row0 * 8;
    if constexpr (KT) {   // the 64 tokens in flight lie inside one aligned group of 128: its 128 meta rows x 4 B
      const uint4 *gp = (const uint4 *)(head + tv.k_meta_off + (row0 & ~127) * 4 + kg * 128);
#pragma unroll
      for (int i = 0; i < 8; ++i) t.gm[i] = gp[i];
    }
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const uint32_t row = FULL ? tt * 16 + n : min(tt * 16 + n, nv - 1);   // rows past the end re-read the last live row
      const uint32_t ko = FULL ? kdoff + tt * 16 * FK::ROWB : row * FK::ROWB + kg * 16;
      const uint32_t vo = FULL ? vdoff + tt * 16 * FV::ROWB : row * FV::ROWB + kg * 16;
#pragma unroll
      for (int x = 0; x < NLK; ++x) t.kw[tt][x] = *(const uint4 *)(kb + ko + 64 * x);
#pragma unroll
      for (int x = 0; x < NLV; ++x) t.vw[tt][x] = *(const uint4 *)(vb + vo + 64 * x);
      if constexpr (VQ) t.vmeta[tt] = *(const uint2 *)(vmb + row * 8);
    }
  };

  // ---- PF: the same rows as asynchronous copies into the wave's LDS and reads from there.
  // LDS of the wave: K rows at 0, V rows at 4 KiB (row r at r ROWB, its piece p at 16 (p ^ swz(r))), then the two
  // buffers of meta planes.
  constexpr int PK = FK::ROWB / 16, PV = FV::ROWB / 16;              // pieces per row
  constexpr int NDK = TT * FK::ROWB / 1024, NDV = TT * FV::ROWB / 1024;   // copy instructions of 1 KiB per half
  constexpr int N_K = NDK + 4, N_V = NDV;                              // with the four meta planes
  static_assert(!PF || PF64 || (NT == 2 && ((PK == 8 && NDK == 4) || (PK == 4 && NDK == 2)) && (NDV == 4 || NDV == 2)),
                "the batch the LDS readers cover");
  auto swz = [](int pieces, int r) { return pieces == 4 ? (r >> 2) & 3 : (r >> 1) & 7; };
  // value rows: also different for the rows that the lanes of a transposing read name in different tiles
  auto swzv = [](int pieces, int r) { return pieces == 4 ? ((r >> 2) ^ (r >> 4)) & 3 : ((r >> 1) & 7) ^ ((r >> 3) & 2); };
  // per-lane byte offset of copy instruction j inside a full batch, minus j KiB: keys even and odd j differ for 8
  // pieces, values by an exchange of pieces (their rows' order is that of j = 0 with vx(j) added by exclusive or)
  uint32_t dko[2];
#pragma unroll
  for (int j = 0; j < 2; ++j) {
    const int rk = j * (64 / PK) + lane / PK;
    dko[j] = rk * FK::ROWB + ((lane % PK) ^ swz(PK, rk)) * 16 - j * 1024;
  }
  const uint32_t dvo = lane / PV * FV::ROWB + ((lane % PV) ^ swzv(PV, lane / PV)) * 16;
  constexpr auto vx = [](int j) { return PV == 4 ? j * 16 : (j & 1) * 64 + (j >> 1) * 32; };
  const uint32_t lds0 = (uint32_t)(uintptr_t)(las_ptr)wbuf;
  // the lane's 8 bytes of the 32-byte stretch x of row n: half kg % 2 of piece 2 x + kg / 2
  uint32_t lka[4];
#pragma unroll
  for (int x = 0; x < 4; ++x) {
    const int p = (2 * x) % PK + (kg >> 1);
    lka[x] = lds0 + n * FK::ROWB + ((p ^ swz(PK, n)) * 16) + 8 * (kg & 1);
  }
  // what the lane names to the transposing value reads: its row's first piece (the others by exclusive or with 16 x piece)
  uint32_t lva = lds0 + 4096 + lane * 16;
  if constexpr (PF && !VT) {
    const int r4 = 2 * (n & 1) + 16 * ((n >> 1) & 1) + ((n >> 2) & 1) + 4 * kg;   // kTok[n % 8] + 4 kg
    const int row = PV == 8 ? ((n >> 1) & 3) + 16 * (n >> 3) + 4 * kg : PF64 ? r4 + 32 * (n >> 3) : r4;
    const int half = PV == 8 ? n & 1 : PF64 ? 0 : n >> 3;
    lva = lds0 + 4096 + row * FV::ROWB + swzv(PV, row) * 16 + 8 * half;
  }
  uint32_t meta_in = 0, meta_cur = 0;   // meta buffer (byte offset) of the batch being issued / computed
  const uint8_t *nx_head = nullptr;   // batch whose K half was issued last
  int nx_row0 = 0, nx_nv = 0;
  auto issue_k = [&](int i0) {
    nx_head = locate(i0, nx_row0);
    nx_nv = min(TT, c1 - i0);
    const uint8_t *kb = nx_head + nx_row0 * FK::ROWB, *kmb = nx_head + tv.k_meta_off + nx_row0 * 8;
    if (nx_nv == TT) {
      dma16<0>(kb + dko[0], wbuf); dma16<1024>(kb + dko[1], wbuf);
      if constexpr (NDK == 4) {
        dma16<2048>(kb + dko[0], wbuf); dma16<3072>(kb + dko[1], wbuf);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NDK; ++j) {
        const int r = j * (64 / PK) + lane / PK;   // LDS row; rows past the end repeat the last live row
        dma16(kb + min(r, nx_nv - 1) * FK::ROWB + ((lane % PK) ^ swz(PK, r)) * 16, wbuf + j * 1024);
      }
    }
    const uint32_t mo = min(lane, nx_nv - 1) * 8;   // one lane per token (TT = 32: the upper lanes repeat the last row)
    dma4(kmb + mo, wbuf + kTileRowsLds + meta_in);
    dma4(kmb + mo + 4, wbuf + kTileRowsLds + meta_in + 256);
    const uint8_t *vmb = nx_head + tv.v_meta_off + nx_row0 * 8;   // the values' too: their scales are looked at with the scores
    dma4(vmb + mo, wbuf + kTileRowsLds + meta_in + 512);
    dma4(vmb + mo + 4, wbuf + kTileRowsLds + meta_in + 768);
    meta_in ^= kMetaLds;
  };
  auto issue_v = [&]() {
    const uint8_t *vb = nx_head + tv.v_off + nx_row0 * FV::ROWB;
    if constexpr (VT) {   // whole 2 KiB groups (lengths are multiples of 32), copied as they lie
      dma16<0>(vb + lane * 16, wbuf + 4096); dma16<1024>(vb + lane * 16, wbuf + 4096);
      if constexpr (PF64) {   // the second group: inside the record even when the run ends before it (its weights are 0)
        dma16<2048>(vb + lane * 16, wbuf + 4096); dma16<3072>(vb + lane * 16, wbuf + 4096);
      }
    } else if (nx_nv == TT) {
      dma16<0>(vb + dvo, wbuf + 4096); dma16<1024>(vb + (dvo ^ vx(1)), wbuf + 4096);
      if constexpr (NDV == 4) {
        dma16<2048>(vb + (dvo ^ vx(2)), wbuf + 4096); dma16<3072>(vb + (dvo ^ vx(3)), wbuf + 4096);
      }
    } else {
#pragma unroll
      for (int j = 0; j < NDV; ++j) {
        const int r = j * (64 / PV) + lane / PV;
        dma16(vb + min(r, nx_nv - 1) * FV::ROWB + ((lane % PV) ^ swzv(PV, r)) * 16, wbuf + 4096 + j * 1024);
      }
    }
  };
  // Rows in pinned host memory: the whole batch through registers into the same places (over PCIe the asynchronous
  // copies were 3-4 % slower, and the streaming hint has nothing to gain there).  Lane (n, kg) moves piece kg (+ 4) of
  // row n of every tile, one lane per token its meta words.
  auto bring_host = [&](int i0) {
    int row0;
    const uint8_t *head = locate(i0, row0);
    const int nv = min(TT, c1 - i0);
    const uint8_t *kb = head + row0 * FK::ROWB, *vb = head + tv.v_off + row0 * FV::ROWB;
    uint4 kw[NT][NLK], vw[NT][NLV];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const uint32_t row = min(tt * 16 + n, nv - 1);   // rows past the end repeat the last live row
#pragma unroll
      for (int x = 0; x < NLK; ++x) kw[tt][x] = *(const uint4 *)(kb + row * FK::ROWB + kg * 16 + 64 * x);
      if constexpr (VT) {
        // piece hh = tt % 2 of the 32-token group tt / 2 (a group past the end repeats the last live one)
        vw[tt][0] = *(const uint4 *)(vb + min(tt / 2, (nv - 1) / 32) * 2048 + (tt & 1) * 1024 + lane * 16);
      } else {
#pragma unroll
        for (int x = 0; x < NLV; ++x) vw[tt][x] = *(const uint4 *)(vb + row * FV::ROWB + kg * 16 + 64 * x);
      }
    }
    const uint32_t mo = (row0 + min(lane, nv - 1)) * 8;
    const uint2 km = *(const uint2 *)(head + tv.k_meta_off + mo), vm = *(const uint2 *)(head + tv.v_meta_off + mo);
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
      for (int x = 0; x < NLK; ++x)
        *(uint4 *)(wbuf + (tt * 16 + n) * FK::ROWB + (((kg + 4 * x) ^ swz(PK, n)) * 16)) = kw[tt][x];
      if constexpr (VT) {
        *(uint4 *)(wbuf + 4096 + tt * 1024 + lane * 16) = vw[tt][0];
      } else {
#pragma unroll
        for (int x = 0; x < NLV; ++x)
          *(uint4 *)(wbuf + 4096 + (tt * 16 + n) * FV::ROWB + (((kg + 4 * x) ^ swzv(PV, tt * 16 + n)) * 16)) = vw[tt][x];
      }
    }
    uint32_t *m = (uint32_t *)(wbuf + kTileRowsLds) + lane;   // buffer 0
    m[0] = km.x;
    m[64] = km.y;
    m[128] = vm.x;
    m[192] = vm.y;
  };
  auto fetch_k = [&](auto &t) {   // generic: compiled only where it is called, i.e. for the formats of PF
    u32x2 w[8];
    if constexpr (PK == 8) lds_keys_i8(lka[0], lka[1], lka[2], lka[3], w);
    else lds_keys_i4(lka[0], lka[1], w);
#pragma unroll
    for (int tt = 0; tt < NT; ++tt)
#pragma unroll
      for (int x = 0; x < NLK; ++x) {
        const u32x2 v0 = w[2 * (tt * NLK + x)], v1 = w[2 * (tt * NLK + x) + 1];
        t.kw[tt][x] = uint4{v0.x, v0.y, v1.x, v1.y};
      }
  };
  auto fetch_v = [&](auto &t) {
    if constexpr (VT) {   // word w of piece hh: block 4 hh + w
      u32x4 w[4];
      lds_pieces<NT>(lva, w);
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int pr = 0; pr < NT / 2; ++pr) t.vop[pr][s][0] = w[2 * pr + s / 4][s % 4];
    } else {
      u32x2 w[8];
      if constexpr (PV == 8) {
        uint32_t va = lva;
        asm volatile("" : "+v"(va));   // formed again in every batch: kept, the eight addresses made the loop spill
        lds_values_i8(va, va ^ 16, va ^ 32, va ^ 48, w);
        lds_values_i8(va ^ 64, va ^ 80, va ^ 96, va ^ 112, w + 4);
      } else if constexpr (PF64) {
        lds_values_i4x4(lva, lva ^ 16, lva ^ 32, lva ^ 48, w);
      } else {
        lds_values_i4x2(lva, lva ^ 16, lva ^ 32, lva ^ 48, w);
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if constexpr (PV == 8) {
          t.vop[0][s][0] = w[s].x;
          t.vop[0][s][1] = w[s].y;
        } else if constexpr (PF64) {
          t.vop[0][s][0] = w[s].x;
          t.vop[1][s][0] = w[s].y;
        } else {
          t.vop[0][s][0] = s % 2 ? w[s / 2].y : w[s / 2].x;
        }
      }
    }
  };

  // before_v runs between the softmax and the first use of the batch's V half.
  auto compute_tiles = [&](TileRegs &t, int nv, auto full_tag, auto before_v) {
    constexpr bool FULL = decltype(full_tag)::value;
    // ---- KT: q . k = sum_d (q_d s_d) (c_d - 8) + sum_d q_d (z_d + 8 s_d) with s, z of the token group.  q_d s_d
    // is carried as two fp16 operands (rounded product and exact remainder), both multiplied with the codes;
    // the sums over q s and q z are exact products accumulated in fp32 and leave with the initial value.
    uint32_t qh[KT ? 16 : 1], ql[KT ? 16 : 1];
    float off_t = 0.0f;
    if constexpr (KT) {
      float se = 0.0f, so = 0.0f, qz = 0.0f;
#pragma unroll
      for (int dd = 0; dd < 4; ++dd) {
        const uint32_t m8[8] = {t.gm[2 * dd].x, t.gm[2 * dd].y, t.gm[2 * dd].z, t.gm[2 * dd].w,
                                t.gm[2 * dd + 1].x, t.gm[2 * dd + 1].y, t.gm[2 * dd + 1].z, t.gm[2 * dd + 1].w};
#pragma unroll
        for (int j = 0; j < 4; ++j) {   // operand register 4 dd + j holds channels (8 dd + j, 8 dd + j + 4) of the slice
          const int r = 4 * dd + j;
          const h2 s2 = as_h2(__builtin_amdgcn_perm(m8[j + 4], m8[j], 0x05040100u));
          const h2 z2 = as_h2(__builtin_amdgcn_perm(m8[j + 4], m8[j], 0x07060302u));
          const h2 q2 = as_h2(qB[r]);
          const h2 hi = q2 * s2;
          qh[r] = __builtin_bit_cast(uint32_t, hi);
          ql[r] = __builtin_bit_cast(uint32_t, __builtin_elementwise_fma(q2, s2, -hi));
          if (r & 1) so = __builtin_amdgcn_fdot2(q2, s2, so, false);
          else se = __builtin_amdgcn_fdot2(q2, s2, se, false);
          qz = __builtin_amdgcn_fdot2(q2, z2, qz, false);
        }
      }
      // splice offsets 1024 / 64 plus the centre 8, minus the zero-point sum; summed over the four channel slices
      off_t = fmaf(1032.0f, se, 72.0f * so) - fmaf(8.0f, se + so, qz);
      off_t += __shfl_xor(off_t, 16);
      off_t += __shfl_xor(off_t, 32);
    }

    // ---- scores (log2 domain), column n of tokens 4 kg + i
    f4 S[NT];
    float mt = -INFINITY;
    uint32_t top = 0;   // PF: the largest value scale of the lane's own token (one lane per token)
    u32x4 km[4];   // the meta words of the lane's tokens 4 kg + i of two tiles, straight in the score layout
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      if constexpr (KQ)
        if (tt % 2 == 0) {
          const uint32_t plane = lds0 + kTileRowsLds + meta_cur;
          if (tt == 0) {
            u32x2 own;
            lds_meta_own(plane + 16 * kg, plane + 512 + 4 * lane, km, &own);
            top = halves_max(own.x, own.y);                       // scales are not negative
            top = V4 ? top & 0xffffu : max(top & 0xffffu, top >> 16);
          } else {
            lds_meta(plane + 64 * tt + 16 * kg, km);
          }
        }
      uint32_t kr[16];
#pragma unroll
      for (int x = 0; x < NLK; ++x) unpack16<KF>(t.kw[tt][x], kr + x * (16 / NLK), sp);
      // one product chain per channel group
      f4 sv[NGK];
#pragma unroll
      for (int gr = 0; gr < NGK; ++gr) {
        if constexpr (KT) {
          sv[gr] = f4{-off_t, -off_t, -off_t, -off_t};
#pragma unroll
          for (int s = 0; s < 4; ++s) {
            sv[gr] = mma32<false>(kr + 4 * s, qh + 4 * s, sv[gr]);
            sv[gr] = mma32<false>(kr + 4 * s, ql + 4 * s, sv[gr]);
          }
        } else {
          sv[gr] = f4{-off[gr], -off[gr], -off[gr], -off[gr]};
#pragma unroll
          for (int s = gr * (4 / NGK); s < (gr + 1) * (4 / NGK); ++s) sv[gr] = mma32<KBF>(kr + 4 * s, qB + 4 * s, sv[gr]);
        }
      }
      const u32x4 m0 = km[2 * (tt & 1)], m1 = km[2 * (tt & 1) + 1];
      f4 sc;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float x = sv[0][i];
        if constexpr (KF == TTKV_I8_SYM_G32) {        // scales of groups 0 .. 3
          x *= half0(m0[i]);
          x = fmaf(sv[1][i], half1(m0[i]), x);
          x = fmaf(sv[2][i], half0(m1[i]), x);
          x = fmaf(sv[3][i], half1(m1[i]), x);
        } else if constexpr (KF == TTKV_I4_ASYM_G64) {   // scale, zero point of group 0; of group 1
          x = fmaf(half1(m0[i]), qs[0], half1(m1[i]) * qs[1]) + fmaf(sv[0][i], half0(m0[i]), sv[1][i] * half0(m1[i]));
        }
        if (!FULL && tt * 16 + 4 * kg + i >= nv) x = -INFINITY;
        sc[i] = x;
        mt = fmaxf(mt, x);
      }
      S[tt] = sc;
    }

    // ---- online softmax (base 2) per column; m is kept in raw score units, the scale enters the exponent
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    if (__any(mt > m || top > s_top)) {
      const float mn = fmaxf(m, mt), old = mcs;
      if constexpr (PF) {
        if (__any(top > s_top)) {
          s_top = wave_max16(top) | 0x3ffu;
          wexp = 29 - max((int)(s_top >> 10), 1);
        }
      }
      mcs = shift_of(mn);
      const float alpha = PF ? __builtin_amdgcn_exp2f(mcs - old) : __builtin_amdgcn_exp2f((m - mn) * cs);
      l *= alpha;
      accz *= alpha;
      if constexpr (V4) {
        zs[0] *= alpha; zs[1] *= alpha;
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[s] *= alpha;
      m = mn;
    }
    const h2 ones = {(_Float16)1.0f, (_Float16)1.0f};

    // ---- weighted V, two 16-token tiles per 32-deep product
    before_v();
    if constexpr (PF) {
      // The codes' words are the A operands of the eight channel blocks after the splice, whose offset leaves exactly
      // (with the centre 8 of 4-bit codes); the scales ride on the weights.  One rounding per product: fp16(p s).
#pragma unroll
      for (int tp = 0; tp < NT; tp += 2) {
        u32x4 vm[4];             // meta words of the lane's tokens 4 kg + i: 4-bit (scale, zero point) of groups 0 and 1, 8-bit scales
        lds_meta(lds0 + kTileRowsLds + meta_cur + 512 + 64 * tp + 16 * kg, vm);
        uint32_t Bg[NGV][4];     // fp16(p_t * s_{t,g}) of the pair's 8 tokens per lane, per channel group g
#pragma unroll
        for (int u = 0; u < 2; ++u) {
          const int tt = tp + u;
          const u32x4 m0 = vm[2 * u], m1 = vm[2 * u + 1];
          float p[4], b[NGV][4];
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            p[i] = __builtin_amdgcn_exp2f(fmaf(S[tt][i], cs, mcs));
            l += p[i];
            if constexpr (V4) {
              zs[0] = fmaf(p[i], fmaf(8.0f, half0(m0[i]), half1(m0[i])), zs[0]);   // zero point + the centre 8 * scale
              zs[1] = fmaf(p[i], fmaf(8.0f, half0(m1[i]), half1(m1[i])), zs[1]);
              b[0][i] = p[i] * half0(m0[i]);
              b[1][i] = p[i] * half0(m1[i]);
            } else {
              b[0][i] = p[i] * half0(m0[i]);
              b[1][i] = p[i] * half1(m0[i]);
              b[2][i] = p[i] * half0(m1[i]);
              b[3][i] = p[i] * half1(m1[i]);
            }
          }
#pragma unroll
          for (int gr = 0; gr < NGV; ++gr) {
            Bg[gr][2 * u] = pk(b[gr][0], b[gr][1]);
            Bg[gr][2 * u + 1] = pk(b[gr][2], b[gr][3]);
          }
        }
#pragma unroll
        for (int s = 0; s < 8; ++s) {
          uint32_t vr[4];
          const int gr = s / (8 / NGV);
          if constexpr (V4) {
            splice4(t.vop[tp / 2][s][0], vr, sp);
#pragma unroll
            for (int r = 0; r < 4; ++r) vr[r] = __builtin_bit_cast(uint32_t, as_h2(vr[r]) + as_h2((r & 1) ? no_b : no_a));
          } else {
#pragma unroll
            for (int h = 0; h < 2; ++h) {
              const uint32_t x = t.vop[tp / 2][s][h] ^ 0x80808080u;               // byte -> code + 128
              vr[2 * h] = __builtin_amdgcn_perm(0x64646464u, x, 0x04010400u);      // (1024 + b0, 1024 + b1)
              vr[2 * h + 1] = __builtin_amdgcn_perm(0x64646464u, x, 0x04030402u);
            }
#pragma unroll
            for (int r = 0; r < 4; ++r) vr[r] = __builtin_bit_cast(uint32_t, as_h2(vr[r]) + as_h2(no_c));
          }
          acc[s] = mma32<false>(vr, Bg[gr], acc[s]);
        }
      }
    } else {
#pragma unroll
    for (int tp = 0; tp < NT; tp += 2) {
      uint32_t pB[4];          // softmax weights of the pair, rounded to fp16: the B operand
      uint32_t vr[2][16];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int tt = tp + u;
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(S[tt][i], cs, mcs));
        pB[2 * u] = pk(p[0], p[1]);
        pB[2 * u + 1] = pk(p[2], p[3]);
        l = __builtin_amdgcn_fdot2(as_h2(pB[2 * u]), ones, l, false);       // the row sum uses the rounded weights
        l = __builtin_amdgcn_fdot2(as_h2(pB[2 * u + 1]), ones, l, false);

#pragma unroll
        for (int x = 0; x < NLV; ++x) unpack16<VF>(t.vw[tt][x], vr[u] + x * (16 / NLV), sp);
        if constexpr (VQ) {
          // codes -> code * scale in fp16 with one rounding (to nearest even), while the lane still owns one token
          // and one group.  The splice holds offset + code; the centred code (code - 8) is taken out first, which is exact, and then scaled, so that the one rounding is relative to a value of
          // the size of the element itself (scaling offset + code in one fused step and removing offset * scale
          // afterwards would round a value up to the row's whole range: an error of range x 2^-11 on its smallest
          // elements).  The int4 centre 8 * scale rejoins with the zero points at the end.
          const h2 vs2 = as_h2(__builtin_amdgcn_perm(t.vmeta[tt].y, t.vmeta[tt].x, vsel));
#pragma unroll
          for (int r = 0; r < 16; ++r) vr[u][r] = __builtin_bit_cast(uint32_t, (as_h2(vr[u][r]) + as_h2((r & 1) ? no_b : no_a)) * vs2);
        }
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        const f4 d0 = mma<VBF>(vr[0][2 * s], vr[0][2 * s + 1], id0, id1, zero4);
        const f4 d1 = mma<VBF>(vr[1][2 * s], vr[1][2 * s + 1], id0, id1, zero4);
        const uint32_t A[4] = {pk(d0[0], d0[1]), pk(d0[2], d0[3]), pk(d1[0], d1[1]), pk(d1[2], d1[3])};
        acc[s] = mma32<false>(A, pB, acc[s]);
      }
      if constexpr (VF == TTKV_I4_ASYM_G64) {
        // the meta words transposed like a 4-channel V: every row group of four then accumulates
        // sum_t p_t * (s0, z0, s1, z1)
        const f4 d0 = mma<false>(t.vmeta[tp].x, t.vmeta[tp].y, id0, id1, zero4);
        const f4 d1 = mma<false>(t.vmeta[tp + 1].x, t.vmeta[tp + 1].y, id0, id1, zero4);
        const uint32_t A[4] = {pk(d0[0], d0[1]), pk(d0[2], d0[3]), pk(d1[0], d1[1]), pk(d1[2], d1[3])};
        accz = mma32<false>(A, pB, accz);
      }
    }
    }
  };

  // ---- fp16 / bf16 rows through LDS: a half (K or V rows of a batch of 32 tokens) is 8 KiB, so the wave's LDS
  // takes one half at a time: K of batch i is read out, V of batch i is copied in while the scores are computed,
  // read out, K of batch i + 1 copied in while the weighted values are computed.  Row r keeps its 16 pieces in the
  // order p ^ (r & 15).
  constexpr bool PF2 = (KF == TTKV_F16 || KF == TTKV_BF16) && KF == VF;
  const uint8_t *cur_head = nullptr;
  int cur_row0 = 0, cur_nv = 0;
  auto issue_fp = [&](const uint8_t *rows, int nv) {   // rows: the half's first row
    if (nv == 32) {
      const uint32_t r0 = lane >> 4, s0 = (lane & 15) ^ r0;   // copy j: row 4 j + r0, piece s0 ^ 4 (j & 3)
      const uint8_t *a0 = rows + r0 * 256 + s0 * 16, *a1 = rows + r0 * 256 + (s0 ^ 4) * 16;
      const uint8_t *a2 = rows + r0 * 256 + (s0 ^ 8) * 16, *a3 = rows + r0 * 256 + (s0 ^ 12) * 16;
      dma16<0>(a0, wbuf); dma16<1024>(a1, wbuf); dma16<2048>(a2, wbuf); dma16<3072>(a3, wbuf);
      dma16<0>(a0 + 4096, wbuf + 4096); dma16<1024>(a1 + 4096, wbuf + 4096);
      dma16<2048>(a2 + 4096, wbuf + 4096); dma16<3072>(a3 + 4096, wbuf + 4096);
    } else {
#pragma unroll
      for (int j = 0; j < 8; ++j) {
        const int r = 4 * j + (lane >> 4);   // LDS row; rows past the end repeat the last live row
        dma16(rows + min(r, nv - 1) * 256 + (((lane & 15) ^ (r & 15)) * 16), wbuf + j * 1024);
      }
    }
  };
  auto fetch_fp = [&](auto *dst) {   // dst: kw or vw of the tile registers
    const uint32_t base = (uint32_t)(uintptr_t)(las_ptr)wbuf + n * 256 + ((kg ^ (n & 3)) * 16);
    const uint32_t hi = n >> 2;   // piece kg + 4 x sits at slot (kg ^ (n & 3)) + 4 (x ^ hi)
    u32x4 w[8];
    lds_half_fp(base + ((0 ^ hi) << 6), base + ((1 ^ hi) << 6), base + ((2 ^ hi) << 6), base + ((3 ^ hi) << 6), w);
#pragma unroll
    for (int tt = 0; tt < 2; ++tt)
#pragma unroll
      for (int x = 0; x < 4; ++x) {
        const u32x4 v = w[4 * tt + x];
        dst[tt][x] = uint4{v.x, v.y, v.z, v.w};
      }
  };
  auto fp_loop = [&](auto &ra) {   // generic: compiled only for the formats of PF2
    int i0 = c0 + wave * TT;
    if (i0 < c1) {
      cur_head = locate(i0, cur_row0);
      cur_nv = min(TT, c1 - i0);
      issue_fp(cur_head + cur_row0 * 256, cur_nv);
    }
    auto step = [&](int nv, auto full_tag) {
      wait_vmcnt<0>();
      fetch_fp(ra.kw);
      issue_fp(cur_head + tv.v_off + cur_row0 * 256, cur_nv);
      compute_tiles(ra, nv, full_tag, [&]() {
        wait_vmcnt<0>();
        fetch_fp(ra.vw);
        if (i0 + 4 * TT < c1) {   // wave-uniform
          cur_head = locate(i0 + 4 * TT, cur_row0);
          cur_nv = min(TT, c1 - i0 - 4 * TT);
          issue_fp(cur_head + cur_row0 * 256, cur_nv);
        }
      });
    };
    for (; i0 + TT <= c1; i0 += 4 * TT) step(TT, std::true_type{});
    if (i0 < c1) step(c1 - i0, std::false_type{});
  };

  auto register_loop = [&]() {
    TileRegs ra;
    int i0 = c0 + wave * TT;
    for (; i0 + TT <= c1; i0 += 4 * TT) {
      load_tiles(ra, i0, TT, std::true_type{});
      compute_tiles(ra, TT, std::true_type{}, []() {});
    }
    if (i0 < c1) {
      load_tiles(ra, i0, c1 - i0, std::false_type{});
      compute_tiles(ra, c1 - i0, std::false_type{}, []() {});
    }
  };
  if constexpr (PF) {
    TileRegs ra;
    int i0 = c0 + wave * TT;
    if (!tv.in_host) {
      // While batch i is computed the copies of batch i + 1 are in flight: its K half is issued once batch i's K
      // rows are in registers, its V half once batch i's V rows are.  Loads complete in order, so "at most as
      // many outstanding as were issued after it" means a half has landed.
      if (i0 < c1) {
        issue_k(i0);
        issue_v();
      }
      auto step = [&](int nv, auto full_tag) {
        const bool more = i0 + 4 * TT < c1;   // wave-uniform
        wait_vmcnt<N_V>();
        fetch_k(ra);
        if (more) issue_k(i0 + 4 * TT);
        compute_tiles(ra, nv, full_tag, [&]() {
          if (more) wait_vmcnt<N_K>();
          else wait_vmcnt<0>();
          fetch_v(ra);
          if (more) issue_v();
        });
        meta_cur ^= kMetaLds;
      };
      for (; i0 + TT <= c1; i0 += 4 * TT) step(TT, std::true_type{});
      if (i0 < c1) step(c1 - i0, std::false_type{});
    } else {
      for (; i0 < c1; i0 += 4 * TT) {
        bring_host(i0);
        fetch_k(ra);
        compute_tiles(ra, min(TT, c1 - i0), std::false_type{}, [&]() { fetch_v(ra); });
      }
    }
  } else if constexpr (PF2) {
    static_assert(!PF2 || (TT == 32 && NT == 2 && NLK == 4 && NLV == 4), "the batch the LDS readers cover");
    // also for a tier in pinned host memory: the copies read whole 256-byte rows, where the register loads ask
    // for 64 bytes of a row per instruction -- over PCIe 55.7 against 42.8 GB/s (measured)
    TileRegs ra;
    fp_loop(ra);
  } else {
    register_loop();
  }

  // ---- the wave's result: column n < G of lane (n, kg) holds, in acc[s][i], the row channel of slice element
  // chan(s, i); the zero-point sums of that channel's group are added here
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  float z[2] = {0.0f, 0.0f};   // zero-point sum of the channels' group
  if constexpr (KT)   // sum_t p_t * (zero + 8 * scale)
    z[0] = z[1] = (kg >> 1) ? fmaf(8.0f, accz[2], accz[3]) : fmaf(8.0f, accz[0], accz[1]);
  if constexpr (V4) {   // per channel group: the lanes' zero-point sums over their tokens
#pragma unroll
    for (int g2 = 0; g2 < 2; ++g2) {
      zs[g2] += __shfl_xor(zs[g2], 16);
      zs[g2] += __shfl_xor(zs[g2], 32);
      z[g2] = zs[g2];
    }
  }
  // what the weights are relative to (log2 domain), and the power of two they carry
  const float wcol = PF && fabsf(m * cs) < 4194304.0f ? (float)wexp : 0.0f, unscale = pow2(-(int)wcol);
  const float m2 = PF ? wcol - mcs : m * cs;
  float (*w_acc)[128] = (float (*)[128])wbuf;   // [head][channel]; the wave's last batch has been consumed
  if (n < Gr) {
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        if constexpr (PF) w_acc[n][16 * s + 4 * kg + i] = (acc[s][i] + z[s / 4]) * unscale;   // block s row 4 kg + i, as the product leaves it
        else w_acc[n][slice_channel<VF>(kg, chan<VF>(s, i))] = acc[s][i] + z[s / 4];
      }
    if (kg == 0) {
      s_m[wave][n] = m2;
      s_l[wave][n] = l * unscale;
    }
  }
}

// FOUR_BIT: the launch has a tier with 4-bit keys or values.  Those cases are held to two workgroups per CU (the plan counts on it); the
// others run three.  T128: also one whose keys are grouped over 128 tokens per channel.
template <bool FOUR_BIT, bool T128>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(FOUR_BIT ? 2 : 3, FOUR_BIT ? 2 : 3))) void attn_mfma_kernel(const FusedArgs a) {
  static_assert(kTileLds >= 16 * 128 * 4, "the wave's result fits its tile buffer");
  __shared__ __attribute__((aligned(256))) char s_buf[4 * kTileLds];   // per wave: batch in flight, then [head][channel] floats
  __shared__ float s_m[4][16], s_l[4][16];

  // Linear workgroup id -> (item, KV head, block of heads).  More heads per KV head than one tile takes are cut
  // into blocks of mfma_heads; the blocks of one (item, KV head) read the same bytes and get ids 8 apart, so that
  // they run on the same XCD at the same time and the later readers are served from its L2.
  const int Gtot = a.Hq / a.Hkv;
  const uint32_t n_hb = (Gtot + a.mfma_heads - 1) / a.mfma_heads;
  const uint32_t id = blockIdx.x;
  const uint32_t base = ((id >> 3) / n_hb) * 8 + (id & 7);
  if (base >= (uint32_t)a.n_items * a.Hkv) return;
  const int item = base / a.Hkv;
  const int hkv = base % a.Hkv;
  const int hb0 = ((id >> 3) % n_hb) * a.mfma_heads;          // first head of the block within the KV head's heads
  const int hq0 = hkv * Gtot + hb0;
  const int G = min(a.mfma_heads, Gtot - hb0);                // heads in this block

  int lo = 0, hi = a.n_entries - 1;
  while (lo < hi) {
    const int mid = (lo + hi + 1) >> 1;
    if (a.e[mid].item_start <= item) lo = mid; else hi = mid - 1;
  }
  RunView en = run_view(a, lo);
  const int tier = en.tier, seq = en.seq, item_start = a.e[lo].item_start;
  TierView tv = a.tv[tier];
  if (en.flags & kEntryNoTable) tv.table = nullptr;   // the run names pool records directly
  int chunk_tokens = a.chunk[tier];
  const bool equal_items = chunk_tokens == 0;
  if (equal_items) chunk_tokens = even_chunk(en.len, (lo + 1 < a.n_entries ? a.e[lo + 1].item_start : a.n_items) - item_start);
  const int part = en.part_base + item - item_start;   // this item's partial
  int chunk = item - item_start;
  const int32_t *sel = resolve_selected(a, tv, en, seq, equal_items, chunk_tokens, chunk);

  const int combo = tv.k_fmt * 8 + tv.v_fmt;
#define TTKV_MFMA_CASE(KF, VF) process_mfma<KF, VF>(a, tv, en, sel, chunk_tokens, chunk, seq, hq0, G, hkv, s_buf, s_m, s_l)
  switch (combo) {
    case TTKV_F16 * 8 + TTKV_F16: TTKV_MFMA_CASE(TTKV_F16, TTKV_F16); break;
    case TTKV_BF16 * 8 + TTKV_BF16: TTKV_MFMA_CASE(TTKV_BF16, TTKV_BF16); break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I8_SYM_G32: TTKV_MFMA_CASE(TTKV_I8_SYM_G32, TTKV_I8_SYM_G32); break;
    case TTKV_I4_ASYM_T128 * 8 + TTKV_I4_ASYM_G64:
      if constexpr (T128) TTKV_MFMA_CASE(TTKV_I4_ASYM_T128, TTKV_I4_ASYM_G64);
      break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I4_ASYM_G64:
      if constexpr (FOUR_BIT) TTKV_MFMA_CASE(TTKV_I8_SYM_G32, TTKV_I4_ASYM_G64);
      break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I4_ASYM_G64_T32:
      if constexpr (FOUR_BIT) TTKV_MFMA_CASE(TTKV_I8_SYM_G32, TTKV_I4_ASYM_G64_T32);
      break;
    case TTKV_I4_ASYM_G64 * 8 + TTKV_I4_ASYM_G64_T32:
      if constexpr (FOUR_BIT) TTKV_MFMA_CASE(TTKV_I4_ASYM_G64, TTKV_I4_ASYM_G64_T32);
      break;
    default:
      if constexpr (FOUR_BIT) TTKV_MFMA_CASE(TTKV_I4_ASYM_G64, TTKV_I4_ASYM_G64);
      break;
  }
#undef TTKV_MFMA_CASE
  __syncthreads();

  // ---- merge the four waves (each with its own running max) and write the item's partials
  for (int idx = threadIdx.x; idx < G * 128; idx += 256) {
    const int g = idx >> 7, dch = idx & 127;
    const float M = fmaxf(fmaxf(s_m[0][g], s_m[1][g]), fmaxf(s_m[2][g], s_m[3][g]));
    float o = 0.0f, ll = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = s_m[w][g] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(s_m[w][g] - M);
      o = fmaf(((const float *)(s_buf + w * kTileLds))[g * 128 + dch], wgt, o);
      ll = fmaf(s_l[w][g], wgt, ll);
    }
    const int64_t prow = ((int64_t)seq * a.Hq + hq0 + g) * a.part_stride + part;
    a.pacc[prow * 128 + dch] = o;
    if (dch == 0) {
      a.pm[prow] = M * kLn2;  // natural-log units outside the kernel
      a.pl[prow] = ll;
    }
  }
}

}  // namespace

// Do the kernel's cases take these formats?  From two query heads per KV head on (measured against the vector kernel's
// head pair at two heads: fp16 6.4 against 6.2 TB/s, int8 6.2 against 5.3, int4 5.2 against 4.5, K 8-bit / V 4-bit 6.0
// against 4.3, keys grouped over tokens 4.4 against 3.5).
bool attn_mfma_fits(int k_fmt, int v_fmt, int G) {
  if (G < 2) return false;
  if (v_fmt == TTKV_I4_ASYM_G64_T32) return k_fmt == TTKV_I8_SYM_G32 || k_fmt == TTKV_I4_ASYM_G64;
  if (k_fmt == TTKV_I4_ASYM_G64) return v_fmt == k_fmt;
  return true;
}

bool attn_mfma_four_bit(int k_fmt, int v_fmt) { return !is_fp(k_fmt) && !(k_fmt == TTKV_I8_SYM_G32 && v_fmt == k_fmt); }

namespace {
// Key formats that stay with the vector kernel's head pairs when keys grouped over tokens are in the same launch: the
// former score product had no case for them.  This one has, and the pairs are not the faster route any more (2 x 51K
// tokens, 8 heads per KV head 129 us against 41, 16 heads 134 against 29).
bool pairs_beside_t128(int k_fmt, int G) { return (k_fmt == TTKV_I8_SYM_G32 && G > 4) || (k_fmt == TTKV_I4_ASYM_G64 && G > 8); }

// What one launch needs: heads per block, 4-bit tiers, keys grouped over tokens.  ok: the kernel takes it.
struct MfmaShape {
  int heads;
  bool four_bit, t128, ok;
};
MfmaShape mfma_shape(const FusedArgs &a) {
  const int G = a.Hq / a.Hkv;
  MfmaShape m{std::min(16, G), false, false, true};
  bool pairs = false;
  for (int j = 0; j < a.n_entries; ++j) {
    const TierView &tv = a.tv[entry_tier(a.e[j])];
    m.ok &= attn_mfma_fits(tv.k_fmt, tv.v_fmt, G);
    m.four_bit |= attn_mfma_four_bit(tv.k_fmt, tv.v_fmt);
    m.t128 |= tv.k_fmt == TTKV_I4_ASYM_T128;
    pairs |= pairs_beside_t128(tv.k_fmt, G);
  }
  m.ok &= !(m.t128 && pairs);
  return m;
}
}  // namespace

bool attn_mfma_eligible(const FusedArgs &a) { return mfma_shape(a).ok; }

hipError_t launch_attn_mfma(const FusedArgs &a0, hipStream_t s) {
  const MfmaShape m = mfma_shape(a0);
  FusedArgs a = a0;
  a.mfma_heads = m.heads;
  const int G = a.Hq / a.Hkv;
  const uint32_t n_hb = (G + m.heads - 1) / m.heads;
  const dim3 grid(((uint32_t)a.n_items * a.Hkv + 7) / 8 * 8 * n_hb);
  if (m.t128) hipLaunchKernelGGL((attn_mfma_kernel<true, true>), grid, dim3(256), 0, s, a);
  else if (m.four_bit) hipLaunchKernelGGL((attn_mfma_kernel<true, false>), grid, dim3(256), 0, s, a);
  else hipLaunchKernelGGL((attn_mfma_kernel<false, false>), grid, dim3(256), 0, s, a);
  return hipGetLastError();
}

}  // namespace ttkv
