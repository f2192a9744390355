// Grouped-query variant of the split-K decode attention partials (Alg. 1: Attn on the
// fast tier, Decompress + Attn per slow-tier block): all query heads that share a KV
// head are served by ONE pass over that head's K/V bytes, with the two contractions on
// the matrix cores (v_mfma_f32_16x16x32 f16 / bf16 for q.k and p.v, v_mfma_f32_16x16x16 for
// the layout changes).  Same work items, same partials and same record layout as the vector
// kernel; only the lane mapping differs.
//
// One 16-token tile, lane = (c = lane % 16, kg = lane / 16); a K row reaches the product as 32 channels of token c per lane
// in four 32-deep steps.
//
// Quantized tiers (process_quant): heads are the rows and tokens the columns of the score product,
//       S[head][token] = sum_d Q[head][d] K[token][d],
//   with the heads of up to four tiles in the 16 rows (QuantShape), so that the softmax has 4 scores per lane and chain at any
//   number of heads, all of one token, whose scales and zero points are the lane's own.  The lane's channels are 8 bytes of
//   each 32-byte stretch of the row, so a step (or two, int4) stays inside one channel group and every group has a product
//   chain of its own.  Codes enter as fp16 subnormals: no splice constant, no offset (int8: 128).
//   Values: gfx950's transposing LDS reads (ds_read_b64_tr_b4 / _b8) hand lane (c, kg) the codes of ONE channel of eight
//   tokens of a 32-token pair of tiles -- with the masks applied the A operand of
//       O[channel][group, head] += sum_token V^T[channel][token] * P[token][group, head],
//   and the token's scale rides on the other operand, P = p_t s_{t,g}, whose (channel group, head) pairs fill the product's
//   16 columns; it goes through LDS (stored per token, read transposed per head: ds_read_b64_tr_b16) as an fp16 number and
//   its remainder, 22 bits.  The weights p carry a power of two that keeps both in fp16's range whatever the size of the
//   values (wexp below).  The codes' centre (128; 8) leaves with a product of the same weights with a constant, the int4
//   zero points and the centre come back as sum_t p_t (z_{t,g} + 8 s_{t,g}) in fp32.  Values stored channel-major per 32
//   tokens (TTKV_I4_ASYM_G64_T32) are those operand words as they lie.
//
// fp16 / bf16 tiers and keys grouped over tokens (process_rows): tokens are the rows, heads the columns of S; lane (c, kg)
//   holds head c of tokens 4 kg .. 4 kg + 3 and the softmax is per column.  V rows like K's (int4 ones dequantized in packed
//   fp16); a product with the identity matrix brings the tile from [token][channel] to [channel][token]: the fp32 result
//   (exact) has lane (c, kg) holding channel-row c for tokens 4 kg .. 4 kg + 3, the A layout.  Two 16-token tiles feed
//   one 32-deep product.  The zero points and scales ride along as a 4-channel V.  P meets an fp16 / bf16 V with 22 bits, as an
//   fp16 number and its remainder, eight products per 32 tokens that cost no time beside the memory's (steps of fp16 alone,
//   1 x 30K to 64 x 2K tokens, within 1 % either way); error against 64 bits, 2 x 8192 tokens: fp16 9.0e-5 -> 5e-7, bf16 9.1e-5
//   -> 5e-7, 64 sequences of 1003 fp16 + up to 3072 int8 tokens 4.3e-5 -> 6e-6.
//   Keys grouped over 128 tokens per channel have no channel groups; the token group's scales fold into the q operand,
//   carried as fp16 rounded product + exact remainder (two products per step), rebuilt for every 64 tokens in flight.
//
// Bound: the memory system; vector instructions where they are too many.  Quantized loop, 32 / 8 heads, vector
// instructions per 64 tokens of int4 (32 of int8): 624 -> 280 (337 -> 160) against the form with heads as columns of both
// products, one rounding of p s and splice constants; one step, us, before -> now: 128K tokens of three formats 42.9 -> 39.2,
// 16 ragged sequences of K int4 / V4c 187 -> 177, block-sparse recall 125 -> 115; 64 / 4 heads, K int8 / V int4, 84.8 -> 81.7
// (77 with everything but copies and LDS reads taken out).  Error against 64 bits (2-norm, keys with outlier channels,
// 4K to 64K tokens): int8 0.9e-4 -> 1.4e-5 to 4.3e-5, int4 1e-4 -> 1e-5 to 2e-5, int4 with scores eight times as large 8e-5 ->
// 1.9e-5.  One power of two serves a wave's weights: channels whose values are 2^-14 of other channels' keep this error, at
// 2^-18 it is 1e-4 and at 2^-20 5e-4 (one rounding: 1e-4).  More heads per KV head than 16 are cut into blocks of 16, one
// workgroup and one pass over the bytes per block.
#include "ttkv_attn_dev.h"

#include <algorithm>
#include <type_traits>

namespace ttkv {

namespace {

using namespace dev;

typedef _Float16 h4 __attribute__((ext_vector_type(4)));
typedef short s4 __attribute__((ext_vector_type(4)));
typedef float f4 __attribute__((ext_vector_type(4)));
typedef float f4_any __attribute__((ext_vector_type(4), aligned(4)));

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
// of the lane's slice (j = 4 s + i in unpack order for fp16 / bf16) is therefore row channel:
template <int F>
__device__ __forceinline__ constexpr int slice_channel(int kg, int j) {
  if (is_i4<F>()) return 32 * kg + j;     // one piece of 32 channels
  return 32 * (j / 8) + 8 * kg + j % 8;   // four pieces of 8
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

// ---- tiles of quantized rows prefetched through LDS
// The rows of a batch of tiles are copied global -> LDS asynchronously (no registers in between), the K half and
// the V half separately, while the batch before is being computed; the copy instructions read whole rows (whole
// 128-byte lines, so they carry the streaming hint), and the lanes then read their pieces from LDS in the operand
// layout.  Inside LDS row r keeps its pieces in the order p ^ swz(r), which spreads the 16 rows that the
// lanes of one piece read at a time over the banks; the copy realises the order by choosing which piece each lane fetches.
// Per wave: a batch's K rows, V rows and four planes of meta words (K words 0 and 1 of the batch's tokens, V words 0 and
// 1), then the weights.  At the end the wave's result takes the first 8 KiB, its sums the meta planes behind them.  (Two
// batches in flight gained nothing: 86 against 87 us for 8 x 64K tokens of K int8 / V int4.)
constexpr int kTileRowsLds = 8 * 1024, kMetaLds = 4 * 256, kBatchLds = kTileRowsLds + kMetaLds, kWeightsLds = 2 * 2048;
constexpr int kTileLds = kBatchLds + kWeightsLds;
// Behind the four waves' places, int8 keys: the rows' offsets per channel group, [group][kg].  All waves of a workgroup have
// the same queries and store the same numbers.  (A copy per wave would make three workgroups 1280 bytes larger than a CU's
// LDS: it is given out in units of 1280 bytes, and 54272 become 55040.  With two resident, 16 sequences of 2664 fp16 + 8704
// int8 tokens, 32 / 8 heads, take 85.4 us instead of 79.)
constexpr int kOffLds = 256;
constexpr int lds_given(int bytes) { return (bytes + 1279) / 1280 * 1280; }
constexpr int kSumsLds = kTileRowsLds + 512;   // 16 references, 16 sums of weights
typedef const __attribute__((address_space(1))) void *gas_ptr;
typedef __attribute__((address_space(3))) void *las_ptr;
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4_any __attribute__((ext_vector_type(4), aligned(2)));
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
// The same with off[g], the four rows' offsets of group g, from o.
__device__ __forceinline__ void lds_keys_i8(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, uint32_t o, u32x2 *w, f4 *off) {
  asm volatile("ds_read_b64 %0, %12\n\tds_read_b64 %1, %13\n\tds_read_b64 %2, %14\n\tds_read_b64 %3, %15\n\t"
               "ds_read_b64 %4, %12 offset:2048\n\tds_read_b64 %5, %13 offset:2048\n\t"
               "ds_read_b64 %6, %14 offset:2048\n\tds_read_b64 %7, %15 offset:2048\n\t"
               "ds_read_b128 %8, %16\n\tds_read_b128 %9, %16 offset:64\n\tds_read_b128 %10, %16 offset:128\n\t"
               "ds_read_b128 %11, %16 offset:192\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7]),
                 "=&v"(off[0]), "=&v"(off[1]), "=&v"(off[2]), "=&v"(off[3])
               : "v"(a0), "v"(a1), "v"(a2), "v"(a3), "v"(o) : "memory");
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
// the largest value of the lane's row of 16
__device__ __forceinline__ float row_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));
  return fmaxf(v, dpp<0x140>(v));
}
__device__ __forceinline__ float pow2(int e) { return __uint_as_float((uint32_t)(127 + e) << 23); }   // |e| < 127
// fp16 halves of a meta word
__device__ __forceinline__ float half0(uint32_t w) { return (float)as_h2(w).x; }
__device__ __forceinline__ float half1(uint32_t w) { return (float)as_h2(w).y; }

// Head section and row inside it of the item's token i, of a run or of the blocks that `sel` names.  The block table
// does not change during the launch and the index is wave-uniform: it is read through the constant address space (a
// scalar load); so are the selected ids, written by the launch before this one.
struct Place {
  int block, row;   // ring block (selected: index into the ids), row inside it
};
typedef const __attribute__((address_space(4))) int32_t *const_i32;
__device__ __forceinline__ Place place_of(const TierView &tv, const RunView &en, int i) {
  int tok = en.first_tok + i;
  const int ring_tokens = tv.ring_blocks * tv.bt;
  if (tok >= ring_tokens) tok -= ring_tokens;
  const int rb = div_bt(tok, tv.bt, tv.bt_magic);
  return Place{rb, tok - rb * tv.bt};
}
__device__ __forceinline__ const uint8_t *head_at(const TierView &tv, const RunView &en, const int32_t *sel, int seq, int hkv, int block) {
  int rb = block;
  if (sel) rb = ring_of_id(((const_i32)(uintptr_t)sel)[rb], en, tv);
  const int64_t rec = tv.table ? (int64_t)((const_i32)(uintptr_t)tv.table)[(int64_t)seq * tv.ring_blocks + rb]
                               : (int64_t)en.rec_base + rb;
  return tv.base + rec * tv.rec_bytes + (int64_t)hkv * tv.head_bytes;
}

// fp16 / bf16 tiers, and keys grouped over tokens: any number of query heads up to 16 (the columns of both products).
template <int KF, int VF>
__device__ __forceinline__ void process_rows(const FusedArgs &a, const TierView &tv, const RunView &en, const int32_t *sel,
                                             int chunk_tokens, int chunk, int seq, int hq0, int Gr, int hkv, char *wbuf) {
  // wbuf: the wave's LDS, a batch of tiles in flight, at the end its result
  // sel: null, or the block ids behind a run made of selected blocks (ring block of token i: sel[i / bt])
  // hq0, Gr: first query head and number of heads of this workgroup's block of heads (all heads of the KV head,
  // or a block of up to 16 of them)
  using FK = Fmt<KF>;
  using FV = Fmt<VF>;
  constexpr int NLK = FK::ROWB / 64, NLV = FV::ROWB / 64;   // 16-byte loads per lane per 16-token tile
  constexpr int NT = NLK == 4 ? 2 : 4 / NLK;   // tiles in flight per wave (int4 on register loads: 4; with 2 that kernel is 10 % slower)
  constexpr int TT = 16 * NT;
  constexpr bool VQ = n_groups<VF>() > 1;
  constexpr bool KT = KF == TTKV_I4_ASYM_T128;   // keys grouped over 128 tokens per channel: the scales fold into q
  constexpr bool KBF = KF == TTKV_BF16, VBF = VF == TTKV_BF16;
  // Weights with their remainders; not beside grouped keys, whose values are rounded as they are dequantized: nothing would be
  // gained (1.9e-4 either way), and that loop is bound by its instructions (3-4 % slower).
  constexpr bool REST = !VQ;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kg = lane >> 4;
  const int c0 = chunk * chunk_tokens;
  const int c1 = min(en.len, c0 + chunk_tokens);
  const float cs = a.scale * kLog2e;       // scores are kept in the log2 domain

  const bool col_on = n < Gr;   // column = query head

  // ---- q operand: 16 packed registers (step s: 4 s .. 4 s + 3)
  uint32_t qB[16];
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
#pragma unroll
    for (int r = 0; r < 16; ++r) {
      uint32_t w = qw[r];
      if constexpr (is_i4<KF>()) {
        const int dd = r / 4, e = r % 4;
        w = __builtin_amdgcn_perm(qw[4 * dd + 2 + e / 2], qw[4 * dd + e / 2], (e & 1) ? 0x07060302u : 0x05040100u);
      }
      qB[r] = col_on ? w : 0u;
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
  // minus (splice offset + centre) as packed fp16 pairs: -(1024 + 8), -(64 + 8)
  uint32_t no_a = 0xE408E408u, no_b = 0xD480D480u;
  asm volatile("" : "+s"(no_a), "+s"(no_b));

  const f4 zero4 = f4{0.0f, 0.0f, 0.0f, 0.0f};
  f4 acc[8], accz = zero4;
#pragma unroll
  for (int s = 0; s < 8; ++s) acc[s] = zero4;
  float m = -INFINITY, l = 0.0f, mcs = INFINITY;   // a token's weight: exp2(score cs + mcs)
  // The weights carry 2^14: rounded to fp16 they keep their 11 bits down to 2^-28 of the largest one instead of 2^-14 (fp16's
  // subnormals), so that the error does not grow with the tokens of an item, among which the largest weight is found.  As for
  // the quantized tiers a reference beyond 4 million carries none, and f - mcs, the reference of the result, is exact.
  float f = 0.0f;
  Splice sp;
  sp.init();

  struct TileRegs {
    uint4 kw[NT][NLK], vw[NT][NLV];
    uint2 vmeta[NT];
    uint4 gm[KT ? 8 : 1];   // KT: {scale, zero} of the lane's 32 channels for the token group of these tiles
  };
  const uint32_t kdoff = n * FK::ROWB + kg * 16, vdoff = n * FV::ROWB + kg * 16;

  // Plain loads here, not the non-temporal ones of the vector kernel: the load instructions of a tile share
  // cache lines (each reads 64 of a line's 128 bytes), and lines fetched with the streaming hint do not
  // survive until the next instruction.
  auto locate = [&](int i, int &row0) -> const uint8_t * {
    const Place p = place_of(tv, en, i);
    row0 = p.row;
    return head_at(tv, en, sel, seq, hkv, p.block);
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
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      uint32_t kr[16];
#pragma unroll
      for (int x = 0; x < NLK; ++x) unpack16<KF>(t.kw[tt][x], kr + x * (16 / NLK), sp);
      f4 sv = KT ? f4{-off_t, -off_t, -off_t, -off_t} : zero4;
#pragma unroll
      for (int s = 0; s < 4; ++s) {
        if constexpr (KT) {
          sv = mma32<false>(kr + 4 * s, qh + 4 * s, sv);
          sv = mma32<false>(kr + 4 * s, ql + 4 * s, sv);
        } else {
          sv = mma32<KBF>(kr + 4 * s, qB + 4 * s, sv);
        }
      }
      f4 sc;
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float x = sv[i];
        if (!FULL && tt * 16 + 4 * kg + i >= nv) x = -INFINITY;
        sc[i] = x;
        mt = fmaxf(mt, x);
      }
      S[tt] = sc;
    }

    // ---- online softmax (base 2) per column; m is kept in raw score units, the scale enters the exponent
    mt = fmaxf(mt, __shfl_xor(mt, 16));
    mt = fmaxf(mt, __shfl_xor(mt, 32));
    if (__any(mt > m)) {
#pragma clang fp contract(off)
      const float mn = fmaxf(m, mt), r = mn * cs, was = f;
      if constexpr (REST) f = fabsf(r) < 4194304.0f ? 14.0f : 0.0f;
      mcs = f - r;
      const float alpha = __builtin_amdgcn_exp2f(REST ? (m - mn) * cs + (f - was) : (m - mn) * cs);
      l *= alpha;
      accz *= alpha;
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[s] *= alpha;
      m = mn;
    }

    // ---- weighted V, two 16-token tiles per 32-deep product
    before_v();
#pragma unroll
    for (int tp = 0; tp < NT; tp += 2) {
      uint32_t pB[4], pR[4];   // softmax weights of the pair, rounded to fp16, and their remainders: the B operands
      uint32_t vr[2][16];
#pragma unroll
      for (int u = 0; u < 2; ++u) {
        const int tt = tp + u;
        float p[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) p[i] = __builtin_amdgcn_exp2f(fmaf(S[tt][i], cs, mcs));
        if constexpr (REST) l += (p[0] + p[1]) + (p[2] + p[3]);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
          const uint32_t w = pk(p[2 * i], p[2 * i + 1]);
          pB[2 * u + i] = w;
          if constexpr (REST) pR[2 * u + i] = pk(p[2 * i] - half0(w), p[2 * i + 1] - half1(w));
          else l = __builtin_amdgcn_fdot2(as_h2(w), h2{(_Float16)1.0f, (_Float16)1.0f}, l, false);   // the sum of the rounded weights
        }

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
        if constexpr (REST) acc[s] = mma32<false>(A, pR, acc[s]);
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
  if constexpr (PF2) {
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
  float z = 0.0f;   // zero-point sum of the channels' group
  if constexpr (KT)   // sum_t p_t * (zero + 8 * scale)
    z = (kg >> 1) ? fmaf(8.0f, accz[2], accz[3]) : fmaf(8.0f, accz[0], accz[1]);
  float (*w_acc)[128] = (float (*)[128])wbuf;   // [head][channel]; the wave's last batch has been consumed
  if (n < Gr) {
    const float unscale = !REST || f == 0.0f ? 1.0f : 0x1p-14f;
#pragma unroll
    for (int s = 0; s < 8; ++s)
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        w_acc[n][slice_channel<VF>(kg, chan<VF>(s, i))] = (acc[s][i] + z) * unscale;
      }
    if (kg == 0) {
      ((float *)(wbuf + kSumsLds))[n] = f - mcs;
      ((float *)(wbuf + kSumsLds))[16 + n] = l * unscale;
    }
  }
}

// ---------------------------------------------------------------- quantized tiers
// How the heads of a workgroup and the tiles of a batch share the rows of a score product (heads are its rows, tokens
// its columns).  HS: 4, 8 or 16 places for heads (the smallest that holds the block's heads); the 16 rows then take the
// heads of 16 / HS tiles at once, each tile's product with the queries in its own rows and zeros in the others.  So the
// softmax works on 4 tokens x heads per lane whatever HS is (with the heads as columns, 12 of 16 lanes had nothing to
// do at four heads per KV head), every lane has one token of a chain, and that token's scales are the lane's own.
template <int KF, int VF, int HS>
struct QuantShape {
  static constexpr int NT = KF == TTKV_I8_SYM_G32 ? 2 : 4, TT = 16 * NT;   // tiles, tokens of a batch
  static constexpr int TPC = NT < 16 / HS ? NT : 16 / HS, NC = NT / TPC;   // tiles per score chain, chains
  static constexpr int KPT = 4 / TPC, NE = HS / KPT;   // lanes' kg per tile; rows used of a lane's four
  // row 4 kg + i, i < NE: tile kg / KPT of the chain, head (kg % KPT) NE + i
  static constexpr int NGK = n_groups<KF>(), NGV = n_groups<VF>();
  static constexpr bool K4 = KF == TTKV_I4_ASYM_G64, V4 = VF != TTKV_I8_SYM_G32, VT = VF == TTKV_I4_ASYM_G64_T32;
  // The weights' way to the value product, whose columns are (channel group, head) pairs, 16 per operand set:
  static constexpr int GR = HS * NGV > 32 ? 2 : NGV, NR = NGV / GR;   // channel groups that pass LDS at a time
  static constexpr int RB = GR * HS * 2;                             // bytes per token there
  static constexpr bool BY_PAIR = TT * RB > 2048;                    // only a pair of tiles at a time
  static constexpr int NB = GR * HS > 16 ? GR * HS / 16 : 1, GPS = GR / NB, SETS = NB * NR;   // operand sets; groups in each
  // A tile's weights in LDS: slots of 16 tokens x U bytes, one per kg of the tile (and half of the groups, where a lane has
  // 32 bytes of a token); the tokens of slot q lie at (token U) ^ 64 q, so that the four slots a transposing read touches
  // at a time, and the 16 tokens a store does, fall into different banks (rows of a token's 64 bytes before: four-way
  // conflicts, 128 cycles per batch of 32 tokens and 16 heads).
  static constexpr int U = GR * NE * 2 >= 16 ? 16 : 8;
  static constexpr bool HALVES = GR * NE * 2 == 32;
  static __device__ __forceinline__ uint32_t place(int slot, int token) { return slot * 16 * U + ((token * U) ^ (U == 16 ? slot * 64 : 0)); }
  static_assert(NE == 4 || (NE == 2 && HS == 4), "rows per lane");
  static_assert((BY_PAIR ? 32 : TT) * RB <= 2048, "the weights' place in LDS");
  // column n of operand set b
  static __device__ __forceinline__ int head_of(int n) {
    return NE == 4 ? 4 * ((n >> 2) % KPT) + (n & 3) : 2 * ((n >> 2) & 1) + (n & 1);
  }
  static __device__ __forceinline__ int group_of(int n) {   // within the set
    return NE == 4 ? ((n >> 2) / KPT) % GPS : (2 * (n >> 3) + ((n >> 1) & 1)) % GPS;
  }
  static __device__ __forceinline__ bool spare(int n) { return n >= GPS * HS; }   // a column that repeats another one
};

// The weights of four rows of 16 halves for lane c = one of 16: column c of them (transposing reads); from a0, their
// remainders 2 KiB further: w[2 i] and w[2 i + 1] for O_i.
template <int O0, int O1>
__device__ __forceinline__ void lds_weights(uint32_t a0, u32x2 *w) {
  asm volatile("ds_read_b64_tr_b16 %0, %4 offset:%5\n\tds_read_b64_tr_b16 %1, %4 offset:%7\n\t"
               "ds_read_b64_tr_b16 %2, %4 offset:%6\n\tds_read_b64_tr_b16 %3, %4 offset:%8\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
               : "v"(a0), "n"(O0), "n"(O1), "n"(O0 + 2048), "n"(O1 + 2048) : "memory");
}
template <int O0, int O1, int O2, int O3>   // the last two from a1
__device__ __forceinline__ void lds_weights(uint32_t a0, uint32_t a1, u32x2 *w) {
  asm volatile("ds_read_b64_tr_b16 %0, %8 offset:%10\n\tds_read_b64_tr_b16 %1, %8 offset:%14\n\t"
               "ds_read_b64_tr_b16 %2, %8 offset:%11\n\tds_read_b64_tr_b16 %3, %8 offset:%15\n\t"
               "ds_read_b64_tr_b16 %4, %9 offset:%12\n\tds_read_b64_tr_b16 %5, %9 offset:%16\n\t"
               "ds_read_b64_tr_b16 %6, %9 offset:%13\n\tds_read_b64_tr_b16 %7, %9 offset:%17\n\ts_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
               : "v"(a0), "v"(a1), "n"(O0), "n"(O1), "n"(O2), "n"(O3), "n"(O0 + 2048), "n"(O1 + 2048), "n"(O2 + 2048),
                 "n"(O3 + 2048) : "memory");
}
// 32 channels of a query, 8 from each address
__device__ __forceinline__ void lds_query(uint32_t a0, uint32_t a1, uint32_t a2, uint32_t a3, u32x4 *w) {
  asm volatile("ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
               "s_waitcnt lgkmcnt(0)"
               : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]) : "v"(a0), "v"(a1), "v"(a2), "v"(a3) : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_put(uint32_t a0, u32x4 w) {
  asm volatile("ds_write_b128 %0, %1 offset:%2" ::"v"(a0), "v"(w), "n"(OFF) : "memory");
}
template <int OFF>
__device__ __forceinline__ void lds_put(uint32_t a0, u32x2 w) {
  asm volatile("ds_write_b64 %0, %1 offset:%2" ::"v"(a0), "v"(w), "n"(OFF) : "memory");
}
// The four meta words of the lane's token of NC chains: w[2 j] = the keys', w[2 j + 1] = the values'; chains STEP bytes
// apart, the second word of a pair one plane (256 bytes) further, the values' two planes.
template <int NC, int STEP>
__device__ __forceinline__ void lds_meta(uint32_t a0, u32x2 *w) {
  if constexpr (NC == 1) {
    asm volatile("ds_read2_b32 %0, %2 offset1:64\n\tds_read2_b32 %1, %2 offset0:128 offset1:192\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]) : "v"(a0) : "memory");
  } else if constexpr (NC == 2) {
    asm volatile("ds_read2_b32 %0, %4 offset1:64\n\tds_read2_b32 %1, %4 offset0:128 offset1:192\n\t"
                 "ds_read2_b32 %2, %4 offset0:%5 offset1:%6\n\tds_read2_b32 %3, %4 offset0:%7 offset1:%8\n\ts_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3])
                 : "v"(a0), "n"(STEP / 4), "n"(STEP / 4 + 64), "n"(STEP / 4 + 128), "n"(STEP / 4 + 192) : "memory");
  } else {
    static_assert(STEP == 64, "the offsets below");
    asm volatile("ds_read2_b32 %0, %8 offset1:64\n\tds_read2_b32 %1, %8 offset0:128 offset1:192\n\t"
                 "ds_read2_b32 %2, %8 offset0:16 offset1:80\n\tds_read2_b32 %3, %8 offset0:144 offset1:208\n\t"
                 "ds_read2_b32 %4, %8 offset0:32 offset1:96\n\tds_read2_b32 %5, %8 offset0:160 offset1:224\n\t"
                 "ds_read2_b32 %6, %8 offset0:48 offset1:112\n\tds_read2_b32 %7, %8 offset0:176 offset1:240\n\t"
                 "s_waitcnt lgkmcnt(0)"
                 : "=&v"(w[0]), "=&v"(w[1]), "=&v"(w[2]), "=&v"(w[3]), "=&v"(w[4]), "=&v"(w[5]), "=&v"(w[6]), "=&v"(w[7])
                 : "v"(a0) : "memory");
  }
}
// Codes as fp16 bit patterns, i.e. as subnormal numbers: the matrix cores take them as they are, there is no offset to
// remove and no rounding.  The products are aligned by the operands' exponents before they are added, so a code in the
// lowest bits loses what its leading zeros take: in the sums over thousands of values that showed (2e-4 of the result at
// 64K tokens, biased), so int4 values sit four bits up: (n0, n4) (n1, n5) (n2, n6) (n3, n7) as 16 code x 2^-24.  Keys,
// summed over 64 channels, save two operations: registers 0 and 2 hold code x 2^-24, and the factor 16 sits on the queries
// (a score's error stays below 2e-6 of its terms).  Where 16 q would leave fp16's range they are taken like values, by a loop
// of its own: no factor on the queries then, whose smaller heads would lose bits by one below 1.  Four int8 codes:
// (code + 128) x 2^-24.
constexpr uint32_t kCodeMask = 0x000F000Fu, kCodeFlip = 0x80808080u;
struct CodeMasks {
  uint32_t lo, hi, flip;   // in registers: a literal would be fetched with every instruction
  __device__ __forceinline__ CodeMasks() : lo(kCodeMask), hi(kCodeMask << 4), flip(kCodeFlip) { asm volatile("" : "+s"(lo), "+s"(hi), "+s"(flip)); }
};
__device__ __forceinline__ void key_codes4(uint32_t x, uint32_t *r, const CodeMasks &k) {
  const uint32_t y = x >> 8;
  r[0] = x & k.lo;
  r[1] = x & k.hi;
  r[2] = y & k.lo;
  r[3] = y & k.hi;
}
__device__ __forceinline__ void value_codes4(uint32_t x, uint32_t *r, const CodeMasks &k) {
  r[0] = (x << 4) & k.hi;
  r[1] = x & k.hi;
  r[2] = (x >> 4) & k.hi;
  r[3] = (x >> 8) & k.hi;
}
// both halves of a register times f
__device__ __forceinline__ uint32_t pk_scale(uint32_t w, _Float16 f) { return __builtin_bit_cast(uint32_t, as_h2(w) * h2{f, f}); }
__device__ __forceinline__ void codes8(uint32_t w, uint32_t *r, const CodeMasks &k) {
  const uint32_t x = w ^ k.flip;
  r[0] = __builtin_amdgcn_perm(0u, x, 0x0c010c00u);
  r[1] = __builtin_amdgcn_perm(0u, x, 0x0c030c02u);
}
// The same value, as if formed here: what is derived from it is not kept in registers through the loop.
__device__ __forceinline__ uint32_t fresh(uint32_t v) {
  asm volatile("" : "+v"(v));
  return v;
}

template <int KF, int VF, int HS, bool OFF_LDS>
__device__ __forceinline__ void process_quant(const FusedArgs &a, const TierView &tv, const RunView &en, const int32_t *sel,
                                              int chunk_tokens, int chunk, int n_items, int seq, int hq0, int Gr, int hkv, char *wbuf) {
  // sel, hq0, Gr, wbuf: as process_rows.  n_items: 0, the item is chunk_tokens tokens in a row; else the run's items take
  // turns at its batches, so that at any time they read one stretch of memory (8 x 64K tokens of K int8 / V int4, 64 / 4 heads,
  // 84.2 -> 83.0 us, block-sparse recall 119.5 -> 117.6; in turn over caches of 2.3 GB together, so that each is read cold, 85.5 ->
  // 83.5 and 121.0 -> 118.9; 128K tokens, ragged and short sequences within 0.5 us either way, cold or not).
  using FK = Fmt<KF>;
  using FV = Fmt<VF>;
  using Q = QuantShape<KF, VF, HS>;
  constexpr int NT = Q::NT, TT = Q::TT, TPC = Q::TPC, NC = Q::NC, KPT = Q::KPT, NE = Q::NE, NGK = Q::NGK, NGV = Q::NGV;
  constexpr bool K4 = Q::K4, V4 = Q::V4, VT = Q::VT;
  constexpr int PK = FK::ROWB / 16, PV = FV::ROWB / 16;                   // 16-byte pieces per row
  constexpr int NDK = TT * FK::ROWB / 1024, NDV = TT * FV::ROWB / 1024;   // copy instructions of 1 KiB per half
  constexpr int N_K = NDK + 4, N_V = NDV;                                 // with the four meta planes
  static_assert(NDK == 4 && (NDV == 4 || NDV == 2), "the batch the LDS readers cover");
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int n = lane & 15, kg = lane >> 4;
  const int step_tokens = 4 * TT * max(n_items, 1);
  const int c0 = n_items ? chunk * 4 * TT : chunk * chunk_tokens;
  const int c1 = n_items ? en.len : min(en.len, c0 + chunk_tokens);

  // ---- where a batch lies, and its copies into the wave's LDS: K rows at 0, V rows at 4 KiB (row r at r ROWB, its
  // piece p at 16 (p ^ swz(r))), then the four meta planes, then the weights.
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
  const uint8_t *nx_head = nullptr;     // batch whose K half was issued last
  int nx_row0 = 0, nx_nv = 0;
  // The wave's batches lie step_tokens apart: block and row move on by additions, and the next batch's record is looked up
  // before it is asked for.
  const int first = c0 + wave * TT;
  const int step_blocks = div_bt(step_tokens, tv.bt, tv.bt_magic), step_rows = step_tokens - step_blocks * tv.bt;
  Place at = place_of(tv, en, min(first, en.len - 1));
  const uint8_t *at_head = head_at(tv, en, sel, seq, hkv, at.block);
  auto advance = [&](int i0) {   // to the batch after i0, if there is one
    if (i0 + step_tokens >= c1) return;
    at.row += step_rows;
    at.block += step_blocks;
    if (at.row >= tv.bt) {
      at.row -= tv.bt;
      ++at.block;
    }
    if (!sel && at.block >= tv.ring_blocks) at.block -= tv.ring_blocks;
    at_head = head_at(tv, en, sel, seq, hkv, at.block);
  };
  auto issue_k = [&](int i0) {
    nx_head = at_head;
    nx_row0 = at.row;
    nx_nv = min(TT, c1 - i0);
    const uint8_t *kb = nx_head + nx_row0 * FK::ROWB, *kmb = nx_head + tv.k_meta_off + nx_row0 * 8;
    if (nx_nv == TT) {
      dma16<0>(kb + dko[0], wbuf); dma16<1024>(kb + dko[1], wbuf);
      dma16<2048>(kb + dko[0], wbuf); dma16<3072>(kb + dko[1], wbuf);
    } else {
      const int ln = (int)fresh(lane);
#pragma unroll
      for (int j = 0; j < NDK; ++j) {
        const int r = j * (64 / PK) + ln / PK;   // LDS row; rows past the end repeat the last live row
        dma16(kb + min(r, nx_nv - 1) * FK::ROWB + ((ln % PK) ^ swz(PK, r)) * 16, wbuf + j * 1024);
      }
    }
    const uint32_t mo = min(lane, nx_nv - 1) * 8;   // one lane per token (TT = 32: the upper lanes repeat the last row)
    dma4(kmb + mo, wbuf + kTileRowsLds);
    dma4(kmb + mo + 4, wbuf + kTileRowsLds + 256);
    const uint8_t *vmb = nx_head + tv.v_meta_off + nx_row0 * 8;   // the values' too: their scales are looked at with the scores
    dma4(vmb + mo, wbuf + kTileRowsLds + 512);
    dma4(vmb + mo + 4, wbuf + kTileRowsLds + 768);
  };
  auto issue_v = [&](int i0) {   // of the batch at i0, whose K half was issued last
    const uint8_t *vb = nx_head + tv.v_off + nx_row0 * FV::ROWB;
    if constexpr (VT) {   // whole 2 KiB groups (lengths are multiples of 32), copied as they lie
      dma16<0>(vb + lane * 16, wbuf + 4096); dma16<1024>(vb + lane * 16, wbuf + 4096);
      if constexpr (NT == 4) {   // the second group: inside the record even when the run ends before it (its weights are 0)
        dma16<2048>(vb + lane * 16, wbuf + 4096); dma16<3072>(vb + lane * 16, wbuf + 4096);
      }
    } else if (nx_nv == TT) {
      dma16<0>(vb + dvo, wbuf + 4096); dma16<1024>(vb + (dvo ^ vx(1)), wbuf + 4096);
      if constexpr (NDV == 4) {
        dma16<2048>(vb + (dvo ^ vx(2)), wbuf + 4096); dma16<3072>(vb + (dvo ^ vx(3)), wbuf + 4096);
      }
    } else {
      const int ln = (int)fresh(lane);
#pragma unroll
      for (int j = 0; j < NDV; ++j) {
        const int r = j * (64 / PV) + ln / PV;
        dma16(vb + min(r, nx_nv - 1) * FV::ROWB + ((ln % PV) ^ swzv(PV, r)) * 16, wbuf + 4096 + j * 1024);
      }
    }
    advance(i0);
  };
  // Rows in pinned host memory: the whole batch through registers into the same places (over PCIe the asynchronous
  // copies were 3-4 % slower, and the streaming hint has nothing to gain there).  Lane (n, kg) moves piece kg (+ 4) of
  // row n of every tile, one lane per token its meta words.
  constexpr int NLK = FK::ROWB / 64, NLV = FV::ROWB / 64;   // 16-byte loads per lane per 16-token tile
  auto bring_host = [&](int i0) {
    const int lane = (int)fresh(threadIdx.x & 63), n = lane & 15, kg = lane >> 4;
    const uint8_t *const head = at_head;
    const int nv = min(TT, c1 - i0), row0 = at.row;
    advance(i0);
    const uint8_t *kb = head + row0 * FK::ROWB, *vb = head + tv.v_off + row0 * FV::ROWB;
    u32x4 kw[NT][NLK], vw[NT][NLV];
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
      const uint32_t row = min(tt * 16 + n, nv - 1);   // rows past the end repeat the last live row
#pragma unroll
      for (int x = 0; x < NLK; ++x) kw[tt][x] = *(const u32x4 *)(kb + row * FK::ROWB + kg * 16 + 64 * x);
      if constexpr (VT) {
        // piece hh = tt % 2 of the 32-token group tt / 2 (a group past the end repeats the last live one)
        vw[tt][0] = *(const u32x4 *)(vb + min(tt / 2, (nv - 1) / 32) * 2048 + (tt & 1) * 1024 + lane * 16);
      } else {
#pragma unroll
        for (int x = 0; x < NLV; ++x) vw[tt][x] = *(const u32x4 *)(vb + row * FV::ROWB + kg * 16 + 64 * x);
      }
    }
    const uint32_t mo = (row0 + min(lane, nv - 1)) * 8;
    const uint2 km = *(const uint2 *)(head + tv.k_meta_off + mo), vm = *(const uint2 *)(head + tv.v_meta_off + mo);
#pragma unroll
    for (int tt = 0; tt < NT; ++tt) {
#pragma unroll
      for (int x = 0; x < NLK; ++x)
        *(u32x4 *)(wbuf + (tt * 16 + n) * FK::ROWB + (((kg + 4 * x) ^ swz(PK, n)) * 16)) = kw[tt][x];
      if constexpr (VT) {
        *(u32x4 *)(wbuf + 4096 + tt * 1024 + lane * 16) = vw[tt][0];
      } else {
#pragma unroll
        for (int x = 0; x < NLV; ++x)
          *(u32x4 *)(wbuf + 4096 + (tt * 16 + n) * FV::ROWB + (((kg + 4 * x) ^ swzv(PV, tt * 16 + n)) * 16)) = vw[tt][x];
      }
    }
    uint32_t *m = (uint32_t *)(wbuf + kTileRowsLds) + lane;
    m[0] = km.x;
    m[64] = km.y;
    m[128] = vm.x;
    m[192] = vm.y;
  };

  if (first >= c1) {   // no batch for this wave (wave-uniform): an empty part
    if (lane < 16) {
      ((float *)(wbuf + kSumsLds))[lane] = -INFINITY;
      ((float *)(wbuf + kSumsLds))[16 + lane] = 0.0f;
    }
    for (int idx = lane; idx < Gr * 32; idx += 64) ((float4 *)wbuf)[idx] = float4{0.0f, 0.0f, 0.0f, 0.0f};
    return;
  }

  // ---- the queries.  Their rows come through LDS like everything else, in front of the first batch, so that a count of
  // the copies behind them says when they have landed: they are prepared while the batch is on its way (loads into
  // registers are waited for with everything in flight wherever paths with other counts meet; so 3.1 us passed from the
  // look-up of the item to its first keys).  Up to 8 heads wait in the weights' place, 16 in that of the values, which are
  // then copied after them.
  constexpr bool Q_IN_V = HS == 16;
  char *const q_lds = wbuf + (Q_IN_V ? 4096 : kBatchLds);
  // The copies take addresses of 16-byte alignment; queries that a caller keeps elsewhere (a view into a larger tensor) come
  // through registers.
  const bool q_aligned = ((uintptr_t)a.q & 15) == 0;
#pragma unroll
  for (int i = 0; i < HS / 4; ++i) {
    const int h = min(4 * i + (lane >> 4), Gr - 1);
    const uint8_t *const src = (const uint8_t *)a.q + ((int64_t)seq * a.Hq + hq0 + h) * 256 + n * 16;
    if (q_aligned) dma16(src, q_lds + 1024 * i);
    else *(u32x4 *)(q_lds + 1024 * i + 16 * lane) = *(const u32x4_any *)src;
  }
  if (tv.in_host) {
    wait_vmcnt<0>();
  } else {
    issue_k(first);
    if constexpr (!Q_IN_V) issue_v(first);
    wait_vmcnt<N_K + (Q_IN_V ? 0 : N_V)>();
  }
  const int my_row = n & 3, row_kg = n >> 2;                       // row n = 4 row_kg + my_row
  const int row_head = (row_kg % KPT) * NE + my_row;
  uint32_t qw[16];            // lane (c = n, kg): 32 channels of the head of row c
  {
    u32x4 w[4];
    const uint32_t q0 = (uint32_t)(uintptr_t)(las_ptr)q_lds + min(row_head, HS - 1) * 256;
    lds_query(q0 + key_channel<KF>(kg, 0) * 2, q0 + key_channel<KF>(kg, 8) * 2, q0 + key_channel<KF>(kg, 16) * 2,
              q0 + key_channel<KF>(kg, 24) * 2, w);
#pragma unroll
    for (int i = 0; i < 16; ++i) qw[i] = w[i / 4][i % 4];
  }
  if constexpr (Q_IN_V)
    if (!tv.in_host) issue_v(first);
  // A score is its product times this, in the log2 domain.  Finite for every scale, or a score of zero would be NaN.
  const float unit = fminf(a.scale * kLog2e * (K4 ? 0x1p20f : 0x1p24f), 3.402823466e38f);
  uint32_t qA[TPC][16];      // row operand of the chain's tiles
  // Int8: minus what the code offset 128 adds to a row's product, per channel group.  OFF_LDS: where these 16 registers would
  // make the loop spill, and a reload from scratch waits for every copy in flight (28 / 4 heads, 2 x 23K tokens 22.0 -> 23.3
  // us), they are read from LDS with the keys; elsewhere that costs 1-2 %.
  const uint32_t lds_off = lds0 + (4 - wave) * kTileLds;
  f4 off[NGK];
  float qs[K4 ? 2 : 1][NE];  // int4: a row's sum per channel group (for the zero points), in the product's units
  bool big = false;          // int4: some |q| of the workgroup's heads is 4095 or more
  {
    if (a.q_fmt == TTKV_BF16) {   // bf16 -> fp16 (exact inside the fp16 normal range, clamped outside)
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        const float lo = fminf(fmaxf(__uint_as_float(qw[i] << 16), -65504.0f), 65504.0f);
        const float hi = fminf(fmaxf(__uint_as_float(qw[i] & 0xffff0000u), -65504.0f), 65504.0f);
        qw[i] = (uint32_t)__half_as_ushort(__float2half_rn(lo)) | ((uint32_t)__half_as_ushort(__float2half_rn(hi)) << 16);
      }
    }
    const bool row_on = my_row < NE && row_head < Gr;
#pragma unroll
    for (int i = 0; i < 16; ++i) qw[i] = row_on ? qw[i] : 0u;
    if constexpr (K4) {
      // 16 q on the even registers, unless that leaves fp16's range
      uint32_t top = 0;
#pragma unroll
      for (int i = 0; i < 16; ++i) top = halves_max(top, qw[i] & 0x7fff7fffu);
      big = __any((top & 0xffffu) > 0x6bffu || (top >> 16) > 0x6bffu);
      const _Float16 fe = big ? (_Float16)1.0f : (_Float16)16.0f;
      uint32_t t[16];
#pragma unroll
      for (int r = 0; r < 16; ++r) {   // register r = 4 d + e: elements (8 d + e, 8 d + e + 4) of the slice
        const int dd = r / 4, e = r % 4;
        t[r] = __builtin_amdgcn_perm(qw[4 * dd + 2 + e / 2], qw[4 * dd + e / 2], (e & 1) ? 0x07060302u : 0x05040100u);
        if (r % 2 == 0) t[r] = pk_scale(t[r], fe);
      }
#pragma unroll
      for (int r = 0; r < 16; ++r) qw[r] = t[r];
    }
    // the rows' sums per channel group, by a product with ones: in every lane those of its own rows
#pragma unroll
    for (int gr = 0; gr < NGK; ++gr) {
      const uint32_t ev = K4 && !big ? 0x2C002C00u : 0x3C003C00u, one4[4] = {ev, 0x3C003C00u, ev, 0x3C003C00u};   // 1/16 for 16 q
      f4 sum = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int s = gr * (4 / NGK); s < (gr + 1) * (4 / NGK); ++s) sum = mma32<false>(qw + 4 * s, one4, sum);
      if constexpr (K4) {
#pragma unroll
        for (int e = 0; e < NE; ++e) qs[gr][e] = sum[e] * 0x1p-20f;
      } else {
        off[gr] = sum * (-128.0f * 0x1p-24f);
        if constexpr (OFF_LDS)   // the 16 lanes of a kg store the same; as an opaque store, which waits for no copy in flight
          lds_put<0>(lds_off + 64 * gr + 16 * kg, __builtin_bit_cast(u32x4, off[gr]));
      }
    }
#pragma unroll
    for (int u = 0; u < TPC; ++u)
#pragma unroll
      for (int r = 0; r < 16; ++r) qA[u][r] = TPC == 1 || row_kg / KPT == u ? qw[r] : 0u;
  }

  // ---- addresses of the LDS reads
  // the lane's 8 bytes of the first 32-byte stretch of row n: half kg % 2 of piece kg / 2 (stretch x: by exclusive or with 32 x)
  const uint32_t lka = lds0 + n * FK::ROWB + (((kg >> 1) ^ swz(PK, n)) * 16) + 8 * (kg & 1);
  // what the lane names to the transposing value reads: its row's first piece (the others by exclusive or with 16 x piece)
  uint32_t lva = lds0 + 4096 + lane * 16;
  if constexpr (!VT) {
    const int r4 = 2 * (n & 1) + 16 * ((n >> 1) & 1) + ((n >> 2) & 1) + 4 * kg;   // kTok[n % 8] + 4 kg
    const int row = PV == 8 ? ((n >> 1) & 3) + 16 * (n >> 3) + 4 * kg : NT == 4 ? r4 + 32 * (n >> 3) : r4;
    const int half = PV == 8 ? n & 1 : NT == 4 ? 0 : n >> 3;
    lva = lds0 + 4096 + row * FV::ROWB + swzv(PV, row) * 16 + 8 * half;
  }
  const int my_tok = 16 * (kg / KPT) + n;                             // the lane's token of chain 0
  const uint32_t lma = lds0 + kTileRowsLds + 4 * my_tok;
  // weights: where the lane's go (the second half of its groups a slot distance further), and what it names to a transposing
  // read: quad n % 4 of token 4 kg + n / 4
  const uint32_t lp0 = lds0 + kBatchLds;
  const uint32_t lpw = lp0 + (my_tok & ~15) * Q::RB + Q::place(kg % KPT, n);
  const int quad = n & 3;
  const uint32_t lpr = lp0 + (NE == 4 ? Q::place(quad % KPT, 4 * kg + (n >> 2)) + ((quad / KPT) % Q::GPS) * 8
                                      : Q::place(quad & 1, 4 * kg + (n >> 2)) + ((quad >> 1) % (Q::GR / 2)) * 8);
  // KPT slots further: 16 U KPT bytes, and the tokens' turn by exclusive or
  auto second_half = [&](uint32_t at) -> uint32_t { return Q::HALVES ? (fresh(at) ^ (64 * KPT)) + 16 * Q::U * KPT : at; };

  const f4 zero4 = f4{0.0f, 0.0f, 0.0f, 0.0f};
  f4 acc[8], accc[Q::SETS];       // accc: the centre's share of every channel's sum (the same in all four rows)
  float zs[V4 ? 2 : 1][NE];       // sum_t p_t (z_{t,g} + 8 s_{t,g}) over the lane's tokens
  float l[NE], mcs[NE];           // a token's weight: exp2(score unit + mcs)
#pragma unroll
  for (int s = 0; s < 8; ++s) acc[s] = zero4;
#pragma unroll
  for (int b = 0; b < Q::SETS; ++b) accc[b] = zero4;
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    l[e] = 0.0f;
    mcs[e] = INFINITY;
#pragma unroll
    for (int g = 0; g < (V4 ? 2 : 1); ++g) zs[g][e] = 0.0f;
  }
  // The value operand is fp16(p s), and with p <= 1 that falls into fp16's subnormals or to zero for value scales well
  // below 1 (std 0.02 beside a token 7 above the rest: an error of 1.7e-2 of the output).  So the weights carry a power
  // of two, 2^wexp, that brings the largest value scale the wave has met, with room for twice as large ones, to [2^8, 2^9); it is in l, zs and acc alike and
  // leaves them at the end.  s_top: the largest fp16 number (as bits, ordered like the numbers) of that scale's binade,
  // so that only a scale beyond that room takes the branch below.
  // The weights' reference is a score that no other one exceeds by more than a factor 2^kHeadroom in weight: it moves
  // once or twice per item, where the running maximum of 16 heads moves in most batches.
  constexpr int kHeadroom = 5;
  uint32_t s_top = 0;
  int wexp = 0;
  float limit = -INFINITY;         // of the exponents; the first batch always exceeds it
  // A reference beyond 4 million has no bits left for the power of two: weights of such a head carry none, and no headroom
  // either (32 times a value scale of 8736, as int4 values that span fp16's range have, is beyond fp16).  Product and
  // difference are rounded one after the other: factor - mcs, the reference of the item's result, is then exact.
  uint32_t plain = 0;              // bit e: the weights of element e's head carry no power of two

  const CodeMasks codes;
  u32x4 centre = {0x00800080u, 0x00800080u, 0x00800080u, 0x00800080u};   // the centre as a code: int4 16 x 8, int8 128
  if constexpr (K4) asm volatile("" : "+v"(centre));   // with two loops below it would be formed in every batch

  u32x2 kw[8], meta[2 * NC];
  uint32_t vop[NT / 2][8][VF == TTKV_I8_SYM_G32 ? 2 : 1];   // codes of channel 16 s + n, the pair's 8 tokens of this kg
  auto fetch_k = [&]() {
    const uint32_t ka = fresh(lka);
    if constexpr (PK == 8 && OFF_LDS) lds_keys_i8(ka, ka ^ 32, ka ^ 64, ka ^ 96, lds_off + 16 * kg, kw, off);
    else if constexpr (PK == 8) lds_keys_i8(ka, ka ^ 32, ka ^ 64, ka ^ 96, kw);
    else lds_keys_i4(ka, ka ^ 32, kw);
    lds_meta<NC, 64 * TPC>(lma, meta);
  };
  auto fetch_v = [&]() {
    const uint32_t va = fresh(lva);
    if constexpr (VT) {   // word w of piece hh: block 4 hh + w
      u32x4 w[4];
      lds_pieces<NT>(va, w);
#pragma unroll
      for (int s = 0; s < 8; ++s)
#pragma unroll
        for (int pr = 0; pr < NT / 2; ++pr) vop[pr][s][0] = w[2 * pr + s / 4][s % 4];
    } else {
      u32x2 w[8];
      if constexpr (PV == 8) {
        lds_values_i8(va, va ^ 16, va ^ 32, va ^ 48, w);
        lds_values_i8(va ^ 64, va ^ 80, va ^ 96, va ^ 112, w + 4);
      } else if constexpr (NT == 4) {
        lds_values_i4x4(va, va ^ 16, va ^ 32, va ^ 48, w);
      } else {
        lds_values_i4x2(va, va ^ 16, va ^ 32, va ^ 48, w);
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) {
        if constexpr (PV == 8) {
          vop[0][s][0] = w[s].x;
          vop[0][s][1] = w[s].y;
        } else if constexpr (NT == 4) {
          vop[0][s][0] = w[s].x;
          vop[1][s][0] = w[s].y;
        } else {
          vop[0][s][0] = s % 2 ? w[s / 2].y : w[s / 2].x;
        }
      }
    }
  };

  // before_v runs between the softmax and the first use of the batch's V half.
  auto compute = [&](int nv, auto big_tag, auto before_v) __attribute__((always_inline)) {
    // ---- scores: element e of chain j is head (kg % KPT) NE + e of token 16 TPC j + my_tok
    float x[NC][NE];
    uint32_t top = 0;   // the largest value scale of the lane's tokens
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const uint32_t m0 = meta[2 * j].x, m1 = meta[2 * j].y;
      float v[NE];
      // One product chain per channel group, all before the first result is used: one after the other each result was waited
      // for (64 / 4 heads, 8 x 64K tokens of K int8 / V int4 81.0 -> 80.0 us; 64 / 2 heads, 24 x 21K tokens 86.4 -> 85.3).
      f4 sv[NGK];
#pragma unroll
      for (int gr = 0; gr < NGK; ++gr) {
        sv[gr] = K4 ? zero4 : off[gr];
#pragma unroll
        for (int u = 0; u < TPC; ++u) {
          const u32x2 w = kw[(j * TPC + u) * NGK + gr];   // the lane's 8 bytes of the group
          if constexpr (K4) {
            uint32_t kr[8];
            auto take = [&](uint32_t x, uint32_t *r) {
              if constexpr (decltype(big_tag)::value) value_codes4(x, r, codes);
              else key_codes4(x, r, codes);
            };
            take(w.x, kr);
            take(w.y, kr + 4);
            sv[gr] = mma32<false>(qA[u] + 8 * gr, kr, sv[gr]);
            sv[gr] = mma32<false>(qA[u] + 8 * gr + 4, kr + 4, sv[gr]);
          } else {
            uint32_t kr[4];
            codes8(w.x, kr, codes);
            codes8(w.y, kr + 2, codes);
            sv[gr] = mma32<false>(qA[u] + 4 * gr, kr, sv[gr]);
          }
        }
      }
#pragma unroll
      for (int gr = 0; gr < NGK; ++gr)
#pragma unroll
        for (int e = 0; e < NE; ++e) {
          if constexpr (K4) {   // the group's zero point and scale
            const uint32_t m = gr ? m1 : m0;
            v[e] = gr ? fmaf(half1(m), qs[gr][e], v[e]) : half1(m) * qs[gr][e];
            v[e] = fmaf(sv[gr][e], half0(m), v[e]);
          } else {              // the group's scale
            const uint32_t m = gr / 2 ? m1 : m0;
            v[e] = gr ? fmaf(sv[gr][e], gr % 2 ? half1(m) : half0(m), v[e]) : sv[gr][e] * half0(m);
          }
        }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        x[j][e] = v[e];
      }
      const uint32_t t = halves_max(meta[2 * j + 1].x, meta[2 * j + 1].y);   // scales are not negative
      top = max(top, V4 ? t & 0xffffu : max(t & 0xffffu, t >> 16));
    }

    if (nv < TT)   // wave-uniform
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int e = 0; e < NE; ++e) x[j][e] = 16 * TPC * j + my_tok < nv ? x[j][e] : -INFINITY;

    // ---- online softmax (base 2)
    float p[NC][NE];   // exponents, then weights
    float most = -INFINITY;
#pragma unroll
    for (int j = 0; j < NC; ++j)
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        p[j][e] = fmaf(x[j][e], unit, mcs[e]);
        most = fmaxf(most, p[j][e]);
      }
    if (__any(most > limit || top > s_top)) {
      const int before = wexp;
      if (__any(top > s_top)) {
        s_top = (wave_max16(top) | 0x3ffu) + 0x400u;   // a binade of room
        wexp = 29 - kHeadroom - max((int)(s_top >> 10), 1);
      }
      float alpha[NE];
      limit = INFINITY;
      const uint32_t was_plain = plain;
      plain = 0;
#pragma unroll
      for (int e = 0; e < NE; ++e) {
#pragma clang fp contract(off)
        float mx = x[0][e];
#pragma unroll
        for (int j = 1; j < NC; ++j) mx = fmaxf(mx, x[j][e]);
        mx = row_max(mx);   // over the 16 tokens, then the chain's tiles
        if constexpr (TPC == 4) mx = fmaxf(both16(mx).x, both16(mx).y);
        if constexpr (TPC >= 2) mx = fmaxf(both32(mx).x, both32(mx).y);
        // the reference so far: factor - mcs, minus infinity before the first batch
        const float old = mcs[e];
        const float r_old = ((was_plain >> e) & 1 ? 0.0f : (float)before) - old;
        const float r = fmaxf(r_old, mx * unit);
        const bool none = !(fabsf(r) < 4194304.0f);
        const float f = none ? 0.0f : (float)wexp;
        plain |= none ? 1u << e : 0u;
        mcs[e] = f - r;
        limit = fminf(limit, none ? 0.0f : f + (float)kHeadroom);
        alpha[e] = __builtin_amdgcn_exp2f(mcs[e] - old);
        l[e] *= alpha[e];
        if constexpr (V4) {
          zs[0][e] *= alpha[e];
          zs[1][e] *= alpha[e];
        }
      }
      // a column's factor: that of its head
      float ac = 0.0f;
      const int h = Q::head_of((int)fresh(n));
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        const float v = KPT == 1 ? alpha[e] : __shfl(alpha[e], 16 * (h / NE));   // one kg per tile: every lane has all heads
        if (h % NE == e) ac = v;
      }
#pragma unroll
      for (int s = 0; s < 8; ++s) acc[s] *= ac;
#pragma unroll
      for (int b = 0; b < Q::SETS; ++b) accc[b] *= ac;
#pragma unroll
      for (int j = 0; j < NC; ++j)
#pragma unroll
        for (int e = 0; e < NE; ++e) p[j][e] = fmaf(x[j][e], unit, mcs[e]);
    }
    float vs[NC][NGV];   // the values' scales as they meet the weights
#pragma unroll
    for (int j = 0; j < NC; ++j) {
      const uint32_t m0 = meta[2 * j + 1].x, m1 = meta[2 * j + 1].y;
      float z[2] = {0.0f, 0.0f};
      if constexpr (V4) {   // zero point + the centre 8 x scale
        z[0] = fmaf(8.0f, half0(m0), half1(m0));
        z[1] = fmaf(8.0f, half0(m1), half1(m1));
        vs[j][0] = half0(m0);
        vs[j][1] = half0(m1);
      } else {
        vs[j][0] = half0(m0); vs[j][1] = half1(m0);
        vs[j][2] = half0(m1); vs[j][3] = half1(m1);
      }
#pragma unroll
      for (int e = 0; e < NE; ++e) {
        p[j][e] = __builtin_amdgcn_exp2f(p[j][e]);
        l[e] += p[j][e];
        if constexpr (V4) {
          zs[0][e] = fmaf(p[j][e], z[0], zs[0][e]);
          zs[1][e] = fmaf(p[j][e], z[1], zs[1][e]);
        }
      }
    }

    // ---- weighted V, two 16-token tiles per 32-deep product.  The codes' words are the A operands of the eight channel
    // blocks; the weights, times the scales of a channel group, go through LDS into the B operand's layout (rows of a
    // token in, columns of a (group, head) out).  They meet the values with 22 bits, as fp16(p s) and its remainder: two
    // products, which are not what bounds the loop.  (With fp16(p s) alone the error is 1e-4, and keeping it there takes
    // the running maximum as reference, so that the largest weight is a power of two.)
    auto put_weights = [&](int j, int round, auto at_tag) __attribute__((always_inline)) {   // chain j, channel groups GR round ..
      constexpr int AT = decltype(at_tag)::value;
      uint32_t w[Q::GR * NE / 2], r[Q::GR * NE / 2];
#pragma unroll
      for (int g = 0; g < Q::GR; ++g)
#pragma unroll
        for (int e = 0; e < NE; e += 2) {
          const float s = vs[j][Q::GR * round + g];
          const uint32_t x = pk(p[j][e] * s, p[j][e + 1] * s);
          w[(g * NE + e) / 2] = x;
          r[(g * NE + e) / 2] = pk(fmaf(p[j][e], s, -half0(x)), fmaf(p[j][e + 1], s, -half1(x)));
        }
      if constexpr (Q::GR * NE == 4) {
        lds_put<AT>(lpw, u32x2{w[0], w[1]});
        lds_put<AT + 2048>(lpw, u32x2{r[0], r[1]});
      } else {
        lds_put<AT>(lpw, u32x4{w[0], w[1], w[2], w[3]});
        lds_put<AT + 2048>(lpw, u32x4{r[0], r[1], r[2], r[3]});
        if constexpr (Q::HALVES) {
          lds_put<AT>(second_half(lpw), u32x4{w[4], w[5], w[6], w[7]});
          lds_put<AT + 2048>(second_half(lpw), u32x4{r[4], r[5], r[6], r[7]});
        }
      }
    };
    auto product = [&](int pr, int b, const u32x2 *w) __attribute__((always_inline)) {   // pair pr, operand set b
      const uint32_t B[4] = {w[0].x, w[0].y, w[2].x, w[2].y}, R[4] = {w[1].x, w[1].y, w[3].x, w[3].y};
      constexpr int BPG = 8 / NGV;   // channel blocks per group
#pragma unroll
      for (int s = b * Q::GPS * BPG; s < (b + 1) * Q::GPS * BPG; ++s) {
        uint32_t vr[4];
        if constexpr (V4) {
          value_codes4(vop[pr][s][0], vr, codes);
        } else {
          codes8(vop[pr][s][0], vr, codes);
          codes8(vop[pr][s][VF == TTKV_I8_SYM_G32 ? 1 : 0], vr + 2, codes);
        }
        acc[s] = mma32<false>(vr, R, acc[s]);
        acc[s] = mma32<false>(vr, B, acc[s]);
      }
      const uint32_t cc[4] = {centre.x, centre.y, centre.z, centre.w};
      accc[b] = mma32<false>(cc, R, accc[b]);
      accc[b] = mma32<false>(cc, B, accc[b]);
    };
    constexpr int T16 = 16 * Q::RB, SET = Q::HALVES ? 0 : Q::GPS * 8;   // bytes of a tile's weights; to the second operand set
    if constexpr (Q::BY_PAIR) {
      static_assert(!Q::BY_PAIR || (NC == 4 && Q::NR == 1 && Q::NB == 2), "one tile per chain, two sets");
      u32x2 w[16];
      put_weights(0, 0, std::integral_constant<int, 0>{});
      put_weights(1, 0, std::integral_constant<int, T16>{});
      lds_weights<0, T16, Q::GPS * 8, T16 + Q::GPS * 8>(lpr, lpr, w);
      put_weights(NC - 2, 0, std::integral_constant<int, 0>{});
      put_weights(NC - 1, 0, std::integral_constant<int, T16>{});
      lds_weights<0, T16, Q::GPS * 8, T16 + Q::GPS * 8>(lpr, lpr, w + 8);
      before_v();
#pragma unroll
      for (int pr = 0; pr < NT / 2; ++pr)
#pragma unroll
        for (int b = 0; b < Q::NB; ++b) product(pr, b, w + 8 * pr + 4 * b);
    } else if constexpr (NT == 4) {   // one operand set, both pairs
      static_assert(NT != 4 || Q::BY_PAIR || (Q::SETS == 1 && Q::NR == 1), "one set");
      put_weights(0, 0, std::integral_constant<int, 0>{});
      if constexpr (NC == 2) put_weights(NC - 1, 0, std::integral_constant<int, 2 * T16>{});
      u32x2 w[8];
      lds_weights<0, T16, 2 * T16, 3 * T16>(lpr, lpr, w);
      before_v();
      product(0, 0, w);
      product(NT / 2 - 1, 0, w + 4);
    } else {
#pragma unroll
      for (int round = 0; round < Q::NR; ++round) {   // a round's products before the next one's weights: half as many in registers
        u32x2 w[4 * Q::NB];
        put_weights(0, round, std::integral_constant<int, 0>{});
        if constexpr (NC == 2) put_weights(NC - 1, round, std::integral_constant<int, T16>{});
        if constexpr (Q::NB == 2) lds_weights<0, T16, SET, T16 + SET>(lpr, second_half(lpr), w);
        else lds_weights<0, T16>(lpr, w);
        if (round == 0) before_v();
#pragma unroll
        for (int b = 0; b < Q::NB; ++b) product(0, Q::NB * round + b, w + 4 * b);
      }
    }
  };

  // While batch i is computed the copies of batch i + 1 are in flight: its K half is issued once batch i's K rows and meta
  // words are in registers, its V half once batch i's V rows are.  Loads complete in order, so "at most as many
  // outstanding as were issued after it" means a half has landed.
  auto loop = [&](auto big_tag) __attribute__((always_inline)) {
    for (int i0 = first; i0 < c1; i0 += step_tokens) {
      const bool more = !tv.in_host && i0 + step_tokens < c1;   // wave-uniform
      if (tv.in_host) bring_host(i0);
      else wait_vmcnt<N_V>();
      fetch_k();
      if (more) issue_k(i0 + step_tokens);
      compute(min(TT, c1 - i0), big_tag, [&]() {
        if (more) wait_vmcnt<N_K>();
        else wait_vmcnt<0>();
        fetch_v();
        if (more) issue_v(i0 + step_tokens);
      });
    }
  };
  if (!K4 || !big) {
    loop(std::false_type{});
  } else {
    if constexpr (K4) loop(std::true_type{});
  }

  // ---- the wave's result.  Sums over the lane's tokens come together; a head's zero-point sums, and what its weights
  // carry, reach the columns through LDS.
  float *const s_head = (float *)(wbuf + kTileRowsLds);   // [head][4], where the meta words were
#pragma unroll
  for (int e = 0; e < NE; ++e) {
    auto over_tokens = [&](float v) {
      v = group_sum<16>(v);
      if constexpr (TPC == 4) v = both16(v).x + both16(v).y;
      if constexpr (TPC >= 2) v = both32(v).x + both32(v).y;
      return v;
    };
    l[e] = over_tokens(l[e]);
    float z[2] = {0.0f, 0.0f};
    if constexpr (V4) {
      z[0] = over_tokens(zs[0][e]);
      z[1] = over_tokens(zs[1][e]);
    }
    const float w = (plain >> e) & 1 ? 0.0f : (float)wexp, unscale = pow2(-(int)w);
    const int h = (kg % KPT) * NE + e;
    if (n == 0 && kg < KPT) {
      s_head[4 * h] = z[0] * unscale;
      s_head[4 * h + 1] = z[1] * unscale;
      s_head[4 * h + 2] = unscale * (V4 ? 0x1p20f : 0x1p24f);
      ((float *)(wbuf + kSumsLds))[h] = w - mcs[e];   // log2 domain
      ((float *)(wbuf + kSumsLds))[16 + h] = l[e] * unscale;
    }
  }
  const int h = Q::head_of(n);
  if (h < Gr && !Q::spare(n)) {
    float (*w_acc)[128] = (float (*)[128])wbuf;   // [head][channel]; the wave's last batch has been consumed
    const float back = s_head[4 * h + 2];
#pragma unroll
    for (int s = 0; s < 8; ++s) {
      const int g = s / (8 / NGV), b = g / Q::GPS;
      if (g % Q::GPS != Q::group_of(n)) continue;
      const float z = V4 ? s_head[4 * h + g] : 0.0f;
#pragma unroll
      for (int i = 0; i < 4; ++i) w_acc[h][16 * s + 4 * kg + i] = fmaf(acc[s][i] - accc[b][i], back, z);
    }
  }
}

// What the tiers of a launch hold: each kind is compiled without the cases it does not meet, so that their registers do
// not count.  With 4-bit keys or values two workgroups per CU, otherwise three (int8 and 16 heads with two: 64 / 2 heads, 98K
// tokens 39.5 us against 37.1, 24 x 21K tokens 104.3 against 102.8; 64 / 4 heads, 16 x 16K tokens 61.0 against 59.5).
// HS: places for heads (QuantShape).
enum LaunchKind { FP_ONLY, WITH_INT8, WITH_4BIT, WITH_T128 };
// Key formats that stay with the vector kernel's head pairs when keys grouped over tokens are in the same launch: those
// have fp32 weights, where process_rows rounds the weights of the grouped keys, and the values beside them, to 16 bits.  Error
// against 64 bits and time of 2 sequences of 8192 tokens of the format and 16384 of grouped keys, pairs and matrix cores: 16 / 2
// heads, int8 3.0e-5 in 35.6 us, 1.5e-4 in 16.8; 32 / 2 heads 2.9e-5 in 54.9, 1.7e-4 in 18.4, int4 4.0e-5 in 55.3, 1.7e-4 in 16.8
// (with 22-bit weights still 1.3e-4 to 1.9e-4).  Launches that took the matrix cores before there was a faster way for all of
// them stay there.
constexpr bool pairs_beside_t128(int k_fmt, int G) { return (k_fmt == TTKV_I8_SYM_G32 && G > 4) || (k_fmt == TTKV_I4_ASYM_G64 && G > 8); }
constexpr int waves_per_simd(int kind) { return kind == FP_ONLY || kind == WITH_INT8 ? 3 : 2; }
// Two tiles' rows of queries (8 places), or three workgroups per CU with 16.
constexpr bool offsets_in_lds(int kind, int hs) { return hs == 8 || (hs == 16 && kind == WITH_INT8); }
template <int KIND, int HS>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(waves_per_simd(KIND), waves_per_simd(KIND)))) void attn_mfma_kernel(const FusedArgs a) {
  static_assert(kTileRowsLds >= 16 * 128 * 4 && 3 * lds_given(4 * kTileLds + kOffLds) <= 160 * 1024, "the wave's result; three workgroups per CU");
  __shared__ __attribute__((aligned(256))) char s_buf[4 * kTileLds + kOffLds];   // per wave: batches in flight, then [head][channel] floats
  char *const wbuf = s_buf + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6) * kTileLds;

  // Linear workgroup id -> (item, KV head, block of heads).  More heads per KV head than one tile takes are cut
  // into blocks of mfma_heads; the blocks of one (item, KV head) read the same bytes and get ids 8 apart, so that
  // they run on the same XCD at the same time and the later readers are served from its L2.
  touch_arguments(a);
  const int Gtot = a.G;
  const uint32_t id = blockIdx.x;
  const bool blocks = Gtot > a.mfma_heads;                    // more than one block of heads
  const uint32_t n_hb = blocks ? (Gtot + a.mfma_heads - 1) / a.mfma_heads : 1;
  const uint32_t base = blocks ? ((id >> 3) / n_hb) * 8 + (id & 7) : id;
  if (base >= (uint32_t)a.n_items * a.Hkv) return;
  const int item = item_of(a, base);
  const int hkv = base - item * a.Hkv;
  const int hb0 = blocks ? ((id >> 3) % n_hb) * a.mfma_heads : 0;          // first head of the block within the KV head's heads
  const int hq0 = hkv * Gtot + hb0;
  const int G = min(a.mfma_heads, Gtot - hb0);                // heads in this block

  const int lo = find_run(a, item);
  RunView en = run_view(a, lo);
  const int tier = en.tier, seq = en.seq, item_start = a.start[lo];
  TierView tv = a.tv[tier];
  if (en.flags & kEntryNoTable) tv.table = nullptr;   // the run names pool records directly
  int chunk_tokens = a.chunk[tier];
  const bool equal_items = chunk_tokens == 0;
  const int n_even = equal_items ? (lo + 1 < a.n_entries ? a.start[lo + 1] : a.n_items) - item_start : 0;
  if (equal_items) chunk_tokens = even_chunk(en.len, n_even);
  const int part = en.part_base + item - item_start;   // this item's partial
  int chunk = item - item_start;
  if ((en.flags & kEntrySelected) && a.host_ids && chunk == 0 && hq0 == 0) report_selected(a, tv, en, seq, equal_items);
  const int32_t *sel = resolve_selected(a, tv, en, seq, equal_items, chunk_tokens, chunk);

  constexpr bool K8 = KIND != WITH_T128 || !pairs_beside_t128(TTKV_I8_SYM_G32, HS), K4 = KIND != WITH_T128 || !pairs_beside_t128(TTKV_I4_ASYM_G64, HS);
  const int combo = tv.k_fmt * 8 + tv.v_fmt;
#define TTKV_ROWS(KF, VF) process_rows<KF, VF>(a, tv, en, sel, chunk_tokens, chunk, seq, hq0, G, hkv, wbuf)
#define TTKV_QUANT(KF, VF)                                                                               \
  process_quant<KF, VF, HS, KF == TTKV_I8_SYM_G32 && offsets_in_lds(KIND, HS)>(a, tv, en, sel, chunk_tokens, chunk, n_even, seq, hq0, G, \
                                                                               hkv, wbuf)
  switch (combo) {
    case TTKV_F16 * 8 + TTKV_F16: TTKV_ROWS(TTKV_F16, TTKV_F16); break;
    case TTKV_BF16 * 8 + TTKV_BF16: TTKV_ROWS(TTKV_BF16, TTKV_BF16); break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I8_SYM_G32:
      if constexpr (KIND >= WITH_INT8 && K8) TTKV_QUANT(TTKV_I8_SYM_G32, TTKV_I8_SYM_G32);
      break;
    case TTKV_I4_ASYM_T128 * 8 + TTKV_I4_ASYM_G64:
      if constexpr (KIND == WITH_T128) TTKV_ROWS(TTKV_I4_ASYM_T128, TTKV_I4_ASYM_G64);
      break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I4_ASYM_G64:
      if constexpr (KIND >= WITH_4BIT && K8) TTKV_QUANT(TTKV_I8_SYM_G32, TTKV_I4_ASYM_G64);
      break;
    case TTKV_I8_SYM_G32 * 8 + TTKV_I4_ASYM_G64_T32:
      if constexpr (KIND >= WITH_4BIT && K8) TTKV_QUANT(TTKV_I8_SYM_G32, TTKV_I4_ASYM_G64_T32);
      break;
    case TTKV_I4_ASYM_G64 * 8 + TTKV_I4_ASYM_G64_T32:
      if constexpr (KIND >= WITH_4BIT && K4) TTKV_QUANT(TTKV_I4_ASYM_G64, TTKV_I4_ASYM_G64_T32);
      break;
    default:
      if constexpr (KIND >= WITH_4BIT && K4) TTKV_QUANT(TTKV_I4_ASYM_G64, TTKV_I4_ASYM_G64);
      break;
  }
#undef TTKV_ROWS
#undef TTKV_QUANT
  __syncthreads();

  // ---- merge the four waves (each with its own running max) and write the item's partials: four channels per thread, so
  // that 16 heads take two turns of a chain of LDS reads and exponentials, not eight (64 / 4 heads, 4 x 6K tokens 17.9 -> 16.8
  // us, 64 / 2 heads 82K tokens 38.4 -> 35.8).  Partials are 16-byte stores to addresses of 8-byte alignment (4, if
  // the caller's workspace is), which the merge reads alike.
  for (int idx = threadIdx.x; idx < G * 32; idx += 256) {
    const int g = idx >> 5, c4 = idx & 31;
    float m[4], l[4];
    f4 x[4];
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float *sums = (const float *)(s_buf + w * kTileLds + kSumsLds);
      m[w] = sums[g];
      l[w] = sums[16 + g];
      x[w] = ((const f4 *)(s_buf + w * kTileLds))[idx];
    }
    const float M = fmaxf(fmaxf(m[0], m[1]), fmaxf(m[2], m[3]));
    f4 o = f4{0.0f, 0.0f, 0.0f, 0.0f};
    float ll = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      const float wgt = m[w] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(m[w] - M);
#pragma unroll
      for (int i = 0; i < 4; ++i) o[i] = fmaf(x[w][i], wgt, o[i]);
      ll = fmaf(l[w], wgt, ll);
    }
    const int64_t prow = ((int64_t)seq * a.Hq + hq0 + g) * a.part_stride + part;
    *(f4_any *)(a.pacc + prow * 128 + c4 * 4) = o;
    if (c4 == 0) {
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
// What one launch needs: heads per block, quantized tiers, 4-bit ones, keys grouped over tokens.  ok: the kernel takes it.
struct MfmaShape {
  int heads;
  bool quantized, four_bit, t128, ok;
};
MfmaShape mfma_shape(const FusedArgs &a) {
  const int G = a.Hq / a.Hkv;
  MfmaShape m{std::min(16, G), false, false, false, true};
  bool pairs = false;
  for (int j = 0; j < a.n_entries; ++j) {
    const TierView &tv = a.tv[entry_tier(a.e[j])];
    m.ok &= attn_mfma_fits(tv.k_fmt, tv.v_fmt, G);
    m.quantized |= !is_fp(tv.k_fmt);
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
  auto go = [&](auto hs) {
    constexpr int HS = decltype(hs)::value;
    if (m.t128) hipLaunchKernelGGL((attn_mfma_kernel<WITH_T128, HS>), grid, dim3(256), 0, s, a);
    else if (m.four_bit) hipLaunchKernelGGL((attn_mfma_kernel<WITH_4BIT, HS>), grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL((attn_mfma_kernel<WITH_INT8, HS>), grid, dim3(256), 0, s, a);
  };
  if (!m.quantized) hipLaunchKernelGGL((attn_mfma_kernel<FP_ONLY, 4>), grid, dim3(256), 0, s, a);
  else if (m.heads <= 4) go(std::integral_constant<int, 4>{});
  else if (m.heads <= 8) go(std::integral_constant<int, 8>{});
  else go(std::integral_constant<int, 16>{});
  return hipGetLastError();
}

}  // namespace ttkv
