// Device helpers shared by the attention kernels: row geometry per format, the
// splice of int4 / int8 codes into fp16 mantissas, DPP lane exchanges.
#pragma once
#include "ttkv_internal.h"

#include <hip/hip_fp16.h>

namespace ttkv {
namespace dev {

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

typedef _Float16 h2 __attribute__((ext_vector_type(2)));
typedef __bf16 b2 __attribute__((ext_vector_type(2)));

template <int F> struct Fmt;
template <> struct Fmt<TTKV_F16> { static constexpr int ROWB = 256, LPT = 16, TPL = 4, EPL = 8; };
template <> struct Fmt<TTKV_BF16> { static constexpr int ROWB = 256, LPT = 16, TPL = 4, EPL = 8; };
template <> struct Fmt<TTKV_I8_SYM_G32> { static constexpr int ROWB = 128, LPT = 8, TPL = 8, EPL = 16; };
template <> struct Fmt<TTKV_I4_ASYM_G64> { static constexpr int ROWB = 64, LPT = 4, TPL = 16, EPL = 32; };
template <> struct Fmt<TTKV_I4_ASYM_T128> { static constexpr int ROWB = 64, LPT = 4, TPL = 16, EPL = 32; };   // rows as int4
template <> struct Fmt<TTKV_I4_ASYM_G64_T32> { static constexpr int ROWB = 64, LPT = 4, TPL = 16, EPL = 32; };   // bytes per token as int4
template <int F> constexpr bool is_i4() { return F == TTKV_I4_ASYM_G64 || F == TTKV_I4_ASYM_T128 || F == TTKV_I4_ASYM_G64_T32; }

// Streaming loads: K/V bytes are read exactly once per launch, so they are fetched with the
// non-temporal hint (no reuse expected).  On MI355X a load-only kernel moves 6.5-7.0 TB/s this way
// against 5.7-6.1 TB/s with plain loads (measured, 2 GiB, same access pattern).
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ uint4 ld_stream(const uint4 *p) {
  const u32x4 v = __builtin_nontemporal_load((const u32x4 *)p);
  return uint4{v.x, v.y, v.z, v.w};
}
__device__ __forceinline__ uint2 ld_stream(const uint2 *p) {
  const u32x2 v = __builtin_nontemporal_load((const u32x2 *)p);
  return uint2{v.x, v.y};
}
__device__ __forceinline__ uint32_t ld_stream(const uint32_t *p) { return __builtin_nontemporal_load(p); }
__device__ __forceinline__ uint16_t ld_stream(const uint16_t *p) { return __builtin_nontemporal_load(p); }

__device__ __forceinline__ float h2f(uint16_t h) { return __half2float(__ushort_as_half(h)); }
__device__ __forceinline__ h2 as_h2(uint32_t u) { return __builtin_bit_cast(h2, u); }
__device__ __forceinline__ b2 as_b2(uint32_t u) { return __builtin_bit_cast(b2, u); }

// Position of element e of a lane's 16-byte slice inside the packed pair registers:
// register e/2-ish and half, per format (see unpack16).
//   F16 / BF16 / I8 : pair r = e/2 holds (e, e+1)                      -> natural
//   I4              : dword d = e/8, pairs (0,4) (1,5) (2,6) (3,7)     -> r = 4d + e%4, half = (e%8)/4
template <int F>
__device__ __forceinline__ constexpr int pair_reg(int e) {
  return is_i4<F>() ? 4 * (e / 8) + (e % 4) : e / 2;
}
template <int F>
__device__ __forceinline__ constexpr int pair_half(int e) {
  return is_i4<F>() ? (e % 8) / 4 : e % 2;
}
// Offset o_e that unpack16 leaves on element e.
template <int F>
__device__ __forceinline__ constexpr float elem_offset(int e) {
  return is_i4<F>() ? ((e % 2) ? 64.0f : 1024.0f) : (F == TTKV_I8_SYM_G32 ? 1152.0f : 0.0f);
}

// Bit patterns used to splice int4 codes into fp16 mantissas.  They are kept in
// registers the compiler cannot see through (two SGPR masks, two VGPR constants):
// gfx9 VOP3 encodings take no literals, and with literals the compiler falls back
// to v_and + v_or instead of one v_and_or_b32 per pair.
struct Splice {
  uint32_t m0, m1, c0, c1;
  __device__ __forceinline__ void init() {
    m0 = 0x000F000Fu; m1 = 0x00F000F0u; c0 = 0x64006400u; c1 = 0x54005400u;
    asm volatile("" : "+s"(m0), "+s"(m1), "+v"(c0), "+v"(c1));
  }
};

// Eight 4-bit codes -> four registers of packed fp16 pairs, offsets 1024 (even registers) and 64 (odd ones) included.
__device__ __forceinline__ void splice4(uint32_t x, uint32_t *r, const Splice &k) {
  const uint32_t y = x >> 8;
  r[0] = (x & k.m0) | k.c0;   // (1024 + n0, 1024 + n4)
  r[1] = (x & k.m1) | k.c1;   // (  64 + n1,   64 + n5)
  r[2] = (y & k.m0) | k.c0;   // (1024 + n2, 1024 + n6)
  r[3] = (y & k.m1) | k.c1;   // (  64 + n3,   64 + n7)
}

// 16 bytes of a row -> EPL/2 registers of packed 16-bit pairs (fp16, or bf16 for the bf16 tier).
template <int F>
__device__ __forceinline__ void unpack16(const uint4 &w, uint32_t *r, const Splice &k) {
  const uint32_t u[4] = {w.x, w.y, w.z, w.w};
  if constexpr (F == TTKV_F16 || F == TTKV_BF16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = u[i];
  } else if constexpr (F == TTKV_I8_SYM_G32) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const uint32_t x = u[i] ^ 0x80808080u;                       // byte -> code + 128 in [1, 255]
      r[2 * i] = __builtin_amdgcn_perm(0x64646464u, x, 0x04010400u);      // (1024 + b0, 1024 + b1)
      r[2 * i + 1] = __builtin_amdgcn_perm(0x64646464u, x, 0x04030402u);  // (1024 + b2, 1024 + b3)
    }
  } else {
#pragma unroll
    for (int i = 0; i < 4; ++i) splice4(u[i], r + 4 * i, k);
  }
}

template <int CTRL>
__device__ __forceinline__ float dpp(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), CTRL, 0xf, 0xf, true));
}
// sum / max over groups of LPT consecutive lanes (LPT = 4, 8, 16) -- every lane gets the result
template <int LPT>
__device__ __forceinline__ float group_sum(float v) {
  v += dpp<0xB1>(v);                       // quad_perm [1,0,3,2]
  v += dpp<0x4E>(v);                       // quad_perm [2,3,0,1]: every lane holds its quad's sum
  if constexpr (LPT >= 8) v += dpp<0x141>(v);   // row_half_mirror: lane i <- lane 7-i = the other quad's sum
  if constexpr (LPT >= 16) v += dpp<0x140>(v);  // row_mirror: lane i <- lane 15-i = the other half's sum
  return v;
}
// One run of the launch, unpacked.
struct RunView {
  int tier, seq, part_base;
  uint32_t flags;
  int rec_base;    // record of ring block 0 (no block table) or the run's first pool record
  int first_tok;   // ring token index of the run's first token, 0 for runs that name records; selected: newest block id
  int len;
  int id_base;     // of a run of selected blocks: the multiple of the ring's blocks below the newest id
};
// Ring block of a selected id, which is less than a ring older than the newest one (a remainder is worked out on the vector
// unit, some 30 instructions for every batch of a wave).
__device__ __forceinline__ int ring_of_id(int id, const RunView &en, const TierView &tv) {
  const int rb = id - en.id_base;
  return rb < 0 ? rb + tv.ring_blocks : rb;
}
__device__ __forceinline__ RunView run_view(const FusedArgs &a, int i) {
  const Entry e = a.e[i];
  RunView r;
  r.tier = entry_tier(e);
  r.seq = (e.head >> 20) & 63;
  r.part_base = e.head & (TTKV_MAX_PARTS - 1);
  r.flags = e.head & (kEntryNoTable | kEntrySelected);
  const bool direct = r.flags & kEntryNoTable;
  r.rec_base = direct ? e.at : r.seq * a.tv[r.tier].ring_blocks;
  r.first_tok = direct ? 0 : e.at;
  r.len = e.len;
  r.id_base = 0;
  return r;
}
// Asks for what the look-up of an item reads, all at once and before anything is worked out: a launch's arguments are in no
// cache when its first workgroups start, and every load that waits for another one costs some 0.2 us of them.
__device__ __forceinline__ void touch_arguments(const FusedArgs &a) {
  asm volatile("" ::"s"(a.n_entries), "s"(a.n_items), "s"(a.Hkv), "s"(a.G), "s"(a.hkv_magic), "s"(a.start[0]), "s"(a.start[15]),
               "s"(a.tv[0].bt), "s"(a.tv[1].bt), "s"(a.tv[2].bt), "s"(a.tv[3].bt), "s"(a.e[0].len), "s"(a.e[5].len),
               "s"(a.e[10].len), "s"(a.chunk[0]), "s"(a.q_fmt));
}
// The first workgroup of a run of selected blocks also stores their ids and number to the caller's pinned memory: the
// stores cross PCIe while the launch streams (two copies behind it took 2-3 us of the stream; stored by the ranking kernel,
// whose end waits for them, as much).
__device__ __forceinline__ void report_selected(const FusedArgs &a, const TierView &tv, const RunView &en, int seq, bool equal_items) {
  const int n = equal_items ? en.len / tv.bt : en.len;
  for (int i = threadIdx.x; i < n; i += blockDim.x) a.host_ids[seq * a.sel_stride + i] = a.sel_ids[seq * a.sel_stride + i];
  if (threadIdx.x == 0) a.host_count[seq] = n;
}
// A run whose blocks are named by the device-side selection (ids ascending, so only the last can be the tier's
// partly filled newest block).  Two forms, told apart by the tier's item size in the launch arguments:
//   fixed items (host tiers): item `chunk` of the run is sub-chunk chunk % ipb of the run's (chunk / ipb)-th
//     selected block; the entry is rewritten into a run over that one block;
//   equal items (tiers in HBM): the tokens of all selected blocks form ONE run of len tokens, cut like any other
//     run; token i of it lies in block ids[i / bt], which the tile address look-up follows (`sel`), so an item may
//     span several blocks and small blocks cost no more than large ones.
// Either way everything after this sees an ordinary run.  Returns the run's id list for the second form.
__device__ __forceinline__ const int32_t *resolve_selected(const FusedArgs &a, const TierView &tv, RunView &en, int seq,
                                                           bool equal_items, int chunk_tokens, int &chunk) {
  if (!(en.flags & kEntrySelected)) return nullptr;
  const int32_t *ids = a.sel_ids + seq * a.sel_stride;
  if (equal_items) {
    if (ids[en.len / tv.bt - 1] == en.first_tok) en.len -= tv.bt - a.sel_last_ntok[seq];
    en.id_base = __builtin_amdgcn_readfirstlane(en.first_tok - en.first_tok % tv.ring_blocks);
    en.first_tok = 0;
    return ids;
  }
  const int ipb = (tv.bt + chunk_tokens - 1) / chunk_tokens;
  const int blk = chunk / ipb;
  chunk -= blk * ipb;
  const int32_t id = ids[blk];
  en.len = id == en.first_tok ? a.sel_last_ntok[seq] : tv.bt;
  en.first_tok = (id % tv.ring_blocks) * tv.bt;
  return nullptr;
}

// the two values of the lanes 16 (32) apart by exclusive or, in the same order in both
typedef float f2 __attribute__((ext_vector_type(2)));
__device__ __forceinline__ f2 both16(float v) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f2{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
__device__ __forceinline__ f2 both32(float v) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
  return f2{__uint_as_float(r[0]), __uint_as_float(r[1])};
}
// Over the wave, in every lane, without LDS (an exchange through it costs some 60 ns, a sum of 64 lanes six of them).
__device__ __forceinline__ float wave_max(float v) {
  v = fmaxf(v, dpp<0xB1>(v));
  v = fmaxf(v, dpp<0x4E>(v));
  v = fmaxf(v, dpp<0x141>(v));             // row_half_mirror
  v = fmaxf(v, dpp<0x140>(v));             // row_mirror
  v = fmaxf(both16(v).x, both16(v).y);
  return fmaxf(both32(v).x, both32(v).y);
}
__device__ __forceinline__ float wave_sum(float v) {   // the order of sums of a tree over lanes 1, 2, 4, .. apart
  v = group_sum<16>(v);
  v = both16(v).x + both16(v).y;
  return both32(v).x + both32(v).y;
}

}  // namespace dev
}  // namespace ttkv
