// Internal declarations shared by the translation units of libttkv (gfx950 only).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>
#include <stdlib.h>

#include <vector>

#include "ttkv.h"
#include "ttkv_bench.h"

namespace ttkv {

// ---------------------------------------------------------------- layout
// Per token-head byte counts of one format (K or V alone).
struct FmtBytes {
  int code, meta;
};
inline FmtBytes fmt_bytes(int fmt) {
  switch (fmt) {
    case TTKV_F16:
    case TTKV_BF16: return {256, 0};
    case TTKV_I8_SYM_G32: return {128, 8};
    case TTKV_I4_ASYM_G64:
    case TTKV_I4_ASYM_G64_T32: return {64, 8};
    case TTKV_I4_ASYM_T128: return {64, 4};   // 128 tokens x 4 B = 128 channels x fp16 {scale, zero}
    default: return {0, 0};
  }
}

// Byte geometry of one block record of a tier (see the header's "Block record").
struct Layout {
  int32_t bt;          // tokens per record
  int32_t kc, km, vc, vm;
  int32_t k_meta_off;  // offsets inside one head part
  int32_t v_off, v_meta_off;
  int32_t head_bytes;
  int64_t rec_bytes;
};
inline Layout make_layout(const ttkv_tier &t, int n_kv_heads) {
  Layout L{};
  FmtBytes k = fmt_bytes(t.k_fmt), v = fmt_bytes(t.v_fmt);
  L.bt = t.block_tokens;
  L.kc = k.code; L.km = k.meta; L.vc = v.code; L.vm = v.meta;
  L.k_meta_off = L.bt * L.kc;
  L.v_off = L.k_meta_off + L.bt * L.km;
  L.v_meta_off = L.v_off + L.bt * L.vc;
  L.head_bytes = L.v_meta_off + L.bt * L.vm;
  L.rec_bytes = (int64_t)L.head_bytes * n_kv_heads;
  return L;
}

// What a kernel needs to find a token of a tier (or of a staging slot that holds
// a few consecutive records of it).
struct TierView {
  uint8_t *base;          // record pool (device) or staging slot
  const int32_t *table;   // device block table or nullptr
  int64_t rec_bytes;
  int32_t head_bytes, k_meta_off, v_off, v_meta_off;
  int32_t bt, ring_blocks;
  int32_t k_fmt, v_fmt;
  int32_t in_host;        // the records are pinned host memory, read over PCIe
  uint32_t bt_magic;      // ring tokens / bt by a multiplication (div_bt); 0: by a division
};
// A division by the block size (a multiple of 64) for every look-up of a token costs some 25 instructions and a chain of
// latencies: x / d = (x ceil(2^31 / d)) >> 31 exactly as long as x d < 2^31, with x = token / 64 and d = bt / 64.
inline uint32_t magic_bt(int64_t ring_tokens, int32_t bt) {
  const int64_t d = bt / 64;
  return bt % 64 == 0 && d > 0 && (ring_tokens / 64 + 1) * d < (1ll << 31) ? (uint32_t)(((1ll << 31) + d - 1) / d) : 0;
}
__host__ __device__ inline uint32_t mul_high(uint32_t x, uint32_t y) { return (uint32_t)(((uint64_t)x * y) >> 32); }
__host__ __device__ inline int div_bt(int tok, int bt, uint32_t magic) {
  return magic ? (int)mul_high((uint32_t)tok >> 6 << 1, magic) : tok / bt;
}

// ---------------------------------------------------------------- the split-K plan of one attention call
// One run of consecutive tokens of one (tier, sequence) attended by the fused
// kernel in place: a device tier, a host tier read over PCIe by the kernel itself,
// or a run of selected blocks.
struct Run {
  int tier, b;
  int32_t rec_base;   // no_table: first pool record
  int32_t first_tok, len;
  bool no_table;
  bool selected;   // blocks named by the device-side selection (first_tok: newest block id; len: their number for a host
                   // tier, their tokens for a tier in HBM)
  int part_base, n_chunks;
  int64_t item_bytes;   // of one of its items (one KV head)
};
// Selection left on the device by the top-k kernel: ids [batch][stride], min(k, live blocks) of them per sequence.
struct DevSel {
  const int32_t *ids;
  int32_t k, stride;
  int32_t *host_ids, *host_count;   // nullable: where the attention launch stores them for the caller
};
// One staged copy: consecutive pool records of a host tier brought into a slot.
struct Fetch {
  int tier, b;
  int64_t rec;     // first pool record
  int nrec;        // consecutive records in this copy
  int ntok;        // live tokens covered
  int part_base;
  int chunk;
};
// Lives in the handle and is rebuilt by every call: the vectors keep their storage, so a call allocates host
// memory only when its plan is larger than any before it (ttkv_create reserves TTKV_PLAN_RESERVE entries).
#define TTKV_PLAN_RESERVE 4096
// What the search for the split-K item size settled on, kept while the cache keeps its shape.
struct SplitMemo {
  bool valid;
  uint32_t sig;      // tiers, formats, head counts, batch, slots and shortest items planned with
  int n_runs;
  int step;          // index into the table of rounds
  int64_t bytes;     // bytes of one pass over one KV head when it was chosen
};
struct Plan {
  SplitMemo memo[2];   // of the plans over everything, and of those with a device-side selection
  std::vector<Run> runs;
  std::vector<Fetch> fetch;
  std::vector<const Run *> order;   // launch order of `runs`
  int chunk[TTKV_MAX_TIERS];
  bool even[TTKV_MAX_TIERS];   // the tier's runs are cut into items of equal size each (chunk[] is then the size aimed at)
  int parts[TTKV_MAX_BATCH];
  int max_parts;
  int resident_items;   // the kernel's default split (default_items)
  bool few;             // some runs may be in items of 128 tokens (finest_item)
  size_t slot_bytes;
  ttkv_status status;
};

// ---------------------------------------------------------------- handle
struct Handle {
  Plan plan;
  int device;
  bool have_events;
  hipEvent_t ready[TTKV_MAX_SLOTS];
  hipEvent_t freed[TTKV_MAX_SLOTS];
  hipEvent_t fence;     // orders the copy stream behind earlier compute work
  hipEvent_t fence2;    // orders device->host eviction copies behind the quantize kernel
  ttkv_stats stats;
  // optional per-call timing of one device tier's partial kernel
  bool time_on;
  int target_items;     // split-K granularity of the fused launch
  bool check_tables;    // every call checks every host block-table entry against pool_blocks
  int time_max, time_n;
  hipEvent_t *time_ev;  // 2 * time_max events
  int32_t *time_reps;   // launches between the events of each sample
  int time_repeat;      // how often a timed call issues its attention launch(es)
};

#define TTKV_HIP(h, expr)                                   \
  do {                                                      \
    hipError_t e_ = (expr);                                 \
    if (e_ != hipSuccess) {                                 \
      if (h) (h)->stats.last_hip_error = (int32_t)e_;       \
      return TTKV_ERR_HIP;                                  \
    }                                                       \
  } while (0)

inline bool is_fp(int f) { return f == TTKV_F16 || f == TTKV_BF16; }
inline bool is_tier_fmt(int f) {
  return (f >= TTKV_F16 && f <= TTKV_I4_ASYM_G64) || f == TTKV_I4_ASYM_T128 || f == TTKV_I4_ASYM_G64_T32;
}

ttkv_status validate_cache(const ttkv_cache *c, bool check_tables = true);

// ---------------------------------------------------------------- launchers (defined in the .hip files)
struct ConvSource {
  // flat source [n_seq][Hkv][n][128] indexed by launch entry, or a tier view
  const void *k_flat, *v_flat;
  int32_t flat_fmt;
  int32_t from_tier;    // 0: flat source, 1: read rows of `src`
  TierView src;
  int32_t src_first_tok[TTKV_MAX_BATCH];  // ring token index of the first row to read, per entry
  int32_t src_rec_base[TTKV_MAX_BATCH];
};
struct ConvArgs {
  ConvSource s;
  TierView dst;
  int32_t n_seq, Hkv, n_tokens;            // rows per entry and head
  int32_t seq_id[TTKV_MAX_BATCH];
  int32_t dst_first_tok[TTKV_MAX_BATCH];   // ring token index where the first row lands
  int32_t dst_rec_base[TTKV_MAX_BATCH];
  int32_t to_host;                         // the rows belong to a pinned tier: stored there directly, or copied from staging records
  int32_t n_via;                           // intermediate formats a value passes through first
  uint32_t via_k, via_v;                   // 8 bits each, the first in the low ones
  // summaries of the destination tier (nullable)
  float *k_sum;
  uint16_t *k_summary;
  // (their ring is the tier's own, also where the rows themselves go to staging records)
  const int32_t *sum_table;                // device block table of the destination pool for the summaries
  int32_t sum_first_block[TTKV_MAX_BATCH]; // ring block of the first row
  int32_t sum_ring_blocks;
  float inv_bt;
};
hipError_t launch_convert(const ConvArgs &a, hipStream_t s, int *n_kernels);
// Two conversions of which neither reads what the other writes, in one launch where that pays; else one after the other.
hipError_t launch_convert_pair(const ConvArgs &a, const ConvArgs &b, hipStream_t s, int *n_kernels);

// One launch of the fused attention kernel: up to TTKV_MAX_ENTRIES runs of tokens,
// each belonging to one (tier, sequence), all passed by value (no per-step upload).  16 bytes per run, so that one
// launch takes three tiers of 64 sequences: with 24 (120 runs) the 128 runs of 64 sequences in two tiers made two
// launches, the second one nearly empty (64 x 4K tokens: 118.3 us per step, 110.3 in one launch).
#define TTKV_MAX_ENTRIES 208
struct Entry {
  // bits 0-19 first partial index of the run, 20-25 sequence, 26-27 tier, 28: the run names pool records directly
  // (no block table), 29: it is made of blocks named by the device-side selection
  uint32_t head;
  int32_t at;           // ring token index of the run's first token (multiple of 64); bit 28: its first pool record;
                        // bit 29: id of the tier's newest live block
  int32_t len;          // tokens; bit 29: the number of blocks (tier cut into fixed items) or their tokens (equal items)
};
constexpr uint32_t kEntryNoTable = 1u << 28, kEntrySelected = 1u << 29;
inline Entry make_entry(int tier, int seq, int part_base, uint32_t flags, int32_t at, int32_t len) {
  return Entry{(uint32_t)part_base | (uint32_t)seq << 20 | (uint32_t)tier << 26 | flags, at, len};
}
__host__ __device__ inline int entry_tier(const Entry &e) { return (e.head >> 26) & 3; }
static_assert(TTKV_MAX_BATCH <= 64 && TTKV_MAX_TIERS <= 4, "an entry's sequence and tier fields");
#define TTKV_MAX_PARTS (1 << 20)
// A run of `len` tokens cut into n items of equal size, a multiple of 64 tokens (the last item may be shorter).
// The host plans with it and the kernels derive an item's size from the run's length and item count with it.
__host__ __device__ inline int even_chunk(int len, int n) { return ((len + n - 1) / n + 63) / 64 * 64; }
struct FusedArgs {
  // what every workgroup reads first, in one line
  int32_t n_entries, n_items;
  int32_t Hq, Hkv;
  int32_t G;               // query heads per KV head
  int32_t mfma_heads;      // set by the matrix-core launcher: query heads one workgroup serves
  uint32_t hkv_magic;      // workgroup / Hkv by a multiplication; 0: by a division
  int32_t part_stride;
  const void *q;
  float *pm, *pl, *pacc;
  // First work item (chunk) of each run in this launch, INT32_MAX behind the last one, and of every sixteenth run: an item
  // finds its run by one or two loads of 64 bytes whatever their number (a binary search is a chain of up to seven).
  int32_t start[TTKV_MAX_ENTRIES], coarse[TTKV_MAX_ENTRIES / 16];
  int32_t q_fmt;
  float scale;
  int32_t sel_stride;
  TierView tv[TTKV_MAX_TIERS];
  int32_t chunk[TTKV_MAX_TIERS];   // tokens per item of the tier's runs; 0: every run in items of equal size (even_chunk)
  Entry e[TTKV_MAX_ENTRIES];
  const int32_t *sel_ids;                    // device: block ids (Eq. 1) chosen by the top-k kernel [batch][sel_stride], for selected runs
  int32_t sel_last_ntok[TTKV_MAX_BATCH];     // live tokens in the newest block of the selected tier, per sequence
  int32_t *host_ids, *host_count;            // nullable: the caller's copies of them in pinned memory ([batch][sel_stride], [batch])
};
static_assert(sizeof(FusedArgs) <= 4096, "kernel arguments are passed by value");
static_assert(TTKV_MAX_ENTRIES % 16 == 0, "coarse");
void set_items(FusedArgs &a, int n_entries, int n_items);   // the look-up tables behind `start`
// The run that holds an item: start <= item < next run's.
__host__ __device__ inline int find_run(const FusedArgs &a, int item) {
  int seg = 0;
  if (a.n_entries > 16) {
#pragma unroll
    for (int k = 1; k < TTKV_MAX_ENTRIES / 16; ++k) seg += a.coarse[k] <= item;
  }
  const int32_t *s = a.start + 16 * seg;
  int lo = 16 * seg - 1;
#pragma unroll
  for (int k = 0; k < 16; ++k) lo += s[k] <= item;
  return lo;
}
// Workgroup -> (item, KV head).
__host__ __device__ inline int item_of(const FusedArgs &a, uint32_t base) {
  if (a.Hkv == 1) return base;
  return a.hkv_magic ? (int)mul_high(base, a.hkv_magic) : (int)(base / (uint32_t)a.Hkv);
}
hipError_t launch_attn(const FusedArgs &a, hipStream_t s, int *n_kernels, int *n_mfma);
bool attn_supported(int k_fmt, int v_fmt, int G);
int attn_group_width(int Gtot);
// Grouped-query kernel on the matrix cores: all query heads of a KV head in one pass over its bytes.
bool attn_mfma_fits(int k_fmt, int v_fmt, int G);
bool attn_mfma_four_bit(int k_fmt, int v_fmt);
bool attn_mfma_eligible(const FusedArgs &a);
hipError_t launch_attn_mfma(const FusedArgs &a, hipStream_t s);

struct MergeArgs {
  const float *m, *l, *acc;
  int32_t n_parts, part_stride, rows;
  int32_t rows_per_seq;         // > 0: cnt[sequence] parts per row (the rows of a sequence lie together), 0: cnt[0] in every row
  const int32_t *n_parts_row;   // device, nullable: parts of each row
  float *out, *lse;
  // The step's new token (k_new nullable; then rows = batch x Hq): its term (score q.k_new, weight 1, value
  // v_new) joins the merge, and its row is stored at the tail of tier 0, whose fp format it has.
  const void *q, *k_new, *v_new;   // q [batch][Hq][128]; k_new, v_new [batch][Hkv][128]
  int32_t q_fmt, new_fmt, G, Hkv;  // G: query heads per KV head
  uint32_t g_magic;                // head / G by a multiplication; 0: by a division
  float scale;
  TierView dst;                    // tier 0
  int32_t cnt[TTKV_MAX_BATCH];
  int32_t new_block[TTKV_MAX_BATCH], new_row[TTKV_MAX_BATCH];   // ring block and row in it where the sequence's row lands
};
// head / G = mul_high(head, magic_heads) as long as head G < 2^32; 0: by a division.
inline uint32_t magic_heads(int32_t Hq, int32_t G) { return G > 1 && (int64_t)Hq * G < (1ll << 32) ? (uint32_t)(((1ll << 32) + G - 1) / G) : 0; }
// Threads per row of the merge (merge_kernel); a launch holds fewer than 2^32 threads.
inline int merge_threads(int32_t n_parts, int32_t rows) {
  if (n_parts <= 32) return 128;
  if (n_parts <= 64 || rows >= 1 << 22) return 256;
  return n_parts < 192 && rows > 256 ? 256 : 1024;
}
hipError_t launch_merge(const MergeArgs &a, hipStream_t s);

struct SelectArgs {
  const void *q;
  int32_t q_fmt;
  const uint16_t *k_summary;
  const int32_t *table;          // device block table of the last tier or nullptr
  int32_t ring_blocks, Hq, Hkv, k, sel_stride, n_seq;
  int32_t G;                     // query heads per KV head
  uint32_t g_magic;              // head / G by a multiplication; 0: by a division
  int32_t rec_base[TTKV_MAX_BATCH];
  int32_t first_block[TTKV_MAX_BATCH];   // ring index of the oldest live block
  int64_t first_block_id[TTKV_MAX_BATCH];  // its block id (Eq. 1)
  int32_t n_blocks[TTKV_MAX_BATCH];
  int32_t max_blocks;
  float *scores;                 // [n_seq][max_blocks]
  int32_t *sel_out;              // [n_seq][sel_stride + 1]: count then ids relative to first_block_id
};
hipError_t launch_select(const SelectArgs &a, hipStream_t s);

// Load-only kernel over `bytes` (rounded down to 64 KiB) of device memory; sink: 4 writable bytes.
hipError_t launch_stream_read(const void *src, int64_t bytes, uint32_t *sink, hipStream_t s);

}  // namespace ttkv
