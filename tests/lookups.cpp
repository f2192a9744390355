// The attention kernels' index arithmetic (token -> ring block, workgroup -> item and KV head, item -> run) against plain
// divisions and a linear search.  Prints nothing and returns 0, or names the first disagreement.
#include "ttkv_internal.h"

#include <cstdio>
#include <cstring>
#include <random>

using namespace ttkv;

static int fail(const char *what, long a, long b, long c) {
  printf("%s: %ld %ld %ld\n", what, a, b, c);
  return 1;
}

// every token next to a block boundary, at the ends of the ring and a few thousand others
static int division(int64_t ring_blocks, int bt, std::mt19937_64 &g, bool *by_product) {
  const int64_t ring = ring_blocks * bt;
  const uint32_t magic = magic_bt(ring, bt);
  *by_product = magic != 0;
  auto check = [&](int64_t tok) { return tok < 0 || tok >= ring || div_bt((int)tok, bt, magic) == (int)(tok / bt); };
  for (int i = 0; i < 4000; ++i) {
    const int64_t b = i < 64 ? i : i < 128 ? ring_blocks - 1 - (i - 64) : (int64_t)(g() % (uint64_t)ring_blocks);
    for (int64_t tok : {b * bt - 1, b * bt, b * bt + 1, b * bt + bt - 64, b * bt + bt - 1})
      if (!check(tok)) return fail("div_bt", (long)tok, bt, (long)ring_blocks);
  }
  for (int i = 0; i < 4000; ++i)
    if (!check((int64_t)(g() % (uint64_t)ring))) return fail("div_bt", i, bt, (long)ring_blocks);
  return 0;
}

static int divisions() {
  std::mt19937_64 g(1976970);
  for (int bt : {64, 128, 192, 256, 320, 448, 512, 576, 1024, 1088, 4160, 8192, 8256, 65536, 131072, 1000000 / 64 * 64}) {
    const int64_t most = INT32_MAX / bt, d = bt / 64;
    // the product is used while (ring / 64 + 1) d < 2^31, i.e. below about 2^31 / d^2 blocks: both sides of that bound
    const int64_t bound = ((1ll << 31) / d - 1) / d;
    bool yes = false, last = false, beyond = true;
    for (int64_t n : {(int64_t)1, (int64_t)2, (int64_t)3, (int64_t)97, (int64_t)1024, most / 3, most - 1, most})
      if (n >= 1 && n <= most && division(n, bt, g, &yes)) return 1;
    if (bound >= 1 && bound <= most) {
      int64_t n = bound;
      while (n > 1 && !magic_bt(n * bt, bt)) --n;
      if (division(n, bt, g, &last)) return 1;
      if (!last) return fail("no product below its bound", bt, (long)n, 0);
      if (n + 2 <= most) {
        if (division(n + 2, bt, g, &beyond)) return 1;
        if (beyond) return fail("a product beyond its bound", bt, (long)n, 0);
      }
    }
  }
  if (magic_bt(1 << 20, 96) != 0) return fail("a block size that is no multiple of 64", 96, 0, 0);
  return 0;
}

static int heads() {
  static FusedArgs a;
  std::mt19937_64 g(1976971);
  for (int hkv = 1; hkv <= TTKV_MAX_KV_HEADS; hkv = hkv < 70 ? hkv + 1 : hkv + 13) {
    const int64_t bound = (1ll << 31) / ((int64_t)hkv * hkv);
    for (int64_t items : {(int64_t)1, (int64_t)2, (int64_t)777, bound - 1, bound, bound + 1, (int64_t)INT32_MAX / hkv}) {
      if (items < 1 || items > INT32_MAX / hkv) continue;
      memset(&a, 0, sizeof a);
      a.Hkv = hkv;
      a.Hq = 2 * hkv;
      set_items(a, 1, (int)items);
      if (a.G != 2) return fail("G", hkv, a.G, 0);
      if (hkv > 1 && items < bound && !a.hkv_magic) return fail("no product below its bound", hkv, (long)items, 0);
      for (int i = 0; i < 600; ++i) {
        const int64_t item = i < 100 ? i : i < 200 ? items - 1 - (i - 100) : (int64_t)(g() % (uint64_t)items);
        if (item < 0 || item >= items) continue;
        for (int h : {0, hkv / 2, hkv - 1})
          if (item_of(a, (uint32_t)(item * hkv + h)) != item) return fail("item_of", (long)item, hkv, (long)items);
      }
    }
  }
  return 0;
}

static int runs() {
  static FusedArgs a;
  std::mt19937_64 g(1976972);
  for (int n : {1, 2, 14, 15, 16, 17, 31, 32, 33, 63, 64, 65, 111, 112, 113, 128, 192, 193, 207, 208})
    for (int most : {1, 3, 40}) {
      memset(&a, 0xee, sizeof a);   // whatever an earlier launch left behind
      a.Hkv = 4;
      a.Hq = 4;
      int items = 0, owner[208 * 40];
      for (int r = 0; r < n; ++r) {
        a.start[r] = items;
        for (int k = 1 + (int)(g() % most); k; --k) owner[items++] = r;
      }
      set_items(a, n, items);
      for (int i = 0; i < items; ++i)
        if (find_run(a, i) != owner[i]) return fail("find_run", n, i, find_run(a, i));
    }
  return 0;
}

// the merge's threads per row: whole waves, and a launch of fewer than 2^32 threads as far as 256 of them allow
static int merges() {
  for (int parts : {0, 1, 32, 33, 64, 65, 191, 192, 256, 1 << 20})
    for (int rows : {1, 256, 257, (1 << 22) - 1, 1 << 22, (1 << 24) - 1}) {
      const int t = merge_threads(parts, rows);
      if ((t != 128 && t != 256 && t != 1024) || (uint64_t)t * (uint64_t)rows >> 32) return fail("merge_threads", parts, rows, t);
    }
  return 0;
}

int main() { return divisions() || heads() || runs() || merges(); }
