// Workspace plans and device facts shared by the C ABI and the launchers (host
// code only).
#include <algorithm>
#include <atomic>

#include "gca_plan.hpp"

namespace gca {

int device_cus() {
  // one slot per device ordinal; 0 = not yet queried
  static std::atomic<int> cached[64];
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0) {
    (void)hipGetLastError();
    return 256;
  }
  if (dev < 64) {
    const int c = cached[dev].load(std::memory_order_relaxed);
    if (c > 0) return c;
  }
  int n = 0;
  if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n < 1) {
    (void)hipGetLastError();
    n = 256;
  }
  if (dev < 64) cached[dev].store(n, std::memory_order_relaxed);
  return n;
}

// ----------------------------------------------------------- decode ----

namespace {
constexpr int64_t kScanTarget = 256, kScanWaves = 4;
// Fewest keys per wave (never more for a longer past: see decode_workspace).  One group of
// 8 spreads a short past over the chip; for k > 8 merging the longer lists that this leaves
// can cost more than the scan gains.  64 / 8 keys, us a call: k = 32, 3,000 chunks 96 / 122;
// k = 12, per-head landmarks (width 64), 256 chunks 28 / 30, 768 30 / 33, 2,000 31 / 33,
// 6,000 34 / 34; k = 9, width 256, 128 chunks 25.7 / 26.9, 200 29.1 / 26.5; width 512, 64
// chunks 24.3 / 26.6, 100 26.8 / 26.5.  k <= 8 takes the same time or less with 8.
int64_t scan_floor(const Shape& s) {
  const int64_t key = (int64_t)s.D * (s.bf16 ? 2 : 4);
  const bool cheap = s.D <= 64 || s.nKV * key <= 64 * 1024;  // to scan
  return s.topk > 16 || (s.topk > 8 && cheap) ? 64 : 8;
}
}

DecodePlan decode_plan(const Shape& s) {
  // about 256 scan workgroups in all, every wave at least scan_floor keys
  const int64_t rows = (int64_t)s.B * s.Hr;
  int64_t wgs = kScanTarget / rows;
  if (wgs < 1) wgs = 1;
  int64_t pw = (s.nKV + wgs * kScanWaves - 1) / (wgs * kScanWaves);
  pw = std::max((pw + 7) & ~int64_t(7), scan_floor(s));
  DecodePlan p;
  p.pw = pw;
  p.wgs = ((s.nKV + pw - 1) / pw + kScanWaves - 1) / kScanWaves;
  p.lists = p.wgs * kScanWaves;  // a wave whose groups all lie past the keys leaves an empty list
  return p;
}

// Sized by the most lists that any past of up to nKV chunks needs, which grows with nKV
// (the plan's own count falls wherever pw steps up), so that one workspace sized for a
// program's longest past serves every shorter one.
size_t decode_workspace(const Shape& s) {
  const int64_t rows = (int64_t)s.B * s.Hr;
  const int64_t most = rows < kScanTarget ? kScanTarget / rows : 1;  // workgroups per row
  const int64_t least = kScanWaves * scan_floor(s);  // chunks of a workgroup but the last
  const int64_t wgs = std::min(most, (s.nKV + least - 1) / least);
  const size_t n = (size_t)(rows * wgs * kScanWaves) * s.topk;
  return align256(n * sizeof(float)) + align256(n * sizeof(int));
}
float* decode_list_scores(const Shape&, void* ws) { return reinterpret_cast<float*>(ws); }
int* decode_list_chunks(const Shape& s, void* ws) {
  const size_t n = (size_t)s.B * s.Hr * decode_plan(s).lists * s.topk;
  return reinterpret_cast<int*>(reinterpret_cast<char*>(ws) + align256(n * sizeof(float)));
}

// ----------------------------------------------------- fused select ----

SelectPlan select_plan(const Shape& s) {
  SelectPlan p{};
  // landmark queries stay in registers (bf16 up to 512 columns, fp32 up to 256) next
  // to each lane's best-16 list at most; wider ones are staged through LDS in tiles of
  // kWideTile keys
  const bool wide = s.bf16 ? s.D > 512 : s.D > 256;
  // Wide landmarks of few chunks stay with the one-pass form: their triangle is too few
  // tiles to split, and clearing and merging take two more launches.  A forward of width
  // 1,024, k = 4, one-pass / split: 1 x 64 chunks 31 / 48 us, 1 x 128 52 / 71, 1 x 200 80 /
  // 84, 1 x 256 92 / 88; 8 x 64 94 / 104, 8 x 128 189 / 196, 8 x 160 235 / 230, 8 x 256
  // 363 / 331; k = 16 and fp32 alike.
  const int64_t rows = (int64_t)s.B * s.Hr * s.nQ;
  p.split = s.causal && s.topk <= 16 && (!wide || s.nKV >= 256 || (s.nKV > 128 && rows >= 1024));
  p.blocks = (s.nQ + kSelRows - 1) / kSelRows;
  p.tile = wide ? kWideTile : kSelTile;
  p.tiles = (s.nKV + p.tile - 1) / p.tile;
  // tiles per part, a power of two.  Narrow: 2,048 keys.  Wide: 1,024 (a tile is twice
  // the work or more), and as many as it takes for a row's lists and threshold to fit
  // in the space of one query chunk of one head (their scratch is the output).
  p.tiles_per_part = wide ? 8 : 64;
  // the largest row block needs every key tile
  const int64_t per_class = (p.tiles + kSelClasses - 1) / kSelClasses;
  for (;; p.tiles_per_part *= 2) {
    p.parts_max = (per_class + p.tiles_per_part - 1) / p.tiles_per_part;
    if (p.parts_max < 1) p.parts_max = 1;
    p.lists = kSelClasses * p.parts_max;
    if (!wide || p.parts_max == 1 ||
        p.lists * s.topk * 8 + 64 <= (int64_t)kChunk * kChunk * (s.bf16 ? 2 : 4))
      break;
  }
  if (!p.split) return p;
  // items of one class: sum over row blocks of its parts there
  int64_t items = 0;
  for (int64_t r = 0; r < p.blocks; ++r) {
    // row block r reaches key chunks below its last row: tiles [0, nt)
    const int64_t last_row = (r + 1) * kSelRows - 1 < s.nQ - 1 ? (r + 1) * kSelRows - 1 : s.nQ - 1;
    int64_t nt = (last_row - 1) / p.tile + 1;  // key chunks j <= last_row - 1
    if (last_row < 1) nt = 0;
    if (nt > p.tiles) nt = p.tiles;
    const int64_t c0 = nt > 0 ? (nt + kSelClasses - 1) / kSelClasses : 0;  // class 0 has the most tiles
    items += (c0 + p.tiles_per_part - 1) / p.tiles_per_part;
  }
  p.items_per_class = items;
  return p;
}

namespace {
size_t select_bytes(const Shape& s, const SelectPlan& p) {
  const size_t n = (size_t)s.B * s.Hr * s.nQ * p.lists * s.topk;
  // the lists' scores and chunks, then one published threshold per row
  return align256(n * sizeof(float)) + align256(n * sizeof(int)) +
         align256(sizeof(uint32_t) * (size_t)s.B * s.Hr * s.nQ);
}
}  // namespace

size_t fused_workspace(const Shape& s) {
  const SelectPlan p = select_plan(s);
  return p.split && p.tile == kSelTile ? select_bytes(s, p) : 0;
}

size_t wide_select_bytes(const Shape& s) {
  const SelectPlan p = select_plan(s);
  return p.split && p.tile == kWideTile ? select_bytes(s, p) : 0;
}

// --------------------------------------------------------- backward ----

namespace {
struct Carver {
  char* p;
  size_t used = 0;
  template <typename X>
  X* take(size_t count) {
    X* r = reinterpret_cast<X*>(p ? p + used : nullptr);
    used += align256(sizeof(X) * count);
    return r;
  }
};

BwdWs carve(const Shape& s, Carver& c) {
  const size_t BHr = (size_t)s.B * s.Hr, BH = (size_t)s.B * s.H;
  BwdWs w;
  w.w = c.take<float>(BHr * s.nQ * s.topk);
  w.Dbuf = c.take<float>(BH * s.nQ * s.Sq * s.topk);
  w.Lbuf = c.take<float>(BH * s.nQ * s.Sq * s.topk);
  w.dwp = c.take<float>(BH * s.nQ * s.topk * 2);
  w.offs = c.take<int>(BHr * (s.nKV + 1));
  w.unsorted = c.take<int>(BHr * s.nQ * s.topk);
  w.sorted = c.take<int>(BHr * s.nQ * s.topk);
  w.head = c.take<int>(BHr * s.nKV * kHeadInts);
  return w;
}
}  // namespace

BwdWs bwd_carve(const Shape& s, void* base) {
  Carver c{reinterpret_cast<char*>(base)};
  return carve(s, c);
}

size_t bwd_workspace(const Shape& s) {
  Carver c{nullptr};
  carve(s, c);
  return c.used;
}

}  // namespace gca
