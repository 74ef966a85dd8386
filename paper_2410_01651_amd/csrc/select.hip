// Causal relevance scores and top-k without the score matrix (Eq. 1 of the
// method) for long sequences: the split select and its merge.
#include "gca_device.hpp"
#include "gca_launch.hpp"

#include <algorithm>
#include <type_traits>

namespace gca {
namespace {

// --------------------------------------- split causal select (no matrix) ----
//
// The work of a long causal selection is a triangle of (landmark row, key
// chunk) pairs.  It is cut into work items: a block of kSelRows rows against a
// part of the key tiles (kSelTile key chunks each) that the block reaches, the
// tiles of one item all of one class (tile index mod 8, one class per XCD, so
// that each XCD's L2 holds one eighth of the landmark keys).  Each item leaves
// the best k of its candidates for every one of its rows in the workspace, and
// a merge pass takes each row's best k over its lists: an exact top-k, since
// any member of a row's top k is among the best k of its own item.
//
// An item is one workgroup of 4 waves, two per CU; wave w owns 32 of the
// block's rows and keeps their landmark queries in registers as MFMA B operands
// (queries are the product's columns), so a lane holds, per 32-key tile, 16
// candidate scores of one row in registers and folds them into its own
// running best-k list; the two lanes of a row share their lists' thresholds
// once per tile, so that a candidate below the k-th best of either list is
// dropped with one compare.  Key tiles (32 keys x D columns) are staged in LDS
// by direct-to-LDS copies, two tiles deep.

template <typename T> struct SelMax;
template <> struct SelMax<__bf16> { static constexpr int kCh = 8; };  // D <= 512 in registers
template <> struct SelMax<float> { static constexpr int kCh = 4; };   // D <= 256
constexpr int kSelThreads = 256;
constexpr int kSelWaves = kSelThreads / 64;
static_assert(kSelWaves * 32 == kSelRows, "one 32-row column block per wave");

struct SelParams {
  uint32_t* gthr;  // per landmark row: the best published k-th score (order bits of a packed key), 0 = none
  int64_t nQ, nKV, tiles, blocks, items_per_class, parts_max, lists;
  int D, K, tile, tpp, tpp_shift;  // keys per tile; tiles per part, a power of two (parts need no division)
  float scale;
  uint64_t seed;
};

// Key tiles row block r reaches (key chunks below its last row).
__device__ __forceinline__ int64_t sel_block_tiles(const SelParams& p, int64_t r) {
  const int64_t last = min((r + 1) * kSelRows - 1, p.nQ - 1);
  if (last < 1) return 0;
  return min((last - 1) / p.tile + 1, p.tiles);
}
// Tiles of class x among the first nt; parts they form.
__device__ __forceinline__ int64_t sel_class_tiles(int64_t nt, int x) {
  return nt > x ? (nt - x + kSelClasses - 1) / kSelClasses : 0;
}

// Block -> (retrieval slice, class, row block, part): items of a class in order of
// descending row block, so the longest items start first.  False: no such item.
struct SelItem {
  int64_t bhr, r, part;
  int x, nu;  // class; tiles of the item
};
__device__ __forceinline__ bool sel_item(const SelParams& p, SelItem& it) {
  it.x = (int)(blockIdx.x % kSelClasses);
  const int64_t rest = blockIdx.x / kSelClasses;
  it.bhr = rest / p.items_per_class;
  int64_t i = rest % p.items_per_class;
  for (it.r = p.blocks - 1; it.r >= 0; --it.r) {
    const int64_t ncls = sel_class_tiles(sel_block_tiles(p, it.r), it.x);
    const int64_t np = (ncls + p.tpp - 1) >> p.tpp_shift;
    if (i < np) {
      it.part = i;
      it.nu = (int)min<int64_t>(p.tpp, ncls - i * p.tpp);
      return true;
    }
    i -= np;
  }
  return false;  // this class has fewer items
}

// The row's threshold: the better k-th best of its two lanes' lists and of what
// the row's other items have published (each is the score of a candidate beaten by
// k - 1 others, so a candidate below it cannot be in the row's top k).  This lane
// pair publishes its own with an atomic maximum, which returns the best published so
// far; a value read late is only a weaker filter, never a wrong one.  Split in two so
// that products can run while the atomic is away.
template <int KM>
__device__ __forceinline__ uint32_t sel_publish(const SelParams& p, const TopKeys<KM>& L, int64_t bhr, int64_t t,
                                                uint32_t& own) {
  uint32_t pa, pb;
  pair32((uint32_t)(L.k[KM - 1] >> 32), pa, pb);
  own = pa > pb ? pa : pb;
  uint32_t pub = 0u;
  if ((threadIdx.x & 32) == 0 && t < p.nQ && own != 0u)
    pub = __hip_atomic_fetch_max(p.gthr + bhr * p.nQ + t, own, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  return pub;
}
__device__ __forceinline__ float sel_threshold(uint32_t own, uint32_t pub) {
  uint32_t qa, qb;
  pair32(pub, qa, qb);
  const uint32_t hi = max(own, max(qa, qb));  // the best threshold's score bits
  return hi == 0u ? -kMaxFloat : key_score((uint64_t)hi << 32);
}

// Folds the 16 scores a lane holds of 32 keys from key0 (row t's, S^T in the
// accumulator layout: register i holds key 8 (i / 4) + 4 hh + i % 4; four consecutive
// keys per group of four registers, so one generator call gives their Gumbel noise)
// into its list.  The candidates are filtered against the threshold into a bit mask;
// then every lane inserts its surviving candidates one per round, so a round costs one
// insert for the wave however many rows have a survivor, and the wave runs as many
// rounds as its lane with the most survivors.  Only finite scores (with noise) are
// candidates: a threshold is never below the lowest finite value, which drops -inf and
// NaN in the filter, and +inf is dropped at its insertion.  full: every key is in range.
template <int KM, bool GUMBEL>
__device__ __forceinline__ void sel_fold(const SelParams& p, TopKeys<KM>& L, f32x16 a, int64_t key0, int64_t bhr,
                                         int64_t t, float ts, bool full) {
  const int hh = (threadIdx.x >> 5) & 1;
  uint32_t mask = 0u;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    const int64_t jg = key0 + 8 * g + 4 * hh;
    f32x4 nz = f32x4{0.f, 0.f, 0.f, 0.f};
    if constexpr (GUMBEL) nz = gumbel_noise4(p.seed, (uint32_t)bhr, (uint32_t)t, (uint32_t)(jg >> 2));
#pragma unroll
    for (int m = 0; m < 4; ++m) {
      a[4 * g + m] = a[4 * g + m] * p.scale + nz[m];
      mask |= (uint32_t)(a[4 * g + m] >= ts) << (4 * g + m);
    }
  }
  if (!full) {
    // keys at or past the row (and rows past the end) are not candidates
    const int64_t lim = t < p.nQ ? t - (key0 + 4 * hh) : 0;  // keys below the row, from this lane's first
    uint32_t okm = 0u;
#pragma unroll
    for (int i = 0; i < 16; ++i) okm |= (uint32_t)(8 * (i >> 2) + (i & 3) < lim) << i;
    mask &= okm;
  }
  while (__builtin_amdgcn_ballot_w64(mask != 0u)) {
    if (mask != 0u) {
      const int i = __builtin_ctz(mask);
      mask &= mask - 1u;
      // a[i] by a four-level select on the bits of i
      float v8[8], v4[4], v2[2];
#pragma unroll
      for (int e = 0; e < 8; ++e) v8[e] = (i & 1) ? a[2 * e + 1] : a[2 * e];
#pragma unroll
      for (int e = 0; e < 4; ++e) v4[e] = (i & 2) ? v8[2 * e + 1] : v8[2 * e];
#pragma unroll
      for (int e = 0; e < 2; ++e) v2[e] = (i & 4) ? v4[2 * e + 1] : v4[2 * e];
      const float v = (i & 8) ? v2[1] : v2[0];
      // (the empty key displaces nothing)
      L.insert(v <= kMaxFloat ? pack_key(v, (int)(key0 + 8 * (i >> 2) + 4 * hh + (i & 3))) : 0);
    }
  }
}

// The item's best k of row t: the partner lane's list entries inserted into this
// lane's (the two lanes hold disjoint keys, so the partner's entry is the one that
// differs from this lane's; equal entries are both empty), and stored.
template <int KM>
__device__ __forceinline__ void sel_store(const SelParams& p, TopKeys<KM>& L, const SelItem& it, int64_t t,
                                          float* __restrict__ ls, int* __restrict__ lj) {
  uint64_t pk[KM];
#pragma unroll
  for (int e = 0; e < KM; ++e) {
    uint32_t la, lb, ha, hb;
    pair32((uint32_t)L.k[e], la, lb);
    pair32((uint32_t)(L.k[e] >> 32), ha, hb);
    const bool own_first = la == (uint32_t)L.k[e] && ha == (uint32_t)(L.k[e] >> 32);
    pk[e] = own_first ? ((uint64_t)hb << 32 | lb) : ((uint64_t)ha << 32 | la);
  }
#pragma unroll
  for (int e = 0; e < KM; ++e)
    if (pk[e] != 0) L.insert(pk[e]);
  if ((threadIdx.x & 32) == 0 && t < p.nQ) {
    const int64_t o = ((it.bhr * p.nQ + t) * p.lists + it.x * p.parts_max + it.part) * p.K;
#pragma unroll
    for (int e = 0; e < KM; ++e) {
      if (e < p.K) {
        const bool real = L.k[e] != 0;
        ls[o + e] = real ? key_score(L.k[e]) : -INFINITY;
        lj[o + e] = real ? key_chunk(L.k[e]) : -1;
      }
    }
  }
}

// NCH: 64-column chunks of the landmark width (D / 64), a compile-time count so
// that the chunks' fragment reads and products form one straight schedule.
template <typename T, int KM, bool GUMBEL, int NCH>
__global__ __launch_bounds__(kSelThreads, 2) void select_part_kernel(const T* __restrict__ lq,
                                                                     const T* __restrict__ lk,
                                                                     float* __restrict__ ls, int* __restrict__ lj,
                                                                     SelParams p) {
  constexpr int TILE = kSelTile * kD;  // one 64-column chunk of a key tile
  static_assert(NCH >= 1 && NCH <= SelMax<T>::kCh, "landmark width held in registers");
  __shared__ __attribute__((aligned(16))) T stage[2 * NCH * TILE];

  SelItem it;
  if (!sel_item(p, it)) return;
  const int x = it.x, nu = it.nu;
  const int64_t bhr = it.bhr, r = it.r, part = it.part;
  auto tile_of = [&](int u) -> int64_t { return x + kSelClasses * (part * p.tpp + u); };

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t t0w = r * kSelRows + 32 * wave;  // this wave's first row
  const int64_t t = t0w + l32;                   // this lane's row
  const T* qrow = lq + (bhr * p.nQ + min(t, p.nQ - 1)) * p.D;
  Frag<T> qf[NCH][4];
#pragma unroll
  for (int c = 0; c < NCH; ++c)
#pragma unroll
    for (int kb = 0; kb < 4; ++kb)
      qf[c][kb] = load_frag(qrow + c * kD + 16 * kb + 8 * hh);

  // copies: every wave copies its share of each 32 x 64 chunk of a tile; the
  // last key tile may hold fewer than 32 keys (rows past it repeat the last)
  const TileCopy<T, kSelWaves, kSelTile> cp_full(wave, lane, p.D, kSelTile);
  const int last_rows = (int)(p.nKV - (p.tiles - 1) * kSelTile);
  const TileCopy<T, kSelWaves, kSelTile> cp_last(wave, lane, p.D, last_rows);
  const T* kbase = lk + bhr * p.nKV * p.D;
  auto issue = [&](int u) __device__ {
    const int64_t j = tile_of(u);
    const T* src = kbase + j * kSelTile * p.D;
    T* dst = stage + (u & 1) * NCH * TILE;
    const bool last = j == p.tiles - 1;
#pragma unroll
    for (int c = 0; c < NCH; ++c) {
      if (last) cp_last.issue(src + c * kD, dst + c * TILE);
      else cp_full.issue(src + c * kD, dst + c * TILE);
    }
  };

  TopKeys<KM> L;
  L.init();
  issue(0);
  for (int u = 0; u < nu; ++u) {
    wait_vmem<0>();
    block_barrier();  // tile u is in; every wave is done with the other slot
    if (u + 1 < nu) issue(u + 1);
    const int64_t j0 = tile_of(u) * kSelTile;  // first key chunk of the tile
    // wave-uniform: some (row, key) pair of this wave's block is a candidate
    if (j0 < t0w + 31 && t0w < p.nQ) {
      uint32_t own;
      const uint32_t pub = sel_publish(p, L, bhr, t, own);
      const T* sK = stage + (u & 1) * NCH * TILE;
      // S^T of the tile's 32 keys against the wave's 32 rows
      auto half_scores = [&](int key0) __device__ {
        f32x16 a = zero16();
#pragma unroll
        for (int c = 0; c < NCH; ++c)
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) mma32(a, lds_frag(sK + c * TILE, key0 + l32, 16 * kb + 8 * hh), qf[c][kb]);
        return a;
      };
      const f32x16 acc = half_scores(0);
      const float ts = sel_threshold(own, pub);
      // full tile: every key below every row of the wave (and inside the keys)
      const bool full = j0 + kSelTile <= t0w && j0 + kSelTile <= p.nKV && t0w + 31 < p.nQ;
      sel_fold<KM, GUMBEL>(p, L, acc, j0, bhr, t, ts, full);
    }
  }
  sel_store(p, L, it, t, ls, lj);
}

// Wide landmarks (their queries do not fit in registers): both operands go through
// LDS.  An item is again 128 rows against its class's key tiles, here of kWideTile
// keys; wave w owns 32 rows and computes S^T of all 128 keys against them, so a row's
// candidates stay in one wave's two lanes as above.  The landmark width is walked in
// 64-column chunks of both operands, two stages deep, the next chunk (the next tile's
// first included) in flight during the current one's products.
//
// Bound by the LDS: per chunk a wave reads 4 + 16 fragments for 16 products (2 waves
// per SIMD: about 1,250 LDS cycles against 1,024 of the matrix cores).  12,288 landmark
// rows of width 1,024: 2,370 us for the one-pass form (fused_select_kernel, 192
// workgroups there) -> 420 us (370 TFLOP/s) + 24 us for the merge.
template <typename T, int KM, bool GUMBEL>
__global__ __launch_bounds__(kSelThreads, 2) void select_wide_kernel(const T* __restrict__ lq,
                                                                     const T* __restrict__ lk,
                                                                     float* __restrict__ ls, int* __restrict__ lj,
                                                                     SelParams p) {
  constexpr int TILE = kS * kD;  // 64 rows of one 64-column chunk
  __shared__ __attribute__((aligned(16))) T stage[2 * 4 * TILE];  // per stage: rows 0-63, 64-127, keys 0-63, 64-127
  SelItem it;
  if (!sel_item(p, it)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int64_t r0 = it.r * kSelRows, t0w = r0 + 32 * wave;  // the block's and this wave's first row
  const int64_t t = t0w + l32;                               // this lane's row
  // rows and keys past the end repeat the last one (their scores are no candidates);
  // a 64-row half that does not exist at all copies the one before it
  auto half_of = [](int64_t first, int h, int64_t n) -> int64_t { return first + 64 * h < n ? first + 64 * h : first; };
  const int64_t q0 = half_of(r0, 0, p.nQ), q1 = half_of(r0, 1, p.nQ);
  const TileCopy<T, kSelWaves> cq0(wave, lane, p.D, (int)min<int64_t>(64, p.nQ - q0));
  const TileCopy<T, kSelWaves> cq1(wave, lane, p.D, (int)min<int64_t>(64, p.nQ - q1));
  const TileCopy<T, kSelWaves> cfull(wave, lane, p.D, 64);
  const int64_t klast = (p.tiles - 1) * kWideTile;
  const int64_t e0 = half_of(klast, 0, p.nKV), e1 = half_of(klast, 1, p.nKV);
  const TileCopy<T, kSelWaves> ce0(wave, lane, p.D, (int)min<int64_t>(64, p.nKV - e0));
  const TileCopy<T, kSelWaves> ce1(wave, lane, p.D, (int)min<int64_t>(64, p.nKV - e1));
  const T* const qbase = lq + it.bhr * p.nQ * p.D;
  const T* const kbase = lk + it.bhr * p.nKV * p.D;
  constexpr int kLoads = 4 * TileCopy<T, kSelWaves>::kN;  // one wave's copies of one chunk
  const int nch = p.D / kD;
  auto tile_of = [&](int u) -> int64_t { return it.x + kSelClasses * (it.part * p.tpp + u); };
  auto issue = [&](int u, int c, int st) __device__ {
    T* dst = stage + st * 4 * TILE;
    cq0.issue(qbase + q0 * p.D + c * kD, dst);
    cq1.issue(qbase + q1 * p.D + c * kD, dst + TILE);
    const int64_t j = tile_of(u);
    if (j == p.tiles - 1) {
      ce0.issue(kbase + e0 * p.D + c * kD, dst + 2 * TILE);
      ce1.issue(kbase + e1 * p.D + c * kD, dst + 3 * TILE);
    } else {
      cfull.issue(kbase + j * kWideTile * p.D + c * kD, dst + 2 * TILE);
      cfull.issue(kbase + (j * kWideTile + 64) * p.D + c * kD, dst + 3 * TILE);
    }
  };

  TopKeys<KM> L;
  L.init();
  int st = 0;
  issue(0, 0, 0);
  for (int u = 0; u < it.nu; ++u) {
    const int64_t j0 = tile_of(u) * kWideTile;  // first key chunk of the tile
    // wave-uniform: some (row, key) pair of this wave's block is a candidate
    const bool live = j0 < t0w + 31 && t0w < p.nQ;
    f32x16 acc[kWideTile / 32];
#pragma unroll
    for (int b = 0; b < kWideTile / 32; ++b) acc[b] = zero16();
    for (int c = 0; c < nch; ++c) {
      const bool more = c + 1 < nch || u + 1 < it.nu;
      if (more) {
        if (c + 1 < nch) issue(u, c + 1, st ^ 1);
        else issue(u + 1, 0, st ^ 1);
        wait_vmem<kLoads>();
      } else {
        wait_vmem<0>();
      }
      block_barrier();  // every wave's copies of this chunk are in
      if (live) {
        const T* sq = stage + st * 4 * TILE + (wave >> 1) * TILE;
        const T* sk = stage + st * 4 * TILE + 2 * TILE;
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          const Frag<T> qf = lds_frag(sq, 32 * (wave & 1) + l32, 16 * kb + 8 * hh);
#pragma unroll
          for (int b = 0; b < kWideTile / 32; ++b)
            mma32(acc[b], lds_frag(sk + (b >> 1) * TILE, 32 * (b & 1) + l32, 16 * kb + 8 * hh), qf);
        }
      }
      block_barrier();  // the stage is free for the copy issued in the next step
      st ^= 1;
    }
    if (live) {
      uint32_t own;
      const uint32_t pub = sel_publish(p, L, it.bhr, t, own);
      const float ts = sel_threshold(own, pub);
      const bool full = j0 + kWideTile <= t0w && j0 + kWideTile <= p.nKV && t0w + 31 < p.nQ;
#pragma unroll
      for (int b = 0; b < kWideTile / 32; ++b) sel_fold<KM, GUMBEL>(p, L, acc[b], j0 + 32 * b, it.bhr, t, ts, full);
    }
  }
  sel_store(p, L, it, t, ls, lj);
}

__global__ void sel_clear_kernel(uint32_t* __restrict__ p, int64_t n) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < n; i += (int64_t)gridDim.x * blockDim.x)
    p[i] = 0u;
}

// One wave per landmark row: the best k over the row's lists, written in
// ascending chunk order (GUMBEL: the lists rank noisy scores; sel gets the
// chosen chunks' raw scores, recomputed from the landmark rows).
template <typename T, int KM, bool GUMBEL>
__global__ __launch_bounds__(256) void select_merge_kernel(const float* __restrict__ ls, const int* __restrict__ lj,
                                                           int32_t* __restrict__ idx, float* __restrict__ sel,
                                                           const T* __restrict__ lq, const T* __restrict__ lk,
                                                           int64_t rows, SelParams p) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (row >= rows) return;
  const int64_t t = row % p.nQ, bhr = row / p.nQ;
  const int64_t nt = sel_block_tiles(p, t / kSelRows);
  TopList<KM> L;
  L.init();
  const int64_t base = row * p.lists * p.K;
  // entry e of the row: class e / (parts_max K), part, rank
  const int64_t per_class = p.parts_max * p.K;
  for (int64_t e = lane; e < p.lists * p.K; e += 64) {
    const int x = (int)(e / per_class);
    const int64_t in_class = e % per_class;
    const int64_t parts = (sel_class_tiles(nt, x) + p.tpp - 1) >> p.tpp_shift;
    if (in_class / p.K < parts) {
      const int jj = lj[base + e];
      if (jj >= 0) L.insert(ls[base + e], jj);
    }
  }
  float ms;
  int mj, cnt;
  wave_merge(L, p.K, ms, mj, cnt);
  if constexpr (GUMBEL) {
    if (lane < cnt) ms = p.scale * dot_rows(lq + (bhr * p.nQ + t) * p.D, lk + (bhr * p.nKV + mj) * p.D, p.D);
  }
  const int rank = rank_by_chunk(mj, cnt);
  int32_t* io = idx + row * p.K;
  float* so = sel + row * p.K;
  if (lane < cnt) {
    io[rank] = mj;
    so[rank] = ms;
  } else if (lane < p.K) {
    io[lane] = -1;
    so[lane] = -INFINITY;
  }
}

// NCH: landmark chunks held in registers (select_part_kernel); 0: select_wide_kernel.
template <typename T, int KM, bool GUMBEL, int NCH>
hipError_t launch_split_select_n(const Shape& s, const void* lq, const void* lk, int32_t* idx, float* sel, void* ws,
                               hipStream_t st) {
  const SelectPlan plan = select_plan(s);
  SelParams p;
  p.nQ = s.nQ;
  p.nKV = s.nKV;
  p.tiles = plan.tiles;
  p.blocks = plan.blocks;
  p.items_per_class = plan.items_per_class;
  p.parts_max = plan.parts_max;
  p.lists = plan.lists;
  p.D = s.D;
  p.K = s.topk;
  p.tile = plan.tile;
  p.tpp = plan.tiles_per_part;
  p.tpp_shift = __builtin_ctz((unsigned)plan.tiles_per_part);
  p.scale = s.score_scale;
  p.seed = s.gumbel_seed;
  const int64_t BHr = (int64_t)s.B * s.Hr;
  const size_t n = (size_t)BHr * s.nQ * plan.lists * s.topk;
  float* ls = reinterpret_cast<float*>(ws);
  int* lj = reinterpret_cast<int*>(reinterpret_cast<char*>(ws) + align256(n * sizeof(float)));
  p.gthr = reinterpret_cast<uint32_t*>(reinterpret_cast<char*>(ws) + 2 * align256(n * sizeof(float)));
  const int64_t nrows = BHr * s.nQ;
  launch_kernel("sel_clear_kernel", sel_clear_kernel, dim3((unsigned)std::min<int64_t>((nrows + 255) / 256, 1024)),
                dim3(256), 0, st, p.gthr, nrows);
  const int64_t items = BHr * kSelClasses * plan.items_per_class;
  if (items > 0) {
    if constexpr (NCH > 0)
      launch_kernel("select_part_kernel", select_part_kernel<T, KM, GUMBEL, NCH>, dim3((unsigned)items),
                    dim3(kSelThreads), 0, st, (const T*)lq, (const T*)lk, ls, lj, p);
    else
      launch_kernel("select_wide_kernel", select_wide_kernel<T, KM, GUMBEL>, dim3((unsigned)items),
                    dim3(kSelThreads), 0, st, (const T*)lq, (const T*)lk, ls, lj, p);
  }
  const int64_t rows = BHr * s.nQ;
  launch_kernel("select_merge_kernel", select_merge_kernel<T, KM, GUMBEL>, dim3((unsigned)((rows + 3) / 4)),
                dim3(256), 0, st, ls, lj, idx, sel, (const T*)lq, (const T*)lk, rows, p);
  return take_launch_error();
}

template <typename T, int KM, bool GUMBEL>
hipError_t launch_split_select(const Shape& s, const void* lq, const void* lk, int32_t* idx, float* sel, void* ws,
                               hipStream_t st) {
  if (select_plan(s).tile == kWideTile) return launch_split_select_n<T, KM, GUMBEL, 0>(s, lq, lk, idx, sel, ws, st);
  switch (s.D / kD) {
    case 1: return launch_split_select_n<T, KM, GUMBEL, 1>(s, lq, lk, idx, sel, ws, st);
    case 2: return launch_split_select_n<T, KM, GUMBEL, 2>(s, lq, lk, idx, sel, ws, st);
    case 3: return launch_split_select_n<T, KM, GUMBEL, 3>(s, lq, lk, idx, sel, ws, st);
    case 4: return launch_split_select_n<T, KM, GUMBEL, 4>(s, lq, lk, idx, sel, ws, st);
    default: break;
  }
  if constexpr (SelMax<T>::kCh > 4) {
    switch (s.D / kD) {
      case 5: return launch_split_select_n<T, KM, GUMBEL, 5>(s, lq, lk, idx, sel, ws, st);
      case 6: return launch_split_select_n<T, KM, GUMBEL, 6>(s, lq, lk, idx, sel, ws, st);
      case 7: return launch_split_select_n<T, KM, GUMBEL, 7>(s, lq, lk, idx, sel, ws, st);
      case 8: return launch_split_select_n<T, KM, GUMBEL, 8>(s, lq, lk, idx, sel, ws, st);
      default: break;
    }
  }
  return hipErrorInvalidValue;  // the plan keeps wider landmarks off this path
}

}  // namespace

hipError_t launch_fused_select(const Shape& s, const void* lmk_q, const void* lmk_k, int32_t* idx, float* sel,
                               void* ws, hipStream_t stream) {
  if (!select_plan(s).split || !ws) return launch_fused_rowblocks(s, lmk_q, lmk_k, idx, sel, stream);
  auto run = [&](auto tag, auto gumbel) {
    using T = decltype(tag);
    constexpr bool G = decltype(gumbel)::value;
    if (s.topk <= 8) return launch_split_select<T, 8, G>(s, lmk_q, lmk_k, idx, sel, ws, stream);
    return launch_split_select<T, 16, G>(s, lmk_q, lmk_k, idx, sel, ws, stream);
  };
  if (s.bf16) return s.gumbel ? run(__bf16{}, std::true_type{}) : run(__bf16{}, std::false_type{});
  return s.gumbel ? run(float{}, std::true_type{}) : run(float{}, std::false_type{});
}

}  // namespace gca
