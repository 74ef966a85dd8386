// Backward of grouped cross attention (Algorithm 2 of the method's appendix)
// and of the retrieval scores (Eq. 2) and landmark vectors (Eq. 1).
//
// With P_s = softmax of one (query chunk, retrieved chunk j) tile, recomputed
// from the saved log-sum-exp, dP_s = dO V_j^T, D_s = rowsum(P_s o dP_s) and
// dS_s = w_s P_s o (dP_s - D_s):
//   dQ_c  += scale * dS_s K_j           (query-stationary kernel)
//   dV_j  += (w_s P_s)^T dO_c           (key-stationary kernel)
//   dK_j  += scale * dS_s^T Q_c         (key-stationary kernel)
//   dw[t,s] = sum over the group's heads and the chunk's rows of D_s
// D_s equals rowsum(dO o O'_s) of Algorithm 2, computed here on chip from the
// same tile, so the per-chunk outputs O'_s are never stored.
//
// With an LMK row per chunk (S + 1 query rows against S-row key chunks) the
// 65th row takes the same steps as a vector against the tiles the waves hold:
// in the query-stationary pass one wave per slot (alternating) forms its
// scores, dP, D and dS with one key per lane and accumulates its dQ row, and
// in the key-stationary pass every wave adds the row's rank-one terms to dV and
// dK with one more, mostly zero, 16-deep MFMA step.
//
// No floating-point atomics: every output element is produced by exactly one
// workgroup.  The key-stationary pass needs, for each chunk j, the list of
// (row t, slot s) that retrieved it, in (t, s) order (bwd_prep_kernel), so the
// summation order, and hence the result, is the same on every run.
#include "gca_device.hpp"
#include "gca_launch.hpp"

#include <algorithm>
#include <type_traits>

namespace gca {
namespace {

// query-stationary pass: wave pairs per workgroup (one, so that a round's
// barrier couples only the two waves sharing a ring), four workgroups per CU
constexpr int kPairs = 1;
constexpr int kThreads = 128 * kPairs;
constexpr int kWgPerCu = 4 / kPairs;

struct BwdParams {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* idx;
  const float* sel;
  const float* lse;
  const void* dout;
  void* dq;
  void* dk;
  void* dv;
  BwdWs ws;
  int B, H, Hr, K;
  int64_t nQ, nKV;
  int causal;
  float attn_scale;
  bool windows;  // dQ stream order (StreamOrder), the forward's
};

// the LMK row's per-chunk exchange between the two waves of a dQ pair
template <typename T>
struct LmkShared {
  T q[2][kD];      // the row's Q and dO, by chunk parity
  T d[2][kD];
  T p[2][kS];      // per wave: the current slot's dS (one per key)
  float o[2][kD];  // per wave: its slots' share of the row's dQ
  float dl[2][32]; // per slot: -D and the shifted lse of the row
};

// ------------------------------------------------------------ helpers ----

// ----------------------------------- fusion weights and inverse index ----

// An entry (t, s) is listed under chunk idx[t, s] when row t feeds a query chunk that
// exists (causal: t + 1 < nQ).  Each list ends up ascending by (t, s): an entry's
// position is the number of smaller entries in its list (entries are distinct), so the
// order does not depend on the order of collection.  Two forms:
//
// Slices of up to kPrepEntries entries, and decode (one landmark row): one launch.
// Workgroup g of a (batch, retrieval head) slice
//  - writes the fusion weights (Eq. 2, as the forward computed them) of the g-th `per`
//    landmark rows;
//  - builds the inverse index (CSR) of the g-th `per` key chunks: it reads the whole
//    slice's retrieval lists, counts the entries of earlier chunks (the offset of its
//    own lists) and collects its own.
// Every workgroup reads all of its slice's lists (32 KiB at 1,024 chunks, from the L2)
// instead of a launch per step that each wait for the one before: latency is all that
// bounds this step while slices are short.
//
// Longer slices: weights and counts, scan, fill and sort as launches of their own, whose
// work grows with the entries only (the one launch's reads grow with entries x groups).
// One slice, k = 8, one launch / its steps as launches: 1,024 chunks 16 / 28 us, 4,000
// chunks 32 / 34, 4,200 41 / 35, 8,000 58 / 42; k = 32, 1,500 chunks 72 / 86, 2,500 200 /
// 95.  Where many slices fill the chip the line lies a little lower or higher (16 slices of
// 4,000 chunks 126 / 131, 64 of 2,000 187 / 206).
constexpr int kPrepThreads = 256;
constexpr int kPrepPool = 2048;   // entries collected in LDS; more go through global memory
constexpr int kPrepMax = 1024;    // most chunks per workgroup
constexpr int64_t kPrepEntries = 32768;
// Chunks per workgroup, such that the first group of a causal slice with evenly spread
// lists fits the pool: chunk j of n is then retrieved about k ln(n / j) times, so the
// first `per` chunks hold per k (1 + ln(n / per)) entries.  16 are about 660 at 1,024
// chunks and k = 8 (64 took 46 us there); k = 32 takes 8, 1,500 entries; from 4,096
// chunks up at most 256 workgroups read a slice, and its kPrepEntries bound the first
// group by 840.
inline int prep_chunks(int64_t nKV, int K) {
  int per = K > 16 ? 8 : 16;
  while (per < kPrepMax && nKV > (int64_t)per * 256) per *= 2;
  return per;
}
// Position of e in an ascending order of list[lo .. hi): the smaller entries.
__device__ __forceinline__ int prep_rank(const int* list, int lo, int hi, int e) {
  int rank = 0, u = lo;
  for (; u + 8 <= hi; u += 8) {
    int v[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) v[i] = list[u + i];
#pragma unroll
    for (int i = 0; i < 8; ++i) rank += v[i] < e ? 1 : 0;
  }
  for (; u < hi; ++u) rank += list[u] < e ? 1 : 0;
  return rank;
}
__global__ __launch_bounds__(kPrepThreads) void bwd_prep_kernel(const int32_t* __restrict__ idx,
                                                                const float* __restrict__ sel, BwdWs ws,
                                                                int64_t nQ, int K, int64_t nKV, int causal,
                                                                int per, int64_t groups) {
  __shared__ int sE[kPrepPool];             // collected entries ...
  __shared__ unsigned short sJ[kPrepPool];  // ... and their chunks (less the group's first)
  __shared__ int sList[kPrepPool];          // the same grouped by chunk
  __shared__ int sCnt[kPrepMax], sCur[kPrepMax], sOff[kPrepMax + 1];
  __shared__ int sBelow, sM;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int64_t bhr = blockIdx.x / groups, g = blockIdx.x % groups;
  const int64_t j0 = g * per;
  const int nj = (int)min<int64_t>(per, nKV - j0);
  const int32_t* lists = idx + bhr * nQ * K;
  const int n = (int)((nQ - causal) * K);  // entries of rows that feed a chunk: a prefix
  for (int i = tid; i < (per + 63 & ~63); i += kPrepThreads) {
    sCnt[i] = 0;
    sCur[i] = 0;
  }
  if (tid == 0) {
    sBelow = 0;
    sM = 0;
  }
  __syncthreads();

  constexpr int kB = 16;  // loads in flight per thread
  int below = 0;
  for (int64_t e0 = 0; e0 < n; e0 += kPrepThreads * kB) {
    int j[kB];
#pragma unroll
    for (int m = 0; m < kB; ++m) {
      const int64_t e = e0 + m * kPrepThreads + tid;
      j[m] = e < n ? lists[e] : -1;
    }
#pragma unroll
    for (int m = 0; m < kB; ++m) {
      const bool valid = j[m] >= 0 && j[m] < nKV;
      const int64_t d = j[m] - j0;
      below += valid && d < 0 ? 1 : 0;
      const bool mine = valid && d >= 0 && d < per;
      const uint64_t mask = __ballot(mine);
      if (mask == 0) continue;  // one reservation per wave
      int at = 0;
      if (lane == 0) at = atomicAdd(&sM, __popcll(mask));
      at = __builtin_amdgcn_readfirstlane(at) + lanes_below(mask);
      if (mine) {
        atomicAdd(&sCnt[d], 1);
        if (at < kPrepPool) {
          sE[at] = (int)(e0 + m * kPrepThreads + tid);
          sJ[at] = (unsigned short)d;
        }
      }
    }
  }
  // (a slice has fewer than 2^31 entries)
  for (int o = 32; o > 0; o >>= 1) below += __shfl_xor(below, o);
  if (lane == 0) atomicAdd(&sBelow, below);
  __syncthreads();
  if (wave == 0) {  // exclusive scan of the counts
    int carry = 0;
    for (int i0 = 0; i0 < per; i0 += 64) {
      const int v = sCnt[i0 + lane];
      int x = v;
#pragma unroll
      for (int o = 1; o < 64; o <<= 1) {
        const int y = __shfl_up(x, o);
        if (lane >= o) x += y;
      }
      sOff[i0 + lane] = carry + x - v;
      carry += __shfl(x, 63);
    }
    if (lane == 0) sOff[per] = carry;
  }
  __syncthreads();
  const int base = sBelow, m = sM;
  int* offs = ws.offs + bhr * (nKV + 1);
  int* sorted = ws.sorted + bhr * nQ * K;
  int* head = ws.head + (bhr * nKV + j0) * kHeadInts;
  for (int d = tid; d < nj; d += kPrepThreads) {
    offs[j0 + d] = base + sOff[d];
    head[d * kHeadInts] = base + sOff[d];
    head[d * kHeadInts + 1] = sCnt[d];
  }
  if (tid == 0 && g == groups - 1) offs[nKV] = base + m;

  if (m <= kPrepPool) {
    for (int i = tid; i < m; i += kPrepThreads) {
      const int d = sJ[i];
      sList[sOff[d] + atomicAdd(&sCur[d], 1)] = sE[i];
    }
    __syncthreads();
    for (int i = tid; i < m; i += kPrepThreads) {
      const int d = sJ[i], e = sE[i], lo = sOff[d], hi = sOff[d + 1];
      const int rank = prep_rank(sList, lo, hi, e);
      sorted[base + lo + rank] = e;
      if (rank < kHeadEntries) head[d * kHeadInts + 2 + rank] = e;
    }
  } else {
    int* list = ws.unsorted + bhr * nQ * K + base;
    for (int64_t e = tid; e < n; e += kPrepThreads) {
      const int j = lists[e];
      if (j < 0 || j >= nKV) continue;
      const int64_t d = j - j0;
      if (d >= 0 && d < per) list[sOff[d] + atomicAdd(&sCur[d], 1)] = (int)e;
    }
    __syncthreads();  // the workgroup's own global writes are visible to it
    for (int d = wave; d < nj; d += kPrepThreads / 64) {
      const int lo = sOff[d], hi = sOff[d + 1];
      for (int i = lo + lane; i < hi; i += 64) {
        const int e = list[i];
        const int rank = prep_rank(list, lo, hi, e);
        sorted[base + lo + rank] = e;
        if (rank < kHeadEntries) head[d * kHeadInts + 2 + rank] = e;
      }
    }
  }

  // fusion weights: the rows' chunks and scores through LDS (the pool's space, read
  // above) a few rows at a time, then one (row, slot) per thread
  const int64_t r1 = min<int64_t>((g + 1) * per, nQ);
  const int rows = kPrepPool / K;
  for (int64_t r0 = g * per; r0 < r1; r0 += rows) {
    const int64_t at0 = (bhr * nQ + r0) * K;
    const int ne = (int)min<int64_t>(rows, r1 - r0) * K;
    __syncthreads();
    for (int e = tid; e < ne; e += kPrepThreads) {
      sE[e] = idx[at0 + e];
      sList[e] = __float_as_int(sel[at0 + e]);
    }
    __syncthreads();
    for (int e = tid; e < ne; e += kPrepThreads) {
      const int row = e / K * K;
      float wv;
      int jv;
      row_weight(sE + row, reinterpret_cast<const float*>(sList) + row, K, nKV, e - row, wv, jv);
      ws.w[at0 + e] = wv;
    }
  }
}

// The long form.  A slice's counts, then its fill cursors, sit at the start of its part of
// ws.sorted, which the last launch overwrites.
__global__ void bwd_prep_clear_kernel(int* __restrict__ sorted, int64_t BHr, int64_t nQ, int K, int64_t nKV) {
  for (int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x; i < BHr * nKV; i += (int64_t)gridDim.x * blockDim.x)
    sorted[i / nKV * nQ * K + i % nKV] = 0;
}

__global__ void bwd_prep_count_kernel(const int32_t* __restrict__ idx, const float* __restrict__ sel, BwdWs ws,
                                      int64_t BHr, int64_t nQ, int K, int64_t nKV, int causal) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= BHr * nQ * K) return;
  const int64_t row = e / K;
  float wv;
  int j;
  row_weight(idx + row * K, sel + row * K, K, nKV, (int)(e % K), wv, j);
  ws.w[e] = wv;
  if (j >= 0 && row % nQ + causal < nQ) atomicAdd(&ws.sorted[row / nQ * nQ * K + j], 1);
}

// Exclusive scan of one slice's counts: offs[0 .. nKV], and the cursors in their place.
constexpr int kPrepScan = 1024;
__global__ __launch_bounds__(kPrepScan) void bwd_prep_scan_kernel(BwdWs ws, int64_t nQ, int K, int64_t nKV) {
  __shared__ int sWave[kPrepScan / 64];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int* cur = ws.sorted + (int64_t)blockIdx.x * nQ * K;
  int* off = ws.offs + (int64_t)blockIdx.x * (nKV + 1);
  int carry = 0;
  for (int64_t base = 0; base < nKV; base += kPrepScan) {
    const int64_t i = base + tid;
    const int v = i < nKV ? cur[i] : 0;
    int x = v;  // inclusive scan within the wave
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const int y = __shfl_up(x, o);
      if (lane >= o) x += y;
    }
    if (lane == 63) sWave[wave] = x;
    __syncthreads();
    int before = 0, all = 0;
    for (int w = 0; w < kPrepScan / 64; ++w) {
      before += w < wave ? sWave[w] : 0;
      all += sWave[w];
    }
    if (i < nKV) {
      off[i] = carry + before + x - v;
      cur[i] = carry + before + x - v;
    }
    carry += all;
    __syncthreads();
  }
  if (tid == 0) off[nKV] = carry;
}

__global__ void bwd_prep_fill_kernel(const int32_t* __restrict__ idx, BwdWs ws, int64_t BHr, int64_t nQ, int K,
                                     int64_t nKV, int causal) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= BHr * nQ * K) return;
  const int64_t slice = e / (nQ * K), local = e % (nQ * K);  // t * K + s
  const int j = idx[e];
  if (j >= 0 && j < nKV && local / K + causal < nQ)
    ws.unsorted[slice * nQ * K + atomicAdd(&ws.sorted[slice * nQ * K + j], 1)] = (int)local;
}

// One wave per chunk.
__global__ __launch_bounds__(256) void bwd_prep_sort_kernel(BwdWs ws, int64_t BHr, int64_t nQ, int K, int64_t nKV) {
  const int64_t wv = (int64_t)blockIdx.x * 4 + (threadIdx.x >> 6);
  if (wv >= BHr * nKV) return;
  const int lane = threadIdx.x & 63;
  const int64_t slice = wv / nKV, j = wv % nKV;
  const int lo = ws.offs[slice * (nKV + 1) + j], hi = ws.offs[slice * (nKV + 1) + j + 1];
  const int* src = ws.unsorted + slice * nQ * K;
  int* head = ws.head + wv * kHeadInts;
  if (lane == 0) {
    head[0] = lo;
    head[1] = hi - lo;
  }
  for (int i = lo + lane; i < hi; i += 64) {
    const int e = src[i], rank = prep_rank(src, lo, hi, e);
    ws.sorted[slice * nQ * K + lo + rank] = e;
    if (rank < kHeadEntries) head[2 + rank] = e;
  }
}

// ------------------------------------------------- query-stationary dQ ----

// Persistent workgroups of one wave pair, four per CU; each pair is a stream of
// (batch, head, query chunk) items, taking the chunk's retrieved chunks one per round
// from its two LDS ring slots (K_j and V_j tiles, copied one round ahead), each
// wave owning 32 query tokens.  Per retrieved chunk it writes D_s and the
// shifted log-sum-exp used by the key-stationary pass, and the wave's partial
// sum of D_s for dw; dQ stays in registers until the chunk ends.  The work order
// is the forward's (StreamOrder, chosen the same way).
// STAGE (k <= kDqStageK): the per-(token, slot) values are staged in LDS and
// stored once per chunk.
constexpr int kDqStageK = 8;
template <typename T, bool STAGE, bool XR>
__global__ __launch_bounds__(kThreads, kWgPerCu) void bwd_dq_kernel(BwdParams p, int64_t nwork) {
  constexpr int TILE = kS * kD;
  constexpr int SQ = XR ? kS + 1 : kS;  // query rows per chunk
  static_assert(kPairs == 1, "the LMK row exchange assumes one pair per workgroup");
  __shared__ __attribute__((aligned(16))) LmkShared<T> sX[1];  // used with XR only
  __shared__ __attribute__((aligned(16))) T ring[kPairs * 2 * 2 * TILE];  // pair p: slots 2p, 2p+1
  __shared__ int sJ[kPairs][2][32];     // [pair][chunk parity][slot]: chunk index or -1
  __shared__ int sSlot[kPairs][2][32];  // compacted valid slots: slot, chunk, weight
  __shared__ int sJc[kPairs][2][32];
  __shared__ float sWc[kPairs][2][32];
  __shared__ int sN[kPairs][2];
  // per wave, the (-D, shifted lse) pairs of its 32 tokens x k slots and its dw
  // partials (k <= 8), stored at the end of the chunk: a store still in flight
  // holds up the next round's wait for its copies, so none is issued per round
  constexpr int kStageK = STAGE ? kDqStageK : 1;
  __shared__ float sDL[2 * kPairs][2][kStageK][32];
  __shared__ float sDw[2 * kPairs][kStageK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5;
  const int pair = wave >> 1, half = wave & 1;
  const int xcd = (int)(blockIdx.x & 7);
  const int64_t st_wg = (int64_t)(blockIdx.x >> 3) * kPairs;
  auto order_of = [&](int q) {
    return StreamOrder((int64_t)(gridDim.x >> 3) * kPairs, st_wg + q, xcd, nwork, p.windows);
  };
  const StreamOrder ord = order_of(pair);
  const int64_t my_n = ord.length();
  int64_t nch = 0;  // all pairs of the workgroup run nch chunks of rounds
  for (int q = 0; q < kPairs; ++q) nch = max(nch, order_of(q).length());
  if (nch == 0) return;
  const int64_t c_begin = ord.item(0);
  const int K = p.K;
  const int qi = 32 * half + (lane & 31);
  const int l32 = lane & 31;
  const float sc = p.attn_scale * kLog2e;
  const int cb = 16 * ((lane >> 4) & 1);

  // retrieval row t of a chunk: its offset in idx / w, or -1
  auto row_off_of = [&](const Geo& g) -> int64_t {
    const int hr = p.Hr == 1 ? 0 : g.h;
    const int64_t t = p.causal ? g.c - 1 : 0;
    return t >= 0 ? ((g.b * p.Hr + hr) * p.nQ + t) * K : -1;
  };
  struct Meta {
    int j;
    float w;
  };
  auto load_meta = [&](const Geo& g) -> Meta {
    Meta m{-1, 0.f};
    const int64_t ro = row_off_of(g);
    if (ro >= 0 && lane < K) {
      m.j = p.idx[ro + lane];
      m.w = p.ws.w[ro + lane];
    }
    return m;
  };
  // first wave of a pair: the pair's compacted slot list of a chunk
  auto make_slots = [&](const Meta& m, int buf) __device__ {
    const bool valid = lane < K && m.j >= 0 && m.j < p.nKV;
    const uint64_t mask = __ballot(valid);
    if (lane < 32) sJ[pair][buf][lane] = valid ? m.j : -1;
    if (valid) {
      const int rk = lanes_below(mask);
      sSlot[pair][buf][rk] = lane;
      sJc[pair][buf][rk] = m.j;
      sWc[pair][buf][rk] = m.w;
    }
    if (lane == 0) sN[pair][buf] = __popcll(mask);
  };
  auto tok_of = [&](const Geo& g) -> int64_t { return ((g.b * p.H + g.h) * p.nQ + g.c) * SQ; };
  const int64_t lq_len = p.nQ * SQ;  // query tokens per (batch, head)
  // the LMK row's Q and dO rows: copied straight into LDS (wave 0 the Q row, wave
  // 1 the dO row, one 16-byte piece per lane below kXPieces) with the chunk's
  // Q/dO fragment loads; visible to both waves after the next wait and barrier
  constexpr int kXPieces = kD * (int)sizeof(T) / 16;
  const int xh = __builtin_amdgcn_readfirstlane(half);  // the wave's half, in a scalar register

  // ---- prologue
  Frag<T> qf[4], df[4];  // the current chunk's Q and dO rows of this lane's query
  Meta meta{-1, 0.f};
  Geo g0(c_begin, p.nQ, p.H);
  Geo g1 = g0, g2 = g0;  // (the range order steps without divisions)
  if (p.windows) {
    g1 = Geo(ord.item(1), p.nQ, p.H);
    g2 = Geo(ord.item(2), p.nQ, p.H);
  } else {
    g1.next(p.nQ, p.H, ord.S);
    g2 = g1;
    g2.next(p.nQ, p.H, ord.S);
  }
  auto load_qdo = [&](const Geo& g, Frag<T>* qd, Frag<T>* dd, int xbuf) __device__ {
    const int64_t row = tok_of(g) + (XR ? opaque(qi) : qi);
    const T* qr = reinterpret_cast<const T*>(p.q) + row * kD;
    const T* dr = reinterpret_cast<const T*>(p.dout) + row * kD;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      qd[kb] = load_frag(qr + 16 * kb + 8 * hh);
      dd[kb] = load_frag(dr + 16 * kb + 8 * hh);
    }
    if (XR && lane < kXPieces) {
      const int64_t xrow = (tok_of(g) + kS) * kD;
      const T* src = reinterpret_cast<const T*>(xh == 0 ? p.q : p.dout) + xrow;
      dma_row16(src, lane * 16u, xh == 0 ? &sX[0].q[xbuf][0] : &sX[0].d[xbuf][0]);
    }
  };
  if (my_n > 0) {
    const Meta m0 = load_meta(g0);
    load_qdo(g0, qf, df, 0);
    if (half == 0) make_slots(m0, 0);
    if (my_n > 1) meta = load_meta(g1);
  }
  wait_vmem<0>();
  __syncthreads();

  const TileCopy<T, 2> cp(half, lane);
  const T* const gk = reinterpret_cast<const T*>(p.k);
  const T* const gv = reinterpret_cast<const T*>(p.v);
  auto slice_of = [&](const Geo& g) __device__ { return (g.b * p.H + g.h) * p.nKV * TILE; };
  auto issue_item = [&](int64_t kvb, int j, int slot) __device__ {
    j = min(max(j, 0), (int)p.nKV - 1);  // lists hold valid chunks; never copy from outside the slice
    T* dst = ring + (2 * pair + slot) * (2 * TILE);
    cp.issue(gk + kvb + (int64_t)j * TILE, dst);
    cp.issue(gv + kvb + (int64_t)j * TILE, dst + TILE);
  };
  int ls = sSlot[pair][0][l32], lj = sJc[pair][0][l32];
  float lw = sWc[pair][0][l32];
  int64_t kvb = uniform64(slice_of(g0)), kvb_n = 0;
  int cs = 0;
  // this lane's saved lse of the next item to compute (loaded a round ahead),
  // and the LMK row's
  float lse_next = 0.f, lsex_next = 0.f;
  if (my_n > 0 && sN[pair][0] > 0) {
    issue_item(kvb, __builtin_amdgcn_readlane(lj, 0), cs);
    lse_next = p.lse[(tok_of(g0) + qi) * K + __builtin_amdgcn_readlane(ls, 0)];
    if (XR) lsex_next = p.lse[(tok_of(g0) + kS) * K + __builtin_amdgcn_readlane(ls, 0)];
  }

  constexpr bool kB16 = std::is_same<T, __bf16>::value;
  constexpr uint32_t kTileB = TILE * sizeof(T), kRowB = kD * sizeof(T);
  const lds_char* const lds0 = (const lds_char*)(ring);
  uint32_t kofs[4], tofs[2][2];
  {
    const uint32_t pb = (uint32_t)pair * 4 * kTileB;
    const int s16 = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kofs[kb] = pb + Swz<T>::off(lane & 31, 16 * kb + 8 * hh) * sizeof(T);
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        tofs[dh][r8] = pb + Swz<T>::off(8 * r8 + 4 * hh + (s16 >> 2), 32 * dh + cb + 4 * (s16 & 3)) * sizeof(T);
  }

  f32x16 g0a = zero16(), g1a = zero16();  // dQ^T, d rows 0-31 / 32-63
  // cbase: element of (this slice, slot 0, this chunk's first token) in Dbuf / Lbuf
  // pre: this is the chunk's last item and a next chunk follows; its Q and dO rows
  // are loaded as soon as this item's products have read qf/df, so that the
  // next chunk's first round does not wait out the whole load
  float ox0 = 0.f, ox1 = 0.f;  // LMK row: this lane's partial dQ for d = l%32 and 32 + l%32
  auto run = [&](int slot, int u, float lse_q, float lse_x, int64_t cbase, int64_t t, bool pre, int buf) __device__ {
    const uint32_t co = (uint32_t)slot * 2 * kTileB;
    // With the LMK row every register counts: the other fragment offsets are
    // derived from the first two each round by their swizzle's fixed XOR
    // patterns (key block kb: bits 5-6; transposed halves: bit 6, and rows +8:
    // bits 4 and 10), instead of being held across the whole loop.
    uint32_t k0b = kofs[0], t0b = tofs[0][0];
    if constexpr (XR && kB16) {
      k0b = (uint32_t)opaque((int)k0b);
      t0b = (uint32_t)opaque((int)t0b);
    }
    auto KO = [&](int kb) -> uint32_t { return (XR && kB16) ? (k0b ^ (uint32_t)(kb << 5)) : kofs[kb]; };
    auto TO = [&](int dh, int r8) -> uint32_t {
      return (XR && kB16) ? (t0b ^ (uint32_t)((dh << 6) | (r8 ? 1040 : 0))) : tofs[dh][r8];
    };
    const int s = __builtin_amdgcn_readlane(ls, u);
    const float ws = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(lw), u));
    const bool xr = XR && (u & 1) == xh;  // this wave takes the LMK row of slot u
    const T* sK = ring + (2 * pair + slot) * (2 * TILE);
    const T* sV = sK + TILE;
    // the LMK row: scores and dP with one key per lane (row fragments of K and V
    // against the row's Q and dO, the two dimension halves added across l ^ 32),
    // w P, D, dS, and its dQ against the K^T fragments
    float Dx = 0.f;
    if (xr) {
      __builtin_amdgcn_sched_barrier(0);  // the row's reads start after the tile's products
      float a0 = 0.f, a1 = 0.f, b0 = 0.f, b1 = 0.f;
#pragma unroll
      for (int kb = 0; kb < 8; ++kb) {
        __builtin_amdgcn_sched_barrier(0);  // one key block's fragments live at a time
        const int kk = kb & 3;
        const bool vt = kb >= 4;  // blocks 0-3: K against the row's Q; 4-7: V against its dO
        const Frag<T> xv = vec_frag(vt ? &sX[0].d[buf][0] : &sX[0].q[buf][0], 16 * kk + 8 * hh);
        Frag<T> r0, r1;
        if constexpr (kB16) {
          const lds_char* kp = lds0 + (KO(kk) + co) + (vt ? kTileB : 0u);
          r0 = lds_b128_at(kp);
          r1 = lds_b128_at(kp + 32 * kRowB);
        } else {
          r0 = lds_frag(vt ? sV : sK, lane & 31, 16 * kk + 8 * hh);
          r1 = lds_frag(vt ? sV : sK, 32 + (lane & 31), 16 * kk + 8 * hh);
        }
        if (vt) {
          b0 = frag_dot(r0, xv, b0);
          b1 = frag_dot(r1, xv, b1);
        } else {
          a0 = frag_dot(r0, xv, a0);
          a1 = frag_dot(r1, xv, a1);
        }
      }
      a0 = sum_xor32(a0);
      a1 = sum_xor32(a1);
      b0 = sum_xor32(b0);
      b1 = sum_xor32(b1);
      const float xs = hh ? a1 : a0, xdp = hh ? b1 : b0;  // key `lane`
      const float wsf = fmaxf(ws, 1e-30f);
      const float offx = lse_x * kLog2e - __builtin_amdgcn_logf(wsf);
      const float wpx = __builtin_amdgcn_exp2f(fmaf(xs, sc, -offx));
      Dx = sum64(wpx * xdp) * __builtin_amdgcn_rcpf(wsf);
      sX[0].p[xh][lane] = (T)(wpx * (xdp - Dx));
      wave_lds_order();  // one from each lane ...
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        __builtin_amdgcn_sched_barrier(0);  // one key block's fragments live at a time
        Frag<T> k0, k1;
        if constexpr (kB16) {
          k0 = lds_tr2(lds0 + (TO(0, 0) + co) + 16 * kb * kRowB, lds0 + (TO(0, 1) + co) + 16 * kb * kRowB);
          k1 = lds_tr2(lds0 + (TO(1, 0) + co) + 16 * kb * kRowB, lds0 + (TO(1, 1) + co) + 16 * kb * kRowB);
        } else {
          k0 = lds_frag_t(sK, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, cb);
          k1 = lds_frag_t(sK, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, 32 + cb);
        }
        const Frag<T> xf = vec_frag_t(&sX[0].p[xh][0], 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh);
        ox0 = frag_dot(k0, xf, ox0);
        ox1 = frag_dot(k1, xf, ox1);
      }
      wave_lds_order();  // ... which the next slot's overwrite after this
      if (lane == 0) {
        sX[0].dl[0][s] = -Dx;
        sX[0].dl[1][s] = lse_x * kLog2e - __builtin_amdgcn_logf(ws);
      }
      __builtin_amdgcn_sched_barrier(0);  // the tile's own products start after the row's
    }
    f32x16 s0 = zero16(), s1 = zero16(), p0 = zero16(), p1 = zero16();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (kB16) {
        const lds_char* kp = lds0 + (KO(kb) + co);
        mma32(s0, lds_b128_at(kp), qf[kb]);
        mma32(s1, lds_b128_at(kp + 32 * kRowB), qf[kb]);
        mma32(p0, lds_b128_at(kp + kTileB), df[kb]);
        mma32(p1, lds_b128_at(kp + (kTileB + 32 * kRowB)), df[kb]);
      } else {
        mma32(s0, lds_frag(sK, lane & 31, 16 * kb + 8 * hh), qf[kb]);
        mma32(s1, lds_frag(sK, 32 + (lane & 31), 16 * kb + 8 * hh), qf[kb]);
        mma32(p0, lds_frag(sV, lane & 31, 16 * kb + 8 * hh), df[kb]);
        mma32(p1, lds_frag(sV, 32 + (lane & 31), 16 * kb + 8 * hh), df[kb]);
      }
    }
    if (pre) load_qdo(g1, qf, df, buf ^ 1);
    // w P^T (the weight folded into the exponent: wsf = max(ws, 1e-30) keeps the
    // shift finite), D = rowsum(P o dP) for this lane's query, w dS
    const float wsf = fmaxf(ws, 1e-30f);
    const float off = lse_q * kLog2e - __builtin_amdgcn_logf(wsf);
    float Dw = 0.f;
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s0[i] = __builtin_amdgcn_exp2f(fmaf(s0[i], sc, -off));
      s1[i] = __builtin_amdgcn_exp2f(fmaf(s1[i], sc, -off));
      Dw = fmaf(s0[i], p0[i], Dw);
      Dw = fmaf(s1[i], p1[i], Dw);
    }
    const float Dq = sum_xor32(Dw) * __builtin_amdgcn_rcpf(wsf);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      s0[i] = s0[i] * (p0[i] - Dq);
      s1[i] = s1[i] * (p1[i] - Dq);
    }
    Frag<T> f[4];
    frag_from_acc(f[0], s0, 0, 1.f);
    frag_from_acc(f[1], s0, 1, 1.f);
    frag_from_acc(f[2], s1, 0, 1.f);
    frag_from_acc(f[3], s1, 1, 1.f);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (kB16) {
        mma32(g0a, lds_tr2(lds0 + (TO(0, 0) + co) + 16 * kb * kRowB, lds0 + (TO(0, 1) + co) + 16 * kb * kRowB),
              f[kb]);
        mma32(g1a, lds_tr2(lds0 + (TO(1, 0) + co) + 16 * kb * kRowB, lds0 + (TO(1, 1) + co) + 16 * kb * kRowB),
              f[kb]);
      } else {
        mma32(g0a, lds_frag_t(sK, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, cb), f[kb]);
        mma32(g1a, lds_frag_t(sK, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, 32 + cb), f[kb]);
      }
    }
    // D_s (negated: it seeds the dP accumulator there) and the shifted lse of this
    // (query, slot) for the key-stationary pass
    if (hh == 0) {
      const float dneg = -Dq, lsh = lse_q * kLog2e - __builtin_amdgcn_logf(ws);
      if constexpr (STAGE) {
        sDL[wave][0][s][l32] = dneg;
        sDL[wave][1][s][l32] = lsh;
      } else {
        const int64_t o = cbase + s * lq_len + (XR ? opaque(qi) : qi);
        p.ws.Dbuf[o] = dneg;
        p.ws.Lbuf[o] = lsh;
      }
    }
    // this wave's 32 queries' share of dw[t, s] (and the LMK row's D)
    const float dsum = sum32(Dq) + Dx;
    if (lane == 0) {
      if constexpr (STAGE) sDw[wave][s] = dsum;
      else p.ws.dwp[(t * K + s) * 2 + half] = dsum;
    }
  };

  for (int64_t ci = 0; ci < nch; ++ci) {
    const bool live = ci < my_n, live_next = ci + 1 < my_n;
    const int buf = (int)(ci & 1);
    const int n = live ? sN[pair][buf] : 0;
    const int64_t tok0 = tok_of(g0);
    const int64_t cbase = (g0.b * p.H + g0.h) * K * lq_len + g0.c * SQ;
    const int64_t tglob = (g0.b * p.H + g0.h) * p.nQ + (p.causal ? g0.c - 1 : 0);  // dw row (b, h, t)
    const int64_t tok_n = tok_of(g1);
    for (int u = 0; u < K; ++u) {
      wait_vmem<0>();
      block_barrier();
      if (u == 0) {
        if (ci > 0 && live) {
          ls = sSlot[pair][buf][l32];
          lj = sJc[pair][buf][l32];
          lw = sWc[pair][buf][l32];
          kvb = kvb_n;
        }
        if (live_next) {
          if (half == 0) make_slots(meta, buf ^ 1);
          if (ci + 2 < my_n) meta = load_meta(g2);
          kvb_n = uniform64(slice_of(g1));
        }
        if (K == 1) block_barrier();  // the next chunk's list is needed this round
      }
      const bool comp = u < n;
      const int is = comp ? cs ^ 1 : cs;
      const float lse_q = lse_next, lse_x = lsex_next;
      if (u + 1 < n) {
        issue_item(kvb, __builtin_amdgcn_readlane(lj, u + 1), is);
        lse_next = p.lse[(tok0 + (XR ? opaque(qi) : qi)) * K + __builtin_amdgcn_readlane(ls, u + 1)];
        if (XR) lsex_next = p.lse[(tok0 + kS) * K + __builtin_amdgcn_readlane(ls, u + 1)];
      } else if (u == K - 1 && live_next && sN[pair][buf ^ 1] > 0) {
        issue_item(kvb_n, sJc[pair][buf ^ 1][0], is);
        lse_next = p.lse[(tok_n + (XR ? opaque(qi) : qi)) * K + sSlot[pair][buf ^ 1][0]];
        if (XR) lsex_next = p.lse[(tok_n + kS) * K + sSlot[pair][buf ^ 1][0]];
      }
      if (comp) {
        run(cs, u, lse_q, lse_x, cbase, tglob, live_next && u == n - 1, buf);
        cs ^= 1;
      }
      // a chunk without items loads the next chunk's Q and dO rows in its first round
      if (n == 0 && u == 0 && live_next) load_qdo(g1, qf, df, buf ^ 1);
    }

    // ---- finish the chunk: dQ rows of this wave; zero dw partials of empty slots
    if (live) {
      const float as = p.attn_scale;
      T* drow = reinterpret_cast<T*>(p.dq) + (tok0 + (XR ? opaque(qi) : qi)) * kD;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        store4(drow + 8 * g + 4 * hh, as * g0a[4 * g], as * g0a[4 * g + 1], as * g0a[4 * g + 2],
               as * g0a[4 * g + 3]);
        store4(drow + 32 + 8 * g + 4 * hh, as * g1a[4 * g], as * g1a[4 * g + 1], as * g1a[4 * g + 2],
               as * g1a[4 * g + 3]);
      }
      const bool has_row = !p.causal || g0.c > 0;
      if constexpr (XR) {
        // the LMK row: add the two waves' shares of its dQ, store it and its
        // per-slot -D and shifted lse
        const float t0 = sum_xor32(ox0), t1 = sum_xor32(ox1);
        sX[0].o[xh][lane] = hh ? t1 : t0;  // lane l: d = l
        block_barrier();
        if (xh == 0) {
          // (lane-dependent addresses are formed here, not kept in registers
          // across the whole loop)
          const int ln = opaque(lane);
          const int64_t tx = tok0 + kS;
          reinterpret_cast<T*>(p.dq)[tx * kD + ln] = (T)(as * (sX[0].o[0][lane] + sX[0].o[1][lane]));
          if (lane < K && sJ[pair][buf][lane] >= 0) {
            const int64_t o = cbase + ln * lq_len + kS;
            p.ws.Dbuf[o] = sX[0].dl[0][lane];
            p.ws.Lbuf[o] = sX[0].dl[1][lane];
          }
        }
        ox0 = 0.f;
        ox1 = 0.f;
      }
      if constexpr (STAGE) {
        // this wave's staged values: per valid slot one contiguous run of 32 tokens
        wave_lds_order();  // other lanes staged them ...
        for (int e = lane; e < 32 * K; e += 64) {
          const int sl = e >> 5, q = e & 31;
          if (sJ[pair][buf][sl] >= 0) {
            const int64_t o = cbase + sl * lq_len + 32 * half + (XR ? opaque(q) : q);
            p.ws.Dbuf[o] = sDL[wave][0][sl][q];
            p.ws.Lbuf[o] = sDL[wave][1][sl][q];
          }
        }
        if (has_row && lane < K) {
          const int sl = opaque(lane);
          p.ws.dwp[(tglob * K + sl) * 2 + xh] = sJ[pair][buf][lane] >= 0 ? sDw[wave][lane] : 0.f;
        }
        wave_lds_order();  // ... and the next chunk's are staged after this
      } else if (has_row && n < K && lane < K && sJ[pair][buf][lane] < 0) {
        const int sl = opaque(lane);
        p.ws.dwp[(tglob * K + sl) * 2 + xh] = 0.f;
      }
    }
    g0a = zero16();
    g1a = zero16();
    g0 = g1;
    g1 = g2;
    if (p.windows)
      g2 = Geo(ord.item(ci + 3), p.nQ, p.H);
    else
      g2.next(p.nQ, p.H, ord.S);
  }
}

// The same pass for few query chunks (few_pairs): one workgroup of several wave pairs per
// chunk, the pairs taking its slots side by side (two resident slots per pair in bf16,
// one in fp32) and adding their dQ through LDS in pair order, instead of one pair taking
// them one after another on a chip that is mostly idle.
template <typename T, int PAIRS>
__global__ __launch_bounds__(128 * PAIRS, PAIRS == 4 ? 1 : 2) void bwd_dq_few_kernel(BwdParams p) {
  constexpr int TILE = kS * kD;
  constexpr bool kB16 = std::is_same<T, __bf16>::value;
  constexpr int SP = kB16 ? 2 : 1;  // resident slots per pair
  constexpr int kPerRound = PAIRS * SP;
  constexpr uint32_t kTileB = TILE * sizeof(T), kRowB = kD * sizeof(T);
  __shared__ __attribute__((aligned(16))) T ring[PAIRS * SP * 2 * TILE];  // K and V tiles; then the partial dQ
  __shared__ int sSlot[32], sJc[32];
  __shared__ float sWc[32];
  __shared__ int sN;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5, l32 = lane & 31;
  const int pair = wave >> 1, half = wave & 1;
  const int64_t wi = blockIdx.x;  // (batch, head, query chunk)
  const int64_t bh = wi / p.nQ, c = wi % p.nQ;
  const int64_t b = bh / p.H;
  const int h = (int)(bh % p.H);
  const int K = p.K;
  const bool has_row = !p.causal || c > 0;
  const int64_t t = p.causal && has_row ? c - 1 : c;
  const int64_t ro = ((b * p.Hr + (p.Hr == 1 ? 0 : h)) * p.nQ + t) * K;
  const int64_t tglob = bh * p.nQ + t;  // dw row (b, h, t)
  const int qi = 32 * half + l32;
  const int64_t tok0 = wi * kS, lq_len = p.nQ * kS;
  const int64_t cbase = bh * K * lq_len + c * kS;
  const float sc = p.attn_scale * kLog2e;
  const int cb = 16 * ((lane >> 4) & 1);

  Frag<T> qf[4], df[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    qf[kb] = load_frag(reinterpret_cast<const T*>(p.q) + (tok0 + qi) * kD + 16 * kb + 8 * hh);
    df[kb] = load_frag(reinterpret_cast<const T*>(p.dout) + (tok0 + qi) * kD + 16 * kb + 8 * hh);
  }
  if (wave == 0) {
    int j = -1;
    float w = 0.f;
    if (has_row && lane < K) {
      j = p.idx[ro + lane];
      w = p.ws.w[ro + lane];
    }
    const bool valid = j >= 0 && j < p.nKV;
    const uint64_t mask = __ballot(valid);
    if (valid) {
      const int rk = lanes_below(mask);
      sSlot[rk] = lane;
      sJc[rk] = j;
      sWc[rk] = w;
    } else if (has_row && lane < K) {
      // a slot without a chunk: zero dw partials
      p.ws.dwp[(tglob * K + lane) * 2] = 0.f;
      p.ws.dwp[(tglob * K + lane) * 2 + 1] = 0.f;
    }
    if (lane == 0) sN = __popcll(mask);
  }
  __syncthreads();
  const int n = sN;
  const TileCopy<T, 2> cp(half, lane);
  const T* const gk = reinterpret_cast<const T*>(p.k) + bh * p.nKV * TILE;
  const T* const gv = reinterpret_cast<const T*>(p.v) + bh * p.nKV * TILE;
  const lds_char* const lds0 = (const lds_char*)(ring);
  const F32Offsets f32(lane);
  uint32_t kofs[4], tofs[2][2];
  {
    const uint32_t pb = (uint32_t)pair * SP * 2 * kTileB;
    const int s16 = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kofs[kb] = pb + Swz<T>::off(l32, 16 * kb + 8 * hh) * sizeof(T);
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        tofs[dh][r8] = pb + Swz<T>::off(8 * r8 + 4 * hh + (s16 >> 2), 32 * dh + cb + 4 * (s16 & 3)) * sizeof(T);
  }
  f32x16 g0 = zero16(), g1 = zero16();  // dQ^T, d rows 0-31 / 32-63
  auto run = [&](int slot, int i, float lse_q) __device__ {
    const int s = sSlot[i];
    const float ws = sWc[i];
    const uint32_t co = (uint32_t)slot * 2 * kTileB;
    const lds_char* const tl = lds0 + (uint32_t)(pair * SP + slot) * 2 * kTileB;
    auto row = [&](int kb, int half32, bool v) __device__ -> Frag<T> {
      if constexpr (kB16)
        return lds_b128_at(lds0 + (kofs[kb] + co) + (v ? kTileB : 0u) + half32 * 32 * kRowB);
      else
        return f32.row_frag(tl + (v ? kTileB : 0u), kb, half32);
    };
    f32x16 s0 = zero16(), s1 = zero16(), p0 = zero16(), p1 = zero16();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      mma32(s0, row(kb, 0, false), qf[kb]);
      mma32(s1, row(kb, 1, false), qf[kb]);
      mma32(p0, row(kb, 0, true), df[kb]);
      mma32(p1, row(kb, 1, true), df[kb]);
      if (!kB16) __builtin_amdgcn_sched_barrier(0);  // one key block's fragments live at a time
    }
    // as in bwd_dq_kernel
    const float wsf = fmaxf(ws, 1e-30f);
    const float off = lse_q * kLog2e - __builtin_amdgcn_logf(wsf);
    float Dw = 0.f;
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s0[e] = __builtin_amdgcn_exp2f(fmaf(s0[e], sc, -off));
      s1[e] = __builtin_amdgcn_exp2f(fmaf(s1[e], sc, -off));
      Dw = fmaf(s0[e], p0[e], Dw);
      Dw = fmaf(s1[e], p1[e], Dw);
    }
    const float Dq = sum_xor32(Dw) * __builtin_amdgcn_rcpf(wsf);
#pragma unroll
    for (int e = 0; e < 16; ++e) {
      s0[e] = s0[e] * (p0[e] - Dq);
      s1[e] = s1[e] * (p1[e] - Dq);
    }
    Frag<T> f[4];
    frag_from_acc(f[0], s0, 0, 1.f);
    frag_from_acc(f[1], s0, 1, 1.f);
    frag_from_acc(f[2], s1, 0, 1.f);
    frag_from_acc(f[3], s1, 1, 1.f);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (kB16) {
        mma32(g0, lds_tr2(lds0 + (tofs[0][0] + co) + 16 * kb * kRowB, lds0 + (tofs[0][1] + co) + 16 * kb * kRowB), f[kb]);
        mma32(g1, lds_tr2(lds0 + (tofs[1][0] + co) + 16 * kb * kRowB, lds0 + (tofs[1][1] + co) + 16 * kb * kRowB), f[kb]);
      } else {
        mma32(g0, f32.col_frag(tl, kb, 0), f[kb]);
        mma32(g1, f32.col_frag(tl, kb, 1), f[kb]);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (hh == 0) {
      p.ws.Dbuf[cbase + s * lq_len + qi] = -Dq;
      p.ws.Lbuf[cbase + s * lq_len + qi] = lse_q * kLog2e - __builtin_amdgcn_logf(ws);
    }
    const float dsum = sum32(Dq);
    if (lane == 0) p.ws.dwp[(tglob * K + s) * 2 + half] = dsum;
  };
  for (int r0 = 0; r0 < n; r0 += kPerRound) {
    if (r0 > 0) block_barrier();  // the last round's tiles have been read
    const int i0 = r0 + pair * SP;
    float lse_q[SP];
#pragma unroll
    for (int e = 0; e < SP; ++e) lse_q[e] = i0 + e < n ? p.lse[(tok0 + qi) * K + sSlot[i0 + e]] : 0.f;
#pragma unroll
    for (int e = 0; e < SP; ++e) {
      if (i0 + e < n) {
        const int64_t j = min(max(sJc[i0 + e], 0), (int)p.nKV - 1);
        T* dst = ring + (pair * SP + e) * (2 * TILE);
        cp.issue(gk + j * TILE, dst);
        cp.issue(gv + j * TILE, dst + TILE);
      }
    }
    wait_vmem<0>();
    block_barrier();
#pragma unroll
    for (int e = 0; e < SP; ++e)
      if (i0 + e < n) run(e, i0 + e, lse_q[e]);
  }

  // the pairs' partial dQ: part[pair][row][16 float4 blocks], block c of row r at c ^ (r mod 16)
  block_barrier();
  float* part = reinterpret_cast<float*>(ring);
  static_assert(sizeof(ring) >= PAIRS * kS * kD * sizeof(float), "partial dQ fits in the tiles");
  {
    const int sw = qi & 15;
    float* pr = part + (pair * kS + qi) * kD;
#pragma unroll
    for (int g = 0; g < 4; ++g) {
      *reinterpret_cast<f32x4*>(pr + 4 * ((2 * g + hh) ^ sw)) =
          f32x4{g0[4 * g], g0[4 * g + 1], g0[4 * g + 2], g0[4 * g + 3]};
      *reinterpret_cast<f32x4*>(pr + 4 * ((8 + 2 * g + hh) ^ sw)) =
          f32x4{g1[4 * g], g1[4 * g + 1], g1[4 * g + 2], g1[4 * g + 3]};
    }
  }
  __syncthreads();
  constexpr int kTpr = 2 * PAIRS;  // threads per row
  const int rr = tid / kTpr;
  T* drow = reinterpret_cast<T*>(p.dq) + (tok0 + rr) * kD;
  const float as = p.attn_scale;
#pragma unroll
  for (int e = 0; e < 16 / kTpr; ++e) {
    const int cblk = 16 / kTpr * (tid % kTpr) + e;
    f32x4 acc = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int q = 0; q < PAIRS; ++q)
      acc += *reinterpret_cast<const f32x4*>(part + (q * kS + rr) * kD + 4 * (cblk ^ (rr & 15)));
    store4(drow + 4 * cblk, as * acc[0], as * acc[1], as * acc[2], as * acc[3]);
  }
}

// Wave pairs per item for few items: as many as fit in a CU's LDS while every item runs
// at once (bf16: 4 up to one item per CU, 2 up to two; fp32, whose rounds are five times
// longer, 4 up to two), else 1, the form that keeps four items per CU.  2.4K tokens (444
// items, bf16): dQ 20 -> 14 us and dK/dV 33 -> 24 us a launch (four pairs in two rounds of
// workgroups took 19 and 31); 16 chunks of one head in fp32: dQ 18 -> 13 us.
inline int few_pairs(int64_t items, bool bf16) {
  const int64_t cus = device_cus();
  if (items > 2 * cus) return 1;
  return items <= cus || !bf16 ? 4 : 2;
}
// For dQ, unless lists of one entry (k = 1) leave nothing to share out: the whole backward
// at 504 items, few_pairs' pairs / one: 86 / 72 us in fp32, 31.5 / 29.9 in bf16; at 240
// fp32 items 54 / 51.
inline int q_pairs_of(int64_t items, int K, bool bf16) { return K == 1 ? 1 : few_pairs(items, bf16); }
// The same for dK/dV, whose longest list bounds a causal launch for longer in fp32: 4 up to
// four items per CU, 2 beyond (800 items, k = 8: 202 us with two pairs, 165 with four;
// 2,000 items 343 / 397; one pair with two ring slots 286 and 374) and for k = 1, whose
// lists leave most pairs nothing to do (the whole backward, four pairs / two: 240 items
// 54 / 51 us, 504 86 / 77, 768 99 / 91, 1,020 114 / 100).
// In bf16 one pair is as good or better from three items per CU (1,200 items 47 us
// each way, 6,400 items 148 against 184 us).
inline int kv_pairs(int64_t items, int K, bool bf16) {
  if (bf16) return few_pairs(items, bf16);
  return K > 1 && items <= 4 * (int64_t)device_cus() ? 4 : 2;
}

// ---------------------------------------------- key-stationary dK, dV ----

// One workgroup of two waves per (batch, head, key chunk j), four per CU; the pair
// takes the retrievers (row t, slot s) of chunk j in list order through a
// two-slot LDS ring (Q_c and dO_c tiles plus the shifted-lse and D columns of
// slot s, which the query-stationary pass wrote), each wave owning 32 of chunk
// j's keys, so a workgroup's barrier couples only its two waves and no partial
// sums are exchanged.  With the shifted lse L = log2(e) lse - log2(w_s),
// exp2(S log2(e) scale - L) is w_s P_s directly.
//
// In fp32 (without the LMK row) a ring has one slot, copied between rounds: a tile pair is
// 32 KiB and a round's products take five times as long as in bf16, so a second slot
// hides little, while its LDS holds another pair (two waves per SIMD instead of one).
template <typename T, bool XR>
constexpr bool kOneSlot = sizeof(T) == 4 && !XR;

// PAIRS > 1 (kv_pairs): a workgroup of that many wave pairs, each with its own
// ring, pair i taking retrievers i, i + PAIRS, ...; the pairs' sums are added through LDS
// in pair order at the end.  A list is a chain of rounds (1.3 us each in bf16, 7 us in
// fp32), and causal problems have a few long ones (a slice's first chunks), so on a
// chip with room to spare the longest list is what a launch takes.
template <typename T, bool XR, int PAIRS>
__global__ __launch_bounds__(128 * PAIRS, (kOneSlot<T, XR> ? 2 : PAIRS == 1 ? 4 : PAIRS == 2 ? 2 : 1)) void bwd_dkdv_kernel(BwdParams p, int64_t nwork) {
  constexpr int kKvThreads = 128 * PAIRS;
  static_assert(PAIRS == 1 || !XR, "the LMK row staging assumes one pair");
  constexpr int TILE = kS * kD;
  constexpr int SQ = XR ? kS + 1 : kS;  // query rows per chunk
  // ring slot: Q_c tile, dO_c tile, shifted-lse column, D column; with the LMK
  // row also its Q and dO rows and its shifted lse and -D (16 bytes)
  constexpr int XOFF = 2 * TILE + 2 * kS * (int)(sizeof(float) / sizeof(T));
  constexpr int ENTRY = XOFF + (XR ? 2 * kD + 16 / (int)sizeof(T) : 0);
  // fp32 (without the LMK row): one ring slot, see kOneSlot
  constexpr int SLOTS = kOneSlot<T, XR> ? 1 : 2;
  __shared__ __attribute__((aligned(16))) T rings[PAIRS * SLOTS * ENTRY];
  constexpr int NE = 256;  // retrievers staged in LDS per batch
  __shared__ int sE[NE];
  // LMK rows: up to kXGroup retrievers' rows staged for one padded contraction
  // step: Q and dO rows transposed ([d][retriever]) and, per key, w P and dS
  // ([key][retriever])
  constexpr int kXGroup = 8;
  __shared__ __attribute__((aligned(16))) T sXst[XR ? 4 : 1][XR ? kD : 1][kXGroup];

  const int64_t wid = xcd_swizzle(blockIdx.x, gridDim.x);
  if (wid >= nwork) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5;
  const int half = PAIRS == 1 ? wave : wave & 1, pair = PAIRS == 1 ? 0 : wave >> 1;
  T* const ring = rings + pair * SLOTS * ENTRY;
  const int64_t j = wid % p.nKV;
  const int64_t bh = wid / p.nKV;
  const int h = (int)(bh % p.H);
  const int64_t b = bh / p.H;
  const int hr = p.Hr == 1 ? 0 : h;
  const int K = p.K;
  const int64_t bhr = b * p.Hr + hr;
  // the chunk's header row: lane i < kHeadInts holds int i
  const int hv = lane < kHeadInts ? p.ws.head[(bhr * p.nKV + j) * kHeadInts + lane] : 0;
  const int lo = __builtin_amdgcn_readlane(hv, 0), n = __builtin_amdgcn_readlane(hv, 1);
  const int* list_g = p.ws.sorted + bhr * p.nQ * K + lo;

  const int64_t key0 = (bh * p.nKV + j) * kS;  // first key token of chunk j
  T* dk = reinterpret_cast<T*>(p.dk) + key0 * kD;
  T* dv = reinterpret_cast<T*>(p.dv) + key0 * kD;
  if (n == 0) {
    for (int e = tid; e < kS * kD / 4; e += kKvThreads) {
      store4(dk + 4 * e, 0.f, 0.f, 0.f, 0.f);
      store4(dv + 4 * e, 0.f, 0.f, 0.f, 0.f);
    }
    return;
  }

  // this wave's 32 keys of chunk j as B operands (K^T, V^T columns)
  const int kr = 32 * half + (lane & 31);
  const T* krow = reinterpret_cast<const T*>(p.k) + (key0 + kr) * kD;
  const T* vrow = reinterpret_cast<const T*>(p.v) + (key0 + kr) * kD;
  Frag<T> kf[4], vf[4];
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    kf[kb] = load_frag(krow + 16 * kb + 8 * hh);
    vf[kb] = load_frag(vrow + 16 * kb + 8 * hh);
  }

  const int64_t lq_len = p.nQ * SQ;  // query tokens per (batch, head)
  const T* qb = reinterpret_cast<const T*>(p.q) + bh * lq_len * kD;
  const T* ob = reinterpret_cast<const T*>(p.dout) + bh * lq_len * kD;
  const float* Lb = p.ws.Lbuf + bh * lq_len * K;
  const float* Db = p.ws.Dbuf + bh * lq_len * K;

  const TileCopy<T, 2> cp(half, lane);
  const uint32_t col_off = (uint32_t)(lane * sizeof(float));
  constexpr int kXPieces = kD * (int)sizeof(T) / 16;  // 16-byte pieces of one row
  const int xw = __builtin_amdgcn_readfirstlane(half);  // LMK row copies: wave 0 Q and L, wave 1 dO and -D
  const T* const xrow_src = xw == 0 ? qb : ob;
  const float* const xcol_src = xw == 0 ? Lb : Db;
  auto enc = [&](int e) { return ((e / K + p.causal) << 5) | (e % K); };  // list entry t*K+s -> (query chunk << 5) | slot
  auto issue = [&](int slot, int cs) __device__ {
    const int64_t c = cs >> 5;
    const int s = cs & 31;
    T* dst = ring + slot * ENTRY;
    cp.issue(qb + c * SQ * kD, dst);
    cp.issue(ob + c * SQ * kD, dst + TILE);
    float* cols = reinterpret_cast<float*>(dst + 2 * TILE);
    if (half == 0) dma_column_s(Lb + s * lq_len + c * SQ, col_off, cols);
    else dma_column_s(Db + s * lq_len + c * SQ, col_off, cols + kS);
    if constexpr (XR) {
      // the LMK row (row S of the chunk): wave 0 its Q row and shifted lse, wave 1
      // its dO row and -D (addresses in scalar registers)
      const int64_t xr = c * SQ + kS;
      T* xdst = dst + XOFF;
      float* xcol = reinterpret_cast<float*>(xdst + 2 * kD);
      if (lane < kXPieces) dma_row16(xrow_src + xr * kD, lane * 16u, xdst + xw * kD);
      if (lane == 0) dma_column_s(xcol_src + s * lq_len + xr, 0u, xcol + xw);
    }
  };

  f32x16 dv0 = zero16(), dv1 = zero16(), dk0 = zero16(), dk1 = zero16();
  const float sc = p.attn_scale * kLog2e;
  const int cb = 16 * ((lane >> 4) & 1);

  // bf16 fragment addresses: this lane's byte offsets inside a ring slot, computed
  // once; a round adds its slot's offset and every fragment read is one of these
  // addresses plus an immediate (row +32, key block, dO tile, transposed-row gap)
  constexpr bool kB16 = std::is_same<T, __bf16>::value;
  constexpr uint32_t kTileB = TILE * sizeof(T), kRowB = kD * sizeof(T), kEntryB = ENTRY * sizeof(T);
  const lds_char* const lds0 = (const lds_char*)(rings) + (uint32_t)pair * SLOTS * kEntryB;
  const F32Offsets f32(lane);
  uint32_t rofs[4], tofs[2][2];
  {
    const int s16 = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) rofs[kb] = Swz<T>::off(lane & 31, 16 * kb + 8 * hh) * sizeof(T);
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        tofs[dh][r8] = Swz<T>::off(8 * r8 + 4 * hh + (s16 >> 2), 32 * dh + cb + 4 * (s16 & 3)) * sizeof(T);
  }
  auto row_frag = [&](uint32_t so, int kb, int half32) __device__ -> Frag<T> {
    if constexpr (kB16) {
      return lds_b128_at(lds0 + (rofs[kb] + so) + half32 * 32 * kRowB);
    } else {
      return f32.row_frag(lds0 + so, kb, half32);
    }
  };
  auto col_frag = [&](uint32_t so, int kb, int dh) __device__ -> Frag<T> {
    if constexpr (kB16) {
      return lds_tr2(lds0 + (tofs[dh][0] + so) + 16 * kb * kRowB, lds0 + (tofs[dh][1] + so) + 16 * kb * kRowB);
    } else {
      return f32.col_frag(lds0 + so, kb, dh);
    }
  };

  auto run = [&](int slot, int u, bool last) __device__ {
    const T* sQ = ring + slot * ENTRY;
    const T* sO = sQ + TILE;
    const uint32_t qo = (uint32_t)slot * kEntryB, oo = qo + kTileB;
    const float* sL = reinterpret_cast<const float*>(sQ + 2 * TILE);
    const float* sD = sL + kS;
    if constexpr (XR || !kB16) {
      // with the LMK row, and in fp32, the 64 queries go in two halves of 32, one after
      // the other (the same products in the same order per accumulator, half the
      // score and dP registers live at a time)
#pragma unroll
      for (int qh = 0; qh < 2; ++qh) {
        f32x16 pp, ss = zero16();
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 d0 = *reinterpret_cast<const f32x4*>(sD + 32 * qh + 8 * g + 4 * hh);
#pragma unroll
          for (int r = 0; r < 4; ++r) pp[4 * g + r] = d0[r];
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          mma32(ss, row_frag(qo, kb, qh), kf[kb]);
        }
#pragma unroll
        for (int kb = 0; kb < 4; ++kb) {
          mma32(pp, row_frag(oo, kb, qh), vf[kb]);
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
          const f32x4 l0 = *reinterpret_cast<const f32x4*>(sL + 32 * qh + 8 * g + 4 * hh);
#pragma unroll
          for (int r = 0; r < 4; ++r) ss[4 * g + r] = __builtin_amdgcn_exp2f(fmaf(ss[4 * g + r], sc, -l0[r]));
        }
        Frag<T> wp2[2], ds2[2];
        frag_from_acc(wp2[0], ss, 0, 1.f);
        frag_from_acc(wp2[1], ss, 1, 1.f);
#pragma unroll
        for (int i = 0; i < 16; ++i) pp[i] *= ss[i];
        frag_from_acc(ds2[0], pp, 0, 1.f);
        frag_from_acc(ds2[1], pp, 1, 1.f);
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          mma32(dv0, col_frag(oo, 2 * qh + kk, 0), wp2[kk]);
          mma32(dv1, col_frag(oo, 2 * qh + kk, 1), wp2[kk]);
        }
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
          mma32(dk0, col_frag(qo, 2 * qh + kk, 0), ds2[kk]);
          mma32(dk1, col_frag(qo, 2 * qh + kk, 1), ds2[kk]);
        }
      }
    } else {
      // accumulator row i of a 32-query tile holds query 32*qt + 8*(i/4) + 4*hh + i%4,
      // so four consecutive registers take one 16-byte column read.
      // dP - D = dO V^T + (-D): the accumulators start from the stored -D column
      f32x16 p0, p1;
  #pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 d0 = *reinterpret_cast<const f32x4*>(sD + 8 * g + 4 * hh);
        const f32x4 d1 = *reinterpret_cast<const f32x4*>(sD + 32 + 8 * g + 4 * hh);
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          p0[4 * g + r] = d0[r];
          p1[4 * g + r] = d1[r];
        }
      }
      // S = Q K^T for this wave's keys (queries 0-31 in s0, 32-63 in s1), and dP
      f32x16 s0 = zero16(), s1 = zero16();
  #pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        mma32(s0, row_frag(qo, kb, 0), kf[kb]);
        mma32(s1, row_frag(qo, kb, 1), kf[kb]);
      }
  #pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        mma32(p0, row_frag(oo, kb, 0), vf[kb]);
        mma32(p1, row_frag(oo, kb, 1), vf[kb]);
      }
      // w P (fp32), then dS = w P o (dP - D)
  #pragma unroll
      for (int g = 0; g < 4; ++g) {
        const f32x4 l0 = *reinterpret_cast<const f32x4*>(sL + 8 * g + 4 * hh);
        const f32x4 l1 = *reinterpret_cast<const f32x4*>(sL + 32 + 8 * g + 4 * hh);
  #pragma unroll
        for (int r = 0; r < 4; ++r) {
          s0[4 * g + r] = __builtin_amdgcn_exp2f(fmaf(s0[4 * g + r], sc, -l0[r]));
          s1[4 * g + r] = __builtin_amdgcn_exp2f(fmaf(s1[4 * g + r], sc, -l1[r]));
        }
      }
      Frag<T> wp[4], ds[4];
      frag_from_acc(wp[0], s0, 0, 1.f);
      frag_from_acc(wp[1], s0, 1, 1.f);
      frag_from_acc(wp[2], s1, 0, 1.f);
      frag_from_acc(wp[3], s1, 1, 1.f);
  #pragma unroll
      for (int i = 0; i < 16; ++i) {
        p0[i] *= s0[i];
        p1[i] *= s1[i];
      }
      frag_from_acc(ds[0], p0, 0, 1.f);
      frag_from_acc(ds[1], p0, 1, 1.f);
      frag_from_acc(ds[2], p1, 0, 1.f);
      frag_from_acc(ds[3], p1, 1, 1.f);
      // dV^T += dO^T (w P) and dK^T += Q^T dS  (contractions over the 64 queries)
  #pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        mma32(dv0, col_frag(oo, kb, 0), wp[kb]);
        mma32(dv1, col_frag(oo, kb, 1), wp[kb]);
      }
  #pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        mma32(dk0, col_frag(qo, kb, 0), ds[kb]);
        mma32(dk1, col_frag(qo, kb, 1), ds[kb]);
      }
    }
    if constexpr (XR) {
      // the LMK row against this wave's keys, after the tile's products (so its
      // registers do not add to theirs): its score and dP for key kr (row
      // fragments of K and V held in registers, the dimension halves added
      // across l ^ 32), w P and dS, staged with the row's Q and dO as retriever
      // u % kXGroup; every kXGroup retrievers (and at the end of a batch) the
      // staged rows enter dV^T += dO_X^T (w P_X) and dK^T += Q_X^T dS_X as one
      // contraction step padded to 16 with zeros
      __builtin_amdgcn_sched_barrier(0);
      const T* sqx = sQ + XOFF;
      const T* sdx = sqx + kD;
      const float* slx = reinterpret_cast<const float*>(sdx + kD);
      float a = 0.f, b = 0.f;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        a = frag_dot(kf[kb], vec_frag(sqx, 16 * kb + 8 * hh), a);
        b = frag_dot(vf[kb], vec_frag(sdx, 16 * kb + 8 * hh), b);
      }
      a = sum_xor32(a);
      b = sum_xor32(b);
      const float wpx = __builtin_amdgcn_exp2f(fmaf(a, sc, -slx[0]));
      const float xd = wpx * (b + slx[1]);
      const int e = u % kXGroup;
      if (hh == 0) {
        sXst[2][kr][e] = (T)wpx;
        sXst[3][kr][e] = (T)xd;
      }
      sXst[half][lane][e] = (half == 0 ? sqx : sdx)[lane];  // wave 0 the Q row, wave 1 the dO row
      if (e == kXGroup - 1 || last) {
        block_barrier();
        __builtin_amdgcn_sched_barrier(0);
        const int filled = e + 1, r = lane & 31;
        Frag<T> ad0 = zero_frag<T>(), ad1 = ad0, aq0 = ad0, aq1 = ad0, bp = ad0, bs = ad0;
        if (hh == 0) {
          // entries past `filled` hold an earlier group's values or bits never
          // written: both operands are cut to the filled ones (0 * NaN is NaN)
          ad0 = frag_prefix<T>(load_frag(&sXst[1][r][0]), filled);
          ad1 = frag_prefix<T>(load_frag(&sXst[1][32 + r][0]), filled);
          aq0 = frag_prefix<T>(load_frag(&sXst[0][r][0]), filled);
          aq1 = frag_prefix<T>(load_frag(&sXst[0][32 + r][0]), filled);
          bp = frag_prefix<T>(load_frag(&sXst[2][kr][0]), filled);
          bs = frag_prefix<T>(load_frag(&sXst[3][kr][0]), filled);
        }
        mma32(dv0, ad0, bp);
        mma32(dv1, ad1, bp);
        mma32(dk0, aq0, bs);
        mma32(dk1, aq1, bs);
      }
    }
  };

  // the retriever list is staged through LDS in batches, each streamed through
  // the ring (one item in flight ahead of the compute) and drained at its end.
  // The first batch: its first copy straight from the header, its first entries
  // from the header and the rest from the list, in flight with that copy and the
  // K/V fragments (round 0's barrier makes them visible)
  for (int b0 = 0; b0 < n; b0 += NE) {
    const int nb = min(NE, n - b0);
    const int mine = pair < nb ? (nb - pair + PAIRS - 1) / PAIRS : 0;  // this pair's items of the batch
    if (b0 == 0) {
      static_assert(PAIRS <= kHeadEntries, "every pair's first item is in the header");
      if (PAIRS == 1 || mine > 0) issue(0, enc(__builtin_amdgcn_readlane(hv, 2 + pair)));
      const int e_head = __shfl(hv, (lane + 2) & 63);  // lane i: header entry i
      if (wave == 0 && lane < kHeadEntries && lane < nb) sE[lane] = enc(e_head);
      for (int i = kHeadEntries + tid; i < nb; i += kKvThreads) sE[i] = enc(list_g[i]);
    } else {
      __syncthreads();
      for (int i = tid; i < nb; i += kKvThreads) sE[i] = enc(list_g[b0 + i]);
      __syncthreads();
      if (PAIRS == 1 || mine > 0) issue(0, sE[pair]);
    }
    const int rounds = (nb + PAIRS - 1) / PAIRS;  // the first pair's items: every pair meets its barriers
    for (int u = 0; u < rounds; ++u) {
      if (SLOTS == 1 && u > 0) {
        block_barrier();  // both waves have read the slot
        if (u < mine) issue(0, sE[u * PAIRS + pair]);
      }
      wait_vmem<0>();
      block_barrier();
      if (SLOTS == 2 && u + 1 < mine) issue((u + 1) & 1, sE[(u + 1) * PAIRS + pair]);
      if (PAIRS == 1 || u < mine) run(SLOTS == 2 ? u & 1 : 0, u, u + 1 == nb);
    }
  }
  if constexpr (PAIRS > 1) {
    // the other pairs' sums into the first's, in pair order (the rings are free: every
    // copy has been waited for)
    float* part = reinterpret_cast<float*>(rings);
    static_assert(sizeof(rings) >= (PAIRS - 1) * 2 * 64 * 64 * sizeof(float), "partial sums fit in the rings");
    auto each = [&](auto f) {
#pragma unroll
      for (int i = 0; i < 16; ++i) {
        f(dv0, i, i);
        f(dv1, i, 16 + i);
        f(dk0, i, 32 + i);
        f(dk1, i, 48 + i);
      }
    };
    __syncthreads();
    if (pair > 0)
      each([&](f32x16& v, int i, int r) { part[(((pair - 1) * 2 + half) * 64 + r) * 64 + lane] = v[i]; });
    __syncthreads();
    if (pair > 0) return;
    for (int q = 0; q < PAIRS - 1; ++q)
      each([&](f32x16& v, int i, int r) { v[i] += part[((q * 2 + half) * 64 + r) * 64 + lane]; });
  }

  // accumulators are transposed: lane holds key kr, d = 32*dt + 8*g + 4*hh + 0..3
  const float as = p.attn_scale;
  T* dkr = dk + kr * kD;
  T* dvr = dv + kr * kD;
#pragma unroll
  for (int g = 0; g < 4; ++g) {
    store4(dvr + 8 * g + 4 * hh, dv0[4 * g], dv0[4 * g + 1], dv0[4 * g + 2], dv0[4 * g + 3]);
    store4(dvr + 32 + 8 * g + 4 * hh, dv1[4 * g], dv1[4 * g + 1], dv1[4 * g + 2], dv1[4 * g + 3]);
    store4(dkr + 8 * g + 4 * hh, as * dk0[4 * g], as * dk0[4 * g + 1], as * dk0[4 * g + 2], as * dk0[4 * g + 3]);
    store4(dkr + 32 + 8 * g + 4 * hh, as * dk1[4 * g], as * dk1[4 * g + 1], as * dk1[4 * g + 2],
           as * dk1[4 * g + 3]);
  }
}

// -------------------------------------- score and landmark gradients ----

// dw[t, s] of one row: the per-head, per-wave-half partials summed over the
// group's heads as kDwClasses interleaved classes (head h in class (h - h0) mod
// kDwClasses), each class summed in head order and the classes added in class
// order, so that both kernels that form dsel round identically.
constexpr int kDwClasses = 8;
__device__ __forceinline__ float dw_class(const float* __restrict__ dwp, int64_t b, int64_t t, int s, int H, int Hr,
                                          int hr, int64_t nQ, int K, int cls) {
  const int h0 = Hr == 1 ? 0 : hr, h1 = Hr == 1 ? H : hr + 1;
  float acc = 0.f;
  for (int h = h0 + cls; h < h1; h += kDwClasses) {
    const float* d2 = dwp + (((b * H + h) * nQ + t) * K + s) * 2;
    acc += d2[0] + d2[1];
  }
  return acc;
}

// dsel[t, s] = w_s (dw_s - sum_s' w_s' dw_s'), dw summed over the group's heads.
__global__ __launch_bounds__(64) void dsel_kernel(const float* __restrict__ w, const float* __restrict__ dwp,
                                                  float* __restrict__ dsel, int64_t nQ, int H, int Hr, int K,
                                                  int causal) {
  const int64_t row = blockIdx.x;  // (b, hr, t)
  const int64_t t = row % nQ;
  const int64_t bhr = row / nQ;
  const int64_t b = bhr / Hr;
  const int hr = (int)(bhr % Hr);
  const int s = threadIdx.x;
  float dw = 0.f, ws = 0.f;
  if (s < K) {
    ws = w[row * K + s];
    if (t + causal < nQ) {
      for (int c = 0; c < kDwClasses; ++c) dw += dw_class(dwp, b, t, s, H, Hr, hr, nQ, K, c);
    }
  }
  float tot = ws * dw;
  tot = sum64(tot);
  if (s < K) dsel[row * K + s] = ws * (dw - tot);
}

// Weighted sum of gathered landmark rows by a team of NT threads (a workgroup, or one
// wave of it):
//   out[x] = scale * sum_u w_u src[off_u + x],  x < D,
// for the n (row offset, weight) pairs staged in sOff / sW.  A thread owns a 16-byte
// column block and a residue class of u (the groups), so every load is an
// independent 16-byte read; the groups' partial sums are added in a fixed order
// (deterministic).  256 threads keep four reads in flight each; 64 threads, with a
// quarter of the groups, 8 or 16.
constexpr int kMaxGatherPasses = 8;  // D <= 8192: at most 8 passes of 256 blocks (fp32); one pass of 64 threads

// column blocks per pass and retriever groups
struct GatherShape {
  int pass_cols, groups;
};
inline GatherShape gather_shape(int D, int elem_bytes, int threads) {
  const int nb = D / (16 / elem_bytes);
  GatherShape g;
  g.pass_cols = nb < threads ? nb : threads;
  g.groups = threads / g.pass_cols;
  return g;
}

template <typename T>
__device__ __forceinline__ float elem16(const u32x4& r, int m) {
  if constexpr (sizeof(T) == 2) return __uint_as_float((m & 1) ? (r[m >> 1] & 0xffff0000u) : (r[m >> 1] << 16));
  else return __uint_as_float(r[m]);
}

// N entries of one thread's residue class from u on; entries past the list add nothing.
template <int N, typename T>
__device__ __forceinline__ void gather_batch(const T* __restrict__ src, const int64_t* sOff, const float* sW, int n,
                                             int u, int step, bool active, float (&acc)[16 / sizeof(T)]) {
  constexpr int V = 16 / sizeof(T);
  u32x4 f[N];
  float w[N];
#pragma unroll
  for (int i = 0; i < N; ++i) {
    const int at = min(u + i * step, n - 1);
    f[i] = *reinterpret_cast<const u32x4*>(src + sOff[at]);
    w[i] = sW[at];
  }
#pragma unroll
  for (int i = 0; i < N; ++i)
    if (active && u + i * step < n)
#pragma unroll
      for (int m = 0; m < V; ++m) acc[m] += w[i] * elem16<T>(f[i], m);
}

template <typename T, int NT, int PASSES>
__device__ __forceinline__ void gather_rows(const T* __restrict__ src, int D, const int64_t* sOff, const float* sW,
                                            int n, float (&acc)[PASSES][16 / sizeof(T)], GatherShape gs) {
  constexpr int V = 16 / sizeof(T);
  const int tid = threadIdx.x % NT, cb = tid % gs.pass_cols, grp = tid / gs.pass_cols, groups = gs.groups;
  const int nb = D / V;
  if constexpr (NT == 64) {
    static_assert(PASSES == 1, "one wave covers a row");
    for (int u0 = 0; u0 < n; u0 += 8 * groups)
      gather_batch<8>(src + cb * V, sOff, sW, n, u0 + grp, groups, grp < groups, acc[0]);
    return;
  }
  auto ld = [&](int u, int b) { return *reinterpret_cast<const u32x4*>(src + sOff[u] + b * V); };
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int b = pass * gs.pass_cols + cb;
    if (pass * gs.pass_cols >= nb) break;
    if (grp < groups && b < nb) {
      int u = grp;
      for (; u + 3 * groups < n; u += 4 * groups) {
        const u32x4 f0 = ld(u, b), f1 = ld(u + groups, b), f2 = ld(u + 2 * groups, b), f3 = ld(u + 3 * groups, b);
        const float w0 = sW[u], w1 = sW[u + groups], w2 = sW[u + 2 * groups], w3 = sW[u + 3 * groups];
#pragma unroll
        for (int m = 0; m < V; ++m)
          acc[pass][m] += w0 * elem16<T>(f0, m) + w1 * elem16<T>(f1, m) + w2 * elem16<T>(f2, m) +
                          w3 * elem16<T>(f3, m);
      }
      for (; u < n; u += groups) {
        const u32x4 f0 = ld(u, b);
#pragma unroll
        for (int m = 0; m < V; ++m) acc[pass][m] += sW[u] * elem16<T>(f0, m);
      }
    }
  }
}

// LDS written by the team is visible to it.
template <int NT>
__device__ __forceinline__ void gather_sync() {
  if constexpr (NT == 64) wave_lds_order();
  else __syncthreads();
}

template <typename T, int NT, int PASSES>
__device__ __forceinline__ void gather_store(float* __restrict__ out, int D, float scale, float* sAcc,
                                             float (&acc)[PASSES][16 / sizeof(T)], GatherShape gs) {
  constexpr int V = 16 / sizeof(T);
  const int tid = threadIdx.x % NT, cb = tid % gs.pass_cols, grp = tid / gs.pass_cols, groups = gs.groups;
  const int nb = D / V;
#pragma unroll
  for (int pass = 0; pass < PASSES; ++pass) {
    const int b = pass * gs.pass_cols + cb;
    if (pass * gs.pass_cols >= nb) break;
    gather_sync<NT>();
    if (grp < groups && b < nb)
#pragma unroll
      for (int m = 0; m < V; ++m) sAcc[(grp * gs.pass_cols + cb) * V + m] = acc[pass][m];
    gather_sync<NT>();
    if (grp == 0 && b < nb) {
      float r[V];
#pragma unroll
      for (int m = 0; m < V; ++m) r[m] = sAcc[cb * V + m];
      for (int g = 1; g < groups; ++g)
#pragma unroll
        for (int m = 0; m < V; ++m) r[m] += sAcc[(g * gs.pass_cols + cb) * V + m];
#pragma unroll
      for (int m = 0; m < V; m += 4)
        store4(out + b * V + m, scale * r[m], scale * r[m + 1], scale * r[m + 2], scale * r[m + 3]);
    }
  }
}

// dlmk_q[t] = score_scale * sum_s dsel[t, s] lmk_k[idx[t, s]]
// The row's dsel (as dsel_kernel computes it, the same summation order) is
// formed here and written out, so the backward needs no separate dsel launch
// when the landmark-query gradient is wanted: all threads read the head
// classes of the dw partials, and the first wave forms dsel.
template <typename T, int NT>
__global__ __launch_bounds__(NT) void dlmk_q_kernel(const T* __restrict__ lk, const int32_t* __restrict__ idx,
                                                     const float* __restrict__ w, const float* __restrict__ dwp,
                                                     float* __restrict__ dsel, float* __restrict__ dlq,
                                                     int64_t nQ, int64_t nKV, int D, int K, int H, int Hr,
                                                     int causal, float scale, GatherShape gs) {
  constexpr int V = 16 / sizeof(T), PASSES = NT == 64 ? 1 : kMaxGatherPasses;
  __shared__ int64_t sOff[32];
  __shared__ float sW[32];
  __shared__ int sN;
  __shared__ float sAcc[NT * 8];
  __shared__ float sCls[kDwClasses][32];
  const int64_t row = blockIdx.x;
  const int64_t bhr = row / nQ;
  const int64_t t = row % nQ;
  const int64_t b = bhr / Hr;
  const int hr = (int)(bhr % Hr);
  {
    // the dw partials of every head are read by all threads at once: thread
    // (class c, slot s) sums head class c of slot s
    const int s = threadIdx.x & 31;
#pragma unroll
    for (int c = threadIdx.x >> 5; c < kDwClasses; c += NT / 32)
      sCls[c][s] = (s < K && t + causal < nQ) ? dw_class(dwp, b, t, s, H, Hr, hr, nQ, K, c) : 0.f;
  }
  __syncthreads();
  if (threadIdx.x < 64) {
    const int s = threadIdx.x;
    float dw = 0.f, ws = 0.f;
    if (s < K) {
      ws = w[row * K + s];
      for (int c = 0; c < kDwClasses; ++c) dw += sCls[c][s];
    }
    const float tot = sum64(ws * dw);
    const float ds = ws * (dw - tot);
    if (s < K) dsel[row * K + s] = ds;
    const int j = s < K ? idx[row * K + s] : -1;
    const bool ok = j >= 0 && j < nKV;
    const uint64_t mask = __ballot(ok);
    if (ok) {
      const int rk = __popcll(mask & ((1ull << s) - 1));
      sOff[rk] = (bhr * nKV + j) * D;
      sW[rk] = ds;
    }
    if (s == 0) sN = __popcll(mask);
  }
  __syncthreads();
  float acc[PASSES][V];
  for (int q = 0; q < PASSES; ++q)
    for (int m = 0; m < V; ++m) acc[q][m] = 0.f;
  gather_rows<T, NT>(lk, D, sOff, sW, sN, acc, gs);
  gather_store<T, NT>(dlq + row * D, D, scale, sAcc, acc, gs);
}

// dlmk_k[j] = score_scale * sum over the rows (t, s) that retrieved j of dsel[t, s] lmk_q[t],
// in (t, s) order within each group of the list, by a team of NT threads.
template <typename T, int NT, int PASSES>
__device__ __forceinline__ void dlmk_k_row(const T* __restrict__ lq, const int* __restrict__ sorted,
                                           const float* __restrict__ dsel, float* __restrict__ dlk, int64_t nQ,
                                           int D, int K, float scale, int64_t row, uint32_t slice, int lo, int hi,
                                           int64_t* sOff, float* sW, float* sAcc, GatherShape gs) {
  constexpr int V = 16 / sizeof(T);
  const int tid = threadIdx.x % NT;
  const int64_t q0 = slice * nQ;  // the slice's first landmark row
  float acc[PASSES][V];
  for (int q = 0; q < PASSES; ++q)
    for (int m = 0; m < V; ++m) acc[q][m] = 0.f;
  for (int b0 = lo; b0 < hi; b0 += NT) {
    const int nb = min(NT, hi - b0);
    gather_sync<NT>();
    if (tid < nb) {
      const int e = sorted[q0 * K + b0 + tid];  // t * K + s
      sOff[tid] = (q0 + e / K) * D;
      sW[tid] = dsel[q0 * K + e];
    }
    gather_sync<NT>();
    gather_rows<T, NT>(lq, D, sOff, sW, nb, acc, gs);
  }
  gather_store<T, NT>(dlk + row * D, D, scale, sAcc, acc, gs);
}

// One row (b, hr, j) per workgroup (rows fit 31 bits).
template <typename T>
__global__ __launch_bounds__(256) void dlmk_k_kernel(const T* __restrict__ lq, const int* __restrict__ offs,
                                                     const int* __restrict__ sorted, const float* __restrict__ dsel,
                                                     float* __restrict__ dlk, int64_t nQ, uint32_t nKV, int D, int K,
                                                     float scale, GatherShape gs) {
  __shared__ int64_t sOff[256];
  __shared__ float sW[256];
  __shared__ float sAcc[256 * 8];
  const int64_t row = blockIdx.x;
  const uint32_t slice = blockIdx.x / nKV;
  const int* off = offs + row + slice;  // (nKV + 1 offsets per slice)
  dlmk_k_row<T, 256, kMaxGatherPasses>(lq, sorted, dsel, dlk, nQ, D, K, scale, row, slice, off[0], off[1], sOff, sW,
                                       sAcc, gs);
}

// Landmarks of at most 64 column blocks, many rows (dlmk_k_waves): each wave of a
// workgroup takes a row of its own, except rows with long lists, which the four waves
// then take together.  The workgroup's rows lie a quarter of all rows apart, shifted
// against each other, so that the hot chunks of a slice, and the first ones of several
// slices, fall to different workgroups.
template <typename T>
__global__ __launch_bounds__(256, 4) void dlmk_k_rows_kernel(const T* __restrict__ lq, const int* __restrict__ offs,
                                                          const int* __restrict__ sorted,
                                                          const float* __restrict__ dsel, float* __restrict__ dlk,
                                                          uint32_t rows, int64_t nQ, uint32_t nKV, int D, int K,
                                                          float scale, GatherShape one, GatherShape four) {
  __shared__ int64_t sOff[256];
  __shared__ float sW[256];
  __shared__ float sAcc[256 * 8];
  const int wave = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));
  const uint32_t G = gridDim.x;
  const int longest = 32 * one.groups;  // of a list that one wave takes
  uint32_t row[4], slice[4];
  int lo[4], n[4];
#pragma unroll
  for (int w = 0; w < 4; ++w) {
    uint32_t x = blockIdx.x + 37 * w;
    while (x >= G) x -= G;
    row[w] = min(w * G + x, rows - 1);
    slice[w] = row[w] / nKV;
    const int* off = offs + row[w] + slice[w];
    lo[w] = off[0];
    n[w] = w * G + x < rows ? off[1] - lo[w] : -1;  // -1: no such row
  }
  uint32_t own = row[0], own_slice = slice[0];
  int own_lo = lo[0], own_n = n[0];
#pragma unroll
  for (int w = 1; w < 4; ++w)
    if (wave == w) {
      own = row[w];
      own_slice = slice[w];
      own_lo = lo[w];
      own_n = n[w];
    }
  if (own_n >= 0 && own_n <= longest)
    dlmk_k_row<T, 64, 1>(lq, sorted, dsel, dlk, nQ, D, K, scale, own, own_slice, own_lo, own_lo + own_n,
                         sOff + 64 * wave, sW + 64 * wave, sAcc + 512 * wave, one);
  if (max(max(n[0], n[1]), max(n[2], n[3])) <= longest) return;
#pragma unroll 1
  for (int w = 0; w < 4; ++w) {
    auto pick = [&](auto& a) { return w == 0 ? a[0] : w == 1 ? a[1] : w == 2 ? a[2] : a[3]; };
    if (pick(n) > longest) {
      __syncthreads();
      dlmk_k_row<T, 256, 1>(lq, sorted, dsel, dlk, nQ, D, K, scale, pick(row), pick(slice), pick(lo),
                            pick(lo) + pick(n), sOff, sW, sAcc, four);
    }
  }
}

// Landmark gradients one wave per row: where a wave covers a row and the rows fill the
// chip many times over, what counts is the rows in flight; below, a row's own chain of
// reads and sums, which a workgroup shortens (the more, the wider the row).  A workgroup /
// a wave per row, bf16, k = 8: dlmk_q 2,048 rows of width 64 9.0 / 4.7 us, of 512 8.4 / 5.4,
// 11,200 of 64 (k = 16) 46 / 12; 500 rows with 16 heads' classes to add 4.9 / 6.2.  dlmk_k
// 1,400 rows of width 64 7.9 / 5.0, of 256 6.9 / 7.3; 2,048 of 256 9.6 / 7.7, of 512
// 10.4 / 11.4; 4,000 of 512 20.4 / 12.5; 11,200 of 64 (k = 16) 50 / 18.  A list of 1,000
// on one wave took 22 us at width 64 and 96 at 512, on four 11.5 and 36.
inline bool dlmk_q_waves(int64_t rows, int D, int elem_bytes) {
  return D * elem_bytes <= 64 * 16 && rows >= 4 * (int64_t)device_cus();
}
inline bool dlmk_k_waves(int64_t rows, int D, int elem_bytes) {
  const int blocks = D * elem_bytes / 16;  // 16-byte column blocks
  return dlmk_q_waves(rows, D, elem_bytes) && rows * 16 >= blocks * (int64_t)device_cus() * 3;
}

template <typename T>
hipError_t launch_bwd_t(const Shape& s, BwdParams& p, float* dsel, const void* lmk_q, const void* lmk_k,
                        float* dlmk_q, float* dlmk_k, hipStream_t st) {
  const int64_t BHr = (int64_t)s.B * s.Hr, BH = (int64_t)s.B * s.H;
  BwdWs& w = p.ws;
  if (!s.causal || s.nQ * s.topk <= kPrepEntries) {
    // (decode has one landmark row: the groups of its past cover it too)
    const int per = prep_chunks(s.nKV, s.topk);
    const int64_t groups = (s.nKV + per - 1) / per;
    launch_kernel("bwd_prep_kernel", bwd_prep_kernel, dim3((unsigned)(BHr * groups)), dim3(kPrepThreads), 0, st,
                  p.idx, p.sel, w, s.nQ, s.topk, s.nKV, s.causal, per, groups);
  } else {
    const dim3 ent((unsigned)((BHr * s.nQ * s.topk + 255) / 256)), chunks((unsigned)((BHr * s.nKV + 3) / 4));
    launch_kernel("bwd_prep_clear_kernel", bwd_prep_clear_kernel,
                  dim3((unsigned)std::min<int64_t>((BHr * s.nKV + 255) / 256, 4096)), dim3(256), 0, st, w.sorted, BHr,
                  s.nQ, s.topk, s.nKV);
    launch_kernel("bwd_prep_count_kernel", bwd_prep_count_kernel, ent, dim3(256), 0, st, p.idx, p.sel, w, BHr, s.nQ,
                  s.topk, s.nKV, s.causal);
    launch_kernel("bwd_prep_scan_kernel", bwd_prep_scan_kernel, dim3((unsigned)BHr), dim3(kPrepScan), 0, st, w, s.nQ,
                  s.topk, s.nKV);
    launch_kernel("bwd_prep_fill_kernel", bwd_prep_fill_kernel, ent, dim3(256), 0, st, p.idx, w, BHr, s.nQ, s.topk,
                  s.nKV, s.causal);
    launch_kernel("bwd_prep_sort_kernel", bwd_prep_sort_kernel, chunks, dim3(256), 0, st, w, BHr, s.nQ, s.topk,
                  s.nKV);
  }
  const int64_t nq_work = BH * s.nQ, nk_work = BH * s.nKV;
  // persistent: kWgPerCu workgroups per CU, kPairs chunk streams each
  const int64_t dq_wgs =
      std::min<int64_t>(round8((int64_t)device_cus() * kWgPerCu), round8((nq_work + kPairs - 1) / kPairs));
  const bool xr = s.Sq != kS;  // LMK row per query chunk
  auto dq = [&](auto kernel) {
    launch_kernel("bwd_dq_kernel", kernel, dim3((unsigned)dq_wgs), dim3(kThreads), 0, st, p, nq_work);
  };
  constexpr bool kB16 = sizeof(T) == 2;
  const int q_pairs = xr ? 1 : q_pairs_of(nq_work, s.topk, kB16), k_pairs = xr ? 1 : kv_pairs(nk_work, s.topk, kB16);
  if (q_pairs > 1)
    launch_kernel("bwd_dq_kernel", q_pairs == 4 ? bwd_dq_few_kernel<T, 4> : bwd_dq_few_kernel<T, kB16 ? 2 : 4>,
                  dim3((unsigned)nq_work), dim3(128 * q_pairs), 0, st, p);
  else if (s.topk <= kDqStageK)
    xr ? dq(bwd_dq_kernel<T, true, true>) : dq(bwd_dq_kernel<T, true, false>);
  else
    xr ? dq(bwd_dq_kernel<T, false, true>) : dq(bwd_dq_kernel<T, false, false>);
  auto kv = [&](auto kernel, int pairs) {
    launch_kernel("bwd_dkdv_kernel", kernel, dim3((unsigned)round8(nk_work)), dim3(128 * pairs), 0, st, p, nk_work);
  };
  if (xr) kv(bwd_dkdv_kernel<T, true, 1>, 1);
  else if (k_pairs == 4) kv(bwd_dkdv_kernel<T, false, 4>, 4);
  else if (k_pairs == 2) kv(bwd_dkdv_kernel<T, false, 2>, 2);
  else kv(bwd_dkdv_kernel<T, false, kB16 ? 1 : 2>, kB16 ? 1 : 2);
  if (dlmk_q) {
    // dsel is formed inside the landmark-query gradient kernel
    const bool waves = dlmk_q_waves(BHr * s.nQ, s.D, sizeof(T));
    launch_kernel("dlmk_q_kernel", waves ? dlmk_q_kernel<T, 64> : dlmk_q_kernel<T, 256>, dim3((unsigned)(BHr * s.nQ)),
                  dim3(waves ? 64 : 256), 0, st, (const T*)lmk_k, p.idx, w.w, w.dwp, dsel, dlmk_q, s.nQ, s.nKV, s.D,
                  s.topk, s.H, s.Hr, s.causal, s.score_scale, gather_shape(s.D, sizeof(T), waves ? 64 : 256));
  } else {
    launch_kernel("dsel_kernel", dsel_kernel, dim3((unsigned)(BHr * s.nQ)), dim3(64), 0, st, w.w, w.dwp, dsel,
                  s.nQ, s.H, s.Hr, s.topk, s.causal);
  }
  if (dlmk_k) {
    const int64_t rows = BHr * s.nKV;
    if (dlmk_k_waves(rows, s.D, sizeof(T)))
      launch_kernel("dlmk_k_kernel", dlmk_k_rows_kernel<T>, dim3((unsigned)((rows + 3) / 4)), dim3(256), 0, st,
                    (const T*)lmk_q, w.offs, w.sorted, dsel, dlmk_k, (uint32_t)rows, s.nQ, (uint32_t)s.nKV, s.D, s.topk,
                    s.score_scale, gather_shape(s.D, sizeof(T), 64), gather_shape(s.D, sizeof(T), 256));
    else
      launch_kernel("dlmk_k_kernel", dlmk_k_kernel<T>, dim3((unsigned)rows), dim3(256), 0, st, (const T*)lmk_q, w.offs,
                    w.sorted, dsel, dlmk_k, s.nQ, (uint32_t)s.nKV, s.D, s.topk, s.score_scale,
                    gather_shape(s.D, sizeof(T), 256));
  }
  return take_launch_error();
}

}  // namespace

hipError_t launch_xattn_bwd(const Shape& s, const void* q, const void* k, const void* v, const int32_t* idx,
                            const float* sel, const float* lse, const void* dout, void* dq, void* dk, void* dv,
                            float* dsel, const void* lmk_q, const void* lmk_k, float* dlmk_q, float* dlmk_k,
                            void* ws, hipStream_t stream) {
  BwdParams p;
  p.q = q; p.k = k; p.v = v; p.idx = idx; p.sel = sel; p.lse = lse; p.dout = dout;
  p.dq = dq; p.dk = dk; p.dv = dv;
  p.ws = bwd_carve(s, ws);
  p.B = s.B; p.H = s.H; p.Hr = s.Hr; p.K = s.topk;
  p.nQ = s.nQ; p.nKV = s.nKV;
  p.causal = s.causal;
  p.attn_scale = s.attn_scale;
  p.windows = use_window_order(s.nKV, s.bf16 ? 2 : 4);
  return s.bf16 ? launch_bwd_t<__bf16>(s, p, dsel, lmk_q, lmk_k, dlmk_q, dlmk_k, stream)
                : launch_bwd_t<float>(s, p, dsel, lmk_q, lmk_k, dlmk_q, dlmk_k, stream);
}

}  // namespace gca
