// Grouped cross attention forward (Eq. 2-3 of the method; Algorithm 1 in the
// appendix is its tiled form).
//
// Persistent workgroups of one wave pair, four per CU: each pair is a stream of
// (batch, head, query chunk) work items, and within a pair each wave owns 32 of
// the chunk's 64 query tokens and keeps their Q fragments in registers.  A pair
// takes its chunk's retrieved chunks one per round; their keys and values stream
// through the pair's two LDS ring slots, filled by asynchronous direct-to-LDS
// copies one round ahead of the compute (two waves per SIMD hide each other's
// MFMA, LDS and cross-lane latencies).  For every retrieved chunk (slot) a wave
// computes S^T = K Q^T on the matrix cores, takes each query's softmax over the
// 64 keys (one retrieved chunk is exactly one tile, so no running rescale is
// needed), folds the fusion weight w_s / l_s into P, and accumulates
// O^T += V^T (w_s P_s)^T in registers; at the end of the chunk each wave stores
// its rows.  The per-chunk outputs O'_s of Algorithm 1 are never written; the
// log-sum-exp of every (row, slot) is.
//
// Computing the transposed products keeps every query's statistics inside one
// lane (query = accumulator column): the softmax needs one cross-lane step, and
// the probability tile feeds the PV product straight from registers.  V^T
// fragments come from the row-major V tile through LDS transpose reads.
//
// With an LMK row per chunk (S + 1 query rows), the 65th row meets the same
// tiles: one wave per slot (the waves alternate) takes it as a vector against
// the K and V^T fragments it already holds, with one key per lane for the
// softmax, and the waves' partial outputs are added through LDS at the end of
// the chunk.
#include "gca_device.hpp"
#include "gca_launch.hpp"

#include <type_traits>

namespace gca {
namespace {

// wave pairs per workgroup: one, so that a round's barrier couples only the two
// waves that share a ring; four workgroups per CU
constexpr int kPairs = 1;
constexpr int kThreads = 128 * kPairs;
constexpr int kWgPerCu = 4 / kPairs;

struct FwdParams {
  const void* q;
  const void* k;
  const void* v;
  const int32_t* idx;
  const float* sel;
  void* out;
  float* lse;
  float* w;
  int H, Hr, topk;
  int64_t nQ, nKV, nwork;
  int causal;
  float attn_scale;
  bool windows;  // stream order (StreamOrder)
};

// the LMK row's per-chunk exchange between the two waves of a pair
template <typename T>
struct LmkShared {
  T q[2][kD];       // the row's queries, by chunk parity
  T p[2][kS];       // per wave: the current slot's weighted probabilities (one per key)
  float o[2][kD];   // per wave: its slots' share of the row's output
  float lse[32];    // per slot: the row's log-sum-exp
};

// Per-lane retrieval metadata of one landmark row: lane s < K holds slot s's
// chunk index and raw score (chunk -1 for lanes >= K or rows that do not exist).
struct RowMeta {
  int j;
  float sv;
};

__device__ __forceinline__ RowMeta load_row_meta(const FwdParams& p, int64_t row_off, bool exists) {
  const int lane = threadIdx.x & 63;
  RowMeta m{-1, -INFINITY};
  if (exists && lane < p.topk) {
    m.j = p.idx[row_off + lane];
    m.sv = p.sel[row_off + lane];
  }
  return m;
}

template <typename T, bool OBO, bool XR, bool ONE>
__global__ __launch_bounds__(kThreads, (ONE ? 2 : kWgPerCu)) void xattn_fwd_kernel(FwdParams p) {
  static_assert(!ONE || (sizeof(T) == 4 && !XR), "one ring slot is for fp32 without the LMK row");
  constexpr int TILE = kS * kD;
  constexpr int SQ = XR ? kS + 1 : kS;  // query rows per chunk
  static_assert(kPairs == 1, "the LMK row exchange assumes one pair per workgroup");
  __shared__ __attribute__((aligned(16))) LmkShared<T> sX[1];  // used with XR only
  // ONE (fp32 without the LMK row, whose registers leave one wave per SIMD anyway): one
  // ring slot, copied between rounds while the CU's other workgroups compute.  In fp32 a
  // tile pair is 32 KiB and a round's products take five times as long as in bf16, so a
  // second slot hides little and costs the second wave per SIMD (two workgroups per CU
  // instead of four).  See fp32_two_slots for where that pays.
  __shared__ __attribute__((aligned(16))) T ring[kPairs * (ONE ? 1 : 2) * 2 * TILE];  // pair p: slots 2p, 2p+1 (K and V tiles)
  __shared__ int sJ[kPairs][2][32];     // [pair][chunk parity][slot]: chunk index or -1
  __shared__ int sSlot[kPairs][2][32];  // compacted lists of the valid slots: slot, chunk, weight
  __shared__ int sJc[kPairs][2][32];
  __shared__ float sWc[kPairs][2][32];
  __shared__ int sN[kPairs][2];
  // per wave, the log-sum-exp of its 32 tokens x k slots (k <= 8), stored to
  // HBM in one contiguous run at the end of the chunk instead of k scattered
  // 4-byte writes per token
  constexpr int kStageK = 8;
  __shared__ float sLse[2 * kPairs][32][kStageK];

  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, hh = lane >> 5;
  const int pair = wave >> 1, half = wave & 1;
  // Work order: workgroups are dealt to the eight XCDs round-robin (blockIdx mod
  // 8) and each wave pair is a stream of query chunks in StreamOrder (XCD ranges,
  // or chip-wide windows for long slices).
  const int xcd = (int)(blockIdx.x & 7);
  const int64_t st_wg = (int64_t)(blockIdx.x >> 3) * kPairs;
  auto order_of = [&](int q) {
    return StreamOrder((int64_t)(gridDim.x >> 3) * kPairs, st_wg + q, xcd, p.nwork, p.windows);
  };
  const StreamOrder ord = order_of(pair);
  const int64_t my_n = ord.length();
  int64_t nch = 0;  // all pairs of the workgroup run nch chunks of rounds
  for (int q = 0; q < kPairs; ++q) nch = max(nch, order_of(q).length());
  if (nch == 0) return;
  const int64_t c_begin = ord.item(0);
  const int K = p.topk;
  const int qi = 32 * half + (lane & 31);  // this lane's query token within a chunk
  const float sc = p.attn_scale * kLog2e;
  const int cb = 16 * ((lane >> 4) & 1);
  const int l32 = lane & 31;

  // work item w = (b, h, c): geometry helpers
  auto row_of = [&](const Geo& g, int64_t& row_off, bool& exists, bool& owner) __device__ {
    const int hr = p.Hr == 1 ? 0 : g.h;
    const int64_t t = p.causal ? g.c - 1 : 0;
    exists = t >= 0;
    row_off = ((g.b * p.Hr + hr) * p.nQ + (exists ? t : 0)) * K;
    owner = p.Hr != 1 || g.h == 0;  // writes the row's weights
  };
  // first wave of a pair: turn a row's metadata into the pair's compacted slot list
  auto make_slots = [&](const RowMeta& m, const Geo& g, int buf) __device__ {
    int64_t row_off;
    bool exists, owner;
    row_of(g, row_off, exists, owner);
    const bool valid = lane < K && m.j >= 0 && m.j < p.nKV;
    float mx = valid ? m.sv : -INFINITY;
    mx = max64(mx);
    const float e = valid ? expf(m.sv - mx) : 0.f;
    float sum = e;
    sum = sum64(sum);
    const float wv = valid ? e / sum : 0.f;
    const uint64_t mask = __ballot(valid);
    if (lane < 32) sJ[pair][buf][lane] = valid ? m.j : -1;
    if (valid) {
      const int rk = __popcll(mask & ((1ull << lane) - 1));
      sSlot[pair][buf][rk] = lane;
      sJc[pair][buf][rk] = m.j;
      sWc[pair][buf][rk] = wv;
    }
    if (lane == 0) sN[pair][buf] = __popcll(mask);
    if (p.w && exists && owner && lane < K) p.w[row_off + lane] = wv;
  };
  auto qrow_ptr = [&](int64_t w) __device__ {
    return reinterpret_cast<const T*>(p.q) + (w * SQ + qi) * kD;
  };
  // the LMK row's queries, copied by the first wave straight into LDS (one
  // 16-byte piece per lane below kXPieces); visible to both waves after the
  // next wait and barrier
  constexpr int kXPieces = kD * (int)sizeof(T) / 16;
  const int xh = __builtin_amdgcn_readfirstlane(half);  // the wave's half, in a scalar register
  auto load_qx = [&](int64_t w, int xbuf) __device__ {
    if (lane < kXPieces) dma_row16(reinterpret_cast<const T*>(p.q) + (w * SQ + kS) * kD, lane * 16u, &sX[0].q[xbuf][0]);
  };

  // ---- prologue: the first chunk's slot list and Q, the second chunk's metadata
  Frag<T> qf[4], qn[4];
  RowMeta meta{-1, -INFINITY};
  Geo g0(c_begin, p.nQ, p.H);  // geometry of the current chunk and of the two after it
  Geo g1 = g0, g2 = g0;  // (the range order steps without divisions)
  if (p.windows) {
    g1 = Geo(ord.item(1), p.nQ, p.H);
    g2 = Geo(ord.item(2), p.nQ, p.H);
  } else {
    g1.next(p.nQ, p.H, ord.S);
    g2 = g1;
    g2.next(p.nQ, p.H, ord.S);
  }
  if (my_n > 0) {
    int64_t ro;
    bool ex, ow;
    row_of(g0, ro, ex, ow);
    const RowMeta m0 = load_row_meta(p, ro, ex);
    const T* qr = qrow_ptr(c_begin);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) qf[kb] = load_frag(qr + 16 * kb + 8 * hh);
    if (XR && xh == 0) load_qx(c_begin, 0);
    if (half == 0) make_slots(m0, g0, 0);
    if (my_n > 1) {
      row_of(g1, ro, ex, ow);
      meta = load_row_meta(p, ro, ex);
    }
  }
  wait_vmem<0>();
  __syncthreads();

  // the pair's two ring slots alternate: cs is the slot of the next item to compute
  const TileCopy<T, 2> cp(half, lane);
  const T* const gk = reinterpret_cast<const T*>(p.k);
  const T* const gv = reinterpret_cast<const T*>(p.v);
  // element offset of the (batch, head) key/value slice of chunk w
  auto slice_of = [&](const Geo& g) __device__ { return (g.b * p.H + g.h) * p.nKV * TILE; };
  auto issue_item = [&](int64_t kvb, int j, int slot) __device__ {
    j = min(max(j, 0), (int)p.nKV - 1);  // lists hold valid chunks; never copy from outside the slice
    T* dst = ring + (2 * pair + slot) * (2 * TILE);
    cp.issue(gk + kvb + (int64_t)j * TILE, dst);
    cp.issue(gv + kvb + (int64_t)j * TILE, dst + TILE);
  };
  // lane u < 32 of the lists holds valid item u of the current chunk (slot, chunk,
  // weight); items are picked with a lane read
  int ls = sSlot[pair][0][l32], lj = sJc[pair][0][l32];
  float lw = sWc[pair][0][l32];
  int64_t kvb = uniform64(slice_of(g0)), kvb_n = 0;
  int cs = 0;
  if (my_n > 0 && sN[pair][0] > 0) issue_item(kvb, __builtin_amdgcn_readlane(lj, 0), cs);

  // bf16 fragment addresses: this lane's byte offsets inside its pair's first ring
  // slot, computed once; a round adds its slot's offset and every fragment read is
  // one of these six addresses plus an immediate (row +32, key block, V tile,
  // transposed-row gap).
  constexpr bool kB16 = std::is_same<T, __bf16>::value;
  constexpr uint32_t kTileB = TILE * sizeof(T), kRowB = kD * sizeof(T);
  const lds_char* const lds0 = (const lds_char*)(ring);
  const F32Offsets f32o(lane);  // used with ONE
  uint32_t kofs[4], vofs[2][2];
  {
    const uint32_t pb = (uint32_t)pair * 4 * kTileB;
    const int s16 = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kofs[kb] = pb + Swz<T>::off(lane & 31, 16 * kb + 8 * hh) * sizeof(T);
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        vofs[dh][r8] =
            pb + kTileB + Swz<T>::off(8 * r8 + 4 * hh + (s16 >> 2), 32 * dh + cb + 4 * (s16 & 3)) * sizeof(T);
  }

  // one retrieved chunk (item u of the current chunk, tokens from tok0) against
  // this wave's 32 queries; its tiles are in the pair's ring slot `slot`
  float ox0 = 0.f, ox1 = 0.f;  // LMK row: this lane's partial outputs for d = l%32 and 32 + l%32
  auto compute = [&](int slot, int u, int64_t tok0, int buf, f32x16& o0, f32x16& o1) __device__ {
    const uint32_t co = (uint32_t)slot * 2 * kTileB;
    const F32Offsets f32 = ONE ? f32o.fresh() : f32o;
    const int s = __builtin_amdgcn_readlane(ls, u);
    const bool xr = XR && (u & 1) == xh;  // this wave takes the LMK row of slot u
    const T* sK = ring + (2 * pair + slot) * (2 * TILE);
    const T* sV = sK + TILE;
    // all K fragments first, so the eight products issue back to back
    Frag<T> ka[ONE ? 1 : 8];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (ONE) {
        // (read where they are used)
      } else if constexpr (kB16) {
        const lds_char* kp = lds0 + (kofs[kb] + co);
        ka[2 * kb] = lds_b128_at(kp);
        ka[2 * kb + 1] = lds_b128_at(kp + 32 * kRowB);
      } else {
        ka[2 * kb] = lds_frag(sK, lane & 31, 16 * kb + 8 * hh);
        ka[2 * kb + 1] = lds_frag(sK, 32 + (lane & 31), 16 * kb + 8 * hh);
      }
    }
    f32x16 st0 = zero16(), st1 = zero16();
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (ONE) {
        mma32(st0, f32.row_frag(lds0, kb, 0), qf[kb]);
        mma32(st1, f32.row_frag(lds0, kb, 1), qf[kb]);
      } else {
        mma32(st0, ka[2 * kb], qf[kb]);
        mma32(st1, ka[2 * kb + 1], qf[kb]);
      }
    }
    // LMK row scores while the products run: lane l holds keys l%32 and 32 + l%32
    // over its half of the dimensions; the halves are added across l ^ 32
    float xs = 0.f;
    if (xr) {
      float a0 = 0.f, a1 = 0.f;
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        const Frag<T> xf = vec_frag(&sX[0].q[buf][0], 16 * kb + 8 * hh);
        a0 = frag_dot(ka[2 * kb], xf, a0);
        a1 = frag_dot(ka[2 * kb + 1], xf, a1);
      }
      a0 = sum_xor32(a0);
      a1 = sum_xor32(a1);
      xs = hh ? a1 : a0;  // the score of key `lane`
    }
    // V^T fragments are read while the softmax runs
    Frag<T> va[ONE ? 1 : 8];
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (ONE) {
      } else if constexpr (kB16) {
        va[2 * kb] = lds_tr2(lds0 + (vofs[0][0] + co) + 16 * kb * kRowB, lds0 + (vofs[0][1] + co) + 16 * kb * kRowB);
        va[2 * kb + 1] =
            lds_tr2(lds0 + (vofs[1][0] + co) + 16 * kb * kRowB, lds0 + (vofs[1][1] + co) + 16 * kb * kRowB);
      } else {
        va[2 * kb] = lds_frag_t(sV, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, cb);
        va[2 * kb + 1] = lds_frag_t(sV, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, 32 + cb);
      }
    }
    float mx = max_xor32(max_of(st0, st1)) * sc;
    if (OBO) mx = fmaxf(mx, 0.f);
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      st0[i] = __builtin_amdgcn_exp2f(fmaf(st0[i], sc, -mx));
      st1[i] = __builtin_amdgcn_exp2f(fmaf(st1[i], sc, -mx));
    }
    float sum = st0[0] + st1[0];
#pragma unroll
    for (int i = 1; i < 16; ++i) sum += st0[i] + st1[i];
    sum = sum_xor32(sum);
    if (OBO) sum += __builtin_amdgcn_exp2f(-mx);
    if (p.lse && hh == 0) {
      const float lv = (mx + __builtin_amdgcn_logf(sum)) * kLn2;
      if (K <= kStageK)
        sLse[wave][l32][s] = lv;
      else
        p.lse[(tok0 + qi) * K + s] = lv;
    }
    const int coef_bits = __builtin_amdgcn_readlane(__float_as_int(lw), u);
    const float coef = __int_as_float(coef_bits) * __builtin_amdgcn_rcpf(sum);
    if (xr) {
      // the LMK row's softmax over the chunk's 64 keys, one key per lane
      float xm = max64(xs) * sc;
      if (OBO) xm = fmaxf(xm, 0.f);
      const float xe = __builtin_amdgcn_exp2f(fmaf(xs, sc, -xm));
      float xsum = sum64(xe);
      if (OBO) xsum += __builtin_amdgcn_exp2f(-xm);
      if (lane == 0) sX[0].lse[s] = (xm + __builtin_amdgcn_logf(xsum)) * kLn2;
      sX[0].p[xh][lane] = (T)(xe * (__int_as_float(coef_bits) * __builtin_amdgcn_rcpf(xsum)));
    }
    Frag<T> pf[4];
    frag_from_acc(pf[0], st0, 0, coef);
    frag_from_acc(pf[1], st0, 1, coef);
    frag_from_acc(pf[2], st1, 0, coef);
    frag_from_acc(pf[3], st1, 1, coef);
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      if constexpr (ONE) {
        mma32(o0, f32.col_frag(lds0 + kTileB, kb, 0), pf[kb]);
        mma32(o1, f32.col_frag(lds0 + kTileB, kb, 1), pf[kb]);
      } else {
        mma32(o0, va[2 * kb], pf[kb]);
        mma32(o1, va[2 * kb + 1], pf[kb]);
      }
    }
    if (xr) {
      // LMK row output: (w P) V against the V^T fragments, read again now that
      // the products have taken theirs
      wave_lds_order();  // the probabilities, one from each lane ...
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) {
        __builtin_amdgcn_sched_barrier(0);  // one key block's fragments live at a time
        Frag<T> v0, v1;
        if constexpr (kB16) {
          v0 = lds_tr2(lds0 + (vofs[0][0] + co) + 16 * kb * kRowB, lds0 + (vofs[0][1] + co) + 16 * kb * kRowB);
          v1 = lds_tr2(lds0 + (vofs[1][0] + co) + 16 * kb * kRowB, lds0 + (vofs[1][1] + co) + 16 * kb * kRowB);
        } else {
          v0 = lds_frag_t(sV, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, cb);
          v1 = lds_frag_t(sV, 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh, 32 + cb);
        }
        const Frag<T> xf = vec_frag_t(&sX[0].p[xh][0], 16 * kb + 4 * hh, 16 * kb + 8 + 4 * hh);
        ox0 = frag_dot(v0, xf, ox0);
        ox1 = frag_dot(v1, xf, ox1);
      }
      wave_lds_order();  // ... which the next slot's overwrite after this
    }
  };

  // Every chunk takes K rounds (a pair whose chunk has fewer valid slots, or that
  // has run out of chunks, idles), so both pairs meet the same barriers.  Each
  // round: wait for this wave's copies, barrier (the partner's copies are visible
  // and the slot read last round is free), copy the pair's next item into that
  // slot, then compute this round's item.
  f32x16 o0 = zero16(), o1 = zero16();
  for (int64_t ci = 0; ci < nch; ++ci) {
    const bool live = ci < my_n, live_next = ci + 1 < my_n;
    const int buf = (int)(ci & 1);
    const int n = live ? sN[pair][buf] : 0;
    const int64_t w = ord.item(ci), w_next = ord.item(ci + 1);
    const int64_t tok0 = w * SQ;
    for (int u = 0; u < K; ++u) {
      wait_vmem<0>();
      block_barrier();
      if (u == 0) {
        if (!XR && !ONE && ci > 0 && live) {
#pragma unroll
          for (int kb = 0; kb < 4; ++kb) qf[kb] = qn[kb];
        }
        if (ci > 0 && live) {
          ls = sSlot[pair][buf][l32];
          lj = sJc[pair][buf][l32];
          lw = sWc[pair][buf][l32];
          kvb = kvb_n;
        }
        if (live_next) {
          if constexpr (ONE) {
          } else if constexpr (!XR) {
            const T* qr = qrow_ptr(w_next);
#pragma unroll
            for (int kb = 0; kb < 4; ++kb) qn[kb] = load_frag(qr + 16 * kb + 8 * hh);
          } else if (xh == 0) {
            load_qx(w_next, buf ^ 1);
          }
          if (half == 0) make_slots(meta, g1, buf ^ 1);
          if (ci + 2 < my_n) {
            int64_t ro;
            bool ex, ow;
            row_of(g2, ro, ex, ow);
            meta = load_row_meta(p, ro, ex);
          }
          kvb_n = uniform64(slice_of(g1));
        }
        if (K == 1) block_barrier();  // the next chunk's list is needed this round
      }
      const bool comp = u < n;
      const int is = comp && !ONE ? cs ^ 1 : cs;
      if (ONE && comp) {
        compute(cs, u, tok0, buf, o0, o1);
        block_barrier();  // both waves have read the slot
      }
      if (u + 1 < n) {
        issue_item(kvb, __builtin_amdgcn_readlane(lj, u + 1), is);
      } else if (u == K - 1 && live_next && sN[pair][buf ^ 1] > 0) {
        issue_item(kvb_n, sJc[pair][buf ^ 1][0], is);
      }
      if (!ONE && comp) {
        compute(cs, u, tok0, buf, o0, o1);
        cs ^= 1;
      }
    }
    // with the LMK row the next chunk's Q rows are loaded only now, straight into
    // the fragments (the registers of a prefetch are what the row's own work
    // needs); the next round's wait covers them
    if ((XR || ONE) && live_next) {
      const T* qr = qrow_ptr(w_next);
#pragma unroll
      for (int kb = 0; kb < 4; ++kb) qf[kb] = load_frag(qr + 16 * kb + 8 * hh);
    }

    // ---- finish the chunk: each wave stores its 32 query rows
    if (live) {
      T* orow = reinterpret_cast<T*>(p.out) + (tok0 + qi) * kD;
#pragma unroll
      for (int gq = 0; gq < 4; ++gq) {
        store4(orow + 8 * gq + 4 * hh, o0[4 * gq], o0[4 * gq + 1], o0[4 * gq + 2], o0[4 * gq + 3]);
        store4(orow + 32 + 8 * gq + 4 * hh, o1[4 * gq], o1[4 * gq + 1], o1[4 * gq + 2], o1[4 * gq + 3]);
      }
      if (p.lse && K <= kStageK) {
        // this wave's tokens are one contiguous run of 32 k entries; slots
        // without a chunk read -inf
        const int64_t base = (tok0 + 32 * half) * K;
        wave_lds_order();  // other lanes' log-sum-exps ...
        for (int e = lane; e < 32 * K; e += 64) {
          const int tk = e / K, sl = e - tk * K;
          p.lse[base + e] = sJ[pair][buf][sl] < 0 ? -INFINITY : sLse[wave][tk][sl];
        }
        wave_lds_order();  // ... which the next chunk's overwrite after this
      } else if (p.lse && n < K && hh == 0) {
        float* lse = p.lse + (tok0 + qi) * K;
        for (int s = 0; s < K; ++s)
          if (sJ[pair][buf][s] < 0) lse[s] = -INFINITY;
      }
      if constexpr (XR) {
        // the LMK row: add the two waves' shares (each lane first adds its key
        // half to the partner lane's), then one wave stores the row and its lse
        const float t0 = sum_xor32(ox0), t1 = sum_xor32(ox1);
        sX[0].o[xh][lane] = hh ? t1 : t0;  // lane l: d = l
        block_barrier();
        if (xh == 0) {
          const int64_t tx = tok0 + kS;
          reinterpret_cast<T*>(p.out)[tx * kD + lane] = (T)(sX[0].o[0][lane] + sX[0].o[1][lane]);
          if (p.lse && lane < K) p.lse[tx * K + lane] = sJ[pair][buf][lane] < 0 ? -INFINITY : sX[0].lse[lane];
        }
        ox0 = 0.f;
        ox1 = 0.f;
      }
      // the causal last row feeds no chunk: its weights go out with chunk 0
      if (p.w && p.causal && g0.c == 0 && half == 1) {
        int64_t ro;
        bool ex, ow;
        row_of(g0, ro, ex, ow);
        if (ow) {
          const int64_t last_off = (g0.b * p.Hr + (p.Hr == 1 ? 0 : g0.h)) * p.nQ * K + (p.nQ - 1) * K;
          float wv;
          int jv;
          wave_row_weight(p.idx, p.sel, last_off, K, p.nKV, wv, jv);
          if (lane < K) p.w[last_off + lane] = wv;
        }
      }
    }
    o0 = zero16();
    o1 = zero16();
    g0 = g1;
    g1 = g2;
    if (p.windows)
      g2 = Geo(ord.item(ci + 3), p.nQ, p.H);
    else
      g2.next(p.nQ, p.H, ord.S);
  }
}

// ------------------------------ one wave per query chunk (bf16, k <= kWaveMaxK) ----
//
// The same products with the work split differently: a workgroup is one wave that
// owns a whole query chunk, its 64 tokens as two halves of 32, and eight of them
// share a CU (two waves per SIMD).  Against a pair of waves per chunk, a tile's K
// and V^T fragments are read from LDS once for all 64 queries instead of once per
// half, no barrier couples two waves, and one half's products can run beside the
// other half's softmax (the longest phase: 32 exponentials per lane).
//
// K and V each have one LDS tile, filled by asynchronous copies issued piece by piece
// between the products and the exponentials: V's during the score products of the tile
// itself (its last reader was the tile before), the next K's during the first half's
// softmax (the K fragments sit in registers by then).  Everything that a chunk switch
// needs is found one chunk ahead: the landmark row comes by an asynchronous copy and its
// fusion weights stay in registers (lane s: slot s), so the loop holds no load that the
// compiler would wait for behind the copies.  The next chunk's queries are loaded after
// the last score products and waited for with the next keys.
//
// What bounds it: the waves' issue (VALU 0.54, matrix cores 0.28, both 0.11 of the
// SIMD cycles at 16K) under the board's power limit (the clock falls to 1.7-2.0 GHz as
// it gets denser); the copies are waited for 8 % of a tile's time.
// Measured, MI355X, the launch alone, pair form above -> this: 64K tokens (B = 2,
// H = 16, k = 8) 549 -> 487 us, 16K (B = 8, H = 12) 459 -> 411 us, 1M (H = 8, bound by
// the gather past the L2) 2,580 -> 2,540 us.  Few chunks (12 heads, k = 8): 528 16.8 ->
// 15.4 us, 768 17.2 -> 16.7, 1,032 23.6 -> 24.2, 1,200 24.2 -> 24.7, 1,536 30.5 -> 26.0,
// 2,400 44.3 -> 40.0, 6,144 97 -> 84, 24,576 404 -> 374; k = 1 to 4 alike.  It loses where
// its 2,048 waves start a pass that the pair form's 1,024 pairs have just finished: 3,120
// 49.3 -> 52.7, 3,360 55.8 -> 51.7.
// One wave per SIMD (512 registers, tiles two ahead, every product under a softmax) took
// 524 and 410 us: nothing hides a chunk switch there.  Lists longer than kWaveMaxK stay
// with the pair form: their log-sum-exps do not fit in LDS beside the tiles (8 x 20 KiB per
// CU), and storing them per item made this form no faster (k = 16: 339 us against 336 us).
constexpr int kWaveMaxK = 8;
constexpr int kWavesPerCu = 8;
template <bool OBO>
__global__ __launch_bounds__(64, 2) void xattn_fwd_wave_kernel(FwdParams p) {
  using T = __bf16;
  constexpr int TILE = kS * kD;
  constexpr uint32_t kTileB = TILE * sizeof(T), kRowB = kD * sizeof(T);
  __shared__ __attribute__((aligned(16))) T ring[2 * TILE];  // K tile, V tile
  __shared__ int sMj[32];          // the next landmark row's chunks and scores
  __shared__ float sMs[32];
  __shared__ float sLse[2][32 * kWaveMaxK];  // per half: its 32 tokens x K log-sum-exps

  const int lane = threadIdx.x & 63, hh = lane >> 5, l32 = lane & 31;
  // (all counts below fit 32 bits: the launcher's work items and landmark rows do)
  const int S = (int)(gridDim.x >> 3), st = (int)(blockIdx.x >> 3), xcd = (int)(blockIdx.x & 7);
  const int nQ = (int)p.nQ, nKV = (int)p.nKV, H = p.H;
  const StreamOrder ord(S, st, xcd, p.nwork, p.windows);
  const int my_n = __builtin_amdgcn_readfirstlane((int)ord.length());
  if (my_n == 0) return;
  const int K = p.topk;
  const float sc = p.attn_scale * kLog2e;
  const int cb = 16 * ((lane >> 4) & 1);
  const T* const gq = reinterpret_cast<const T*>(p.q);
  T* const go = reinterpret_cast<T*>(p.out);

  // ---- the stream's chunks, found one ahead of the copies: position pos of the
  // stream is work item wd, chunk cd of (batch, head) bd * H + hd
  int pos = 0, wd = __builtin_amdgcn_readfirstlane((int)ord.item(0));
  int cd = wd % nQ, bd = wd / nQ / H, hd = wd / nQ % H;
  auto row_of = [&]() { return (int64_t)(p.Hr == 1 ? bd : bd * H + hd) * nQ + (p.causal ? cd - 1 : 0); };
  auto fetch_meta = [&]() {
    if (pos < my_n && (!p.causal || cd > 0)) {
      const int64_t ro = row_of() * K;
      if (lane < K) {
        dma_column_s(reinterpret_cast<const float*>(p.idx) + ro, (uint32_t)lane * 4, reinterpret_cast<float*>(sMj));
        dma_column_s(p.sel + ro, (uint32_t)lane * 4, sMs);
      }
    }
  };
  // A query chunk with something to attend to: its work item, (batch, head), mask
  // of valid slots, and in lane s < K slot s's key chunk and fusion weight.
  struct Chunk {
    int w, bh;
    uint32_t mask;
    int j;
    float wt;
  };
  auto discover = [&](Chunk& x) {  // the next such chunk of the stream; false at its end
    bool found = false;
    while (!found && pos < my_n) {
      const bool has = !p.causal || cd > 0, owner = p.Hr != 1 || hd == 0;
      const bool in = has && lane < K;
      const int mj = in ? sMj[l32] : -1;
      const float ms = in ? sMs[l32] : 0.f;
      const bool valid = in && mj >= 0 && mj < nKV;
      const uint64_t mask = __ballot(valid);
      // the valid lanes (slots) all sit in the lower half
      const float mx = max64(valid ? ms : -INFINITY);
      const float e = valid ? expf(ms - mx) : 0.f;
      const float sum = sum32(e);
      const float wv = valid ? e / sum : 0.f;
      if (p.w && owner && in) p.w[row_of() * K + lane] = wv;
      x.w = wd;
      x.bh = bd * H + hd;
      x.mask = (uint32_t)__builtin_amdgcn_readfirstlane((int)mask);
      x.j = mj;
      x.wt = wv;
      found = x.mask != 0;
      if (!found) {
        // nothing retrieved: zero output
        const int64_t tok = (int64_t)wd * kS;
#pragma unroll 1
        for (int e2 = lane; e2 < kS * kD / 8; e2 += 64)
          *reinterpret_cast<u32x4*>(go + tok * kD + e2 * 8) = u32x4{0, 0, 0, 0};
        if (p.lse)
#pragma unroll 1
          for (int e2 = lane; e2 < kS * K; e2 += 64) p.lse[tok * K + e2] = -INFINITY;
        if (p.w && p.causal && cd == 0 && owner) {
          // the causal last row feeds no chunk: its weights go out with chunk 0
          float w2;
          int j2;
          const int64_t last = ((int64_t)(p.Hr == 1 ? bd : bd * H + hd) * nQ + nQ - 1) * K;
          wave_row_weight(p.idx, p.sel, last, K, nKV, w2, j2);
          if (lane < K) p.w[last + lane] = w2;
        }
      }
      if (++pos < my_n) {
        if (p.windows) {
          wd = __builtin_amdgcn_readfirstlane((pos * 8 + ((xcd + pos) & 7)) * S + st);
          cd = wd % nQ;
          bd = wd / nQ / H;
          hd = wd / nQ % H;
        } else {
          wd += S;
          cd += S;
          while (cd >= nQ) {
            cd -= nQ;
            if (++hd == H) {
              hd = 0;
              ++bd;
            }
          }
        }
      }
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // sMj / sMs have been read
      fetch_meta();
      if (!found) wait_tiles<0>();  // the next row's chunks and scores
    }
    return found;
  };
  fetch_meta();
  wait_tiles<0>();
  Chunk x0, x1;
  if (!discover(x0)) return;
  wait_tiles<0>();
  bool more = discover(x1);
  if (!more) x1 = x0;
  auto tile_of = [&](const Chunk& x, uint32_t rest) {  // element offset of the K and V tiles of the first slot in rest
    const int j = min(max(__builtin_amdgcn_readlane(x.j, __builtin_ctz(rest)), 0), nKV - 1);
    return ((int64_t)x.bh * nKV + j) * TILE;
  };

  const TileCopy<T, 1> cp(0, lane);
  const T* const gk = reinterpret_cast<const T*>(p.k);
  const T* const gv = reinterpret_cast<const T*>(p.v);
  const lds_char* const lds0 = (const lds_char*)(ring);
  uint32_t kofs[4], vofs[2][2];
  {
    const int s16 = lane & 15;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) kofs[kb] = Swz<T>::off(l32, 16 * kb + 8 * hh) * sizeof(T);
#pragma unroll
    for (int dh = 0; dh < 2; ++dh)
#pragma unroll
      for (int r8 = 0; r8 < 2; ++r8)
        vofs[dh][r8] = kTileB + Swz<T>::off(8 * r8 + 4 * hh + (s16 >> 2), 32 * dh + cb + 4 * (s16 & 3)) * sizeof(T);
  }

  uint32_t rest = x0.mask;  // the current chunk's slots still to do
  Frag<T> qa[4], qb[4];
  const uint32_t qoff = (uint32_t)(l32 * kD + 8 * hh);  // this lane's part of 32 query rows
  auto load_q = [&](int w) {
    const T* r = gq + (int64_t)w * kS * kD;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      qa[kb] = load_frag(r + (qoff + 16 * kb));
      qb[kb] = load_frag(r + (qoff + 32 * kD + 16 * kb));
    }
  };
  load_q(x0.w);
  int64_t off_v = tile_of(x0, rest);
  {
    cp.issue(gk + off_v, ring);
  }
  f32x16 oa0 = zero16(), oa1 = zero16(), ob0 = zero16(), ob1 = zero16();
  f32x16 sa0, sa1, sb0, sb1;
  Frag<T> kf[8], vf[8], pa[4], pb[4];
  auto read_k = [&]() {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      kf[2 * kb] = lds_b128_at(lds0 + kofs[kb]);
      kf[2 * kb + 1] = lds_b128_at(lds0 + kofs[kb] + 32 * kRowB);
    }
  };
  auto read_v = [&]() {
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      vf[2 * kb] = lds_tr2(lds0 + vofs[0][0] + 16 * kb * kRowB, lds0 + vofs[0][1] + 16 * kb * kRowB);
      vf[2 * kb + 1] = lds_tr2(lds0 + vofs[1][0] + 16 * kb * kRowB, lds0 + vofs[1][1] + 16 * kb * kRowB);
    }
  };
  // One half's softmax over the tile's 64 keys; part(i, mx) is called eight times
  // between the exponentials, which take the mx it leaves (it orders what it issues).
  auto softmax = [&](f32x16& s0, f32x16& s1, int half, int s, float wt, Frag<T>* pf, auto part) {
    float mx = max_xor32(max_of(s0, s1)) * sc;
    if (OBO) mx = fmaxf(mx, 0.f);
    float sum = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      part(i, mx);
#pragma unroll
      for (int e = 2 * i; e < 2 * i + 2; ++e) {
        s0[e] = __builtin_amdgcn_exp2f(fmaf(s0[e], sc, -mx));
        s1[e] = __builtin_amdgcn_exp2f(fmaf(s1[e], sc, -mx));
      }
      sum += (s0[2 * i] + s1[2 * i]) + (s0[2 * i + 1] + s1[2 * i + 1]);
    }
    sum = sum_xor32(sum);
    if (OBO) sum += __builtin_amdgcn_exp2f(-mx);
    // both lanes of a query hold the same value
    sLse[half][l32 * K + s] = (mx + __builtin_amdgcn_logf(sum)) * kLn2;
    const float coef = wt * __builtin_amdgcn_rcpf(sum);
    frag_from_acc(pf[0], s0, 0, coef);
    frag_from_acc(pf[1], s0, 1, coef);
    frag_from_acc(pf[2], s1, 0, coef);
    frag_from_acc(pf[3], s1, 1, coef);
  };
  auto store_half = [&](int half, f32x16& o0_, f32x16& o1_) {
    const int64_t tok = (int64_t)x0.w * kS + 32 * half;
    T* orow = go + tok * kD;
#pragma unroll
    for (int m = 0; m < 2; ++m) {
      store_rows16(orow + (qoff + 16 * m), o0_, 8 * m);
      store_rows16(orow + (qoff + 32 + 16 * m), o1_, 8 * m);
    }
    if (p.lse) {
      const uint32_t full = (1u << K) - 1u;
#pragma unroll 1
      for (int s = 0; x0.mask != full && s < K; ++s)
        if (!((x0.mask >> s) & 1u)) sLse[half][l32 * K + s] = -INFINITY;
      wave_lds_order();  // other lanes' log-sum-exps ...
      float v[kWaveMaxK / 2];
#pragma unroll
      for (int i = 0; i < kWaveMaxK / 2; ++i) v[i] = sLse[half][64 * i + lane];
      wave_lds_order();  // ... which the next chunk's overwrite after this
      float* lse = p.lse + tok * K;
#pragma unroll
      for (int i = 0; i < kWaveMaxK / 2; ++i)
        if (64 * i + lane < 32 * K) lse[(uint32_t)(64 * i + lane)] = v[i];
    }
    o0_ = zero16();
    o1_ = zero16();
  };

  while (true) {
    const int s = __builtin_ctz(rest);
    const float wt = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(x0.wt), s));
    rest &= rest - 1u;
    const bool last = rest == 0u;
    // the next item (past the last one: a copy nothing reads)
    const int64_t off = last ? tile_of(x1, x1.mask) : tile_of(x0, rest);
    sa0 = zero16();
    sa1 = zero16();
    sb0 = zero16();
    sb1 = zero16();
    wait_tiles<0>();  // this item's keys
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // the last item's values have been read: their tile is free
#pragma unroll
    for (int i = 0; i < 4; ++i) asm volatile("" : "+v"(qa[i]), "+v"(qb[i]));
    read_k();
    {
      const typename TileCopy<T, 1>::Cursor cv = cp.cursor(gv + off_v, ring + TILE);
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        if (i & 1) mma32(sa1, kf[i], qa[i >> 1]);
        else mma32(sa0, kf[i], qa[i >> 1]);
        cp.issue_piece(cv, i, sc);
      }
    }
    const typename TileCopy<T, 1>::Cursor ck = cp.cursor(gk + off, ring);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // this item's keys have been read
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & 1) mma32(sb1, kf[i], qb[i >> 1]);
      else mma32(sb0, kf[i], qb[i >> 1]);
    }
    softmax(sa0, sa1, 0, s, wt, pa, [&](int i, float& mx) { mx = cp.issue_piece(ck, i, mx); });
    if (last) load_q(x1.w);
    if (last) wait_tiles<16>();
    else wait_tiles<8>();  // this item's values
    read_v();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & 1) mma32(oa1, vf[i], pa[i >> 1]);
      else mma32(oa0, vf[i], pa[i >> 1]);
    }
    softmax(sb0, sb1, 1, s, wt, pb, [&](int, float&) {});
    off_v = off;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      if (i & 1) mma32(ob1, vf[i], pb[i >> 1]);
      else mma32(ob0, vf[i], pb[i >> 1]);
    }
    if (last) {
      store_half(0, oa0, oa1);
      store_half(1, ob0, ob1);
      if (!more) break;
      x0 = x1;
      rest = x0.mask;
      more = discover(x1);
      if (!more) x1 = x0;  // an empty chunk's mask names no tile to copy
    }
  }
  wait_tiles<0>();  // no copy outlives the workgroup's LDS
}

// Ring slots of the fp32 pair form (without the LMK row): two where the items fill whole
// passes of two workgroups per CU but not of four.  A pass of the two-slot form takes
// 43 us at k = 8 for up to two items per CU; the one-slot form's passes of four take 35,
// 73, 76 and 78 us for 1 to 4 items per CU (two workgroups on a CU share SIMDs).
// Two slots / one, k = 8: 504 items (2 per CU) 46 / 74 us, 516 53 / 76, 600 84 / 76, 1,020
// (4) 87 / 80, 1,032 88 / 113, 1,056 97 / 114, 1,116 123 / 114, 1,284 124 / 144, 1,536 (6)
// 128 / 146, 1,548 163 / 149, 2,052 200 / 178, 2,340 (10) 206 / 214, 2,568 242 / 221, 8,000
// 666 / 609; k = 2 and 16 alike (2,340 items, k = 2: 68 / 64).
inline bool fp32_two_slots(int64_t items) {
  const int64_t cus = device_cus(), per_cu = (items + cus - 1) / cus;
  return 8 * items <= 17 * cus || (items > 4 * cus && 4 * items <= 17 * cus) || per_cu == 6 || per_cu == 10;
}

}  // namespace

hipError_t launch_xattn_fwd(const Shape& s, const void* q, const void* k, const void* v,
                            const int32_t* idx, const float* sel, void* out, float* lse, float* w,
                            hipStream_t stream) {
  // Decode, and causal problems whose query chunks all run at once in the decode kernel
  // (two workgroups per CU in bf16, one in fp32): the kernels below would take a chunk's
  // slots one after another on a chip that is mostly idle; that one takes them side by
  // side.  444 chunks, k = 8, bf16: 15.7 -> 12.0 us; 16 in fp32, k = 2: 14.2 -> 10.4 us.
  // One slot (k = 1) leaves nothing to take side by side: 504 chunks in bf16 7.1 us there,
  // 6.0 below, 252 in fp32 11.2 and 10.3.
  const int64_t items = (int64_t)s.B * s.H * s.nQ;
  if (!s.causal || (s.Sq == kS && s.topk > 1 && items <= (s.bf16 ? 2 : 1) * (int64_t)device_cus()))
    return launch_xattn_decode(s, nullptr, nullptr, q, k, v, const_cast<int32_t*>(idx), const_cast<float*>(sel), out,
                               lse, w, nullptr, nullptr, stream);
  FwdParams p;
  p.q = q; p.k = k; p.v = v; p.idx = idx; p.sel = sel;
  p.out = out; p.lse = lse; p.w = w;
  p.H = s.H; p.Hr = s.Hr; p.topk = s.topk;
  p.nQ = s.nQ; p.nKV = s.nKV;
  p.nwork = (int64_t)s.B * s.H * s.nQ;
  p.causal = s.causal;
  p.attn_scale = s.attn_scale;
  p.windows = use_window_order(s.nKV, s.bf16 ? 2 : 4);
  const bool xr = s.Sq != kS;
  // persistent workgroups: kWgPerCu per CU, a multiple of 8 (one share per XCD),
  // each running kPairs chunk streams
  const int64_t target = round8((int64_t)device_cus() * kWgPerCu), wgs = (p.nwork + kPairs - 1) / kPairs;
  const dim3 grid((unsigned)(wgs < target ? round8(wgs) : target)), block(kThreads);
  auto go = [&](auto kernel) { launch_kernel("xattn_fwd_kernel", kernel, grid, block, 0, stream, p); };
  // one wave per chunk for short lists in bf16 (see there); the LMK row's extra state
  // does not fit its registers
  if (s.bf16 && !xr && s.topk <= kWaveMaxK) {
    const int64_t waves = round8((int64_t)device_cus() * kWavesPerCu);
    const dim3 wgrid((unsigned)(p.nwork < waves ? round8(p.nwork) : waves));
    auto wave = [&](auto kernel) { launch_kernel("xattn_fwd_kernel", kernel, wgrid, dim3(64), 0, stream, p); };
    s.off_by_one ? wave(xattn_fwd_wave_kernel<true>) : wave(xattn_fwd_wave_kernel<false>);
    return take_launch_error();
  }
  if (s.bf16) {
    if (xr) s.off_by_one ? go(xattn_fwd_kernel<__bf16, true, true, false>) : go(xattn_fwd_kernel<__bf16, false, true, false>);
    else s.off_by_one ? go(xattn_fwd_kernel<__bf16, true, false, false>) : go(xattn_fwd_kernel<__bf16, false, false, false>);
  } else if (xr) {
    s.off_by_one ? go(xattn_fwd_kernel<float, true, true, false>) : go(xattn_fwd_kernel<float, false, true, false>);
  } else if (fp32_two_slots(items)) {
    s.off_by_one ? go(xattn_fwd_kernel<float, true, false, false>) : go(xattn_fwd_kernel<float, false, false, false>);
  } else {
    s.off_by_one ? go(xattn_fwd_kernel<float, true, false, true>) : go(xattn_fwd_kernel<float, false, false, true>);
  }
  return take_launch_error();
}

}  // namespace gca
