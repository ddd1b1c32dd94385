// gfx950 kernels of libkvs: eviction-masked attention forward and backward.
//
// Mask (Section 2, "KV-streams"): query i of a trace sees key j iff
// j <= i < evict_at[j].  Kernels skip EMPTY tiles, run FULL tiles without
// mask arithmetic and mask PARTIAL tiles element by element.
//
// Row kernels (forward, dQ): a workgroup owns 32*TC query tokens of HG
// q-heads that share one KV head; each wave owns 32 tokens of one q-head.
// K/V tiles of 64 keys are staged once in LDS (double-buffered) and read by
// every wave of the workgroup, so the G heads of a GQA group share them.
// Scores are computed transposed, S^T = K Q^T (keys on the MFMA M axis,
// queries on N), so each lane holds 16 scores of a single query and the row
// max / row sum need one cross-lane exchange per tile.
//
// Column kernel (dK, dV): a workgroup owns 128 keys of one KV head (K held in
// registers, V in LDS) and walks the contiguous range of query rows that can
// see any of them, for each q-head of the group, in steps of 64 rows whose Q,
// dO, LSE and Delta are staged in LDS; a wave takes 32 keys x 32 rows of a step.
//
// All MFMAs are v_mfma_f32_32x32x16_bf16 (bf16 in, fp32 accumulate).
// Operand layouts (per lane l, h = l / 32):  A[m = l%32][k = 8h .. 8h+7],
// B[k = 8h .. 8h+7][n = l%32], C[m = 8(r/4) + 4h + r%4][n = l%32], r = 0..15.
#include "kvs_device.h"
#include "kvs_launch.h"

#include <algorithm>
#include <climits>
#include <mutex>
#include <type_traits>

namespace kvs {

// ---------------------------------------------------------------- kernel arguments
struct RowArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const int* evict;
  const int* cu;
  const int2* kstats;
  uint16_t* o;          // forward output
  float* lse;           // forward output
  const uint16_t* dout; // dQ kernel input
  const float* lse_in;  // dQ kernel input
  const float* delta;   // dQ kernel input
  uint16_t* dq;         // dQ kernel output
  int B, T, Hq, Hkv, G, HG, TC, nhg, nqt, ntok;
  int varlen;
  int flags;            // kFlagNoEmptySkip | kFlagFullAsPartial (consistency checks; 0 normally)
  float scale_log2;     // softmax_scale * log2(e)
  float scale;
};

struct ColArgs {
  const uint16_t* q;
  const uint16_t* k;
  const uint16_t* v;
  const uint16_t* dout;
  const float* lse;
  const float* delta;
  const int* evict;
  const int* cu;
  uint16_t* dk;
  uint16_t* dv;
  const int* plan;      // [B * nkt][2]: parts of the key block (1 = not split), first slot; NULL: none is split
  const int2* items;    // [B * nkt + capE]: (key block, part) work items, longest first; NULL: one per key block
  int* ctl;             // PlanCtl
  float* part;          // [capE * Hkv][2][kColKeys][D] fp32 partial dV, dK of split blocks
  int B, T, Hq, Hkv, G, nkt, ntok;
  int nq;               // work queues (queue_count)
  int varlen;
  int flags;            // as in RowArgs
  float scale_log2;
  float scale;
};

// Parts of a split key block, in steps of 64 query rows x one q-head (see
// split_plan_kernel): at least kMinChunk steps, at most kSplitRowSteps row-steps
// (times G q-heads); kSplitShare parts make up one CU's share of all steps.
constexpr int kSplitRowSteps = 64;
constexpr int kMinChunk = 8;
constexpr int kSplitShare = 3;
constexpr int kCUs = 256;

// Control words of the column kernel, written by the plan: the number of work
// items, of split blocks, and the work queues' next items.
struct PlanCtl {
  int nitems, nsplit;
  int next[kCUs];
};
// One queue per KV head where the KV heads divide the CUs (workgroup w then
// keeps to head w % Hkv, and with it an XCD to few heads) and `bytes` hold
// their counters, else one for all.
static int queue_count(int Hkv, size_t bytes) {
  return kCUs % Hkv == 0 && offsetof(PlanCtl, next) + Hkv * sizeof(int) <= bytes ? Hkv : 1;
}

// LSE / Delta layout: fixed [B][Hq][T], varlen [Hq][ntok].
__device__ __forceinline__ long long lse_index(int varlen, int ntok, int Hq, int T, int b, int h, int tok0, int i) {
  return varlen ? (long long)h * ntok + tok0 + i : ((long long)b * Hq + h) * T + i;
}

// ---------------------------------------------------------------- key-tile statistics
// min and max of min(evict_at[j], L) over the keys j < L of the tile [j0, j0 + BN).
__device__ __forceinline__ int2 key_tile_stats(const int* __restrict__ evict, const Trace& tr, int j0, int BN) {
  int mn = INT_MAX, mx = INT_MIN;
  const int j1 = min(j0 + BN, tr.L);
  for (int j = j0; j < j1; ++j) {
    const int e = min(evict[tr.tok0 + j], tr.L);
    mn = min(mn, e);
    mx = max(mx, e);
  }
  return make_int2(mn, mx);
}

// Statistics of the 64-key tiles of all traces: one wave a tile, one lane a
// key, four tiles a workgroup of 256 threads (group wg of tg per trace).  Bound
// by one memory latency; one thread a tile walked its 64 keys in series, 6.0 us
// for 512 tokens and 7.4 for 8,191, against 2.3 and 4.6 (a launch's own time).
__device__ __forceinline__ void kstats_group(const int* __restrict__ evict, const int* __restrict__ cu, int T, int ntok,
                                             int wg, int tg, int2* __restrict__ out) {
  const int b = wg / tg, kt = (wg - b * tg) * 4 + (threadIdx.x >> 6), lane = threadIdx.x & 63;
  const Trace tr = trace_of(cu, b, T, ntok);
  const int j0 = kt * kKeyTile;
  if (j0 >= tr.L) return;
  const int e = min(evict[tr.tok0 + min(j0 + lane, tr.L - 1)], tr.L);   // lanes past the end repeat the last key
  const int mn = wave_min(e), mx = wave_max(e);
  if (lane == 0) out[kstat_index(b, tr.tok0, kt, kKeyTile)] = make_int2(mn, mx);
}
__host__ __device__ __forceinline__ int kstats_groups(int T) { return ((T + kKeyTile - 1) / kKeyTile + 3) / 4; }

__global__ void __launch_bounds__(256) kstats_kernel(const int* __restrict__ evict, const int* __restrict__ cu, int T,
                                                     int ntok, int2* __restrict__ out) {
  kstats_group(evict, cu, T, ntok, blockIdx.x, kstats_groups(T), out);
}

// ---------------------------------------------------------------- tile-class grid
// One thread per (trace, q-tile, k-tile); grids of all traces concatenated.
// With cu_seqlens, T is the packed token count (every trace length is clamped
// to it, so the grids never outgrow what the host sized from the same offsets).
__global__ void __launch_bounds__(64) classify_kernel(const int* __restrict__ evict, const int* __restrict__ cu,
                                                      int B, int T, int BM, int BN, uint8_t* __restrict__ out) {
  const int kt = blockIdx.x * kWave + threadIdx.x;
  const int qt = blockIdx.y, b = blockIdx.z;
  const Trace tr = trace_of(cu, b, T, T);
  const int nq = (tr.L + BM - 1) / BM, nk = (tr.L + BN - 1) / BN;
  if (qt >= nq || kt >= nk) return;
  long long off = 0;
  for (int bb = 0; bb < b; ++bb) {
    const Trace t2 = trace_of(cu, bb, T, T);
    off += (long long)((t2.L + BM - 1) / BM) * ((t2.L + BN - 1) / BN);
  }
  const int2 st = key_tile_stats(evict, tr, kt * BN, BN);
  out[off + (long long)qt * nk + kt] =
      (uint8_t)tile_class(qt * BM, qt * BM + BM, kt * BN, kt * BN + BN, tr.L, st.x, st.y);
}

// ---------------------------------------------------------------- evict_at validation
__device__ unsigned long long g_first_bad;
__device__ int g_cu_bad;

__global__ void check_init_kernel() {
  g_first_bad = ULLONG_MAX;
  g_cu_bad = 0;
}

__global__ void __launch_bounds__(256) check_kernel(const int* __restrict__ evict, const int* __restrict__ cu,
                                                    int B, int T, int ntok) {
  const int b = blockIdx.y;
  if (cu) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      const int a = cu[b], z = cu[b + 1];
      if ((b == 0 && a != 0) || z < a || (b == B - 1 && z != ntok) || z > ntok) atomicOr(&g_cu_bad, 1);
    }
  }
  const Trace tr = trace_of(cu, b, T, ntok);
  if (tr.L <= 0) return;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < tr.L; j += gridDim.x * blockDim.x) {
    if (evict[tr.tok0 + j] <= j) atomicMin(&g_first_bad, (unsigned long long)(tr.tok0 + j));
  }
}

// ---------------------------------------------------------------- key-tile walker
// Every wave of a workgroup walks the same sequence of non-EMPTY key tiles of
// its query rows [i0, i1): 64 candidate tiles are classified at a time (one
// per lane) and the non-EMPTY ones kept as a ballot.  Each lane keeps the
// evict_at statistics of its candidate tile, so the statistics of the tile
// walker_next returns are read from a register (walker_stats) instead of from
// memory, whose latency the wave would otherwise wait out on every tile.
struct TileWalker {
  int base, lim;
  unsigned long long live;
  int emin, emax;   // statistics of candidate tile base + lane
};

__device__ __forceinline__ void walker_load(TileWalker& w, const int2* __restrict__ ks, int kidx0, int i0, int i1,
                                            int L, int flags) {
  const int kt = w.base + (threadIdx.x & 63);
  bool ne = false;
  int2 st = make_int2(0, 0);
  if (kt < w.lim) {
    st = ks[kidx0 + kt];
    ne = adjust_class(tile_class(i0, i1, kt * kKeyTile, kt * kKeyTile + kKeyTile, L, st.x, st.y), flags) != kEmpty;
  }
  w.live = __ballot(ne);
  w.emin = st.x;
  w.emax = st.y;
}

__device__ __forceinline__ int walker_next(TileWalker& w, const int2* __restrict__ ks, int kidx0, int i0, int i1,
                                           int L, int flags) {
  while (w.live == 0ull) {
    w.base += 64;
    if (w.base >= w.lim) return -1;
    walker_load(w, ks, kidx0, i0, i1, L, flags);
  }
  const int bit = __builtin_ctzll(w.live);
  w.live &= w.live - 1ull;
  return w.base + bit;
}

// evict_at minimum and maximum of tile kt, the tile the last walker_next call returned (kt >= 0)
__device__ __forceinline__ int2 walker_stats(const TileWalker& w, int kt) {
  const int l = kt - w.base;
  return make_int2(__builtin_amdgcn_readlane(w.emin, l), __builtin_amdgcn_readlane(w.emax, l));
}

// ---------------------------------------------------------------- operand reads from swizzled tiles
// S^T block (32 keys x 32 queries) of the current tile: A = K rows from LDS, B = Q^T in registers.
// rl = Lay<D, COMPACT>::row_lane(lane).
template <int D, bool COMPACT = false>
__device__ __forceinline__ f32x16 scores_t(const uint16_t* tile, int row0, const bf16x8* breg,
                                           typename Lay<D, COMPACT>::RowLane rl, f32x16 s = f32x16{}) {
  using LY = Lay<D, COMPACT>;
  const uint16_t* base = tile + row0 * LY::PITCH;
#pragma unroll
  for (int ks = 0; ks < D / 16; ++ks) s = mfma32(lds_read_b128(base + LY::row_at(rl, ks)), breg[ks], s);
  return s;
}

// Mask of a PARTIAL tile for S^T blocks: element r of block kb is key
// j = j0 + 32 kb + 8 (r/4) + 4 half + r%4 and query i.
__device__ __forceinline__ void mask_t(f32x16& s, const int* sE, int kb, int j0, int i, int L, int half) {
#pragma unroll
  for (int q4 = 0; q4 < 4; ++q4) {
    const int jl = 32 * kb + 8 * q4 + 4 * half;
    const int4 e4 = *reinterpret_cast<const int4*>(sE + jl);
    const int ev[4] = {e4.x, e4.y, e4.z, e4.w};
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      const int j = j0 + jl + t;
      const bool vis = (j <= i) && (i < ev[t]) && (i < L);
      if (!vis) s[4 * q4 + t] = -INFINITY;
    }
  }
}

// Head grouping of a row-kernel workgroup.
struct RowTile {
  int g, h, b, i0, i1, i0w, hh;
  Trace tr;
};

// Launch order: blockIdx % Hkv is the KV head (consecutive workgroups go to
// different XCDs, so each XCD's L2 serves one head's K/V); then the head
// group; then the traces one after another, each trace's query tiles from the
// last to the first (later tiles see more keys: start them first).  Taking
// the traces one at a time keeps an XCD's K/V working set to one trace.
__device__ __forceinline__ bool row_tile(const RowArgs& a, RowTile& t) {
  int wg = blockIdx.x;
  t.g = wg % a.Hkv;
  wg /= a.Hkv;
  const int hgrp = wg % a.nhg;
  wg /= a.nhg;
  const int qt = a.nqt - 1 - wg % a.nqt;
  t.b = wg / a.nqt;
  t.tr = trace_of(a.cu, t.b, a.T, a.ntok);
  const int BMt = 32 * a.TC;
  t.i0 = qt * BMt;
  t.i1 = t.i0 + BMt;
  if (t.i0 >= t.tr.L) return false;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  t.hh = wave % a.HG;
  t.h = t.g * a.G + hgrp * a.HG + t.hh;
  t.i0w = t.i0 + 32 * (wave / a.HG);
  return true;
}

// Asynchronous staging of one 64-key K/V (and evict_at) tile of KV head g
// (compact layout: two workgroups of the dQ kernel share a CU).
template <int D>
using KVStager = RowStager<D, kKeyTile, 4, true>;   // row kernels: 4 waves

// Rows of an O or dQ accumulator to memory: 32 rows (lane % 32) x D, acc[d][r]
// = column 32 d + 8 (r / 4) + 4 half + r % 4, scaled and rounded to bf16.  They
// go through the wave's own LDS buffer (at least 32 x (D + 8) elements), so that
// a store instruction writes whole rows: from the accumulator layout it writes
// 16 bytes of each of 32 rows, which cost the 24 short traces of 100 to 1,500
// tokens 10 of the forward's 82 us and 9 of dQ's 107 us, the 16k trace 1%.
template <int D>
__device__ __forceinline__ void store_rows(const f32x16* acc, float sc, uint16_t* buf, uint16_t* __restrict__ dst,
                                           long long row_stride, int nrows, int lane) {
  constexpr int P = D + 8;   // row pitch: rows 8 bytes x 2 banks apart
  const int half = lane >> 5, col = lane & 31;
#pragma unroll
  for (int d = 0; d < D / 32; ++d)
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4)
      *reinterpret_cast<uint2*>(buf + col * P + 32 * d + 8 * q4 + 4 * half) =
          pack4_bf16(acc[d][4 * q4] * sc, acc[d][4 * q4 + 1] * sc, acc[d][4 * q4 + 2] * sc, acc[d][4 * q4 + 3] * sc);
  asm volatile("" ::: "memory");   // the same bytes are read back as another type; LDS keeps a wave's order
  constexpr int LPR = D / 8, RPI = kWave / LPR;   // lanes per row, rows per store
  const int r0 = lane / LPR, c = 8 * (lane % LPR);
#pragma unroll
  for (int it = 0; it < 32 / RPI; ++it) {
    const int r = it * RPI + r0;
    const uint4 v = *reinterpret_cast<const uint4*>(buf + r * P + c);
    if (r < nrows) *reinterpret_cast<uint4*>(dst + r * row_stride + c) = v;
  }
}

// ---------------------------------------------------------------- forward
// K/V are staged in sub-tiles of BN keys (D = 128: 32, so that a workgroup
// needs 37 KB of LDS and three workgroups, three waves per SIMD, share a CU;
// D = 64: 64 keys, 37 KB, four workgroups at 128 VGPRs per wave), walked in
// the order of the non-EMPTY 64-key tiles.  The sub-tiles are double-buffered
// in two distinct LDS arrays each; the loop body alternates between them so
// the compiler can tell that the asynchronous fill of the next buffer never
// aliases the reads of the current one (and does not wait for the fill
// before reading).  A sub-tile's class comes from the statistics of its
// 64-key tile, which can only report PARTIAL where FULL would hold or
// non-EMPTY where EMPTY would: a conservative, exact choice.
template <int D>
constexpr int fwd_bn() { return D == 128 ? 32 : 64; }

template <int D>
using FwdStager = RowStager<D, fwd_bn<D>(), 4, true>;   // 4 waves

template <int D>
__global__ void __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(D == 128 ? 3 : 4, D == 128 ? 3 : 4)))
fwd_kernel(RowArgs a) {
  constexpr int KS = D / 16, DB = D / 32, BN = fwd_bn<D>(), NKB = BN / 32, NSUB = kKeyTile / BN;
  __shared__ __attribute__((aligned(1024))) uint16_t sK0[BN * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sK1[BN * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sV0[BN * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sV1[BN * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(256))) int sE0[BN];
  __shared__ __attribute__((aligned(256))) int sE1[BN];

  RowTile rt;
  if (!row_tile(a, rt)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const Trace tr = rt.tr;
  const int i = rt.i0w + col;
  const bool row_ok = i < tr.L;
  const auto rl = Lay<D, true>::row_lane(lane);
  const int tl = Lay<D, true>::tr_lo(lane), th = Lay<D, true>::tr_hi(lane);
  FwdStager<D> kvst;
  kvst.init(wave, lane, (long long)a.Hkv * D);
  // Asynchronous staging of the BN keys from j0 on (j0 < L) of KV head g.
  // Byte offsets are formed with one 32 x 32 -> 64 bit product: the copies
  // stand at the head of every sub-tile, in front of all its products.
  const uint32_t row_bytes = 2u * (uint32_t)a.Hkv * D;
  const char* kbase = (const char*)uniform_ptr(a.k + ((long long)tr.tok0 * a.Hkv + rt.g) * D);
  const char* vbase = (const char*)uniform_ptr(a.v + ((long long)tr.tok0 * a.Hkv + rt.g) * D);
  const char* ebase = (const char*)uniform_ptr(a.evict + tr.tok0);
  auto stage = [&](uint16_t* sK, uint16_t* sV, int* sE, int j0) __attribute__((always_inline)) {
    const uint64_t off = (uint64_t)(uint32_t)j0 * row_bytes;
    const int dr = tr.L - 1 - j0;
    const uint32_t lim = FwdStager<D>::limit(dr, (long long)a.Hkv * D);
    kvst.issue_at(lds_addr(sK), kbase + off, lim, wave);
    kvst.issue_at(lds_addr(sV), vbase + off, lim, wave);
    if (wave == nw - 1) {
      if (BN == kWave || lane < BN) stage_words_at(lds_addr(sE), ebase + 4u * (uint32_t)j0, dr, lane);
    }
  };

  bf16x8 qreg[KS];
  {
    const uint16_t* qrow = a.q + ((size_t)(tr.tok0 + min(i, tr.L - 1)) * a.Hq + rt.h) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) qreg[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(qrow + 16 * ks));
  }

  f32x16 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x16{};
  // Running reference maximum of the row (log2 units), the offset the
  // exponentials use (0 until the row has seen a visible key), and the raw
  // score above which the reference must move: m_run + 8 in score units.
  float m_run = -INFINITY, l_run = 0.f, m_use = 0.f, thr = -INFINITY;
  const float inv_scale_log2 = 1.f / a.scale_log2;

  const int kidx0 = kstat_index(rt.b, tr.tok0, 0, kKeyTile);
  TileWalker w{0, (min(rt.i1, tr.L) + kKeyTile - 1) / kKeyTile, 0ull, 0, 0};
  walker_load(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags);
  int kt = __builtin_amdgcn_readfirstlane(walker_next(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags));
  int2 kst = kt >= 0 ? walker_stats(w, kt) : make_int2(0, 0);

  // The products and the softmax of the sub-tile of BN keys from j0 on.
  auto compute = [&](const uint16_t* cK, const uint16_t* cV, const int* cE, int j0) __attribute__((always_inline)) {
    const int cls = adjust_class(tile_class(rt.i0w, rt.i0w + 32, j0, j0 + BN, tr.L, kst.x, kst.y), a.flags);
    if (cls != kEmpty) {
      f32x16 s[NKB];
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb) {
        s[kb] = scores_t<D, true>(cK, 32 * kb, qreg, rl);
        if (cls == kPartial) mask_t(s[kb], cE, kb, j0, i, tr.L, half);
      }
      float mx = -INFINITY;   // maximum of this lane's half of the row
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, s[kb][r]);
      // The reference max of a row only moves when the tile's max exceeds it by
      // more than 8 (log2 units): probabilities are then at most 2^8, exact to
      // rescale later, and the accumulator rescale is skipped for most tiles.
      // The row's max exceeds the threshold iff one of its two halves does, so
      // the halves are combined only when some row of the wave moves.  The
      // ballot moves every row of the wave, including rows that have not seen
      // a visible key yet and see none here (m_run = row max = -inf): their
      // factor is 1, not exp2(-inf - -inf) = NaN.
      if (__ballot(mx > thr)) {
        const float m_new = fmaxf(m_run, fmaxf(mx, wave_xor32(mx)) * a.scale_log2);
        const float alpha = m_new == m_run ? 1.f : __builtin_amdgcn_exp2f(m_run - m_new);   // 0 on the first visible tile
        l_run *= alpha;
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[d][r] *= alpha;
        m_run = m_new;
        m_use = (m_run == -INFINITY) ? 0.f : m_run;
        thr = (m_run + 8.f) * inv_scale_log2;
      }
      float ls = 0.f;
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[kb][r], a.scale_log2, -m_use));
          s[kb][r] = p;
          ls += p;
        }
      l_run += ls;
      // Raised wave priority for the PV products: the SIMD then runs this wave's
      // MFMAs back to back while the other resident waves do their softmax work,
      // instead of the waves drifting into the same phase (measured: 2-3%).
      __builtin_amdgcn_s_setprio(3);
#pragma unroll
      for (int kb = 0; kb < NKB; ++kb)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bf16x8 pb = pack8(s[kb], 8 * t);
#pragma unroll
          for (int d = 0; d < DB; ++d)
            acc[d] = mfma32(tr_operand<D, true>(cV, 32 * kb + 16 * t, 32 * d, tl, th), pb, acc[d]);
        }
      __builtin_amdgcn_s_setprio(0);
    }
  };

  // Next key tile and its statistics, from the walker's registers (no memory
  // access); called behind a sub-tile's products, so that its scalar work runs
  // while the matrix core still has some of them to do.
  int nkt = -1;
  int2 nkst = make_int2(0, 0);
  auto walk = [&]() __attribute__((always_inline)) {
    nkt = __builtin_amdgcn_readfirstlane(walker_next(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags));
    if (nkt >= 0) nkst = walker_stats(w, nkt);
  };
  const int jend = min(rt.i1, tr.L);   // no row of the workgroup sees a key from here on

  if (kt >= 0) stage(sK0, sV0, sE0, kt * kKeyTile);
  if (NSUB == 1 && kt >= 0) walk();
  wait_vm();
  __syncthreads();
  while (kt >= 0) {
    const int j0 = kt * kKeyTile;
    if (NSUB == 2) {
      // the two halves of a 64-key tile; where no row sees the second one it is the last tile
      const bool second = j0 + BN < jend;
      if (second) stage(sK1, sV1, sE1, j0 + BN);
      compute(sK0, sV0, sE0, j0);
      if (!second) break;
      walk();
      wait_vm();
      __syncthreads();
      if (nkt >= 0) stage(sK0, sV0, sE0, nkt * kKeyTile);
      compute(sK1, sV1, sE1, j0 + BN);
      if (nkt < 0) break;
      kt = nkt;
      kst = nkst;
      wait_vm();
      __syncthreads();
    } else {
      if (nkt >= 0) stage(sK1, sV1, sE1, nkt * kKeyTile);
      compute(sK0, sV0, sE0, j0);
      kt = nkt;
      kst = nkst;
      if (kt >= 0) walk();
      wait_vm();
      __syncthreads();
      if (kt < 0) break;
      if (nkt >= 0) stage(sK0, sV0, sE0, nkt * kKeyTile);
      compute(sK1, sV1, sE1, kt * kKeyTile);
      kt = nkt;
      kst = nkst;
      if (kt >= 0) walk();
      wait_vm();
      __syncthreads();
    }
  }

  const float l_tot = l_run + wave_xor32(l_run);
  const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
  __syncthreads();   // the tile buffers are free
  store_rows<D>(acc, inv, wave < 2 ? (wave ? sK1 : sK0) : (wave == 2 ? sV0 : sV1),
                a.o + ((size_t)(tr.tok0 + rt.i0w) * a.Hq + rt.h) * D, (long long)a.Hq * D, tr.L - rt.i0w, lane);
  if (row_ok && half == 0)
    a.lse[lse_index(a.varlen, a.ntok, a.Hq, a.T, rt.b, rt.h, tr.tok0, i)] =
        (m_run + __log2f(l_tot)) * 0.6931471805599453f;
}

// ---------------------------------------------------------------- backward: Delta = rowsum(dO * O), stored as -Delta
// Also writes LSE * log2(e), the form in which the backward kernels use it.
// The first nks workgroups take the key-tile statistics instead (a launch less
// ahead of the backward's main kernels).
template <int D>
__global__ void __launch_bounds__(256) bwd_pre_kernel(const uint16_t* __restrict__ o, const uint16_t* __restrict__ dout,
                                                      const float* __restrict__ lse, float* __restrict__ delta,
                                                      float* __restrict__ lse2, int ntok, int Hq, int T, int varlen,
                                                      const int* __restrict__ evict, const int* __restrict__ cu,
                                                      int nks, int2* __restrict__ kstats) {
  if ((int)blockIdx.x < nks) {
    kstats_group(evict, cu, T, ntok, blockIdx.x, kstats_groups(T), kstats);
    return;
  }
  constexpr int PER = D / 16;  // elements per lane, 16 lanes per row
  const int sub = threadIdx.x & 15;
  const long long row = (long long)(blockIdx.x - nks) * (blockDim.x / 16) + (threadIdx.x >> 4);
  const bool ok = row < (long long)ntok * Hq;
  float s = 0.f;
  if (ok) {
    const size_t off = (size_t)row * D + sub * PER;
#pragma unroll
    for (int e = 0; e < PER; ++e) {
      const float x = (float)__builtin_bit_cast(__bf16, o[off + e]);
      const float y = (float)__builtin_bit_cast(__bf16, dout[off + e]);
      s += x * y;
    }
  }
#pragma unroll
  for (int m = 8; m > 0; m >>= 1) s += __shfl_xor(s, m);
  if (ok && sub == 0) {
    const int tok = (int)(row / Hq), h = (int)(row % Hq);
    const long long idx = varlen ? (long long)h * ntok + tok : ((long long)(tok / T) * Hq + h) * T + tok % T;
    delta[idx] = -s;   // stored negated: both backward kernels add it
    lse2[idx] = lse[idx] * 1.4426950408889634f;
  }
}

// ---------------------------------------------------------------- backward: dQ (row kernel)
template <int D>
__global__ void __launch_bounds__(512) dq_kernel(RowArgs a) {
  constexpr int KS = D / 16, DB = D / 32;
  __shared__ __attribute__((aligned(1024))) uint16_t sK0[kKeyTile * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sK1[kKeyTile * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sV0[kKeyTile * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(1024))) uint16_t sV1[kKeyTile * Lay<D, true>::PITCH];
  __shared__ __attribute__((aligned(256))) int sE0[kKeyTile];
  __shared__ __attribute__((aligned(256))) int sE1[kKeyTile];

  RowTile rt;
  if (!row_tile(a, rt)) return;
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6), nw = blockDim.x >> 6;
  const int half = lane >> 5, col = lane & 31;
  const Trace tr = rt.tr;
  const int i = rt.i0w + col;
  const auto rl = Lay<D, true>::row_lane(lane);
  const int tl = Lay<D, true>::tr_lo(lane), th = Lay<D, true>::tr_hi(lane);
  KVStager<D> kvst;
  kvst.init(wave, lane, (long long)a.Hkv * D);
  // asynchronous staging of the 64 keys from j0 on (j0 < L) of KV head g, as in the forward
  const uint32_t row_bytes = 2u * (uint32_t)a.Hkv * D;
  const char* kbase = (const char*)uniform_ptr(a.k + ((long long)tr.tok0 * a.Hkv + rt.g) * D);
  const char* vbase = (const char*)uniform_ptr(a.v + ((long long)tr.tok0 * a.Hkv + rt.g) * D);
  const char* ebase = (const char*)uniform_ptr(a.evict + tr.tok0);
  auto stage = [&](uint16_t* sK, uint16_t* sV, int* sE, int j0) __attribute__((always_inline)) {
    const uint64_t off = (uint64_t)(uint32_t)j0 * row_bytes;
    const int dr = tr.L - 1 - j0;
    const uint32_t lim = KVStager<D>::limit(dr, (long long)a.Hkv * D);
    kvst.issue_at(lds_addr(sK), kbase + off, lim, wave);
    kvst.issue_at(lds_addr(sV), vbase + off, lim, wave);
    if (wave == nw - 1) stage_words_at(lds_addr(sE), ebase + 4u * (uint32_t)j0, dr, lane);
  };
  const int ic = min(i, tr.L - 1);

  bf16x8 qreg[KS], oreg[KS];
  float lse2, ndlt;
  {
    const size_t roff = ((size_t)(tr.tok0 + ic) * a.Hq + rt.h) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      qreg[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(a.q + roff + 16 * ks));
      oreg[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(a.dout + roff + 16 * ks));
    }
    const long long li = lse_index(a.varlen, a.ntok, a.Hq, a.T, rt.b, rt.h, tr.tok0, ic);
    lse2 = a.lse_in[li];   // already scaled by log2(e)
    ndlt = a.delta[li];   // -Delta
  }

  f32x16 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x16{};

  const int kidx0 = kstat_index(rt.b, tr.tok0, 0, kKeyTile);
  TileWalker w{0, (min(rt.i1, tr.L) + kKeyTile - 1) / kKeyTile, 0ull, 0, 0};
  walker_load(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags);
  int kt = __builtin_amdgcn_readfirstlane(walker_next(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags));
  int2 kst = kt >= 0 ? walker_stats(w, kt) : make_int2(0, 0);

  // The next tile and its statistics come from the walker's registers (no
  // memory access), one tile ahead and behind the current tile's products.
  int nkt = -1;
  int2 nkst = make_int2(0, 0);
  auto walk = [&]() __attribute__((always_inline)) {
    nkt = __builtin_amdgcn_readfirstlane(walker_next(w, a.kstats, kidx0, rt.i0, rt.i1, tr.L, a.flags));
    if (nkt >= 0) nkst = walker_stats(w, nkt);
  };
  auto body = [&](const uint16_t* cK, const uint16_t* cV, const int* cE, uint16_t* nK, uint16_t* nV, int* nE) {
    if (nkt >= 0) stage(nK, nV, nE, nkt * kKeyTile);
    const int j0 = kt * kKeyTile;
    const int cls = adjust_class(tile_class(rt.i0w, rt.i0w + 32, j0, j0 + kKeyTile, tr.L, kst.x, kst.y), a.flags);
    if (cls != kEmpty) {
#pragma unroll
      for (int kb = 0; kb < 2; ++kb) {
        f32x16 s = scores_t<D, true>(cK, 32 * kb, qreg, rl);
        if (cls == kPartial) mask_t(s, cE, kb, j0, i, tr.L, half);
        // dP - Delta: the product starts at -Delta
        f32x16 d0;
#pragma unroll
        for (int r = 0; r < 16; ++r) d0[r] = ndlt;
        const f32x16 dp = scores_t<D, true>(cV, 32 * kb, oreg, rl, d0);
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const float p = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], a.scale_log2, -lse2));
          s[r] = p * dp[r];
        }
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          const bf16x8 dsb = pack8(s, 8 * t);
#pragma unroll
          for (int d = 0; d < DB; ++d)
            acc[d] = mfma32(tr_operand<D, true>(cK, 32 * kb + 16 * t, 32 * d, tl, th), dsb, acc[d]);
        }
      }
    }
    kt = nkt;
    kst = nkst;
    if (kt < 0) return;   // the last tile: nothing staged, no buffer reused
    walk();
    wait_vm();
    __syncthreads();
  };

  if (kt >= 0) {
    stage(sK0, sV0, sE0, kt * kKeyTile);
    walk();
  }
  wait_vm();
  __syncthreads();
  while (kt >= 0) {
    body(sK0, sV0, sE0, sK1, sV1, sE1);
    if (kt < 0) break;
    body(sK1, sV1, sE1, sK0, sV0, sE0);
  }

  __syncthreads();   // the tile buffers are free
  store_rows<D>(acc, a.scale, wave < 2 ? (wave ? sK1 : sK0) : (wave == 2 ? sV0 : sV1),
                a.dq + ((size_t)(tr.tok0 + rt.i0w) * a.Hq + rt.h) * D, (long long)a.Hq * D, tr.L - rt.i0w, lane);
}

// ---------------------------------------------------------------- backward: dK, dV (column kernel)
// One workgroup: 128 keys of one KV head, 8 waves.  The workgroup walks the
// query rows that can see any of its keys in steps of 64 rows x one q-head of
// the group; Q, dO, LSE and Delta of a step are staged once in LDS for all
// eight waves.  Wave w computes the 32 keys 32 (w % 4) .. and the 32-row block
// w / 4 of every step, all of it by itself:
//   S = Q K^T,  P = exp2(S * scale * log2 e - LSE * log2 e) (masked),  dV^T += dO^T P,
//   dP = dO V^T - Delta,  dS = P dP,  dK^T += Q^T dS
// so the waves of a SIMD (w and w + 4) exchange nothing inside an item and P
// stays in registers.  K is held in registers; V, which does not fit beside the
// dK and dV accumulators (2 x 64 registers at D = 128 of a wave's 256), is
// staged in LDS once per item.  At the item's end the two row halves are added
// through the (then free) tile buffers: wave w < 4 stores dV, wave w + 4 dK.
// Bound by the matrix cores (busy 58% of the kernel's cycles on the 16k trace) at
// the clock their power leaves: each wave is one chain of S, dP, the exponentials,
// dV and dK, and two waves a SIMD cover each other's.  A pair of waves that splits
// the products instead (one S and dV, the other dP and dK of the same block, P
// through LDS in 16 bits) is locked together by every step's barrier: 17% more
// cycles, 50% busy, at a higher clock.  That against this, kernel traces of one
// run, us: 16k trace (32/8 heads, D = 128) 1,852 -> 1,711, two of 4,097 340 -> 318,
// 24 of 100 to 1,500 (16/2) 135 -> 118, 8,191 tokens (24/8, D = 64) 208 -> 179, 512
// tokens (4/4, D = 64) 14.9 -> 13.7.
template <int D>
__global__ void __launch_bounds__(512) __attribute__((amdgpu_waves_per_eu(2, 2))) dkdv_kernel(ColArgs a) {
  constexpr int KS = D / 16, DB = D / 32, PITCH = Lay<D>::PITCH, kHalf = kQStep * PITCH, kTile = 2 * kHalf;
  using LV = Lay<D, true>;
  constexpr int AHEAD = 2, OPS = 2;
  // ring of three tiles: [Q rows, dO rows], and their [LSE * log2 e, -Delta].  One array each, indexed by the
  // step: with an array a tile, every tile's operand addresses would be held in registers (24 of them spilled).
  __shared__ __attribute__((aligned(1024))) uint16_t sT[3 * kTile];
  __shared__ __attribute__((aligned(1024))) uint16_t sV[kColKeys * LV::PITCH];
  __shared__ __attribute__((aligned(256))) float sW[3 * 2 * kQStep];
  __shared__ int sEmax[4];
  __shared__ int sNext;

  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const bool role_dk = wave >= 4;       // what the wave stores at the item's end
  const int kw = wave & 3;              // its keys
  const int rb = 32 * (wave >> 2);      // its rows of a step
  // The second wave of a SIMD gets its copies out last; with priority it catches up with the first one's products
  // instead of ending every step behind it (16k trace, backward: 2,975 -> 2,950 us, with the early reads below).
  if (role_dk) __builtin_amdgcn_s_setprio(1);

  // Work items (longest first, see split_plan_kernel): a whole key block, or
  // one part of a split block; one KV head each.  The grid is one workgroup a
  // CU (it fills the CU); each takes the next item of its queue when it is
  // done, the first one by its index.  Every item is an iteration, and the
  // queue's counter only grows, so each workgroup ends after at most all items.
  // (One workgroup per possible item left those without one to be started and
  // ended in turn behind the last items, as many as there are unused slots.)
  PlanCtl* ctl = reinterpret_cast<PlanCtl*>(a.ctl);
  const int nq = a.nq, queue = nq > 1 ? blockIdx.x % a.Hkv : 0;
  const int nitems = a.items ? ctl->nitems : a.B * a.nkt;
  const int nidx = nq > 1 ? nitems : nitems * a.Hkv;
  int idx = nq > 1 ? blockIdx.x / a.Hkv : blockIdx.x;
  const bool more = (int)gridDim.x / nq < nidx;   // items beyond the first ones
  while (idx < nidx) {
  const int g = nq > 1 ? queue : idx % a.Hkv;
  const int2 item = a.items ? a.items[nq > 1 ? idx : idx / a.Hkv] : make_int2(nq > 1 ? idx : idx / a.Hkv, 0);
  const int b = item.x / a.nkt, kt = item.x % a.nkt, chunk = item.y;
  const int nchunk = a.plan ? a.plan[2 * item.x] : 1, slot0 = a.plan ? a.plan[2 * item.x + 1] : 0;
  const Trace tr = trace_of(a.cu, b, a.T, a.ntok);
  const int j0 = kt * kColKeys;
  if (j0 >= tr.L) break;   // only without a plan, where every workgroup has one item; the plan lists no such block
  // per-lane constants are recomputed for every item: held across items they cost registers the loop lacks
  int lane = threadIdx.x & 63;
  asm volatile("" : "+v"(lane));
  const int half = lane >> 5, col = lane & 31;
  const auto rl = Lay<D>::row_lane(lane);
  const int vl = LV::row_lane(lane).even + 32 * kw * LV::PITCH;
  const int tl = Lay<D>::tr_lo(lane), th = Lay<D>::tr_hi(lane);
  {
    // V of the block's keys (rows past the trace's end repeat its last 16 bytes and are masked)
    RowStager<D, kColKeys, 8, true> vst;
    vst.init(wave, lane, (long long)a.Hkv * D);
    vst.issue(lds_addr(sV), a.v + ((size_t)tr.tok0 * a.Hkv + g) * D, (long long)a.Hkv * D, j0, tr.L - 1, wave);
  }
  RowStager<D, kQStep, 8> qst;
  qst.init(wave, lane, (long long)a.Hq * D);
  const int j = j0 + 32 * kw + col;
  const bool key_ok = j < tr.L;
  const int jc = min(j, tr.L - 1);
  const int ej = key_ok ? min(a.evict[tr.tok0 + j], tr.L) : 0;
  const unsigned kspan = key_ok ? (unsigned)(ej - j) : 0u;   // rows j .. ej - 1 see this key
  int emin_w = key_ok ? ej : INT_MAX, emax_w = key_ok ? ej : INT_MIN;
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    emin_w = min(emin_w, __shfl_xor(emin_w, off));
    emax_w = max(emax_w, __shfl_xor(emax_w, off));
  }
  emin_w = __builtin_amdgcn_readfirstlane(emin_w);
  emax_w = __builtin_amdgcn_readfirstlane(emax_w);
  if (!role_dk && lane == 0) sEmax[kw] = emax_w;

  // K of this lane's key: the B operand of S
  bf16x8 kreg[KS];
  {
    const uint16_t* src = a.k + ((size_t)(tr.tok0 + jc) * a.Hkv + g) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) kreg[ks] = as_bf16x8(*reinterpret_cast<const uint4*>(src + 16 * ks));
  }
  __syncthreads();
  const int emax_wg = max(max(sEmax[0], sEmax[1]), max(sEmax[2], sEmax[3]));
  const int qs_lo = j0 / kQStep;
  const int qs_hi = (emax_wg + kQStep - 1) / kQStep;
  int steps = max(qs_hi - qs_lo, 0) * a.G, step0 = 0;   // this item: steps step0 .. step0 + steps - 1 of the block's
  if (nchunk > 1) {
    const int per = (steps + nchunk - 1) / nchunk;
    step0 = min(chunk * per, steps);
    steps = min(per, steps - step0);
  }

  f32x16 av[DB], ak[DB];   // dV^T and dK^T of the wave's rows: rows d, column = this lane's key
#pragma unroll
  for (int d = 0; d < DB; ++d) av[d] = ak[d] = f32x16{};

  // First row of a step and the byte offsets of its first Q / dO row and its
  // first LSE / Delta value, advanced step by step: from the step number they
  // are a division by G and some forty scalar instructions of every wave,
  // ahead of the step's copies.
  struct Pos {
    int i0, hh;   // first row, q-head of the group
  };
  struct Src {
    Pos at;
    long long row, word;
  };
  const long long row_step = 2ll * D, row_wrap = 2ll * D * ((long long)kQStep * a.Hq - a.G);
  const long long word_step = 4ll * (a.varlen ? a.ntok : a.T), word_wrap = 4ll * kQStep - a.G * word_step;
  auto advance = [&](Pos& p) __attribute__((always_inline)) {
    const bool wrap = ++p.hh == a.G;
    p.hh = wrap ? 0 : p.hh;
    p.i0 += wrap ? kQStep : 0;
    return wrap;
  };
  const Pos first = {(qs_lo + step0 / a.G) * kQStep, step0 % a.G};
  Src next = {first, row_step * ((long long)(tr.tok0 + first.i0) * a.Hq + g * a.G + first.hh),
              4ll * lse_index(a.varlen, a.ntok, a.Hq, a.T, b, g * a.G + first.hh, tr.tok0, first.i0)};   // staged next
  Pos cur = first;                                                                                       // computed next
  const uint32_t tile_lds = lds_addr(sT), word_lds = lds_addr(sW);
  auto stage = [&](int buf) __attribute__((always_inline)) {
    const int dr = tr.L - 1 - next.at.i0;
    const uint32_t lim = qst.limit(dr, (long long)a.Hq * D);
    qst.issue_at(tile_lds + 2 * buf * kTile, (const char*)a.q + next.row, lim, wave);
    qst.issue_at(tile_lds + 2 * (buf * kTile + kHalf), (const char*)a.dout + next.row, lim, wave);
    if (wave == 6) stage_words_at(word_lds + 8 * buf * kQStep, (const char*)a.lse + next.word, dr, lane);   // LSE * log2(e)
    if (wave == 7) stage_words_at(word_lds + 8 * buf * kQStep + 4 * kQStep, (const char*)a.delta + next.word, dr, lane);
    const bool wrap = advance(next.at);
    next.row += row_step + (wrap ? row_wrap : 0);
    next.word += word_step + (wrap ? word_wrap : 0);
  };
  const int jw0 = j0 + 32 * kw;

  f32x16 dp;   // dP - Delta: the product starts at -Delta
  bf16x8 qa[AHEAD], oa[AHEAD], va[AHEAD];
  auto read_ks = [&](int buf, int ks) __attribute__((always_inline)) {
    const uint16_t *cQ = sT + buf * kTile, *cO = cQ + kHalf;
    qa[ks % AHEAD] = lds_read_b128(cQ + rb * PITCH + Lay<D>::row_at(rl, ks));
    oa[ks % AHEAD] = lds_read_b128(cO + rb * PITCH + Lay<D>::row_at(rl, ks));
    va[ks % AHEAD] = lds_read_b128(sV + LV::row_at({vl}, ks));
  };
  // the first operands of a tile: read ahead of the barrier in front of its step (in registers the step before
  // has done with), unused if the block turns out EMPTY
  auto read_first = [&](int buf) __attribute__((always_inline)) {
#pragma unroll
    for (int ks = 0; ks < AHEAD; ++ks) read_ks(buf, ks);
    const float* cD = sW + buf * 2 * kQStep + kQStep;
#pragma unroll
    for (int q4 = 0; q4 < 4; ++q4) {
      const float4 d4 = *reinterpret_cast<const float4*>(cD + rb + 8 * q4 + 4 * half);
      dp[4 * q4] = d4.x;
      dp[4 * q4 + 1] = d4.y;
      dp[4 * q4 + 2] = d4.z;
      dp[4 * q4 + 3] = d4.w;
    }
  };
  // The wave's block of a step.  C layout of S and dP: lane <-> key, element r
  // <-> row rb + 8 (r/4) + 4 half + r%4 of the staged tile.  Operands are read
  // AHEAD k-steps (S, dP) or OPS products (dV, dK) before their product, and the
  // arithmetic of one group of products stands between the products of the
  // group before it; fences keep the compiler from moving the reads back to
  // their products (which waits out an LDS latency per product).
  auto compute = [&](int buf) __attribute__((always_inline)) {
    const int ib = cur.i0 + rb;
    const int cls = adjust_class(tile_class(ib, ib + 32, jw0, jw0 + 32, tr.L, emin_w, emax_w), a.flags);
    if (cls == kEmpty) return;
    const uint16_t *cQ = sT + buf * kTile, *cO = cQ + kHalf;
    const float* cL = sW + buf * 2 * kQStep;
    f32x16 x = {};
    float4 l4[4];
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      x = mfma32(qa[ks % AHEAD], kreg[ks], x);
      dp = mfma32(oa[ks % AHEAD], va[ks % AHEAD], dp);
      if (ks + AHEAD < KS) read_ks(buf, ks + AHEAD);
      if (ks + AHEAD == KS) {
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) l4[q4] = *reinterpret_cast<const float4*>(cL + rb + 8 * q4 + 4 * half);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    // operand n of dV (n < 2 DB) and dK
    auto operand = [&](int n) __attribute__((always_inline)) {
      return tr_operand<D>(n < 2 * DB ? cO : cQ, rb + 16 * ((n / DB) & 1), 32 * (n % DB), tl, th);
    };
    bf16x8 op[OPS + 1];
#pragma unroll
    for (int n = 0; n < OPS; ++n) op[n] = operand(n);
    if (cls == kPartial) {
#pragma unroll
      for (int r = 0; r < 16; ++r) {
        const bool vis = (unsigned)(ib + 8 * (r >> 2) + 4 * half + (r & 3) - j) < kspan;
        x[r] = vis ? x[r] : -INFINITY;
      }
    }
    auto prob = [&](int r) __attribute__((always_inline)) {
      const float lv[4] = {l4[r >> 2].x, l4[r >> 2].y, l4[r >> 2].z, l4[r >> 2].w};
      x[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(x[r], a.scale_log2, -lv[r & 3]));
    };
#pragma unroll
    for (int r = 0; r < 8; ++r) prob(r);
    bf16x8 pk[2];   // P, then dS, of the rows of each half of the products
    pk[0] = pack8(x, 0);
    __builtin_amdgcn_sched_barrier(0);
    constexpr int E = 8 / DB;   // elements a product's arithmetic takes
#pragma unroll
    for (int n = 0; n < 4 * DB; ++n) {
      f32x16& acc = n < 2 * DB ? av[n % DB] : ak[n % DB];
      acc = mfma32(op[n % (OPS + 1)], pk[(n / DB) & 1], acc);
      if (n + OPS < 4 * DB) op[(n + OPS) % (OPS + 1)] = operand(n + OPS);
#pragma unroll
      for (int e = 0; e < E; ++e) {
        const int r = E * (n % DB) + e;
        if (n < DB) prob(8 + r);
        else if (n < 2 * DB) x[r] *= dp[r];
        else if (n < 3 * DB) x[8 + r] *= dp[8 + r];
      }
      if (n == DB - 1) pk[1] = pack8(x, 8);
      if (n == 2 * DB - 1) pk[0] = pack8(x, 0);
      if (n == 3 * DB - 1) pk[1] = pack8(x, 8);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

  // Three-stage ring: during step s tile s is read and tile s + 2 copied into
  // the buffer tile s - 1 used.  Every wave waits for its copies of tile s + 2
  // ahead of the barrier that ends step s, so tile s + 1 is whole all through
  // step s and its first operands may be read before that barrier.  The barrier
  // itself only orders the copies behind the reads of step s, whose values the
  // products have taken by then: no wait for LDS stands in front of it.
  {
    if (steps > 0) stage(0);
    if (steps > 1) stage(1);
    wait_vm();
    __syncthreads();
    int buf = 0;
    read_first(0);
    for (int step = 0; step < steps; ++step) {
      const int nbuf = buf == 2 ? 0 : buf + 1;
      if (step + 2 < steps) stage(buf == 0 ? 2 : buf - 1);
      compute(buf);
      advance(cur);
      read_first(nbuf);
      __builtin_amdgcn_sched_barrier(0);
      wait_vm();
      asm volatile("" ::: "memory");
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");
      buf = nbuf;
    }
  }

  int next_idx = nidx;   // asked for ahead of the stores, waited for behind them
  if (threadIdx.x == 0 && more) next_idx = atomicAdd(&ctl->next[queue], 1);
  // The row halves' sums: each wave hands the partner (w ^ 4) the accumulators
  // it does not store, through its own buffer among the tiles', which are free.
  auto buffer = [&](int w) { return w < 6 ? sT + w * kHalf : sV + (w - 6) * 64 * LV::PITCH; };
  uint16_t *buf = buffer(wave), *other = buffer(wave ^ 4);
  {
    float* give = reinterpret_cast<float*>(buf) + 4 * lane;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const f32x16& x = role_dk ? av[d] : ak[d];
        *reinterpret_cast<float4*>(give + (4 * d + q4) * 4 * kWave) =
            make_float4(x[4 * q4], x[4 * q4 + 1], x[4 * q4 + 2], x[4 * q4 + 3]);
      }
  }
  __syncthreads();
  f32x16 acc[DB];
  {
    const float* take = reinterpret_cast<const float*>(other) + 4 * lane;
#pragma unroll
    for (int d = 0; d < DB; ++d) {
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[d][r] = role_dk ? ak[d][r] : av[d][r];
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4) {
        const float4 v = *reinterpret_cast<const float4*>(take + (4 * d + q4) * 4 * kWave);
        acc[d][4 * q4] += v.x;
        acc[d][4 * q4 + 1] += v.y;
        acc[d][4 * q4 + 2] += v.z;
        acc[d][4 * q4 + 3] += v.w;
      }
    }
  }
  if (nchunk > 1) {
    // fp32 partial sums of this part: [slot][dV, dK][32-key group], each group
    // as the accumulators lie, [d][q4][lane][4], so that a store instruction
    // writes 1 KB in a row (split_reduce_kernel turns the sums)
    float* dst = a.part + ((((size_t)(slot0 + chunk) * a.Hkv + g) * 2 + (role_dk ? 1 : 0)) * 4 + kw) * 32 * D + 4 * lane;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<float4*>(dst + (4 * d + q4) * 4 * kWave) =
            make_float4(acc[d][4 * q4], acc[d][4 * q4 + 1], acc[d][4 * q4 + 2], acc[d][4 * q4 + 3]);
  } else {
    // whole rows through LDS, in the buffer this wave has just read (its own is still the partner's to read)
    asm volatile("" ::: "memory");
    store_rows<D>(acc, role_dk ? a.scale : 1.f, other,
                  (role_dk ? a.dk : a.dv) + ((size_t)(tr.tok0 + jw0) * a.Hkv + g) * D, (long long)a.Hkv * D, tr.L - jw0,
                  lane);
  }
  if (threadIdx.x == 0) sNext = next_idx;
  __syncthreads();   // sNext; and every wave is done with the LDS of this item
  idx = __builtin_amdgcn_readfirstlane(sNext);
  }
}

// ---------------------------------------------------------------- work plan of the column kernel
// A key block whose keys stay visible for many query rows (the prompt,
// long-lived summaries) would be one long workgroup and set the kernel's
// critical path.  A dK/dV workgroup fills a CU, so a CU's share of the work is
// total steps x Hkv / kCUs.  Blocks longer than that share are cut into equal
// parts of at most 1 / kSplitShare of it; shorter ones start early enough whole.
// Parts stay within [kMinChunk, kSplitRowSteps * G] steps (below, a workgroup's
// start and end outweigh its steps; above, long traces would be left with a
// long last item) and blocks of up to two of the bound are not cut.  Every part
// gets a slot of fp32 partial sums, and the parts are added in order afterwards
// (deterministic).  Slots are granted in key-block order while capE lasts;
// later blocks stay whole.  All work items (whole blocks and parts) are then
// listed longest first (counting sort on the step count).  One workgroup of
// 1024 threads; block spans come from the 64-key tile statistics.
// dK/dV kernel with parts of 64 row-steps only, cut beyond 128, and with these
// (kernel traces of one run, its products split over pairs of waves on both
// sides): 24 traces of 100 to 1,500 tokens (16/2 heads, D = 128) 336 -> 139 us, two
// of 4,097 (32/8) 462 -> 354, one of 8,191 (24/8, D = 64) 474 -> 217; plan and
// reduce take 15 to 18 us of that back.  Parts of 1/2 and 1/4 share and a
// threshold of 2/3 or 4/5 share: within 5%.
__global__ void __launch_bounds__(1024) split_plan_kernel(const int2* __restrict__ kstats, const int* __restrict__ cu,
                                                          int B, int T, int ntok, int nkt, int G, int Hkv, int capE,
                                                          int grid, int nq, int* __restrict__ plan, int2* __restrict__ items,
                                                          int* __restrict__ split, PlanCtl* __restrict__ ctl) {
  constexpr int NBK = 2048, NW = 1024 / kWave;   // sort buckets, waves
  __shared__ int bucket[NBK];
  __shared__ int wsum[4][NW];
  __shared__ int nsplit_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int nblocks = B * nkt;
  bucket[tid] = bucket[tid + 1024] = 0;
  if (tid == 0) nsplit_s = 0;
  if (tid < nq) ctl->next[tid] = grid / nq;   // the first items are taken by index
  const int per = (nblocks + 1023) / 1024;
  const int b0 = min(tid * per, nblocks), b1 = min(b0 + per, nblocks);
  // row-steps of a block: [j0/64, ceil(emax/64)); 0 past the trace
  auto read_rows = [&](int blk) {
    const int b = blk / nkt, kt = blk % nkt;
    const Trace tr = trace_of(cu, b, T, ntok);
    const int j0 = kt * kColKeys;
    if (j0 >= tr.L) return 0;
    const int t0 = j0 / kKeyTile, nt = (tr.L + kKeyTile - 1) / kKeyTile;
    int emax = kstats[kstat_index(b, tr.tok0, t0, kKeyTile)].y;
    if (t0 + 1 < nt) emax = max(emax, kstats[kstat_index(b, tr.tok0, t0 + 1, kKeyTile)].y);
    return max((emax + kQStep - 1) / kQStep - j0 / kQStep, 1);
  };
  // at most one block a thread: its steps and parts stay in registers
  const int own = per == 1 && b0 < b1 ? read_rows(b0) * G : 0;
  int own_parts = 1;
  auto steps_of = [&](int blk) { return per == 1 ? own : read_rows(blk) * G; };
  int sum = 0, steps_sum = 0;   // row-steps: at most 2^14 a block, 2^13 blocks of the longest traces
  for (int blk = b0; blk < b1; ++blk) sum += steps_of(blk) / G;
  steps_sum = wave_last(wave_scan(sum));
  if (lane == 0) wsum[0][wave] = steps_sum;
  __syncthreads();
  long long total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) total += wsum[0][w];
  const long long share = total * G * Hkv / kCUs;   // steps of one CU
  const long long most = max((long long)kSplitRowSteps * G, (long long)kMinChunk);
  const int chunk = (int)min(max(share / kSplitShare, (long long)kMinChunk), most);
  const int whole = (int)min(max(share, 2ll * kMinChunk), 2 * most);
  auto parts_of = [&](int steps) { return steps > whole ? (steps + chunk - 1) / chunk : 0; };
  int tot = 0, top = 1;   // requested slots; longest item
  for (int blk = b0; blk < b1; ++blk) {
    const int steps = steps_of(blk), w = parts_of(steps);
    tot += w;
    top = max(top, w > 0 ? (steps + w - 1) / w : steps);
  }
  int incl = wave_scan(tot);
  top = wave_max(top);
  if (lane == kWave - 1) wsum[1][wave] = incl;
  if (lane == 0) wsum[2][wave] = top;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) incl += wsum[1][w];
    top = max(top, wsum[2][w]);
  }
  int run = incl - tot;   // exclusive prefix of requested slots
  // Sort key (larger first): the step count in equal classes (blocks left
  // whole for want of slots may exceed the last one).  One trace (or more than
  // NBK / 8): NBK classes.  Otherwise the class, then the trace, so that items
  // of one trace with about the same length are listed together and run side
  // by side (they share Q / dO rows in an XCD's L2); the classes are then at
  // least 8 row-steps wide, or a quarter of a chunk if that is less; the
  // longest class still starts first, so the tail grows by less than a class.
  // Keys stay below NBK: nclass * B <= NBK.
  const bool by_trace = B > 1 && B <= NBK / 8;
  const int nclass = by_trace ? NBK / B : NBK;
  const int width = max((top + nclass) / nclass, by_trace ? min(8 * G, max(chunk / 4, 1)) : 1);
  auto key_of = [&](int steps, int blk) {
    const int c = min(steps / width, nclass - 1);
    return by_trace ? c * B + blk / nkt : c;
  };
  for (int blk = b0; blk < b1; ++blk) {
    const int steps = steps_of(blk), w = parts_of(steps);
    const bool grant = w > 0 && run + w <= capE;
    own_parts = grant ? w : 1;
    if (plan) {
      plan[2 * blk] = own_parts;
      plan[2 * blk + 1] = grant ? run : 0;
    }
    if (grant) split[atomicAdd(&nsplit_s, 1)] = blk;
    run += w;
    if (steps == 0) continue;
    const int len = (steps + own_parts - 1) / own_parts;
    for (int c = 0; c < own_parts; ++c) atomicAdd(&bucket[key_of(max(min(len, steps - c * len), 0), blk)], 1);
  }
  __syncthreads();
  // bucket start positions, longest first: thread t owns buckets NBK-1-2t and NBK-2-2t
  const int khi = NBK - 1 - 2 * tid, klo = khi - 1;
  const int chi = bucket[khi], clo = bucket[klo];
  incl = wave_scan(chi + clo);
  if (lane == kWave - 1) wsum[3][wave] = incl;
  __syncthreads();
  int all = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    if (w < wave) incl += wsum[3][w];
    all += wsum[3][w];
  }
  bucket[khi] = incl - chi - clo;
  bucket[klo] = incl - clo;
  if (tid == 0) {
    ctl->nitems = all;
    ctl->nsplit = nsplit_s;
  }
  __syncthreads();
  for (int blk = b0; blk < b1; ++blk) {
    const int steps = steps_of(blk), nc = per == 1 ? own_parts : plan ? plan[2 * blk] : 1;
    if (steps == 0) continue;
    const int len = (steps + nc - 1) / nc;
    for (int c = 0; c < nc; ++c)
      items[atomicAdd(&bucket[key_of(max(min(len, steps - c * len), 0), blk)], 1)] = make_int2(blk, c);
  }
}

// Sum of the parts' partials of split key blocks, in part order; dK scaled.
// The split blocks are listed by the plan, and a fixed grid walks the 32-key
// groups of dV and dK of all of them.  Bound by reading the partials, so every
// thread keeps several parts' loads in flight; the sums are turned in LDS and
// stored as whole rows.
constexpr int kReduceGrid = 2048;
template <int D>
__global__ void __launch_bounds__(256) split_reduce_kernel(const PlanCtl* __restrict__ ctl,
                                                           const int* __restrict__ plan, const int* __restrict__ split,
                                                           const float* __restrict__ part, const int* __restrict__ cu,
                                                           uint16_t* __restrict__ dk, uint16_t* __restrict__ dv, int B,
                                                           int T, int ntok, int nkt, int Hkv, float scale) {
  constexpr int P = D + 8, NF = D / 32;              // LDS row pitch; float4s of a thread: fragments of 256
  constexpr size_t kSlot = (size_t)2 * kColKeys * D;    // floats of one slot
  __shared__ __attribute__((aligned(16))) uint16_t buf[32 * P];
  const int tid = threadIdx.x, lane = tid & 63, half = lane >> 5, col = lane & 31;
  const int tasks = ctl->nsplit * Hkv * 8;
  for (int t = blockIdx.x; t < tasks; t += gridDim.x) {
    const int grp = t & 7, bg = t >> 3, g = bg % Hkv, blk = split[bg / Hkv];   // group: dV 0..3, dK 4..7
    const int nc = plan[2 * blk], s0 = plan[2 * blk + 1];
    const int b = blk / nkt, kt = blk % nkt;
    const float* src = part + ((size_t)s0 * Hkv + g) * kSlot + (size_t)grp * 32 * D + 4 * tid;
    float4 sum[NF];
#pragma unroll
    for (int n = 0; n < NF; ++n) sum[n] = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 2
    for (int c = 0; c < nc; ++c) {
      float4 v[NF];
#pragma unroll
      for (int n = 0; n < NF; ++n) v[n] = *reinterpret_cast<const float4*>(src + (size_t)c * Hkv * kSlot + n * 1024);
#pragma unroll
      for (int n = 0; n < NF; ++n) {
        sum[n].x += v[n].x;
        sum[n].y += v[n].y;
        sum[n].z += v[n].z;
        sum[n].w += v[n].w;
      }
    }
    const float sc = grp >= 4 ? scale : 1.f;
    // float4 n of wave w is fragment 4 n + w: columns 32 n + 8 w + 4 half of key `col`
#pragma unroll
    for (int n = 0; n < NF; ++n)
      *reinterpret_cast<uint2*>(buf + col * P + 32 * n + 8 * (tid >> 6) + 4 * half) =
          pack4_bf16(sum[n].x * sc, sum[n].y * sc, sum[n].z * sc, sum[n].w * sc);
    asm volatile("" ::: "memory");   // the same bytes are read back as another type
    __syncthreads();
    const Trace tr = trace_of(cu, b, T, ntok);
    constexpr int LPR = D / 8;
#pragma unroll
    for (int n = 0; n < 32 * LPR / 256; ++n) {
      const int r = (n * 256 + tid) / LPR, c = 8 * (tid % LPR), j = kt * kColKeys + 32 * (grp & 3) + r;
      const uint4 v = *reinterpret_cast<const uint4*>(buf + r * P + c);
      if (j < tr.L) *reinterpret_cast<uint4*>((grp >= 4 ? dk : dv) + ((size_t)(tr.tok0 + j) * Hkv + g) * D + c) = v;
    }
    __syncthreads();
  }
}

// Explicit instantiations: every kernel the launchers use is emitted, with its host stub.
template __global__ void fwd_kernel<64>(RowArgs);
template __global__ void fwd_kernel<128>(RowArgs);
template __global__ void dq_kernel<64>(RowArgs);
template __global__ void dq_kernel<128>(RowArgs);
template __global__ void dkdv_kernel<64>(ColArgs);
template __global__ void dkdv_kernel<128>(ColArgs);
template __global__ void split_reduce_kernel<64>(const PlanCtl*, const int*, const int*, const float*, const int*, uint16_t*, uint16_t*,
                                                  int, int, int, int, int, float);
template __global__ void split_reduce_kernel<128>(const PlanCtl*, const int*, const int*, const float*, const int*, uint16_t*, uint16_t*,
                                                  int, int, int, int, int, float);

// ---------------------------------------------------------------- library-owned scratch (allocation-free forward)
// Per-key-tile statistics of kvs_evict_attn_fwd_noalloc.  In host code the
// name `scratch` is only a host-side stand-in: its device address (one per
// GPU) comes from hipGetSymbolAddress, taken once per device with that device
// current, and only that address is ever passed to a kernel.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

hipError_t noalloc_scratch(void** ptr) {
  static std::mutex mu;
  static void* per_device[kMaxDevices] = {};
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lk(mu);
  if (!per_device[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    per_device[dev] = p;
  }
  *ptr = per_device[dev];
  return hipSuccess;
}

// ---------------------------------------------------------------- launchers
size_t ws_kstats_bytes(int B, int ntok) {
  const size_t n = (size_t)B + (size_t)ntok / kKeyTile + 2;
  return (n * sizeof(int2) + 255) & ~(size_t)255;
}

// -Delta followed by LSE * log2(e), each [Hq][ntok] (or [B][Hq][T]) fp32.
size_t ws_delta_bytes(int Hq, int ntok) { return 2 * (((size_t)Hq * ntok * sizeof(float) + 255) & ~(size_t)255); }

static size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }

// Slots of parts per KV head that the plan can use, at most 2048 over all KV
// heads.  Up to 2 * kSplitRowSteps row-steps only the CUs' shares ask for
// parts: kSplitShare kCUs of them if every block is cut, and one more for each
// of at most kCUs cut blocks.  None when no block can span more than two least
// parts.
static int split_cap(int B, int T, int Hkv, int G) {
  const long long max_span = (T + kQStep - 1) / kQStep, max_steps = max_span * G;
  if (max_steps <= 2 * kMinChunk) return 0;
  const long long nkt = (T + kColKeys - 1) / kColKeys;
  const long long slots = max_span <= 2 * kSplitRowSteps ? std::min(2048, (kSplitShare + 1) * kCUs) : 2048;
  const long long per_block = (max_steps + kMinChunk - 1) / kMinChunk;
  return (int)std::min<long long>(slots / Hkv, (long long)B * nkt * per_block);
}

// Workspace of the column kernel for `cap` slots per KV head: plan [B * nkt][2]
// int, work items [B * nkt + cap] int2, PlanCtl, the split blocks [cap] int,
// partial sums [cap * Hkv][2][kColKeys][D] fp32.  Without slots no plan is
// kept, and the counters (as many as fit) stand in its place.
struct SplitSpace {
  size_t plan, items, ctl, split, part;
  size_t bytes() const { return plan + items + ctl + split + part; }
};
static SplitSpace split_space(int B, int T, int Hkv, int D, int cap) {
  const size_t blocks = (size_t)B * ((T + kColKeys - 1) / kColKeys);
  if (cap == 0) return {0, round256(blocks * sizeof(int2)), round256(blocks * 2 * sizeof(int)), 0, 0};
  return {round256(blocks * 2 * sizeof(int)), round256((blocks + cap) * sizeof(int2)), round256(sizeof(PlanCtl)),
          round256((size_t)cap * sizeof(int)), round256((size_t)cap * Hkv * 2 * kColKeys * D * sizeof(float))};
}
size_t ws_split_bytes(int B, int T, int Hkv, int G, int D) { return split_space(B, T, Hkv, D, split_cap(B, T, Hkv, G)).bytes(); }
// The least a call takes: no partial sums up to 2 * kSplitRowSteps row-steps, beyond which a block that is not cut
// would be the kernel's critical path.
size_t ws_split_least(int B, int T, int Hkv, int D) {
  const long long max_span = (T + kQStep - 1) / kQStep, nkt = (T + kColKeys - 1) / kColKeys;
  const size_t whole = split_space(B, T, Hkv, D, 0).bytes();
  if (max_span <= 2 * kSplitRowSteps) return whole;
  const size_t cap = std::min<long long>(2048 / Hkv, B * nkt * ((max_span + kSplitRowSteps - 1) / kSplitRowSteps));
  return whole - round256((size_t)B * nkt * sizeof(int2)) + round256(((size_t)B * nkt + cap) * sizeof(int2)) +
         round256(cap * Hkv * 2 * kColKeys * D * sizeof(float));
}
// Slots per KV head in `bytes` of workspace: blocks that get none stay whole.
static int split_fit(int B, int T, int Hkv, int G, int D, size_t bytes) {
  int cap = split_cap(B, T, Hkv, G);
  if (split_space(B, T, Hkv, D, cap).bytes() <= bytes) return cap;
  cap = (int)std::min<size_t>(cap, bytes / ((size_t)Hkv * 2 * kColKeys * D * sizeof(float)));
  while (cap > 0 && split_space(B, T, Hkv, D, cap).bytes() > bytes) --cap;
  return cap;
}
static size_t half_delta_bytes(int Hq, int ntok) { return ws_delta_bytes(Hq, ntok) / 2; }

static RowArgs row_args(const Problem& p, const int2* kstats) {
  RowArgs a{};
  a.q = (const uint16_t*)p.q;
  a.k = (const uint16_t*)p.k;
  a.v = (const uint16_t*)p.v;
  a.evict = p.evict;
  a.cu = p.cu;
  a.kstats = kstats;
  a.o = (uint16_t*)p.o;
  a.lse = p.lse;
  a.dout = (const uint16_t*)p.dout;
  a.lse_in = p.lse_in;
  a.dq = (uint16_t*)p.dq;
  a.B = p.B;
  a.T = p.T;
  a.Hq = p.Hq;
  a.Hkv = p.Hkv;
  a.G = p.G;
  a.HG = p.HG;
  a.TC = p.TC;
  a.nhg = p.nhg;
  a.nqt = (p.T + 32 * p.TC - 1) / (32 * p.TC);
  a.ntok = p.ntok;
  a.varlen = p.cu != nullptr;
  a.flags = p.flags;
  a.scale = p.scale;
  a.scale_log2 = p.scale * 1.4426950408889634f;
  return a;
}

constexpr int kMaxTraces = 65535;   // keeps every grid and workgroup index within 31 bits

hipError_t launch_kstats(const Problem& p, int2* kstats) {
  if (p.B > kMaxTraces) return hipErrorInvalidConfiguration;
  prof_begin("classify", p.stream);
  hipLaunchKernelGGL(kstats_kernel, dim3((unsigned)((long long)kstats_groups(p.T) * p.B)), dim3(256), 0, p.stream,
                     p.evict, p.cu, p.T, p.ntok, kstats);
  prof_end(p.stream);
  return hipGetLastError();
}

hipError_t launch_fwd(const Problem& p, const int2* kstats) {
  RowArgs a = row_args(p, kstats);
  const long long nblk = (long long)a.nqt * p.B * p.Hkv * p.nhg;
  dim3 grid((unsigned)nblk), block(64 * p.HG * p.TC);   // 4 waves
  prof_begin("fwd", p.stream);
  if (p.D == 128) hipLaunchKernelGGL(fwd_kernel<128>, grid, block, 0, p.stream, a);
  else hipLaunchKernelGGL(fwd_kernel<64>, grid, block, 0, p.stream, a);
  prof_end(p.stream);
  return hipGetLastError();
}

hipError_t launch_bwd_pre(const Problem& p, int2* kstats, float* delta) {
  if (p.B > kMaxTraces) return hipErrorInvalidConfiguration;
  const long long rows = (long long)p.ntok * p.Hq;
  float* lse2 = (float*)((char*)delta + half_delta_bytes(p.Hq, p.ntok));
  const PreGrid pg = bwd_pre_grid(rows, (long long)kstats_groups(p.T) * p.B);
  if (!pg.with_kstats) {
    hipError_t e = launch_kstats(p, kstats);
    if (e != hipSuccess) return e;
  }
  const int nks = pg.with_kstats ? kstats_groups(p.T) * p.B : 0;
  dim3 grid(pg.blocks), block(256);
  prof_begin("bwd_pre", p.stream);
  if (p.D == 128)
    hipLaunchKernelGGL(bwd_pre_kernel<128>, grid, block, 0, p.stream, (const uint16_t*)p.o_in,
                       (const uint16_t*)p.dout, p.lse_in, delta, lse2, p.ntok, p.Hq, p.T, (int)(p.cu != nullptr),
                       p.evict, p.cu, nks, kstats);
  else
    hipLaunchKernelGGL(bwd_pre_kernel<64>, grid, block, 0, p.stream, (const uint16_t*)p.o_in,
                       (const uint16_t*)p.dout, p.lse_in, delta, lse2, p.ntok, p.Hq, p.T, (int)(p.cu != nullptr),
                       p.evict, p.cu, nks, kstats);
  prof_end(p.stream);
  return hipGetLastError();
}

hipError_t launch_bwd_dkdv(const Problem& p, const int2* kstats, const float* delta, void* split_ws,
                           size_t split_bytes) {
  ColArgs a{};
  a.q = (const uint16_t*)p.q;
  a.k = (const uint16_t*)p.k;
  a.v = (const uint16_t*)p.v;
  a.dout = (const uint16_t*)p.dout;
  a.lse = (const float*)((const char*)delta + half_delta_bytes(p.Hq, p.ntok));   // LSE * log2(e)
  a.delta = delta;
  a.evict = p.evict;
  a.cu = p.cu;
  a.dk = (uint16_t*)p.dk;
  a.dv = (uint16_t*)p.dv;
  a.B = p.B;
  a.T = p.T;
  a.Hq = p.Hq;
  a.Hkv = p.Hkv;
  a.G = p.G;
  a.nkt = (p.T + kColKeys - 1) / kColKeys;
  a.ntok = p.ntok;
  a.varlen = p.cu != nullptr;
  a.flags = p.flags;
  a.scale = p.scale;
  a.scale_log2 = p.scale * 1.4426950408889634f;
  const int cap = split_fit(p.B, p.T, p.Hkv, p.G, p.D, split_bytes);
  const SplitSpace sp = split_space(p.B, p.T, p.Hkv, p.D, cap);
  // one workgroup a CU, fewer if there cannot be as many items
  const int grid = (int)std::min<long long>(kCUs, ((long long)a.nkt * p.B + cap) * p.Hkv);
  char* w = (char*)split_ws;
  int* plan = cap ? (int*)w : nullptr;
  int2* items = (int2*)(w += sp.plan);
  PlanCtl* ctl = (PlanCtl*)(w += sp.items);
  int* split = (int*)(w += sp.ctl);   // split blocks
  a.part = (float*)(w + sp.split);
  a.nq = queue_count(p.Hkv, sp.ctl);
  a.plan = plan;
  // Without parts, and where every block starts at once, there is nothing to plan (5 us, and a launch).
  if (cap > 0 || (long long)p.B * a.nkt * p.Hkv > grid) {
    a.items = items;
    a.ctl = (int*)ctl;
    hipLaunchKernelGGL(split_plan_kernel, dim3(1), dim3(1024), 0, p.stream, kstats, p.cu, p.B, p.T, p.ntok, a.nkt, p.G,
                       p.Hkv, cap, grid, a.nq, plan, items, split, ctl);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  prof_begin("bwd_dkdv", p.stream);
  if (p.D == 128) hipLaunchKernelGGL(dkdv_kernel<128>, dim3(grid), dim3(512), 0, p.stream, a);
  else hipLaunchKernelGGL(dkdv_kernel<64>, dim3(grid), dim3(512), 0, p.stream, a);
  prof_end(p.stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || cap == 0) return e;
  if (p.D == 128)
    hipLaunchKernelGGL(split_reduce_kernel<128>, dim3(kReduceGrid), dim3(256), 0, p.stream, ctl, a.plan, split, a.part, p.cu,
                       (uint16_t*)p.dk, (uint16_t*)p.dv, p.B, p.T, p.ntok, a.nkt, p.Hkv, p.scale);
  else
    hipLaunchKernelGGL(split_reduce_kernel<64>, dim3(kReduceGrid), dim3(256), 0, p.stream, ctl, a.plan, split, a.part, p.cu,
                       (uint16_t*)p.dk, (uint16_t*)p.dv, p.B, p.T, p.ntok, a.nkt, p.Hkv, p.scale);
  return hipGetLastError();
}

hipError_t launch_bwd_dq(const Problem& p, const int2* kstats, const float* delta) {
  RowArgs a = row_args(p, kstats);
  a.delta = delta;
  a.lse_in = (const float*)((const char*)delta + half_delta_bytes(p.Hq, p.ntok));   // LSE * log2(e)
  const long long nblk = (long long)a.nqt * p.B * p.Hkv * p.nhg;
  dim3 grid((unsigned)nblk), block(64 * p.HG * p.TC);
  prof_begin("bwd_dq", p.stream);
  if (p.D == 128) hipLaunchKernelGGL(dq_kernel<128>, grid, block, 0, p.stream, a);
  else hipLaunchKernelGGL(dq_kernel<64>, grid, block, 0, p.stream, a);
  prof_end(p.stream);
  return hipGetLastError();
}

hipError_t launch_classify(const int32_t* evict, const int32_t* cu, int B, int T, int BM, int BN, uint8_t* out,
                           hipStream_t stream) {
  const int nk = (T + BN - 1) / BN, nq = (T + BM - 1) / BM;
  hipLaunchKernelGGL(classify_kernel, dim3((nk + kWave - 1) / kWave, nq, B), dim3(kWave), 0, stream, evict, cu, B,
                     T, BM, BN, out);
  return hipGetLastError();
}

hipError_t launch_check(const int32_t* evict, const int32_t* cu, int B, int T, int ntok, int64_t* first_bad,
                        int* cu_bad, hipStream_t stream) {
  hipLaunchKernelGGL(check_init_kernel, dim3(1), dim3(1), 0, stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  const int blocks = (T + 255) / 256 < 1024 ? (T + 255) / 256 : 1024;
  hipLaunchKernelGGL(check_kernel, dim3(blocks > 0 ? blocks : 1, B), dim3(256), 0, stream, evict, cu, B, T, ntok);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  unsigned long long fb = 0;
  int cb = 0;
  e = hipMemcpyFromSymbolAsync(&fb, HIP_SYMBOL(g_first_bad), sizeof(fb), 0, hipMemcpyDeviceToHost, stream);
  if (e != hipSuccess) return e;
  e = hipMemcpyFromSymbolAsync(&cb, HIP_SYMBOL(g_cu_bad), sizeof(cb), 0, hipMemcpyDeviceToHost, stream);
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(stream);
  if (e != hipSuccess) return e;
  *first_bad = (fb == ULLONG_MAX) ? -1 : (int64_t)fb;
  *cu_bad = cb;
  return hipSuccess;
}

}  // namespace kvs
