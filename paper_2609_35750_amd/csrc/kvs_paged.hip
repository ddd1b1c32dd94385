// gfx950 kernels of the streamed paged KV cache (the inference side of
// KV-streams: Section 2, "KV-streams"; Section 4, "Inference engine
// implementation").  The engine appends one (K, V) entry per generated token
// to a paged cache and drops evicted entries for good; a query attends over
// exactly the entries that are live when it is generated.
//
// Cache layout: K, V [num_blocks][Hkv][block_size][D] bf16 (a block holds one
// contiguous run of block_size rows per KV head); slot_pos [num_blocks *
// block_size] int32 holds the trace position of the token in a slot (slot =
// block * block_size + row), or -1 (empty or evicted).  A sequence's blocks are
// listed in its row of the block table.
//
// Decode: one wave per (sequence, KV head, split); how many splits a sequence
// gets follows from its blocks (decode_unit).  The wave walks its split's
// cache slots in tiles of 32, gathering each tile's K and V rows from their
// blocks into LDS with asynchronous global-to-LDS copies (double-buffered, no
// workgroup barrier: each wave owns its buffers), computes S^T = K Q^T with the
// G q-heads of the group as the MFMA N columns, masks slots that are empty,
// evicted or past the sequence's last slot, runs the online softmax per
// column and accumulates O^T += V^T P^T.  Partial (max, sum, O) of every split
// go to the workspace; a combine kernel merges them into O and LSE.
#include "kvs_decode_plan.h"
#include "kvs_device.h"
#include "kvs_launch.h"

#include <algorithm>
#include <climits>
#include <cstdlib>

namespace kvs {

// ---------------------------------------------------------------- append / evict
// Token t of the batch goes to cache slot slots[t]; slots outside [0, num_slots) are skipped.
template <int D>
__global__ void __launch_bounds__(256) paged_append_kernel(const uint16_t* __restrict__ kn,
                                                           const uint16_t* __restrict__ vn,
                                                           const int* __restrict__ pos, const int* __restrict__ slots,
                                                           int n, uint16_t* __restrict__ kc, uint16_t* __restrict__ vc,
                                                           int* __restrict__ slot_pos, int num_slots, int Hkv, int BS) {
  const long long per_tok = (long long)Hkv * (D / 8);   // 16-byte chunks per token and tensor
  const long long chunks = (long long)n * per_tok;
  for (long long c = (long long)blockIdx.x * blockDim.x + threadIdx.x; c < chunks;
       c += (long long)gridDim.x * blockDim.x) {
    const long long t = c / per_tok, r = c - t * per_tok;
    const int slot = slots[t];
    if ((unsigned)slot >= (unsigned)num_slots) continue;
    const int h = (int)(r / (D / 8)), d8 = (int)(r - (long long)h * (D / 8));
    const long long dst = ((((long long)(slot / BS) * Hkv + h) * BS + slot % BS) * D) + 8 * d8;
    *reinterpret_cast<uint4*>(kc + dst) = *reinterpret_cast<const uint4*>(kn + c * 8);
    *reinterpret_cast<uint4*>(vc + dst) = *reinterpret_cast<const uint4*>(vn + c * 8);
    if (r == 0) slot_pos[slot] = pos[t];
  }
}

__global__ void __launch_bounds__(256) paged_evict_kernel(const int* __restrict__ slots, int n,
                                                          int* __restrict__ slot_pos, int num_slots) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < n; i += gridDim.x * blockDim.x) {
    const int slot = slots[i];
    if ((unsigned)slot < (unsigned)num_slots) slot_pos[slot] = -1;
  }
}

// The same from slot lists the host holds, run by run: the slots a block manager
// hands out lie in a few runs (a block's rows, and often blocks in a row), which
// fit the launch's arguments, so nothing is uploaded.  Token i of a run: slot +
// i * step, position + i.  Workgroups by run (run_grid): with the longest
// run's number for each, one long run beside many short ones, which is what a
// fragmented free list hands out, starts up to 128 times what it needs.  4,096
// tokens in a row and 100 by themselves (8 heads, D = 128): append 47 us that
// way, 14 with a list of the runs' first workgroups (RunList).  Looking them up takes
// 0.6 us, as long as some 4,000 idle workgroups; up to that the run is blockIdx.y.
// The workgroup's run, the first of its items there, and how many of them it has.
__device__ __forceinline__ int run_of(const SlotRuns&, const NoRunList&, long long& begin, long long& items) {
  begin = blockIdx.x * 256ll;
  items = LLONG_MAX;   // in strides of the grid
  return blockIdx.y;
}
__device__ __forceinline__ int run_of(const SlotRuns& runs, const RunList& list, long long& begin, long long& items) {
  const int lane = threadIdx.x & 63;
  int k = -1;   // the last run that begins at or before this workgroup
#pragma unroll
  for (int h = 0; h < kMaxRuns; h += kWave)
    k += __builtin_popcountll(__ballot(h + lane < runs.n && list.first[h + lane] <= (int)blockIdx.x));
  k = __builtin_amdgcn_readfirstlane(k);
  items = list.items;
  begin = (blockIdx.x - list.first[k]) * items;
  return k;
}

template <int D, class L>
__global__ void __launch_bounds__(256) paged_append_runs_kernel(const uint16_t* __restrict__ kn,
                                                                const uint16_t* __restrict__ vn, SlotRuns runs,
                                                                uint16_t* __restrict__ kc, uint16_t* __restrict__ vc,
                                                                int* __restrict__ slot_pos, int num_slots, int Hkv,
                                                                int BS, L list) {
  long long begin, items;
  const SlotRun run = runs.r[run_of(runs, list, begin, items)];
  const long long per_tok = (long long)Hkv * (D / 8), chunks = (long long)(run.len < 0 ? -run.len : run.len) * per_tok;
  const long long end = items < chunks - begin ? begin + items : chunks, step = L::kListed ? 256 : gridDim.x * 256ll;
  for (long long c = begin + threadIdx.x; c < end; c += step) {
    const long long i = c / per_tok, r = c - i * per_tok, src = ((long long)run.tok + i) * per_tok + r;
    const long long slot = run.slot + (run.len < 0 ? -i : i);
    if (slot < 0 || slot >= num_slots) continue;
    const int h = (int)(r / (D / 8)), d8 = (int)(r - (long long)h * (D / 8));
    const long long dst = (((slot / BS) * Hkv + h) * BS + slot % BS) * D + 8 * d8;
    *reinterpret_cast<uint4*>(kc + dst) = *reinterpret_cast<const uint4*>(kn + src * 8);
    *reinterpret_cast<uint4*>(vc + dst) = *reinterpret_cast<const uint4*>(vn + src * 8);
    if (r == 0) slot_pos[slot] = (int)(run.pos + i);
  }
}

template <class L>
__global__ void __launch_bounds__(256) paged_evict_runs_kernel(SlotRuns runs, int* __restrict__ slot_pos,
                                                               int num_slots, L list) {
  long long begin, items;
  const SlotRun run = runs.r[run_of(runs, list, begin, items)];
  const int n = run.len < 0 ? -run.len : run.len, end = items < n - begin ? (int)(begin + items) : n;
  for (int i = (int)begin + threadIdx.x; i < end; i += L::kListed ? 256 : gridDim.x * 256) {
    const long long slot = (long long)run.slot + (run.len < 0 ? -i : i);
    if (slot >= 0 && slot < num_slots) slot_pos[slot] = -1;
  }
}

// ---------------------------------------------------------------- decode
struct DecodeArgs {
  const uint16_t* q;      // [S][Hq][D]
  const uint16_t* kc;     // [num_blocks][BS][Hkv][D]
  const uint16_t* vc;
  const int* slot_pos;    // [num_blocks * BS]
  const int* table;       // [S][max_blocks]
  const int* nblk;        // [S]
  // rows of the partials: partial_units * Hq, sequence s from partial_row * Hq on as [q-head][its units]
  float* part;            // [rows][D]: unnormalised O of each split (relative to its max)
  float2* part_ml;        // [rows]: max (log2 units), sum
  int plan;               // DecodePlan: how a wave finds its unit
  int2* seq_units;        // kByWave: [S], partial_row and number of units of the sequence
  int4* unit_seq;         // kListed: [units], sequence, its slots, its first unit, its units (0: no such unit)
  int* cut;               // kListed: number of cut sequences, their first units
  uint16_t* o;            // [S][Hq][D]: written here for sequences of one unit, by the merge for the others
  float* lse;             // [S][Hq]
  int S, Hq, Hkv, G, max_blocks, BS, num_blocks, units;
  float scale_log2;       // softmax_scale * log2(e)
};

__device__ __forceinline__ int partial_row(const DecodeArgs& a, int s, int first) {
  return partial_row(a.S, a.units, s, first);
}

// One unit a sequence; each wave plans by itself; looked up in unit_seq, which the plan kernel wrote.
enum DecodePlan : int { kOneUnit = 0, kByWave = 1, kListed = 2 };

// The 32-slot tile's K or V rows (D = 128: 18 x 16-byte slots per padded LDS
// row, 9 pieces of 64 lanes; D = 64: 9 per row, 4.5 pieces -> 5 with a guard).
template <int D>
struct GatherStager {
  using LY = Lay<D, true>;
  static constexpr int SLOTS = kDecTile * LY::CPRP;
  static constexpr int NI = (SLOTS + kWave - 1) / kWave;
  int row[NI];   // tile row of this lane's 16-byte slot (-1: none)
  int col[NI];   // element column in the source row
  __device__ __forceinline__ void init(int lane) {
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int q = i * kWave + lane;
      const int r = q / LY::CPRP, pc = q - r * LY::CPRP;
      row[i] = q < SLOTS ? r : -1;
      col[i] = (q < SLOTS && pc < LY::CPR) ? 8 * (pc ^ LY::flip(r)) : 0;
    }
  }
  // K and V rows of one tile.  roff: element offset of tile row (lane % 32)
  // in the caches (lanes 0..31, a valid row).  The offsets of all pieces are
  // exchanged first (one LDS round trip), then the copies are issued back to back.
  __device__ __forceinline__ void issue(uint32_t ldsK, uint32_t ldsV, const uint16_t* __restrict__ kb,
                                        const uint16_t* __restrict__ vb, long long roff) const {
    int lo[NI], hi[NI];
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      const int r = row[i] < 0 ? 0 : row[i];
      lo[i] = __shfl((int)(uint32_t)roff, r);
      hi[i] = __shfl((int)(roff >> 32), r);
    }
    __builtin_amdgcn_sched_barrier(0);   // all exchanges before the first copy
#pragma unroll
    for (int i = 0; i < NI; ++i) {
      if (i * kWave + kWave <= SLOTS || row[i] >= 0) {
        const long long off = (long long)(((uint64_t)(uint32_t)hi[i] << 32) | (uint32_t)lo[i]) + col[i];
        dma_b128_global(kb + off, ldsK + i * kWave * 16);
        dma_b128_global(vb + off, ldsV + i * kWave * 16);
      }
    }
  }
};

// The split of the decode's work (kvs_decode_plan.h).  Each wave finds its unit
// by itself from seq_blocks where that costs less than a plan of its own (up
// to four sequences a lane, and few rounds of waves: see launch_paged_decode);
// otherwise paged_plan_kernel lists the units once.  The lookup is one scalar
// load, and the merge walks the cut sequences only.
// Cutting every sequence into the same number of splits instead: 24 rollouts
// of 200 to 9,000 entries (D = 64, 195 MB) 51.8 -> 39.9 us, 40 of 500 to 8,000
// (D = 128, 674 MB) 162 -> 119 us, one of 16,000 beside 63 of 200 378 -> 36 us
// (these with the streamed gather).
struct DecodeUnit {
  int s, nslots, first, n, chunk;   // sequence, its slots, its first unit, its units, this one among them
};

// x / y for x >= 0, y >= 1: float quotient, corrected, where x is exact in fp32 (an integer division of the
// compiler's is several times the dependent instructions, on every wave's way to its first load)
__device__ __forceinline__ int quick_div(int x, int y) {
  if (x > kTileCap) return x / y;
  int q = (int)((float)x * __builtin_amdgcn_rcpf((float)y));
  const int r = x - q * y;
  return q + (r >= y) - (r < 0);
}

// slots of the blocks sequence s uses (clamped to the table width; some may be evicted)
__device__ __forceinline__ int slots_of(const DecodeArgs& a, int s) { return min(max(a.nblk[s], 0), a.max_blocks) * a.BS; }

// The unit u of up to 64 REGS sequences: its sequence, that one's slots, first unit and units.  False past the last one.
template <int REGS>
__device__ __forceinline__ bool plan_by_wave(const DecodeArgs& a, int u, int lane, int& s, int& ns, int& first, int& n) {
  int sl[REGS];   // slots of sequences 64 k + lane; -1: none
#pragma unroll
  for (int k = 0; k < REGS; ++k) {
    const int i = k * kWave + lane;
    sl[k] = k * kWave < a.S ? slots_of(a, min(i, a.S - 1)) : -1;
    if (i >= a.S) sl[k] = -1;
  }
  int sum = 0, top = 0;   // at most 2^28
#pragma unroll
  for (int k = 0; k < REGS; ++k) {
    const int t = plan_tiles(max(sl[k], 0));
    sum += t;
    top = max(top, t);
  }
  const int total = wave_last(wave_scan(sum));
  auto count = [&](int slots, int c, float rc) __attribute__((always_inline)) {
    return slots < 0 ? 0 : unit_count(plan_tiles(slots), c, rc);
  };
  auto units_at = [&](int c) __attribute__((always_inline)) {
    const float rc = __builtin_amdgcn_rcpf((float)c);
    int m = 0;
#pragma unroll
    for (int k = 0; k < REGS; ++k)
      if (k * kWave < a.S) m += count(sl[k], c, rc);
    return wave_last(wave_scan(m));
  };
  auto upper = [&]() __attribute__((always_inline)) {
    return min(wave_max(top), quick_div(total, a.units - a.S) + 1);
  };
  const int C = unit_size(quick_div(max(total - 1, 0), a.units) + 1, a.units, 30, units_at, upper);
  const float rc = __builtin_amdgcn_rcpf((float)C);
  int base = 0, l = -1;
#pragma unroll
  for (int k = 0; k < REGS; ++k) {
    if (k * kWave < a.S && l < 0) {
      const int m = count(sl[k], C, rc), incl = wave_scan(m);
      const unsigned long long hit = __ballot(u < base + incl);
      if (hit != 0ull) {
        l = __builtin_ctzll(hit);
        s = k * kWave + l;
        ns = __builtin_amdgcn_readlane(sl[k], l);
        n = __builtin_amdgcn_readlane(m, l);
        first = base + __builtin_amdgcn_readlane(incl, l) - n;
      }
      base += wave_last(incl);
    }
  }
  return l >= 0;
}

// The unit and KV head of workgroup `wg`; s = -1 past the last one.  All lanes
// of the wave take part.  A sequence's workgroups are consecutive, its units
// fastest, then the KV heads.
__device__ __forceinline__ DecodeUnit decode_unit(const DecodeArgs& a, int wg, int lane, int& g) {
  const int u = __builtin_amdgcn_readfirstlane(quick_div(wg, a.Hkv));
  g = wg - u * a.Hkv;
  if (a.plan == kOneUnit) return {u, slots_of(a, u), u, 1, 0};
  int s = 0, ns = 0, first = 0, n = 0;
  if (a.plan == kListed) {
    const int4 m = a.unit_seq[u];
    s = m.x, ns = m.y, first = m.z, n = m.w;
    if (n == 0) return {-1, 0, 0, 0, 0};
  } else if (a.S <= kWave ? !plan_by_wave<1>(a, u, lane, s, ns, first, n) : !plan_by_wave<kPlanRegs>(a, u, lane, s, ns, first, n)) {
    return {-1, 0, 0, 0, 0};
  }
  const int rem = wg - first * a.Hkv;
  g = __builtin_amdgcn_readfirstlane(quick_div(rem, n));
  return {s, ns, first, n, rem - g * n};
}

// The plan of all sequences in one workgroup: unit_seq and cut.
__global__ void __launch_bounds__(1024) paged_plan_kernel(DecodeArgs a) {
  constexpr int NW = 1024 / kWave, KEEP = 4;   // waves; sequences a thread keeps in registers
  __shared__ long long wsum[NW];
  __shared__ int wtop[NW], wcnt[2][NW], ncut;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  auto tiles = [&](int s) { return plan_tiles(slots_of(a, s)); };
  int t[KEEP];
#pragma unroll
  for (int k = 0; k < KEEP; ++k) t[k] = k * 1024 + tid < a.S ? tiles(k * 1024 + tid) : 0;
  if (tid == 0) ncut = 0;
  long long sum = 0;
  int top = 0;
  auto take = [&](int x) {
    sum += x;
    top = max(top, x);
  };
#pragma unroll
  for (int k = 0; k < KEEP; ++k) take(t[k]);
  for (int s = KEEP * 1024 + tid; s < a.S; s += 1024) take(tiles(s));
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) sum += __shfl_xor(sum, off);
  top = wave_max(top);
  if (lane == 0) {
    wsum[wave] = sum;
    wtop[wave] = top;
  }
  __syncthreads();
  long long total = 0;
#pragma unroll
  for (int w = 0; w < NW; ++w) {
    total += wsum[w];
    top = max(top, wtop[w]);
  }
  int turn = 0;   // of two sets of counts: a wave may be one count ahead of the slowest reader
  auto units_at = [&](int c) {
    const float rc = __builtin_amdgcn_rcpf((float)c);
    int m = 0;
#pragma unroll
    for (int k = 0; k < KEEP; ++k) m += k * 1024 + tid < a.S ? unit_count(t[k], c, rc) : 0;
    for (int s = KEEP * 1024 + tid; s < a.S; s += 1024) m += unit_count(tiles(s), c, rc);
    m = wave_last(wave_scan(m));
    turn ^= 1;
    if (lane == 0) wcnt[turn][wave] = m;
    __syncthreads();
    m = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) m += wcnt[turn][w];
    return m;
  };
  auto upper = [&]() { return (int)min((long long)top, total / (a.units - a.S) + 1); };
  const int C = unit_size((int)((max(total, 1ll) - 1) / a.units) + 1, a.units, 4, units_at, upper);
  const float rc = __builtin_amdgcn_rcpf((float)C);
  int base = 0;
  for (int s0 = 0; s0 < a.S; s0 += 1024) {
    const int s = s0 + tid, ns = s < a.S ? slots_of(a, s) : 0;
    const int m = s < a.S ? unit_count(plan_tiles(ns), C, rc) : 0, incl = wave_scan(m);
    turn ^= 1;
    if (lane == kWave - 1) wcnt[turn][wave] = incl;
    __syncthreads();
    int first = base + incl - m;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const int x = wcnt[turn][w];
      first += w < wave ? x : 0;
      base += x;
    }
    for (int i = 0; i < m; ++i) a.unit_seq[first + i] = make_int4(s, ns, first, m);
    if (m > 1) a.cut[1 + atomicAdd(&ncut, 1)] = first;
  }
  for (int u = base + tid; u < a.units; u += 1024) a.unit_seq[u] = make_int4(0, 0, 0, 0);
  __syncthreads();
  if (tid == 0) a.cut[0] = ncut;
}

// Copies in flight per wave: a ring of kDecRing tiles (K, V and the tile's
// slot_pos values), one ahead of the one being computed.  D = 128 uses 37 KB
// of LDS per wave, so four waves (one per SIMD) share a CU; D = 64 18 KB
// (eight).  A deeper ring costs SIMDs: four stages at two waves per CU
// measured 20% slower on the 64-rollout decode.
constexpr int kDecRing = 2;

// Wait until at most N vector memory operations of this wave are outstanding (N <= 63).
template <int N>
__device__ __forceinline__ void wait_vm_le() {
  static_assert(N >= 0 && N < 64, "vmcnt is six bits");
  __builtin_amdgcn_s_waitcnt(0x0F70 | (N & 15) | ((N >> 4) << 14));
}

// Every global read of the decode loop is an asynchronous copy to LDS, so all
// of them complete in issue order under one counter and each wait is exact
// (R = kDecRing):
// step n reads the block-table entries of tile n + R - 1 (copied during step
// n - 1), issues the table copy of tile n + R, the K/V copy of tile n + R - 1
// and the copy of its slot_pos values, and computes tile n once at most the
// copies of the R - 1 later steps are outstanding.  (A compiler-visible load
// consumed while copies are in flight would make the compiler wait for all
// of them, since it cannot see them.)
template <int D>
__global__ void __launch_bounds__(64) paged_decode_kernel(DecodeArgs a) {
  constexpr int KS = D / 16, DB = D / 32, PITCH = Lay<D, true>::PITCH, TILE = kDecTile * PITCH, R = kDecRing;
  constexpr int OPS_KV = 2 * GatherStager<D>::NI;   // K and V copy instructions per tile
  constexpr int OPS_STEP = OPS_KV + 2;             // plus the table and slot_pos copies
  static_assert((R - 1) * OPS_STEP < 64, "outstanding copies must fit vmcnt");
  __shared__ __attribute__((aligned(1024))) uint16_t sK[R * TILE];
  __shared__ __attribute__((aligned(1024))) uint16_t sV[R * TILE];
  __shared__ __attribute__((aligned(256))) int sTab[2][kWave];   // block-table entries of a tile's rows
  __shared__ __attribute__((aligned(256))) int sPos[R][kWave];   // slot_pos of a tile's rows

  const int lane = threadIdx.x, half = lane >> 5, col = lane & 31;
  int g;
  const DecodeUnit du = decode_unit(a, blockIdx.x, lane, g);
  if (du.s < 0) return;
  const int s = du.s;
  const auto rl = Lay<D, true>::row_lane(lane);
  const int tl = Lay<D, true>::tr_lo(lane), th = Lay<D, true>::tr_hi(lane);

  const int nslots = du.nslots;
  // the sequence's tiles in du.n equal runs
  const int tiles = (int)(((unsigned)nslots + kDecTile - 1) / kDecTile);
  const long long per = (long long)__builtin_amdgcn_readfirstlane(quick_div(tiles + du.n - 1, du.n)) * kDecTile;
  const int c_begin = (int)min(du.chunk * per, (long long)nslots);
  const int c_end = (int)min(c_begin + per, (long long)nslots);
  const int ntile = c_end > c_begin ? (int)(((unsigned)(c_end - c_begin) + kDecTile - 1) / kDecTile) : 0;

  // Q^T operand: column n = q-head g * G + n of the group (zero for n >= G)
  const int hcol = g * a.G + col;
  const bool col_ok = col < a.G;
  bf16x8 qreg[KS];
  {
    const uint16_t* qrow = a.q + ((size_t)s * a.Hq + (col_ok ? hcol : g * a.G)) * D + 8 * half;
#pragma unroll
    for (int ks = 0; ks < KS; ++ks) {
      const uint4 u = *reinterpret_cast<const uint4*>(qrow + 16 * ks);
      qreg[ks] = as_bf16x8(col_ok ? u : make_uint4(0u, 0u, 0u, 0u));
    }
  }
  f32x16 acc[DB];
#pragma unroll
  for (int d = 0; d < DB; ++d) acc[d] = f32x16{};
  float m_run = -INFINITY, l_run = 0.f;

  const int* trow = a.table + (size_t)s * a.max_blocks;
  const long long blk_stride = (long long)a.Hkv * a.BS * D;   // elements per cache block
  const uint16_t* kbase = a.kc + (long long)g * a.BS * D;
  const uint16_t* vbase = a.vc + (long long)g * a.BS * D;
  GatherStager<D> gst;
  gst.init(lane);

  // sequence-local slot index of tile row `col` of tile t (rows past c_end
  // repeat the split's last slot and are masked)
  auto slot_index = [&](int t) __attribute__((always_inline)) { return min(c_begin + t * kDecTile + col, c_end - 1); };
  // copy the block-table entries of tile t's rows (lanes 0..31) into sTab[t & 1]
  auto copy_table = [&](int t) __attribute__((always_inline)) {
    const int c = slot_index(t);
    if (lane < 32) dma_b32_global(trow + c / a.BS, lds_addr(&sTab[t & 1][0]));
  };

  unsigned valid_q[R] = {};   // rows of tiles n .. n + R - 1 that hold a slot of the split (index 0 = tile n)
  if (ntile > 0) copy_table(0);
  wait_vm_le<0>();   // Q and the first table entries are in (no compiler-visible load stays pending in the loop)
  for (int n = -(R - 1); n < ntile; ++n) {
    const int tn = n + R - 1;   // tile whose copies this step issues
    if (tn < ntile) {
      if (n > -(R - 1)) wait_vm_le<OPS_KV + 1>();   // table entries of tile tn have landed
      const int c = slot_index(tn);
      const int blk = sTab[tn & 1][col];
      // a table entry outside the cache reads slot 0 and is masked
      const bool bok = (unsigned)blk < (unsigned)a.num_blocks;
      const int slot = bok ? blk * a.BS + c % a.BS : 0;
      const long long roff = bok ? (long long)blk * blk_stride + (long long)(c % a.BS) * D : 0;
      copy_table(min(tn + 1, ntile - 1));   // always one copy, so that every step issues the same count
      gst.issue(lds_addr(sK + (tn % R) * TILE), lds_addr(sV + (tn % R) * TILE), kbase, vbase, roff);
      if (lane < 32) dma_b32_global(a.slot_pos + slot, lds_addr(&sPos[tn % R][0]));
      valid_q[R - 1] = (unsigned)__ballot(lane < 32 && c_begin + tn * kDecTile + col < c_end && bok);
      if (n >= 0) wait_vm_le<(R - 1) * OPS_STEP>();   // tile n has landed
    } else if (n >= 0) {
      wait_vm_le<0>();
    }
    if (n >= 0) {
      const unsigned live_cur = valid_q[0] & (unsigned)__ballot(lane < 32 && sPos[n % R][col] >= 0);
      const uint16_t* cK = sK + (n % R) * TILE;
      const uint16_t* cV = sV + (n % R) * TILE;
      if (live_cur != 0u) {
        // S^T block: keys on M (tile rows), q-heads on N
        f32x16 sc = f32x16{};
        bf16x8 ka[KS];
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) ka[ks] = lds_read_b128(cK + Lay<D, true>::row_at(rl, ks));
#pragma unroll
        for (int ks = 0; ks < KS; ++ks) sc = mfma32(ka[ks], qreg[ks], sc);
        // element r <-> tile row 8 (r / 4) + 4 half + r % 4
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          const int row = 8 * (r >> 2) + 4 * half + (r & 3);
          if (!((live_cur >> row) & 1u)) sc[r] = -INFINITY;
        }
        float mx = -INFINITY;
#pragma unroll
        for (int r = 0; r < 16; ++r) mx = fmaxf(mx, sc[r]);
        mx = halves_max(mx) * a.scale_log2;
        // P is taken against the tile's own maximum, not the running one: what bf16 makes of it (the largest is 1,
        // exactly) then depends on the tile alone and not on how many tiles the unit has.
        const float m_tile = mx == -INFINITY ? 0.f : mx;
        float l_tile = 0.f;
#pragma unroll
        for (int r = 0; r < 16; ++r) {
          sc[r] = __builtin_amdgcn_exp2f(__builtin_fmaf(sc[r], a.scale_log2, -m_tile));
          l_tile += sc[r];
        }
        f32x16 ot[DB] = {};
#pragma unroll
        for (int t2 = 0; t2 < 2; ++t2) {
          const bf16x8 pb = pack8(sc, 8 * t2);
#pragma unroll
          for (int d = 0; d < DB; ++d) ot[d] = mfma32(tr_operand<D, true>(cV, 16 * t2, 32 * d, tl, th), pb, ot[d]);
        }
        if (mx > m_run) {   // per column (lane)
          const float alpha = __builtin_amdgcn_exp2f(m_run - mx);   // 0 on the first live tile
          l_run *= alpha;
#pragma unroll
          for (int d = 0; d < DB; ++d)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[d][r] *= alpha;
          m_run = mx;
        }
        const float beta = __builtin_amdgcn_exp2f(mx - (m_run == -INFINITY ? 0.f : m_run));
        l_run = __builtin_fmaf(l_tile, beta, l_run);
#pragma unroll
        for (int d = 0; d < DB; ++d)
#pragma unroll
          for (int r = 0; r < 16; ++r) acc[d][r] = __builtin_fmaf(ot[d][r], beta, acc[d][r]);
      }
    }
#pragma unroll
    for (int i = 0; i < R - 1; ++i) valid_q[i] = valid_q[i + 1];
    valid_q[R - 1] = 0u;
  }

  if (a.plan == kByWave && lane == 0 && g == 0 && du.chunk == 0) a.seq_units[s] = make_int2(partial_row(a, s, du.first), du.n);
  const float l_tot = halves_sum(l_run);
  if (!col_ok) return;
  if (du.n == 1) {   // the sequence's only unit: O and LSE directly
    const float inv = l_tot > 0.f ? 1.f / l_tot : 0.f;
    uint16_t* orow = a.o + ((size_t)s * a.Hq + hcol) * D;
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<uint2*>(orow + 32 * d + 8 * q4 + 4 * half) =
            pack4_bf16(acc[d][4 * q4] * inv, acc[d][4 * q4 + 1] * inv, acc[d][4 * q4 + 2] * inv,
                       acc[d][4 * q4 + 3] * inv);
    if (half == 0) a.lse[(size_t)s * a.Hq + hcol] = l_tot > 0.f ? (m_run + __log2f(l_tot)) * 0.6931471805599453f : -INFINITY;
    return;
  }
  // partial of this unit for q-head column `col`
  const size_t pidx = (size_t)partial_row(a, s, du.first) * a.Hq + (size_t)hcol * du.n + du.chunk;
  float* dst = a.part + pidx * D;
  if (l_tot > 0.f) {   // an empty unit leaves its O unwritten (the merge skips it)
#pragma unroll
    for (int d = 0; d < DB; ++d)
#pragma unroll
      for (int q4 = 0; q4 < 4; ++q4)
        *reinterpret_cast<float4*>(dst + 32 * d + 8 * q4 + 4 * half) =
            make_float4(acc[d][4 * q4], acc[d][4 * q4 + 1], acc[d][4 * q4 + 2], acc[d][4 * q4 + 3]);
  }
  if (half == 0) a.part_ml[pidx] = make_float2(m_run, l_tot);
}

// Merge the splits of one (sequence, q-head): W waves.  The split weights
// exp2(m_i - M) are computed in parallel (one thread per split) and kept in
// LDS, then D / 4 lanes read one split's partial each as float4 and the
// 64 W / (D / 4) groups of lanes take the splits in turn.  Bound by the
// latency of its reads: one wave walking the splits in series took 71.6 us
// for 32 rows of 128 splits (one 16,000-token rollout, 32 q-heads), four waves
// 7.1, sixteen with the first partials requested before the weights are known
// about 4.5; 8.7 -> 4.5 us for 576 rows of 11 splits.
constexpr int kMaxSplit = 2048;   // splits of one sequence: at most one round of resident waves, see paged_units
template <int D, int W>
__device__ __forceinline__ void combine_row(const DecodeArgs& a, int r, int2 su) {
  constexpr int LPS = D / 4, P = kWave * W / LPS;   // lanes per split, splits per pass
  __shared__ float sw[kMaxSplit];
  __shared__ float sred[2][W];
  __shared__ float4 sx[kWave * W];
  const int tid = threadIdx.x, wave = tid >> 6;
  const int nsplit = min(su.y, kMaxSplit);
  const size_t row0 = (size_t)su.x * a.Hq + (size_t)(r % a.Hq) * su.y;   // split i is row row0 + i
  const float2* ml = a.part_ml + row0;
  const float4* pv = reinterpret_cast<const float4*>(a.part + row0 * D) + (tid & (LPS - 1));
  // the first passes' partials are requested before the weights are known
  constexpr int PRE = 4;
  float4 pre[PRE];
#pragma unroll
  for (int k = 0; k < PRE; ++k) pre[k] = pv[(size_t)min(tid / LPS + k * P, nsplit - 1) * LPS];
  float M = -INFINITY;
  for (int i = tid; i < nsplit; i += kWave * W) M = fmaxf(M, ml[i].x);
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) M = fmaxf(M, __shfl_xor(M, off));
  if (W > 1) {
    if ((tid & 63) == 0) sred[0][wave] = M;
    __syncthreads();
#pragma unroll
    for (int k = 0; k < W; ++k) M = fmaxf(M, sred[0][k]);
  }
  float L = 0.f;
  for (int i = tid; i < nsplit; i += kWave * W) {
    const float2 v = ml[i];
    const float w = v.y <= 0.f ? -1.f : __builtin_amdgcn_exp2f(v.x - M);   // -1: empty split, its O is unwritten
    sw[i] = w;
    if (!(w < 0.f)) L += v.y * w;
  }
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) L += __shfl_xor(L, off);
  if (W > 1 && (tid & 63) == 0) sred[1][wave] = L;
  __syncthreads();
  if (W > 1) {
    L = 0.f;
#pragma unroll
    for (int k = 0; k < W; ++k) L += sred[1][k];
  }
  float4 x = make_float4(0.f, 0.f, 0.f, 0.f);
  auto add = [&](const float4& v, float w) __attribute__((always_inline)) {
    if (w < 0.f) return;
    x.x += v.x * w;
    x.y += v.y * w;
    x.z += v.z * w;
    x.w += v.w * w;
  };
#pragma unroll
  for (int k = 0; k < PRE; ++k) {
    const int i = tid / LPS + k * P;
    if (i < nsplit) add(pre[k], sw[i]);
  }
#pragma unroll 4
  for (int i = tid / LPS + PRE * P; i < nsplit; i += P) add(pv[(size_t)i * LPS], sw[i]);
  sx[tid] = x;
  __syncthreads();
  if (tid < LPS) {
#pragma unroll
    for (int k = 1; k < P; ++k) {
      const float4 v = sx[tid + k * LPS];
      x.x += v.x;
      x.y += v.y;
      x.z += v.z;
      x.w += v.w;
    }
    const float inv = L > 0.f ? 1.f / L : 0.f;
    reinterpret_cast<uint2*>(a.o + (size_t)r * D)[tid] = pack4_bf16(x.x * inv, x.y * inv, x.z * inv, x.w * inv);
    if (tid == 0) a.lse[r] = L > 0.f ? (M + __log2f(L)) * 0.6931471805599453f : -INFINITY;
  }
}

// One row a workgroup (those of one split the decode has written itself), or, where they are listed, all rows of
// the cut sequences.
template <int D, int W, bool LISTED>
__global__ void __launch_bounds__(64 * W) paged_combine_kernel(DecodeArgs a) {
  if (!LISTED) {
    const int2 su = a.seq_units[blockIdx.x / a.Hq];
    if (su.y > 1) combine_row<D, W>(a, blockIdx.x, su);
    return;
  }
  const int rows = a.cut[0] * a.Hq;
  for (int i = blockIdx.x; i < rows; i += gridDim.x) {
    const int4 m = a.unit_seq[a.cut[1 + i / a.Hq]];
    combine_row<D, W>(a, m.x * a.Hq + i % a.Hq, make_int2(partial_row(a, m.x, m.z), m.w));
    __syncthreads();   // the next row's weights
  }
}

template __global__ void paged_append_kernel<64>(const uint16_t*, const uint16_t*, const int*, const int*, int,
                                                 uint16_t*, uint16_t*, int*, int, int, int);
template __global__ void paged_append_kernel<128>(const uint16_t*, const uint16_t*, const int*, const int*, int,
                                                  uint16_t*, uint16_t*, int*, int, int, int);
#define KVS_RUNS(LL)                                                                                               \
  template __global__ void paged_append_runs_kernel<64, LL>(const uint16_t*, const uint16_t*, SlotRuns, uint16_t*, \
                                                            uint16_t*, int*, int, int, int, LL);                   \
  template __global__ void paged_append_runs_kernel<128, LL>(const uint16_t*, const uint16_t*, SlotRuns, uint16_t*, \
                                                             uint16_t*, int*, int, int, int, LL);                  \
  template __global__ void paged_evict_runs_kernel<LL>(SlotRuns, int*, int, LL)
KVS_RUNS(NoRunList);
KVS_RUNS(RunList);
#undef KVS_RUNS
template __global__ void paged_decode_kernel<64>(DecodeArgs);
template __global__ void paged_decode_kernel<128>(DecodeArgs);
template __global__ void paged_combine_kernel<64, 1, false>(DecodeArgs);
template __global__ void paged_combine_kernel<64, 4, false>(DecodeArgs);
template __global__ void paged_combine_kernel<64, 16, false>(DecodeArgs);
template __global__ void paged_combine_kernel<128, 1, false>(DecodeArgs);
template __global__ void paged_combine_kernel<128, 4, false>(DecodeArgs);
template __global__ void paged_combine_kernel<128, 16, false>(DecodeArgs);
template __global__ void paged_combine_kernel<64, 4, true>(DecodeArgs);
template __global__ void paged_combine_kernel<128, 4, true>(DecodeArgs);

// ---------------------------------------------------------------- launchers
template <class L>
static void launch_append_runs(dim3 grid, const void* kn, const void* vn, const SlotRuns& runs, void* kc, void* vc,
                               int* slot_pos, int num_slots, int BS, int Hkv, int D, const L& list, hipStream_t stream) {
  const auto kernel = D == 128 ? paged_append_runs_kernel<128, L> : paged_append_runs_kernel<64, L>;
  hipLaunchKernelGGL(kernel, grid, dim3(256), 0, stream, (const uint16_t*)kn, (const uint16_t*)vn, runs, (uint16_t*)kc,
                     (uint16_t*)vc, slot_pos, num_slots, Hkv, BS, list);
}
hipError_t launch_paged_append_runs(const void* kn, const void* vn, const SlotRuns& runs, void* kc, void* vc,
                                    int* slot_pos, int num_slots, int BS, int Hkv, int D, hipStream_t stream) {
  RunList list;
  const dim3 grid = run_grid(runs, (long long)Hkv * (D / 8), &list);
  if (list.items) launch_append_runs(grid, kn, vn, runs, kc, vc, slot_pos, num_slots, BS, Hkv, D, list, stream);
  else launch_append_runs(grid, kn, vn, runs, kc, vc, slot_pos, num_slots, BS, Hkv, D, NoRunList{}, stream);
  return hipGetLastError();
}

hipError_t launch_paged_evict_runs(const SlotRuns& runs, int* slot_pos, int num_slots, hipStream_t stream) {
  RunList list;
  const dim3 grid = run_grid(runs, 1, &list);
  if (list.items)
    hipLaunchKernelGGL(paged_evict_runs_kernel<RunList>, grid, dim3(256), 0, stream, runs, slot_pos, num_slots, list);
  else
    hipLaunchKernelGGL(paged_evict_runs_kernel<NoRunList>, grid, dim3(256), 0, stream, runs, slot_pos, num_slots,
                       NoRunList{});
  return hipGetLastError();
}

static size_t round256(size_t n) { return (n + 255) & ~(size_t)255; }
// Partial results and what the waves and the merge look units up in; nothing for one unit a sequence.
static size_t units_bytes(int S, int Hq, int D, int units) {
  if (units <= S) return 0;
  const size_t rows = (size_t)partial_units(S, units) * Hq;
  return round256(rows * D * sizeof(float)) + round256(rows * sizeof(float2)) + round256((size_t)S * sizeof(int2)) +
         round256((size_t)units * sizeof(int4));
}
// Partial results of equal splits, as many a sequence as make one round of waves, of four tiles of the table's width
// at least.
static size_t equal_splits_bytes(int S, int Hq, int Hkv, int max_blocks, int BS, int D) {
  const long long waves = (long long)S * Hkv, most = std::max(1ll, (long long)max_blocks * BS / (4 * kDecTile));
  const size_t rows = (size_t)S * Hq * std::min((decode_round(D) + waves - 1) / waves, most);
  return round256(rows * D * sizeof(float)) + round256(rows * sizeof(float2));
}
// What the query gives; never less than equal splits took.
size_t paged_ws_bytes(int S, int Hq, int Hkv, int max_blocks, int BS, int D) {
  return std::max(units_bytes(S, Hq, D, paged_units(S, Hkv, max_blocks, BS, D)),
                  equal_splits_bytes(S, Hq, Hkv, max_blocks, BS, D));
}
// At most `want` units that fit `bytes`.
static int fitting_units(int S, int Hq, int D, int want, size_t bytes) {
  while (want > S && units_bytes(S, Hq, D, want) > bytes) --want;
  return want;
}
// The least a call takes: that of equal splits where it holds all but a sixteenth of the units (short of the query
// by what they are looked up in), the query's size where it does not (narrow tables, whose units may be shorter than
// four tiles).
size_t paged_ws_least(int S, int Hq, int Hkv, int max_blocks, int BS, int D) {
  const int want = paged_units(S, Hkv, max_blocks, BS, D);
  const size_t equal = equal_splits_bytes(S, Hq, Hkv, max_blocks, BS, D);
  return units_bytes(S, Hq, D, std::max(S, want - want / 16)) <= equal ? equal
                                                                     : paged_ws_bytes(S, Hq, Hkv, max_blocks, BS, D);
}

hipError_t launch_paged_append(const void* kn, const void* vn, const int* pos, const int* slots, int n, void* kc,
                               void* vc, int* slot_pos, int num_slots, int BS, int Hkv, int D, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const long long chunks = (long long)n * Hkv * (D / 8);
  const int blocks = (int)std::min<long long>((chunks + 255) / 256, 65535);
  if (D == 128)
    hipLaunchKernelGGL(paged_append_kernel<128>, dim3(blocks), dim3(256), 0, stream, (const uint16_t*)kn,
                       (const uint16_t*)vn, pos, slots, n, (uint16_t*)kc, (uint16_t*)vc, slot_pos, num_slots, Hkv, BS);
  else
    hipLaunchKernelGGL(paged_append_kernel<64>, dim3(blocks), dim3(256), 0, stream, (const uint16_t*)kn,
                       (const uint16_t*)vn, pos, slots, n, (uint16_t*)kc, (uint16_t*)vc, slot_pos, num_slots, Hkv, BS);
  return hipGetLastError();
}

hipError_t launch_paged_evict(const int* slots, int n, int* slot_pos, int num_slots, hipStream_t stream) {
  if (n == 0) return hipSuccess;
  const int blocks = std::min((n + 255) / 256, 4096);
  hipLaunchKernelGGL(paged_evict_kernel, dim3(blocks), dim3(256), 0, stream, slots, n, slot_pos, num_slots);
  return hipGetLastError();
}

// One wave a row while it covers the splits in four passes (8 splits at D = 128, 16 at D = 64): many rows
// then, and one wave without a cross-wave exchange takes 4.9 us for 2,048 rows of two splits.  Beyond that
// few rows with many splits each: four waves (11.3 -> 4.0 us for 256 rows of 16 splits), sixteen
// beyond sixteen passes (9.8 -> 6.2 us for 32 rows of 128).  These rows had equal splits: the width follows the
// average, so that a lone long sequence of a ragged batch is merged by one wave (63 splits beside 63 sequences of
// one).  Listed sequences are few and long: four waves.
template <int W, bool LISTED>
static void launch_combine(int D, int grid, const DecodeArgs& a, hipStream_t stream) {
  if (D == 128) hipLaunchKernelGGL((paged_combine_kernel<128, W, LISTED>), dim3(grid), dim3(kWave * W), 0, stream, a);
  else hipLaunchKernelGGL((paged_combine_kernel<64, W, LISTED>), dim3(grid), dim3(kWave * W), 0, stream, a);
}
static void launch_combine(int D, const DecodeArgs& a, hipStream_t stream) {
  const int pass = D == 128 ? 2 : 4, avg = a.units / a.S;   // splits one wave reads at a time; units per sequence
  if (a.plan == kListed)
    launch_combine<4, true>(D, (int)std::min(std::min(a.S, a.units - a.S) * (long long)a.Hq, 2048ll), a, stream);
  else if (avg > 16 * pass) launch_combine<16, false>(D, a.S * a.Hq, a, stream);
  else if (avg > 4 * pass) launch_combine<4, false>(D, a.S * a.Hq, a, stream);
  else launch_combine<1, false>(D, a.S * a.Hq, a, stream);
}

// Rounds of waves up to which each wave plans by itself (about 1 us a round, in every wave), beyond which a plan
// kernel does (4 to 6 us, and a launch).  By wave against listed: 64 sequences of 200 entries (one round) 18.4 and
// 22.0 us, 128 (1.5 rounds) 24.4 and 27.5, 256 (2.5 rounds) 45.3 and 46.4 (32/8 heads, D = 128).  More than kPlanSeqs
// sequences were planned by wave too, at a cost that grows with their square: 2,048 of 200 347 us with no plan, 501
// by wave, 294 now; 4,096 of 100 394, 1,050, 349; 1,024 of 300 under a wide table (8/2, D = 64) 31.7, 41.7, 35.9; one
// of 16,000 beside 299 of 200 749, 78.5, 72.0.
constexpr int kPlanRounds = 3;

hipError_t launch_paged_decode(const PagedDecode& p) {
  DecodeArgs a{};
  a.q = (const uint16_t*)p.q;
  a.kc = (const uint16_t*)p.k_cache;
  a.vc = (const uint16_t*)p.v_cache;
  a.slot_pos = p.slot_pos;
  a.table = p.block_table;
  a.nblk = p.seq_blocks;
  a.S = p.S;
  a.Hq = p.Hq;
  a.Hkv = p.Hkv;
  a.G = p.Hq / p.Hkv;
  a.max_blocks = p.max_blocks;
  a.BS = p.block_size;
  a.num_blocks = p.num_blocks;
  a.units = fitting_units(p.S, p.Hq, p.D, paged_units(p.S, p.Hkv, p.max_blocks, p.block_size, p.D), p.ws_bytes);
  a.o = (uint16_t*)p.o;
  a.lse = p.lse;
  const size_t rows = (size_t)partial_units(p.S, a.units) * p.Hq;
  a.part = (float*)p.ws;
  a.part_ml = (float2*)((char*)p.ws + round256(rows * p.D * sizeof(float)));
  a.seq_units = (int2*)((char*)a.part_ml + round256(rows * sizeof(float2)));
  a.cut = (int*)a.seq_units;   // their number and no more than S first units: at most S + 1 of 2 S words
  a.unit_seq = (int4*)((char*)a.seq_units + round256((size_t)p.S * sizeof(int2)));
  a.scale_log2 = p.scale * 1.4426950408889634f;
  const dim3 grid((unsigned)((long long)a.units * p.Hkv));
  a.plan = a.units == p.S ? kOneUnit
           : p.S <= kPlanSeqs && (long long)a.units * p.Hkv <= kPlanRounds * decode_round(p.D) ? kByWave : kListed;
  if (a.plan == kListed) hipLaunchKernelGGL(paged_plan_kernel, dim3(1), dim3(1024), 0, p.stream, a);
  prof_begin("paged_decode", p.stream);
  if (p.D == 128) hipLaunchKernelGGL(paged_decode_kernel<128>, grid, dim3(64), 0, p.stream, a);
  else hipLaunchKernelGGL(paged_decode_kernel<64>, grid, dim3(64), 0, p.stream, a);
  prof_end(p.stream);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess || a.plan == kOneUnit) return e;
  launch_combine(p.D, a, p.stream);
  return hipGetLastError();
}

}  // namespace kvs
