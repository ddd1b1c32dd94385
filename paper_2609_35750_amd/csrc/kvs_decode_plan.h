// The split of the paged decode's work into units, as plain arithmetic that
// the host (grid and workspace sizes) and the device (the plan itself) share.
//
// A unit is a run of a sequence's 32-slot tiles that one wave walks per KV
// head; every sequence gets at least one.  All sequences are cut with one size
// C, close to the smallest for which the units fit the grid (paged_units), so
// ragged sequences give equal waves and a table wider than what it holds costs
// nothing.
#pragma once

#include <hip/hip_runtime.h>

#include <algorithm>
#include <climits>

namespace kvs {

constexpr int kDecTile = 32;   // cache slots per tile
// Least tiles of a unit.  A lone wave takes about 2 us a tile (one memory
// latency), so small batches want many short units until the merge's reads
// outweigh it: one rollout of 4,096 entries took 14.0 us with 4, 11.6 with 2.
constexpr int kMinTiles = 2;
// Tiles of one sequence the plan tells apart (33 M slots); exact in fp32, and 1,024 of them in 31 bits.
constexpr int kTileCap = 1 << 20;
constexpr int kPlanRegs = 4, kPlanSeqs = kPlanRegs * 64;   // sequences a wave can plan for by itself

inline long long decode_round(int D) { return (D == 128 ? 4ll : 8ll) * 256; }   // resident waves of the chip

// Units of the decode grid per KV head: one round of the resident waves (D =
// 128: four per CU, D = 64: eight), and for more sequences than that half a
// round on top of one unit each, so that long sequences of a ragged batch can
// still be cut; at most one unit per kMinTiles tiles of the table width.
// Under a narrow table every sequence is one unit, which needs neither plan
// nor merge (6 to 9 us): up to two least units where waves are left over, and
// where one unit each fills the chip up to 8 tiles and 4 more a round, which
// bounds what cutting the longest possible sequence could save.  At that line
// (32/8 heads, D = 128, 512 slots wide, 256 sequences): all of 200 entries 47.2
// -> 41.3 us, eight of 512 beside 248 of 16 22.2 -> 30.4.
inline int paged_units(int S, int Hkv, int max_blocks, int BS, int D) {
  const long long round = decode_round(D), waves = (long long)S * Hkv;
  const long long tiles = ((long long)max_blocks * BS + kDecTile - 1) / kDecTile;
  if (tiles <= (waves < round ? 2 * kMinTiles : 8 + 4 * (waves / round))) return S;
  const long long slack = waves <= (1 << 20) ? (round / 2 + Hkv - 1) / Hkv : 0;
  const long long per_seq = (tiles + kMinTiles - 1) / kMinTiles;
  return (int)std::min(std::max((round + Hkv - 1) / Hkv, S + slack), S * per_seq);
}

// Rows of partial results, per q-head.  A sequence of n units needs n of them if n > 1 and none if n = 1, and the
// sequences before s have first - s units beyond their first: from row 2 (first - s) on it has 2 (n - 1) to itself.
// Where that is less than a row for every unit, it saves the rows of the sequences that are not cut.
__host__ __device__ __forceinline__ bool partials_paired(int S, int units) { return units < 2ll * S; }
__host__ __device__ __forceinline__ int partial_units(int S, int units) {
  return partials_paired(S, units) ? 2 * (units - S) : units;
}
__host__ __device__ __forceinline__ int partial_row(int S, int units, int s, int first) {
  return partials_paired(S, units) ? 2 * (first - s) : first;
}

// 32-slot tiles of ns slots, as the plan counts them
__host__ __device__ __forceinline__ int plan_tiles(int ns) {
  const unsigned t = ((unsigned)ns + kDecTile - 1) / kDecTile;
  return t < (unsigned)kTileCap ? (int)t : kTileCap;
}

// max(1, ceil(t / C)) for 0 <= t <= kTileCap, C >= 1, rcpC within 2^-22 of 1 / C (t rcpC is then within one of the
// quotient for every C >= 1)
__host__ __device__ __forceinline__ int unit_count(int t, int C, float rcpC) {
  int q = (int)((float)t * rcpC);
  int r = t - q * C;
  if (r < 0) --q, r += C;
  if (r >= C) ++q, r -= C;
  const int n = q + (r > 0);
  return n > 1 ? n : 1;
}

// Unit size for S sequences of `total` tiles in all, the longest of tmax, on
// `units` > S units.  least = ceil(total / units), below which they cannot fit;
// upper() = min(tmax, total / (units - S) + 1), where they do: from tmax on
// each is one unit, and sum max(1, ceil(t / C)) <= total / C + S.  Bisection
// between the two, to within one part in 2^fine.  units_at(C): units of size C.
template <class F, class H>
__host__ __device__ __forceinline__ int unit_size(int least, int units, int fine, F units_at, H upper) {
  int lo = least > kMinTiles ? least : kMinTiles;
  if (units_at(lo) <= units) return lo;
  int hi = upper();
  while (hi - lo > 1 + (hi >> fine)) {
    const int c = lo + (hi - lo) / 2;
    if (units_at(c) <= units) hi = c;
    else lo = c;
  }
  return hi;
}

}  // namespace kvs
