// Internal interface between the C ABI layer (kvs_api.cpp) and the kernel
// launchers (kvs_kernels.hip).  Not part of the public ABI.
#pragma once

#include <hip/hip_runtime_api.h>
#include <stdint.h>

namespace kvs {

// Problem description after host-side validation.
struct Problem {
  const void* q;
  const void* k;
  const void* v;
  const void* o_in;      // backward: forward output O
  const void* dout;      // backward: dO
  const float* lse_in;   // backward: forward LSE
  const int32_t* evict;
  const int32_t* cu;     // NULL: fixed length
  void* o;               // forward output
  float* lse;            // forward output
  void* dq;
  void* dk;
  void* dv;
  int B;
  int T;        // fixed: trace length; varlen: max_seqlen
  int ntok;     // total packed tokens
  int Hq, Hkv, D, G;
  int HG, TC, nhg;   // q-heads per workgroup, 32-token chunks per workgroup, head groups per KV head
  int flags;         // tile-classifier switches (kFlagNoEmptySkip, kFlagFullAsPartial); 0 normally
  float scale;
  void* ws;
  size_t ws_bytes;   // backward
  hipStream_t stream;
};

// Workspace pieces (byte offsets from the workspace start).
size_t ws_kstats_bytes(int B, int ntok);

// Library-owned scratch of the allocation-free forward: kNoAllocScratchBytes
// per GPU (device address of this device's copy in *ptr; taken once per device).
constexpr size_t kNoAllocScratchBytes = 256 * 1024;
constexpr int kMaxDevices = 64;
hipError_t noalloc_scratch(void** ptr);
size_t ws_delta_bytes(int Hq, int ntok);
size_t ws_split_bytes(int B, int T, int Hkv, int G, int D);   // that the dK/dV work plan can use
size_t ws_split_least(int B, int T, int Hkv, int D);          // that it needs

// Grid of the backward's preprocess: 16 rows a workgroup of 256 threads, and the workgroups of the key-tile statistics
// in front of them where a launch, of at most 2^32 - 1 threads, holds both.
struct PreGrid {
  unsigned blocks;
  bool with_kstats;
};
inline PreGrid bwd_pre_grid(long long rows, long long kstats_blocks) {
  const long long blocks = (rows + 15) / 16;
  const bool both = (blocks + kstats_blocks) * 256 <= 0xffffffffll;
  return {(unsigned)(both ? blocks + kstats_blocks : blocks), both};
}

// Launchers.  Each returns the hipError_t of its launch(es).
hipError_t launch_kstats(const Problem& p, int2* kstats);
hipError_t launch_fwd(const Problem& p, const int2* kstats);
hipError_t launch_bwd_pre(const Problem& p, int2* kstats, float* delta);   // and the key-tile statistics
hipError_t launch_bwd_dkdv(const Problem& p, const int2* kstats, const float* delta, void* split_ws,
                           size_t split_bytes);
hipError_t launch_bwd_dq(const Problem& p, const int2* kstats, const float* delta);
hipError_t launch_classify(const int32_t* evict, const int32_t* cu, int B, int T, int BM, int BN,
                           uint8_t* out, hipStream_t stream);
hipError_t launch_check(const int32_t* evict, const int32_t* cu, int B, int T, int ntok,
                        int64_t* first_bad, int* cu_bad, hipStream_t stream);

// Paged decode over the streamed KV cache (after host-side validation).
struct PagedDecode {
  const void* q;            // [S][Hq][D] bf16
  const void* k_cache;      // [num_blocks][Hkv][block_size][D] bf16
  const void* v_cache;
  const int32_t* slot_pos;  // [num_blocks * block_size]
  const int32_t* block_table;   // [S][max_blocks]
  const int32_t* seq_blocks;    // [S]
  void* o;                  // [S][Hq][D] bf16
  float* lse;               // [S][Hq]
  int S, Hq, Hkv, D, max_blocks, block_size, num_blocks;
  float scale;
  void* ws;
  size_t ws_bytes;
  hipStream_t stream;
};
// Slots of a host-held list as runs: |len| tokens from `tok` on, positions pos, pos + 1, ..., slots slot, slot + 1,
// ... (or slot, slot - 1, ... for len < 0).  Passed by value: 2 KB of launch arguments.
struct SlotRun {
  int tok, slot, pos, len;
};
constexpr int kMaxRuns = 128;
struct SlotRuns {
  int n;
  SlotRun r[kMaxRuns];
};
// How the run kernels share the runs' work, per_tok items a token.  Without a list: x workgroups for every run (y), in
// strides of 256 x items.  Where runs of unequal length would leave more than kIdleGroups of those without any: run i
// has workgroups first[i] to first[i + 1] - 1, of `items` items each (256, more beyond 65,535 workgroups).
struct NoRunList {
  static constexpr bool kListed = false;
};
struct RunList {
  static constexpr bool kListed = true;
  long long items;   // 0: no list
  int first[kMaxRuns];
};
constexpr int kIdleGroups = 4096;
inline dim3 run_grid(const SlotRuns& runs, long long per_tok, RunList* list) {
  auto work = [&](int i) { return (runs.r[i].len < 0 ? -(long long)runs.r[i].len : runs.r[i].len) * per_tok; };
  long long all = 0, busy = 0, each = 0;   // items; workgroups of all runs, of the longest
  for (int i = 0; i < runs.n; ++i) {
    const long long groups = (work(i) + 255) / 256;
    all += work(i);
    busy += groups;
    each = groups > each ? groups : each;
  }
  list->items = 0;
  if (each * runs.n - busy <= kIdleGroups) return dim3((unsigned)(each < 4096 ? each : 4096), (unsigned)runs.n);
  list->items = 256 * ((all + 256ll * 65535 - 1) / (256ll * 65535));
  unsigned wg = 0;
  for (int i = 0; i < runs.n; ++i) {
    list->first[i] = (int)wg;
    wg += (unsigned)((work(i) + list->items - 1) / list->items);
  }
  return dim3(wg);
}
hipError_t launch_paged_append_runs(const void* kn, const void* vn, const SlotRuns& runs, void* kc, void* vc,
                                    int* slot_pos, int num_slots, int BS, int Hkv, int D, hipStream_t stream);
hipError_t launch_paged_evict_runs(const SlotRuns& runs, int* slot_pos, int num_slots, hipStream_t stream);
size_t paged_ws_bytes(int S, int Hq, int Hkv, int max_blocks, int BS, int D);   // that the decode can use
size_t paged_ws_least(int S, int Hq, int Hkv, int max_blocks, int BS, int D);   // that it needs
hipError_t launch_paged_append(const void* kn, const void* vn, const int* pos, const int* slots, int n, void* kc,
                               void* vc, int* slot_pos, int num_slots, int BS, int Hkv, int D, hipStream_t stream);
hipError_t launch_paged_evict(const int* slots, int n, int* slot_pos, int num_slots, hipStream_t stream);
hipError_t launch_paged_decode(const PagedDecode& p);

// Per-kernel event bracketing (benchmark timing).
void prof_begin(const char* name, hipStream_t s);
void prof_end(hipStream_t s);

}  // namespace kvs
