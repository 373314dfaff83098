// Parts of the kernels that lay out expert segments, in 1024-thread workgroups:
// an inclusive scan over the workgroup, and the pads.
#pragma once
#include "common.hpp"

namespace moe {

constexpr int kPermThreads = 1024;

// Inclusive scan inside each 16-lane row of the wave with DPP shifts
// (row_shr:n, 0x110 + n; lanes whose source falls before the row read 0):
// VALU lane moves in place of ds_bpermute round trips.
__device__ __forceinline__ int row_inclusive_scan(int v) {
  v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xF, 0xF, true);
  v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xF, 0xF, true);
  return v;
}

// Inclusive scan of one int per thread across the block (blockDim = 1024):
// rows of 16 lanes, then the rows of each wave joined with row_bcast:15
// (0x142: lane 15 of rows 0 and 2 added to rows 1 and 3) and row_bcast:31
// (0x143: lane 31 added to rows 2 and 3), then the waves through LDS.
__device__ __forceinline__ int block_inclusive_scan(int v, int* wave_tot) {
  const int lane = lane_id(), wv = threadIdx.x >> 6;
  v = row_inclusive_scan(v);
  v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xA, 0xF, false);
  v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xC, 0xF, false);
  if (lane == 63) wave_tot[wv] = v;
  __syncthreads();
  if (wv == 0) {
    static_assert(kPermThreads / 64 <= 16, "the wave totals fit one row");
    int t = lane < (kPermThreads / 64) ? wave_tot[lane] : 0;
    t = row_inclusive_scan(t);
    if (lane < (kPermThreads / 64)) wave_tot[lane] = t;
  }
  __syncthreads();
  if (wv > 0) v += wave_tot[wv - 1];
  return v;
}

// Pad ids n of workgroup c of nc: a wave per segment, whose pads are positions
// [pad_begin[e], pad_end[e]), and the tail [total, cap), both spread over the
// workgroups (a thread per segment in one workgroup wrote up to block_m - 1 pads
// one after the other: 16 us for 300 tokens, 256 experts and 128-row tiles, 6.8
// this way).
__device__ __forceinline__ void write_pads(const int* pad_begin, const int* pad_end, int E, int total, int cap, int n,
                                           int32_t* sorted_ids, int c, int nc) {
  for (int e = c * (kPermThreads / 64) + (threadIdx.x >> 6); e < E; e += nc * (kPermThreads / 64))
    for (int p = pad_begin[e] + lane_id(); p < pad_end[e]; p += 64) sorted_ids[p] = n;
  for (int p = total + c * kPermThreads + threadIdx.x; p < cap; p += nc * kPermThreads) sorted_ids[p] = n;
}

}  // namespace moe
