// MoE Gate and permute of a small batch in one launch (the first node of the
// skeleton of Fig. 1 and the data movement in front of the second): one
// workgroup, one wave per token for the selection (gate_select.hpp), then the
// same stable permutation as permute.hip on the ids in LDS.
//
// Both steps are latency, most of it launch, first loads and the drain between
// them, and the permute read back ids that the gate had just written: 16 tokens
// took 7.1 + 5.8 us over 128 experts and 9.2 + 7.5 us over 256 in two launches,
// 11.5 and 15.3 us in one (9.5 and 13.2 with the gate's later arg-max).  One token per wave of the
// workgroup; where one CU is too few for them, two launches are faster
// (gate_permute_fits).
#include "block_scan.hpp"
#include "gate_select.hpp"
#include "launch.hpp"

namespace moe {

constexpr int kGpMaxT = kPermThreads / 64;
constexpr int kGpMaxE = 256;
constexpr int kGpMaxN = kGpMaxT * MOE_GATE_MAX_K;  // routed rows

// PART: the logits are the KS router partials lg[ks][T][E], summed in slice
// order (and written to logits_out, if given); else lg is the logits [T][E].
template <int EPL, bool PART>
__global__ __launch_bounds__(kPermThreads) void gate_permute_kernel(
    const float* __restrict__ lg, int KS, const float* __restrict__ bias, int T, int E, int k, int mode, int renorm,
    float scale, float* __restrict__ logits_out, int32_t* __restrict__ ids, float* __restrict__ w,
    int32_t* __restrict__ ids2, float* __restrict__ w2, int block_m, int32_t* __restrict__ offsets,
    int32_t* __restrict__ sorted_ids, int32_t* __restrict__ inv_pos, int cap) {
  constexpr bool RANK = EPL <= 1;  // as in the gate: ranks up to 64 experts, arg-max rounds above
  constexpr int NW = kPermThreads / 64;
  __shared__ uint32_t bitmap[64 * EPL * (kGpMaxN / 32)];  // [expert][W]: bit f % 32 of word f / 32: id f routes there
  __shared__ int32_t sid[kGpMaxN];
  __shared__ float slg[PART ? NW : 1][PART ? EPL * 64 : 1];
  __shared__ __attribute__((aligned(16))) double skey[RANK ? NW : 1][RANK ? EPL * 64 : 1];
  __shared__ double sval[RANK ? NW : 1][RANK ? EPL * 64 : 1];
  __shared__ double ssel[RANK ? NW : 1][RANK ? MOE_GATE_MAX_K : 1];
  __shared__ int base[64 * EPL], pad_begin[64 * EPL], pad_end[64 * EPL];
  __shared__ int wave_tot[NW];
  __shared__ int total_padded;
  const int tid = threadIdx.x, wv = tid >> 6, lane = lane_id();
  const int n = T * k, W = (n + 31) / 32;
  for (int i = tid; i < E * W; i += kPermThreads) bitmap[i] = 0;

  if (wv < T) {  // wave wv selects for token wv
    const float* row = lg + static_cast<size_t>(wv) * E;
    if constexpr (PART) {
#pragma unroll
      for (int i = 0; i < EPL; ++i) {
        const int e = lane + 64 * i;
        if (e >= E) continue;
        const float v = sum_slices<kRouterMaxKS>(row + e, KS, static_cast<size_t>(T) * E);
        slg[wv][e] = v;  // read back below by this same lane only
        if (logits_out) logits_out[static_cast<size_t>(wv) * E + e] = v;
      }
      row = slg[wv];
    }
    const int o = wv * k;
    if constexpr (RANK)
      gate_rank_row<EPL>(row, bias, E, k, mode, renorm, scale, sid + o, w + o, nullptr, w2 ? w2 + o : nullptr,
                         skey[wv], sval[wv], ssel[wv]);
    else
      gate_argmax_row<EPL>(row, bias, E, k, mode, renorm, scale, sid + o, w + o, nullptr, w2 ? w2 + o : nullptr);
  }
  __syncthreads();

  int my_e = -1;
  if (tid < n) {
    my_e = sid[tid];
    ids[tid] = my_e;
    if (ids2) ids2[tid] = my_e;
    if (my_e >= 0 && my_e < E) atomicOr(&bitmap[my_e * W + (tid >> 5)], 1u << (tid & 31));
    else my_e = -1;
  }
  __syncthreads();
  int tot = 0;
  if (tid < E)
    for (int i = 0; i < W; ++i) tot += __popc(bitmap[tid * W + i]);
  const int padded = (tot + block_m - 1) / block_m * block_m;
  const int incl = block_inclusive_scan(tid < E ? padded : 0, wave_tot);
  if (tid < E) {
    const int seg0 = incl - padded;
    base[tid] = seg0;
    pad_begin[tid] = seg0 + tot;
    pad_end[tid] = incl;
    offsets[tid] = seg0;
    if (tid == E - 1) {
      offsets[E] = incl;
      total_padded = incl;
    }
  }
  __syncthreads();
  write_pads(pad_begin, pad_end, E, total_padded, cap, n, sorted_ids, 0, 1);
  if (tid >= n) return;
  if (my_e < 0) {
    inv_pos[tid] = -1;
    return;
  }
  const uint32_t* row = bitmap + my_e * W;
  const int wi = tid >> 5;
  int pos = base[my_e] + __popc(row[wi] & ((1u << (tid & 31)) - 1u));
  for (int i = 0; i < wi; ++i) pos += __popc(row[i]);
  sorted_ids[pos] = tid;
  inv_pos[tid] = pos;
}

// Up to 8 tokens (two waves per SIMD) one launch is always the faster form: the
// whole layer, H = 256, I = 128, 8 tokens: 8 experts, top 2, 17.9 us, in two launches 20.1;
// 256 experts, top 8, 24.4 and 28.2, top 32, 64.7 and 67.4; with a router 23.7 and
// 24.3, 31.9 and 34.6, 72.9 and 73.6.  From 9 to 16 tokens the arg-max rounds of
// up to four waves per SIMD get in each other's way (16 tokens, 256 experts: top
// 8 34.6 and 36.4, top 12 50.0 and 50.2, top 16 56.7 and 55.6, top 32 85.4 and
// 77.3; rank selection up to 64 experts, top 32, 37.7 and 38.6), and so do the
// loads of the router's slices (8 experts 25.5 and 24.8, 256 experts, top 8, 46.7 and 43.3).
bool gate_permute_fits(int T, int E, int k, bool router) {
  if (T < 1 || T > kGpMaxT || E > kGpMaxE || k > MOE_GATE_MAX_K) return false;
  return T <= 8 || (!router && (E <= 64 || k <= 12));
}

hipError_t launch_gate_permute(const float* lg, int KS, const float* bias, int T, int E, int k, int mode, int renorm,
                               float scale, float* logits_out, int32_t* ids, float* w, int32_t* ids2, float* w2,
                               int block_m, int32_t* offsets, int32_t* sorted_ids, int32_t* inv_pos, int cap,
                               hipStream_t s) {
  if (!gate_permute_fits(T, E, k, KS > 0) || KS < 0 || KS > kRouterMaxKS) return hipErrorInvalidValue;
  const int epl = (E + 63) / 64;
#define MOE_GP_CASE(N, P)                                                                                         \
  hipLaunchKernelGGL((gate_permute_kernel<N, P>), dim3(1), dim3(kPermThreads), 0, s, lg, KS, bias, T, E, k, mode, \
                     renorm, scale, logits_out, ids, w, ids2, w2, block_m, offsets, sorted_ids, inv_pos, cap)
  if (KS > 0) {
    if (epl <= 1) MOE_GP_CASE(1, true);
    else if (epl <= 2) MOE_GP_CASE(2, true);
    else MOE_GP_CASE(4, true);
  } else {
    if (epl <= 1) MOE_GP_CASE(1, false);
    else if (epl <= 2) MOE_GP_CASE(2, false);
    else MOE_GP_CASE(4, false);
  }
#undef MOE_GP_CASE
  return hipGetLastError();
}

}  // namespace moe
