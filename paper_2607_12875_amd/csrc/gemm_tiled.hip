// Grouped expert GEMMs, LDS-tiled, for the three weight formats (the "Fused
// MoE" node of the paper's skeleton, Fig. 1 / Fig. 3; the quantised formats
// carry the numeric semantics Sec. 6.2 asks of quantised routes):
//   GEMM1  a = SiLU(x W1[e,:I]^T) * (x W1[e,I:]^T)     (SiLU*up epilogue)
//   GEMM2  y = a W2[e]^T
//
//  bf16  A, B bf16; v_mfma_f32_32x32x16_bf16.
//  fp8   A (activations) and B (weights) OCP e4m3; v_mfma_f32_32x32x64_f8f6f4
//        with W as the first operand (the product is formed transposed),
//        one 128-wide K block at a time into a fresh partial, then
//        acc += partial * s_row(A) * s_block(B) on the VALU, overlapped with
//        the next blocks' MFMAs.  The GEMM1 epilogue requantises the
//        intermediate per (row, 128 columns): the tile holds exactly one such
//        group per row.
//  int4  A bf16; B signed int4 words decoded in registers to the exact bf16
//        136 + q right before the bf16 MFMA, never materialised; the bias comes
//        off through the activations' group sums and the group scale is applied
//        to the fp32 sums.  The decode takes 7 operations per word; on long K
//        it is interleaved with the MFMAs, one workgroup per CU and 256
//        elements per step, so that each weight row gives whole lines: a layer of
//        512 tokens, 4096 x 1536 x 128 experts, top 8, takes 365 us (388 with
//        128-element steps and two workgroups per CU, where the decode sets the
//        time; 433 with 14 and 28 operations per word).  Short K with many tiles
//        takes the 128-element steps.
//  mxfp4 A bf16; B OCP MX E2M1 codes with an E8M0 scale per 32 elements,
//        decoded by v_cvt_scalef32_pk_bf16_fp4 (exact: the bf16 result is the
//        code's value times a power of two) right before the bf16 MFMA.
// Every GEMM2 but int4's (whose scales and biases fit the direct layout) also
// forms its product transposed (four consecutive output columns per lane, so y
// goes out in 16-byte stores).
//
// Each K step streams KB bytes of every A row through LDS -- 128 (64 bf16 /
// 128 fp8 elements), 256 for the 4-bit weights (128 elements beside bf16
// activations, where each weight row gives 64 bytes, half a cache line; 256 beside
// MXFP8, a whole one) or 512 (256 elements, int4) -- in 16-byte chunks XOR-swizzled by row
// so that the fragment reads are bank-conflict free; B rows likewise.
//
// Scheduling is persistent and XCD-aware: the launch has a few workgroups per
// CU; workgroups that land on one XCD (block ids congruent mod 8) own one
// contiguous range of logical tiles, ordered expert by expert in chunks of at
// most GM row tiles x all column tiles, so that concurrently running workgroups
// share a weight slab and row tiles in L2 as long as they stay in step.  The
// number of real row tiles is read on the device from expert_offsets[E]
// (segments are padded to BM).
#include <algorithm>
#include <type_traits>

#include "common.hpp"
#include "launch.hpp"
#include "lds_dma.hpp"

namespace moe {

constexpr int kXcds = 8;
constexpr int MOE_MAX_EXPERTS_DEV = 1024;  // the ABI's expert limit

// Sixteen zero bytes: the source of every bf16 copy chunk that lies past the
// end of K (K a multiple of 8 but not of the 64-element step), so a ragged
// last step multiplies zeros and reads nothing beyond a row.
__device__ __align__(16) const uint8_t kZeroChunk[16] = {};

// 8 signed nibbles -> 8 bf16 values 136 + q, exact: the bits are 0x4300 | (q + 8)
// (128 + (q + 8), the nibble in the low mantissa bits of 128), and q + 8 = n ^ 8.
// Dword d takes nibbles d and d + 4, so slot s of the result holds element
// {0,4,1,5,2,6,3,7}[s] of the word and each dword is one v_bitop3 on the word
// shifted right by 4 d (truth table of (S0 & S1) ^ S2 over (0xF0, 0xCC, 0xAA):
// 0x6A): 7 operations per word, where the word's own order took 14.  The
// activations are stored in the same order (hidden by group_sum_kernel, the
// intermediate by GEMM1's epilogue).  `mask` is 0x000F000F, or 0 to turn every
// code into q = 0.
__device__ __forceinline__ bf16x8 int4x8_biased_bf16(uint32_t w, uint32_t mask) {
  auto dw = [&](uint32_t v) { return static_cast<uint32_t>(__builtin_amdgcn_bitop3_b32(v, mask, 0x43084308u, 0x6A)); };
  return as_bf16x8(u32x4{dw(w), dw(w >> 4), dw(w >> 8), dw(w >> 12)});
}

// One output of the int4 second product, sum over k of a[k] * (q[k] * s[k / 128])
// in fp32, for the values that the tile's biased form cannot hold (below): `a`
// an intermediate row in the codes' order, `w` and `s` a weight row's codes and
// group scales.
__device__ float int4_dot(const uint16_t* a, const uint32_t* w, const uint16_t* s, int K) {
  float sum = 0.f;
  for (int k8 = 0; k8 < K / 8 && sum == sum; ++k8) {
    const float sc = bf16_to_f32(s[k8 / 16]);
    const uint32_t word = w[k8];
    const u32x4 x = ld16(a + 8 * k8);
#pragma unroll
    for (int j = 0; j < 8; ++j) {  // element j: half j / 4 of dword j % 4
      const float q = static_cast<float>(static_cast<int>(word << (28 - 4 * j)) >> 28);
      sum = fmaf(__uint_as_float(j < 4 ? x[j % 4] << 16 : x[j % 4] & 0xFFFF0000u), q * sc, sum);
    }
  }
  return sum;
}

// XOR swizzle of the 16-byte chunks of a 128-byte LDS row: row r stores its
// chunk c in slot c ^ swz<KB>(r).  For the fragment reads (32 consecutive rows,
// lanes l and l+32 on neighbouring chunks of one row) (r >> 1) & 7 measured
// 1.6x the LDS read throughput of r & 7 on gfx950.
// With 64-byte rows (4 chunks) the analogous choice is (r >> 2) & 3; a
// 256-byte row spans all 64 banks, so there the slot alone must tell 16
// consecutive rows apart: r & 15.
template <int KB>
__device__ __forceinline__ int swz(int r) { return KB >= 256 ? r & 15 : KB == 128 ? (r >> 1) & 7 : (r >> 2) & 3; }
// int4 B rows (32 or 64 bytes: 2 or 4 chunks)
// (128-byte 4-bit rows, 256-element MXFP8 steps: as swz<128>)
template <int BB>
__device__ __forceinline__ int swz_b(int r) { return BB == 32 ? (r >> 2) & 1 : BB == 64 ? (r >> 2) & 3 : (r >> 1) & 7; }

// Four math waves, one per SIMD and side by side in the tile's columns, and four
// copy waves.  Only the copy waves issue the global->LDS copies and the math waves
// never touch global memory in the main loop, so a stalled load queue
// (L1 waiting on L2) cannot hold up the MFMA stream behind an in-order copy
// instruction.
// OPT, a sum of: kNoSums (int4: no group sums of the rows are there, the bias comes
// off by MFMAs), kOnce (experts with one row tile copy their weights with the
// non-temporal hint).
constexpr int kNoSums = 1, kOnce = 2;
constexpr int kMathWaves = 4, kCopyWaves = 4;
template <int FMT, bool GEMM1, int BM, int BNW, int GM, int KBT, int STAGES, int OPT = 0>
// The 128-element int4 steps are held to 128 registers, which keeps two workgroups per CU.
__global__ __launch_bounds__((kMathWaves + kCopyWaves) * 64) __attribute__((amdgpu_waves_per_eu(FMT == 2 && KBT < 512 ? 4 : 1)))
void moe_gemm_tiled(GroupedGemm g) {
  constexpr int NW = kMathWaves, WN = NW, NT = (NW + kCopyWaves) * 64;
  constexpr int LW = kCopyWaves;
  constexpr bool F4B = FMT == 2 || FMT == 4;  // 4-bit weights (int4, MXFP4), bf16 activations
  constexpr bool MX8 = FMT == 5;              // MXFP4 weights, MXFP8 activations
  constexpr bool SUMS = !(OPT & kNoSums), ONCE = OPT & kOnce;
  constexpr bool A8 = FMT == 1 || MX8;        // one-byte (e4m3) activations
  constexpr bool B4 = F4B || MX8;             // 4-bit weight rows
  static_assert(FMT == 2 ? KBT == 256 || KBT == 512 : FMT == 4 ? KBT == 256 : MX8 ? KBT == 128 || KBT == 256 : KBT == 128, "step");
  constexpr int KB = KBT;                                       // A bytes per row per step
  constexpr int KE = A8 ? KB : KB / 2;                                 // K elements per step
  constexpr int BB = B4 ? KE / 2 : KB;                                 // B bytes per row per step
  constexpr int LPB = BB / 16;                                         // lanes per 4-bit B row in a copy
  // bf16 and MXFP4 GEMM2 form their product transposed, as fp8 does (16-byte
  // y stores, one pad check per row; bf16 prefill 4 % faster, GEMM1 was not)
  constexpr bool TRB = !A8 && !GEMM1 && FMT != 2;
  constexpr int RPI = 1024 / KB, LPR = KB / 16;  // rows per DMA instruction, lanes per row
  constexpr int WTN = BNW / WN;
  constexpr int TM = BM / 32, TN = WTN / 32;
  constexpr int NC = GEMM1 ? BNW / 2 : BNW;  // output columns per tile
  // 16-byte DMA instructions per copy wave per stage (each moves 1 KB)
  constexpr int A_CH = BM * KB / 1024 / LW, B_CH = BNW * BB / 1024 / LW;
  static_assert(A_CH >= 1 && B_CH >= 1 && A_CH * LW * 1024 == BM * KB && B_CH * LW * 1024 == BNW * BB, "");
  static_assert(!GEMM1 || TN % 2 == 0, "gate/up pairs");
  static_assert(FMT != 1 || !GEMM1 || NC == 128, "fp8 requant needs one 128-column group per tile");
  // per-stage scale block: NW slots of 256 bytes, one 4-byte DMA instruction
  // each (64 floats); fp8: slots [0, BM/64) the row scales of A, slot BM/64
  // the block scales of B; int4: slots [0, BNW/64) the bf16 pair holding each
  // B row's group scale and slots [BNW/64, BNW/64 + BM/64) the
  // rows' biased group sums (GEMM1: x_gsum; GEMM2: in y).  Copy wave lw fills slots lw, lw + LW, ...
  // MXFP8: MXD E8M0 dwords per row per step (four 32-element blocks each);
  // slots [0, MXD BM/64) the A rows' dwords (slot d BM/64 + g: dword d of
  // row group g), then MXD BNW/64 slots of the B rows' likewise; slots past
  // those load a harmless dummy.
  constexpr bool GSUM = FMT == 2;
  static_assert(SUMS || (GSUM && KBT < 512), "group sums are int4's; the 256-element steps need them");
  constexpr int GD = GSUM ? KE / 128 : 1;  // int4: scale groups per step
  constexpr int MXD = MX8 ? KE / 128 : 1;
  constexpr int NSLOT = FMT == 0 ? 0 : (MX8 ? MXD * (BM + BNW) / 64 : (GSUM ? 2 : 1) * NW);
  constexpr int SC = (NSLOT + LW - 1) / LW;  // scale loads per copy wave per stage
  static_assert(FMT != 1 || BM / 64 < NW, "fp8 scale DMA layout");
  static_assert(!F4B || BNW / 64 <= NW, "4-bit scale DMA layout");
  static_assert(!GSUM || (BNW / 64 + GD * BM / 64 <= 2 * NW && STAGES == 2), "int4 group-sum DMA layout");
  static_assert(STAGES >= 2 && STAGES <= 4 && (STAGES - 2) * (A_CH + B_CH + SC) < 64, "vmcnt range");
  constexpr int A_BYTES = BM * KB, B_BYTES = BNW * BB, S_BYTES = SC * LW * 256;
  constexpr int STAGE = A_BYTES + B_BYTES + S_BYTES;
  constexpr int N_DMA = A_CH + B_CH + SC;  // loads per copy wave per stage

  __shared__ __attribute__((aligned(1024))) uint8_t smem[STAGES][STAGE];
  __shared__ float lds_amax[FMT == 1 && GEMM1 ? WN : 1][FMT == 1 && GEMM1 ? BM : 1];
  __shared__ int lds_off[MOE_MAX_EXPERTS_DEV + 1];  // expert_offsets, read once per workgroup
  // copy waves: the next tile's row ids, one slot per copy wave
  __shared__ int lds_sid[LW][BM];

  const int tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int wn = wave % WN;
  const bool is_math = wave < NW;             // uniform per wave
  const int lw = is_math ? 0 : wave - NW;     // copy-wave index
  const int l32 = lane & 31, kg = lane >> 5;
  const int K = GEMM1 ? g.H : g.I;
  const int N = GEMM1 ? g.I : g.H;       // output columns of the product
  // bf16 only: K and N multiples of 8 -- a ragged last K step (zero chunks)
  // and a ragged last column tile (weight rows clamped, stores masked); the
  // quantised formats have K and N multiples of 128
  const int nk = (K + KE - 1) / KE;
  const int n_tiles_n = (N + NC - 1) / NC;
  for (int i = tid; i <= g.E; i += NT) lds_off[i] = g.offsets[i];
  __syncthreads();
  const int n_tiles_m = lds_off[g.E] / BM;
  const int total = n_tiles_m * n_tiles_n;

  // this workgroup's share of the logical tiles: a contiguous range per XCD
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int per_xcd = gridDim.x / kXcds;
  const int chunk = (total + kXcds - 1) / kXcds;
  const int t_end = min(total, (xcd + 1) * chunk);
  const uint32_t smem0 = lds_addr(&smem[0][0]);

  // Logical tile order: expert by expert; inside expert e (row tiles
  // [base, base+cnt)) chunks of at most GM row tiles, each chunk swept
  // column tile by column tile with its row tiles adjacent.  Workgroups
  // running together then share one expert's weight slab and a few row tiles.
  auto coords = [&](int t, int& e, int& m0, int& n0) {
    e = find_segment(lds_off, g.E, (t / n_tiles_n) * BM);
    const int base = lds_off[e] / BM, cnt = (lds_off[e + 1] - lds_off[e]) / BM;
    const int local = t - base * n_tiles_n;
    const int c = local / (GM * n_tiles_n), within = local % (GM * n_tiles_n);
    const int sz = min(GM, cnt - c * GM);
    const int mt = base + c * GM + within % sz, nt = within / sz;
    m0 = mt * BM;
    n0 = nt * NC;
  };

  constexpr int NSL = SC > 0 ? SC : 1;
  struct Src {
    const uint8_t* a[A_CH];  // A rows
    int am[A_CH];            // A step-advance mask: -1, or 0 for a pad row (its source is the zero chunk)
    const uint8_t* b[B_CH];  // B rows
    const uint8_t* s[NSL];   // scale words
    int ss[NSL];             // scale advance per step
    bool once;               // the expert has one row tile: its weight rows are read once (uniform)
  };
  // staged: the tile's BM row ids are in this copy wave's lds_sid slot (else
  // they are read from sorted_ids)
  auto sources = [&](int e, int m0, int n0, Src& src, bool staged) {
    // per-lane DMA sources of the tile.  Instruction i of copy wave lw fills the 1 KB
    // block (i*LW + lw) of a stage: 1024/KB rows of A / of fp8-bf16 B (KB/16
    // lanes per row, one 16-byte slot each) or 64/LPB rows of int4 B (LPB
    // lanes per row).  Slot s of row r holds the row's chunk s ^ swz(r), the
    // XOR swizzle the fragment reads undo.
    // GEMM1 gathers its A rows by token: every row id this lane needs (A rows,
    // fp8 row scales) is requested before the first is used, so the tile
    // pays one memory round trip.  A pad row (id n_routed) of either product
    // copies the zero chunk at every step: one cache line per instruction
    // rather than a row's eight, and zeros in LDS; its products are never
    // read.  Scale sources of pad rows read the last token's.
    // Weights of an expert with one row tile are read once: the hint keeps
    // them from displacing what other tiles share.  With two or more row tiles
    // it costs the sharing (prefill GEMM1 675 -> 973 us with it everywhere).
    // Chosen once per step: a choice per copy cost the bf16 layer of 4096
    // tokens 7 %.
    src.once = ONCE && __builtin_amdgcn_readfirstlane(lds_off[e + 1] - lds_off[e]) == BM;
    int sid[A_CH + NSL];
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int r = (i * LW + lw) * RPI + lane / LPR;
      sid[i] = staged ? lds_sid[lw][r] : g.sorted_ids[m0 + r];
    }
    if constexpr (GEMM1) {
#pragma unroll
      for (int k = 0; k < NSL; ++k) {
        const int r = (lw + k * LW) * 64 + lane;
        int v = 0;
        if (A8 && lw + k * LW < MXD * (BM / 64)) {
          const int ra = ((lw + k * LW) % (BM / 64)) * 64 + lane;  // A row of the slot
          v = staged ? lds_sid[lw][ra] : g.sorted_ids[m0 + ra];
        }
        const int rg = (lw + k * LW - BNW / 64) % (BM / 64) * 64 + lane;  // group-sum slot row
        if (GSUM && lw + k * LW >= BNW / 64 && lw + k * LW < BNW / 64 + GD * BM / 64) {
          v = staged ? lds_sid[lw][rg] : g.sorted_ids[m0 + rg];
        }
        sid[A_CH + k] = v;
      }
    }
    auto token = [&](int v) {
      return static_cast<size_t>(static_cast<unsigned>(min(v, g.n_routed - 1)) / static_cast<unsigned>(g.top_k));
    };
#pragma unroll
    for (int i = 0; i < A_CH; ++i) {
      const int r = (i * LW + lw) * RPI + lane / LPR;
      const uint8_t* row;
      if (GEMM1) {
        row = static_cast<const uint8_t*>(g.x) + token(sid[i]) * g.H * (A8 ? 1 : 2);
      } else {
        row = static_cast<const uint8_t*>(g.inter) + static_cast<size_t>(m0 + r) * g.I * (A8 ? 1 : 2);
      }
      const bool pad = sid[i] >= g.n_routed;
      src.a[i] = pad ? static_cast<const uint8_t*>(kZeroChunk) : row + (((lane % LPR) ^ swz<KB>(r)) << 4);
      src.am[i] = pad ? 0 : -1;
    }
    const size_t w_row_bytes = FMT == 0 ? K * 2 : (FMT == 1 ? K : K / 2);
    const uint8_t* wbase = static_cast<const uint8_t*>(GEMM1 ? g.w1 : g.w2) +
                           static_cast<size_t>(e) * (GEMM1 ? 2 * g.I : g.H) * w_row_bytes;
#pragma unroll
    for (int i = 0; i < B_CH; ++i) {
      const int blk = i * LW + lw;
      const int r = B4 ? blk * (64 / LPB) + lane / LPB : blk * RPI + lane / LPR;
      const int sl = B4 ? (lane % LPB) ^ swz_b<BB>(r) : (lane % LPR) ^ swz<KB>(r);
      // weight rows past N (a ragged last column tile) read the last row:
      // their columns are never stored
      int n;
      if (GEMM1) n = r < NC ? min(n0 + r, g.I - 1) : g.I + min(n0 + (r - NC), g.I - 1);
      else n = min(n0 + r, g.H - 1);
      src.b[i] = wbase + static_cast<size_t>(n) * w_row_bytes + (sl << 4);
    }
    // scale DMA sources of this lane, one per slot lw + k*LW (advanced by one
    // K block / half group per step); slots without a scale role load a
    // harmless dummy
#pragma unroll
    for (int k = 0; k < NSL; ++k) {
      const int sl = lw + k * LW;
      src.s[k] = src.a[0];
      src.ss[k] = 0;
      if constexpr (FMT == 1) {
        if (sl < BM / 64) {
          const int r = sl * 64 + lane;
          if (GEMM1) {
            src.s[k] = reinterpret_cast<const uint8_t*>(g.x_scale + token(sid[A_CH + k]) * (g.H / 128));
          } else {
            src.s[k] = reinterpret_cast<const uint8_t*>(g.inter_scale + static_cast<size_t>(m0 + r) * (g.I / 128));
          }
          src.ss[k] = 4;
        } else if (sl == BM / 64) {
          // lane l: block row of W (GEMM1: l odd -> up half, even -> gate half;
          // GEMM2: block row n0/128 + l % (BNW/128))
          const float* wsc = static_cast<const float*>(GEMM1 ? g.w1_scale : g.w2_scale) +
                             static_cast<size_t>(e) * ((GEMM1 ? 2 * g.I : g.H) / 128) * (K / 128);
          const int br = GEMM1 ? ((lane & 1) ? (g.I + n0) / 128 : n0 / 128) : n0 / 128 + lane % (BNW / 128);
          src.s[k] = reinterpret_cast<const uint8_t*>(wsc + static_cast<size_t>(br) * (K / 128));
          src.ss[k] = 4;
        }
      } else if constexpr (FMT == 2) {
        if (sl < BNW / 64) {
          const int r = sl * 64 + lane;
          const int n = GEMM1 ? (r < NC ? n0 + r : g.I + n0 + (r - NC)) : n0 + r;
          // bf16 scale [n][group] of K step kt sits at element n*(K/128) + kt/2;
          // the dword holding it starts at the even element below
          src.s[k] = reinterpret_cast<const uint8_t*>(static_cast<const uint16_t*>(GEMM1 ? g.w1_scale : g.w2_scale) +
                                                      (static_cast<size_t>(e) * (GEMM1 ? 2 * g.I : g.H) + n) * (K / 128));
          src.ss[k] = 1;  // advanced per step in elements below
        } else if (SUMS && sl < BNW / 64 + GD * BM / 64) {
          // tile row (sl - BNW/64) % (BM/64) * 64 + lane: its sum over the
          // step's group (sl - BNW/64) / (BM/64); GEMM1 GD floats per step,
          // GEMM2 (64 rows, one slot per group) as launch_tile_sums lays them out
          static_assert(!SUMS || BM == 64, "one slot per group");
          const int d = (sl - BNW / 64) / (BM / 64), r = (sl - BNW / 64) % (BM / 64) * 64 + lane;
          if (GEMM1) src.s[k] = reinterpret_cast<const uint8_t*>(g.x_gsum + token(sid[A_CH + k]) * (g.H / 128) + d);
          else src.s[k] = reinterpret_cast<const uint8_t*>(static_cast<const float*>(g.y) + static_cast<size_t>(m0) * g.H + n0 + 64 * d + lane);
          src.ss[k] = 4 * GD;
        }
      } else if constexpr (MX8) {
        if (sl < MXD * (BM / 64)) {
          // A row (sl % (BM/64))*64 + lane: its E8M0 bytes [K/32]; dword sl / (BM/64) of step kt
          const int r = (sl % (BM / 64)) * 64 + lane, d = sl / (BM / 64);
          if (GEMM1) src.s[k] = g.x_mx + token(sid[A_CH + k]) * (g.H / 32) + 4 * d;
          else src.s[k] = g.inter_mx + static_cast<size_t>(m0 + r) * (g.I / 32) + 4 * d;
          src.ss[k] = 4 * MXD;
        } else if (sl < MXD * (BM / 64 + BNW / 64)) {
          const int sb2 = sl - MXD * (BM / 64);
          const int r = (sb2 % (BNW / 64)) * 64 + lane, d = sb2 / (BNW / 64);
          const int n = GEMM1 ? (r < NC ? n0 + r : g.I + n0 + (r - NC)) : n0 + r;
          src.s[k] = static_cast<const uint8_t*>(GEMM1 ? g.w1_scale : g.w2_scale) +
                     (static_cast<size_t>(e) * (GEMM1 ? 2 * g.I : g.H) + n) * (K / 32) + 4 * d;
          src.ss[k] = 4 * MXD;
        }
      } else if constexpr (FMT == 4) {
        if (sl < BNW / 64) {
          // E8M0 bytes [n][K/32]: the four of K step kt are one dword at byte 4 kt
          const int r = sl * 64 + lane;
          const int n = GEMM1 ? (r < NC ? n0 + r : g.I + n0 + (r - NC)) : n0 + r;
          src.s[k] = static_cast<const uint8_t*>(GEMM1 ? g.w1_scale : g.w2_scale) +
                     (static_cast<size_t>(e) * (GEMM1 ? 2 * g.I : g.H) + n) * (K / 32);
          src.ss[k] = 4;
        }
      }
    }
  };

  // issue this copy wave's N_DMA loads of step kt of the tile `src` describes
  // into LDS buffer `buf`
  // bf16 ragged K: in the last step a lane whose 8-element chunk starts at
  // or past K copies the zero chunk instead (A row chunk (lane % LPR) ^ swz(r),
  // r the row the instruction's lane covers; the bf16 B rows likewise)
  const bool k_ragged = FMT == 0 && K % KE != 0;
  auto tail_src = [&](const uint8_t* p, int blk, int kt) {
    const int r = blk * RPI + lane / LPR;
    const int c = (lane % LPR) ^ swz<KB>(r);
    return kt * KE + 8 * c >= K ? static_cast<const uint8_t*>(kZeroChunk) : p;
  };
  auto issue = [&](const Src& src, int kt, int buf) {
    const uint32_t base = smem0 + buf * STAGE;
    if (FMT == 0 && k_ragged && kt == nk - 1) {  // uniform: only the last step of a ragged K
#pragma unroll
      for (int i = 0; i < A_CH; ++i)
        dma16(tail_src(src.a[i] + (kt * KB & src.am[i]), i * LW + lw, kt), base + (i * LW + lw) * 1024);
#pragma unroll
      for (int i = 0; i < B_CH; ++i)
        dma16(tail_src(src.b[i] + kt * BB, i * LW + lw, kt), base + A_BYTES + (i * LW + lw) * 1024);
    } else {
#pragma unroll
      for (int i = 0; i < A_CH; ++i)
        dma16(src.a[i] + (kt * KB & src.am[i]), base + (i * LW + lw) * 1024);
      if (ONCE && src.once) {
#pragma unroll
        for (int i = 0; i < B_CH; ++i)
          dma16_nt(src.b[i] + kt * BB, base + A_BYTES + (i * LW + lw) * 1024);
      } else {
#pragma unroll
        for (int i = 0; i < B_CH; ++i)
          dma16(src.b[i] + kt * BB, base + A_BYTES + (i * LW + lw) * 1024);
      }
    }
#pragma unroll
    for (int k = 0; k < SC; ++k) {
      // int4 (two stages, so every wait drains all loads and the
      // per-wave load counts need not match) skips its empty slots
      if (GSUM && src.ss[k] == 0) continue;
      const uint32_t dst = base + A_BYTES + B_BYTES + (lw + k * LW) * 256;
      if constexpr (FMT == 1 || FMT == 4 || MX8) {
        dma4(src.s[k] + kt * src.ss[k], dst);
      } else if constexpr (FMT == 2) {
        // B scale words (ss 1): element kt*KE/128 of the row, rounded down to
        // an even element (4-byte aligned); group sums advance one float per
        // group (ss 4 GD) or as they lie in y; dummies stay put (ss 0)
        const uint8_t* p = src.s[k] + kt * src.ss[k];
        if (src.ss[k] == 1) {
          const uintptr_t a = reinterpret_cast<uintptr_t>(src.s[k]) + ((kt * KE) / 128) * 2;
          p = reinterpret_cast<const uint8_t*>(a & ~static_cast<uintptr_t>(3));
        } else if (SUMS && !GEMM1) {
          const int at = 64 * GD * kt;
          p = src.s[k] + (static_cast<size_t>(at / BNW) * g.H + at % BNW) * 4;
        }
        dma4(p, dst);
      }
    }
  };
  // this copy wave's loads for a step have landed once at most `ahead`
  // later steps (N_DMA loads each) are still in flight
  auto wait_ahead = [&](int ahead) {
    if constexpr (STAGES >= 4) { if (ahead == 2) { vm_wait<2 * N_DMA>(); return; } }
    if constexpr (STAGES >= 3) { if (ahead == 1) { vm_wait<N_DMA>(); return; } }
    vm_wait<0>();
  };

  // K steps are numbered across this workgroup's tiles, and step s of the
  // sequence lives in LDS buffer s % STAGES; `sb` is the buffer of a tile's
  // step 0.  STAGES-1 steps are loaded ahead: step s+STAGES-1 goes into the
  // buffer read in step s-1, issued once the barrier of step s shows every
  // wave is past it.  The next tile's first STAGES-1 steps
  // are issued right after the barrier of the current tile's last step (their
  // buffers were read in earlier steps), so they load during that step and
  // the epilogue.
  const int t0 = xcd * chunk + slot;
  Src cur;
  if (!is_math) {
    // copy waves: one barrier per step, the same sequence as the math waves
    if (t0 < t_end) {
      int e, m0, n0;
      coords(t0, e, m0, n0);
      sources(e, m0, n0, cur, false);
#pragma unroll
      for (int q = 0; q < STAGES - 1; ++q)
        if (q < nk) issue(cur, q, q);
    }
    // the next tile's sources are computed in step kc; its row ids,
    // copied to this wave's LDS slot ahead of step STAGES-1's loads, have
    // landed by then: in-order completion, and the wait of step kt covers
    // every load issued before step kt+1 (all of them in the last step)
    const int kc = min(STAGES - 2, nk - 1);
    for (int t = t0, sb = 0; t < t_end; t += per_xcd, sb = (sb + nk) % STAGES) {
      const int tn = t + per_xcd;
      const bool next = tn < t_end;
      Src nxt;
      int en = 0, m0n = 0, n0n = 0;
      if (next) {
        coords(tn, en, m0n, n0n);
#pragma unroll
        for (int q = 0; q < BM / 64; ++q) dma4(g.sorted_ids + m0n + q * 64 + lane, lds_addr(&lds_sid[lw][q * 64]));
      }
      // Tiles of at most 32 steps (the second products here) run with
      // the next tile as one sequence of steps: step j of it is issued in
      // step j - (STAGES - 1), so the next tile's first steps load STAGES - 1
      // steps ahead like every other step, and the wait keeps them in
      // flight across the boundary (fp8 GEMM2 -2.4 %, prefill GEMM2 -2 %).
      // Longer tiles measured no gain, and tiles of fewer than 2 STAGES
      // steps may not have the next tile's sources ready in time: both
      // issue the next tile's first steps together in their last step.
      const bool flow = next && nk >= 2 * STAGES && nk <= 32;  // uniform
      for (int kt = 0; kt < nk; ++kt) {
        wait_ahead(flow ? STAGES - 2 : min(STAGES - 2, nk - 1 - kt));
        bar();
        if (next && kt == kc) sources(en, m0n, n0n, nxt, true);
        const int j = kt + STAGES - 1;
        if (j < nk) issue(cur, j, (sb + j) % STAGES);
        else if (flow) issue(nxt, j - nk, (sb + j) % STAGES);
        if (next && !flow && kt == nk - 1) {
#pragma unroll
          for (int q = 0; q < STAGES - 1; ++q)
            if (q < nk) issue(nxt, q, (sb + nk + q) % STAGES);
        }
      }
      if constexpr (FMT == 1 && GEMM1) {  // the two barriers of the requant epilogue
        bar();
        bar();
      }
      if (next) cur = nxt;
    }
    return;
  }

  for (int t = t0, sb = 0; t < t_end; t += per_xcd, sb = (sb + nk) % STAGES) {
    int e, m0, n0;
    coords(t, e, m0, n0);
    // GEMM2: the ids of this lane's output rows, for the epilogue's pad-row
    // check, requested before the K loop (landed long before it is used)
    int sid_ep[GEMM1 ? 1 : TM];
    bool live_row = false;  // int4: row m0 + lane of the tile
    if constexpr (!GEMM1 && FMT == 2) {
      live_row = g.sorted_ids[m0 + lane] < g.n_routed;
    } else if constexpr (!GEMM1) {
#pragma unroll
      for (int i = 0; i < TM; ++i) sid_ep[i] = g.sorted_ids[m0 + i * 32 + l32];
    }
    f32x16 acc[TM][TN];
#pragma unroll
    for (int i = 0; i < TM; ++i)
#pragma unroll
      for (int j = 0; j < TN; ++j) acc[i][j] = f32x16{};
    float seff[TN];  // int4: the scale each column's accumulators are divided by (0: none yet)
#pragma unroll
    for (int j = 0; j < TN; ++j) seff[j] = 0.f;
    float least = 1.f;  // int4 GEMM2: the smallest ratio of this lane's columns' scales, group to group

    // B row (within the tile) of wave tile j
#define brow(j) (GEMM1 ? ((j) < TN / 2 ? wn * (WTN / 2) + (j) * 32 : NC + wn * (WTN / 2) + ((j) - TN / 2) * 32) \
                       : wn * WTN + (j) * 32)

    // Row blocks (of 32) of the tile that hold routed rows: the last tile of an
    // expert is padded, on average by half a tile, and the loops below
    // leave the blocks of pads out (every wave holds all BM rows, so all gain alike).
    // Layer with all blocks and without those of pads: bf16, 4096 x 1408 x 64
    // experts, top 6, 777 tokens 490 and 479 us, 2500 tokens 861 and 847, 4096 tokens (384
    // rows per expert) 1223 and 1233; MXFP4, 7168 x 2048 x 256 experts, top 8, 2000 tokens
    // 2345 and 2098, 8192 tokens 6377 and 6288; MXFP4 x MXFP8 3634 and 3594; fp8, the
    // same layer, 300 tokens 1241 and 1159, 8192 tokens 4266 and 4172; int4, 4096 x
    // 1536 x 128 experts, top 8, 512 tokens 394 and 371.  The ids are
    // waited for at the start of each tile.  Tiles that take unequal time let the
    // workgroups that share operands drift apart: GEMM1 reads 2.26 GB from HBM with all
    // blocks and 3.93 without for bf16 at 4096 tokens, 6.91 and 16.8 for MXFP4 at 8192,
    // 9.54 and 10.6 for fp8, which takes back what the MFMAs save in large bf16 batches.
    constexpr bool I4P = FMT == 2 && KB == 512;  // int4 on the software-pipelined loop
    constexpr bool SKIP = FMT != 2 || I4P;
    static_assert(TM == 4 || TM == 2, "every wave holds all row blocks");
    int nb = TM;
    if constexpr (SKIP) nb = __popcll(__ballot(lane < TM && g.sorted_ids[m0 + 32 * (lane % TM)] < g.n_routed));
    auto for_blocks = [&](auto loop) {
      if (TM >= 4 && nb >= 4) loop(std::integral_constant<int, TM >= 4 ? 4 : 1>{});
      else if (TM >= 4 && nb == 3) loop(std::integral_constant<int, TM >= 4 ? 3 : 1>{});
      else if (nb == 2) loop(std::integral_constant<int, 2>{});
      else loop(std::integral_constant<int, 1>{});
    };
    if constexpr (FMT == 0) {
      // Math waves of a split bf16 launch: fragments are read one MFMA K
      // substep ahead into a double buffer.  The barrier for stage kt+1 sits
      // before the last substep's MFMAs of step kt (once this wave's reads of
      // stage kt are complete), so the next stage's first fragments load
      // while those MFMAs run; the barrier count is still one per step.
      constexpr int NKK = KE / 16;
      static_assert(NKK % 2 == 0, "substep parity");
      for_blocks([&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        bf16x8 fa[2][NB], fb[2][TN];
        auto read_frags = [&](int kt, int kk, int buf) {
          const uint8_t* As = &smem[(sb + kt) % STAGES][0];
          const uint8_t* Bs = As + A_BYTES;
          const int ch = 2 * kk + kg;
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int r = i * 32 + l32;
            fa[buf][i] = as_bf16x8(ld16(As + r * KB + ((ch ^ swz<KB>(r)) << 4)));
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int r = brow(j) + l32;
            fb[buf][j] = as_bf16x8(ld16(Bs + r * BB + ((ch ^ swz<KB>(r)) << 4)));
          }
        };
        bar();  // stage 0 has landed
        read_frags(0, 0, 0);
        for (int kt = 0; kt < nk; ++kt) {
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            if (kk + 1 < NKK) {
              read_frags(kt, kk + 1, (kk + 1) & 1);
            } else if (kt + 1 < nk) {
              __atomic_signal_fence(__ATOMIC_SEQ_CST);
              lds_wait();  // stage kt is in registers
              bar();                               // stage kt+1 has landed; buffer kt is free
              read_frags(kt + 1, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = TRB ? mfma32x32x16(fb[kk & 1][j], fa[kk & 1][i], acc[i][j])
                                : mfma32x32x16(fa[kk & 1][i], fb[kk & 1][j], acc[i][j]);
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      });
    }
    if constexpr (FMT == 1) {
      // fp8 math waves of a split launch (two waves per SIMD, so at most 256
      // registers each): transposed product as below, but one 32x32 block
      // at a time -- its two K halves are MFMAs on one partial, and the
      // VALU folds the previous block's partial in between them -- with
      // the A fragments read per row block, one block ahead.
      for_blocks([&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        for (int kt = 0; kt < nk; ++kt) {
          bar();  // every stage-kt copy of every copy wave has landed
          const uint8_t* As = &smem[(sb + kt) % STAGES][0];
          const uint8_t* Bs = As + A_BYTES;
          const uint8_t* Ss = Bs + B_BYTES;
          auto read8 = [&](const uint8_t* row, int r, int kk) {  // K half kk of a row: this lane's 32 bytes
            const int c0 = 4 * kk + 2 * kg;
            const i32x4 lo = __builtin_bit_cast(i32x4, ld16(row + ((c0 ^ swz<KB>(r)) << 4)));
            const i32x4 hi = __builtin_bit_cast(i32x4, ld16(row + (((c0 + 1) ^ swz<KB>(r)) << 4)));
            return i32x8(__builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
          };
          i32x8 bq[TN][2];
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int r = brow(j) + l32;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) bq[j][kk] = read8(Bs + r * BB, r, kk);
          }
          i32x8 af[2][2];  // [buffer][K half] of one row block
          auto read_a = [&](int i, int buf) {
            const int r = i * 32 + l32;
#pragma unroll
            for (int kk = 0; kk < 2; ++kk) af[buf][kk] = read8(As + r * KB, r, kk);
          };
          read_a(0, 0);
          const float* sA = reinterpret_cast<const float*>(Ss);                    // [BM]
          const float* sB = reinterpret_cast<const float*>(Ss + (BM / 64) * 256);  // [64]
          float fa[NB], sw[TN];
#pragma unroll
          for (int i = 0; i < NB; ++i) fa[i] = sA[i * 32 + l32];
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int r = brow(j);
            sw[j] = GEMM1 ? sB[r < NC ? 0 : 1] : sB[(r / 128) % (BNW / 128)];
          }
          f32x16 part[2];
          // blocks row-major: b = i*TN + j
#pragma unroll
          for (int b = 0; b <= NB * TN; ++b) {
            const int i = b / TN, j = b % TN;
            const int ip = (b - 1) / TN, jp = (b - 1) % TN;  // the block folded in this iteration
            if (b < NB * TN && j == 0 && i + 1 < NB) read_a(i + 1, (i + 1) & 1);
            __builtin_amdgcn_sched_barrier(0);
            const float f = b > 0 ? fa[ip] * sw[jp] : 0.f;
            if (b < NB * TN) part[b & 1] = mfma32x32x64_fp8(bq[j][0], af[i & 1][0], f32x16{});
            if (b > 0) {
#pragma unroll
              for (int v = 0; v < 8; ++v) acc[ip][jp][v] = fmaf(part[(b - 1) & 1][v], f, acc[ip][jp][v]);
            }
            if (b < NB * TN) part[b & 1] = mfma32x32x64_fp8(bq[j][1], af[i & 1][1], part[b & 1]);
            if (b > 0) {
#pragma unroll
              for (int v = 8; v < 16; ++v) acc[ip][jp][v] = fmaf(part[(b - 1) & 1][v], f, acc[ip][jp][v]);
            }
            // keep the order written: each MFMA, then eight fmas that run on the
            // VALU while it executes (the compiler otherwise pairs the MFMAs and
            // stalls the fmas behind the second one)
            if (b > 0 && b < NB * TN) {
              __builtin_amdgcn_sched_group_barrier(0x002, 1, 0);  // the scale product
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
              __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        }
      });
    }
    if constexpr (FMT == 4) {
      // Math waves of a split MXFP4 launch.  One math wave per SIMD issues in
      // order, so decoding a substep's weights and then multiplying them ran
      // the VALU (its conversions) and the matrix pipe one after the
      // other.  Here the next substep's conversions are interleaved with this
      // substep's MFMAs; fragments are read one substep
      // ahead, and the barrier for stage kt+1 sits before the last substep's
      // MFMAs as in the bf16 loop above.
      // Lane group kg covers elements [64 kg, 64 kg + 64) of the step, the
      // 32-element blocks 2 kg and 2 kg + 1: their E8M0 bytes are bytes
      // 2 kg and 2 kg + 1 of the row's scale dword, passed as float(s << 23).
      constexpr int NKK = KE / 16;
      static_assert(NKK == 8, "two 32-element blocks per lane group, four substeps each");
      for_blocks([&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        bf16x8 fa[2][NB], fb[2][TN];
        u32x4 bw[2][TN];  // [block][column tile]
        uint32_t sd[TN];  // this lane group's two scale bytes
        float sc[2][TN];
        auto stage = [&](int kt) { return &smem[(sb + kt) % STAGES][0]; };
        auto read_a = [&](int kt, int kk, int buf) {
          const uint8_t* As = stage(kt);
          const int ch = NKK * kg + kk;
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const int r = i * 32 + l32;
            fa[buf][i] = as_bf16x8(ld16(As + r * KB + ((ch ^ swz<KB>(r)) << 4)));
          }
        };
        auto read_w = [&](int kt, int h) {
          const uint8_t* Bs = stage(kt) + A_BYTES;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const int r = brow(j) + l32;
            bw[h][j] = ld16(Bs + r * BB + (((2 * kg + h) ^ swz_b<BB>(r)) << 4));
          }
        };
        auto read_s = [&](int kt) {
          const uint32_t* sW = reinterpret_cast<const uint32_t*>(stage(kt) + A_BYTES + B_BYTES);
#pragma unroll
          for (int j = 0; j < TN; ++j) sd[j] = sW[brow(j) + l32];
        };
        auto scales = [&]() {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            sc[0][j] = __uint_as_float((sd[j] >> (16 * kg) & 0xFFu) << 23);
            sc[1][j] = __uint_as_float((sd[j] >> (16 * kg + 8) & 0xFFu) << 23);
          }
        };
        auto decode = [&](int kk, int j, int buf) {
          fb[buf][j] = as_bf16x8(mxfp4x8_to_bf16(bw[kk / 4][j][kk % 4], sc[kk / 4][j]));
        };
        bar();  // stage 0 has landed
        read_s(0);
        read_w(0, 0);
        read_a(0, 0, 0);
        scales();
#pragma unroll
        for (int j = 0; j < TN; ++j) decode(0, j, 0);
        // the last step stands apart: a branch around its missing barrier would
        // let the compiler sink the earlier substeps' MFMAs past it
        auto step = [&](int kt, auto last) {
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            const bool more = kk + 1 < NKK || !decltype(last)::value;  // a later substep follows
            if (kk + 1 < NKK) {
              if (kk == 0) read_w(kt, 1);
              read_a(kt, kk + 1, (kk + 1) & 1);
            } else if (more) {
              __atomic_signal_fence(__ATOMIC_SEQ_CST);
              lds_wait();  // stage kt is in registers
              bar();       // stage kt+1 has landed; buffer kt is free
              read_s(kt + 1);
              read_w(kt + 1, 0);
              read_a(kt + 1, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) {
              if (kk + 1 == NKK) scales();
#pragma unroll
              for (int j = 0; j < TN; ++j) decode((kk + 1) % NKK, j, (kk + 1) & 1);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j)
                acc[i][j] = TRB ? mfma32x32x16(fb[kk & 1][j], fa[kk & 1][i], acc[i][j])
                                : mfma32x32x16(fa[kk & 1][i], fb[kk & 1][j], acc[i][j]);
            if (kk + 1 < NKK) {
#pragma unroll
              for (int q = 0; q < NB * TN; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x002, (4 + NB - 1) / NB, 0);
              }
            } else if (more) {
              // the next stage's words arrive under the first half of the MFMAs
              __builtin_amdgcn_sched_group_barrier(0x008, NB * TN / 2, 0);
#pragma unroll
              for (int q = 0; q < NB * TN / 2; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x002, (8 + NB - 1) / NB + 4, 0);
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        for (int kt = 0; kt + 1 < nk; ++kt) step(kt, std::false_type{});
        step(nk - 1, std::true_type{});
      });
    }
    if constexpr (MX8) {
      // Math waves of an MXFP4 x MXFP8 launch, formed transposed like fp8
      // (the weight fragment is the first operand).  MFMA kk of the step
      // covers K [64 kk, 64 kk + 64) in two 32-element scale blocks, and lane
      // group kg supplies block kg's E8M0 byte for both operands (byte
      // 2 (kk % 2) + kg of the row's dword kk / 2 for the step; the
      // instruction applies the scales itself, so the products accumulate
      // in place: no rescale on the VALU).  Weights: lane group kg holds
      // block kg, 16 bytes (chunk 2 kk + kg of the row's KE/2 bytes).
      // Activations: the e4m3 operand interleaves the blocks in 16-element
      // halves -- lane group kg holds elements [16 kg, +16) of block 0,
      // then of block 1, i.e. chunks 4 kk + kg and 4 kk + 2 + kg of the
      // row's KE bytes.  Fragments are read one substep ahead; chunk addresses
      // are one XOR on the stage's (rows aligned to their bytes).  With the row
      // blocks of pads left out, 7168 x 2048 x 256 experts, top 8: 8192 tokens
      // 3693 and 3664 us, 2000 tokens 1453 and 1411, 64 tokens 675 and 653.
      for_blocks([&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        constexpr int NKK = 2 * MXD;
        static_assert(STAGE % 256 == 0 && A_BYTES % 256 == 0, "rows aligned to their bytes");
        i32x8 fa[2][NB];
        i32x4 fb[2][TN];
        int da[2][NB], db[2][TN];  // the rows' scale dwords
        const int ra = l32, rb = brow(0) + l32;
        const uint32_t oa = ra * KB + ((kg ^ swz<KB>(ra)) << 4);
        const uint32_t ob = A_BYTES + rb * BB + ((kg ^ swz_b<BB>(rb)) << 4);
        typedef const __attribute__((address_space(3))) int* lds_i32;
        auto read_frags = [&](int kt, int kk, int buf) {
          const uint32_t st = smem0 + ((sb + kt) % STAGES) * STAGE;
          const uint32_t pa = st + oa, pb = st + ob;
          const uint32_t sa = st + A_BYTES + B_BYTES + (kk / 2) * BM * 4 + ra * 4;                  // [MXD][BM]
          const uint32_t sw = st + A_BYTES + B_BYTES + MXD * BM * 4 + (kk / 2) * BNW * 4 + rb * 4;  // [MXD][BNW]
#pragma unroll
          for (int i = 0; i < NB; ++i) {
            const i32x4 lo = __builtin_bit_cast(i32x4, lds16((pa ^ (4 * kk) << 4) + i * 32 * KB));
            const i32x4 hi = __builtin_bit_cast(i32x4, lds16((pa ^ (4 * kk + 2) << 4) + i * 32 * KB));
            fa[buf][i] = __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7);
            da[buf][i] = *(lds_i32)(sa + i * 32 * 4);
          }
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            fb[buf][j] = __builtin_bit_cast(i32x4, lds16((pb ^ (2 * kk) << 4) + (brow(j) - brow(0)) * BB));
            db[buf][j] = *(lds_i32)(sw + (brow(j) - brow(0)) * 4);
          }
        };
        bar();  // stage 0 has landed
        read_frags(0, 0, 0);
        auto step = [&](int kt, auto last) {  // the last step apart, as above
#pragma unroll
          for (int kk = 0; kk < NKK; ++kk) {
            if (kk + 1 < NKK) {
              read_frags(kt, kk + 1, (kk + 1) & 1);
            } else if (!decltype(last)::value) {
              __atomic_signal_fence(__ATOMIC_SEQ_CST);
              lds_wait();  // stage kt is in registers
              bar();       // stage kt+1 has landed; buffer kt is free
              read_frags(kt + 1, 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            int sw[TN];
#pragma unroll
            for (int j = 0; j < TN; ++j) sw[j] = static_cast<int>(static_cast<uint32_t>(db[kk & 1][j]) >> (8 * kg));
#pragma unroll
            for (int i = 0; i < NB; ++i) {
              const int sa = static_cast<int>(static_cast<uint32_t>(da[kk & 1][i]) >> (8 * kg));
#pragma unroll
              for (int j = 0; j < TN; ++j) {
                const i32x4 q = fb[kk & 1][j];
                const i32x8 w = __builtin_shufflevector(q, q, 0, 1, 2, 3, 0, 1, 2, 3);  // upper half unused
                acc[i][j] = (kk & 1) ? mfma32x32x64_f4f8<2>(w, fa[kk & 1][i], sw[j], sa, acc[i][j])
                                     : mfma32x32x64_f4f8<0>(w, fa[kk & 1][i], sw[j], sa, acc[i][j]);
              }
            }
            // the products stay in their substep: without a use here they were
            // moved past the later substeps' reads, whose fragments then spilled
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));
            __builtin_amdgcn_sched_barrier(0);
          }
        };
        for (int kt = 0; kt + 1 < nk; ++kt) step(kt, std::false_type{});
        step(nk - 1, std::true_type{});
      });
    }
    if constexpr (I4P) {
      // int4, 256 K elements (two scale groups) per step, so every weight row
      // gives a whole 128-byte line: the number of lines through the vector
      // L1 set the time of the 128-element steps below, which ask for half
      // lines.  The stages leave room for one workgroup per CU, one math wave
      // per SIMD, so the next substep's decode and the group's rescale are
      // interleaved with the MFMAs.  The arithmetic is that of the
      // 128-element loop below.  512 tokens, 4096 x 1536 x 128 experts, top 8:
      // the layer 388 us with the 128-element steps, 365 with these.
      // Substep t: K elements [128 (t/8) + 64 kg + 8 (t%8), +8) of the step,
      // chunk 16 (t/8) + 8 kg + t%8 of an activation row, word t%4 of chunk
      // t/4 + 2 kg + 2 (t/8) of a weight row.
      for_blocks([&](auto nbc) {
        constexpr int NB = decltype(nbc)::value;
        static_assert(STAGE % 512 == 0 && A_BYTES % 512 == 0, "rows aligned to their bytes");
        bf16x8 fa[2][NB], fb[2][TN];
        u32x4 bw[2][TN];
        uint32_t sd[TN], keep[TN];
        float ratio[TN];
        f32x16 rs[NB];
        const int ra = l32, rb = brow(0) + l32;
        const uint32_t oa = ra * KB + (((8 * kg) ^ swz<KB>(ra)) << 4);
        const uint32_t ob = A_BYTES + rb * BB + (((2 * kg) ^ swz_b<BB>(rb)) << 4);
        auto stage = [&](int kt) { return smem0 + ((sb + kt) % STAGES) * STAGE; };
        auto read_a = [&](int kt, int t, int buf) {
          const uint32_t pa = stage(kt) + oa;
#pragma unroll
          for (int i = 0; i < NB; ++i)
            fa[buf][i] = as_bf16x8(lds16((pa ^ (16 * (t / 8) + t % 8) << 4) + i * 32 * KB));
        };
        auto read_w = [&](int kt, int h) {  // words of substeps [4 h, 4 h + 4)
          const uint32_t pb = stage(kt) + ob;
#pragma unroll
          for (int j = 0; j < TN; ++j)
            bw[h & 1][j] = lds16((pb ^ (4 * (h / 2) + h % 2) << 4) + (brow(j) - brow(0)) * BB);
        };
        auto read_s = [&](int kt) {
          const uint8_t* Ss = &smem[(sb + kt) % STAGES][A_BYTES + B_BYTES];
#pragma unroll
          for (int j = 0; j < TN; ++j) sd[j] = reinterpret_cast<const uint32_t*>(Ss)[brow(j) + l32];
        };
        auto read_r = [&](int kt, int q) {  // the rows' biased sums over group q
          const uint32_t sr = stage(kt) + A_BYTES + B_BYTES + (BNW / 64 + q * (BM / 64)) * 256 + 16 * kg;
#pragma unroll
          for (int i = 0; i < NB; ++i)
#pragma unroll
            for (int b4 = 0; b4 < 4; ++b4) {
              const u32x4 v = lds16(sr + i * 128 + b4 * 32);  // rows 32 i + 8 b4 + 4 kg + [0, 4)
#pragma unroll
              for (int c = 0; c < 4; ++c) rs[i][4 * b4 + c] = __uint_as_float(v[c]);
            }
        };
        auto scales = [&](int q) {
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            const float sc = __uint_as_float(q ? sd[j] & 0xFFFF0000u : sd[j] << 16);
            const bool z = sc == 0.f;
            const float se = z ? seff[j] : sc;
            ratio[j] = seff[j] == 0.f ? 0.f : seff[j] * __builtin_amdgcn_rcpf(se);
            if (!GEMM1) least = fminf(least, seff[j] == 0.f ? 1.f : fabsf(ratio[j]));
            seff[j] = se;
            keep[j] = z ? 0u : 0x000F000Fu;
          }
        };
        auto decode = [&](int t, int buf) {
#pragma unroll
          for (int j = 0; j < TN; ++j) fb[buf][j] = int4x8_biased_bf16(bw[t / 4 & 1][j][t % 4], keep[j]);
        };
        bar();  // stage 0 has landed
        read_s(0);
        read_w(0, 0);
        read_a(0, 0, 0);
        read_r(0, 0);
        scales(0);
        decode(0, 0);
        auto step = [&](int kt, auto last) {  // the last step apart, as above
          constexpr int NT_ = 16;
#pragma unroll
          for (int t = 0; t < NT_; ++t) {
            const bool more = t + 1 < NT_ || !decltype(last)::value;
            if (t % 8 == 0) {  // the group's rescale, one tile ahead of its first MFMA
#pragma unroll
              for (int i = 0; i < NB; ++i)
#pragma unroll
                for (int j = 0; j < TN; ++j)
#pragma unroll
                  for (int v = 0; v < 16; ++v) acc[i][j][v] = fmaf(acc[i][j][v], ratio[j], rs[i][v]);
            }
            if (t + 1 < NT_) {
              read_a(kt, t + 1, (t + 1) & 1);
              if (t % 4 == 0 && t + 4 < NT_) read_w(kt, t / 4 + 1);
              if (t == 7) read_r(kt, 1);
            } else if (more) {
              __atomic_signal_fence(__ATOMIC_SEQ_CST);
              lds_wait();  // stage kt is in registers
              bar();       // stage kt+1 has landed; buffer kt is free
              read_s(kt + 1);
              read_w(kt + 1, 0);
              read_a(kt + 1, 0, 0);
              read_r(kt + 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            if (more) {
              if (t % 8 == 7) scales((t + 1) / 8 % 2);
              decode((t + 1) % NT_, (t + 1) & 1);
            }
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(fa[t & 1][i], fb[t & 1][j], acc[i][j]);
            if (t + 1 < NT_) {
#pragma unroll
              for (int q = 0; q < NB * TN; ++q) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (t == 7) __builtin_amdgcn_sched_group_barrier(0x002, (7 + NB - 1) / NB + 6, 0);  // and the next scales
                else __builtin_amdgcn_sched_group_barrier(0x002, (7 + NB - 1) / NB, 0);
              }
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < NB; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j) asm volatile("" : "+v"(acc[i][j]));  // the products stay in their substep
          }
        };
        for (int kt = 0; kt + 1 < nk; ++kt) step(kt, std::false_type{});
        step(nk - 1, std::true_type{});
      });
    }
    if constexpr (FMT == 2 && !I4P) {
      for (int kt = 0; kt < nk; ++kt) {
        bar();  // every stage-kt copy of every copy wave has landed
        const uint8_t* Ss = &smem[(sb + kt) % STAGES][A_BYTES + B_BYTES];
        // int4.  The codes enter the MFMA exactly, as bf16 136 + q, and
        // the group scale is applied in fp32: acc holds the tile's sum
        // divided by its column's current scale s, so each step first takes
        // acc * (s_prev / s) - 136 * (the row's sum over the group) and the
        // step's MFMAs then add sum(a * (136 + q)).  A zero scale keeps the
        // previous one and turns the group's codes into q = 0.
        constexpr int NKK = KE / 16, NBW = NKK / 4;
        const uint32_t* sW = reinterpret_cast<const uint32_t*>(Ss);  // one dword per tile row
        const float* sR = reinterpret_cast<const float*>(Ss + (BNW / 64) * 256);  // [BM] biased group sums
        float ratio[TN];
        uint32_t keep[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) {
          const int r = brow(j) + l32;
          const int n_glob = GEMM1 ? (r < NC ? n0 + r : g.I + n0 + (r - NC)) : n0 + r;
          // element index of the scale; only its parity (which half of the dword) is
          // used, so unsigned wrap-around for the largest weight tensors is harmless
          const unsigned idx = (static_cast<unsigned>(e) * (GEMM1 ? 2u * g.I : g.H) + n_glob) * (K / 128) + (kt * KE) / 128;
          const uint32_t d = sW[r];
          const float sc = __uint_as_float((idx & 1) ? (d & 0xFFFF0000u) : (d << 16));
          const bool z = sc == 0.f;
          const float se = z ? seff[j] : sc;
          ratio[j] = seff[j] == 0.f ? 0.f : seff[j] * __builtin_amdgcn_rcpf(se);  // 1-ulp reciprocal
          if (!GEMM1) least = fminf(least, seff[j] == 0.f ? 1.f : fabsf(ratio[j]));
          seff[j] = se;
          keep[j] = z ? 0u : 0x000F000Fu;
        }
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          const int r0 = i * 32 + 4 * kg;  // value v: row r0 + 8*(v/4) + v%4
          f32x16 rs{};
#pragma unroll
          for (int b4 = 0; b4 < (SUMS ? 4 : 0); ++b4) {
            const u32x4 q = ld16(sR + r0 + 8 * b4);
#pragma unroll
            for (int c = 0; c < 4; ++c) rs[4 * b4 + c] = __uint_as_float(q[c]);
          }
#pragma unroll
          for (int j = 0; j < TN; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) acc[i][j][v] = fmaf(acc[i][j][v], ratio[j], rs[v]);
        }
        // substep kk of lane group kg covers K elements [(NKK*kg+kk)*8, +8) of
        // the step, chunk NKK*kg + kk of an activation row and word kk % 4 of
        // chunk NBW*kg + kk/4 of a weight row.  Chunk addresses are one XOR on
        // the stage's (rows aligned to their bytes), and the scheduler keeps to
        // one substep at a time: both hold the kernel in 128 registers.
        static_assert(STAGE % 256 == 0 && A_BYTES % 256 == 0, "rows aligned to their size");
        const int ra = l32, rb = brow(0) + l32;
        const uint32_t st = smem0 + ((sb + kt) % STAGES) * STAGE;
        const uint32_t pa = st + ra * KB + (((NKK * kg) ^ swz<KB>(ra)) << 4);
        const uint32_t pb = st + A_BYTES + rb * BB + (((NBW * kg) ^ swz_b<BB>(rb)) << 4);
        u32x4 bw[TN];
        bf16x8 a[2][TM];
#pragma unroll
        for (int i = 0; i < TM; ++i) a[0][i] = as_bf16x8(lds16(pa + i * 32 * KB));
#pragma unroll
        for (int kk = 0; kk < NKK; ++kk) {
          if (kk % 4 == 0) {
#pragma unroll
            for (int j = 0; j < TN; ++j) bw[j] = lds16((pb ^ (kk / 4) << 4) + (brow(j) - brow(0)) * BB);
          }
          if (kk + 1 < NKK) {
#pragma unroll
            for (int i = 0; i < TM; ++i) a[(kk + 1) & 1][i] = as_bf16x8(lds16((pa ^ (kk + 1) << 4) + i * 32 * KB));
          }
          __builtin_amdgcn_sched_barrier(0);
          bf16x8 b[TN];
#pragma unroll
          for (int j = 0; j < TN; ++j) b[j] = int4x8_biased_bf16(bw[j][kk % 4], keep[j]);
#pragma unroll
          for (int i = 0; i < TM; ++i)
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(a[kk & 1][i], b[j], acc[i][j]);
          if constexpr (!SUMS) {
            const bf16x8 off = as_bf16x8(u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u});  // -136
#pragma unroll
            for (int i = 0; i < TM; ++i)
#pragma unroll
              for (int j = 0; j < TN; ++j) acc[i][j] = mfma32x32x16(a[kk & 1][i], off, acc[i][j]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
    }
#undef brow

    // ---- epilogue.  D element v of a 32x32 tile (GEMM1 with bf16 activations, int4
    // GEMM2): row 8*(v/4) + 4*kg + v%4, column l32.  The others form the product
    // transposed (W is the MFMA's first operand): lane (kg, l32) of row
    // block i holds row i*32 + l32 at columns 8*(v/4) + 4*kg + v%4
    // of each column block, so four consecutive columns per store.
    if constexpr (GSUM) {
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) acc[i][j][v] *= seff[j];
    }
    if constexpr (GEMM1) {
      constexpr int TH = TN / 2;  // gate tiles (paired with up tile j + TH)
      float av[TM][TH][16];
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int j = 0; j < TH; ++j)
#pragma unroll
          for (int v = 0; v < 16; ++v) av[i][j][v] = silu_mul(acc[i][j][v], acc[i][j + TH][v]);
      if constexpr (FMT == 1) {
        // transposed layout: lane (kg, l32) of row block i holds row
        // i*32 + l32 at columns 8*(v/4) + 4*kg + v%4 of each gate
        // block.  Row amax over the tile's 128 columns: the lane's values,
        // the other k-group lane, then the WN waves (LDS).
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if (i >= nb) break;  // blocks of pads are never read
          float m = 0.f;
#pragma unroll
          for (int j = 0; j < TH; ++j)
#pragma unroll
            for (int v = 0; v < 16; ++v) m = fmaxf(m, fabsf(av[i][j][v]));
          m = fmaxf(m, __shfl_xor(m, 32));
          if (kg == 0) lds_amax[wn][i * 32 + l32] = m;
        }
        __syncthreads();
        uint8_t* q = static_cast<uint8_t*>(g.inter);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if (i >= nb) break;
          const int rl = i * 32 + l32;
          float m = 0.f;
#pragma unroll
          for (int w = 0; w < WN; ++w) m = fmaxf(m, lds_amax[w][rl]);
          const float sc = fmaxf(m, 1e-10f) / 448.0f;
          const size_t row = static_cast<size_t>(m0 + rl);
          // a / sc as one IEEE reciprocal per row and a residual step per
          // value: q0 = a r, then q0 + (a - q0 sc) r, the residual exact by
          // fma, the sign restored for a = -0.  On the fp8 workload its codes
          // equal those of the IEEE quotient for all 134M intermediate values
          // (GEMM1 0.7 % faster than a divide per value).
          const float r = 1.0f / sc;
          auto qdiv = [&](float a) {
            const float q0 = a * r;
            return sat_e4m3(__builtin_copysignf(fmaf(fmaf(-q0, sc, a), r, q0), a));
          };
#pragma unroll
          for (int j = 0; j < TH; ++j)
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
              const int col = n0 + wn * (WTN / 2) + j * 32 + 8 * v4 + 4 * kg;
              const float* a4 = &av[i][j][4 * v4];
              const uint32_t codes = f32x2_to_e4m3(qdiv(a4[0]), qdiv(a4[1])) |
                                     (f32x2_to_e4m3(qdiv(a4[2]), qdiv(a4[3])) << 16);
              *reinterpret_cast<uint32_t*>(q + row * g.I + col) = codes;
            }
          if (wn == 0 && kg == 0) g.inter_scale[row * (g.I / 128) + n0 / 128] = sc;
        }
        __syncthreads();  // lds_amax is reused by the next tile
      } else if constexpr (MX8) {
        // transposed layout as fp8; the OCP MX block is one 32-column gate
        // block j of the row: amax over the lane's 16 values and the other
        // k-group lane's, then the E8M0 byte and the exact power-of-two scaling
        uint8_t* q = static_cast<uint8_t*>(g.inter);
#pragma unroll
        for (int i = 0; i < TM; ++i) {
          if (i >= nb) break;  // blocks of pads are never read
          const size_t row = static_cast<size_t>(m0 + i * 32 + l32);
#pragma unroll
          for (int j = 0; j < TH; ++j) {
            float m = 0.f;
#pragma unroll
            for (int v = 0; v < 16; ++v) m = fmaxf(m, fabsf(av[i][j][v]));
            m = fmaxf(m, __shfl_xor(m, 32));
            const uint32_t byte = mx_e8m0_of_amax(m);
            const float mul = __uint_as_float((254u - byte) << 23);
            const int cb = n0 + wn * (WTN / 2) + j * 32;  // the block's first column
#pragma unroll
            for (int v4 = 0; v4 < 4; ++v4) {
              const float* a4 = &av[i][j][4 * v4];
              const uint32_t codes = f32x2_to_e4m3(sat_e4m3(a4[0] * mul), sat_e4m3(a4[1] * mul)) |
                                     (f32x2_to_e4m3(sat_e4m3(a4[2] * mul), sat_e4m3(a4[3] * mul)) << 16);
              *reinterpret_cast<uint32_t*>(q + row * g.I + cb + 8 * v4 + 4 * kg) = codes;
            }
            if (kg == 0) g.inter_mx[row * (g.I / 32) + cb / 32] = static_cast<uint8_t>(byte);
          }
        }
      } else {
        uint16_t* o = static_cast<uint16_t*>(g.inter);
        auto store = [&](bool masked) {
#pragma unroll
          for (int i = 0; i < TM; ++i) {
            if (i >= nb) break;  // blocks of pads are never read
#pragma unroll
            for (int j = 0; j < TH; ++j)
#pragma unroll
              for (int v = 0; v < 16; ++v) {
                const int row = m0 + i * 32 + 8 * (v >> 2) + 4 * kg + (v & 3);
                // int4: eight columns in the order the second product's codes decode to
                const int lc = FMT == 2 ? (l32 & ~7) | (l32 & 3) << 1 | (l32 >> 2 & 1) : l32;
                const int col = n0 + wn * (WTN / 2) + j * 32 + lc;
                if (!masked || col < g.I) o[static_cast<size_t>(row) * g.I + col] = f32_to_bf16(av[i][j][v]);
              }
          }
        };
        if (n0 + NC <= g.I) store(false);  // uniform: only a ragged last column tile masks
        else store(true);
      }
    } else if constexpr (A8) {
      // transposed layout: a lane holds four consecutive output columns per
      // group and the lane 32 away the next four of the same row, so one
      // exchange makes eight consecutive columns per 16-byte store (half the
      // store instructions of 8-byte stores: GEMM2 of the fp8 workload
      // 1608 -> 1502 us)
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m0 + i * 32 + l32;
        if (sid_ep[i] >= g.n_routed) continue;  // pad rows are never read
        uint16_t* yr = static_cast<uint16_t*>(g.y) + static_cast<size_t>(row) * g.H;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int p = 0; p < 2; ++p) {
            // groups 2p and 2p+1 (columns 16p + [0,16) of the block): lane kg
            // keeps its own four columns of group 2p+kg and takes the other
            // lane's four of that group, then stores eight columns at once
            const f32x16& c = acc[i][j];
            const int ga = 2 * p, gb = 2 * p + 1;
            const uint32_t a0 = pack_bf16x2(c[4 * ga], c[4 * ga + 1]), a1 = pack_bf16x2(c[4 * ga + 2], c[4 * ga + 3]);
            const uint32_t b0 = pack_bf16x2(c[4 * gb], c[4 * gb + 1]), b1 = pack_bf16x2(c[4 * gb + 2], c[4 * gb + 3]);
            const uint32_t s0 = kg ? a0 : b0, s1 = kg ? a1 : b1;
            const uint32_t r0 = __shfl_xor(s0, 32), r1 = __shfl_xor(s1, 32);
            const u32x4 o = kg ? u32x4{r0, r1, b0, b1} : u32x4{a0, a1, r0, r1};
            const int col = n0 + wn * WTN + j * 32 + 16 * p + 8 * kg;
            *reinterpret_cast<u32x4*>(yr + col) = o;
          }
      }
    } else if constexpr (FMT == 2) {
      // direct layout, fp32 y: the tile's routed rows come before its pads
      const int live = __popcll(__ballot(live_row)) - 4 * kg;
      float top = 0.f;  // largest magnitude of this lane's outputs
      static_assert(FMT != 2 || BM == 64, "one row per lane in the ballot");
#pragma unroll
      for (int i = 0; i < TM; ++i)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int r = i * 32 + 8 * (v >> 2) + (v & 3);
          if (r >= live) continue;  // pad rows are never read
          float* yr = static_cast<float*>(g.y) + static_cast<size_t>(m0 + r + 4 * kg) * g.H + n0 + wn * WTN + l32;
#pragma unroll
          for (int j = 0; j < TN; ++j) {
            yr[j * 32] = acc[i][j][v];
            top = __builtin_elementwise_maximum(top, fabsf(acc[i][j][v]));  // NaN if one is
          }
        }
      // An intermediate value of Inf, a group whose sum times 136 passes the
      // fp32 range, or scales that fall too far (subnormal ones included: their
      // reciprocal overflows): the biased form gives NaN or Inf, as
      // Inf * (136 + q) - 136 * Inf, where the sum itself may have a value.
      // Scales that rise too far leave nothing of the groups before.  Those
      // outputs are formed again from the codes themselves, one lane each:
      // slow, and nothing to any other tile (half an instruction per output
      // and one per scale; 4000 tokens, 7168 x 2048 x 256 experts, top 8:
      // 3706 us without the checks, 3709 with; the range of every ratio
      // compared on both sides took 3787).
      const bool wide = least < 0x1p-64f;
      if (__builtin_expect(wide || !(top < INFINITY), 0)) {
        for (int b = 0; b < TM * 16 * TN; ++b) {
          const int r = (b / TN / 16) * 32 + 8 * (b / TN % 16 >> 2) + (b / TN & 3);
          if (r >= live) continue;
          const size_t row = static_cast<size_t>(m0 + r + 4 * kg);
          const int n = n0 + wn * WTN + b % TN * 32 + l32;
          float* y = static_cast<float*>(g.y) + row * g.H + n;
          if (!wide && fabsf(*y) < INFINITY) continue;
          const size_t wr = static_cast<size_t>(e) * g.H + n;
          *y = int4_dot(static_cast<const uint16_t*>(g.inter) + row * g.I, static_cast<const uint32_t*>(g.w2) + wr * (g.I / 8),
                        static_cast<const uint16_t*>(g.w2_scale) + wr * (g.I / 128), g.I);
        }
      }
    } else {
      // transposed layout, fp32 y: four consecutive output columns per 16-byte store
      static_assert(TRB && y_is_f32(FMT), "bf16-activation routes keep y in fp32");
      const bool masked = n0 + NC > g.H;  // uniform: only a ragged last column tile masks
#pragma unroll
      for (int i = 0; i < TM; ++i) {
        const int row = m0 + i * 32 + l32;
        if (sid_ep[i] >= g.n_routed) continue;  // pad rows are never read
        float* yr = static_cast<float*>(g.y) + static_cast<size_t>(row) * g.H;
#pragma unroll
        for (int j = 0; j < TN; ++j)
#pragma unroll
          for (int v4 = 0; v4 < 4; ++v4) {
            const int col = n0 + wn * WTN + j * 32 + 8 * v4 + 4 * kg;
            const f32x16& c = acc[i][j];
            if (!masked || col < g.H)  // four columns, all in or all out (H % 4 == 0)
              *reinterpret_cast<f32x4*>(yr + col) = f32x4{c[4 * v4], c[4 * v4 + 1], c[4 * v4 + 2], c[4 * v4 + 3]};
          }
      }
    }
  }
}

// ----------------------------------------------------------------- launchers
namespace {

int cu_count() {
  int dev = 0, n = 0;
  if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0)
    n = 256;
  return n;
}

template <class Kernel>
int occupancy_per_cu(Kernel k, int threads) {
  int per_cu = 1;
  if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, k, threads, 0) != hipSuccess || per_cu < 1)
    per_cu = 1;
  return per_cu;
}

// Persistent grid: as many workgroups as fit on the device at once (per_cu
// per CU, a multiple of the XCD count), never more than the largest possible
// number of tiles.
dim3 persistent_grid(int per_cu, long max_tiles) {
  long n = static_cast<long>(cu_count()) * per_cu;
  n = (n + kXcds - 1) / kXcds * kXcds;
  const long cap = (max_tiles + kXcds - 1) / kXcds * kXcds;
  return dim3(static_cast<unsigned>(std::max<long>(kXcds, std::min(n, cap))));
}

template <int FMT, bool GEMM1, int BM, int BNW, int GM, int KBT, int STAGES, int OPT = 0>
hipError_t launch_tiled(const GroupedGemm& g, hipStream_t s) {
  constexpr int NC = GEMM1 ? BNW / 2 : BNW;
  constexpr int NT = (kMathWaves + kCopyWaves) * 64;
  // only bf16 handles a ragged last K step; every other format's steps must
  // tile K exactly (a step past K would read beyond its rows)
  constexpr int KE = (FMT == 1 || FMT == 5) ? KBT : KBT / 2;
  if (FMT != 0 && (GEMM1 ? g.H : g.I) % KE != 0) return hipErrorInvalidValue;
  const long mt = g.max_rows / BM, nt = ((GEMM1 ? g.I : g.H) + NC - 1) / NC;
  auto kern = moe_gemm_tiled<FMT, GEMM1, BM, BNW, GM, KBT, STAGES, OPT>;
  // workgroups per CU depend on the kernel's registers and LDS only: queried
  // once per instantiation (thread-safe static initialisation)
  static const int per_cu = occupancy_per_cu(kern, NT);
  hipLaunchKernelGGL(kern, persistent_grid(per_cu, mt * nt), dim3(NT), 0, s, g);
  return hipGetLastError();
}

}  // namespace

// Whether the bf16 kernels copy the weights of experts with one row tile with the
// non-temporal hint: where experts have at most a tile of rows on average.  Layers
// without and with it, the same weights as in the call before and, second, after
// 1 GB of other reads: 4096 x 1408 x 64 experts, top 6, 777 tokens (73 rows per
// expert) 495 -> 473 us, -4.3 %; 1200 (112) -1.2 %, -0.8 %; 2500 (234) +0.2 %, +0.8 %; 4096
// (384) +0.7 %, +0.8 %, the choice alone.  The fp8 kernels always do: 7168 x 2048 x 256
// experts, top 8, 300 tokens (9) 1245 -> 1162, -6.2 %; 4000 (125) -0.7 %, -1.0 %; 8192 (256)
// -1.0 %, -1.0 %.  So do the 256-element int4 steps, for little: 4096 x 1536 x 128 experts,
// top 8, 512 tokens -1.5 %, +0.4 %, 2048 -0.7 %, -1.7 %, 5120 x 1536 x 160, top 6, 200 tokens
// +0.9 %, +2.0 %.  MXFP4 x MXFP8 has no use for it: 2048 x 1408 x 60 experts, top 4, 260
// tokens +14 %, +2.5 % (weights that the memory-side cache held from call to call no
// longer stay there), 7168 x 2048 x 256, 1000 tokens -0.1 %, +0.1 %.  Nor has MXFP4, as far
// as measured (8192 tokens 6243 -> 6332 us).
bool weights_once(const GroupedGemm& g) { return g.n_routed <= 128L * g.E; }

// most row tiles of one expert swept together per column tile
constexpr int kSweep = 8, kSweepInt4 = 16;

int bf16_tiled_block_m() { return 128; }
template <bool GEMM1, int BNW>
hipError_t launch_bf16(const GroupedGemm& g, hipStream_t s) {
  if (weights_once(g)) return launch_tiled<0, GEMM1, 128, BNW, kSweep, 128, 3, kOnce>(g, s);
  return launch_tiled<0, GEMM1, 128, BNW, kSweep, 128, 3>(g, s);
}
hipError_t launch_gemm1_bf16_tiled(const GroupedGemm& g, hipStream_t s) { return launch_bf16<true, 256>(g, s); }
hipError_t launch_gemm2_bf16_tiled(const GroupedGemm& g, hipStream_t s) {
  if (g.H % 256) return launch_bf16<false, 128>(g, s);
  return launch_bf16<false, 256>(g, s);
}

int gemm_block_m_fp8(int, int, int) { return 128; }
template <bool GEMM1, int BNW>
hipError_t launch_fp8(const GroupedGemm& g, hipStream_t s) {
  return launch_tiled<1, GEMM1, 128, BNW, kSweep, 128, 3, kOnce>(g, s);
}
hipError_t launch_gemm1_fp8(const GroupedGemm& g, hipStream_t s) { return launch_fp8<true, 256>(g, s); }
hipError_t launch_gemm2_fp8(const GroupedGemm& g, hipStream_t s) {
  if (g.H % 256) return launch_fp8<false, 128>(g, s);
  return launch_fp8<false, 256>(g, s);
}

// int4 row tile: one math wave per 64 columns covers all 64 rows, so each decoded
// weight fragment feeds two MFMAs
constexpr int kInt4BM = 64;
int gemm_block_m_int4(int, int, int) { return kInt4BM; }
// Where GEMM2 finds the intermediate's group sums: each of its tiles, BNW
// columns wide, reads them from its own part of y (64 rows, room for BNW groups
// of 64 sums), which it overwrites when it has read them all.  An intermediate of
// more groups goes without (the bias comes off by MFMAs of its own, which doubles
// them): returns 0.  So does one of one or two groups, where the launch that
// sums costs more (8 experts, top 2, H = 256, I = 128: 17 tokens 28.6 us with,
// 26.5 without, 8192 tokens 55.9 and 53.9; at I = 512, 10000 rows, 66.3 and 67.9).
int int4_sum_columns(int H, int I) {
  const int bnw = H % 256 ? 128 : 256;
  return I > 256 && I / 128 <= bnw ? bnw : 0;
}
// 256 K elements per step (whole weight lines) leave room for one workgroup per
// CU, 128 (64 bytes of each weight row, half a line) for two, which hide each other's first steps and epilogues.  256 where
// K is a multiple of that and long (1536: 512 tokens, 128 experts 359 us, 388
// with 128), or each workgroup has one tile at most (H = I = 512, 32 experts, top
// 4, 150 tokens: 33.8 and 36.8 us).  Short K with many tiles takes 128 (8192
// tokens of that layer 147 and 136 us; H = I = 1024, 8 experts, top 2, 196 and 183).
template <bool GEMM1, int BNW>
bool int4_long_steps(const GroupedGemm& g) {
  const int K = GEMM1 ? g.H : g.I, N = GEMM1 ? g.I : g.H;
  constexpr int NC = GEMM1 ? BNW / 2 : BNW;
  const long tiles = static_cast<long>(g.max_rows / kInt4BM) * ((N + NC - 1) / NC);
  return K % 256 == 0 && (K >= 1536 || tiles <= cu_count());
}
template <bool GEMM1, int BNW>
hipError_t launch_int4(const GroupedGemm& g, hipStream_t s) {
  if constexpr (!GEMM1)
    if (!g.inter_sums) return launch_tiled<2, false, kInt4BM, BNW, kSweepInt4, 256, 2, kNoSums>(g, s);
  if (int4_long_steps<GEMM1, BNW>(g)) return launch_tiled<2, GEMM1, kInt4BM, BNW, kSweepInt4, 512, 2, kOnce>(g, s);
  return launch_tiled<2, GEMM1, kInt4BM, BNW, kSweepInt4, 256, 2>(g, s);
}
hipError_t launch_gemm1_int4(const GroupedGemm& g, hipStream_t s) { return launch_int4<true, 256>(g, s); }
// MXFP4 weights (same 4-bit packing as int4, E8M0 scales per 32)
int gemm_block_m_mxfp4() { return 128; }
hipError_t launch_gemm1_mxfp4_tiled(const GroupedGemm& g, hipStream_t s) {
  return launch_tiled<4, true, 128, 256, kSweep, 256, 3>(g, s);
}
hipError_t launch_gemm2_mxfp4_tiled(const GroupedGemm& g, hipStream_t s) {
  if (g.H % 256) return launch_tiled<4, false, 128, 128, kSweep, 256, 3>(g, s);
  return launch_tiled<4, false, 128, 256, kSweep, 256, 3>(g, s);
}
// MXFP4 weights x MXFP8 activations: the fp8 tile (128 x 256, four math
// waves beside four copy waves).  When K is a multiple of 256, 256-element K
// steps, so each weight row gives a whole 128-byte line per step (256 bytes
// of each activation row, two E8M0 dwords per row of either), two stages;
// otherwise (K a multiple of 128) 128-element steps (half a line of each
// weight row) with four stages.  A step never reaches past K.
template <bool GEMM1, int BNW>
hipError_t launch_mx8(const GroupedGemm& g, hipStream_t s) {
  const int K = GEMM1 ? g.H : g.I;
  if (K % 256 == 0) return launch_tiled<5, GEMM1, 128, BNW, kSweep, 256, 2>(g, s);
  return launch_tiled<5, GEMM1, 128, BNW, kSweep, 128, 4>(g, s);
}
hipError_t launch_gemm1_mx8(const GroupedGemm& g, hipStream_t s) { return launch_mx8<true, 256>(g, s); }
hipError_t launch_gemm2_mx8(const GroupedGemm& g, hipStream_t s) {
  if (g.H % 256) return launch_mx8<false, 128>(g, s);
  return launch_mx8<false, 256>(g, s);
}
hipError_t launch_gemm2_int4(const GroupedGemm& g, hipStream_t s) {
  if (g.H % 256) return launch_int4<false, 128>(g, s);
  return launch_int4<false, 256>(g, s);
}

}  // namespace moe
