// prefill.hip -- causal QK4PV8 prefill for gfx950 (Algorithm 1 main loop).
//
// One workgroup = 8 waves = 256 query rows of one query head; each wave owns
// 32 rows, the columns of one 32x32 MFMA.  Per 128-key tile (visited from the
// block's last tile down to tile 0, Sec. 4.1):
//   * the workgroup stages the tile in LDS: NVFP4 K dequantized once to exact
//     FP16 (group scale applied, tensor scale factored out), FP8 V in its
//     channel-major page layout, and the compensation vector Delta_S;
//   * each wave computes S^T = K Q^T on FP16 MFMA (32x32x16) starting from
//     the rank-one term 1 Delta_S^T (Sec. 4.3 Eq. 11): loaded from LDS as the
//     accumulator input, or (MPFA_SEED_MFMA) formed by one BF16 rank-one MFMA
//     per 32x32 block as in Sec. 5.2;
//   * mask, row max, P = 2^(lambda (S - m) + log2 448), row sum of the FP32 P,
//     FP8 conversion in registers; the S^T accumulator layout is already the
//     B-operand layout of the FP8 PV MFMA (O^T = V^T P^T), so P never leaves
//     registers;
//   * O^T rescale (skipped when no row maximum moved) and FP8 MFMA
//     (32x32x64) accumulation.
// The key order inside a 32-row MFMA block is permuted so that the 32 keys a
// lane holds for a PV MFMA are contiguous (tile_key).
#include "prefill_body.h"
#include "prefill_split.h"

namespace mpfa {

namespace {

constexpr int kThreads = kItemWaves * 64;

template <int SEED, bool MX, int PV, int ABL = 0>
__global__ __launch_bounds__(kThreads, 1) void prefill_kernel(PrefillParams p) {
  __shared__ __attribute__((aligned(16))) PrefillSmemT<MX, PV> smem;
  prefill_block<SEED, MX, PV, ABL>(p, blockIdx.x, smem);
}

// Short prompts: a workgroup per 128 rows, with items of 128 rows where that pays, else
// every other one takes 256 (item_rows).  The same bytes.  Taken up to kHalfBlocks
// workgroups (api.cpp): 250 tokens 32:8 16.0 -> 10.8 us, 1600 (416 workgroups) 45 ->
// 36.3.  Above, one prompt would gain (2048 tokens, 512: 56.4 -> 47.3), short batches
// lose (4 x 300 tokens 40:8, 480: 25.8 -> 26.6).
template <bool SMOOTH, bool MX>
__global__ __launch_bounds__(kThreads, 1) void prefill_half_kernel(PrefillParams p) {
  __shared__ __attribute__((aligned(16))) PrefillSmemT<MX, kPvFp8> smem;
  int b, h, rank;
  map_item(p, blockIdx.x, b, h, rank);
  const int blk = p.n_qtiles - 1 - rank;
  if (blk * kHalfRows >= p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b]) return;
  prefill_pick_block<SMOOTH ? kSeedInit : kSeedNone, MX, kHalfRows>(p, b, h, blk, item_rows(p, b), smem);
}

template <int SEED, bool MX>
__global__ __launch_bounds__(kThreads, 1) void prefill_few_kernel(PrefillParams p) {
  __shared__ __attribute__((aligned(16))) FewSmem<MX> sm;
  prefill_few_block<SEED, MX>(p, blockIdx.x, sm);
}

#ifdef MPFA_ABLATION_BUILD
// Characterization library only: softmax ablation level of the method's
// kernels (compensation as accumulator input, FP8 PV), see max_tile.
int g_ablation = 0;
#endif

}  // namespace

#ifdef MPFA_ABLATION_BUILD
// declared in include/mpfa_ablate.h
extern "C" int mpfa_ablation_set_level(int level) {
  if (level < 0 || level > 2) return 1;
  g_ablation = level;
  return 0;
}
#endif

hipError_t launch_prefill(const PrefillParams& p, hipStream_t stream) {
  const unsigned blocks = (unsigned)(p.n_qtiles * p.h_q * p.batch);
  if (blocks == 0) return hipSuccess;
  const dim3 grid(blocks), block(kThreads);
#ifdef MPFA_ABLATION_BUILD
  if (g_ablation > 0 && p.pv == kPvFp8 && p.smooth && !p.seed_mfma && !p.seed_elem) {
    if (p.mx) {
      if (g_ablation == 1) prefill_kernel<kSeedInit, true, kPvFp8, 1><<<grid, block, 0, stream>>>(p);
      else prefill_kernel<kSeedInit, true, kPvFp8, 2><<<grid, block, 0, stream>>>(p);
    } else {
      if (g_ablation == 1) prefill_kernel<kSeedInit, false, kPvFp8, 1><<<grid, block, 0, stream>>>(p);
      else prefill_kernel<kSeedInit, false, kPvFp8, 2><<<grid, block, 0, stream>>>(p);
    }
    return hipGetLastError();
  }
#endif
  if (p.half && !p.few) {
    if (p.mx) {
      if (p.smooth) prefill_half_kernel<true, true><<<grid, block, 0, stream>>>(p);
      else prefill_half_kernel<false, true><<<grid, block, 0, stream>>>(p);
    } else {
      if (p.smooth) prefill_half_kernel<true, false><<<grid, block, 0, stream>>>(p);
      else prefill_half_kernel<false, false><<<grid, block, 0, stream>>>(p);
    }
  } else if (p.few) {
    if (p.mx) {
      if (!p.smooth) prefill_few_kernel<kSeedNone, true><<<grid, block, 0, stream>>>(p);
      else if (p.seed_mfma) prefill_few_kernel<kSeedMfma, true><<<grid, block, 0, stream>>>(p);
      else prefill_few_kernel<kSeedInit, true><<<grid, block, 0, stream>>>(p);
    } else {
      if (!p.smooth) prefill_few_kernel<kSeedNone, false><<<grid, block, 0, stream>>>(p);
      else if (p.seed_mfma) prefill_few_kernel<kSeedMfma, false><<<grid, block, 0, stream>>>(p);
      else prefill_few_kernel<kSeedInit, false><<<grid, block, 0, stream>>>(p);
    }
  } else if (p.pv == kPvBf16) {
    if (!p.smooth) prefill_kernel<kSeedNone, false, kPvBf16><<<grid, block, 0, stream>>>(p);
    else prefill_kernel<kSeedInit, false, kPvBf16><<<grid, block, 0, stream>>>(p);
  } else if (p.pv == kPvNvfp4) {
    if (!p.smooth) prefill_kernel<kSeedNone, false, kPvNvfp4><<<grid, block, 0, stream>>>(p);
    else prefill_kernel<kSeedInit, false, kPvNvfp4><<<grid, block, 0, stream>>>(p);
  } else if (p.mx) {
    if (!p.smooth) prefill_kernel<kSeedNone, true, kPvFp8><<<grid, block, 0, stream>>>(p);
    else if (p.seed_mfma) prefill_kernel<kSeedMfma, true, kPvFp8><<<grid, block, 0, stream>>>(p);
    else if (p.seed_elem) prefill_kernel<kSeedElem, true, kPvFp8><<<grid, block, 0, stream>>>(p);
    else prefill_kernel<kSeedInit, true, kPvFp8><<<grid, block, 0, stream>>>(p);
  } else {
    if (!p.smooth) prefill_kernel<kSeedNone, false, kPvFp8><<<grid, block, 0, stream>>>(p);
    else if (p.seed_mfma) prefill_kernel<kSeedMfma, false, kPvFp8><<<grid, block, 0, stream>>>(p);
    else if (p.seed_elem) prefill_kernel<kSeedElem, false, kPvFp8><<<grid, block, 0, stream>>>(p);
    else prefill_kernel<kSeedInit, false, kPvFp8><<<grid, block, 0, stream>>>(p);
  }
  return hipGetLastError();
}

}  // namespace mpfa
