// mixed.hip -- one launch for a serving step that mixes a causal prefill chunk
// and split-KV decode (Sec. 7.3: prefill and decode requests served together).
//
// The prefill work items (query head, 256-row query tile; matrix-bound) and
// groups of eight decode work items (sequence, KV head, partition; HBM-bound)
// share one grid.  Each decode partition counts itself in a per-(sequence, KV
// head) counter when its state is written; the last one merges the group's
// query heads (log-sum-exp, the same arithmetic as the separate merge kernel)
// and resets the counter, so the step needs no second launch.  A workgroup is
// 512 threads; a prefill item uses 106 KB of LDS for its two tile buffers (MXFP4 59;
// 72 with the few-row items, whose NVFP4 form has 108 bytes of scratch), a group of eight decode items none (their K and V go
// straight to registers).
//
// Placement: a prefill workgroup holds a whole compute unit (its LDS and all
// of its registers), so prefill and decode cannot share a unit at the same
// time; but the prefill's last round of items leaves units idle, and the decode
// groups, dispatched after the prefill items, fill them.  4096 rows behind 16384
// tokens and 64 decoding sequences, 40:8: 1362 us, 1624 with the decode first,
// 1626 for the two calls; 2048 behind 8000 and 32 x 4000 keys 420 / 485 / 470;
// 16384-token prompt and 64 x 6000 keys 2251 / 2258 / 2316; the decode first is the
// better one only for a short prompt beside a long decode (1000 tokens, 16 x
// 30000 keys: 263 / 253 / 204).  Where the decode is the longer part one launch loses
// to the two calls: a unit holds one workgroup of eight decode waves and drains (barrier,
// cache write-back, barrier, perhaps a merge) before the next group starts, where the
// two four-wave workgroups of decode_kernel refill apart.
#include <type_traits>

#include "decode_body.h"
#include "prefill_body.h"
#include "prefill_split.h"

namespace mpfa {

namespace {

// Blocks are dealt to the 8 XCDs round-robin: the prefill items come first, in
// their own order (largest query tiles first), on the XCDs they have in the
// separate launch; then, from the next multiple of 8, the decode groups of 8
// work items.
// FEW: the prefill items are those of prefill_few_kernel (the same bytes as the
// separate calls either way).
template <bool SMOOTH, bool MX, bool FEW>
__global__ __launch_bounds__(512, 1) void mixed_kernel(MixedParams m) {
  __shared__ __attribute__((aligned(16))) std::conditional_t<FEW, FewSmem<MX>, PrefillSmemT<MX, kPvFp8>> lds;
  const int i = blockIdx.x;
  if (i < m.first) {
    if (i >= m.n_pre_blocks) return;
    constexpr int kSeed = SMOOTH ? kSeedInit : kSeedNone;
    if constexpr (FEW) prefill_few_block<kSeed, MX>(m.pre, i, lds);
    else prefill_block<kSeed, MX, kPvFp8>(m.pre, i, lds);
    return;
  }
  // decode group: wave w takes item 8 * group + w = ((b * h_kv + hk) *
  // max_partitions + part)
  const int wave = threadIdx.x >> 6;
  const int item = (i - m.first) * 8 + wave;
  const DecodeParams& p = m.dec;
  const int part = item % p.max_partitions;
  const int hk = (item / p.max_partitions) % p.h_kv;
  const int b = item / (p.max_partitions * p.h_kv);
  const bool live = b < p.batch;
  if (live) decode_partition<SMOOTH, MX>(p, b, hk, part);
  // Release: the group's states become visible device-wide before any of its
  // waves counts itself.  One write-back of the XCD's L2 per workgroup, between
  // two barriers: one per wave (eight times as many) cost more than the decode
  // itself (1000-token prompt and 16 x 30000 keys: 498 -> 253 us).
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // this wave's states are in the L2
  __syncthreads();
  if (wave == 0) __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
  __syncthreads();
  if (!live) return;
  const int np = (p.kv_len[b] + p.partition_tokens - 1) / p.partition_tokens;
  if (part >= np) return;
  uint32_t prev = 0;
  if ((threadIdx.x & 63) == 0) prev = atomicAdd(&m.counters[b * p.h_kv + hk], 1u);
  prev = __shfl(prev, 0);
  if (prev != (uint32_t)(np - 1)) return;
  // the last partition of (b, hk): merge its query heads, reset the counter
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");   // every state counted before is visible
  const int grp = p.h_q / p.h_kv;
  for (int j = 0; j < grp; ++j) merge_head<kMergeChunk>(p, b, hk * grp + j, np);
  if ((threadIdx.x & 63) == 0) atomicExch(&m.counters[b * p.h_kv + hk], 0u);
}

template <bool SMOOTH, bool MX>
void launch_form(const MixedParams& m, dim3 grid, dim3 block, hipStream_t stream) {
  if (m.pre.few) mixed_kernel<SMOOTH, MX, true><<<grid, block, 0, stream>>>(m);
  else mixed_kernel<SMOOTH, MX, false><<<grid, block, 0, stream>>>(m);
}

}  // namespace

hipError_t launch_mixed(const MixedParams& m, hipStream_t stream) {
  const unsigned blocks = (unsigned)m.n_blocks;
  if (blocks == 0) return hipSuccess;
  const dim3 grid(blocks), block(512);
  if (m.pre.mx) {
    if (m.pre.smooth) launch_form<true, true>(m, grid, block, stream);
    else launch_form<false, true>(m, grid, block, stream);
  } else {
    if (m.pre.smooth) launch_form<true, false>(m, grid, block, stream);
    else launch_form<false, false>(m, grid, block, stream);
  }
  return hipGetLastError();
}

}  // namespace mpfa
