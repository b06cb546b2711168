// decode.hip -- split-KV QK4PV8 decode over the paged cache for gfx950
// (Sec. 5.3), plus the log-sum-exp merge of the partition states.
//
// One wave = one (sequence, KV head, partition).  The G = H_q / H_kv query
// heads of the KV head are packed into the 16-wide MFMA column dimension
// (GQA packing); the compensation becomes a rank-G term (Delta_S differs per
// query head), loaded as the input accumulator of the first QK MFMA: each
// lane's four accumulator rows are four consecutive keys of one query head,
// one 8-byte load per 16-key block.  K and V stream straight
// from HBM into registers (no LDS): each lane loads 16 contiguous bytes of
// NVFP4 codes per key it owns and 32 contiguous FP8 bytes of the channel-major
// V page, dequantizes K exactly to FP16 and runs the same S^T = K Q^T /
// O^T = V^T P^T MFMA chain as prefill.  The reduction (head) dimension is
// permuted (lane group g, step ks, element e -> channel 32g + 8ks + e) so that
// every lane's code bytes are contiguous; Q uses the same permutation.
#include "decode_body.h"

#include <mutex>

namespace mpfa {

// Partition states of mpfa_decode_paged_static: one array per GPU, created
// with the code object and held until the process ends.  Host code never uses
// the name itself (on the host it only stands for the symbol); it uses the
// device address that hipGetSymbolAddress returns for the current device.
static __device__ __align__(256) uint8_t scratch[kStaticScratchBytes];

namespace {
constexpr int kMaxDevices = 64;
std::mutex scratch_mu;
void* scratch_addr[kMaxDevices] = {};
}  // namespace

hipError_t static_decode_scratch(void** ptr) {
  int dev = -1;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(scratch_mu);
  if (!scratch_addr[dev]) {
    void* a = nullptr;
    e = hipGetSymbolAddress(&a, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    scratch_addr[dev] = a;
  }
  *ptr = scratch_addr[dev];
  return hipSuccess;
}

namespace {

// Block -> work map.  Workgroups are dealt to the 8 XCDs round-robin by block
// id.  The (sequence, group of kWavesPerBlock partitions) pairs that hold work
// are numbered k = 0, 1, ... in sequence order, so no workgroup is spent on a
// partition past a short sequence's end.  Pair k takes the 8 blocks of slot k
// (one per XCD), and the KV head run on XCD x is (x - k) mod 8: each pair's
// heads spread over all XCDs and every XCD sees every head, so the XCDs share
// the work evenly whatever the sequence lengths.  KV head counts above 8 take
// ceil(h_kv / 8) consecutive slots per pair.  A block finds its pair by a
// prefix sum of the sequences' group counts across the wave's lanes, 64
// sequences at a time.  That lookup costs every block O(batch), so batches
// above kDecodePackedMaxBatch sequences use the plain grid (partition group, KV
// head, sequence) instead, with an odd group count so that each (KV head,
// sequence) row still spreads over the XCDs.  Either map gives every
// partition to exactly one wave; the results do not depend on it.
__device__ __forceinline__ int partition_groups(int kvl, int partition_tokens) {
  const int np = (kvl + partition_tokens - 1) / partition_tokens;
  return (np + kWavesPerBlock - 1) / kWavesPerBlock;
}

template <bool SMOOTH, bool MX, bool PACKED>
__global__ __launch_bounds__(kWavesPerBlock * 64, 2) void decode_kernel(DecodeParams p) {
  const int wave = threadIdx.x >> 6;
  if (!PACKED) {
    // grid (partition group, KV head, sequence); groups past the sequence's
    // partitions return inside decode_partition
    decode_partition<SMOOTH, MX>(p, blockIdx.z, blockIdx.y, blockIdx.x * kWavesPerBlock + wave);
    return;
  }
  const int xcd = blockIdx.x & 7, slot = blockIdx.x >> 3;
  const int hrows = (p.h_kv + 7) >> 3;
  const int k = slot / hrows, hk = (slot % hrows) * 8 + ((xcd - k) & 7);
  if (hk >= p.h_kv) return;
  const int lane = threadIdx.x & 63;
  int b = -1, grp = 0, base = 0;
  for (int b0 = 0; b0 < p.batch && b < 0; b0 += 64) {
    const int bb = b0 + lane;
    const int cnt = bb < p.batch ? partition_groups(p.kv_len[bb], p.partition_tokens) : 0;
    int incl = cnt;   // inclusive prefix sum over the lanes
#pragma unroll
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d);
      if (lane >= d) incl += up;
    }
    const int total = __shfl(incl, 63);
    if (k < base + total) {
      const uint64_t past = __ballot(base + incl > k);   // lanes whose sequence ends after pair k
      const int first = __ffsll((unsigned long long)past) - 1;
      b = b0 + first;
      grp = k - (base + __shfl(incl, first) - __shfl(cnt, first));
    }
    base += total;
  }
  if (b < 0) return;   // the grid is sized for batch * ceil(max_partitions / 4) pairs
  decode_partition<SMOOTH, MX>(p, b, hk, grp * kWavesPerBlock + wave);
}

// Merge of the partition states, one workgroup per (query head, sequence).  A
// separate launch: merging in the last-arriving decode wave needs the partition
// states made visible across the XCDs' L2 caches (an L2 write-back per wave, or
// write-through stores and an arrival counter), which measured slower than this
// second launch.  Up to 32 partitions one wave merges them (17 partitions 5.6 ->
// 3.5 us).
template <int N>
__global__ __launch_bounds__(64) void merge_kernel(DecodeParams p) {
  const int h = blockIdx.x, b = blockIdx.y;
  merge_head<N>(p, b, h, (p.kv_len[b] + p.partition_tokens - 1) / p.partition_tokens);
}

// More than one chunk: WAVES waves share the chunks, a round of WAVES at a time.
// The states are read once, a chunk's 32 rows in flight per wave; what it costs is
// the round trips and what one compute unit can fetch (512 partitions: 266 KB per
// head), so few heads are merged by two workgroups of 64 channels each (CH = 1
// channel per lane instead of 2), of sixteen waves.  The sums and their order are
// the same in each.  One sequence of 131072 keys, 40 heads: 75 us by one wave, 10
// by eight, 7.5 by 2 x 16 (the whole call 48.0 -> 45.2; 500000 keys 181.7 ->
// 175.8).  With more heads the two read the (m, l) twice for nothing (2 x 30000
// keys 32:8 24.7 / 24.3, but 4 x 30000 41.3 / 41.3, 4 x 9000 40:8 22.3 / 24.4, 8 x
// 30000 89.2 / 92.0).
constexpr int kSplitMergeHeads = 64;

template <int WAVES, int CH>
__global__ __launch_bounds__(WAVES * 64) void merge_wide_kernel(DecodeParams p) {
  constexpr int SLICES = 2 / CH;
  const int h = blockIdx.x / SLICES, b = blockIdx.y;
  const int np = (p.kv_len[b] + p.partition_tokens - 1) / p.partition_tokens;
  __shared__ float wave_top[WAVES];
  __shared__ float part_o[WAVES][CH][64];
  __shared__ float part_l[WAVES];
  const float* st = head_states(p, b, h);
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int ch = (blockIdx.x % SLICES) * 64 + CH * lane;   // this lane's first channel
  float o[kMergeChunk][CH];
  float2 ml = {};
  auto load = [&](int q0) {   // all in flight; past np the last partition repeats and is not used
    ml = merge_ml(st, q0, np);
#pragma unroll
    for (int j = 0; j < kMergeChunk; ++j) {
      const float* row = st + (int64_t)min(q0 + j, np - 1) * (kD + 2) + 2 + ch;
      if constexpr (CH == 2) {
        const float2 v = *reinterpret_cast<const float2*>(row);
        o[j][0] = v.x;
        o[j][1] = v.y;
      } else {
        o[j][0] = *row;
      }
    }
  };
  if (wave * kMergeChunk < np) load(wave * kMergeChunk);
  float M = -INFINITY;
  for (int q = threadIdx.x; q < np; q += WAVES * 64) M = fmaxf(M, st[(int64_t)q * (kD + 2)]);
  M = wave_max64(M);
  if (lane == 0) wave_top[wave] = M;
  __syncthreads();
#pragma unroll
  for (int w = 0; w < WAVES; ++w) M = fmaxf(M, wave_top[w]);
  float L = 0.0f, O[CH] = {};   // wave 0
  for (int r0 = 0; r0 < np; r0 += WAVES * kMergeChunk) {
    const int q0 = r0 + wave * kMergeChunk;
    if (q0 < np) {
      if (r0 > 0) load(q0);
      const float f = __builtin_amdgcn_exp2f(ml.x - M);
      float l = 0.0f, s[CH] = {};
#pragma unroll
      for (int j = 0; j < kMergeChunk; ++j) {
        if (q0 + j < np) {
          const float fj = __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(f), j));
          l = __builtin_fmaf(fj, __uint_as_float(__builtin_amdgcn_readlane(__float_as_uint(ml.y), j)), l);
#pragma unroll
          for (int i = 0; i < CH; ++i) s[i] = __builtin_fmaf(fj, o[j][i], s[i]);
        }
      }
#pragma unroll
      for (int i = 0; i < CH; ++i) part_o[wave][i][lane] = s[i];
      if (lane == 0) part_l[wave] = l;
    }
    __syncthreads();
    if (wave == 0) {
      for (int w = 0; w < WAVES && r0 + w * kMergeChunk < np; ++w) {
        L += part_l[w];
#pragma unroll
        for (int i = 0; i < CH; ++i) O[i] += part_o[w][i][lane];
      }
    }
    __syncthreads();
  }
  if (wave != 0) return;
  if constexpr (CH == 2) merge_store(p, b, h, L, O[0], O[1], np > 0);
  else p.out[((int64_t)b * p.h_q + h) * kD + ch] = (uint16_t)bf16_rne(np > 0 ? __fdiv_rn(O[0], L) : 0.0f);
}

// Short contexts: one workgroup per (KV head, sequence) whose waves are its
// partitions; the states stay in LDS and wave j merges query heads j, j + WAVES,
// ... after a barrier.  Saves the merge launch and its round trips to memory
// (group_decode says when).
template <bool SMOOTH, bool MX, int WAVES>
__global__ __launch_bounds__(WAVES * 64, 1) void decode_group_kernel(DecodeParams p) {
  extern __shared__ __attribute__((aligned(16))) float states[];   // [WAVES][grp][kD + 2]
  const int hk = blockIdx.x, b = blockIdx.y, wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int grp = p.h_q / p.h_kv, slice = grp * (kD + 2);
  decode_partition<SMOOTH, MX, true>(p, b, hk, wave, states + wave * slice);
  __syncthreads();
  const int np = (p.kv_len[b] + p.partition_tokens - 1) / p.partition_tokens;
  for (int j = wave; j < grp; j += WAVES) {
    const float* st = states + j * (kD + 2);
    float M = -INFINITY, L = 0.0f, O0 = 0.0f, O1 = 0.0f;
    for (int q = 0; q < np; ++q) M = fmaxf(M, st[q * slice]);
    for (int q = 0; q < np; ++q) {
      const float* sq = st + q * slice;
      const float f = __builtin_amdgcn_exp2f(sq[0] - M);
      L = __builtin_fmaf(f, sq[1], L);
      O0 = __builtin_fmaf(f, sq[2 + 2 * lane], O0);
      O1 = __builtin_fmaf(f, sq[3 + 2 * lane], O1);
    }
    merge_store(p, b, hk * grp + j, L, O0, O1, np > 0);
  }
}

template <bool SMOOTH, bool MX>
hipError_t launch_decode_group(const DecodeParams& p, hipStream_t stream) {
  const dim3 grid(p.h_kv, p.batch);
  const size_t slice = (size_t)(p.h_q / p.h_kv) * (kD + 2) * sizeof(float);
  if (p.max_partitions <= 1) decode_group_kernel<SMOOTH, MX, 1><<<grid, dim3(64), slice, stream>>>(p);
  else if (p.max_partitions <= 2) decode_group_kernel<SMOOTH, MX, 2><<<grid, dim3(128), 2 * slice, stream>>>(p);
  else if (p.max_partitions <= 4) decode_group_kernel<SMOOTH, MX, 4><<<grid, dim3(256), 4 * slice, stream>>>(p);
  else decode_group_kernel<SMOOTH, MX, 8><<<grid, dim3(512), 8 * slice, stream>>>(p);
  return hipGetLastError();
}

// When a call takes decode_group_kernel (times of the whole call, 32:8 heads; the
// two launches / one): up to 4 partitions while there are at most kGroupMaxWaves
// waves, two per SIMD of the chip: 1 x 60 keys 12.0 / 9.0 us, 900 keys x 16 14.0
// / 10.0, 500 x 256 (4096 waves) 50.1 / 44.1.  5 to 8 partitions only when the
// packed grid's workgroups would share compute units anyway (more than 256 of
// them): 1500 keys x 32 22.1 / 17.3 us, x 64 35.9 / 32.9, but x 8 13.1 / 14.4 (a
// unit then has eight waves' keys to fetch where two workgroups had two).
constexpr int kGroupWaves = 8, kGroupMaxWaves = 4096;

bool group_decode(const DecodeParams& p) {
  if (p.max_partitions > kGroupWaves) return false;
  const int w = p.max_partitions <= 2 ? p.max_partitions : (p.max_partitions <= 4 ? 4 : kGroupWaves);
  if ((int64_t)p.batch * p.h_kv * w > kGroupMaxWaves) return false;
  return w <= 4 || (int64_t)p.batch * 2 * ((p.h_kv + 7) / 8 * 8) > 256;
}

}  // namespace

hipError_t launch_decode(const DecodeParams& p, hipStream_t stream) {
  if (p.batch == 0) return hipSuccess;
  if (group_decode(p)) {
    if (p.mx) return p.smooth ? launch_decode_group<true, true>(p, stream) : launch_decode_group<false, true>(p, stream);
    return p.smooth ? launch_decode_group<true, false>(p, stream) : launch_decode_group<false, false>(p, stream);
  }
  const int groups = (p.max_partitions + kWavesPerBlock - 1) / kWavesPerBlock;
  const dim3 block(kWavesPerBlock * 64);
  if (p.batch <= kDecodePackedMaxBatch) {
    const int64_t pairs = (int64_t)p.batch * groups;
    const dim3 grid((unsigned)(pairs * ((p.h_kv + 7) / 8 * 8)));
    if (p.mx) {
      if (p.smooth) decode_kernel<true, true, true><<<grid, block, 0, stream>>>(p);
      else decode_kernel<false, true, true><<<grid, block, 0, stream>>>(p);
    } else {
      if (p.smooth) decode_kernel<true, false, true><<<grid, block, 0, stream>>>(p);
      else decode_kernel<false, false, true><<<grid, block, 0, stream>>>(p);
    }
  } else {
    const dim3 grid(groups | 1, p.h_kv, p.batch);
    if (p.mx) {
      if (p.smooth) decode_kernel<true, true, false><<<grid, block, 0, stream>>>(p);
      else decode_kernel<false, true, false><<<grid, block, 0, stream>>>(p);
    } else {
      if (p.smooth) decode_kernel<true, false, false><<<grid, block, 0, stream>>>(p);
      else decode_kernel<false, false, false><<<grid, block, 0, stream>>>(p);
    }
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (p.max_partitions <= 8) merge_kernel<8><<<dim3(p.h_q, p.batch), dim3(64), 0, stream>>>(p);
  else if (p.max_partitions <= 16) merge_kernel<16><<<dim3(p.h_q, p.batch), dim3(64), 0, stream>>>(p);
  else if (p.max_partitions <= kMergeChunk) merge_kernel<kMergeChunk><<<dim3(p.h_q, p.batch), dim3(64), 0, stream>>>(p);
  else if (p.h_q * (int64_t)p.batch <= kSplitMergeHeads) merge_wide_kernel<16, 1><<<dim3(2 * p.h_q, p.batch), dim3(1024), 0, stream>>>(p);
  else merge_wide_kernel<8, 2><<<dim3(p.h_q, p.batch), dim3(512), 0, stream>>>(p);
  return hipGetLastError();
}

}  // namespace mpfa
