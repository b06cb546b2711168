// quantize.hip -- Algorithm 1 stage one on gfx950: sequence statistics (Eq. 7),
// centering, NVFP4 quantization of Q and K (Sec. 2.1 Eq. 1), FP8 V, and the
// Delta_S compensation vector (Eq. 9) written into the paged side cache
// (Sec. 6).  Memory-bound; every rounding follows the ABI contract exactly so
// that codes are bit-reproducible.
#include "mpfa_device.h"
#include "mpfa_internal.h"

#pragma clang fp contract(off)

namespace mpfa {

// ---------------------------------------------------------------------------
// Sequence statistics (Eq. 7) and tensor scales.
//
// stats_partial_kernel: one workgroup per (sequence, 128-token block).  Lane
// groups of 16 own one head row (8 channels per lane, 16-byte loads); each lane
// sums its channels over the block's tokens in token order (FP32) and keeps
// their max and min.  The amax of the centered values needs no second read:
// x -> fl(x - mean) is monotone, so max_t |fl(x_t - mean)| is reached at the
// channel's max or min.  A one-block sequence is finished in place; otherwise
// the block partials (sum, max, min) are parked in the q_codes rows of the
// sequence, which quantize_kernel overwrites later on the same stream.
// stats_final_kernel adds the block partials in block order and finishes.
// ---------------------------------------------------------------------------
constexpr int kStatUnits = 4;   // (head, 8-channel) units per thread and pass

struct StatsShape {
  int hs;                 // heads with statistics: h_q, plus h_kv with stats_k
  bool want_sum, want_amax;
};

__device__ __forceinline__ StatsShape stats_shape(const QuantParams& p) {
  StatsShape s;
  s.hs = p.h_q + (p.stats_k ? p.h_kv : 0);
  s.want_sum = p.compute_stats && p.smooth;
  s.want_amax = !(p.tscale_unit || p.mx);
  return s;
}

// block partials of block blk: float [3][hs][128] (sum, max, min).  Block i <
// nblk-1 uses the q_codes rows of its own 128 tokens; the last block uses the
// rows of block nblk-2 after that block's partials (2 * 1536 * hs bytes fit in
// the 8192 * h_q bytes of 128 token rows since hs <= 2 h_q).
__device__ __forceinline__ float* partial_ptr(const QuantParams& p, int64_t t0, int nblk, int blk, int hs) {
  const bool last = blk == nblk - 1;
  const int64_t r = last ? nblk - 2 : blk;
  uint8_t* base = p.q_codes + (t0 + r * 128) * (int64_t)p.h_q * 64;
  if (last) base += (int64_t)3 * hs * kD * 4;
  return reinterpret_cast<float*>(base);
}

// the per-head arrival counters (uint32 [hs]) and slice amaxes (float [hs][4])
__device__ __forceinline__ uint8_t* fin_scratch(const QuantParams& p, int64_t t0, int hs) {
  return p.q_codes + t0 * (int64_t)p.h_q * 64 + (int64_t)6 * hs * kD * 4;
}

// mean of head hh (0..h_q-1: Q, then K) and its BF16 output row
__device__ __forceinline__ uint16_t* mean_row(const QuantParams& p, int b, int hh) {
  return hh < p.h_q ? p.q_mean + ((int64_t)b * p.h_q + hh) * kD
                    : p.k_mean + ((int64_t)b * p.h_kv + (hh - p.h_q)) * kD;
}

__device__ __forceinline__ void write_tscale(const QuantParams& p, int b, int hh, float amax) {
  const float ts = (p.tscale_unit || p.mx) ? 1.0f : tensor_scale(amax);
  if (hh < p.h_q) p.q_tscale[b * p.h_q + hh] = ts;
  else p.k_tscale[b * p.h_kv + (hh - p.h_q)] = ts;
}

// Rows read once by the workgroup, past the caches' ordinary replacement: 131072
// tokens 40:8, 864 -> 812 us of the whole call (1.6 GB read by this kernel, 326 us
// before); nothing lost where the inputs fit in the last-level cache (9000 tokens).
__device__ __forceinline__ u32x4 load_stream(const u32x4* src) { return __builtin_nontemporal_load(src); }

__global__ __launch_bounds__(256) void stats_partial_kernel(QuantParams p) {
  const int b = blockIdx.y, blk = blockIdx.x;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int nblk = (n + 127) >> 7;
  if (blk >= nblk) return;
  const StatsShape ss = stats_shape(p);
  const int tb = blk * 128, te = min(n, tb + 128);
  const int nunits = ss.hs * 16;
  if (nblk >= 2 && blk == 0)   // arrival counters of stats_final_kernel
    for (int i = threadIdx.x; i < ss.hs; i += blockDim.x) reinterpret_cast<uint32_t*>(fin_scratch(p, t0, ss.hs))[i] = 0u;
  for (int u0 = 0; u0 < nunits; u0 += 256 * kStatUnits) {
    const u32x4* src[kStatUnits];
    int64_t stride[kStatUnits];   // in 16-byte words per token
    bool act[kStatUnits];
    float sm[kStatUnits][8], mx[kStatUnits][8], mn[kStatUnits][8];
#pragma unroll
    for (int k = 0; k < kStatUnits; ++k) {
      const int u = u0 + k * 256 + threadIdx.x;
      act[k] = u < nunits;
      const int hh = act[k] ? u >> 4 : 0, oct = u & 15;
      const bool isq = hh < p.h_q;
      const int H = isq ? p.h_q : p.h_kv;
      const int h = isq ? hh : hh - p.h_q;
      const uint16_t* base = isq ? p.q : p.k;
      src[k] = reinterpret_cast<const u32x4*>(base + ((t0 + tb) * H + h) * kD + oct * 8);
      stride[k] = (int64_t)H * (kD / 8);
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        sm[k][e] = 0.0f;
        mx[k][e] = -INFINITY;
        mn[k][e] = INFINITY;
      }
    }
    for (int t = tb; t < te; t += 4) {
      u32x4 w[4][kStatUnits];
#pragma unroll
      for (int j = 0; j < 4; ++j)
#pragma unroll
        for (int k = 0; k < kStatUnits; ++k)
          w[j][k] = (act[k] && t + j < te) ? load_stream(src[k] + (int64_t)(t - tb + j) * stride[k]) : u32x4{0, 0, 0, 0};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        if (t + j < te) {
#pragma unroll
          for (int k = 0; k < kStatUnits; ++k) {
            const uint32_t wd[4] = {w[j][k].x, w[j][k].y, w[j][k].z, w[j][k].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = __uint_as_float((e & 1) ? (wd[e >> 1] & 0xFFFF0000u) : (wd[e >> 1] << 16));
              sm[k][e] += x;
              mx[k][e] = fmaxf(mx[k][e], x);
              mn[k][e] = fminf(mn[k][e], x);
            }
          }
        }
      }
    }
#pragma unroll
    for (int k = 0; k < kStatUnits; ++k) {
      const int u = u0 + k * 256 + threadIdx.x;
      const int hh = u >> 4, oct = u & 15;
      if (nblk == 1) {
        // one block: its partial sum is the total (0 + partial, exact)
        float amax = 0.0f;
        if (act[k]) {
          uint16_t* mrow = mean_row(p, b, hh) + oct * 8;
          float mu[8];
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            uint16_t m = 0;
            if (ss.want_sum) m = bf16_rne(__fdiv_rn(sm[k][e], (float)n));
            else if (!p.compute_stats && p.smooth) m = mrow[e];
            if (p.compute_stats) mrow[e] = m;
            mu[e] = bf16_to_f32(m);
          }
#pragma unroll
          for (int e = 0; e < 8; ++e)
            amax = fmaxf(amax, fmaxf(__builtin_fabsf(mx[k][e] - mu[e]), __builtin_fabsf(mn[k][e] - mu[e])));
        }
        // 16 lanes of one head row (units of one head are 16 consecutive lanes)
        for (int off = 1; off < 16; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
        if (act[k] && oct == 0) write_tscale(p, b, hh, amax);
      } else if (act[k]) {
        float* part = partial_ptr(p, t0, nblk, blk, ss.hs) + hh * kD + oct * 8;
#pragma unroll
        for (int e = 0; e < 8; e += 4) {
          *reinterpret_cast<float4*>(part + e) = make_float4(sm[k][e], sm[k][e + 1], sm[k][e + 2], sm[k][e + 3]);
          *reinterpret_cast<float4*>(part + ss.hs * kD + e) =
              make_float4(mx[k][e], mx[k][e + 1], mx[k][e + 2], mx[k][e + 3]);
          *reinterpret_cast<float4*>(part + 2 * ss.hs * kD + e) =
              make_float4(mn[k][e], mn[k][e + 1], mn[k][e + 2], mn[k][e + 3]);
        }
      }
    }
  }
}

// Sequence and block of the idx-th block of 2^SHIFT tokens of the call; false past the
// last.  For the grids of one workgroup per block that the call has: those of (blocks of
// the longest sequence) x (sequences) are mostly empty in a batch of one long prompt and
// many short ones, and an empty workgroup costs about 0.3 ns of the chip.
template <int SHIFT>
__device__ __forceinline__ bool packed_block(const QuantParams& p, int idx, int& b, int& blk) {
  const int lane = threadIdx.x & 63;
  for (int b0 = 0; b0 < p.batch; b0 += 64) {
    const int i = b0 + lane;
    const int n = i < p.batch ? (p.cu_seqlens[i + 1] - p.cu_seqlens[i] + (1 << SHIFT) - 1) >> SHIFT : 0;
    int incl = n;
    for (int d = 1; d < 64; d <<= 1) {
      const int up = __shfl_up(incl, d);
      if (lane >= d) incl += up;
    }
    const int total = __builtin_amdgcn_readlane(incl, 63);
    if (idx < total) {
      const int at = __ffsll((unsigned long long)__ballot(incl > idx)) - 1;
      b = b0 + at;
      blk = idx - (__builtin_amdgcn_readlane(incl, at) - __builtin_amdgcn_readlane(n, at));
      return true;
    }
    idx -= total;
  }
  return false;
}

// The same for few blocks: one wave per (head, block, sequence), two channels
// per lane and 32 tokens in flight.  A block is a serial walk over its tokens,
// so with too few workgroups to fill the chip its latency counts: 16 lanes a
// head with 8 channels each spend 20 us on the 4096 vector operations and 8
// round trips of a block, this shape 2 channels' 1024 and 4 (see launch_quantize
// for the line between the two).  Per channel the tokens add in the same order.
template <bool PACKED>
__global__ __launch_bounds__(64) void stats_partial_wave_kernel(QuantParams p) {
  constexpr int kAhead = 32;
  const int hh = blockIdx.x, lane = threadIdx.x;
  int blk = blockIdx.y, b = blockIdx.z;
  if (PACKED && !packed_block<7>(p, blockIdx.y, b, blk)) return;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int nblk = (n + 127) >> 7;
  if (blk >= nblk) return;
  const StatsShape ss = stats_shape(p);
  const int tb = blk * 128, cnt = min(n - tb, 128);
  if (nblk >= 2 && blk == 0 && lane == 0)   // arrival counter of stats_final_kernel
    reinterpret_cast<uint32_t*>(fin_scratch(p, t0, ss.hs))[hh] = 0u;
  const bool isq = hh < p.h_q;
  const int H = isq ? p.h_q : p.h_kv;
  const uint32_t* src =
      reinterpret_cast<const uint32_t*>((isq ? p.q : p.k) + ((t0 + tb) * H + (isq ? hh : hh - p.h_q)) * kD) + lane;
  const int64_t stride = (int64_t)H * (kD / 2);
  float s0 = 0.0f, s1 = 0.0f, x0 = -INFINITY, x1 = -INFINITY, m0 = INFINITY, m1 = INFINITY;
  for (int t = 0; t < cnt; t += kAhead) {
    uint32_t w[kAhead];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) w[j] = src[(int64_t)min(t + j, cnt - 1) * stride];
#pragma unroll
    for (int j = 0; j < kAhead; ++j) {
      const float a = __uint_as_float(w[j] << 16), c = __uint_as_float(w[j] & 0xFFFF0000u);
      if (t + j < cnt) {
        s0 += a;
        s1 += c;
      }
      // past the block's end the last token repeats: no change to max and min
      x0 = fmaxf(x0, a);
      x1 = fmaxf(x1, c);
      m0 = fminf(m0, a);
      m1 = fminf(m1, c);
    }
  }
  if (nblk == 1) {
    // one block: its partial sum is the total (0 + partial, exact)
    uint16_t* mrow = mean_row(p, b, hh) + 2 * lane;
    uint16_t v0 = 0, v1 = 0;
    if (ss.want_sum) {
      v0 = bf16_rne(__fdiv_rn(s0, (float)n));
      v1 = bf16_rne(__fdiv_rn(s1, (float)n));
    } else if (!p.compute_stats && p.smooth) {
      v0 = mrow[0];
      v1 = mrow[1];
    }
    if (p.compute_stats) {
      mrow[0] = v0;
      mrow[1] = v1;
    }
    const float u0 = bf16_to_f32(v0), u1 = bf16_to_f32(v1);
    float amax = fmaxf(fmaxf(__builtin_fabsf(x0 - u0), __builtin_fabsf(m0 - u0)),
                       fmaxf(__builtin_fabsf(x1 - u1), __builtin_fabsf(m1 - u1)));
    for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (lane == 0) write_tscale(p, b, hh, amax);
  } else {
    float* part = partial_ptr(p, t0, nblk, blk, ss.hs) + hh * kD + 2 * lane;
    *reinterpret_cast<float2*>(part) = make_float2(s0, s1);
    *reinterpret_cast<float2*>(part + ss.hs * kD) = make_float2(x0, x1);
    *reinterpret_cast<float2*>(part + 2 * ss.hs * kD) = make_float2(m0, m1);
  }
}

// stats_final_kernel: one workgroup of 256 threads per (head, 32-channel
// slice, sequence), so that the partials of one head are read by four compute
// units.  The slice's partials arrive in LDS 256 blocks at a time (coalesced
// 128-byte rows, the next chunk in flight while the current one is added);
// 32 lanes of wave 0 own one channel each and add its partials strictly in block
// order, then FP32 divide and BF16 rounding; waves 1 and 2 take the maxima and
// minima beside them (one wave for the three walked the chunk three times as
// long: 131072 tokens 40:8 34.5 -> 27 us, 75 MB of partials).  The tensor scale needs the amax
// of the whole head: each slice stores its own and counts itself in the
// head's arrival counter; the fourth arrival takes the maximum and writes the
// scale.  Counters and slice amaxes live in the spare bytes of the first
// block's q_codes rows (zeroed by stats_partial_kernel), which the quantizer
// overwrites later.  Sequences whose statistics need no partials (frozen
// statistics, empty or one-block sequences) are handled by slice 0 alone.
constexpr int kFinThreads = 256;
constexpr int kFinSlice = 32;                                        // channels per workgroup
constexpr int kFinChunk = 256;                                       // blocks per chunk
constexpr int kFinLoads = 3 * kFinChunk * (kFinSlice / 4) / kFinThreads;   // float4 loads per thread and chunk

__device__ __forceinline__ void fin_load(const QuantParams& p, int64_t t0, int nblk, int hs, int hh, int c0,
                                         int blk0, float4 (&r)[kFinLoads]) {
#pragma unroll
  for (int i = 0; i < kFinLoads; ++i) {
    const int idx = i * kFinThreads + (int)threadIdx.x;
    const int arr = idx / (kFinChunk * (kFinSlice / 4)), rem = idx % (kFinChunk * (kFinSlice / 4));
    const int blk = blk0 + rem / (kFinSlice / 4), q4 = rem % (kFinSlice / 4);
    r[i] = make_float4(0.f, 0.f, 0.f, 0.f);
    if (blk < nblk)
      r[i] = *reinterpret_cast<const float4*>(partial_ptr(p, t0, nblk, blk, hs) + (int64_t)arr * hs * kD + hh * kD +
                                              c0 + 4 * q4);
  }
}

__global__ __launch_bounds__(kFinThreads) void stats_final_kernel(QuantParams p) {
  __shared__ float4 chunk[3 * kFinChunk * (kFinSlice / 4)];   // [sum, max, min][block][channel / 4]: 96 KB
  const int hh = blockIdx.x >> 2, slice = blockIdx.x & 3, b = blockIdx.y, t = threadIdx.x;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int nblk = (n + 127) >> 7;
  if (p.need_partials && nblk == 1) return;   // finished by stats_partial_kernel
  const StatsShape ss = stats_shape(p);
  const bool have = p.need_partials && nblk >= 2;
  if (!have) {
    // no partials: the (frozen or zero) means and a zero amax, by slice 0
    if (slice != 0) return;
    if (t < kD) {
      uint16_t* mrow = mean_row(p, b, hh);
      uint16_t m = 0;
      if (!p.compute_stats && p.smooth) m = mrow[t];
      if (p.compute_stats) mrow[t] = m;
    }
    if (t == 0) write_tscale(p, b, hh, 0.0f);
    return;
  }
  const int c0 = slice * kFinSlice, c = c0 + t;
  float tot = 0.0f, mx = -INFINITY, mn = INFINITY;
  {
    const int arr = t >> 6, lane = t & 63;   // waves 0, 1, 2: sum, max, min
    float4 r[kFinLoads];
    fin_load(p, t0, nblk, ss.hs, hh, c0, 0, r);
    for (int blk0 = 0; blk0 < nblk; blk0 += kFinChunk) {
#pragma unroll
      for (int i = 0; i < kFinLoads; ++i) chunk[i * kFinThreads + t] = r[i];
      __syncthreads();
      if (blk0 + kFinChunk < nblk) fin_load(p, t0, nblk, ss.hs, hh, c0, blk0 + kFinChunk, r);
      if (lane < kFinSlice) {
        const float* cs = reinterpret_cast<const float*>(chunk) + arr * kFinChunk * kFinSlice + lane;
        const int nb = min(kFinChunk, nblk - blk0);
        // unrolled so that the LDS reads run ahead of the dependent operations
        if (arr == 0) {
#pragma unroll 16
          for (int j = 0; j < nb; ++j) tot += cs[j * kFinSlice];
        } else if (arr == 1) {
#pragma unroll 16
          for (int j = 0; j < nb; ++j) mx = fmaxf(mx, cs[j * kFinSlice]);
        } else if (arr == 2) {
#pragma unroll 16
          for (int j = 0; j < nb; ++j) mn = fminf(mn, cs[j * kFinSlice]);
        }
      }
      __syncthreads();
    }
    float* ends = reinterpret_cast<float*>(chunk);   // [max, min][channel]
    if (lane < kFinSlice && arr == 1) ends[lane] = mx;
    if (lane < kFinSlice && arr == 2) ends[kFinSlice + lane] = mn;
    __syncthreads();
    if (t < kFinSlice) {
      mx = ends[t];
      mn = ends[kFinSlice + t];
    }
  }
  if (t < 64) {   // one wave: the slice's 32 channels
    float amax = 0.0f;
    if (t < kFinSlice) {
      uint16_t* mrow = mean_row(p, b, hh);
      uint16_t m = 0;
      if (ss.want_sum) m = bf16_rne(__fdiv_rn(tot, (float)n));
      else if (!p.compute_stats && p.smooth) m = mrow[c];
      if (p.compute_stats) mrow[c] = m;
      const float mu = bf16_to_f32(m);
      amax = fmaxf(__builtin_fabsf(mx - mu), __builtin_fabsf(mn - mu));
    }
    for (int off = 16; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (t == 0) {
      uint8_t* scr = fin_scratch(p, t0, ss.hs);
      uint32_t* cnt = reinterpret_cast<uint32_t*>(scr) + hh;
      float* samax = reinterpret_cast<float*>(scr + ss.hs * 4) + hh * 4;
      samax[slice] = amax;
      // release: the slice amax is visible before the arrival is counted
      __builtin_amdgcn_fence(__ATOMIC_RELEASE, "agent");
      if (atomicAdd(cnt, 1u) == 3u) {   // the head's last slice
        __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "agent");
        const float a = fmaxf(fmaxf(samax[0], samax[1]), fmaxf(samax[2], samax[3]));
        write_tscale(p, b, hh, a);
      }
    }
  }
}

// The same for sequences of few blocks: one workgroup of 128 threads per (head,
// sequence), one channel per thread, its partials read straight from memory
// (kShortBatch blocks in flight) and added in block order.  No LDS chunk, no
// arrival counters: with at most kShortBlocks blocks the reads are a few round
// trips, where the kernel above spends its time on whole 256-block chunks.
constexpr int kShortBlocks = 64;
constexpr int kShortBatch = 32;

__global__ __launch_bounds__(kD) void stats_final_short_kernel(QuantParams p) {
  __shared__ float wave_amax[2];
  const int hh = blockIdx.x, b = blockIdx.y, c = threadIdx.x;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int nblk = (n + 127) >> 7;
  if (p.need_partials && nblk == 1) return;   // finished by stats_partial_kernel
  const StatsShape ss = stats_shape(p);
  const bool have = p.need_partials && nblk >= 2;
  float tot = 0.0f, mx = -INFINITY, mn = INFINITY;
  if (have) {
    for (int blk0 = 0; blk0 < nblk; blk0 += kShortBatch) {
      float s[kShortBatch], x[kShortBatch], m[kShortBatch];
#pragma unroll
      for (int j = 0; j < kShortBatch; ++j) {
        const float* part = partial_ptr(p, t0, nblk, min(blk0 + j, nblk - 1), ss.hs) + hh * kD + c;
        s[j] = part[0];
        x[j] = part[ss.hs * kD];
        m[j] = part[2 * ss.hs * kD];
      }
#pragma unroll
      for (int j = 0; j < kShortBatch; ++j)
        if (blk0 + j < nblk) {
          tot += s[j];
          mx = fmaxf(mx, x[j]);
          mn = fminf(mn, m[j]);
        }
    }
  }
  uint16_t* mrow = mean_row(p, b, hh);
  uint16_t m = 0;
  if (have && ss.want_sum) m = bf16_rne(__fdiv_rn(tot, (float)n));
  else if (!p.compute_stats && p.smooth) m = mrow[c];
  if (p.compute_stats) mrow[c] = m;
  const float mu = bf16_to_f32(m);
  float amax = have ? fmaxf(__builtin_fabsf(mx - mu), __builtin_fabsf(mn - mu)) : 0.0f;
  for (int off = 32; off >= 1; off >>= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
  if ((c & 63) == 0) wave_amax[c >> 6] = amax;
  __syncthreads();
  if (c == 0) write_tscale(p, b, hh, fmaxf(wave_amax[0], wave_amax[1]));
}

// NVFP4 quantization (Sec. 2.1 Eq. 1) of a 16-channel group of centered FP32
// values, in two steps so that the group may be spread over lanes: the scale
// from the group amax, then the codes of 8 channels at a time.
// rcp_sd[c] = RN(1 / e4m3_value(c)) for the positive E4M3 codes; with a
// power-of-two t, RN(1 / (t * sd)) = rcp_sd / t and RN(1 / (6 t)) = RN(1/6) / t.
struct Nv4Scale {
  uint32_t code;   // E4M3 scale byte
  float scale;     // t * sd (exact)
  float r;         // RN(1 / scale)
  int mode;        // 0: all codes are signed zeros; 1: product quotients; 2: IEEE division
};

__device__ __forceinline__ Nv4Scale nvfp4_scale(float a, float t, const float* rcp_sd) {
  const int kt = ilog2f(t);
  float q = div_by_scale(a, 6.0f * t, __builtin_ldexpf(kRcp6, -kt));   // RN(amax / (6 t))
  if (!(q < 0x1p100f)) q = 0x1p100f;   // an overflowing quotient saturates like +inf would
  Nv4Scale s;
  s.code = fp8_sat_pair(0u, q, 0.0f, false) & 0xFFu;                   // E4M3_RNE_sat
  const float sd = e4m3_value(s.code);
  s.scale = t * sd;   // exact: t is a power of two
  s.r = __builtin_ldexpf(rcp_sd[s.code], -kt);
  // quotients near the FP32 range (a frozen K tensor scale far below a later
  // token) take the IEEE division and the saturating encoder
  s.mode = sd == 0.0f ? 0 : (a * s.r < 0x1p100f ? 1 : 2);
  return s;
}

// Codes of 8 channels (element i in nibble i) under the group scale s.
__device__ __forceinline__ uint32_t nvfp4_encode8(const float* x, const Nv4Scale& s) {
  uint32_t w = 0;
  if (s.mode == 0) {
#pragma unroll
    for (int i = 0; i < 8; ++i) w |= ((__float_as_uint(x[i]) >> 28) & 8u) << (4 * i);
  } else if (s.mode == 1) {
#pragma unroll
    for (int j = 0; j < 4; ++j)
      w = fp4_pair(w, div_by_scale(x[2 * j], s.scale, s.r), div_by_scale(x[2 * j + 1], s.scale, s.r), 1.0f, j);
  } else {
#pragma unroll
    for (int i = 0; i < 8; ++i) w |= e2m1_rne_sat(__fdiv_rn(x[i], s.scale)) << (4 * i);
  }
  return w;
}

// One whole group: 8 code bytes (as a 64-bit word, low nibble first) and the
// scale byte.
__device__ __forceinline__ uint64_t nvfp4_group(const float* xc, float t, const float* rcp_sd,
                                                uint32_t* scale_code) {
  float a = 0.0f;
#pragma unroll
  for (int i = 0; i < 16; ++i) a = fmaxf(a, __builtin_fabsf(xc[i]));
  const Nv4Scale s = nvfp4_scale(a, t, rcp_sd);
  *scale_code = s.code;
  return (uint64_t)nvfp4_encode8(xc, s) | ((uint64_t)nvfp4_encode8(xc + 8, s) << 32);
}

// MXFP4 quantization of one 32-channel block held as 32 centered FP32 values:
// X = 2^e, e = floor(log2 amax) - 2 clamped to [-127, 127] (-127 for an
// all-zero block); codes E2M1_RNE_sat(x / X).  Returns 16 code bytes (element
// 2j in the low nibble of byte j).
__device__ __forceinline__ u32x4 mxfp4_group(const float* xc, uint32_t* scale_code) {
  float a = 0.0f;
#pragma unroll
  for (int i = 0; i < 32; ++i) a = fmaxf(a, __builtin_fabsf(xc[i]));
  int e = -127;
  if (a > 0.0f) e = max(-127, min(127, ilog2f(a) - 2));
  *scale_code = (uint32_t)(e + 127);
  // e = -127 only for an all-zero block, whose codes keep just the signs under
  // any scale; 2^-126 keeps the scale operand a normal number
  const float pw = __builtin_ldexpf(1.0f, max(e, -126));
  u32x4 w = {0u, 0u, 0u, 0u};
#pragma unroll
  for (int q = 0; q < 4; ++q)
#pragma unroll
    for (int j = 0; j < 4; ++j) w[q] = fp4_pair(w[q], xc[8 * q + 2 * j], xc[8 * q + 2 * j + 1], pw, j);
  return w;
}

// ---------------------------------------------------------------------------
// Quantization and cache write.  One workgroup (256 threads) per (sequence,
// 64-token chunk).
//   Q: group u of the chunk's rows is at u * group_elems in the packed input,
//   so consecutive lanes read and write consecutive groups; each lane has the
//   loads of several groups in flight before it quantizes them.
//   K and Delta_S: one lane per (token, KV head) row, the lanes of a wave on
//   consecutive tokens of one head.  The lane reads its row once; each group's
//   centered values feed both the quantizer and the Delta_S chains, so K is
//   read from HBM once.  Codes, scale rows and Delta_S entries of consecutive
//   tokens are consecutive in the cache pages: the stores are contiguous.
//   V: when the chunk's 64 tokens fill one cache page in order (the common
//   prefill case), each lane converts two channels of all 64 tokens and writes
//   their two channel-major 64-byte page rows whole; otherwise one byte per
//   (token, channel).
// ---------------------------------------------------------------------------
constexpr int kChunk = 64;
constexpr int kMeanStride = kD * 2 + 16;   // bytes per BF16 mean row in LDS (padded: rows on distinct banks)

// 8 centered values (x - mean, FP32) of the BF16 words v and m.
__device__ __forceinline__ void center8(const uint4 v, const uint4 m, float* xc) {
  const uint32_t vv[4] = {v.x, v.y, v.z, v.w}, mm[4] = {m.x, m.y, m.z, m.w};
#pragma unroll
  for (int e = 0; e < 8; ++e) {
    const bool lo = (e & 1) == 0;
    const float xv = __uint_as_float(lo ? (vv[e >> 1] << 16) : (vv[e >> 1] & 0xFFFF0000u));
    const float mv = __uint_as_float(lo ? (mm[e >> 1] << 16) : (mm[e >> 1] & 0xFFFF0000u));
    xc[e] = xv - mv;
  }
}

// Max over the lanes of one quantization group (lane pairs, or quads for
// MXFP4): DPP swaps inside each quad of lanes.
template <bool MX>
__device__ __forceinline__ float group_max(float a) {
  a = fmaxf(a, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0xB1, 0xF, 0xF, false)));  // lane ^ 1
  if (MX) a = fmaxf(a, __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(a), 0x4E, 0xF, 0xF, false)));  // lane ^ 2
  return a;
}

// Codes and scale of one lane's 8 centered channels (c8: which of the row's 16
// lanes): every lane of a group derives the group's scale.
template <bool MX>
__device__ __forceinline__ uint32_t encode_lane(const float* xc, float t, const float* rcp_sd, uint32_t* scale_code) {
  float a = 0.0f;
#pragma unroll
  for (int i = 0; i < 8; ++i) a = fmaxf(a, __builtin_fabsf(xc[i]));
  a = group_max<MX>(a);
  if (MX) {
    int e = -127;
    if (a > 0.0f) e = max(-127, min(127, ilog2f(a) - 2));
    *scale_code = (uint32_t)(e + 127);
    const float pw = __builtin_ldexpf(1.0f, max(e, -126));
    uint32_t w = 0u;
#pragma unroll
    for (int j = 0; j < 4; ++j) w = fp4_pair(w, xc[2 * j], xc[2 * j + 1], pw, j);
    return w;
  }
  const Nv4Scale s = nvfp4_scale(a, t, rcp_sd);
  *scale_code = s.code;
  return nvfp4_encode8(xc, s);
}

// Q rows: one lane per 8 channels (16 bytes) of a row, so a wave reads and
// writes 4 whole rows; the lanes of a group (2 for NVFP4, 4 for MXFP4) share
// its amax.  Each lane has U units in flight before it quantizes them.
template <bool MX>
__device__ __forceinline__ void quant_q_rows(const QuantParams& p, const uint8_t* mean_base, const float* tscale,
                                             int64_t tok0, int cnt, const float* rcp_sd) {
  constexpr int L = MX ? 4 : 2;          // lanes per group
  constexpr int U = 8;                   // units per lane in flight
  const int H = p.h_q;
  const int nun = cnt * H * 16;          // a multiple of 16: the lanes of a group act together
  const uint4* src = reinterpret_cast<const uint4*>(p.q + (tok0 * H) * kD);
  for (int u0 = threadIdx.x; u0 < nun; u0 += 256 * U) {
    uint4 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      v[k] = src[min(u0 + 256 * k, nun - 1)];   // past the end: not stored
      // the loads issue in unit order, all before the first unit is used
      __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int u = u0 + 256 * k;
      if (u < nun) {
        const int r = u >> 4, c8 = u & 15, h = r % H, g = c8 / L;
        float xc[8];
        center8(v[k], *reinterpret_cast<const uint4*>(mean_base + h * kMeanStride + c8 * 16), xc);
        const int64_t row = tok0 * H + r;
        uint32_t sc;
        const uint32_t w = encode_lane<MX>(xc, MX ? 1.0f : tscale[h], rcp_sd, &sc);
        *reinterpret_cast<uint32_t*>(p.q_codes + row * 64 + c8 * 4) = w;
        if (c8 % L == 0) {
          p.q_scales[row * 8 + g] = (uint8_t)sc;
          if (MX) p.q_scales[row * 8 + 4 + g] = 0;
        }
      }
    }
  }
}

// codes[q] = w for a runtime q (selects, no indexed register access)
__device__ __forceinline__ void codes_put(u32x4 (&codes)[4], int q, u32x4 w) {
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (i == q) codes[i] = w;
}

// One K row: NVFP4 / MXFP4 codes and scale row into the cache, and
// Delta_S[h] = BF16(sum_c Qbar[h][c] * K_c[c]) as an FMA chain over c from +0
// (Eq. 9) for the query heads of the KV head's group, eight at a time.  The
// row is read a quarter (32 channels) at a time, the next quarter's loads in
// flight while the current one is used.
template <bool MX>
__device__ __forceinline__ void quant_k_rows(const QuantParams& p, const uint8_t* kmean_s, const uint8_t* qmean_s,
                                             const float* tscale, int64_t tok0, int cnt, const float* rcp_sd) {
  const int H = p.h_kv, grp = p.h_q / p.h_kv;
  for (int r = threadIdx.x; r < kChunk * H; r += 256) {
    const int i = r % kChunk, hk = r / kChunk;
    if (i >= cnt) continue;
    const uint4* kr = reinterpret_cast<const uint4*>(p.k + ((tok0 + i) * H + hk) * kD);
    const uint4* km = reinterpret_cast<const uint4*>(kmean_s + hk * kMeanStride);
    const int64_t slot = p.slot_mapping[tok0 + i];
    const int64_t crow = ((slot / kPage) * H + hk) * kPage + slot % kPage;
    const float t = tscale[hk];
    uint32_t scw[2] = {0u, 0u};
    u32x4 codes[4];   // the row's 64 code bytes, stored whole (partial-line stores cost write-backs)
    // the first pass over the row also quantizes it
    for (int j0 = 0; j0 == 0 || (p.smooth && j0 < grp); j0 += 8) {
      const int nj = p.smooth ? min(8, grp - j0) : 0;
      const uint8_t* qm = qmean_s + (hk * grp + j0) * kMeanStride;
      float d[8];
#pragma unroll
      for (int j = 0; j < 8; ++j) d[j] = 0.0f;
      uint4 nxt[4];
#pragma unroll
      for (int w = 0; w < 4; ++w) nxt[w] = kr[w];
#pragma unroll 1
      for (int qt = 0; qt < 4; ++qt) {   // channels 32 qt .. 32 qt + 31
        uint4 v[4];
#pragma unroll
        for (int w = 0; w < 4; ++w) v[w] = nxt[w];
        if (qt < 3) {
#pragma unroll
          for (int w = 0; w < 4; ++w) nxt[w] = kr[4 * (qt + 1) + w];
        }
        float xc[32];
#pragma unroll
        for (int w = 0; w < 4; ++w) center8(v[w], km[4 * qt + w], xc + 8 * w);
        if (j0 == 0) {
          uint32_t sc;
          if (MX) {
            const u32x4 cw = mxfp4_group(xc, &sc);
            codes_put(codes, qt, cw);
            scw[0] |= sc << (8 * qt);
          } else {
            uint32_t sc1;
            const uint64_t c0 = nvfp4_group(xc, t, rcp_sd, &sc);
            const uint64_t c1 = nvfp4_group(xc + 16, t, rcp_sd, &sc1);
            codes_put(codes, qt, (u32x4){(uint32_t)c0, (uint32_t)(c0 >> 32), (uint32_t)c1, (uint32_t)(c1 >> 32)});
            scw[qt >> 1] |= (sc | (sc1 << 8)) << (16 * (qt & 1));
          }
        }
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          if (j < nj) {
#pragma unroll
            for (int w = 0; w < 4; ++w) {
              const uint4 qv = *reinterpret_cast<const uint4*>(qm + j * kMeanStride + (4 * qt + w) * 16);
              const uint32_t q4[4] = {qv.x, qv.y, qv.z, qv.w};
#pragma unroll
              for (int e = 0; e < 8; ++e) {
                const float qx = __uint_as_float((e & 1) == 0 ? (q4[e >> 1] << 16) : (q4[e >> 1] & 0xFFFF0000u));
                d[j] = __builtin_fmaf(qx, xc[8 * w + e], d[j]);
              }
            }
          }
        }
      }
      if (j0 == 0) {
        u32x4* co = reinterpret_cast<u32x4*>(p.k_codes + crow * 64);
#pragma unroll
        for (int q = 0; q < 4; ++q) co[q] = codes[q];
        *reinterpret_cast<uint2*>(p.k_scales + crow * 8) = make_uint2(scw[0], scw[1]);
      }
      uint16_t* dsrow = p.ds + ((slot / kPage) * p.h_q + hk * grp + j0) * kPage + slot % kPage;
#pragma unroll
      for (int j = 0; j < 8; ++j)
        if (j < nj) dsrow[(int64_t)j * kPage] = bf16_rne(d[j]);
    }
  }
}

// V of 16 tokens and two adjacent channels, w[j] both values of token j: FP8 bytes of the
// channel rows.
__device__ __forceinline__ void v_fp8_16(const uint32_t (&w)[16], u32x4& r0, u32x4& r1) {
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    const uint32_t* wq = w + 4 * q;
    uint32_t a = fp8_sat_pair(0u, __uint_as_float(wq[0] << 16), __uint_as_float(wq[1] << 16), false);
    a = fp8_sat_pair(a, __uint_as_float(wq[2] << 16), __uint_as_float(wq[3] << 16), true);
    uint32_t c = fp8_sat_pair(0u, __uint_as_float(wq[0] & 0xFFFF0000u), __uint_as_float(wq[1] & 0xFFFF0000u), false);
    c = fp8_sat_pair(c, __uint_as_float(wq[2] & 0xFFFF0000u), __uint_as_float(wq[3] & 0xFFFF0000u), true);
    r0[q] = a;
    r1[q] = c;
  }
}

// The characterization copies of the same tokens (qq .. qq + 15 of the page) in channel
// rows crow, crow + 1: BF16 rows (page_run: all 64 tokens present), or an NVFP4 group.
__device__ __forceinline__ void v_aux_16(const QuantParams& p, const uint32_t (&w)[16], int64_t crow, int qq,
                                         bool page_run, const float* rcp_sd) {
  if (p.pv == 1 && page_run) {   // 16 keys of each channel, 32 bytes
    uint32_t b0[8], b1[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      b0[j] = (w[2 * j] & 0xFFFFu) | (w[2 * j + 1] << 16);
      b1[j] = (w[2 * j] >> 16) | (w[2 * j + 1] & 0xFFFF0000u);
    }
    uint16_t* a16 = reinterpret_cast<uint16_t*>(p.v_aux) + crow * kPage + qq;
    *reinterpret_cast<u32x4*>(a16) = (u32x4){b0[0], b0[1], b0[2], b0[3]};
    *reinterpret_cast<u32x4*>(a16 + 8) = (u32x4){b0[4], b0[5], b0[6], b0[7]};
    *reinterpret_cast<u32x4*>(a16 + kPage) = (u32x4){b1[0], b1[1], b1[2], b1[3]};
    *reinterpret_cast<u32x4*>(a16 + kPage + 8) = (u32x4){b1[4], b1[5], b1[6], b1[7]};
  }
  if (p.pv == 2) {   // one NVFP4 group per channel: these 16 keys (absent ones zero)
    const int64_t aux_scales = p.num_pages * p.h_kv * kD * 32;   // scale plane offset
    float x0[16], x1[16];
#pragma unroll
    for (int j = 0; j < 16; ++j) {
      x0[j] = __uint_as_float(w[j] << 16);
      x1[j] = __uint_as_float(w[j] & 0xFFFF0000u);
    }
    uint32_t sc0, sc1;
    const uint64_t c0 = nvfp4_group(x0, 1.0f, rcp_sd, &sc0);
    const uint64_t c1 = nvfp4_group(x1, 1.0f, rcp_sd, &sc1);
    *reinterpret_cast<uint64_t*>(p.v_aux + crow * 32 + qq / 2) = c0;
    *reinterpret_cast<uint64_t*>(p.v_aux + (crow + 1) * 32 + qq / 2) = c1;
    p.v_aux[aux_scales + crow * 4 + qq / 16] = (uint8_t)sc0;
    p.v_aux[aux_scales + (crow + 1) * 4 + qq / 16] = (uint8_t)sc1;
  }
}

template <bool MX>
__global__ __launch_bounds__(256) void quantize_kernel(QuantParams p) {
  __shared__ int page_start;   // 1: the chunk's tokens are slots 0, 1, ... of one page, in order
  __shared__ float rcp_sd[128];
  // [h_q + h_kv][kMeanStride] BF16 mean rows, then [h_q + h_kv] tensor scales
  extern __shared__ __attribute__((aligned(16))) uint8_t sm_mean[];
  // last tokens first: the statistics pass ended with them, so they are the ones
  // still in the last-level cache (20000 + 9000 + 30000 + 12345 tokens 32:8 636 ->
  // 509 us with the streaming loads of that pass, 598 with those alone)
  const int b = gridDim.y - 1 - blockIdx.y;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int i0 = (int)(gridDim.x - 1 - blockIdx.x) * kChunk;
  if (i0 >= n) return;
  const int cnt = min(kChunk, n - i0);
  const int64_t tok0 = t0 + i0;
  const int tid = threadIdx.x;

  if (tid < 64) {
    const int64_t s0 = p.slot_mapping[tok0];
    const bool ok = (s0 % kPage == 0) && (tid >= cnt || p.slot_mapping[tok0 + tid] == s0 + tid);
    const bool all = __builtin_amdgcn_ballot_w64(!ok) == 0;
    if (tid == 0) page_start = all ? 1 : 0;
  }
  if (!MX && tid < 128) rcp_sd[tid] = (tid & 0x7F) && tid < 0x7F ? __fdiv_rn(1.0f, e4m3_value(tid)) : 0.0f;
  // the sequence's Q and K means (zero rows without smoothing)
  for (int u = tid; u < (p.h_q + p.h_kv) * (kD / 8); u += blockDim.x) {
    const int hh = u / (kD / 8), w = u % (kD / 8);
    uint4 m = make_uint4(0, 0, 0, 0);
    if (p.smooth) {
      const uint16_t* row = hh < p.h_q ? p.q_mean + ((int64_t)b * p.h_q + hh) * kD
                                       : p.k_mean + ((int64_t)b * p.h_kv + (hh - p.h_q)) * kD;
      m = reinterpret_cast<const uint4*>(row)[w];
    }
    *reinterpret_cast<uint4*>(sm_mean + hh * kMeanStride + w * 16) = m;
  }
  float* ts_s = reinterpret_cast<float*>(sm_mean + (p.h_q + p.h_kv) * kMeanStride);
  for (int hh = tid; hh < p.h_q + p.h_kv; hh += blockDim.x)
    ts_s[hh] = hh < p.h_q ? p.q_tscale[b * p.h_q + hh] : p.k_tscale[b * p.h_kv + (hh - p.h_q)];
  __syncthreads();
  const uint8_t* qmean_s = sm_mean;
  const uint8_t* kmean_s = sm_mean + p.h_q * kMeanStride;

  // Q rows (packed output); K rows (cache) with Delta_S
  quant_q_rows<MX>(p, qmean_s, ts_s, tok0, cnt, rcp_sd);
  quant_k_rows<MX>(p, kmean_s, qmean_s, ts_s + p.h_q, tok0, cnt, rcp_sd);
  __syncthreads();

  // V -> E4M3, channel-major page rows (plus the characterization copies in
  // v_aux: BF16 rows, or NVFP4 16-key groups along each channel row)
  const bool page_run = page_start && cnt == kChunk;   // whole page rows can be written
  if (page_run || (p.pv == 2 && page_start)) {
    const int64_t page = p.slot_mapping[tok0] / kPage;
    for (int u = tid; u < p.h_kv * (kD / 2); u += blockDim.x) {
      const int h = u / (kD / 2), cp = u % (kD / 2);
      const uint32_t* src = reinterpret_cast<const uint32_t*>(p.v + (tok0 * p.h_kv + h) * kD) + cp;
      const int64_t tstride = (int64_t)p.h_kv * (kD / 2);
      const int64_t crow = (page * p.h_kv + h) * kD + 2 * cp;   // channel row 2cp; 2cp+1 follows
      uint8_t* dst = p.v_codes + crow * kPage;
      // the two 64-byte channel rows (one 128-byte line) are stored whole after
      // all 64 tokens are converted: stores of line pieces far apart in time
      // cost partial-line write-backs
      u32x4 r0s[kPage / 16], r1s[kPage / 16];
      // 16 tokens at a time: 16 bytes of each of the two channel rows
#pragma unroll
      for (int qq = 0; qq < kPage; qq += 16) {
        uint32_t w[16];
#pragma unroll
        for (int j = 0; j < 16; ++j) w[j] = qq + j < cnt ? src[(int64_t)(qq + j) * tstride] : 0u;
        if (page_run) v_fp8_16(w, r0s[qq / 16], r1s[qq / 16]);
        v_aux_16(p, w, crow, qq, page_run, rcp_sd);
      }
      if (page_run) {
#pragma unroll
        for (int q = 0; q < kPage / 16; ++q) {
          *reinterpret_cast<u32x4*>(dst + 16 * q) = r0s[q];
          *reinterpret_cast<u32x4*>(dst + kPage + 16 * q) = r1s[q];
        }
      }
    }
  }
  if (!page_run) {
    for (int u = tid; u < cnt * p.h_kv * kD; u += blockDim.x) {
      const int c = u % kD, ih = u / kD;
      const int h = ih % p.h_kv, i = ih / p.h_kv;
      const int64_t slot = p.slot_mapping[tok0 + i];
      const uint16_t vb = p.v[(tok0 + i) * p.h_kv * kD + (int64_t)h * kD + c];
      const int64_t at = (((slot / kPage) * p.h_kv + h) * kD + c) * kPage + slot % kPage;
      p.v_codes[at] = (uint8_t)e4m3_rne_sat(bf16_to_f32(vb));
      if (p.pv == 1) reinterpret_cast<uint16_t*>(p.v_aux)[at] = vb;
    }
  }
}

// ---------------------------------------------------------------------------
// Few tokens: one workgroup (256 threads) per (64-token chunk, KV head with its
// group of query heads, sequence).  Everything a chunk writes for one KV head
// depends on that head group alone, so the chunk splits over the KV heads.
// quantize_kernel above is the better one when the chunks alone fill the chip;
// with few chunks its long serial lanes show (a K row there is one lane's work:
// 8 groups, then a 128-step chain per query head, about 40 us however few the
// rows).  Here 16 lanes share a K row as they do a Q row, the centered values
// go to LDS, and one lane per (token, query head) runs its Delta_S chain.
// Same arithmetic in the same order: the bytes are those of quantize_kernel.
// ---------------------------------------------------------------------------
constexpr int kMaxGroupLds = 16;             // query heads per KV head the group kernels take
constexpr int kKcStride = kD + 4;            // floats per centered K row in LDS (padded: rows on distinct banks)

struct GroupSmem {
  float kc[kChunk * kKcStride];              // centered K rows
  float rcp_sd[128];
  float ts[kMaxGroupLds + 1];                // tensor scales: the group's Q heads, then K
  int page_start;                            // 1: the chunk's tokens are slots 0, 1, ... of one page, in order
  __attribute__((aligned(16))) uint8_t mean[(kMaxGroupLds + 1) * kMeanStride];   // BF16 mean rows, Q heads then K
};

// V of 16 tokens (qq .. qq + 15 of the chunk) and channels 2cp, 2cp + 1 of head
// h: FP8 into the page rows (page_run: all 64 slots present), and the
// characterization copies.
__device__ __forceinline__ void quant_v_part(const QuantParams& p, int64_t tok0, int cnt, int64_t page, int h, int cp,
                                             int qq, bool page_run, const float* rcp_sd) {
  const uint32_t* src = reinterpret_cast<const uint32_t*>(p.v + (tok0 * p.h_kv + h) * kD) + cp;
  const int64_t tstride = (int64_t)p.h_kv * (kD / 2);
  const int64_t crow = (page * p.h_kv + h) * kD + 2 * cp;   // channel row 2cp; 2cp+1 follows
  uint32_t w[16];
#pragma unroll
  for (int j = 0; j < 16; ++j) w[j] = qq + j < cnt ? src[(int64_t)(qq + j) * tstride] : 0u;
  if (page_run) {
    u32x4 r0, r1;
    v_fp8_16(w, r0, r1);
    *reinterpret_cast<u32x4*>(p.v_codes + crow * kPage + qq) = r0;
    *reinterpret_cast<u32x4*>(p.v_codes + (crow + 1) * kPage + qq) = r1;
  }
  v_aux_16(p, w, crow, qq, page_run, rcp_sd);
}

// Parts of a head group's work, which need nothing of each other: separate
// workgroups take one part each (their latencies then run side by side: a chunk
// of 64 tokens takes 18 us in one workgroup whatever the number of chunks).
enum GroupPart { kPartK = 1, kPartQ = 2, kPartV = 4, kPartAll = 7 };   // kPartK: K rows and Delta_S

// Quantization and cache write of cnt (1..64) tokens from tok0 for KV head hk and
// its query heads; sm.mean, sm.ts, sm.rcp_sd and sm.page_start are filled.
template <bool MX>
__device__ __forceinline__ void quant_group(const QuantParams& p, GroupSmem& sm, int64_t tok0, int cnt, int hk,
                                            int parts) {
  constexpr int L = MX ? 4 : 2;          // lanes per quantization group
  constexpr int U = 8;                   // Q units per lane in flight
  const int grp = p.h_q / p.h_kv, tid = threadIdx.x;

  // K rows: 16 lanes each, the loads of all of a lane's units in flight
  constexpr int UK = kChunk * 16 / 256;
  if (parts & kPartK) {
    int64_t slot[UK];
    uint4 kv[UK];
#pragma unroll
    for (int k = 0; k < UK; ++k) {
      const int i = min((tid >> 4) + 16 * k, cnt - 1);   // past the end: not stored
      slot[k] = p.slot_mapping[tok0 + i];
      kv[k] = reinterpret_cast<const uint4*>(p.k + ((tok0 + i) * p.h_kv + hk) * kD)[tid & 15];
    }
#pragma unroll
    for (int k = 0; k < UK; ++k) {
      const int i = (tid >> 4) + 16 * k, c8 = tid & 15;
      if (i >= cnt) continue;
      const int64_t crow = ((slot[k] / kPage) * p.h_kv + hk) * kPage + slot[k] % kPage;
      float xc[8];
      center8(kv[k], *reinterpret_cast<const uint4*>(sm.mean + grp * kMeanStride + c8 * 16), xc);
      if (p.smooth) {
        float* dst = sm.kc + i * kKcStride + c8 * 8;
        *reinterpret_cast<float4*>(dst) = make_float4(xc[0], xc[1], xc[2], xc[3]);
        *reinterpret_cast<float4*>(dst + 4) = make_float4(xc[4], xc[5], xc[6], xc[7]);
      }
      uint32_t sc;
      const uint32_t w = encode_lane<MX>(xc, MX ? 1.0f : sm.ts[grp], sm.rcp_sd, &sc);
      *reinterpret_cast<uint32_t*>(p.k_codes + crow * 64 + c8 * 4) = w;
      if (c8 % L == 0) {
        p.k_scales[crow * 8 + c8 / L] = (uint8_t)sc;
        if (MX) p.k_scales[crow * 8 + 4 + c8 / L] = 0;
      }
    }
  }
  __syncthreads();   // the centered rows

  // Q rows: 16 lanes each
  const int nun = (parts & kPartQ) ? cnt * grp * 16 : 0;   // a multiple of 16: the lanes of a group act together
  for (int u0 = tid; u0 < nun; u0 += 256 * U) {
    uint4 v[U];
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int r = min(u0 + 256 * k, nun - 1) >> 4;   // past the end: not stored
      v[k] = reinterpret_cast<const uint4*>(p.q + ((tok0 + r / grp) * p.h_q + hk * grp + r % grp) * kD)[u0 & 15];
    }
#pragma unroll
    for (int k = 0; k < U; ++k) {
      const int u = u0 + 256 * k;
      if (u < nun) {
        const int r = u >> 4, c8 = u & 15, j = r % grp;
        const int64_t row = (tok0 + r / grp) * p.h_q + hk * grp + j;
        float xc[8];
        center8(v[k], *reinterpret_cast<const uint4*>(sm.mean + j * kMeanStride + c8 * 16), xc);
        uint32_t sc;
        const uint32_t w = encode_lane<MX>(xc, MX ? 1.0f : sm.ts[j], sm.rcp_sd, &sc);
        *reinterpret_cast<uint32_t*>(p.q_codes + row * 64 + c8 * 4) = w;
        if (c8 % L == 0) {
          p.q_scales[row * 8 + c8 / L] = (uint8_t)sc;
          if (MX) p.q_scales[row * 8 + 4 + c8 / L] = 0;
        }
      }
    }
  }

  // Delta_S: one lane per (token, query head), lanes on consecutive tokens; the
  // last lanes first, so that a few chains do not follow the waves' Q rows
  if (p.smooth && (parts & kPartK)) {
    for (int u = 255 - tid; u < cnt * grp; u += 256) {
      const int i = u % cnt, j = u / cnt;
      const float* x = sm.kc + i * kKcStride;
      const uint8_t* qm = sm.mean + j * kMeanStride;
      float d = 0.0f;
#pragma unroll 4
      for (int w = 0; w < 16; ++w) {
        const uint4 qv = *reinterpret_cast<const uint4*>(qm + 16 * w);
        const float4 x0 = *reinterpret_cast<const float4*>(x + 8 * w), x1 = *reinterpret_cast<const float4*>(x + 8 * w + 4);
        const uint32_t q4[4] = {qv.x, qv.y, qv.z, qv.w};
        const float xv[8] = {x0.x, x0.y, x0.z, x0.w, x1.x, x1.y, x1.z, x1.w};
#pragma unroll
        for (int e = 0; e < 8; ++e)
          d = __builtin_fmaf(__uint_as_float((e & 1) == 0 ? (q4[e >> 1] << 16) : (q4[e >> 1] & 0xFFFF0000u)), xv[e], d);
      }
      const int64_t slot = p.slot_mapping[tok0 + i];
      p.ds[((slot / kPage) * p.h_q + hk * grp + j) * kPage + slot % kPage] = bf16_rne(d);
    }
  }

  // V: whole channel rows where the chunk is one page, else a byte per (token, channel)
  if (!(parts & kPartV)) return;
  const bool page_run = sm.page_start && cnt == kChunk;
  if (page_run || (p.pv == 2 && sm.page_start))
    quant_v_part(p, tok0, cnt, p.slot_mapping[tok0] / kPage, hk, tid & 63, (tid >> 6) * 16, page_run, sm.rcp_sd);
  if (!page_run) {
    for (int u = tid; u < cnt * kD; u += 256) {
      const int c = u % kD, i = u / kD;
      const int64_t slot = p.slot_mapping[tok0 + i];
      const uint16_t vb = p.v[((tok0 + i) * p.h_kv + hk) * kD + c];
      const int64_t at = (((slot / kPage) * p.h_kv + hk) * kD + c) * kPage + slot % kPage;
      p.v_codes[at] = (uint8_t)e4m3_rne_sat(bf16_to_f32(vb));
      if (p.pv == 1) reinterpret_cast<uint16_t*>(p.v_aux)[at] = vb;
    }
  }
}

// sm.rcp_sd and, for cnt >= 1 tokens from tok0, sm.page_start (no barrier)
__device__ __forceinline__ void group_tables(const QuantParams& p, GroupSmem& sm, int64_t tok0, int cnt) {
  const int tid = threadIdx.x;
  if (tid < 64 && cnt > 0) {
    const int64_t s0 = p.slot_mapping[tok0];
    const bool ok = (s0 % kPage == 0) && (tid >= cnt || p.slot_mapping[tok0 + tid] == s0 + tid);
    const bool all = __builtin_amdgcn_ballot_w64(!ok) == 0;
    if (tid == 0) sm.page_start = all ? 1 : 0;
  }
  if (tid >= 128) sm.rcp_sd[tid - 128] = (tid & 0x7F) && (tid & 0x7F) < 0x7F ? __fdiv_rn(1.0f, e4m3_value(tid & 0x7F)) : 0.0f;
}

template <bool MX, bool PACKED>
__global__ __launch_bounds__(256) void quantize_group_kernel(QuantParams p) {
  __shared__ GroupSmem sm;
  const int tid = threadIdx.x;
  int b = blockIdx.z, chunk = blockIdx.x;
  if (PACKED && !packed_block<6>(p, blockIdx.x, b, chunk)) return;
  const int hk = blockIdx.y % p.h_kv;
  const int parts = (int)gridDim.y == p.h_kv ? kPartAll : 1 << (blockIdx.y / p.h_kv);   // 1 or 3 workgroups a group
  const int64_t t0 = p.cu_seqlens[b];
  const int n = p.cu_seqlens[b + 1] - (int)t0;
  const int i0 = chunk * kChunk;
  if (i0 >= n) return;
  const int cnt = min(kChunk, n - i0), grp = p.h_q / p.h_kv;
  group_tables(p, sm, t0 + i0, cnt);
  for (int u = tid; u < (grp + 1) * (kD / 8); u += 256) {
    const int j = u / (kD / 8), w = u % (kD / 8);
    uint4 m = make_uint4(0, 0, 0, 0);
    if (p.smooth) m = reinterpret_cast<const uint4*>(mean_row(p, b, j < grp ? hk * grp + j : p.h_q + hk))[w];
    *reinterpret_cast<uint4*>(sm.mean + j * kMeanStride + w * 16) = m;
  }
  if (tid <= grp) sm.ts[tid] = tid < grp ? p.q_tscale[b * p.h_q + hk * grp + tid] : p.k_tscale[b * p.h_kv + hk];
  __syncthreads();
  quant_group<MX>(p, sm, t0 + i0, cnt, hk, parts);
}

// The whole pass in one launch for calls whose sequences have at most 64 tokens
// (a decode step's cache write, a short prompt): the statistics of a head group
// need the group's tokens only, and one chunk holds them all.  The sums run
// over the tokens in order, as in stats_partial_kernel.
template <bool MX>
__global__ __launch_bounds__(256) void quantize_short_kernel(QuantParams p) {
  __shared__ GroupSmem sm;
  // one workgroup for all parts (grid z = 1) or one each (3); the Q part, or the
  // only workgroup, writes the Q statistics, the K part those of K
  const int hk = blockIdx.x, b = blockIdx.y, tid = threadIdx.x;
  const int parts = gridDim.z == 1 ? kPartAll : 1 << blockIdx.z;
  const int64_t t0 = p.cu_seqlens[b];
  const int n = min(p.cu_seqlens[b + 1] - (int)t0, kChunk);   // at most max_seqlen by contract
  const int grp = p.h_q / p.h_kv;
  const bool want_sum = p.compute_stats && p.smooth;
  group_tables(p, sm, t0, n);
  // 16 lanes per head row (the group's Q heads, then K), 8 channels per lane
  for (int u0 = 0; u0 < (grp + 1) * 16; u0 += 256) {
    const int u = u0 + tid, j = u >> 4, oct = u & 15;
    const bool act = j <= grp, isq = j < grp;
    const int hh = isq ? hk * grp + j : p.h_q + hk;
    float sum[8], mx[8], mn[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      sum[e] = 0.0f;
      mx[e] = -INFINITY;
      mn[e] = INFINITY;
    }
    // the V part needs no statistics; the K part those of Q only for their means
    const bool want = parts == kPartAll || parts == kPartQ || (parts == kPartK && (want_sum || !isq));
    const bool own = parts & (isq ? kPartQ : kPartK);
    if (act && want && p.need_partials && (isq || p.stats_k)) {
      const int H = isq ? p.h_q : p.h_kv;
      const uint4* src = reinterpret_cast<const uint4*>((isq ? p.q : p.k) + (t0 * H + (isq ? hh : hk)) * kD) + oct;
      for (int t = 0; t < n; t += 8) {
        uint4 w[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) w[k] = src[(int64_t)min(t + k, n - 1) * H * (kD / 8)];
#pragma unroll
        for (int k = 0; k < 8; ++k) {
          if (t + k < n) {
            const uint32_t wd[4] = {w[k].x, w[k].y, w[k].z, w[k].w};
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              const float x = __uint_as_float((e & 1) ? (wd[e >> 1] & 0xFFFF0000u) : (wd[e >> 1] << 16));
              sum[e] += x;
              mx[e] = fmaxf(mx[e], x);
              mn[e] = fminf(mn[e], x);
            }
          }
        }
      }
    }
    float amax = 0.0f;
    if (act) {
      uint16_t* mrow = mean_row(p, b, hh) + oct * 8;
      uint32_t mw[4] = {0u, 0u, 0u, 0u};
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        uint16_t m = 0;
        if (want_sum && n > 0) m = bf16_rne(__fdiv_rn(sum[e], (float)n));
        else if (!p.compute_stats && p.smooth) m = mrow[e];
        if (p.compute_stats && own) mrow[e] = m;
        mw[e >> 1] |= (uint32_t)m << (16 * (e & 1));
        if (p.need_partials && want && n > 0) {
          const float mu = bf16_to_f32(m);
          amax = fmaxf(amax, fmaxf(__builtin_fabsf(mx[e] - mu), __builtin_fabsf(mn[e] - mu)));
        }
      }
      *reinterpret_cast<uint4*>(sm.mean + j * kMeanStride + oct * 16) = make_uint4(mw[0], mw[1], mw[2], mw[3]);
    }
    for (int off = 1; off < 16; off <<= 1) amax = fmaxf(amax, __shfl_xor(amax, off));
    if (act && oct == 0) {
      float ts;
      if (!isq && !p.stats_k) {
        ts = p.k_tscale[b * p.h_kv + hk];   // frozen
      } else {
        ts = (p.tscale_unit || p.mx) ? 1.0f : tensor_scale(amax);
        if (own) write_tscale(p, b, hh, amax);
      }
      sm.ts[j] = ts;
    }
  }
  __syncthreads();
  if (n > 0) quant_group<MX>(p, sm, t0, n, hk, parts);
}

__global__ void convert_kernel(int fmt, const float* x, int64_t n, uint8_t* out) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= n) return;
  uint32_t c;
  if (fmt >= 0x400) {   // reference for 0x200 + b: exact scaling, then the software encoder
    c = e2m1_rne_sat(__builtin_ldexpf(x[i], 127 - (fmt & 0xFF)));
  } else if (fmt >= 0x300) {   // reference for 0x100 + c: IEEE division, then the software encoder
    c = e2m1_rne_sat(__fdiv_rn(x[i], e4m3_value(fmt & 0xFF)));
  } else if (fmt >= 0x200) {   // MXFP4 element: x / 2^e, e = (fmt & 0xFF) - 127 >= -126
    c = fp4_pair(0u, x[i], 0.0f, __builtin_ldexpf(1.0f, (fmt & 0xFF) - 127), 0) & 0xFu;
  } else if (fmt >= 0x100) {   // NVFP4 element: x / e4m3_value(fmt & 0xFF), the quantizer's division
    const float s = e4m3_value(fmt & 0xFF), r = __fdiv_rn(1.0f, s);
    if (__builtin_fabsf(x[i]) * r < 0x1p100f) c = fp4_pair(0u, div_by_scale(x[i], s, r), 0.0f, 1.0f, 0) & 0xFu;
    else c = e2m1_rne_sat(__fdiv_rn(x[i], s));   // the quantizer's fallback near the FP32 range
  } else {
    switch (fmt) {
      case 0: c = e4m3_rne_sat(x[i]); break;
      case 1: c = e2m1_rne_sat(x[i]); break;
      case 2: c = fp8_sat_pair(0u, x[i], 0.0f, false) & 0xFFu; break;
      default: c = fp4_pair(0u, x[i], 0.0f, 1.0f, 0) & 0xFu; break;
    }
  }
  out[i] = (uint8_t)c;
}

// Where the launch shapes change (all give the same bytes; times of the whole
// call on one MI355X, 32:8 heads unless noted):
//  - at most 64 tokens per sequence: one launch (32 x 1 token 52 -> 9.2 us, 8 x
//    64 tokens of 40:8 131 -> 23.6 us);
//  - statistics by one wave per (head, block) up to kWaveStats waves, about 18
//    per SIMD: 4048 tokens in four prompts 213 -> 154 us, 32768 tokens 40:8 (12K
//    waves) 265 -> 254 us, 65536 tokens 8:2 (5K) 137 -> 100 us; at 65536 tokens
//    40:8 (25K) the 256-thread shape is the better one, 452 against 463 us;
//  - the short finish up to kShortBlocks blocks of the longest sequence: 16 x
//    2000 tokens 303 -> 240 us; 64 blocks 63.9 -> 62.6 us; 128 blocks 102.2
//    against 104.8 us;
//  - quantization by KV head group up to kGroupChunks chunks: 4096 tokens 40:8
//    171 -> 94 us, 16 x 2000 tokens (516 chunks) 303 -> 280 us, 32768 tokens
//    40:8 (513) 254 -> 250 us; 65536 tokens 40:8 (1025) 463 against 499 us;
//  - a workgroup per part up to kPartGroups head groups, about two per CU: 65
//    tokens 24.8 -> 19.2 us, 777 tokens 23.8 -> 20.4 us; 16 x 2000 tokens (4128
//    groups) 206 us in one part against 215 us.
//  - grids of the blocks that the call has (packed_block) instead of (longest) x
//    (sequences) where the latter are more than twice as many: 30000 + 31 x 1 tokens
//    243 -> 201 us, 3000 + 200 x 1 83 -> 59, 60000 + 63 x 1 of 8:2 187 -> 108; up to
//    kPackedBatch sequences, eight steps of the search.
constexpr int64_t kWaveStats = 18432, kGroupChunks = 520, kPartGroups = 512;
constexpr int kPackedGrid = 2, kPackedBatch = 512;
constexpr int kOnePartTokens = 8;   // so few tokens that the parts cost more than they overlap

hipError_t launch_quantize(const QuantParams& p, hipStream_t stream) {
  const int hs = p.h_q + (p.stats_k ? p.h_kv : 0);
  const bool group_ok = p.h_q / p.h_kv <= kMaxGroupLds;
  if (p.max_seqlen <= kChunk && group_ok) {
    const bool split = p.max_seqlen > kOnePartTokens && (int64_t)p.batch * p.h_kv <= kPartGroups;
    const dim3 grid(p.h_kv, p.batch, split ? 3 : 1);
    if (p.mx) quantize_short_kernel<true><<<grid, dim3(256), 0, stream>>>(p);
    else quantize_short_kernel<false><<<grid, dim3(256), 0, stream>>>(p);
    return hipGetLastError();
  }
  // chunks and blocks of the call, at most (the sequence lengths are on the device)
  const int64_t blocks = (int64_t)p.total_tokens / 128 + p.batch;
  const int64_t chunks = (int64_t)p.total_tokens / kChunk + p.batch;
  const bool packed = p.batch <= kPackedBatch;
  if (p.need_partials && p.max_seqlen > 0) {
    const unsigned nb = (p.max_seqlen + 127) / 128;
    if (blocks * hs <= kWaveStats && p.max_seqlen <= 128 * 65535) {
      if (packed && blocks * kPackedGrid < (int64_t)nb * p.batch)
        stats_partial_wave_kernel<true><<<dim3(hs, (unsigned)blocks), dim3(64), 0, stream>>>(p);
      else
        stats_partial_wave_kernel<false><<<dim3(hs, nb, p.batch), dim3(64), 0, stream>>>(p);
    } else {
      stats_partial_kernel<<<dim3(nb, p.batch), dim3(256), 0, stream>>>(p);
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
  }
  if (p.max_seqlen <= kShortBlocks * 128)
    stats_final_short_kernel<<<dim3(hs, p.batch), dim3(kD), 0, stream>>>(p);
  else
    stats_final_kernel<<<dim3(hs * 4, p.batch), dim3(kFinThreads), 0, stream>>>(p);
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (p.total_tokens > 0 && p.max_seqlen > 0) {
    const unsigned nc = (p.max_seqlen + kChunk - 1) / kChunk;
    if (group_ok && chunks <= kGroupChunks) {
      const unsigned groups = p.h_kv * (chunks * p.h_kv <= kPartGroups ? 3 : 1);
      if (packed && chunks * kPackedGrid < (int64_t)nc * p.batch) {
        const dim3 grid((unsigned)chunks, groups);
        if (p.mx) quantize_group_kernel<true, true><<<grid, dim3(256), 0, stream>>>(p);
        else quantize_group_kernel<false, true><<<grid, dim3(256), 0, stream>>>(p);
      } else {
        const dim3 grid(nc, groups, p.batch);
        if (p.mx) quantize_group_kernel<true, false><<<grid, dim3(256), 0, stream>>>(p);
        else quantize_group_kernel<false, false><<<grid, dim3(256), 0, stream>>>(p);
      }
    } else {
      const dim3 grid(nc, p.batch);
      const size_t lds = (size_t)(p.h_q + p.h_kv) * (kMeanStride + sizeof(float));
      if (p.mx) quantize_kernel<true><<<grid, dim3(256), lds, stream>>>(p);
      else quantize_kernel<false><<<grid, dim3(256), lds, stream>>>(p);
    }
    e = hipGetLastError();
  }
  return e;
}

hipError_t launch_convert(int fmt, const float* x, int64_t n, uint8_t* out, hipStream_t stream) {
  if (n <= 0) return hipSuccess;
  const int64_t blocks = (n + 255) / 256;
  convert_kernel<<<dim3((unsigned)blocks), dim3(256), 0, stream>>>(fmt, x, n, out);
  return hipGetLastError();
}

}  // namespace mpfa
