// prefill_split.h -- the prefill work item for calls with few query rows: 32 query
// rows of one head per workgroup, its KV tiles spread over the eight waves.
//
// prefill_item walks a row block's tiles one after the other, so a call whose row
// blocks do not fill the chip (a short prompt, a chunk behind a long prefix, few
// heads on a tensor-parallel shard) takes (tiles) x (latency of a tile step).
// Here the scores and the softmax of eight tiles run side by side and only the PV
// product, the short part of a step, walks the tiles in order:
//   * wave w takes the tiles j with j % 8 == 7 - w, one per round: K and its own
//     scores go straight to registers as in the decode (no LDS staging, K is
//     dequantized per wave instead of once per workgroup: about 250 more vector
//     instructions per tile and 32 rows);
//   * the method quantizes P at the running maximum, so the waves exchange their
//     tiles' row maxima through LDS; each then has the running maxima before and
//     after its tile in the sequential order (last tile to first), and with them
//     the tile's P codes, rescale factor and row sum, which it leaves in LDS;
//   * a round later wave w < 4 accumulates O of channels 32w .. 32w + 31 over the
//     eight tiles in that order, the other waves being in their softmax meanwhile
//     (one such wave per SIMD).
// prefill_few_kernel spills 13 registers in NVFP4 with the compensation (44 bytes a
// lane), none without it or in MXFP4.
// Every FP32 operation has the operands and the order it has in prefill_item, so
// the bytes are the same whichever of the two a call takes.
#pragma once
#include "prefill_body.h"

namespace mpfa {

namespace {

constexpr int kSplitWaves = 8;
constexpr int kPvWaves = 4;       // 32 channels each

struct SplitSmem {
  float top[2][kSplitWaves][kWaveRows];        // row maxima of a round's tiles
  float alpha[2][kSplitWaves][kWaveRows];      // their rescale factors
  float ps[2][kSplitWaves][64];                // the lanes' row sums
  u32x4 p[2][kSplitWaves][4][64];              // P codes as PV operands: [16-byte part][lane]
};

// K side of one tile in registers: lane (row r = lane % 32, half hf) holds, for
// the key of MFMA row r of each 32-key block, channels 64hf .. +63 (NVFP4), or
// 32hf .. +31 and 64 + 32hf .. +31 (MXFP4), the row's scales and the key's Delta_S.
struct SplitK {
  u32x4 c[4][2];
  uint2 sc[4];
  uint32_t ds[4];
};

template <bool MX, bool SMOOTH>
__device__ __forceinline__ void split_load_k(SplitK& r, const PrefillParams& p, const ItemState& st, int pg0, int pg1) {
  // tile_key(lc, kb) within its page is key0 + 16 (kb % 2)
  const uint32_t key0 = 32u * ((st.lc >> 2) & 1) + 4u * (st.lc >> 3) + (st.lc & 3);
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    const int pg = kb < 2 ? pg0 : pg1;
    const int64_t row = (int64_t)pg * p.h_kv + st.hk;
    const uint8_t* cb = p.k_codes + row * (kPage * 64);
    const uint8_t* sb = p.k_scales + row * (kPage * 8);
    const int so = 16 * (kb & 1);   // keys, as a scalar offset
    if (MX) {
      r.c[kb][0] = page_load16(cb, kPage * 64, key0 * 64 + 16 * st.hf, so * 64);
      r.c[kb][1] = page_load16(cb, kPage * 64, key0 * 64 + 16 * st.hf, so * 64 + 32);
      r.sc[kb].x = page_load4(sb, kPage * 8, key0 * 8, so * 8);
    } else {
      r.c[kb][0] = page_load16(cb, kPage * 64, key0 * 64 + 32 * st.hf, so * 64);
      r.c[kb][1] = page_load16(cb, kPage * 64, key0 * 64 + 32 * st.hf, so * 64 + 16);
      r.sc[kb] = page_load8(sb, kPage * 8, key0 * 8, so * 8);
    }
    if (SMOOTH)
      r.ds[kb] = page_load2(p.ds + ((int64_t)pg * p.h_q + st.h) * kPage, kPage * 2, key0 * 2, so * 2);
  }
}

// S^T = 1 Delta_S^T + K Q^T of the tile; the rank-one term is formed by a BF16
// MFMA (bit-identical to the accumulator input, and one value per lane and block).
template <bool MX, bool SMOOTH>
__device__ __forceinline__ void split_qk(f32x16 (&s)[4], const SplitK& r, const ItemState& st) {
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
    f32x16 acc = {};
    if (SMOOTH) {
      // exact: a BF16 value times a power of two stays a BF16 value
      const uint32_t v = bf16_rne(bf16_to_f32((uint16_t)r.ds[kb]) * st.seed_scale);
      const u32x4 a = {v, 0u, 0u, 0u};
      acc = mfma32_bf16(__builtin_bit_cast(bf16x8, a), st.bseed, acc);
    }
    if (MX) {
      const int sc = (int)(r.sc[kb].x >> (8 * st.hf));   // bytes 0, 2: blocks hf, 2 + hf
      acc = mfma32_fp4<0>(r.c[kb][0], st.qraw[0], acc, sc, st.qscale[0]);
      acc = mfma32_fp4<2>(r.c[kb][1], st.qraw[1], acc, sc, st.qscale[1]);
    } else {
      // MFMA ks takes channels 16ks + 8hf .. +7, code dword 2ks + hf of the row.
      // A lane half holds dwords 8hf .. +7: the swap of the upper half of dword 2t
      // with the lower half of dword 2t + 1 gives the operands of ks = t and 4 + t.
      uint32_t w[8];
#pragma unroll
      for (int t = 0; t < 4; ++t) {
        const auto x = __builtin_amdgcn_permlane32_swap(r.c[kb][t >> 1][2 * (t & 1)], r.c[kb][t >> 1][2 * (t & 1) + 1],
                                                        false, false);
        w[t] = x[0];
        w[4 + t] = x[1];
      }
      const f16x2 a = e4m3_pair_f16(r.sc[kb].x), b = e4m3_pair_f16(r.sc[kb].x >> 16);
      const f16x2 c = e4m3_pair_f16(r.sc[kb].y), d = e4m3_pair_f16(r.sc[kb].y >> 16);
      const _Float16 g[8] = {a[0], a[1], b[0], b[1], c[0], c[1], d[0], d[1]};
#pragma unroll
      for (int ks = 0; ks < 8; ++ks) acc = mfma32_f16(dequant8h(w[ks], g[ks]), st.qop[ks], acc);
    }
    s[kb] = acc;
  }
}

// V of channel block db of one tile (pages pg0, pg1): the A operands of its two
// 64-key MFMAs.
__device__ __forceinline__ void split_load_v(u32x4 (&v)[2][2], const PrefillParams& p, const ItemState& st, int db,
                                             int pg0, int pg1) {
#pragma unroll
  for (int kk = 0; kk < 2; ++kk) {
    const uint8_t* vb = p.v_codes + ((int64_t)(kk ? pg1 : pg0) * p.h_kv + st.hk) * (kD * kPage);
#pragma unroll
    for (int w = 0; w < 2; ++w)
      v[kk][w] = page_load16(vb, kD * kPage, st.lc * kPage + 32 * st.hf, 32 * db * kPage + 16 * w);
  }
}

template <bool SMOOTH, bool MX>
__device__ __forceinline__ void prefill_split_item(const PrefillParams& p, int b, int h, int r0, SplitSmem& sm) {
  ItemState st;
  item_setup<MX>(p, b, h, r0, kWaveRows, r0, st);
  const int wave = __builtin_amdgcn_readfirstlane(st.wave);
  const bool pv_wave = wave < kPvWaves;
  const int32_t* ptab = p.page_table + (int64_t)st.b * p.max_pages;
  const int npg = (st.kvl + 63) >> 6;
  // the 16 pages of tile group q (tiles 8q .. 8q + 7), one per lane, clamped to
  // mapped ones for tiles outside the sequence, whose data is not used
  auto window = [&](int q) { return ptab[min(max(16 * q + (st.lane & 15), 0), npg - 1)]; };

  f32x16 o = {};                            // waves 0 .. 3: O^T of their channels
  float l = 0.0f;                           // and this lane's share of the row sum
  float mround = -INFINITY;                 // running maximum after all tiles of the earlier rounds
  SoftState ss;
  f32x16 s[4];
  PTile pt;
  SplitK k;
  constexpr int kAheadV = 4;                // V tiles in flight
  // MXFP4: K and V are loaded as soon as their registers are free (512 rows behind
  // 32000 tokens, 32:8: 270 -> 261 us).  NVFP4 has 32 query and 4 scale registers
  // more and spills so (379 us against 325); it loads K and the last two V tiles
  // after the first PV products.
  constexpr bool kEarly = MX;
  u32x4 v[kAheadV][2][2];

  // V of tile t (of eight, last first) of the tile group whose pages are in win
  auto load_v = [&](int t, int win) {
    split_load_v(v[t % kAheadV], p, st, wave, __builtin_amdgcn_readlane(win, 2 * (7 - t)),
                 __builtin_amdgcn_readlane(win, 2 * (7 - t) + 1));
  };
  // PV of tile t of tile group q, whose P is in buffer buf
  auto pv = [&](int t, int buf, int q) {
    const float alpha = sm.alpha[buf][t][st.lc];
    l = __builtin_fmaf(alpha, l, sm.ps[buf][t][st.lane]);
    if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) o *= alpha;
    u32x4 (&vt)[2][2] = v[t % kAheadV];
    const int nvalid = st.kvl - (8 * q + 7 - t) * kTile;   // keys of the tile before kv_len
    if (nvalid < kTile) {   // uniform: the sequence's last keys
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int w = 0; w < 2; ++w) vt[kk][w] = zero_tail(vt[kk][w], nvalid - 64 * kk - 32 * st.hf - 16 * w);
    }
#pragma unroll
    for (int kk = 0; kk < 2; ++kk) {
      const u32x4 pa = sm.p[buf][t][2 * kk][st.lane], pc = sm.p[buf][t][2 * kk + 1][st.lane];
      const i32x8 vop = {(int)vt[kk][0][0], (int)vt[kk][0][1], (int)vt[kk][0][2], (int)vt[kk][0][3],
                         (int)vt[kk][1][0], (int)vt[kk][1][1], (int)vt[kk][1][2], (int)vt[kk][1][3]};
      const i32x8 pop = {(int)pa[0], (int)pa[1], (int)pa[2], (int)pa[3], (int)pc[0], (int)pc[1], (int)pc[2], (int)pc[3]};
      o = mfma32_fp8(vop, pop, o);
    }
  };

  const int rounds = (st.j_hi >> 3) + 1;
  int q = rounds - 1;                       // tile group of the round; this wave's tile is 8q + 7 - wave
  const int e0 = 2 * (kSplitWaves - 1 - wave);
  int wprev = 0, wcur = window(q), wnext = window(q - 1);
  split_load_k<MX, SMOOTH>(k, p, st, __builtin_amdgcn_readlane(wcur, e0), __builtin_amdgcn_readlane(wcur, e0 + 1));
  auto load_next_k = [&]() {
    split_load_k<MX, SMOOTH>(k, p, st, __builtin_amdgcn_readlane(wnext, e0), __builtin_amdgcn_readlane(wnext, e0 + 1));
  };
  for (int r = 0; r < rounds; ++r, --q) {
    const bool have_pv = pv_wave && r > 0;
    const int key0 = (8 * q + kSplitWaves - 1 - wave) * kTile;
    if (have_pv) {
#pragma unroll
      for (int t = 0; t < kAheadV; ++t) load_v(t, wprev);
    }
    __builtin_amdgcn_sched_barrier(0);
    // A tile past the row block (first round only) reads mapped pages, is masked
    // whole and adds nothing.
    split_qk<MX, SMOOTH>(s, k, st);
    __builtin_amdgcn_sched_barrier(0);
    if (kEarly) load_next_k();
    if (key0 + kTile - 1 > st.wpos_min) mask_tile(s, key0, st);
    float mxa = -INFINITY, mxb = -INFINITY;
#pragma unroll
    for (int kb = 0; kb < 4; kb += 2)
#pragma unroll
      for (int i = 0; i < 16; i += 2) {
        mxa = fmaxf(fmaxf(mxa, s[kb][i]), s[kb][i + 1]);
        mxb = fmaxf(fmaxf(mxb, s[kb + 1][i]), s[kb + 1][i + 1]);
      }
    const float mx = wave_max32(fmaxf(mxa, mxb));
    sm.top[r & 1][wave][st.lc] = mx;   // both lane halves hold it
    // this round's row maxima and the last one's P are there after it; the buffers
    // of the round before that are free again
    __syncthreads();
    // running maximum before this wave's tile: the earlier rounds' and the tiles before it
    ss.m = mround;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float t = sm.top[r & 1][w][st.lc];
      mround = fmaxf(mround, t);
      if (w < wave) ss.m = fmaxf(ss.m, t);
    }
    if (have_pv) {
#pragma unroll
      for (int t = 0; t < kAheadV; ++t) {
        pv(t, (r - 1) & 1, q + 1);
        if (kEarly || t < 2) load_v(t + kAheadV, wprev);
        __builtin_amdgcn_sched_barrier(0);
      }
    }
    if (!kEarly) load_next_k();
    __builtin_amdgcn_sched_barrier(0);
    const float mnew = fmaxf(ss.m, mx);
    const float muse = (mnew == -INFINITY) ? 0.0f : mnew;
    const float alpha = (ss.m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f((ss.m - muse) * st.lam2);
    ss.bias = __builtin_fmaf(-muse, st.lam2, kLog2PScale<kPvFp8>);
    float ps = 0.0f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      ps += exp_block<kPvFp8, 0>(s[kb], kb, st, ss, pt);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (!kEarly && have_pv) {
      load_v(6, wprev);
      load_v(7, wprev);
    }
    sm.alpha[r & 1][wave][st.lc] = alpha;
    sm.ps[r & 1][wave][st.lane] = ps;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const i32x8& x = pt.pb[i >> 1];
      const int f = 4 * (i & 1);
      sm.p[r & 1][wave][i][st.lane] = (u32x4){(uint32_t)x[f], (uint32_t)x[f + 1], (uint32_t)x[f + 2], (uint32_t)x[f + 3]};
    }
    if (have_pv) {
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int t = kAheadV; t < kSplitWaves; ++t) pv(t, (r - 1) & 1, q + 1);
    }
    wprev = wcur;
    wcur = wnext;
    wnext = window(q - 2);
    __builtin_amdgcn_sched_barrier(0);
  }
  if (pv_wave) {
#pragma unroll
    for (int t = 0; t < kAheadV; ++t) load_v(t, wprev);
  }
  __syncthreads();
  if (!pv_wave) return;
#pragma unroll
  for (int t = 0; t < kSplitWaves; ++t) {
    pv(t, (rounds - 1) & 1, 0);
    if (t + kAheadV < kSplitWaves) load_v(t + kAheadV, wprev);
  }
  asm volatile("" : "+v"(o));   // full-wave MFMAs (see prefill_item)
  const float lt = l + __shfl_xor(l, 32);
  const int row = st.wrow0 + st.lc;
  if (row < st.nq) store_channels(p, st, row, wave, __frcp_rn(lt), o);
}

// A call with few row blocks (PrefillParams::few): one workgroup per 32 query
// rows, which either splits their KV tiles over its waves, or, where the context
// is too short for that to pay, takes the rows of a whole item (prefill_pick_block).
// The choice is per sequence, from its context on the device.  Model of the call, in
// us: whole items 5 + 1.75 (MXFP4 1.45) per tile of the longest for 128 rows, 2.65 (2.0)
// for 256, all resident; split items 4, and 7.5 + 5 per eight tiles each (MXFP4 6.5 +
// 4), as many one after the other as there are blocks per compute unit.  Measured,
// 32:8 heads, whole items / split: 512 rows behind 16000 tokens 234 / 170 us, 64 behind
// 16000 221 / 82, 256 behind 2000 40 / 25, 8:2 heads 1024 behind 16000 239 / 88, 2000
// tokens 34.9 / 29.7 (MXFP4 28.7 / 23.1); not split: 1024 behind 16000 240 (split 340),
// 500 behind 2000 43.7 (47.2), 1024-token prompt 22.3 (53.9), 256-token prompt 10.8
// (17.7).  In a batch the count of blocks per unit is more than a split of one sequence
// waits for, and the line stays at 2.65 (2.0) for either item: 40:8 heads, 91, 147 and 53
// rows behind 155, 1928, 618 tokens 38.8 us at 1.75, 28.0 so.
template <bool MX>
struct FewSmem {
  union {
    SplitSmem split;
    PrefillSmemT<MX, kPvFp8> item;
  };
};

template <int SEED, bool MX>
__device__ __forceinline__ void prefill_few_block(const PrefillParams& p, int bid, FewSmem<MX>& sm) {
  int b, h, rank;
  map_item(p, bid, b, h, rank);
  const int nq = p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b];
  const int blks = (nq + kWaveRows - 1) / kWaveRows;
  // 32-row block, the last first; of one sequence first those that end 128 rows, the
  // only ones with work where its tiles are not split (1300 tokens 32:8, wide table, 37
  // -> 31 us; but 18, 506 and 401 rows behind 612, 611, 214 tokens 8:2 20.3 -> 24.2)
  int blk = p.n_qtiles - 1 - rank;
  if (p.batch == 1) {
    const int quads = p.n_qtiles / 4;
    if (rank < quads) {
      blk = 4 * (quads - 1 - rank);
      if (blk < blks) blk = min(blk + 3, blks - 1);
    } else {
      blk = blk / 3 * 4 + blk % 3;
      if (blk == blks - 1) return;   // its last 128 rows are fewer: taken above
    }
  }
  if (blk >= blks) return;
  int blocks = 0;   // 32-row blocks of one head over the batch
  for (int i = threadIdx.x & 63; i < p.batch; i += 64)
    blocks += (p.cu_seqlens_q[i + 1] - p.cu_seqlens_q[i] + kWaveRows - 1) / kWaveRows;
  const int per_cu = (wave_sum_all(blocks) * p.h_q + kComputeUnits - 1) / kComputeUnits;
  const int item = item_rows(p, b);
  const float per_tile = item == kHalfRows && p.batch == 1 ? (MX ? 1.45f : 1.75f) : (MX ? 2.0f : 2.65f);
  const float start = (float)p.q_start[b], rows = (float)nq;
  const float most = (start + rows) * (1.0f / kTile), mean = (start + 0.5f * rows) * (1.0f / kTile);
  const float split = MX ? 6.5f + 0.5f * mean : 7.5f + 0.625f * mean;
  if (4.0f + (float)per_cu * split < 5.0f + per_tile * most)
    prefill_split_item<SEED != kSeedNone, MX>(p, b, h, blk * kWaveRows, sm.split);
  else
    prefill_pick_block<SEED, MX, kWaveRows>(p, b, h, blk, item, sm.item);
}

}  // namespace

}  // namespace mpfa
