// prefill_split.h -- the prefill work item for calls with few query rows: 32 query
// rows of one head per workgroup, its KV tiles spread over the eight waves.
//
// prefill_item walks a row block's tiles one after the other, so a call whose row
// blocks do not fill the chip (a short prompt, a chunk behind a long prefix, few
// heads on a tensor-parallel shard) takes (tiles) x (latency of a tile step).
// Here wave w takes the tiles j with j % 8 == 7 - w, one per round.  The method
// quantizes P at the running maximum, so a round first takes every tile's row
// maximum, exchanges them through LDS, and each wave then uses the running
// maximum its tile has in the sequential order (last tile to first): the same P
// codes.  Every wave accumulates its own l and O relative to the maximum of its
// latest tile; they are added at the end, scaled to the final maximum.  Only the
// order of FP32 sums differs from prefill_item.
//
// A tile is used by one wave, so K and V go straight to registers as in the
// decode (no LDS staging, and K is dequantized per wave instead of once per
// workgroup: about 250 more vector instructions per tile and 32 rows).  That is
// why prefill_item stays for calls that fill the chip (prefill_few_block has the
// rule).
#pragma once
#include "prefill_body.h"

namespace mpfa {

namespace {

constexpr int kSplitWaves = 8;
constexpr int kSplitStride = kD + 4;   // floats per O row in LDS (padded: rows on distinct banks)

struct SplitSmem {
  float top[2][kSplitWaves][kWaveRows];          // row maxima of a round's tiles
  float m[kSplitWaves][kWaveRows], l[kSplitWaves][kWaveRows];
  float o[kSplitWaves][kWaveRows * kSplitStride];
};

// K side of one tile in registers: lane (row r = lane % 32, half hf) holds, for
// the key of MFMA row r of each 32-key block, channels 64hf .. +63 (NVFP4), or
// 32hf .. +31 and 64 + 32hf .. +31 (MXFP4), their scales and the key's Delta_S.
struct SplitK {
  u32x4 c[4][2];
  uint32_t sc[4];
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
    const int so = 16 * (kb & 1);   // keys, as a scalar offset
    if (MX) {
      r.c[kb][0] = page_load16(cb, kPage * 64, key0 * 64 + 16 * st.hf, so * 64);
      r.c[kb][1] = page_load16(cb, kPage * 64, key0 * 64 + 16 * st.hf, so * 64 + 32);
      r.sc[kb] = page_load4(p.k_scales + row * (kPage * 8), kPage * 8, key0 * 8, so * 8);
    } else {
      r.c[kb][0] = page_load16(cb, kPage * 64, key0 * 64 + 32 * st.hf, so * 64);
      r.c[kb][1] = page_load16(cb, kPage * 64, key0 * 64 + 32 * st.hf, so * 64 + 16);
      r.sc[kb] = page_load4(p.k_scales + row * (kPage * 8), kPage * 8, key0 * 8 + 4 * st.hf, so * 8);
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
      const int sc = (int)(r.sc[kb] >> (8 * st.hf));   // bytes 0, 2: blocks hf, 2 + hf
      acc = mfma32_fp4<0>(r.c[kb][0], st.qraw[0], acc, sc, st.qscale[0]);
      acc = mfma32_fp4<2>(r.c[kb][1], st.qraw[1], acc, sc, st.qscale[1]);
    } else {
      const f16x2 s01 = e4m3_pair_f16(r.sc[kb]), s23 = e4m3_pair_f16(r.sc[kb] >> 16);
#pragma unroll
      for (int ks = 0; ks < 8; ++ks)
        acc = mfma32_f16(dequant8h(r.c[kb][ks >> 2][ks & 3], ks < 4 ? s01[ks >> 1] : s23[(ks >> 1) - 2]), st.qop[ks], acc);
    }
    s[kb] = acc;
  }
}

// V of 64 keys (page pg) of the tile: A operands of the four channel blocks.
__device__ __forceinline__ void split_load_v(u32x4 (&v)[4][2], const PrefillParams& p, const ItemState& st, int pg) {
  const uint8_t* vb = p.v_codes + ((int64_t)pg * p.h_kv + st.hk) * (kD * kPage);
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int w = 0; w < 2; ++w)
      v[db][w] = page_load16(vb, kD * kPage, st.lc * kPage + 32 * st.hf, 32 * db * kPage + 16 * w);
}

// nvalid: keys of these 64 before kv_len (bytes past them are cleared)
__device__ __forceinline__ void split_pv(u32x4 (&v)[4][2], const i32x8& pb, f32x16 (&o)[4], const ItemState& st,
                                         int nvalid) {
  if (nvalid < kPage) {   // uniform: the sequence's last keys
#pragma unroll
    for (int db = 0; db < 4; ++db)
#pragma unroll
      for (int w = 0; w < 2; ++w) v[db][w] = zero_tail(v[db][w], nvalid - 32 * st.hf - 16 * w);
  }
#pragma unroll
  for (int db = 0; db < 4; ++db) {
    const i32x8 vop = {(int)v[db][0][0], (int)v[db][0][1], (int)v[db][0][2], (int)v[db][0][3],
                       (int)v[db][1][0], (int)v[db][1][1], (int)v[db][1][2], (int)v[db][1][3]};
    o[db] = mfma32_fp8(vop, pb, o[db]);
  }
}

template <bool SMOOTH, bool MX>
__device__ __forceinline__ void prefill_split_item(const PrefillParams& p, int b, int h, int r0, SplitSmem& sm) {
  ItemState st;
  item_setup<MX, kSplitWaves, true>(p, b, h, r0, st);
  const int wave = __builtin_amdgcn_readfirstlane(st.wave);
  const int32_t* ptab = p.page_table + (int64_t)st.b * p.max_pages;
  const int npg = (st.kvl + 63) >> 6;
  auto page = [&](int i) { return ptab[min(max(i, 0), npg - 1)]; };

  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db) o[db] = (f32x16){};
  SoftState ss = {-INFINITY, 0.0f, 0.0f};   // m: running maximum after this wave's latest tile
  float mround = -INFINITY;                 // running maximum after all tiles of the earlier rounds
  f32x16 s[4];
  PTile pt;
  SplitK k;
  u32x4 v[4][2];

  const int rounds = (st.j_hi >> 3) + 1;
  int j = 8 * (rounds - 1) + 7 - wave;      // this wave's tile of the round
  int c0 = __builtin_amdgcn_readfirstlane(page(2 * j)), c1 = __builtin_amdgcn_readfirstlane(page(2 * j + 1));
  int n0 = page(2 * (j - 8)), n1 = page(2 * (j - 8) + 1);   // the next round's pages
  split_load_k<MX, SMOOTH>(k, p, st, c0, c1);
  for (int r = 0; r < rounds; ++r, j -= 8) {
    // A tile past the row block (first round only) reads mapped pages, is masked
    // whole and adds nothing.
    split_qk<MX, SMOOTH>(s, k, st);
    __builtin_amdgcn_sched_barrier(0);
    split_load_v(v, p, st, c0);
    if (j * kTile + kTile - 1 > st.wpos_min) mask_tile(s, j * kTile, st);
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
    __syncthreads();
    // running maximum of this wave's tile: the earlier rounds' and the tiles up to it
    float mine = mround;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float t = sm.top[r & 1][w][st.lc];
      mround = fmaxf(mround, t);
      if (w <= wave) mine = fmaxf(mine, t);
    }
    const float muse = (mine == -INFINITY) ? 0.0f : mine;
    const float alpha = (ss.m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f((ss.m - muse) * st.lam2);
    ss.m = mine;
    ss.bias = __builtin_fmaf(-muse, st.lam2, kLog2PScale<kPvFp8>);
    rescale(o, alpha);
    float ps = 0.0f;
#pragma unroll
    for (int kb = 0; kb < 4; ++kb) {
      ps += exp_block<kPvFp8, 0>(s[kb], kb, st, ss, pt);
      __builtin_amdgcn_sched_barrier(0);
    }
    ss.l = alpha * ss.l + ps;
    const int key0 = j * kTile;
    split_pv(v, pt.pb[0], o, st, st.kvl - key0);
    __builtin_amdgcn_sched_barrier(0);
    split_load_v(v, p, st, c1);
    c0 = __builtin_amdgcn_readfirstlane(n0);
    c1 = __builtin_amdgcn_readfirstlane(n1);
    split_load_k<MX, SMOOTH>(k, p, st, c0, c1);
    n0 = page(2 * (j - 16));
    n1 = page(2 * (j - 16) + 1);
    __builtin_amdgcn_sched_barrier(0);
    split_pv(v, pt.pb[1], o, st, st.kvl - key0 - kPage);
    __builtin_amdgcn_sched_barrier(0);
  }

  // add the waves' states, scaled to the final maximum (mround)
  const float lt = ss.l + __shfl_xor(ss.l, 32);
#pragma unroll
  for (int db = 0; db < 4; ++db) asm volatile("" : "+v"(o[db]));   // full-wave MFMAs (see prefill_item)
  if (st.lane < 32) {
    sm.m[wave][st.lc] = ss.m;
    sm.l[wave][st.lc] = lt;
  }
#pragma unroll
  for (int db = 0; db < 4; ++db)
#pragma unroll
    for (int i = 0; i < 4; ++i)
      *reinterpret_cast<f32x4*>(&sm.o[wave][st.lc * kSplitStride + 32 * db + 8 * i + 4 * st.hf]) =
          (f32x4){o[db][4 * i], o[db][4 * i + 1], o[db][4 * i + 2], o[db][4 * i + 3]};
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kWaveRows / kSplitWaves; ++i) {   // four rows per wave, two channels per lane
    const int row = wave * (kWaveRows / kSplitWaves) + i;
    float M = -INFINITY, L = 0.0f, a0 = 0.0f, a1 = 0.0f;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) M = fmaxf(M, sm.m[w][row]);
    const float muse = (M == -INFINITY) ? 0.0f : M;
#pragma unroll
    for (int w = 0; w < kSplitWaves; ++w) {
      const float f = __builtin_amdgcn_exp2f((sm.m[w][row] - muse) * st.lam2);
      const float2 ov = *reinterpret_cast<const float2*>(&sm.o[w][row * kSplitStride + 2 * st.lane]);
      L = __builtin_fmaf(f, sm.l[w][row], L);
      a0 = __builtin_fmaf(f, ov.x, a0);
      a1 = __builtin_fmaf(f, ov.y, a1);
    }
    if (st.wrow0 + row < st.nq) {
      const float inv = __frcp_rn(L);
      *reinterpret_cast<uint32_t*>(p.out + ((int64_t)(st.q0 + st.wrow0 + row) * p.h_q + st.h) * kD + 2 * st.lane) =
          (uint32_t)bf16_rne(a0 * inv) | ((uint32_t)bf16_rne(a1 * inv) << 16);
    }
  }
}

// A call with few row blocks (PrefillParams::few): one workgroup per 32 query
// rows, which either splits their KV tiles over its waves, or, where the context
// is too short for that to pay, one of each eight takes the 256 rows as a whole.
// The choice is per sequence, from its context on the device.  Model of the
// call, in us: whole items, all resident, 5 + 2.65 (MXFP4 2.0) per tile of the
// longest; split items 4, and 7.5 + 5 per eight tiles each, as many one after
// the other as there are blocks per compute unit.  Measured, whole items / this
// kernel: 512 rows behind 32000 tokens 32:8 700 / 319 us, 64 behind 20000 266 /
// 102, 256 behind 16000 8:2 355 / 80, 1000-token prompt 8:2 33 / 14.5, 1024
// behind 16000 32:8 377 / 341; not split: 2048 behind 16000 430 (split 696),
// 2048-token prompt 57 (124), 250-token prompt 16.1 (17).
template <bool SMOOTH, bool MX>
struct FewSmem {
  union {
    SplitSmem split;
    PrefillSmemT<MX, kPvFp8> item;
  };
};

template <bool SMOOTH, bool MX>
__device__ __forceinline__ void prefill_few_block(const PrefillParams& p, int bid, FewSmem<SMOOTH, MX>& sm) {
  int b, h, rank;
  map_item(p, bid, b, h, rank);
  const int blk = p.n_qtiles - 1 - rank;   // 32-row block
  const int nq = p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b];
  if (blk * kWaveRows >= nq) return;
  int blocks = 0;   // 32-row blocks of one head over the batch
  for (int i = threadIdx.x & 63; i < p.batch; i += 64)
    blocks += (p.cu_seqlens_q[i + 1] - p.cu_seqlens_q[i] + kWaveRows - 1) / kWaveRows;
  const int per_cu = (wave_sum_all(blocks) * p.h_q + kComputeUnits - 1) / kComputeUnits;
  const float start = (float)p.q_start[b], rows = (float)nq;
  const float most = (start + rows) * (1.0f / kTile), mean = (start + 0.5f * rows) * (1.0f / kTile);
  if (4.0f + (float)per_cu * (7.5f + 0.625f * mean) < 5.0f + (MX ? 2.0f : 2.65f) * most) {
    prefill_split_item<SMOOTH, MX>(p, b, h, blk * kWaveRows, sm.split);
    return;
  }
  const int item = blk / kItemWaves, last = min((item + 1) * kItemWaves, (nq + kWaveRows - 1) / kWaveRows) - 1;
  if (blk == last)   // the first of the eight in dispatch order
    prefill_item<SMOOTH ? kSeedInit : kSeedNone, MX, kPvFp8, kItemWaves>(p, b, h, item * kItemRows, sm.item);
}

}  // namespace

}  // namespace mpfa
