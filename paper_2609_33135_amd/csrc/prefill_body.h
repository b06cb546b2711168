// prefill_body.h -- the causal prefill work item (Algorithm 1 main loop) as a
// device function, shared by the prefill kernel and the fused mixed-step kernel.
#pragma once
#include "mpfa_device.h"
#include "mpfa_internal.h"

namespace mpfa {

namespace {

constexpr int kWaveRows = 32;                // query rows per wave: the columns of one 32x32 MFMA
constexpr int kItemWaves = 8;
constexpr int kItemRows = kItemWaves * kWaveRows;
constexpr int kHalfRows = kItemRows / 2;

// Precision of the PV product: the method's FP8 (P * 448 and V in E4M3), or
// the two other assignments compared in Sec. 3.1 / Fig. 3a, BF16 P and V, and
// NVFP4 P (2688 P quantized per 16 keys with dynamic E4M3 scales) with NVFP4 V
// (16-key groups per channel, tensor scale 1), both on FP16 / BF16 MFMA after
// exact dequantization.
enum PvMode { kPvFp8 = 0, kPvBf16 = 1, kPvNvfp4 = 2 };

// Two K and two V tile buffers.  Rows are padded by 16 bytes: 16 consecutive
// lanes of an MFMA operand read (16 consecutive rows of one 16-byte chunk) then
// cover all banks, and every chunk of every row block is a constant offset from
// one lane address.
template <bool MX, int PV>
struct PrefillSmemT {
  // K rows in MFMA order (row r of key block kb is LDS row 32 kb + r).  NVFP4:
  // exact FP16; MXFP4: raw codes, then the E8M0 scales as [MFMA row][lane
  // half][64-channel half][key block].
  static constexpr int kKStride = MX ? 64 + 16 : 256 + 16;
  static constexpr int kKBytes = kTile * kKStride + (MX ? 512 : 0);
  // V: [channel][key], FP8 bytes or BF16 / exact FP16
  static constexpr int kVStride = (PV == kPvFp8 ? kTile : 2 * kTile) + 16;
  uint8_t k[2][kKBytes];
  uint8_t v[2][kD * kVStride];
  float ds[2][kTile];       // seed values (BF16 values in accumulator units) as FP32, key order
  uint16_t dss[2][kTile];   // the same values, BF16, in seed_slot order
};

// Key order inside a tile.  MFMA row r of 32-key block kb (accumulator rows of
// S^T = K Q^T) is key 64*(kb/2) + 32*((r/4)%2) + 16*(kb%2) + 4*(r/8) + r%4: the
// 16 accumulator registers of block kb in lane half hf are then the 16
// consecutive keys from 64*(kb/2) + 32*hf + 16*(kb%2), and the registers of
// blocks 2kk, 2kk+1 the 32 consecutive keys that lane half hf supplies to the
// kk-th 64-key PV MFMA: P never leaves the lane.
__device__ __forceinline__ int tile_key(int r, int kb) {
  return 64 * (kb >> 1) + 32 * ((r >> 2) & 1) + 16 * (kb & 1) + 4 * (r >> 3) + (r & 3);
}
__device__ __forceinline__ int key_row(int key) { return 8 * ((key >> 2) & 3) + 4 * ((key >> 5) & 1) + (key & 3); }
__device__ __forceinline__ int key_blk(int key) { return 2 * (key >> 6) + ((key >> 4) & 1); }
// position in dss of key `key`: the four blocks' values of one MFMA row are contiguous
__device__ __forceinline__ int seed_slot(int key) { return key_row(key) * 4 + key_blk(key); }

__device__ __forceinline__ u32x4 zero_tail(u32x4 w, int nvalid) {
  // keep bytes [0, nvalid) of the 16-byte word
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    int keep = nvalid - 4 * i;
    uint32_t mask = keep >= 4 ? 0xFFFFFFFFu : (keep <= 0 ? 0u : ((1u << (8 * keep)) - 1u));
    w[i] &= mask;
  }
  return w;
}

// Raw bytes of one unit (32 elements) of a K and of a V tile held in registers
// between the global load and the LDS store.  A page of one KV head is 256
// units, contiguous in unit order: unit i of K is key i/4, channels 32 (i%4) ..
// +31; unit i of V is channel i/2, keys 32 (i%2) .. +31.
struct KRegs {
  u32x4 c;         // code bytes
  uint32_t sc;     // their E4M3 scales (two), or their E8M0 scale
  uint32_t ds;     // BF16 Delta_S of key i (i < 64)
};
template <int PV>
struct VRegs {
  static constexpr int kWords = PV == kPvFp8 ? 2 : (PV == kPvBf16 ? 4 : 1);   // FP8, BF16 or E2M1 codes
  u32x4 v[kWords];
  uint32_t sc;     // NVFP4: their two E4M3 scales
};

// Loads from a page of `bytes` bytes at a wave-uniform base, through a buffer
// resource in scalar registers: the lane's 32-bit offset is the only address
// register (a 64-bit pointer per plane costs the loop 10 VGPRs it needs).
__device__ __forceinline__ __amdgpu_buffer_rsrc_t page_rsrc(const void* base, int bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), 0, bytes, 0x00027000);
}
__device__ __forceinline__ u32x4 page_load16(const void* base, int bytes, uint32_t off, int scalar_off = 0) {
  return __builtin_amdgcn_raw_buffer_load_b128(page_rsrc(base, bytes), off, scalar_off, 0);
}
__device__ __forceinline__ uint2 page_load8(const void* base, int bytes, uint32_t off, int scalar_off = 0) {
  const auto w = __builtin_amdgcn_raw_buffer_load_b64(page_rsrc(base, bytes), off, scalar_off, 0);
  return make_uint2(w[0], w[1]);
}
__device__ __forceinline__ uint32_t page_load4(const void* base, int bytes, uint32_t off, int scalar_off = 0) {
  return __builtin_amdgcn_raw_buffer_load_b32(page_rsrc(base, bytes), off, scalar_off, 0);
}
__device__ __forceinline__ uint32_t page_load2(const void* base, int bytes, uint32_t off, int scalar_off = 0) {
  return (uint16_t)__builtin_amdgcn_raw_buffer_load_b16(page_rsrc(base, bytes), off, scalar_off, 0);
}
__device__ __forceinline__ uint32_t page_load1(const void* base, int bytes, uint32_t off) {
  return (uint8_t)__builtin_amdgcn_raw_buffer_load_b8(page_rsrc(base, bytes), off, 0, 0);
}

// Every address lies in a mapped page, so the loads are unconditional: what
// slots at or past kv_len hold is masked (K) or cleared (V) later.
template <bool MX, bool SMOOTH>
__device__ __forceinline__ void fetch_k(KRegs& r, const PrefillParams& p, int pg, int hk, int h, uint32_t i) {
  const int64_t row = (int64_t)pg * p.h_kv + hk;
  r.c = page_load16(p.k_codes + row * (kPage * 64), kPage * 64, i * 16u);
  const uint8_t* sb = p.k_scales + row * (kPage * 8);
  r.sc = MX ? page_load1(sb, kPage * 8, (i >> 2) * 8u + (i & 3u)) : page_load2(sb, kPage * 8, i * 2u);
  if (SMOOTH) r.ds = page_load2(p.ds + ((int64_t)pg * p.h_q + h) * kPage, kPage * 2, (i & 63u) * 2u);
}
template <int PV>
__device__ __forceinline__ void fetch_v(VRegs<PV>& r, const PrefillParams& p, int pg, int hk, uint32_t i) {
  const int64_t row = (int64_t)pg * p.h_kv + hk;
  if (PV == kPvFp8) {
    const uint8_t* src = p.v_codes + row * (kD * kPage);
#pragma unroll
    for (int w = 0; w < 2; ++w) r.v[w % VRegs<PV>::kWords] = page_load16(src, kD * kPage, i * 32u + 16u * w);
  } else if (PV == kPvBf16) {
    const uint8_t* src = p.v_aux + row * (kD * kPage * 2);
#pragma unroll
    for (int w = 0; w < 4; ++w) r.v[w % VRegs<PV>::kWords] = page_load16(src, kD * kPage * 2, i * 64u + 16u * w);
  } else {
    r.v[0] = page_load16(p.v_aux + row * (kD * 32), kD * 32, i * 16u);
    r.sc = page_load2(p.v_aux + p.num_pages * p.h_kv * (kD * 32) + row * (kD * 4), kD * 4, i * 2u);
  }
}

// How the compensation 1 Delta_S^T (Sec. 4.3 Eq. 11) enters the score
// accumulator before the QK product:
//  kSeedMfma  one BF16 rank-one MFMA per 32-key block (A = the block's Delta_S
//             in reduction slot 0, B = ones in slot 0);
//  kSeedInit  the same rank-one matrix loaded directly as the accumulator input
//             of the first FP16 MFMA (bit-identical: both start the accumulator
//             at the FP32 value of the BF16 Delta_S);
//  kSeedNone  no compensation (the unsmoothed "direct" variant);
//  kSeedElem  the placement the rank-one seed replaces (Sec. 3.2, Fig. 10):
//             the accumulator starts at zero and Delta_S is added to every
//             score in FP32 after the QK product, on the softmax path.  Same
//             values up to the FP32 rounding order.
enum SeedMode { kSeedNone = 0, kSeedMfma = 1, kSeedInit = 2, kSeedElem = 3 };

// half: which 64 keys of the tile the unit's page holds
template <int SEED, bool MX, int PV>
__device__ __forceinline__ void store_k(PrefillSmemT<MX, PV>& sm, int buf, const KRegs& r, float seed_scale, int half,
                                        int i) {
  const int key = 64 * half + (i >> 2), qt = i & 3;
  uint8_t* rowp = sm.k[buf] + (32 * key_blk(key) + key_row(key)) * sm.kKStride;
  if (MX) {
    *reinterpret_cast<u32x4*>(rowp + qt * 16) = r.c;
    sm.k[buf][kTile * sm.kKStride + (key_row(key) * 2 + (qt & 1)) * 8 + (qt >> 1) * 4 + key_blk(key)] = (uint8_t)r.sc;
  } else {
    const f16x2 s2 = e4m3_pair_f16(r.sc);
#pragma unroll
    for (int w = 0; w < 4; ++w)
      *reinterpret_cast<f16x8*>(rowp + qt * 64 + w * 16) = dequant8h(r.c[w], s2[w >> 1]);
  }
  if (SEED != kSeedNone) {
    // exact: a BF16 value times a power of two stays a BF16 value.  The four
    // waves of a page hold the same values; all store them (no branch).
    const float v = bf16_to_f32(bf16_rne(bf16_to_f32((uint16_t)r.ds) * seed_scale));
    const int dkey = 64 * half + (i & 63);
    if (SEED == kSeedMfma) sm.dss[buf][seed_slot(dkey)] = (uint16_t)(__float_as_uint(v) >> 16);
    else sm.ds[buf][dkey] = v;
  }
}
// nvalid: keys of the tile before kv_len (V bytes past them are cleared)
template <bool MX, int PV>
__device__ __forceinline__ void store_v(PrefillSmemT<MX, PV>& sm, int buf, const VRegs<PV>& r, int half, int i,
                                        int nvalid) {
  constexpr int kE = PV == kPvFp8 ? 1 : 2;
  const int d = i >> 1, key = 64 * half + 32 * (i & 1);
  uint8_t* dst = sm.v[buf] + d * sm.kVStride + key * kE;
  if (PV == kPvNvfp4) {
    // finite whatever the bytes, and P is 0 on keys past kv_len: nothing to clear
#pragma unroll
    for (int w = 0; w < 4; ++w)   // 8 codes of keys 8w .. +7, the scale of their 16-key group
      *reinterpret_cast<f16x8*>(dst + 16 * w) = dequant8(r.v[0][w], split_e4m3((r.sc >> (8 * (w >> 1))) & 0xFFu));
  } else {
    constexpr int kW = VRegs<PV>::kWords;
    u32x4 v[kW];
#pragma unroll
    for (int w = 0; w < kW; ++w) v[w] = r.v[w];
    if (nvalid < kTile) {   // uniform: the sequence's last tile
#pragma unroll
      for (int w = 0; w < kW; ++w) v[w] = zero_tail(v[w], kE * (nvalid - key) - 16 * w);
    }
#pragma unroll
    for (int w = 0; w < kW; ++w) *reinterpret_cast<u32x4*>(dst + 16 * w) = v[w];
  }
}

// Per-item state of one wave: the work item, the query operands, the softmax
// scale and the row positions.
struct ItemState {
  int b, h, hk, q0, nq, qs, kvl, j_hi;
  int lane, wave, hf, lc;   // lane half (l / 32) and query column (l % 32)
  int wrow0, wpos_min;
  bool wave_active;
  float lam2, seed_scale;
  int pos;             // absolute position of the lane's query
  f16x8 qop[8];        // NVFP4: exact FP16 query operands, tensor scale factored out
  u32x4 qraw[2];       // MXFP4: raw codes of channels 64i + 32hf .. +31
  int qscale[2];       // MXFP4: their E8M0 scales
  bf16x8 bseed;        // B operand of the rank-one seed MFMA: 1 in slot 0 of lanes 0..31
};

// Sequence, query head and row-tile rank of dispatch position `bid`.
__device__ __forceinline__ void map_item(const PrefillParams& p, int bid, int& b, int& h, int& rank) {
  if (p.xcd_remap) {
    // block ids are dealt round-robin to the 8 XCDs; give each XCD the query
    // heads of a fixed subset of KV heads so their K/V tiles share its L2.
    const int xcd = bid & 7, slot = bid >> 3;
    const int kvpx = p.h_kv / 8, grp = p.h_q / p.h_kv;
    const int ipr = kvpx * grp * p.batch;
    rank = slot / ipr;
    int r = slot % ipr;
    const int hk = xcd * kvpx + r % kvpx;
    r /= kvpx;
    h = hk * grp + r % grp;
    b = r / grp;
  } else {
    const int per = p.h_q * p.batch;
    rank = bid / per;
    const int rem = bid % per;
    h = rem % p.h_q;
    b = rem / p.h_q;
  }
}

// Sum over the wave (DPP, no LDS round trips), in every lane.
__device__ __forceinline__ int wave_sum_all(int x) {
  x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xF, 0xF, true);   // row_shr 1, 2, 4, 8
  x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xF, 0xF, true);
  x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xA, 0xF, false);  // row_bcast 15
  x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xC, 0xF, false);  // row_bcast 31
  return __builtin_amdgcn_readlane(x, 63);
}

// Dispatch order of a batch whose sequences start at different positions (chunks
// behind prefixes): position pos is the pos-th longest row tile of the batch, by
// KV tiles to visit, found by a binary search over the tile count; lanes hold
// the sequences.  By row-tile index alone a short chunk behind a long prefix,
// the longest items of all, starts last (chunks of 512, 2048, 1000 rows behind
// 30000, 5001, 12345 tokens, 32:8: 821 -> 670 us).  Sequences that start
// together are in that order already.  Returns false past the last item.
__device__ __forceinline__ bool longest_item(const PrefillParams& p, int pos, int& b, int& tile) {
  const int lane = threadIdx.x & 63;
  int qs = 0, nq = 0;
  if (lane < p.batch) {
    qs = p.q_start[lane];
    nq = p.cu_seqlens_q[lane + 1] - p.cu_seqlens_q[lane];
  }
  const int items = (nq + kItemRows - 1) / kItemRows;
  if (pos >= wave_sum_all(items)) return false;
  // first item of the lane's sequence that visits at least c + 1 tiles (its last tile is >= c)
  auto first = [&](int c) { const int x = c * kTile - qs; return nq - 1 < x ? items : (x > 0 ? x / kItemRows : 0); };
  int lo = 0, hi = p.max_pages / 2 + 1;   // the pos-th longest item's last tile is in [lo, hi)
  while (hi - lo > 1) {
    const int mid = (lo + hi) >> 1;
    if (wave_sum_all(items - first(mid)) > pos) lo = mid;
    else hi = mid;
  }
  const int f0 = first(lo), f1 = first(lo + 1);
  const int rest = pos - wave_sum_all(items - f1);   // among the items whose last tile is lo
  int incl = f1 - f0;
  for (int d = 1; d < kOrderMaxBatch; d <<= 1) {
    const int up = __shfl_up(incl, d);
    if (lane >= d) incl += up;
  }
  const uint64_t past = __ballot(incl > rest);
  b = __ffsll((unsigned long long)past) - 1;
  tile = __builtin_amdgcn_readlane(f0, b) + rest - (__builtin_amdgcn_readlane(incl, b) - __builtin_amdgcn_readlane(f1 - f0, b));
  return true;
}

// Whether the sequences' first positions differ by more than a row tile.
__device__ __forceinline__ bool starts_differ(const PrefillParams& p) {
  if (!p.order) return false;
  const int lane = threadIdx.x & 63;
  const int x = p.q_start[min(lane, p.batch - 1)], x0 = __builtin_amdgcn_readfirstlane(x);
  return __ballot(abs(x - x0) > kItemRows) != 0;
}

// State of one wave of the work item (query head h, rows r0 .. r0 + rows - 1 of
// sequence b, r0 below its row count); wrow0: the wave's first row.  Loads the
// wave's query operands.
template <bool MX>
__device__ __forceinline__ void item_setup(const PrefillParams& p, int b, int h, int r0, int rows, int wrow0,
                                           ItemState& st) {
  const int q0 = p.cu_seqlens_q[b];
  const int nq = p.cu_seqlens_q[b + 1] - q0;
  const int end = min(r0 + rows, nq);

  st.b = b;
  st.h = h;
  st.q0 = q0;
  st.nq = nq;
  st.qs = p.q_start[b];
  st.kvl = p.kv_len[b];
  st.hk = h / (p.h_q / p.h_kv);
  st.lane = threadIdx.x & 63;
  st.wave = threadIdx.x >> 6;
  st.hf = st.lane >> 5;
  st.lc = st.lane & 31;
  st.j_hi = (st.qs + end - 1) >> 7;

  const float tq = p.q_tscale[b * p.h_q + h], tk = p.k_tscale[b * p.h_kv + st.hk];
  const int eqk = ilog2f(tq) + ilog2f(tk);
  st.lam2 = __builtin_ldexpf(p.lam, eqk);        // lambda * tQ * tK
  st.seed_scale = __builtin_ldexpf(1.0f, -eqk);  // Delta_S in accumulator units

  st.wrow0 = wrow0;
  st.wave_active = wrow0 < end;
  st.wpos_min = st.qs + st.wrow0;

  // ---- Q operands (B of S^T = K Q^T).  NVFP4: exact FP16, tensor scale
  // factored out.  MXFP4: the raw codes and E8M0 scales (the lane's 32-element
  // blocks of the scaled FP4 MFMA).
  const int row = st.wrow0 + st.lc;
  const bool valid = row < nq;
  st.pos = st.qs + min(row, nq - 1);
  const int64_t tok = q0 + (valid ? row : 0);
  const uint8_t* qc = p.q_codes + (tok * p.h_q + h) * 64;
  const uint8_t* qsc = p.q_scales + (tok * p.h_q + h) * 8;
  if (MX) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      st.qraw[i] = valid ? *reinterpret_cast<const u32x4*>(qc + 32 * i + 16 * st.hf) : (u32x4){0u, 0u, 0u, 0u};
      st.qscale[i] = valid ? qsc[2 * i + st.hf] : 127;
    }
  } else {
    // the lane's channels: 16ks + 8hf .. +7 (group ks); scale times code is exact in FP16
    const uint2 sw = valid ? *reinterpret_cast<const uint2*>(qsc) : make_uint2(0u, 0u);
    const f16x2 a = e4m3_pair_f16(sw.x), b2 = e4m3_pair_f16(sw.x >> 16), c = e4m3_pair_f16(sw.y), d = e4m3_pair_f16(sw.y >> 16);
    const _Float16 g[8] = {a[0], a[1], b2[0], b2[1], c[0], c[1], d[0], d[1]};
#pragma unroll
    for (int ks = 0; ks < 8; ++ks) {
      const uint32_t cw = valid ? *reinterpret_cast<const uint32_t*>(qc + 8 * ks + 4 * st.hf) : 0u;
      st.qop[ks] = dequant8h(cw, g[ks]);
    }
  }
  st.bseed = (bf16x8){};
  if (st.lane < 32) st.bseed[0] = (__bf16)1.0f;
}

// S^T = seed + K Q^T of one 32-key block (Algorithm 1, scores).
template <int SEED, bool MX, int PV>
__device__ __forceinline__ void qk_block(f32x16& s, int kb, const PrefillSmemT<MX, PV>& sm, int buf,
                                         const ItemState& st) {
  const int hf = st.hf, lc = st.lc;
  f32x16 seed = {};
  if (SEED == kSeedMfma) {
    // every lane reads the value of its row lc; only reduction slot 0 of lanes
    // 0..31 meets a nonzero B element
    const u32x4 a = {(uint32_t)sm.dss[buf][4 * lc + kb], 0u, 0u, 0u};
    seed = mfma32_bf16(__builtin_bit_cast(bf16x8, a), st.bseed, seed);
  } else if (SEED == kSeedInit) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(&sm.ds[buf][64 * (kb >> 1) + 32 * hf + 16 * (kb & 1) + 4 * i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) seed[4 * i + e] = w[e];
    }
  }
  s = seed;
  const uint8_t* kp = sm.k[buf] + (32 * kb + lc) * sm.kKStride + 16 * hf;
  if (MX) {
    const uint2 ks8 = *reinterpret_cast<const uint2*>(sm.k[buf] + kTile * sm.kKStride + (lc * 2 + hf) * 8);
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      const int sk = (int)(ks ? ks8.y : ks8.x);
      const u32x4 kop = *reinterpret_cast<const u32x4*>(kp + 32 * ks);
      if (kb == 0) s = mfma32_fp4<0>(kop, st.qraw[ks], s, sk, st.qscale[ks]);
      else if (kb == 1) s = mfma32_fp4<1>(kop, st.qraw[ks], s, sk, st.qscale[ks]);
      else if (kb == 2) s = mfma32_fp4<2>(kop, st.qraw[ks], s, sk, st.qscale[ks]);
      else s = mfma32_fp4<3>(kop, st.qraw[ks], s, sk, st.qscale[ks]);
    }
  } else {
#pragma unroll
    for (int ks = 0; ks < 8; ++ks)
      s = mfma32_f16(*reinterpret_cast<const f16x8*>(kp + 32 * ks), st.qop[ks], s);
  }
  if (SEED == kSeedElem) {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const f32x4 w = *reinterpret_cast<const f32x4*>(&sm.ds[buf][64 * (kb >> 1) + 32 * hf + 16 * (kb & 1) + 4 * i]);
#pragma unroll
      for (int e = 0; e < 4; ++e) s[4 * i + e] += w[e];
    }
  }
}

// P operands of the PV product of one tile: FP8 words (kPvFp8), eight BF16 values
// per MFMA (kPvBf16), or their E2M1 codes and the scales of 16 keys (kPvNvfp4),
// made exact FP16 next to the MFMA: held as such from the softmax on they are 20
// registers more, and the pipelined step spilled 29 (131072 tokens, 40:8: 263 ms
// so, 212.5 with the codes and no spill).
struct PTile {
  i32x8 pb[2];     // keys 64kk + 32hf .. +31
  f16x8 ph[8];     // keys 64(t/4) + 32hf + 8(t%4) .. +7
  uint32_t pc[8];  // the same keys
  uint32_t psc[4]; // E4M3 scale of codes 2i, 2i + 1
};

// Softmax state of the wave's query column.
struct SoftState {
  float m, l;          // running maximum and (this lane's share of the) row sum
  float bias;          // exponent bias of the tile whose scores are held
};

// log2 of the fixed factor the P quantizer applies: 448 (FP8), 1 (BF16),
// 2688 = 6 * 448 (NVFP4: the largest P, 1, maps to the top E2M1 code
// under the largest E4M3 scale)
template <int PV>
constexpr float kLog2PScale = PV == kPvFp8 ? kLog2_448 : (PV == kPvBf16 ? 0.0f : 11.392317422778760f);

// Causal mask of the scores of the tile at key0.
__device__ __forceinline__ void mask_tile(f32x16 (&s)[4], int key0, const ItemState& st) {
  // key 64(kb/2) + 32hf + 16(kb%2) + r of the tile lies after query position pos
  const int lim = st.pos - key0 - 32 * st.hf;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) {
#pragma unroll
    for (int q = 0; q < 4; ++q) {
#pragma unroll
      for (int i = 0; i < 4; ++i)
        if (64 * (kb >> 1) + 16 * (kb & 1) + 4 * q + i > lim) s[kb][4 * q + i] = -INFINITY;
      // keep each compare next to its select: scheduled as one batch, the
      // 64 compare masks exhaust the scalar registers
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// Running maximum over the tile's scores, the rescale factor and the exponent bias.
// ABL > 0 only in the characterization library (built with
// MPFA_ABLATION_BUILD), whose outputs are meaningless by design: the cost of
// a softmax stage is the time difference to the build without it (Sec. 3.2,
// Fig. 3c).  ABL 1: P = its exponent argument (no exp2); ABL 2: also no row
// maximum, row sum or O rescale.
template <int PV, int ABL>
__device__ __forceinline__ float max_tile(const f32x16 (&s)[4], const ItemState& st, SoftState& ss) {
  // two independent chains of v_max3 (two new scores per instruction)
  float mxa = -INFINITY, mxb = -INFINITY;
#pragma unroll
  for (int kb = 0; kb < 4; kb += 2) {
#pragma unroll
    for (int r = 0; r < 16; r += 2) {
      mxa = fmaxf(fmaxf(mxa, s[kb][r]), s[kb][r + 1]);
      mxb = fmaxf(fmaxf(mxb, s[kb + 1][r]), s[kb + 1][r + 1]);
    }
  }
  const float mx = ABL >= 2 ? 0.0f : wave_max32(fmaxf(mxa, mxb));
  const float mnew = fmaxf(ss.m, mx);
  const float muse = (mnew == -INFINITY) ? 0.0f : mnew;
  const float alpha = (ss.m == -INFINITY) ? 0.0f : __builtin_amdgcn_exp2f((ss.m - muse) * st.lam2);
  ss.m = mnew;
  ss.bias = ABL >= 2 ? kLog2PScale<PV> : __builtin_fmaf(-muse, st.lam2, kLog2PScale<PV>);
  return alpha;
}

// P of one 32-key block from its scores; returns the lane's sum of it.
template <int PV, int ABL>
__device__ __forceinline__ float exp_block(const f32x16& s, int kb, const ItemState& st, const SoftState& ss,
                                           PTile& pt) {
  float ps = 0.0f;
  float ev[16];
#pragma unroll
  for (int q = 0; q < 4; ++q) {
    float e[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float arg = __builtin_fmaf(s[4 * q + i], st.lam2, ss.bias);
      e[i] = ABL >= 1 ? arg : __builtin_amdgcn_exp2f(arg);
    }
    if (ABL < 2) {
      const float q4 = (e[0] + e[1]) + (e[2] + e[3]);
      ps = q == 0 ? q4 : ps + q4;
    }
    if (PV == kPvFp8) {
      int w = (int)pack_fp8x4(e[0], e[1], e[2], e[3]);
      // keeps the exponentials here: P is only used by the PV product, and the
      // compiler would otherwise sink them past the branches before it
      asm volatile("" : "+v"(w), "+v"(ps));
      pt.pb[kb >> 1][4 * (kb & 1) + q] = w;
    } else {
#pragma unroll
      for (int i = 0; i < 4; ++i) ev[4 * q + i] = e[i];
    }
  }
  if (PV == kPvBf16) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      bf16x8 b;
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = (__bf16)ev[8 * t + i];
      pt.ph[2 * kb + t] = __builtin_bit_cast(f16x8, b);
    }
  } else if (PV == kPvNvfp4) {
    // the lane's 16 keys of the block are one 16-key group: scale
    // E4M3(amax / 6), codes E2M1(P'/scale)
    float amax = 0.0f;
#pragma unroll
    for (int i = 0; i < 16; ++i) amax = fmaxf(amax, ev[i]);
    const uint32_t sc = fp8_sat_pair(0u, div_by_scale(amax, 6.0f, kRcp6), 0.0f, false) & 0xFFu;
    const float sd = e4m3_value(sc);
    uint32_t cw[2] = {0u, 0u};
    if (sd > 0.0f) {
      const float r = __fdiv_rn(1.0f, sd);
#pragma unroll
      for (int w = 0; w < 2; ++w)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          cw[w] = fp4_pair(cw[w], div_by_scale(ev[8 * w + 2 * j], sd, r), div_by_scale(ev[8 * w + 2 * j + 1], sd, r),
                           1.0f, j);
    }
    uint32_t scale = sc;
    asm volatile("" : "+v"(cw[0]), "+v"(cw[1]), "+v"(scale), "+v"(ps));   // the codes are formed here (see the FP8 words)
    pt.pc[2 * kb] = cw[0];
    pt.pc[2 * kb + 1] = cw[1];
    pt.psc[kb] = scale;
  }
  return ps;
}

// O *= alpha, only when one of the wave's maxima moved.
__device__ __forceinline__ void rescale(f32x16 (&o)[4], float alpha) {
  if (__builtin_amdgcn_ballot_w64(alpha != 1.0f) != 0) {
#pragma unroll
    for (int db = 0; db < 4; ++db) o[db] *= alpha;
  }
}

// O^T += V^T P^T with V of the tile in sm.
template <bool MX, int PV>
__device__ __forceinline__ void pv_tile(const PrefillSmemT<MX, PV>& sm, int buf, const PTile& pt, f32x16 (&o)[4],
                                        const ItemState& st) {
  const int hf = st.hf, lc = st.lc;
  const uint8_t* vp = sm.v[buf] + lc * sm.kVStride + (PV == kPvFp8 ? 32 : 64) * hf;
  if (PV == kPvFp8) {
#pragma unroll
    for (int kk = 0; kk < 2; ++kk)
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const u32x4 va = *reinterpret_cast<const u32x4*>(vp + 32 * db * sm.kVStride + 64 * kk);
        const u32x4 vb = *reinterpret_cast<const u32x4*>(vp + 32 * db * sm.kVStride + 64 * kk + 16);
        const i32x8 vop = {(int)va[0], (int)va[1], (int)va[2], (int)va[3],
                           (int)vb[0], (int)vb[1], (int)vb[2], (int)vb[3]};
        o[db] = mfma32_fp8(vop, pt.pb[kk], o[db]);
      }
  } else {
    // eight 16-key MFMAs per channel block: MFMA t reduces keys
    // 64(t/4) + 32hf + 8(t%4) .. +7 of each lane half, so A (the V row chunk of
    // those keys) and B (the lane's own P values) pair the same keys
#pragma unroll
    for (int t = 0; t < 8; ++t) {
      const f16x8 ph = PV == kPvNvfp4 ? dequant8h(pt.pc[t], e4m3_pair_f16(pt.psc[t >> 1])[0]) : pt.ph[t];
#pragma unroll
      for (int db = 0; db < 4; ++db) {
        const u32x4 va =
            *reinterpret_cast<const u32x4*>(vp + 32 * db * sm.kVStride + 128 * (t >> 2) + 16 * (t & 3));
        if (PV == kPvBf16)
          o[db] = mfma32_bf16(__builtin_bit_cast(bf16x8, va), __builtin_bit_cast(bf16x8, ph), o[db]);
        else
          o[db] = mfma32_f16(__builtin_bit_cast(f16x8, va), ph, o[db]);
      }
    }
  }
}

// out = O / (448 l) as BF16 (for the other PV precisions the factor is the
// one their P carries): channels 32 db .. +31 of one row, inv = 1 / l.
__device__ __forceinline__ void store_channels(const PrefillParams& p, const ItemState& st, int row, int db, float inv,
                                               const f32x16& o) {
  uint16_t* dst = p.out + ((int64_t)(st.q0 + row) * p.h_q + st.h) * kD + 32 * db + 4 * st.hf;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const uint32_t lo = (uint32_t)bf16_rne(o[4 * i] * inv) | ((uint32_t)bf16_rne(o[4 * i + 1] * inv) << 16);
    const uint32_t hi = (uint32_t)bf16_rne(o[4 * i + 2] * inv) | ((uint32_t)bf16_rne(o[4 * i + 3] * inv) << 16);
    *reinterpret_cast<uint2*>(dst + 8 * i) = make_uint2(lo, hi);
  }
}

__device__ __forceinline__ void store_output(const PrefillParams& p, const ItemState& st, float l,
                                             const f32x16 (&o)[4]) {
  const float lt = l + __shfl_xor(l, 32);
  const int row = st.wrow0 + st.lc;
  if (row < st.nq) {
    const float inv = __frcp_rn(lt);
#pragma unroll
    for (int db = 0; db < 4; ++db) store_channels(p, st, row, db, inv, o[db]);
  }
}

// One prefill work item (query head h, query rows r0 .. r0 + rows - 1 of sequence b)
// executed by a whole workgroup of eight waves, 32 rows each.
//
// What bounds it: the matrix pipe and the softmax's vector work on the same
// SIMD, and, on long prefills, the card's power (large library products sustain
// 1.07 PFLOP/s in FP16 and 3.1 in FP8 there).  Run one after the
// other (QK, softmax, PV per tile, both waves of a SIMD in step at the tile
// barrier) they leave the matrix pipe 40 % busy.  So step j is software
// pipelined: the QK MFMAs of tile j-1 run among the exponentials of tile j,
// block by block in the same 64 score registers (block kb of tile j-1 takes the
// registers whose scores became P a moment before), and the PV MFMAs of tile j
// among the row maximum of tile j-1 and the exponentials of its first block.
// 32x32 MFMAs take half the instructions and operand registers of the 16x16
// ones, one query per lane halves the per-row softmax state, and constant LDS
// offsets and buffer loads keep the address registers few enough for the whole
// step to fit 256 registers.  Measured on one card: 131072 tokens, 40:8 heads 133.8 ->
// 121.4 ms (matrix pipe 40 -> 48 % busy, clock 2.38 -> 2.14 GHz), 16384 tokens, 32:8
// heads 1.80 -> 1.65 ms, MXFP4 65536 tokens, 40:8 heads 25.4 -> 22.5 ms.
//
// LDS buffers: K(j-1) and V(j) are read in step j; K(j-2) is stored over K(j)
// and V(j-1) over V(j+1), both read in step j+1, before its barrier.
template <int SEED, bool MX, int PV, int ABL = 0>
__device__ __forceinline__ void prefill_item(const PrefillParams& p, int b, int h, int r0, PrefillSmemT<MX, PV>& sm,
                                             int rows = kItemRows) {
  constexpr bool kSmooth = SEED != kSeedNone;
  // BF16 V: its 16 registers per thread are held only across the PV product
  // (across the whole step they spill)
  constexpr bool kLateV = PV == kPvBf16;
  ItemState st;
  item_setup<MX>(p, b, h, r0, rows, r0 + (int)(threadIdx.x >> 6) * kWaveRows, st);

  SoftState ss = {-INFINITY, 0.0f, 0.0f};
  f32x16 o[4];
#pragma unroll
  for (int db = 0; db < 4; ++db) o[db] = (f32x16){};

  const int32_t* ptab = p.page_table + (int64_t)st.b * p.max_pages;
  const int npg = (st.kvl + 63) >> 6;
  const int wv = __builtin_amdgcn_readfirstlane(st.wave);
  const int i = threadIdx.x & 255;   // unit of the page
  // the page of tile j that holds this wave's units, one per thread (clamped to a
  // mapped one for tiles outside the sequence, whose data is not used)
  const int half = wv >> 2;
  auto page = [&](int j) { return ptab[min(max(2 * j + half, 0), npg - 1)]; };
  KRegs kr;
  VRegs<PV> vr;
  // page of the next K tile to load (and, a step later, of its V tile): the
  // index is loaded a step before it is used
  int pgk, pgv, pgn;
  auto next_pages = [&](int j) {   // tile j's page starts to load, the one before becomes current
    pgv = pgk;
    pgk = __builtin_amdgcn_readfirstlane(pgn);
    pgn = page(j);
  };
  auto load_k = [&]() { fetch_k<MX, kSmooth>(kr, p, pgk, st.hk, st.h, i); };
  auto load_v = [&]() { fetch_v<PV>(vr, p, pgv, st.hk, i); };
  auto put_k = [&](int j) { store_k<SEED, MX, PV>(sm, j & 1, kr, st.seed_scale, half, i); };
  auto put_v = [&](int j, int nvalid) { store_v<MX, PV>(sm, j & 1, vr, half, i, nvalid); };
  const int j_hi = st.j_hi;
  pgk = page(j_hi);
  pgn = page(j_hi - 1);
  load_k();
  pgv = pgk;
  load_v();
  put_k(j_hi);
  next_pages(j_hi - 2);
  if (j_hi > 0) load_k();
  put_v(j_hi, st.kvl - j_hi * kTile);
  if (j_hi > 0) put_k(j_hi - 1);
  __syncthreads();
  if (!st.wave_active) {   // a wave without rows only moves its share of the tiles
    if (j_hi > 0) __syncthreads();
    for (int j = j_hi; j > 0; --j) {
      next_pages(j - 3);
      load_k();
      load_v();
      put_k(j - 2);
      put_v(j - 1, kTile);
      __syncthreads();
    }
    return;
  }

  f32x16 s[4];
  PTile pt;
#pragma unroll
  for (int kb = 0; kb < 4; ++kb) qk_block<SEED, MX, PV>(s[kb], kb, sm, j_hi & 1, st);
  if (j_hi > 0) __syncthreads();   // K of tile j_hi is read: the first step stores over it
  if (j_hi * kTile + kTile - 1 > st.wpos_min) mask_tile(s, j_hi * kTile, st);
  float alpha = max_tile<PV, ABL>(s, st, ss);
  float ps = exp_block<PV, ABL>(s[0], 0, st, ss, pt);
  for (int j = j_hi; j > 0; --j) {
    next_pages(j - 3);
    load_k();                    // tile j - 2
    if (!kLateV) load_v();       // tile j - 1
    const int kbuf = (j - 1) & 1;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int kb = 0; kb < 3; ++kb) {
      qk_block<SEED, MX, PV>(s[kb], kb, sm, kbuf, st);
      ps += exp_block<PV, ABL>(s[kb + 1], kb + 1, st, ss, pt);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (ABL < 2) ss.l = __builtin_fmaf(alpha, ss.l, ps);
    qk_block<SEED, MX, PV>(s[3], 3, sm, kbuf, st);
    put_k(j - 2);
    if (!kLateV) put_v(j - 1, kTile);
    __builtin_amdgcn_sched_barrier(0);
    if (j * kTile - 1 > st.wpos_min) mask_tile(s, (j - 1) * kTile, st);
    if (ABL < 2) rescale(o, alpha);
    if (kLateV) load_v();
    pv_tile<MX, PV>(sm, j & 1, pt, o, st);
    if (kLateV) put_v(j - 1, kTile);
    if (PV == kPvNvfp4) __builtin_amdgcn_sched_barrier(0);
    alpha = max_tile<PV, ABL>(s, st, ss);
    ps = exp_block<PV, ABL>(s[0], 0, st, ss, pt);
    __syncthreads();
  }
#pragma unroll
  for (int kb = 1; kb < 4; ++kb) ps += exp_block<PV, ABL>(s[kb], kb, st, ss, pt);
  if (ABL < 2) {
    ss.l = __builtin_fmaf(alpha, ss.l, ps);
    rescale(o, alpha);
  }
  pv_tile<MX, PV>(sm, 0, pt, o, st);
  // The scaled MFMA may otherwise be sunk into the row check of the store, where
  // lanes without a row are switched off and their operand rows read as zero.
#pragma unroll
  for (int db = 0; db < 4; ++db) asm volatile("" : "+v"(o[db]));
  store_output(p, st, ss.l, o);
}

// The item at position `bid` of the dispatch order (largest row tiles first).
template <int SEED, bool MX, int PV, int ABL = 0>
__device__ __forceinline__ void prefill_block(const PrefillParams& p, int bid, PrefillSmemT<MX, PV>& sm) {
  int b, h, rank;
  map_item(p, bid, b, h, rank);
  int tile = p.n_qtiles - 1 - rank;
  if (starts_differ(p) && !longest_item(p, rank * p.batch + b, b, tile)) return;
  const int r0 = tile * kItemRows;
  if (r0 >= p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b]) return;
  prefill_item<SEED, MX, PV, ABL>(p, b, h, r0, sm);
}

// Rows of the items that sequence b is cut into.  Of 128 rows, four waves compute (one
// per SIMD) and the other four only move their share of the tiles; such a step takes
// 1.75 us where one of 256 rows takes 2.9 (MXFP4 1.45, 2.2), so they are the better
// ones while all of them are resident at once (kHalfAll), and past that (kHalfAsk)
// while a compute unit's share of the tiles is not much more than the longest of them.
// 32:8 heads, 128 / 256 rows: 777 tokens 18.8 / 28 us, 777 behind 8000 132 / 203, 1600
// 36.3 / 45, 1600 behind 500 51.0 / 56.5, 1300 behind 1000 57.6 / 62.0, but 1300 behind
// 4000 142 / 129, 1600 behind 2000 93 / 90.
__device__ __forceinline__ int item_rows(const PrefillParams& p, int b) {
  if (p.half != kHalfAsk) return p.half == kHalfAll ? kHalfRows : kItemRows;
  int blocks = 0, tiles = 0;   // 128-row blocks of one head over the batch, and the KV tiles they visit
  for (int i = threadIdx.x & 63; i < p.batch; i += 64) {
    const int n = (p.cu_seqlens_q[i + 1] - p.cu_seqlens_q[i] + kHalfRows - 1) / kHalfRows;
    blocks += n;
    tiles += n * min(p.q_start[i] / kTile, 1 << 20) + n * (n + 1) / 2;
  }
  if (wave_sum_all(blocks) * p.h_q <= kComputeUnits) return kHalfRows;
  const float share = (float)wave_sum_all(tiles) * (float)p.h_q / kComputeUnits;
  const int longest = (p.q_start[b] + p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b] + kTile - 1) / kTile;
  return share <= 1.15f * (float)longest ? kHalfRows : kItemRows;
}

// Block blk of ROWS rows of sequence b, head h, whose items have `rows` rows.  An item is
// taken by its last block, the first of them in dispatch order; in a call of one sequence
// items of 256 rows by the last block of one of their halves, which of them changes every
// other item: the workgroups of an XCD are dealt to its four shader engines in turn, and
// with the working ones eight apart all ran on one of them (6000 rows behind 4000 tokens,
// 8:2 heads, 513 us; so 228).
template <int SEED, bool MX, int ROWS>
__device__ __forceinline__ void prefill_pick_block(const PrefillParams& p, int b, int h, int blk, int rows,
                                                   PrefillSmemT<MX, kPvFp8>& sm) {
  constexpr int kPer = kHalfRows / ROWS;
  const int nq = p.cu_seqlens_q[b + 1] - p.cu_seqlens_q[b];
  int item = blk / kPer;
  if (blk != min(item * kPer + kPer, (nq + ROWS - 1) / ROWS) - 1) return;
  if (rows == kItemRows) {
    const bool second = item & 1;
    item >>= 1;
    const bool pick = p.batch > 1 || ((item >> 1) & 1);
    if (second != (pick && item * kItemRows + kHalfRows < nq)) return;
  }
  prefill_item<SEED, MX, kPvFp8>(p, b, h, item * rows, sm, rows);
}

}  // namespace

}  // namespace mpfa
