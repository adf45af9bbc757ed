// Causal grouped-query attention over the paged KV cache.
//
// Cache geometry per layer: [num_blocks][n_kv][2][16 * d]; plane 0 holds K,
// plane 1 holds V, each as whole 1 KB MFMA operand fragments (kv_k_offset
// and kv_v_offset in packed.hpp).
//
// * attn_decode_bf16: one wave per (decode token, kv head, key split); the 16
//   MFMA rows are the G query heads sharing the kv head (padded to 16).
//     S^T[key][row] = K[key][:] . Q[row][:]        v_mfma_f32_16x16x32_bf16
//     O^T[d][row]  += V^T[d][key] . P^T[key][row]  v_mfma_f32_16x16x16_bf16
//   Every operand is one contiguous fragment load. The C layout of the first
//   product (lane l: row l%16, keys (l/16)*4 + r) is exactly the B layout
//   the second needs, and each lane keeps the online softmax statistics of
//   its own row (4-lane row reductions). A token's only split writes the
//   finished row; several splits leave (max, sum, unnormalised output) in a
//   workspace, and attn_merge_kernel combines them.
// * attn_decode_item_bf16: the same products, one 8-wave workgroup per (decode
//   token, kv head): the waves share the token's keys and combine in LDS.
// * attn_prefill_bf16: one 4-wave workgroup per (128 rows of a chunk, kv
//   head); rows are (position, head) pairs of the chunk, keys run from 0 to
//   the last position of the chunk (the chunk's own keys are already in the
//   cache), with the causal mask applied per row. Both products on
//   v_mfma_f32_32x32x16_bf16, with operands gathered per lane from the same
//   fragments (staged in LDS). Few, long chunks share an item's keys between
//   several workgroups, whose parts attn_prefill_merge combines.
// * attn_f32_kernel: the fp32 mode, prefill and decode rows alike: one
//   workgroup per (up to 16 (token, head) rows, kv head) on fp32 MFMA.
#include <type_traits>

#include "common.hpp"
#include "kernels.hpp"
#include "packed.hpp"

namespace stage_k {

namespace {

constexpr float kLog2e = 1.4426950408889634f;

// 2^x with the hardware instruction alone. Softmax arguments are <= 8 here
// and results below 2^-126 are negligible next to the row sum, so the
// denormal range handling of exp2f (several more instructions per value, on
// a path bound by these exponentials) is not needed.
__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }
// Online softmax: move the reference maximum only when a block's maximum
// exceeds it by more than this (log2 units).
constexpr float kLazyRescale = 8.0f;

__device__ __forceinline__ const int32_t* seq_table(const SegTables& t, int seq) {
  return seq < t.nseq0 ? t.bt0 + (size_t)seq * t.stride0
                       : t.bt1 + (size_t)(seq - t.nseq0) * t.stride1;
}

// Block ids of a wave's key range are read 64 at a time into one VGPR (lane
// i holds entry w + i) and taken back with v_readlane. A scalar load of each
// entry inside the key loop stalls the loop on every scalar-cache miss before
// the next block's loads can be issued; a conditional refill inside the loop
// makes the compiler wait for all outstanding loads at every readlane. So
// the key loop runs per window: refill, one wait, then the ping-pong over
// the window's blocks.
__device__ __forceinline__ int fill_window(const int32_t* bt, int w, int we, int lane) {
  const int ids = w + lane < we ? bt[w + lane] : 0;
  __builtin_amdgcn_s_waitcnt(0);
  return ids;
}

// K fragments of one 16-token block (kv_k_offset layout): fragment j, lane l
// = token l%16, d = j*32 + (l/16)*8 .. +7; each load reads 1 KB contiguously.
template <int D>
struct KFrag {
  static constexpr int NJ = D / 32;
  u32x4_t v[NJ];
  __device__ __forceinline__ void load(const bf16_t* kplane, int lane) {
    const bf16_t* p = kplane + lane * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) v[j] = ldg128(p + j * 512);
  }
  // streaming (non-temporal) variant for data read once
  __device__ __forceinline__ void load_nt(const bf16_t* kplane, int lane) {
    const bf16_t* p = kplane + lane * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) v[j] = __builtin_nontemporal_load((const u32x4_t*)(p + j * 512));
  }
};

// V^T fragments of one block (kv_v_offset layout): 1 KB fragment p, lane l
// holds d = 32p + l%16 (words 0-1) and d = 32p + 16 + l%16 (words 2-3), each
// for tokens (l/16)*4 .. +3.
template <int D>
struct VFrag {
  static constexpr int NP = D / 32;
  u32x4_t v[NP];
  __device__ __forceinline__ void load(const bf16_t* vplane, int lane) {
    const bf16_t* p = vplane + lane * 8;
#pragma unroll
    for (int j = 0; j < NP; ++j) v[j] = ldg128(p + j * 512);
  }
  __device__ __forceinline__ void load_nt(const bf16_t* vplane, int lane) {
    const bf16_t* p = vplane + lane * 8;
#pragma unroll
    for (int j = 0; j < NP; ++j) v[j] = __builtin_nontemporal_load((const u32x4_t*)(p + j * 512));
  }
  // A operand of d tile t (16 d values)
  __device__ __forceinline__ u32x2_t tile(int t) const {
    const u32x4_t& w = v[t >> 1];
    return (t & 1) ? u32x2_t{w[2], w[3]} : u32x2_t{w[0], w[1]};
  }
};

// Lanes l, l^16, l^32 and l^48 hold the same row of a 16x16 C tile; combine
// their values with the gfx950 lane swaps (VALU only, no LDS round trip).
// IEEE maximum (NaN-propagating): unlike fmaxf it needs no quieting of its
// operands, and chains of it become three-operand maximum instructions.
__device__ __forceinline__ float vmax(float a, float b) { return __builtin_elementwise_maximum(a, b); }

__device__ __forceinline__ float row4_max(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = vmax(__uint_as_float(a[0]), __uint_as_float(a[1]));
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return vmax(__uint_as_float(b[0]), __uint_as_float(b[1]));
}
__device__ __forceinline__ float row4_sum(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  x = __uint_as_float(a[0]) + __uint_as_float(a[1]);
  auto b = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(b[0]) + __uint_as_float(b[1]);
}

// Online-softmax state of the row owned by this lane (row l%16 of a tile).
struct RowState {
  float m, l;
};

// Process one key block for one 16-row tile: scores -> P -> O^T update.
// `s` holds the 4 raw scores (already scaled to log2 units and masked).
template <int D>
__device__ __forceinline__ void softmax_pv(f32x4_t s, RowState& st, f32x4_t* oacc,
                                           const VFrag<D>& vf) {
  const float bm = row4_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
  const float mn = fmaxf(st.m, bm);
  // A row can only be fully masked in a block after an earlier block gave it
  // a finite max, so mn is finite here. (No data-dependent branch here: a
  // branch inside the pipelined key loop makes the compiler wait for every
  // outstanding load at the join.)
  const float alpha = fast_exp2(st.m - mn);
  float p[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) p[r] = fast_exp2(s[r] - mn);
  const float ps = row4_sum(p[0] + p[1] + p[2] + p[3]);
  st.l = st.l * alpha + ps;
  st.m = mn;
  u32x2_t pb;
  pb[0] = pack_bf16x2(p[0], p[1]);
  pb[1] = pack_bf16x2(p[2], p[3]);
#pragma unroll
  for (int t = 0; t < D / 16; ++t) {
    oacc[t] *= alpha;
    oacc[t] = mfma16x16x16(vf.tile(t), pb, oacc[t]);
  }
}

// One wave over the 16-key blocks [b0, b1) of an item's keys for one kv head:
// unnormalised output and softmax state of the group's rows (none: st.m =
// -inf, zeros).
template <int D>
__device__ __forceinline__ void decode_blocks(const bf16_t* __restrict__ q,
                                              const bf16_t* __restrict__ kv, int n_kv,
                                              const SegTables& tabs, const DecodeItem& it, int kvh,
                                              int n_q, int b0, int b1, RowState& st,
                                              f32x4_t (&oacc)[D / 16]) {
  const int lane = threadIdx.x & 63;
  const int G = n_q / n_kv;
  const int row = lane & 15;  // query head within the group
  const bool row_ok = row < G;
  const float scale = kLog2e / sqrtf((float)D);

  // Q^T fragments (B operand): lane l holds head row, same d offsets as K.
  constexpr int NJ = D / 32;
  u32x4_t qf[NJ];
  {
    const bf16_t* qp = q + ((size_t)it.tok * n_q + kvh * G + (row_ok ? row : 0)) * D +
                       (lane >> 4) * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) qf[j] = row_ok ? ldg128(qp + j * 32) : u32x4_t{0u, 0u, 0u, 0u};
  }

  const int32_t* bt = seq_table(tabs, it.seq);
  const size_t plane = (size_t)kBlock * D;
  const size_t head_stride = 2 * plane;
  st = RowState{-INFINITY, 0.f};
#pragma unroll
  for (int t = 0; t < D / 16; ++t) oacc[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Two register sets in ping-pong (no copies between them), so a block's
  // loads stay in flight while the previous block is processed; the
  // prefetch index is clamped to the window's last block and its data is
  // unused.
  KFrag<D> kx, ky;
  VFrag<D> vx, vy;
  int w = 0, we = 0, ids = 0;
  auto load = [&](KFrag<D>& kf, VFrag<D>& vf, int b) {
    b = b < we ? b : we - 1;
    const bf16_t* kp = kv + ((size_t)__builtin_amdgcn_readlane(ids, b - w) * n_kv + kvh) * head_stride;
    // each (block, kv head) plane is read by exactly one wave of the step:
    // stream it (plain loads that allocate in the caches were ~15% slower)
    kf.load_nt(kp, lane);
    vf.load_nt(kp + plane, lane);
  };
  auto step = [&](const KFrag<D>& kf, const VFrag<D>& vf, int b) {
    f32x4_t s = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int j = 0; j < NJ; ++j) s = mfma16x16x32(kf.v[j], qf[j], s);
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int key = b * kBlock + (lane >> 4) * 4 + r;
      s[r] = key < it.k1 ? s[r] * scale : -INFINITY;
    }
    softmax_pv<D>(s, st, oacc, vf);
  };
  for (w = b0; w < b1; w += 64) {
    we = min(w + 64, b1);
    ids = fill_window(bt, w, we, lane);
    load(kx, vx, w);
    int b = w;
    for (; b + 1 < we; b += 2) {
      load(ky, vy, b + 1);
      __builtin_amdgcn_sched_barrier(0);
      step(kx, vx, b);
      __builtin_amdgcn_sched_barrier(0);
      load(kx, vx, b + 2);
      __builtin_amdgcn_sched_barrier(0);
      step(ky, vy, b + 1);
      __builtin_amdgcn_sched_barrier(0);
    }
    if (b < we) step(kx, vx, b);
  }
}

template <int D>
__global__ __launch_bounds__(256) void attn_decode_bf16(const bf16_t* __restrict__ q,
                                                        const bf16_t* __restrict__ kv, int n_kv,
                                                        SegTables tabs,
                                                        const DecodeItem* __restrict__ items,
                                                        const int32_t* __restrict__ order,
                                                        int n_items, int n_q,
                                                        float* __restrict__ part_o,
                                                        float* __restrict__ part_ml) {
  const int lane = threadIdx.x & 63;
  const int kvh = blockIdx.y * 4 + (threadIdx.x >> 6);
  if (kvh >= n_kv) return;
  const int idx = order[blockIdx.x];
  const DecodeItem it = items[idx];
  // items of one token are adjacent, from key 0 on: alone if the next item
  // starts at key 0 again
  const bool alone = it.k0 == 0 && (idx + 1 == n_items || items[idx + 1].k0 == 0);
  const int G = n_q / n_kv, row = lane & 15;
  RowState st;
  f32x4_t oacc[D / 16];
  decode_blocks<D>(q, kv, n_kv, tabs, it, kvh, n_q, it.k0 / kBlock, (it.k1 + kBlock - 1) / kBlock,
                   st, oacc);
  if (row >= G) return;
  if (alone) {
    const float inv = 1.0f / st.l;
    bf16_t* out = (bf16_t*)tabs.attn_out;
    const int col = (kvh * G + row) * D + (lane >> 4) * 4;
#pragma unroll
    for (int t = 0; t < D / 16; ++t) {
      u32x2_t w;
      w[0] = pack_bf16x2(oacc[t][0] * inv, oacc[t][1] * inv);
      w[1] = pack_bf16x2(oacc[t][2] * inv, oacc[t][3] * inv);
      *(u32x2_t*)(out + packed_a_offset(it.tok, col + t * 16, n_q * D)) = w;
    }
    return;
  }
  const size_t ob = ((size_t)idx * n_q + kvh * G + row);
  float* po = part_o + ob * D;
#pragma unroll
  for (int t = 0; t < D / 16; ++t)
    *(f32x4_t*)(po + t * 16 + (lane >> 4) * 4) = oacc[t];
  if (lane < 16) {
    part_ml[ob * 2 + 0] = st.m;
    part_ml[ob * 2 + 1] = st.l;
  }
}

// Items that hold all keys of their token, one workgroup of kItemWaves waves
// per (item, kv head): each wave takes an eighth of the blocks and the parts
// meet in LDS, so that a small step of middling contexts needs neither
// partials in memory nor the merge's launch. (Not for long contexts or large
// batches, where splits of equal size over the whole chip balance better.)
constexpr int kItemWaves = 8;

template <int D>
__global__ __launch_bounds__(kItemWaves * 64) void attn_decode_item_bf16(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ kv, int n_kv, SegTables tabs,
    const DecodeItem* __restrict__ items, const int32_t* __restrict__ order, int n_q) {
  constexpr int NW = kItemWaves;
  __shared__ float2 s_ml[NW][16];
  __shared__ f32x4_t s_o[NW][16][D / 4 + 1];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kvh = blockIdx.y, G = n_q / n_kv, row = lane & 15;
  const DecodeItem it = items[order[blockIdx.x]];
  const int nb = (it.k1 + kBlock - 1) / kBlock, per = (nb + NW - 1) / NW;
  RowState st;
  f32x4_t oacc[D / 16];
  decode_blocks<D>(q, kv, n_kv, tabs, it, kvh, n_q, min(wave * per, nb), min((wave + 1) * per, nb),
                   st, oacc);
  if (lane < 16) s_ml[wave][row] = make_float2(st.m, st.l);
#pragma unroll
  for (int t = 0; t < D / 16; ++t) s_o[wave][row][t * 4 + (lane >> 4)] = oacc[t];
  __syncthreads();
  for (int e = threadIdx.x; e < G * D / 4; e += NW * 64) {
    const int r = e / (D / 4), c = e % (D / 4);
    float M = s_ml[0][r].x;  // wave 0 has at least one block
#pragma unroll
    for (int w = 1; w < NW; ++w) M = fmaxf(M, s_ml[w][r].x);
    float l = 0.f;
    f32x4_t o = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int w = 0; w < NW; ++w) {
      const float f = exp2f(s_ml[w][r].x - M);
      l += f * s_ml[w][r].y;
      o += f * s_o[w][r][c];
    }
    o *= 1.0f / l;
    u32x2_t v;
    v[0] = pack_bf16x2(o[0], o[1]);
    v[1] = pack_bf16x2(o[2], o[3]);
    *(u32x2_t*)((bf16_t*)tabs.attn_out +
                packed_a_offset(it.tok, (kvh * G + r) * D + 4 * c, n_q * D)) = v;
  }
}

// Combine the key splits of each decode token. WPT waves per (token, kv
// head): wave w takes splits 4 w .. 4 w + 3, then the 4 WPT further on. Lane l
// serves query head row l / LPR of the group and DPL consecutive d values (a
// multiple of 4). Bound by latency: a wave's chain is one memory round trip
// per 4 splits, so batches that are small enough to leave CUs free (and whose
// tokens then have many splits) share the chain between waves: one token of 8
// kv heads, 11.7 us for 32 splits with one wave each, 6.8 for 55 with eight;
// 32 tokens of 14 splits and one kv head 6.1 -> 4.2.
template <int D, int G, int WPT>
__global__ __launch_bounds__(WPT == 1 ? 256 : WPT * 64) void attn_merge_kernel(
    const float* __restrict__ part_o, const float* __restrict__ part_ml,
    const int32_t* __restrict__ item_start, const int32_t* __restrict__ tok_rows, int n_q,
    int n_kv, bf16_t* __restrict__ out) {
  constexpr int LPR = (64 / G) < (D / 4) ? (64 / G) : (D / 4);  // lanes per head row
  constexpr int DPL = D / LPR;                                    // d values per lane
  __shared__ float2 s_ml[WPT][G];
  __shared__ float4 s_o[WPT > 1 ? WPT : 1][WPT > 1 ? G * D / 4 : 1];
  const int t = blockIdx.x;
  const int wave = threadIdx.x >> 6, lane = threadIdx.x & 63;
  const int kvh = WPT > 1 ? blockIdx.y : blockIdx.y * 4 + wave;
  const int i0 = item_start[t], i1 = item_start[t + 1];
  if (i1 - i0 == 1) return;  // written by its item
  const bool on = lane < G * LPR;
  if (WPT == 1 && (kvh >= n_kv || !on)) return;
  const int h = kvh * G + (on ? lane / LPR : 0);
  const int d0 = (lane % LPR) * DPL;
  // Online merge over chunks of 4 splits: a chunk's loads are all issued
  // before any is used (indices past the last split are clamped and masked).
  float M = -INFINITY, L = 0.f;
  float4 o[DPL / 4];
#pragma unroll
  for (int c = 0; c < DPL / 4; ++c) o[c] = make_float4(0.f, 0.f, 0.f, 0.f);
  for (int i = i0 + (WPT > 1 ? 4 * wave : 0); i < i1; i += 4 * WPT) {
    float mu[4], lu[4];
    float4 v[4][DPL / 4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t b = (size_t)min(i + u, i1 - 1) * n_q + h;
      mu[u] = part_ml[b * 2];
      lu[u] = part_ml[b * 2 + 1];
      const float4* po = (const float4*)(part_o + b * D + d0);
#pragma unroll
      for (int c = 0; c < DPL / 4; ++c) v[u][c] = po[c];
    }
    float cm = M;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (i + u < i1) cm = fmaxf(cm, mu[u]);
    const float sc = exp2f(M - cm);  // 0 for the first chunk (M = -inf)
    L *= sc;
#pragma unroll
    for (int c = 0; c < DPL / 4; ++c) {
      o[c].x *= sc;
      o[c].y *= sc;
      o[c].z *= sc;
      o[c].w *= sc;
    }
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float w = i + u < i1 ? exp2f(mu[u] - cm) : 0.f;
      L += w * lu[u];
#pragma unroll
      for (int c = 0; c < DPL / 4; ++c) {
        o[c].x += w * v[u][c].x;
        o[c].y += w * v[u][c].y;
        o[c].z += w * v[u][c].z;
        o[c].w += w * v[u][c].w;
      }
    }
    M = cm;
  }
  const int row = tok_rows[t], K = n_q * D;
  if constexpr (WPT == 1) {
    const float inv = 1.0f / L;
#pragma unroll
    for (int c = 0; c < DPL / 4; ++c) {
      u32x2_t wv;
      wv[0] = pack_bf16x2(o[c].x * inv, o[c].y * inv);
      wv[1] = pack_bf16x2(o[c].z * inv, o[c].w * inv);
      *(u32x2_t*)(out + packed_a_offset(row, h * D + d0 + 4 * c, K)) = wv;
    }
  } else {
    // the waves' parts; a wave without splits has M = -inf and weight 0
    // (wave 0 always has some, so the common maximum is one of the splits')
    const int r = lane / LPR;
    if (on && lane % LPR == 0) s_ml[wave][r] = make_float2(M, L);
    if (on) {
#pragma unroll
      for (int c = 0; c < DPL / 4; ++c) s_o[wave][(r * D + d0) / 4 + c] = o[c];
    }
    __syncthreads();
    for (int e = threadIdx.x; e < G * D / 4; e += WPT * 64) {
      const int er = e / (D / 4);
      float cm = s_ml[0][er].x;
#pragma unroll
      for (int w = 1; w < WPT; ++w) cm = fmaxf(cm, s_ml[w][er].x);
      float l = 0.f;
      float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll
      for (int w = 0; w < WPT; ++w) {
        const float f = exp2f(s_ml[w][er].x - cm);
        l += f * s_ml[w][er].y;
        const float4 b = s_o[w][e];
        a.x += f * b.x;
        a.y += f * b.y;
        a.z += f * b.z;
        a.w += f * b.w;
      }
      const float inv = 1.0f / l;
      u32x2_t wv;
      wv[0] = pack_bf16x2(a.x * inv, a.y * inv);
      wv[1] = pack_bf16x2(a.z * inv, a.w * inv);
      *(u32x2_t*)(out + packed_a_offset(row, kvh * G * D + 4 * e, K)) = wv;
    }
  }
}

// Prefill: one workgroup of kPfWaves waves per (item, kv head). Row r of
// the workgroup (r < kPfWaves * 32) is query position r / G of the item and
// head kvh*G + r % G; wave w owns rows 32w .. 32w + 31 as one 32-row tile of
// v_mfma_f32_32x32x16_bf16 (lane l: row l % 32). Keys run in stages of BPS
// 16-token blocks: each stage's K and V fragments are copied once into LDS
// (direct loads, two buffers each; K two stages ahead, V one) and read by all
// waves, so a key is fetched once per workgroup instead of once per 32 rows.
// The score products of a stage run between the exponentials of the stage
// before it, in program order, so that a wave overlaps its own matrix and
// vector work and the LDS reads of K hide behind both (one stage at a time,
// the two waves of a SIMD mostly alternated: 2048 rows behind 61440 keys 4217
// us with MFMA busy 54%, now 4050). Scores of a whole stage
// are reduced together; the running maximum is only moved (and the
// accumulators rescaled) when it grows by more than 2^8, so P stays below
// 256 and the rescale is rare after the first stage.
//
// The 32x32x16 form: one wave alone keeps the MFMA pipe nearly full with it
// (2.37 PFLOP/s in a probe, against 1.4 for 16x16x32), which matters here
// because a wave's MFMA work alternates with its softmax arithmetic.
//   S^T[key][row] (32 keys = two blocks x 32 rows): A = K, lane l: key l % 32
//     (block (l / 16) % 2, token l % 16), d 16 ds + 8 (l / 32) .. + 7, read
//     per lane from the blocks' K fragments; B = Q^T, lane l: row l % 32,
//     the same d. C, lane l, value v: row l % 32, key 8 (v / 4) + 4 (l / 32)
//     + v % 4.
//   O^T[d][row] += V^T[d][key] P^T[key][row], 16 keys (one block z of the
//     pair) per product: B = P^T is values 8z .. 8z + 7 of the lane's S^T
//     tile as they stand (k index 8 (l / 32) + e <-> key 8 (e / 4) + 4 (l /
//     32) + e % 4), and A = V^T, lane l: d 32 t + l % 32, the same keys: two
//     8-byte pieces of the block's V fragment t.
constexpr int kPfWaves = 4;
constexpr int kPfBPS = 4;
static_assert(kPfWaves * 32 == kPrefillRows, "rows of a prefill work item");

typedef __attribute__((address_space(3))) void* lds_ptr_t;

__device__ __forceinline__ float row2_max(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return vmax(__uint_as_float(a[0]), __uint_as_float(a[1]));
}
__device__ __forceinline__ float row2_sum(float x) {
  auto a = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  return __uint_as_float(a[0]) + __uint_as_float(a[1]);
}

// Two workgroups per CU (64 KB of LDS each) need the register budget of two
// waves per SIMD; one would leave no other wave to overlap a wave's
// exponentials with MFMA work.
template <int D>
__global__ __launch_bounds__(kPfWaves * 64) __attribute__((amdgpu_waves_per_eu(2)))
void attn_prefill_bf16(
    const bf16_t* __restrict__ q, const bf16_t* __restrict__ kv, int n_kv, SegTables tabs,
    const PrefillItem* __restrict__ items, int n_q, bf16_t* __restrict__ out) {
  constexpr int BPS = kPfBPS;
  static_assert(BPS * kBlock == kPrefillStage, "keys per stage");
  constexpr int NJ = D / 32;           // K fragments per block (and V fragments)
  constexpr int KF = BPS * NJ;         // K fragments per stage (and V fragments)
  constexpr int PER = KF / kPfWaves;   // K copies per wave and stage (and V copies)
  constexpr int NP = BPS / 2;          // 32-key tiles per stage
  constexpr int ND = D / 16;           // 16-wide d slices (score products per tile)
  constexpr int NT = D / 32;           // 32-wide d tiles of O^T
  static_assert(KF % kPfWaves == 0, "stage split");
  static_assert(BPS % 2 == 0, "score tiles take key blocks in pairs");
  __shared__ u32x4_t lds[4][KF * 64];  // K of even and odd stages, then V
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int l32 = lane & 31, hi = lane >> 5;
  // Workgroup b runs on XCD b % 8, each XCD with its own L2. Take the kv head
  // from the linear id modulo n_kv, so every XCD serves a fixed set of kv
  // heads and a sequence's K/V for one head is pulled into one L2 only (not
  // into all eight); items stay in their longest-first order.
  const int lin = blockIdx.x + blockIdx.y * gridDim.x;
  const int kvh = lin % n_kv;
  const PrefillItem it = items[lin / n_kv];
  const int G = n_q / n_kv;
  const float scale = kLog2e / sqrtf((float)D);

  const int r = wave * 32 + l32;  // this lane's row of the workgroup
  const int pi = r / G;
  const bool rok = pi < it.npos;
  const int pc = rok ? pi : it.npos - 1;
  const int rpos = it.p0 + pc;    // its position
  u32x4_t qf[ND];
  {
    const bf16_t* qp = q + ((size_t)(it.t0 + pc) * n_q + kvh * G + r % G) * D + hi * 8;
#pragma unroll
    for (int s = 0; s < ND; ++s) qf[s] = ldg128(qp + s * 16);
  }

  const int32_t* bt = seq_table(tabs, it.seq);
  const size_t plane = (size_t)kBlock * D;
  const int kend = it.p0 + it.npos;  // keys [0, kend)
  const int nb = (kend + kBlock - 1) / kBlock;
  // the stages [s0, nst) of this block (all of them unless the step is split)
  int s0 = 0, nst = (nb + BPS - 1) / BPS;
  const int parts = prefill_parts(tabs.parts.stages, it.p0, nst);
  if ((int)blockIdx.z >= parts) return;
  if (parts > 1) {
    s0 = blockIdx.z * tabs.parts.stages;
    if ((int)blockIdx.z + 1 < parts) nst = s0 + tabs.parts.stages;
  }

  RowState st{-INFINITY, 0.f};
  f32x16_t oacc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int v = 0; v < 16; ++v) oacc[t][v] = 0.f;

  // Block ids, 64 at a time (a multiple of BPS, so a stage never straddles
  // two windows). `window` before the copies of a stage that may open a new one.
  int wbase = 0, ids = 0;
  auto window = [&](int stg) {
    if (stg * BPS - wbase >= 64) {
      wbase = stg * BPS;
      ids = fill_window(bt, wbase, min(wbase + 64, nb), lane);
    }
  };
  // copies of a stage's K (plane 0) or V (plane 1) fragments into LDS
  auto issue = [&](int stg, int vp) {
    const int buf = 2 * vp + (stg & 1);
#pragma unroll
    for (int p = 0; p < PER; ++p) {
      const int f = wave * PER + p;
      int b = stg * BPS + f / NJ;
      b = b < nb ? b : nb - 1;  // past the end: a valid block, never used
      const bf16_t* src = kv + ((size_t)__builtin_amdgcn_readlane(ids, b - wbase) * n_kv + kvh) *
                                   (2 * plane) +
                          vp * plane + (f % NJ) * 512 + lane * 8;
      __builtin_amdgcn_global_load_lds((const void*)src, (lds_ptr_t)&lds[buf][f * 64], 16, 0, 0);
    }
  };

  // lane offsets inside a block's fragments (u32x4 units): K of d slice s
  // at (s / 2) * 64 + kslot + 32 (s % 2) of block 2 tile + kblk; V pieces
  // at vslot and vslot + 32 (in 8-byte units, half vhalf)
  const int kblk = (lane >> 4) & 1;
  const int kslot = (lane & 15) + 16 * hi;
  const int vslot = (lane & 15) + 16 * hi, vhalf = (lane >> 4) & 1;

  // operand and product number i of a stage's raw scores (one 32-key tile per
  // pair of blocks)
  auto kload = [&](const u32x4_t* L, int i) {
    const int sl = i / NP, t = i % NP;
    return L[((2 * t + kblk) * NJ + sl / 2) * 64 + kslot + 32 * (sl % 2)];
  };
  auto score = [&](f32x16_t (&sc)[NP], u32x4_t kf, int i) {
    if (i < NP) {
#pragma unroll
      for (int v = 0; v < 16; ++v) sc[i][v] = 0.f;
    }
    sc[i % NP] = mfma32x32x16(kf, qf[i / NP], sc[i % NP]);
  };

  // One stage of BPS key blocks, whose raw scores are in sc. The scores of the
  // next stage (`more`) go to sn, their products between this stage's
  // exponentials. Stages whose last key is at or before the first query
  // position of the item need no causal mask (for a long context, nearly all).
  auto stage = [&](auto masked, auto more, int stg, f32x16_t (&sc)[NP], f32x16_t (&sn)[NP]) {
    constexpr bool kMask = decltype(masked)::value, kMore = decltype(more)::value;
    if constexpr (kMore) {
      issue(stg + 1, 1);
      if (stg + 2 < nst) {
        window(stg + 2);
        issue(stg + 2, 0);
      }
    }
    if constexpr (kMask) {
#pragma unroll
      for (int t = 0; t < NP; ++t)
#pragma unroll
        for (int v = 0; v < 16; ++v) {
          const int key = (stg * BPS + 2 * t) * kBlock + 8 * (v >> 2) + 4 * hi + (v & 3);
          sc[t][v] = key <= rpos ? sc[t][v] : -INFINITY;
        }
    }
    // softmax statistics of the stage (log2 units: score * scale), then P
    float bm = -INFINITY;
#pragma unroll
    for (int t = 0; t < NP; ++t)
#pragma unroll
      for (int v = 0; v < 16; ++v) bm = vmax(bm, sc[t][v]);
    bm = row2_max(bm) * scale;
    const bool grow = bm > st.m + kLazyRescale;
    const float mn = grow ? bm : st.m;
    const float alpha = fast_exp2(st.m - mn);  // exactly 1 unless the maximum moved
    if (__builtin_amdgcn_ballot_w64(grow) != 0) {
#pragma unroll
      for (int t = 0; t < NT; ++t) oacc[t] *= alpha;
    }
    // P and, product by product between its arithmetic, the next stage's
    // scores: one product, the read of the operand KD products further on,
    // and EP exponentials, in this order (the scheduling barriers keep it).
    constexpr int MF = ND * NP, KD = 4, EP = NP * 16 / MF;
    const u32x4_t* LK = lds[(stg + 1) & 1];
    u32x4_t kf[MF];
    if constexpr (kMore) {
#pragma unroll
      for (int i = 0; i < KD; ++i) kf[i] = kload(LK, i);
    }
    u32x4_t pb[NP][2];
    float ps = 0.f;
#pragma unroll
    for (int i = 0; i < MF; ++i) {
      if constexpr (kMore) {
        __builtin_amdgcn_sched_barrier(0);
        score(sn, kf[i], i);
        if (i + KD < MF) kf[i + KD] = kload(LK, i + KD);
      }
#pragma unroll
      for (int e = 0; e < EP; e += 2) {
        const int v = i * EP + e, t = v / 16, u = v % 16;
        const float p0 = fast_exp2(fmaf(sc[t][u], scale, -mn));
        const float p1 = fast_exp2(fmaf(sc[t][u + 1], scale, -mn));
        ps += p0 + p1;
        pb[t][u / 8][u % 8 / 2] = pack_bf16x2(p0, p1);
      }
    }
    __builtin_amdgcn_sched_barrier(0);
    st.l = st.l * alpha + row2_sum(ps);
    st.m = mn;
    // O^T += V^T P^T, block by block. The two 8-byte pieces of each V^T
    // operand are read from LDS straight into adjacent registers (volatile
    // reads, so that the compiler does not merge them with neighbouring
    // pieces and then assemble the operands with register moves).
    typedef const volatile u32x2_t __attribute__((address_space(3)))* lds_u32x2_ptr;
    const lds_u32x2_ptr L2 = (lds_u32x2_ptr)lds[2 + (stg & 1)];
    auto vload = [&](int blk, int t) {
      const int f = blk * NJ + t;
      const u32x2_t a0 = L2[(f * 64 + vslot) * 2 + vhalf];
      const u32x2_t a1 = L2[(f * 64 + vslot + 32) * 2 + vhalf];
      return u32x4_t{a0[0], a0[1], a1[0], a1[1]};
    };
    // Groups g of two products (one block, two d tiles); the V operands of
    // group g + 2 are read while the products of group g run.
    constexpr int NG = BPS * NT / 2, PD = 2;
    u32x4_t va[PD + 1], vb[PD + 1];
    auto vgroup = [&](int g) {
      const int blk = g / (NT / 2), t = 2 * (g % (NT / 2));
      va[g % (PD + 1)] = vload(blk, t);
      vb[g % (PD + 1)] = vload(blk, t + 1);
    };
#pragma unroll
    for (int g = 0; g < PD; ++g) vgroup(g);
    // The compiler's scheduler would otherwise move each read down to just
    // before its product (fewest live registers); these group barriers keep
    // the order: the first PD groups' reads, then per group the reads of
    // group g + PD followed by the products of group g.
    __builtin_amdgcn_sched_group_barrier(0x100, 4 * PD, 0);
#pragma unroll
    for (int g = 0; g < NG; ++g) {
      if (g + PD < NG) vgroup(g + PD);
      const int blk = g / (NT / 2), t = 2 * (g % (NT / 2));
      const u32x4_t pp = pb[blk / 2][blk % 2];
      oacc[t] = mfma32x32x16(va[g % (PD + 1)], pp, oacc[t]);
      oacc[t + 1] = mfma32x32x16(vb[g % (PD + 1)], pp, oacc[t + 1]);
      if (g + PD < NG) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);  // 4 LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);                    // then the MFMAs
    }
    __builtin_amdgcn_s_waitcnt(0);  // the copies have landed in LDS
    __syncthreads();
  };

  wbase = s0 * BPS;
  ids = fill_window(bt, wbase, min(wbase + 64, nb), lane);
  issue(s0, 0);
  issue(s0, 1);
  if (s0 + 1 < nst) issue(s0 + 1, 0);  // (a stage is never a window's last)
  __builtin_amdgcn_s_waitcnt(0);
  __syncthreads();
  f32x16_t sa[NP], sb[NP];
#pragma unroll
  for (int i = 0; i < ND * NP; ++i) score(sa, kload(lds[s0 & 1], i), i);
  __syncthreads();  // every wave has read the first K
  const int nfull = min(nst, (it.p0 + 1) / (BPS * kBlock));
  // stages in pairs, their scores alternating between sa and sb
  const std::true_type yes{};
  const std::false_type no{};
  int stg = s0;
  for (; stg + 1 < min(nfull, nst - 1); stg += 2) {
    stage(no, yes, stg, sa, sb);
    stage(no, yes, stg + 1, sb, sa);
  }
  for (; stg + 1 < nst; ++stg) {
    stage(yes, yes, stg, sa, sb);
#pragma unroll
    for (int t = 0; t < NP; ++t) sa[t] = sb[t];
  }
  stage(yes, no, stg, sa, sb);

  if (!rok) return;
  if (parts > 1) {
    // [d / 8][row][d % 8] of unnormalised output, then (max, sum) per row
    float* po = tabs.parts.buf +
                (((size_t)blockIdx.z * n_kv + kvh) * gridDim.x + lin / n_kv) * prefill_part_floats(D);
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
      for (int qd = 0; qd < 4; ++qd)
        *(f32x4_t*)(po + ((size_t)(t * 4 + qd) * kPrefillRows + r) * 8 + 4 * hi) =
            f32x4_t{oacc[t][4 * qd], oacc[t][4 * qd + 1], oacc[t][4 * qd + 2], oacc[t][4 * qd + 3]};
    if (hi == 0) *(float2*)(po + kPrefillRows * D + 2 * r) = make_float2(st.m, st.l);
    return;
  }
  const float inv = 1.0f / st.l;
  // packed activation layout (the O projection's input); 4 consecutive
  // columns share one 8-byte piece of a fragment lane
  const int row = it.t0 + pi;
  const int col0 = (kvh * G + r % G) * D + 4 * hi;
#pragma unroll
  for (int t = 0; t < NT; ++t)
#pragma unroll
    for (int qd = 0; qd < 4; ++qd) {
      u32x2_t w;
      w[0] = pack_bf16x2(oacc[t][4 * qd] * inv, oacc[t][4 * qd + 1] * inv);
      w[1] = pack_bf16x2(oacc[t][4 * qd + 2] * inv, oacc[t][4 * qd + 3] * inv);
      *(u32x2_t*)(out + packed_a_offset(row, col0 + 32 * t + 8 * qd, n_q * D)) = w;
    }
}

// Combine the parts of split prefill items: grid (item, kv head, 8-column
// group); a thread takes 4 of the 8 columns of one row, in the layout the
// parts were written in.
template <int D>
__global__ __launch_bounds__(2 * kPrefillRows) void attn_prefill_merge(
    SegTables tabs, const PrefillItem* __restrict__ items, int n_q, bf16_t* __restrict__ out) {
  const int n_items = gridDim.x, n_kv = gridDim.y, kvh = blockIdx.y;
  const PrefillItem it = items[blockIdx.x];
  const int nst = (it.p0 + it.npos + kPrefillStage - 1) / kPrefillStage;
  const int parts = prefill_parts(tabs.parts.stages, it.p0, nst);
  const int r = threadIdx.x >> 1, hi = threadIdx.x & 1;
  const int G = n_q / n_kv, pi = r / G;
  if (parts == 1 || pi >= it.npos) return;
  const size_t step = (size_t)n_kv * n_items * prefill_part_floats(D);
  const float* po = tabs.parts.buf + ((size_t)kvh * n_items + blockIdx.x) * prefill_part_floats(D);
  const float* pm = po + kPrefillRows * D + 2 * r;
  po += ((size_t)blockIdx.z * kPrefillRows + r) * 8 + 4 * hi;
  float M = -INFINITY, L = 0.f;
  f32x4_t o = f32x4_t{0.f, 0.f, 0.f, 0.f};
  for (int i = 0; i < parts; i += 4) {  // 4 parts' loads in flight
    float2 ml[4];
    f32x4_t v[4];
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const size_t off = (size_t)min(i + u, parts - 1) * step;
      ml[u] = *(const float2*)(pm + off);
      v[u] = *(const f32x4_t*)(po + off);
    }
    float cm = M;
#pragma unroll
    for (int u = 0; u < 4; ++u) cm = fmaxf(cm, ml[u].x);
    const float sc = exp2f(M - cm);
    L *= sc;
    o *= sc;
#pragma unroll
    for (int u = 0; u < 4; ++u) {
      const float w = i + u < parts ? exp2f(ml[u].x - cm) : 0.f;
      L += w * ml[u].y;
      o += w * v[u];
    }
    M = cm;
  }
  o *= 1.0f / L;
  u32x2_t w;
  w[0] = pack_bf16x2(o[0], o[1]);
  w[1] = pack_bf16x2(o[2], o[3]);
  *(u32x2_t*)(out + packed_a_offset(it.t0 + pi, (kvh * G + r % G) * D + 8 * blockIdx.z + 4 * hi,
                                    n_q * D)) = w;
}

// fp32 mode, prefill and decode rows alike: one workgroup of kF32Waves waves
// per (P consecutive tokens, kv head, run); its rows (at most 16) are the tokens'
// (token, head) pairs. A run is the tokens of one sequence among the P; each
// run has a block of its own (blockIdx.z; the blocks past the last run leave
// at once), so that neither its chain of keys nor its values mix with another
// request's. Wave w takes every kF32Waves-th 16-key block, in fp32
// throughout, on v_mfma_f32_16x16x4_f32:
//   S^T[key][row]: A = K, lane l: key l % 16, B = Q^T, lane l: row l % 16,
//     step (j, e): d 32 j + 8 (l / 16) + e, the 8 consecutive floats the lane
//     holds of K fragment j. C, lane l, value r: row l % 16, key 4 (l / 16) + r.
//   O^T[d][row] += V^T P^T, step r: B = value r of the S^T tile as it stands,
//     A = V^T, lane l: d 16 t + l % 16, the same key: of the lane's 8 floats
//     of V fragment t / 2, number 4 (t % 2) + r.
// The waves' (max, sum, output) are combined through LDS at the end. The fp32
// mode's batches are small, so what bounds it is the chain of one row's keys:
// eight waves share it, and a key that is read serves up to 16 rows. 454 rows
// of 8 heads, up to 900 keys each: 117 us with one wave per (token, head), 45
// with the runs of a block one after another, 26 with a block per run.
constexpr int kF32Waves = 8;

template <int D>
__global__ __launch_bounds__(kF32Waves * 64) void attn_f32_kernel(
    const float* __restrict__ q, const float* __restrict__ kv, int n_kv, SegTables tabs,
    const int32_t* __restrict__ tok_seq, const int32_t* __restrict__ tok_pos, int t_begin,
    int t_end, int P, int n_q, float* __restrict__ out) {
  constexpr int NW = kF32Waves, NJ = D / 32, NT = D / 16;
  __shared__ float s_ml[NW][2][16];
  __shared__ float s_o[NW / 2][16][D + 4];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int kvh = blockIdx.y;
  int t0 = t_begin + blockIdx.x * P, np = min(P, t_end - t0);
  for (int z = 0;; ++z) {  // tokens [t0, t0 + np): this block's run
    int r1 = 1;
    while (r1 < np && tok_seq[t0 + r1] == tok_seq[t0]) ++r1;
    if (z == (int)blockIdx.z) {
      np = r1;
      break;
    }
    if (r1 == np) return;  // fewer runs than blocks
    t0 += r1;
    np -= r1;
  }
  const int G = n_q / n_kv;
  const float scale = 1.0f / sqrtf((float)D);
  const int row = lane & 15, quad = lane >> 4;
  const int rt = row / G;               // this row's token of the run
  const int tc = t0 + min(rt, np - 1);  // (rows past the run are masked, and not stored)
  const int rpos = rt < np ? tok_pos[tc] : -1;
  f32x4_t qf[NJ][2];
  {
    const float* qp = q + ((size_t)tc * n_q + kvh * G + row % G) * D + quad * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      qf[j][0] = *(const f32x4_t*)(qp + j * 32);
      qf[j][1] = *(const f32x4_t*)(qp + j * 32 + 4);
    }
  }
  const size_t plane = (size_t)kBlock * D;
  float m = -INFINITY, l = 0.f;
  f32x4_t o[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) o[t] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  const int32_t* bt = seq_table(tabs, tok_seq[t0]);
  // positions grow along a run, so its last token sees the most keys
  const int first = tok_pos[t0], last = tok_pos[t0 + np - 1];
  const int nb = last / kBlock + 1;
  // K is loaded a block ahead, V at the start of its block
  f32x4_t kf[NJ][2], vf[NJ][2], kn[NJ][2];
  const float *vp = nullptr, *vn = nullptr;
  int ids = 0, w0 = 0;  // lane i: id of this wave's block number w0 + i
  auto load = [&](int b) {
    const int i = (b - wave) / NW;
    if (i - w0 >= 64 || i == 0) {
      w0 = i;
      ids = bt[min(b + lane * NW, nb - 1)];
    }
    const int id = __builtin_amdgcn_readlane(ids, i - w0);
    const float* kp = kv + ((size_t)id * n_kv + kvh) * 2 * plane + lane * 8;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      kn[j][0] = *(const f32x4_any_t*)(kp + j * 512);
      kn[j][1] = *(const f32x4_any_t*)(kp + j * 512 + 4);
    }
    vn = kp + plane;
  };
  if (wave < nb) load(wave);
  for (int b = wave; b < nb; b += NW) {
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      kf[j][0] = kn[j][0];
      kf[j][1] = kn[j][1];
    }
    vp = vn;
#pragma unroll
    for (int j = 0; j < NJ; ++j) {
      vf[j][0] = *(const f32x4_any_t*)(vp + j * 512);
      vf[j][1] = *(const f32x4_any_t*)(vp + j * 512 + 4);
    }
    if (b + NW < nb) load(b + NW);
    // two chains of products, so that one's latency hides behind the other
    f32x4_t s0 = f32x4_t{0.f, 0.f, 0.f, 0.f}, s1 = s0;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        s0 = mfma16x16x4(kf[j][0][e], qf[j][0][e], s0);
        s1 = mfma16x16x4(kf[j][1][e], qf[j][1][e], s1);
      }
    float sc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r)
      sc[r] = b * kBlock + quad * 4 + r <= rpos ? (s0[r] + s1[r]) * scale : -INFINITY;
    const float bm = row4_max(fmaxf(fmaxf(sc[0], sc[1]), fmaxf(sc[2], sc[3])));
    const float mn = fmaxf(m, bm);
    // a row whose keys are all masked so far keeps weight 0 everywhere
    const float ref = mn == -INFINITY ? 0.f : mn;
    const float alpha = expf(m - ref);
    float p[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) p[r] = expf(sc[r] - ref);
    l = l * alpha + row4_sum((p[0] + p[1]) + (p[2] + p[3]));
    m = mn;
    auto pv = [&](bool take) {  // other rows keep their output
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        f32x4_t n = o[t] * alpha;
#pragma unroll
        for (int r = 0; r < 4; ++r) n = mfma16x16x4(vf[t / 2][t % 2][r], p[r], n);
        o[t] = take ? n : o[t];
      }
    };
    // drop the values of keys past `end` (slots not written yet, or later
    // tokens of the run)
    auto drop_past = [&](int end) {
#pragma unroll
      for (int j = 0; j < NJ; ++j)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const bool in = b * kBlock + quad * 4 + r <= end;
          vf[j][0][r] = in ? vf[j][0][r] : 0.f;
          vf[j][1][r] = in ? vf[j][1][r] : 0.f;
        }
    };
    if (b * kBlock + kBlock - 1 <= first) {
      pv(true);
      continue;
    }
    // A block that some rows of the run see only in part: a weight of zero
    // does not keep a later token's infinities and NaN out of a product.
    drop_past(last);
    bool bad = false;
#pragma unroll
    for (int j = 0; j < NJ; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        bad |= !(fabsf(vf[j][0][r]) < INFINITY) || !(fabsf(vf[j][1][r]) < INFINITY);
    if (np == 1 || __builtin_amdgcn_ballot_w64(bad) == 0) {
      pv(true);
      continue;
    }
    for (int i = np - 1; i >= 0; --i) {  // token by token, from the last
      drop_past(tok_pos[t0 + i]);
      pv(rt == i);
    }
  }

  if (quad == 0) {
    s_ml[wave][0][row] = m;
    s_ml[wave][1][row] = l;
  }
  __syncthreads();
  float M = -INFINITY, L = 0.f;
#pragma unroll
  for (int w = 0; w < NW; ++w) M = fmaxf(M, s_ml[w][0][row]);
#pragma unroll
  for (int w = 0; w < NW; ++w) L += expf(s_ml[w][0][row] - M) * s_ml[w][1][row];
  const float f = expf(m - M) / L;  // a token's row sees key 0, so M is finite there
  // the upper half of the waves, then the lower half on top of it
  if (wave >= NW / 2) {
#pragma unroll
    for (int t = 0; t < NT; ++t) *(f32x4_t*)&s_o[wave - NW / 2][row][t * 16 + quad * 4] = o[t] * f;
  }
  __syncthreads();
  if (wave < NW / 2) {
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      f32x4_t* e = (f32x4_t*)&s_o[wave][row][t * 16 + quad * 4];
      *e = *e + o[t] * f;
    }
  }
  __syncthreads();
  for (int i = threadIdx.x; i < 16 * D; i += NW * 64) {
    const int r = i / D, d = i % D;
    if (r / G >= np) continue;
    float v = 0.f;
#pragma unroll
    for (int w = 0; w < NW / 2; ++w) v += s_o[w][r][d];
    out[((size_t)(t0 + r / G) * n_q + kvh * G + r % G) * D + d] = v;
  }
}

}  // namespace

hipError_t attn_decode(DType dt, const void* q, KVLayer kv, SegTables tabs,
                       const DecodeItem* items, const int32_t* order, int n_items, int n_q,
                       float* part_o, float* part_ml, hipStream_t s) {
  if (n_items == 0) return hipSuccess;
  if (dt != DT_BF16) return hipErrorInvalidValue;
  if (tabs.whole_items) {
    const dim3 g(n_items, kv.n_kv);
    if (kv.head_dim == 128)
      attn_decode_item_bf16<128><<<g, kItemWaves * 64, 0, s>>>(
          (const bf16_t*)q, (const bf16_t*)kv.base, kv.n_kv, tabs, items, order, n_q);
    else if (kv.head_dim == 64)
      attn_decode_item_bf16<64><<<g, kItemWaves * 64, 0, s>>>(
          (const bf16_t*)q, (const bf16_t*)kv.base, kv.n_kv, tabs, items, order, n_q);
    else
      return hipErrorInvalidValue;
    return hipGetLastError();
  }
  dim3 grid(n_items, (kv.n_kv + 3) / 4);
  if (kv.head_dim == 128)
    attn_decode_bf16<128><<<grid, 256, 0, s>>>((const bf16_t*)q, (const bf16_t*)kv.base, kv.n_kv,
                                               tabs, items, order, n_items, n_q, part_o, part_ml);
  else if (kv.head_dim == 64)
    attn_decode_bf16<64><<<grid, 256, 0, s>>>((const bf16_t*)q, (const bf16_t*)kv.base, kv.n_kv,
                                              tabs, items, order, n_items, n_q, part_o, part_ml);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

// Waves per (token, kv head): one while these alone fill the chip's SIMDs,
// then as many as keep the launch near one wave per SIMD.
template <int D, int G>
static void launch_merge_g(const float* part_o, const float* part_ml, const int32_t* starts,
                           const int32_t* rows, int n_tok, int n_q, int n_kv, bf16_t* out,
                           hipStream_t s) {
  const int pairs = n_tok * n_kv;
  if (pairs > 256)
    attn_merge_kernel<D, G, 1><<<dim3(n_tok, (n_kv + 3) / 4), 256, 0, s>>>(part_o, part_ml, starts,
                                                                            rows, n_q, n_kv, out);
  else if (pairs > 128 || G == 16)  // (G = 16 and 8 waves: more than 64 KB of LDS)
    attn_merge_kernel<D, G, 4><<<dim3(n_tok, n_kv), 256, 0, s>>>(part_o, part_ml, starts, rows,
                                                                 n_q, n_kv, out);
  else
    attn_merge_kernel<D, G, G == 16 ? 4 : 8><<<dim3(n_tok, n_kv), (G == 16 ? 4 : 8) * 64, 0, s>>>(
        part_o, part_ml, starts, rows, n_q, n_kv, out);
}

template <int D>
static hipError_t launch_merge(const float* part_o, const float* part_ml, const int32_t* starts,
                               const int32_t* rows, int n_tok, int n_q, int n_kv, bf16_t* out,
                               hipStream_t s) {
  switch (n_q / n_kv) {
    case 1: launch_merge_g<D, 1>(part_o, part_ml, starts, rows, n_tok, n_q, n_kv, out, s); break;
    case 2: launch_merge_g<D, 2>(part_o, part_ml, starts, rows, n_tok, n_q, n_kv, out, s); break;
    case 4: launch_merge_g<D, 4>(part_o, part_ml, starts, rows, n_tok, n_q, n_kv, out, s); break;
    case 8: launch_merge_g<D, 8>(part_o, part_ml, starts, rows, n_tok, n_q, n_kv, out, s); break;
    case 16: launch_merge_g<D, 16>(part_o, part_ml, starts, rows, n_tok, n_q, n_kv, out, s); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t attn_merge(DType dt, const float* part_o, const float* part_ml,
                      const int32_t* tok_item_start, const int32_t* tok_rows, int n_tok, int n_q,
                      int n_kv, int head_dim, void* out, hipStream_t s) {
  if (n_tok == 0) return hipSuccess;
  if (dt != DT_BF16) return hipErrorInvalidValue;
  if (head_dim == 128)
    return launch_merge<128>(part_o, part_ml, tok_item_start, tok_rows, n_tok, n_q, n_kv,
                             (bf16_t*)out, s);
  if (head_dim == 64)
    return launch_merge<64>(part_o, part_ml, tok_item_start, tok_rows, n_tok, n_q, n_kv,
                            (bf16_t*)out, s);
  return hipErrorInvalidValue;
}

template <int D>
static void launch_prefill(dim3 grid, hipStream_t s, const void* q, KVLayer kv, SegTables tabs,
                           const PrefillItem* items, int n_q, void* out) {
  grid.z = tabs.parts.most;
  attn_prefill_bf16<D><<<grid, kPfWaves * 64, 0, s>>>(
      (const bf16_t*)q, (const bf16_t*)kv.base, kv.n_kv, tabs, items, n_q, (bf16_t*)out);
  if (grid.z == 1) return;
  grid.z = D / 8;
  attn_prefill_merge<D><<<grid, 2 * kPrefillRows, 0, s>>>(tabs, items, n_q, (bf16_t*)out);
}

hipError_t attn_prefill(DType dt, const void* q, KVLayer kv, SegTables tabs,
                        const PrefillItem* items, int n_items, int n_q, void* out,
                        hipStream_t s) {
  if (n_items == 0) return hipSuccess;
  if (dt != DT_BF16) return hipErrorInvalidValue;
  if (kPrefillRows % (n_q / kv.n_kv) != 0) return hipErrorInvalidValue;
  dim3 grid(n_items, kv.n_kv);
  if (kv.head_dim == 128)
    launch_prefill<128>(grid, s, q, kv, tabs, items, n_q, out);
  else if (kv.head_dim == 64)
    launch_prefill<64>(grid, s, q, kv, tabs, items, n_q, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

hipError_t attn_f32(const float* q, KVLayer kv, SegTables tabs, const int32_t* tok_seq,
                    const int32_t* tok_pos, int t_begin, int n_tok, int n_q, float* out,
                    hipStream_t s) {
  if (n_tok == 0) return hipSuccess;
  // whole 16-row tiles, unless that leaves more than half of the CUs without
  // a block: then fewer tokens (and more padding rows) per block
  int P = 16 / (n_q / kv.n_kv);
  while (P > 1 && (long)((n_tok + P - 1) / P) * kv.n_kv < kCus / 2) P /= 2;
  dim3 grid((n_tok + P - 1) / P, kv.n_kv, P);
  if (kv.head_dim == 128)
    attn_f32_kernel<128><<<grid, kF32Waves * 64, 0, s>>>(q, (const float*)kv.base, kv.n_kv, tabs,
                                                         tok_seq, tok_pos, t_begin,
                                                         t_begin + n_tok, P, n_q, out);
  else if (kv.head_dim == 64)
    attn_f32_kernel<64><<<grid, kF32Waves * 64, 0, s>>>(q, (const float*)kv.base, kv.n_kv, tabs,
                                                        tok_seq, tok_pos, t_begin,
                                                        t_begin + n_tok, P, n_q, out);
  else
    return hipErrorInvalidValue;
  return hipGetLastError();
}

}  // namespace stage_k
