// Split-K partial attention for work with at most 16 query rows per kv head (decode: one
// token x the GQA group).  Bandwidth-bound: every K/V byte is used once (paper Section 4.2:
// the memory-bound side of max(4Cd/F, 4Cd/B_mem)).
//
// One workgroup = one unit (a few query tokens x a chunk of the slot list) for `unit_heads` kv heads
// (1, 2, 4 or 8; a divisor of kv_heads, or 8 with idle waves).  Its 8 waves are dealt to (head, slice) pairs: wave w takes
// head unit_heads * head_block + w % unit_heads and, of the chunk's 32-token tiles, every
// (8 / unit_heads)-th from w / unit_heads on; the slices of a head are added up through LDS at the end,
// so that a unit gives one partial whatever the deal.  With 8 heads the workgroup as a whole reads
// whole token rows of the slot (2 KB contiguous) and no wave shares a head: the form for batches that
// fill the GPU.  The others are for layers with fewer kv heads (a layer split over GPUs), where waves
// without a head would idle, and for batches of so few units that their heads have to be spread over
// workgroups to occupy the CUs (plan_unit_heads_log2).  Each wave streams its head's K and V in tiles
// of 32 tokens: global -> registers (prefetched one tile ahead) -> wave-private LDS -> MFMA 16x16x32
// operands.  The 8 (or fewer) GQA rows ride in a 16-row MFMA tile.
#pragma once

#include "attn_common.h"

// Each wave stages its kv head's tiles in an LDS region of its own, and a wave's LDS
// operations execute in program order, so no workgroup barrier is needed between the
// wave's writes and its reads: a compiler-level ordering point is enough.
#define TL_UNIT_SYNC() do { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront"); __builtin_amdgcn_wave_barrier(); } while (0)

namespace tl {
namespace unit {

constexpr int kThreads = 512;
constexpr int kWaves = 8;
constexpr int kTok = 32;                                   // kv tokens per wave tile
constexpr int kWaveElems = kTok * (kLdsStride + kVStrideUnit);   // K tile + V tile, bf16 elements
constexpr size_t kLdsBytes = (size_t)kWaves * kWaveElems * sizeof(uint16_t);
// what a wave leaves in its LDS region for the sum over slices: O as 8 x 64 lanes x 4, then the 16 rows'
// reference, row sum and rounded row sum
constexpr int kSliceStats = 8 * 64 * 4;                    // offset of the statistics, in floats
static_assert((kSliceStats + 3 * 16) * sizeof(float) <= kWaveElems * sizeof(uint16_t), "a slice fits its wave's region");

// The plan's lists through the constant address space: nothing in a launch writes them.  In a kernel that the
// compiler cannot see this of (row tiles beside units), it would take the cursor's loads through the vector unit,
// whose wait is for the tile in flight as well: 128 requests of 500 to 32k tokens 713 us there, 634 with scalar loads.
template <typename T>
__device__ __forceinline__ const __attribute__((address_space(4))) T* scalar_loads(const T* p) {
  return (const __attribute__((address_space(4))) T*)(uintptr_t)p;
}

// Whole workgroups, or a wave per head (waves that share a head meet at a barrier: none may be without one).
inline bool can_deal(const AttnArgs& a) {
  return a.unit_heads_log2 == 3 || (a.unit_heads_log2 >= 0 && a.unit_heads_log2 < 3 && !(a.kv_heads & ((1 << a.unit_heads_log2) - 1)));
}

// IN_TURN: the workgroup takes several units, one after the other.
template <int VREAD, bool IN_TURN, typename Args>
__device__ __forceinline__ void splitk_unit(const Args& a, const Work wk, const int head_block, uint16_t* lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, l16 = lane & 15, c4 = lane >> 4;
  const int heads = 1 << a.unit_heads_log2, slices = kWaves >> a.unit_heads_log2;
  const int slice = wave >> a.unit_heads_log2;          // scalar, as the tile cursor has to be
  const int g = head_block * heads + (wave & (heads - 1));
  if (g >= a.kv_heads) return;                          // 8 heads to a workgroup, no barrier below
  const int G = a.group;
  uint16_t* kt = lds + wave * kWaveElems;
  uint16_t* vt = kt + kTok * kLdsStride;

  const int tok_local = l16 / G;
  const int j = l16 - tok_local * G;
  const bool row_ok = tok_local < wk.n_tok;
  int token = 0;
  if (!IN_TURN) {
    token = row_ok ? a.tok[wk.tok_off + tok_local] : 0;
  } else {
    // by scalar loads, 16 entries of the token array whatever their number (the plan's block goes on for 256 bytes behind its last
    // array), each lane its own: a vector load would wait for the last unit's stores.  (Where every unit has a workgroup
    // of its own, 0.2 us longer than the vector load.)
    const auto* toks = scalar_loads(a.tok + wk.tok_off);
#pragma unroll
    for (int t = 0; t < kUnitRows; ++t) {
      const int of_t = toks[t];
      if (row_ok && tok_local == t) token = of_t;
    }
  }

  // Q as B operand of 16x16x32: lane holds row l16, head-dim 32 s + 8 c4 .. +7
  bf16x8 qreg[4];
  {
    const uint4* qp = (const uint4*)(a.q + ((size_t)token * a.q_heads + g * G + j) * kHeadDim);
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      uint4 u = make_uint4(0, 0, 0, 0);
      if (row_ok) u = qp[4 * s + c4];
      qreg[s] = as_bf16x8(u);
    }
  }

  f32x4 o[8];
#pragma unroll
  for (int d = 0; d < 8; ++d) o[d] = f32x4{0.f, 0.f, 0.f, 0.f};
  // two row sums: the unrounded fp32 one gives the LSE, the one over the probabilities as rounded
  // to bf16 for the second product normalises O (a convex combination of V rows whatever the rounding)
  float m_run = -INFINITY, l_run = 0.f, lr_run = 0.f;
  const float c = a.scale_log2e;
  const size_t kv_row = (size_t)a.kv_heads * kHeadDim;

  // address = (tile's first row and head: wave-uniform, scalar registers) + (this lane's constant 32-bit
  // offset) + (a multiple of four rows), so that a tile costs hardly any per-lane address arithmetic
  const unsigned lane_off = (unsigned)((lane >> 4) * kv_row * 2 + (lane & 15) * 16);
  const unsigned row4 = (unsigned)(4 * kv_row * 2);
  uint4 kst[8], vst[8];
  auto gload = [&](int base, int valid) {
    base = __builtin_amdgcn_readfirstlane(base);
    valid = __builtin_amdgcn_readfirstlane(valid);
    const size_t tile = ((size_t)base * kv_row + (size_t)g * kHeadDim) * 2;
    const char* ksrc = (const char*)a.k + tile;
    const char* vsrc = (const char*)a.v + tile;
    if (valid == kTok) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        kst[i] = *(const uint4*)(ksrc + (lane_off + row4 * i));
        vst[i] = *(const uint4*)(vsrc + (lane_off + row4 * i));
      }
    } else {
      // rows beyond `valid` are taken as zero: 0 * garbage cannot make NaN
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        kst[i] = make_uint4(0, 0, 0, 0);
        vst[i] = make_uint4(0, 0, 0, 0);
        if ((lane >> 4) + 4 * i < valid) {
          kst[i] = *(const uint4*)(ksrc + (lane_off + row4 * i));
          vst[i] = *(const uint4*)(vsrc + (lane_off + row4 * i));
        }
      }
    }
  };
  auto lstore = [&]() {
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int cidx = lane + 64 * i;
      const int tr = cidx >> 4, part = cidx & 15;
      *(uint4*)&kt[tr * kLdsStride + part * 8] = kst[i];
      *(uint4*)&vt[tr * kVStrideUnit + part * 8] = vst[i];
    }
  };

  // tile cursor over the unit's slots (uniform across the wave: each slice takes its own tiles); an entry
  // of the list is (first kv row of the slot, valid tokens)
  // (a slot that the unit's run lists m times is walked once; its keys weigh m: lm = log2 m is
  // added to the exponent of the tile's probabilities)
  const auto* entries = scalar_loads((const int2*)a.unit_slots + wk.kv_off);
  const auto* lms = scalar_loads(a.slot_lm + wk.kv_off);
  int li = 0, kk = slice;
  auto next_tile = [&](int& base, int& valid, float& lm) __attribute__((always_inline)) -> bool {
    int i = li, k = kk, first = 0, f = 0;
    for (; i < wk.kv_len; ++i) {
      first = entries[i].x;
      f = entries[i].y;
      if (k * kTok < f) break;
      k -= (f + kTok - 1) / kTok;
    }
    const bool found = i < wk.kv_len;
    if (found) {
      base = first + k * kTok;
      valid = min(kTok, f - k * kTok);
      lm = a.slot_lm ? lms[i] : 0.f;
    }
    li = i;
    kk = k + slices;
    return found;
  };

  int base = 0, valid = 0;
  float lm = 0.f;
  bool have = next_tile(base, valid, lm);
  if (have) gload(base, valid);

  while (have) {
    lstore();
    int nbase = 0, nvalid = 0;
    float nlm = 0.f;
    const bool have_next = next_tile(nbase, nvalid, nlm);
    if (have_next) gload(nbase, nvalid);
    TL_UNIT_SYNC();

    // S^T = K Q^T : two blocks of 16 tokens
    f32x4 s0 = {0.f, 0.f, 0.f, 0.f}, s1 = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) {
      const bf16x8 a0 = *(const bf16x8*)&kt[l16 * kLdsStride + 32 * s + 8 * c4];
      const bf16x8 a1 = *(const bf16x8*)&kt[(16 + l16) * kLdsStride + 32 * s + 8 * c4];
      s0 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a0, qreg[s], s0, 0, 0, 0);
      s1 = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a1, qreg[s], s1, 0, 0, 0);
    }
    if (valid < kTok) {
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if (4 * c4 + r >= valid) s0[r] = -INFINITY;
        if (16 + 4 * c4 + r >= valid) s1[r] = -INFINITY;
      }
    }
    float mx = fmaxf(fmaxf(fmaxf(s0[0], s0[1]), fmaxf(s0[2], s0[3])), fmaxf(fmaxf(s1[0], s1[1]), fmaxf(s1[2], s1[3])));
    mx = fmaxf(mx, __shfl_xor(mx, 16));
    mx = fmaxf(mx, __shfl_xor(mx, 32));
    const float m_new = fmaxf(m_run, mx);
    const float m_use = (m_new == -INFINITY) ? 0.f : m_new;
    const float alpha = fast_exp2((m_run - m_use) * c);
    m_run = m_new;
    const float mc = m_use * c - lm;
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      s0[r] = fast_exp2(fmaf(s0[r], c, -mc));
      s1[r] = fast_exp2(fmaf(s1[r], c, -mc));
      lsum += s0[r] + s1[r];
    }
    l_run = l_run * alpha + lsum;
    // P^T operand: elements 0..3 = block 0 (tokens 4 c4 + r), 4..7 = block 1 (16 + 4 c4 + r)
    const bf16x8 pb = pack_bf16x8(s0[0], s0[1], s0[2], s0[3], s1[0], s1[1], s1[2], s1[3]);
    {
      typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
      const u32x4 w = __builtin_bit_cast(u32x4, pb);
      float lr = lr_run * alpha;
#pragma unroll
      for (int i = 0; i < 4; ++i) lr = add_bf16_pair(lr, w[i]);
      lr_run = lr;
    }
#pragma unroll
    for (int d = 0; d < 8; ++d) {
      bf16x8 av;
      if (VREAD == 0) {
        const uint16_t* p = vt + (4 * c4 + (l16 >> 2)) * kVStrideUnit + 16 * d + 4 * (l16 & 3);
        av = join_tr(lds_read_tr(p), lds_read_tr(p + 16 * kVStrideUnit));
      } else {
        s16x8 t;
#pragma unroll
        for (int e = 0; e < 8; ++e) t[e] = (short)vt[(16 * (e >> 2) + 4 * c4 + (e & 3)) * kVStrideUnit + 16 * d + l16];
        av = __builtin_bit_cast(bf16x8, t);
      }
      f32x4 acc = o[d];
      acc[0] *= alpha; acc[1] *= alpha; acc[2] *= alpha; acc[3] *= alpha;
      o[d] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(av, pb, acc, 0, 0, 0);
    }
    TL_UNIT_SYNC();
    have = have_next;
    base = nbase;
    valid = nvalid;
    lm = nlm;
  }

  float l_tot = l_run + __shfl_xor(l_run, 16);
  l_tot += __shfl_xor(l_tot, 32);
  float lr_tot = lr_run + __shfl_xor(lr_run, 16);
  lr_tot += __shfl_xor(lr_tot, 32);
  const size_t orow = (size_t)(wk.out_row + tok_local) * a.q_heads + g * G + j;
  if (slices == 1) {
    if (row_ok) {
      const float inv = lr_tot > 0.f ? 1.f / lr_tot : 0.f;
      float* op = a.out + orow * kHeadDim;
#pragma unroll
      for (int d = 0; d < 8; ++d)
        *(float4*)&op[16 * d + 4 * c4] = make_float4(o[d][0] * inv, o[d][1] * inv, o[d][2] * inv, o[d][3] * inv);
      if (c4 == 0) a.lse[orow] = l_tot > 0.f ? m_run * a.scale + __logf(l_tot) : -INFINITY;
    }
    return;
  }
  // ---- the slices of each head, added up: M = max m_s, weights 2^(c (m_s - M)) (0 for a slice without
  // keys) on O_s, l_s and lr_s alike.  Wave (head, slice) finishes an even share of the 8 channel blocks.
  {
    float* mine = (float*)kt;
#pragma unroll
    for (int d = 0; d < 8; ++d) *(f32x4*)&mine[(d * 64 + lane) * 4] = o[d];
    if (c4 == 0) {
      mine[kSliceStats + l16] = m_run;
      mine[kSliceStats + 16 + l16] = l_tot;
      mine[kSliceStats + 32 + l16] = lr_tot;
    }
  }
  __syncthreads();
  const float* first = (const float*)(lds + (wave & (heads - 1)) * kWaveElems);      // the head's slice 0
  const int slice_step = heads * kWaveElems / 2;                                       // floats from slice to slice
  float M = -INFINITY;
  for (int s = 0; s < slices; ++s) M = fmaxf(M, first[s * slice_step + kSliceStats + l16]);
  const float m_use = (M == -INFINITY) ? 0.f : M;
  float L = 0.f, LR = 0.f;
  const int per = 8 / slices, d0 = slice * per;
  f32x4 acc[4];
#pragma unroll
  for (int u = 0; u < 4; ++u) acc[u] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int s = 0; s < slices; ++s) {
    const float* src = first + s * slice_step;
    const float w = fast_exp2((src[kSliceStats + l16] - m_use) * c);
    L += w * src[kSliceStats + 16 + l16];
    LR += w * src[kSliceStats + 32 + l16];
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < per) {
        const f32x4 x = *(const f32x4*)&src[((d0 + u) * 64 + lane) * 4];
        acc[u][0] += w * x[0]; acc[u][1] += w * x[1]; acc[u][2] += w * x[2]; acc[u][3] += w * x[3];
      }
  }
  if (row_ok) {
    const float inv = LR > 0.f ? 1.f / LR : 0.f;
    float* op = a.out + orow * kHeadDim;
#pragma unroll
    for (int u = 0; u < 4; ++u)
      if (u < per)
        *(float4*)&op[16 * (d0 + u) + 4 * c4] = make_float4(acc[u][0] * inv, acc[u][1] * inv, acc[u][2] * inv, acc[u][3] * inv);
    if (slice == 0 && c4 == 0) a.lse[orow] = L > 0.f ? M * a.scale + __logf(L) : -INFINITY;
  }
}

}  // namespace unit
}  // namespace tl
