// Row-tile partial attention (paper Section 4, first paragraph: query rows attend to cache
// segments independently and emit a partial output plus normalizer; Section 2.1: the new
// tokens' self-attention is one more such partial).
//
// One workgroup = 8 wavefronts = 256 query rows of one kv head (row = (token, head in the
// GQA group)); wave w owns rows 32w..32w+31 (two waves per SIMD).  The workgroup walks the work
// item's kv tokens in tiles of 64, brought into LDS by direct global->LDS loads (16 bytes per
// lane, whole 256-byte rows, three tile buffers each for K and V).
//
// With 32x32x16 bf16 MFMA, per 32-token block and wave:
//   S^T[kv, row] = K[kv, :] . Q[row, :]      A = K block from LDS, B = Q (registers)
//   softmax numerators down the kv axis       lane l holds row l%32; its partner l^32 holds
//                                             the other half of that row's kv values
//   O^T[d, row] += V^T[d, kv] . P^T[kv, row]  A = V block read transposed from LDS, B = P
// Scores never leave registers between the two products.
//
// Fast path (completely filled tiles): the stream of 32-token blocks is software-pipelined
// inside each wave.  While the vector ALU turns the scores of block i into probabilities, the
// matrix unit computes the scores of block i+1 and accumulates block i-1; the three touch
// different registers, so neither unit waits for the other.  (Measured on gfx950: MFMA and
// vector-ALU instructions of the SAME wave overlap, those of two waves of a SIMD hardly do, and
// both kinds leave through one issue port, so the vector-ALU instruction count per MFMA is what
// the loop is trimmed for: LDS addresses are loop-invariant registers plus immediates -- the
// loop is unrolled over the three tile buffers -- and LDS operands are fetched three operand
// groups ahead of their MFMA.)  The exponent's reference point is fixed from the first block
// (any reference gives the same normalised result), which leaves the loop free of branches and
// of rescaling; if a row sum ends up above 2^60 or not finite -- scores far above the reference
// -- the workgroup discards the result and redoes the full tiles on the careful path.
// Careful path (tiles cut short by a slot's fill, tiles on the causal diagonal, and the
// redo): one tile at a time, masked, running maximum raised (and O rescaled) when a block
// exceeds it by more than 2^8; the next tile streams into the same LDS buffers meanwhile, and the first one
// comes behind the fast path's last tile as if it were one more of them, so that nothing waits for it.
// (Staged through registers, a masked tile cost 8.2k cycles, three of the fast path's; now 4.9k, with the phase's first loads
// issued ahead of its lists: 8 prompts of 700 to 4096 tokens 559 -> 548 us, 7 of 261 to 1044 with 16 heads 55.2 -> 50.5.)
// Repeated slots: a work item's list may name a slot several times (a multiset); the plan's tile
// lists hold each distinct slot once with log2 of its multiplicity, which is added to the exponent
// of the tile's probabilities (m equal keys weigh m exp(s) in numerator and denominator alike).
//
// Normalisation.  The probabilities enter the second product rounded to bf16, so O should be
// divided by the sum of the ROUNDED values -- it is then a convex combination of V rows whatever
// the rounding did to the weights -- while the normalizer that leaves the kernel (LSE) needs the
// sum of the unrounded fp32 values.  The kernel keeps the fp32 sum l and, beside it, a
// correction d ~= sum(rounded) - sum(unrounded); O is divided by l + d, LSE = m + ln l.
//  * careful path: d is exact (v_dot2c_f32_bf16 sums each packed pair as the matrix unit sees it);
//  * fast path: a second exact sum of every tile would cost 7 % of the kernel's time (the dot
//    instructions share the matrix pipeline), so a tile gets its exact d only if it raised some
//    lane's row sum by more than a sixteenth (one compare per tile; both blocks' packed
//    probabilities are still in registers then).  That is every tile at the start of a phase and
//    hardly any later on, unless a row is peaked: with a fixed exponent reference a dominant
//    probability is a rounded number like any other (with a running maximum it would be exactly
//    1), and its rounding is what the error of a peaked row consists of.  What remains is the
//    error of terms from tiles that added little, sum_j w_j e_j (v_j - O) with |e_j| <= 2^-8 over
//    those terms: no more than in a kernel that keeps a running maximum.
#include <type_traits>

#include "attn_common.h"
#include "splitk_unit.h"

namespace tl {

namespace {

constexpr int kRG = 1;                                    // 32-row groups per wave
constexpr int kWaves = kRowTile / (32 * kRG);             // 8
constexpr int kThreads = 64 * kWaves;                     // 512
constexpr int kKS = kHeadDim;        // K row stride in LDS (bf16): unpadded, 16-byte chunks swizzled
constexpr int kVS = kHeadDim;        // V row stride in LDS (bf16): unpadded, 16-byte chunks swizzled
constexpr int kKTile = kKvTile * kKS;
constexpr int kVTile = kKvTile * kVS;
constexpr int kIdxRing = 512;        // tile-base entries kept in LDS (ring over the work item's tile list)
constexpr int kBufs = 3;             // LDS tile buffers: K(t+2) and V(t+1) stream in while tile t is computed
constexpr int kQWave = 32 * kHeadDim;              // a wave's queries, staged through LDS: waves 0 and 1 in the third K buffer, the others from the
                                                   // second V buffer on, which the first tiles leave free, and kQExtra behind the third
constexpr int kQExtra = 6 * kQWave - 2 * kVTile;
static_assert(2 * kQWave == kKTile && kQExtra >= 0, "the queries fit beside the first tiles");
constexpr size_t kLdsBytes = (size_t)(kBufs * (kKTile + kVTile) + kQExtra) * sizeof(uint16_t) + (2 * kIdxRing + 4) * sizeof(int32_t);
constexpr int kOutStride = 2 * kHeadDim + 16;    // epilogue: bytes from row to row of a wave's stretch of LDS (half an fp32 row or a bf16 one, and
                                                 // 16 so that eight rows' 16-byte writes fall in different banks)
static_assert(kWaves * 32 * kOutStride <= kBufs * (kKTile + kVTile) * (int)sizeof(uint16_t), "the rows of a tile fit the LDS of its kv tiles");
constexpr int kPriorWave = 32 * 4 * kHeadDim;    // epilogue of one-pass tails: bytes of a wave's rows of one prior partial
template <int MODE>
constexpr size_t kLds = MODE == 2 && kWaves * kPriorWave > kLdsBytes ? kWaves * kPriorWave : kLdsBytes;
constexpr float kRescaleLog2 = 8.0f;             // careful path: raise the maximum when exceeded by 2^8
constexpr float kFastPathLimit = 1.152921504606846976e18f;  // 2^60
constexpr int kDmaPerWave = 16 / kWaves;                  // direct-load instructions per wave per K (or V) tile
constexpr float kExactCorrectionGrowth = 1.0625f;   // fast path: growth of a lane's row sum over one tile from which the tile's correction is exact
constexpr int kDepth = 3;            // LDS operands in flight ahead of the MFMA that uses them (ring of kDepth + 1)

// Lanes l and l^32 exchange x: returns {own, partner} in some order.  The swap instruction
// exchanges the upper half of its first operand with the lower half of its second; the second
// copy of x is laundered through an empty asm so that the compiler treats the two operands
// (and hence the two results) as unrelated values.
__device__ __forceinline__ void xor32_pair(float x, float& r0, float& r1) {
  unsigned a = __builtin_bit_cast(unsigned, x), b = a;
  asm volatile("" : "+v"(b));
  auto r = __builtin_amdgcn_permlane32_swap(a, b, false, false);
  unsigned u0 = r[0], u1 = r[1];
  asm volatile("" : "+v"(u0), "+v"(u1));
  r0 = __builtin_bit_cast(float, u0);
  r1 = __builtin_bit_cast(float, u1);
}

__device__ __forceinline__ float xor32_max(float x) {
  float r0, r1;
  xor32_pair(x, r0, r1);
  return fmaxf(r0, r1);
}

__device__ __forceinline__ float xor32_sum(float x) {
  float r0, r1;
  xor32_pair(x, r0, r1);
  return r0 + r1;
}

// a packed bf16 operand held as four 32-bit words, so that a pair of elements is one register write
typedef unsigned u32x4 __attribute__((ext_vector_type(4)));
// word `pair` (0..3) of a packed operand := (a, b) rounded to bf16
__device__ __forceinline__ void set_pair(u32x4& p, int pair, float a, float b) {
  typedef float f32x2_t __attribute__((ext_vector_type(2)));
  typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
  p[pair] = __builtin_bit_cast(unsigned, __builtin_convertvector(f32x2_t{a, b}, bf16x2_t));
}

__device__ __forceinline__ float max16(const f32x16& s) {
  float a = fmaxf(fmaxf(s[0], s[1]), s[2]);
  float b = fmaxf(fmaxf(s[3], s[4]), s[5]);
  float c = fmaxf(fmaxf(s[6], s[7]), s[8]);
  float d = fmaxf(fmaxf(s[9], s[10]), s[11]);
  float e = fmaxf(fmaxf(s[12], s[13]), s[14]);
  return fmaxf(fmaxf(fmaxf(a, b), fmaxf(c, d)), fmaxf(e, s[15]));
}

// 16 bytes from any address
__device__ __forceinline__ uint4 load_any(const char* p) {
  uint4 x;
  __builtin_memcpy(&x, p, sizeof(x));
  return x;
}

__host__ __device__ inline unsigned unit_blocks(const AttnArgs& a) { return ((unsigned)a.unit_lanes + 7u) & ~7u; }

// MODE 0: pool work item (tile lists) -> partial.  MODE 1: causal block of the new tokens ->
// partial.  MODE 2: both in one pass -- the row tile walks its request's pool tiles, then the
// new tokens up to its own rows -- and writes the final, normalised output: such rows have one
// partial, so they need no merge.
//
// JOINT (MODE 0): row tiles of the pool and split-K units in one launch: units first, which are bound by HBM and by their own
// chain, in as many workgroups as the plan says (plan_unit_lanes), then row tiles, which find the CUs that the units leave and finish evenly on all of them.  The first
// row tile's block is a multiple of eight, so that a kv head stays on its XCD.  One launch after the other, the
// first leaves CUs idle at its end and HBM idles through the row tiles: 4 chunks of 300 to 600 tokens beside 48 decoded
// ones 614 us a step, together 520; over 120 random batches tl_segment_attn takes 0.87 of its time in two launches, 0.99
// at most.  (Groups of eight blocks of each kind in turn: a unit takes a whole round whatever runs beside it, so the
// units' second round ends late, a tenth slower.)  The branch is in the kernel itself, not around a function that both
// kernels call.  IN_TURN: fewer workgroups than units, each takes several (a kernel of its own: units with a workgroup
// each fetch their tokens 0.2 us faster without, splitk_unit).
//
// READ: how memory is read.  Bit 0: scalar LDS reads of V in place of transposing ones.  Bit 1 (kOffGrid): some tensor does not
// start on a 16-byte boundary, which direct loads to LDS ask for; what they bring goes through registers instead, to the
// same places in the same order, so that the results are the same bits.  (A variant of its own: aligned tensors pay nothing.)
constexpr int kScalarV = 1, kOffGrid = 2;
template <int MODE, int READ, bool JOINT = false, bool IN_TURN = false>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(2 / kRG, 2 / kRG))) void row_tile_attn_kernel(const AttnArgs a) {
  extern __shared__ __attribute__((aligned(16))) uint16_t lds[];
  // Arguments for the parts behind the loops, and for each of several units, are read from the kernel's argument block where
  // they are needed: held in scalar registers from the start they push others of the loop's out.  (The empty asm keeps the loads in their place.)
  auto late_args = []() __attribute__((always_inline)) {
    auto p = (const __attribute__((address_space(4))) AttnArgs*)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(p));
    return p;
  };
  if (JOINT && blockIdx.x < unit_blocks(a)) {
    const int n = a.n_units * unit_head_blocks(a.kv_heads, a.unit_heads_log2), lanes = a.unit_lanes, lane_no = blockIdx.x;
    if (lane_no >= lanes) return;
    if constexpr (!IN_TURN) {
      unit::splitk_unit<READ & kScalarV, false>(a, a.units[lane_no % a.n_units], lane_no / a.n_units, lds);
    } else {
      for (int first = 0; first < n; first += lanes) {          // forth and back, as the units come longest first
        const int i = (first / lanes) & 1 ? first + lanes - 1 - lane_no : first + lane_no;
        if (first > 0) __syncthreads();                           // the LDS is free again
        if (i >= n) return;
        const auto args = late_args();
        const auto* w = unit::scalar_loads((const int32_t*)(args->units + i % args->n_units));     // (a vector load would wait for the last unit's stores)
        unit::splitk_unit<READ & kScalarV, true>(*args, Work{w[0], w[1], w[2], w[3], w[4]}, i / args->n_units, lds);
      }
    }
    return;
  }
  const int block = JOINT ? (int)(blockIdx.x - unit_blocks(a)) : (int)blockIdx.x;   // (unsigned: 0.7 % slower on 128k lists, 6414 -> 6462 us)
  uint16_t* lds_k = lds;                 // [kBufs][64][kKS]
  uint16_t* lds_v = lds + kBufs * kKTile;    // [kBufs][64][kVS]
  int32_t* lds_idx = (int32_t*)(lds + kBufs * (kKTile + kVTile) + kQExtra);   // [kIdxRing]
  float* lds_lm = (float*)(lds_idx + kIdxRing);   // [kIdxRing] log2(multiplicity) of the same tiles
  int32_t* lds_flag = lds_idx + 2 * kIdxRing;

  const int g = block % a.kv_heads;
  // a row tile as two workgroups: the first halves of all, then the second ones, of which some may be empty
  int item = block / a.kv_heads;
  const bool second = a.halve && item >= a.n_work;
  if (second) item -= a.n_work;
  Work wk = a.work[item];
  if (a.halve) {
    const int first = half_row_tile(a.group), skip = second ? first : 0;
    if (skip >= wk.n_tok) return;
    const int n = second ? wk.n_tok - first : min(first, wk.n_tok);
    wk.tok_off += skip;
    wk.out_row += skip;
    wk.kv_len -= wk.n_tok - skip - n;          // (new tokens visible to the half's last row; not used by pool work)
    wk.n_tok = n;
  }
  const int tid = threadIdx.x;
  const int wave = tid >> 6, lane = tid & 63, l32 = lane & 31, h = lane >> 5;
  const int G = a.group;
  constexpr bool kHasPool = MODE != 1, kHasSelf = MODE != 0;
  const int first_token = wk.tok_off;          // causal work: tokens of a tile are consecutive, and the token array starts with
                                               // every token in order (one dependent load less before the queries)
  // K/V of the new tokens: the launch's main K/V for the causal block alone, the second pair when fused
  auto self_k = [&]() __attribute__((always_inline)) { const auto args = late_args(); return MODE == 2 ? args->k2 : args->k; };
  auto self_v = [&]() __attribute__((always_inline)) { const auto args = late_args(); return MODE == 2 ? args->v2 : args->v; };

  // per row group: this lane's row, its token and head
  int tok_local[kRG], head_j[kRG], token[kRG], q_row[kRG];
  bool row_ok[kRG];
#pragma unroll
  for (int rg = 0; rg < kRG; ++rg) {
    const int row = wave * (32 * kRG) + 32 * rg + l32;
    tok_local[rg] = row / G;                    // any group size: the last 256 % G rows of a tile are idle
    head_j[rg] = row - tok_local[rg] * G;
    row_ok[rg] = tok_local[rg] < wk.n_tok;
    const int at = row_ok[rg] ? tok_local[rg] : 0;         // a row that does not exist takes the queries of the tile's first
    const int t = kHasSelf ? first_token + at : a.tok[wk.tok_off + at];
    token[rg] = row_ok[rg] ? t : -1;
    q_row[rg] = t * a.q_heads + g * G + (row_ok[rg] ? head_j[rg] : 0);
  }

  // the last token that one of this wave's rows belongs to, -1 for a wave without rows (the item's last row tile)
  const int n_rows = wk.n_tok * G, wave_row = __builtin_amdgcn_readfirstlane(wave) * (32 * kRG);
  const int wave_last = wave_row >= n_rows ? -1 : first_token + (min(wave_row + 32 * kRG, n_rows) - 1) / G;

  bf16x8 qreg[kRG][8];    // Q as the B operand: lane holds its row, head-dim elements 16 s + 8 h .. +7 of step s

  // O^T accumulators: o[rg][d][r] = channel 32 d + 8 (r/4) + 4 h + r%4 of the lane's row in group rg
  f32x16 o[kRG][4];
  float m_ref[kRG];   // reference point of the exponent (raw score units), -inf before any key
  float l_run[kRG];   // this lane's share of sum exp(s - m_ref), unrounded (-> LSE)
  float lr_run[kRG];  // correction: (sum of the values as rounded to bf16 for the second product) - (unrounded sum)
  auto reset_state = [&]() __attribute__((always_inline)) {
#pragma unroll
    for (int rg = 0; rg < kRG; ++rg) {
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[rg][d][r] = 0.f;
      m_ref[rg] = -INFINITY;
      l_run[rg] = 0.f;
      lr_run[rg] = 0.f;
    }
  };
  reset_state();
  const float c = a.scale_log2e;

  // which tiles are full (no masking needed for any row of this workgroup)
  const int nf_pool = kHasPool ? wk.n_full : 0, np_pool = kHasPool ? wk.n_part : 0;
  int nf_self = 0, np_self = 0;
  if (kHasSelf) {
    nf_self = (first_token - wk.kv_off + 1) / kKvTile;
    np_self = (wk.kv_len + kKvTile - 1) / kKvTile - nf_self;
  }
  // first kv row of a full pool tile comes from the item's tile list, kept in an LDS ring (a
  // dependent global load per iteration would stall the wave); that of a full tile of new tokens
  // is arithmetic
  auto ring_fill = [&](int first, int count) __attribute__((always_inline)) {   // entries [first, first+count) of the list
    for (int i = first + tid; i < first + count && i < nf_pool + 1; i += kThreads) {
      if (i < nf_pool) {
        lds_idx[i & (kIdxRing - 1)] = a.tile_base[wk.full_off + i];
        if (a.tile_lm) lds_lm[i & (kIdxRing - 1)] = a.tile_lm[wk.full_off + i];
      } else if (np_pool > 0) {       // one entry more: the first tile cut short
        lds_idx[i & (kIdxRing - 1)] = a.part_tile[2 * wk.part_off];
      }
    }
  };

  const unsigned kv_bytes = (unsigned)a.kv_heads * (2 * kHeadDim);        // from kv row to kv row
  // ---- staging: direct global -> LDS load of a whole tile.  A tile is 16 wave
  // instructions; wave w issues instructions w + kWaves u, instruction i filling rows 4 i .. 4 i + 3;
  // lane L lands at row 4 i + L / 16, position L % 16, so it fetches the logical chunk that belongs there
  unsigned dma_off_k[kDmaPerWave], dma_off_v[kDmaPerWave];
#pragma unroll
  for (int u = 0; u < kDmaPerWave; ++u) {
    const int r_ = 4 * (wave + kWaves * u) + (lane >> 4), pos = lane & 15;
    dma_off_k[u] = (r_ * kv_bytes + (unsigned)g * (2 * kHeadDim) + 16 * (pos ^ (r_ & 15)));
    dma_off_v[u] = (r_ * kv_bytes + (unsigned)g * (2 * kHeadDim) + 16 * (pos ^ (4 * (r_ & 3))));
  }
  // (issued as inline assembly: the compiler does not see these loads, so it puts no wait for them
  // in front of the LDS reads that follow; dma_wait() before the iteration's barrier is the wait)
  const unsigned lds_base_addr = __builtin_amdgcn_readfirstlane((unsigned)(size_t)(__attribute__((address_space(3))) void*)lds);
  const unsigned dma_wave_off = __builtin_amdgcn_readfirstlane(wave) * (4 * kHeadDim * 2);
  static_assert(kDmaPerWave == 2, "dma_tile issues exactly two direct loads per wave");
  auto dma_tile = [&](const uint16_t* src, int base, uint16_t* tile, const unsigned (&off)[kDmaPerWave]) {
    const char* trow = (const char*)src + (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(base) * kv_bytes;
    const unsigned dst0 = lds_base_addr + (unsigned)(tile - lds) * 2u + dma_wave_off;
    const unsigned dst1 = dst0 + (unsigned)(kWaves * 4 * kHeadDim) * 2u;
    if constexpr (READ & kOffGrid) {
      char* at = (char*)tile + dma_wave_off;
      ((uint4*)at)[lane] = load_any(trow + off[0]);
      ((uint4*)(at + kWaves * 4 * kHeadDim * 2))[lane] = load_any(trow + off[1]);
      return;
    }
    // address = wave-uniform 64-bit tile base (scalar registers) + this lane's constant 32-bit offset;
    // the LDS destination travels in M0, which the compiler does not accept as a clobber: its value
    // is put back before the statement ends
    unsigned saved_m0;
    asm volatile(
        "s_mov_b32 %[sv], m0\n\t"
        "s_mov_b32 m0, %[d0]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o0], %[b]\n\t"
        "s_mov_b32 m0, %[d1]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o1], %[b]\n\t"
        "s_mov_b32 m0, %[sv]"
        : [sv] "=&s"(saved_m0)
        : [o0] "v"(off[0]), [o1] "v"(off[1]), [d0] "s"(dst0), [d1] "s"(dst1), [b] "s"(trow)
        : "memory");
  };
  // the same for the first `rows` rows of a tile; the others' places in LDS keep what they hold
  auto dma_rows = [&](const uint16_t* src, int base, int rows, uint16_t* tile, const unsigned (&off)[kDmaPerWave]) __attribute__((always_inline)) {
    const char* trow = (const char*)src + (uint64_t)(unsigned)__builtin_amdgcn_readfirstlane(base) * kv_bytes;
#pragma unroll
    for (int u = 0; u < kDmaPerWave; ++u) {
      const unsigned dst = lds_base_addr + (unsigned)(tile - lds) * 2u + dma_wave_off + (unsigned)(u * kWaves * 4 * kHeadDim) * 2u;
      unsigned saved_m0;
      if (4 * (wave + kWaves * u) + (lane >> 4) >= rows) continue;
      if constexpr (READ & kOffGrid)
        ((uint4*)((char*)tile + dma_wave_off + u * kWaves * 4 * kHeadDim * 2))[lane] = load_any(trow + off[u]);
      else
        asm volatile("s_mov_b32 %[sv], m0\n\ts_mov_b32 m0, %[d]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[o], %[b]\n\ts_mov_b32 m0, %[sv]"
                     : [sv] "=&s"(saved_m0)
                     : [o] "v"(off[u]), [d] "s"(dst), [b] "s"(trow)
                     : "memory");
    }
  };
  // wait for all of this wave's direct loads (vmcnt(0); the other counters are left alone so that
  // LDS operand reads already in flight stay in flight); for its LDS writes where they take the loads' place
  auto dma_wait = [&]() __attribute__((always_inline)) {
    if constexpr (READ & kOffGrid) asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
    else __builtin_amdgcn_s_waitcnt(0x0F70);
  };

  // ---- queries: a wave's 32 rows by direct loads, 256 bytes of a row by 16 lanes, in the swizzle of a K tile; to
  // registers once the first tiles are on their way too.  (Loaded by the lanes that hold them, 16 bytes of 32 rows an
  // instruction, they kept the first tiles waiting: prologue and first loads 8.0k cycles, now 5.1k; 64 sessions with shared
  // runs 1736 -> 1723 us, one 32k prompt 264.3 -> 261.3, 24 chunks of 150 to 301 tokens on short prefixes 71.5 -> 68.3.)
  static_assert(kRG == 1, "one K-shaped stretch of 32 rows a wave");
  const int wave_u = __builtin_amdgcn_readfirstlane(wave);
  uint16_t* q_lds = wave_u < 2 ? lds_k + 2 * kKTile + wave_u * kQWave : lds_v + kVTile + (wave_u - 2) * kQWave;
  {
    const unsigned dst0 = lds_base_addr + (unsigned)(q_lds - lds) * 2u;
    auto q_chunk = [&](int i) __attribute__((always_inline)) -> const char* {       // of row 4 i + lane / 16
      const int r_ = 4 * i + (lane >> 4);
      return (const char*)a.q + (size_t)__shfl(q_row[0], r_) * (2 * kHeadDim) + 16 * ((lane & 15) ^ (r_ & 15));
    };
    if constexpr (READ & kOffGrid) {
#pragma unroll 1
      for (int i = 0; i < 8; ++i) ((uint4*)((char*)q_lds + i * (4 * kHeadDim * 2)))[lane] = load_any(q_chunk(i));
    } else {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        unsigned saved_m0;
        asm volatile("s_mov_b32 %[sv], m0\n\ts_mov_b32 m0, %[d]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[p], off\n\ts_mov_b32 m0, %[sv]"
                     : [sv] "=&s"(saved_m0)
                     : [p] "v"(q_chunk(i)), [d] "s"(dst0 + (unsigned)i * (4 * kHeadDim * 2))
                     : "memory");
      }
    }
  }

  // ---- building blocks ----
  // LDS tiles are unpadded rows of 256 B = 16 chunks of 16 B, written by direct global->LDS
  // loads (one wave instruction fills 4 rows contiguously).  Bank conflicts are avoided by
  // storing logical chunk c of row r at position c ^ swz(r):
  //   K: swz(r) = r & 15      -> the 16 rows that 16 lanes read at one logical chunk hit 16 positions
  //   V: swz(r) = 4 (r & 3)   -> the 4 rows x 4 chunks of one transposing read hit 16 positions
  auto k_operand = [&](const uint16_t* kt, int hb, int s8) __attribute__((always_inline)) -> bf16x8 {
    return *(const bf16x8*)&kt[(32 * hb + l32) * kKS + 8 * ((2 * s8 + h) ^ (l32 & 15))];
  };
  // V^T operand of accumulation step (sp, d) of block hb: channels 32 d .. 32 d + 31, block
  // tokens 16 sp + {4h..4h+3, 8+4h..8+4h+3} -- the order in which the score registers hold them
  auto v_operand = [&](const uint16_t* vt, int hb, int sp, int d) __attribute__((always_inline)) -> bf16x8 {
    const int kvb = 32 * hb + 16 * sp;
    if constexpr (!(READ & kScalarV)) {
      const int blk = lane >> 4, jj = lane & 15;
      // logical chunk 4 d + 2 (blk & 1) + (jj & 3) / 2 of row kvb + 4 (blk >> 1) + jj / 4 (row & 3 = jj / 4)
      const int chunk = (4 * d + 2 * (blk & 1) + ((jj & 3) >> 1)) ^ (4 * (jj >> 2));
      const uint16_t* p = vt + (kvb + 4 * (blk >> 1) + (jj >> 2)) * kVS + 8 * chunk + 4 * (jj & 1);
      return join_tr(lds_read_tr(p), lds_read_tr(p + 8 * kVS));
    } else {
      s16x8 t;
#pragma unroll
      for (int e = 0; e < 8; ++e) {
        const int r_ = kvb + 8 * (e >> 2) + 4 * h + (e & 3), col = 32 * d + l32;
        t[e] = (short)vt[r_ * kVS + 8 * ((col >> 3) ^ (4 * (r_ & 3))) + (col & 7)];
      }
      return __builtin_bit_cast(bf16x8, t);
    }
  };
  // scores of block hb of the K tile at kt, for every row group of the wave
  auto qk_block = [&](const uint16_t* kt, int hb, f32x16 (&s)[kRG]) {
    const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s8 = 0; s8 < 8; ++s8) {
      const bf16x8 ak = k_operand(kt, hb, s8);
#pragma unroll
      for (int rg = 0; rg < kRG; ++rg)
        s[rg] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ak, qreg[rg][s8], s8 == 0 ? zero : s[rg], 0, 0, 0);
    }
  };
  // probabilities of a block against the reference: p = 2^(c (s - m_ref)); B operands pb[sp]
  // hold registers 8 sp .. 8 sp + 7
  auto exp_block = [&](int rg, f32x16& s, bf16x8 (&pb)[2], float lm) {
    const float mc = m_ref[rg] * c - lm;   // lm = log2(times the tile's slot is listed): p = m 2^(c (s - m_ref))
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = fast_exp2(fmaf(s[r], c, -mc));
    pb[0] = pack_bf16x8(s[0], s[1], s[2], s[3], s[4], s[5], s[6], s[7]);
    pb[1] = pack_bf16x8(s[8], s[9], s[10], s[11], s[12], s[13], s[14], s[15]);
    // the normalizer (LSE) sums the probabilities before their rounding to bf16, in fp32 ...
    float lsum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) lsum += s[r];
    l_run[rg] += lsum;
    // ... and O is divided by the sum of what the matrix unit is given: lr = that sum, exactly
    float lr = 0.f;
#pragma unroll
    for (int sp = 0; sp < 2; ++sp) {
      const u32x4 w = __builtin_bit_cast(u32x4, pb[sp]);
#pragma unroll
      for (int i = 0; i < 4; ++i) lr = add_bf16_pair(lr, w[i]);
    }
    lr_run[rg] += lr - lsum;
  };
  auto pv_block = [&](const uint16_t* vt, int hb, const bf16x8 (&pb)[kRG][2]) {
#pragma unroll
    for (int sp = 0; sp < 2; ++sp)
#pragma unroll
      for (int d = 0; d < 4; ++d) {
        const bf16x8 av = v_operand(vt, hb, sp, d);
#pragma unroll
        for (int rg = 0; rg < kRG; ++rg)
          o[rg][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(av, pb[rg][sp], o[rg][d], 0, 0, 0);
      }
  };
  // careful path: raise the reference maximum if the block's scores exceed it by too much
  auto maybe_rescale = [&](int rg, const f32x16& s) __attribute__((always_inline)) {
    const float mx = xor32_max(max16(s));
    const bool need = (mx - m_ref[rg]) * c > kRescaleLog2 || m_ref[rg] == -INFINITY;
    if (__builtin_amdgcn_ballot_w64(need) != 0) {
      const float m_new = fmaxf(m_ref[rg], mx);
      const float alpha = (m_new == -INFINITY) ? 1.f : fast_exp2((m_ref[rg] - m_new) * c);
      m_ref[rg] = m_new;
      l_run[rg] *= alpha;
      lr_run[rg] *= alpha;
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[rg][d][r] *= alpha;
    }
  };
  // Tiles that are masked or walked carefully, by number t in a phase's list: the kv row at the tile's first place, the
  // places [lo, hi) that are the tile's, log2 of the multiplicity.  Pool: the full tiles, then those cut short by a
  // fill; new tokens: in order.  (The lists' places are held in scalar registers, for which the one-pass kernel puts three others
  // aside once on the way to its masked pool tiles; read from the argument block tile by tile, nothing is put aside and the tiny
  // configuration takes 14.4 us, 13.2 so.)
  struct Tile {
    int base, lo, hi;
    float lm;
  };
  auto tile_at = [&](auto SELF, int t) __attribute__((always_inline)) -> Tile {
    if constexpr (decltype(SELF)::value) return {wk.kv_off + kKvTile * t, 0, min(kKvTile, wk.kv_len - kKvTile * t), 0.f};
    if (t < nf_pool) return {unit::scalar_loads(a.tile_base)[wk.full_off + t], 0, kKvTile, a.tile_lm ? unit::scalar_loads(a.tile_lm)[wk.full_off + t] : 0.f};
    const int pt = wk.part_off + t - nf_pool;
    return {unit::scalar_loads(a.part_tile)[2 * pt], 0, unit::scalar_loads(a.part_tile)[2 * pt + 1], a.part_lm ? unit::scalar_loads(a.part_lm)[pt] : 0.f};
  };
  // where the fast path loads 64 rows for tile t of the new tokens: inside the memory (there is a full tile, hence 64 rows).
  // (A pool tile's 64 rows are always its slot's: seg_len is a multiple of 64.)
  auto self_load_base = [&](int t) __attribute__((always_inline)) -> int { return min(wk.kv_off + kKvTile * t, a.n_tokens - kKvTile); };
  // a barrier for LDS alone: direct loads on their way stay on their way
  auto lds_barrier = [&]() __attribute__((always_inline)) {
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
  };
  // a phase's first loads: the list's first entries come by scalar loads
  auto first_loads = [&](auto SELF, const uint16_t* src_k, const uint16_t* src_v, const int n_load) __attribute__((always_inline)) {
    constexpr bool CAUSAL = decltype(SELF)::value;
    const int first_base = tile_at(SELF, 0).base;
    dma_tile(src_k, first_base, lds_k, dma_off_k);
    dma_tile(src_v, first_base, lds_v, dma_off_v);
    if (n_load > 1) dma_tile(src_k, CAUSAL ? self_load_base(1) : tile_at(SELF, 1).base, lds_k + kKTile, dma_off_k);
  };
  // careful path: tiles [from, to) of a phase, tile t in LDS buffers t % kBufs; the next tile is on its way while one is
  // computed.  `loaded`: tile `from` is there already, fetched by the fast path behind its last full tile.
  auto careful_tiles = [&](auto SELF, const uint16_t* src_k, const uint16_t* src_v, const int from, const int to, const bool loaded) __attribute__((always_inline)) {
    constexpr bool CAUSAL = decltype(SELF)::value;
    if (from >= to) return;
    Tile cur = tile_at(SELF, from);
    int buf = from % kBufs;
    if (loaded) {
      if constexpr (CAUSAL) {
        cur.lo = cur.base - self_load_base(from);
        cur.hi += cur.lo;
        cur.base -= cur.lo;
      }
    } else {
      dma_rows(src_k, cur.base, cur.hi, lds_k + buf * kKTile, dma_off_k);
      dma_rows(src_v, cur.base, cur.hi, lds_v + buf * kVTile, dma_off_v);
      dma_wait();
      lds_barrier();
    }
#pragma unroll 1
    for (int t = from; t < to; ++t) {
      const uint16_t* kt = lds_k + buf * kKTile;
      uint16_t* vt = lds_v + buf * kVTile;
      buf = buf + 1 == kBufs ? 0 : buf + 1;
      Tile next = cur;
      if (t + 1 < to) {
        next = tile_at(SELF, t + 1);
        dma_rows(src_k, next.base, next.hi, lds_k + buf * kKTile, dma_off_k);
        dma_rows(src_v, next.base, next.hi, lds_v + buf * kVTile, dma_off_v);
      }
      if (cur.hi - cur.lo < kKvTile) {
        // places of V that are not the tile's are zero: 0 * garbage cannot make NaN (their scores are hidden below)
        for (int i = tid; i < 16 * kKvTile; i += kThreads)
          if (i < 16 * cur.lo || i >= 16 * cur.hi) ((uint4*)vt)[i] = make_uint4(0, 0, 0, 0);
        lds_barrier();
      }
#pragma unroll 1
      for (int hb = 0; hb < 2; ++hb) {
        if (32 * hb >= cur.hi || (CAUSAL ? cur.base + 32 * hb > wave_last : wave_last < 0)) break;   // wave-uniform
        f32x16 s[kRG];
        qk_block(kt, hb, s);
        bf16x8 pb[kRG][2];
#pragma unroll
        for (int rg = 0; rg < kRG; ++rg) {
          // register r of the lane is place 32 hb + 4 h + (8 (r / 4) + r % 4) of the tile: visible before `end`
          const int end = (CAUSAL ? min(cur.hi, token[rg] + 1 - cur.base) : cur.hi) - 32 * hb - 4 * h;
#pragma unroll
          for (int r = 0; r < 16; ++r) {
            if (8 * (r >> 2) + (r & 3) >= end) s[rg][r] = -INFINITY;
          }
          if (CAUSAL && cur.lo > 32 * hb) {
#pragma unroll
            for (int r = 0; r < 16; ++r)
              if (8 * (r >> 2) + (r & 3) < cur.lo - 32 * hb - 4 * h) s[rg][r] = -INFINITY;
          }
          maybe_rescale(rg, s[rg]);
          if (m_ref[rg] == -INFINITY) {
            // every key so far is hidden from this row: probabilities are zero
            pb[rg][0] = pack_bf16x8(0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f);
            pb[rg][1] = pb[rg][0];
          } else {
            exp_block(rg, s[rg], pb[rg], cur.lm);
          }
        }
        pv_block(vt, hb, pb);
      }
      dma_wait();
      lds_barrier();
      cur = next;
    }
  };

  // ======================= fast path: full tiles, software-pipelined by 32-token block =======================
  // Steady state, per block i of the tile stream (two blocks per tile = two steps per iteration):
  //   MFMA:  scores(block i+1)  and  accumulate(block i-1)      16 kRG MFMA each
  //   VALU:  probabilities(block i)
  // An iteration is 32 operand groups: one LDS operand (a K fragment, or a transposed V fragment)
  // and the kRG MFMAs that use it, plus a slice of the probabilities; the operand is fetched
  // kDepth groups earlier.  sched_barrier(0) after every group keeps the compiler to this order.
  // Runs the n_full (> 0) full tiles of one phase; have_ref says whether the exponent's reference
  // point exists already.  Returns false if the result overflowed and has to be discarded.
  // A masked tile behind the full ones (`more`) is fetched like one more of them.  `started`: the first loads are on their way.
  auto fast_phase = [&](auto SELF, const uint16_t* src_k, const uint16_t* src_v, const int n_full, const bool more, const bool started, const bool have_ref) __attribute__((always_inline)) -> bool {
    constexpr bool CAUSAL = decltype(SELF)::value;
    auto full_base = [&](int t) __attribute__((always_inline)) -> int { return CAUSAL ? self_load_base(t) : lds_idx[t & (kIdxRing - 1)]; };
    const int n_load = n_full + (more ? 1 : 0);
    if (!started) first_loads(SELF, src_k, src_v, n_load);
    if (tid == 0) *lds_flag = 0;
    if (!CAUSAL) ring_fill(0, kIdxRing);
    if (wave_u == 4 || wave_u == 5) {
      // "tile -1" (V buffer kBufs-1) is multiplied by zero probabilities in the first iteration; written by the waves
      // whose queries were there
      static_assert(kBufs == 3 && 2 * kQWave == kVTile, "the third V buffer is waves 4 and 5's");
      const uint4 z = make_uint4(0, 0, 0, 0);
#pragma unroll
      for (int i = 0; i < kQWave / 8 / 64; ++i) ((uint4*)(lds_v + (kBufs - 1) * kVTile + (wave_u - 4) * kQWave))[64 * i + lane] = z;
    }
    dma_wait();
    __syncthreads();

    if (wave_row >= n_rows) {
      // A wave without rows (a short chunk, an item's last row tile) brings its share of the tiles and leaves the matrix unit
      // to the wave it shares a SIMD with: a row tile of 128 rows or less takes 0.71 to 0.76 us a tile by itself, 1.12
      // when the idle waves multiplied zeros (the tiny configuration, 128 rows: 17.7 -> 14.6 us); of 129 rows or more no change.
      int buf = 0;
#pragma unroll 1
      for (int t = 0; t < n_full; ++t) {
        const int next = buf + 1 == kBufs ? 0 : buf + 1, prev = buf == 0 ? kBufs - 1 : buf - 1;
        if (!CAUSAL && t > 0 && (t & (kIdxRing / 2 - 1)) == 0) ring_fill(t + kIdxRing / 2, kIdxRing / 2);
        if (t + 2 < n_load) dma_tile(src_k, full_base(t + 2), lds_k + prev * kKTile, dma_off_k);
        if (t + 1 < n_load) dma_tile(src_v, full_base(t + 1), lds_v + next * kVTile, dma_off_v);
        buf = next;
        dma_wait();
        lds_barrier();
      }
      __syncthreads();
      const bool redo = *lds_flag != 0;
      __syncthreads();
      return !redo;
    }

    float l_prev[kRG];                  // the lane's row sum before the current tile
#pragma unroll
    for (int rg = 0; rg < kRG; ++rg) l_prev[rg] = l_run[rg];
    f32x16 s0[kRG], s1[kRG];            // scores of block 0 / block 1 of a tile (then their probabilities)
    u32x4 p0[kRG][2], p1[kRG][2];       // packed probabilities (bf16 pairs)
    qk_block(lds_k, 0, s0);
    float mc[kRG];
#pragma unroll
    for (int rg = 0; rg < kRG; ++rg) {
      if (!have_ref) m_ref[rg] = xor32_max(max16(s0[rg]));   // reference: the first block's row maximum
      mc[rg] = m_ref[rg] * c;
      p1[rg][0] = u32x4{0u, 0u, 0u, 0u};
      p1[rg][1] = p1[rg][0];
      p0[rg][0] = p0[rg][1] = p1[rg][0];
    }

    // operand group g of an iteration (0..31): step g / 16; even = K operand (head-dim step g%16 / 2),
    // odd = V operand ((sp, d) = g%16 / 2).  Step 0: K(t, block 1), V(t-1, block 1); step 1:
    // K(t+1, block 0), V(t, block 0).
    auto operand = [&](int gq, const uint16_t* k_t, const uint16_t* k_n, const uint16_t* v_p, const uint16_t* v_t) __attribute__((always_inline)) -> bf16x8 {
      const int step = gq >> 4, idx = (gq & 15) >> 1;
      if ((gq & 1) == 0) return k_operand(step == 0 ? k_t : k_n, step == 0 ? 1 : 0, idx);
      return v_operand(step == 0 ? v_p : v_t, step == 0 ? 1 : 0, idx >> 2, idx & 3);
    };
    bf16x8 ring[kDepth + 1];
    {
      const uint16_t* k_t = lds_k;
      const uint16_t* k_n = lds_k + kKTile;
      const uint16_t* v_p = lds_v + (kBufs - 1) * kVTile;
      const uint16_t* v_t = lds_v;
#pragma unroll
      for (int gq = 0; gq < kDepth; ++gq) ring[gq] = operand(gq, k_t, k_n, v_p, v_t);
    }
    __builtin_amdgcn_sched_barrier(0);

    // first rows of the tiles that the coming iteration streams in, K(t+2) and V(t+1) (indices past
    // the end are clamped: such a value is never used for a load)
    int base_k = full_base(min(2, n_load - 1)), base_v = full_base(min(1, n_load - 1));
    // log2 of the multiplicity of the tile whose probabilities the coming iteration forms
    // (a.tile_lm is null when no list of the plan names a slot twice: then nothing is read)
    auto tile_lm = [&](int t) __attribute__((always_inline)) -> float { return CAUSAL || !a.tile_lm ? 0.f : lds_lm[t & (kIdxRing - 1)]; };
    float lm_cur = tile_lm(0);
    // one tile; kb = t % kBufs is a compile-time constant (the loop below is unrolled kBufs times),
    // so that every LDS address is a loop-invariant per-lane register plus an immediate offset
    auto tile_iteration = [&](auto KB, int t) __attribute__((always_inline)) {
      constexpr int kb = decltype(KB)::value;
      constexpr int kb1 = kb + 1 == kBufs ? 0 : kb + 1;
      constexpr int km1 = kb == 0 ? kBufs - 1 : kb - 1;
      constexpr int km2 = km1 == 0 ? kBufs - 1 : km1 - 1;
      const uint16_t* k_t = lds_k + kb * kKTile;     // K(t), V(t)
      const uint16_t* v_t = lds_v + kb * kVTile;
      const uint16_t* k_n = lds_k + kb1 * kKTile;    // K(t+1), V(t+1)
      const uint16_t* v_n = lds_v + kb1 * kVTile;
      const uint16_t* v_p = lds_v + km1 * kVTile;    // V(t-1)
      if (!CAUSAL && t > 0 && (t & (kIdxRing / 2 - 1)) == 0) ring_fill(t + kIdxRing / 2, kIdxRing / 2);
      // K(t+2) replaces K(t-1), V(t+1) replaces V(t-2): both were last read before the previous barrier
      if (t + 2 < n_load) dma_tile(src_k, base_k, lds_k + km1 * kKTile, dma_off_k);
      if (t + 1 < n_load) dma_tile(src_v, base_v, lds_v + km2 * kVTile, dma_off_v);
      int base_k_next = 0, base_k_next_v = 0;
      float lm_next = 0.f;
      float nmc[kRG];               // exponent offset of this tile's probabilities: p = m 2^(c (s - m_ref))
#pragma unroll
      for (int rg = 0; rg < kRG; ++rg) nmc[rg] = lm_cur - mc[rg];
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int gq = 0; gq < 32; ++gq) {
        const int step = gq >> 4, gi = gq & 15, idx = gi >> 1;
        // read early and made wave-uniform well before the next iteration's start needs it
        if (gq == 6) {
          base_k_next_v = full_base(min(t + 3, n_load - 1));
          lm_next = tile_lm(min(t + 1, n_full - 1));
        }
        if (gq == 20) {
          base_k_next = __builtin_amdgcn_readfirstlane(base_k_next_v);
        }
        // fetch ahead (the first groups of the next iteration read tiles that are already resident)
        {
          const int gp = gq + kDepth;
          ring[gp % (kDepth + 1)] = gp < 32 ? operand(gp, k_t, k_n, v_p, v_t) : operand(gp - 32, k_n, k_n, v_t, v_n);
        }
        const bf16x8 x = ring[gq % (kDepth + 1)];
        // kRG MFMAs share the operand; each is followed by its own slice of the probabilities of
        // the block whose scores are complete (one element), so that matrix and vector
        // instructions alternate in the wave's instruction stream
#pragma unroll
        for (int j = 0; j < kRG; ++j) {
          if ((gi & 1) == 0) {
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (step == 0) s1[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qreg[j][idx], idx == 0 ? zero : s1[j], 0, 0, 0);
            else s0[j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, qreg[j][idx], idx == 0 ? zero : s0[j], 0, 0, 0);
          } else {
            const int sp = idx >> 2, d = idx & 3;
            o[j][d] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(x, __builtin_bit_cast(bf16x8, step == 0 ? p1[j][sp] : p0[j][sp]), o[j][d], 0, 0, 0);
          }
          __builtin_amdgcn_sched_barrier(0);   // the MFMA first, then its slice (+0.8 % over leaving the order to the compiler)
          const int e = gi * kRG + j, rg = e >> 4, r = e & 15;
          f32x16& s = step == 0 ? s0[rg] : s1[rg];
          s[r] = fast_exp2(fmaf(s[r], c, nmc[rg]));
          // The row sum and the packing to bf16 trail the exponentials by one element / one pair, so
          // that every slice carries the same few vector instructions (a burst of eight adds and
          // four converts in one place would hold up the MFMA behind it) and none of them waits
          // for the exponential issued just before it.
          u32x4 (&pp)[2] = step == 0 ? p0[rg] : p1[rg];
          if (r >= 1) l_run[rg] += s[r - 1];
          if (r >= 2 && (r & 1) == 0) set_pair(pp[(r - 2) >> 3], ((r - 2) & 7) >> 1, s[r - 2], s[r - 1]);
          if (r == 15) {
            l_run[rg] += s[15];
            set_pair(pp[1], 3, s[14], s[15]);
          }
          __builtin_amdgcn_sched_barrier(0);
        }
      }
      // A tile that raised some lane's row sum by more than a sixteenth gets its exact correction: the sum
      // of its 32 probabilities per lane as rounded (both blocks' packed values are still in registers)
      // minus what they added to the row sum.  Rare after the first few tiles of a phase.
      {
        bool big = false;
#pragma unroll
        for (int rg = 0; rg < kRG; ++rg) big = big || l_run[rg] > kExactCorrectionGrowth * l_prev[rg];
        if (__builtin_amdgcn_ballot_w64(big) != 0) {
#pragma unroll
          for (int rg = 0; rg < kRG; ++rg) {
            float lr = 0.f;
#pragma unroll
            for (int sp = 0; sp < 2; ++sp)
#pragma unroll
              for (int i = 0; i < 4; ++i) {
                lr = add_bf16_pair(lr, p0[rg][sp][i]);
                lr = add_bf16_pair(lr, p1[rg][sp][i]);
              }
            lr_run[rg] += lr - (l_run[rg] - l_prev[rg]);
          }
        }
#pragma unroll
        for (int rg = 0; rg < kRG; ++rg) l_prev[rg] = l_run[rg];
      }
      // this wave's share of K(t+2) / V(t+1) has landed; after the barrier everybody's has, and
      // everybody is done reading K(t) block 1 and V(t-1), the buffers the next loads overwrite
      dma_wait();
      __builtin_amdgcn_s_barrier();
      asm volatile("" ::: "memory");   // no memory access moves across the barrier at compile time
      __builtin_amdgcn_sched_barrier(0);
      base_v = base_k;
      base_k = base_k_next;
      lm_cur = lm_next;
    };
    {
      int t = 0;
      while (true) {
        tile_iteration(std::integral_constant<int, 0>{}, t);
        if (++t == n_full) break;
        tile_iteration(std::integral_constant<int, 1>{}, t);
        if (++t == n_full) break;
        tile_iteration(std::integral_constant<int, 2>{}, t);
        if (++t == n_full) break;
      }
    }
    // drain: accumulate block 1 of the last tile
    {
      bf16x8 pl[kRG][2];
#pragma unroll
      for (int rg = 0; rg < kRG; ++rg) {
        pl[rg][0] = __builtin_bit_cast(bf16x8, p1[rg][0]);
        pl[rg][1] = __builtin_bit_cast(bf16x8, p1[rg][1]);
      }
      pv_block(lds_v + ((n_full - 1) % kBufs) * kVTile, 1, pl);
    }

    // did the fixed reference hold?  (row sums are sums of positive terms: one huge term shows)
    bool bad = false;
#pragma unroll
    for (int rg = 0; rg < kRG; ++rg) bad = bad || !(l_run[rg] < kFastPathLimit);
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && lane == 0) *lds_flag = 1;
    __syncthreads();
    const bool redo = *lds_flag != 0;
    __syncthreads();
    return !redo;
  };

  // ======================= the phases =======================
  // A phase is its full tiles on the fast path, then its masked ones.  Where the fixed reference fails the full
  // tiles are walked carefully too; in the second phase everything so far is spoilt and starts again.
  const std::false_type kPoolPhase{};
  const std::true_type kSelfPhase{};
  // the first phase's first loads, then the queries to registers (four loads or six left behind them, or none)
  const bool self_first = kHasSelf && nf_pool + np_pool == 0;
  const bool started = self_first ? nf_self > 0 : nf_pool > 0;
  if (kHasPool && nf_pool > 0) first_loads(kPoolPhase, a.k, a.v, nf_pool + (np_pool > 0));
  if (kHasSelf && self_first && nf_self > 0) first_loads(kSelfPhase, self_k(), self_v(), nf_self + (np_self > 0));
  if (started) asm volatile("s_waitcnt vmcnt(4)" ::: "memory");
  else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
#pragma unroll
  for (int s = 0; s < 8; ++s) qreg[0][s] = k_operand(q_lds, 0, s);
  if constexpr (kHasPool) {
    int from = 0;
    if (nf_pool > 0) {
      if (fast_phase(kPoolPhase, a.k, a.v, nf_pool, np_pool > 0, true, false)) from = nf_pool;
      else reset_state();
    }
    careful_tiles(kPoolPhase, a.k, a.v, from, nf_pool + np_pool, from > 0);
  }
  if constexpr (kHasSelf) {
    const uint16_t *new_k = self_k(), *new_v = self_v();
    int from = 0;
    if (nf_self > 0) {
      if (fast_phase(kSelfPhase, new_k, new_v, nf_self, np_self > 0, self_first, kHasPool && nf_pool + np_pool > 0)) {
        from = nf_self;
      } else {
        reset_state();
        if constexpr (kHasPool) careful_tiles(kPoolPhase, a.k, a.v, 0, nf_pool + np_pool, false);
      }
    }
    careful_tiles(kSelfPhase, new_k, new_v, from, nf_self + np_self, from > 0);     // the last ones are on the diagonal
  }

  // ---- epilogue: normalise, LSE, store ----
  const auto args = late_args();
  if (wave_row >= n_rows) return;
  // place of the lane's row behind the tile's first, in rows of the output; -1: the row does not exist
  const size_t out_row0 = (size_t)wk.out_row * args->q_heads + g * G;      // (one-pass rows: out_row is the tile's first token)
  char* mine = (char*)lds + wave_u * (MODE == 2 ? kPriorWave : 32 * kOutStride);      // the wave's stretch of LDS
  auto lane_order = []() __attribute__((always_inline)) {       // the wave's LDS writes above, its reads below, as issued
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
  };
#pragma unroll
  for (int rg = 0; rg < kRG; ++rg) {
    const float l_tot = xor32_sum(l_run[rg]);
    const float lr_tot = l_tot + xor32_sum(lr_run[rg]);
    const int row = wave_row + 32 * rg + l32, row_tok = row / args->group;         // (again: two registers less through the loops)
    const int rel = row_tok < wk.n_tok ? row_tok * args->q_heads + row - row_tok * args->group : -1;
    float inv = lr_tot > 0.f ? 1.f / lr_tot : 0.f;
    float lse_val = l_tot > 0.f ? m_ref[rg] * args->scale + __logf(l_tot) : -INFINITY;
    if (MODE == 2 && wk.n_prior > 0) {
      // One-pass tail: the row's partials in the work items above it (shared runs, computed by an
      // earlier launch) are merged in with the rule of the merge kernel,
      //   M = max LSE_j, w_j = exp(LSE_j - M), O = sum w_j O_j / sum w_j, LSE = M + ln sum w_j,
      // taken one partial at a time: (M, W, acc) <- (max(M, L), W e^(M-M') + e^(L-M'), acc e^(M-M') + O_j e^(L-M')).
      // The accumulators are brought to their normalised values first.
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int r = 0; r < 16; ++r) o[rg][d][r] *= inv;
      float M = lse_val, W = lse_val > -INFINITY ? 1.f : 0.f;
      // (a row that does not exist takes the first one's: it is not written)
      const int own = max(rel, 0);
      const unsigned prior_lds = lds_base_addr + (unsigned)wave_u * kPriorWave;
      for (int j = 0; j < wk.n_prior; ++j) {
        // the wave's 32 rows of 512 bytes through LDS, 16-byte chunk c of row r at place c ^ r (by loads of 16 bytes of 32 rows
        // each: 3 chunks of 88 to 177 tokens with six partials a row 111 us, 104.5; one partial a row in 2048 workgroups is bound by
        // HBM, 134 MB read as the row tiles of a round end together, either way)
        const size_t prow0 = (size_t)(unit::scalar_loads(args->prior_rows)[wk.prior_off + j] + wk.out_row - wk.kv_off) * args->q_heads + g * G;
        asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
        auto prior_chunk = [&](int i) __attribute__((always_inline)) -> const float* {     // of row 2 i + lane / 32
          const int r_ = 2 * i + (lane >> 5);
          return args->prior_out + (prow0 + __shfl(own, r_)) * kHeadDim + 4 * ((lane & 31) ^ r_);
        };
        if constexpr (READ & kOffGrid) {
#pragma unroll 1
          for (int i = 0; i < 16; ++i) ((uint4*)(mine + i * 1024))[lane] = load_any((const char*)prior_chunk(i));
        } else {
#pragma unroll 2
          for (int i = 0; i < 16; ++i) {
            unsigned saved_m0;
            asm volatile("s_mov_b32 %[sv], m0\n\ts_mov_b32 m0, %[d]\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %[p], off\n\ts_mov_b32 m0, %[sv]"
                         : [sv] "=&s"(saved_m0)
                         : [p] "v"(prior_chunk(i)), [d] "s"(prior_lds + (unsigned)i * 1024u)
                         : "memory");
          }
        }
        const float L = args->prior_lse[prow0 + own];
        dma_wait();
        lane_order();
        if (!(L > -INFINITY)) continue;              // a partial without keys has weight 0
        const float Mn = fmaxf(M, L);
        const float ea = M > -INFINITY ? __expf(M - Mn) : 0.f, eb = __expf(L - Mn);
#pragma unroll
        for (int d = 0; d < 4; ++d)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4) {
            const float4 x = *(const float4*)(mine + l32 * 512 + 16 * ((8 * d + 2 * q4 + h) ^ l32));
            o[rg][d][4 * q4 + 0] = o[rg][d][4 * q4 + 0] * ea + x.x * eb;
            o[rg][d][4 * q4 + 1] = o[rg][d][4 * q4 + 1] * ea + x.y * eb;
            o[rg][d][4 * q4 + 2] = o[rg][d][4 * q4 + 2] * ea + x.z * eb;
            o[rg][d][4 * q4 + 3] = o[rg][d][4 * q4 + 3] * ea + x.w * eb;
          }
        W = W * ea + eb;
        M = Mn;
      }
      lane_order();
      inv = W > 0.f ? 1.f / W : 0.f;
      lse_val = W > 0.f ? M + __logf(W) : -INFINITY;
    }
    float* lse_out = MODE == 2 ? args->final_lse : args->lse;
    if (h == 0 && rel >= 0 && lse_out) lse_out[out_row0 + rel] = lse_val;
    // The accumulators hold a row in two lanes, 16 bytes of it here and there.  They go to memory by way of the wave's own
    // stretch of LDS (the tiles are done with), so that 16 lanes write 256 bytes of one row.
    int rel_of[8];                       // of row 4 i + lane / 16, which this lane helps to write
#pragma unroll
    for (int i = 0; i < 8; ++i) rel_of[i] = __shfl(rel, 4 * i + (lane >> 4));
    const int col = 16 * (lane & 15);
    auto write_rows = [&](char* out, int row_bytes) __attribute__((always_inline)) {
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        const uint4 x = *(const uint4*)(mine + (4 * i + (lane >> 4)) * kOutStride + col);
        if (rel_of[i] >= 0) *(uint4*)(out + (size_t)rel_of[i] * row_bytes + col) = x;
      }
    };
    if (MODE == 2 && args->final_is_bf16) {
#pragma unroll
      for (int d = 0; d < 4; ++d)
#pragma unroll
        for (int q4 = 0; q4 < 4; ++q4) {
          const bf16x4 b = __builtin_convertvector(
              f32x4{o[rg][d][4 * q4 + 0] * inv, o[rg][d][4 * q4 + 1] * inv, o[rg][d][4 * q4 + 2] * inv, o[rg][d][4 * q4 + 3] * inv}, bf16x4);
          *(uint2*)(mine + l32 * kOutStride + 2 * (32 * d + 8 * q4 + 4 * h)) = __builtin_bit_cast(uint2, b);
        }
      lane_order();
      write_rows((char*)args->final_out + out_row0 * (2 * kHeadDim), 2 * kHeadDim);
      lane_order();
    } else {
      char* out = (char*)(MODE == 2 ? (float*)args->final_out : args->out) + out_row0 * (4 * kHeadDim);
#pragma unroll
      for (int half = 0; half < 2; ++half) {
#pragma unroll
        for (int d = 2 * half; d < 2 * half + 2; ++d)
#pragma unroll
          for (int q4 = 0; q4 < 4; ++q4)
            *(float4*)(mine + l32 * kOutStride + 4 * (32 * (d & 1) + 8 * q4 + 4 * h)) =
                make_float4(o[rg][d][4 * q4 + 0] * inv, o[rg][d][4 * q4 + 1] * inv, o[rg][d][4 * q4 + 2] * inv, o[rg][d][4 * q4 + 3] * inv);
        lane_order();
        write_rows(out + half * (2 * kHeadDim), 4 * kHeadDim);
        lane_order();
      }
    }
  }
}

static_assert(kThreads == unit::kThreads, "one block size for both kinds");

template <int MODE>
tl_status launch_row_tiles(const AttnArgs& a, int n_work, hipStream_t st) {
  if (n_work == 0) return TL_OK;
  const dim3 grid((unsigned)n_work * a.kv_heads * (a.halve ? 2 : 1)), block(kThreads);
  static std::atomic<uint64_t> allowed[4];
  const int read = (get_option_vread() ? kScalarV : 0) | (a.off_grid ? kOffGrid : 0);
  constexpr decltype(&row_tile_attn_kernel<MODE, 0>) kernels[4] = {row_tile_attn_kernel<MODE, 0>, row_tile_attn_kernel<MODE, 1>,
                                                                    row_tile_attn_kernel<MODE, 2>, row_tile_attn_kernel<MODE, 3>};
  auto kern = kernels[read];
  const tl_status rc = allow_lds((const void*)kern, kLds<MODE>, allowed[read]);
  if (rc != TL_OK) return rc;
  hipLaunchKernelGGL(kern, grid, block, kLds<MODE>, st, a);
  TL_HIP(hipGetLastError());
  return TL_OK;
}

}  // namespace

tl_status launch_pool_row_tiles(const AttnArgs& a, int n_work, hipStream_t st) { return launch_row_tiles<0>(a, n_work, st); }
tl_status launch_tiles_and_units(const AttnArgs& a, hipStream_t st) {
  if (!unit::can_deal(a))
    TL_FAIL(TL_EINVAL, "launch_tiles_and_units: %d kv heads cannot be dealt %d to a workgroup", a.kv_heads, 1 << a.unit_heads_log2);
  if (a.off_grid) TL_FAIL(TL_EINVAL, "launch_tiles_and_units: tensors off the 16-byte grid go in two launches");
  const dim3 grid(unit_blocks(a) + (unsigned)a.n_work * a.kv_heads), block(kThreads);
  static std::atomic<uint64_t> allowed[4];
  const bool scalar_v = get_option_vread() != 0, in_turn = a.unit_lanes < a.n_units * unit_head_blocks(a.kv_heads, a.unit_heads_log2);
  constexpr decltype(&row_tile_attn_kernel<0, 0, true>) kernels[4] = {row_tile_attn_kernel<0, 0, true>, row_tile_attn_kernel<0, 1, true>,
                                                                       row_tile_attn_kernel<0, 0, true, true>, row_tile_attn_kernel<0, 1, true, true>};
  const int which = 2 * in_turn + scalar_v;
  auto kern = kernels[which];
  constexpr size_t lds_bytes = kLdsBytes > unit::kLdsBytes ? kLdsBytes : unit::kLdsBytes;
  const tl_status rc = allow_lds((const void*)kern, lds_bytes, allowed[which]);
  if (rc != TL_OK) return rc;
  hipLaunchKernelGGL(kern, grid, block, lds_bytes, st, a);
  TL_HIP(hipGetLastError());
  return TL_OK;
}
tl_status launch_causal_row_tiles(const AttnArgs& a, int n_work, hipStream_t st) { return launch_row_tiles<1>(a, n_work, st); }
tl_status launch_fused_row_tiles(const AttnArgs& a, int n_work, hipStream_t st) { return launch_row_tiles<2>(a, n_work, st); }

}  // namespace tl
