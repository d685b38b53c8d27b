// Non-causal attention softmax(q k^T / sqrt(dh)) v for the DiT's 3D
// self-attention and text cross-attention.
//
// bfloat16 path (dh = 128): a flash-style kernel on CDNA4 matrix cores.  A
// workgroup of 8 waves owns 256 queries, 32 per wave (two blocks of 16).  Per 64-key
// tile each wave forms the transposed logits S^T = K Q^T with
// v_mfma_f32_16x16x32_bf16 (K tile from LDS as the MFMA "A" operand, the wave's Q
// fragments held in registers as "B"), so each lane's accumulators of a block belong
// to a single query and only the max is exchanged between lanes.  The reference max
// moves only when a tile's max exceeds it by more than ATT_TAU (log2 units), which
// bounds every probability by 2^ATT_TAU and spares most rescales of O; while a row's
// max stays within [ATT_MLO, ATT_TAU] the reference is 0, and a wave whose rows all
// have reference 0 takes each probability as the plain exp2 of its logit.  With QLOG2
// q arrives multiplied by the softmax scale log2(e) / sqrt(dh) (the forward's RMSNorm
// writes it so, inside its one rounding), without it each logit is scaled first.
// The probabilities are packed to bf16 and used as the "B" operand of
// O^T += V^T P^T, with V^T read from LDS; V arrives pre-transposed ([dh, keys]).  The
// softmax denominators are sums of those same bf16 probabilities, formed on the
// matrix cores too: one more MFMA per 32 keys with ones as "A".
//
// What bounds it: the matrix pipe is busy 68% of the cycles (12 heads, 16384 x 16384:
// 1.711e9 of 1024 SIMDs x 2.44e6), the softmax between the two products takes most of the
// rest, and the clock under this work is 1.95 - 2.0 GHz of 2.4 (1310 - 1350 W of 1400).
// A first form with 32x32x16 MFMAs took 9% fewer cycles at a clock that was lower by as
// much or more (1.48 against 1.61 GHz under the counters): the 16x16x32 shape moves half
// the accumulator bytes per FLOP, so it gains where its cycles can be kept down.  That
// took a loop body of one tile without a second exit (the masked last tile is a template
// instance, ring slots switch by an XOR), so that the accumulators are updated in place:
// 153 - 189 registers and no VGPR spilled (the item loop's TAIL 4 instances keep 7 SGPRs in
// vector lanes), where two unrolled tiles took 250 and the short-key kernel spilled; and
// fragments read one by one ATT_LA = 3 ahead of their MFMAs (2: up to 7% slower, 5: 2%,
// 7: 1%).  Both forms in turn on seven cards, 2 x 12 heads 32760 x 32760: 0.98, 1.01, 1.01,
// 1.03, 1.04, 1.05 and 1.05 times as fast (9.83 - 10.32 ms, 1280 - 1342 TFLOP/s); one card,
// 40 heads 8190 x 8190 1101 -> 1063 us, 2 x 12 heads 3000 x 3000 145.0 -> 143.8.
// Measured and left out: 48 queries a wave, or 12 waves of 32 (2 - 3% faster in whole
// rounds of whole tiles, slower wherever 384-query blocks leave a round part empty).
#include <math.h>

#include <algorithm>
#include <cstdlib>

#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace track {

constexpr int ATT_D = 128;
// log2 headroom before the reference max is moved (lazy rescale): probabilities
// stay below 2^64, which bf16 P and the float32 sums of up to 2^31 keys carry
constexpr float ATT_TAU = 64.0f;
constexpr float ATT_MLO = -64.0f;  // below this row max the reference leaves 0

// Maxima over the four 16-lane groups (lanes l, l + 16, l + 32, l + 48) of a and
// of b: lanes 0..31 return that of a, lanes 32..63 that of b.
__device__ __forceinline__ float group_max2(float a, float b) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(a), __float_as_uint(b), false, false);
  const float x = __uint_as_float(r[0]), y = __uint_as_float(r[1]);
  const float m = fmaxf(x, y);
  const auto t = __builtin_amdgcn_permlane16_swap(__float_as_uint(m), __float_as_uint(m), false, false);
  const float u = __uint_as_float(t[0]), v = __uint_as_float(t[1]);
  return fmaxf(u, v);
}

// K and V^T tiles travel from global memory straight into LDS
// (buffer_load ... lds, 16 bytes per lane) through a ring of two slots, with
// no register staging and no LDS store instructions.  Per tile the K source
// is a buffer resource starting at the tile's first key, so keys past Lk read
// as zero; V^T columns are addressed through the vector offset (row and
// column together), so the resource's range check covers every V^T read.
// A DMA copy lands lane-contiguously, so every layout choice is made on the
// source side: each lane picks the 16-byte chunk that belongs at its LDS
// position.  The XOR swizzles keep the 16-row fragment reads conflict free:
// K rows are 256 bytes (unit u of row r at u ^ (r & 15)); V^T rows are 128
// bytes (unit u at u ^ att_vswz(r)).  Each lane's fragment offsets are computed
// once and switch slots with an XOR.  Rows are permuted within every 32: LDS row
// 16 h + 4 q + j holds key (or channel) 8 q + 4 h + j.  A lane's logits of a pair of
// 16-key blocks are
// then 8 consecutive keys, the P operand's k-block, which meets one contiguous
// 16-byte V^T chunk, and its outputs of a pair of 16-channel blocks are 8
// consecutive channels, one 16-byte store.
__device__ __forceinline__ int att_perm(int row) {
  return (row & ~31) | (((row >> 2) & 3) << 3) | (((row >> 4) & 1) << 2) | (row & 3);
}

typedef __attribute__((address_space(3))) void* att_lds_ptr_t;

// The lane index, computed where it is used (opaque to the compiler, which would
// otherwise keep values derived from it live across long loops).
__device__ __forceinline__ int att_lane() {
  int ln;
  asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(ln));
  return ln;
}

template <int N>
__device__ __forceinline__ void att_wait_vmcnt() {
  // s_waitcnt vmcnt(N) (gfx9 encoding), expcnt and lgkmcnt not waited on
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

constexpr int ATT_NW = 8, ATT_BKV = 64;
constexpr int ATT_BQ = 32 * ATT_NW;                 // queries per workgroup
constexpr int ATT_K_BYTES = ATT_BKV * ATT_D * 2;    // K tile, 16 KB
constexpr int ATT_VROW = ATT_BKV * 2;               // V^T tile row, 128 bytes
constexpr int ATT_V_BYTES = ATT_D * ATT_VROW;       // V^T tile, 16 KB
constexpr int ATT_SLOT = ATT_K_BYTES + ATT_V_BYTES;  // one ring slot, 32 KB
// key sequences of at most this many 64-key tiles (an even number) take the item-loop kernel
constexpr int ATT_ITEMS_MAX_TILES = 32;

__device__ __forceinline__ int att_vswz(int row) { return ((row & 7) ^ ((row >> 3) & 1)) & 6; }

constexpr int ATT_LA = 3;  // fragments read ahead of their MFMAs
constexpr int ATT_QB = 2;  // 16-query blocks per wave

// What a lane keeps of its wave's 32 queries (lane l holds query 16 b + l % 16 of
// block b) across the tiles.
struct AttState {
  f32x4 o[ATT_D / 16][ATT_QB];  // O^T: channels att_perm of 16 f + 4 (l / 16) + 0..3, of query block b
  f32x4 lsum[ATT_QB];           // row sums (every element the sum of the lane's query)
  float ms;                     // reference max: block 0's in lanes 0..31, block 1's in lanes 32..63
  bool zref;                    // every row of the wave has reference 0
  __device__ __forceinline__ void reset() {
#pragma unroll
    for (int b = 0; b < ATT_QB; ++b) {
#pragma unroll
      for (int f = 0; f < ATT_D / 16; ++f) o[f][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
      lsum[b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
    }
    ms = -INFINITY;
    zref = false;
  }
};

// The value of the lane's query of block b, of one kept as ms is.
__device__ __forceinline__ float att_of_block(float v, int b, int lane) {
  const int src = (32 * b + (lane & 15)) << 2;
  return __int_as_float(__builtin_amdgcn_ds_bpermute(src, __float_as_int(v)));
}

// One 64-key tile for one wave's 32 queries: S^T = K Q^T from the slot's K
// tile, the online-softmax update (lazy rescale), and O^T += V^T P^T from the
// slot's V^T tile.  ko / vo are the lane's fragment offsets (depth step 0, key chunk
// 0; the others differ in one XOR); with MASK, keys at or past Lk get probability
// zero.  KB 16-key blocks of the tile (2: the half that ko and vo point at).  With SAFE
// a row whose logits so far are all -inf (a wave of a split sequence can begin with
// such a tile) takes reference 0 instead.
// FIRST: the sequence's first tile, which starts O and the sums (no rescale, nothing to
// zero) and the references: 212.7 -> 207.3 us at 2 x 12 heads, 32760 x 512, 12 times a CU.
template <bool MASK, bool QLOG2, int KB = ATT_BKV / 16, bool SAFE = false, bool FIRST = false>
__device__ __forceinline__ void att_tile(const uint8_t* kb, const bf16x8 (&qf)[ATT_D / 32][ATT_QB], uint32_t ko,
                                         uint32_t vo, AttState& st, int key0, int Lk, float scale_log2) {
  constexpr int QB = ATT_QB;
  typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
  const uint8_t* vb = kb + ATT_K_BYTES;
  f32x4 s[KB][QB];
#pragma unroll
  for (int i = 0; i < KB; ++i)
#pragma unroll
    for (int b = 0; b < QB; ++b) s[i][b] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  // fragment j: 16-key block j % KB of depth step j / KB
  auto kfrag = [&](int j) {
    return __builtin_bit_cast(bf16x8, *(const u32x4*)(kb + (j % KB) * 4096 + (ko ^ (uint32_t)(j / KB * 64))));
  };
  constexpr int KF = ATT_D / 32 * KB;
  bf16x8 kf[ATT_LA + 1];
#pragma unroll
  for (int j = 0; j < ATT_LA; ++j) kf[j] = kfrag(j);
#pragma unroll
  for (int j = 0; j < KF; ++j) {
    if (j + ATT_LA < KF) kf[(j + ATT_LA) % (ATT_LA + 1)] = kfrag(j + ATT_LA);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int b = 0; b < QB; ++b)
      s[j % KB][b] =
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[j % (ATT_LA + 1)], qf[j / KB][b], s[j % KB][b], 0, 0, 0);
  }
  float mx[QB];
#pragma unroll
  for (int b = 0; b < QB; ++b) mx[b] = -INFINITY;
  // valid keys from this lane's first on
  const int lim = MASK ? Lk - key0 - 8 * (att_lane() >> 4) : 0;
#pragma unroll
  for (int i = 0; i < KB; ++i)
#pragma unroll
    for (int b = 0; b < QB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        if constexpr (MASK) {
          if (32 * (i >> 1) + 4 * (i & 1) + r >= lim) s[i][b][r] = -INFINITY;
        }
        mx[b] = fmaxf(mx[b], s[i][b][r]);
      }
  const float mt = QLOG2 ? group_max2(mx[0], mx[1]) : group_max2(mx[0], mx[1]) * scale_log2;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (FIRST) {
    st.ms = mt >= ATT_MLO && mt <= ATT_TAU ? 0.0f : fmaxf(-INFINITY, mt);
    st.zref = !__ballot(st.ms != 0.0f);
  } else if (__ballot(mt > st.ms + ATT_TAU)) {
    float mn = fmaxf(st.ms, mt);
    if (mn >= ATT_MLO && mn <= ATT_TAU) mn = 0.0f;
    const float alpha = SAFE && mn == -INFINITY ? 1.0f : __builtin_amdgcn_exp2f(st.ms - mn);
    st.ms = mn;
    st.zref = !__ballot(mn != 0.0f);
    const int lane = att_lane();
#pragma unroll
    for (int b = 0; b < QB; ++b) {
      const float al = att_of_block(alpha, b, lane);
#pragma unroll
      for (int r = 0; r < 4; ++r) st.lsum[b][r] *= al;
#pragma unroll
      for (int f = 0; f < ATT_D / 16; ++f)
#pragma unroll
        for (int r = 0; r < 4; ++r) st.o[f][b][r] *= al;
    }
  }
  // probabilities exp2(s c - m) (c = 1 with QLOG2); without the shift while every row
  // of the wave has reference 0, a wave-uniform branch
  bf16x8 pf[KB / 2][QB];
  auto probs = [&](auto shift_tag) {
    constexpr bool SHIFT = decltype(shift_tag)::value;
    float nm[QB];
    if constexpr (SHIFT) {
      const int lane = att_lane();
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        nm[b] = -att_of_block(st.ms, b, lane);
        if (SAFE && nm[b] == INFINITY) nm[b] = 0.0f;
      }
    }
#pragma unroll
    for (int c = 0; c < KB / 2; ++c)
#pragma unroll
      for (int b = 0; b < QB; ++b) {
        uint32_t w[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          float x[2];
#pragma unroll
          for (int k = 0; k < 2; ++k) {
            x[k] = s[2 * c + (e >> 1)][b][2 * (e & 1) + k];
            if constexpr (SHIFT) x[k] = QLOG2 ? x[k] + nm[b] : fmaf(x[k], scale_log2, nm[b]);
            else if constexpr (!QLOG2) x[k] *= scale_log2;
          }
          const bf16x2 pb =
              __builtin_convertvector(f32x2{__builtin_amdgcn_exp2f(x[0]), __builtin_amdgcn_exp2f(x[1])}, bf16x2);
          w[e] = __builtin_bit_cast(uint32_t, pb);
        }
        pf[c][b] = __builtin_bit_cast(bf16x8, u32x4{w[0], w[1], w[2], w[3]});
      }
  };
  if (st.zref) probs(std::false_type{});
  else probs(std::true_type{});
  const bf16x8 ones = __builtin_bit_cast(bf16x8, u32x4{0x3f803f80u, 0x3f803f80u, 0x3f803f80u, 0x3f803f80u});
  // fragment j: 16-channel block j / (KB / 2), key chunk j % (KB / 2)
  auto vfrag = [&](int j) {
    return __builtin_bit_cast(
        bf16x8, *(const u32x4*)(vb + j / (KB / 2) * 16 * ATT_VROW + (vo ^ (uint32_t)(j % (KB / 2) * 64))));
  };
  constexpr int VF = ATT_D / 16 * (KB / 2);
  bf16x8 vf[ATT_LA + 1];
#pragma unroll
  for (int j = 0; j < ATT_LA; ++j) vf[j] = vfrag(j);
#pragma unroll
  for (int c = 0; c < KB / 2; ++c)
#pragma unroll
    for (int b = 0; b < QB; ++b)
      st.lsum[b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[c][b], FIRST && c == 0 ? zero : st.lsum[b], 0, 0, 0);
#pragma unroll
  for (int j = 0; j < VF; ++j) {
    if (j + ATT_LA < VF) vf[(j + ATT_LA) % (ATT_LA + 1)] = vfrag(j + ATT_LA);
    __builtin_amdgcn_sched_barrier(0);
    const int f = j / (KB / 2), c = j % (KB / 2);
#pragma unroll
    for (int b = 0; b < QB; ++b)
      st.o[f][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vf[j % (ATT_LA + 1)], pf[c][b],
                                                           FIRST && c == 0 ? zero : st.o[f][b], 0, 0, 0);
  }
}

// The wave's 32 rows from q0 on of one (batch, head): op points at row 0, channel 0.
__device__ __forceinline__ void att_store(const AttState& st, bf16_t* __restrict__ op, int64_t ldo, int q0, int Lq,
                                          int lane) {
  const bool wide = (((uintptr_t)op | (uintptr_t)(ldo * 2)) & 15) == 0;  // rows may be 8-byte aligned only
#pragma unroll
  for (int b = 0; b < ATT_QB; ++b) {
    const float inv = 1.0f / st.lsum[b][0];
    const int qi = q0 + 16 * b + (lane & 15);
    if (qi < Lq) {
      bf16_t* orow = op + (int64_t)qi * ldo + 8 * (lane >> 4);
#pragma unroll
      for (int p = 0; p < ATT_D / 32; ++p) {
        const f32x4 &x = st.o[2 * p][b], &y = st.o[2 * p + 1][b];
        const u32x4 pk = {pack_bf2(x[0] * inv, x[1] * inv), pack_bf2(x[2] * inv, x[3] * inv),
                          pack_bf2(y[0] * inv, y[1] * inv), pack_bf2(y[2] * inv, y[3] * inv)};
        if (wide) {
          *(u32x4*)(orow + 32 * p) = pk;
        } else {
          *(u32x2*)(orow + 32 * p) = u32x2{pk[0], pk[1]};
          *(u32x2*)(orow + 32 * p + 4) = u32x2{pk[2], pk[3]};
        }
      }
    }
  }
}

// TAIL: 16-key blocks computed of a ragged last tile, which is masked: 2 where it holds
// at most 32 keys, else 4; 0 if Lk is whole tiles.
template <int KIND, bool QLOG2, int TAIL>
__global__ __launch_bounds__(512) void flash_attn_bf16_kernel(const bf16_t* __restrict__ q, int64_t ldq,
                                                      const bf16_t* __restrict__ k, int64_t ldk,
                                                      const bf16_t* __restrict__ vt, int64_t ldv,
                                                      bf16_t* __restrict__ out, int64_t ldo, int H,
                                                      int Lq, int Lk, float scale_log2) {
  constexpr int BKV = ATT_BKV, D = ATT_D, BQ = ATT_BQ;
  constexpr int K_BYTES = ATT_K_BYTES, VROW = ATT_VROW, SLOT = ATT_SLOT;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * SLOT];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jq = lane & 15;
  const int g = lane >> 4;
  const int h = blockIdx.y;
  const int b = blockIdx.z;
  const int q0 = blockIdx.x * BQ + wave * 32;

  const bf16_t* kbase = k + (int64_t)b * Lk * ldk + (int64_t)h * D;
  const bf16_t* vbase = vt + ((int64_t)b * H + h) * D * ldv;

  bf16x8 qf[D / 32][ATT_QB];
#pragma unroll
  for (int i = 0; i < ATT_QB; ++i) {
    const int qi = min(q0 + 16 * i + jq, Lq - 1);
    const bf16_t* qp = q + (int64_t)b * Lq * ldq + (int64_t)h * D + (int64_t)qi * ldq + g * 8;
#pragma unroll
    for (int kc = 0; kc < D / 32; ++kc) qf[kc][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + kc * 32));
  }
  // copy i (0, 1) of this wave fills its 1 KB block 2 wave + i of the K (or
  // V^T) region; per-lane byte offsets within the tile's rows
  uint32_t koffg[2], voffg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * wave + 4 * i + (lane >> 4);
    koffg[i] = (uint32_t)((att_perm(row) * ldk + ((lane & 15) ^ (row & 15)) * 8) * 2);
    const int vr = 16 * wave + 8 * i + (lane >> 3);
    voffg[i] = (uint32_t)((att_perm(vr) * ldv + ((lane & 7) ^ att_vswz(vr)) * 8) * 2);
  }
  const int ntiles = (Lk + BKV - 1) / BKV;
  // V^T of this (batch, head): D rows of ldv keys
  // (the host keeps D * ldv * 2 and Lk * ldk * 2 below 2^32, the size field's range)
  const __amdgpu_buffer_rsrc_t rsV =
      __builtin_amdgcn_make_buffer_rsrc((void*)vbase, (short)0, (int)(uint32_t)(D * ldv * 2), 0x00020000);
  // tile t (past the end: the last tile again) into slot S
  int slot = 0;
  auto issue = [&](int t) {
    const int tt = min(t, ntiles - 1);
    const int key0 = tt * BKV;
    // K rows key0 .. Lk - 1 of this head; rows past Lk read as zero
    const __amdgpu_buffer_rsrc_t rsK = __builtin_amdgcn_make_buffer_rsrc((void*)(kbase + (int64_t)key0 * ldk), (short)0,
                                                                         (int)(uint32_t)((Lk - key0) * ldk * 2), 0x00020000);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsK, (att_lds_ptr_t)(smem + slot + wave * 2048 + i * 1024), 16, koffg[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsV, (att_lds_ptr_t)(smem + slot + K_BYTES + wave * 2048 + i * 1024), 16,
                                               voffg[i] + (uint32_t)(key0 * 2), 0, 0, 0);
    slot ^= SLOT;
  };

  // per-lane LDS fragment offsets (slot and 32-row block are immediates)
  uint32_t ko = jq * 256 + ((g ^ jq) << 4), vo = jq * VROW + ((g ^ att_vswz(jq)) << 4);

  AttState st;

  auto tile = [&](int t, auto tail_tag, auto first_tag) {
    issue(t + 1);
    constexpr int NB = decltype(tail_tag)::value;
    att_tile<(NB > 0), QLOG2, NB ? NB : BKV / 16, false, decltype(first_tag)::value>(smem, qf, ko, vo, st, t * BKV, Lk,
                                                                                     scale_log2);
    ko ^= SLOT;
    vo ^= SLOT;
    att_wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt((15 << 0) | (3 << 14) | (7 << 4) | (0 << 8));  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };

  issue(0);
  att_wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  const int whole = TAIL > 0 ? ntiles - 1 : ntiles;
  using Whole = std::integral_constant<int, 0>;
  if (TAIL == 0 || whole > 0) tile(0, Whole{}, std::true_type{});
  else st.reset();
  for (int t = 1; t < whole; ++t) tile(t, Whole{}, std::false_type{});
  if constexpr (TAIL > 0) tile(whole, std::integral_constant<int, TAIL>{}, std::false_type{});
  att_wait_vmcnt<0>();

  att_store(st, out + (int64_t)b * Lq * ldo + (int64_t)h * D, ldo, q0, Lq, lane);
}

// Split attention, for shapes whose 256-query blocks leave most CUs idle.  A
// workgroup's 8 waves are 8 / KS groups of 32 queries times KS shares of the keys:
// fewer queries per workgroup, so KS times the workgroups, each with 1 / KS of the
// steps.  A ring slot holds 128 keys (two of the tiles above); with KS = 2 a wave takes
// one tile of it, with KS = 4 one 32-key half of one.  The shares' sums meet through
// LDS at the end: 16 KB of float32 O a wave, in the ring's space.  3 heads, 1000 x 1000:
// 28.7 us with 1 share, 20.3 with 2, 15.6 with 4; 8 heads, 3001 x 3001: 71.8 / 57.6 / 83.3.
template <int KS, bool QLOG2>
__global__ __launch_bounds__(512) void flash_attn_split_kernel(const bf16_t* __restrict__ q, int64_t ldq,
                                                               const bf16_t* __restrict__ k, int64_t ldk,
                                                               const bf16_t* __restrict__ vt, int64_t ldv,
                                                               bf16_t* __restrict__ out, int64_t ldo, int H, int Lq,
                                                               int Lk, float scale_log2) {
  static_assert(KS == 2 || KS == 4, "key shares");
  constexpr int D = ATT_D, KB = KS == 2 ? 4 : 2, STEP = 2 * ATT_BKV, NK = 16 * KB;
  constexpr int STEP_BYTES = 2 * ATT_SLOT;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * STEP_BYTES];
  __shared__ float sm[8][32], sl[8][32];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int ks = wave % KS, qw = wave / KS;
  const int jq = lane & 15;
  const int g = lane >> 4;
  const int h = blockIdx.y;
  const int b = blockIdx.z;
  const int q0 = blockIdx.x * (256 / KS) + qw * 32;

  const bf16_t* kbase = k + (int64_t)b * Lk * ldk + (int64_t)h * D;
  const bf16_t* vbase = vt + ((int64_t)b * H + h) * D * ldv;
  bf16x8 qf[D / 32][2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int qi = min(q0 + 16 * i + jq, Lq - 1);
    const bf16_t* qp = q + (int64_t)b * Lq * ldq + (int64_t)h * D + (int64_t)qi * ldq + g * 8;
#pragma unroll
    for (int kc = 0; kc < D / 32; ++kc) qf[kc][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qp + kc * 32));
  }
  uint32_t koffg[2], voffg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * wave + 4 * i + (lane >> 4);
    koffg[i] = (uint32_t)((att_perm(row) * ldk + ((lane & 15) ^ (row & 15)) * 8) * 2);
    const int vr = 16 * wave + 8 * i + (lane >> 3);
    voffg[i] = (uint32_t)((att_perm(vr) * ldv + ((lane & 7) ^ att_vswz(vr)) * 8) * 2);
  }
  const __amdgpu_buffer_rsrc_t rsV =
      __builtin_amdgcn_make_buffer_rsrc((void*)vbase, (short)0, (int)(uint32_t)(D * ldv * 2), 0x00020000);
  int slot = 0;  // byte offset of the slot copied into next
  auto issue = [&](int step) {
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int key0 = step * STEP + t * ATT_BKV;
      // K rows key0 .. Lk - 1 of this head; a tile past Lk reads zeros (and the
      // last V^T tile again), which no wave uses
      const int rows = max(0, Lk - key0);
      const __amdgpu_buffer_rsrc_t rsK = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(kbase + (int64_t)min(key0, Lk) * ldk), (short)0, (int)(uint32_t)(rows * ldk * 2), 0x00020000);
      uint8_t* const dst = smem + slot + t * ATT_SLOT + wave * 2048;
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsK, (att_lds_ptr_t)(dst + i * 1024), 16, koffg[i], 0, 0, 0);
#pragma unroll
      for (int i = 0; i < 2; ++i)
        __builtin_amdgcn_raw_ptr_buffer_load_lds(rsV, (att_lds_ptr_t)(dst + ATT_K_BYTES + i * 1024), 16,
                                                 voffg[i] + (uint32_t)(min(key0, (Lk - 1) & ~(ATT_BKV - 1)) * 2), 0, 0, 0);
    }
    slot ^= STEP_BYTES;
  };

  // the lane's fragment offsets in the wave's share of slot 0
  const int share = (KS == 2 ? ks : ks >> 1) * ATT_SLOT, half = KS == 2 ? 0 : ks & 1;
  uint32_t ko = share + half * 8192 + jq * 256 + ((g ^ jq) << 4);
  uint32_t vo = share + jq * ATT_VROW + (((4 * half + g) ^ att_vswz(jq)) << 4);

  AttState st;
  st.reset();

  issue(0);
  att_wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  const int nsteps = (Lk + STEP - 1) / STEP;
  auto next = [&]() {
    ko ^= STEP_BYTES;
    vo ^= STEP_BYTES;
    att_wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt((15 << 0) | (3 << 14) | (7 << 4) | (0 << 8));  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  int key0 = ks * NK;  // the wave's first key of the step
  for (int step = 0; step + 1 < nsteps; ++step, key0 += STEP) {
    issue(step + 1);
    att_tile<false, QLOG2, KB, true>(smem, qf, ko, vo, st, key0, Lk, scale_log2);
    next();
  }
  // the last step: whole, ragged or past the end for this wave
  if (key0 < Lk) att_tile<true, QLOG2, KB, true>(smem, qf, ko, vo, st, key0, Lk, scale_log2);
  next();

  // join the shares: [wave][8 channel blocks][2 query blocks][lane] of float32 quads
  f32x4* const so = (f32x4*)smem;
#pragma unroll
  for (int f = 0; f < D / 16; ++f)
#pragma unroll
    for (int i = 0; i < 2; ++i) so[(wave * 16 + f * 2 + i) * 64 + lane] = st.o[f][i];
  const float mref[2] = {att_of_block(st.ms, 0, lane), att_of_block(st.ms, 1, lane)};
  if (g == 0) {
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      sm[wave][16 * i + jq] = mref[i];
      sl[wave][16 * i + jq] = st.lsum[i][0];
    }
  }
  __syncthreads();
  float wt[2][KS], inv[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int qr = 16 * i + jq;
    float mx = sm[qw * KS][qr], sum = 0.0f;
#pragma unroll
    for (int w = 1; w < KS; ++w) mx = fmaxf(mx, sm[qw * KS + w][qr]);
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      const float mi = sm[qw * KS + w][qr];
      wt[i][w] = mi == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(mi - mx);  // a share without keys
      sum = fmaf(wt[i][w], sl[qw * KS + w][qr], sum);
    }
    inv[i] = 1.0f / sum;
  }
  bf16_t* op = out + (int64_t)b * Lq * ldo + (int64_t)h * D + 8 * g;
  // this wave's channel blocks of the group's queries
#pragma unroll
  for (int fi = 0; fi < 8 / KS; ++fi) {
    const int f = ks * (8 / KS) + fi;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const int qi = q0 + 16 * i + jq;
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < KS; ++w) {
        const f32x4 u = so[((qw * KS + w) * 16 + f * 2 + i) * 64 + lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(wt[i][w], u[r], v[r]);
      }
      if (qi < Lq)
        *(u32x2*)(op + (int64_t)qi * ldo + 32 * (f >> 1) + 4 * (f & 1)) =
            u32x2{pack_bf2(v[0] * inv[i], v[1] * inv[i]), pack_bf2(v[2] * inv[i], v[3] * inv[i])};
    }
  }
}

// Attention over a short key sequence (text cross-attention: Lk = 512, 8
// tiles).  With one workgroup per (query block, head, batch) as above, each
// workgroup would pay its Q load, the first tile's copy and its output stores
// for only 8 tiles.  Here one workgroup per CU walks the work items
// it = (b H + h) nqb + qb, taking p, p + G, p + 2G, ...; the K / V^T copy
// ring runs on from one item's last tile into the next item's first, and each
// wave copies the Q rows of its next item into LDS (buffer_load ... lds, rows
// past Lq read as zero) while the current item runs, so an item starts with 8
// LDS reads instead of a global load.  Every wave reads back only the Q rows
// that it copied itself, so those copies need no barrier.  ntiles must be
// even: a tile's ring slot is then its index within the item modulo 2.
//
// All workgroups finish their items together, and the burst of output stores
// (16 MB over the chip) takes longer than a tile.  vmcnt counts loads and stores
// alike, in issue order (the compiler's own waits rely on it), so a copy issued
// behind the stores would make the next item's
// first tile wait for them.  The next item's first two tiles are therefore
// copied (and its Q registers read) before the stores are issued, and its first
// tile waits only for what precedes them; the Q copies, as many bytes again, are
// spread over an item's last tiles, and the outputs leave through LDS as whole 256-byte
// rows.  2 x 12 heads, 32760 queries, the three steps: 240.9 -> 227.4 us at 512 keys, 187 ->
// 161 at 226; with the present tile body 216.8 (0.95 PFLOP/s) and 137.
template <int KIND, bool QLOG2, int TAIL>
__global__ __launch_bounds__(512) void flash_attn_items_kernel(const bf16_t* __restrict__ q, int64_t ldq,
                                                               const bf16_t* __restrict__ k, int64_t ldk,
                                                               const bf16_t* __restrict__ vt, int64_t ldv,
                                                               bf16_t* __restrict__ out, int64_t ldo, int H, int Lq,
                                                               int Lk, float scale_log2, int nitems) {
  constexpr int BKV = ATT_BKV, D = ATT_D, BQ = ATT_BQ;
  constexpr int K_BYTES = ATT_K_BYTES, VROW = ATT_VROW, SLOT = ATT_SLOT;
  constexpr int QROW = D * 2;  // 256-byte Q rows in LDS
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * SLOT + BQ * QROW];
  uint8_t* const qs = smem + 2 * SLOT;

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int jq = lane & 15;
  const int g = lane >> 4;
  const int nqb = (Lq + BQ - 1) / BQ;
  const int ntiles = (Lk + BKV - 1) / BKV;
  const int G = gridDim.x;
  // item -> (query block, head, batch); the divisions run on the vector ALU,
  // readfirstlane returns the (wave-uniform) results to scalar registers so the
  // buffer resources built from them stay scalar
  auto split = [&](int it, int& qb, int& h, int& b) {
    const int bh = __builtin_amdgcn_readfirstlane(it / nqb);
    qb = __builtin_amdgcn_readfirstlane(it - bh * nqb);
    b = __builtin_amdgcn_readfirstlane(bh / H);
    h = __builtin_amdgcn_readfirstlane(bh - b * H);
  };

  uint32_t koffg[2], voffg[2];
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const int row = 8 * wave + 4 * i + (lane >> 4);
    koffg[i] = (uint32_t)((att_perm(row) * ldk + ((lane & 15) ^ (row & 15)) * 8) * 2);
    const int vr = 16 * wave + 8 * i + (lane >> 3);
    voffg[i] = (uint32_t)((att_perm(vr) * ldv + ((lane & 7) ^ att_vswz(vr)) * 8) * 2);
  }
  uint32_t ko = jq * 256 + ((g ^ jq) << 4), vo = jq * VROW + ((g ^ att_vswz(jq)) << 4);

  int slot = 0;  // byte offset of the slot copied into next
  // K / V^T tile t of item it into the next slot (no copy past the last item)
  auto issue = [&](int it, int t) {
    if (it >= nitems) return;
    int qb, h, b;
    split(it, qb, h, b);
    const int key0 = t * BKV;
    const __amdgpu_buffer_rsrc_t rsK =
        __builtin_amdgcn_make_buffer_rsrc((void*)(k + ((int64_t)b * Lk + key0) * ldk + (int64_t)h * D), (short)0,
                                          (int)(uint32_t)((Lk - key0) * ldk * 2), 0x00020000);
    const __amdgpu_buffer_rsrc_t rsV = __builtin_amdgcn_make_buffer_rsrc(
        (void*)(vt + ((int64_t)b * H + h) * D * ldv), (short)0, (int)(uint32_t)(D * ldv * 2), 0x00020000);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsK, (att_lds_ptr_t)(smem + slot + wave * 2048 + i * 1024), 16,
                                               koffg[i], 0, 0, 0);
#pragma unroll
    for (int i = 0; i < 2; ++i)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsV, (att_lds_ptr_t)(smem + slot + K_BYTES + wave * 2048 + i * 1024),
                                               16, voffg[i] + (uint32_t)(key0 * 2), 0, 0, 0);
    slot ^= SLOT;
  };
  // pieces i0 .. i1 - 1 (of 8) of this wave's 32 Q rows of item it into LDS (rows
  // past Lq read as zero)
  auto issue_q = [&](int it, int i0, int i1) {
    if (it >= nitems || i0 >= i1) return;
    int qb, h, b;
    split(it, qb, h, b);
    const int r0 = qb * BQ + wave * 32;
    const int nrows = __builtin_amdgcn_readfirstlane(max(0, min(32, Lq - r0)));  // (clamped on the vector ALU)
    const __amdgpu_buffer_rsrc_t rsQ =
        __builtin_amdgcn_make_buffer_rsrc((void*)(q + ((int64_t)b * Lq + r0) * ldq + (int64_t)h * D), (short)0,
                                          (int)(uint32_t)(nrows * ldq * 2), 0x00020000);
    // piece i fills LDS rows 4 i .. 4 i + 3 of the wave's 32 (1 KB);
    // unit u of row r sits at u ^ (r & 15).  The lane index is made opaque so
    // that these offsets are formed here, not kept live across the tiles.
    const int ln = att_lane();
    for (int i = i0; i < i1; ++i) {
      const int r = 4 * i + (ln >> 4);
      const uint32_t off = (uint32_t)((r * ldq + ((ln & 15) ^ (r & 15)) * 8) * 2);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsQ, (att_lds_ptr_t)(qs + wave * 32 * QROW + i * 1024), 16, off, 0, 0, 0);
    }
  };
  bf16x8 qf[D / 32][2];
  auto read_q = [&]() {
#pragma unroll
    for (int kc = 0; kc < D / 32; ++kc)
#pragma unroll
      for (int i = 0; i < 2; ++i)
        // the same row / unit layout as a K tile: ko (in slot 0 between items) doubles as the offset
        qf[kc][i] = __builtin_bit_cast(bf16x8, *(const u32x4*)(qs + (wave * 32 + 16 * i) * QROW + (ko ^ (uint32_t)(kc * 64))));
    __builtin_amdgcn_s_waitcnt((15 << 0) | (3 << 14) | (7 << 4) | (0 << 8));  // lgkmcnt(0): Q buffer free again
  };

  AttState st;
  // 16-byte output stores of an item per wave.  They go through a buffer resource
  // (rows past Lq are dropped there, not masked), so every wave issues as many.
  constexpr int NST = D / 16;
  // Q pieces per tile: the 8 pieces over the item's last tiles, away from the stores
  const int qper = ntiles > 8 ? 1 : (ntiles > 4 ? 2 : (ntiles > 2 ? 4 : 8));
  auto store_item = [&](int it) {
    int qb, h, b;
    split(it, qb, h, b);
    const int r0 = qb * BQ + wave * 32;
    const int nrows = __builtin_amdgcn_readfirstlane(max(0, min(32, Lq - r0)));
    const __amdgpu_buffer_rsrc_t rsO =
        __builtin_amdgcn_make_buffer_rsrc((void*)(out + ((int64_t)b * Lq + r0) * ldo + (int64_t)h * D), (short)0,
                                          (int)(uint32_t)(nrows * ldo * 2), 0x00020000);
    // the lane index, formed here so that neither it nor the offset is spilled
    // across the tiles (a reload would wait for the copies just issued)
    const int ln = att_lane();
    // through the wave's Q rows in LDS (free until the next Q pieces; unit u of row r
    // at u ^ (r & 15)), so that a store covers four whole 256-byte rows
    uint8_t* const ob = qs + wave * 32 * QROW;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
      const float inv = 1.0f / st.lsum[i][0];
      const int r = 16 * i + (ln & 15);
#pragma unroll
      for (int p = 0; p < D / 32; ++p) {
        const f32x4 &x = st.o[2 * p][i], &y = st.o[2 * p + 1][i];
        *(u32x4*)(ob + r * QROW + (((4 * p + (ln >> 4)) ^ (ln & 15)) << 4)) =
            u32x4{pack_bf2(x[0] * inv, x[1] * inv), pack_bf2(x[2] * inv, x[3] * inv),
                  pack_bf2(y[0] * inv, y[1] * inv), pack_bf2(y[2] * inv, y[3] * inv)};
      }
    }
#pragma unroll
    for (int i = 0; i < NST; ++i) {
      const int r = 4 * i + (ln >> 4), u = ln & 15;
      const u32x4 v = *(const u32x4*)(ob + r * QROW + ((u ^ (r & 15)) << 4));
      __builtin_amdgcn_raw_buffer_store_b128(v, rsO, (uint32_t)(r * ldo * 2 + u * 16), 0, 0);
    }
  };
  // tile t of item it, the copy of the tile after it in flight (the first tile's
  // successor is under way already, before the last item's stores)
  auto tile = [&](int it, int t, auto tail_tag, auto first_tag, bool stores_behind) {
    if constexpr (!decltype(first_tag)::value) {
      if (t + 1 < ntiles) issue(it, t + 1);
      else issue(it + G, 0);
      const int i1 = 8 - (ntiles - 1 - t) * qper;  // the last tiles copy the next item's Q
      issue_q(it + G, max(0, i1 - qper), min(i1, 8));
    }
    constexpr int NB = decltype(tail_tag)::value;
    att_tile<(NB > 0), QLOG2, NB ? NB : BKV / 16, false, decltype(first_tag)::value>(smem, qf, ko, vo, st, t * BKV, Lk,
                                                                                     scale_log2);
    ko ^= SLOT;
    vo ^= SLOT;
    if (stores_behind) att_wait_vmcnt<NST>();
    else att_wait_vmcnt<0>();
    __builtin_amdgcn_s_waitcnt((15 << 0) | (3 << 14) | (7 << 4) | (0 << 8));  // lgkmcnt(0)
    __builtin_amdgcn_s_barrier();
  };
  // the Q of item it to registers, the item's second tile on its way
  auto begin = [&](int it) {
    if (it >= nitems) return;
    read_q();
    issue(it, 1);
    __builtin_amdgcn_sched_barrier(0);
  };

  int it = blockIdx.x;
  issue_q(it, 0, 8);
  issue(it, 0);
  att_wait_vmcnt<0>();
  __builtin_amdgcn_s_barrier();
  begin(it);
  for (bool first = true; it < nitems; it += G, first = false) {
    const int whole = TAIL ? ntiles - 1 : ntiles;  // at least one: ntiles is even
    using Whole = std::integral_constant<int, 0>;
    tile(it, 0, Whole{}, std::true_type{}, !first);
    for (int t = 1; t < whole; ++t) tile(it, t, Whole{}, std::false_type{}, false);
    if constexpr (TAIL > 0) tile(it, whole, std::integral_constant<int, TAIL>{}, std::false_type{}, false);
    begin(it + G);
    store_item(it);
  }
  att_wait_vmcnt<0>();
}

// float32 path on v_mfma_f32_16x16x4_f32 (float32 products and sums).  A wave
// owns 16 queries and walks the keys 16 at a time: S^T = K Q^T (k index i of
// channel group c: channels 16 c + 4 g + i, g = lane / 16), then O^T += V^T P^T,
// where the logits a lane holds (keys 4 g + 0..3 of its query) are the P operand
// as they are.  K and V^T go from global memory to registers 16 bytes per lane
// (VEC; element loads where rows are not 16-byte aligned), the next 16 keys' while
// this one's are multiplied: no LDS and no barrier in the loop.  A short sequence
// leaves most of the chip idle, so with KS = 4 the workgroup's waves share one
// query block and take every fourth key block, joined at the end through LDS; with
// KS = 1 they take four query blocks and the same keys, which they then share in
// the CU's cache.
//
// It replaces one thread per query, which read V^T uncoalesced behind a serial
// chain over all keys: 2 x 4 heads of 32, 64 x 64: 35.6 -> 8.2 us; 8 heads of 64, 300 x
// 300: 303 -> 9.8 us; 2 x 8 heads of 128, 1500 x 1500: 19.9 -> 0.37 ms (50 TFLOP/s, bound by
// the L2 reads of K and V^T), each with a smaller error against float64.
template <bool VEC>
__device__ __forceinline__ f32x4 att_load4(const float* __restrict__ p) {
  if constexpr (VEC) return *(const f32x4*)p;
  else return f32x4{p[0], p[1], p[2], p[3]};
}

template <int D, int KS, bool VEC, bool VROWS>
__global__ __launch_bounds__(256) void attn_f32_kernel(const float* __restrict__ q, int64_t ldq,
                                                       const float* __restrict__ k, int64_t ldk,
                                                       const float* __restrict__ vt, int64_t ldv,
                                                       float* __restrict__ out, int64_t ldo, int H, int64_t Lq,
                                                       int64_t Lk, float scale_log2, const float* __restrict__ q_gain) {
  static_assert(KS == 1 || KS == 4, "waves per query block");
  constexpr int C = D / 16;
  __shared__ f32x4 so[KS == 4 ? 4 : 1][KS == 4 ? C : 1][64];
  __shared__ float sm[4][16], sl[4][16];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int jq = lane & 15, g = lane >> 4;
  const int h = blockIdx.y, b = blockIdx.z;
  const int64_t q0 = KS == 4 ? (int64_t)blockIdx.x * 16 : ((int64_t)blockIdx.x * 4 + wave) * 16;
  if (KS == 1 && q0 >= Lq) return;
  const int64_t qi = q0 + jq;
  const float* qp = q + ((int64_t)b * Lq + (qi < Lq ? qi : Lq - 1)) * ldq + (int64_t)h * D + 4 * g;
  const float* kb = k + (int64_t)b * Lk * ldk + (int64_t)h * D + 4 * g;
  const float* vb = VROWS ? vt + ((int64_t)b * Lk + 4 * g) * ldv + (int64_t)h * D + jq
                          : vt + (((int64_t)b * H + h) * D + jq) * ldv + 4 * g;
  f32x4 qf[C], kf[C], vf[C], o[C];
  // K row key0 + jq (the last key again past the end) and the V^T columns
  // key0 + 4 g + 0..3, zero past the end
  auto load_k = [&](int64_t key0, f32x4 (&d)[C]) {
    const float* p = kb + (key0 + jq < Lk ? key0 + jq : Lk - 1) * ldk;
#pragma unroll
    for (int c = 0; c < C; ++c) d[c] = att_load4<VEC>(p + 16 * c);
  };
  auto load_v = [&](int64_t key0, f32x4 (&d)[C]) {
    if constexpr (VROWS) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bool in = key0 + 4 * g + j < Lk;
        const float* p = vb + (in ? key0 + j : -4 * g) * ldv;
#pragma unroll
        for (int c = 0; c < C; ++c) d[c][j] = in ? p[16 * c] : 0.0f;
      }
    } else if (key0 + 16 <= Lk) {
#pragma unroll
      for (int c = 0; c < C; ++c) d[c] = att_load4<VEC>(vb + 16 * c * ldv + key0);
    } else {
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int j = 0; j < 4; ++j) d[c][j] = key0 + 4 * g + j < Lk ? vb[16 * c * ldv + key0 + j] : 0.0f;
    }
  };
#pragma unroll
  for (int c = 0; c < C; ++c) {
    qf[c] = att_load4<VEC>(qp + 16 * c);
    o[c] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  }
  if (q_gain) {  // RMSNorm of the query rows over all heads, times the gain
    const float* row = qp - (int64_t)h * D;
    float sq = 0.0f;
#pragma unroll 4
    for (int c = 0; c < H * C; ++c) {
      const f32x4 v = att_load4<VEC>(row + 16 * c);
      sq = fmaf(v[0], v[0], fmaf(v[1], v[1], fmaf(v[2], v[2], fmaf(v[3], v[3], sq))));
    }
    sq += __shfl_xor(sq, 16);
    sq += __shfl_xor(sq, 32);
    const float rstd = 1.0f / sqrtf(sq / (float)(H * D) + 1e-6f);
#pragma unroll
    for (int c = 0; c < C; ++c) {
      const f32x4 gn = att_load4<VEC>(q_gain + (int64_t)h * D + 16 * c + 4 * g);
#pragma unroll
      for (int r = 0; r < 4; ++r) qf[c][r] = qf[c][r] * rstd * gn[r];
    }
  }
  float m = -INFINITY, l = 0.0f;  // reference max (log2 units), the lane's share of the denominator
  int64_t key0 = KS == 4 ? 16 * wave : 0;
  if (key0 < Lk) {
    load_k(key0, kf);
    load_v(key0, vf);
  }
  for (; key0 < Lk; key0 += 16 * KS) {
    f32x4 kn[C], vn[C];
    const bool more = key0 + 16 * KS < Lk;
    if (more) {
      load_k(key0 + 16 * KS, kn);
      load_v(key0 + 16 * KS, vn);
    }
    f32x4 s0 = {0.0f, 0.0f, 0.0f, 0.0f}, s1 = s0;
#pragma unroll
    for (int c = 0; c < C; ++c) {
#pragma unroll
      for (int i = 0; i < 4; i += 2) {
        s0 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][i], qf[c][i], s0, 0, 0, 0);
        s1 = __builtin_amdgcn_mfma_f32_16x16x4f32(kf[c][i + 1], qf[c][i + 1], s1, 0, 0, 0);
      }
    }
    float x[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = key0 + 4 * g + r < Lk ? s0[r] + s1[r] : -INFINITY;
    const float t = fmaxf(fmaxf(x[0], x[1]), fmaxf(x[2], x[3]));
    const float mn = fmaxf(m, group_max2(t, t) * scale_log2);
    if (__ballot(mn > m)) {
      const float alpha = __builtin_amdgcn_exp2f(m - mn);
      l *= alpha;
#pragma unroll
      for (int c = 0; c < C; ++c)
#pragma unroll
        for (int r = 0; r < 4; ++r) o[c][r] *= alpha;
      m = mn;
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) x[r] = __builtin_amdgcn_exp2f(fmaf(x[r], scale_log2, -m));
    l += (x[0] + x[1]) + (x[2] + x[3]);
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int c = 0; c < C; ++c) o[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(vf[c][j], x[j], o[c], 0, 0, 0);
    if (more) {
#pragma unroll
      for (int c = 0; c < C; ++c) {
        kf[c] = kn[c];
        vf[c] = vn[c];
      }
    }
  }
  l += __shfl_xor(l, 16);
  l += __shfl_xor(l, 32);
  float* op = out + ((int64_t)b * Lq + qi) * ldo + (int64_t)h * D + 4 * g;
  auto store = [&](int c, const f32x4& v) {
    if (qi >= Lq) return;
    if constexpr (VEC) {
      *(f32x4*)(op + 16 * c) = v;
    } else {
#pragma unroll
      for (int r = 0; r < 4; ++r) op[16 * c + r] = v[r];
    }
  };
  if constexpr (KS == 1) {
    const float inv = 1.0f / l;
#pragma unroll
    for (int c = 0; c < C; ++c) store(c, f32x4{o[c][0] * inv, o[c][1] * inv, o[c][2] * inv, o[c][3] * inv});
  } else {
#pragma unroll
    for (int c = 0; c < C; ++c) so[wave][c][lane] = o[c];
    if (g == 0) {
      sm[wave][jq] = m;
      sl[wave][jq] = l;
    }
    __syncthreads();
    const float mx = fmaxf(fmaxf(sm[0][jq], sm[1][jq]), fmaxf(sm[2][jq], sm[3][jq]));
    float wt[4], sum = 0.0f;
#pragma unroll
    for (int w = 0; w < 4; ++w) {
      wt[w] = sm[w][jq] == -INFINITY ? 0.0f : __builtin_amdgcn_exp2f(sm[w][jq] - mx);  // a wave without keys
      sum = fmaf(wt[w], sl[w][jq], sum);
    }
    const float inv = 1.0f / sum;
    for (int c = wave; c < C; c += 4) {
      f32x4 v = {0.0f, 0.0f, 0.0f, 0.0f};
#pragma unroll
      for (int w = 0; w < 4; ++w) {
        const f32x4 u = so[w][c][lane];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = fmaf(wt[w], u[r], v[r]);
      }
      store(c, f32x4{v[0] * inv, v[1] * inv, v[2] * inv, v[3] * inv});
    }
  }
}

// Key shares per query block (1, 2 or 4), by an estimate of the time: rounds of
// workgroups over the CUs, times steps of a workgroup and its fixed cost.  The constants
// are fits to all three at 19 shapes (1 - 5000 queries, 1 - 40 heads), where the pick is
// within 5% of the best: a step is a 64-key tile with 1 share (1.55 us), 128 keys with 2
// (2.2: the copies of 64 KB) or 4 (1.72: half the work per wave).  A shape that fills the
// chip keeps one share: 2 x 12 heads, 1560 x 1560: 44 us, 68 with 2, 75 with 4.
// TRACK_ATTN_SPLIT = 1, 2 or 4 (read at every call) forces one, for tests.
static int pick_split(int64_t Lq, int64_t Lk, int64_t heads) {
  const char* v = getenv("TRACK_ATTN_SPLIT");
  if (v && (v[0] == '1' || v[0] == '2' || v[0] == '4')) return v[0] - '0';
  const int64_t cus = device_cus();
  const double step_us[3] = {1.55, 2.2, 1.72}, fixed_us[3] = {5.5, 8.5, 6.0};
  int best = 1;
  double best_t = 0.0;
  for (int i = 0; i < 3; ++i) {
    const int ks = 1 << i, per = i == 0 ? 64 : 128;
    const int64_t wgs = (Lq * ks + 255) / 256 * heads, rounds = (wgs + cus - 1) / cus;
    const double t = (double)rounds * ((double)((Lk + per - 1) / per) * step_us[i] + fixed_us[i]);
    if (i == 0 || t < best_t) {
      best = ks;
      best_t = t;
    }
  }
  return best;
}

float attn_log2_scale(int head_dim) { return (float)(1.4426950408889634 / sqrt((double)head_dim)); }

static track_status attention_f32(int B, int H, int head_dim, int64_t Lq, int64_t Lk, const float* q, int64_t ldq,
                                  const float* k, int64_t ldk, const float* v, int64_t ldv, float* out, int64_t ldo,
                                  bool vrows, const float* q_gain, hipStream_t s) {
  const float scale_log2 = attn_log2_scale(head_dim);
  const int64_t nqb = (Lq + 15) / 16;
  // four waves a query block until the blocks alone give every SIMD a wave
  const bool split = nqb * H * B < 4 * (int64_t)device_cus();
  const bool vec = ((ldq | ldk | ldv | ldo) & 3) == 0 &&
                   (((uintptr_t)q | (uintptr_t)k | (uintptr_t)v | (uintptr_t)out | (uintptr_t)q_gain) & 15) == 0;
  if (vrows && !vec) return fail(TRACK_E_INVALID, "attention_f32_vrows: needs 16-byte aligned rows");
  dim3 grid((unsigned)(split ? nqb : (nqb + 3) / 4), H, B);
#define TRACK_ATT_F32_K(DH, KS, VEC, VR) \
  attn_f32_kernel<DH, KS, VEC, VR><<<grid, 256, 0, s>>>(q, ldq, k, ldk, v, ldv, out, ldo, H, Lq, Lk, scale_log2, q_gain)
#define TRACK_ATT_F32(DH)                                          \
  do {                                                             \
    if (vrows && split) TRACK_ATT_F32_K(DH, 4, true, true);        \
    else if (vrows) TRACK_ATT_F32_K(DH, 1, true, true);            \
    else if (split && vec) TRACK_ATT_F32_K(DH, 4, true, false);    \
    else if (split) TRACK_ATT_F32_K(DH, 4, false, false);          \
    else if (vec) TRACK_ATT_F32_K(DH, 1, true, false);             \
    else TRACK_ATT_F32_K(DH, 1, false, false);                     \
  } while (0)
  switch (head_dim) {
    case 32: TRACK_ATT_F32(32); break;
    case 64: TRACK_ATT_F32(64); break;
    case 128: TRACK_ATT_F32(128); break;
    default: return fail(TRACK_E_UNSUPPORTED, "attention: float32 path supports head_dim 32, 64, 128 (got %d)", head_dim);
  }
#undef TRACK_ATT_F32
#undef TRACK_ATT_F32_K
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

track_status attention(int dtype, int B, int H, int head_dim, int64_t Lq, int64_t Lk, const void* q, int64_t ldq,
                       const void* k, int64_t ldk, const void* vt, int64_t ldv, void* out, int64_t ldo,
                       hipStream_t s, int prof_kind, bool q_log2) {
  if (B < 1 || H < 1 || Lq < 0 || Lk < 1) return fail(TRACK_E_SHAPE, "attention: bad sizes B=%d H=%d Lq=%lld Lk=%lld", B, H, (long long)Lq, (long long)Lk);
  if (!q || !k || !vt || !out) return fail(TRACK_E_INVALID, "attention: null pointer");
  const int64_t width = (int64_t)H * head_dim;
  if (ldq < width || ldk < width || ldo < width || ldv < Lk) return fail(TRACK_E_SHAPE, "attention: leading dimension too small");
  if (q_log2 && dtype != TRACK_DTYPE_BF16) return fail(TRACK_E_INVALID, "attention: pre-scaled q is a bf16-path input");
  if (Lq == 0) return TRACK_OK;
  ProfScope prof(prof_kind, s);
  if (dtype == TRACK_DTYPE_BF16) {
    if (head_dim != ATT_D) return fail(TRACK_E_UNSUPPORTED, "attention: bf16 path needs head_dim 128 (got %d)", head_dim);
    if (ldv % 8) return fail(TRACK_E_SHAPE, "attention: bf16 path needs ldv %% 8 == 0");
    if (ldq % 8 || ldk % 8 || ldo % 4 || ((uintptr_t)q & 15) || ((uintptr_t)k & 15) || ((uintptr_t)vt & 15) ||
        ((uintptr_t)out & 7))
      return fail(TRACK_E_INVALID, "attention: bf16 path needs 16-byte aligned rows");
    if (Lq > INT32_MAX / 2 || Lk > INT32_MAX / 2) return fail(TRACK_E_SHAPE, "attention: sequence too long");
    // the K and V^T copies address one head through 32-bit buffer offsets
    if (Lk * ldk * 2 > (int64_t)UINT32_MAX || (int64_t)ATT_D * ldv * 2 > (int64_t)UINT32_MAX)
      return fail(TRACK_E_SHAPE, "attention: K or V^T of one head spans more than 4 GiB");
    const float scale_log2 = attn_log2_scale(head_dim);
    const int cross = prof_kind == TRACK_PROF_ATTN_CROSS;
    dim3 grid((unsigned)((Lq + 255) / 256), H, B);
    const bf16_t *qq = (const bf16_t*)q, *kk = (const bf16_t*)k, *vv = (const bf16_t*)vt;
    bf16_t* oo = (bf16_t*)out;
    const int64_t ntiles = (Lk + ATT_BKV - 1) / ATT_BKV;
    // the instance of a kernel for (cross, q_log2, masked last tile)
#define TRACK_ATT_TAILS(KIND, QL, LAUNCH)  \
  do {                                     \
    if (tail == 0) LAUNCH(KIND, QL, 0);    \
    else if (tail <= 32) LAUNCH(KIND, QL, 2); \
    else LAUNCH(KIND, QL, 4);              \
  } while (0)
#define TRACK_ATT_ALL(LAUNCH)                               \
  do {                                                      \
    const int tail = (int)(Lk % ATT_BKV);                   \
    if (cross && q_log2) TRACK_ATT_TAILS(1, true, LAUNCH);  \
    else if (cross) TRACK_ATT_TAILS(1, false, LAUNCH);      \
    else if (q_log2) TRACK_ATT_TAILS(0, true, LAUNCH);      \
    else TRACK_ATT_TAILS(0, false, LAUNCH);                 \
  } while (0)
    // TRACK_ATTN_ITEMS=0 keeps short sequences on the per-block kernel (both
    // give identical bits; the tests compare them)
    const char* items_env = getenv("TRACK_ATTN_ITEMS");
    const bool items_ok = !(items_env && items_env[0] == '0');
    // (either setting leaves the sequence unsplit)
    const int ksplit = items_env ? 1 : pick_split(Lq, Lk, (int64_t)H * B);
    if (ksplit > 1) {
      dim3 sgrid((unsigned)((Lq * ksplit + 255) / 256), H, B);
#define TRACK_ATT_SPLIT(KS, QL) \
  flash_attn_split_kernel<KS, QL><<<sgrid, 512, 0, s>>>(qq, ldq, kk, ldk, vv, ldv, oo, ldo, H, (int)Lq, (int)Lk, scale_log2)
      if (ksplit == 2) {
        if (q_log2) TRACK_ATT_SPLIT(2, true);
        else TRACK_ATT_SPLIT(2, false);
      } else {
        if (q_log2) TRACK_ATT_SPLIT(4, true);
        else TRACK_ATT_SPLIT(4, false);
      }
#undef TRACK_ATT_SPLIT
      TRACK_LAUNCH_CHECK();
      return TRACK_OK;
    }
    // (the items kernel addresses 32 output rows through a 32-bit buffer size)
    if (items_ok && ntiles % 2 == 0 && ntiles <= ATT_ITEMS_MAX_TILES && ldo < ((int64_t)1 << 25)) {
      // short key sequence: one workgroup per CU over all (query block, head, batch) items
      const int64_t nitems = (int64_t)grid.x * H * B;
      if (nitems > INT32_MAX) return fail(TRACK_E_SHAPE, "attention: too many query blocks");
      const int g = (int)std::min<int64_t>(nitems, device_cus());
#define TRACK_ATT_ITEMS(KIND, QL, TAIL)                                                                          \
  flash_attn_items_kernel<KIND, QL, TAIL><<<g, 512, 0, s>>>(qq, ldq, kk, ldk, vv, ldv, oo, ldo, H, (int)Lq, (int)Lk, \
                                                            scale_log2, (int)nitems)
      TRACK_ATT_ALL(TRACK_ATT_ITEMS);
#undef TRACK_ATT_ITEMS
    } else {
#define TRACK_ATT_BLOCKS(KIND, QL, TAIL)                                                                        \
  flash_attn_bf16_kernel<KIND, QL, TAIL><<<grid, 512, 0, s>>>(qq, ldq, kk, ldk, vv, ldv, oo, ldo, H, (int)Lq, (int)Lk, \
                                                              scale_log2)
      TRACK_ATT_ALL(TRACK_ATT_BLOCKS);
#undef TRACK_ATT_BLOCKS
    }
#undef TRACK_ATT_ALL
#undef TRACK_ATT_TAILS
    TRACK_LAUNCH_CHECK();
    return TRACK_OK;
  }
  if (dtype != TRACK_DTYPE_F32) return fail(TRACK_E_INVALID, "attention: bad dtype %d", dtype);
  return attention_f32(B, H, head_dim, Lq, Lk, (const float*)q, ldq, (const float*)k, ldk, (const float*)vt, ldv,
                       (float*)out, ldo, false, nullptr, s);
}

track_status attention_f32_vrows(int B, int H, int head_dim, int64_t Lq, int64_t Lk, const float* q, int64_t ldq,
                                 const float* k, int64_t ldk, const float* v, int64_t ldv, float* out, int64_t ldo,
                                 const float* q_gain, hipStream_t s, int prof_kind) {
  const int64_t width = (int64_t)H * head_dim;
  if (B < 1 || H < 1 || Lq < 1 || Lk < 1 || ldq < width || ldk < width || ldv < width || ldo < width)
    return fail(TRACK_E_SHAPE, "attention_f32_vrows: bad sizes");
  ProfScope prof(prof_kind, s);
  return attention_f32(B, H, head_dim, Lq, Lk, q, ldq, k, ldk, v, ldv, out, ldo, true, q_gain, s);
}

}  // namespace track
