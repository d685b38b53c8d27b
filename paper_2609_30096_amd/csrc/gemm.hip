// Projection GEMMs of the denoiser: out = epilogue(A W^T + b).
//
// A is the activation matrix [M tokens, K] and W a linear weight [N, K]
// (both K-contiguous).  The bfloat16 kernel runs on CDNA4 matrix cores
// (v_mfma_f32_16x16x32_bf16) with the weight tile as the MFMA "A" operand and
// the token tile as the "B" operand, so each lane's accumulators hold one
// token and runs of consecutive output features; the epilogue then writes
// 16-byte vectors.  Epilogues fuse the bias, the tanh GELU of the MLP, and the
// adaLN gate with the float32 residual update; one variant swaps the operands
// and stores the output transposed per batch (V^T for attention).
#include <algorithm>
#include <cstdlib>
#include <type_traits>

#include "common.h"
#include "kernels.h"

namespace track {

struct EpiArgs {
  const void* bias;   // [N], weight dtype
  const float* gate;  // [N] float32 (gated residual only)
  void* out;          // output or residual
  int64_t ldo;
  // transposed output (EPI_BIAS_VT): column n of row m goes to
  // vt[((m / L) * N + n) * ldv + m % L], m counted from m_off
  void* vt = nullptr;
  int64_t ldv = 0, L = 1, m_off = 0;
  int nv = 0;  // N
  // products of a batch (blockIdx.z): element strides of W and bias (one stride), and of out
  int64_t zw = 0, zo = 0;
};

// Persistent-kernel epilogue that writes the output transposed per batch
// (V^T for attention); internal to the library (linear_vt), not an ABI
// epilogue code.
constexpr int EPI_BIAS_VT = 16;

// ------------------------------------------------------------------ epilogues
template <int EPI, typename T>
__device__ __forceinline__ void epi_store1(const EpiArgs& e, int64_t m, int n, float v) {
  v += ldf((const T*)e.bias + n);
  if constexpr (EPI == TRACK_EPI_BIAS || EPI == TRACK_EPI_BIAS_GELU) {
    if constexpr (EPI == TRACK_EPI_BIAS_GELU) v = gelu_tanh(v);
    stf((T*)e.out + m * e.ldo + n, v);
  } else if constexpr (EPI == TRACK_EPI_GATE_RESID) {
    float* o = (float*)e.out + m * e.ldo + n;
    *o = fmaf(e.gate[n], v, *o);
  } else if constexpr (EPI == TRACK_EPI_RESID) {
    float* o = (float*)e.out + m * e.ldo + n;
    *o += v;
  } else {
    ((float*)e.out)[m * e.ldo + n] = v;
  }
}

// Epilogue of an MFMA tile: lane holds token m_base + 32 ti and features
// n_base + 32 fi + 8 g + {0..3}.  The lane's bias values are loaded (packed
// bf16) before any store, and the output pointer is declared unaliased, so
// the loads are not serialised behind the stores.
template <int EPI, int FI, int TI>
__device__ __forceinline__ void epilogue(const EpiArgs& e, const f32x16 (&acc)[FI][TI], int64_t M, int64_t m_base,
                                         int n_base) {
  const bf16_t* __restrict__ bias_p = (const bf16_t*)e.bias;
  const float* __restrict__ gate_p = e.gate;
#pragma unroll
  for (int fi = 0; fi < FI; ++fi) {
    u32x2 bias[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) bias[g] = *(const u32x2*)(bias_p + n_base + fi * 32 + 8 * g);
#pragma unroll
    for (int ti = 0; ti < TI; ++ti) {
      const int64_t m = m_base + ti * 32;
      if (m >= M) continue;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        const int n = n_base + fi * 32 + 8 * g;
        const u32x2 bv = bias[g];
        float v[4];
        v[0] = acc[fi][ti][4 * g + 0] + __uint_as_float(bv[0] << 16);
        v[1] = acc[fi][ti][4 * g + 1] + __uint_as_float(bv[0] & 0xffff0000u);
        v[2] = acc[fi][ti][4 * g + 2] + __uint_as_float(bv[1] << 16);
        v[3] = acc[fi][ti][4 * g + 3] + __uint_as_float(bv[1] & 0xffff0000u);
        if constexpr (EPI == TRACK_EPI_BIAS || EPI == TRACK_EPI_BIAS_GELU) {
          if constexpr (EPI == TRACK_EPI_BIAS_GELU) {
#pragma unroll
            for (int j = 0; j < 4; ++j) v[j] = gelu_tanh(v[j]);
          }
          u32x2 pk;
          pk[0] = pack_bf2(v[0], v[1]);
          pk[1] = pack_bf2(v[2], v[3]);
          bf16_t* __restrict__ o = (bf16_t*)e.out + m * e.ldo + n;
          *(u32x2*)o = pk;
        } else if constexpr (EPI == TRACK_EPI_GATE_RESID || EPI == TRACK_EPI_RESID) {
          float* __restrict__ o = (float*)e.out + m * e.ldo + n;
          f32x4 x = *(f32x4*)o;
          if constexpr (EPI == TRACK_EPI_GATE_RESID) {
            const f32x4 gt = *(const f32x4*)(gate_p + n);
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] = fmaf(gt[j], v[j], x[j]);
          } else {
#pragma unroll
            for (int j = 0; j < 4; ++j) x[j] += v[j];
          }
          *(f32x4*)o = x;
        } else {
          float* __restrict__ o = (float*)e.out + m * e.ldo + n;
          *(f32x4*)o = f32x4{v[0], v[1], v[2], v[3]};
        }
      }
    }
  }
}

// ------------------------------------------------------------------ bf16 MFMA kernel
// 16-byte chunk swizzle of a 128-byte LDS row: 8 consecutive rows get
// distinct chunks, and rows r and r + 8 differ as well, so 32-row fragment
// reads are conflict free whether LDS serves 8 or 16 lanes per cycle.
__device__ __forceinline__ int lds_swz(int row) { return (row & 7) ^ ((row >> 3) & 1); }

// Any leading dimension (64-bit addresses).  Block tile BM tokens x BN features
// x 64 (K); four waves in a 2 x 2 grid, each owning (BM/2) x (BN/2) as 32 x 32
// MFMA blocks.  Tiles are staged
// through LDS, double buffered, rows of 64 bf16 (128 B) with the 16-byte
// chunk index XOR-swizzled (lds_swz) so that the 32-row fragment reads are
// bank-conflict free.  Global loads of the next K-slab are issued before
// the MFMAs of the current one.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                        const bf16_t* __restrict__ W, int64_t M, int N, int K,
                                                        EpiArgs e) {
  constexpr int BM = 128, BN = 64, BK = 64;
  constexpr int WM = BM / 2, WN = BN / 2;
  constexpr int TI = WM / 32, FI = WN / 32;
  constexpr int AC = BM / 32;  // 16-byte chunks per thread for the A tile (BM * 8 / 256)
  constexpr int WC = BN / 32;
  constexpr int TILE_BYTES = (BM + BN) * 128;
  __shared__ __attribute__((aligned(16))) uint8_t smem[2 * TILE_BYTES];

  const int tid = threadIdx.x;
  const int lane = tid & 63;
  const int wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;

  // tile order: XCD-aware remap, then bands of 8 M-tiles swept across N
  const int num_tm = (int)((M + BM - 1) / BM);
  const int num_tn = N / BN;
  const int pid = xcd_remap(blockIdx.x, gridDim.x);
  constexpr int G = 8;
  const int band = pid / (G * num_tn);
  const int first_tm = band * G;
  const int gsz = min(num_tm - first_tm, G);
  const int in_band = pid - band * G * num_tn;
  const int tm = first_tm + in_band % gsz;
  const int tn = in_band / gsz;
  const int64_t m0 = (int64_t)tm * BM;
  const int n0 = tn * BN;

  // staging: thread handles chunk column c = tid & 7 of rows (tid >> 3) + 32 i
  const int c = tid & 7;
  const int r0 = tid >> 3;
  const bf16_t* a_ptr[AC];
#pragma unroll
  for (int i = 0; i < AC; ++i) {
    int64_t row = m0 + r0 + 32 * i;
    if (row > M - 1) row = M - 1;
    a_ptr[i] = A + row * lda + c * 8;
  }
  const bf16_t* w_ptr = W + (int64_t)(n0 + r0) * K + c * 8;

  u32x4 ra[AC], rw[WC];
  auto load_global = [&](int kt) {
    const int k0 = kt * BK;
#pragma unroll
    for (int i = 0; i < AC; ++i) ra[i] = *(const u32x4*)(a_ptr[i] + k0);
#pragma unroll
    for (int i = 0; i < WC; ++i) rw[i] = *(const u32x4*)(w_ptr + (int64_t)32 * i * K + k0);
  };
  auto store_lds = [&](int buf) {
    uint8_t* base = smem + buf * TILE_BYTES;
#pragma unroll
    for (int i = 0; i < AC; ++i) {
      const int row = r0 + 32 * i;
      *(u32x4*)(base + row * 128 + ((c ^ lds_swz(row)) << 4)) = ra[i];
    }
#pragma unroll
    for (int i = 0; i < WC; ++i) {
      const int row = r0 + 32 * i;
      *(u32x4*)(base + (BM + row) * 128 + ((c ^ lds_swz(row)) << 4)) = rw[i];
    }
  };

  f32x16 acc[FI][TI];
#pragma unroll
  for (int fi = 0; fi < FI; ++fi)
#pragma unroll
    for (int ti = 0; ti < TI; ++ti)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[fi][ti][r] = 0.0f;

  const int KT = K / BK;
  load_global(0);
  store_lds(0);
  __syncthreads();

  const int frow = lane & 31;
  const int fhalf = lane >> 5;
  for (int kt = 0; kt < KT; ++kt) {
    const int cur = kt & 1;
    if (kt + 1 < KT) load_global(kt + 1);
    const uint8_t* base = smem + cur * TILE_BYTES;
#pragma unroll
    for (int kk = 0; kk < BK / 16; ++kk) {
      const int ch = kk * 2 + fhalf;
      bf16x8 fw[FI], fa[TI];
#pragma unroll
      for (int fi = 0; fi < FI; ++fi) {
        const int row = wn * WN + fi * 32 + frow;
        fw[fi] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + (BM + row) * 128 + ((ch ^ lds_swz(row)) << 4)));
      }
#pragma unroll
      for (int ti = 0; ti < TI; ++ti) {
        const int row = wm * WM + ti * 32 + frow;
        fa[ti] = __builtin_bit_cast(bf16x8, *(const u32x4*)(base + row * 128 + ((ch ^ lds_swz(row)) << 4)));
      }
#pragma unroll
      for (int fi = 0; fi < FI; ++fi)
#pragma unroll
        for (int ti = 0; ti < TI; ++ti)
          acc[fi][ti] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fw[fi], fa[ti], acc[fi][ti], 0, 0, 0);
    }
    if (kt + 1 < KT) store_lds(cur ^ 1);
    __syncthreads();
  }

  // epilogue: lane holds token (lane & 31) and features 8g + 4 (lane >> 5) + {0..3}
  epilogue<EPI, FI, TI>(e, acc, M, m0 + wm * WM + frow, n0 + wn * WN + 4 * fhalf);
}

// ------------------------------------------------------------------ persistent bf16 MFMA kernel
// One workgroup per CU loops over the 256 x 256 output tiles p, p + G, p + 2G,
// ... (p the XCD-remapped block index, G the grid), so the copy pipeline runs
// on from one tile into the next and a tile's epilogue overlaps the loads of
// the next tile's first slabs.  Four waves in a 2 x 2 grid own 128 x 128 each as
// 8 x 8 blocks of v_mfma_f32_16x16x32_bf16.
//
// K-slabs of 64 (128-byte rows) travel global -> LDS through a 2-slot ring
// with buffer_load ... lds (16 bytes per lane, lane-contiguous in LDS); a
// buffer resource per tile makes rows past M read as zero.  A slab is two
// 32-deep steps of 64 MFMAs.  The fragments of a step are read one per MFMA
// during the step before it, into the other half of a register double buffer,
// so a slab's last reads are over a third of the way into it: its one barrier
// sits there, after which the slot is refilled with slab g + 2 (one copy per
// PK_DPM MFMAs, in program order; 3 or 4 stalls the wave behind the load unit,
// 2-8% slower) while two thirds of slab g are still to be multiplied.  LDS rows carry a
// 32-byte-granular XOR swizzle applied on the global side: no bank conflicts on
// the 16-row fragment reads, and lane pairs keep contiguous 32-byte pieces of a
// row, which the load path coalesces better than a 16-byte permutation (3% slower).
//
// The 16x16x32 shape moves half the accumulator bytes of 32x32x16 per FLOP, and
// the chip's clock under matrix work follows that: a stream of it
// (mfma_stream_kernel) holds 1950-2020 TFLOP/s on N(0,1) operands where 32x32x16
// holds 1720-1835, and this kernel ran 6-9% faster with it at every Wan projection
// (14B FFN1 6994 -> 6468 us, 1.3B O 393 -> 371; on another card q/k 5.02 -> 4.57
// ms, 1378 -> 1505 TFLOP/s).  What bounds it now (s_memtime copy, 14B q/k): 2470 of
// the 2048 cycles per slab the MFMAs need, 140 of the excess the copies' issue
// waiting on L2 misses, 10 k cycles of output stores per tile (220 k).  The
// accumulators fill the 256 AGPRs; 3-4 VGPRs (10 in the transposed form) are
// spilled, and reloaded once a tile, outside the slab loop.
__device__ __forceinline__ int lds_swz16(int row) { return ((row & 7) ^ ((row >> 3) & 1)) & ~1; }

typedef __attribute__((address_space(3))) void* lds_ptr_t;

template <int N>
__device__ __forceinline__ void wait_vmcnt() {
  // s_waitcnt with vmcnt = N (gfx9 encoding: low 4 bits and bits 15:14),
  // expcnt and lgkmcnt left at their maxima (no wait)
  static_assert(N >= 0 && N < 64, "vmcnt range");
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | (7 << 4) | (15 << 8));
}

__device__ __forceinline__ void wait_lgkm0() { __builtin_amdgcn_s_waitcnt((15 << 0) | (3 << 14) | (7 << 4) | (0 << 8)); }

constexpr int PK_F = 8;     // 16-row fragments per wave and operand
constexpr int PK_RS = 2;    // MFMAs per fragment read
constexpr int PK_BAR = 40;  // the slab's barrier follows MFMA 40 of its first step
constexpr int PK_DPM = 5;   // MFMAs per copy

// The MFMA "A" operand's rows (features; tokens in the transposed-output
// kernels) sit permuted in LDS, within every 32 rows: row 16 h + 4 q + j holds
// row 8 q + 4 h + j.  A lane's accumulators of the fragment pair 2 p, 2 p + 1
// (rows 4 q + j of each) are then 8 consecutive rows 32 p + 8 q + 0..7: whole
// 16-byte bf16 stores without a lane exchange.
//
// Epilogue of a tile with bfloat16 output (bias, bias + GELU): the lane holds
// tokens m_base + 16 y and features n_base + 32 p + 0..7, one 16-byte store to a row
// that need only be 8-byte aligned (ldo % 4 == 0).  Every bias value is
// loaded before the first store (a load issued after a store would wait for
// it).  Token blocks outermost: the 64-byte pieces of a token row's 128-byte
// line are stored back to back, so the L2 holds whole lines when it writes
// them back (feature blocks outermost left lines half written long enough to be
// evicted and written twice: 20% more HBM writes).
template <int EPI, int XF, int YF>
__device__ __forceinline__ void epilogue_bf16(const EpiArgs& e, const f32x4 (&acc)[XF][YF], int64_t M,
                                              int64_t m_base, int n_base) {
  const bf16_t* __restrict__ bias_p = (const bf16_t*)e.bias + n_base;
  u32x2 bias[XF];
#pragma unroll
  for (int f = 0; f < XF; ++f) bias[f] = *(const u32x2*)(bias_p + 32 * (f >> 1) + 4 * (f & 1));
#pragma unroll
  for (int y = 0; y < YF; ++y) {
    const int64_t m = m_base + y * 16;
    bf16_t* __restrict__ orow = (bf16_t*)e.out + m * e.ldo + n_base;
#pragma unroll
    for (int p = 0; p < XF / 2; ++p) {
      u32x4 pk;
#pragma unroll
      for (int h = 0; h < 2; ++h) {
        const u32x2 bv = bias[2 * p + h];
        const f32x4& c = acc[2 * p + h][y];
        float v[4];
        v[0] = c[0] + __uint_as_float(bv[0] << 16);
        v[1] = c[1] + __uint_as_float(bv[0] & 0xffff0000u);
        v[2] = c[2] + __uint_as_float(bv[1] << 16);
        v[3] = c[3] + __uint_as_float(bv[1] & 0xffff0000u);
        if constexpr (EPI == TRACK_EPI_BIAS_GELU) {
#pragma unroll
          for (int j = 0; j < 4; ++j) v[j] = gelu_tanh(v[j]);
        }
        pk[2 * h] = pack_bf2(v[0], v[1]);
        pk[2 * h + 1] = pack_bf2(v[2], v[3]);
      }
      if (m < M) *(u32x4_a8*)(orow + 32 * p) = pk;
    }
  }
}

// Epilogue of a tile with float32 output (gated residual, residual, plain).
// The bias and gate values are loaded first, and the residual rows of token
// block y + 1 before the stores of block y are issued, so no load waits behind
// a store of the same tile.
template <int XF>
__device__ __forceinline__ void load_resid(const EpiArgs& e, int64_t M, int64_t m, int n_base, f32x4 (&x)[XF]) {
  const float* __restrict__ out = (const float*)e.out + n_base;
#pragma unroll
  for (int f = 0; f < XF; ++f)
    x[f] = m < M ? *(const f32x4*)(out + m * e.ldo + 32 * (f >> 1) + 4 * (f & 1)) : f32x4{0, 0, 0, 0};
}

template <int EPI, int XF, int YF>
__device__ __forceinline__ void epilogue_f32(const EpiArgs& e, const f32x4 (&acc)[XF][YF], int64_t M,
                                             int64_t m_base, int n_base) {
  constexpr bool RES = EPI == TRACK_EPI_GATE_RESID || EPI == TRACK_EPI_RESID;
  constexpr bool GATE = EPI == TRACK_EPI_GATE_RESID;
  const bf16_t* __restrict__ bias_p = (const bf16_t*)e.bias + n_base;
  float* __restrict__ out = (float*)e.out + n_base;
  u32x2 bias[XF];
  f32x4 gate[XF];
  f32x4 x[2][XF];
#pragma unroll
  for (int f = 0; f < XF; ++f) {
    bias[f] = *(const u32x2*)(bias_p + 32 * (f >> 1) + 4 * (f & 1));
    if constexpr (GATE) gate[f] = *(const f32x4*)(e.gate + n_base + 32 * (f >> 1) + 4 * (f & 1));
  }
  if constexpr (RES) load_resid<XF>(e, M, m_base, n_base, x[0]);
#pragma unroll
  for (int y = 0; y < YF; ++y) {
    if constexpr (RES) {
      if (y + 1 < YF) load_resid<XF>(e, M, m_base + (y + 1) * 16, n_base, x[(y + 1) & 1]);
    }
    __builtin_amdgcn_sched_barrier(0);  // keep those loads ahead of this block's stores
    const int64_t m = m_base + y * 16;
#pragma unroll
    for (int f = 0; f < XF; ++f) {
      const u32x2 bv = bias[f];
      const f32x4& c = acc[f][y];
      f32x4 v;
      v[0] = c[0] + __uint_as_float(bv[0] << 16);
      v[1] = c[1] + __uint_as_float(bv[0] & 0xffff0000u);
      v[2] = c[2] + __uint_as_float(bv[1] << 16);
      v[3] = c[3] + __uint_as_float(bv[1] & 0xffff0000u);
      if constexpr (GATE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = fmaf(gate[f][j], v[j], x[y & 1][f][j]);
      } else if constexpr (RES) {
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = x[y & 1][f][j] + v[j];
      }
      if (m < M) *(f32x4*)(out + m * e.ldo + 32 * (f >> 1) + 4 * (f & 1)) = v;
    }
  }
}

// Epilogue of the transposed-output GEMM: out^T per batch.  Tokens are the
// MFMA "A" operand here, so the lane holds feature feat + 16 y and 8
// consecutive tokens tok0 + 32 p + 8 q + 0..7: one 16-byte store along the
// output row.  Requires L % 8 == 0, so that 8 tokens starting at a multiple of
// 8 share a batch, L >= 128 (the wave's at most 128 tokens then cross at most
// one batch boundary) and ldv % 8 == 0.
template <int XF, int YF>
__device__ __forceinline__ void epilogue_vt(const EpiArgs& e, const f32x4 (&acc)[XF][YF], int64_t M, int64_t tok0,
                                            int q, int feat) {
  static_assert(XF <= 8, "a wave's tokens cross at most one batch boundary");
  const int64_t mg0 = e.m_off + tok0;
  const int64_t b0 = mg0 / e.L;
  const int64_t l0 = mg0 - b0 * e.L;
  bf16_t* __restrict__ vt = (bf16_t*)e.vt;
  const bf16_t* __restrict__ bias_p = (const bf16_t*)e.bias + feat;
  float bias[YF];
#pragma unroll
  for (int y = 0; y < YF; ++y) bias[y] = bf2f(bias_p[16 * y]);
#pragma unroll
  for (int y = 0; y < YF; ++y) {
#pragma unroll
    for (int p = 0; p < XF / 2; ++p) {
      const f32x4 &c0 = acc[2 * p][y], &c1 = acc[2 * p + 1][y];
      const float bv = bias[y];
      const u32x4 pk = {pack_bf2(c0[0] + bv, c0[1] + bv), pack_bf2(c0[2] + bv, c0[3] + bv),
                        pack_bf2(c1[0] + bv, c1[1] + bv), pack_bf2(c1[2] + bv, c1[3] + bv)};
      const int t = 32 * p + 8 * q;
      if (tok0 + t < M) {
        int64_t l = l0 + t, b = b0;
        if (l >= e.L) {
          l -= e.L;
          ++b;
        }
        *(u32x4*)(vt + (b * e.nv + feat + 16 * y) * e.ldv + l) = pk;
      }
    }
  }
}

// The tile epilogue of `EPI`: tokens tok0 .. and features feat0 .. are the
// wave's, frow = lane % 16, q = lane / 16.
template <int EPI, int XF, int YF>
__device__ __forceinline__ void tile_epilogue(const EpiArgs& e, const f32x4 (&acc)[XF][YF], int64_t M, int64_t tok0,
                                              int feat0, int frow, int q) {
  if constexpr (EPI == EPI_BIAS_VT)
    epilogue_vt<XF, YF>(e, acc, M, tok0, q, feat0 + frow);
  else if constexpr (EPI == TRACK_EPI_BIAS || EPI == TRACK_EPI_BIAS_GELU)
    epilogue_bf16<EPI, XF, YF>(e, acc, M, tok0 + frow, feat0 + 8 * q);
  else
    epilogue_f32<EPI, XF, YF>(e, acc, M, tok0 + frow, feat0 + 8 * q);
}

template <int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_persist_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                                const bf16_t* __restrict__ W, int64_t M, int N,
                                                                int K, EpiArgs e, int ntiles, int GB) {
  constexpr int BM = 256, BN = 256, BK = 64, NWV = 4;
  constexpr int ROWB = BK * 2;                               // 128-byte LDS rows, 8 chunks of 16 bytes
  constexpr int STAGE_BYTES = (BM + BN) * ROWB;              // 64 KB per slot: A tile, then W tile
  constexpr int LOADS = (BM + BN) / 8 / NWV;                 // 16 per wave and slab
  constexpr int F = PK_F;
  constexpr bool VT = EPI == EPI_BIAS_VT;
  __shared__ __attribute__((aligned(1024))) uint8_t smem[2 * STAGE_BYTES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  const int num_tm = (int)((M + BM - 1) / BM), num_tn = N / BN;
  const int G = gridDim.x;
  const int p = xcd_remap(blockIdx.x, G);
  // tile order: bands of GB M-tiles swept across N
  auto tile_mn = [&](int T, int64_t& m0, int& n0) {
    const int band = T / (GB * num_tn);
    const int first_tm = band * GB;
    const int gsz = min(num_tm - first_tm, GB);
    const int in_band = T - band * GB * num_tn;
    m0 = (int64_t)(first_tm + in_band % gsz) * BM;
    n0 = (in_band / gsz) * BN;
  };

  // Load i of a wave fills the 8 LDS rows 32 (i % 8) + 8 wave .. + 7 of the A
  // tile (i < 8) or of the W tile, lane -> row + lane / 8, fetching the global
  // chunk that the swizzle puts at LDS chunk lane % 8.
  const int lrow = lane >> 3;
  const int lcol = ((lane & 7) ^ lds_swz16(wave * 8 + lrow)) * 8;
  const int plain_row = wave * 8 + lrow;
  const int perm_row = 8 * (2 * (wave & 1) + (lrow >> 2)) + 4 * (wave >> 1) + (lrow & 3);
  const uint32_t voffA = (uint32_t)(((VT ? perm_row : plain_row) * lda + lcol) * 2);
  const uint32_t voffW = (uint32_t)(((VT ? plain_row : perm_row) * (int64_t)K + lcol) * 2);
  __amdgpu_buffer_rsrc_t rsA, rsW;
  auto set_src = [&](int T) {
    int64_t m0;
    int n0;
    tile_mn(T, m0, n0);
    // the host keeps (M - m0) * lda * 2 below 2^31
    rsA = __builtin_amdgcn_make_buffer_rsrc((void*)(A + m0 * lda), (short)0, (int)((M - m0) * lda * 2), 0x00020000);
    rsW = __builtin_amdgcn_make_buffer_rsrc((void*)(W + (int64_t)n0 * K), (short)0, (int)((int64_t)BN * K * 2), 0x00020000);
  };
  const int KT = K / BK;
  int ld_T = p, ld_kt = 0, ld_slot = 0;
  set_src(p);
  // The A row of a load is part of its vector offset and only the slab's
  // column offset (less than a row) is scalar, so a row past M lies beyond
  // the resource's size whatever the scalar part, and an in-range row's
  // address stays inside that row.
  uint32_t voA[LOADS / 2];
  // formed anew for every tile (the lane offset is made opaque), so that they
  // are not kept, and spilled, across the epilogue
  auto set_vo = [&]() {
    uint32_t v = voffA;
    asm volatile("" : "+v"(v));
#pragma unroll
    for (int i = 0; i < LOADS / 2; ++i) voA[i] = v + (uint32_t)(i * 32 * lda * 2);
  };
  auto issue_one = [&](int i) {
    lds_ptr_t d = (lds_ptr_t)(smem + ld_slot * STAGE_BYTES + (i * 32 + wave * 8) * ROWB);
    if (i < LOADS / 2)
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsA, d, 16, voA[i], ld_kt * BK * 2, 0, 0);
    else
      __builtin_amdgcn_raw_ptr_buffer_load_lds(rsW, d, 16, voffW, (int)(((i - LOADS / 2) * 32 * (int64_t)K + ld_kt * BK) * 2), 0, 0);
  };
  // After the last slab of the last tile the loads keep re-fetching that tile
  // (in bounds, into a slot nobody reads again).
  auto advance_ld = [&]() {
    ld_slot ^= 1;
    if (++ld_kt == KT) {
      ld_kt = 0;
      if (ld_T + G < ntiles) {
        ld_T += G;
        set_src(ld_T);
      }
    }
  };

  // LDS byte offsets of the lane's fragments, 32-deep step 0 of slot 0: lane ->
  // row lane % 16, chunk lane / 16 (step 1: chunk + 4, an XOR of 64 bytes
  // either way; fragment f: + 2048 f)
  const int frow = lane & 15, q = lane >> 4;
  const uint32_t foff = (uint32_t)(frow * ROWB + ((q ^ lds_swz16(frow)) << 4));
  const uint32_t offA = (uint32_t)(wm * 128 * ROWB) + foff, offW = (uint32_t)((BM + wn * 128) * ROWB) + foff;
  uint32_t xo = VT ? offA : offW, yo = VT ? offW : offA;  // MFMA "A" and "B" operand
  auto frag = [&](uint32_t o, int f) { return __builtin_bit_cast(bf16x8, *(const u32x4*)(smem + o + f * 16 * ROWB)); };

  f32x4 acc[F][F];
  bf16x8 fx[2][F], fy[2][F];
  // MFMAs j0 .. j1 of a step, with the reads of the next step's fragments (one
  // per PK_RS MFMAs from MFMA 0 on) and, with load0 >= 0, the copies from load0 on
  auto mfmas = [&](int kk, int j0, int j1, bool zero, uint32_t nx, uint32_t ny, int load0, int dpm) {
    bf16x8 *rx = fx[kk ^ 1], *ry = fy[kk ^ 1];
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      if (j % PK_RS == 0 && j / PK_RS < 2 * F) {
        const int r = j / PK_RS;
        if (r < F) ry[r] = frag(ny, r);
        else rx[r - F] = frag(nx, r - F);
      }
      const int x = j / F, y = j % F;
      acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[kk][x], fy[kk][y], zero ? f32x4{0, 0, 0, 0} : acc[x][y], 0, 0, 0);
      if (load0 >= 0 && (j - j0) % dpm == 0 && load0 + (j - j0) / dpm < LOADS) issue_one(load0 + (j - j0) / dpm);
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  constexpr int L0 = (64 - PK_BAR + PK_DPM - 1) / PK_DPM;  // loads issued during step 0
  static_assert(PK_BAR > PK_RS * (2 * F - 1) && PK_BAR <= 64 && L0 + (64 + PK_DPM - 1) / PK_DPM >= LOADS, "slab schedule");
  auto slab = [&](auto first_tag) {
    constexpr bool FIRST = decltype(first_tag)::value;
    mfmas(0, 0, PK_BAR, FIRST, xo ^ 64, yo ^ 64, -1, 1);
    // slab g + 1 has landed for this wave (and, at a tile's first slab, the
    // previous epilogue's stores are complete) and the wave holds all of slab
    // g's fragments; after the barrier both hold for every wave
    wait_vmcnt<0>();
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(0, PK_BAR, 64, FIRST, xo ^ 64, yo ^ 64, 0, PK_DPM);  // slab g + 2 into slab g's slot
    xo ^= STAGE_BYTES;
    yo ^= STAGE_BYTES;
    mfmas(1, 0, 64, false, xo, yo, L0, PK_DPM);
    advance_ld();
  };

  // prologue: slabs 0 and 1, slab 0's first fragments
  set_vo();
#pragma unroll
  for (int i = 0; i < LOADS; ++i) issue_one(i);
  advance_ld();
#pragma unroll
  for (int i = 0; i < LOADS; ++i) issue_one(i);
  advance_ld();
  wait_vmcnt<LOADS>();
  __builtin_amdgcn_s_barrier();
#pragma unroll
  for (int f = 0; f < F; ++f) {
    fx[0][f] = frag(xo, f);
    fy[0][f] = frag(yo, f);
  }

  const int my_tiles = (ntiles - p + G - 1) / G;
  for (int t = 0; t < my_tiles; ++t) {
    set_vo();
    slab(std::true_type{});
    for (int kt = 1; kt < KT; ++kt) slab(std::false_type{});
    int64_t cm0;
    int cn0;
    tile_mn(p + t * G, cm0, cn0);
    tile_epilogue<EPI, F, F>(e, acc, M, cm0 + wm * 128, cn0 + wn * 128, frow, q);
  }
  // the last copies must land before the workgroup's LDS is released
  wait_vmcnt<0>();
}

// ------------------------------------------------------------------ bf16 MFMA kernel, one tile per workgroup
// The same slab schedule for every shape whose 256 x 256 tiles would leave CUs
// idle: X rows x Y rows of 32 XF x 32 YF (X the MFMA "A" operand: features, or
// tokens in the transposed-output form), four waves in a 2 x 2 grid of
// 16 XF x 16 YF, NS ring slots.  Slab g + NS is copied into slab g's slot after
// the slab's barrier, so NS - 1 slabs are in flight while one is multiplied.
// Copies past the last slab go through an empty buffer resource (they fetch
// nothing; the counts the waits rely on stay the same).
template <int XF, int YF, int NS, int EPI>
__global__ __launch_bounds__(256) void gemm_bf16_tile_kernel(const bf16_t* __restrict__ A, int64_t lda,
                                                             const bf16_t* __restrict__ W, int64_t M, int N, int K,
                                                             EpiArgs e, int GB) {
  if constexpr (EPI == TRACK_EPI_BIAS) {
    W += blockIdx.z * e.zw;
    e.bias = (const bf16_t*)e.bias + blockIdx.z * e.zw;
    e.out = (bf16_t*)e.out + blockIdx.z * e.zo;
  }
  constexpr bool VT = EPI == EPI_BIAS_VT;
  constexpr int BX = 32 * XF, BY = 32 * YF, BM = VT ? BX : BY, BN = VT ? BY : BX;
  constexpr int BK = 64, ROWB = 128, NWV = 4;
  constexpr int STAGE_BYTES = (BX + BY) * ROWB;
  constexpr int LOADS = XF + YF;  // per wave and slab
  constexpr int NM = XF * YF;     // MFMAs per 32-deep step
  __shared__ __attribute__((aligned(1024))) uint8_t smem[NS * STAGE_BYTES];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wx = wave & 1, wy = wave >> 1;
  // tile order: XCD-aware remap, then bands of GB M-tiles swept across N
  const int num_tm = (int)((M + BM - 1) / BM), num_tn = N / BN;
  const int p = xcd_remap(blockIdx.x, gridDim.x);
  const int band = p / (GB * num_tn);
  const int gsz = min(num_tm - band * GB, GB);
  const int in_band = p - band * GB * num_tn;
  const int64_t m0 = (int64_t)(band * GB + in_band % gsz) * BM;
  const int n0 = (in_band / gsz) * BN;

  const int lrow = lane >> 3;
  const int lcol = ((lane & 7) ^ lds_swz16(wave * 8 + lrow)) * 8;
  const int plain_row = wave * 8 + lrow;
  const int perm_row = 8 * (2 * (wave & 1) + (lrow >> 2)) + 4 * (wave >> 1) + (lrow & 3);
  // the host keeps BM * lda * 2 and BN * K * 2 below 2^31; rows past M lie
  // beyond the resource through their vector offset
  const int64_t arows = M - m0 < BM ? M - m0 : BM;
  const bf16_t *xp = VT ? A + m0 * lda : W + (int64_t)n0 * K, *yp = VT ? W + (int64_t)n0 * K : A + m0 * lda;
  const int64_t ldx = VT ? lda : K, ldy = VT ? K : lda;
  const int xbytes = (int)((VT ? arows * lda : (int64_t)BN * K) * 2), ybytes = (int)((VT ? (int64_t)BN * K : arows * lda) * 2);
  uint32_t vox[XF], voy[YF];
#pragma unroll
  for (int i = 0; i < XF; ++i) vox[i] = (uint32_t)(((i * 32 + perm_row) * ldx + lcol) * 2);
#pragma unroll
  for (int i = 0; i < YF; ++i) voy[i] = (uint32_t)(((i * 32 + plain_row) * ldy + lcol) * 2);
  const int KT = K / BK;
  int ld_kt = 0, ld_off = wave * 8 * ROWB;  // slab and LDS offset of the next copy
  __amdgpu_buffer_rsrc_t rx, ry;
  auto set_rsrc = [&]() {
    rx = __builtin_amdgcn_make_buffer_rsrc((void*)xp, (short)0, ld_kt < KT ? xbytes : 0, 0x00020000);
    ry = __builtin_amdgcn_make_buffer_rsrc((void*)yp, (short)0, ld_kt < KT ? ybytes : 0, 0x00020000);
  };
  // (plain types only: the builtin is not accepted with type-dependent arguments)
  uint8_t* const ring = smem;
  auto copy16 = [&](__amdgpu_buffer_rsrc_t r, int dst, uint32_t voff) {
    __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_ptr_t)(ring + dst), 16, voff, ld_kt * 128, 0, 0);
  };
  auto issue_one = [&](int i) {
    if (i < XF) copy16(rx, ld_off + i * 32 * ROWB, vox[i < XF ? i : 0]);
    else copy16(ry, ld_off + i * 32 * ROWB, voy[i < XF ? 0 : i - XF]);
  };
  auto advance_ld = [&]() {
    ++ld_kt;
    ld_off += STAGE_BYTES;
    if (ld_off >= NS * STAGE_BYTES) ld_off -= NS * STAGE_BYTES;
    set_rsrc();
  };

  const int frow = lane & 15, q = lane >> 4;
  const uint32_t foff = (uint32_t)(frow * ROWB + ((q ^ lds_swz16(frow)) << 4));
  const uint32_t xo = (uint32_t)(wx * 16 * XF * ROWB) + foff, yo = (uint32_t)((BX + wy * 16 * YF) * ROWB) + foff;
  uint32_t rd = 0;  // ring offset of the slab being read
  auto frag = [&](uint32_t o, int f) { return __builtin_bit_cast(bf16x8, *(const u32x4*)(smem + o + f * 16 * ROWB)); };

  f32x4 acc[XF][YF];
#pragma unroll
  for (int x = 0; x < XF; ++x)
#pragma unroll
    for (int y = 0; y < YF; ++y) acc[x][y] = f32x4{0, 0, 0, 0};
  bf16x8 fx[2][XF], fy[2][YF];
  // fragment reads r0 .. r1 (y first) of a step into buffer b
  auto reads = [&](int b, uint32_t nx, uint32_t ny, int r0, int r1) {
#pragma unroll
    for (int r = r0; r < r1; ++r) {
      if (r < YF) fy[b][r < YF ? r : 0] = frag(ny, r);
      else fx[b][r < YF ? 0 : r - YF] = frag(nx, r - YF);
    }
  };
  // MFMAs j0 .. j1 of step kk, with reads (from r0 on) or copies (from c0 on) spread over them
  auto mfmas = [&](int kk, int j0, int j1, int r0, uint32_t nx, uint32_t ny, int c0, int c1) {
#pragma unroll
    for (int j = j0; j < j1; ++j) {
      const int a = j - j0, n = j1 - j0;
      if (r0 >= 0) reads(kk ^ 1, nx, ny, r0 + a * (LOADS - r0) / n, r0 + (a + 1) * (LOADS - r0) / n);
      acc[j / YF][j % YF] =
          __builtin_amdgcn_mfma_f32_16x16x32_bf16(fx[kk][j / YF], fy[kk][j % YF], acc[j / YF][j % YF], 0, 0, 0);
#pragma unroll
      for (int c = c0 + a * (c1 - c0) / n; c < c0 + (a + 1) * (c1 - c0) / n; ++c) issue_one(c);
      __builtin_amdgcn_sched_barrier(0);
    }
  };

#pragma unroll
  for (int s = 0; s < NS; ++s) {
    set_rsrc();
#pragma unroll
    for (int i = 0; i < LOADS; ++i) issue_one(i);
    advance_ld();
  }
  wait_vmcnt<(NS - 1) * LOADS>();
  __builtin_amdgcn_s_barrier();
  reads(0, xo, yo, 0, LOADS);
  constexpr int HALF = NM / 2;  // the barrier's place: step 0's second half covers the wait of a partner
  for (int kt = 0; kt < KT; ++kt) {
    // every fragment of the slab's second step read by the middle of its first
    mfmas(0, 0, HALF, 0, rd + (xo ^ 64), rd + (yo ^ 64), 0, 0);
    // slab kt + 1 has landed for this wave and the wave holds all of slab kt's
    // fragments; after the barrier both hold for every wave
    wait_vmcnt<(NS - 2) * LOADS>();
    wait_lgkm0();
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    mfmas(0, HALF, NM, -1, 0, 0, 0, LOADS / 3);  // slab kt + NS into slab kt's slot
    rd += STAGE_BYTES;
    if (rd >= NS * STAGE_BYTES) rd -= NS * STAGE_BYTES;
    mfmas(1, 0, NM, 0, rd + xo, rd + yo, LOADS / 3, LOADS);
    advance_ld();
  }
  wait_vmcnt<0>();  // the last copies must land before the workgroup's LDS is released
  tile_epilogue<EPI, XF, YF>(e, acc, M, m0 + (VT ? wx * 16 * XF : wy * 16 * YF),
                             n0 + (VT ? wy * 16 * YF : wx * 16 * XF), frow, q);
}

// ------------------------------------------------------------------ float32 kernel
// Plain LDS-tiled FMA GEMM (64 x 64 tile, K-slab 16, 4 x 4 outputs per
// thread) for the float32 parity path; any M, N, K.
template <int EPI>
__global__ __launch_bounds__(256) void gemm_f32_kernel(const float* __restrict__ A, int64_t lda,
                                                       const float* __restrict__ W, int64_t M, int N, int K,
                                                       EpiArgs e) {
  __shared__ float As[16][65];
  __shared__ float Ws[16][65];
  const int tid = threadIdx.x;
  const int tx = tid & 15, ty = tid >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 64;
  const int n0 = blockIdx.x * 64;
  float acc[4][4] = {};
  for (int k0 = 0; k0 < K; k0 += 16) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int idx = tid + 256 * i;  // 0..1023 over a 64 x 16 tile
      const int row = idx >> 4, kk = idx & 15;
      const int64_t gm = m0 + row;
      const int gn = n0 + row;
      const int gk = k0 + kk;
      As[kk][row] = (gm < M && gk < K) ? A[gm * lda + gk] : 0.0f;
      Ws[kk][row] = (gn < N && gk < K) ? W[(int64_t)gn * K + gk] : 0.0f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < 16; ++kk) {
      float a[4], w[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        a[i] = As[kk][ty * 4 + i];
        w[i] = Ws[kk][tx * 4 + i];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) acc[i][j] = fmaf(a[i], w[j], acc[i][j]);
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int64_t m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n < N) epi_store1<EPI, float>(e, m, n, acc[i][j]);
    }
  }
}

// K-sharing float32 GEMM on v_mfma_f32_16x16x4_f32 (float32 products and sums): a
// workgroup owns 16 T x 16 T outputs and its four waves share K, every fourth
// 16-deep chunk each, joined through LDS.  The small float32 models' products (128
// rows, K 128 - 512) are a latency chain: here one global load and K / 64 short
// steps, where the LDS tiles above took a load, two barriers and a store per 16 of
// K on a handful of CUs.  K-index i of chunk kc is k = 16 kc + 4 (lane / 16) + i, so
// every lane loads 16 bytes.  Needs K % 4 == 0 and 16-byte aligned rows.
//
// With LN the rows of A are LayerNorm inputs: a wave's share of its rows (K up to
// SF_LN_K) stays in registers, the rows' means and centred square sums are joined over
// the lanes and (LDS) the waves, and the normalised, modulated values go straight into the
// products, in place of a launch that writes them and another that reads them.
constexpr int SF_LN_CH = 8, SF_LN_K = 4 * 16 * SF_LN_CH;

// Sums over a row's four 16-lane groups and the four waves, for T rows a lane.
template <int T>
__device__ __forceinline__ void small_row_sums(float (&v)[T], float (*red)[16 * T], int wave, int j, int g) {
#pragma unroll
  for (int t = 0; t < T; ++t) {
    v[t] += __shfl_xor(v[t], 16);
    v[t] += __shfl_xor(v[t], 32);
    if (g == 0) red[wave][16 * t + j] = v[t];
  }
  __syncthreads();
#pragma unroll
  for (int t = 0; t < T; ++t)
    v[t] = (red[0][16 * t + j] + red[1][16 * t + j]) + (red[2][16 * t + j] + red[3][16 * t + j]);
}

template <int EPI, int T, bool LN>
__global__ __launch_bounds__(256) void gemm_f32_small_kernel(const float* __restrict__ A, int64_t lda,
                                                             const float* __restrict__ W, int64_t M, int N, int K,
                                                             EpiArgs e, const float* __restrict__ ln_scale,
                                                             const float* __restrict__ ln_shift) {
  if constexpr (EPI == TRACK_EPI_BIAS) {
    W += blockIdx.z * e.zw;
    e.bias = (const float*)e.bias + blockIdx.z * e.zw;
    e.out = (float*)e.out + blockIdx.z * e.zo;
  }
  __shared__ f32x4 red[4][T * T][64];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int j = lane & 15, g = lane >> 4;
  const int64_t m0 = (int64_t)blockIdx.y * 16 * T;
  const int n0 = blockIdx.x * 16 * T;
  const float *ap[T], *wp[T];
#pragma unroll
  for (int t = 0; t < T; ++t) {
    const int64_t m = m0 + 16 * t + j;
    const int n = n0 + 16 * t + j;
    ap[t] = A + (m < M ? m : M - 1) * lda + 4 * g;
    wp[t] = W + (int64_t)(n < N ? n : N - 1) * K + 4 * g;
  }
  // thread -> token threadIdx / 16, feature threadIdx % 16 of each 16 x 16 block in
  // the epilogue; what it adds there is fetched with the operands
  const int tm = threadIdx.x >> 4, tn = threadIdx.x & 15;
  float pre_bias[T], pre_gate[T], pre_out[T][T];
#pragma unroll
  for (int x = 0; x < T; ++x) {
    const int n = min(n0 + 16 * x + tn, N - 1);
    pre_bias[x] = ((const float*)e.bias)[n];
    pre_gate[x] = EPI == TRACK_EPI_GATE_RESID ? e.gate[n] : 1.0f;
#pragma unroll
    for (int y = 0; y < T; ++y) {
      const int64_t m = m0 + 16 * y + tm;
      pre_out[x][y] = EPI == TRACK_EPI_GATE_RESID || EPI == TRACK_EPI_RESID
                          ? ((const float*)e.out)[(m < M ? m : M - 1) * e.ldo + n]
                          : 0.0f;
    }
  }
  f32x4 acc[T][T];  // features 4 g + r of block x, token j of block y
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y) acc[x][y] = f32x4{0.0f, 0.0f, 0.0f, 0.0f};
  const int chunks = (K + 15) / 16;
  const f32x4 zero = {0.0f, 0.0f, 0.0f, 0.0f};
  if constexpr (LN) {
    __shared__ float rs[2][4][16 * T];
    f32x4 a[SF_LN_CH][T], w[SF_LN_CH][T], sc[SF_LN_CH], sh[SF_LN_CH];
    float sum[T], sq[T];
#pragma unroll
    for (int t = 0; t < T; ++t) sum[t] = sq[t] = 0.0f;
#pragma unroll
    for (int u = 0; u < SF_LN_CH; ++u) {
      const int k0 = 16 * (wave + 4 * u);
#pragma unroll
      for (int t = 0; t < T; ++t) a[u][t] = k0 + 4 * g < K ? *(const f32x4*)(ap[t] + k0) : zero;
    }
    // (the other operands too, so that nothing is waited for after the sums)
#pragma unroll
    for (int u = 0; u < SF_LN_CH; ++u) {
      const int k0 = 16 * (wave + 4 * u);
      const bool in = k0 + 4 * g < K;
#pragma unroll
      for (int t = 0; t < T; ++t) w[u][t] = in ? *(const f32x4*)(wp[t] + k0) : zero;
      sc[u] = ln_scale && in ? *(const f32x4*)(ln_scale + k0 + 4 * g) : zero;
      sh[u] = ln_scale && in ? *(const f32x4*)(ln_shift + k0 + 4 * g) : zero;
    }
#pragma unroll
    for (int u = 0; u < SF_LN_CH; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) sum[t] += (a[u][t][0] + a[u][t][1]) + (a[u][t][2] + a[u][t][3]);
    small_row_sums<T>(sum, rs[0], wave, j, g);
#pragma unroll
    for (int u = 0; u < SF_LN_CH; ++u)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if (16 * (wave + 4 * u) + 4 * g >= K) continue;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          a[u][t][i] -= sum[t] / (float)K;
          sq[t] = fmaf(a[u][t][i], a[u][t][i], sq[t]);
        }
      }
    small_row_sums<T>(sq, rs[1], wave, j, g);
#pragma unroll
    for (int t = 0; t < T; ++t) sq[t] = 1.0f / sqrtf(sq[t] / (float)K + 1e-6f);
#pragma unroll
    for (int u = 0; u < SF_LN_CH; ++u) {
      const int k0 = 16 * (wave + 4 * u);
      if (k0 >= K) break;  // wave-uniform
#pragma unroll
      for (int i = 0; i < 4; ++i) {
        float v[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          v[t] = a[u][t][i] * sq[t];
          if (ln_scale) v[t] = fmaf(v[t], 1.0f + sc[u][i], sh[u][i]);
        }
#pragma unroll
        for (int x = 0; x < T; ++x)
#pragma unroll
          for (int y = 0; y < T; ++y)
            acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][x][i], v[y], acc[x][y], 0, 0, 0);
      }
    }
  } else {
    constexpr int U = 4 / T;  // chunks whose loads are issued together
    for (int kc = wave; kc < chunks; kc += 4 * U) {
      f32x4 a[U][T], w[U][T];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const int k0 = 16 * (kc + 4 * u);
        const bool in = k0 + 4 * g < K;
#pragma unroll
        for (int t = 0; t < T; ++t) {
          a[u][t] = in ? *(const f32x4*)(ap[t] + k0) : zero;
          w[u][t] = in ? *(const f32x4*)(wp[t] + k0) : zero;
        }
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
#pragma unroll
        for (int i = 0; i < 4; ++i)
#pragma unroll
          for (int x = 0; x < T; ++x)
#pragma unroll
            for (int y = 0; y < T; ++y)
              acc[x][y] = __builtin_amdgcn_mfma_f32_16x16x4f32(w[u][x][i], a[u][y][i], acc[x][y], 0, 0, 0);
    }
  }
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y) red[wave][x * T + y][lane] = acc[x][y];
  __syncthreads();
  const int src = (tn >> 2) * 16 + tm, r = tn & 3;
#pragma unroll
  for (int x = 0; x < T; ++x)
#pragma unroll
    for (int y = 0; y < T; ++y) {
      const int64_t m = m0 + 16 * y + tm;
      const int n = n0 + 16 * x + tn;
      if (m >= M || n >= N) continue;
      float v = (red[0][x * T + y][src][r] + red[1][x * T + y][src][r]) +
                (red[2][x * T + y][src][r] + red[3][x * T + y][src][r]) + pre_bias[x];
      if constexpr (EPI == TRACK_EPI_BIAS_GELU) v = gelu_tanh(v);
      if constexpr (EPI == TRACK_EPI_GATE_RESID) v = fmaf(pre_gate[x], v, pre_out[x][y]);
      if constexpr (EPI == TRACK_EPI_RESID) v += pre_out[x][y];
      ((float*)e.out)[m * e.ldo + n] = v;
    }
}

// ------------------------------------------------------------------ launchers
// The register-staged kernel, for leading dimensions whose tiles a buffer
// resource cannot address (BUF_LD and up).
constexpr int64_t BUF_LD = (int64_t)1 << 22;

static void launch_bf16_big_ld(int epi, const bf16_t* A, int64_t lda, const bf16_t* W, int64_t M, int N, int K,
                               const EpiArgs& e, hipStream_t s) {
  dim3 grid((unsigned)((M + 127) / 128) * (unsigned)(N / 64)), block(256);
  switch (epi) {
    case TRACK_EPI_BIAS: gemm_bf16_kernel<TRACK_EPI_BIAS><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); break;
    case TRACK_EPI_BIAS_GELU: gemm_bf16_kernel<TRACK_EPI_BIAS_GELU><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); break;
    case TRACK_EPI_GATE_RESID: gemm_bf16_kernel<TRACK_EPI_GATE_RESID><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); break;
    case TRACK_EPI_RESID: gemm_bf16_kernel<TRACK_EPI_RESID><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); break;
    default: gemm_bf16_kernel<TRACK_EPI_BIAS_F32><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); break;
  }
}

// Compute units of the current device (the persistent grid size).
int device_cus() {
  static int cus[64] = {0};
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 256;
  if (!cus[dev]) {
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || n <= 0) n = 256;
    cus[dev] = n;
  }
  return cus[dev];
}

// The tile kernels (X rows, Y rows in units of 32, ring slots, workgroups a CU
// holds by their LDS); entry 0 is the persistent 256 x 256 kernel.  Ties go to
// the earlier entry, so the deeper ring of two equal tiles comes first.
struct TileCfg {
  int xf, yf, slots, resident;
  bool vt;  // compiled with the transposed output (X the tokens there, Y the features)
};
static const TileCfg kTiles[] = {{8, 8, 2, 1, true},  {8, 4, 3, 1, false}, {4, 8, 3, 1, true},  {4, 5, 4, 1, false},
                                 {4, 5, 2, 2, false}, {4, 4, 4, 1, true},  {4, 3, 4, 1, false}, {4, 2, 3, 2, false},
                                 {2, 4, 3, 2, true},  {2, 2, 4, 2, true},  {2, 1, 4, 3, false}};
constexpr int NTILES = sizeof(kTiles) / sizeof(kTiles[0]);

// Kernel override for tests (TRACK_GEMM_CFG, read at every call): 4 the
// persistent kernel, 10 + i entry i of kTiles, for every shape it supports;
// anything else, and shapes the forced kernel does not take, automatic.
static int gemm_config() {
  const char* v = getenv("TRACK_GEMM_CFG");
  const int c = v ? atoi(v) : 0;
  return c == 4 ? 0 : (c >= 10 && c < 10 + NTILES ? c - 10 : -1);
}

// The tile for a shape, by an estimate of its time.  A slab of a BM x BN tile
// takes at least BM BN / 64 + 70 ns on a CU (its MFMAs at 2 GHz, and the
// barrier, fragment and copy latency of one workgroup), and (BM + BN) 1.47 ns of
// the CU's share of the L2 (16 TB/s over the chip); workgroups that share a CU
// overlap the first but add up in the second.  Tiles run in rounds of what the
// 256 CUs hold; the last round holds what is left.  Fitted over 75 shapes (M
// 130 - 9000, N 64 - 13824, K 64 - 13824), every tile timed at each: the pick is
// within 1% of the fastest tile on average and 13% at worst, where the largest tile
// for all that fill half the chip, and 128 x 128 for the rest, were 1.1 to 4.5 times
// slower (1.3B, 3120 rows: FFN2 154.7 -> 76.3 us, O 35.8 -> 22.8, q/k 51.3 ->
// 29.7, FFN1 111 -> 79; text K/V of 1024 rows 22.9 -> 14.1; 14B, 130 rows: O 61 -> 19).
// A batch of nb products (not for the persistent kernel) counts all their tiles.
static int pick_tile(int64_t M, int64_t N, int64_t K, bool vt, int force, int64_t nb = 1) {
  const int cus = device_cus();
  int best = -1;
  double best_t = 0.0;
  for (int i = 0; i < NTILES; ++i) {
    const TileCfg& c = kTiles[i];
    if ((vt && !c.vt) || (nb > 1 && i == 0)) continue;
    const int64_t bm = 32 * (vt ? c.xf : c.yf), bn = 32 * (vt ? c.yf : c.xf);
    if (N % bn) continue;
    if (i == force) return i;
    const int64_t tiles = (M + bm - 1) / bm * (N / bn) * nb;
    const int64_t round = (int64_t)c.resident * cus, full = tiles / round, rem = tiles % round;
    const double l2 = 1.47 * (double)(bm + bn), one = (double)(bm * bn) / 64.0 + 70.0;
    double t = (double)full * std::max(c.resident * l2, one);
    if (rem) t += std::max((double)((rem + cus - 1) / cus) * l2, one);
    t = t * (double)(K / 64) + 500.0 * (double)(full + (rem != 0));
    if (best < 0 || t < best_t) {
      best = i;
      best_t = t;
    }
  }
  return best;
}

template <int XF, int YF, int NS, bool VT>
static void launch_tile(int epi, const bf16_t* A, int64_t lda, const bf16_t* W, int64_t M, int N, int K,
                        const EpiArgs& e, hipStream_t s, int nb) {
  const int bm = 32 * (epi == EPI_BIAS_VT ? XF : YF), bn = 32 * (epi == EPI_BIAS_VT ? YF : XF);
  dim3 grid((unsigned)((M + bm - 1) / bm) * (unsigned)(N / bn), 1, (unsigned)nb), block(256);
  constexpr int GB = 8;  // height of the bands of M-tiles swept across N
#define TRACK_TK(E) gemm_bf16_tile_kernel<XF, YF, NS, E><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e, GB)
  if constexpr (VT) {
    if (epi == EPI_BIAS_VT) {
      TRACK_TK(EPI_BIAS_VT);
      return;
    }
  }
  switch (epi) {
    case TRACK_EPI_BIAS: TRACK_TK(TRACK_EPI_BIAS); break;
    case TRACK_EPI_BIAS_GELU: TRACK_TK(TRACK_EPI_BIAS_GELU); break;
    case TRACK_EPI_GATE_RESID: TRACK_TK(TRACK_EPI_GATE_RESID); break;
    case TRACK_EPI_RESID: TRACK_TK(TRACK_EPI_RESID); break;
    default: TRACK_TK(TRACK_EPI_BIAS_F32); break;
  }
#undef TRACK_TK
}

// The persistent kernel addresses A through a buffer resource whose size
// field is 32 bits; M is cut into row blocks of at most 2^31 - 1 bytes of A.
static void launch_bf16_persist(int epi, const bf16_t* A, int64_t lda, const bf16_t* W, int64_t M, int N, int K,
                                const EpiArgs& e, int out_elem, hipStream_t s) {
  const int64_t max_rows = ((((int64_t)1 << 31) - 1) / (lda * 2)) / 256 * 256;
  const int cus = device_cus();
  // Height of the bands of M-tiles swept across N (the order in which the
  // CUs take tiles, so what the L2 caches share): measured over the Wan
  // projection shapes, 4 suits long K (5120 and up), 16 wide N at short K,
  // 8 the rest; the order changes no result.
  const int gb = K >= 4096 ? 4 : (N >= 8192 ? 16 : 8);
  for (int64_t r0 = 0; r0 < M; r0 += max_rows) {
    const int64_t rows = M - r0 < max_rows ? M - r0 : max_rows;
    EpiArgs ec = e;
    ec.out = (uint8_t*)e.out + r0 * e.ldo * out_elem;
    ec.m_off = e.m_off + r0;
    const bf16_t* a = A + r0 * lda;
    const int ntiles = (int)((rows + 255) / 256) * (N / 256);
    dim3 grid(ntiles < cus ? ntiles : cus), block(256);
#define TRACK_PK(E) gemm_bf16_persist_kernel<E><<<grid, block, 0, s>>>(a, lda, W, rows, N, K, ec, ntiles, gb)
    switch (epi) {
      case TRACK_EPI_BIAS: TRACK_PK(TRACK_EPI_BIAS); break;
      case TRACK_EPI_BIAS_GELU: TRACK_PK(TRACK_EPI_BIAS_GELU); break;
      case TRACK_EPI_GATE_RESID: TRACK_PK(TRACK_EPI_GATE_RESID); break;
      case TRACK_EPI_RESID: TRACK_PK(TRACK_EPI_RESID); break;
      case EPI_BIAS_VT: TRACK_PK(EPI_BIAS_VT); break;
      default: TRACK_PK(TRACK_EPI_BIAS_F32); break;
    }
#undef TRACK_PK
  }
}

static void launch_bf16(int tile, int epi, const bf16_t* A, int64_t lda, const bf16_t* W, int64_t M, int N, int K,
                        const EpiArgs& e, int out_elem, hipStream_t s, int nb = 1) {
  switch (tile) {
    case 0: launch_bf16_persist(epi, A, lda, W, M, N, K, e, out_elem, s); break;
    case 1: launch_tile<8, 4, 3, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 2: launch_tile<4, 8, 3, true>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 3: launch_tile<4, 5, 4, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 4: launch_tile<4, 5, 2, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 5: launch_tile<4, 4, 4, true>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 6: launch_tile<4, 3, 4, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 7: launch_tile<4, 2, 3, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 8: launch_tile<2, 4, 3, true>(epi, A, lda, W, M, N, K, e, s, nb); break;
    case 9: launch_tile<2, 2, 4, true>(epi, A, lda, W, M, N, K, e, s, nb); break;
    default: launch_tile<2, 1, 4, false>(epi, A, lda, W, M, N, K, e, s, nb); break;
  }
}

// Blocks a side of the K-sharing kernel's workgroup: one until the 16 x 16 blocks fill
// the chip four times over, then two, which was the faster one at all of 15 shapes up to
// 2e12 FLOP (1000 x 1536 x 512 30 us against 74 of the LDS-tiled kernel, 3120 x 4608 x 1536
// 756 / 896, 8192 x 8192 x 2048 4515 / 5132, 200000 x 64 x 512 248 / 334, 65520 x 1536 x 8960
// 30.4 / 33.9 ms).  0: the LDS-tiled kernel, for rows that are not 16-byte aligned, or more
// of them than the grid's second dimension counts.
static int f32_small_blocks(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* W, int64_t nb) {
  const int64_t t16 = ((M + 15) / 16) * ((N + 15) / 16) * nb, cus = device_cus();
  if (K % 4 || lda % 4 || (((uintptr_t)A | (uintptr_t)W) & 15) || (M + 31) / 32 > 65535) return 0;
  return t16 > 4 * cus ? 2 : 1;
}

// ln: the rows of A are LayerNorm inputs (t 1, an epilogue without a residual)
static void launch_f32(int t, int epi, const float* A, int64_t lda, const float* W, int64_t M, int N, int K,
                       const EpiArgs& e, int nb, bool ln, const float* scale, const float* shift, hipStream_t s) {
  const int b = t ? 16 * t : 64;
  dim3 block(256), grid((unsigned)((N + b - 1) / b), (unsigned)((M + b - 1) / b), (unsigned)nb);
#define TRACK_F32_S(E, T, LN) gemm_f32_small_kernel<E, T, LN><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e, scale, shift)
#define TRACK_F32(E)                                                \
  do {                                                              \
    if (t == 1) TRACK_F32_S(E, 1, false);                           \
    else if (t == 2) TRACK_F32_S(E, 2, false);                      \
    else gemm_f32_kernel<E><<<grid, block, 0, s>>>(A, lda, W, M, N, K, e); \
  } while (0)
  if (ln) {
    if (epi == TRACK_EPI_BIAS) TRACK_F32_S(TRACK_EPI_BIAS, 1, true);
    else if (epi == TRACK_EPI_BIAS_GELU) TRACK_F32_S(TRACK_EPI_BIAS_GELU, 1, true);
    else TRACK_F32_S(TRACK_EPI_BIAS_F32, 1, true);
    return;
  }
  switch (epi) {
    case TRACK_EPI_BIAS: TRACK_F32(TRACK_EPI_BIAS); break;
    case TRACK_EPI_BIAS_GELU: TRACK_F32(TRACK_EPI_BIAS_GELU); break;
    case TRACK_EPI_GATE_RESID: TRACK_F32(TRACK_EPI_GATE_RESID); break;
    case TRACK_EPI_RESID: TRACK_F32(TRACK_EPI_RESID); break;
    default: TRACK_F32(TRACK_EPI_BIAS_F32); break;
  }
#undef TRACK_F32
#undef TRACK_F32_S
}

track_status linear(int dtype, int epi, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* W,
                    const void* bias, const float* gate, void* out, int64_t ldo, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0) return fail(TRACK_E_SHAPE, "linear: empty shape M=%lld N=%lld K=%lld", (long long)M, (long long)N, (long long)K);
  if (!A || !W || !bias || !out) return fail(TRACK_E_INVALID, "linear: null pointer");
  if (epi < 0 || epi > TRACK_EPI_BIAS_F32) return fail(TRACK_E_INVALID, "linear: bad epilogue %d", epi);
  if (epi == TRACK_EPI_GATE_RESID && !gate) return fail(TRACK_E_INVALID, "linear: gated residual needs gate");
  if (lda < K || ldo < N) return fail(TRACK_E_SHAPE, "linear: leading dimension too small");
  if (N > (1 << 30) || K > (1 << 30)) return fail(TRACK_E_SHAPE, "linear: N or K too large");
  EpiArgs e{bias, gate, out, ldo};
  ProfScope prof(TRACK_PROF_GEMM, s);
  if (dtype == TRACK_DTYPE_F32) {
    launch_f32(f32_small_blocks(M, N, K, A, lda, W, 1), epi, (const float*)A, lda, (const float*)W, M, (int)N, (int)K, e,
               1, false, nullptr, nullptr, s);
    TRACK_LAUNCH_CHECK();
    return TRACK_OK;
  }
  if (dtype != TRACK_DTYPE_BF16) return fail(TRACK_E_INVALID, "linear: bad dtype %d", dtype);
  if (K % 64 || N % 64) return fail(TRACK_E_UNSUPPORTED, "linear: bf16 path needs N, K multiples of 64 (N=%lld K=%lld)", (long long)N, (long long)K);
  if (lda % 8 || ldo % 4 || ((uintptr_t)A & 15) || ((uintptr_t)W & 15) || ((uintptr_t)out & 15) ||
      ((uintptr_t)bias & 7) || (gate && ((uintptr_t)gate & 15)))
    return fail(TRACK_E_INVALID, "linear: bf16 path needs 16-byte aligned rows");
  const bf16_t* a = (const bf16_t*)A;
  const bf16_t* w = (const bf16_t*)W;
  const int n = (int)N, k = (int)K;
  const int out_elem = (epi == TRACK_EPI_BIAS || epi == TRACK_EPI_BIAS_GELU) ? 2 : 4;
  if (lda >= BUF_LD || K >= BUF_LD)
    launch_bf16_big_ld(epi, a, lda, w, M, n, k, e, s);
  else
    launch_bf16(pick_tile(M, N, K, false, gemm_config()), epi, a, lda, w, M, n, k, e, out_elem, s);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

track_status linear_batch(int dtype, int nb, int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* W,
                          const void* bias, int64_t wstride, void* out, int64_t ldo, int64_t ostride, hipStream_t s) {
  const size_t es = dtype == TRACK_DTYPE_BF16 ? 2 : 4;
  const bool bf = dtype == TRACK_DTYPE_BF16;
  const int t = bf ? 0 : f32_small_blocks(M, N, K, A, lda, W, nb);
  // one launch on the kernels that take a batch, within their alignment needs
  const bool batch = nb > 1 && nb < 65536 && M > 0 && N > 0 && K > 0 && A && W && bias && out && lda >= K && ldo >= N &&
                     N <= (1 << 30) && K <= (1 << 30) &&
                     (bf ? K % 64 == 0 && N % 64 == 0 && lda % 8 == 0 && ldo % 4 == 0 && wstride % 8 == 0 &&
                               ostride % 8 == 0 && (((uintptr_t)A | (uintptr_t)W | (uintptr_t)out) & 15) == 0 &&
                               ((uintptr_t)bias & 7) == 0 && lda < BUF_LD && K < BUF_LD
                         : t > 0 && wstride % 4 == 0);
  if (!batch) {
    for (int i = 0; i < nb; ++i) {
      const track_status st =
          linear(dtype, TRACK_EPI_BIAS, M, N, K, A, lda, (const uint8_t*)W + i * wstride * es,
                 (const uint8_t*)bias + i * wstride * es, nullptr, (uint8_t*)out + i * ostride * es, ldo, s);
      if (st != TRACK_OK) return st;
    }
    return TRACK_OK;
  }
  EpiArgs e{bias, nullptr, out, ldo};
  e.zw = wstride;
  e.zo = ostride;
  ProfScope prof(TRACK_PROF_GEMM, s);
  if (bf)
    launch_bf16(pick_tile(M, N, K, false, -1, nb), TRACK_EPI_BIAS, (const bf16_t*)A, lda, (const bf16_t*)W, M, (int)N,
                (int)K, e, 2, s, nb);
  else
    launch_f32(t, TRACK_EPI_BIAS, (const float*)A, lda, (const float*)W, M, (int)N, (int)K, e, nb, false, nullptr,
               nullptr, s);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

track_status layernorm_linear(int dtype, int epi, int64_t M, int64_t N, int64_t K, const float* X, const float* scale,
                              const float* shift, void* Y, const void* W, const void* bias, const float* gate,
                              void* out, int64_t ldo, hipStream_t s) {
  // (only where one 16 x 16 block a workgroup covers the product: the rows' sums are formed
  // again for every 16 features.  8 blocks of a float32 model, LayerNorm inside all products
  // against in launches of its own: width 128, 64 tokens 330 / 421 us, 512 tokens 482 / 486;
  // width 512, 64 tokens 522 / 541, but 256 tokens (1536 - 2048 such blocks) 793 / 767 and
  // 1024 tokens 2391 / 2311)
  const bool takes = dtype == TRACK_DTYPE_F32 && K <= SF_LN_K && M > 0 && N > 0 && ldo >= N && N <= (1 << 30) && bias &&
                     out && (epi == TRACK_EPI_BIAS || epi == TRACK_EPI_BIAS_GELU || epi == TRACK_EPI_BIAS_F32) &&
                     (((uintptr_t)scale | (uintptr_t)shift) & 15) == 0;
  const int t = takes ? f32_small_blocks(M, N, K, X, K, W, 1) : 0;
  if (t != 1) {
    const track_status st = layernorm(dtype, M, (int)K, X, scale, shift, Y, s);
    if (st != TRACK_OK) return st;
    return linear(dtype, epi, M, N, K, Y, K, W, bias, gate, out, ldo, s);
  }
  ProfScope prof(TRACK_PROF_GEMM, s);
  launch_f32(1, epi, X, K, (const float*)W, M, (int)N, (int)K, EpiArgs{bias, gate, out, ldo}, 1, true, scale, shift, s);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

track_status linear_vt(int64_t M, int64_t N, int64_t K, const void* A, int64_t lda, const void* W, const void* bias,
                       int64_t L, void* vt, int64_t ldv, hipStream_t s) {
  if (M <= 0 || N <= 0 || K <= 0 || L <= 0) return fail(TRACK_E_SHAPE, "linear_vt: empty shape");
  if (!A || !W || !bias || !vt) return fail(TRACK_E_INVALID, "linear_vt: null pointer");
  if (lda < K || ldv < L) return fail(TRACK_E_SHAPE, "linear_vt: leading dimension too small");
  if (N % 256 || K % 64 || L % 8 || L < 128 || M % L || ldv % 8 || lda % 8 || lda >= ((int64_t)1 << 22) ||
      N > (1 << 30) || K > (1 << 30))
    return fail(TRACK_E_UNSUPPORTED, "linear_vt: needs N %% 256 == 0, K %% 64 == 0, L, ldv, lda %% 8 == 0, L >= 128, "
                "M %% L == 0 (N=%lld K=%lld L=%lld M=%lld)", (long long)N, (long long)K, (long long)L, (long long)M);
  if (((uintptr_t)A & 15) || ((uintptr_t)W & 15) || ((uintptr_t)vt & 15) || ((uintptr_t)bias & 7))
    return fail(TRACK_E_INVALID, "linear_vt: needs 16-byte aligned buffers");
  EpiArgs e{bias, nullptr, nullptr, 0};
  e.vt = vt;
  e.ldv = ldv;
  e.L = L;
  e.m_off = 0;
  e.nv = (int)N;
  ProfScope prof(TRACK_PROF_GEMM, s);
  launch_bf16(K < BUF_LD ? pick_tile(M, N, K, true, gemm_config()) : 0, EPI_BIAS_VT, (const bf16_t*)A, lda,
              (const bf16_t*)W, M, (int)N, (int)K, e, 2, s);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}


// ------------------------------------------------------------------ matrix-core stream
// The sustained matrix-core rate, the ceiling the MFMA-bound kernels are
// measured against besides the published peak: one 8-wave workgroup per CU; the
// two waves of a SIMD share the iterations (one wave alone loses 8% to the loop's
// branch), each iteration 16 independent v_mfma_f32_16x16x32_bf16 (the
// instruction of those kernels) on operands the wave loaded once (four A and four
// B fragments, caller data).  The chip's clock under matrix work depends on how
// many operand bits toggle, so the caller picks data like that of the kernel it
// compares.
constexpr int MFMA_STREAM_CHAINS = 16;
constexpr int64_t MFMA_STREAM_VECS = 4096;  // 16-byte operand vectors read

__global__ __launch_bounds__(512) void mfma_stream_kernel(const bf16x8* __restrict__ ops, float* __restrict__ sink,
                                                          int iters) {
  const int g = blockIdx.x * 512 + threadIdx.x;
  bf16x8 a[4], b[4];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    a[i] = ops[(g * 3 + i * 131) & (MFMA_STREAM_VECS - 1)];
    b[i] = ops[(g * 5 + i * 977 + 7) & (MFMA_STREAM_VECS - 1)];
  }
  f32x4 c[MFMA_STREAM_CHAINS];
#pragma unroll
  for (int j = 0; j < MFMA_STREAM_CHAINS; ++j) c[j] = f32x4{};
  const int mine = __builtin_amdgcn_readfirstlane(iters / 2 + (threadIdx.x < 256 ? iters % 2 : 0));
  for (int it = 0; it < mine; ++it) {
#pragma unroll
    for (int j = 0; j < MFMA_STREAM_CHAINS; ++j) {
      c[j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[j & 3], b[j >> 2], c[j], 0, 0, 0);
      __builtin_amdgcn_sched_barrier(0);  // in order, so that each chain stays in its registers
    }
  }
  float s = 0.f;
#pragma unroll
  for (int j = 0; j < MFMA_STREAM_CHAINS; ++j)
#pragma unroll
    for (int e = 0; e < 4; ++e) s += c[j][e];
  // reaches memory only for a value a caller would have to plant, so the
  // chains cannot be dropped
  if (s == 0x1.5p-99f) sink[0] = s;
}

track_status mfma_stream(const void* operands, int64_t iters, float* sink, int64_t* flop, hipStream_t s) {
  if (!operands || !sink || !flop) return fail(TRACK_E_INVALID, "mfma_stream: null pointer");
  if (iters <= 0 || iters > INT32_MAX) return fail(TRACK_E_SHAPE, "mfma_stream: iters must be in [1, 2^31)");
  if ((uintptr_t)operands & 15) return fail(TRACK_E_INVALID, "mfma_stream: 16-byte alignment needed");
  const int cus = device_cus();
  *flop = (int64_t)cus * 4 * iters * MFMA_STREAM_CHAINS * (2 * 16 * 16 * 32);
  ProfScope prof(TRACK_PROF_OTHER, s);
  mfma_stream_kernel<<<cus, 512, 0, s>>>((const bf16x8*)operands, sink, (int)iters);
  TRACK_LAUNCH_CHECK();
  return TRACK_OK;
}

}  // namespace track
