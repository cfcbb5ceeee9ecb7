// GEMMs of the quantized linears for 33 to a few thousand tokens (eq. 6 and eq. 1 of the paper):
//   acc[m, n] = sum_k q[m, k] * T[n, k],   Y[m, n] = (acc * d[m]) * alpha,
// from INT8 or INT4 codes x BL_W_GEMM weights (int32 on v_mfma_i32_32x32x32_i8) and from E3M2 codes x BL_W_MX2
// weights (exact integers in float32 on v_mfma_f32_32x32x64_f8f6f4).
//
// What bounds it.  Such a problem has too few 256 x 256 tiles for the chip (2048 tokens x 2048 outputs: 64 of 256
// CUs), so the tiles are smaller and a block is often alone on its CU, one or two waves per SIMD: nothing but the
// waves' own prefetch hides memory.  So every load is issued two steps of 256 channels before its use, and only the
// activations go through LDS: weights are 2-bit codes, which a lane fetches in fragment order (16 bytes serve 64
// channels of one output) and expands in registers between the MFMAs.  For a 128 x 128 tile LDS then takes 32 KB of writes
// and 64 KB of reads per step (about 800 cycles of 1024 of INT8 matrix work), where a tile that also expands the
// weights into LDS moves 64 + 128 KB.  Measured, product alone, weights from HBM (before: 256 x 256 and
// 128 x 128 tiles with one step of prefetch): INT8 200 x 3200 x 8640 44.3 -> 14.3 us, 1000 x 4096 x 11008 55.5 -> 40.7,
// 2048 x 2048 x 5460 55.5 -> 23.2, 2048 x 4096 x 11008 109 -> 74 (2.5 POPS); INT4 200 x 9600 x 3200 22.4 -> 13.1, gate/up of
// 130 x 2 x 8640 x 3200 25.7 -> 16.9.  64 tokens (before: the kernel that keeps the codes in LDS, and a second launch for the sums
// where K is split, which is still the better one for long K and few outputs: gr_long_k): INT8 64 x 4096 x 4096 12.5 -> 9.1,
// 64 x 12288 x 4096 17.8 -> 9.7, 64 x 2048 x 5460 12.2 -> 11.4; gate/up of 64 x 2 x 11008 x 4096 18.4 -> 14.2.
//
// Structure.  A group of 4 waves (2 x 2; block-float, mostly 1 x 4) owns a tile of 64 TM x 64 TN; a wave has TM x TN MFMA tiles (row operand =
// weights, column operand = tokens, so a lane ends up with groups of 4 consecutive outputs of one token).  One step =
// 256 channels = NSUB sub-steps of TM TN MFMAs.  Two LDS stages, two register sets per operand:
//   first sub-steps        write the activations of step s + 1 into the other stage, refill their registers (s + 3)
//   before the last one    barrier (the other stage is whole; every read of the own stage has been issued and waited for)
//   every sub-step         reads the token fragments and expands the weight fragments of the next sub-step
// The order of the channels inside a step is free as long as both operands agree: lane half lh takes the channels that
// its 16-byte weight piece covers.
// Where the tiles leave SIMDs short of waves, G groups of a block share out K and add their sums in LDS at the end
// (exact integers in either number format, so the order does not matter).
#include "common.h"

#define GM_THREADS 256                // of one K group

typedef int v2i __attribute__((ext_vector_type(2)));
typedef int v16i __attribute__((ext_vector_type(16)));
typedef float v16f __attribute__((ext_vector_type(16)));

enum { GM_I8 = 0, GM_I4 = 1, GM_MX = 2 };
enum { GM_ROWS = 0, GM_ANY = 1 };

// Tile of 64 TM tokens x 64 TN outputs, G groups of four waves that share out K.
template <int FMT, int TM, int TN, int G>
struct GmFmt {
  static constexpr bool mx = FMT == GM_MX;
  static_assert(!mx || TM <= 2, "block-float tiles are 64 tokens");
  static constexpr int wn = mx && TM == 2 ? 4 : 2;         // waves across the outputs; the rest across the tokens
  static constexpr int bm = 32 * (4 / wn) * TM, bn = 32 * wn * TN;
  static constexpr int nsub = mx ? 4 : 8;                  // MFMA sub-steps per step of 256 channels
  static constexpr int la = (FMT == GM_I8 ? 64 : FMT == GM_I4 ? 32 : 48) * bm / 1024;   // 16-byte activation loads per thread and step
  static constexpr int per_sub = FMT == GM_I8 ? TM : 1;    // of them written to LDS per sub-step
  static constexpr int stage = mx ? 2 * 6144 : bm * 256;
  static constexpr int shift = FMT == GM_I8 ? 6 : FMT == GM_I4 ? 10 : 0;   // the int8 expansion scales the sums by 2^shift
  static constexpr int tb_row = bn * 2 + 16;               // epilogue: one token's outputs in LDS, padded against conflicts
  static constexpr int sums = (G - 1) * bm * bn * 4;       // epilogue: accumulators of groups 1 ...
  static constexpr int max2(int a, int b) { return a > b ? a : b; }
  static constexpr int lds = max2(G * 2 * stage, max2(bm * tb_row, sums));
};

__device__ __forceinline__ __amdgpu_buffer_rsrc_t gm_rsrc(const unsigned char* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, 0x7FFFFFFF, 0x00027000);
}
__device__ __forceinline__ v4i gm_load16(__amdgpu_buffer_rsrc_t r, u32 voff, int soff) {
  return __builtin_bit_cast(v4i, __builtin_amdgcn_raw_buffer_load_b128(r, (int)voff, soff, 0));
}

__device__ __forceinline__ v4i gm_acc4(const v16i& c, int q) { return (v4i){c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]}; }
__device__ __forceinline__ v4i gm_acc4(const v16f& c, int q) {
  return __builtin_bit_cast(v4i, (v4f){c[4 * q], c[4 * q + 1], c[4 * q + 2], c[4 * q + 3]});
}
__device__ __forceinline__ void gm_acc4_add(v16i& c, int q, v4i v) {
#pragma unroll
  for (int r = 0; r < 4; ++r) c[4 * q + r] += v[r];
}
__device__ __forceinline__ void gm_acc4_add(v16f& c, int q, v4i v) {   // (whole numbers below 2^24: exact in any order)
#pragma unroll
  for (int r = 0; r < 4; ++r) c[4 * q + r] += __builtin_bit_cast(v4f, v)[r];
}

// OUT: GM_ROWS = bfloat16 rows through LDS; GM_ANY = either output type by elements, and the accumulators if asked
// for.  GLU (GM_I4 or GM_MX, GM_ROWS, TN = 2): a tile is 64 outputs of the gate and of the up matrix, column
// tile 0 of a wave is G and column tile 1 is U of the same 32 outputs; H = bf16(U * max(G, 0)^2).
template <int FMT, int OUT, bool GLU, int TM, int TN, int G>
__global__ __launch_bounds__(GM_THREADS * G, 2) void gemm_mid_kernel(
    const unsigned char* __restrict__ A, const float* __restrict__ scale, int M, int KT,
    const unsigned char* __restrict__ Wp, const unsigned char* __restrict__ Wp2, const float* __restrict__ alpha_p,
    const float* __restrict__ alpha2_p, int N, void* __restrict__ Y, int y_bf16, int32_t* __restrict__ acc_out,
    int MT, int NTB) {
  typedef GmFmt<FMT, TM, TN, G> F;
  constexpr bool MX = F::mx;
  constexpr int NSUB = F::nsub, LA = F::la, STAGE = F::stage;
  typedef typename std::conditional<MX, v16f, v16i>::type Acc;
  extern __shared__ __align__(16) unsigned char gm_smem[];
  const int tid = threadIdx.x & (GM_THREADS - 1), lane = tid & 63;   // (tid: within the K group)
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int group = G > 1 ? __builtin_amdgcn_readfirstlane(threadIdx.x >> 8) : 0;
  const int wm = F::wn == 4 ? 0 : wave >> 1, wn = F::wn == 4 ? wave : wave & 1;
  const int l32 = lane & 31, lh = lane >> 5;
  int m0, n0;
  bl_tile_origin((int)blockIdx.x, MT * NTB, MT, NTB, F::bm, F::bn, m0, n0);
  // this group's steps (a group without any multiplies zeros: every group takes part in the barriers)
  const int kt0 = min(group * KT / G, KT - 1);
  const int ns = (group + 1) * KT / G - group * KT / G, ns_block = (KT + G - 1) / G;
  const int s_max = max(ns, 1) - 1;
  unsigned char* const lds = gm_smem + group * 2 * STAGE;

  // ---- activation sources.  Row-major codes: piece i of a thread is row (tid / PR) + (256 / PR) i, 16-byte piece
  // tid % PR of the step's PR pieces per row; block form: a wave copies half of the 6 KB of a 32-token block in order.
  // Rows (blocks) past the end re-read the last one; their results are not stored.
  constexpr int PR = FMT == GM_I4 ? 8 : 16;
  constexpr int A_STEP = MX ? 6144 : PR * 16;              // bytes of one step along a row (block row)
  const int A_WAVE = (wave & 1) * 3072;                    // (block form: two waves share a block row, 3 KB each)
  const unsigned char* a_base;
  u32 a_off[MX ? 1 : LA];
  if constexpr (MX) {
    const int MB = (M + 31) >> 5;
    a_base = A + ((size_t)min((m0 >> 5) + (wave >> 1), MB - 1) * KT + kt0) * 6144;
    a_off[0] = A_WAVE + lane * 16;
  } else {
    const u32 row_bytes = (u32)KT * (PR * 16);
    a_base = A + (size_t)m0 * row_bytes + (size_t)kt0 * A_STEP;
#pragma unroll
    for (int i = 0; i < LA; ++i) a_off[i] = (u32)min(tid / PR + (GM_THREADS / PR) * i, M - 1 - m0) * row_bytes + (tid % PR) * 16;
  }
  // (buffer loads: one uniform descriptor and step offset plus a 32-bit lane offset, where flat loads made the
  // compiler keep a 64-bit address per load and spill; every offset is in range by the clamps, so no size is set)
  const __amdgpu_buffer_rsrc_t a_rsrc = gm_rsrc(a_base);
  v4i a_reg[2][LA];
  auto load_a = [&](int set, int i, int s) {
    const int so = min(s, s_max) * A_STEP;                // (past the last step: loads that nobody uses)
    if constexpr (MX) a_reg[set][i] = gm_load16(a_rsrc, a_off[0] + i * 1024, so);
    else a_reg[set][i] = gm_load16(a_rsrc, a_off[i], so);
  };
  // LDS: a row's 256 bytes cover all banks, its 16-byte chunk c sits at c ^ (row % 16); block form as it comes
  const int a_dst = MX ? (wave >> 1) * 6144 + A_WAVE + lane * 16
                       : (tid / PR) * 256 + (((FMT == GM_I4 ? 2 * (tid % PR) : tid % PR) ^ ((tid / PR) & 15)) << 4);
  auto store_a = [&](int st, int set, int i) {
    unsigned char* d = lds + st * STAGE + a_dst;
    const v4i v = a_reg[set][i];
    if constexpr (MX) {
      *reinterpret_cast<v4i*>(d + i * 1024) = v;
    } else if constexpr (FMT == GM_I8) {
      *reinterpret_cast<v4i*>(d + i * (16 * 256)) = v;
    } else {
      // rows of load i sit 32 i rows further down; nibbles to the top of their bytes (16 q)
      constexpr u32 MA = 0xF0F0F0F0u;
      unsigned char* d2 = lds + st * STAGE + (a_dst ^ 16);
      *reinterpret_cast<v4i*>(d + i * (32 * 256)) =
          (v4i){(int)(((u32)v[0] << 4) & MA), (int)((u32)v[0] & MA), (int)(((u32)v[1] << 4) & MA), (int)((u32)v[1] & MA)};
      *reinterpret_cast<v4i*>(d2 + i * (32 * 256)) =
          (v4i){(int)(((u32)v[2] << 4) & MA), (int)((u32)v[2] & MA), (int)(((u32)v[3] << 4) & MA), (int)((u32)v[3] & MA)};
    }
  };

  // ---- weight sources: piece h of column tile a is 16 bytes = 64 channels of output row 32 a + l32
  const unsigned char* w_base[TN];
  u32 w_off[TN];
  constexpr int W_STEP = MX ? 2048 : 1024;                 // bytes of one step along a block / tile row
  constexpr int W_HALF = MX ? 1024 : 512;                  // piece 1 against piece 0
  if constexpr (MX) {
    const int NB = (N + 31) >> 5;
#pragma unroll
    for (int a = 0; a < TN; ++a) {
      const int nb = GLU ? (n0 >> 6) + wn : (n0 >> 5) + TN * wn + a;
      w_base[a] = (GLU && a ? Wp2 : Wp) + ((size_t)min(nb, NB - 1) * KT + kt0) * W_STEP;
      w_off[a] = l32 * 32 + ((lh ^ ((l32 >> 4) & 1)) << 4);   // units 2 lh, 2 lh + 1 of the row (swapped for odd (l32 / 8))
    }
  } else {
    const int nt_max = ((N + 15) >> 4) - 1;
#pragma unroll
    for (int a = 0; a < TN; ++a) {
      const int nt = GLU ? (n0 >> 5) + 2 * wn : (n0 >> 4) + 2 * TN * wn + 2 * a;
      w_base[a] = (GLU && a ? Wp2 : Wp) + ((size_t)min(nt, nt_max) * KT + kt0) * W_STEP;
      w_off[a] = ((l32 >> 4) && nt < nt_max ? (u32)KT * 1024 : 0u) + (lh * 16 + (l32 & 15)) * 16;
    }
  }
  const __amdgpu_buffer_rsrc_t w_rsrc[2] = {gm_rsrc(w_base[0]), gm_rsrc(w_base[TN - 1])};
  v4i w_reg[2][TN][2];                                     // [set][column tile][piece]
  auto load_w = [&](int set, int a, int h, int s) {
    w_reg[set][a][h] = gm_load16(w_rsrc[a], w_off[a] + h * W_HALF, min(s, s_max) * W_STEP);
  };

  // ---- fragments
  typedef typename std::conditional<MX, v8i, v4i>::type Frag;
  Frag xf[2][TM], wf[2][TN];                                // [sub-step parity][tile]
  int x_off[NSUB];                                         // 16-byte part; compile-time index
  int xq_off[2];
  if constexpr (MX) {
#pragma unroll
    for (int j = 0; j < NSUB; ++j)
      x_off[j] = wm * 6144 + (j >> 1) * 3072 + l32 * 64 + (((2 * lh + (j & 1)) ^ ((l32 >> 2) & 3)) << 4);
#pragma unroll
    for (int e = 0; e < 2; ++e) xq_off[e] = wm * 6144 + 2048 + l32 * 32 + (((2 * lh + e) ^ ((l32 >> 3) & 3)) << 3);
  } else {
#pragma unroll
    for (int j = 0; j < NSUB; ++j)
      x_off[j] = (wm * 32 * TM + l32) * 256 + (((4 * (2 * (j >> 2) + lh) + (j & 3)) ^ (l32 & 15)) << 4);
  }
  auto read_x = [&](int st, int j, int b) -> Frag {
    if constexpr (MX) {
      const unsigned char* p = lds + st * STAGE + b * 6144;
      const v4i lo = *reinterpret_cast<const v4i*>(p + x_off[j]);
      const v2i hi = *reinterpret_cast<const v2i*>(p + xq_off[j & 1] + (j >> 1) * 3072);
      return (v8i){lo[0], lo[1], lo[2], lo[3], hi[0], hi[1], 0, 0};
    } else {
      return *reinterpret_cast<const v4i*>(lds + st * STAGE + b * (32 * 256) + x_off[j]);
    }
  };
  const bool w_swap = (l32 >> 3) & 1;
  auto expand_w = [&](int set, int j, int a, u32 mask) -> Frag {
    if constexpr (MX) {                                    // 2-bit codes -> E2M1 nibbles
      const v4i c = w_reg[set][a][j >> 1];
      const u32 w0 = (u32)((w_swap != (bool)(j & 1)) ? c[2] : c[0]), w1 = (u32)((w_swap != (bool)(j & 1)) ? c[3] : c[1]);
      return (v8i){(int)(w0 & mask), (int)((w0 << 1) & mask), (int)(w1 & mask), (int)((w1 << 1) & mask), 0, 0, 0, 0};
    } else {                                               // 2-bit codes to the top of their bytes (64 T)
      const u32 w = (u32)w_reg[set][a][j >> 2][j & 3];
      return (v4i){(int)((w << 6) & mask), (int)((w << 4) & mask), (int)((w << 2) & mask), (int)(w & mask)};
    }
  };
  constexpr u32 W_MASK = MX ? 0xAAAAAAAAu : 0xC0C0C0C0u;
  constexpr int W_SUBS = NSUB / 2;                         // sub-steps served by one weight piece

  Acc acc[TN][TM];
#pragma unroll
  for (int a = 0; a < TN; ++a)
#pragma unroll
    for (int b = 0; b < TM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[a][b][r] = 0;

  // the loads of step t's slots, in the order in which the loop issues them (the compiler derives the loop's wait
  // counts from the order of the loads in flight on every path into it): activations of step t + 3, weights of t + 2
  auto refill = [&](int set_a, int set_w, int t) {
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
#pragma unroll
      for (int e = 0; e < F::per_sub; ++e)
        if (j * F::per_sub + e < LA) load_a(set_a, j * F::per_sub + e, t + 3);
      if (j % W_SUBS == W_SUBS - 2) {
#pragma unroll
        for (int a = 0; a < TN; ++a) load_w(set_w, a, j / W_SUBS, t + 2);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // ---- prologue: step 0 in stage 0, activations of steps 1, 2 and weights of steps 0, 1 in registers
#pragma unroll
  for (int i = 0; i < LA; ++i) load_a(0, i, 0);
  __builtin_amdgcn_sched_barrier(0);
  refill(1, 0, -2);
#pragma unroll
  for (int i = 0; i < LA; ++i) store_a(0, 0, i);
  __builtin_amdgcn_sched_barrier(0);
  refill(0, 1, -1);
  __syncthreads();
#pragma unroll
  for (int b = 0; b < TM; ++b) xf[0][b] = read_x(0, 0, b);
  const u32 mask0 = ns > 0 ? W_MASK : 0u;
#pragma unroll
  for (int a = 0; a < TN; ++a) wf[0][a] = expand_w(0, 0, a, mask0);

  auto step = [&](auto par, int s) {
    constexpr int P = decltype(par)::value;
    const u32 mask = s < ns ? W_MASK : 0u, mask_next = s + 1 < ns ? W_MASK : 0u;
#pragma unroll
    for (int j = 0; j < NSUB; ++j) {
      constexpr int LAST = NSUB - 1;
      const int c = j & 1, d = c ^ 1;
      if (j == LAST) __syncthreads();
      __builtin_amdgcn_sched_barrier(0);
#pragma unroll
      for (int b = 0; b < TM; ++b) xf[d][b] = j < LAST ? read_x(P, j + 1, b) : read_x(P ^ 1, 0, b);
#pragma unroll
      for (int e = 0; e < F::per_sub; ++e) {
        const int i = j * F::per_sub + e;
        if (i < LA) {
          store_a(P ^ 1, P ^ 1, i);
          load_a(P ^ 1, i, s + 3);
        }
      }
#pragma unroll
      for (int a = 0; a < TN; ++a) wf[d][a] = j < LAST ? expand_w(P, j + 1, a, mask) : expand_w(P ^ 1, 0, a, mask_next);
      // piece h has been expanded for the last time one sub-step before its last use
      if (j % W_SUBS == W_SUBS - 2) {
#pragma unroll
        for (int a = 0; a < TN; ++a) load_w(P, a, j / W_SUBS, s + 2);
      }
#pragma unroll
      for (int a = 0; a < TN; ++a)
#pragma unroll
        for (int b = 0; b < TM; ++b) {
          if constexpr (MX)
            acc[a][b] = __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(wf[c][a], xf[c][b], acc[a][b], 4, 3, 0, 0, 0, 0);
          else
            acc[a][b] = __builtin_amdgcn_mfma_i32_32x32x32_i8(wf[c][a], xf[c][b], acc[a][b], 0, 0, 0);
        }
      // one MFMA, then what fits into its shadow
#pragma unroll
      for (int k = 0; k < TM * TN; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        __builtin_amdgcn_sched_group_barrier(0x100, TM * TN == 1 ? 2 : 1, 0);   // LDS read
        __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);   // LDS write
        __builtin_amdgcn_sched_group_barrier(0x002, TM * TN == 4 ? 4 : 8, 0);   // vector arithmetic
        __builtin_amdgcn_sched_group_barrier(0x020, 1, 0);   // global load
      }
      __builtin_amdgcn_sched_barrier(0);
    }
  };
  // Two steps per turn, one exit (a second one makes the compiler copy accumulators); an odd last step is followed by
  // one on its own data again whose weights are masked to zero.
  for (int s = 0; s < ns_block; s += 2) {
    step(std::integral_constant<int, 0>{}, s);
    step(std::integral_constant<int, 1>{}, s + 1);
  }

  // ---- epilogue.  acc[a][b][r] is output n = 64 wn + 32 a + 8 (r / 4) + 4 lh + r % 4 (GLU: 32 wn + ...) of token
  // m = 64 wm + 32 b + l32 of the tile, times 2^shift in integer formats.
  auto value = [&](const Acc& c, int i) {
    if constexpr (MX) return c[i];
    else return (float)(c[i] >> F::shift);
  };
  if constexpr (G > 1) {                                   // sums of the other groups, added by group 0
    __syncthreads();
    v4i* const sp = reinterpret_cast<v4i*>(gm_smem) + tid;
    if (group > 0) {
#pragma unroll
      for (int i = 0; i < 4 * TN * TM; ++i)
        sp[((group - 1) * 4 * TN * TM + i) * GM_THREADS] = gm_acc4(acc[i / (4 * TM)][(i / 4) % TM], i % 4);
    }
    __syncthreads();
    if (group == 0) {
#pragma unroll
      for (int g = 0; g < G - 1; ++g)
#pragma unroll
        for (int i = 0; i < 4 * TN * TM; ++i) gm_acc4_add(acc[i / (4 * TM)][(i / 4) % TM], i % 4, sp[(g * 4 * TN * TM + i) * GM_THREADS]);
    }
  }
  const bool mine = G == 1 || group == 0;                  // (the other groups help to store rows)
  {
    const float alpha = alpha_p[0];
    float dsc[TM];
#pragma unroll
    for (int b = 0; b < TM; ++b) dsc[b] = scale[min(m0 + wm * 32 * TM + b * 32 + l32, M - 1)];
    if constexpr (OUT == GM_ROWS) {
      constexpr int TB = F::tb_row;
      constexpr int BNO = GLU ? F::bn / 2 : F::bn;                 // outputs per token of this tile
      const float alpha2 = GLU ? alpha2_p[0] : 0.0f;
      __syncthreads();                                     // the stages become the transpose space
#pragma unroll
      for (int b = 0; b < TM; ++b) {
        if (!mine) break;
        unsigned char* trow = gm_smem + (wm * 32 * TM + b * 32 + l32) * TB;
#pragma unroll
        for (int a = 0; a < (GLU ? 1 : TN); ++a)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            float fv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              const float g = (value(acc[a][b], 4 * q + r) * dsc[b]) * alpha;
              if constexpr (GLU) {
                const float u = (value(acc[TN - 1][b], 4 * q + r) * dsc[b]) * alpha2;
                const float rl = fmaxf(g, 0.0f);
                const float rr = rl * rl;
                fv[r] = u * rr;
              } else {
                fv[r] = g;
              }
            }
            uint2 p;
            p.x = bl_pack_bf16(fv[0], fv[1]);
            p.y = bl_pack_bf16(fv[2], fv[3]);
            *reinterpret_cast<uint2*>(trow + ((GLU ? 32 : 32 * TN) * wn + 32 * a + 8 * q + 4 * lh) * 2) = p;
          }
      }
      __syncthreads();
      constexpr int LPR = BNO / 8;                         // lanes per token row
      const int rr = threadIdx.x / LPR, cc = threadIdx.x % LPR;
      const int nb = (GLU ? n0 >> 1 : n0) + cc * 8, n_left = N - nb;
      uint16_t* yp = (uint16_t*)Y + (size_t)(m0 + rr) * N + nb;
#pragma unroll
      for (int i = 0; i < (F::bm * LPR + GM_THREADS * G - 1) / (GM_THREADS * G); ++i) {
        const int row = i * (GM_THREADS * G / LPR);
        if (rr + row >= F::bm) break;                        // (small tile, many groups: more threads than pieces)
        const v4i v = *reinterpret_cast<const v4i*>(gm_smem + (rr + row) * TB + cc * 16);
        if (m0 + rr + row < M && n_left > 0) {
          if (n_left >= 8) *reinterpret_cast<v4i_align2*>(yp + (size_t)row * N) = v;
          else bl_store_tail8(yp + (size_t)row * N, v, n_left);
        }
      }
    } else if (mine) {
#pragma unroll
      for (int b = 0; b < TM; ++b) {
        const int m = m0 + wm * 32 * TM + b * 32 + l32;
#pragma unroll
        for (int a = 0; a < TN; ++a)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            const int n = n0 + wn * 32 * TN + a * 32 + 8 * q + 4 * lh;
            const size_t o = (size_t)m * N + n;
            float fv[4];
            int iv[4];
#pragma unroll
            for (int r = 0; r < 4; ++r) {
              fv[r] = (value(acc[a][b], 4 * q + r) * dsc[b]) * alpha;
              iv[r] = MX ? (int)acc[a][b][4 * q + r] : (int)acc[a][b][4 * q + r] >> F::shift;
            }
            if (m >= M) continue;
            if ((N & 3) == 0) {
              if (n < N) {
                if (y_bf16) *reinterpret_cast<uint2*>((uint16_t*)Y + o) = make_uint2(bl_pack_bf16(fv[0], fv[1]), bl_pack_bf16(fv[2], fv[3]));
                else *reinterpret_cast<float4*>((float*)Y + o) = make_float4(fv[0], fv[1], fv[2], fv[3]);
                if (acc_out) *reinterpret_cast<int4*>(acc_out + o) = make_int4(iv[0], iv[1], iv[2], iv[3]);
              }
            } else {
#pragma unroll
              for (int r = 0; r < 4; ++r) {
                if (n + r < N) {
                  if (y_bf16) ((uint16_t*)Y)[o + r] = bl_f32_to_bf16_rne(fv[r]);
                  else ((float*)Y)[o + r] = fv[r];
                  if (acc_out) acc_out[o + r] = iv[r];
                }
              }
            }
          }
      }
    }
  }
}

template <int FMT, int OUT, bool GLU, int TM, int TN, int G>
static int gm_go(const void* q, const float* scale, int M, int KT, const void* Wp, const void* Wp2, const float* alpha,
                 const float* alpha2, int N, void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  typedef GmFmt<FMT, TM, TN, G> F;
  constexpr int BNO = GLU ? F::bn / 2 : F::bn;
  const int MT = (M + F::bm - 1) / F::bm, NTB = (N + BNO - 1) / BNO;
  if (!bl_grid_ok((int64_t)MT * NTB)) return BL_ESHAPE;
  BL_SET_MAX_LDS_ONCE((gemm_mid_kernel<FMT, OUT, GLU, TM, TN, G>), F::lds);
  gemm_mid_kernel<FMT, OUT, GLU, TM, TN, G><<<(unsigned)(MT * NTB), GM_THREADS * G, F::lds, s>>>(
      (const unsigned char*)q, scale, M, KT, (const unsigned char*)Wp, (const unsigned char*)Wp2, alpha, alpha2, N, Y,
      ydt == BL_BF16 ? 1 : 0, acc_out, MT, NTB);
  BL_HIP_CHECK_LAUNCH();
  return BL_OK;
}

// ---- dispatch rules.  Costs in turns of the chip (tiles over CUs, rounded up).  (The figures below are of repeated calls on one
// weight matrix; with weights from HBM few tokens take 1 to 2 us more on either side.)
static int64_t gm_turns(int64_t M, int64_t N, int bm, int bn, int64_t cus = bl_num_cus()) {
  const int64_t tiles = ((M + bm - 1) / bm) * ((N + bn - 1) / bn);
  return (tiles + cus - 1) / cus;
}

// Integer codes: a 256 x 256 tile takes 3.5 times as long as a 128 x 128 tile (2.84 against 0.81 us per 256 channels
// with every CU busy), so the large tiles are left where they need as many turns: 4096 x 4096 x 11008 122 us against
// 140, 8192 x 3200 x 8640 174 against 180; on the other side 2048 x 4096 x 11008 100 against 71.
bool bl_gemm_mid_ok(int64_t M, int64_t N) { return 7 * gm_turns(M, N, 256, 256) > 2 * gm_turns(M, N, 128, 128); }

// Block-float codes: 64 x 256 tiles against 256 x 256, in turns of the small ones; where these do not fill their last turn, blocks
// that share a CU finish sooner, which counts for 0.3 of it.  The lines lie where whole layers (qkv, o, gate and up, down in a row, about
// 400 sizes of 90 to 10500 tokens, 1024 to 4096 channels) say so as well: the kernel that is the faster one alone may slow down what runs
// after it, under the power limit.
// One matrix: a turn of the large tiles is 3.05 small ones, the first one 2.8 from 2048 channels on, less below (a small tile's start and
// end weigh more).  Product alone, large / small, us: 500 x 12288 x 4096 23.1 / 20.3, 1500 x 12288 x 4096 60.4 / 50.0, 1000 x 12288 x 4096
// 33.8 / 34.9, 2048 x 12288 x 4096 62.0 / 64.9, 2048 x 9600 x 3200 51.4 / 47.9, 4096 x 9600 x 3200 78.8 / 87.7, 1700 x 3072 x 1024 9.8 / 9.4,
// 3000 x 3072 x 1024 14.1 / 15.8; two layers: 6000 tokens, 1024 channels 268.8 / 259.1, 1600 tokens, 3200 channels 409.7 / 386.5, 900 tokens,
// 4096 channels 348.4 / 348.2, 1850 tokens, 4096 channels 566.7 / 573.2.
// Gate and up: 3.1 small turns, the first 2.65, at any length of rows (the large tiles end slowly).  Two layers, large / small, us:
// 1106 tokens, 2944 channels, 2 x 7832 outputs 284.7 / 266.4, 1250 tokens, 2944 channels 290.1 / 273.8, 2400 tokens, 2560 channels 400.7 / 380.9;
// 1000 tokens, 4096 channels 354.2 / 353.7, 2048 tokens, 4096 channels 574.9 / 608.3, 1600 tokens, 2944 channels 351.7 / 356.9.
bool bl_gemm_mid_mx_ok(int64_t M, int64_t N, int64_t K, bool glu) {
  const int64_t n_cols = glu ? 2 * N : N;                  // the outputs of both matrices
  const int64_t cus = bl_num_cus();
  const double share = (double)(((M + 63) / 64) * ((n_cols + 255) / 256)) / cus;
  const double KT = (double)(bl_round_up(K, BL_KPAD) >> 8);
  const double small = 0.7 * (double)gm_turns(M, n_cols, 64, 256, cus) + 0.3 * share, large = (double)gm_turns(M, n_cols, 256, 256, cus);
  if (glu) return small < 3.1 * large - 0.45;
  return small < (3.05 * large - 0.25) * (large == 1.0 && KT < 8.0 ? 0.6 + 0.05 * KT : 1.0);
}

#define GM_CALL(FMT, OUT, GLU, TM, TN, G) \
  gm_go<FMT, OUT, GLU, TM, TN, G>(q, scale, (int)M, KT, Wp, Wp2, alpha, alpha2, (int)N, Y, ydt, acc_out, s)

// Integer codes: 64 x 64 tiles and two K groups while these fill one turn (200 x 3200 x 8640: 12.8 us, 64 x 128 tiles 17.6,
// 128 x 128 25.9), then 64 x 128 while those do (400 x 3200 x 8640: 18.5, 128 x 128 26.8, 64 x 64 21.0), then 128 x 128
// (600 x 4096 x 4096: 15.6 against 16.4 and more; never for tokens that fill only half of it).
template <int FMT, int OUT>
static int gm_int(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha, int64_t N,
                  void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8);
  const void* Wp2 = nullptr;
  const float* alpha2 = nullptr;
  if (gm_turns(M, N, 64, 64) == 1) return GM_CALL(FMT, OUT, false, 1, 1, 2);
  if (M <= 64 || gm_turns(M, N, 64, 128) == 1) return GM_CALL(FMT, OUT, false, 1, 2, 2);
  return GM_CALL(FMT, OUT, false, 2, 2, 1);
}

// Block-float codes.  What bounds a step is the CU's vector loads (about 53 bytes per clock): with the four waves side by side
// (1 x 4, every wave with all 64 tokens) the weights are fetched once instead of by two waves, 20 KB a step for 64 x 128 instead of
// 28, and 28 KB for 64 x 256.  So 64 x 256 tiles wherever they save a turn or more (a turn of theirs is 1.4 times as long), else 64 x
// 128.  Product alone, weights from HBM, 2 x 2 waves / 64 x 128 / 64 x 256, us: 200 x 9600 x 3200 13.2 / 12.4 / 10.9, 300 x 12288 x 4096 17.2 / 16.7 /
// 14.2, 700 x 9600 x 3200 25.0 / 25.0 / 21.5.
// Where 64 x 128 tiles fill no more than one turn, the blocks are few and short: 2 x 2 waves start sooner than 1 x 4, and beyond 3584
// channels two K groups of them are faster still.  Quantizer and product, mean over 65 to 400 tokens, 2 x 2 / 1 x 4 / two groups: 4608 x 1536 9.3 /
// 9.4 / 10.5, 9600 x 3200 12.5 / 12.8 / 13.3, 11136 x 3712 13.2 / 13.5 / 13.6; with weights in the last-level cache 8.7 / 8.9 / 9.6, 12.1 / 12.7 /
// 12.2, 12.8 / 13.4 / 12.2.
// Where 64 x 256 tiles leave their third turn nearly empty and rows are up to 3072 channels, 64 x 128 are about level and don't slow
// down what follows: the product inside a layer and two layers, both under the profiler, 64 x 128 / 64 x 256: 1400 x 6144 x 2048 19.1 / 20.8 and 236 / 240, 927 x 8832 x 2944 24.3 / 24.1
// and 247 / 250; longer rows 751 x 12288 x 4096 31.6 / 28.6 and 348 / 341.
template <int OUT>
static int gm_mx(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha, int64_t N,
                 void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8);
  const void* Wp2 = nullptr;
  const float* alpha2 = nullptr;
  const int64_t cus = bl_num_cus(), t128 = gm_turns(M, N, 64, 128, cus), t256 = gm_turns(M, N, 64, 256, cus);
  if (t128 == 1) return KT >= 15 ? GM_CALL(GM_MX, OUT, false, 1, 2, 2) : GM_CALL(GM_MX, OUT, false, 1, 2, 1);
  if (7 * t256 <= 5 * t128 && !(t256 == 3 && t128 == 5 && KT <= 12)) return GM_CALL(GM_MX, OUT, false, 2, 2, 1);
  return GM_CALL(GM_MX, OUT, false, 2, 1, 1);
}

int bl_launch_gemm_mid(const void* q, const float* scale, bl_act_mode mode, int64_t M, int64_t K, const void* Wp,
                       const float* alpha, int64_t N, void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  const bool rows = ydt == BL_BF16 && !acc_out;
#define GM_INT(FMT, OUT) gm_int<FMT, OUT>(q, scale, M, K, Wp, alpha, N, Y, ydt, acc_out, s)
  if (mode == BL_ACT_INT4_ABSMEAN) return rows ? GM_INT(GM_I4, GM_ROWS) : GM_INT(GM_I4, GM_ANY);
  return rows ? GM_INT(GM_I8, GM_ROWS) : GM_INT(GM_I8, GM_ANY);
#undef GM_INT
}

int bl_launch_gemm_mid_mx(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha,
                          int64_t N, void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  if (ydt == BL_BF16 && !acc_out) return gm_mx<GM_ROWS>(q, scale, M, K, Wp, alpha, N, Y, ydt, acc_out, s);
  return gm_mx<GM_ANY>(q, scale, M, K, Wp, alpha, N, Y, ydt, acc_out, s);
}

int bl_launch_gemm_mid_mx_glu(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha,
                              const void* Wp2, const float* alpha2, int64_t N, void* Y, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8);
  const bl_dtype ydt = BL_BF16;
  int32_t* acc_out = nullptr;
  // 64 outputs of either matrix per block while those blocks fill one turn, else 128 (1 x 4 waves): 128 x 2 x 5460 x 2048 6.6 us /
  // 7.3; 200 x 2 x 5460 x 2048 9.1 / 7.6, 100 x 2 x 11008 x 4096 15.2 / 12.0, 700 x 2 x 11008 x 4096 51.5 / 40.3
  if (gm_turns(M, 2 * N, 64, 128) == 1) return GM_CALL(GM_MX, GM_ROWS, true, 1, 2, 1);
  return GM_CALL(GM_MX, GM_ROWS, true, 2, 2, 1);
}

// INT4 codes x two BL_W_GEMM matrices (33 to 64 tokens): 64 outputs of either per block, two K groups.
int bl_launch_gemm_mid_a4_glu(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha,
                              const void* Wp2, const float* alpha2, int64_t N, void* Y, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8);
  const bl_dtype ydt = BL_BF16;
  int32_t* acc_out = nullptr;
  return GM_CALL(GM_I4, GM_ROWS, true, 1, 2, 2);
}
