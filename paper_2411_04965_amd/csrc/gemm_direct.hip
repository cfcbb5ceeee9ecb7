// GEMMs of the quantized linears for a few dozen to a few hundred tokens, without LDS in the K loop (eq. 6 and eq. 1):
//   acc[m, n] = sum_k q[m, k] * T[n, k],   Y[m, n] = (acc * d[m]) * alpha,
// INT8 or INT4 codes x BL_W_GEMM weights on v_mfma_i32_16x16x64_i8.
//
// What bounds it.  A decode-sized product is a chain of latencies, not of bytes: a launch starts, its first loads come
// back, sums are added, rows are stored.  Kernels that keep the codes in LDS wait for all of them before the first
// product and, where K does not fit, split it over blocks and pay a second launch; tiles whose waves share K steps meet
// at a barrier per step.  Here a block owns 16 MT tokens x 16 NT outputs over the whole of K and its eight waves share out
// K in tiles of 256 channels.  A wave reads a tile of both operands straight into MFMA registers and requests the next one
// into the same registers once its products are issued; other waves and blocks of the CU fill its waits, and nothing waits for
// another wave until the one LDS reduction at the end (exact integers: any order).  (Two and four tiles in flight per wave were no
// faster: the blocks that share a CU then have fewer registers.)  A CU fetches every byte it needs once; how many those are
// decides the tile (gx_pick).
//
// Both operands come as whole 1 KB runs per load: the weights because BL_W_GEMM is in fragment order, the codes because the
// quantizer writes them that way for this kernel (a private order in the caller's workspace; from row-major codes a load
// touches 64 separate 16-byte pieces and the CU gets a quarter of the bytes per cycle: 32 x 4096 x 11008 17.6 us).
//   Codes in fragment order: token tile t (16 tokens, R = min(16, M - 16 t) of them there), channel tile kt (256 channels):
//   INT8 at t * 16 * Kp + kt * 256 R, four pieces of 64 R bytes; piece j, lane group g (0 .. 3), token i: the 16 bytes at
//   (g R + i) * 16 are channels 256 kt + 64 g + 16 j ...  INT4 at half of these offsets, two pieces of 64 R bytes; piece j:
//   the 32 nibbles (eight to a word as in the row-major form) of channels 256 kt + 64 g + 32 j ...
#include "common.h"

#define GX_WAVES 8
#define GX_THREADS (64 * GX_WAVES)


__device__ __forceinline__ __amdgpu_buffer_rsrc_t gx_rsrc(const unsigned char* base) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(base), 0, 0x7FFFFFFF, 0x00027000);
}

// GLU: the NT output tiles are NT / 2 of the gate matrix and the same NT / 2 of the up matrix;
// H = bf16(U * max(G, 0)^2) (eq. 5) is what is stored.
template <bool A4, bool GLU, int MT, int NT>
__global__ __launch_bounds__(GX_THREADS, 1) void gemm_direct_kernel(
    const unsigned char* __restrict__ A, const float* __restrict__ scale, int M, int KT,
    const unsigned char* __restrict__ Wp, const unsigned char* __restrict__ Wp2, const float* __restrict__ alpha_p,
    const float* __restrict__ alpha2_p, int N, void* __restrict__ Y, int y_bf16, int32_t* __restrict__ acc_out, int MG,
    int n_blocks) {
  constexpr int NTM = GLU ? NT / 2 : NT;                   // output tiles of one matrix
  constexpr int LX = A4 ? 2 : 4;                           // pieces (16-byte loads) per token tile and K tile
  constexpr int SHIFT = A4 ? 10 : 6;                       // weights carry 64 T, nibble codes 16 q
  extern __shared__ __align__(16) unsigned char gx_smem[];
  v4i* const red = reinterpret_cast<v4i*>(gx_smem);        // [entry][wave][lane]
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, lg = lane >> 4;
  // blocks go round robin to the 8 XCDs: token groups of one output group (its weights) to one XCD
  const int bq = n_blocks >> 3, brm = n_blocks & 7, xcd = (int)blockIdx.x & 7;
  const int pid = xcd * bq + min(xcd, brm) + ((int)blockIdx.x >> 3);
  const int mt0 = (pid % MG) * MT, nt0 = (pid / MG) * NTM;
  const int nt_max = ((N + 15) >> 4) - 1;

  // ---- sources.  Rows past the last token re-read it; output tiles past the end re-read the last one; their results are not
  // stored.  K tiles past the end are loads outside the descriptor: zeros, and no traffic.
  const int rows0 = M - mt0 * 16;                          // tokens from this block's first on
  u32 a_off[MT], a_step[MT];
#pragma unroll
  for (int b = 0; b < MT; ++b) {
    const int bb = min(b, (rows0 - 1) >> 4);               // (a token tile past the end re-reads the last one)
    const int r = min(16, rows0 - 16 * bb);
    a_off[b] = (u32)bb * 16 * KT * (A4 ? 128 : 256) + (u32)(lg * r + min(li, r - 1)) * 16;
    a_step[b] = 64 * r;                                    // bytes of one piece
  }
  const unsigned char* const a_base = A + (size_t)mt0 * 16 * KT * (A4 ? 128 : 256);
  const unsigned char* const w_base = Wp + (size_t)nt0 * KT * 1024;
  const unsigned char* const w2_base = (GLU ? Wp2 : Wp) + (size_t)nt0 * KT * 1024;
  int w_tile[NT];                                          // byte offset of the output tile
#pragma unroll
  for (int a = 0; a < NT; ++a) w_tile[a] = min(a % NTM, nt_max - nt0) * KT * 1024;

  v4i xr[MT][LX], wr[NT];
  const __amdgpu_buffer_rsrc_t ar = gx_rsrc(a_base), w1 = gx_rsrc(w_base), w2 = gx_rsrc(w2_base);
  auto load = [&](int kt) {
    const u32 past = kt < KT ? 0u : 0x80000000u;           // wave-uniform; past the end: outside the descriptor
    const int kc = min(kt, KT - 1);
#pragma unroll
    for (int a = 0; a < NT; ++a)
      wr[a] = __builtin_bit_cast(
          v4i, __builtin_amdgcn_raw_buffer_load_b128(GLU && a >= NTM ? w2 : w1, (int)(lane * 16 | past), w_tile[a] + kc * 1024, 0));
#pragma unroll
    for (int b = 0; b < MT; ++b)
#pragma unroll
      for (int e = 0; e < LX; ++e)
        xr[b][e] = __builtin_bit_cast(
            v4i, __builtin_amdgcn_raw_buffer_load_b128(ar, (int)(a_off[b] | past), (int)a_step[b] * (LX * kc + e), 0));
  };
  load(wave);

  v4i acc[NT][MT];
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) acc[a][b] = (v4i){0, 0, 0, 0};
  auto products = [&]() {
#pragma unroll
    for (int t = 0; t < 4; ++t) {
      v4i x[MT];
#pragma unroll
      for (int b = 0; b < MT; ++b) {
        if constexpr (A4) {                                // nibbles to the top of their bytes (16 q)
          const u32 w0 = (u32)xr[b][t >> 1][2 * (t & 1)], w1_ = (u32)xr[b][t >> 1][2 * (t & 1) + 1];
          x[b] = (v4i){(int)((w0 << 4) & 0xF0F0F0F0u), (int)(w0 & 0xF0F0F0F0u), (int)((w1_ << 4) & 0xF0F0F0F0u),
                       (int)(w1_ & 0xF0F0F0F0u)};
        } else {
          x[b] = xr[b][t];
        }
      }
#pragma unroll
      for (int a = 0; a < NT; ++a) {
        const u32 w = (u32)wr[a][t], mask = 0xC0C0C0C0u;
        const v4i wo = (v4i){(int)((w << 6) & mask), (int)((w << 4) & mask), (int)((w << 2) & mask), (int)(w & mask)};
#pragma unroll
        for (int b = 0; b < MT; ++b) acc[a][b] = __builtin_amdgcn_mfma_i32_16x16x64_i8(wo, x[b], acc[a][b], 0, 0, 0);
      }
    }
  };
  // one K tile per wave and round, the same number of rounds for every wave; the last one requests nothing any more
  // (loads that nobody needs cost their address cycles all the same: 32 x 12288 x 4096 INT4 6.2 us with them, 5.7 without)
  for (int k0 = 0; k0 + GX_WAVES < KT; k0 += GX_WAVES) {
    products();
    load(k0 + GX_WAVES + wave);
  }
  products();

  // ---- sums over the waves: entry (tile b of tokens, tile a of one matrix) is finished by wave (entry % 8)
#pragma unroll
  for (int a = 0; a < NT; ++a)
#pragma unroll
    for (int b = 0; b < MT; ++b) red[((b * NT + a) * GX_WAVES + wave) * 64 + lane] = acc[a][b];
  __syncthreads();
  auto entry_sum = [&](int e, int (&iv)[4]) {
    v4i s = (v4i){0, 0, 0, 0};
#pragma unroll
    for (int w = 0; w < GX_WAVES; ++w) s += red[(e * GX_WAVES + w) * 64 + lane];
#pragma unroll
    for (int r = 0; r < 4; ++r) iv[r] = s[r] >> SHIFT;
  };
  const float alpha = alpha_p[0], alpha2 = GLU ? alpha2_p[0] : 0.0f;
#pragma unroll
  for (int i = 0; i < (NTM * MT + GX_WAVES - 1) / GX_WAVES; ++i) {
    const int e = wave + GX_WAVES * i;
    if (e >= NTM * MT) break;
    const int b = e / NTM, a = e % NTM;
    const int m = (mt0 + b) * 16 + li, n = (nt0 + a) * 16 + 4 * lg;
    if (m >= M || n >= N) continue;
    const float d = scale[m];
    const size_t o = (size_t)m * N + n;
    int ig[4];
    float fg[4];
    entry_sum(b * NT + a, ig);
#pragma unroll
    for (int r = 0; r < 4; ++r) fg[r] = ((float)ig[r] * d) * alpha;
    if constexpr (GLU) {
      int iu[4];
      float h[4];
      entry_sum(b * NT + NTM + a, iu);
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const float u = ((float)iu[r] * d) * alpha2;
        const float rl = fmaxf(fg[r], 0.0f);
        const float rr = rl * rl;
        h[r] = u * rr;
      }
      bl_store_out4(Y, 1, nullptr, o, n, N, iu, h);
    } else {
      bl_store_out4(Y, y_bf16, acc_out, o, n, N, ig, fg);
    }
  }
}

template <bool A4, bool GLU, int MT, int NT>
static int gx_go(const void* q, const float* scale, int M, int KT, const void* Wp, const void* Wp2, const float* alpha,
                 const float* alpha2, int N, void* Y, int ybf, int32_t* acc_out, hipStream_t s) {
  constexpr int NTM = GLU ? NT / 2 : NT;
  constexpr size_t smem = (size_t)MT * NT * GX_WAVES * 1024;
  static_assert(smem <= 160 * 1024, "the reduction fits the LDS");
  const int64_t MG = (M + 16 * MT - 1) / (16 * MT), NG = ((N + 15) / 16 + NTM - 1) / NTM;
  if (!bl_grid_ok(MG * NG)) return BL_ESHAPE;
  BL_SET_MAX_LDS_ONCE((gemm_direct_kernel<A4, GLU, MT, NT>), smem);
  gemm_direct_kernel<A4, GLU, MT, NT><<<(unsigned)(MG * NG), GX_THREADS, smem, s>>>(
      (const unsigned char*)q, scale, M, KT, (const unsigned char*)Wp, (const unsigned char*)Wp2, alpha, alpha2, N, Y, ybf,
      acc_out, (int)MG, (int)(MG * NG));
  BL_HIP_CHECK_LAUNCH();
  return BL_OK;
}

// ---- tile choice.  What a block costs goes with the 1 KB loads of its K loop (INT8 codes: four per token tile and K tile, INT4
// two; one per output tile) plus the sums of its accumulator tiles, worth 6 loads each.  Blocks beyond one per CU come in turns;
// where their sums leave LDS for two blocks on a CU (up to 10 accumulator tiles), a turn costs less and a part of one counts as such.
// Against the best of all tiles at 96 sizes (4 to 320 tokens, 1024 to 12288 outputs, 1024 to 11008 channels, weights from HBM) the
// choice is within 8 % everywhere.  Products alone, before (resident codes and split K, or 64 x 64 tiles with a barrier per step) -> here, us:
//   INT8   32 x 4096 x 4096 7.9 -> 4.2, 32 x 4096 x 11008 13.1 -> 7.1, 57 x 2048 x 5460 9.5 -> 4.7, 64 x 4096 x 11008 16.7 -> 8.8,
//          200 x 3200 x 8640 14.3 -> 11.2, 256 x 4096 x 4096 9.4 -> 7.8
//   INT4   32 x 12288 x 4096 8.9 -> 5.6, 64 x 12288 x 4096 9.5 -> 7.4; gate and up 32 x 2 x 11008 x 4096 12.8 -> 8.0,
//          64 x 2 x 5460 x 2048 8.0 -> 5.2
struct GxTile { int mt, nt; };

template <int COUNT>
static int gx_pick(const GxTile (&tiles)[COUNT], int64_t M, int64_t N, int KT, int code_loads, bool glu) {
  const int cus = bl_num_cus(), m16 = (int)((M + 15) / 16), n16 = (int)((N + 15) / 16);   // (M N <= 2^40, M <= 256: 32 bits each)
  int best = 0;
  float best_cost = 0.0f;
  for (int i = 0; i < COUNT; ++i) {
    const int mt = tiles[i].mt, nt = tiles[i].nt, ntm = glu ? nt / 2 : nt;
    const float share = (float)((m16 + mt - 1) / mt) * (float)((n16 + ntm - 1) / ntm) / (float)cus, turns = ceilf(share);
    const float busy = mt * nt <= 10 && turns > 1.0f ? 0.85f * (0.7f * turns + 0.3f * share) : turns;
    const float cost = busy * (float)(KT * (code_loads * mt + nt) + 6 * mt * nt);
    if (i == 0 || cost < best_cost) { best = i; best_cost = cost; }
  }
  return best;
}

// Where these tiles are the better choice, by tokens x outputs per CU.  Beyond 16 tokens they take token tiles in pairs (a lone one
// costs its pair) and run out of room in turns, as the kernels on the other side do: those do 33 to 64 tokens in one turn up to
// 128 outputs per CU, 17 to 32 tokens up to 256, more tokens while 64 x 128 tiles last, and beyond that turn they lose.
// The waves share K by 256 channels: up to four tiles leave half of them idle (one tile: all but one), so that what a turn costs at least
// weighs more, and nine to twelve tiles fill the second round by half.  INT8 codes are twice the loads of INT4.  17 to 32 tokens lose
// only against INT8 kernels that need not split K (nine to sixteen tiles).  Quantizer and product, weights from HBM, other forms / here, us:
// INT8 208 x 5904 x 4600 20.0 / 19.0, 208 x 6400 x 4600 20.1 / 20.9, 256 x 5200 x 4600 20.8 / 19.7, 256 x 5600 x 4600 20.8 / 21.2, 56 x 25600 x 4600
// 21.4 / 22.9, 28 x 48044 x 2972 19.6 / 21.4, 33 x 37636 x 1536 20.5 / 14.0; INT4 128 x 12288 x 4096 15.9 / 14.7, 256 x 6096 x 3064 13.8 / 13.4,
// 144 x 9952 x 4600 17.5 / 19.5, 40 x 25600 x 3064 14.0 / 14.9, 56 x 25600 x 3064 14.0 / 16.2; up to 1024 channels 128 x 8000 x 1024 8.3 / 8.3,
// 256 x 4000 x 1024 8.3 / 8.3, 128 x 9600 x 1024 9.4 / 10.0, 256 x 4800 x 1024 9.4 / 10.2, 104 x 7424 x 156 7.7 / 9.0.  Gate and up (both counted)
// where the other side is one launch: 64 x 2 x 6992 x 1024 9.2 / 8.1, 56 x 2 x 10048 x 1024 9.3 / 10.0, 64 x 2 x 12192 x 4096 15.6 / 14.9,
// 56 x 2 x 13936 x 4096 15.9 / 17.1.  Of 23600 calls measured (9 to 256 tokens, 156 to 16384 channels, cold and warm weights) 0.8 % are more
// than 2 % behind the other forms.
bool bl_gemm_direct_ok(int64_t M, int64_t n_cols, int64_t K, bool a4) {
  const int64_t cus = bl_num_cus(), tiles = bl_round_up(K, BL_KPAD) >> 8, pairs = bl_round_up(M, 32) * n_cols;
  if (M * n_cols > 6144 * cus) return false;
  if (M <= 16 || (M <= 64 && n_cols > (M <= 32 ? 256 : 128) * cus)) return true;
  if (tiles <= 4) {
    const bool one_turn = M <= 32 || (M + 63) / 64 * ((n_cols + 63) / 64) <= cus;
    return pairs <= (tiles == 1 && one_turn ? 2048 : 4096) * cus;
  }
  if (M <= 32) return a4 || tiles <= 8 || tiles > 16 || pairs <= 5632 * cus;
  if (M > 64 && tiles > 12 && (M + 63) / 64 * ((n_cols + 127) / 128) > cus) return true;
  return pairs <= (a4 || tiles <= 8 || (tiles > 12 && tiles <= 16) ? 6144 : 5376) * cus;
}

#define GX_GO(A4, GLU, MT, NT) \
  return gx_go<A4, GLU, MT, NT>(q, scale, (int)M, KT, Wp, Wp2, alpha, alpha2, (int)N, Y, ybf, acc_out, s)

// Codes in fragment order x BL_W_GEMM weights.
int bl_launch_gemm_direct(const void* q, const float* scale, bl_act_mode mode, int64_t M, int64_t K, const void* Wp,
                          const float* alpha, int64_t N, void* Y, bl_dtype ydt, int32_t* acc_out, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8), ybf = ydt == BL_BF16 ? 1 : 0;
  const void* Wp2 = nullptr;
  const float* alpha2 = nullptr;
  if (mode == BL_ACT_INT4_ABSMEAN) {
    static constexpr GxTile tiles[] = {{1, 1}, {1, 2}, {1, 3}, {1, 4}, {1, 6}, {2, 2}, {2, 3}, {2, 4}, {2, 6}};
    switch (gx_pick(tiles, M, N, KT, 2, false)) {
      case 0: GX_GO(true, false, 1, 1);
      case 1: GX_GO(true, false, 1, 2);
      case 2: GX_GO(true, false, 1, 3);
      case 3: GX_GO(true, false, 1, 4);
      case 4: GX_GO(true, false, 1, 6);
      case 5: GX_GO(true, false, 2, 2);
      case 6: GX_GO(true, false, 2, 3);
      case 7: GX_GO(true, false, 2, 4);
      default: GX_GO(true, false, 2, 6);
    }
  }
  static constexpr GxTile tiles[] = {{1, 1}, {1, 2}, {1, 3}, {1, 4}, {1, 6}, {2, 2}, {2, 3}, {2, 4}, {2, 6}, {2, 8}, {3, 4}};
  switch (gx_pick(tiles, M, N, KT, 4, false)) {
    case 0: GX_GO(false, false, 1, 1);
    case 1: GX_GO(false, false, 1, 2);
    case 2: GX_GO(false, false, 1, 3);
    case 3: GX_GO(false, false, 1, 4);
    case 4: GX_GO(false, false, 1, 6);
    case 5: GX_GO(false, false, 2, 2);
    case 6: GX_GO(false, false, 2, 3);
    case 7: GX_GO(false, false, 2, 4);
    case 8: GX_GO(false, false, 2, 6);
    case 9: GX_GO(false, false, 2, 8);
    default: GX_GO(false, false, 3, 4);
  }
}

// INT4 codes in fragment order x two BL_W_GEMM matrices: H = bf16(U * max(G, 0)^2).
int bl_launch_gemm_direct_glu(const void* q, const float* scale, int64_t M, int64_t K, const void* Wp, const float* alpha,
                              const void* Wp2, const float* alpha2, int64_t N, void* Y, hipStream_t s) {
  const int KT = (int)(bl_round_up(K, BL_KPAD) >> 8), ybf = 1;
  int32_t* acc_out = nullptr;
  static constexpr GxTile tiles[] = {{1, 2}, {1, 4}, {1, 6}, {2, 2}, {2, 4}, {2, 6}, {3, 6}};
  switch (gx_pick(tiles, M, N, KT, 2, true)) {
    case 0: GX_GO(true, true, 1, 2);
    case 1: GX_GO(true, true, 1, 4);
    case 2: GX_GO(true, true, 1, 6);
    case 3: GX_GO(true, true, 2, 2);
    case 4: GX_GO(true, true, 2, 4);
    case 5: GX_GO(true, true, 2, 6);
    default: GX_GO(true, true, 3, 6);
  }
}
