// Absmean ternarisation of a latent weight matrix and 2-bit packing (eq. 2 of the paper):
//   alpha = mean|W|,  T = RoundClip(W / (alpha + eps), -1, 1).
// Two kernels: a float64 partial-sum reduction of |W|, then ternarise + pack.  Every block of
// the second kernel re-adds the partial sums in one fixed order, so alpha is identical in all
// blocks and from run to run.
//
// Both are bound by reading W (float32 9600 x 3200: 123 MB, 24 us at the 5.1 TB/s of a plain copy).  So loads are
// 16 bytes per lane and several are in flight, and the ternary code of a weight is a comparison, not the division of
// eq. 2 (pt_ternary_bits).
#include "common.h"

#define PT_THREADS 256
#define PT_MAX_PARTIALS 1024

template <typename T> __device__ __forceinline__ float pt_load(const T* p, int64_t i);
template <> __device__ __forceinline__ float pt_load<float>(const float* p, int64_t i) { return p[i]; }
template <> __device__ __forceinline__ float pt_load<uint16_t>(const uint16_t* p, int64_t i) {
  return bl_bf16_to_f32(p[i]);
}

// Four consecutive elements at a multiple of their size.
__device__ __forceinline__ void pt_load4(const float* p, int64_t i, float (&v)[4]) {
  const float4 x = *reinterpret_cast<const float4*>(p + i);
  v[0] = x.x; v[1] = x.y; v[2] = x.z; v[3] = x.w;
}
__device__ __forceinline__ void pt_load4(const uint16_t* p, int64_t i, float (&v)[4]) {
  const uint2 x = *reinterpret_cast<const uint2*>(p + i);
  v[0] = __uint_as_float(x.x << 16); v[1] = __uint_as_float(x.x & 0xFFFF0000u);
  v[2] = __uint_as_float(x.y << 16); v[3] = __uint_as_float(x.y & 0xFFFF0000u);
}

// One load of an element per turn, as the loop was, kept too little in flight: 9600 x 3200 38 us alone.
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void abs_sum_partial_kernel(const T* __restrict__ W,
                                                                     int64_t n,
                                                                     double* __restrict__ partial) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const int64_t step = (int64_t)gridDim.x * PT_THREADS, first = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  double a[4] = {0.0, 0.0, 0.0, 0.0};
  const int64_t n4 = n >> 2;                // (W is 16-byte aligned: checked at the entry point)
  constexpr int U = 4;
  int64_t i = first;
  for (; i + (U - 1) * step < n4; i += U * step) {
    float v[U][4];
#pragma unroll
    for (int u = 0; u < U; ++u) pt_load4(W, 4 * (i + u * step), v[u]);
#pragma unroll
    for (int u = 0; u < U; ++u)
#pragma unroll
      for (int e = 0; e < 4; ++e) a[e] += (double)fabsf(v[u][e]);
  }
  for (; i < n4; i += step) {
    float v[4];
    pt_load4(W, 4 * i, v);
#pragma unroll
    for (int e = 0; e < 4; ++e) a[e] += (double)fabsf(v[e]);
  }
  for (int64_t j = 4 * n4 + first; j < n; j += step) a[0] += (double)fabsf(pt_load<T>(W, j));
  double acc = (a[0] + a[1]) + (a[2] + a[3]);
  acc = bl_wave_sum_f64(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) {
    double s = 0.0;
    for (int w = 0; w < PT_THREADS / BL_WAVE; ++w) s += red[w];
    partial[blockIdx.x] = s;
  }
}

// alpha from the partial sums, same order in every block.
template <int THREADS = PT_THREADS>
__device__ __forceinline__ float pt_alpha(const double* __restrict__ partial, int n_partial,
                                          int64_t n_elem, double* red) {
  double acc = 0.0;
  if (THREADS == PT_THREADS || threadIdx.x < PT_THREADS)     // (the same order in every layout's kernel)
    for (int i = threadIdx.x; i < n_partial; i += PT_THREADS) acc += partial[i];
  acc = bl_wave_sum_f64(acc);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  double s = 0.0;
  for (int w = 0; w < THREADS / BL_WAVE; ++w) s += red[w];
  return (float)(s / (double)n_elem);
}

__device__ __forceinline__ u32 pt_code(float w, float t) {
  float r = rintf(w / t);                 // IEEE divide, round half to even
  r = fminf(fmaxf(r, -1.0f), 1.0f);
  int c = (int)r;                          // -1, 0, 1
  return (u32)c & 3u;                      // two's complement 2-bit: 00, 01, 11
}
// The same code by comparison.  The rounded quotient is 0 unless |w| / t, rounded to float32, exceeds 0.5, that is
// unless |w| > t/2 + t 2^-25 (a quotient no further from 0.5 rounds to 0.5, whose mantissa is even).  t/2 is a float32 here,
// and for t = m 2^e, 1 <= m < 2, the next float32 above it exceeds it by 2^(e-24), which is strictly more than
// t 2^-25 = m 2^(e-25): for a float32 |w| the condition is |w| > t/2.
// Wants a finite t, which says that every weight is finite, and t/2 free of rounding (t well above the subnormals).
__device__ __forceinline__ u32 pt_ternary_bits(float w, float half) {
  const u32 u = __float_as_uint(w);
  return (u & 0x7FFFFFFFu) > __float_as_uint(half) ? 1u | ((u >> 30) & 2u) : 0u;
}
__device__ __forceinline__ bool pt_compare_ok(float t) { return t >= 0x1p-100f && t <= 0x1p100f; }

// body(code): code(w) is the ternary code of a weight.
template <typename Body>
__device__ __forceinline__ void pt_with_code(float t, Body body) {
  if (pt_compare_ok(t)) {
    const float half = 0.5f * t;
    body([=](float w) { return pt_ternary_bits(w, half); });
  } else {
    body([=](float w) { return pt_code(w, t); });
  }
}

// Tiled GEMM layout: a wave ternarises 4 output rows x 256 input channels (a quarter of a tile), 4 rows of 4 consecutive
// channels per lane, so that a wave reads whole rows of 1 KB.  Channel c of a word sits in field 4 (c % 4) + c / 4: the four
// lanes of a word hold disjoint fields, which two exchanges inside the quad put together; lane q of the quad then
// stores the word of row q (64-byte runs).  One thread per word with 16 loads of 4 bytes, 64 bytes apart between lanes,
// as it was: 9600 x 3200 99 us.
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void ternarize_pack_gemm_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, int64_t Kp, float eps, int vec,
    const double* __restrict__ partial, int n_partial, u32* __restrict__ out,
    float* __restrict__ alpha_out, int64_t n_tiles) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const float alpha = pt_alpha(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  const float t = alpha + eps;
  const int lane = threadIdx.x & 63, i0 = (threadIdx.x >> 6) * 4;   // rows i0 ... i0 + 3 of the tile
  const int q = lane & 3, g = lane >> 4, wt = (lane >> 2) & 3;
  const int64_t k_tiles = Kp / 256;
  pt_with_code(t, [&](auto code) {
    for (int64_t tile = blockIdx.x; tile < n_tiles; tile += gridDim.x) {
      const int64_t nt = tile / k_tiles, kt = tile - nt * k_tiles;
      const int64_t n0 = nt * 16 + i0, k = kt * 256 + 4 * lane;
      float v[4][4];
#pragma unroll
      for (int r = 0; r < 4; ++r) {
#pragma unroll
        for (int e = 0; e < 4; ++e) v[r][e] = 0.0f;       // (code 0 either way)
        if (n0 + r < N) {
          if (vec) {
            if (k < K) pt_load4(W, (n0 + r) * K + k, v[r]);
          } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
              if (k + e < K) v[r][e] = pt_load<T>(W, (n0 + r) * K + k + e);
          }
        }
      }
      u32 mine = 0;
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        u32 w = 0;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const bool pad = !(n0 + r < N && k + e < K);
          w |= (pad ? 0u : code(v[r][e])) << (2 * (4 * e + q));
        }
        w |= (u32)__builtin_amdgcn_mov_dpp((int)w, 0xB1, 0xF, 0xF, true);   // quad_perm [1, 0, 3, 2]
        w |= (u32)__builtin_amdgcn_mov_dpp((int)w, 0x4E, 0xF, 0xF, true);   // quad_perm [2, 3, 0, 1]
        if (r == q) mine = w;
      }
      out[tile * 256 + (g * 16 + i0 + q) * 4 + wt] = mine;
    }
  });
}

// Input-channel-major layout (column blocks of 512 outputs, 128 bytes per channel and block): a workgroup takes 64
// channels of one column block, a thread 4 of the channels and the 16 outputs of a word (16 loads of 16 bytes in flight, 256-byte
// runs of a row of W per 16 lanes); the words meet in LDS and leave as one run of 8 KB.  One thread per word and
// each word stored where it falls, 128 bytes apart between lanes, as it was: 9600 x 3200 46 us.
#define PT_KM_THREADS 512
template <typename T>
__global__ __launch_bounds__(PT_KM_THREADS) void ternarize_pack_kmajor_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, float eps, int vec,
    const double* __restrict__ partial, int n_partial, u32* __restrict__ out,
    float* __restrict__ alpha_out, int64_t k_blocks) {
  __shared__ double red[PT_KM_THREADS / BL_WAVE];
  __shared__ u32 words[64 * 33];
  const int64_t cb = blockIdx.x / k_blocks, k0 = (blockIdx.x - cb * k_blocks) * 64;
  const int c4 = (threadIdx.x & 15) * 4, d = threadIdx.x >> 4;          // channels k0 + c4 ... + 3, word d of 32
  const int64_t k = k0 + c4, n0 = cb * 512 + d * 16;
  float v[16][4];
#pragma unroll
  for (int f = 0; f < 16; ++f) {
#pragma unroll
    for (int e = 0; e < 4; ++e) v[f][e] = 0.0f;
    if (n0 + f < N) {
      if (vec) {
        if (k < K) pt_load4(W, (n0 + f) * K + k, v[f]);
      } else {
#pragma unroll
        for (int e = 0; e < 4; ++e)
          if (k + e < K) v[f][e] = pt_load<T>(W, (n0 + f) * K + k + e);
      }
    }
  }
  const float alpha = pt_alpha<PT_KM_THREADS>(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  pt_with_code(alpha + eps, [&](auto code) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      u32 word = 0;
#pragma unroll
      for (int f = 0; f < 16; ++f)
        if (n0 + f < N) word |= code(v[f][e]) << (2 * f);
      words[(c4 + e) * 33 + d] = word;
    }
  });
  __syncthreads();
  u32* dst = out + (cb * K + k0) * 32;
#pragma unroll
  for (int i = threadIdx.x; i < 64 * 32; i += PT_KM_THREADS)
    if (k0 + (i >> 5) < K) dst[i] = words[(i >> 5) * 33 + (i & 31)];
}

// The same layout, one thread per 32-bit word (channel k, 16 outputs; consecutive threads take consecutive channels, so reads
// are coalesced and each word is stored where it falls): for matrices with too few blocks of the kernel above.
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void ternarize_pack_kmajor_words_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, float eps, const double* __restrict__ partial, int n_partial,
    u32* __restrict__ out, float* __restrict__ alpha_out, int64_t n_words) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const float alpha = pt_alpha(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  const int64_t id = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  if (id >= n_words) return;
  const int64_t k = id % K, d = id / K;
  u32 word = 0;
  pt_with_code(alpha + eps, [&](auto code) {
#pragma unroll
    for (int f = 0; f < 16; ++f) {
      const int64_t n = d * 16 + f;
      if (n < N) word |= code(pt_load<T>(W, n * K + k)) << (2 * f);
    }
  });
  out[((d >> 5) * K + k) * 32 + (d & 31)] = word;
}

// One thread per 32-bit word of the block-float GEMM layout: blocks of 32 outputs x 128 input
// channels (2048 bytes); inside, row r = n % 32 takes 64 bytes, its 16-byte piece p holds the
// 32 channels of unit u = p ^ ((r / 4) % 4) as E2M1 nibbles (0 -> 0000, +1 -> 0010, -1 -> 1010),
// low nibble first.  A word covers 8 consecutive channels.
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void ternarize_pack_mx4_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, int64_t Kp, float eps,
    const double* __restrict__ partial, int n_partial, u32* __restrict__ out,
    float* __restrict__ alpha_out, int64_t n_words) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const float alpha = pt_alpha(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  const float t = alpha + eps;
  const int64_t w = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  if (w >= n_words) return;
  const int64_t blk = w >> 9;               // 512 words per block
  const int in = (int)(w & 511);
  const int r = in >> 4, p = (in >> 2) & 3, j = in & 3;
  const int64_t KB = Kp / 128;
  const int64_t n = (blk / KB) * 32 + r;
  const int64_t k0 = (blk % KB) * 128 + 32 * (p ^ ((r >> 2) & 3)) + 8 * j;
  u32 word = 0;
  pt_with_code(t, [&](auto code) {
    if (n >= N) return;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int64_t k = k0 + i;
      if (k < K) {
        const u32 c = code(pt_load<T>(W, n * K + k));        // 00, 01, 11
        word |= (((c & 2u) << 2) | ((c & 1u) << 1)) << (4 * i);    // sign to bit 3, magnitude 1.0 = 010
      }
    }
  });
  out[w] = word;
}

// One thread per 32-bit word of the 2-bit block-float GEMM layout: blocks of 32 outputs x 128 input
// channels (1024 bytes); inside, row r = n % 32 takes 32 bytes, its 8-byte piece p holds the 32
// channels of unit u = p ^ ((r / 8) % 4) as two words of 16 channels: nibble j of a word keeps
// channels j and 8 + j as (sign j, sign 8+j, magnitude j, magnitude 8+j) from bit 3 down, so that
// one mask, and one shift and mask, give their E2M1 nibbles (sign 0 magnitude 0).
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void ternarize_pack_mx2_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, int64_t Kp, float eps,
    const double* __restrict__ partial, int n_partial, u32* __restrict__ out,
    float* __restrict__ alpha_out, int64_t n_words) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const float alpha = pt_alpha(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  const float t = alpha + eps;
  const int64_t w = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  if (w >= n_words) return;
  const int64_t blk = w >> 8;               // 256 words per block
  const int in = (int)(w & 255);
  const int r = in >> 3, p = (in >> 1) & 3, h = in & 1;
  const int64_t KB = Kp / 128;
  const int64_t n = (blk / KB) * 32 + r;
  const int64_t k0 = (blk % KB) * 128 + 32 * (p ^ ((r >> 3) & 3)) + 16 * h;
  u32 word = 0;
  pt_with_code(t, [&](auto code) {
    if (n >= N) return;
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      if (k0 + j < K) {
        const u32 c = code(pt_load<T>(W, n * K + k0 + j));            // 00, 01, 11
        word |= (((c & 2u) << 2) | ((c & 1u) << 1)) << (4 * j);
      }
      if (k0 + 8 + j < K) {
        const u32 c = code(pt_load<T>(W, n * K + k0 + 8 + j));
        word |= (((c & 2u) << 1) | (c & 1u)) << (4 * j);
      }
    }
  });
  out[w] = word;
}

// One thread per 32-bit word of the output-channel-major layout: row n, channels 16 w .. 16 w + 15,
// channel 16 w + f in bits 2 f, 2 f + 1.
template <typename T>
__global__ __launch_bounds__(PT_THREADS) void ternarize_pack_rows_kernel(
    const T* __restrict__ W, int64_t N, int64_t K, int64_t Kp, float eps,
    const double* __restrict__ partial, int n_partial, u32* __restrict__ out,
    float* __restrict__ alpha_out, int64_t n_words) {
  __shared__ double red[PT_THREADS / BL_WAVE];
  const float alpha = pt_alpha(partial, n_partial, N * K, red);
  if (blockIdx.x == 0 && threadIdx.x == 0) alpha_out[0] = alpha;
  const float t = alpha + eps;
  const int64_t w = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  if (w >= n_words) return;
  const int64_t wpr = Kp / 16, n = w / wpr, k0 = (w % wpr) * 16;
  u32 word = 0;
  pt_with_code(t, [&](auto code) {
#pragma unroll
    for (int f = 0; f < 16; ++f)
      if (k0 + f < K) word |= code(pt_load<T>(W, n * K + k0 + f)) << (2 * f);
  });
  out[w] = word;
}

__global__ __launch_bounds__(PT_THREADS) void unpack_ternary_kernel(const u32* __restrict__ packed,
                                                                    int64_t N, int64_t K,
                                                                    int64_t Kp, int64_t Np,
                                                                    int layout,
                                                                    int8_t* __restrict__ T) {
  const int64_t id = (int64_t)blockIdx.x * PT_THREADS + threadIdx.x;
  if (id >= N * K) return;
  const int64_t n = id / K, k = id % K;
  u32 word;
  int f;
  if (layout == BL_W_MX4) {
    const int r = (int)(n & 31), u = (int)((k >> 5) & 3), i = (int)(k & 31);
    const u32 w4 = packed[((n >> 5) * (Kp / 128) + (k >> 7)) * 512 + r * 16 + ((u ^ ((r >> 2) & 3)) << 2) + (i >> 3)];
    const u32 c = (w4 >> (4 * (i & 7))) & 15u;
    T[id] = (int8_t)(c == 0 ? 0 : ((c & 8u) ? -1 : 1));
    return;
  }
  if (layout == BL_W_MX2) {
    const int r = (int)(n & 31), u = (int)((k >> 5) & 3), i = (int)(k & 31);
    word = packed[((n >> 5) * (Kp / 128) + (k >> 7)) * 256 + r * 8 + ((u ^ ((r >> 3) & 3)) << 1) + (i >> 4)];
    const u32 nib = (word >> (4 * (i & 7))) << ((i >> 3) & 1);       // channel's sign in bit 3, magnitude in bit 1
    T[id] = (int8_t)((nib & 2u) ? ((nib & 8u) ? -1 : 1) : 0);
    return;
  } else if (layout == BL_W_ROWS) {
    word = packed[n * (Kp / 16) + (k >> 4)];
    f = (int)(k & 15);
  } else if (layout == BL_W_GEMM) {
    const int64_t nt = n >> 4, kt = k >> 8;
    const int i = (int)(n & 15), g = (int)((k >> 6) & 3), t = (int)((k >> 4) & 3);
    const int kk = (int)(k & 15);
    f = 4 * (kk & 3) + (kk >> 2);
    word = packed[(nt * (Kp / 256) + kt) * 256 + (g * 16 + i) * 4 + t];
  } else {
    word = packed[((n >> 9) * K + k) * 32 + ((n >> 4) & 31)];
    f = (int)(n & 15);
  }
  const u32 c = (word >> (2 * f)) & 3u;
  T[id] = (int8_t)((int)(c << 30) >> 30);   // sign-extend the 2-bit field
}

static int pt_num_partials(int64_t n) {
  int64_t b = (n + (int64_t)PT_THREADS * 16 - 1) / ((int64_t)PT_THREADS * 16);
  if (b < 1) b = 1;
  if (b > PT_MAX_PARTIALS) b = PT_MAX_PARTIALS;
  return (int)b;
}

extern "C" size_t pack_ternary_workspace_bytes(int64_t N, int64_t K) {
  (void)N; (void)K;
  return PT_MAX_PARTIALS * sizeof(double);
}

template <typename T>
static int pt_run(const T* W, int64_t N, int64_t K, float eps, bl_w_layout layout, void* out,
                  float* alpha, void* ws, hipStream_t s) {
  const int64_t n = N * K;
  const int np = pt_num_partials(n);
  double* partial = (double*)ws;
  const int vec = K % 4 == 0 ? 1 : 0;              // rows of whole, aligned groups of four
  abs_sum_partial_kernel<T><<<np, PT_THREADS, 0, s>>>(W, n, partial);
  BL_HIP_CHECK_LAUNCH();
  if (layout == BL_W_MX4) {
    const int64_t Kp = bl_round_up(K, BL_KPAD), Np = bl_round_up(N, 32);
    const int64_t n_words = Np * Kp / 8;
    const int64_t blocks = (n_words + PT_THREADS - 1) / PT_THREADS;
    ternarize_pack_mx4_kernel<T><<<(unsigned)blocks, PT_THREADS, 0, s>>>(
        W, N, K, Kp, eps, partial, np, (u32*)out, alpha, n_words);
  } else if (layout == BL_W_MX2) {
    const int64_t Kp = bl_round_up(K, BL_KPAD), Np = bl_round_up(N, 32);
    const int64_t n_words = Np * Kp / 16;
    const int64_t blocks = (n_words + PT_THREADS - 1) / PT_THREADS;
    ternarize_pack_mx2_kernel<T><<<(unsigned)blocks, PT_THREADS, 0, s>>>(
        W, N, K, Kp, eps, partial, np, (u32*)out, alpha, n_words);
  } else if (layout == BL_W_ROWS) {
    const int64_t Kp = bl_round_up(K, BL_KPAD);
    const int64_t n_words = N * Kp / 16;
    const int64_t blocks = (n_words + PT_THREADS - 1) / PT_THREADS;
    ternarize_pack_rows_kernel<T><<<(unsigned)blocks, PT_THREADS, 0, s>>>(
        W, N, K, Kp, eps, partial, np, (u32*)out, alpha, n_words);
  } else if (layout == BL_W_GEMM) {
    const int64_t Kp = bl_round_up(K, BL_KPAD);
    const int64_t n_tiles = bl_round_up(N, 16) / 16 * (Kp / 256);
    // (8 workgroups per CU: each adds the partial sums once for all its tiles)
    const int64_t blocks = n_tiles < 8 * (int64_t)bl_num_cus() ? n_tiles : 8 * (int64_t)bl_num_cus();
    ternarize_pack_gemm_kernel<T><<<(unsigned)blocks, PT_THREADS, 0, s>>>(
        W, N, K, Kp, eps, vec, partial, np, (u32*)out, alpha, n_tiles);
  } else {
    const int64_t k_blocks = (K + 63) / 64, blocks = bl_round_up(N, 512) / 512 * k_blocks;
    // One word per thread where the 64 x 512 blocks leave too much of the chip idle for their longer chains: fewer than 100 of
    // them (1024 x 1024, 32 blocks: float32 8.6 us against 9.8, bfloat16 8.6 / 10.5; 1536 x 2048, 96: 10.7 / 11.0, 10.5 / 11.5;
    // on the other side 2048 x 2048, 128: 13.5 / 11.8, 11.4 / 11.7), or no more than one per CU where rows are not whole groups of four
    // (1000 x 1001, 32: 8.7 / 14.3, 8.8 / 13.6; 2048 x 4095, 256: 20.4 / 20.6, 17.1 / 20.9).
    if (vec ? blocks < 100 : blocks <= bl_num_cus()) {
      const int64_t n_words = K * (bl_round_up(N, 512) / 16);
      ternarize_pack_kmajor_words_kernel<T><<<(unsigned)((n_words + PT_THREADS - 1) / PT_THREADS), PT_THREADS, 0, s>>>(
          W, N, K, eps, partial, np, (u32*)out, alpha, n_words);
    } else {
      ternarize_pack_kmajor_kernel<T><<<(unsigned)blocks, PT_KM_THREADS, 0, s>>>(
          W, N, K, eps, vec, partial, np, (u32*)out, alpha, k_blocks);
    }
  }
  BL_HIP_CHECK_LAUNCH();
  return BL_OK;
}

int bl_launch_pack_ternary(const void* W, bl_dtype dt, int64_t N, int64_t K, float eps,
                           bl_w_layout layout, void* out, float* alpha, void* ws, hipStream_t s) {
  if (dt == BL_F32) return pt_run<float>((const float*)W, N, K, eps, layout, out, alpha, ws, s);
  return pt_run<uint16_t>((const uint16_t*)W, N, K, eps, layout, out, alpha, ws, s);
}

int bl_launch_unpack_ternary(const void* packed, int64_t N, int64_t K, bl_w_layout layout,
                             int8_t* T, hipStream_t s) {
  const int64_t blocks = (N * K + PT_THREADS - 1) / PT_THREADS;
  unpack_ternary_kernel<<<(unsigned)blocks, PT_THREADS, 0, s>>>(
      (const u32*)packed, N, K, bl_round_up(K, BL_KPAD), bl_round_up(N, 512), (int)layout, T);
  BL_HIP_CHECK_LAUNCH();
  return BL_OK;
}
