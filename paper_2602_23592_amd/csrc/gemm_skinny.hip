// Weight-streaming GEMMs for launches of a few rows (bf16 in, fp32 accumulate): C[M, N] = A[M, K] . B[N, K]^T.
//
// With so few rows the work is reading the weights once: these kernels are bound by HBM, not by the matrix cores.
// They carry greedy decoding (one row), short instructions over a reused prompt and the caching of one short memory
// unit (Section 4.1).  k_gemv (up to 16 rows, weights in bf16 or in the 4-bit form; wide bf16 projections of 8 to 16 rows
// are k_gemm_stream's) finishes its outputs itself;
// k_gemm_skinny_w4 (17 to 32 or 40 rows, 4-bit form only) writes K slices that k_skinny_finish adds.
#include <algorithm>

#include "keep_internal.h"

namespace keep {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(16))) float f32x16;

constexpr int SK_BN = 64;       // weight rows per workgroup
constexpr size_t SK_MAX_PART_FLOATS = (size_t)64 * 65536;  // capacity of the partials workspace

size_t gemm_skinny_ws_bytes() { return SK_MAX_PART_FLOATS * sizeof(float); }

struct SkinnyEpi {       // what the finishing pass needs
  int epilogue;          // GemmEpilogue
  int N;                 // output columns (SwiGLU: gate and up each have N)
  const bf16_t* residual;
  void* C;
};

// One output element from the S slices, summed in slice order.
__device__ __forceinline__ void skinny_store(const float* __restrict__ part, int n_splits, int ld, int M, int m, int n,
                                             const SkinnyEpi& e) {
  float s0 = 0.f, s1 = 0.f;
  for (int z = 0; z < n_splits; ++z) {
    const float* p = part + ((size_t)z * M + m) * ld;
    s0 += p[n];
    if (e.epilogue == EPI_SWIGLU_STORE) s1 += p[e.N + n];
  }
  const size_t idx = (size_t)m * e.N + n;
  if (e.epilogue == EPI_STORE_F32) {
    reinterpret_cast<float*>(e.C)[idx] = s0;
  } else if (e.epilogue == EPI_RESIDUAL_STORE) {
    reinterpret_cast<bf16_t*>(e.C)[idx].bits = f32_to_bf16_bits(bf16_bits_to_f32(e.residual[idx].bits) + s0);
  } else {
    reinterpret_cast<bf16_t*>(e.C)[idx].bits = f32_to_bf16_bits(s0 / (1.0f + __expf(-s0)) * s1);
  }
}

// C = epilogue(sum over the K slices, in slice order)
__global__ void __launch_bounds__(256)
    k_skinny_finish(const float* __restrict__ part, int n_splits, int ld, int M, SkinnyEpi e) {
  const int n = blockIdx.x * 256 + threadIdx.x;
  const int m = blockIdx.y;
  if (n >= e.N || m >= M) return;
  skinny_store(part, n_splits, ld, M, m, n, e);
}

// ---------------------------------------------------------------------------------------------
// INT4 weight-only variant (Section 6.1: the 32B model runs with INT4 weight-only quantisation).
// The weights the model computes with are  w = bf16((q - z) * s)  per group of 128 input features
// (codes q and zero z of 4 bits, scale s in bf16).  Launches of a few dozen rows are bound by
// reading the weights, so they read the 4-bit form (a quarter of the bytes) and expand it in
// registers to exactly those bf16 values; launches with many rows are bound by the matrix cores
// and use a bf16 copy expanded once by k_dequant_int4.
//
// Storage (rows a multiple of 32): codes in blocks of 32 rows x 128 features, ordered by (row block, feature
// group), 2048 bytes each; inside a block 64 bytes per row; within a run of 8 features byte t holds feature t
// (low nibble) and feature t + 4 (high nibble).  One 32-bit word per (row, group): scale bits | zero << 16,
// in the same block order, 32 words per block.  A wave step of the GEMM below reads one such block per row
// tile: one contiguous 2 KB request for the codes, one 128-byte request for the words.
// ---------------------------------------------------------------------------------------------
constexpr int W4_GROUP = 128;
constexpr int W4_ROWS = 32;                          // rows per storage block
constexpr int W4_BLOCK_BYTES = W4_ROWS * W4_GROUP / 2;  // 2048

// Eight weights of one code word -> 8 bf16 (4 packed words), in feature order.
// (q - z) * s has <= 13 significant bits, so fma(q, s, -z*s) is exact and the only rounding is the
// conversion to bf16 (round to nearest even).
// byte N of a word as a float (v_cvt_f32_ubyteN: the shift, the mask and the conversion in one instruction)
#define W4_UBYTE(N, DST, SRC) asm("v_cvt_f32_ubyte" #N " %0, %1" : "=v"(DST) : "v"(SRC))
__device__ __forceinline__ void w4_expand8(uint32_t d, float sc, float nzs, uint32_t out[4]) {
  const uint32_t lo = d & 0x0F0F0F0Fu, hi = (d >> 4) & 0x0F0F0F0Fu;  // features 0..3 and 4..7 as bytes
  float f[8];
  W4_UBYTE(0, f[0], lo); W4_UBYTE(1, f[1], lo); W4_UBYTE(2, f[2], lo); W4_UBYTE(3, f[3], lo);
  W4_UBYTE(0, f[4], hi); W4_UBYTE(1, f[5], hi); W4_UBYTE(2, f[6], hi); W4_UBYTE(3, f[7], hi);
#pragma unroll
  for (int t = 0; t < 8; ++t) f[t] = __builtin_fmaf(f[t], sc, nzs);
#pragma unroll
  for (int t = 0; t < 4; ++t) out[t] = pack_bf16x2(f[2 * t], f[2 * t + 1]);
}
#undef W4_UBYTE

__device__ __forceinline__ void w4_scale_zero(uint32_t word, float& sc, float& nzs) {
  sc = __uint_as_float(word << 16);
  nzs = -(float)((word >> 16) & 0xFu) * sc;  // exact: 4 bits times 8 bits
}

// one code word (8 features of one row) per thread, in storage order
__global__ void __launch_bounds__(256)
    k_dequant_int4(const uint32_t* __restrict__ codes, const uint32_t* __restrict__ scale_zero, long n_words,
                   int groups, int K, uint4* __restrict__ out) {
  const long i = (long)blockIdx.x * 256 + threadIdx.x;
  if (i >= n_words) return;
  const long block = i / (W4_BLOCK_BYTES / 4);                 // (row block, group)
  const int within = (int)(i - block * (W4_BLOCK_BYTES / 4));  // word inside the block: row * 16 + run of 8
  const int r = within >> 4, run = within & 15;
  const long rb = block / groups;
  const int kg = (int)(block - rb * groups);
  float sc, nzs;
  w4_scale_zero(scale_zero[block * W4_ROWS + r], sc, nzs);
  uint32_t o[4];
  w4_expand8(codes[i], sc, nzs, o);
  const size_t row = (size_t)rb * W4_ROWS + r;
  out[(row * K + (size_t)kg * W4_GROUP + 8 * run) / 8] = make_uint4(o[0], o[1], o[2], o[3]);
}

void launch_dequant_int4(const void* codes, const void* scale_zero, int32_t rows, int32_t K, void* out, hipStream_t s) {
  const long n_words = (long)rows * (K / 8);
  if (n_words <= 0) return;
  hipLaunchKernelGGL(k_dequant_int4, dim3((unsigned)((n_words + 255) / 256)), dim3(256), 0, s,
                     reinterpret_cast<const uint32_t*>(codes), reinterpret_cast<const uint32_t*>(scale_zero), n_words,
                     K / W4_GROUP, K, reinterpret_cast<uint4*>(out));
}

// ---------------------------------------------------------------------------------------------
// k_gemv: up to 16 rows.
//
// Bound by HBM.  A workgroup owns tiles of 16 weight rows over the WHOLE of K; its eight waves take the K steps
// round-robin and add their partial tiles through LDS, so nothing is written for another kernel to finish and the
// epilogue (residual, SwiGLU, or bias + RoPE + scatter into the cache) runs in place.  The weights are the A operand
// of v_mfma_f32_16x16x32_bf16 (lane l: row l % 16, eight k of block l / 16), the activations its B operand.
// Operands go global -> registers (no weight is shared between waves) through buffer loads: a lane whose row or step
// lies past the end reads zeros and costs no memory traffic, which keeps the loop one straight line of loads with
// exact wait counts, DEPTH steps ahead of their use, also across the ends of tiles.
// With one row (decoding) the activations sit in LDS, and the RMSNorm in front of the projection is done there by
// every workgroup for itself while its first weights are on their way: the row is 10 KB, and the launch that did it
// took 4.6 us, as did the RoPE/scatter launch behind QKV and each launch that added K slices.
// Per decoded token and layer at hidden 5120, FFN 13824 (550 MB of weights): 104 us = 5.3 TB/s, where K slices written
// as partials and added by a second kernel, a norm and a RoPE/scatter kernel took 146 us; gate/up alone 49.0 us
// (5.8 TB/s), vocabulary of 152064 rows 251 us (6.2 TB/s).  With 16 rows every wave reads its activations from L2 beside
// the weights: gate/up 55 us, output and down projection 25 us on average, QKV 21 us (64, 26 and 23 us where a cache of
// 135 MB per layer is read and written in between).
// ---------------------------------------------------------------------------------------------
struct GemvArgs {
  const bf16_t* A;
  int M, K, N;            // N: output columns
  int units;              // output columns (SwiGLU, RoPE: column pairs) of a workgroup's tile, at most 16 per MFMA tile
  int tiles, red_offset;  // tiles of `units` in all; byte offset of the partial sums in LDS
  const bf16_t* norm_w;   // one row: RMSNorm weights to apply to A first, or NULL
  float eps;
  const void* w[3];       // bf16 rows or 4-bit codes; SwiGLU: gate, up
  const uint32_t* sz[3];  // 4-bit form: scale / zero words
  int begin[4];           // first output column of each part (SwiGLU: unused)
  const bf16_t* residual;
  void* C;
  QkvEpilogue qe;
};

constexpr int GV_WAVES = 8;
constexpr int GV_MAX_ROWS = 16;
constexpr int GV_MAX_LDS = 158 * 1024;
constexpr uint32_t GV_PAST_END = 0x40000000u;  // beyond every tile's record count: the load returns zero
constexpr int GV_RS = 20;  // floats per (wave, MFMA tile, activation row) of the partial sums
constexpr int GV_RSRC_FLAGS = 0x00020000;      // raw buffer, 32-bit data format

typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;

template <typename P>
__device__ __forceinline__ P* uniform_ptr(P* p) {
  const uint64_t u = reinterpret_cast<uint64_t>(p);
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)u), hi = __builtin_amdgcn_readfirstlane((uint32_t)(u >> 32));
  return reinterpret_cast<P*>((uint64_t)hi << 32 | lo);
}

template <int EPI, int NT, bool ONE_ROW, bool W4>
__global__ void __launch_bounds__(GV_WAVES * 64, ONE_ROW ? 4 : 2) k_gemv(GemvArgs g) {
  constexpr int T = GV_WAVES * 64;
  constexpr int KS = W4 ? 128 : 64;                      // K per wave step
  constexpr int LD = W4 ? 1 : 2;                         // 16-byte loads per tile and step
  // Steps requested ahead.  Two are enough (with bf16 weights 16 waves of a CU have NT x 64 KB on their way), and more is
  // slower: the gate/up launch at 27648 x 5120 (NT = 2) takes 49.0 us with two, 50.1 with three, 51.7 with four.
  constexpr int DEPTH = W4 && NT == 1 ? 3 : 2;
  constexpr int MF = KS / 32;                            // MFMAs per tile and step
  constexpr int ADEPTH = ONE_ROW ? 1 : DEPTH;
  extern __shared__ __attribute__((aligned(16))) char gv_smem[];
  __shared__ float s_norm[GV_WAVES];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int row = lane & 15, kg = lane >> 4;
  const int M = g.M, K = g.K;
  const int units = g.units, N = g.N;
  // With several parts (q | k | v) a block has one tile, and the tile lies in one part: units is 16 or, of pairs, 8 or
  // 16, which divide the parts (and a head's 64 pairs).
  int first = 0, last = EPI == EPI_QKV_ROPE ? N / 2 : N, part = 0;  // the part's units, and which it is
  const void *base0 = g.w[0], *base1 = g.w[1], *bias = nullptr;
  const uint32_t *sz0 = g.sz[0], *sz1 = g.sz[1];
  if (EPI == EPI_QKV_ROPE || EPI == EPI_STORE_F32) {
    constexpr int D = EPI == EPI_QKV_ROPE ? 2 : 1;
    const int u = blockIdx.x * units;
    bias = g.qe.bias[0];
    if (u * D >= g.begin[2]) {
      part = 2, first = g.begin[2] / D, base0 = g.w[2], sz0 = g.sz[2], bias = g.qe.bias[2];
    } else if (u * D >= g.begin[1]) {
      part = 1, first = g.begin[1] / D, last = g.begin[2] / D, base0 = g.w[1], sz0 = g.sz[1], bias = g.qe.bias[1];
    } else {
      last = g.begin[1] / D;
    }
  }
  constexpr bool PAIRS = EPI == EPI_SWIGLU_STORE || EPI == EPI_QKV_ROPE;
  constexpr int UT = PAIRS ? NT / 2 : NT;  // MFMA tiles of 16 units
  // ---- a tile of units (output columns, or the column pairs of SwiGLU and RoPE): u0 .. u0 + count - 1 of one part
  struct Units {
    int u0, count;
  };
  auto units_of = [&](int tile) {
    Units q;
    q.u0 = tile * units - first;
    q.count = min(units, last - first - q.u0);
    return q;
  };
  const char* wp[NT];
  const uint32_t* zp[NT];
  int wn[NT], zn[NT];
  uint32_t w_lane[NT], z_lane[NT];
  auto aim = [&](int tile) {  // point the loads at a tile
    const Units q = units_of(tile);
#pragma unroll
    for (int t = 0; t < NT; ++t) {
      // weight rows rb .. re of the MFMA tile (consecutive units are consecutive rows; RoPE pairs column c of a head
      // with c + 64); lanes past them read nothing
      const int ub = q.u0 + min((t % UT) * 16, q.count - 1), n_rows = min(16, q.count - (t % UT) * 16);
      const int rb = EPI == EPI_QKV_ROPE ? (ub >> 6) * 128 + (ub & 63) + (t / UT) * 64 : ub;
      const int r = rb + max(0, min(row, n_rows - 1)), re = rb + max(0, n_rows - 1);
      const void* base = EPI == EPI_SWIGLU_STORE && t >= UT ? base1 : base0;
      const uint32_t* sz = EPI == EPI_SWIGLU_STORE && t >= UT ? sz1 : sz0;
      if (W4) {  // storage block (r / 32, step): 2048 code bytes, 32 words
        const int groups = K / W4_GROUP, db = (r >> 5) - (rb >> 5), nb = (re >> 5) - (rb >> 5) + 1;
        wp[t] = reinterpret_cast<const char*>(base) + (size_t)(rb >> 5) * groups * W4_BLOCK_BYTES;
        zp[t] = sz + (size_t)(rb >> 5) * groups * W4_ROWS;
        w_lane[t] = db * groups * W4_BLOCK_BYTES + (r & 31) * 64 + kg * 16;
        z_lane[t] = (db * groups * W4_ROWS + (r & 31)) * 4;
        wn[t] = nb * groups * W4_BLOCK_BYTES;
        zn[t] = nb * groups * W4_ROWS * 4;
      } else {
        wp[t] = reinterpret_cast<const char*>(base) + (size_t)rb * K * 2;
        w_lane[t] = (uint32_t)(r - rb) * K * 2 + kg * 16;
        wn[t] = (re - rb + 1) * K * 2;
        zp[t] = nullptr;
        z_lane[t] = zn[t] = 0;
      }
      if (row >= n_rows) w_lane[t] = z_lane[t] = GV_PAST_END;
      // (the descriptors in scalar registers: where the compiler cannot prove it, it loops over lanes at every load)
      wp[t] = uniform_ptr(wp[t]);
      wn[t] = __builtin_amdgcn_readfirstlane(wn[t]);
      zp[t] = uniform_ptr(zp[t]);
      zn[t] = __builtin_amdgcn_readfirstlane(zn[t]);
    }
  };
  const uint32_t a_lane = (uint32_t)row * K * 2 + kg * (W4 ? 64 : 16);
  const int steps = K / KS;
  const int n_i = wave < steps ? (steps - wave + GV_WAVES - 1) / GV_WAVES : 0;  // this wave's steps of a tile: wave, + 8, ...
  const int n_p = max(1, (n_i + DEPTH - 1) / DEPTH) * DEPTH;  // padded, so that every tile starts at buffer 0
  const int n_tiles = (g.tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;  // this block's: blockIdx, + grid, ...

  // The steps of all its tiles are one sequence: the loads run DEPTH steps ahead of the products, over the ends of
  // tiles and the barriers there (lt, li: tile and step the next load is for).
  int lt = 0, li = 0;
  u32x4 w[DEPTH][NT][LD];
  uint32_t z[DEPTH][NT];
  u32x4 a[ADEPTH][MF];
#define GV_RSRC(P, N) __builtin_amdgcn_make_buffer_rsrc(const_cast<char*>(reinterpret_cast<const char*>(P)), 0, (N), GV_RSRC_FLAGS)
#define GV_LOAD(BUF)                                                                                               \
  {                                                                                                                \
    const bool live_ = lt < n_tiles && li < n_i;                                                                   \
    const int st_ = wave + li * GV_WAVES;                                                                          \
    const uint32_t wo_ = live_ ? (uint32_t)st_ * (W4 ? W4_BLOCK_BYTES : KS * 2) : GV_PAST_END;                     \
    _Pragma("unroll") for (int t = 0; t < NT; ++t) {                                                               \
      _Pragma("unroll") for (int c = 0; c < LD; ++c) w[BUF][t][c] =                                                \
          __builtin_amdgcn_raw_buffer_load_b128(GV_RSRC(wp[t], wn[t]), w_lane[t] + wo_ + c * 64, 0, 0);            \
      if (W4) z[BUF][t] = __builtin_amdgcn_raw_buffer_load_b32(                                                    \
          GV_RSRC(zp[t], zn[t]), z_lane[t] + (live_ ? (uint32_t)st_ * (W4_ROWS * 4) : GV_PAST_END), 0, 0);         \
    }                                                                                                              \
    if (!ONE_ROW) {                                                                                                \
      const uint32_t ao_ = a_lane + (live_ ? (uint32_t)st_ * (KS * 2) : GV_PAST_END);                              \
      _Pragma("unroll") for (int c = 0; c < MF; ++c) a[(BUF) % ADEPTH][c] =                                        \
          __builtin_amdgcn_raw_buffer_load_b128(GV_RSRC(g.A, M * K * 2), ao_ + c * (W4 ? 16 : 64), 0, 0);          \
    }                                                                                                              \
    if (++li >= n_p) {                                                                                             \
      li = 0;                                                                                                      \
      if (++lt < n_tiles) aim(blockIdx.x + lt * gridDim.x);                                                        \
    }                                                                                                              \
  }

  // ---- one row: the activations (normalised where asked) into LDS, behind the first weights' requests
  bf16_t* act = reinterpret_cast<bf16_t*>(gv_smem);
  // 16-byte vectors per thread kept in registers: rows of up to 8192 (the hidden width; 28672 where the FFN's width
  // may come); longer ones loop
  constexpr int XV = NT == 1 ? 7 : 2;
  u32x4 xv[XV], gv[2] = {};
  const u32x4* xs = reinterpret_cast<const u32x4*>(g.A);
  const u32x4* gs = reinterpret_cast<const u32x4*>(g.norm_w);
  const int nv = K / 8;
  if (ONE_ROW) {
#pragma unroll
    for (int j = 0; j < XV; ++j)
      if (j * T < nv) xv[j] = __builtin_amdgcn_raw_buffer_load_b128(GV_RSRC(xs, K * 2), (tid + j * T) * 16, 0, 0);
    if (g.norm_w) {
#pragma unroll
      for (int j = 0; j < 2; ++j)
        if (j * T < nv) gv[j] = __builtin_amdgcn_raw_buffer_load_b128(GV_RSRC(gs, K * 2), (tid + j * T) * 16, 0, 0);
    }
  }
  aim(blockIdx.x);
#pragma unroll
  for (int j = 0; j < DEPTH; ++j) GV_LOAD(j)
  if (ONE_ROW) {
    u32x4* av = reinterpret_cast<u32x4*>(act);
    if (g.norm_w) {
      auto sumsq = [](const u32x4& v) {
        float s = 0.f;
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float lo = __uint_as_float(v[e] << 16), hi = __uint_as_float(v[e] & 0xffff0000u);
          s += lo * lo + hi * hi;
        }
        return s;
      };
      auto scaled = [](const u32x4& v, const u32x4& gw, float inv) {
        u32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e)
          o[e] = pack_bf16x2(__uint_as_float(v[e] << 16) * inv * __uint_as_float(gw[e] << 16),
                             __uint_as_float(v[e] & 0xffff0000u) * inv * __uint_as_float(gw[e] & 0xffff0000u));
        return o;
      };
      float ss = 0.f;  // (vectors past the row's end were read as zeros)
#pragma unroll
      for (int j = 0; j < XV; ++j)
        if (j * T < nv) ss += sumsq(xv[j]);
      for (int i = tid + XV * T; i < nv; i += T) ss += sumsq(xs[i]);
#pragma unroll
      for (int o = 32; o > 0; o >>= 1) ss += __shfl_xor(ss, o, 64);
      if (lane == 0) s_norm[wave] = ss;
      __syncthreads();
      float tot = 0.f;
#pragma unroll
      for (int i = 0; i < GV_WAVES; ++i) tot += s_norm[i];
      const float inv = 1.0f / sqrtf(tot / (float)K + g.eps);
#pragma unroll
      for (int j = 0; j < XV; ++j) {
        const int i = tid + j * T;
        if (i < nv) av[i] = scaled(xv[j], j < 2 ? gv[j & 1] : gs[i], inv);
      }
      for (int i = tid + XV * T; i < nv; i += T) av[i] = scaled(xs[i], gs[i], inv);
    } else {
#pragma unroll
      for (int j = 0; j < XV; ++j)
        if (tid + j * T < nv) av[tid + j * T] = xv[j];
      for (int i = tid + XV * T; i < nv; i += T) av[i] = xs[i];
    }
    __syncthreads();
  }

  f32x4 acc[NT];
#pragma unroll
  for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
  // ---- the end of a tile: add the eight waves' products, apply the epilogue.
  // acc[t][e]: weight row 4 kg + e of MFMA tile t, activation row lane % 16
  auto finish = [&](int tile_no, float* red) {
    if (row < M) {
#pragma unroll
      for (int t = 0; t < NT; ++t) *reinterpret_cast<f32x4*>(red + ((wave * NT + t) * M + row) * GV_RS + 4 * kg) = acc[t];
    }
#pragma unroll
    for (int t = 0; t < NT; ++t) acc[t] = f32x4{0.f, 0.f, 0.f, 0.f};
    __syncthreads();
    const Units q = units_of(blockIdx.x + tile_no * gridDim.x);
    auto total = [&](int m, int t, int r) {
      float s = 0.f;
  #pragma unroll
      for (int wv = 0; wv < GV_WAVES; ++wv) s += red[((wv * NT + t) * M + m) * GV_RS + r];
      return s;
    };
    for (int it = tid; it < M * q.count; it += T) {
      const int m = it / q.count, ul = it - m * q.count, t = ul >> 4, r = ul & 15;
      const int u = q.u0 + ul;
      if constexpr (EPI == EPI_QKV_ROPE) {
        const QkvEpilogue& qe = g.qe;
        const int kind = part, rc = u & 63;
        const int hc = (u >> 6) * 128 + rc;  // low column of the pair inside q / k / v
        float lo = total(m, t, r), hi = total(m, t + UT, r);
        const bf16_t* bp = reinterpret_cast<const bf16_t*>(bias);
        if (bp) {
          lo += bf16_bits_to_f32(bp[hc].bits);
          hi += bf16_bits_to_f32(bp[hc + 64].bits);
        }
        const int pos = qe.row_pos[m];
        if (kind == 2) {
          bf16_t* dst = reinterpret_cast<bf16_t*>(qe.v_cache) + (size_t)pos * qe.kv_dim + hc;
          dst[0].bits = f32_to_bf16_bits(lo);
          dst[64].bits = f32_to_bf16_bits(hi);
        } else {
          const int rp = pos - (qe.row_lo ? qe.row_lo[m] : 0);
          const float cc = qe.rope_cos[(size_t)rp * 64 + rc], ss = qe.rope_sin[(size_t)rp * 64 + rc];
          const uint16_t olo = f32_to_bf16_bits(lo * cc - hi * ss), ohi = f32_to_bf16_bits(hi * cc + lo * ss);
          bf16_t* d1 = kind == 0 ? reinterpret_cast<bf16_t*>(qe.q) + (size_t)m * qe.q_dim + hc
                                 : reinterpret_cast<bf16_t*>(qe.k_compact) + (size_t)m * qe.kv_dim + hc;
          d1[0].bits = olo;
          d1[64].bits = ohi;
          if (kind == 1) {
            bf16_t* d2 = reinterpret_cast<bf16_t*>(qe.k_cache) + (size_t)pos * qe.kv_dim + hc;
            d2[0].bits = olo;
            d2[64].bits = ohi;
          }
        }
      } else if constexpr (EPI == EPI_SWIGLU_STORE) {
        const float s0 = total(m, t, r), s1 = total(m, t + UT, r);
        reinterpret_cast<bf16_t*>(g.C)[(size_t)m * N + u].bits = f32_to_bf16_bits(s0 / (1.0f + __expf(-s0)) * s1);
      } else {
        const size_t idx = (size_t)m * N + first + u;
        const float s0 = total(m, t, r);
        if (EPI == EPI_STORE_F32)
          reinterpret_cast<float*>(g.C)[idx] = s0;
        else
          reinterpret_cast<bf16_t*>(g.C)[idx].bits = f32_to_bf16_bits(bf16_bits_to_f32(g.residual[idx].bits) + s0);
      }
    }
  };
  float* red0 = reinterpret_cast<float*>(gv_smem + g.red_offset);  // two buffers: a tile's sums are read while the next is written
  const int red_floats = GV_WAVES * NT * M * GV_RS;
  for (int ct = 0; ct < n_tiles; ++ct) {
    for (int i0 = 0; i0 < n_p; i0 += DEPTH) {
#pragma unroll
      for (int j = 0; j < DEPTH; ++j) {
        const int i = i0 + j;
        if (i < n_i) {
        bf16x8 av[MF];
#pragma unroll
        for (int c = 0; c < MF; ++c) {
          // the k a lane feeds to MFMA c: bf16 c * 32 + kg * 8 .., 4-bit kg * 32 + c * 8 .. (its 16 code bytes in order)
          if (ONE_ROW)
            av[c] = *reinterpret_cast<const bf16x8*>(act + (wave + i * GV_WAVES) * KS + (W4 ? kg * 32 + c * 8 : c * 32 + kg * 8));
          else
            av[c] = __builtin_bit_cast(bf16x8, a[j % ADEPTH][c]);
        }
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          if (W4) {
            float sc, nzs;
            w4_scale_zero(z[j][t], sc, nzs);
#pragma unroll
            for (int c = 0; c < MF; ++c) {
              uint32_t o[4];
              w4_expand8(w[j][t][0][c], sc, nzs, o);
              const u32x4 ov = {o[0], o[1], o[2], o[3]};
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, ov), av[c], acc[t], 0, 0, 0);
            }
          } else {
#pragma unroll
            for (int c = 0; c < MF; ++c)
              acc[t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, w[j][t][c % LD]), av[c], acc[t], 0, 0, 0);
          }
        }
      }
      GV_LOAD(j)
      }
    }
    finish(ct, red0 + (ct & 1) * red_floats);
  }
#undef GV_LOAD
#undef GV_RSRC
}

template <int EPI, int NT, bool ONE_ROW, bool W4>
static void launch_gemv_cfg(GemvArgs g, hipStream_t s) {
  constexpr int CAP = (EPI == EPI_SWIGLU_STORE || EPI == EPI_QKV_ROPE ? NT / 2 : NT) * 16;  // units a tile can hold
  // Two workgroups per CU are resident, 512 in all, and a workgroup streams at its own pace however many others
  // there are: a last round of 320 takes as long as one of 512.  So the units are dealt out evenly, as tiles of equal
  // size, over 512 persistent workgroups (256 where half as many rows would leave the tiles mostly empty): at
  // 5120 rows of output, K = 5120 and 13824, 19.1 us on average against 25.6 us with tiles of 16 rows.  With several
  // activation rows every workgroup reads them all from L2, so there are 256 workgroups of twice the tiles
  // (16 rows, same shapes: 26.1 us against 32.8).  QKV is not dealt out: its tiles are 8 or 16 column pairs, one per
  // workgroup, so that none straddles q, k, v or a head.  7168 rows, K = 5120: 224 workgroups of 16 pairs, 16.9 us with
  // one row (4.3 TB/s).
  const int total = EPI == EPI_QKV_ROPE ? g.N / 2 : g.N;
  const int slots = ONE_ROW && (total + 511) / 512 > CAP / 2 ? 512 : 256;
  const int rounds = (total + slots * CAP - 1) / (slots * CAP);
  g.units = std::min(CAP, (total + rounds * slots - 1) / (rounds * slots));
  if (EPI == EPI_QKV_ROPE) g.units = g.units > 8 ? 16 : 8;
  if (EPI == EPI_STORE_F32 && g.begin[1] < g.N) g.units = 16;  // several parts: no tile straddles two
  g.tiles = (total + g.units - 1) / g.units;
  const size_t red = (size_t)2 * GV_WAVES * NT * g.M * GV_RS * sizeof(float);
  g.red_offset = ONE_ROW ? (g.K * 2 + 15) / 16 * 16 : 0;
  const size_t sh = (size_t)g.red_offset + red;
  const bool parts = EPI == EPI_QKV_ROPE || (EPI == EPI_STORE_F32 && g.begin[1] < g.N);
  const int blocks = parts ? g.tiles : std::min(g.tiles, slots);
  auto kern = k_gemv<EPI, NT, ONE_ROW, W4>;
  static std::atomic<uint64_t> attr_done{0};
  set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(kern), GV_MAX_LDS);
  hipLaunchKernelGGL(kern, dim3(blocks), dim3(GV_WAVES * 64), sh, s, g);
}

template <bool ONE_ROW, bool W4>
static void launch_gemv_rows(const GemvArgs& g, int epilogue, hipStream_t s) {
  if (epilogue == EPI_QKV_ROPE)
    launch_gemv_cfg<EPI_QKV_ROPE, 2, ONE_ROW, W4>(g, s);
  else if (epilogue == EPI_SWIGLU_STORE)
    launch_gemv_cfg<EPI_SWIGLU_STORE, ONE_ROW ? 2 : 4, ONE_ROW, W4>(g, s);
  else if (epilogue == EPI_RESIDUAL_STORE)
    launch_gemv_cfg<EPI_RESIDUAL_STORE, ONE_ROW ? 1 : 2, ONE_ROW, W4>(g, s);
  else if (g.N >= 512 * 16)
    launch_gemv_cfg<EPI_STORE_F32, 2, ONE_ROW, W4>(g, s);
  else
    launch_gemv_cfg<EPI_STORE_F32, 1, ONE_ROW, W4>(g, s);
}

// Rows, K and the parts' widths k_gemv takes (32-bit offsets into a tile of weight rows bound K, beyond any model).
static bool gemv_fits(int32_t M, int32_t K, const GemmB& B) {
  if (M < 1 || M > GV_MAX_ROWS || K % 64 || (size_t)16 * K * 2 >= GV_PAST_END) return false;
  for (int p = 0; p + 1 < B.n_parts; ++p)
    if (B.n_rows[p] % 16) return false;
  return true;
}

// A single row is kept in LDS where it fits beside the partial sums (up to 64 KB of it leave room for two workgroups per
// CU); a longer one is read like several rows, by every wave for itself.
static bool gemv_row_in_lds(int32_t M, int32_t K) { return M == 1 && (size_t)K * 2 + 8192 <= (size_t)GV_MAX_LDS; }

struct SkinnyW4 {
  const uint8_t* codes[3];
  const uint32_t* sz[3];
  int32_t begin[4];  // first output column of each part; unused parts never match
};

// 17 to 40 rows on the 4-bit form.  A workgroup owns 64 weight rows (output columns) and one of S slices of K; its
// four waves take the slice's steps round-robin, add their tiles through LDS and write fp32 partials [S][M][ld].
// (Letting the workgroup that finishes a column tile last add the slices, found by a ticket counter, was measured
// and dropped: the device-wide release each workgroup then needs writes back the XCD's L2.)  A wave step covers one
// quantisation group (128 input features): the half-wave g reads the 32 code bytes of features 64 g .. 64 g + 63 of each of its two weight rows
// (two 16-byte loads per row) and one scale/zero word per row; a row tile's 32 rows are one storage block.
template <int MT>
__global__ void __launch_bounds__(256, 2)
    k_gemm_skinny_w4(const bf16_t* __restrict__ A, int M, int K, SkinnyW4 B, int n_rows_b, int n_splits,
                     float* __restrict__ part, int ld) {
  __shared__ float s_red[4][MT * 32][SK_BN + 1];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int g = lane >> 5, lq = lane & 31;
  const int n0 = blockIdx.x * SK_BN;
  const int z = blockIdx.y;
  const int steps = K / W4_GROUP;
  const int s_begin = (int)((long)z * steps / n_splits), s_end = (int)((long)(z + 1) * steps / n_splits);

  const uint8_t* cp[2];
  const uint32_t* zp[2];
#pragma unroll
  for (int ct = 0; ct < 2; ++ct) {
    const int n = min(n0 + ct * 32 + lq, n_rows_b - 1);
    int p = 0;
    if (n >= B.begin[1]) p = 1;
    if (n >= B.begin[2]) p = 2;
    // row r of the part: block row r / 32, row r % 32 inside the block; step s of the wave is block (r / 32, s)
    const size_t r = (size_t)(n - B.begin[p]);
    const size_t blk0 = (r / W4_ROWS) * (size_t)steps;
    cp[ct] = B.codes[p] + blk0 * W4_BLOCK_BYTES + (r % W4_ROWS) * (W4_GROUP / 2) + 32 * g;
    zp[ct] = B.sz[p] + blk0 * W4_ROWS + (r % W4_ROWS);
  }
  const bf16_t* ap[MT];
#pragma unroll
  for (int rt = 0; rt < MT; ++rt) ap[rt] = A + (size_t)min(rt * 32 + lq, M - 1) * K + 64 * g;

  f32x16 acc[MT][2];
#pragma unroll
  for (int rt = 0; rt < MT; ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[rt][ct][e] = 0.f;

  // Code words (the HBM stream) and, with one row tile, the activations are requested one step ahead in
  // two register buffers; with two row tiles the activations (from L2) are single-buffered and requested
  // before the next step's codes, so that waiting for them leaves the code loads in flight.
  constexpr int AB = MT == 1 ? 2 : 1;
  uint4 cw[2][2][2];   // [buffer][weight row][half of the 32 bytes]
  uint32_t zw[2][2];   // scale / zero words
  bf16x8 a[AB][MT][8];
#define W4_LOAD_B(BUF, STEP)                                                                        \
  {                                                                                                 \
    _Pragma("unroll") for (int ct = 0; ct < 2; ++ct) {                                              \
      const uint4* src_ = reinterpret_cast<const uint4*>(cp[ct] + (size_t)(STEP) * W4_BLOCK_BYTES); \
      cw[BUF][ct][0] = src_[0];                                                                     \
      cw[BUF][ct][1] = src_[1];                                                                     \
      zw[BUF][ct] = zp[ct][(size_t)(STEP) * W4_ROWS];                                               \
    }                                                                                               \
  }
#define W4_LOAD_A(BUF, STEP)                                                                        \
  {                                                                                                 \
    _Pragma("unroll") for (int rt = 0; rt < MT; ++rt) _Pragma("unroll") for (int c = 0; c < 8; ++c) \
        a[(BUF) % AB][rt][c] = *reinterpret_cast<const bf16x8*>(ap[rt] + (size_t)(STEP) * W4_GROUP + 8 * c); \
  }
#define W4_COMPUTE(BUF)                                                                             \
  {                                                                                                 \
    _Pragma("unroll") for (int ct = 0; ct < 2; ++ct) {                                              \
      float sc_, nzs_;                                                                              \
      w4_scale_zero(zw[BUF][ct], sc_, nzs_);                                                        \
      const uint32_t d_[8] = {cw[BUF][ct][0].x, cw[BUF][ct][0].y, cw[BUF][ct][0].z, cw[BUF][ct][0].w, \
                              cw[BUF][ct][1].x, cw[BUF][ct][1].y, cw[BUF][ct][1].z, cw[BUF][ct][1].w}; \
      _Pragma("unroll") for (int c = 0; c < 8; ++c) {                                               \
        uint32_t o_[4];                                                                             \
        w4_expand8(d_[c], sc_, nzs_, o_);                                                           \
        typedef uint32_t u32x4_ __attribute__((ext_vector_type(4)));                                \
        const u32x4_ ov_ = {o_[0], o_[1], o_[2], o_[3]};                                            \
        const bf16x8 b_ = __builtin_bit_cast(bf16x8, ov_);                                          \
        _Pragma("unroll") for (int rt = 0; rt < MT; ++rt) acc[rt][ct] =                             \
            __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[(BUF) % AB][rt][c], b_, acc[rt][ct], 0, 0, 0); \
      }                                                                                             \
    }                                                                                               \
  }
  // This wave's steps: s_begin + wave, + 4, ... (n_i of them).  Every request is issued unconditionally
  // (past the end the last step is requested again and never used): with no branch around the loads the
  // compiler's wait counts are exact, and a step waits for its own operands only, not for the newer requests.
  const int first = s_begin + wave;
  const int n_i = first < s_end ? (s_end - first + 3) / 4 : 0;
  if (n_i > 0) {
    const int last = first + 4 * (n_i - 1);
    int st = first;
    W4_LOAD_A(0, st)
    W4_LOAD_B(0, st)
    for (int i = 0; i < n_i; i += 2) {  // two steps per trip so that the register buffers keep fixed names
      int nx = min(st + 4, last);
      if (AB == 2) W4_LOAD_A(1, nx)
      W4_LOAD_B(1, nx)
      W4_COMPUTE(0)
      if (i + 1 >= n_i) break;
      st = nx;
      if (AB == 1) W4_LOAD_A(1, st)
      nx = min(st + 4, last);
      if (AB == 2) W4_LOAD_A(0, nx)
      W4_LOAD_B(0, nx)
      W4_COMPUTE(1)
      st = nx;
      if (AB == 1) W4_LOAD_A(0, st)
    }
  }
#undef W4_LOAD_A
#undef W4_LOAD_B
#undef W4_COMPUTE

#pragma unroll
  for (int rt = 0; rt < MT; ++rt)
#pragma unroll
    for (int ct = 0; ct < 2; ++ct)
#pragma unroll
      for (int e = 0; e < 16; ++e) s_red[wave][rt * 32 + 8 * (e >> 2) + 4 * g + (e & 3)][ct * 32 + lq] = acc[rt][ct][e];
  __syncthreads();
  float* dst = part + (size_t)z * M * ld;
  for (int i = tid; i < MT * 32 * SK_BN; i += 256) {
    const int r = i / SK_BN, cidx = i % SK_BN;
    const float v = (s_red[0][r][cidx] + s_red[1][r][cidx]) + (s_red[2][r][cidx] + s_red[3][r][cidx]);
    if (r < M && n0 + cidx < n_rows_b) dst[(size_t)r * ld + n0 + cidx] = v;
  }
}

bool gemm_skinny_fits(int32_t M, int32_t K, const GemmB& B, int32_t N, int epilogue) {
  const long rows = epilogue == EPI_SWIGLU_STORE ? 2L * N : N;
  const long ld = (rows + SK_BN - 1) / SK_BN * SK_BN;
  if (rows >= (1L << 24) || (epilogue == EPI_SWIGLU_STORE && B.n_parts != 1)) return false;
  if (epilogue == EPI_QKV_ROPE) {  // whole heads of 128 columns in every part
    if (B.n_parts != 3) return false;
    for (int p = 0; p < 3; ++p)
      if (B.n_rows[p] % 128) return false;
  }
  if (B.has_w4) {  // whole groups along K; every part a whole number of column tiles (two storage blocks)
    if (K % W4_GROUP) return false;
    for (int p = 0; p < B.n_parts; ++p)
      if (B.n_rows[p] % SK_BN) return false;
    if (epilogue == EPI_SWIGLU_STORE && N % SK_BN) return false;
  }
  // Where this kernel is the faster one, in us per layer of a unit cached on its own, all launches of a layer, at the
  // 7B / 14B / 32B shapes.  k_gemv holds up to 16 rows in one MFMA tile:
  //   bf16: what gemm_stream_fits leaves (the figures stand there).  Against the matrix-core tiles: 2 rows 124 / 137 / 207
  //   against 147 / 160 / 260, 16 rows 143 / 150 / 231 against 150 / 158 / 253.
  //   4-bit, k_gemv against k_gemm_skinny_w4: 2 rows 78 / 81 / 113 against 86 / 96 / 120, 8 rows 81 / 84 / 116 against
  //   90 / 99 / 125, 16 rows 93 / 94 / 133 against 96 / 101 / 133.
  // k_gemm_skinny_w4 goes on from there as far as the 4-bit form is read.
  if (gemv_fits(M, K, B)) return true;
  return reads_w4(B, M, K, N) && M > GV_MAX_ROWS && epilogue != EPI_QKV_ROPE && (size_t)M * (size_t)ld <= SK_MAX_PART_FLOATS;
}

bool gemm_fuses_norm(int32_t M, int32_t K, const GemmB& B, int32_t N, int epilogue, bool have_ws) {
  return have_ws && gemv_row_in_lds(M, K) && gemv_fits(M, K, B) && gemm_skinny_fits(M, K, B, N, epilogue);
}

void launch_gemm_skinny(const bf16_t* A, int32_t M, int32_t K, const GemmB& B, const void* B2, int32_t N, int epilogue,
                        const bf16_t* residual, void* C, void* ws, hipStream_t s, const QkvEpilogue* qkv,
                        const RowNorm* norm) {
  const bool swiglu = epilogue == EPI_SWIGLU_STORE;
  int begin[4], acc = 0;
  for (int p = 0; p < 3; ++p) {
    begin[p] = acc;
    if (p < B.n_parts) acc += B.n_rows[p];
  }
  begin[3] = acc;
  if (gemv_fits(M, K, B)) {
    GemvArgs g{};
    g.A = A;
    g.M = M;
    g.K = K;
    g.N = N;
    g.norm_w = norm ? reinterpret_cast<const bf16_t*>(norm->w) : nullptr;
    g.eps = norm ? norm->eps : 0.f;
    for (int p = 0; p < B.n_parts; ++p) {
      g.w[p] = B.has_w4 ? B.w4_codes[p] : B.ptr[p];
      g.sz[p] = reinterpret_cast<const uint32_t*>(B.w4_scale_zero[p]);
    }
    if (swiglu) {
      g.w[1] = B.has_w4 ? B.w4_codes_b2 : B2;
      g.sz[1] = reinterpret_cast<const uint32_t*>(B.w4_scale_zero_b2);
    }
    for (int p = 0; p < 4; ++p) g.begin[p] = begin[p];
    g.residual = residual;
    g.C = C;
    if (qkv) g.qe = *qkv;
    const bool one_row = gemv_row_in_lds(M, K);
    if (B.has_w4)
      one_row ? launch_gemv_rows<true, true>(g, epilogue, s) : launch_gemv_rows<false, true>(g, epilogue, s);
    else
      one_row ? launch_gemv_rows<true, false>(g, epilogue, s) : launch_gemv_rows<false, false>(g, epilogue, s);
    return;
  }
  // 17 to 40 rows, 4-bit form
  SkinnyW4 q{};
  for (int p = 0; p < B.n_parts; ++p) {
    q.codes[p] = reinterpret_cast<const uint8_t*>(B.w4_codes[p]);
    q.sz[p] = reinterpret_cast<const uint32_t*>(B.w4_scale_zero[p]);
  }
  for (int p = 0; p < 4; ++p) q.begin[p] = begin[p];
  if (swiglu) {  // gate rows, then up rows
    q.codes[1] = reinterpret_cast<const uint8_t*>(B.w4_codes_b2);
    q.sz[1] = reinterpret_cast<const uint32_t*>(B.w4_scale_zero_b2);
    q.begin[1] = N;
    q.begin[2] = q.begin[3] = acc = 2 * N;
  }
  const int rows = acc;
  const int tiles = (rows + SK_BN - 1) / SK_BN;
  const int ld = tiles * SK_BN;
  const int steps = K / W4_GROUP;
  // K slices: the chip holds 512 workgroups at a time (two per CU), and a count just above a multiple of 512
  // leaves most of it idle during the last round.  Among the slice counts that keep at least 4 steps per
  // workgroup and fit the workspace, take the one with the least estimated time, in bytes at the streaming
  // rate: per round of 512 workgroups their share of the weight bytes plus a fixed cost (a round's start-up
  // and its reduction through LDS, ~2 us), plus the partials written and read back.
  int smax = std::max(1, steps / 4);
  smax = (int)std::min<long>(smax, (long)(SK_MAX_PART_FLOATS / ((size_t)M * ld)));
  smax = std::max(1, std::min(smax, 64));
  const double w_bytes = (double)rows * K * 0.53;
  int splits = 1;
  double best = 0.0;
  for (int sp = 1; sp <= smax; ++sp) {
    const long wgs = (long)tiles * sp;
    const double est = (double)((wgs + 511) / 512) * (512.0 * (w_bytes / wgs) + 9.0e6) + 2.0 * M * (double)ld * sp * 4.0;
    if (sp == 1 || est < best) {
      best = est;
      splits = sp;
    }
  }
  float* part = reinterpret_cast<float*>(ws);
  const dim3 grid(tiles, splits);
  SkinnyEpi e;
  e.epilogue = epilogue;
  e.N = N;
  e.residual = residual;
  e.C = C;
  if (M <= 32)
    hipLaunchKernelGGL(k_gemm_skinny_w4<1>, grid, dim3(256), 0, s, A, M, K, q, rows, splits, part, ld);
  else
    hipLaunchKernelGGL(k_gemm_skinny_w4<2>, grid, dim3(256), 0, s, A, M, K, q, rows, splits, part, ld);
  const dim3 fgrid((N + 255) / 256, M);
  hipLaunchKernelGGL(k_skinny_finish, fgrid, dim3(256), 0, s, part, splits, ld, M, e);
}

}  // namespace keep
