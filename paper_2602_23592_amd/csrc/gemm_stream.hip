// bf16 GEMM for 8 to 128 rows: C[M, N] = A[M, K] . W[N, K]^T (fp32 accumulate) with the epilogues of a layer.
//
// With so few rows the work is still reading the weights once, but every workgroup also needs all the activations, so
// what counts is that all 256 CUs stream an equal share of the weights from the first slice to the last.  The output
// columns are therefore dealt out evenly (20 columns per workgroup for 5120, 54 gate/up pairs for 13824): one workgroup
// per CU owns its columns over the WHOLE of K and finishes them itself, with no cuts along K and no pass that adds them.
// Weights and activations go global -> LDS through a ring of three to eight stages of 64 or 128 deep slices, one barrier
// per stage, so that 70 to 140 KB per CU are on their way: tiles of 128x128 with two stages had half of that, on 0.6 to
// 0.85 of the chip, and each launch a second one behind it.  The weights are the A operand of v_mfma_f32_16x16x32_bf16,
// 16 columns per tile, the activations the B operand, 16 rows per tile; a wave owns one or two of the activation tiles.
// The loads run on over the ends of a workgroup's tiles.
//
// Where the weight rows are a multiple of 4 KB apart, workgroups that walk K side by side ask the same memory channels at the
// same time, so they start at different slices and go round (us, side by side / spread; k_gemv or tiles before them): gate/up
// 4096 x 28672, 8 rows 43.3: 46.1 / 41.3, 64 rows 56.1: 47.7 / 42.7; 4096 x 22016, 8 rows 34.2: 37.4 / 33.1; 4096 x 49152, 64
// rows 100.6: 85.1 / 72.3; down 16384 x 6144, 8 rows 41.8: 48.4 / 37.2, 64 rows 47.4: 52.3 / 39.8; QKV 8192 x 10240, 64 rows
// 40.0: 47.0 / 35.7.  Other distances, O, and cuts of at most 64 columns a workgroup lose 1 to 3 % and start side by side.
//
// Where the activations of the whole of K would cost a CU more than its few columns of weights (down projections, O and QKV
// from 17 or 33 rows on), K is cut in 4 or 8: a workgroup then has 4 or 8 times the columns of one split, writes fp32 sums,
// and k_stream_add adds the splits in order and applies the epilogue.
#include <algorithm>
#include <type_traits>

#include "keep_internal.h"

namespace keep {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;

namespace {

constexpr int ST_WGS = 256;      // workgroups resident on the chip: one per CU
constexpr int ST_MAX_ROWS = 128;

struct StreamArgs {
  const bf16_t* A;
  int M, K, N;       // N: output columns
  int units, tiles;  // output columns (SwiGLU, RoPE: pairs) of a tile, and tiles
  const bf16_t* w[3];  // weight parts; SwiGLU: gate, up
  int begin[4];        // first output column of each part (SwiGLU: unused)
  const bf16_t* residual;
  void* C;
  float* part;  // cut along K: fp32 sums [splits][M][N]
  int splits;
  const bf16_t* norm_w;  // k_stream_add_norm
  float eps;
  bf16_t* norm_out;
  QkvEpilogue qe;
};

__device__ __forceinline__ constexpr int st_vmcnt(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// element offset of 16-byte chunk `chunk` of row `row` in a [rows][64] tile: 16 consecutive rows cover all banks
__device__ __forceinline__ int st_off(int row, int chunk) { return row * 64 + ((chunk ^ ((row >> 1) & 7)) << 3); }

// (One workgroup per CU: the ring leaves no LDS for another.  The widest tiles need more than half of the registers; for the
// narrower ones the bound keeps the accumulators in vector registers.)
template <int EPI, int UT, int MT, int SUB, int ST>
__global__ void __launch_bounds__(256, UT >= 14 ? 1 : 2) k_gemm_stream(StreamArgs g) {
  constexpr bool PAIRS = EPI == EPI_SWIGLU_STORE || EPI == EPI_QKV_ROPE;
  constexpr bool CUT = EPI == EPI_STORE_F32;       // one of the splits along K, one tile: fp32 sums for k_stream_add
  constexpr int UH = PAIRS ? UT / 2 : UT;          // weight tiles of 16 units
  constexpr int ROWS = (UT + MT) * 16;             // LDS rows of a slice: weights, then activations
  constexpr int SLICE = ROWS * 64, STAGE = SLICE * SUB;  // elements
  constexpr int LPS = ROWS / 8 / 4;                // loads of a wave per slice (8 rows each)
  constexpr int L = LPS * SUB;                     // ... per stage
  constexpr int AW = MT == 8 ? 2 : 1;              // activation tiles of a wave
  constexpr int KB = UT * AW <= 16 ? 2 : 1;        // 32-deep k-steps whose operands are read at once
  static_assert(ROWS % 32 == 0 && (ST - 2) * L < 64, "loads must split over the waves and fit the wait counter");
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = g.M, K = g.K, N = g.N;
  const int total = PAIRS && EPI == EPI_QKV_ROPE ? N / 2 : N;
  // Cut along K, the workgroups of an XCD (blockIdx % 8) take the same split or two: its L2 holds that part of the activations.
  const int per_split = CUT ? 8 / g.splits : 1, xcd = blockIdx.x & 7;
  const int z = CUT ? xcd / per_split : 0;
  const int wg = CUT ? (blockIdx.x >> 3) * per_split + xcd % per_split : blockIdx.x;
  if (CUT && wg >= g.tiles) return;
  const int n_all = K / (64 * SUB), it0 = CUT ? z * n_all / g.splits : 0;
  const int n_it = CUT ? (z + 1) * n_all / g.splits - it0 : n_all;
  const int n_tiles = CUT ? 1 : (g.tiles - wg + (int)gridDim.x - 1) / (int)gridDim.x;  // this workgroup's: wg, + grid, ...
  typedef const void __attribute__((address_space(1))) * gptr_t;
  typedef void __attribute__((address_space(3))) * lptr_t;

  // ---- loads: the wave's rows of a slice are (wave * LPS + i) * 8 + lane / 8; the lane fetches the chunk that the swizzle
  // keeps at its place.  Rows past the tile's last unit or past M read the last one again (no memory traffic).
  const bf16_t* src[LPS];
  auto aim = [&](int tile) {
    const int u0 = tile * g.units, count = min(g.units, total - u0);
#pragma unroll
    for (int i = 0; i < LPS; ++i) {
      const int r = (wave * LPS + i) * 8 + lane / 8, c = (lane & 7) ^ ((r >> 1) & 7);
      const bf16_t* row;
      if (r < UT * 16) {
        const int half = r / (UH * 16), u = u0 + min(r % (UH * 16), count - 1);
        if (EPI == EPI_SWIGLU_STORE) {
          row = (half ? g.w[1] : g.w[0]) + (size_t)u * K;
        } else {
          const int n = EPI == EPI_QKV_ROPE ? (u >> 6) * 128 + (u & 63) + half * 64 : u;  // RoPE pairs column c of a head with c + 64
          const bf16_t* base = g.w[0];
          int first = 0;
          if (EPI != EPI_RESIDUAL_STORE && n >= g.begin[1]) base = g.w[1], first = g.begin[1];
          if (EPI != EPI_RESIDUAL_STORE && n >= g.begin[2]) base = g.w[2], first = g.begin[2];
          row = base + (size_t)(n - first) * K;
        }
      } else {
        row = g.A + (size_t)min(r - UT * 16, M - 1) * K;
      }
      src[i] = row + c * 8 + (size_t)it0 * SUB * 64;
    }
  };
  int lt = 0, li = 0, slot = 0;  // tile, stages of it requested and place in the ring of the next stage to request
  const bool apart = K % 2048 == 0 && (CUT ? g.units > 64 : PAIRS);
  int at = !apart ? 0 : (CUT ? wg * 3 % n_it : wg * n_it / ST_WGS);  // stage along K
  auto request = [&]() {
#pragma unroll
    for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
      for (int i = 0; i < LPS; ++i)
        __builtin_amdgcn_global_load_lds((gptr_t)(src[i] + ((size_t)at * SUB + sub) * 64),
                                         (lptr_t)(smem + slot * STAGE + sub * SLICE + (wave * LPS + i) * 512), 16, 0, 0);
    slot = slot + 1 == ST ? 0 : slot + 1;
    at = at + 1 == n_it ? 0 : at + 1;
    if (++li == n_it) {
      li = 0;
      if (++lt < n_tiles) aim(wg + lt * gridDim.x);
    }
  };

  f32x4 acc[UT][AW];
  const int row16 = lane & 15, kg = lane >> 4;
  int w_off[2], a_off[2];
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    w_off[ks] = st_off(row16, ks * 4 + kg);
    a_off[ks] = st_off(UT * 16 + (wave % MT) * 16 + row16, ks * 4 + kg);
  }
  const bool works = wave < MT && (wave * 16 < M);  // (a wave without rows of its own only loads)
  // acc[t][a][e]: unit 16 t + 4 kg + e of the tile (pairs: t and t + UH), row 16 (wave + 4 a) + row16
  auto finish = [&](int tile) {
    const int u0 = tile * g.units, count = min(g.units, total - u0);
#pragma unroll
    for (int a = 0; a < AW; ++a) {
      const int m = (wave + 4 * a) * 16 + row16;
      if (m >= M) continue;
      if constexpr (CUT) {  // (four columns of a lane: N and the tiles' widths are multiples of four)
#pragma unroll
        for (int t = 0; t < UT; ++t)
          if (t * 16 + 4 * kg < count)
            *reinterpret_cast<f32x4*>(g.part + ((size_t)z * M + m) * N + u0 + t * 16 + 4 * kg) = acc[t][a];
        continue;
      }
      int pos = 0, rp = 0;
      if (EPI == EPI_QKV_ROPE) {
        pos = g.qe.row_pos[m];
        rp = pos - (g.qe.row_lo ? g.qe.row_lo[m] : 0);
      }
#pragma unroll
      for (int t = 0; t < UH; ++t)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const int ul = t * 16 + 4 * kg + e;
          if (ul >= count) continue;
          const int u = u0 + ul;
          if constexpr (EPI == EPI_QKV_ROPE) {
            const QkvEpilogue& qe = g.qe;
            float lo = acc[t][a][e], hi = acc[t + UH][a][e];
            const int rc = u & 63, n = (u >> 6) * 128 + rc;
            const int kind = n >= g.begin[2] ? 2 : (n >= g.begin[1] ? 1 : 0);
            const int hc = n - (kind == 2 ? g.begin[2] : (kind == 1 ? g.begin[1] : 0));
            const bf16_t* bp = reinterpret_cast<const bf16_t*>(kind == 2 ? qe.bias[2] : (kind == 1 ? qe.bias[1] : qe.bias[0]));
            if (bp) {
              lo += bf16_bits_to_f32(bp[hc].bits);
              hi += bf16_bits_to_f32(bp[hc + 64].bits);
            }
            if (kind == 2) {
              bf16_t* dst = reinterpret_cast<bf16_t*>(qe.v_cache) + (size_t)pos * qe.kv_dim + hc;
              dst[0].bits = f32_to_bf16_bits(lo);
              dst[64].bits = f32_to_bf16_bits(hi);
            } else {
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
            const float s0 = acc[t][a][e];
            reinterpret_cast<bf16_t*>(g.C)[(size_t)m * N + u].bits =
                f32_to_bf16_bits(s0 / (1.0f + __expf(-s0)) * acc[t + UH][a][e]);
          } else if constexpr (EPI == EPI_RESIDUAL_STORE) {
            const size_t idx = (size_t)m * N + u;
            reinterpret_cast<bf16_t*>(g.C)[idx].bits = f32_to_bf16_bits(bf16_bits_to_f32(g.residual[idx].bits) + acc[t][a][e]);
          }
        }
    }
  };
  auto clear = [&]() {
#pragma unroll
    for (int t = 0; t < UT; ++t)
#pragma unroll
      for (int a = 0; a < AW; ++a) acc[t][a] = f32x4{0.f, 0.f, 0.f, 0.f};
  };
  int cs = 0;  // ring place of the stage in hand
  auto compute = [&]() {
    if (works) {
      const uint16_t* base = smem + cs * STAGE;
#pragma unroll
      for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
        for (int k0 = 0; k0 < 2; k0 += KB) {
          bf16x8 x[KB][AW], w[KB][UT];
#pragma unroll
          for (int ks = 0; ks < KB; ++ks) {
#pragma unroll
            for (int a = 0; a < AW; ++a)
              x[ks][a] = *reinterpret_cast<const bf16x8*>(base + sub * SLICE + a_off[k0 + ks] + a * 64 * 64);
#pragma unroll
            for (int t = 0; t < UT; ++t)
              w[ks][t] = *reinterpret_cast<const bf16x8*>(base + sub * SLICE + w_off[k0 + ks] + t * 16 * 64);
          }
#pragma unroll
          for (int ks = 0; ks < KB; ++ks)
#pragma unroll
            for (int t = 0; t < UT; ++t)
#pragma unroll
              for (int a = 0; a < AW; ++a)
                acc[t][a] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w[ks][t], x[ks][a], acc[t][a], 0, 0, 0);
        }
      // (one wave per SIMD: reads first, or the compiler pairs every read with a wait)
#pragma unroll
      for (int b = 0; b < SUB * 2 / KB; ++b) {
        __builtin_amdgcn_sched_group_barrier(0x100, KB * (AW + UT), 0);
        if (KB == 1 || b + 1 == SUB * 2 / KB) __builtin_amdgcn_sched_group_barrier(0x008, KB == 1 ? UT * AW : 2 * SUB * UT * AW, 0);
      }
    }
    cs = cs + 1 == ST ? 0 : cs + 1;
  };

  // All stages of all its tiles are one sequence, requested ST - 1 ahead.  A barrier shows that every wave's loads of the
  // stage in hand have landed and that every wave is done with the one before, whose place is requested next.
  const int n_seq = n_tiles * n_it;
  int seq = 0, ct = 0, ci = 0;
  aim(wg);
  clear();
  for (int s = 0; s < ST - 1; ++s) request();
  auto step = [&]() {
    compute();
    ++seq;
    if (++ci == n_it) {
      if (works) finish(wg + ct * gridDim.x);
      clear();
      ci = 0;
      ++ct;
    }
  };
  while (seq + ST - 1 < n_seq) {
    __builtin_amdgcn_s_waitcnt(st_vmcnt((ST - 2) * L));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    request();
    step();
    __builtin_amdgcn_sched_barrier(0);
  }
  auto last = [&](auto self, auto left) -> void {  // the last ST - 1 stages are all on their way
    __builtin_amdgcn_s_waitcnt(st_vmcnt((decltype(left)::value - 1) * L));
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    asm volatile("" ::: "memory");
    step();
    __builtin_amdgcn_sched_barrier(0);
    if constexpr (decltype(left)::value > 1) self(self, std::integral_constant<int, decltype(left)::value - 1>{});
  };
  last(last, std::integral_constant<int, ST - 1>{});
}

// Adds the splits, in order, and applies the epilogue.  A thread owns four columns of a row, with RoPE four of the low half
// of a head and their partners.
template <int EPI, int S>
__global__ void __launch_bounds__(256) k_stream_add(StreamArgs g) {
  const int M = g.M, N = g.N;
  const int per_row = EPI == EPI_QKV_ROPE ? N / 8 : N / 4;
  const int i = blockIdx.x * 256 + threadIdx.x;
  if (i >= M * per_row) return;
  const int m = i / per_row, c4 = i - m * per_row;
  const size_t step = (size_t)M * N;
  if constexpr (EPI == EPI_RESIDUAL_STORE) {
    const size_t idx = (size_t)m * N + c4 * 4;
    f32x4 v[S];
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = *reinterpret_cast<const f32x4*>(g.part + z * step + idx);
    const uint2 r = *reinterpret_cast<const uint2*>(g.residual + idx);
#pragma unroll
    for (int z = 1; z < S; ++z) v[0] += v[z];
    uint2 o;
    o.x = pack_bf16x2(bf16_bits_to_f32((uint16_t)(r.x & 0xffff)) + v[0][0], bf16_bits_to_f32((uint16_t)(r.x >> 16)) + v[0][1]);
    o.y = pack_bf16x2(bf16_bits_to_f32((uint16_t)(r.y & 0xffff)) + v[0][2], bf16_bits_to_f32((uint16_t)(r.y >> 16)) + v[0][3]);
    *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(g.C) + idx) = o;
  } else {
    const QkvEpilogue& qe = g.qe;
    const int rc = (c4 & 15) * 4, n = (c4 >> 4) * 128 + rc;
    const int kind = n >= g.begin[2] ? 2 : (n >= g.begin[1] ? 1 : 0);
    const int hc = n - (kind == 2 ? g.begin[2] : (kind == 1 ? g.begin[1] : 0));
    const float* p = g.part + (size_t)m * N + n;
    f32x4 lo[S], hi[S];
#pragma unroll
    for (int z = 0; z < S; ++z) {
      lo[z] = *reinterpret_cast<const f32x4*>(p + z * step);
      hi[z] = *reinterpret_cast<const f32x4*>(p + z * step + 64);
    }
    const int pos = qe.row_pos[m], rp = pos - (qe.row_lo ? qe.row_lo[m] : 0);
#pragma unroll
    for (int z = 1; z < S; ++z) lo[0] += lo[z], hi[0] += hi[z];
    const bf16_t* bp = reinterpret_cast<const bf16_t*>(kind == 2 ? qe.bias[2] : (kind == 1 ? qe.bias[1] : qe.bias[0]));
    if (bp) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        lo[0][e] += bf16_bits_to_f32(bp[hc + e].bits);
        hi[0][e] += bf16_bits_to_f32(bp[hc + 64 + e].bits);
      }
    }
    f32x4 ol = lo[0], oh = hi[0];
    if (kind != 2) {
      const f32x4 cc = *reinterpret_cast<const f32x4*>(qe.rope_cos + (size_t)rp * 64 + rc);
      const f32x4 ss = *reinterpret_cast<const f32x4*>(qe.rope_sin + (size_t)rp * 64 + rc);
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        ol[e] = lo[0][e] * cc[e] - hi[0][e] * ss[e];
        oh[e] = hi[0][e] * cc[e] + lo[0][e] * ss[e];
      }
    }
    uint2 l, h;
    l.x = pack_bf16x2(ol[0], ol[1]), l.y = pack_bf16x2(ol[2], ol[3]);
    h.x = pack_bf16x2(oh[0], oh[1]), h.y = pack_bf16x2(oh[2], oh[3]);
    auto put = [&](void* base, size_t row, int dim) {
      bf16_t* dst = reinterpret_cast<bf16_t*>(base) + row * dim + hc;
      *reinterpret_cast<uint2*>(dst) = l;
      *reinterpret_cast<uint2*>(dst + 64) = h;
    };
    if (kind == 0) put(qe.q, m, qe.q_dim);
    if (kind == 1) put(qe.k_compact, m, qe.kv_dim);
    if (kind == 1) put(qe.k_cache, pos, qe.kv_dim);
    if (kind == 2) put(qe.v_cache, pos, qe.kv_dim);
  }
}

// The same with a residual and the RMSNorm of the finished rows behind it, a workgroup per row: one launch for two (64 rows of
// 5120: 4.0 + 4.5 us before, 4.8 now).  The row's squares are added as k_rmsnorm adds them, so the outputs are the same.
constexpr int ADD_THREADS = 1024;
template <int S>
__global__ void __launch_bounds__(ADD_THREADS) k_stream_add_norm(StreamArgs g) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];  // the row, rounded
  __shared__ float s_red[4];
  const int N = g.N, tid = threadIdx.x;
  const size_t row = (size_t)blockIdx.x * N, step = (size_t)g.M * N;
  for (int i = tid; i < N / 4; i += ADD_THREADS) {
    f32x4 v[S];
#pragma unroll
    for (int z = 0; z < S; ++z) v[z] = *reinterpret_cast<const f32x4*>(g.part + z * step + row + i * 4);
    const uint2 r = *reinterpret_cast<const uint2*>(g.residual + row + i * 4);
#pragma unroll
    for (int z = 1; z < S; ++z) v[0] += v[z];
    uint2 o;
    o.x = pack_bf16x2(bf16_bits_to_f32((uint16_t)(r.x & 0xffff)) + v[0][0], bf16_bits_to_f32((uint16_t)(r.x >> 16)) + v[0][1]);
    o.y = pack_bf16x2(bf16_bits_to_f32((uint16_t)(r.y & 0xffff)) + v[0][2], bf16_bits_to_f32((uint16_t)(r.y >> 16)) + v[0][3]);
    *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(g.C) + row + i * 4) = o;
    *reinterpret_cast<uint2*>(smem + i * 4) = o;
  }
  __syncthreads();
  if (tid < 256) {
    float ss = 0.f;
    for (int i = tid; i < N / 8; i += 256) {
      const uint4 u = *reinterpret_cast<const uint4*>(smem + i * 8);
      const uint32_t d[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const float a = __uint_as_float(d[e] << 16), b = __uint_as_float(d[e] & 0xffff0000u);
        ss += a * a;
        ss += b * b;
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off, 64);
    if ((tid & 63) == 0) s_red[tid >> 6] = ss;
  }
  __syncthreads();
  const float inv = 1.0f / sqrtf((s_red[0] + s_red[1] + s_red[2] + s_red[3]) / (float)N + g.eps);
  for (int i = tid; i < N / 4; i += ADD_THREADS) {
    const uint2 x = *reinterpret_cast<const uint2*>(smem + i * 4), w = *reinterpret_cast<const uint2*>(g.norm_w + i * 4);
    auto n = [&](uint32_t a, uint32_t b) {
      return pack_bf16x2(__uint_as_float(a << 16) * inv * __uint_as_float(b << 16),
                         __uint_as_float(a & 0xffff0000u) * inv * __uint_as_float(b & 0xffff0000u));
    };
    *reinterpret_cast<uint2*>(g.norm_out + row + i * 4) = uint2{n(x.x, w.x), n(x.y, w.y)};
  }
}

// columns of a workgroup where K is cut: a multiple of four
int cut_columns(int N, int splits) { return ((N * splits + ST_WGS - 1) / ST_WGS + 3) / 4 * 4; }

template <int EPI, int UT, int MT, int SUB, int ST>
void launch_stream_cfg(StreamArgs g, hipStream_t s) {
  constexpr bool PAIRS = EPI == EPI_SWIGLU_STORE || EPI == EPI_QKV_ROPE;
  constexpr int CAP = (PAIRS ? UT / 2 : UT) * 16;
  const int total = EPI == EPI_QKV_ROPE ? g.N / 2 : g.N;
  if (EPI == EPI_STORE_F32) {
    g.units = cut_columns(g.N, g.splits);
    g.tiles = (g.N + g.units - 1) / g.units;
  } else {
    const int rounds = (total + ST_WGS * CAP - 1) / (ST_WGS * CAP);
    g.units = (total + rounds * ST_WGS - 1) / (rounds * ST_WGS);
    g.tiles = (total + g.units - 1) / g.units;
  }
  constexpr int sh = ST * SUB * (UT + MT) * 16 * 64 * 2;
  static_assert(sh <= 160 * 1024, "the ring does not fit LDS");
  auto kern = k_gemm_stream<EPI, UT, MT, SUB, ST>;
  static std::atomic<uint64_t> attr_done{0};
  set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(kern), sh);
  hipLaunchKernelGGL(kern, dim3(EPI == EPI_STORE_F32 ? ST_WGS : std::min(g.tiles, ST_WGS)), dim3(256), sh, s, g);
}

template <int EPI, int UT, int MT, int SUB>
void launch_stream_ring(const StreamArgs& g, hipStream_t s) {  // as many stages as fit 144 KB, at most eight
  constexpr int FIT = 144 / (SUB * (UT + MT) * 2);
  launch_stream_cfg<EPI, UT, MT, SUB, (FIT < 8 ? FIT : 8)>(g, s);
}

template <int MT>
void launch_stream_cut(const StreamArgs& g, int epilogue, hipStream_t s) {
  const int columns = cut_columns(g.N, g.splits);
  if (columns <= 64)
    launch_stream_ring<EPI_STORE_F32, 4, MT, 1>(g, s);
  else if (columns <= 96)
    launch_stream_ring<EPI_STORE_F32, 6, MT, 1>(g, s);
  else if (columns <= 128)
    launch_stream_ring<EPI_STORE_F32, 8, MT, 1>(g, s);
  else if (columns <= 160)
    launch_stream_ring<EPI_STORE_F32, 10, MT, 1>(g, s);
  else if constexpr (MT <= 4)
    launch_stream_ring<EPI_STORE_F32, 14, MT, 1>(g, s);
  const int threads = g.M * (epilogue == EPI_QKV_ROPE ? g.N / 8 : g.N / 4);
  if (g.norm_out) {
    hipLaunchKernelGGL(g.splits == 8 ? k_stream_add_norm<8> : k_stream_add_norm<4>, dim3(g.M), dim3(ADD_THREADS), g.N * 2, s, g);
    return;
  }
  auto add = [&](void (*kern)(StreamArgs)) { hipLaunchKernelGGL(kern, dim3((threads + 255) / 256), dim3(256), 0, s, g); };
  if (epilogue == EPI_QKV_ROPE)
    add(g.splits == 8 ? k_stream_add<EPI_QKV_ROPE, 8> : k_stream_add<EPI_QKV_ROPE, 4>);
  else
    add(g.splits == 8 ? k_stream_add<EPI_RESIDUAL_STORE, 8> : k_stream_add<EPI_RESIDUAL_STORE, 4>);
}

template <int MT>
void launch_stream_rows(const StreamArgs& g, int epilogue, hipStream_t s) {
  if constexpr (MT <= 4) {  // (with more rows QKV and O are cut along K, or not here)
    if (epilogue == EPI_QKV_ROPE) return launch_stream_ring<EPI_QKV_ROPE, 2, MT, 2>(g, s);
    if (epilogue == EPI_RESIDUAL_STORE) return launch_stream_ring<EPI_RESIDUAL_STORE, 2, MT, 2>(g, s);
  }
  const int pairs = (g.N + ST_WGS - 1) / ST_WGS;  // gate/up: of a workgroup, if it takes one tile
  if (pairs <= 32)
    launch_stream_ring<EPI_SWIGLU_STORE, 4, MT, 1>(g, s);
  else if (pairs <= 64)
    launch_stream_ring<EPI_SWIGLU_STORE, 8, MT, 1>(g, s);
  else if (pairs <= 80)
    launch_stream_ring<EPI_SWIGLU_STORE, 10, MT, 1>(g, s);
  else if constexpr (MT <= 4)
    launch_stream_ring<EPI_SWIGLU_STORE, 14, MT, 1>(g, s);
  else  // (two accumulators per weight tile: 14 tiles would not fit the registers)
    launch_stream_ring<EPI_SWIGLU_STORE, 8, MT, 1>(g, s);
}

// Splits along K of a projection whose columns are too few to share the activations over: 0 (none), 4 or 8.
// Every CU reads the activations of its split, and gets about 60 bytes a nanosecond to its LDS: with 20 columns of the whole
// of K per CU that alone takes longer than the weights from HBM.  The sums cost a second launch (3 to 4 us).  Measured, us,
// without cuts (or tiles of 128x128 cut along K where those won; k_gemv up to 16 rows) / 4 splits / 8 splits:
//   down 13824 x 5120: 4 rows 26.5 / 27.4, 8 rows 28.6 / 27.2, 16 rows 32.9 / 27.1, 64 rows 32.6 / 29.4 / 30.1, 96 rows 39.4 /
//   38.6 / 34.3, 128 rows 42.5 / 39.8 / 36.4; 18944 x 3584: 8 rows 32.3 / 26.1, 16 rows 38.3 / 26.3, 64 rows 34.9 / 28.7,
//   128 rows 43.1 / 40.0 / 36.3; 27648 x 5120: 16 rows 62.7 / 51.5, 64 rows 60.9 / 57.3 / 56.2, 128 rows 73.9 / 75.8 / 65.2;
//   8192 x 2048: 16 rows 16.6 / 12.5, 64 rows 16.3 / 14.3, 96 rows 17.7 / 18.7.
//   O at 5120: 17 rows 14.2 / 14.1 / 14.6, 48 rows 17.8 / 15.1 / 16.6, 64 rows 20.0 / 16.4 / 17.8, 128 rows 25.8 / 21.0 / 22.2;
//   at 3584: 12 rows 10.1 / 9.7, 17 rows 10.3 / 9.8, 64 rows 13.7 / 12.0, 128 rows 21.4 / 15.3; at 2048: 17 rows 6.9 / 7.3, 48
//   rows 8.4 / 7.6, 128 rows 14.1 / 10.9.
//   QKV at 5120: 17 rows 16.3 / 18.3 / 19.1, 32 rows 18.1 / 18.6, 48 rows 21.1 / 20.1 / 22.1, 128 rows 30.2 / 26.7 / 30.7; at
//   3584: 32 rows 12.4 / 12.4, 48 rows 14.7 / 13.2, 128 rows 22.8 / 18.1; at 2048: 32 rows 8.8 / 8.5, 128 rows 17.2 / 13.0.
int stream_splits(int M, int K, int N, int epilogue, bool have_ws) {
  if (epilogue == EPI_SWIGLU_STORE || !have_ws || N % 8) return 0;
  if (M < (epilogue == EPI_QKV_ROPE || K < 3584 ? 33 : (K < 8192 ? 17 : 8))) return 0;
  const int splits = M > 64 && K >= 8192 ? 8 : 4;
  // (at least eight slices each, for the ring; the widest tile, whose sums still fit the registers and the workspace)
  return K >= 512 * splits && cut_columns(N, splits) <= (M > 64 ? 160 : 224) ? splits : 0;
}

}  // namespace

bool gemm_stream_fits(int32_t M, int32_t K, const GemmB& B, int32_t N, int epilogue, bool have_ws) {
  if (M > ST_MAX_ROWS || K % 128 || K < 1024) return false;  // (stages of two slices; at least eight of them)
  if (reads_w4(B, M, K, N)) return false;
  if (!parts_aligned16(B)) return false;
  // Up to 16 rows k_gemv streams as well, with every wave's activations from L2 beside its weights, us, k_gemv / this kernel:
  //   gate/up 5120 x 27648: 4 rows 49.8 / 50.4, 8 rows 51.1 / 50.5, 16 rows 54.2 / 50.6; 3584 x 37888: 8 rows 49.8 / 48.3,
  //   16 rows 53.9 / 48.3; wider ones stay with k_gemv: 8192 x 57344, 8 rows 160 / 192, 16 rows 165 / 192 (though at 5120 x 55296
  //   this kernel would win: 8 rows 99.2 / 96.8, 16 rows 108.0 / 97.2).
  //   QKV at 5120: 4 rows 16.0 / 15.5, 8 rows 17.0 / 15.6, 16 rows 18.9 / 16.2; at 3584: 8 rows 12.2 / 11.6, 16 rows 13.5 /
  //   11.8; but at 2048, 16 rows: 7.7 / 8.3.
  //   O at 5120: 12 rows 13.5 / 13.7, 16 rows 14.4 / 13.9; but 3584 x 3584, 13 rows: 10.1 / 10.2.
  const bool cut = stream_splits(M, K, N, epilogue, have_ws) != 0;
  if (!cut && M <= 16) {
    if (epilogue == EPI_SWIGLU_STORE ? M < 8 || K < 3584 || N > 80 * ST_WGS
                                     : (epilogue == EPI_QKV_ROPE ? M < 8 || K < 3584 : M < 13 || K < 5120 || N < 5120))
      return false;
  } else if (!cut && epilogue != EPI_SWIGLU_STORE && (K > 5120 || M > (K <= 4096 ? 64 : 48))) {
    // Tiles of 128x128 cut along K / this kernel without cuts, us:
    //   gate/up 5120 x 27648, 64 rows 70.8 / 57.0, 128 rows 81.1 / 72.6; 3584 x 37888 68.3 / 51.6, 80.9 / 64.5; 5120 x 55296,
    //   64 rows 131 / 102; 2048 x 16384 22.3 / 17.5, 28.9 / 21.0: always here.
    //   O and QKV at 5120: 32 rows 16.6 / 14.8 and 20.1 / 18.0, 48 rows 19.6 / 18.1 and 22.3 / 21.2, 64 rows 20.2 / 19.9 and
    //   23.2 / 24.4; at 3584, 64 rows: 16.7 / 13.7 and 17.2 / 15.6, 80 rows: 17.9 / 18.7 and 20.2 / 21.9; at 2048, 64 rows:
    //   11.8 / 8.7 and 13.3 / 10.7.
    //   Down (13824 x 5120): 32 rows 29.0 / 31.5, 64 rows 32.7 / 44.8: not here.
    return false;
  }
  if (epilogue == EPI_QKV_ROPE) {
    if (B.n_parts != 3) return false;
    for (int p = 0; p < 3; ++p)
      if (B.n_rows[p] % 128) return false;  // whole heads
    return true;
  }
  return B.n_parts == 1 && (epilogue == EPI_SWIGLU_STORE || epilogue == EPI_RESIDUAL_STORE);
}

bool gemm_norms_output(int32_t M, int32_t K, const GemmB& B, int32_t N, bool have_ws) {
  return gemm_stream_fits(M, K, B, N, EPI_RESIDUAL_STORE, have_ws) && stream_splits(M, K, N, EPI_RESIDUAL_STORE, have_ws);
}

void launch_gemm_stream(const bf16_t* A, int32_t M, int32_t K, const GemmB& B, const void* B2, int32_t N, int epilogue,
                        const bf16_t* residual, void* C, hipStream_t s, void* ws, const QkvEpilogue* qkv,
                        const RowNorm* norm, void* norm_out) {
  StreamArgs g{};
  g.A = A;
  g.M = M;
  g.K = K;
  g.N = N;
  int acc = 0;
  for (int p = 0; p < 3; ++p) {
    g.begin[p] = acc;
    if (p < B.n_parts) {
      g.w[p] = reinterpret_cast<const bf16_t*>(B.ptr[p]);
      acc += B.n_rows[p];
    }
  }
  g.begin[3] = acc;
  if (epilogue == EPI_SWIGLU_STORE) g.w[1] = reinterpret_cast<const bf16_t*>(B2);
  g.residual = residual;
  g.C = C;
  if (qkv) g.qe = *qkv;
  g.splits = stream_splits(M, K, N, epilogue, ws != nullptr);
  if (g.splits) {
    g.part = reinterpret_cast<float*>(ws);
    if (norm_out) {
      g.norm_w = reinterpret_cast<const bf16_t*>(norm->w);
      g.eps = norm->eps;
      g.norm_out = reinterpret_cast<bf16_t*>(norm_out);
    }
    if (M <= 32)
      launch_stream_cut<2>(g, epilogue, s);
    else if (M <= 64)
      launch_stream_cut<4>(g, epilogue, s);
    else
      launch_stream_cut<8>(g, epilogue, s);
    return;
  }
  if (M <= 32)
    launch_stream_rows<2>(g, epilogue, s);
  else if (M <= 64)
    launch_stream_rows<4>(g, epilogue, s);
  else
    launch_stream_rows<8>(g, epilogue, s);
}

}  // namespace keep
