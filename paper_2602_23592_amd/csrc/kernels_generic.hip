// Generic (fp32-accumulate) kernels: the kernel family used for fp32
// storage and for shapes the bf16 MFMA kernels do not take.  LDS-tiled GEMM, flash-style
// attention and per-row group scores on the fp32 matrix instruction.
#include "keep_internal.h"

namespace keep {

// ---------------------------------------------------------------------------
// C[M,N] = A[M,K] . W[N,K]^T, 64x64 tile, 16-deep K slices, 4x4 outputs per thread
// ---------------------------------------------------------------------------
struct BRows {
  const void* ptr[3];
  int32_t begin[4];  // first global column of each part, begin[n_parts] = N
  int32_t n_parts;
};

template <typename T, int EPI>
__global__ void __launch_bounds__(256)
    k_gemm_generic(const T* __restrict__ A, int M, int K, BRows B, const T* __restrict__ B2, int N,
                   const T* __restrict__ residual, void* __restrict__ Cv) {
  constexpr int BM = 64, BN = 64, BK = 16;
  __shared__ float As[BK][BM + 1];
  __shared__ float Bs[BK][BN + 1];
  __shared__ float Bs2[EPI == EPI_SWIGLU_STORE ? BK : 1][BN + 1];
  const int tid = threadIdx.x;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BN;
  const int lrow = tid >> 2, lk = (tid & 3) * 4;  // 64 rows x 4 chunks of 4 k
  const int tx = tid & 15, ty = tid >> 4;         // 16 x 16 threads, 4x4 outputs each
  float acc[4][4] = {}, acc2[4][4] = {};

  // resolve this thread's B row once
  const int bn = n0 + lrow;
  const T* brow = nullptr;
  if (bn < N) {
    const void* base = B.ptr[0];
    int first = 0;
    if (B.n_parts > 1 && bn >= B.begin[1]) {
      base = B.ptr[1];
      first = B.begin[1];
    }
    if (B.n_parts > 2 && bn >= B.begin[2]) {
      base = B.ptr[2];
      first = B.begin[2];
    }
    brow = reinterpret_cast<const T*>(base) + (size_t)(bn - first) * K;
  }
  const T* brow2 = (EPI == EPI_SWIGLU_STORE && bn < N) ? B2 + (size_t)bn * K : nullptr;
  const int am = m0 + lrow;
  const T* arow = am < M ? A + (size_t)am * K : nullptr;

  for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int k = k0 + lk + e;
      As[lk + e][lrow] = (arow && k < K) ? ldf(arow + k) : 0.f;
      Bs[lk + e][lrow] = (brow && k < K) ? ldf(brow + k) : 0.f;
      if (EPI == EPI_SWIGLU_STORE) Bs2[lk + e][lrow] = (brow2 && k < K) ? ldf(brow2 + k) : 0.f;
    }
    __syncthreads();
#pragma unroll
    for (int kk = 0; kk < BK; ++kk) {
      float a[4], b[4], b2[4];
#pragma unroll
      for (int i = 0; i < 4; ++i) a[i] = As[kk][ty * 4 + i];
#pragma unroll
      for (int j = 0; j < 4; ++j) b[j] = Bs[kk][tx * 4 + j];
      if (EPI == EPI_SWIGLU_STORE) {
#pragma unroll
        for (int j = 0; j < 4; ++j) b2[j] = Bs2[kk][tx * 4 + j];
      }
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          acc[i][j] += a[i] * b[j];
          if (EPI == EPI_SWIGLU_STORE) acc2[i][j] += a[i] * b2[j];
        }
    }
    __syncthreads();
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int m = m0 + ty * 4 + i;
    if (m >= M) continue;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const int n = n0 + tx * 4 + j;
      if (n >= N) continue;
      const size_t idx = (size_t)m * N + n;
      if (EPI == EPI_STORE_F32) {
        reinterpret_cast<float*>(Cv)[idx] = acc[i][j];
      } else if (EPI == EPI_RESIDUAL_STORE) {
        stf(reinterpret_cast<T*>(Cv) + idx, ldf(residual + idx) + acc[i][j]);
      } else {
        const float g = acc[i][j];
        stf(reinterpret_cast<T*>(Cv) + idx, g / (1.0f + expf(-g)) * acc2[i][j]);
      }
    }
  }
}

// ---------------------------------------------------------------------------
// The same product for fp32 storage on v_mfma_f32_16x16x4_f32 (fp32 operands and accumulation).
//
// Small fp32 models are bound by latency: few tiles, each a chain of K slabs.  So a slab is 64 deep, the next one is
// on its way to registers (16-byte loads) while the present one is multiplied from LDS, and tiles are 32x32 unless
// 64x64 ones fill the chip twice.  A lane's 16-byte LDS read holds k = 4 (lane / 16) .. + 3 of its row, one element
// per MFMA: both operands permute k alike.  Rows are padded to 68 floats, so the 16 lanes of a read cover all banks.
// The 2-layer, 256-wide fp32 prefill of 1088 tokens spent 576 us in the scalar kernel's products and spends 60 in these.
// Its caches' error against 64 bits is unchanged (3.0e-7 and 3.4e-7 in the 2-norm at the two layers, with either kernel).
// ---------------------------------------------------------------------------
typedef __attribute__((ext_vector_type(4))) float f32x4;

template <int MI, int EPI>
__global__ void __launch_bounds__(256)
    k_gemm_f32(const float* __restrict__ A, int M, int K, BRows B, const float* __restrict__ B2, int N,
               const float* __restrict__ residual, float* __restrict__ C) {
  constexpr int BM = 32 * MI, BK = 64, LD = BK + 4;
  constexpr int NB = EPI == EPI_SWIGLU_STORE ? 2 : 1;  // weight matrices
  __shared__ __attribute__((aligned(16))) float As[BM][LD];
  __shared__ __attribute__((aligned(16))) float Bs[NB][BM][LD];
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  const int wm = wave >> 1, wn = wave & 1;
  const int m0 = blockIdx.y * BM, n0 = blockIdx.x * BM;
  // staging: 16 threads per row, rows tid / 16 + 16 i
  constexpr int LPT = BM / 16;
  const int sr = tid >> 4, sk = (tid & 15) * 4;
  const float* ap[LPT];
  const float* bp[NB][LPT];
#pragma unroll
  for (int i = 0; i < LPT; ++i) {
    const int m = m0 + sr + 16 * i, n = n0 + sr + 16 * i;
    ap[i] = m < M ? A + (size_t)m * K : nullptr;
    const void* base = B.ptr[0];
    int first = 0;
    if (B.n_parts > 1 && n >= B.begin[1]) base = B.ptr[1], first = B.begin[1];
    if (B.n_parts > 2 && n >= B.begin[2]) base = B.ptr[2], first = B.begin[2];
    bp[0][i] = n < N ? reinterpret_cast<const float*>(base) + (size_t)(n - first) * K : nullptr;
    if (NB == 2) bp[NB - 1][i] = n < N ? B2 + (size_t)n * K : nullptr;
  }
  f32x4 ra[LPT], rb[NB][LPT];
  auto fetch = [&](int k0) {
    const int k = k0 + sk;
    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      ra[i] = ap[i] && k < K ? *reinterpret_cast<const f32x4*>(ap[i] + k) : zero;
#pragma unroll
      for (int b = 0; b < NB; ++b) rb[b][i] = bp[b][i] && k < K ? *reinterpret_cast<const f32x4*>(bp[b][i] + k) : zero;
    }
  };
  f32x4 acc[NB][MI][MI];
#pragma unroll
  for (int b = 0; b < NB; ++b)
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < MI; ++j) acc[b][i][j] = f32x4{0.f, 0.f, 0.f, 0.f};
  const int row = lane & 15, kg = lane >> 4;
  fetch(0);
  for (int k0 = 0; k0 < K; k0 += BK) {
#pragma unroll
    for (int i = 0; i < LPT; ++i) {
      *reinterpret_cast<f32x4*>(&As[sr + 16 * i][sk]) = ra[i];
#pragma unroll
      for (int b = 0; b < NB; ++b) *reinterpret_cast<f32x4*>(&Bs[b][sr + 16 * i][sk]) = rb[b][i];
    }
    __syncthreads();
    if (k0 + BK < K) fetch(k0 + BK);
#pragma unroll
    for (int c = 0; c < BK / 16; ++c) {
      f32x4 a[MI], w[NB][MI];
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        a[i] = *reinterpret_cast<const f32x4*>(&As[(wm * MI + i) * 16 + row][c * 16 + kg * 4]);
#pragma unroll
        for (int b = 0; b < NB; ++b)
          w[b][i] = *reinterpret_cast<const f32x4*>(&Bs[b][(wn * MI + i) * 16 + row][c * 16 + kg * 4]);
      }
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int b = 0; b < NB; ++b)
#pragma unroll
          for (int i = 0; i < MI; ++i)
#pragma unroll
            for (int j = 0; j < MI; ++j)
              acc[b][i][j] = __builtin_amdgcn_mfma_f32_16x16x4f32(a[i][e], w[b][j][e], acc[b][i][j], 0, 0, 0);
    }
    __syncthreads();
  }
  // acc[..][i][j][e]: row 4 (lane / 16) + e, column lane % 16 of the 16x16 tile
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int m = m0 + (wm * MI + i) * 16 + 4 * kg + e;
      if (m >= M) continue;
#pragma unroll
      for (int j = 0; j < MI; ++j) {
        const int n = n0 + (wn * MI + j) * 16 + row;
        if (n >= N) continue;
        const size_t idx = (size_t)m * N + n;
        const float v = acc[0][i][j][e];
        if (EPI == EPI_STORE_F32)
          C[idx] = v;
        else if (EPI == EPI_RESIDUAL_STORE)
          C[idx] = residual[idx] + v;
        else
          C[idx] = v / (1.0f + expf(-v)) * acc[NB - 1][i][j][e];
      }
    }
}

template <int EPI>
static void launch_gemm_f32(const float* A, int M, int K, const BRows& br, const float* B2, int N, const float* residual,
                            float* C, hipStream_t s) {
  const long tiles64 = (long)((M + 63) / 64) * ((N + 63) / 64);
  if (tiles64 >= 512)
    hipLaunchKernelGGL((k_gemm_f32<2, EPI>), dim3((N + 63) / 64, (M + 63) / 64), dim3(256), 0, s, A, M, K, br, B2, N,
                       residual, C);
  else
    hipLaunchKernelGGL((k_gemm_f32<1, EPI>), dim3((N + 31) / 32, (M + 31) / 32), dim3(256), 0, s, A, M, K, br, B2, N,
                       residual, C);
}

template <typename T>
void launch_gemm_generic(const T* A, int32_t M, int32_t K, const GemmB& B, const void* B2, int32_t N, int epilogue,
                         const T* residual, void* C, hipStream_t s) {
  if (M <= 0 || N <= 0) return;
  BRows br;
  br.n_parts = B.n_parts;
  int acc = 0;
  for (int p = 0; p < 3; ++p) {
    br.ptr[p] = p < B.n_parts ? B.ptr[p] : nullptr;
    br.begin[p] = acc;
    if (p < B.n_parts) acc += B.n_rows[p];
  }
  br.begin[3] = acc;
  dim3 grid((N + 63) / 64, (M + 63) / 64), block(256);
  const T* b2 = reinterpret_cast<const T*>(B2);
  if constexpr (sizeof(T) == 4) {
    // 16-byte loads along K: whole vectors, aligned rows
    uintptr_t at = reinterpret_cast<uintptr_t>(A) | reinterpret_cast<uintptr_t>(B2);
    for (int p = 0; p < B.n_parts; ++p) at |= reinterpret_cast<uintptr_t>(B.ptr[p]);
    if (K % 4 == 0 && at % 16 == 0) {
      float* c = reinterpret_cast<float*>(C);
      if (epilogue == EPI_STORE_F32)
        launch_gemm_f32<EPI_STORE_F32>(A, M, K, br, b2, N, residual, c, s);
      else if (epilogue == EPI_RESIDUAL_STORE)
        launch_gemm_f32<EPI_RESIDUAL_STORE>(A, M, K, br, b2, N, residual, c, s);
      else
        launch_gemm_f32<EPI_SWIGLU_STORE>(A, M, K, br, b2, N, residual, c, s);
      return;
    }
  }
  switch (epilogue) {
    case EPI_STORE_F32:
      hipLaunchKernelGGL((k_gemm_generic<T, EPI_STORE_F32>), grid, block, 0, s, A, M, K, br, b2, N, residual, C);
      break;
    case EPI_RESIDUAL_STORE:
      hipLaunchKernelGGL((k_gemm_generic<T, EPI_RESIDUAL_STORE>), grid, block, 0, s, A, M, K, br, b2, N, residual, C);
      break;
    default:
      hipLaunchKernelGGL((k_gemm_generic<T, EPI_SWIGLU_STORE>), grid, block, 0, s, A, M, K, br, b2, N, residual, C);
      break;
  }
}

// Four consecutive elements of a head as floats (16 or 8 bytes).
__device__ __forceinline__ f32x4 ld4(const float* p) { return *reinterpret_cast<const f32x4*>(p); }
__device__ __forceinline__ f32x4 ld4(const bf16_t* p) {
  const uint2 u = *reinterpret_cast<const uint2*>(p);
  return f32x4{__uint_as_float(u.x << 16), __uint_as_float(u.x & 0xffff0000u), __uint_as_float(u.y << 16),
               __uint_as_float(u.y & 0xffff0000u)};
}

// A head of NT * 16 elements as an operand of v_mfma_f32_16x16x4_f32: the lane's row is lane % 16, and it holds the
// elements 16 c + 4 (lane / 16) .. + 3 of it, one per MFMA.  (Both operands permute the dot's elements alike.)
template <int NT, typename T>
__device__ __forceinline__ void load_head(const T* row, int kg, f32x4 (&v)[NT]) {
#pragma unroll
  for (int c = 0; c < NT; ++c) v[c] = ld4(row + 16 * c + 4 * kg);
}
// 16 x 16 dots: the lane gets those of A's rows 4 (lane / 16) .. + 3 with B's row lane % 16
template <int NT>
__device__ __forceinline__ f32x4 dots(const f32x4 (&a)[NT], const f32x4 (&b)[NT]) {
  f32x4 d = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int c = 0; c < NT; ++c)
#pragma unroll
    for (int e = 0; e < 4; ++e) d = __builtin_amdgcn_mfma_f32_16x16x4f32(a[c][e], b[c][e], d, 0, 0, 0);
  return d;
}

// ---------------------------------------------------------------------------
// Attention of the recomputed rows over the cache rows 0..p in fp32 (online softmax).
//
// Bound by latency at the sizes this family serves, so the keys of one item are spread over eight waves: a workgroup
// owns one KV head and 16 query rows (a recomputed row paired with one of the KV head's query heads), each wave takes
// every eighth tile of 16 keys, and the waves' maxima, sums and outputs are joined through LDS in wave order
// (reproducible).  Scores are formed transposed, S^T = K . Q^T, so that the lane owns a query row and its four
// probabilities are, as they stand, the operand of O^T += V^T . P^T.  Operands come straight from the cache: a K row's
// 64 bytes are one request of four lanes, and the next tile's K is requested before the present one is used.  Of a V row a
// lane reads four consecutive elements, one for each of four products: acc[4 g + u] holds in element e the output dimension
// 64 g + 16 (lane / 16) + 4 e + u (what is left of the width in tiles of 16: 16 c + 4 (lane / 16) + e).
// 2-layer, 4-head, 64-wide fp32 prefill of 1088 tokens (1088 and 320 rows): 24 us per layer on average against 84 with a
// workgroup per (row, head) and a key per thread, which read the cache once per query row.  One row over 20 000 keys, two KV
// heads of 256: 1.0 ms (4.5 ms with an element of V per load, each waited for in front of its product: a tile then costs as
// many round trips as loads).
// ---------------------------------------------------------------------------
constexpr int AG_WAVES = 8;

template <typename T, int NT>
__global__ void __launch_bounds__(AG_WAVES * 64)
    k_attn_generic(const T* __restrict__ q, const T* __restrict__ k_cache, const T* __restrict__ v_cache,
                   const int32_t* __restrict__ row_pos, const int32_t* __restrict__ row_lo, int n_rows, int n_q_heads,
                   int n_kv_heads, T* __restrict__ o, float* __restrict__ lse) {
  constexpr int DH = NT * 16, LD = DH + 4;
  constexpr bool AHEAD = NT <= 8;  // (wider heads leave no registers for a second tile, nor for K and V at once)
  extern __shared__ __attribute__((aligned(16))) float ag_smem[];  // [wave][16][LD]: outputs, then max and sum
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int lq = lane & 15, kg = lane >> 4;
  const int rep = n_q_heads / n_kv_heads, hk = blockIdx.y, kv_dim = n_kv_heads * DH;
  const int x = min((int)blockIdx.x * 16 + lq, n_rows * rep - 1);  // this lane's query row (past the end: the last again)
  const int r = x / rep, head = hk * rep + x % rep;
  const int pos = row_pos[r], lo = row_lo ? row_lo[r] : 0;  // (lo: a unit cached on its own sees only itself)
  int last = pos, first = lo, all_from = lo, all_to = pos;  // keys some row sees, keys every row sees
#pragma unroll
  for (int off = 8; off > 0; off >>= 1) {
    last = max(last, __shfl_xor(last, off, 64));
    first = min(first, __shfl_xor(first, off, 64));
    all_from = max(all_from, __shfl_xor(all_from, off, 64));
    all_to = min(all_to, __shfl_xor(all_to, off, 64));
  }
  const int n_tiles = (last + 1 - first + 15) / 16;
  const float scale = 1.0f / sqrtf((float)DH);
  f32x4 qf[NT], kf[NT], kn[AHEAD ? NT : 1], acc[NT];
  load_head<NT>(q + ((size_t)r * n_q_heads + head) * DH, kg, qf);
#pragma unroll
  for (int c = 0; c < NT; ++c) acc[c] = f32x4{0.f, 0.f, 0.f, 0.f};
  const T* kh = k_cache + hk * DH;
  const T* vh = v_cache + hk * DH;
  auto k_row = [&](int t) { return kh + (size_t)min(first + t * 16 + lq, last) * kv_dim; };
  if (AHEAD && wave < n_tiles) load_head<NT>(k_row(wave), kg, kf);
  float m_run = -INFINITY, l_run = 0.f;
  for (int t = wave; t < n_tiles; t += AG_WAVES) {
    const int key0 = first + t * 16 + 4 * kg;  // the lane's four keys
    f32x4 v[4][(NT + 3) / 4];
    auto load_v = [&]() {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const T* vr = vh + (size_t)min(key0 + e, last) * kv_dim;
#pragma unroll
        for (int g = 0; g < NT / 4; ++g) v[e][g] = ld4(vr + 64 * g + 4 * lq);
#pragma unroll
        for (int c = NT / 4 * 4; c < NT; ++c) v[e][c / 4][c % 4] = ldf(vr + 16 * c + lq);
      }
      __builtin_amdgcn_sched_barrier(0);  // (the loads go out together, not each in front of its product)
    };
    if constexpr (AHEAD) {
      load_v();
      load_head<NT>(k_row(min(t + AG_WAVES, n_tiles - 1)), kg, kn);
    } else {
      load_head<NT>(k_row(t), kg, kf);
    }
    f32x4 s = dots<NT>(kf, qf);
    if constexpr (!AHEAD) load_v();
    float tmax = -INFINITY;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      s[e] = key0 + e <= pos && key0 + e >= lo ? s[e] * scale : -INFINITY;
      tmax = fmaxf(tmax, s[e]);
    }
    tmax = fmaxf(tmax, __shfl_xor(tmax, 16, 64));
    tmax = fmaxf(tmax, __shfl_xor(tmax, 32, 64));
    const float m_new = fmaxf(m_run, tmax);
    const float base = m_new == -INFINITY ? 0.f : m_new;  // (nothing visible yet: all weights zero)
    const float alpha = m_run == m_new ? 1.f : expf(m_run - base);
    float psum = 0.f;
    f32x4 p;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      p[e] = expf(s[e] - base);
      psum += p[e];
    }
    l_run = l_run * alpha + psum;
    m_run = m_new;
#pragma unroll
    for (int c = 0; c < NT; ++c) acc[c] *= alpha;
    // A weight of zero does not hide an infinity or NaN from a row that does not see its key, so where rows differ in what
    // they see such values stay out of the products and are added for the rows that see them.
    const int tile0 = __builtin_amdgcn_readfirstlane(first + t * 16);
    bool not_finite = false;
    if (tile0 < __builtin_amdgcn_readfirstlane(all_from) || tile0 + 15 > __builtin_amdgcn_readfirstlane(all_to)) {
#pragma unroll
      for (int e = 0; e < 4; ++e)
#pragma unroll
        for (int c = 0; c < NT; ++c) {
          const float x = v[e][c / 4][c % 4];
          const bool finite = fabsf(x) < INFINITY;
          not_finite |= !finite;
          v[e][c / 4][c % 4] = finite ? x : 0.f;
        }
    }
#pragma unroll
    for (int e = 0; e < 4; ++e)
#pragma unroll
      for (int c = 0; c < NT; ++c)
        acc[c] = __builtin_amdgcn_mfma_f32_16x16x4f32(v[e][c / 4][c % 4], p[e], acc[c], 0, 0, 0);
    if (__any(not_finite)) {
#pragma unroll 1
      for (int g = 0; g < 4; ++g)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          const float w = __shfl(p[e], g * 16 + lq, 64);
          const int key = tile0 + 4 * g + e;
          if (key < lo || key > pos) continue;
          const T* vr = vh + (size_t)key * kv_dim;
#pragma unroll
          for (int c = 0; c < NT; ++c)
#pragma unroll
            for (int i = 0; i < 4; ++i) {
              const float x = ldf(vr + (c < NT / 4 * 4 ? c / 4 * 64 + 16 * kg + 4 * i + c % 4 : 16 * c + 4 * kg + i));
              if (!(fabsf(x) < INFINITY)) acc[c][i] += w * x;
            }
        }
    }
    if constexpr (AHEAD) {
#pragma unroll
      for (int c = 0; c < NT; ++c) kf[c] = kn[c];
    }
  }
  l_run += __shfl_xor(l_run, 16, 64);
  l_run += __shfl_xor(l_run, 32, 64);
  float* mine = ag_smem + (wave * 16 + lq) * LD;
#pragma unroll
  for (int g = 0; g < NT / 4; ++g)
#pragma unroll
    for (int e = 0; e < 4; ++e)
      *reinterpret_cast<f32x4*>(mine + 64 * g + 16 * kg + 4 * e) =
          f32x4{acc[4 * g][e], acc[4 * g + 1][e], acc[4 * g + 2][e], acc[4 * g + 3][e]};
#pragma unroll
  for (int c = NT / 4 * 4; c < NT; ++c) *reinterpret_cast<f32x4*>(mine + 16 * c + 4 * kg) = acc[c];
  if (kg == 0) {
    mine[DH] = m_run;
    mine[DH + 1] = l_run;
  }
  __syncthreads();
  for (int it = tid; it < 16 * DH; it += AG_WAVES * 64) {
    const int row = it / DH, d = it - row * DH, xr = blockIdx.x * 16 + row;
    if (xr >= n_rows * rep) break;
    float m_all = -INFINITY;
#pragma unroll
    for (int w = 0; w < AG_WAVES; ++w) m_all = fmaxf(m_all, ag_smem[(w * 16 + row) * LD + DH]);
    const float base = m_all == -INFINITY ? 0.f : m_all;
    float l_all = 0.f, v = 0.f;
#pragma unroll
    for (int w = 0; w < AG_WAVES; ++w) {
      const float* pw = ag_smem + (w * 16 + row) * LD;
      const float weight = expf(pw[DH] - base);
      l_all += pw[DH + 1] * weight;
      v += pw[d] * weight;
    }
    const size_t at = (size_t)(xr / rep) * n_q_heads + hk * rep + xr % rep;
    stf(o + at * DH + d, v / l_all);
    if (d == 0) lse[at] = m_all + logf(l_all);
  }
}

// one instance per head width (a multiple of 16, at most 256)
#define FOR_HEAD_TILES(NT_, CALL)                                                                                     \
  switch (NT_) {                                                                                                      \
    case 1: CALL(1); break;                                                                                           \
    case 2: CALL(2); break;                                                                                           \
    case 3: CALL(3); break;                                                                                           \
    case 4: CALL(4); break;                                                                                           \
    case 5: CALL(5); break;                                                                                           \
    case 6: CALL(6); break;                                                                                           \
    case 7: CALL(7); break;                                                                                           \
    case 8: CALL(8); break;                                                                                           \
    case 9: CALL(9); break;                                                                                           \
    case 10: CALL(10); break;                                                                                         \
    case 11: CALL(11); break;                                                                                         \
    case 12: CALL(12); break;                                                                                         \
    case 13: CALL(13); break;                                                                                         \
    case 14: CALL(14); break;                                                                                         \
    case 15: CALL(15); break;                                                                                         \
    default: CALL(16); break;                                                                                         \
  }

template <typename T, int NT>
static void launch_attn_cfg(const T* q, const T* k_cache, const T* v_cache, const int32_t* d_row_pos, int32_t n_rows,
                            int32_t n_q_heads, int32_t n_kv_heads, T* o, float* lse, hipStream_t s,
                            const int32_t* d_row_lo) {
  const size_t sh = (size_t)AG_WAVES * 16 * (NT * 16 + 4) * sizeof(float);  // at most 130 KB
  static std::atomic<uint64_t> attr_done{0};
  set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(k_attn_generic<T, NT>), (int)sh);
  const int tiles = (int)(((long)n_rows * (n_q_heads / n_kv_heads) + 15) / 16);
  hipLaunchKernelGGL((k_attn_generic<T, NT>), dim3(tiles, n_kv_heads), dim3(AG_WAVES * 64), sh, s, q, k_cache, v_cache,
                     d_row_pos, d_row_lo, n_rows, n_q_heads, n_kv_heads, o, lse);
}

template <typename T>
void launch_attn_generic(const T* q, const T* k_cache, const T* v_cache, const int32_t* d_row_pos, int32_t n_rows,
                         int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim, T* o, float* lse, hipStream_t s,
                         const int32_t* d_row_lo) {
  if (n_rows <= 0) return;
#define GO(NT) launch_attn_cfg<T, NT>(q, k_cache, v_cache, d_row_pos, n_rows, n_q_heads, n_kv_heads, o, lse, s, d_row_lo)
  FOR_HEAD_TILES(head_dim / 16, GO)
#undef GO
}

// ---------------------------------------------------------------------------
// attention mass of the recomputed rows towards each candidate memory
//   rowmass[t, j] = sum_h sum_{s in block j, s <= t} exp(q_t,h . k_s / sqrt(dh) - lse[t,h])
// Rows and candidate keys are both in compact (prompt) order, so causality is s <= t.
//
// A product gives the dots of 16 rows with 16 keys.  Heads times key tiles of 16 rows and a candidate block are dealt out
// evenly over the eight waves of a workgroup, in runs (a wave loads the rows' queries anew only where the head changes) with
// the next tile's keys requested ahead; the waves' sums are added in wave order.  Rows that all lie in the block itself, or
// in front of it, have nothing to do.  Bound by latency, hence the waves: 20 rows of an instruction towards one memory
// of 1500 tokens, whose own rows are not counted, 16 heads of 128 in fp32, whole call: 367 us, 1467 with one wave per block.
// Where many short blocks fill the chip, a wave takes a block alone (ALONE): see the launch.
// ---------------------------------------------------------------------------
constexpr int SG_WAVES = 8, SG_ALONE_WAVES = 4;

template <typename T, int NT, bool ALONE>
__global__ void __launch_bounds__((ALONE ? SG_ALONE_WAVES : SG_WAVES) * 64)
    k_score_rows_generic(const T* __restrict__ q, const T* __restrict__ k_compact, const float* __restrict__ lse,
                         const int32_t* __restrict__ row_start, int m, int n_rows, int n_q_heads, int n_kv_heads,
                         float* __restrict__ rowmass) {
  constexpr int DH = NT * 16;
  __shared__ float s_sum[SG_WAVES][16];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int lq = lane & 15, kg = lane >> 4;
  const int j = ALONE ? blockIdx.y * SG_ALONE_WAVES + wave : blockIdx.y, t0 = blockIdx.x * 16;
  if (ALONE && j >= m) return;
  const int rep = n_q_heads / n_kv_heads, kv_dim = n_kv_heads * DH;
  const float scale = 1.0f / sqrtf((float)DH);
  const int t = t0 + lq, tc = min(t, n_rows - 1);  // the lane's row
  const int s0 = row_start[j], s_end = row_start[j + 1];
  const int t_end = min(t0 + 16, n_rows);
  const bool own = tc >= s0 && tc < s_end;  // a memory's attention to itself does not count
  const int s1 = t0 >= s0 && t_end <= s_end ? s0 : min(s_end, t_end);  // keys some row of the tile may see
  const int seen = own ? s0 : min(s_end, tc + 1);                      // ... this row
  float sum = 0.f;
  if (s0 < s1) {
    f32x4 qf[NT], kf[NT];
    float l = 0.f;
    auto queries = [&](int h) {
      load_head<NT>(q + ((size_t)tc * n_q_heads + h) * DH, kg, qf);
      l = lse[(size_t)tc * n_q_heads + h];
    };
    auto keys = [&](int h, int c, f32x4 (&v)[NT]) {
      load_head<NT>(k_compact + (size_t)min(s0 + 16 * c + lq, s1 - 1) * kv_dim + (h / rep) * DH, kg, v);
    };
    auto add = [&](int c) {
      const f32x4 d = dots<NT>(kf, qf);
#pragma unroll
      for (int e = 0; e < 4; ++e) sum += s0 + 16 * c + 4 * kg + e < seen ? expf(d[e] * scale - l) : 0.f;
    };
    const int tiles = (s1 - s0 + 15) / 16;
    if constexpr (ALONE) {
      for (int h = 0; h < n_q_heads; ++h) {
        queries(h);
        for (int c = 0; c < tiles; ++c) {
          keys(h, c, kf);
          add(c);
        }
      }
    } else {
      const int items = n_q_heads * tiles, i_end = (int)((long)(wave + 1) * items / SG_WAVES);
      int i = (int)((long)wave * items / SG_WAVES), h = i / tiles, c = i - h * tiles, loaded = -1;
      f32x4 kn[NT];
      if (i < i_end) keys(h, c, kf);
      for (; i < i_end; ++i) {
        if (h != loaded) queries(loaded = h);
        const int at = c;
        if (++c == tiles) c = 0, ++h;
        if (i + 1 < i_end) keys(h, c, kn);
        add(at);
#pragma unroll
        for (int u = 0; u < NT; ++u) kf[u] = kn[u];
      }
    }
    sum += __shfl_xor(sum, 16, 64);
    sum += __shfl_xor(sum, 32, 64);
    if constexpr (!ALONE) {
      if (kg == 0) s_sum[wave][lq] = sum;
      __syncthreads();
      if (wave == 0) {
        sum = 0.f;
#pragma unroll
        for (int w = 0; w < SG_WAVES; ++w) sum += s_sum[w][lq];
      }
    }
  }
  if ((ALONE || wave == 0) && kg == 0 && t < n_rows) rowmass[(size_t)t * m + j] = sum;
}

template <typename T>
void launch_score_rows_generic(const T* q, const T* k_compact, const float* lse, const int32_t* d_row_start, int32_t m,
                               int32_t n_rows, int32_t n_q_heads, int32_t n_kv_heads, int32_t head_dim,
                               float* rowmass, hipStream_t s) {
  if (n_rows <= 0 || m <= 0) return;
  // Many short blocks fill the chip with one wave each, and eight waves that find little to do cost more than they save.
  // 4000 rows, 250 blocks of 16 tokens, whole call in us, one wave / eight: 8 heads of 256 1019 / 1276, 6 heads of 48
  // 185 / 210; from 32 heads times key tiles on the same (32 heads of 64: equal).
  const long pairs = (long)((n_rows + 15) / 16) * m;
  const bool alone = pairs >= 4096 && (long)n_q_heads * ((n_rows / m + 15) / 16) < 32;
  auto launch = [&](auto kern, int blocks_y, int waves) {
    hipLaunchKernelGGL(kern, dim3((n_rows + 15) / 16, blocks_y), dim3(waves * 64), 0, s, q, k_compact, lse, d_row_start, m,
                       n_rows, n_q_heads, n_kv_heads, rowmass);
  };
#define GO(NT)                                                                                                        \
  alone ? launch(k_score_rows_generic<T, NT, true>, (m + SG_ALONE_WAVES - 1) / SG_ALONE_WAVES, SG_ALONE_WAVES)        \
        : launch(k_score_rows_generic<T, NT, false>, m, SG_WAVES)
  FOR_HEAD_TILES(head_dim / 16, GO)
#undef GO
}
#undef FOR_HEAD_TILES

// S[a, b] = (sum over the rows t of block a, ascending, of rowmass[t, b]) / (heads * len_a * len_b); S[a, a] = 0
__global__ void k_score_finish(const float* __restrict__ rowmass, const int32_t* __restrict__ row_start, int m,
                               int n_q_heads, float* __restrict__ S) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  const int a = blockIdx.y;
  if (b >= m) return;
  float v = 0.f;
  if (a != b) {
    const int t0 = row_start[a], t1 = row_start[a + 1];
    float sum = 0.f;
#pragma unroll 16
    for (int t = t0; t < t1; ++t) sum += rowmass[(size_t)t * m + b];
    const float len_a = (float)(t1 - t0), len_b = (float)(row_start[b + 1] - row_start[b]);
    v = sum / ((float)n_q_heads * len_a * len_b);
  }
  S[(size_t)a * m + b] = v;
}

void launch_score_finish(const float* rowmass, const int32_t* d_row_start, int32_t m, int32_t n_q_heads, float* S,
                         hipStream_t s) {
  if (m <= 0) return;
  hipLaunchKernelGGL(k_score_finish, dim3((m + 255) / 256, m + 1), dim3(256), 0, s, rowmass, d_row_start, m, n_q_heads,
                     S);
}

#define INST(T)                                                                                                    \
  template void launch_gemm_generic<T>(const T*, int32_t, int32_t, const GemmB&, const void*, int32_t, int,       \
                                       const T*, void*, hipStream_t);                                              \
  template void launch_attn_generic<T>(const T*, const T*, const T*, const int32_t*, int32_t, int32_t, int32_t,   \
                                       int32_t, T*, float*, hipStream_t, const int32_t*);                          \
  template void launch_score_rows_generic<T>(const T*, const T*, const float*, const int32_t*, int32_t, int32_t,  \
                                             int32_t, int32_t, int32_t, float*, hipStream_t);
INST(float)
INST(bf16_t)
#undef INST

}  // namespace keep
