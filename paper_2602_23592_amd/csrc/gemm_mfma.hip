// bf16 GEMM on the gfx950 matrix cores:  C[M,N] = A[M,K] . W[N,K]^T  (fp32 accumulate)
//
// Both operands are K-contiguous, which is the layout v_mfma_f32_16x16x32_bf16 wants:
// lane l supplies 8 consecutive k of row (l % 16), k-block (l / 16).  (Of the two bf16 shapes this one
// sustains the higher rate under the chip's power limit: a register-only loop on random operands runs at
// 2.03 PFLOP/s against 1.78 PFLOP/s for 32x32x16, and the whole kernel gains 4 %; operand bytes read from
// LDS per flop are the same for both.)  A workgroup owns a
// BM x BN tile of C (256 x 256: k_gemm_256, below, with an order of its own); K is walked in 64-deep slices staged through LDS (two buffers, one
// barrier per slice, next slice streamed global -> LDS by global_load_lds_dwordx4 while the
// current one is multiplied; operand fragments of the next step are read while a step multiplies).  LDS
// rows are 128 B; their 16-byte chunks are XOR-swizzled by the row index so that the
// 16-byte operand reads of consecutive rows spread over all banks.  Workgroups are mapped
// to tiles XCD by XCD so that the tiles resident on one XCD share slices through its L2.
//
// Epilogues: plain fp32 store, residual add (output and down projections),
// SwiGLU: the B tile interleaves rows of W_gate and W_up so that one lane holds
// gate[m, n] and up[m, n] in matching accumulator registers, and the fused QKV epilogue (bias, RoPE,
// compact q / k rows, scatter of K and V into the cache).
#include <algorithm>
#include <type_traits>

#include "keep_internal.h"

namespace keep {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4))) uint32_t u32x4;  // 16-byte register vector (native, so arrays of it stay in VGPRs)

struct MfmaB {
  const bf16_t* ptr[3];
  int32_t begin[4];
  int32_t n_parts;
};

// Element offset of 16-byte chunk `chunk` of row `row` in a [rows][GBK] bf16 tile.  LDS has 64 four-byte
// banks (256 B per bank line); a row is GBK*2 bytes, so 256/(GBK*2) rows share a line.  The chunk index
// is XOR-ed with (row / rows-per-line) % chunks-per-row: 16 consecutive rows then cover all 64 banks
// exactly once for the 16-byte operand reads.
template <int GBK>
__device__ __forceinline__ int lds_off(int row, int chunk) {
  constexpr int CPR = GBK / 8, RPL = 128 / GBK;
  return row * GBK + ((chunk ^ ((row / RPL) & (CPR - 1))) << 3);
}

// s_waitcnt vmcnt(n) with the other counters left alone (gfx9 encoding: vmcnt in bits 3:0 and 15:14)
__device__ __forceinline__ constexpr int vmcnt_imm(int n) { return 0x0F70 | (n & 15) | ((n >> 4) << 14); }

// Position t of the tile list -> tile coordinates: panels of GM tile rows, walked column by column.
template <int BM>
__device__ __forceinline__ void gemm_tile_of(int t, int tiles_m, int tiles_n, int& tile_m, int& tile_n) {
  constexpr int GM = (BM >= 256) ? 4 : 8;
  const int panel = t / (GM * tiles_n);
  const int panel_rows = min(GM, tiles_m - panel * GM);
  const int within = t - panel * GM * tiles_n;
  tile_m = panel * GM + within % panel_rows;
  tile_n = within / panel_rows;
}

template <int BM, int BN, int WM, int WN, int EPI, int GBK, int NST>
__global__ void __launch_bounds__(WM* WN * 64)
    k_gemm_mfma(const bf16_t* __restrict__ A, int M, int K, MfmaB B, const bf16_t* __restrict__ B2, int N,
                const bf16_t* __restrict__ residual, void* __restrict__ Cv, int tiles_m, int tiles_n,
                int full_per_xcd, int split_s, float* __restrict__ part, QkvEpilogue qe) {
  constexpr int T = WM * WN * 64;
  constexpr int TM = BM / WM, TN = BN / WN;
  constexpr int MI = TM / 16, NI = TN / 16;  // 16x16 accumulator tiles per wave
  static_assert(NI % 4 == 0, "a wave's columns are walked in groups of four 16-column tiles");
  static_assert(EPI != EPI_SWIGLU_STORE || (NI % 2 == 0), "SwiGLU needs an even number of N tiles per wave");

  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  constexpr int BUF = (BM + BN) * GBK;  // elements per buffer: A tile then B tile

  const int tid = threadIdx.x;
  const int lane = tid & 63, wave = tid >> 6;
  const int wm = wave / WN, wn = wave % WN;
  // Workgroup -> tile.  Consecutive workgroup ids go round-robin to the 8 XCDs, each with its own L2.
  // XCD x therefore takes the x-th eighth of the tile list, and the list walks panels of GM tile rows
  // column by column, so the ~32 workgroups resident on one XCD cover a GM x (32/GM) patch of C and
  // share their A and B slices through that XCD's L2.
  //
  // The tail of each XCD's list, the tiles that would form a last, partly filled round of workgroups,
  // is cut along K instead: split_s workgroups share a tile, each multiplies its slice of K and writes
  // an fp32 partial tile; k_gemm_fixup adds the slices in order and applies the epilogue.
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  const int xcd = (int)(blockIdx.x & 7), j_x = (int)(blockIdx.x >> 3);
  int tl = j_x, piece = 0, pieces = 1;
  if (j_x >= full_per_xcd) {
    tl = full_per_xcd + (j_x - full_per_xcd) / split_s;
    piece = (j_x - full_per_xcd) % split_s;
    pieces = split_s;
  }
  const int t = xcd * per_xcd + tl;
  if (tl >= per_xcd || t >= n_tiles) return;
  int tile_m, tile_n;
  gemm_tile_of<BM>(t, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM;
  const int n0 = tile_n * BN;  // in B-tile rows (for SwiGLU: BN/2 output columns per block)

  // ---- global -> LDS staging without registers: global_load_lds_dwordx4 writes lane l's 16 bytes at
  // (wave-uniform LDS base) + 16 l, so one instruction fills 8 consecutive 128-byte tile rows.  The
  // XOR swizzle is applied on the global side: the lane whose bytes land in physical chunk pc of row r
  // fetches logical chunk pc ^ ((r / 2) % 8) of that row.
  constexpr int NW = WM * WN;
  constexpr int CPR = GBK / 8;      // 16-byte chunks per tile row
  constexpr int RPL = 128 / GBK;    // tile rows per 256-byte LDS bank line
  constexpr int RPI = 64 / CPR;     // tile rows filled by one wave-wide load instruction (1 KiB)
  constexpr int KS = GBK / 32;      // MFMA k-steps (32 deep) per slice
  constexpr int A_LD = BM / RPI / NW, B_LD = BN / RPI / NW;  // load instructions per wave per slice
  constexpr int LD = A_LD + B_LD;
  static_assert(BM % (RPI * NW) == 0 && BN % (RPI * NW) == 0, "tile rows must split evenly over the waves");
  typedef const void __attribute__((address_space(1))) * gptr_t;
  typedef void __attribute__((address_space(3))) * lptr_t;
  const bf16_t* a_src[A_LD];
  const bf16_t* b_src[B_LD];
#pragma unroll
  for (int i = 0; i < A_LD; ++i) {
    const int r = (wave * A_LD + i) * RPI + lane / CPR, c = (lane % CPR) ^ ((r / RPL) & (CPR - 1));
    const int gm = min(m0 + r, M - 1);
    a_src[i] = A + (size_t)gm * K + c * 8;
  }
#pragma unroll
  for (int i = 0; i < B_LD; ++i) {
    const int r = (wave * B_LD + i) * RPI + lane / CPR, c = (lane % CPR) ^ ((r / RPL) & (CPR - 1));
    const bf16_t* row;
    if (EPI == EPI_SWIGLU_STORE) {
      // tile row r -> wave column block, gate/up half, column inside the half
      const int w = r / TN, within = r % TN, half = within / (TN / 2), col = within % (TN / 2);
      const int gn = (n0 / 2) + w * (TN / 2) + col;
      row = (half ? B2 : B.ptr[0]) + (size_t)gn * K;
    } else {
      const int gn = n0 + r;
      // (selects, not indexed loads: a dynamically indexed kernel-argument array goes to scratch)
      const bf16_t* base = B.ptr[0];
      int first = 0;
      if (B.n_parts > 1 && gn >= B.begin[1]) {
        base = B.ptr[1];
        first = B.begin[1];
      }
      if (B.n_parts > 2 && gn >= B.begin[2]) {
        base = B.ptr[2];
        first = B.begin[2];
      }
      row = base + (size_t)(gn - first) * K;
    }
    b_src[i] = row + c * 8;
  }
  // issue the loads of K-slice `slice` into LDS stage `stage`
#define GEMM_STAGE(slice, stage)                                                                               \
  {                                                                                                            \
    uint16_t* sa_ = smem + (stage) * BUF + (wave * A_LD) * RPI * GBK;                                          \
    uint16_t* sb_ = smem + (stage) * BUF + BM * GBK + (wave * B_LD) * RPI * GBK;                               \
    _Pragma("unroll") for (int i = 0; i < A_LD; ++i)                                                           \
        __builtin_amdgcn_global_load_lds((gptr_t)(a_src[i] + (size_t)(slice) * GBK), (lptr_t)(sa_ + i * RPI * GBK), 16, 0, 0); \
    _Pragma("unroll") for (int i = 0; i < B_LD; ++i)                                                           \
        __builtin_amdgcn_global_load_lds((gptr_t)(b_src[i] + (size_t)(slice) * GBK), (lptr_t)(sb_ + i * RPI * GBK), 16, 0, 0); \
  }

  // Fused QKV epilogue: once the K loop is over the operand tiles in LDS are dead, and the cos / sin rows of the
  // tile's BM rows (64 + 64 floats each, picked by the row's rotation position) are staged there, with the
  // rows' cache positions behind them, so that the epilogue's loads are LDS reads that no global store can
  // delay.  Wave w stages rows 32 w .. 32 w + 31; a load instruction fills two rows (lanes 0-15 / 32-47 the cos
  // chunks, lanes 16-31 / 48-63 the sin chunks).  Tiles that hold only value columns need no table.
#define QKV_STAGE_TABLES                                                                                          \
  {                                                                                                               \
    __syncthreads();                                                                                              \
    float* tab_ = reinterpret_cast<float*>(smem);                                                                 \
    int32_t* spos_ = reinterpret_cast<int32_t*>(smem) + BM * 128;                                                 \
    const int r_ = wave * (BM / NW) + (lane & 31);                                                                \
    const int gmr_ = min(m0 + r_, M - 1);                                                                         \
    const int p_ = qe.row_pos[gmr_];                                                                              \
    const int rp_ = p_ - (qe.row_lo ? qe.row_lo[gmr_] : 0);                                                       \
    if (lane < 32) {                                                                                              \
      spos_[r_] = p_;                                                                                             \
      spos_[BM + r_] = rp_;                                                                                       \
    }                                                                                                             \
    if (n0 < qe.q_dim + qe.kv_dim) {                                                                              \
      _Pragma("unroll") for (int i_ = 0; i_ < 16; ++i_) {                                                         \
        const int rp2_ = __shfl(rp_, 2 * i_ + (lane >> 5), 64);                                                   \
        const int ch_ = lane & 31;                                                                                \
        const float* src_ = (ch_ < 16 ? qe.rope_cos : qe.rope_sin) + (size_t)rp2_ * 64 + (ch_ & 15) * 4;          \
        __builtin_amdgcn_global_load_lds((gptr_t)src_, (lptr_t)(tab_ + (wave * (BM / NW) + 2 * i_) * 128), 16, 0, 0); \
      }                                                                                                           \
    }                                                                                                             \
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));                                                                     \
    __syncthreads();                                                                                              \
  }

  f32x4 acc[MI][NI];
#pragma unroll
  for (int i = 0; i < MI; ++i)
#pragma unroll
    for (int j = 0; j < NI; ++j)
#pragma unroll
      for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;

  // NST LDS stages: slices kt+1 .. kt+NST-1 are in flight (or landed) while slice kt is multiplied
  const int kt_begin = (int)((long)piece * (K / GBK) / pieces);
  const int KT = (int)((long)(piece + 1) * (K / GBK) / pieces);  // end of this workgroup's K slices
  // All NST stages are kept in flight: slice kt+NST is requested as soon as the barrier inside iteration kt
  // has shown that every wave is done reading the current stage (its last operands are in registers by
  // then), so the loads get NST-1 whole iterations to land.
#pragma unroll
  for (int p = 0; p < NST; ++p) GEMM_STAGE(min(kt_begin + p, KT - 1), p)
  __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 1) * LD));  // slice 0 has landed in LDS
  __syncthreads();

  // A wave whose rows all lie past M (the last, partly filled row of tiles) has nothing to multiply: it keeps
  // doing its share of the staging and takes part in every barrier, but issues no operand reads and no MFMAs,
  // which leaves the SIMD's matrix pipe (and its power) to the wave it shares the SIMD with.
  if (m0 + wm * TM >= M) {
    int st_ = 0;
    for (int kt = kt_begin; kt < KT; ++kt) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LD));
      __syncthreads();
      GEMM_STAGE(min(kt + NST, KT - 1), st_)
      st_ = st_ + 1 == NST ? 0 : st_ + 1;
    }
    __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
    if constexpr (EPI == EPI_QKV_ROPE) {
      if (pieces == 1) QKV_STAGE_TABLES  // (its two barriers are the workgroup's: every wave takes part)
    }
    return;
  }

  const int a_row0 = wm * TM + (lane & 15);
  const int b_row0 = wn * TN + (lane & 15);
  const int kg = lane >> 4;
  // LDS element offsets of this lane's operand chunks per k-step (rows differ by multiples of 16,
  // which leaves the swizzle term unchanged, so one offset per k-step serves every row tile)
  int a_off[KS], b_off[KS];
#pragma unroll
  for (int ks = 0; ks < KS; ++ks) {
    a_off[ks] = lds_off<GBK>(a_row0, ks * 4 + kg);
    b_off[ks] = BM * GBK + lds_off<GBK>(b_row0, ks * 4 + kg);
  }

  // A slice is walked in steps (k-step, group of four 16-column tiles): MI x 4 MFMAs each.  The A fragments
  // of a k-step serve all its groups; the B fragments of the next step (and, at the end of a k-step, the next
  // k-step's A fragments) are read while a step multiplies.
  constexpr int NG = NI / 4;        // column groups per k-step
  constexpr int STEPS = KS * NG;    // steps per slice
  static_assert(KS % 2 == 0, "the A fragments' two buffers alternate by k-step and must come out even over a slice");
  bf16x8 af[2][MI], bfr[2][4];
#pragma unroll
  for (int i = 0; i < MI; ++i) af[0][i] = *reinterpret_cast<const bf16x8*>(smem + a_off[0] + i * 16 * GBK);
#pragma unroll
  for (int j = 0; j < 4; ++j) bfr[0][j] = *reinterpret_cast<const bf16x8*>(smem + b_off[0] + j * 16 * GBK);

  int stage = 0;
  for (int kt = kt_begin; kt < KT; ++kt) {
    // (Past the end the last slice is fetched again into the stage just freed: harmless, and it keeps the
    // loop body one straight-line block for the instruction scheduler.)
    const int next_stage = stage + 1 == NST ? 0 : stage + 1;
    const uint16_t* cbuf = smem + stage * BUF;
    const uint16_t* nbuf = smem + next_stage * BUF;
#pragma unroll
    for (int st = 0; st < STEPS; ++st) {
      const int ks = st / NG, g = st % NG;
      const int bc = st & 1, bn = bc ^ 1, ac = ks & 1, an = ac ^ 1;
      // (KS is even, so both buffer parities come out even over a slice and carry over to the next one)
      bool new_a;
      if (st + 1 < STEPS) {
        const int ks1 = (st + 1) / NG, g1 = (st + 1) % NG;
#pragma unroll
        for (int j = 0; j < 4; ++j)
          bfr[bn][j] = *reinterpret_cast<const bf16x8*>(cbuf + b_off[ks1] + (g1 * 4 + j) * 16 * GBK);
        new_a = g1 == 0;
        if (new_a) {
#pragma unroll
          for (int i = 0; i < MI; ++i) af[an][i] = *reinterpret_cast<const bf16x8*>(cbuf + a_off[ks1] + i * 16 * GBK);
        }
      } else {
        // Last step of the slice: its operands are already in registers, so the workgroup waits for
        // slice kt+1 and synchronises BEFORE these MFMAs; the first operand reads of the next slice
        // are then in flight while they run.
        __builtin_amdgcn_s_waitcnt(vmcnt_imm((NST - 2) * LD));
        __syncthreads();
        GEMM_STAGE(min(kt + NST, KT - 1), stage)
#pragma unroll
        for (int j = 0; j < 4; ++j) bfr[bn][j] = *reinterpret_cast<const bf16x8*>(nbuf + b_off[0] + j * 16 * GBK);
#pragma unroll
        for (int i = 0; i < MI; ++i) af[an][i] = *reinterpret_cast<const bf16x8*>(nbuf + a_off[0] + i * 16 * GBK);
        new_a = true;
      }
#pragma unroll
      for (int i = 0; i < MI; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][g * 4 + j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(af[ac][i], bfr[bc][j], acc[i][g * 4 + j], 0, 0, 0);
      // interleave the operand reads issued above with the first half of the step's MFMAs (the second half
      // covers the latency of the last read)
      if (new_a) {
#pragma unroll
        for (int r = 0; r < 4 + MI; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      } else {
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          __builtin_amdgcn_sched_group_barrier(0x008, 2, 0);
          __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        }
      }
    }
    stage = next_stage;
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // no LDS write of this workgroup may outlive it

  // ---- epilogue.  acc[i][j][e]: row = i*16 + 4*(lane/16) + e, col = j*16 + lane%16
  const int col_l = lane & 15;
  const int row_l = 4 * (lane >> 4);
  if (pieces > 1) {  // partial tile [BM][BN] in tile coordinates
    const int rem_per_xcd = per_xcd - full_per_xcd;
    float* pt = part + ((size_t)(xcd * rem_per_xcd + (tl - full_per_xcd)) * split_s + piece) * (BM * BN);
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int r = wm * TM + i * 16 + row_l + e;
#pragma unroll
        for (int j = 0; j < NI; ++j) pt[(size_t)r * BN + wn * TN + j * 16 + col_l] = acc[i][j][e];
      }
    return;
  }
  if constexpr (EPI == EPI_QKV_ROPE) {
    // The wave's TN = 128 columns are one head: query head, key head or value head by where they start.
    // RoPE pairs column c with c + 64: accumulator tiles j and j + 4, same lane, same register.
    static_assert(EPI != EPI_QKV_ROPE || (TN == 128 && NI == 8 && BM / NW == 32),
                  "the fused QKV epilogue needs one head per wave and 32 staged rows per wave");
    QKV_STAGE_TABLES
    const float* tab = reinterpret_cast<const float*>(smem);
    const int32_t* spos = reinterpret_cast<const int32_t*>(smem) + BM * 128;
    const int col0 = n0 + wn * TN;
    const int kind = col0 < qe.q_dim ? 0 : (col0 < qe.q_dim + qe.kv_dim ? 1 : 2);
    const int hcol = kind == 0 ? col0 : (kind == 1 ? col0 - qe.q_dim : col0 - qe.q_dim - qe.kv_dim);  // column inside q / k / v
    const bf16_t* bias = reinterpret_cast<const bf16_t*>(qe.bias[kind]);
    float bl[4] = {0.f, 0.f, 0.f, 0.f}, bh[4] = {0.f, 0.f, 0.f, 0.f};
    if (bias) {
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        bl[j] = bf16_bits_to_f32(bias[hcol + j * 16 + col_l].bits);
        bh[j] = bf16_bits_to_f32(bias[hcol + 64 + j * 16 + col_l].bits);
      }
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int rt = wm * TM + i * 16 + row_l + e;  // row inside the tile
        const int gm = m0 + rt;
        if (gm >= M) continue;
        const int pos = spos[rt];
        if (kind == 2) {
          bf16_t* dst = reinterpret_cast<bf16_t*>(qe.v_cache) + (size_t)pos * qe.kv_dim + hcol;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            dst[j * 16 + col_l].bits = f32_to_bf16_bits(acc[i][j][e] + bl[j]);
            dst[64 + j * 16 + col_l].bits = f32_to_bf16_bits(acc[i][j + 4][e] + bh[j]);
          }
        } else {
          const float* cs = tab + rt * 128;
          const float* sn = cs + 64;
          bf16_t* d1 = kind == 0 ? reinterpret_cast<bf16_t*>(qe.q) + (size_t)gm * qe.q_dim + hcol
                                 : reinterpret_cast<bf16_t*>(qe.k_compact) + (size_t)gm * qe.kv_dim + hcol;
          bf16_t* d2 = reinterpret_cast<bf16_t*>(qe.k_cache) + (size_t)pos * qe.kv_dim + hcol;
#pragma unroll
          for (int j = 0; j < 4; ++j) {
            const int c = j * 16 + col_l;
            const float lo = acc[i][j][e] + bl[j], hi = acc[i][j + 4][e] + bh[j];
            const float cc = cs[c], ss = sn[c];
            const uint16_t olo = f32_to_bf16_bits(lo * cc - hi * ss), ohi = f32_to_bf16_bits(hi * cc + lo * ss);
            d1[c].bits = olo;
            d1[64 + c].bits = ohi;
            if (kind == 1) {
              d2[c].bits = olo;
              d2[64 + c].bits = ohi;
            }
          }
        }
      }
    }
    return;
  }
#pragma unroll
  for (int i = 0; i < MI; ++i) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      const int gm = m0 + wm * TM + i * 16 + row_l + e;
      if (gm >= M) continue;
      if (EPI == EPI_SWIGLU_STORE) {
        const int n_out = N;  // N = ffn_dim (output width)
#pragma unroll
        for (int j = 0; j < NI / 2; ++j) {
          const int gn = (n0 / 2) + wn * (TN / 2) + j * 16 + col_l;
          const float g = acc[i][j][e], u = acc[i][j + NI / 2][e];
          const float v = g / (1.0f + __expf(-g)) * u;
          reinterpret_cast<bf16_t*>(Cv)[(size_t)gm * n_out + gn].bits = f32_to_bf16_bits(v);
        }
      } else {
#pragma unroll
        for (int j = 0; j < NI; ++j) {
          const int gn = n0 + wn * TN + j * 16 + col_l;
          const size_t idx = (size_t)gm * N + gn;
          if (EPI == EPI_STORE_F32) {
            reinterpret_cast<float*>(Cv)[idx] = acc[i][j][e];
          } else {
            const float r = bf16_bits_to_f32(residual[idx].bits);
            reinterpret_cast<bf16_t*>(Cv)[idx].bits = f32_to_bf16_bits(r + acc[i][j][e]);
          }
        }
      }
    }
  }
}

#undef GEMM_STAGE
#undef QKV_STAGE_TABLES

// ---------------------------------------------------------------------------------------------
// k_gemm_256: 256x256 tiles, four waves of 128x128, one per SIMD.
//
// Bound by the matrix cores and by what feeds them: LDS reads (64 KB x 2 per 64-deep slice here; eight waves of 64x128
// read 192 KB), the global -> LDS loads, and the clock, which falls with the power they all draw.  With one wave per SIMD
// nothing but this wave's own instruction order hides latency, so the order is written down: the accumulators sit in the
// accumulation registers (inline assembly: the compiler otherwise copies them to and fro around every product), and each
// k-step of 64 MFMAs carries the 16 operand reads of the next one, two thirds of an MFMA slot apart or more.  The reads of
// a slice's second k-step are done halfway through its first (`X`: every wave has read the stage), so the slice after the
// next is requested from there on, spread evenly, one load in five MFMAs (two in five and more at once stall the wave in
// front of the address unit), and has a slice and a half to arrive (`Y`).
//
// (Inline assembly hides the products from the compiler's hazard checks.  Nothing but products may therefore touch an
// accumulator before the wait behind the last one: the accumulators are read by get(), in assembly too, and the build
// refuses a k_gemm_256 with scratch memory, or with an instruction of the compiler's own that names an accumulator.)
//
// The weights are the A operand and the activations the B operand, and the weight rows of two neighbouring 16-row tiles
// are dealt out alternately by fours: a lane then holds eight consecutive output columns of one row, and the epilogues
// read and write 16 bytes a lane (2 bytes before: 256 stores per wave and as many loads of the residual).
//
// A wave's rows are 64 consecutive ones of either half of the tile, so that in a last tile with at most 128 rows of
// the launch every wave has half its rows and does half its products (MI = 4), or none (MI = 0: loads and barriers only).
//
// Standalone, same card, alternating with eight waves of 64x128 in the order the compiler gave (rows x K x columns, us):
//   gate/up 3328 x 5120 x 27648: 716 against 768 (1.32 PFLOP/s); down 3328 x 13824 x 5120: 350 against 385; O 5120 x 5120 x
//   5120: 216 against 244; QKV 5120 x 5120 x 7168: 296 against 315.  (An approximate reciprocal in SwiGLU: gate/up 703; not
//   kept, its last bit reaches every later layer.)  The loads packed behind
//   one barrier instead (two in eight products): gate/up 8192 rows 7 % slower; the loop on the compiler's own register
//   assignment: 60 % slower (accumulators copied).
// ---------------------------------------------------------------------------------------------
constexpr int G2_THREADS = 256;
constexpr int G2_STAGE = 512 * 64;  // elements of an LDS stage: 256 activation rows, then 256 weight rows

// swizzle of the weight rows' 16-byte chunks: a fragment's 16 lanes read rows 0-3, 8-11, 16-19 and 24-27 of a block of 32
__device__ __forceinline__ int g2_wswz(int row) { return ((row >> 1) & 1) | (((row >> 3) & 3) << 1); }

struct G2Src {  // where the wave's share of a slice comes from
  const bf16_t *a, *b;
  uint32_t a_bytes, b_bytes;
  uint32_t a_off[8], b_off[8];
};

typedef void __attribute__((address_space(3))) * g2_lptr_t;

#define G2_FENCE __builtin_amdgcn_sched_barrier(0)
#define G2_BARRIER                   \
  {                                  \
    G2_FENCE;                        \
    __builtin_amdgcn_s_barrier();    \
    G2_FENCE;                        \
    asm volatile("" ::: "memory");   \
  }

// load r of 16 of slice `s` into stage `st`: even ones activations, odd ones weights, 8 rows each
__device__ __forceinline__ void g2_load(const G2Src& src, uint16_t* smem, int wave, int s, int st, int r) {
  const int i = r >> 1;
  uint16_t* dst = smem + st * G2_STAGE + (r & 1) * (G2_STAGE / 2) + (wave * 8 + i) * 512;
  const auto rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16_t*>(r & 1 ? src.b : src.a), 0,
                                                      r & 1 ? src.b_bytes : src.a_bytes, 0x00020000);
  __builtin_amdgcn_raw_ptr_buffer_load_lds(rsrc, (g2_lptr_t)dst, 16, r & 1 ? src.b_off[i] : src.a_off[i], s * 128, 0, 0);
}

// One slice.  Behind X either slice kt + 2 is requested (NEXT), or, in the last two slices of a tile, what its epilogue
// will read (tail(r), r = 0 .. 15, with `tails`): the stage is free by then and the loads' time is hidden.
enum G2Slice { G2_NEXT, G2_LAST_BUT_ONE, G2_LAST };

template <int MI, G2Slice KIND, typename Tail>
__device__ __forceinline__ void g2_slice(f32x4 (&acc)[8][8], bf16x8 (&wf)[2][8], bf16x8 (&xf)[2][8], const G2Src& src,
                                         uint16_t* smem, int wave, const int (&x_off)[2], const int (&w_off)[2], int kt,
                                         bool tails, const Tail& tail) {
  constexpr int NM = MI ? MI * 8 : 32;          // products per k-step
  constexpr int NR = MI ? MI + 8 : 0;           // operand reads per k-step
  constexpr int X = MI == 8 ? 34 : 22;          // all reads of the second k-step lie in front (every 1.75 products)
  constexpr int DS2 = MI == 8 ? 10 : 5;         // half products between loads
  constexpr int BEHIND_X = (2 * (NM - 2 - X)) / DS2 + 1;  // loads between X and the end of the first k-step
  const int st = kt & 1;
  auto read = [&](int p, int ks, int stage, int r) {
    const uint16_t* base = smem + stage * G2_STAGE;
    if (r < 8)
      wf[p][r] = *reinterpret_cast<const bf16x8*>(base + G2_STAGE / 2 + w_off[ks] + (r >> 1) * 32 * 64 + (r & 1) * 4 * 64);
    else
      xf[p][r - 8] = *reinterpret_cast<const bf16x8*>(base + x_off[ks] + ((r - 8) >> 2) * 128 * 64 + ((r - 8) & 3) * 16 * 64);
  };
#pragma clang loop unroll(full)
  for (int half = 0; half < 2; ++half) {
#pragma clang loop unroll(full)
    for (int n = 0; n < NM; ++n) {
      if (MI)
        asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0"
                     : "+a"(acc[n >> 3][n & 7])
                     : "v"(wf[half][n & 7]), "v"(xf[half][n >> 3]));
      if (half == 0 || KIND != G2_LAST) {
#pragma clang loop unroll(full)
        for (int r = 0; r < NR; ++r)
          if (n == (half ? r * (NM * 3 / 4) / (NR ? NR : 1) : r * 7 / 4)) {
            G2_FENCE;
            read(half ^ 1, half ^ 1, half ? st ^ 1 : st, r);
            G2_FENCE;
          }
      }
      if (half == 0 && n == X) {  // X: this wave's reads of the stage are back, and with the barrier every wave's
        G2_FENCE;
        __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
        G2_BARRIER
      }
#pragma clang loop unroll(full)
      for (int r = 0; r < 16; ++r)
        if (n + half * NM == X + 1 + r * DS2 / 2) {
          G2_FENCE;
          if (KIND == G2_NEXT)
            g2_load(src, smem, wave, kt + 2, st, r);
          else if (tails)
            tail(smem + st * G2_STAGE, KIND == G2_LAST, r);
          G2_FENCE;
        }
    }
    if (half == 0 && KIND != G2_LAST) {  // Y: slice kt + 1 has landed
      G2_FENCE;
      if (KIND == G2_NEXT || tails)
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(BEHIND_X));
      else
        __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      G2_BARRIER
    }
  }
  G2_FENCE;
}

// The slices kt0 .. kt1 - 1 of a tile, at least two; the first two are on their way (16 loads of this wave each).
template <int MI, typename Tail>
__device__ __forceinline__ void g2_loop(f32x4 (&acc)[8][8], const G2Src& src, uint16_t* smem, int wave, int lane, int wm,
                                        int wn, int kt0, int kt1, bool tails, const Tail& tail) {
  bf16x8 wf[2][8], xf[2][8];
  int x_off[2], w_off[2];
  {
    const int l = lane & 15, c = lane >> 4;
    const int wr = 8 * (l >> 2) + (l & 3);  // weight row inside a block of 32 (its tile's other half: + 4)
#pragma unroll
    for (int ks = 0; ks < 2; ++ks) {
      x_off[ks] = lds_off<64>(wm * 64 + l, ks * 4 + c);
      w_off[ks] = (wn * 128 + wr) * 64 + (((ks * 4 + c) ^ g2_wswz(wr)) << 3);
    }
  }
  {  // zeros (while the first slices are on their way), as products: what the compiler cannot rebuild it does not copy
    u32x4 zero = {0, 0, 0, 0};
    asm volatile("s_nop 4" : "+v"(zero));
#pragma unroll
    for (int i = 0; i < MI; ++i)
#pragma unroll
      for (int j = 0; j < 8; ++j) asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %1, 0" : "=a"(acc[i][j]) : "v"(zero));
  }
  __builtin_amdgcn_s_waitcnt(vmcnt_imm(16));  // slice kt0 has landed
  G2_BARRIER
  if (MI) {
    const uint16_t* base = smem + (kt0 & 1) * G2_STAGE;
#pragma unroll
    for (int j = 0; j < 8; ++j)
      wf[0][j] = *reinterpret_cast<const bf16x8*>(base + G2_STAGE / 2 + w_off[0] + (j >> 1) * 32 * 64 + (j & 1) * 4 * 64);
#pragma unroll
    for (int i = 0; i < MI; ++i)
      xf[0][i] = *reinterpret_cast<const bf16x8*>(base + x_off[0] + (i >> 2) * 128 * 64 + (i & 3) * 16 * 64);
  }
  int kt = kt0;
  for (; kt + 2 < kt1; ++kt) g2_slice<MI, G2_NEXT>(acc, wf, xf, src, smem, wave, x_off, w_off, kt, tails, tail);
  g2_slice<MI, G2_LAST_BUT_ONE>(acc, wf, xf, src, smem, wave, x_off, w_off, kt, tails, tail);
  g2_slice<MI, G2_LAST>(acc, wf, xf, src, smem, wave, x_off, w_off, kt + 1, tails, tail);
  asm volatile("s_nop 15\n s_nop 15" ::: "memory");  // the last products are in the accumulators
  G2_FENCE;
}

// eight consecutive values of a row: accumulator tiles 2 jj and 2 jj + 1
__device__ __forceinline__ uint4 g2_pack(const float (&v)[8]) {
  return make_uint4(pack_bf16x2(v[0], v[1]), pack_bf16x2(v[2], v[3]), pack_bf16x2(v[4], v[5]), pack_bf16x2(v[6], v[7]));
}
__device__ __forceinline__ void g2_unpack(const uint4& u, float (&v)[8]) {
  const uint32_t w[4] = {u.x, u.y, u.z, u.w};
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    v[2 * i] = __uint_as_float(w[i] << 16);
    v[2 * i + 1] = __uint_as_float(w[i] & 0xffff0000u);
  }
}

template <int EPI>
__global__ void __launch_bounds__(G2_THREADS, 1)
    k_gemm_256(const bf16_t* __restrict__ A, int M, int K, MfmaB B, const bf16_t* __restrict__ B2, int N,
               const bf16_t* __restrict__ residual, void* __restrict__ Cv, int tiles_m, int tiles_n, int full_per_xcd,
               int split_s, float* __restrict__ part, QkvEpilogue qe) {
  extern __shared__ __attribute__((aligned(16))) uint16_t smem[];
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave >> 1, wn = wave & 1;
  // workgroup -> tile: as in k_gemm_mfma
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  const int xcd = (int)(blockIdx.x & 7), j_x = (int)(blockIdx.x >> 3);
  int tl = j_x, piece = 0, pieces = 1;
  if (j_x >= full_per_xcd) {
    tl = full_per_xcd + (j_x - full_per_xcd) / split_s;
    piece = (j_x - full_per_xcd) % split_s;
    pieces = split_s;
  }
  const int t = xcd * per_xcd + tl;
  if (tl >= per_xcd || t >= n_tiles) return;
  int tile_m, tile_n;
  gemm_tile_of<256>(t, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * 256, n0 = tile_n * 256;  // n0 in rows of the weight tile (SwiGLU: 128 output columns)

  // ---- the wave's 64 rows of either operand, 8 per load: lane l's 16 bytes land at (LDS base) + 16 l, so the lane whose
  // bytes land in chunk pc of a row fetches the chunk that the swizzle keeps there
  G2Src src;
  {
    src.a = A + (size_t)m0 * K;
    src.a_bytes = (uint32_t)min(256, M - m0) * K * 2;
    int first = wave * 64;  // first weight row of the wave's share inside src.b
    if (EPI == EPI_SWIGLU_STORE) {  // waves 0, 2: gate rows, 1, 3: up rows, of column block wave / 2
      src.b = (wave & 1 ? B2 : B.ptr[0]) + (size_t)(n0 / 2) * K;
      first = (wave >> 1) * 64;
    } else {  // (a tile lies in one part: their widths are multiples of 256)
      const bf16_t* base = B.ptr[0];
      int begin = 0;
      if (B.n_parts > 1 && n0 >= B.begin[1]) base = B.ptr[1], begin = B.begin[1];
      if (B.n_parts > 2 && n0 >= B.begin[2]) base = B.ptr[2], begin = B.begin[2];
      src.b = base + (size_t)(n0 - begin) * K;
    }
    src.b_bytes = (uint32_t)(EPI == EPI_SWIGLU_STORE ? 128 : 256) * K * 2;
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const int r = i * 8 + lane / 8, pc = lane & 7;
      src.a_off[i] = (uint32_t)min(wave * 64 + r, M - 1 - m0) * K * 2 + (pc ^ ((r >> 1) & 7)) * 16;
      src.b_off[i] = (uint32_t)(first + r) * K * 2 + (pc ^ g2_wswz(r)) * 16;
    }
  }
  const int kt0 = (int)((long)piece * (K / 64) / pieces), kt1 = (int)((long)(piece + 1) * (K / 64) / pieces);

  const int c8 = 8 * (lane >> 4);  // the lane's output columns: c8 + 32 jj + 0..7 of the wave's 128
  auto rt = [&](int i) { return (i >> 2) * 128 + wm * 64 + (i & 3) * 16 + (lane & 15); };  // its row of tile i

  // ---- what the epilogue reads comes to LDS during the last two slices, the first half of the tile's rows in the first
  // one.  Residual: the 16 bytes of tile i, column block jj land where the lane that fetched them reads them back.
  // Fused QKV: cos / sin rows, picked by each row's rotation position: 32 chunks of 16 bytes (cos, then sin), chunk c
  // kept at c ^ (row % 16); a load fills two rows.  The rows' cache positions sit behind the stages.  (Tiles that hold
  // only value columns need no table.)  Pieces of a tile have no epilogue.
  const bool qkv_table = EPI == EPI_QKV_ROPE && n0 < qe.q_dim + qe.kv_dim;
  const bool tails = pieces == 1 && (EPI == EPI_RESIDUAL_STORE || qkv_table);
  int32_t* spos = reinterpret_cast<int32_t*>(smem + 2 * G2_STAGE);
  int rot = 0;  // rotation position of tile row (lane / 32) * 128 + wave * 32 + lane % 32
  if (EPI == EPI_QKV_ROPE && pieces == 1) {
    const int r = (lane >> 5) * 128 + wave * 32 + (lane & 31), gm = min(m0 + r, M - 1);
    const int p = qe.row_pos[gm];
    spos[r] = p;
    rot = p - (qe.row_lo ? qe.row_lo[gm] : 0);
  }
  const auto res_rsrc = __builtin_amdgcn_make_buffer_rsrc(
      const_cast<bf16_t*>(EPI == EPI_RESIDUAL_STORE ? residual + (size_t)m0 * N + n0 : nullptr), 0,
      (uint32_t)((min(256, M - m0) - 1) * N + min(256, N - n0)) * 2, 0x00020000);
  auto tail = [&](uint16_t* stage, int half, int r) {
    if (EPI == EPI_RESIDUAL_STORE) {
      const int row = min(rt(half * 4 + (r >> 2)), M - 1 - m0);
      __builtin_amdgcn_raw_ptr_buffer_load_lds(res_rsrc, (g2_lptr_t)(stage + (wave * 16 + r) * 512), 16,
                                               (uint32_t)(row * N + wn * 128 + c8 + 32 * (r & 3)) * 2, 0, 0, 0);
    } else if (EPI == EPI_QKV_ROPE) {
      const int even = __builtin_amdgcn_readlane(rot, half * 32 + 2 * r), odd = __builtin_amdgcn_readlane(rot, half * 32 + 2 * r + 1);
      const int ch = (lane & 31) ^ ((2 * r + (lane >> 5)) & 15);
      const float* s = (ch < 16 ? qe.rope_cos : qe.rope_sin) + (size_t)(lane < 32 ? even : odd) * 64 + (ch & 15) * 4;
      __builtin_amdgcn_global_load_lds((const void __attribute__((address_space(1)))*)s,
                                       (g2_lptr_t)(stage + (wave * 32 + 2 * r) * 256), 16, 0, 0);
    }
  };

#pragma unroll
  for (int r = 0; r < 16; ++r) g2_load(src, smem, wave, kt0, kt0 & 1, r);
#pragma unroll
  for (int r = 0; r < 16; ++r) g2_load(src, smem, wave, kt0 + 1, (kt0 & 1) ^ 1, r);
  G2_FENCE;

  auto tile = [&](auto mi) {
    constexpr int MI = decltype(mi)::value;
    f32x4 acc[8][8];  // [activation tile][weight tile]
    g2_loop<MI>(acc, src, smem, wave, lane, wm, wn, kt0, kt1, tails, tail);
    // (the lane's number anew: what the epilogue derives from it is not to be kept in registers through the loop)
    int el = lane;
    asm volatile("" : "+v"(el));
    const int ec8 = 8 * (el >> 4), erow = wm * 64 + (el & 15);
    // Rows past M were computed from row M - 1, as was everything they need: they are stored to that row, the same
    // bytes again.  That keeps the epilogue free of branches, around which the compiler would keep all the accumulators
    // in vector registers at once; the fences have it take them a row at a time.
    auto row_of = [&](int i) { return min((i >> 2) * 128 + (i & 3) * 16 + erow, M - 1 - m0); };
    // (read out of the accumulation registers here: the compiler would do it for all of them behind the last product)
    auto get = [&](int i, int jj, float (&v)[8]) {
#pragma unroll
      for (int e = 0; e < 8; ++e)
        asm volatile("v_accvgpr_read_b32 %0, %1" : "=v"(v[e]) : "a"(acc[i][2 * jj + (e >> 2)][e & 3]));
    };
    if (pieces > 1) {  // partial tile [256][256] in tile coordinates
      const int rem_per_xcd = per_xcd - full_per_xcd;
      float* pt = part + ((size_t)(xcd * rem_per_xcd + (tl - full_per_xcd)) * split_s + piece) * (256 * 256);
#pragma unroll
      for (int i = 0; i < MI; ++i) {
        G2_FENCE;
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          float v[8];
          get(i, jj, v);
          float* dst = pt + row_of(i) * 256 + wn * 128 + 32 * jj + ec8;
          *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
          *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
        }
      }
      return;
    }
    if constexpr (EPI == EPI_QKV_ROPE) {
      // The wave's 128 columns are one head: query head, key head or value head by where they start.  RoPE pairs
      // column c with c + 64: jj and jj + 2, same lane, same register.
      const int col0 = n0 + wn * 128;
      const int kind = col0 < qe.q_dim ? 0 : (col0 < qe.q_dim + qe.kv_dim ? 1 : 2);
      const int hcol = kind == 0 ? col0 : (kind == 1 ? col0 - qe.q_dim : col0 - qe.q_dim - qe.kv_dim);  // column inside q / k / v
      const bf16_t* bias = reinterpret_cast<const bf16_t*>(qe.bias[kind]);
      float bv[4][8] = {};
      if (bias && MI) {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj)
#pragma unroll
          for (int e = 0; e < 8; ++e) bv[jj][e] = bf16_bits_to_f32(bias[hcol + 32 * jj + ec8 + e].bits);
      }
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));
      __syncthreads();  // the tables are there
      auto v_rows = [&]() {
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          G2_FENCE;
          bf16_t* dst = reinterpret_cast<bf16_t*>(qe.v_cache) + (size_t)spos[row_of(i)] * qe.kv_dim + hcol + ec8;
#pragma unroll
          for (int jj = 0; jj < 4; ++jj) {
            float v[8];
            get(i, jj, v);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] += bv[jj][e];
            *reinterpret_cast<uint4*>(dst + 32 * jj) = g2_pack(v);
          }
        }
      };
      auto qk_rows = [&](auto is_key) {
        constexpr bool KEY = decltype(is_key)::value;
        bf16_t* out = reinterpret_cast<bf16_t*>(KEY ? qe.k_compact : qe.q) + hcol + ec8;
        const int ld = KEY ? qe.kv_dim : qe.q_dim;
        // cos / sin of row i: [cos, sin][column block][half of the lane's eight columns]; read a row ahead
        f32x4 tab[2][2][2][2];
        int pos[2] = {0, 0};
        auto read_table = [&](int i) {
          const int row = row_of(i);
          const float* t = reinterpret_cast<const float*>(smem + ((kt1 + (i >> 2)) & 1) * G2_STAGE) + (row & 127) * 128;
#pragma unroll
          for (int k = 0; k < 8; ++k) {
            const int ch = 16 * (k >> 2) + 8 * ((k >> 1) & 1) + (ec8 >> 2) + (k & 1);
            tab[i & 1][k >> 2][(k >> 1) & 1][k & 1] = *reinterpret_cast<const f32x4*>(t + ((ch ^ (row & 15)) << 2));
          }
          if (KEY) pos[i & 1] = spos[row];
        };
        if (MI) read_table(0);
#pragma unroll
        for (int i = 0; i < MI; ++i) {
          G2_FENCE;
          if (i + 1 < MI) read_table(i + 1);
          G2_FENCE;
          bf16_t* d1 = out + (size_t)(m0 + row_of(i)) * ld;
          bf16_t* d2 = reinterpret_cast<bf16_t*>(qe.k_cache) + (size_t)pos[i & 1] * qe.kv_dim + hcol + ec8;
#pragma unroll
          for (int jj = 0; jj < 2; ++jj) {
            float lo[8], hi[8], ol[8], oh[8];
            get(i, jj, lo);
            get(i, jj + 2, hi);
#pragma unroll
            for (int e = 0; e < 8; ++e) {
              lo[e] += bv[jj][e];
              hi[e] += bv[jj + 2][e];
              const float cs = tab[i & 1][0][jj][e >> 2][e & 3], sn = tab[i & 1][1][jj][e >> 2][e & 3];
              ol[e] = lo[e] * cs - hi[e] * sn;
              oh[e] = hi[e] * cs + lo[e] * sn;
            }
            const uint4 pl = g2_pack(ol), ph = g2_pack(oh);
            *reinterpret_cast<uint4*>(d1 + 32 * jj) = pl;
            *reinterpret_cast<uint4*>(d1 + 32 * jj + 64) = ph;
            if (KEY) {
              *reinterpret_cast<uint4*>(d2 + 32 * jj) = pl;
              *reinterpret_cast<uint4*>(d2 + 32 * jj + 64) = ph;
            }
          }
        }
      };
      if (kind == 2)
        v_rows();
      else if (kind == 1)
        qk_rows(std::true_type{});
      else
        qk_rows(std::false_type{});
      return;
    }
    uint4 res[2][4];
    auto read_res = [&](int i) {  // the lane's residual of row i, staged above
#pragma unroll
      for (int jj = 0; jj < 4; ++jj)
        res[i & 1][jj] = *reinterpret_cast<const uint4*>(smem + ((kt1 + (i >> 2)) & 1) * G2_STAGE +
                                                         (wave * 16 + (i & 3) * 4 + jj) * 512 + el * 8);
    };
    if (EPI == EPI_RESIDUAL_STORE) {
      __builtin_amdgcn_s_waitcnt(vmcnt_imm(0));  // (this wave's own loads: no barrier)
      asm volatile("" ::: "memory");
      if (MI) read_res(0);
    }
#pragma unroll
    for (int i = 0; i < MI; ++i) {
      G2_FENCE;
      if (EPI == EPI_RESIDUAL_STORE && i + 1 < MI) read_res(i + 1);
      G2_FENCE;
      const int gm = m0 + row_of(i);
      if (EPI == EPI_SWIGLU_STORE) {
#pragma unroll
        for (int jj = 0; jj < 2; ++jj) {  // N = ffn_dim (output width); gate in jj, up in jj + 2
          float g[8], u[8];
          get(i, jj, g);
          get(i, jj + 2, u);
#pragma unroll
          for (int e = 0; e < 8; ++e) g[e] = g[e] / (1.0f + __expf(-g[e])) * u[e];
          *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(Cv) + (size_t)gm * N + n0 / 2 + wn * 64 + 32 * jj + ec8) = g2_pack(g);
        }
      } else {
#pragma unroll
        for (int jj = 0; jj < 4; ++jj) {
          const size_t idx = (size_t)gm * N + n0 + wn * 128 + 32 * jj + ec8;
          float v[8];
          get(i, jj, v);
          if (EPI == EPI_STORE_F32) {
            float* dst = reinterpret_cast<float*>(Cv) + idx;
            *reinterpret_cast<float4*>(dst) = make_float4(v[0], v[1], v[2], v[3]);
            *reinterpret_cast<float4*>(dst + 4) = make_float4(v[4], v[5], v[6], v[7]);
          } else {
            float r[8];
            g2_unpack(res[i & 1][jj], r);
#pragma unroll
            for (int e = 0; e < 8; ++e) v[e] = r[e] + v[e];
            *reinterpret_cast<uint4*>(reinterpret_cast<bf16_t*>(Cv) + idx) = g2_pack(v);
          }
        }
      }
    }
  };
  if (m0 + 128 + wm * 64 < M)
    tile(std::integral_constant<int, 8>{});
  else if (m0 + wm * 64 < M)
    tile(std::integral_constant<int, 4>{});
  else
    tile(std::integral_constant<int, 0>{});
}

#undef G2_FENCE
#undef G2_BARRIER

// Epilogue of the tiles that were cut along K: partial slices added in slice order (reproducible).
template <int BM, int BN, int WM, int WN, int EPI>
__global__ void __launch_bounds__(256)
    k_gemm_fixup(const float* __restrict__ part, int M, int N, const bf16_t* __restrict__ residual,
                 void* __restrict__ Cv, int tiles_m, int tiles_n, int full_per_xcd, int split_s) {
  constexpr int TN = BN / WN;
  constexpr int OUT_N = EPI == EPI_SWIGLU_STORE ? BN / 2 : BN;  // output columns per tile
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  const int rem_per_xcd = per_xcd - full_per_xcd;
  const int xcd = blockIdx.x / rem_per_xcd, ri = blockIdx.x % rem_per_xcd;
  const int t = xcd * per_xcd + full_per_xcd + ri;
  if (t >= n_tiles) return;
  int tile_m, tile_n;
  gemm_tile_of<BM>(t, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const float* pt = part + (size_t)blockIdx.x * split_s * (BM * BN);
  // one thread per 4 consecutive output columns of one row; the slices' loads are independent
  const int i = (blockIdx.y * 256 + threadIdx.x) * 4;
  if (i >= BM * OUT_N) return;
  const int r = i / OUT_N, c = i % OUT_N;
  const int gm = m0 + r;
  if (gm >= M) return;
  if (EPI == EPI_SWIGLU_STORE) {
    // output column c of the tile: gate in tile column w*TN + col, up in w*TN + TN/2 + col
    const int w = c / (TN / 2), col = c % (TN / 2);
    const float* p = pt + (size_t)r * BN + w * TN + col;
    float4 g = make_float4(0.f, 0.f, 0.f, 0.f), u = g;
#pragma unroll 4
    for (int z = 0; z < split_s; ++z) {
      const float4 gz = *reinterpret_cast<const float4*>(p + (size_t)z * (BM * BN));
      const float4 uz = *reinterpret_cast<const float4*>(p + (size_t)z * (BM * BN) + TN / 2);
      g.x += gz.x; g.y += gz.y; g.z += gz.z; g.w += gz.w;
      u.x += uz.x; u.y += uz.y; u.z += uz.z; u.w += uz.w;
    }
    uint2 o;
    o.x = pack_bf16x2(g.x / (1.0f + __expf(-g.x)) * u.x, g.y / (1.0f + __expf(-g.y)) * u.y);
    o.y = pack_bf16x2(g.z / (1.0f + __expf(-g.z)) * u.z, g.w / (1.0f + __expf(-g.w)) * u.w);
    *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(Cv) + (size_t)gm * N + n0 / 2 + c) = o;
  } else {
    const float* p = pt + (size_t)r * BN + c;
    float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
#pragma unroll 4
    for (int z = 0; z < split_s; ++z) {
      const float4 v = *reinterpret_cast<const float4*>(p + (size_t)z * (BM * BN));
      a.x += v.x; a.y += v.y; a.z += v.z; a.w += v.w;
    }
    const size_t idx = (size_t)gm * N + n0 + c;
    if (EPI == EPI_STORE_F32) {
      *reinterpret_cast<float4*>(reinterpret_cast<float*>(Cv) + idx) = a;
    } else {
      const uint2 rv = *reinterpret_cast<const uint2*>(residual + idx);
      uint2 o;
      o.x = pack_bf16x2(bf16_bits_to_f32((uint16_t)(rv.x & 0xffff)) + a.x, bf16_bits_to_f32((uint16_t)(rv.x >> 16)) + a.y);
      o.y = pack_bf16x2(bf16_bits_to_f32((uint16_t)(rv.y & 0xffff)) + a.z, bf16_bits_to_f32((uint16_t)(rv.y >> 16)) + a.w);
      *reinterpret_cast<uint2*>(reinterpret_cast<bf16_t*>(Cv) + idx) = o;
    }
  }
}

// The same for the fused QKV epilogue: a thread owns 4 consecutive columns c.. of the low half of a head and their
// partners c + 64.. (RoPE pairs), of one row.
template <int BM, int BN>
__global__ void __launch_bounds__(256)
    k_gemm_fixup_qkv(const float* __restrict__ part, int M, int tiles_m, int tiles_n, int full_per_xcd, int split_s,
                     QkvEpilogue qe) {
  const int n_tiles = tiles_m * tiles_n;
  const int per_xcd = (n_tiles + 7) >> 3;
  const int rem_per_xcd = per_xcd - full_per_xcd;
  const int xcd = blockIdx.x / rem_per_xcd, ri = blockIdx.x % rem_per_xcd;
  const int t = xcd * per_xcd + full_per_xcd + ri;
  if (t >= n_tiles) return;
  int tile_m, tile_n;
  gemm_tile_of<BM>(t, tiles_m, tiles_n, tile_m, tile_n);
  const int m0 = tile_m * BM, n0 = tile_n * BN;
  const float* pt = part + (size_t)blockIdx.x * split_s * (BM * BN);
  constexpr int HEADS = BN / 128;               // heads per tile
  constexpr int ITEMS = BM * HEADS * 16;        // (row, head, group of 4 low columns)
  const int it = blockIdx.y * 256 + threadIdx.x;
  if (it >= ITEMS) return;
  const int r = it / (HEADS * 16), hh = (it / 16) % HEADS, c = (it % 16) * 4;
  const int gm = m0 + r;
  if (gm >= M) return;
  const float* p = pt + (size_t)r * BN + hh * 128 + c;
  float4 lo = make_float4(0.f, 0.f, 0.f, 0.f), hi = lo;
#pragma unroll 4
  for (int z = 0; z < split_s; ++z) {
    const float4 a = *reinterpret_cast<const float4*>(p + (size_t)z * (BM * BN));
    const float4 b = *reinterpret_cast<const float4*>(p + (size_t)z * (BM * BN) + 64);
    lo.x += a.x; lo.y += a.y; lo.z += a.z; lo.w += a.w;
    hi.x += b.x; hi.y += b.y; hi.z += b.z; hi.w += b.w;
  }
  float l4[4] = {lo.x, lo.y, lo.z, lo.w}, h4[4] = {hi.x, hi.y, hi.z, hi.w};
  const int col0 = n0 + hh * 128;
  const int kind = col0 < qe.q_dim ? 0 : (col0 < qe.q_dim + qe.kv_dim ? 1 : 2);
  const int hcol = kind == 0 ? col0 : (kind == 1 ? col0 - qe.q_dim : col0 - qe.q_dim - qe.kv_dim);
  const bf16_t* bias = reinterpret_cast<const bf16_t*>(qe.bias[kind]);
  if (bias) {
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      l4[e] += bf16_bits_to_f32(bias[hcol + c + e].bits);
      h4[e] += bf16_bits_to_f32(bias[hcol + 64 + c + e].bits);
    }
  }
  const int pos = qe.row_pos[gm];
  uint2 olo, ohi;
  if (kind == 2) {
    olo.x = pack_bf16x2(l4[0], l4[1]); olo.y = pack_bf16x2(l4[2], l4[3]);
    ohi.x = pack_bf16x2(h4[0], h4[1]); ohi.y = pack_bf16x2(h4[2], h4[3]);
    bf16_t* dst = reinterpret_cast<bf16_t*>(qe.v_cache) + (size_t)pos * qe.kv_dim + hcol;
    *reinterpret_cast<uint2*>(dst + c) = olo;
    *reinterpret_cast<uint2*>(dst + 64 + c) = ohi;
    return;
  }
  const int rpos = pos - (qe.row_lo ? qe.row_lo[gm] : 0);
  const float4 cs = *reinterpret_cast<const float4*>(qe.rope_cos + (size_t)rpos * 64 + c);
  const float4 sn = *reinterpret_cast<const float4*>(qe.rope_sin + (size_t)rpos * 64 + c);
  const float c4[4] = {cs.x, cs.y, cs.z, cs.w}, s4[4] = {sn.x, sn.y, sn.z, sn.w};
  float ol[4], oh[4];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    ol[e] = l4[e] * c4[e] - h4[e] * s4[e];
    oh[e] = h4[e] * c4[e] + l4[e] * s4[e];
  }
  olo.x = pack_bf16x2(ol[0], ol[1]); olo.y = pack_bf16x2(ol[2], ol[3]);
  ohi.x = pack_bf16x2(oh[0], oh[1]); ohi.y = pack_bf16x2(oh[2], oh[3]);
  bf16_t* d1 = kind == 0 ? reinterpret_cast<bf16_t*>(qe.q) + (size_t)gm * qe.q_dim + hcol
                         : reinterpret_cast<bf16_t*>(qe.k_compact) + (size_t)gm * qe.kv_dim + hcol;
  *reinterpret_cast<uint2*>(d1 + c) = olo;
  *reinterpret_cast<uint2*>(d1 + 64 + c) = ohi;
  if (kind == 1) {
    bf16_t* d2 = reinterpret_cast<bf16_t*>(qe.k_cache) + (size_t)pos * qe.kv_dim + hcol;
    *reinterpret_cast<uint2*>(d2 + c) = olo;
    *reinterpret_cast<uint2*>(d2 + 64 + c) = ohi;
  }
}

template <int BM, int BN, int WM, int WN, int EPI, int GBK, int NST>
static auto gemm_kernel() {
  if constexpr (BM == 256)
    return k_gemm_256<EPI>;
  else
    return k_gemm_mfma<BM, BN, WM, WN, EPI, GBK, NST>;
}

constexpr size_t GEMM_SPLIT_WS_BYTES = (size_t)256 * 256 * 256 * sizeof(float);  // 256 partial tiles of 256 x 256

template <int BM, int BN, int WM, int WN, int GBK, int NST>
static void launch_cfg(const bf16_t* A, int M, int K, const MfmaB& b, const bf16_t* B2, int N, int epilogue,
                       const bf16_t* residual, void* C, hipStream_t s, void* ws, const QkvEpilogue& qe) {
  // operand stages; the fused QKV epilogue re-uses them for BM rows of cos / sin (512 B each) and needs 2 BM
  // ints more for the rows' positions
  const size_t sh_ops = (size_t)NST * (BM + BN) * GBK * sizeof(uint16_t);
  const size_t sh = epilogue == EPI_QKV_ROPE ? std::max(sh_ops, (size_t)BM * 512) + (size_t)BM * 8 : sh_ops;
  const dim3 block(WM * WN * 64);
  const int n_tile_rows = epilogue == EPI_SWIGLU_STORE ? 2 * N : N;  // B-tile rows to cover
  const int tiles_n = n_tile_rows / BN, tiles_m = (M + BM - 1) / BM;
  const int per_xcd = (tiles_m * tiles_n + 7) / 8;
  // Workgroups resident per XCD (32 CUs): one per CU for the 256 x 256 tile (128 KB of LDS), two otherwise.
  // What would be a last, partly filled round is cut along K so that it fills the XCD once.
  const int slots = sh_ops > 80 * 1024 ? 32 : 64;
  int full = per_xcd, split = 1;
  if (ws && BM >= 128) {
    const int f = per_xcd / slots * slots, rem = per_xcd - f;
    if (rem > 0) {
      int sp = std::min(16, slots / rem);
      sp = std::min(sp, (K / GBK) / 4);  // at least four K slices per workgroup
      if (sp >= 2 && (size_t)8 * rem * sp * BM * BN * sizeof(float) <= GEMM_SPLIT_WS_BYTES) {
        full = f;
        split = sp;
      }
    }
  }
  const int rem = per_xcd - full;
  const dim3 grid(8 * (full + rem * split));
  float* part = reinterpret_cast<float*>(ws);
#define GO(E)                                                                                              \
  do {                                                                                                     \
    auto kern = gemm_kernel<BM, BN, WM, WN, E, GBK, NST>();                                                \
    static std::atomic<uint64_t> attr_done{0};                                                             \
    set_max_dyn_smem_once(attr_done, reinterpret_cast<const void*>(kern), (int)sh);                        \
    hipLaunchKernelGGL(kern, grid, block, sh, s, A, M, K, b, B2, N, residual, C, tiles_m, tiles_n, full, split, part, qe); \
    if (split > 1 && E != EPI_QKV_ROPE)                                                                    \
      hipLaunchKernelGGL((k_gemm_fixup<BM, BN, WM, WN, E>), dim3(8 * rem, BM * BN / 1024), dim3(256), 0, s, part, M, N, \
                         residual, C, tiles_m, tiles_n, full, split);                                      \
  } while (0)
  if (epilogue == EPI_STORE_F32)
    GO(EPI_STORE_F32);
  else if (epilogue == EPI_RESIDUAL_STORE)
    GO(EPI_RESIDUAL_STORE);
  else if (epilogue == EPI_SWIGLU_STORE)
    GO(EPI_SWIGLU_STORE);
  else if constexpr (BN / WN == 128) {  // one head per wave
    GO(EPI_QKV_ROPE);
    if (split > 1)
      hipLaunchKernelGGL((k_gemm_fixup_qkv<BM, BN>), dim3(8 * rem, (BM * (BN / 128) * 16 + 255) / 256), dim3(256), 0, s,
                         part, M, tiles_m, tiles_n, full, split, qe);
  }
#undef GO
}

size_t gemm_ws_bytes() { return std::max(GEMM_SPLIT_WS_BYTES, gemm_skinny_ws_bytes()); }

// 256x256 tiles (k_gemm_256) or 128x128 (4 waves, 32x128 each); a last, partly filled round of workgroups is cut along K in
// either case.  The large tile moves half the operand bytes per flop but fills its last row of tiles less and starts more
// slowly, so it needs work: tile K slices in all (`work`), a long K, rows that fill the tiles, or rows at which the small
// tiles need a second round.  Measured, small / large, in us (rows x K x columns):
//   at least 8000 with more than 128 rows: 129 x 5120 x 27648 88 / 82, 512 rows 198 / 131; 129 x 3584 x 37888 87 / 82.
//   4000 with K of at least 8192 and 3072 columns: 129 x 13824 x 5120 47.6 / 44.9, 192 rows 56.1 / 51.4; 129 x 18944 x 3584
//   45.5 / 43.8; but 300 x 16384 x 2048 41.4 / 43.3, (2048) 512 x 8192 x 2048 36.7 / 42.9.  4000 with tiles at least 0.8 full: 448 x 5120 x 7168 58.9 / 52.8, but 320 rows
//   45.3 / 46.8, and with a short K 512 x 2048 x 16384 45.9 / 52.2.
//   3200 with more than 512 rows: 513 x 5120 x 5120 51.2 / 46.2, 513 x 5120 x 7168 80.3 / 63.2, 513 x 2048 x 16384 59.5 / 43.1,
//   513 x 6912 x 2560 39.3 / 39.2; but (3072) 513 x 4096 x 4096 34.7 / 36.9.  3000 with more than 600: 700 x 4096 x 4096 43.6 /
//   42.0; but (2352) 768 x 3584 x 3584 41.4 / 42.4, (1152) 513 x 2048 x 3072 23.2 / 30.5.
static bool big_tiles(int32_t M, int32_t K, const GemmB& B, int32_t rows) {
  int acc = 0;
  for (int p = 0; p < B.n_parts; ++p) {
    acc += B.n_rows[p];
    if (acc % 256) return false;
  }
  if (rows % 256 || K < 128) return false;  // (at least two K slices)
  const long tiles_m = (M + 255) / 256, work = tiles_m * (rows / 256) * (K / 64);
  return work >= 10000 || (work >= 8000 && M > 128) ||
         (work >= 4000 && ((K >= 8192 && rows >= 3072 && M > 128) || (K >= 3584 && M * 5L >= tiles_m * 256 * 4))) ||
         (work >= 3200 && M > 512) || (work >= 3000 && M > 600);
}

bool gemm_mfma_fuses_qkv(int32_t M, int32_t K, const GemmB& B, int32_t N, bool have_ws) {
  if (M <= 0 || N <= 0 || B.n_parts != 3) return false;
  if (have_ws && gemm_skinny_fits(M, K, B, N, EPI_QKV_ROPE)) return true;
  if (have_ws && gemm_skinny_fits(M, K, B, N, EPI_STORE_F32)) return false;
  // every part a whole number of 128-column heads, so that a wave's columns never straddle q / k / v
  return B.n_rows[0] % 128 == 0 && B.n_rows[1] % 128 == 0 && B.n_rows[2] % 128 == 0;
}

void launch_gemm_mfma(const bf16_t* A, int32_t M, int32_t K, const GemmB& B, const void* B2, int32_t N, int epilogue,
                      const bf16_t* residual, void* C, hipStream_t s, void* skinny_ws, const QkvEpilogue* qkv,
                      const RowNorm* norm, void* norm_out) {
  if (M <= 0 || N <= 0) return;
  if (gemm_stream_fits(M, K, B, N, epilogue, skinny_ws != nullptr) && aligned16(B2)) {
    launch_gemm_stream(A, M, K, B, B2, N, epilogue, residual, C, s, skinny_ws, qkv, norm, norm_out);
    return;
  }
  if (skinny_ws && gemm_skinny_fits(M, K, B, N, epilogue)) {
    launch_gemm_skinny(A, M, K, B, B2, N, epilogue, residual, C, skinny_ws, s, qkv, norm);
    return;
  }
  MfmaB b;
  b.n_parts = B.n_parts;
  int acc = 0;
  for (int p = 0; p < 3; ++p) {
    b.ptr[p] = p < B.n_parts ? reinterpret_cast<const bf16_t*>(B.ptr[p]) : nullptr;
    b.begin[p] = acc;
    if (p < B.n_parts) acc += B.n_rows[p];
  }
  b.begin[3] = acc;
  const bf16_t* b2 = reinterpret_cast<const bf16_t*>(B2);
  const int rows = epilogue == EPI_SWIGLU_STORE ? 2 * N : N;
  const QkvEpilogue qe = qkv ? *qkv : QkvEpilogue{};
  // (k_gemm_256 also loads the residual straight to LDS)
  if (big_tiles(M, K, B, rows) && parts_aligned16(B) && aligned16(B2) && aligned16(residual))
    launch_cfg<256, 256, 2, 2, 64, 2>(A, M, K, b, b2, N, epilogue, residual, C, s, skinny_ws, qe);
  else if (rows % 128 == 0)
    // (a wave as wide as the tile: a head per wave for the fused QKV epilogue, and where weights bound the launch the
    // waves whose rows lie past M drop out sooner: 64 x 5120 x 5120 20.5 us, 65 x 5120 x 27648 71.6 us, against 20.7
    // and 73.6 us with 64x64 per wave)
    launch_cfg<128, 128, 4, 1, 64, 2>(A, M, K, b, b2, N, epilogue, residual, C, s, skinny_ws, qe);
  else
    launch_cfg<64, 64, 1, 1, 64, 2>(A, M, K, b, b2, N, epilogue, residual, C, s, skinny_ws, qe);
}

}  // namespace keep
