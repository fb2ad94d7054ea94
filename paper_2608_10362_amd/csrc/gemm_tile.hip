// Compute-heavy GEMMs of passes of more than 64 rows (the verify blocks of
// many sequences, prefill chunks):  y[m, n] = s_m * sum_k W[n, k] x[m, k]  with
// bf16 weights from the packed image and x as the stacked bf16 operand its
// producer wrote (put_stacked: hi and lo parts, two products per weight
// fragment for float32 accuracy).
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "gemm_common.h"
#include "internal.h"

namespace specdec {

namespace {

constexpr int kReduceCols = kTileReduceCols;  // columns per block of the split-K reductions (and per ss partial)
constexpr int kMaxSs = 64;                    // ss partials a reduction sums

// Block = WM x WN waves over WM*MTW row tiles x WN*NTW weight tiles of 16; a
// wave owns MTW x NTW of them.  Both operands are already 1 KB fragments in
// MFMA order, so a stage (one k-step of 32: 2 KB of x per row tile, 1 KB per
// weight tile) is copied from memory to LDS as it is, by loads that do not
// pass the registers; ST stages are in flight.  A wave reads the next k-step's
// fragments while it multiplies the current ones, one barrier per k-step (7B
// gate|up, 512 rows: 155 us; reading and multiplying in turn 170).
// The weights are the A operand: D[4 (l/16) + r][l % 16] is weight row 4 (l/16)
// + r, x row l % 16, so each lane stores four consecutive columns of one row;
// a RoPE partner (column ^ 8) is lane ^ 32.
// Bound: the matrix units at the clock they hold (1.1 to 1.3 PFLOP/s of
// products; a large library bf16 product reaches 1.55 on the same card).  7B
// shapes, the reductions included, against staging float32 x through registers:
// 512 rows gate|up 308 -> 153 us, Q|K|V 182 -> 110, O 55 -> 42, down 120 -> 90;
// 112 rows gate|up 64 -> 55, Q|K|V 45 -> 43, O 29 -> 19.5, down 40 -> 32, LM head
// 91 -> 70 (there 3.3 to 3.7 TB/s of weights).
template <int WM, int WN, int MTW, int NTW, int ST, int KIND, bool KEYS>
__global__ __launch_bounds__(64 * WM * WN) void gemm_bf16_tile(GemmArgs a, int n_ctiles, int ks_per_split, int n_split) {
  constexpr int NW = WM * WN, MTB = WM * MTW, NTB = WN * NTW;  // row and weight tiles of the block
  constexpr bool SCALE = KIND != EPI_RESID, SWIGLU = KIND == EPI_SWIGLU;
  constexpr int XFR = 2 * MTB, FR = XFR + NTB;         // 1 KB fragments of a stage: x (hi, lo per row tile), weights
  constexpr int D0 = FR / NW, DX = FR % NW;            // pieces per wave (waves < DX: one more)
  __shared__ u32x4 s_f[ST][FR][kWave];
  __shared__ float scale[16 * MTB];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int wm = wave / WN, wn = wave % WN;
  const int K = a.K, KS = K / 32, M = a.M;
  const int n_rt = (M + 16 * MTB - 1) / (16 * MTB);
  // Blocks go to the 8 XCDs round-robin: the row tiles of one column tile sit 8
  // apart, so they share its weights through one L2 (the grid pads the column
  // tiles to a multiple of 8).
  const int per_split = n_rt * ((n_ctiles + 7) / 8 * 8);
  const int split = (int)blockIdx.x / per_split, bi = (int)blockIdx.x % per_split;
  const int rt = (bi / 8) % n_rt, ct = bi / (8 * n_rt) * 8 + bi % 8;
  if (ct >= n_ctiles) return;
  const int ks_begin = split * ks_per_split, n_k = min(KS, ks_begin + ks_per_split) - ks_begin;
  const int mt0 = rt * MTB, mts = (M + 15) / 16 - mt0;  // the block's first row tile, row tiles left

  // piece j of this wave: fragment f = wave + j * NW of the stage
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&s_f[0][0][0];
  const uint32_t xstep = (uint32_t)a.stt * 1024u;  // bytes of x per k-step
  __amdgpu_buffer_rsrc_t wr[D0 + 1];               // (pieces that are weights)
  uint32_t poff[D0 + 1];
#pragma unroll
  for (int j = 0; j <= D0; ++j) {
    const int f = wave + j * NW;
    // (row tiles past M and weight tiles past N re-read a valid one: their outputs are not stored)
    bool ok;
    const uint16_t* base = weight_tile(a, KIND, ct, 16 * NTB, f >= XFR && f < FR ? f - XFR : 0, KS, ok);
    wr[j] = make_rsrc(base, (uint32_t)KS * 1024u);
    poff[j] = f < XFR ? (2u * (mt0 + min(f >> 1, mts - 1)) + (f & 1)) * 1024u + lane * 16u
                      : (uint32_t)ks_begin * 1024u + lane * 16u;
  }
  auto issue = [&](int i) {  // k-step i of the range into stage i % ST (past the range: the last one again)
    const uint32_t dst = lds0 + (uint32_t)(i % ST) * (FR * 1024u) + wave * 1024u;
    const uint32_t k = (uint32_t)min(i, n_k - 1);
    const __amdgpu_buffer_rsrc_t xr = make_rsrc((const char*)a.xs + (size_t)(ks_begin + k) * xstep, xstep);
#pragma unroll
    for (int j = 0; j <= D0; ++j) {
      if (j == D0 && (DX == 0 || wave >= DX)) break;
      if (wave + j * NW < XFR) load_lds16(dst + j * (NW * 1024u), poff[j], xr);  // (wave-uniform)
      else load_lds16(dst + j * (NW * 1024u), poff[j] + k * 1024u, wr[j]);
    }
  };
  auto wait_stages = [&](auto n) {  // at most n stages' pieces still outstanding
    constexpr int S = decltype(n)::value;
    if (DX != 0 && wave < DX) wait_vm<S * (D0 + 1)>();
    else wait_vm<S * D0>();
  };
  // weight tile j of this wave (SwiGLU: the wave's gate tiles, then the up tiles of the same columns)
  auto btile = [&](int j) {
    return SWIGLU ? (j < NTW / 2 ? wn * (NTW / 2) + j : NTB / 2 + wn * (NTW / 2) + j - NTW / 2) : wn * NTW + j;
  };
  struct Frags {
    u32x4 x[MTW][2], w[NTW];
  };
  auto read = [&](int i, Frags& r) {
    const u32x4(*st)[kWave] = s_f[i % ST];
#pragma unroll
    for (int m = 0; m < MTW; ++m) {
      r.x[m][0] = st[2 * (wm * MTW + m)][lane];
      r.x[m][1] = st[2 * (wm * MTW + m) + 1][lane];
    }
#pragma unroll
    for (int j = 0; j < NTW; ++j) r.w[j] = st[XFR + btile(j)][lane];
  };
  // KEYS (the Q|K|V projections, whose results are rounded to bf16): blocks of at
  // most 128 rows sum hi and lo products apart.  In one accumulator every product
  // of the small lo part rounds the large sum once more (keys and values of a
  // first layer, 120 rows of the 7B shape, that fall on the other bf16 side of
  // their 64-bit value, per 1e5: 37 in one, 27 apart).  Blocks of 256 rows have no
  // registers for it.
  constexpr int HL = KEYS && 16 * MTB <= 128 ? 2 : 1;
  floatx4 acc[MTW][NTW], acl[HL == 2 ? MTW : 1][HL == 2 ? NTW : 1];
#pragma unroll
  for (int m = 0; m < MTW; ++m)
#pragma unroll
    for (int j = 0; j < NTW; ++j) {
      acc[m][j] = floatx4{0.f, 0.f, 0.f, 0.f};
      if constexpr (HL == 2) acl[m][j] = floatx4{0.f, 0.f, 0.f, 0.f};
    }
  auto multiply = [&](const Frags& r) {
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int m = 0; m < MTW; ++m)
#pragma unroll
        for (int j = 0; j < NTW; ++j) {
          floatx4& s = HL == 2 && h == 1 ? acl[HL == 2 ? m : 0][HL == 2 ? j : 0] : acc[m][j];
          s = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, r.w[j]),
                                                      __builtin_bit_cast(bf16x8, r.x[m][h]), s, 0, 0, 0);
        }
  };

#pragma unroll
  for (int i = 0; i < ST; ++i) issue(i);
  if constexpr (SCALE) {
    for (int m = tid; m < 16 * MTB; m += 64 * NW) {
      const int row = mt0 * 16 + m;
      float t = 0.f;
      if (a.ss_in && row < M)
        for (int p = 0; p < a.n_ss; ++p) t += a.ss_in[(size_t)p * a.ss_ld + row];
      scale[m] = a.ss_in && row < M ? 1.0f / sqrtf(t / (float)K + a.eps) : 1.0f;
    }
  }
  Frags ra, rb;
  wait_stages(std::integral_constant<int, ST - 1>{});
  __builtin_amdgcn_s_barrier();
  read(0, ra);
  for (int i = 0; i < n_k; i += 2) {
#pragma unroll
    for (int u = 0; u < 2; ++u) {
      if (i + u >= n_k) break;
      wait_stages(std::integral_constant<int, ST - 2>{});
      asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
      __builtin_amdgcn_s_barrier();
      issue(i + u + ST);
      if (u == 0) {
        read(i + 1, rb);
        multiply(ra);
      } else {
        read(i + 2, ra);
        multiply(rb);
      }
      // the next step's fragment reads spread over this step's products
      constexpr int NR = 2 * MTW + NTW, NM = 2 * MTW * NTW, PER = NM / NR;
#pragma unroll
      for (int k = 0; k < NR; ++k) {
        __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x008, PER, 0);
      }
      __builtin_amdgcn_sched_group_barrier(0x008, NM - NR * PER, 0);
    }
  }
  if constexpr (HL == 2) {
#pragma unroll
    for (int m = 0; m < MTW; ++m)
#pragma unroll
      for (int j = 0; j < NTW; ++j) acc[m][j] += acl[m][j];
  }
  wait_vm<0>();  // (the re-read stages past the range have landed before the block can end)
  __syncthreads();

  const int cl = lane & 15, rg = lane >> 4;
#pragma unroll
  for (int i = 0; i < MTW; ++i) {
    const int ml = (wm * MTW + i) * 16 + cl, m = mt0 * 16 + ml;
    const float sc = SCALE ? scale[ml] : 1.f;
#pragma unroll
    for (int j = 0; j < (SWIGLU ? NTW / 2 : NTW); ++j) {
      f32x4 y = __builtin_bit_cast(f32x4, acc[i][j]);
      if constexpr (KIND == EPI_RESID) {
        const int n = ct * 16 * NTB + 16 * btile(j) + 4 * rg;
        if (m < M && n < a.n_rows) *(f32x4*)(a.ypart + ((size_t)split * M + m) * a.n_rows + n) = y;
      } else if constexpr (KIND == EPI_STORE) {
        const int n = ct * 16 * NTB + 16 * btile(j) + 4 * rg;
        if (m < M && n < a.n_rows) *(f32x4_a4*)(a.out + (size_t)m * a.ldo + n) = y * sc;
      } else if constexpr (SWIGLU) {
        const int n = ct * 8 * NTB + 16 * btile(j) + 4 * rg;
        if (m < M && n < a.n_rows) {
          const f32x4 yu = __builtin_bit_cast(f32x4, acc[i][j + NTW / 2]);
          f32x4 o;
#pragma unroll
          for (int e = 0; e < 4; ++e) o[e] = silu_f(y[e] * sc) * (yu[e] * sc);
          put_stacked4(a.xs_out, a.stt_out, m, n, o);
        }
      } else {
        const int n = ct * 16 * NTB + 16 * btile(j) + 4 * rg;
        y *= sc;
        f32x4 z;
#pragma unroll
        for (int e = 0; e < 4; ++e) z[e] = __shfl_xor(y[e], 32, kWave);
        if (m < M && n < a.n_rows) qkv_store4(a, m, n, y, z);
      }
    }
  }
}

// Split-K partial sums of 4 columns of one row, added in split order; every
// split's load is issued before the first add (the split index is clamped, so
// loads past n_split re-read the last split and are not added).
template <int NS>
__device__ __forceinline__ f32x4 sum_splits_n(const float* yp, size_t split_stride, int n_split) {
  f32x4 v[NS];
#pragma unroll
  for (int s = 0; s < NS; ++s) v[s] = *(const f32x4*)(yp + (size_t)min(s, n_split - 1) * split_stride);
  f32x4 y = f32x4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int s = 0; s < NS; ++s)
    if (s < n_split) y += v[s];
  return y;
}
__device__ __forceinline__ f32x4 sum_splits(const float* yp, size_t split_stride, int n_split) {
  if (n_split <= 4) return sum_splits_n<4>(yp, split_stride, n_split);  // (block-uniform)
  if (n_split <= 8) return sum_splits_n<8>(yp, split_stride, n_split);
  return sum_splits_n<kTileSplitMax>(yp, split_stride, n_split);
}

// RMSNorm scales of rows m0 .. m0+7 into s_scale: the block loads every
// partial sum of squares at once (two per thread), then thread r < 8 adds its
// row's in partial order.
__device__ __forceinline__ void row_scales8(const GemmArgs& a, int m0, float* s_scale, float (*s_ss)[kMaxSs]) {
  const int tid = threadIdx.x;
  float v[2];
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + 256 * k, r = i / kMaxSs, p = i % kMaxSs, m = m0 + r;
    v[k] = a.ss_in && p < a.n_ss && m < a.M ? a.ss_in[(size_t)p * a.ss_ld + m] : 0.f;
  }
#pragma unroll
  for (int k = 0; k < 2; ++k) {
    const int i = tid + 256 * k;
    s_ss[i / kMaxSs][i % kMaxSs] = v[k];
  }
  __syncthreads();
  if (tid < 8) {
    float ss = 0.f;
    for (int p = 0; p < a.n_ss; ++p) ss += s_ss[tid][p];
    s_scale[tid] = a.ss_in ? 1.0f / sqrtf(ss / (float)a.K + a.eps) : 1.0f;
  }
  __syncthreads();
}
static_assert(8 * kMaxSs == 512, "row_scales8: two partials per thread of a 256-thread block");

// Sum of the split-K partials of a residual GEMM in split order, residual
// add, next RMSNorm input and its sums of squares.  Block = 128 columns x 8
// rows; thread = 4 columns of one row; ss partial p = column block p.
__global__ __launch_bounds__(256) void resid_reduce_kernel(GemmArgs a, int n_split) {
  const int tid = threadIdx.x, m = (int)blockIdx.y * 8 + (tid >> 5);
  const int n = (int)blockIdx.x * kReduceCols + 4 * (tid & 31);
  const int M = a.M;
  float t = 0.f;
  if (m < M && n < a.n_rows) {
    const f32x4 y = sum_splits(a.ypart + (size_t)m * a.n_rows + n, (size_t)M * a.n_rows, n_split);
    float* hp = a.out + (size_t)m * a.ldo + n;
    const f32x4 h = *(const f32x4*)hp + y;
    *(f32x4*)hp = h;
    const uint16_t* g = (const uint16_t*)a.gain_out + n;
    const f32x4 x = f32x4{h[0] * bf16_bits_to_f32(g[0]), h[1] * bf16_bits_to_f32(g[1]), h[2] * bf16_bits_to_f32(g[2]),
                          h[3] * bf16_bits_to_f32(g[3])};
    put_stacked4(a.xs_out, a.stt_out, m, n, x);
    t = h[0] * h[0] + h[1] * h[1] + h[2] * h[2] + h[3] * h[3];
  }
#pragma unroll
  for (int o = 16; o > 0; o >>= 1) t += __shfl_xor(t, o, kWave);
  if ((tid & 31) == 0 && m < M) a.ss_out[(size_t)blockIdx.x * a.ss_ld + m] = t;
}

// Sum of the split-K partial sums of a pass's gate and up projections
// (rows [0, F) and [F, 2F) of the partials) in split order, times the row's
// RMSNorm scale, then SwiGLU.  Block = 128 columns x 8 rows; thread = 4 columns of one row.
__global__ __launch_bounds__(256) void swiglu_reduce_kernel(GemmArgs a, int n_split) {
  __shared__ float s_scale[8];
  __shared__ float s_ss[8][kMaxSs];
  const int tid = threadIdx.x, m = (int)blockIdx.y * 8 + (tid >> 5);
  const int f = (int)blockIdx.x * kReduceCols + 4 * (tid & 31);
  const int M = a.M, F = a.n_rows, W = 2 * F;
  // (the splits' loads are issued before the row scales wait for anything)
  const float* yp = a.ypart + (size_t)min(m, M - 1) * W + min(f, F - 4);
  const f32x4 gs = sum_splits(yp, (size_t)M * W, n_split), us = sum_splits(yp + F, (size_t)M * W, n_split);
  row_scales8(a, (int)blockIdx.y * 8, s_scale, s_ss);
  if (m >= M || f >= F) return;
  const float sc = s_scale[tid >> 5];
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = silu_f(gs[e] * sc) * (us[e] * sc);
  put_stacked4(a.xs_out, a.stt_out, m, f, o);
}

// Sum of the split-K partial sums of a pass's Q|K|V projections in split
// order, times the row's RMSNorm scale, then RoPE on the Q and K columns and
// the stores: rotated queries to qr, rotated keys and the values appended to
// the KV cache (valid rows).  Q and K columns come in the packed RoPE order:
// column c of a head's 16-column tile tq is dim 8tq + c for c < 8, hd/2 + 8tq
// + c - 8 otherwise, so each column's rotation partner (c ^ 8) is 8 columns
// away, in the lane ^ 2 of the row's 32 threads.  Block = 128 columns x 8
// rows; thread = 4 columns of one row.
__global__ __launch_bounds__(256) void qkv_reduce_kernel(GemmArgs a, int n_split) {
  __shared__ float s_scale[8];
  __shared__ float s_ss[8][kMaxSs];
  const int tid = threadIdx.x, m = (int)blockIdx.y * 8 + (tid >> 5);
  const int n = (int)blockIdx.x * kReduceCols + 4 * (tid & 31);
  const int M = a.M;
  const bool live = m < M && n < a.n_rows;
  // (the splits' loads are issued before the row scales wait for anything)
  f32x4 y = sum_splits(a.ypart + (size_t)min(m, M - 1) * a.n_rows + min(n, a.n_rows - 4), (size_t)M * a.n_rows, n_split);
  row_scales8(a, (int)blockIdx.y * 8, s_scale, s_ss);
  const float sc = s_scale[tid >> 5];
  f32x4 z;  // (every lane takes part in the shuffles)
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    y[e] *= sc;
    z[e] = __shfl_xor(y[e], 2, kWave);
  }
  if (live) qkv_store4(a, m, n, y, z);
}


// ---------------------------------------------------------------- launchers
struct TileShape {
  int rows, cols;  // of a block
  float us;        // per k-step, every CU at work (measured over the 7B shapes, 256 and 512 rows)
};
constexpr TileShape kShapes[] = {{256, 192, 1.18f}, {256, 128, 0.90f}, {256, 96, 0.69f}, {128, 192, 0.67f},
                                 {128, 128, 0.45f}, {128, 96, 0.42f},  {96, 192, 0.60f}, {96, 128, 0.40f}};
constexpr int kNumShapes = sizeof(kShapes) / sizeof(kShapes[0]);

struct TilePlan {
  int shape = -1, n_split = 1, per = 0;
};

// Block shape and K split of a GEMM over n output columns: the least of rounds
// of the grid x (k-steps x the shape's time per k-step + a block's fixed 4 us)
// + the partial sums' way to memory and back and their reduction launch.  A
// k-step takes no less than its weights at the rate the blocks stream them
// (about 16 bytes per ns and CU; the row tiles of a column share them).
// always_reduce: the GEMM ends in a reduction also without a split.
TilePlan plan_tile(int M, int n, int KS, bool pairs, bool can_split, bool always_reduce, size_t part_floats) {
  const int cus = device_compute_units();
  TilePlan best;
  float best_us = 0.f;
  for (int c = 0; c < kNumShapes; ++c) {
    const TileShape& t = kShapes[c];
    if (t.rows == 96 && M > 96) continue;
    const int rt = (M + t.rows - 1) / t.rows, ct = (n + t.cols - 1) / t.cols;
    const float step = std::max(t.us, (float)t.cols * 64.f / 16e3f / (float)rt);
    for (int s = 1; s <= (can_split ? kTileSplitMax : 1); ++s) {
      const int per = (KS + s - 1) / s;
      if ((KS + per - 1) / per != s) continue;
      const bool reduce = s > 1 || always_reduce;
      if (reduce && (size_t)s * M * n > part_floats) continue;
      if (pairs && s == 1 && (c == 5 || c == 6)) continue;  // (a wave's tiles must be whole gate / up pairs)
      const int rounds = (rt * ct * s + cus - 1) / cus;
      const float us = rounds * (per * step + 4.f) + (reduce ? 3.f + (float)s * M * n * 8e-6f / 4.f : 0.f);
      if (best.shape < 0 || us < best_us) {
        best_us = us;
        best = TilePlan{c, s, per};
      }
    }
  }
  return best;
}

template <int WM, int WN, int MTW, int NTW, int ST, int KIND, bool KEYS>
void launch_shape(const GemmArgs& a, const TilePlan& p, hipStream_t s) {
  constexpr int BM = 16 * WM * MTW, BN = (KIND == EPI_SWIGLU ? 8 : 16) * WN * NTW;
  const int rt = (a.M + BM - 1) / BM, ct = (a.n_rows + BN - 1) / BN;
  hipLaunchKernelGGL((gemm_bf16_tile<WM, WN, MTW, NTW, ST, KIND, KEYS>), dim3(rt * ((ct + 7) / 8 * 8) * p.n_split),
                     dim3(64 * WM * WN), 0, s, a, ct, p.per, p.n_split);
}
template <int KIND, bool KEYS = false>
hipError_t launch_plan(const GemmArgs& a, const TilePlan& p, hipStream_t s) {
  switch (p.shape) {
    case 0: launch_shape<4, 2, 4, 6, 3, KIND, KEYS>(a, p, s); break;
    case 1: launch_shape<4, 2, 4, 4, 3, KIND, KEYS>(a, p, s); break;
    case 2: launch_shape<8, 1, 2, 6, 4, KIND, KEYS>(a, p, s); break;
    case 3: launch_shape<4, 2, 2, 6, 4, KIND, KEYS>(a, p, s); break;
    case 4: launch_shape<2, 4, 4, 2, 4, KIND, KEYS>(a, p, s); break;
    case 7: launch_shape<2, 4, 3, 2, 4, KIND, KEYS>(a, p, s); break;
    default:
      if constexpr (KIND != EPI_SWIGLU) {
        if (p.shape == 5) launch_shape<4, 2, 2, 3, 4, KIND, KEYS>(a, p, s);
        else if (p.shape == 6) launch_shape<2, 4, 3, 3, 4, KIND, KEYS>(a, p, s);
        else return hipErrorInvalidValue;
        break;
      }
      return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

dim3 reduce_grid(const GemmArgs& a) { return dim3((a.n_rows + kReduceCols - 1) / kReduceCols, (a.M + 7) / 8); }

}  // namespace

size_t tile_ypart_floats(int d_model) { return (size_t)kTilePartialRows * d_model; }

hipError_t launch_resid_reduce(const GemmArgs& a, int n_split, hipStream_t s) {
  hipLaunchKernelGGL(resid_reduce_kernel, reduce_grid(a), dim3(256), 0, s, a, n_split);
  return hipGetLastError();
}

hipError_t launch_gemm_tile(const GemmArgs& a, hipStream_t s) {
  if (a.M > kTileLaunchRows || !a.xs || a.stt < 2 * ((a.M + 15) / 16) || a.K % 32 || a.n_rows % 16 || !a.ypart ||
      (a.ss_in && a.n_ss > kMaxSs))
    return hipErrorInvalidValue;
  const int KS = a.K / 32;
  switch (a.kind) {
    case EPI_STORE:
      return launch_plan<EPI_STORE>(a, plan_tile(a.M, a.n_rows, KS, false, false, false, 0), s);
    case EPI_RESID: {
      if (!a.xs_out || !a.gain_bf16) return hipErrorInvalidValue;
      const TilePlan p = plan_tile(a.M, a.n_rows, KS, false, true, true, a.ypart_floats);
      const hipError_t e = launch_plan<EPI_RESID>(a, p, s);
      return e != hipSuccess ? e : launch_resid_reduce(a, p.n_split, s);
    }
    case EPI_QKV: {
      if (a.kv.dtype != SPECDEC_BF16 || a.head_dim % 16 || a.n_seg[0] % a.head_dim || a.n_seg[1] % a.head_dim)
        return hipErrorInvalidValue;
      const TilePlan p = plan_tile(a.M, a.n_rows, KS, false, true, false, a.ypart_floats);
      if (p.n_split == 1) return launch_plan<EPI_QKV, true>(a, p, s);
      GemmArgs g = a;
      g.kind = EPI_RESID;
      const hipError_t e = launch_plan<EPI_RESID, true>(g, p, s);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(qkv_reduce_kernel, reduce_grid(a), dim3(256), 0, s, a, p.n_split);
      return hipGetLastError();
    }
    case EPI_SWIGLU: {
      if (!a.xs_out) return hipErrorInvalidValue;
      const int W = 2 * a.n_rows;
      const TilePlan p = plan_tile(a.M, W, KS, true, true, false, a.ypart_floats);
      if (p.n_split == 1) return launch_plan<EPI_SWIGLU>(a, p, s);
      GemmArgs g = a;  // the gate and up rows as one 2F-row matrix, raw partial sums
      g.kind = EPI_RESID;
      g.n_rows = W;
      g.n_seg[0] = a.n_rows;
      g.n_seg[1] = a.n_rows;
      g.n_seg[2] = 0;
      const hipError_t e = launch_plan<EPI_RESID>(g, p, s);
      if (e != hipSuccess) return e;
      hipLaunchKernelGGL(swiglu_reduce_kernel, reduce_grid(a), dim3(256), 0, s, a, p.n_split);
      return hipGetLastError();
    }
    default: return hipErrorInvalidValue;
  }
}

}  // namespace specdec
