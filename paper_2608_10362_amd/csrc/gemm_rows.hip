// Weight-streaming GEMMs of passes of at most 64 rows (verify blocks, draft
// steps, catch-up and small prefill chunks):
//   y[m, n] = s_m * sum_k W[n, k] x[m, k]
// with bf16 weights from the packed image and x handed over by its producer
// as the stacked bf16 operand (put_stacked: hi and lo parts, x = hi + lo +
// O(2^-17 |x|)), so two products per weight fragment give a float32-accuracy
// result and no kernel converts x again.
#include <algorithm>

#include "device_common.h"
#include "gemm_common.h"
#include "internal.h"

namespace specdec {

namespace {

// One k-step's INT4 code word (8 columns of the lane's row, column e in bits
// 4e..4e+3) as bf16 operands 24 + q in column order: the sign bit flipped makes
// a nibble q + 8, which as the top mantissa bits of 16.0 (0x4180 | (q + 8) << 3)
// is 16 + (q + 8).
__device__ __forceinline__ bf16x8 q4_operand24(uint32_t w) {
  const uint32_t c = w ^ 0x88888888u, lo = c << 3, hi = c >> 1;  // even / odd columns' nibbles at bits 3..6 of their byte
  u32x4 v;
  v[0] = (__builtin_amdgcn_perm(hi, lo, 0x0c040c00u) & 0x00780078u) | 0x41804180u;
  v[1] = (__builtin_amdgcn_perm(hi, lo, 0x0c050c01u) & 0x00780078u) | 0x41804180u;
  v[2] = (__builtin_amdgcn_perm(hi, lo, 0x0c060c02u) & 0x00780078u) | 0x41804180u;
  v[3] = (__builtin_amdgcn_perm(hi, lo, 0x0c070c03u) & 0x00780078u) | 0x41804180u;
  return __builtin_bit_cast(bf16x8, v);
}

// The value of lane ^ 8 (a rotation by 8 within each row of 16 lanes; no LDS round trip).
__device__ __forceinline__ float row_half_swap(float v) {
  return __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xF, 0xF, false));
}

// Block = NW waves, a work unit = T tiles of 16 weight rows over a range of
// k-steps; the unit's k-steps are dealt out to the waves (wave w: w, w + NW,
// ...) and every wave holds the whole unit's T x MT accumulator tiles in
// registers.  So each x fragment is read once per block, straight into the
// registers of the one wave that multiplies it: no staging, no barrier in the
// loop, and 2 MT / T bytes of x (from L2) per weight byte.  Two register
// buffers of UB k-steps keep the next loads, including the next unit's, in
// flight during the products and the epilogue.  Then the waves' sums are added
// in wave order through LDS, each wave finishing whole fragments.
// The weights are the A operand: D[4 (l/16) + r][l % 16] is weight row 4
// (l/16) + r, x row l % 16, so a lane ends with four consecutive columns of
// one row and stores them at once; a RoPE partner (column ^ 8) is lane ^ 32.
// Q4 (INT4 weights): a batch is one group of 128 columns, its codes one 1 KB
// block per tile and its x the fragments of four k-steps (UB = 4).  A code q
// is fed to the products as the bf16 value 24 + q (q4_operand24), the bias is
// cancelled by the product of the same x with -24, shared by the unit's tiles,
// and a group's sum is multiplied by the row's group scale in float32.
// Over at most 16 rows, and in Q|K|V, the hi and lo parts are summed apart and
// added once per unit and wave (APART): in one accumulator every product of the
// small lo part rounds the large sum once more.  Keys and values of a first
// layer that fall on the other bf16 side of their 64-bit value, per 1e5, in one
// accumulator and apart: 8 rows of the 1.1B and the 7B shape 17 and 21, 9 and 16;
// 24 rows 21 and 23, 12 and 16.  (Above 16 rows the other results are not rounded
// to bf16, the logits' error is the same either way, and twice the accumulators
// cost up to 5%.)  XF = 1 (at most 8 rows) has both parts in one fragment, hi in
// x rows 0-7 and lo in rows 8-15 of one product, XF = 2 in two; the sums are the
// same, so a block of rows equals its rows run one by one.
template <int T, int MT, int NW, int UB, int KIND, bool Q4, int XF, bool PEEL>
__global__ __launch_bounds__(64 * NW) void gemm_bf16_rows(GemmArgs a, int n_units, int n_split, int ks_per_split) {
  constexpr int NC = 16 * T, MP = 16 * MT;
  constexpr bool APART = MT == 1 || (!Q4 && KIND == EPI_QKV);
  constexpr int MA = APART ? XF : MT;  // accumulator tiles per weight tile
  static_assert(XF == 2 * MT || (MT == 1 && XF == 1), "fragments of x per k-step");
  constexpr bool SCALE = KIND != EPI_RESID, SWIGLU = KIND == EPI_SWIGLU;
  // fragments per reduction round (a SwiGLU round holds whole gate / up pairs)
  constexpr int RMAX = 128 / NW;
  constexpr int RT = T * MT <= RMAX ? MT : (RMAX / T > 0 ? RMAX / T : 1);  // row tiles per round
  __shared__ f32x4 red[RT * T][NW][kWave];
  __shared__ float scale[MP];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int K = a.K, KS = K / 32, M = a.M;
  const int KG = (K + 127) / 128;  // (Q4: groups)
  const int split = (int)blockIdx.x % n_split, u0 = (int)blockIdx.x / n_split, us = (int)gridDim.x / n_split;
  const int ks_begin = split * ks_per_split, n_k = min(Q4 ? KG : KS, ks_begin + ks_per_split) - ks_begin;
  const int my_ks = n_k > wave ? (n_k - wave + NW - 1) / NW : 0;
  const int nbat = Q4 ? max(1, my_ks) : max(1, (my_ks + UB - 1) / UB);  // (Q4: "k-steps" of the range are groups)
  const int my_units = (n_units - u0 + us - 1) / us;
  const int total = my_units * nbat;

  floatx4 acc[MA][T];
#pragma unroll
  for (int mt = 0; mt < MA; ++mt)
#pragma unroll
    for (int t = 0; t < T; ++t) acc[mt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  constexpr int WB = Q4 ? 1 : UB;  // weight pieces per tile and batch
  u32x4 wA[WB][T], wB[WB][T], xA[UB][XF], xB[UB][XF];
  u32x2 sA[Q4 ? T : 1], sB[Q4 ? T : 1];  // Q4: bf16 scales of the lane's four weight rows

  // (the lanes of rows past M read nothing and hold zeros)
  const uint32_t xlast = (uint32_t)(16 * (MT - 1) + (lane & (XF == 1 ? 7 : 15)) >= M) << 31;
  const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.xs, (uint32_t)KS * XF * 1024u);
  int lu = u0, lb = 0;  // load cursor: unit, batch
  auto load = [&](u32x4 (&wv)[WB][T], u32x4 (&xv)[UB][XF], u32x2 (&sv)[Q4 ? T : 1]) {
    if constexpr (Q4) {
      const int i = min(lb, max(my_ks - 1, 0));
      const uint32_t gr = (uint32_t)(ks_begin + wave + i * NW);
      const uint32_t bad = (uint32_t)(lb >= my_ks) << 31;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        int seg, n;
        bool ok;
        tile_segment(a, KIND, lu, NC, t, seg, n, ok);
        const __amdgpu_buffer_rsrc_t wr =
            make_rsrc((const char*)a.w[seg] + (size_t)(n / 16) * KG * 1024, ok ? (uint32_t)KG * 1024u : 0u);
        wv[0][t] = __builtin_amdgcn_raw_buffer_load_b128(wr, (gr * 1024u + lane * 16u) | bad, 0, kNonTemporal);
        // (a tile or group past the end reads the scales of a valid one; its x or its columns are not used)
        sv[t] = *(const u32x2*)(a.wscale[seg] + ((size_t)(n / 16) * KG + min(gr, (uint32_t)KG - 1u)) * 16 + 4 * (lane >> 4));
      }
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int f = 0; f < XF; ++f) {
          const uint32_t xoff = (((4 * gr + u) * XF + f) * 1024u + lane * 16u) | bad | (f >= XF - 2 ? xlast : 0u);
          xv[u][f] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff, 0, 0);
        }
    } else {
      __amdgpu_buffer_rsrc_t wr[T];
#pragma unroll
      for (int t = 0; t < T; ++t) {
        bool ok;
        const uint16_t* base = weight_tile(a, KIND, lu, NC, t, KS, ok);
        wr[t] = make_rsrc(base, ok ? (uint32_t)KS * 1024u : 0u);
      }
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const int i = lb * UB + u;
        const uint32_t ks = (uint32_t)(ks_begin + wave + i * NW);
        const uint32_t bad = (uint32_t)(i >= my_ks) << 31;
        const uint32_t woff = (ks * 1024u + lane * 16u) | bad;
#pragma unroll
        for (int t = 0; t < T; ++t) wv[u][t] = __builtin_amdgcn_raw_buffer_load_b128(wr[t], woff, 0, kNonTemporal);
#pragma unroll
        for (int f = 0; f < XF; ++f) {
          const uint32_t xoff = ((ks * XF + f) * 1024u + lane * 16u) | bad | (f >= XF - 2 ? xlast : 0u);
          xv[u][f] = __builtin_amdgcn_raw_buffer_load_b128(xr, xoff, 0, 0);
        }
      }
    }
    if (++lb == nbat) { lb = 0; lu += us; }
  };
  auto compute = [&](const u32x4 (&wv)[WB][T], const u32x4 (&xv)[UB][XF], const u32x2 (&sv)[Q4 ? T : 1]) {
    if constexpr (Q4) {
      const bf16x8 m24 = __builtin_bit_cast(bf16x8, u32x4{0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u, 0xC1C0C1C0u});
      floatx4 pb[MT];
#pragma unroll
      for (int mt = 0; mt < MT; ++mt) pb[mt] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int u = 0; u < 4; ++u)
#pragma unroll
        for (int h = 0; h < 2; ++h)
#pragma unroll
          for (int mt = 0; mt < MT; ++mt)
            pb[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(m24, __builtin_bit_cast(bf16x8, xv[u][2 * mt + h]), pb[mt],
                                                             0, 0, 0);
#pragma unroll
      for (int t = 0; t < T; ++t) {
        floatx4 p[MT];
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) p[mt] = pb[mt];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
          const bf16x8 w = q4_operand24(wv[0][t][u]);
#pragma unroll
          for (int h = 0; h < 2; ++h)
#pragma unroll
            for (int mt = 0; mt < MT; ++mt)
              p[mt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(w, __builtin_bit_cast(bf16x8, xv[u][2 * mt + h]), p[mt], 0,
                                                              0, 0);
        }
        const float s4[4] = {__uint_as_float(sv[t][0] << 16), __uint_as_float(sv[t][0] & 0xffff0000u),
                             __uint_as_float(sv[t][1] << 16), __uint_as_float(sv[t][1] & 0xffff0000u)};
#pragma unroll
        for (int mt = 0; mt < MT; ++mt)
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[mt][t][r] = fmaf(s4[r], p[mt][r], acc[mt][t][r]);
      }
    } else {
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int h = 0; h < XF / MA; ++h)
#pragma unroll
          for (int mt = 0; mt < MA; ++mt)
#pragma unroll
            for (int t = 0; t < T; ++t)
              acc[mt][t] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8, wv[u][t]),
                                                                   __builtin_bit_cast(bf16x8, xv[u][XF / MA * mt + h]),
                                                                   acc[mt][t], 0, 0, 0);
    }
  };

  // One finished fragment: y[r] = column n + r of row m (sums over all waves).
  const int cl = lane & 15, rg = lane >> 4;
  auto emit = [&](int unit, int mt, int t, f32x4 y, f32x4 yu) {
    const int m = mt * 16 + cl;
    if constexpr (KIND == EPI_RESID) {
      const int n = unit * NC + 16 * t + 4 * rg;
      if (m < M && n < a.n_rows) *(f32x4*)(a.ypart + ((size_t)split * M + m) * a.n_rows + n) = y;
    } else if constexpr (KIND == EPI_STORE) {
      const int n = unit * NC + 16 * t + 4 * rg;
      if (m < M && n < a.n_rows) *(f32x4_a4*)(a.out + (size_t)m * a.ldo + n) = y * scale[m];
    } else if constexpr (SWIGLU) {
      const int n = unit * (NC / 2) + 16 * t + 4 * rg;
      if (m < M && n < a.n_rows) {
        const float sc = scale[m];
        f32x4 o;
#pragma unroll
        for (int e = 0; e < 4; ++e) o[e] = silu_f(y[e] * sc) * (yu[e] * sc);
        put_stacked4(a.xs_out, a.stt_out, m, n, o);
      }
    } else {
      const int n = unit * NC + 16 * t + 4 * rg;
      y *= m < M ? scale[m] : 0.f;
      f32x4 z;  // (every lane takes part in the shuffles)
#pragma unroll
      for (int e = 0; e < 4; ++e) z[e] = __shfl_xor(y[e], 32, kWave);
      if (m < M && n < a.n_rows) qkv_store4(a, m, n, y, z);
    }
  };
  auto finish = [&](int unit) {
    if constexpr (APART) {  // hi + lo (XF = 1: of row m in lanes of rows m and 8 + m)
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if constexpr (XF == 1) {
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[0][t][r] += row_half_swap(acc[0][t][r]);
        } else {
#pragma unroll
          for (int mt = 0; mt < MT; ++mt) acc[mt][t] = acc[2 * mt][t] + acc[2 * mt + 1][t];
        }
      }
    }
#pragma unroll
    for (int m0 = 0; m0 < MT; m0 += RT) {
#pragma unroll
      for (int i = 0; i < RT; ++i)
#pragma unroll
        for (int t = 0; t < T; ++t)
          if (m0 + i < MT) red[i * T + t][wave][lane] = acc[m0 + i][t];
      __syncthreads();
      constexpr int PF = SWIGLU ? T / 2 : T;  // outputs (or pairs) per row tile
      for (int f = wave; f < RT * PF; f += NW) {
        const int i = f / PF, t = f % PF;
        if (m0 + i < MT) {
          f32x4 y = red[i * T + t][0][lane], yu = y;
#pragma unroll
          for (int w = 1; w < NW; ++w) y += red[i * T + t][w][lane];
          if constexpr (SWIGLU) {
            yu = red[i * T + T / 2 + t][0][lane];
#pragma unroll
            for (int w = 1; w < NW; ++w) yu += red[i * T + T / 2 + t][w][lane];
          }
          emit(unit, m0 + i, t, y, yu);
        }
      }
      __syncthreads();
    }
#pragma unroll
    for (int mt = 0; mt < MA; ++mt)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[mt][t] = floatx4{0.f, 0.f, 0.f, 0.f};
  };

  // Prologue: the row-scale partial sums are requested before the weights
  // (loads complete in order), then both buffers.
  constexpr int RS = (MP + NW - 1) / NW;  // scale rows per wave
  constexpr int RP = MT == 1 ? 4 : 1;     // partial sums per lane held (passes of at most 16 rows: one per 16 columns)
  float rs[SCALE ? RS : 1][RP];
  if constexpr (SCALE) {
    const __amdgpu_buffer_rsrc_t sr = make_rsrc(a.ss_in, a.ss_in ? (uint32_t)a.n_ss * a.ss_ld * 4u : 0u);
#pragma unroll
    for (int r = 0; r < RS; ++r)
#pragma unroll
      for (int i = 0; i < RP; ++i) {
        const int m = wave + r * NW, p = lane + i * kWave;
        const uint32_t off = ((uint32_t)p * a.ss_ld + m) * 4u | ((uint32_t)(m >= M || p >= a.n_ss) << 31);
        rs[r][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, off, 0, 0));
      }
  }
  load(wA, xA, sA);
  if (PEEL || total > 1) load(wB, xB, sB);  // (PEEL, past the last batch: weights out of range)
  if constexpr (SCALE) {
    // s_m = 1/sqrt(sum_p ss[p][m] / K + eps): partial p in lane p % 64, in p order, fixed shuffle tree
    float t[RS];
#pragma unroll
    for (int r = 0; r < RS; ++r) {
      const int m = wave + r * NW;
      t[r] = rs[r][0];
#pragma unroll
      for (int i = 1; i < RP; ++i) t[r] += rs[r][i];
      if (a.ss_in && m < M)
        for (int p = RP * kWave + lane; p < a.n_ss; p += kWave) t[r] += a.ss_in[(size_t)p * a.ss_ld + m];
    }
    wave_sum_n(t);
#pragma unroll
    for (int r = 0; r < RS; ++r) {
      const int m = wave + r * NW;
      if (lane == 0 && m < MP) scale[m] = (a.ss_in && m < M) ? 1.0f / sqrtf(t[r] / (float)K + a.eps) : 1.0f;
    }
  }

  // Refills without a branch, the last batches peeled off (PEEL): with a branch
  // around a refill the compiler waits for both buffers before the first
  // product of either (40 rows, 7B: Q|K|V 28.0 -> 26.8 us, O and down 33.8 ->
  // 32.0 together, LM head 57 -> 50; at most 16 rows: launch_t1).
  int cu = u0, cb = 0, left = total;  // compute cursor, batches left
  auto done = [&]() {
    if (++cb == nbat) { finish(cu); cb = 0; cu += us; }
  };
  if constexpr (!PEEL) {
    while (true) {
      compute(wA, xA, sA);
      if (left > 2) load(wA, xA, sA);
      done();
      if (--left == 0) return;
      compute(wB, xB, sB);
      if (left > 2) load(wB, xB, sB);
      done();
      if (--left == 0) return;
    }
  }
  for (; left > 3; left -= 2) {
    compute(wA, xA, sA);
    load(wA, xA, sA);
    done();
    compute(wB, xB, sB);
    load(wB, xB, sB);
    done();
  }
  compute(wA, xA, sA);
  if (left == 3) load(wA, xA, sA);
  done();
  if (left > 1) {
    compute(wB, xB, sB);
    done();
  }
  if (left == 3) {
    compute(wA, xA, sA);
    done();
  }
}

template <int T, int MT, int NW, int UB, int KIND, bool Q4, int XF, bool PEEL>
void launch_mt(const GemmArgs& a, int n_split, int per_split, hipStream_t s) {
  constexpr int NU = KIND == EPI_SWIGLU ? 8 * T : 16 * T;  // output columns per unit
  const int units = (a.n_rows + NU - 1) / NU;
  const int grid = std::min(units, std::max(1, device_compute_units() / n_split)) * n_split;
  hipLaunchKernelGGL((gemm_bf16_rows<T, MT, NW, UB, KIND, Q4, XF, PEEL>), dim3(grid), dim3(64 * NW), 0, s, a, units,
                     n_split, per_split);
}
// 17 to 64 rows (to 16 MT_MAX).
template <int T, int NW, int UB, int KIND, bool Q4 = false, int MT_MAX = 4>
void launch_t(const GemmArgs& a, int n_split, int per_split, hipStream_t s) {
  const int MT = (a.M + 15) / 16;
  if (MT == 2) launch_mt<T, 2, NW, UB, KIND, Q4, 4, true>(a, n_split, per_split, s);
  else if (MT == 3) launch_mt<T, 3, NW, UB, KIND, Q4, 6, true>(a, n_split, per_split, s);
  else if constexpr (MT_MAX == 4) launch_mt<T, 4, NW, UB, KIND, Q4, 8, true>(a, n_split, per_split, s);
}
// At most 16 rows, whole K; UB1: k-steps per buffer over at most 8 rows.
// Refills without a branch (PEEL) from four batches per unit and wave: 7B verify
// of 5 rows 2973 us (8 batches in all three GEMMs; 3004 with the branch
// everywhere), 1.1B LM head over 16 rows 22.5 (4 batches; 23.2); the 2 batches
// of the 1.1B Q|K|V units gain nothing from the longer code (draft of four slots
// 799 us, 801 with it).
template <int T, int NW, int UB, int KIND, int UB1 = UB>
void launch_t1(const GemmArgs& a, hipStream_t s) {
  const int KS = a.K / 32, per_batch = NW * (a.M <= 8 ? UB1 : UB);
  const bool peel = (KS + per_batch - 1) / per_batch >= 4;
  if (a.M <= 8) {
    if (peel) launch_mt<T, 1, NW, UB1, KIND, false, 1, true>(a, 1, KS, s);
    else launch_mt<T, 1, NW, UB1, KIND, false, 1, false>(a, 1, KS, s);
  } else {
    if (peel) launch_mt<T, 1, NW, UB, KIND, false, 2, true>(a, 1, KS, s);
    else launch_mt<T, 1, NW, UB, KIND, false, 2, false>(a, 1, KS, s);
  }
}

// Rounds of the persistent grid that units of T tiles take, in tiles (plus
// one for what a round costs besides its weights).
int unit_cost(int n_tiles, int T) {
  const int units = (n_tiles + T - 1) / T, cus = device_compute_units();
  return (units + cus - 1) / cus * (T + 1);
}

// Passes of at most 16 rows, bf16 weights: Q|K|V, gate|up and the LM head (the
// residual GEMMs run gemm_bf16_mfma).  Neither the waves nor the unit sizes
// depend on the row count, so a verify block equals its rows run one by one bit
// for bit.  A row tile costs one register set here, so units hold two to four
// k-steps per buffer (over at most 8 rows one or two to four more: 2994 and 3100
// us instead of 2973 for the 7B verify of 5 rows; half in Q|K|V or gate|up: 2973,
// 2982).  Over at most 8 rows x comes in one fragment per k-step: a load takes its
// slot in the texture unit whether its lanes are in range or not.  The 7B LM head
// over 5 rows, among the other launches of a pass: 45.5 us with two fragments,
// 44.5 to 45 with one, 44.0 to 44.8 in buffers of one k-step (43.6 on the
// residual GEMMs' kernel, x held in LDS, but 68 instead of 45 over 9 to 16 rows,
// and the two would add in different orders).
hipError_t launch_one(const GemmArgs& a, hipStream_t s) {
  const int KS = a.K / 32, tiles = a.n_rows / 16;
  if (a.q4) return hipErrorInvalidValue;
  switch (a.kind) {
    case EPI_STORE:
      // (a wave keeps at least 16 k-steps of a unit: fewer waves where K is
      // short; K = 2048, 32000 rows: 22.2 us on 4 waves, 27.7 on 8)
      if (KS >= 128) launch_t1<4, 8, 2, EPI_STORE, 1>(a, s);
      else launch_t1<4, 4, 4, EPI_STORE>(a, s);
      break;
    case EPI_QKV: {
      const int c1 = unit_cost(tiles, 1), c2 = unit_cost(tiles, 2), c3 = unit_cost(tiles, 3);
      if (c3 <= c2 && c3 <= c1) launch_t1<3, 8, 2, EPI_QKV>(a, s);
      else if (c2 <= c1) launch_t1<2, 8, 4, EPI_QKV>(a, s);
      else launch_t1<1, 8, 4, EPI_QKV>(a, s);
      break;
    }
    case EPI_SWIGLU:
      if (unit_cost(2 * tiles, 6) <= unit_cost(2 * tiles, 4)) launch_t1<6, 8, 2, EPI_SWIGLU>(a, s);
      else launch_t1<4, 8, 2, EPI_SWIGLU>(a, s);
      break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

// INT4 weights: 4-wave blocks (a wave holds two groups' x and codes).
hipError_t launch_q4(const GemmArgs& a, hipStream_t s) {
  const int KG = (a.K + 127) / 128, tiles = a.n_rows / 16;
  switch (a.kind) {
    case EPI_QKV: {
      const int c1 = unit_cost(tiles, 1), c3 = unit_cost(tiles, 3);
      if (c3 <= c1) launch_t<3, 4, 4, EPI_QKV, true>(a, 1, KG, s);
      else launch_t<1, 4, 4, EPI_QKV, true>(a, 1, KG, s);
      break;
    }
    case EPI_SWIGLU:
      // (6 tiles over more than 48 rows spill: 101 us against 65 for the 7B shape over 64 rows)
      if (a.M <= 48 && unit_cost(2 * tiles, 6) <= unit_cost(2 * tiles, 4))
        launch_t<6, 4, 4, EPI_SWIGLU, true, 3>(a, 1, KG, s);
      else launch_t<4, 4, 4, EPI_SWIGLU, true>(a, 1, KG, s);
      break;
    case EPI_RESID: {
      const int cus = device_compute_units();
      auto splits = [&](int T) {
        return std::min({kRowsSplitMax, KG, std::max(1, cus / ((tiles + T - 1) / T))});
      };
      const bool four = splits(4) * 4 <= KG;  // (a group for each wave of a split)
      int n_split = four ? splits(4) : splits(2);
      const int per = (KG + n_split - 1) / n_split;
      n_split = (KG + per - 1) / per;
      if (four) launch_t<4, 4, 4, EPI_RESID, true>(a, n_split, per, s);
      else launch_t<2, 4, 4, EPI_RESID, true>(a, n_split, per, s);
      return launch_resid_reduce(a, n_split, s);
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace

hipError_t launch_gemm_rows(const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || a.M > kMaxGemmRows || !a.xs || a.stt != stacked_fragments(a.M) || a.K % 32 || a.n_rows % 16)
    return hipErrorInvalidValue;
  if (a.kind == EPI_QKV && (a.kv.dtype != SPECDEC_BF16 || a.head_dim % 16 || a.n_seg[0] % a.head_dim ||
                            a.n_seg[1] % a.head_dim))
    return hipErrorInvalidValue;
  if (a.kind == EPI_SWIGLU && !a.xs_out) return hipErrorInvalidValue;
  if (a.kind == EPI_RESID && (a.M <= kSkinnyRows || !a.ypart || !a.xs_out || !a.gain_bf16)) return hipErrorInvalidValue;
  if (a.M <= kSkinnyRows) return launch_one(a, s);
  if (a.q4) return launch_q4(a, s);
  const int KS = a.K / 32, tiles = a.n_rows / 16;
  switch (a.kind) {
    case EPI_STORE:
      // Larger units read x fewer times: 8 tiles over more than two row tiles,
      // unless 4 fill the CUs' rounds better (7B LM head, 40 rows: 50 us in 250
      // units of 8; 20 rows: 47.5, in 500 of 4 44.4).  Where K is short a unit
      // of 4 on 4 waves, which keep 16 k-steps each (K = 2048, 32000 rows, 20
      // rows of x: 24.7 us, 27.7 on 8 waves, 28.5 in units of 8).
      if (KS < 128) launch_t<4, 4, 1, EPI_STORE>(a, 1, KS, s);
      else if (a.M > 32 && unit_cost(tiles, 8) <= unit_cost(tiles, 4)) launch_t<8, 4, 1, EPI_STORE>(a, 1, KS, s);
      else launch_t<4, 8, 1, EPI_STORE>(a, 1, KS, s);
      break;
    case EPI_QKV: {
      const int c1 = unit_cost(tiles, 1), c2 = unit_cost(tiles, 2), c3 = unit_cost(tiles, 3);
      if (c3 <= c2 && c3 <= c1) launch_t<3, 8, 1, EPI_QKV>(a, 1, KS, s);
      else if (c2 <= c1) launch_t<2, 8, 1, EPI_QKV>(a, 1, KS, s);
      else launch_t<1, 8, 1, EPI_QKV>(a, 1, KS, s);
      break;
    }
    case EPI_SWIGLU:
      // (pairs of a gate and an up tile: 6 tiles cover three of them; the 7B
      // shape over 40 rows: 38.1 us in 230 units of 6 tiles, 49.5 in 344 of 4)
      if (unit_cost(2 * tiles, 6) <= unit_cost(2 * tiles, 4)) launch_t<6, 4, 2, EPI_SWIGLU>(a, 1, KS, s);
      else launch_t<4, 8, 1, EPI_SWIGLU>(a, 1, KS, s);
      break;
    case EPI_RESID: {
      // Few tiles (7B O and down: 256): units of 4 tiles with K split over the
      // grid, as far as every wave of a split keeps two k-steps; else units of
      // 2.  7B O over 40 rows: 9.8 us in 64 units x 4 splits, 11.2 in 128 x 2.
      const int cus = device_compute_units();
      auto splits = [&](int T) {
        return std::min({kRowsSplitMax, KS, std::max(1, cus / ((tiles + T - 1) / T))});
      };
      const bool four = splits(4) * 16 <= KS;
      int n_split = four ? splits(4) : splits(2);
      const int per = (KS + n_split - 1) / n_split;
      n_split = (KS + per - 1) / per;
      if (four) launch_t<4, 8, 1, EPI_RESID>(a, n_split, per, s);
      else launch_t<2, 8, 1, EPI_RESID>(a, n_split, per, s);
      return launch_resid_reduce(a, n_split, s);
    }
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace specdec
