// Weight-streaming GEMMs of passes of at most 16 rows that gemm_rows.hip does
// not take, the float32 GEMMs, and the weight images:
//   y[m, n] = s_m * sum_k W[n, k] * (x[m, k] * g[k])
// with W streamed once from HBM.  gemm_bf16_mfma: the residual GEMMs (O and
// down projections) of bf16 weights, which add to h and emit the partial sums
// of squares the next RMSNorm needs, and INT4 shapes gemm_q4_lds does not
// cover.  gemm_q4_lds: INT4 layers.  Both run on MFMA (v_mfma_f32_16x16x32_bf16)
// with x as hi + lo bf16 parts (x = hi + lo + O(2^-17 |x|)), so two products
// per weight fragment give float32 accuracy while the weights are read once.
// float32 weights (the tiny configuration) run on a plain vector kernel.
#include <algorithm>
#include <type_traits>

#include "device_common.h"
#include "gemm_common.h"
#include "internal.h"

namespace specdec {

namespace {

constexpr int kMfmaThreads = 1024;  // 16 waves split K
constexpr int kMfmaWaves = kMfmaThreads / kWave;

__device__ __forceinline__ float load_gain(const void* g, int bf16, int n) {
  return bf16 ? bf16_bits_to_f32(((const uint16_t*)g)[n]) : ((const float*)g)[n];
}

// ---------------------------------------------------------------- shared pieces
// Row scale s_m = 1/sqrt(sum_p ss[p][m] / K + eps): one wave per row, lanes
// stride over the partial sums, fixed shuffle tree (deterministic).
template <int MP>
__device__ __forceinline__ void row_scale(const GemmArgs& a, float* scale) {
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, nw = blockDim.x >> 6;
  for (int m = wave; m < MP; m += nw) {
    float t = 0.f;
    if (a.ss_in && m < a.M)
      for (int p = lane; p < a.n_ss; p += kWave) t += a.ss_in[(size_t)p * a.ss_ld + m];
    t = wave_sum(t);
    if (lane == 0) scale[m] = (a.ss_in && m < a.M) ? 1.0f / sqrtf(t / (float)a.K + a.eps) : 1.0f;
  }
}

// Epilogue over this block's final sums yfin[m][c], c < NC columns (store,
// residual, SwiGLU; the MFMA kernel has its own residual and QKV epilogues
// that take their inputs from registers and LDS).
template <int NC, int KIND, int NTH>
__device__ __forceinline__ void epilogue(const GemmArgs& a, int blk, float (*yfin)[NC + 1], const float* scale) {
  const int M = a.M;  // (NTH = threads of the block: a constant, not a read of the dispatch packet)
  if (KIND == EPI_STORE) {
    for (int i = threadIdx.x; i < M * NC; i += NTH) {
      int m = i / NC, c = i % NC;
      int n = blk * NC + c;
      if (n < a.n_rows) a.out[(size_t)m * a.ldo + n] = yfin[m][c] * scale[m];
    }
  } else if (KIND == EPI_RESID) {
    for (int i = threadIdx.x; i < M * NC; i += NTH) {
      int m = i / NC, c = i % NC;
      int n = blk * NC + c;
      float hv = 0.f;
      if (n < a.n_rows) {
        float* hp = a.out + (size_t)m * a.ldo + n;
        hv = *hp + yfin[m][c];
        *hp = hv;
        const float xv = hv * load_gain(a.gain_out, a.gain_bf16, n);
        a.xg_out[(size_t)m * a.ldo + n] = xv;
        if (a.xs_out) put_stacked(a.xs_out, a.stt_out, m, n, xv);
      }
      yfin[m][c] = hv;
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += NTH) {
      float t = 0.f;
      for (int c = 0; c < NC; ++c) t += yfin[m][c] * yfin[m][c];
      a.ss_out[(size_t)blk * a.ss_ld + m] = t;
    }
  } else {  // EPI_SWIGLU: columns [0, NC/2) gate, [NC/2, NC) up
    constexpr int H = NC / 2;
    for (int i = threadIdx.x; i < M * H; i += NTH) {
      int m = i / H, c = i % H;
      int n = blk * H + c;
      if (n < a.n_rows) {
        float g = yfin[m][c] * scale[m];
        float u = yfin[m][H + c] * scale[m];
        const float y = silu_f(g) * u;
        a.out[(size_t)m * a.ldo + n] = y;
        if (a.xs_out) put_stacked(a.xs_out, a.stt_out, m, n, y);
      }
    }
  }
}

// Q|K|V epilogue over this block's final sums yfin[m][c], c < NC columns of
// the concatenated Q|K|V rows (bf16 cache).  Columns of the Q and K segments
// come in RoPE pairs: column c (c % 16 < 8) is dim j = 8 * (tile within the
// head) + c % 8 of its head, column c ^ 8 is dim j + hd/2; x1' = x1 cos - x2
// sin, x2' = x2 cos + x1 sin.  Rotated queries go to qr, K and V into the
// cache at each valid row's position.  s_rows / s_cs: the rows' descriptors
// and cos | sin tables.
template <int NC, int NTH>
__device__ __forceinline__ void qkv_epilogue(const GemmArgs& a, int blk, const float (*yfin)[NC + 1],
                                             const float* scale, const RowDesc* s_rows, const float (*s_cs)[128]) {
  const int M = a.M, hd = a.head_dim, half = hd >> 1, H = a.n_heads;
  const int nq = a.n_seg[0], nqk = nq + a.n_seg[1], cap = a.kv.capacity;
#pragma unroll 1
  for (int i = threadIdx.x; i < M * NC; i += NTH) {
    const int m = i / NC, c = i % NC, n = blk * NC + c;
    if (n >= a.n_rows) continue;
    const float x = yfin[m][c] * scale[m];
    const RowDesc rd = s_rows[m];
    if (n < nqk) {
      const bool is_k = n >= nq;
      const int r = is_k ? n - nq : n;
      const int head = r / hd, w = r % hd, ec = w & 15;
      const int j = 8 * (w >> 4) + (ec & 7);
      const float y = yfin[m][c ^ 8] * scale[m];
      const float cs = s_cs[m][j], sn = s_cs[m][half + j];
      const float out = ec < 8 ? x * cs - y * sn : x * cs + y * sn;
      const int d = ec < 8 ? j : half + j;
      if (!is_k) {
        a.qr[((size_t)m * H + head) * hd + d] = out;
      } else if (rd.valid) {
        uint16_t* kvb = k_block<uint16_t>(a.kv, a.layer, rd.b, head);
        Storage<uint16_t>::store(kvb + KvIndex<uint16_t>::k(rd.pos, d, hd, cap), out);
      }
    } else if (rd.valid) {
      const int r = n - nqk, head = r / hd, d = r % hd;
      uint16_t* kvb = k_block<uint16_t>(a.kv, a.layer, rd.b, head);
      Storage<uint16_t>::store(kvb + KvIndex<uint16_t>::v(rd.pos, d, hd, cap), x);
    }
  }
}

// Row pointer of weight row `r` of the block's concatenated row space.
template <typename WT>
__device__ __forceinline__ const WT* weight_row(const GemmArgs& a, int kind, int blk, int NC, int c, bool& ok) {
  if (kind == EPI_SWIGLU) {
    const int H = NC / 2;
    int seg = c >= H;
    int n = blk * H + (c - seg * H);
    ok = n < a.n_rows;
    if (!ok) n = 0;
    return (const WT*)a.w[seg] + (size_t)n * a.K;
  }
  int n = blk * NC + c;
  ok = n < a.n_rows;
  if (!ok) n = 0;
  int b1 = a.n_seg[0], b2 = b1 + a.n_seg[1];
  if (n < b1) return (const WT*)a.w[0] + (size_t)n * a.K;
  if (n < b2) return (const WT*)a.w[1] + (size_t)(n - b1) * a.K;
  return (const WT*)a.w[2] + (size_t)(n - b2) * a.K;
}

// INT4 image of W [N, K]: per 16-row tile and group of 128 columns a 1 KB
// block in which lane l = 16*(k%32/8) + n%16 holds 16 bytes, the words of
// the group's four k-steps; word j holds the 8 codes of row n at columns
// 128g + 32j + 8*(l/16) .. +7, low nibble first.  Then the group scales
// [N/16][KG][16] (bf16).
struct Q4Frag {
  uint32_t codes;
  uint32_t scale;  // bf16 bits of the group scale of the lane's row (lane % 16)
};

// ---------------------------------------------------------------- MFMA kernel
// Persistent: one 16-wave block per CU loops over row tiles of NC = 16*T
// weight rows (tile = blockIdx.x + i*gridDim.x).  Within a tile, wave w
// reduces k-steps [w*KS/16, (w+1)*KS/16) of 32 columns each, UB k-steps per
// register buffer; the next buffer -- including the first one of the next
// tile -- is loaded while the current one is multiplied, so the weight
// stream keeps going through the cross-wave reduction and the epilogue.
// MFMA operand layout (16x16x32): lane l holds A[l%16][8(l/16)+j] (x rows),
// B[8(l/16)+j][l%16] (= W[n0 + l%16][k0 + 8(l/16) + j]: 16 bytes at lane*16 of
// the packed 1 KB fragment), D[4(l/16)+r][l%16].
template <int T, int UB, int KIND, int XS>
__global__ __launch_bounds__(kMfmaThreads) void gemm_bf16_mfma(GemmArgs a, int n_tiles) {
  // XS = 0: INT4 weights (Q4Frag) and float32 x.  A code q is fed to the MFMA
  // as the bf16 value 136 + q (bits 0x4300 | (q + 8): two byte permutes and an
  // OR per four codes), and the bias is cancelled inside the accumulator by a
  // product of the same x with the constant -136, shared by the unit's tiles;
  // each k-step's product is then multiplied by the lane's row scale in
  // float32, so the effective weights are code * scale.
  // XS > 0: bf16 weights and x as the stacked operand a.xs (put_stacked, XS
  // fragments per k-step, at most 8 rows when XS = 1, 16 when XS = 2): one
  // 16-byte load per fragment and one product per fragment and tile.  The hi
  // and lo parts accumulate apart (accumulator tiles 0 and 1, or rows m and
  // 8 + m of tile 0) and are added once per tile before the cross-wave sums,
  // the same arithmetic for either count of fragments.
  // XS = 3: XS = 1 with each wave's x fragments (at most 8 k-steps, K <= 4096)
  // fetched once into LDS and read from there for every unit of the block.
  constexpr bool Q4 = XS == 0;
  static_assert(Q4 || KIND == EPI_RESID, "bf16 weights: residual GEMMs");
  constexpr int MT = 1;  // (at most kSkinnyRows rows)
  using WReg = std::conditional_t<Q4, Q4Frag, u32x4>;
  constexpr bool XL = XS == 3;
  constexpr int XF = XL ? 1 : XS;   // stacked fragments per k-step
  constexpr int MA = XS ? XF : MT;  // accumulator row tiles
  constexpr int NC = 16 * T;
  constexpr int MP = 16 * MT;
  constexpr int NF = T * MT;              // accumulator fragments per wave
  constexpr int RR = XL ? 1 : (NF <= 2 ? NF : 2);  // fragments reduced per LDS round (XL: LDS goes to x)
  constexpr bool QKV = KIND == EPI_QKV;
  static_assert(MP * NC <= kMfmaThreads, "one epilogue element per thread");
  __shared__ float red[RR][kMfmaWaves][kWave][4];
  __shared__ u32x4 s_xl[XL ? kMfmaWaves : 1][XL ? 8 : 1][kWave];  // XL: wave w's x fragments, k-steps w + 16j
  __shared__ float yfin[MP][NC + 1];
  __shared__ float scale[MP];
  __shared__ RowDesc s_rows[QKV ? MP : 1];
  __shared__ float s_cs[QKV ? MP : 1][QKV ? 128 : 1];  // RoPE cos | sin of each row (head_dim <= 128)

  // The wave index is uniform across the wave; saying so keeps every per-wave
  // quantity derived from it (k-step list, tile, weight segment, buffer
  // descriptors) in scalar registers.
  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int kg = lane >> 4, mrow = lane & 15;
  // Stacked x: the lanes of a fragment's padding rows (rows >= M of its hi and
  // lo halves) read nothing, which keeps them zero; only rows < M reach an
  // output (5 rows: 10 of the 16 fragment rows fetched, 1 row: 2).
  const uint32_t xrbad = XS ? (uint32_t)(((XS == 2 ? mrow : (mrow & 7)) >= a.M)) << 31 : 0u;
  const int K = a.K;
  const int KS = (K + 31) / 32;
#ifdef SPECDEC_KSTEP_CONTIGUOUS
  const int ks0 = (wave * KS) / kMfmaWaves, ks1 = ((wave + 1) * KS) / kMfmaWaves;
  const int kstride = 1;
#else
  // k-steps interleaved across waves (wave w: w, w+16, ...): at any moment the
  // block reads 16 consecutive k-steps = 1 KB contiguous of each of its rows.
  const int ks0 = wave, ks1 = KS;
  const int kstride = kMfmaWaves;
#endif
  const int my_ks = ks1 > ks0 ? (ks1 - ks0 + kstride - 1) / kstride : 0;
  const int nbat = max(1, (my_ks + UB - 1) / UB);
  const int my_tiles = (n_tiles - (int)blockIdx.x + (int)gridDim.x - 1) / (int)gridDim.x;
  const int total = my_tiles * nbat;

  floatx4 acc[T][MA];
#pragma unroll
  for (int t = 0; t < T; ++t)
#pragma unroll
    for (int mt = 0; mt < MA; ++mt) acc[t][mt] = floatx4{0.f, 0.f, 0.f, 0.f};

  WReg wA[UB][T], wB[UB][T];
  f32x4 xA[UB][MA][2], xB[UB][MA][2];  // (stacked x: [u][fragment][0] holds the fragment's 16 bytes)
  // Residual epilogue inputs (old h and the next RMSNorm gain) of the tile whose
  // last batch sits in the matching register buffer, fetched with that batch.
  constexpr bool PRE = KIND == EPI_RESID;
  struct Pre {
    float h;
    uint32_t g;  // bf16 bits of the gain (bf16 models only run this kernel)
  } pA, pB;
  auto epi_fetch = [&](int q, Pre& p) {
    if constexpr (PRE) {
      // (every batch fetches its tile's inputs: no branch; the copy fetched with
      // the tile's last batch is the one its epilogue uses)
      const int tile = blockIdx.x + (q / nbat) * gridDim.x;
      const __amdgpu_buffer_rsrc_t hr = make_rsrc(a.out, (uint32_t)a.M * a.ldo * 4u);
      const __amdgpu_buffer_rsrc_t gr = make_rsrc(a.gain_out, (uint32_t)a.n_rows * 2u);
      const int m = tid / NC, n = tile * NC + tid % NC;
      const uint32_t bad = (uint32_t)(n >= a.n_rows) << 31;  // (rows m >= M fall outside hr)
      p.h = __builtin_bit_cast(
          float, __builtin_amdgcn_raw_buffer_load_b32(hr, (((uint32_t)m * a.ldo + n) * 4u) | bad, 0, 0));
      p.g = __builtin_amdgcn_raw_buffer_load_b16(gr, ((uint32_t)n * 2u) | bad, 0, 0);
    }
  };
  // Loads go through buffer descriptors: an offset past the descriptor's range
  // reads zeros without touching memory, so rows beyond M, tiles beyond N and
  // k-steps beyond the wave's list need no branches (a branch around a load
  // makes the compiler wait for the data where the paths join).
  const __amdgpu_buffer_rsrc_t xr = XS ? make_rsrc(a.xs, (uint32_t)KS * XF * 1024u)
                                       : make_rsrc(a.x, (uint32_t)a.M * a.ldx * 4u);
  // load the q-th batch of this wave's work list (tile q / nbat, k-steps from (q % nbat) * UB)
  auto load = [&](int q, WReg (&wv)[UB][T], f32x4 (&xv)[UB][MA][2]) {
    const int tile = blockIdx.x + (q / nbat) * gridDim.x;
    const int kb = (q % nbat) * UB;  // index into this wave's k-step list
    __amdgpu_buffer_rsrc_t wr[T], sr[T];
#pragma unroll
    for (int t = 0; t < T; ++t) {
      bool rok;
      if constexpr (Q4) {
        int seg, n;
        tile_segment(a, KIND, tile, NC, t, seg, n, rok);
        const int KG = (K + 127) / 128;
        wr[t] = make_rsrc((const char*)a.w[seg] + (size_t)(n / 16) * KG * 1024, rok ? (uint32_t)KG * 1024u : 0u);
        sr[t] = make_rsrc(a.wscale[seg] + (size_t)(n / 16) * KG * 16, rok ? (uint32_t)KG * 32u : 0u);
      } else {
        const uint16_t* base = weight_tile(a, KIND, tile, NC, t, KS, rok);
        wr[t] = make_rsrc(base, rok ? (uint32_t)KS * 1024u : 0u);
      }
    }
#pragma unroll
    for (int u = 0; u < UB; ++u) {
      const int ks = ks0 + (kb + u) * kstride;
      const int k = ks * 32 + kg * 8;
      // (out-of-range flags are OR-ed into the offsets: a select on a wave-uniform
      // flag would become a branch)
      const uint32_t wbad = (uint32_t)((kb + u) >= my_ks || ks >= KS) << 31;
      const uint32_t woff = ((uint32_t)ks * 1024u + lane * 16u) | wbad;
#pragma unroll
      for (int t = 0; t < T; ++t) {
        if constexpr (Q4) {
          const uint32_t qoff = ((uint32_t)(ks >> 2) * 1024u + lane * 16u + (uint32_t)(ks & 3) * 4u) | wbad;
          const uint32_t soff = ((uint32_t)(ks >> 2) * 32u + (lane & 15) * 2u) | wbad;
          wv[u][t].codes = __builtin_amdgcn_raw_buffer_load_b32(wr[t], qoff, 0, kNonTemporal);
          wv[u][t].scale = __builtin_amdgcn_raw_buffer_load_b16(sr[t], soff, 0, 0);
        } else {
          wv[u][t] = __builtin_amdgcn_raw_buffer_load_b128(wr[t], woff, 0, kNonTemporal);
        }
      }
      if constexpr (XL) {
        // (x comes from LDS)
      } else if constexpr (XS) {
#pragma unroll
        for (int f = 0; f < XS; ++f) {
          const uint32_t xoff = (((uint32_t)ks * XS + f) * 1024u + lane * 16u) | wbad | xrbad;
          xv[u][f][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, xoff, 0, 0));
        }
      } else {
#pragma unroll
        for (int mt = 0; mt < MT; ++mt) {
          const int m = mt * 16 + mrow;
          const uint32_t xoff = (((uint32_t)m * a.ldx + k) * 4u) | wbad | ((uint32_t)(k >= K) << 31);
          xv[u][mt][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, xoff, 0, 0));
          xv[u][mt][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, xoff + 16u, 0, 0));
        }
      }
    }
  };
  auto compute = [&](WReg (&wv)[UB][T], f32x4 (&xv)[UB][MA][2], int q) {
    if constexpr (XL) {
      const int kb = (q % nbat) * UB;  // (past the wave's k-steps the weights read zeros)
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        const bf16x8 xf = __builtin_bit_cast(bf16x8, s_xl[wave][min(kb + u, 7)][lane]);
#pragma unroll
        for (int t = 0; t < T; ++t)
          acc[t][0] =
              __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, __builtin_bit_cast(bf16x8, wv[u][t]), acc[t][0], 0, 0, 0);
      }
    } else if constexpr (XS) {
#pragma unroll
      for (int u = 0; u < UB; ++u)
#pragma unroll
        for (int f = 0; f < XS; ++f) {
          const bf16x8 xf = __builtin_bit_cast(bf16x8, xv[u][f][0]);
#pragma unroll
          for (int t = 0; t < T; ++t)
            acc[t][f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xf, __builtin_bit_cast(bf16x8, wv[u][t]), acc[t][f],
                                                                0, 0, 0);
        }
    } else {
#pragma unroll
      for (int u = 0; u < UB; ++u) {
        // the codes of each tile as biased bf16 operands and the row scales
        bf16x8 bq[T];
        float sc[T];
#pragma unroll
        for (int t = 0; t < T; ++t) {
          const uint32_t c = wv[u][t].codes ^ 0x88888888u;  // q + 8 in each nibble
          const uint32_t even = c & 0x0F0F0F0Fu, odd = (c >> 4) & 0x0F0F0F0Fu;  // codes 0,2,4,6 / 1,3,5,7
          u32x4 v;
          // dword j/2 of the operand: code j in its low half, code j+1 in its high half
          v[0] = __builtin_amdgcn_perm(odd, even, 0x0c040c00u) | 0x43004300u;
          v[1] = __builtin_amdgcn_perm(odd, even, 0x0c050c01u) | 0x43004300u;
          v[2] = __builtin_amdgcn_perm(odd, even, 0x0c060c02u) | 0x43004300u;
          v[3] = __builtin_amdgcn_perm(odd, even, 0x0c070c03u) | 0x43004300u;
          bq[t] = __builtin_bit_cast(bf16x8, v);
          sc[t] = bf16_bits_to_f32((uint16_t)wv[u][t].scale);
        }
        bf16x8 hi, lo;
#pragma unroll
        for (int j = 0; j < 8; ++j) {
          const float v = xv[u][0][j >> 2][j & 3];
          const __bf16 h = (__bf16)v;
          hi[j] = h;
          lo[j] = (__bf16)(v - (float)h);
        }
        // -136 * sum_k x[m][k] in every column
        const u32x4 m136 = u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u};
        floatx4 bias = floatx4{0.f, 0.f, 0.f, 0.f};
        bias = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, __builtin_bit_cast(bf16x8, m136), bias, 0, 0, 0);
        bias = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, __builtin_bit_cast(bf16x8, m136), bias, 0, 0, 0);
#pragma unroll
        for (int t = 0; t < T; ++t) {
          floatx4 p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, bq[t], bias, 0, 0, 0);
          p = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, bq[t], p, 0, 0, 0);
#pragma unroll
          for (int r = 0; r < 4; ++r) acc[t][0][r] = fmaf(sc[t], p[r], acc[t][0][r]);
        }
      }
    }
  };
  auto mfma_epilogue = [&](int blk, const Pre& p) {
    const int M = a.M;
    if constexpr (PRE) {
      const int m = tid / NC, c = tid % NC, n = blk * NC + c;
      if (m < M) {
        float hv = 0.f;
        if (n < a.n_rows) {
          hv = p.h + yfin[m][c];
          a.out[(size_t)m * a.ldo + n] = hv;
          const float xv = hv * bf16_bits_to_f32((uint16_t)p.g);
          if (a.xs_out) put_stacked(a.xs_out, a.stt_out, m, n, xv);
          else a.xg_out[(size_t)m * a.ldo + n] = xv;
        }
        yfin[m][c] = hv;
      }
      __syncthreads();
      for (int m = tid; m < M; m += kMfmaThreads) {
        float t = 0.f;
        for (int c = 0; c < NC; ++c) t += yfin[m][c] * yfin[m][c];
        a.ss_out[(size_t)blk * a.ss_ld + m] = t;
      }
    } else if constexpr (KIND == EPI_QKV) {
      qkv_epilogue<NC, kMfmaThreads>(a, blk, yfin, scale, s_rows, s_cs);
    } else {
      epilogue<NC, KIND, kMfmaThreads>(a, blk, yfin, scale);
    }
  };
  // After the last batch of a tile: cross-wave reduction (fixed wave order) and epilogue.
  auto finish = [&](int q, const Pre& p) {
    if (q % nbat != nbat - 1) return;
    const int tile = blockIdx.x + (q / nbat) * gridDim.x;
    if constexpr (XF == 1) {  // hi (rows 0-7, lanes 0-31) + lo (rows 8-15, lanes 32-63)
#pragma unroll
      for (int t = 0; t < T; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          const float v = acc[t][0][r], o = __shfl_xor(v, 32, kWave);
          acc[t][0][r] = lane < 32 ? v + o : 0.f;
        }
    } else if constexpr (XF == 2) {  // hi (tile 0) + lo (tile 1)
#pragma unroll
      for (int t = 0; t < T; ++t) acc[t][0] += acc[t][1];
    }
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += RR) {
#pragma unroll
      for (int f = 0; f < RR; ++f) {
        if (f0 + f < NF) {
          const int t = (f0 + f) / MT, mt = (f0 + f) % MT;
#pragma unroll
          for (int r = 0; r < 4; ++r) red[f][wave][lane][r] = acc[t][mt][r];
        }
      }
      __syncthreads();
      if (tid < 256 * RR && f0 + (tid >> 8) < NF) {
        const int f = tid >> 8, l = tid & 63, r = (tid >> 6) & 3;
        const int t = (f0 + f) / MT, mt = (f0 + f) % MT;
        float s = 0.f;
#pragma unroll
        for (int w = 0; w < kMfmaWaves; ++w) s += red[f][w][l][r];
        yfin[mt * 16 + 4 * (l >> 4) + r][t * 16 + (l & 15)] = s;
      }
      __syncthreads();
    }
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
      for (int mt = 0; mt < MA; ++mt) acc[t][mt] = floatx4{0.f, 0.f, 0.f, 0.f};
    mfma_epilogue(tile, p);
    __syncthreads();  // yfin is reused by the next tile
  };

  // Prologue.  The small operands only the epilogue needs (row-scale partial
  // sums, the QKV tables) are requested first, then both register buffers'
  // weight batches; storing the small ones then waits for them alone (loads
  // complete in order), so no wave waits for a weight batch before its first
  // multiply.
  constexpr int RS_ROWS = (MP + kMfmaWaves - 1) / kMfmaWaves;  // scale rows per wave
  constexpr int RS_P = 4;                                      // partial sums per lane held
  float rs_v[RS_ROWS][RS_P];
  {
    const __amdgpu_buffer_rsrc_t sr = make_rsrc(a.ss_in, a.ss_in ? (uint32_t)a.n_ss * a.ss_ld * 4u : 0u);
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kMfmaWaves;
#pragma unroll
      for (int i = 0; i < RS_P; ++i) {
        const int p = lane + i * kWave;
        const uint32_t off = (m < a.M && p < a.n_ss) ? ((uint32_t)p * a.ss_ld + m) * 4u : kOutOfRange;
        rs_v[r][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, off, 0, 0));
      }
    }
  }
  constexpr int CS_E = QKV ? MP * 128 / kMfmaThreads : 1;  // table entries per thread
  float cs_v[CS_E];
  RowDesc rd_v{0, 0, 0, 0};
  if constexpr (QKV) {
    const __amdgpu_buffer_rsrc_t cr = make_rsrc(a.rope_cs, (uint32_t)a.M * a.head_dim * 4u);
#pragma unroll
    for (int e = 0; e < CS_E; ++e) {
      const int i = tid + e * kMfmaThreads, m = i / 128, j = i % 128;
      const uint32_t off = j < a.head_dim ? ((uint32_t)m * a.head_dim + j) * 4u : kOutOfRange;
      cs_v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(cr, off, 0, 0));
    }
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.rows, (uint32_t)a.M * (uint32_t)sizeof(RowDesc));
    rd_v = __builtin_bit_cast(RowDesc, __builtin_amdgcn_raw_buffer_load_b128(
                                           rr, tid < MP ? (uint32_t)tid * (uint32_t)sizeof(RowDesc) : kOutOfRange, 0, 0));
  }
  int q = 0;
  u32x4 xl[XL ? 8 : 1];
  if constexpr (XL) {  // this wave's x fragments, requested before the weights
#pragma unroll
    for (int j = 0; j < 8; ++j) {
      const int ks = ks0 + j * kstride;
      xl[j] = __builtin_amdgcn_raw_buffer_load_b128(
          xr, ((uint32_t)ks * 1024u + lane * 16u) | ((uint32_t)(j >= my_ks || ks >= KS) << 31) | xrbad, 0, 0);
    }
  }
  if (total > 0) {
    load(0, wA, xA);
    epi_fetch(0, pA);
  }
  if (total > 1) {
    load(1, wB, xB);
    epi_fetch(1, pB);
  }
  if constexpr (XL) {  // (read back by this wave only)
#pragma unroll
    for (int j = 0; j < 8; ++j) s_xl[wave][j][lane] = xl[j];
  }
  // s_m = 1/sqrt(sum_p ss[p][m] / K + eps): lanes sum their partials in p order
  // (held ones first, then any beyond 64*RS_P), fixed shuffle tree.
  {
    float t[RS_ROWS];
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kMfmaWaves;
      t[r] = 0.f;
#pragma unroll
      for (int i = 0; i < RS_P; ++i) t[r] += rs_v[r][i];
      if (a.ss_in && m < a.M)
        for (int p = lane + RS_P * kWave; p < a.n_ss; p += kWave) t[r] += a.ss_in[(size_t)p * a.ss_ld + m];
    }
    wave_sum_n(t);
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kMfmaWaves;
      if (lane == 0 && m < MP) scale[m] = (a.ss_in && m < a.M) ? 1.0f / sqrtf(t[r] / (float)a.K + a.eps) : 1.0f;
    }
  }
  if constexpr (QKV) {
#pragma unroll
    for (int e = 0; e < CS_E; ++e) {
      const int i = tid + e * kMfmaThreads;
      s_cs[i / 128][i % 128] = cs_v[e];
    }
    if (tid < MP) s_rows[tid] = rd_v;
  }
  // A buffer is refilled as soon as its batch has been multiplied, before the
  // tile's reduction and epilogue (which use only the accumulators, LDS and
  // the epilogue inputs fetched with that batch): two batches stay in flight
  // across tile boundaries.
  while (q < total) {
    compute(wA, xA, q);
    if (q + 2 < total) load(q + 2, wA, xA);
    finish(q, pA);
    if (q + 2 < total) epi_fetch(q + 2, pA);
    if (++q >= total) break;
    compute(wB, xB, q);
    if (q + 2 < total) load(q + 2, wB, xB);
    finish(q, pB);
    if (q + 2 < total) epi_fetch(q + 2, pB);
    ++q;
  }
}

// ---------------------------------------------------------------- INT4 kernel for passes of at most 16 rows
// A block (one per CU, 8 waves) owns U units of TU 16-row tiles (unit
// blockIdx.x + i*gridDim.x; a SwiGLU unit pairs a gate tile with an up tile)
// and wave w reduces groups [w*gw, (w+1)*gw) of 128 columns of all of them.
// Every code block (16 bytes per lane, tile and group) and group scale of the
// wave is requested in the prologue, so the block's whole weight share is in
// flight before the first multiply; the activations go through LDS instead
// of registers.  Per window of GPW groups per wave, the block turns its x
// chunks (8 columns of one row) into hi + lo bf16 operands, ordered as the
// code unpacking orders columns; a group's sum over its four k-steps is
// multiplied by the group's scale in float32.
constexpr int kQ4Threads = 512;
constexpr int kQ4Waves = kQ4Threads / kWave;
constexpr int kQ4Rows = 16;                    // rows per launch
constexpr int kQ4RowBlock = 16 * 32 + 16;      // window bytes of one (group, row): 16 chunks, padding
constexpr int kQ4WindowBytes = 128 * 1024;
constexpr int kQ4WindowRows = kQ4WindowBytes / kQ4RowBlock / kQ4Waves;  // GPW * M per window <= this (31)
constexpr int kQ4Chunks = (kQ4Waves * kQ4WindowRows * 16 + kQ4Threads - 1) / kQ4Threads;  // per thread

typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));

// One k-step's code word (8 columns of the lane's row) as biased bf16 MFMA
// operands 136 + q (bits 0x4300 | (q + 8)): element 2d is column d, element
// 2d + 1 column d + 4.  (The nibble's two's-complement sign bit flipped gives
// q + 8; both that flip and the 0x4300 exponent bits are one XOR after the
// mask, since the mask leaves those bits zero.)
__device__ __forceinline__ bf16x8 q4_operand(uint32_t w) {
  u32x4 v;
  v[0] = (w & 0x000F000Fu) ^ 0x43084308u;
  v[1] = ((w >> 4) & 0x000F000Fu) ^ 0x43084308u;
  v[2] = ((w >> 8) & 0x000F000Fu) ^ 0x43084308u;
  v[3] = ((w >> 12) & 0x000F000Fu) ^ 0x43084308u;
  return __builtin_bit_cast(bf16x8, v);
}

template <int U, int TU, int GW, int GPW, int KIND>
__global__ __launch_bounds__(kQ4Threads) void gemm_q4_lds(GemmArgs a, int n_units, int gw) {
  // GPW: groups per wave per window (GPW * M <= kQ4WindowRows); the windows
  // are a compile-time sequence, so no branch joins paths with different
  // loads in flight (which would force waits for every outstanding load).
  constexpr int F = U * TU, NC = 16 * TU, NWIN = (GW + GPW - 1) / GPW;
  constexpr bool QKV = KIND == EPI_QKV;
  __shared__ __align__(16) unsigned char s_win[kQ4WindowBytes];    // x window, then the cross-wave sums
  __shared__ float yfin[U][kQ4Rows][NC + 1];
  __shared__ float scale[kQ4Rows];
  __shared__ RowDesc s_rows[QKV ? kQ4Rows : 1];
  __shared__ float s_cs[QKV ? kQ4Rows : 1][QKV ? 128 : 1];

  const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int M = a.M, K = a.K, G = (K + 127) / 128;
  const int my_g = max(0, min(G - wave * gw, gw));  // groups of this wave
  const int n_chunks = kQ4Waves * GPW * M * 16;      // x chunks per window
  const int chr = (n_chunks + kQ4Threads - 1) / kQ4Threads;  // of them per thread (<= kQ4Chunks)

  // Window wi: chunk c = (slot*M + m)*16 + 4j + kq, slot = wave'*GPW + lgw,
  // holds x[m][128*grp + 32j + 8kq .. +7] of group grp = wave'*gw + wi*GPW + lgw.
  f32x4 xw[kQ4Chunks][2];
  auto load_window = [&](int wi) {
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(a.x, (uint32_t)M * a.ldx * 4u);
#pragma unroll
    for (int i = 0; i < kQ4Chunks; ++i) {
      // (block-uniform: pieces past the window's rows are not requested at all;
      // an out-of-range load still takes its issue slot in the texture unit)
      if (i >= chr) break;
      const int c = tid + i * kQ4Threads, jq = c & 15, r = c >> 4;
      const int m = r % M, slot = r / M, lg = wi * GPW + slot % GPW;
      const int grp = (slot / GPW) * gw + lg;
      const int col = grp * 128 + (jq >> 2) * 32 + (jq & 3) * 8;
      const uint32_t bad = (uint32_t)(c >= n_chunks || lg >= gw || grp >= G || col >= K) << 31;
      const uint32_t off = (((uint32_t)m * a.ldx + col) * 4u) | bad;
      xw[i][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, off, 0, 0));
      xw[i][1] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(xr, off + 16u, 0, 0));
    }
  };
  auto store_window = [&]() {
#pragma unroll
    for (int i = 0; i < kQ4Chunks; ++i) {
      const int c = tid + i * kQ4Threads, jq = c & 15, r = c >> 4;
      if (c < n_chunks) {
        // columns 0, 4, 1, 5, 2, 6, 3, 7 (the order of the unpacked codes)
        const f32x2 p0 = {xw[i][0][0], xw[i][1][0]}, p1 = {xw[i][0][1], xw[i][1][1]};
        const f32x2 p2 = {xw[i][0][2], xw[i][1][2]}, p3 = {xw[i][0][3], xw[i][1][3]};
        const bf16x2 h0 = __builtin_convertvector(p0, bf16x2), h1 = __builtin_convertvector(p1, bf16x2);
        const bf16x2 h2 = __builtin_convertvector(p2, bf16x2), h3 = __builtin_convertvector(p3, bf16x2);
        const f32x2 r0 = p0 - __builtin_convertvector(h0, f32x2), r1 = p1 - __builtin_convertvector(h1, f32x2);
        const f32x2 r2 = p2 - __builtin_convertvector(h2, f32x2), r3 = p3 - __builtin_convertvector(h3, f32x2);
        const u32x4 hv = {__builtin_bit_cast(uint32_t, h0), __builtin_bit_cast(uint32_t, h1),
                          __builtin_bit_cast(uint32_t, h2), __builtin_bit_cast(uint32_t, h3)};
        const u32x4 lv = {__builtin_bit_cast(uint32_t, __builtin_convertvector(r0, bf16x2)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector(r1, bf16x2)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector(r2, bf16x2)),
                          __builtin_bit_cast(uint32_t, __builtin_convertvector(r3, bf16x2))};
        unsigned char* dst = s_win + r * kQ4RowBlock + jq * 32;
        *(u32x4*)dst = hv;
        *(u32x4*)(dst + 16) = lv;
      }
    }
  };

  // Prologue: the first window's x, the row-scale partials and the QKV
  // tables are requested before the scales and codes (loads complete in
  // order, so the conversions below wait for them alone).
  load_window(0);
  constexpr int RS_ROWS = kQ4Rows / kQ4Waves, RS_P = 4;
  float rs_v[RS_ROWS][RS_P];
  {
    const __amdgpu_buffer_rsrc_t sr = make_rsrc(a.ss_in, a.ss_in ? (uint32_t)a.n_ss * a.ss_ld * 4u : 0u);
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kQ4Waves;
#pragma unroll
      for (int i = 0; i < RS_P; ++i) {
        const int p = lane + i * kWave;
        const uint32_t off = (m < M && p < a.n_ss) ? ((uint32_t)p * a.ss_ld + m) * 4u : kOutOfRange;
        rs_v[r][i] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(sr, off, 0, 0));
      }
    }
  }
  constexpr int CS_E = QKV ? kQ4Rows * 128 / kQ4Threads : 1;
  float cs_v[CS_E];
  RowDesc rd_v{0, 0, 0, 0};
  if constexpr (QKV) {
    const __amdgpu_buffer_rsrc_t cr = make_rsrc(a.rope_cs, (uint32_t)M * a.head_dim * 4u);
#pragma unroll
    for (int e = 0; e < CS_E; ++e) {
      const int i = tid + e * kQ4Threads, m = i / 128, j = i % 128;
      const uint32_t off = j < a.head_dim ? ((uint32_t)m * a.head_dim + j) * 4u : kOutOfRange;
      cs_v[e] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(cr, off, 0, 0));
    }
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.rows, (uint32_t)M * (uint32_t)sizeof(RowDesc));
    rd_v = __builtin_bit_cast(RowDesc, __builtin_amdgcn_raw_buffer_load_b128(
                                           rr, tid < kQ4Rows ? (uint32_t)tid * (uint32_t)sizeof(RowDesc) : kOutOfRange,
                                           0, 0));
  }
  // Residual GEMMs (one 16-column unit): the old h and the next RMSNorm gain of
  // this thread's output element.
  constexpr bool PRE = KIND == EPI_RESID && U == 1;
  float pre_h = 0.f;
  uint32_t pre_g = 0u;
  if constexpr (PRE) {
    const int m = tid / 16, n = blockIdx.x * 16 + tid % 16;
    const uint32_t bad = (uint32_t)(m >= M || n >= a.n_rows) << 31;
    const __amdgpu_buffer_rsrc_t hr = make_rsrc(a.out, (uint32_t)M * a.ldo * 4u);
    const __amdgpu_buffer_rsrc_t gr = make_rsrc(a.gain_out, (uint32_t)a.n_rows * 2u);
    pre_h = __builtin_bit_cast(
        float, __builtin_amdgcn_raw_buffer_load_b32(hr, (((uint32_t)m * a.ldo + n) * 4u) | bad, 0, 0));
    pre_g = __builtin_amdgcn_raw_buffer_load_b16(gr, ((uint32_t)n * 2u) | bad, 0, 0);
  }
  // The wave's code blocks and scales, group-major.  All scales come first
  // (a group's products wait for its scales, and loads complete in issue
  // order); the codes of D groups are requested here and each later group's
  // D groups ahead of its products.  A shallow depth keeps the prologue's
  // vector-memory issue short, so it does not hold up the x conversion:
  // deeper requests (up to 8 groups, about 64 KB per CU in flight) measured
  // 2% slower over a 7B verify, and one group is too few below six.
  constexpr int D = F >= 6 ? 1 : 2;
  u32x4 cw[F][GW];
  uint32_t sw[F][GW];
  __amdgpu_buffer_rsrc_t crs[F], srs[F];
#pragma unroll
  for (int f = 0; f < F; ++f) {
    const int unit = blockIdx.x + (f / TU) * gridDim.x;
    int seg, n;
    bool ok;
    tile_segment(a, KIND, unit, NC, f % TU, seg, n, ok);
    ok = ok && unit < n_units;
    crs[f] = make_rsrc((const char*)a.w[seg] + (size_t)(n / 16) * G * 1024, ok ? (uint32_t)G * 1024u : 0u);
    srs[f] = make_rsrc(a.wscale[seg] + (size_t)(n / 16) * G * 16, ok ? (uint32_t)G * 32u : 0u);
  }
#pragma unroll
  for (int lg = 0; lg < GW; ++lg) {
    const uint32_t bad = (uint32_t)(lg >= my_g) << 31;
#pragma unroll
    for (int f = 0; f < F; ++f)
      sw[f][lg] = __builtin_amdgcn_raw_buffer_load_b16(
          srs[f], ((uint32_t)(wave * gw + lg) * 32u + (lane & 15) * 2u) | bad, 0, 0);
  }
  __builtin_amdgcn_sched_barrier(0);
  auto issue_codes = [&](int lg) {
    const uint32_t bad = (uint32_t)(lg >= my_g) << 31;
#pragma unroll
    for (int f = 0; f < F; ++f)
      cw[f][lg] = __builtin_amdgcn_raw_buffer_load_b128(
          crs[f], ((uint32_t)(wave * gw + lg) * 1024u + lane * 16u) | bad, 0, kNonTemporal);
    __builtin_amdgcn_sched_barrier(0);
  };
#pragma unroll
  for (int lg = 0; lg < D && lg < GW; ++lg) issue_codes(lg);

  {
    float t[RS_ROWS];
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kQ4Waves;
      t[r] = 0.f;
#pragma unroll
      for (int i = 0; i < RS_P; ++i) t[r] += rs_v[r][i];
      if (a.ss_in && m < M)
        for (int p = lane + RS_P * kWave; p < a.n_ss; p += kWave) t[r] += a.ss_in[(size_t)p * a.ss_ld + m];
    }
    wave_sum_n(t);
#pragma unroll
    for (int r = 0; r < RS_ROWS; ++r) {
      const int m = wave + r * kQ4Waves;
      if (lane == 0) scale[m] = (a.ss_in && m < M) ? 1.0f / sqrtf(t[r] / (float)K + a.eps) : 1.0f;
    }
  }
  if constexpr (QKV) {
#pragma unroll
    for (int e = 0; e < CS_E; ++e) {
      const int i = tid + e * kQ4Threads;
      s_cs[i / 128][i % 128] = cs_v[e];
    }
    if (tid < kQ4Rows) s_rows[tid] = rd_v;
  }
  store_window();
  __syncthreads();

  floatx4 acc[F];
#pragma unroll
  for (int f = 0; f < F; ++f) acc[f] = floatx4{0.f, 0.f, 0.f, 0.f};
  const int kq = lane >> 4;
  // STACK (at most 8 rows, GPW > 1 implies M <= 7): the hi parts of the rows
  // go to A rows 0..7 and the lo parts to rows 8..15, so one product per
  // k-step covers both; output rows m and m + 8 are added after the
  // cross-wave sums.  Otherwise hi and lo are two products.
  constexpr bool STACK = GPW > 1;
  // The +136 bias of the code operands is cancelled by the product of the same
  // x with -136 (bf16 0xC308), shared by the block's tiles and added to each
  // tile's group sum before the scale.
  const bf16x8 m136 = __builtin_bit_cast(bf16x8, u32x4{0xC308C308u, 0xC308C308u, 0xC308C308u, 0xC308C308u});
  auto compute_group = [&](int lg) {
    const int slot = wave * GPW + lg % GPW;
    floatx4 pb = floatx4{0.f, 0.f, 0.f, 0.f};
    if constexpr (STACK) {
      const unsigned char* xa =
          s_win + (slot * M + min(lane & 7, M - 1)) * kQ4RowBlock + kq * 32 + ((lane >> 3) & 1) * 16;
      floatx4 p[F];
#pragma unroll
      for (int f = 0; f < F; ++f) p[f] = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8 xv = *(const bf16x8*)(xa + j * 128);
        pb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, m136, pb, 0, 0, 0);
#pragma unroll
        for (int f = 0; f < F; ++f)
          p[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(xv, q4_operand(cw[f][lg][j]), p[f], 0, 0, 0);
      }
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const float sc = bf16_bits_to_f32((uint16_t)sw[f][lg]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[f][r] = fmaf(sc, p[f][r] + pb[r], acc[f][r]);
      }
    } else {
      const unsigned char* xb = s_win + (slot * M + min(lane & 15, M - 1)) * kQ4RowBlock + kq * 32;
      floatx4 ph[F], pl[F];
#pragma unroll
      for (int f = 0; f < F; ++f) {
        ph[f] = floatx4{0.f, 0.f, 0.f, 0.f};
        pl[f] = floatx4{0.f, 0.f, 0.f, 0.f};
      }
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const bf16x8 hi = *(const bf16x8*)(xb + j * 128), lo = *(const bf16x8*)(xb + j * 128 + 16);
        pb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, m136, pb, 0, 0, 0);
        pb = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, m136, pb, 0, 0, 0);
#pragma unroll
        for (int f = 0; f < F; ++f) {
          const bf16x8 b = q4_operand(cw[f][lg][j]);
          ph[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(hi, b, ph[f], 0, 0, 0);
          pl[f] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(lo, b, pl[f], 0, 0, 0);
        }
      }
#pragma unroll
      for (int f = 0; f < F; ++f) {
        const float sc = bf16_bits_to_f32((uint16_t)sw[f][lg]);
#pragma unroll
        for (int r = 0; r < 4; ++r) acc[f][r] = fmaf(sc, (ph[f][r] + pl[f][r]) + pb[r], acc[f][r]);
      }
    }
  };
  // (blocks of one tile have the registers to fetch the next window's x while
  // the current one is multiplied; a window past the wave's groups loads
  // nothing and converts zeros)
  constexpr bool PREFETCH = F == 1;
#pragma unroll
  for (int w = 0; w < NWIN; ++w) {
    if (w > 0) {
      __syncthreads();
      if constexpr (!PREFETCH) load_window(w);
      store_window();
      __syncthreads();
    }
    if constexpr (PREFETCH) {
      if (w + 1 < NWIN) load_window(w + 1);
    }
#pragma unroll
    for (int i = 0; i < GPW; ++i) {
      const int lg = w * GPW + i;
      if (lg + D < GW) issue_codes(lg + D);
      if (lg < GW && lg < my_g) compute_group(lg);
    }
  }

  // Cross-wave sums in fixed wave order: red[f][wave][lane][r] -> yfin.
  __syncthreads();
  float* red = (float*)s_win;
#pragma unroll
  for (int f = 0; f < F; ++f) *(floatx4*)&red[((f * kQ4Waves + wave) * kWave + lane) * 4] = acc[f];
  __syncthreads();
  for (int i = tid; i < F * kWave * 4; i += kQ4Threads) {
    const int f = i / (kWave * 4), l = (i / 4) % kWave, r = i % 4;
    float s = 0.f;
#pragma unroll
    for (int w = 0; w < kQ4Waves; ++w) s += red[((f * kQ4Waves + w) * kWave + l) * 4 + r];
    yfin[f / TU][4 * (l >> 4) + r][(f % TU) * 16 + (l & 15)] = s;
  }
  __syncthreads();
  if constexpr (STACK) {  // rows m (hi parts) + m + 8 (lo parts)
    for (int i = tid; i < U * 8 * NC; i += kQ4Threads) {
      const int u = i / (8 * NC), m = (i / NC) % 8, c = i % NC;
      yfin[u][m][c] += yfin[u][m + 8][c];
    }
    __syncthreads();
  }
  if constexpr (PRE) {  // h += y; xg = h * gain; sum of squares of the unit's new h
    const int m = tid / 16, c = tid % 16, n = blockIdx.x * 16 + c;
    if (m < M) {
      float hv = 0.f;
      if (n < a.n_rows) {
        hv = pre_h + yfin[0][m][c];
        a.out[(size_t)m * a.ldo + n] = hv;
        const float xv = hv * bf16_bits_to_f32((uint16_t)pre_g);
        if (a.xs_out) put_stacked(a.xs_out, a.stt_out, m, n, xv);
        else a.xg_out[(size_t)m * a.ldo + n] = xv;
      }
      yfin[0][m][c] = hv;
    }
    __syncthreads();
    if (tid < M) {
      float t = 0.f;
      for (int c2 = 0; c2 < 16; ++c2) t += yfin[0][tid][c2] * yfin[0][tid][c2];
      a.ss_out[(size_t)blockIdx.x * a.ss_ld + tid] = t;
    }
    return;
  }
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int unit = blockIdx.x + u * gridDim.x;
    if (unit >= n_units) break;  // (block-uniform)
    if constexpr (QKV) qkv_epilogue<NC, kQ4Threads>(a, unit, yfin[u], scale, s_rows, s_cs);
    else epilogue<NC, KIND, kQ4Threads>(a, unit, yfin[u], scale);
  }
}

// ---------------------------------------------------------------- vector kernel (float32 weights)
// Block = 4 waves over NC weight rows; each wave takes NC/4 rows, lanes stride
// over K; M processed 8 rows at a time.
template <int NC, int KIND>
__global__ __launch_bounds__(256) void gemm_f32_vector(GemmArgs a) {
  constexpr int MPMAX = kMaxGemmRows;
  __shared__ float yfin[MPMAX][NC + 1];
  __shared__ float scale[MPMAX];
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
  const int blk = blockIdx.x;
  row_scale<MPMAX>(a, scale);
  for (int c = wave; c < NC; c += 4) {
    bool ok;
    const float* wr = weight_row<float>(a, KIND, blk, NC, c, ok);
    for (int m0 = 0; m0 < a.M; m0 += 8) {
      float acc[8];
#pragma unroll
      for (int i = 0; i < 8; ++i) acc[i] = 0.f;
      if (ok) {
        for (int k = lane; k < a.K; k += kWave) {
          float w = wr[k];
#pragma unroll
          for (int i = 0; i < 8; ++i)
            if (m0 + i < a.M) acc[i] += w * a.x[(size_t)(m0 + i) * a.ldx + k];
        }
      }
#pragma unroll
      for (int i = 0; i < 8; ++i) {
        float s = wave_sum(acc[i]);
        if (lane == 0 && m0 + i < a.M) yfin[m0 + i][c] = s;
      }
    }
  }
  __syncthreads();
  epilogue<NC, KIND, 256>(a, blk, yfin, scale);
}

int compute_units() {
  static int cus = [] {
    int dev = 0, n = 0;
    if (hipGetDevice(&dev) != hipSuccess || hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) !=
                                                 hipSuccess || n <= 0)
      n = 256;
    return n;
  }();
  return cus;
}

// k-steps per register buffer: two buffers' W and x fragments stay within the
// 128 VGPRs a wave of a 16-wave block may use.  (INT4 weights: as many, with a
// k-step's fragment a quarter of the bf16 one.  Single-tile units reading one
// stacked x fragment per k-step, from memory or LDS, have the registers for
// four: measured 9.9 -> 9.2 us for the 7B O projection; two fragments per
// k-step or float32 x would spill.)
template <int T, int XS> struct Batch {
  static constexpr int UB = T == 1 ? (XS == 1 || XS == 3 ? 4 : 3) : (T == 2 ? 2 : 1);
};

template <int T, int KIND, int XS>
hipError_t launch_mfma_x(const GemmArgs& a, int tiles, hipStream_t s) {
  const int grid = tiles < compute_units() ? tiles : compute_units();
  hipLaunchKernelGGL((gemm_bf16_mfma<T, Batch<T, XS>::UB, KIND, XS>), dim3(grid), dim3(kMfmaThreads), 0, s, a, tiles);
  return hipGetLastError();
}

// bf16 weights: a residual GEMM, x held in LDS where a wave's share of one
// fragment per k-step fits.
template <int T>
hipError_t launch_mfma_t(const GemmArgs& a, int blocks, hipStream_t s) {
  if (a.stt != (a.M <= 8 ? 1 : 2)) return hipErrorInvalidValue;
  if (a.M > 8) return launch_mfma_x<T, EPI_RESID, 2>(a, blocks, s);
  if ((a.K + 31) / 32 <= 8 * kMfmaWaves) return launch_mfma_x<T, EPI_RESID, 3>(a, blocks, s);
  return launch_mfma_x<T, EPI_RESID, 1>(a, blocks, s);
}

// 16-row tiles per work unit of the bf16 kernel.  More tiles per unit mean
// fewer activation loads per weight byte; the choice balances the units over
// the CUs of the persistent grid (ties go to the larger unit).  SwiGLU pairs
// a gate tile with an up tile.
int mfma_tiles(int kind, int n_rows) {
  if (kind == EPI_SWIGLU) return 2;
  const int cus = compute_units();
  int best = 1;
  double best_eff = 0.0;
  for (int T = 3; T >= 1; --T) {
    const int units = (n_rows + 16 * T - 1) / (16 * T);
    const int rounds = (units + cus - 1) / cus;
    const double eff = (double)units / ((double)rounds * cus);
    if (eff > best_eff + 1e-9) {
      best_eff = eff;
      best = T;
    }
  }
  return best;
}

// One thread per 16-byte piece of the packed image of W [N, K] (row-major).
__global__ void pack_kernel(const uint16_t* __restrict__ src, uint16_t* __restrict__ dst, int N, int K, int KS,
                            int rope_hd) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  const size_t pieces = (size_t)(N / 16) * KS * 64;
  if (i >= pieces) return;
  const int lane = (int)(i % 64);
  const size_t frag = i / 64;
  const int ks = (int)(frag % KS), t = (int)(frag / KS);
  int row = 16 * t + (lane & 15);
  if (rope_hd > 0) {  // tile t of its head: rows 8t' + e and hd/2 + 8t' + e, e < 8
    const int head = (16 * t) / rope_hd, tq = (16 * t) % rope_hd / 16, e = lane & 15;
    row = head * rope_hd + (e < 8 ? 8 * tq + e : rope_hd / 2 + 8 * tq + (e - 8));
  }
  const int k = 32 * ks + 8 * (lane >> 4);
  u32x4 v = u32x4{0u, 0u, 0u, 0u};
  if (k + 8 <= K) {
    v = *(const u32x4*)(src + (size_t)row * K + k);
  } else {
    uint16_t e[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) e[j] = k + j < K ? src[(size_t)row * K + k + j] : 0;
    v = u32x4{e[0] | (uint32_t)e[1] << 16, e[2] | (uint32_t)e[3] << 16, e[4] | (uint32_t)e[5] << 16,
              e[6] | (uint32_t)e[7] << 16};
  }
  *(u32x4*)(dst + i * 8) = v;
}

// INT4 quantization and packing, one thread per (packed row n, group of 128
// columns): s = bf16(max|w| / 7) (IEEE division), q = clamp(rint(w / s), -8, 7)
// (q = 0 where s = 0); the thread writes its row's 16 code words of the
// group and the row's scale.  Rows follow the bf16 image's order (rope_hd).
__global__ void pack_int4_kernel(const uint16_t* __restrict__ src, uint32_t* __restrict__ frag,
                                 uint16_t* __restrict__ scale, int N, int K, int KS, int KG, int rope_hd) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i >= (size_t)N * KG) return;
  const int n = (int)(i / KG), g = (int)(i % KG);
  int row = n;
  if (rope_hd > 0) {
    const int t = n / 16, head = (16 * t) / rope_hd, tq = (16 * t) % rope_hd / 16, e = n & 15;
    row = head * rope_hd + (e < 8 ? 8 * tq + e : rope_hd / 2 + 8 * tq + (e - 8));
  }
  const uint16_t* w = src + (size_t)row * K;
  const int k0 = g * 128, k1 = min(K, k0 + 128);
  float amax = 0.f;
  for (int k = k0; k < k1; ++k) amax = fmaxf(amax, fabsf(bf16_bits_to_f32(w[k])));
  const __bf16 sb = (__bf16)__fdiv_rn(amax, 7.0f);
  const float sf = (float)sb;
  scale[((size_t)(n / 16) * KG + g) * 16 + (n & 15)] = __builtin_bit_cast(uint16_t, sb);
  // (the group's four k-steps: a k-step past K keeps zero codes)
  for (int j = 0; j < 4; ++j)
    for (int kg = 0; kg < 4; ++kg) {
      const int ks = 4 * g + j;
      uint32_t word = 0u;
      for (int e = 0; e < 8; ++e) {
        const int k = ks * 32 + kg * 8 + e;
        int q = 0;
        if (ks < KS && k < K && sf != 0.f)
          q = (int)fminf(fmaxf(rintf(__fdiv_rn(bf16_bits_to_f32(w[k]), sf)), -8.f), 7.f);
        word |= ((uint32_t)q & 0xFu) << (4 * e);
      }
      frag[(((size_t)(n / 16) * KG + g) * 64 + kg * 16 + (n & 15)) * 4 + j] = word;
    }
}

}  // namespace

int device_compute_units() { return compute_units(); }

size_t packed_int4_frag_bytes(int N, int K) { return (size_t)(N / 16) * ((K + 127) / 128) * 1024; }
size_t packed_int4_scale_bytes(int N, int K) { return (size_t)(N / 16) * ((K + 127) / 128) * 32; }

hipError_t launch_pack_int4(const void* src, void* frag, void* scale, int N, int K, int rope_hd, hipStream_t s) {
  if (N % 16 || K % 32) return hipErrorInvalidValue;
  if (rope_hd < 0 || (rope_hd > 0 && (rope_hd % 16 || N % rope_hd))) return hipErrorInvalidValue;
  const int KS = K / 32, KG = (K + 127) / 128;
  const size_t n = (size_t)N * KG;
  hipLaunchKernelGGL(pack_int4_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, (const uint16_t*)src,
                     (uint32_t*)frag, (uint16_t*)scale, N, K, KS, KG, rope_hd);
  return hipGetLastError();
}

size_t packed_elems(int N, int K) { return (size_t)(N / 16) * ((K + 31) / 32) * 512; }

hipError_t launch_pack(const void* src, void* dst, int N, int K, int rope_hd, hipStream_t s) {
  if (N % 16 || K % 8) return hipErrorInvalidValue;
  if (rope_hd < 0 || (rope_hd > 0 && (rope_hd % 16 || N % rope_hd))) return hipErrorInvalidValue;
  const int KS = (K + 31) / 32;
  const size_t pieces = (size_t)(N / 16) * KS * 64;
  hipLaunchKernelGGL(pack_kernel, dim3((unsigned)((pieces + 255) / 256)), dim3(256), 0, s, (const uint16_t*)src,
                     (uint16_t*)dst, N, K, KS, rope_hd);
  return hipGetLastError();
}

bool gemm_wide(int dtype, int M) { return dtype == SPECDEC_BF16 && M > kMaxGemmRows; }
int gemm_launch_rows(int dtype, int M) {
  return gemm_wide(dtype, M) ? kTileLaunchRows : kMaxGemmRows;
}

int gemm_row_blocks(int dtype, int kind, int n_rows, int M) {
  if (kind == EPI_RESID && dtype == SPECDEC_BF16 && M > kSkinnyRows) return (n_rows + kTileReduceCols - 1) / kTileReduceCols;
  if (dtype == SPECDEC_BF16) {
    int nc = 16 * mfma_tiles(kind, n_rows);
    int per = kind == EPI_SWIGLU ? nc / 2 : nc;
    return (n_rows + per - 1) / per;
  }
  int per = kind == EPI_SWIGLU ? 16 : 16;
  return (n_rows + per - 1) / per;
}

// INT4 passes of at most 16 rows on gemm_q4_lds: hipErrorNotSupported where
// its register budget does not cover the shape (the caller then runs the
// skinny kernel's INT4 path).  Groups per wave and window: all of them (one
// window) while the rows allow, else one.
template <int U, int TU, int GW, int KIND>
static void launch_q4_w(const GemmArgs& a, int n_units, int gw, hipStream_t s) {
  const int grid = std::min(n_units, compute_units());
  constexpr int G1 = GW == 4 ? 4 : 6;  // (12 groups: two windows of 6 for up to 5 rows)
  if (G1 * a.M <= kQ4WindowRows)
    hipLaunchKernelGGL((gemm_q4_lds<U, TU, GW, G1, KIND>), dim3(grid), dim3(kQ4Threads), 0, s, a, n_units, gw);
  else
    hipLaunchKernelGGL((gemm_q4_lds<U, TU, GW, 1, KIND>), dim3(grid), dim3(kQ4Threads), 0, s, a, n_units, gw);
}

template <int U, int TU, int KIND>
static hipError_t launch_q4_u(const GemmArgs& a, int n_units, int gw, hipStream_t s) {
  if (gw <= 4) {
    launch_q4_w<U, TU, 4, KIND>(a, n_units, gw, s);
  } else if constexpr (U * TU == 1) {  // (12 groups per wave: single-tile units only)
    if (gw > 12) return hipErrorNotSupported;
    launch_q4_w<U, TU, 12, KIND>(a, n_units, gw, s);
  } else {
    return hipErrorNotSupported;
  }
  return hipGetLastError();
}

static hipError_t launch_q4_lds(const GemmArgs& a, hipStream_t s) {
  if (a.M > kQ4Rows || a.n_rows % 16 || (a.kind == EPI_QKV && a.head_dim > 128)) return hipErrorNotSupported;
  // (residual GEMMs: one tile per unit, as the RMSNorm partials of the consumer expect)
  if (a.kind == EPI_RESID && mfma_tiles(EPI_RESID, a.n_rows) != 1) return hipErrorNotSupported;
  const int n_units = a.n_rows / 16, cus = compute_units();
  const int U = (n_units + cus - 1) / cus;
  const int G = (a.K + 127) / 128, gw = (G + kQ4Waves - 1) / kQ4Waves;
  switch (a.kind) {
    case EPI_QKV:
      if (U == 1) return launch_q4_u<1, 1, EPI_QKV>(a, n_units, gw, s);
      if (U == 2) return launch_q4_u<2, 1, EPI_QKV>(a, n_units, gw, s);
      if (U == 3) return launch_q4_u<3, 1, EPI_QKV>(a, n_units, gw, s);
      break;
    case EPI_SWIGLU:
      if (U == 1) return launch_q4_u<1, 2, EPI_SWIGLU>(a, n_units, gw, s);
      if (U == 2) return launch_q4_u<2, 2, EPI_SWIGLU>(a, n_units, gw, s);
      if (U == 3) return launch_q4_u<3, 2, EPI_SWIGLU>(a, n_units, gw, s);
      break;
    case EPI_RESID:
      if (U == 1) return launch_q4_u<1, 1, EPI_RESID>(a, n_units, gw, s);
      if (U == 2) return launch_q4_u<2, 1, EPI_RESID>(a, n_units, gw, s);
      break;
    default: break;
  }
  return hipErrorNotSupported;
}

hipError_t launch_gemm(int dtype, const GemmArgs& a, hipStream_t s) {
  if (a.M <= 0 || (a.K % 8) != 0 || (a.ldx % 4) != 0) return hipErrorInvalidValue;
  if (a.wide) {
    if (a.q4) return hipErrorInvalidValue;  // (INT4 weights run passes of at most 64 rows)
    if (dtype != SPECDEC_BF16 || (a.kind == EPI_RESID && (!a.gain_bf16 || a.n_rows % 4))) return hipErrorInvalidValue;
    return launch_gemm_tile(a, s);
  }
  if (a.M > kMaxGemmRows) return hipErrorInvalidValue;
  if (dtype == SPECDEC_BF16 && (a.M > kSkinnyRows || (!a.q4 && a.kind != EPI_RESID))) return launch_gemm_rows(a, s);
  const int blocks = gemm_row_blocks(dtype, a.kind, a.n_rows, a.M);
  if (a.q4) {  // INT4 layer weights (passes of at most 64 rows)
    if (dtype != SPECDEC_BF16 || (a.K % 32) != 0) return hipErrorInvalidValue;
    if (a.kind == EPI_RESID && !a.gain_bf16) return hipErrorInvalidValue;
    if (a.kind == EPI_QKV && (a.kv.dtype != SPECDEC_BF16 || a.head_dim % 16 || a.n_seg[0] % a.head_dim ||
                              a.n_seg[1] % a.head_dim))
      return hipErrorInvalidValue;
    const hipError_t e = launch_q4_lds(a, s);
    if (e != hipErrorNotSupported) return e;
    const int T = mfma_tiles(a.kind, a.n_rows);
    switch (a.kind) {
      case EPI_RESID:
        if (!a.gain_bf16) return hipErrorInvalidValue;
        return T == 1 ? launch_mfma_x<1, EPI_RESID, 0>(a, blocks, s)
                      : (T == 2 ? launch_mfma_x<2, EPI_RESID, 0>(a, blocks, s)
                                : launch_mfma_x<3, EPI_RESID, 0>(a, blocks, s));
      case EPI_SWIGLU: return launch_mfma_x<2, EPI_SWIGLU, 0>(a, blocks, s);
      case EPI_QKV:
        if (a.kv.dtype != SPECDEC_BF16 || a.head_dim % 16 || a.n_seg[0] % a.head_dim || a.n_seg[1] % a.head_dim)
          return hipErrorInvalidValue;
        return T == 1 ? launch_mfma_x<1, EPI_QKV, 0>(a, blocks, s)
                      : (T == 2 ? launch_mfma_x<2, EPI_QKV, 0>(a, blocks, s)
                                : launch_mfma_x<3, EPI_QKV, 0>(a, blocks, s));
      default: return hipErrorInvalidValue;
    }
  }
  if (dtype == SPECDEC_BF16) {  // (RESID: the other kinds run launch_gemm_rows)
    if (!a.gain_bf16 || !a.xs || !a.xs_out) return hipErrorInvalidValue;
    const int T = mfma_tiles(EPI_RESID, a.n_rows);
    return T == 1 ? launch_mfma_t<1>(a, blocks, s) : (T == 2 ? launch_mfma_t<2>(a, blocks, s) : launch_mfma_t<3>(a, blocks, s));
  }
  switch (a.kind) {
    case EPI_STORE: hipLaunchKernelGGL((gemm_f32_vector<16, EPI_STORE>), dim3(blocks), dim3(256), 0, s, a); break;
    case EPI_RESID: hipLaunchKernelGGL((gemm_f32_vector<16, EPI_RESID>), dim3(blocks), dim3(256), 0, s, a); break;
    case EPI_SWIGLU: hipLaunchKernelGGL((gemm_f32_vector<32, EPI_SWIGLU>), dim3(blocks), dim3(256), 0, s, a); break;
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

}  // namespace specdec
