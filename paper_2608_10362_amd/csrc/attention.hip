// RoPE + KV append and GQA attention of the verify / draft passes against the
// resident KV cache.
//
// The KV layout (internal.h) stores bf16 caches in MFMA operand order, so
// that every wavefront load of the attention kernel reads 1 KB contiguously.
//
// Attention is split over key chunks (flash-decoding style): one wave per
// (16-query tile, 64-key split, kv head, sequence) computes, for every query
// row of the sequence and every query head of the kv group, the chunk's max,
// exp-sum and unnormalised P V; a combine kernel merges the chunks per (row,
// head).  Query i of a sequence at position pos_i sees keys 0..pos_i (causal
// inside the verify block).
#include <algorithm>

#include "device_common.h"
#include "gemm_common.h"
#include "internal.h"

namespace specdec {

namespace {

// ---------------------------------------------------------------- RoPE + append
// Block (head slot, row): slots [0, H) rotate a query head into qr, [H, H+G)
// rotate a key head and store it at the row's position, [H+G, H+2G) store a
// value head (transposed).  Thread j handles the pair (j, j + hd/2).  (float32
// models; the bf16 Q|K|V GEMMs do this in their epilogues.)
__global__ __launch_bounds__(64) void rope_append_kernel(AttnArgs a) {
  const int hs = blockIdx.x, r = blockIdx.y, j = threadIdx.x;
  const int hd = a.head_dim, half = hd / 2, H = a.n_heads, G = a.n_kv_heads;
  if (j >= half) return;
  const RowDesc rd = a.rows[r];
  const float* src = a.qkv + (size_t)r * (H + 2 * G) * hd + (size_t)hs * hd;
  const float x1 = src[j], x2 = src[j + half];
  const int cap = a.kv.capacity;
  if (hs >= H + G) {  // value head
    if (!rd.valid) return;
    float* blk = k_block<float>(a.kv, a.layer, rd.b, hs - H - G);
    Storage<float>::store(blk + KvIndex<float>::v(rd.pos, j, hd, cap), x1);
    Storage<float>::store(blk + KvIndex<float>::v(rd.pos, j + half, hd, cap), x2);
    return;
  }
  const float* cs = a.rope_cs + (size_t)r * hd;
  const float c = cs[j], s = cs[half + j];
  const float y1 = x1 * c - x2 * s, y2 = x2 * c + x1 * s;
  if (hs < H) {
    float* q = a.qr + ((size_t)r * H + hs) * hd;
    q[j] = y1;
    q[j + half] = y2;
  } else if (rd.valid) {
    float* blk = k_block<float>(a.kv, a.layer, rd.b, hs - H);
    Storage<float>::store(blk + KvIndex<float>::k(rd.pos, j, hd, cap), y1);
    Storage<float>::store(blk + KvIndex<float>::k(rd.pos, j + half, hd, cap), y2);
  }
}

// ---------------------------------------------------------------- split-KV partials
constexpr int kQB = 16;  // queries per pass

template <typename KT>
__global__ __launch_bounds__(256) void attn_partial_kernel(AttnArgs a) {
  extern __shared__ float smem[];
  const int c = blockIdx.x, g = blockIdx.y, b = blockIdx.z;
  const int hd = a.head_dim, H = a.n_heads, G = a.n_kv_heads, group = H / G;
  const int rps = a.rps, r0 = b * rps, chunk = a.chunk;
  int nk = 0;
  for (int i = 0; i < rps; ++i) {
    const RowDesc rd = a.rows[r0 + i];
    if (rd.valid) nk = max(nk, rd.pos + 1);
  }
  const int kbeg = c * chunk;
  if (kbeg >= nk) return;
  const int nkeys = min(chunk, nk - kbeg);

  float* Ks = smem;                           // [chunk][hd+1]
  float* Vs = Ks + chunk * (hd + 1);          // [hd][chunk+1]
  float* qs = Vs + hd * (chunk + 1);          // [kQB][hd]
  float* S = qs + kQB * hd;                   // [kQB][chunk]
  float* ml = S + kQB * chunk;                // [kQB][2]

  const KT* kb = k_block<KT>(a.kv, a.layer, b, g);
  const KT* vb = kb + (size_t)a.kv.capacity * hd;
  for (int i = threadIdx.x; i < nkeys * hd; i += blockDim.x) {
    const int key = i / hd, dd = i % hd;
    Ks[key * (hd + 1) + dd] = Storage<KT>::load(kb + (size_t)(kbeg + key) * hd + dd);
  }
  for (int i = threadIdx.x; i < hd * nkeys; i += blockDim.x) {
    const int dd = i / nkeys, key = i % nkeys;
    Vs[dd * (chunk + 1) + key] = Storage<KT>::load(vb + (size_t)dd * a.kv.capacity + kbeg + key);
  }
  const float scale = 1.0f / sqrtf((float)hd);
  const int nq = rps * group;
  const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;

  for (int qb = 0; qb < nq; qb += kQB) {
    __syncthreads();  // tiles loaded / previous pass done with qs, S
    for (int i = threadIdx.x; i < kQB * hd; i += blockDim.x) {
      const int ql = i / hd, dd = i % hd, qi = qb + ql;
      float v = 0.f;
      if (qi < nq) {
        const int row = r0 + qi / group, head = g * group + qi % group;
        v = a.qr[((size_t)row * H + head) * hd + dd];
      }
      qs[i] = v;
    }
    __syncthreads();
    for (int p = threadIdx.x; p < kQB * chunk; p += blockDim.x) {
      const int ql = p / chunk, key = p % chunk, qi = qb + ql;
      float s = -INFINITY;
      if (qi < nq && key < nkeys) {
        const RowDesc rd = a.rows[r0 + qi / group];
        if (rd.valid && kbeg + key <= rd.pos) {
          const float* qv = qs + ql * hd;
          const float* kv = Ks + key * (hd + 1);
          float t = 0.f;
          for (int dd = 0; dd < hd; ++dd) t += qv[dd] * kv[dd];
          s = t * scale;
        }
      }
      S[p] = s;
    }
    __syncthreads();
    for (int ql = wave; ql < kQB; ql += 4) {
      float mx = -INFINITY;
      for (int key = lane; key < chunk; key += kWave) mx = fmaxf(mx, S[ql * chunk + key]);
      mx = wave_max(mx);
      float sum = 0.f;
      for (int key = lane; key < chunk; key += kWave) {
        const float s = S[ql * chunk + key];
        const float e = (mx == -INFINITY) ? 0.f : expf(s - mx);
        S[ql * chunk + key] = e;
        sum += e;
      }
      sum = wave_sum(sum);
      if (lane == 0) { ml[2 * ql] = mx; ml[2 * ql + 1] = sum; }
    }
    __syncthreads();
    for (int p = threadIdx.x; p < kQB * hd; p += blockDim.x) {
      const int ql = p / hd, dd = p % hd, qi = qb + ql;
      if (qi >= nq || ml[2 * ql] == -INFINITY) continue;
      const float* pr = S + ql * chunk;
      const float* vr = Vs + dd * (chunk + 1);
      float o = 0.f;
      for (int key = 0; key < nkeys; ++key) o += pr[key] * vr[key];
      const int row = r0 + qi / group, head = g * group + qi % group;
      const size_t slot = ((size_t)row * H + head) * a.n_split + c;
      a.o_part[slot * hd + dd] = o;
      if (dd == 0) { a.ml_part[2 * slot] = ml[2 * ql]; a.ml_part[2 * slot + 1] = ml[2 * ql + 1]; }
    }
  }
}

// ---------------------------------------------------------------- MFMA attention partials (bf16 cache)
// The keys [0, 32 n_sub) of each (kv head, sequence) are cut into n_part parts
// of S sub-chunks of 32 keys; the last part also takes the remainder (fewer
// than 2S sub-chunks).  One block per (part, 16-query tile, kv head,
// sequence) and one wave per sub-chunk.  S is chosen on the host so that the
// blocks about fill the CUs once: every CU then streams about the same number
// of K/V bytes.  Per wave, S = Q K^T and O = P V run on
// v_mfma_f32_16x16x32_bf16 with the float32 operands (Q, P) split into hi + lo
// bf16 parts; lane l holds rows 4(l/16)+r of S and O, so the per-row max and
// sum live in the same lanes.  The block merges its waves' (max, sum, O) in
// LDS (fixed wave order) and writes one partial per part.
constexpr int kSubKeys = 32;

__device__ __forceinline__ void split_hilo(const float* v, bf16x8& hi, bf16x8& lo) {
#pragma unroll
  for (int j = 0; j < 8; ++j) {
    const __bf16 h = (__bf16)v[j];
    hi[j] = h;
    lo[j] = (__bf16)(v[j] - (float)h);
  }
}

// One element of the attention output o[row][head * hd + d], into the stacked
// operand of the O projection where the pass hands x over stacked.
__device__ __forceinline__ void put_o(const AttnArgs& a, float* o, int row, int head, int d, float v) {
  if (a.xs) put_stacked(a.xs, a.stt, row, head * a.head_dim + d, v);
  else o[d] = v;
}

// Reductions over the 16 lanes of a row of the wave (lanes 16k .. 16k+15)
// with DPP moves: swaps within quads, then the half-row and row mirrors.
// Every lane ends with the same value (each step combines two equal-order
// partial results, and both operations commute).
template <int CTRL>
__device__ __forceinline__ float dpp_mov(float v) {
  return __builtin_bit_cast(float, __builtin_amdgcn_update_dpp(0, __builtin_bit_cast(int, v), CTRL, 0xF, 0xF, false));
}
__device__ __forceinline__ float group16_max(float v) {
  v = fmaxf(v, dpp_mov<0xB1>(v));   // quad_perm [1,0,3,2]
  v = fmaxf(v, dpp_mov<0x4E>(v));   // quad_perm [2,3,0,1]
  v = fmaxf(v, dpp_mov<0x141>(v));  // row_half_mirror
  return fmaxf(v, dpp_mov<0x140>(v));  // row_mirror
}
__device__ __forceinline__ float group16_sum(float v) {
  v += dpp_mov<0xB1>(v);
  v += dpp_mov<0x4E>(v);
  v += dpp_mov<0x141>(v);
  return v + dpp_mov<0x140>(v);
}

// Dynamic LDS: per wave a P tile [16][36] (the transposed read of P V), then,
// reused once every wave is past P V, the merge buffers [NW][RS][HD + 4] of
// O (rows padded against bank conflicts) and [NW][RS][2] of (max, sum), RS =
// query rows of the tile.
__host__ __device__ inline size_t attn_block_shared(int NW, int RS, int HD) {
  const size_t p = (size_t)NW * 16 * (kSubKeys + 4);
  const size_t m = (size_t)NW * RS * (HD + 6);
  return p > m ? p : m;
}
__host__ __device__ inline size_t attn_block_lds(int NW, int RS, int HD) { return attn_block_shared(NW, RS, HD) * sizeof(float); }

// 16 bytes of a K or V fragment; ONCE: no other block reads them (one query
// tile), so they need not stay in a cache (247 -> 218 us for the 16 long
// sequences below; no difference in the one-round kernel, where each CU reads
// its share at once).
template <bool ONCE>
__device__ __forceinline__ u32x4 load_kv(const uint16_t* p) {
  if constexpr (ONCE) return __builtin_nontemporal_load((const u32x4*)p);
  else return *(const u32x4*)p;
}

constexpr int kMaxPartWaves = 12;  // 3 waves per SIMD: up to 170 VGPRs per lane

template <int HD>
__global__ __launch_bounds__(64 * kMaxPartWaves) void attn_block_kernel(AttnArgs a, int S, int n_sub, int NW) {
  constexpr int KST = HD / 32;  // k-steps of Q K^T
  constexpr int DT = HD / 16;   // 16-wide dimension tiles of P V
  constexpr int NT = kSubKeys / 16;
  extern __shared__ float smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int g = blockIdx.y, b = blockIdx.z;
  const int H = a.n_heads, G = a.n_kv_heads, group = H / G;
  const int rps = a.rps, r0 = b * rps, nq = rps * group;
  const int n_part = a.n_split;
  const int part = blockIdx.x % n_part, mt = blockIdx.x / n_part;
  const int RS = min(16, nq - mt * 16);  // query rows of this tile (> 0 by the grid)
  const int c16 = lane & 15, grp = lane >> 4;
  int sub_here = part == n_part - 1 ? n_sub - part * S : S;
  if (a.seq_bound) {
    // Keys past this sequence's own context are never loaded: within a sequence
    // positions grow with the row index, so its last row (when valid) bounds
    // them.  (Scalar loads; one wait before the K/V loads are issued.)
    const RowDesc last = a.rows[r0 + rps - 1];
    if (last.valid) {
      const int first = part * S * kSubKeys;
      if (first > last.pos) sub_here = 0;  // (block-uniform) no key of this part is visible
      const int need = (last.pos + 1 - first + kSubKeys - 1) / kSubKeys;
      sub_here = need < 0 ? 0 : (need < sub_here ? need : sub_here);
    }
  }
  const uint16_t* kb = k_block<uint16_t>(a.kv, a.layer, b, g);
  const uint16_t* vb = kb + (size_t)a.kv.capacity * HD;

  floatx4 of[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) of[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, sm[4] = {0.f, 0.f, 0.f, 0.f};
  int qpos[4] = {-1, -1, -1, -1};
  float* pbuf = smem + (size_t)wave * 16 * (kSubKeys + 4);

  // Every load of the first sub-chunk is issued before anything waits,
  // smallest first (loads complete in order, so waiting for an early one never
  // waits for a later one): the row descriptors (every wave: the combining
  // block reads them from its lanes too), the K fragments, Q, then the V
  // fragments.  Row descriptors and Q go through range-checked buffer loads.
  // Lane l < 16 holds the descriptor of the row of query l of the tile
  // (queries qa = mt*16 + l; rows r0 + qa / group).  (Only the two fields
  // used: a wider load leaves dead destination registers the allocator
  // reuses, which forces a wait for the load.)
  const int ql = mt * 16 + lane;
  int rd_pos, rd_valid;
  {
    const __amdgpu_buffer_rsrc_t rr = __builtin_amdgcn_make_buffer_rsrc(const_cast<RowDesc*>(a.rows), (short)0,
                                                                         a.M * (int)sizeof(RowDesc), 0x00020000);
    const uint32_t roff = ((uint32_t)(r0 + min(ql, nq - 1) / group) * (uint32_t)sizeof(RowDesc)) |
                          ((uint32_t)(lane >= 16 || ql >= nq) << 31);
    rd_pos = (int)__builtin_amdgcn_raw_buffer_load_b32(rr, roff + offsetof(RowDesc, pos), 0, 0);
    rd_valid = (int)__builtin_amdgcn_raw_buffer_load_b32(rr, roff + offsetof(RowDesc, valid), 0, 0);
  }
  if (wave < sub_here) {  // (wave-uniform) a wave past the part's sub-chunks only joins the merge
    // K fragments of a sub-chunk: 2 x KST contiguous 1 KB fragments (k0 + 32 <= capacity);
    // V fragments: DT contiguous 1 KB fragments (32 positions x 16 dims each).
    u32x4 kf[NT][KST], vf[DT];
    auto load_k = [&](int k0) {
      const uint16_t* kfrag = kb + (size_t)(k0 / 16) * KST * 512 + lane * 8;
#pragma unroll
      for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int c = 0; c < KST; ++c) kf[t][c] = *(const u32x4*)(kfrag + (size_t)(t * KST + c) * 512);
    };
    auto load_v = [&](int k0) {
      const uint16_t* vfrag = vb + (size_t)(k0 / 32) * DT * 512 + lane * 8;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) vf[dt] = *(const u32x4*)(vfrag + (size_t)dt * 512);
    };
    const int k0 = (part * S + wave) * kSubKeys;
    load_k(k0);
    // Q fragments (A operand): query qa = mt*16 + l%16 (zeros past nq).
    f32x4 qv4[KST][2];
    {
      const int qa = mt * 16 + c16;
      const int row = r0 + qa / group, head = g * group + qa % group;
      const __amdgpu_buffer_rsrc_t qrs =
          __builtin_amdgcn_make_buffer_rsrc(a.qr, (short)0, a.M * H * HD * 4, 0x00020000);
      const uint32_t qoff = ((((uint32_t)row * H + head) * HD + 8 * grp) * 4u) | ((uint32_t)(qa >= nq) << 31);
#pragma unroll
      for (int c = 0; c < KST; ++c) {
        qv4[c][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff + 128u * c, 0, 0));
        qv4[c][1] =
            __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff + 128u * c + 16u, 0, 0));
      }
    }
    load_v(k0);
    // (compiler barrier: keeps what follows from being hoisted above the loads)
    asm volatile("" ::: "memory");

    // nk = max(pos) + 1 over the tile's valid query rows: no key past it is read.
    // (Lane reads rather than shuffles: the compiler then waits for the row
    // descriptors alone, with the K, Q and V loads above still in flight; with
    // shuffles it held the Q and V loads back until the descriptors arrived.)
    const int mypos = (lane < 16 && ql < nq && rd_valid) ? rd_pos : -1;
    int lp[16];
#pragma unroll
    for (int i = 0; i < 16; ++i) lp[i] = __builtin_amdgcn_readlane(mypos, i);
    int nk = lp[0] + 1;
#pragma unroll
    for (int i = 1; i < 16; ++i) nk = max(nk, lp[i] + 1);
    // positions of the 4 query rows this lane holds in the C layout (-1: none)
#pragma unroll
    for (int r = 0; r < 4; ++r)
      qpos[r] = grp == 0 ? lp[r] : (grp == 1 ? lp[4 + r] : (grp == 2 ? lp[8 + r] : lp[12 + r]));
    const float scale = 1.0f / sqrtf((float)HD);
    bf16x8 qhi[KST], qlo[KST];
#pragma unroll
    for (int c = 0; c < KST; ++c) {
      float v[8];
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        v[j] = qv4[c][0][j] * scale;
        v[4 + j] = qv4[c][1][j] * scale;
      }
      split_hilo(v, qhi[c], qlo[c]);
    }

    if (k0 < nk) {  // (wave-uniform)
      // keys past the context: zero their V entries (never multiply stale memory)
      const int nvalid = nk - (k0 + 8 * grp);
      if (nvalid < 8) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
#pragma unroll
          for (int q = 0; q < 4; ++q) {
            if (2 * q >= nvalid) vf[dt][q] = 0u;
            else if (2 * q + 1 >= nvalid) vf[dt][q] &= 0xffffu;
          }
      }
      floatx4 sf[NT];
#pragma unroll
      for (int t = 0; t < NT; ++t) {
        floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
        for (int c = 0; c < KST; ++c) {
          const bf16x8 kk = __builtin_bit_cast(bf16x8, kf[t][c]);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qhi[c], kk, acc, 0, 0, 0);
          acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qlo[c], kk, acc, 0, 0, 0);
        }
        const int key = k0 + 16 * t + c16;
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (key > qpos[r]) acc[r] = -INFINITY;
        sf[t] = acc;
      }
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        float m = -INFINITY;
#pragma unroll
        for (int t = 0; t < NT; ++t) m = fmaxf(m, sf[t][r]);
        mx[r] = group16_max(m);
        float sum = 0.f;
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          const float p = mx[r] == -INFINITY || sf[t][r] == -INFINITY ? 0.f : expf(sf[t][r] - mx[r]);
          pbuf[(4 * grp + r) * (kSubKeys + 4) + 16 * t + c16] = p;
          sum += p;
        }
        sm[r] = group16_sum(sum);
      }
      __builtin_amdgcn_wave_barrier();  // P written by all lanes of the wave before the transposed reads
      float pv[8];
#pragma unroll
      for (int q = 0; q < 8; ++q) pv[q] = pbuf[c16 * (kSubKeys + 4) + 8 * grp + q];
      bf16x8 phi, plo;
      split_hilo(pv, phi, plo);
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) {
        const bf16x8 vv = __builtin_bit_cast(bf16x8, vf[dt]);
        of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi, vv, of[dt], 0, 0, 0);
        of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo, vv, of[dt], 0, 0, 0);
      }
    }
  }

  constexpr int DPL = HD >= 64 ? HD / 64 : 1;
  if (NW == 1) {  // (block-uniform) the wave's own (max, sum, O) rows are the part's partials
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * grp + r;
      if (row >= RS || qpos[r] < 0 || mx[r] == -INFINITY) continue;
      const int qc = mt * 16 + row;
      const size_t slot = ((size_t)(r0 + qc / group) * H + g * group + qc % group) * n_part + part;
      if (a.counters) {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt)
          __hip_atomic_store(&a.o_part[slot * HD + dt * 16 + c16], of[dt][r], __ATOMIC_RELAXED,
                             __HIP_MEMORY_SCOPE_AGENT);
        if (c16 == 0) {
          __hip_atomic_store(&a.ml_part[2 * slot], mx[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(&a.ml_part[2 * slot + 1], sm[r], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
      } else {
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) a.o_part[slot * HD + dt * 16 + c16] = of[dt][r];
        if (c16 == 0) {
          a.ml_part[2 * slot] = mx[r];
          a.ml_part[2 * slot + 1] = sm[r];
        }
      }
    }
  } else {
  // Merge the waves' partials of this part (LDS reused: every wave is past P V).
  __syncthreads();
  constexpr int OS = HD + 4;                   // row stride of the O partials
  float* so = smem;                            // [NW][RS][OS]
  float* sml = smem + (size_t)NW * RS * OS;    // [NW][RS][2]
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int row = 4 * grp + r;
    if (row >= RS) continue;
    const bool live = qpos[r] >= 0 && mx[r] != -INFINITY;
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) so[((size_t)wave * RS + row) * OS + dt * 16 + c16] = live ? of[dt][r] : 0.f;
    if (c16 == 0) {
      sml[((size_t)wave * RS + row) * 2] = live ? mx[r] : -INFINITY;
      sml[((size_t)wave * RS + row) * 2 + 1] = live ? sm[r] : 0.f;
    }
  }
  __syncthreads();
  // One wave per row: the waves' weights exp(m_w - M) are uniform across the
  // wave, each lane sums HD / 64 dims over the waves in fixed order.
  constexpr int MAXW = kMaxPartWaves;
  for (int row = wave; row < RS; row += NW) {  // (wave-uniform)
    // The waves' partials in groups of 4: every read of a group first, then
    // the arithmetic (a wave past NW or without keys gets weight 0, and adding
    // 0 * a finite partial changes no sum).
    constexpr int WG = 4;
    float M = -INFINITY;
#pragma unroll
    for (int w0 = 0; w0 < MAXW; w0 += WG) {
      if (w0 >= NW) break;
#pragma unroll
      for (int w = w0; w < w0 + WG; ++w)
        if (w < NW) M = fmaxf(M, sml[((size_t)w * RS + row) * 2]);
    }
    if (M == -INFINITY) continue;  // no key of this part is visible to the row
    float L = 0.f, O[DPL];
#pragma unroll
    for (int j = 0; j < DPL; ++j) O[j] = 0.f;
#pragma unroll
    for (int w0 = 0; w0 < MAXW; w0 += WG) {
      if (w0 >= NW) break;
      float mw[WG], lw[WG], ow[WG][DPL];
#pragma unroll
      for (int i = 0; i < WG; ++i) {
        const size_t wr = (size_t)min(w0 + i, NW - 1) * RS + row;
        mw[i] = sml[wr * 2];
        lw[i] = sml[wr * 2 + 1];
#pragma unroll
        for (int j = 0; j < DPL; ++j) ow[i][j] = lane + 64 * j < HD ? so[wr * OS + lane + 64 * j] : 0.f;
      }
#pragma unroll
      for (int i = 0; i < WG; ++i) {
        const float e = w0 + i < NW && mw[i] != -INFINITY ? expf(mw[i] - M) : 0.f;
        L += e * lw[i];
#pragma unroll
        for (int j = 0; j < DPL; ++j) O[j] += e * ow[i][j];
      }
    }
    const int qc = mt * 16 + row;
    const int qrow = r0 + qc / group, head = g * group + qc % group;
    const size_t slot = ((size_t)qrow * H + head) * n_part + part;
    if (a.counters) {  // (agent-scope stores: visible to the combining block on any XCD once completed)
#pragma unroll
      for (int j = 0; j < DPL; ++j)
        if (lane + 64 * j < HD)
          __hip_atomic_store(&a.o_part[slot * HD + lane + 64 * j], O[j], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      if (lane == 0) {
        __hip_atomic_store(&a.ml_part[2 * slot], M, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        __hip_atomic_store(&a.ml_part[2 * slot + 1], L, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
    } else {  // (read by the combine kernel after this launch)
#pragma unroll
      for (int j = 0; j < DPL; ++j)
        if (lane + 64 * j < HD) a.o_part[slot * HD + lane + 64 * j] = O[j];
      if (lane == 0) {
        a.ml_part[2 * slot] = M;
        a.ml_part[2 * slot + 1] = L;
      }
    }
  }
  }
  // The memory system is idle while the combining blocks finish: blocks that
  // do not combine read their share of the next launch's weights into the
  // last-level cache before they end.
  auto read_ahead = [&]() {
    // (Block i of n: the first kNextWeightsPerBlock bytes of slice i of n.)
    // The loaded words are only kept live to the end (no store), so the loads
    // are issued and waited for and nothing else.
    if (a.next_w) {
      const uint32_t nblk = gridDim.x * gridDim.y * gridDim.z;
      const uint32_t lb = blockIdx.x + gridDim.x * (blockIdx.y + gridDim.y * blockIdx.z);
      const uint32_t slice = (a.next_w_bytes / nblk + 1023u) & ~1023u;
      const __amdgpu_buffer_rsrc_t nr = __builtin_amdgcn_make_buffer_rsrc(const_cast<unsigned char*>(a.next_w),
                                                                          (short)0, a.next_w_bytes, 0x00020000);
      // Wave w reads KB-chunks w, w + NW, ... (at most kNextLoads of them), all
      // issued before the one wait; a dword per lane at a 16-byte stride touches
      // every line of the chunk.  (Offsets past the share or next_w_bytes read
      // nothing: the out-of-range bit and the descriptor's range.)
      constexpr int kNextLoads = 6;
      const uint32_t lim = min(kNextWeightsPerBlock, slice);
      uint32_t v[kNextLoads];
#pragma unroll
      for (int i = 0; i < kNextLoads; ++i) {
        const uint32_t c = ((uint32_t)wave + (uint32_t)i * NW) * 1024u;
        v[i] = __builtin_amdgcn_raw_buffer_load_b32(nr, (lb * slice + c + lane * 16u) | ((uint32_t)(c >= lim) << 31),
                                                    0, 0);
      }
      uint32_t keep = 0;
#pragma unroll
      for (int i = 0; i < kNextLoads; ++i) keep ^= v[i];
      asm volatile("" ::"v"(keep));
    }
  };
  {
    if (!a.counters) return;

    // The last block of this (sequence, tile, kv head) to finish combines the
    // parts: every wave's partial stores have completed before the block's
    // single counter increment, and the combining block reads the partials
    // with agent-scope loads.  The counter goes back to zero for the next launch.
    __shared__ int s_last;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    __syncthreads();
    if (threadIdx.x == 0) {
      uint32_t* ctr = a.counters + ((size_t)b * (gridDim.x / n_part) + mt) * G + g;
      const uint32_t old = __hip_atomic_fetch_add(ctr, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const int last = old == (uint32_t)(n_part - 1);
      if (last) __hip_atomic_store(ctr, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      s_last = last;
    }
    __syncthreads();
    if (!s_last) {
      read_ahead();
      return;
    }
    for (int row = wave; row < RS; row += NW) {  // (wave-uniform) one wave per query row of the tile
      const int qc = mt * 16 + row;
      const int qrow = r0 + qc / group, head = g * group + qc % group;
      RowDesc rd;
      rd.pos = __shfl(rd_pos, row, kWave);  // (lane `row` loaded this query's row descriptor)
      rd.valid = __shfl(rd_valid, row, kWave);
      float* o = a.o + ((size_t)qrow * H + head) * HD;
      if (!rd.valid) {
#pragma unroll
        for (int j = 0; j < DPL; ++j)
          if (lane + 64 * j < HD) put_o(a, o, qrow, head, lane + 64 * j, 0.f);
        continue;
      }
      // parts holding keys <= pos (the last part also holds the remainder)
      const int nch = min(rd.pos / a.chunk + 1, n_part);
      if (rd.pos + 1 > a.max_ctx && lane == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
      const size_t base = ((size_t)qrow * H + head) * n_part;
      // lane p < nch: part p's (max, sum); the first parts' outputs in the same round trip
      constexpr int PB = 8;
      const int pl = min(lane, nch - 1);
      const float mp = __hip_atomic_load(&a.ml_part[2 * (base + pl)], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      const float lp = __hip_atomic_load(&a.ml_part[2 * (base + pl) + 1], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      float acc[DPL];
#pragma unroll
      for (int j = 0; j < DPL; ++j) acc[j] = 0.f;
      float mx = 0.f, wgt = 0.f;
      for (int p0 = 0; p0 < nch; p0 += PB) {  // (wave-uniform)
        float ov[PB][DPL];
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
          const int p = min(p0 + pp, nch - 1);  // (parts past nch get weight 0 below)
#pragma unroll
          for (int j = 0; j < DPL; ++j)
            ov[pp][j] = lane + 64 * j < HD ? __hip_atomic_load(&a.o_part[(base + p) * HD + lane + 64 * j],
                                                               __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)
                                           : 0.f;
        }
        if (p0 == 0) {
          mx = wave_max(lane < nch ? mp : -INFINITY);
          wgt = lane < nch ? expf(mp - mx) : 0.f;
        }
#pragma unroll
        for (int pp = 0; pp < PB; ++pp) {
          const float w = __shfl(wgt, (p0 + pp) & 63, kWave);
          const float wv = p0 + pp < nch ? w : 0.f;
#pragma unroll
          for (int j = 0; j < DPL; ++j) acc[j] += wv * ov[pp][j];
        }
      }
      const float L = wave_sum(wgt * lp);
      const float inv = 1.0f / L;
#pragma unroll
      for (int j = 0; j < DPL; ++j)
        if (lane + 64 * j < HD) put_o(a, o, qrow, head, lane + 64 * j, acc[j] * inv);
    }
  }
}

// ---------------------------------------------------------------- long contexts and batches (bf16 cache)
// More sub-chunks than one round of waves takes: a persistent grid (two blocks
// of 4 waves per CU) over the work itself.  The sub-chunks of every unit
// (sequence, kv head, 16-query tile), each sequence's counted from its own last
// row on the device, form one line, sequence by sequence, and block i takes the
// i-th `per` of them: all blocks stream the same bytes whatever the lengths, and
// a block pays for its start and its merge once or twice instead of per part.
// Within a unit's segment wave w takes sub-chunks w, w + 4, ... with an online
// softmax, then the waves merge in LDS.  A unit inside one block is finished
// there; of a unit that spans blocks every block stores its part, and
// attn_stream_combine_kernel adds the parts.  (Combined by the block that ends
// the unit, which waits for the other parts, instead: at 16 query rows over 30
// and more parts that one block reads 300 KB and more, 25 to 35 us per layer;
// the launch takes 4 to 5.  1.1B shape, 5 rows of one sequence of 8192 keys, two
// layers: 181 us, 137 now; 7B, 4096 keys: 271, 258; no difference where units
// are many and few span blocks, 8 or 16 sequences of the 7B shape.)
// Bound: the key and value stream.  16 sequences of 1024 to 8192 keys (1.26 GB
// per layer of the 7B shape): 250 us in parts sized for 12 blocks per CU (5.0
// TB/s), 216 now with the combine (5.8 TB/s); 8 sequences of 513 to 2048: 54 us,
// 40 now.
constexpr int kLoopWaves = 4;
// Sub-chunks of sequence s: up to its last row's position (the host's count
// where that row is invalid).
__device__ __forceinline__ int stream_subs(const AttnArgs& a, int s, int n_sub) {
  const RowDesc last = a.rows[s * a.rps + a.rps - 1];
  return last.valid ? min(n_sub, last.pos / kSubKeys + 1) : n_sub;
}
// Sub-chunks per block of `nblk` over `tot` in all: a unit spans at most
// kMaxParts blocks, every wave gets a sub-chunk.
__device__ __forceinline__ int stream_per_block(int tot, int nblk, int n_sub) {
  return max(max((tot + nblk - 1) / nblk, (n_sub + kMaxParts - 3) / (kMaxParts - 2)), kLoopWaves);
}
__host__ __device__ inline size_t attn_stream_lds(int RS, int HD) {
  const size_t p = (size_t)kLoopWaves * 16 * (kSubKeys + 4), m = (size_t)kLoopWaves * RS * (HD + 6);
  return (p > m ? p : m) * sizeof(float);
}
template <int HD, bool ONCE>
__global__ __launch_bounds__(64 * kLoopWaves, 2) void attn_stream_kernel(AttnArgs a, int n_sub, int n_mt) {
  constexpr int KST = HD / 32, DT = HD / 16, NT = kSubKeys / 16, NW = kLoopWaves;
  constexpr int DPL = HD >= 64 ? HD / 64 : 1;
  constexpr int OS = HD + 4;
  extern __shared__ float smem[];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int H = a.n_heads, G = a.n_kv_heads, group = H / G;
  const int rps = a.rps, nq = rps * group, B = a.M / rps, U = G * n_mt;
  const int RSM = min(16, nq);
  const int c16 = lane & 15, grp = lane >> 4;
  float* const pbuf = smem + (size_t)wave * 16 * (kSubKeys + 4);
  float* const so = smem;                                   // [NW][RS][OS] (P's place, once every wave is past P V)
  float* const sml = smem + (size_t)NW * RSM * OS;          // [NW][RS][2]

  auto subs_of = [&](int s) { return stream_subs(a, s, n_sub); };
  const int n0 = lane < B ? subs_of(lane) : 0;  // (the first 64 sequences stay in a register)
  int subs = 0;
  for (int c = 0; c < B; c += kWave) {
    int n = c == 0 ? n0 : (c + lane < B ? subs_of(c + lane) : 0);
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) n += __shfl_xor(n, o, kWave);
    subs += n;
  }
  subs = __builtin_amdgcn_readfirstlane(subs);
  const int tot = subs * U, nblk = (int)gridDim.x, blk = (int)blockIdx.x;
  const int per = stream_per_block(tot, nblk, n_sub);
  int x = blk * per;
  const int hi = min(tot, x + per);
  if (x >= tot) return;
  // the sequence that holds x, and the sub-chunks before it
  int b = 0, before = 0;
  for (int c = 0; c < B; c += kWave) {
    const int n = c == 0 ? n0 : (c + lane < B ? subs_of(c + lane) : 0);
    int incl = n;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const int t = __shfl_up(incl, o, kWave);
      if (lane >= o) incl += t;
    }
    const unsigned long long hit = __ballot((before + incl) * U > x);
    if (hit) {
      const int l = __ffsll(hit) - 1;
      b = c + l;
      before += __shfl(incl - n, l, kWave);
      break;
    }
    before += __shfl(incl, kWave - 1, kWave);
  }
  b = __builtin_amdgcn_readfirstlane(b);
  before = __builtin_amdgcn_readfirstlane(before);

  const float scale = 1.0f / sqrtf((float)HD);

  while (x < hi) {  // (block-uniform)
    const int n_b = __builtin_amdgcn_readfirstlane(b < kWave ? __shfl(n0, b & 63, kWave) : subs_of(b));
    const int off = x - before * U, u = off / n_b, j0 = off % n_b, j1 = min(n_b, j0 + hi - x);
    const int g = u / n_mt, mt = u % n_mt, r0 = b * rps;
    const int RS = min(16, nq - mt * 16);
    const int x0 = x - j0;
    const uint16_t* kb = k_block<uint16_t>(a.kv, a.layer, b, g);
    const uint16_t* vb = kb + (size_t)a.kv.capacity * HD;

    floatx4 of[DT];
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) of[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
    float mx[4] = {-INFINITY, -INFINITY, -INFINITY, -INFINITY}, sm[4] = {0.f, 0.f, 0.f, 0.f};
    int qpos[4] = {-1, -1, -1, -1};
    // (loads in the order they are needed: descriptors, K, Q, V; see attn_block_kernel)
    const int ql = mt * 16 + lane;
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(a.rows, (uint32_t)a.M * (uint32_t)sizeof(RowDesc));
    const uint32_t roff = ((uint32_t)(r0 + min(ql, nq - 1) / group) * (uint32_t)sizeof(RowDesc)) |
                          ((uint32_t)(lane >= 16 || ql >= nq) << 31);
    const int rd_pos = (int)__builtin_amdgcn_raw_buffer_load_b32(rr, roff + offsetof(RowDesc, pos), 0, 0);
    const int rd_valid = (int)__builtin_amdgcn_raw_buffer_load_b32(rr, roff + offsetof(RowDesc, valid), 0, 0);
    if (j0 + wave < j1) {  // (wave-uniform)
      u32x4 kf[NT][KST], vf[DT];
      auto load_k = [&](int k0) {
        const uint16_t* kfrag = kb + (size_t)(k0 / 16) * KST * 512 + lane * 8;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
          for (int c = 0; c < KST; ++c) kf[t][c] = load_kv<ONCE>(kfrag + (size_t)(t * KST + c) * 512);
      };
      auto load_v = [&](int k0) {
        const uint16_t* vfrag = vb + (size_t)(k0 / 32) * DT * 512 + lane * 8;
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) vf[dt] = load_kv<ONCE>(vfrag + (size_t)dt * 512);
      };
      int k0 = (j0 + wave) * kSubKeys;
      load_k(k0);
      f32x4 qv4[KST][2];
      {
        const int qa = mt * 16 + c16;
        const int row = r0 + qa / group, head = g * group + qa % group;
        const __amdgpu_buffer_rsrc_t qrs = make_rsrc(a.qr, (uint32_t)a.M * H * HD * 4u);
        const uint32_t qoff = ((((uint32_t)row * H + head) * HD + 8 * grp) * 4u) | ((uint32_t)(qa >= nq) << 31);
#pragma unroll
        for (int c = 0; c < KST; ++c) {
          qv4[c][0] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff + 128u * c, 0, 0));
          qv4[c][1] =
              __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(qrs, qoff + 128u * c + 16u, 0, 0));
        }
      }
      load_v(k0);
      asm volatile("" ::: "memory");  // (keeps what follows from being hoisted above the loads)
      const int mypos = (lane < 16 && ql < nq && rd_valid) ? rd_pos : -1;
      int lp[16];
#pragma unroll
      for (int i = 0; i < 16; ++i) lp[i] = __builtin_amdgcn_readlane(mypos, i);
      int nk = lp[0] + 1;
#pragma unroll
      for (int i = 1; i < 16; ++i) nk = max(nk, lp[i] + 1);
#pragma unroll
      for (int r = 0; r < 4; ++r)
        qpos[r] = grp == 0 ? lp[r] : (grp == 1 ? lp[4 + r] : (grp == 2 ? lp[8 + r] : lp[12 + r]));
      bf16x8 qhi[KST], qlo[KST];
#pragma unroll
      for (int c = 0; c < KST; ++c) {
        float v[8];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          v[j] = qv4[c][0][j] * scale;
          v[4 + j] = qv4[c][1][j] * scale;
        }
        split_hilo(v, qhi[c], qlo[c]);
      }
      for (int j = j0 + wave; j < j1 && k0 < nk; j += NW) {  // (wave-uniform)
        if (j != j0 + wave) {  // the first sub-chunk's fragments were loaded above
          load_k(k0);
          load_v(k0);
        }
        // keys past the context: zero their V entries (never multiply stale memory)
        const int nvalid = nk - (k0 + 8 * grp);
        if (nvalid < 8) {
#pragma unroll
          for (int dt = 0; dt < DT; ++dt)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
              if (2 * q >= nvalid) vf[dt][q] = 0u;
              else if (2 * q + 1 >= nvalid) vf[dt][q] &= 0xffffu;
            }
        }
        floatx4 sf[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) {
          floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
          for (int c = 0; c < KST; ++c) {
            const bf16x8 kk = __builtin_bit_cast(bf16x8, kf[t][c]);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qhi[c], kk, acc, 0, 0, 0);
            acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(qlo[c], kk, acc, 0, 0, 0);
          }
          const int key = k0 + 16 * t + c16;
#pragma unroll
          for (int r = 0; r < 4; ++r)
            if (key > qpos[r]) acc[r] = -INFINITY;
          sf[t] = acc;
        }
        // Online softmax: the running (max, sum, O) of each row is rescaled by
        // exp(old max - new max) when this sub-chunk raises the max.
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          float m = -INFINITY;
#pragma unroll
          for (int t = 0; t < NT; ++t) m = fmaxf(m, sf[t][r]);
          const float mnew = fmaxf(mx[r], group16_max(m));
          const float alpha = mx[r] == -INFINITY ? 0.f : expf(mx[r] - mnew);
          float sum = 0.f;
#pragma unroll
          for (int t = 0; t < NT; ++t) {
            const float p = mnew == -INFINITY || sf[t][r] == -INFINITY ? 0.f : expf(sf[t][r] - mnew);
            pbuf[(4 * grp + r) * (kSubKeys + 4) + 16 * t + c16] = p;
            sum += p;
          }
          sm[r] = sm[r] * alpha + group16_sum(sum);
          mx[r] = mnew;
#pragma unroll
          for (int dt = 0; dt < DT; ++dt) of[dt][r] *= alpha;
        }
        __builtin_amdgcn_wave_barrier();  // P written by all lanes of the wave before the transposed reads
        float pv[8];
#pragma unroll
        for (int q = 0; q < 8; ++q) pv[q] = pbuf[c16 * (kSubKeys + 4) + 8 * grp + q];
        bf16x8 phi, plo;
        split_hilo(pv, phi, plo);
#pragma unroll
        for (int dt = 0; dt < DT; ++dt) {
          const bf16x8 vv = __builtin_bit_cast(bf16x8, vf[dt]);
          of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(phi, vv, of[dt], 0, 0, 0);
          of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(plo, vv, of[dt], 0, 0, 0);
        }
        __builtin_amdgcn_wave_barrier();  // the transposed reads of P done before the next sub-chunk writes it
        k0 += NW * kSubKeys;
      }
    }
    // Merge the waves' partials of the segment (P's LDS reused: every wave is past P V).
    __syncthreads();
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int row = 4 * grp + r;
      if (row >= RS) continue;
      const bool live = qpos[r] >= 0 && mx[r] != -INFINITY;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) so[((size_t)wave * RS + row) * OS + dt * 16 + c16] = live ? of[dt][r] : 0.f;
      if (c16 == 0) {
        sml[((size_t)wave * RS + row) * 2] = live ? mx[r] : -INFINITY;
        sml[((size_t)wave * RS + row) * 2 + 1] = live ? sm[r] : 0.f;
      }
    }
    __syncthreads();
    const bool whole = j0 == 0 && j1 == n_b;
    const int part = blk - x0 / per;
    for (int row = wave; row < RS; row += NW) {  // (wave-uniform) one wave per query row
      const int qc = mt * 16 + row;
      const int qrow = r0 + qc / group, head = g * group + qc % group;
      const int pos = __shfl(rd_pos, row, kWave), valid = __shfl(rd_valid, row, kWave);
      float mw[NW], lw[NW], ow[NW][DPL], M = -INFINITY;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const size_t wr = (size_t)w * RS + row;
        mw[w] = sml[wr * 2];
        lw[w] = sml[wr * 2 + 1];
#pragma unroll
        for (int j = 0; j < DPL; ++j) ow[w][j] = lane + 64 * j < HD ? so[wr * OS + lane + 64 * j] : 0.f;
      }
#pragma unroll
      for (int w = 0; w < NW; ++w) M = fmaxf(M, mw[w]);
      float L = 0.f, O[DPL];
#pragma unroll
      for (int j = 0; j < DPL; ++j) O[j] = 0.f;
#pragma unroll
      for (int w = 0; w < NW; ++w) {
        const float e = mw[w] != -INFINITY ? expf(mw[w] - M) : 0.f;
        L += e * lw[w];
#pragma unroll
        for (int j = 0; j < DPL; ++j) O[j] += e * ow[w][j];
      }
      if (whole) {
        const float inv = valid ? 1.0f / L : 0.f;
        if (valid && pos + 1 > a.max_ctx && lane == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
        float* o = a.o + ((size_t)qrow * H + head) * HD;
#pragma unroll
        for (int j = 0; j < DPL; ++j)
          if (lane + 64 * j < HD) put_o(a, o, qrow, head, lane + 64 * j, valid ? O[j] * inv : 0.f);
      } else {  // (every row, also one that sees no key here or whose scores are all NaN: the combine weighs them by M)
        const size_t slot = ((size_t)qrow * H + head) * a.n_split + part;
#pragma unroll
        for (int j = 0; j < DPL; ++j)
          if (lane + 64 * j < HD) a.o_part[slot * HD + lane + 64 * j] = O[j];
        if (lane == 0) {
          a.ml_part[2 * slot] = M;
          a.ml_part[2 * slot + 1] = L;
        }
      }
    }
    x += j1 - j0;
    if (x == (before + n_b) * U) {
      before += n_b;
      ++b;
    }
    __syncthreads();  // (the merge buffers are P's again)
  }
}

// Adds the parts of attn_stream_kernel: one wave per (head, row), lane p = part
// p.  It finds the unit's place in the line of sub-chunks as the blocks did; a
// unit that one block held whole is finished already.
template <int HD>
__global__ __launch_bounds__(64) void attn_stream_combine_kernel(AttnArgs a, int n_sub, int n_mt, int nblk) {
  constexpr int DPL = HD >= 64 ? HD / 64 : 1, PB = 16;
  const int head = blockIdx.x, r = blockIdx.y, lane = threadIdx.x, H = a.n_heads;
  const int group = H / a.n_kv_heads, U = a.n_kv_heads * n_mt, B = a.M / a.rps, b = r / a.rps;
  const RowDesc rd = a.rows[r];
  const int n_b = stream_subs(a, b, n_sub);
  int subs = 0, before = 0;
  for (int s = lane; s < B; s += kWave) {
    const int n = stream_subs(a, s, n_sub);
    subs += n;
    before += s < b ? n : 0;
  }
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    subs += __shfl_xor(subs, o, kWave);
    before += __shfl_xor(before, o, kWave);
  }
  const int per = stream_per_block(subs * U, nblk, n_sub);
  const int u = head / group * n_mt + ((r - b * a.rps) * group + head % group) / 16;
  const int x0 = before * U + u * n_b, p_first = x0 / per, parts = (x0 + n_b - 1) / per - p_first + 1;
  if (parts == 1) return;
  float* o = a.o + ((size_t)r * H + head) * HD;
  if (!rd.valid) {
#pragma unroll
    for (int j = 0; j < DPL; ++j)
      if (lane + 64 * j < HD) put_o(a, o, r, head, lane + 64 * j, 0.f);
    return;
  }
  if (rd.pos + 1 > a.max_ctx && lane == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
  // parts whose first sub-chunk holds a key <= pos
  const int nch = min((x0 + rd.pos / kSubKeys) / per - p_first + 1, parts);
  const size_t base = ((size_t)r * H + head) * a.n_split;
  const int pl = min(lane, nch - 1);
  const float mp = a.ml_part[2 * (base + pl)], lp = a.ml_part[2 * (base + pl) + 1];
  float acc[DPL], wgt = 0.f;
#pragma unroll
  for (int j = 0; j < DPL; ++j) acc[j] = 0.f;
  for (int p0 = 0; p0 < nch; p0 += PB) {
    float ov[PB][DPL];
#pragma unroll
    for (int pp = 0; pp < PB; ++pp)
#pragma unroll
      for (int j = 0; j < DPL; ++j)
        ov[pp][j] = a.o_part[(base + min(p0 + pp, nch - 1)) * HD + min(lane + 64 * j, HD - 1)];
    if (p0 == 0) {
      const float M = wave_max(lane < nch ? mp : -INFINITY);
      wgt = lane < nch ? expf(mp - M) : 0.f;
    }
#pragma unroll
    for (int pp = 0; pp < PB; ++pp) {
      const float w = __shfl(wgt, (p0 + pp) & 63, kWave);
      const float wv = p0 + pp < nch ? w : 0.f;
#pragma unroll
      for (int j = 0; j < DPL; ++j) acc[j] += wv * ov[pp][j];
    }
  }
  const float inv = 1.0f / wave_sum(wgt * lp);
#pragma unroll
  for (int j = 0; j < DPL; ++j)
    if (lane + 64 * j < HD) put_o(a, o, r, head, lane + 64 * j, acc[j] * inv);
}

// ---------------------------------------------------------------- many query rows (bf16 cache)
// Prefill chunks: enough query rows that K and V are worth sharing.  Block = 64
// queries (4 tiles of 16) of one (kv head, sequence), 8 waves: wave w works on
// tile w % 4 and on every second sub-chunk of 32 keys (w / 4).  Stages of two
// sub-chunks are copied from the cache to LDS as they lie there (1 KB fragments
// in MFMA order, ST stages in flight) and shared by the tiles; every block runs
// through all of its keys, so nothing is written but the output: no partial
// sums, no combine.
// The scores are taken as K Q^T: D[4 (l/16) + r][l % 16] is a key row and a
// query column, so a lane holds 8 scores of one query.  The K rows are read in
// the order that leaves lane group g with keys 8g .. 8g+7 (row i of tile t: key
// 8 (i/4) + 4t + i%4), which is the k order of V's fragments: P feeds O^T = V^T
// P^T from the registers it was made in.  The running maximum is then one value
// per lane (two lane swaps per sub-chunk), the sums stay per lane to the end.
// Bound: the softmax's vector work and the products, 4 waves to a SIMD pair.
template <int HD>
__global__ __launch_bounds__(512) void attn_rows_kernel(AttnArgs a, int n_sub) {
  constexpr int KST = HD / 32, DT = HD / 16, ST = 4;
  constexpr int KP = 4 * KST, NP = KP + 2 * DT;  // 1 KB pieces of a stage: K of two sub-chunks, then V
  constexpr int PW = (NP + 7) / 8;               // per wave
  __shared__ u32x4 s_kv[ST][NP][kWave];
  __shared__ int s_nk[4];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int qt = wave & 3, kg = wave >> 2;
  const int g = blockIdx.y, b = blockIdx.z;
  const int H = a.n_heads, G = a.n_kv_heads, group = H / G;
  const int rps = a.rps, r0 = b * rps, nq = rps * group;
  const int c16 = lane & 15, grp = lane >> 4;
  const uint16_t* kb = k_block<uint16_t>(a.kv, a.layer, b, g);

  // This lane's query: qa of the sequence's rps * group.
  const int qa = ((int)blockIdx.x * 4 + qt) * 16 + c16;
  const int row = r0 + min(qa, nq - 1) / group, head = g * group + min(qa, nq - 1) % group;
  const RowDesc rd = a.rows[row];
  const bool live = qa < nq && rd.valid;
  const int qpos = live ? rd.pos : -1;
  int nk = qpos + 1, lo = live ? qpos : 0x7fffffff;  // keys of the tile; its lowest position
#pragma unroll
  for (int o = 1; o < 16; o <<= 1) {
    nk = max(nk, __shfl_xor(nk, o, kWave));
    lo = min(lo, __shfl_xor(lo, o, kWave));
  }
  nk = __builtin_amdgcn_readfirstlane(nk);
  lo = __builtin_amdgcn_readfirstlane(lo);
  if (kg == 0 && lane == 0) s_nk[qt] = nk;
  if (live && qpos + 1 > a.max_ctx && grp == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong

  // Q as the B operand: lane = query l % 16, dims 32c + 8 (l/16) .. +7
  bf16x8 qhi[KST], qlo[KST];
  const float scale = 1.0f / sqrtf((float)HD);
#pragma unroll
  for (int c = 0; c < KST; ++c) {
    const float* q = a.qr + ((size_t)row * H + head) * HD + 32 * c + 8 * grp;
    float v[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) v[j] = qa < nq ? q[j] * scale : 0.f;
    split_hilo(v, qhi[c], qlo[c]);
  }
  __syncthreads();
  const int bnk = max(max(s_nk[0], s_nk[1]), max(s_nk[2], s_nk[3]));
  const int n_here = min(n_sub, (bnk + kSubKeys - 1) / kSubKeys), n_st = (n_here + 1) / 2;

  const __amdgpu_buffer_rsrc_t kr = make_rsrc(kb, (uint32_t)a.kv.capacity * HD * 2u);
  const __amdgpu_buffer_rsrc_t vr = make_rsrc(kb + (size_t)a.kv.capacity * HD, (uint32_t)a.kv.capacity * HD * 2u);
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) void*)&s_kv[0][0][0];
  auto issue = [&](int st) {
#pragma unroll
    for (int i = 0; i < PW; ++i) {
      const int p = wave * PW + i;
      if (NP % 8 != 0 && p >= NP) break;
      // (sub-chunks past the last one, in the last stages: the last one again)
      const bool is_k = p < KP;
      const int half = is_k ? p / (KP / 2) : (p - KP) / DT, f = is_k ? p % (KP / 2) : (p - KP) % DT;
      const uint32_t sub = (uint32_t)min(2 * st + half, n_here - 1);
      const uint32_t off = (sub * (uint32_t)(is_k ? KP / 2 : DT) + f) * 1024u + lane * 16u;
      load_lds16(lds0 + ((uint32_t)(st % ST) * NP + p) * 1024u, off, is_k ? kr : vr);
    }
  };
  floatx4 of[DT];
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) of[dt] = floatx4{0.f, 0.f, 0.f, 0.f};
  float mx = -INFINITY, sm = 0.f;

  if (n_st > 0) {
#pragma unroll
    for (int i = 0; i < ST - 1; ++i) issue(i);
  }
  // K rows of tile t: key 8 (i/4) + 4t + i%4 of the sub-chunk, i = l % 16
  const int kp0 = 8 * (c16 >> 2) + (c16 & 3);
  for (int st = 0; st < n_st; ++st) {
    wait_vm<(ST - 2) * PW>();
    __syncthreads();  // (stage st has landed for every wave, and every wave is done with stage st - 1)
    issue(st + ST - 1);
    const int k0 = (2 * st + kg) * kSubKeys;
    if (2 * st + kg >= n_here || k0 >= nk) continue;  // (wave-uniform)
    const u32x4(*sk)[kWave] = &s_kv[st % ST][kg * (KP / 2)];
    const u32x4(*sv)[kWave] = &s_kv[st % ST][KP + kg * DT];
    floatx4 sf[2];
#pragma unroll
    for (int t = 0; t < 2; ++t) {
      const int p = kp0 + 4 * t;
      floatx4 acc = floatx4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
      for (int c = 0; c < KST; ++c) {
        const bf16x8 kk = __builtin_bit_cast(bf16x8, sk[(p >> 4) * KST + c][16 * grp + (p & 15)]);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, qhi[c], acc, 0, 0, 0);
        acc = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kk, qlo[c], acc, 0, 0, 0);
      }
      sf[t] = acc;
    }
    if (k0 + kSubKeys - 1 > lo) {  // (wave-uniform) some query does not see the whole sub-chunk
#pragma unroll
      for (int t = 0; t < 2; ++t)
#pragma unroll
        for (int r = 0; r < 4; ++r)
          if (k0 + 8 * grp + 4 * t + r > qpos) sf[t][r] = -INFINITY;
    }
    float m = fmaxf(fmaxf(fmaxf(sf[0][0], sf[0][1]), fmaxf(sf[0][2], sf[0][3])),
                    fmaxf(fmaxf(sf[1][0], sf[1][1]), fmaxf(sf[1][2], sf[1][3])));
    m = fmaxf(m, __shfl_xor(m, 16, kWave));
    m = fmaxf(m, __shfl_xor(m, 32, kWave));
    const float mnew = fmaxf(mx, m);
    if (__any(mnew > mx)) {  // (rescaled only where a maximum rose)
      const float alpha = mx == -INFINITY ? 0.f : expf(mx - mnew);
      sm *= alpha;
#pragma unroll
      for (int dt = 0; dt < DT; ++dt) of[dt] *= alpha;
      mx = mnew;
    }
    float pv[8];
#pragma unroll
    for (int t = 0; t < 2; ++t)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        // (a query that has seen no key yet keeps the maximum -inf)
        pv[4 * t + r] = mx == -INFINITY ? 0.f : expf(sf[t][r] - mx);
        sm += pv[4 * t + r];
      }
    bf16x8 phi, plo;
    split_hilo(pv, phi, plo);
    const int nvalid = nk - (k0 + 8 * grp);
    const bool tail = k0 + kSubKeys > nk;  // (wave-uniform) keys past the tile's: V zeroed, never multiply stale memory
#pragma unroll
    for (int dt = 0; dt < DT; ++dt) {
      u32x4 v = sv[dt][lane];
      if (tail) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
          if (2 * q >= nvalid) v[q] = 0u;
          else if (2 * q + 1 >= nvalid) v[q] &= 0xffffu;
        }
      }
      const bf16x8 vv = __builtin_bit_cast(bf16x8, v);
      of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, phi, of[dt], 0, 0, 0);
      of[dt] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(vv, plo, of[dt], 0, 0, 0);
    }
  }
  sm += __shfl_xor(sm, 16, kWave);
  sm += __shfl_xor(sm, 32, kWave);

  // The two key halves of each tile: waves 4..7 park theirs in LDS, waves 0..3 add them.
  wait_vm<0>();
  __syncthreads();
  float* park = (float*)&s_kv[0][0][0] + (size_t)qt * (4 * DT + 2) * kWave;
  static_assert(4 * (4 * DT + 2) * kWave * 4 <= sizeof(s_kv), "parked sums fit in the stages");
  if (kg == 1) {
#pragma unroll
    for (int dt = 0; dt < DT; ++dt)
#pragma unroll
      for (int r = 0; r < 4; ++r) park[(4 * dt + r) * kWave + lane] = of[dt][r];
    park[4 * DT * kWave + lane] = mx;
    park[(4 * DT + 1) * kWave + lane] = sm;
  }
  __syncthreads();
  if (kg == 1 || qa >= nq) return;
  const float m1 = park[4 * DT * kWave + lane], s1 = park[(4 * DT + 1) * kWave + lane], M = fmaxf(mx, m1);
  const float e0 = mx == -INFINITY ? 0.f : expf(mx - M), e1 = m1 == -INFINITY ? 0.f : expf(m1 - M);
  const float inv = live ? 1.0f / (e0 * sm + e1 * s1) : 0.f;
#pragma unroll
  for (int dt = 0; dt < DT; ++dt) {
    f32x4 o;
#pragma unroll
    for (int r = 0; r < 4; ++r)
      o[r] = live ? (e0 * of[dt][r] + e1 * park[(4 * dt + r) * kWave + lane]) * inv : 0.f;
    put_stacked4(a.xs, a.stt, row, head * HD + 16 * dt + 4 * grp, o);
  }
}

// ---------------------------------------------------------------- combine
// Block (head, row): weights w_c = exp(m_c - max_c m_c) of the row's chunks
// in LDS (fixed-order reductions), then o = sum_c w_c o_c / sum_c w_c l_c with
// the chunk loop unrolled so the partial loads overlap.
__global__ __launch_bounds__(128) void attn_combine_kernel(AttnArgs a) {
  extern __shared__ float wsh[];  // [n_split]
  __shared__ float red[16];
  const int head = blockIdx.x, r = blockIdx.y;
  const int hd = a.head_dim, H = a.n_heads;
  const RowDesc rd = a.rows[r];
  float* o = a.o + ((size_t)r * H + head) * hd;
  if (!rd.valid) {
    for (int dd = threadIdx.x; dd < hd; dd += blockDim.x) put_o(a, o, r, head, dd, 0.f);
    return;
  }
  // splits holding keys <= pos (with parts, the last one also holds the remainder)
  const int nch = min(rd.pos / a.chunk + 1, a.n_split);
  if (rd.pos + 1 > a.max_ctx && threadIdx.x == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
  const size_t base = ((size_t)r * H + head) * a.n_split;
  float mx = -INFINITY;
  for (int c = threadIdx.x; c < nch; c += blockDim.x) mx = fmaxf(mx, a.ml_part[2 * (base + c)]);
  mx = block_max(mx, red);
  float L = 0.f;
  for (int c = threadIdx.x; c < nch; c += blockDim.x) {
    const float w = expf(a.ml_part[2 * (base + c)] - mx);
    wsh[c] = w;
    L += w * a.ml_part[2 * (base + c) + 1];
  }
  L = block_sum(L, red);  // its barrier also publishes wsh
  const float inv = 1.0f / L;
  const float* op = a.o_part + base * hd;
  for (int dd = threadIdx.x; dd < hd; dd += blockDim.x) {
    float acc0 = 0.f, acc1 = 0.f, acc2 = 0.f, acc3 = 0.f;
    int c = 0;
    for (; c + 4 <= nch; c += 4) {
      acc0 += wsh[c] * op[(size_t)c * hd + dd];
      acc1 += wsh[c + 1] * op[(size_t)(c + 1) * hd + dd];
      acc2 += wsh[c + 2] * op[(size_t)(c + 2) * hd + dd];
      acc3 += wsh[c + 3] * op[(size_t)(c + 3) * hd + dd];
    }
    for (; c < nch; ++c) acc0 += wsh[c] * op[(size_t)c * hd + dd];
    put_o(a, o, r, head, dd, ((acc0 + acc1) + (acc2 + acc3)) * inv);
  }
}

// ---------------------------------------------------------------- combine (bf16 path)
// One wave per (row, head).  Every load is issued before the first wait: the
// row's (max, sum) pairs (lane c holds splits c, c+64, ...) and the first 16
// splits' partial outputs (lane holds dims lane, lane+64); each later chunk is
// requested before the current one is accumulated.  o = sum_c w_c o_c /
// sum_c w_c l_c with w_c = exp(m_c - max_c m_c), summed over c in order in four
// interleaved accumulators.
constexpr int kCombineMaxSplits = 256;  // 4 per lane

template <int HD>
__global__ __launch_bounds__(64) void attn_combine_wave_kernel(AttnArgs a) {
  constexpr int DPL = HD >= 64 ? HD / 64 : 1;  // dims per lane
  constexpr int CH = 16;                        // splits per chunk of partial outputs
  const int head = blockIdx.x, r = blockIdx.y, lane = threadIdx.x, H = a.n_heads, ns = a.n_split;
  const size_t base = ((size_t)r * H + head) * ns;
  const __amdgpu_buffer_rsrc_t mlr =
      __builtin_amdgcn_make_buffer_rsrc(a.ml_part + 2 * base, (short)0, ns * 8, 0x00020000);
  const __amdgpu_buffer_rsrc_t opr =
      __builtin_amdgcn_make_buffer_rsrc(a.o_part + base * HD, (short)0, ns * HD * 4, 0x00020000);
  // (two 4-byte loads per pair: this toolchain's 8-byte raw buffer load returns
  // the low word in both elements)
  float mv[4], lv[4];
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    const uint32_t c = lane + 64 * j;
    mv[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mlr, c * 8u, 0, 0));
    lv[j] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(mlr, c * 8u + 4u, 0, 0));
  }
  auto load_chunk = [&](int c0, float (&ov)[CH][DPL]) {
#pragma unroll
    for (int cc = 0; cc < CH; ++cc)
#pragma unroll
      for (int d = 0; d < DPL; ++d) {
        const uint32_t dim = lane + 64 * d;
        const uint32_t off = (((uint32_t)(c0 + cc) * HD + dim) * 4u) | ((uint32_t)(dim >= (uint32_t)HD) << 31);
        ov[cc][d] = __builtin_bit_cast(float, __builtin_amdgcn_raw_buffer_load_b32(opr, off, 0, 0));
      }
  };
  // Partial outputs of NG chunks (64 splits) are requested at once: one memory
  // round trip for contexts up to 64 splits, one more per further 64.
  constexpr int NG = 4;
  float ov[NG][CH][DPL];
#pragma unroll
  for (int g = 0; g < NG; ++g) load_chunk(g * CH, ov[g]);
  asm volatile("" ::: "memory");  // (keep the loads above the exits below)

  const RowDesc rd = a.rows[r];
  float* o = a.o + ((size_t)r * H + head) * HD;
  if (!rd.valid) {
#pragma unroll
    for (int d = 0; d < DPL; ++d)
      if (lane + 64 * d < HD) put_o(a, o, r, head, lane + 64 * d, 0.f);
    return;
  }
  // parts holding keys <= pos (the last part also holds the remainder)
  const int nch = min(rd.pos / a.chunk + 1, ns);
  if (rd.pos + 1 > a.max_ctx && lane == 0) set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
  float mx = -INFINITY;
#pragma unroll
  for (int j = 0; j < 4; ++j)
    if (lane + 64 * j < nch) mx = fmaxf(mx, mv[j]);
  mx = wave_max(mx);
  float wv[4], L = 0.f;
#pragma unroll
  for (int j = 0; j < 4; ++j) {
    wv[j] = lane + 64 * j < nch ? expf(mv[j] - mx) : 0.f;
    L += wv[j] * lv[j];
  }
  L = wave_sum(L);
  float acc[4][DPL];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int d = 0; d < DPL; ++d) acc[i][d] = 0.f;
  for (int g0 = 0; g0 < nch; g0 += NG * CH) {
    if (g0 > 0) {
#pragma unroll
      for (int g = 0; g < NG; ++g) load_chunk(g0 + g * CH, ov[g]);
    }
#pragma unroll
    for (int g = 0; g < NG; ++g)
#pragma unroll
      for (int cc = 0; cc < CH; ++cc) {
        const int c = g0 + g * CH + cc;
        if (c < nch) {
          const float wj = c < 64 ? wv[0] : (c < 128 ? wv[1] : (c < 192 ? wv[2] : wv[3]));
          const float w = __shfl(wj, c & 63, kWave);
#pragma unroll
          for (int d = 0; d < DPL; ++d) acc[cc & 3][d] += w * ov[g][cc][d];
        }
      }
  }
  const float inv = 1.0f / L;
#pragma unroll
  for (int d = 0; d < DPL; ++d)
    if (lane + 64 * d < HD) put_o(a, o, r, head, lane + 64 * d, ((acc[0][d] + acc[1][d]) + (acc[2][d] + acc[3][d])) * inv);
}

// ---------------------------------------------------------------- KV context copy
template <typename KT>
__global__ __launch_bounds__(256) void kv_copy_kernel(KvLayout kv, int layer, int b, int pos0, const KT* k,
                                                      const KT* v, KT* k_out, KT* v_out) {
  const int p = blockIdx.x;
  const int hd = kv.head_dim, G = kv.n_kv_heads;
  for (int i = threadIdx.x; i < G * hd; i += blockDim.x) {
    const int g = i / hd, dd = i % hd;
    KT* blk = k_block<KT>(kv, layer, b, g);
    KT* kc = blk + KvIndex<KT>::k(pos0 + p, dd, hd, kv.capacity);
    KT* vc = blk + KvIndex<KT>::v(pos0 + p, dd, hd, kv.capacity);
    const size_t src = ((size_t)p * G + g) * hd + dd;
    if (k) *kc = k[src];
    if (v) *vc = v[src];
    if (k_out) k_out[src] = *kc;
    if (v_out) v_out[src] = *vc;
  }
}

size_t attn_smem_bytes(int chunk, int hd) {
  return sizeof(float) * ((size_t)chunk * (hd + 1) + (size_t)hd * (chunk + 1) + kQB * hd + kQB * chunk + 2 * kQB);
}

}  // namespace

int attention_chunk(int dtype, int head_dim) {
  if (dtype == SPECDEC_BF16) return kSubKeys;  // (parts are whole numbers of sub-chunks: at most one split each)
  return head_dim >= 128 ? 32 : (head_dim >= 64 ? 64 : 128);
}

hipError_t launch_rope_append(const AttnArgs& a, hipStream_t s) {
  if (a.kv.dtype != SPECDEC_F32) return hipErrorInvalidValue;
  hipLaunchKernelGGL(rope_append_kernel, dim3(a.n_heads + 2 * a.n_kv_heads, a.M), dim3(64), 0, s, a);
  return hipGetLastError();
}

__global__ void fill_u32_kernel(uint32_t* p, size_t n, uint32_t v) {
  const size_t i = blockIdx.x * (size_t)blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

hipError_t launch_fill_u32(uint32_t* p, size_t n, uint32_t v, hipStream_t s) {
  if (n == 0) return hipSuccess;
  hipLaunchKernelGGL(fill_u32_kernel, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, s, p, n, v);
  return hipGetLastError();
}

size_t attention_counter_count(int n_heads, int n_kv_heads, int max_rows) {
  // sequences x query tiles <= max_rows * group / 16 + max_rows
  const size_t group = (size_t)(n_heads / n_kv_heads);
  return (size_t)n_kv_heads * ((size_t)max_rows * group / 16 + (size_t)max_rows + 1);
}

hipError_t launch_attention(const AttnArgs& a, hipStream_t s) {
  const int B = a.M / a.rps;
  AttnArgs ab = a;  // the bf16 path chooses its own parts
  if (a.kv.dtype == SPECDEC_BF16) {
    const int nq = a.rps * (a.n_heads / a.n_kv_heads), n_mt = (nq + 15) / 16, RS = nq < 16 ? nq : 16;
    const int n_sub = (a.max_ctx + kSubKeys - 1) / kSubKeys;
    if (n_sub * kSubKeys > a.kv.capacity || n_sub > a.n_split * (a.chunk / kSubKeys)) return hipErrorInvalidValue;
    const long units = (long)a.n_kv_heads * B * n_mt;
    const int cus = device_compute_units();
    // Many query rows: blocks of 4 tiles that share K and V and need no combine,
    // where there are enough of them for half the CUs.
    const int n_qb = (nq + 63) / 64;
    if (a.xs && nq >= 64 && (long)n_qb * a.n_kv_heads * B * 2 >= cus) {
      const dim3 qgrid(n_qb, a.n_kv_heads, B);
      switch (a.head_dim) {
        case 32: hipLaunchKernelGGL((attn_rows_kernel<32>), qgrid, dim3(512), 0, s, a, n_sub); break;
        case 64: hipLaunchKernelGGL((attn_rows_kernel<64>), qgrid, dim3(512), 0, s, a, n_sub); break;
        case 128: hipLaunchKernelGGL((attn_rows_kernel<128>), qgrid, dim3(512), 0, s, a, n_sub); break;
        default: return hipErrorInvalidValue;
      }
      return hipGetLastError();
    }
    int S = 0, n_part = 0, NW = 0;
    if (n_sub * units <= (long)cus * kMaxPartWaves) {
      // One sub-chunk per wave, one round: parts of S sub-chunks (the last one
      // takes the remainder), the blocks about filling the CUs once.
      S = (int)((n_sub * units + cus / 2) / cus);
      S = S < 1 ? 1 : (S > kMaxPartWaves ? kMaxPartWaves : S);  // (reduced below while the last part is too big)
      // (more units than CUs: a part never holds more sub-chunks than the keys
      // have, so its waves take one sub-chunk each and never loop)
      S = std::max(1, std::min(S, n_sub));
      for (;; --S) {
        n_part = n_sub / S > 0 ? n_sub / S : 1;
        NW = n_sub - (n_part - 1) * S;
        if (S == 1 || (NW <= kMaxPartWaves && attn_block_lds(NW, RS, a.head_dim) <= 65536)) break;
      }
    } else {
      // Long contexts and batches: the persistent kernel over the sub-chunks themselves.
      const dim3 sgrid(2 * cus), sblock(64 * kLoopWaves), cgrid(a.n_heads, a.M);
      const size_t slds = attn_stream_lds(RS, a.head_dim);
#define SD_STREAM(HDV)                                                                                             \
  if (n_mt == 1) hipLaunchKernelGGL((attn_stream_kernel<HDV, true>), sgrid, sblock, slds, s, a, n_sub, 1);         \
  else hipLaunchKernelGGL((attn_stream_kernel<HDV, false>), sgrid, sblock, slds, s, a, n_sub, n_mt);               \
  hipLaunchKernelGGL((attn_stream_combine_kernel<HDV>), cgrid, dim3(64), 0, s, a, n_sub, n_mt, 2 * cus);
      switch (a.head_dim) {
        case 32: SD_STREAM(32) break;
        case 64: SD_STREAM(64) break;
        case 128: SD_STREAM(128) break;
        default: return hipErrorInvalidValue;
      }
#undef SD_STREAM
      return hipGetLastError();
    }
    if (NW > kMaxPartWaves || attn_block_lds(NW, RS, a.head_dim) > 65536) return hipErrorInvalidValue;
    ab.n_split = n_part;
    ab.chunk = S * kSubKeys;
    // In-kernel combine: one part per lane, at most two query rows per wave of
    // the combining block (its rows go one after another); otherwise the
    // separate combine kernel (one wave per row and head).
    if (n_part > kMaxParts || (RS + NW - 1) / NW > 2) ab.counters = nullptr;
    const dim3 grid(n_part * n_mt, a.n_kv_heads, B);
    const size_t lds = attn_block_lds(NW, RS, a.head_dim);
#define SD_ATTN(HDV) hipLaunchKernelGGL((attn_block_kernel<HDV>), grid, dim3(64 * NW), lds, s, ab, S, n_sub, NW);
    switch (a.head_dim) {
      case 32: SD_ATTN(32) break;
      case 64: SD_ATTN(64) break;
      case 128: SD_ATTN(128) break;
      default: return hipErrorInvalidValue;
    }
#undef SD_ATTN
  } else {
    const size_t smem = attn_smem_bytes(a.chunk, a.head_dim);
    dim3 grid(a.n_split, a.n_kv_heads, B);
    hipLaunchKernelGGL((attn_partial_kernel<float>), grid, dim3(256), smem, s, a);
  }
  hipError_t e = hipGetLastError();
  if (e != hipSuccess) return e;
  if (ab.kv.dtype == SPECDEC_BF16 && ab.counters) return hipSuccess;  // combined by the blocks
  if (ab.kv.dtype == SPECDEC_BF16 && ab.n_split <= kCombineMaxSplits) {
    switch (ab.head_dim) {
      case 32: hipLaunchKernelGGL((attn_combine_wave_kernel<32>), dim3(ab.n_heads, ab.M), dim3(64), 0, s, ab); break;
      case 64: hipLaunchKernelGGL((attn_combine_wave_kernel<64>), dim3(ab.n_heads, ab.M), dim3(64), 0, s, ab); break;
      default: hipLaunchKernelGGL((attn_combine_wave_kernel<128>), dim3(ab.n_heads, ab.M), dim3(64), 0, s, ab); break;
    }
  } else {
    hipLaunchKernelGGL(attn_combine_kernel, dim3(ab.n_heads, ab.M), dim3(128), sizeof(float) * ab.n_split, s, ab);
  }
  return hipGetLastError();
}

hipError_t launch_kv_copy(const KvLayout& kv, int layer, int b, int pos0, int n, const void* k, const void* v,
                          void* k_out, void* v_out, hipStream_t s) {
  if (n <= 0) return hipSuccess;
  if (kv.dtype == SPECDEC_BF16)
    hipLaunchKernelGGL((kv_copy_kernel<uint16_t>), dim3(n), dim3(256), 0, s, kv, layer, b, pos0,
                       (const uint16_t*)k, (const uint16_t*)v, (uint16_t*)k_out, (uint16_t*)v_out);
  else
    hipLaunchKernelGGL((kv_copy_kernel<float>), dim3(n), dim3(256), 0, s, kv, layer, b, pos0, (const float*)k,
                       (const float*)v, (float*)k_out, (float*)v_out);
  return hipGetLastError();
}

}  // namespace specdec
