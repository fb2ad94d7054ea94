// Row set-up + embedding gather, the draft's sampling step, the speculative
// accept / resample decision, the fixed-point sampler, Philox draws and the
// KV commit.
//
// Sampling reading (shared with the host documentation in specdec.h): a draw
// from non-negative weights r_j uses R_j = floor(r_j * 2^40) as uint64,
// S = sum R_j, t = floor(x * S / 2^32) for a 32-bit word x, and returns the
// smallest j with R_0 + ... + R_j > t.  Every sum is an integer sum, so the
// result does not depend on how the block splits and orders the reduction.
#include <mutex>

#include "device_common.h"
#include "internal.h"

namespace specdec {

namespace {

constexpr int kSampThreads = 1024;
constexpr int kMaxGamma = 31;

__device__ __forceinline__ uint64_t fp_weight(float r) {
  return r > 0.f ? (uint64_t)(r * 1099511627776.0f) : 0ull;  // exact: r * 2^40, truncation = floor
}
// floor(x * S / 2^32) without a 128-bit product (S < 2^56, x < 2^32).
__device__ __forceinline__ uint64_t scale_word(uint32_t x, uint64_t S) {
  return (uint64_t)x * (S >> 32) + (((uint64_t)x * (S & 0xffffffffull)) >> 32);
}

__device__ __forceinline__ uint64_t shfl_up_u64(uint64_t v, int o) {
  uint32_t lo = __shfl_up((uint32_t)v, o, kWave), hi = __shfl_up((uint32_t)(v >> 32), o, kWave);
  return ((uint64_t)hi << 32) | lo;
}

struct SampShared {
  uint64_t wave_tot[kSampThreads / kWave];
  int token;
};

// Block-wide fixed-point draw over j < V with weights rf(j) (floats >= 0).
// Wave w owns the contiguous segment [w*seg, (w+1)*seg) (seg a multiple of
// 64); lanes read it with unit stride.  Pass 1 sums the integer weights per
// wave; the wave whose range of the running sum holds t then scans its
// segment 64 entries at a time.  Returns the token (same value in every
// thread), or -1 when all weights are zero.
template <typename RF>
__device__ int block_draw(RF rf, int V, uint32_t x, SampShared& sh) {
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6, nw = blockDim.x / kWave;
  const int seg = ((V + nw - 1) / nw + kWave - 1) / kWave * kWave;
  const int j0 = min(V, wave * seg), j1 = min(V, j0 + seg);
  uint64_t mine = 0;
  for (int j = j0 + lane; j < j1; j += kWave) mine += fp_weight(rf(j));
  mine = wave_sum_u64(mine);
  __syncthreads();
  if (lane == 0) sh.wave_tot[wave] = mine;
  if (tid == 0) sh.token = -1;
  __syncthreads();
  uint64_t before = 0, total = 0;
  for (int w = 0; w < nw; ++w) {
    if (w < wave) before += sh.wave_tot[w];
    total += sh.wave_tot[w];
  }
  if (total != 0) {
    const uint64_t t = scale_word(x, total);
    if (mine != 0 && before <= t && t < before + mine) {
      uint64_t cum0 = before;
      for (int c = j0; c < j1; c += kWave) {
        const int j = c + lane;
        uint64_t incl = j < j1 ? fp_weight(rf(j)) : 0ull;
#pragma unroll
        for (int o = 1; o < kWave; o <<= 1) {
          const uint64_t n = shfl_up_u64(incl, o);
          if (lane >= o) incl += n;
        }
        const unsigned long long hit = __ballot(cum0 + incl > t);
        if (hit) {
          const int first = __ffsll(hit) - 1;
          if (lane == 0) sh.token = c + first;
          break;
        }
        cum0 += __shfl(incl, kWave - 1, kWave);
      }
    }
  }
  __syncthreads();
  return sh.token;
}

// (max, sum exp) of z_j = row[j] / T over part of a row; states are merged in a
// fixed order (deterministic).
struct MaxSum {
  float m, s;
};
__device__ __forceinline__ MaxSum ms_merge(MaxSum a, MaxSum b) {
  if (b.m == -INFINITY) return a;
  if (a.m == -INFINITY) return b;
  const float m = fmaxf(a.m, b.m);
  return MaxSum{m, a.s * expf(a.m - m) + b.s * expf(b.m - m)};
}

// ---------------------------------------------------------------- rows + embedding
// Grid (rows, 2): block (r, 0) gathers and scales row r's embedding, block (r,
// 1) computes its RoPE table (in float64: the angle of position p at float32
// resolution needs it) with one thread per cosine and one per sine.  Both are
// latency chains (the table's pow, then cos or sin; the row's state words,
// then its embedding), so they run side by side: 12.8 us for the two one after
// the other over 5 rows of the 7B shape, 6.2 now (at the head of a pass).
template <typename ET>
__global__ __launch_bounds__(256) void rows_embed_kernel(RowsArgs a) {
  __shared__ float red[16];
  const int r = blockIdx.x, b = r / a.rps, i = r % a.rps;
  const bool first = blockIdx.y == 0 && threadIdx.x == 0;  // (writes the row's descriptor and status)
  int pos = 0, tok = 0, valid = 1;
  switch (a.mode) {
    case ROWS_VERIFY:
      pos = a.len[b] + i;
      tok = i == 0 ? a.pending[2 * b + 1] : a.tok_src[(size_t)b * a.ld_tok + i - 1];
      break;
    case ROWS_DRAFT_FIRST: {
      const int np = a.n_pending[b];
      valid = i >= 2 - np;
      pos = a.len[b] + i - (2 - np);
      tok = a.pending[2 * b + i];
      break;
    }
    case ROWS_DRAFT_NEXT:
      pos = a.len[b] + a.n_pending[b] + a.slot - 1;
      tok = a.tok_src[(size_t)b * a.ld_tok + a.slot - 1];
      break;
    default:  // ROWS_PREFILL
      pos = a.len[b] + a.c0 + i;
      tok = a.tok_src[(size_t)b * a.ld_tok + a.c0 + i];
      break;
  }
  if (valid) {
    if (tok < 0 || tok >= a.vocab) {
      if (first) set_status(a.status, kStatusBadToken);
      valid = 0;
    }
    if (pos < 0 || pos >= a.capacity) {
      if (first) set_status(a.status, kStatusKvCapacity);
      valid = 0;
    } else if (pos >= a.max_ctx && first) {
      set_status(a.status, kStatusKvCapacity);  // the host's bound was wrong
    }
  }
  if (!valid) {
    tok = 0;
    pos = 0;
  }
  if (blockIdx.y == 1) {
    const int hd = a.head_dim, half = hd / 2;
    for (int k = threadIdx.x; k < hd; k += blockDim.x) {
      const int j = k < half ? k : k - half;
      const double inv_freq = pow(a.rope_base, -2.0 * (double)j / (double)hd);
      const double ang = (double)pos * inv_freq;
      a.rope_cs[(size_t)r * hd + k] = (float)(k < half ? cos(ang) : sin(ang));
    }
    return;
  }
  if (first) {
    a.rows[r] = RowDesc{b, pos, tok, valid};
  }
  const ET* e = (const ET*)a.embed + (size_t)tok * a.d_model;
  const ET* gn = (const ET*)a.gain;
  float* h = a.h + (size_t)r * a.d_model;
  float* xg = a.xg + (size_t)r * a.d_model;
  float ss = 0.f;
  for (int k = 4 * threadIdx.x; k < a.d_model; k += 4 * blockDim.x) {  // (d_model % 64 == 0)
    f32x4 v, x;
#pragma unroll
    for (int q = 0; q < 4; ++q) {
      v[q] = Storage<ET>::load(e + k + q);
      x[q] = v[q] * Storage<ET>::load(gn + k + q);
    }
    *(f32x4*)(h + k) = v;
    if (a.xs) put_stacked4(a.xs, a.stt, r, k, x);
    else *(f32x4*)(xg + k) = x;
    ss += (v[0] * v[0] + v[1] * v[1]) + (v[2] * v[2] + v[3] * v[3]);
  }
  ss = block_sum(ss, red);
  if (threadIdx.x == 0) a.ss[r] = ss;
}

// ---------------------------------------------------------------- multi-block softmax / accept / draw
// A vocabulary row is cut into NC chunks so that a single decision uses many
// CUs, in two launches:
//   stats         per (chunk, row): online (max, sum exp) of z = x / T, argmax, finiteness
//   decide-draw   per (chunk, sequence): every block merges the chunk statistics
//                 (fixed order) and takes the decision; each sums the integer
//                 weights of its chunk of the row to draw from (the draft's q is
//                 also written here); the last block of the sequence finds the
//                 chunk holding t, scans it and emits the token
constexpr int kChunkThreads = 256;

__host__ __device__ __forceinline__ int n_chunks(int V) {
  int nc = (V + 511) / 512;  // (512-entry chunks: 63 blocks per 32000-entry row; 1024 and 2048 were slower)
  return nc < 1 ? 1 : (nc > 64 ? 64 : nc);
}
// (whole quads: only a row's own end is ragged; the last chunk may be short or empty)
__host__ __device__ __forceinline__ int chunk_size(int V) { return ((V + n_chunks(V) - 1) / n_chunks(V) + 3) / 4 * 4; }

struct StatPart {
  float m, s, amax_v;
  int amax_i, bad;
  uint32_t count;  // of a sequence's first part: blocks of the decide-and-draw launch done (a line of its own per sequence)
  int pad0, pad1;
};
struct DrawPart {
  unsigned long long res, prob;
};
// A sequence's decision, kept in LDS by every block of the decide-and-draw launch.
struct SeqState {
  int A;            // accepted count (-1 error, -2 no draw needed)
  int pad;
  float2 ms[kMaxGamma + 1];  // merged (max, sum) per row
};

struct Scratch {
  StatPart* stats;  // [rows_total][NC]
  DrawPart* draw;   // [B][NC]
};
__host__ __device__ inline size_t align256(size_t x) { return (x + 255) / 256 * 256; }
__host__ __device__ inline Scratch carve(void* base, int B, int rows, int V) {
  const int NC = n_chunks(V);
  char* p = (char*)base;
  Scratch s;
  s.stats = (StatPart*)p;
  p += align256(sizeof(StatPart) * (size_t)B * rows * NC);
  s.draw = (DrawPart*)p;
  return s;
}

// Four consecutive entries of a row of V from j (a multiple of 4), `pad` past
// j1 (a multiple of 4, or V).
__device__ __forceinline__ void load_quad(const float* row, int j, int j1, int V, float pad, float (&v)[4]) {
#pragma unroll
  for (int e = 0; e < 4; ++e) v[e] = pad;
  if ((V & 3) == 0 || j + 4 <= j1) {  // (first test uniform: whole quads need no second path)
    if (j < j1) {
      const f32x4 t = *(const f32x4_a4*)(row + j);
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = t[e];
    }
  } else {
#pragma unroll
    for (int e = 0; e < 4; ++e)
      if (j + e < j1) v[e] = row[j + e];
  }
}

// stats: grid (NC, B * rows_per_seq), block 256.  Row i of sequence b is
// x + (b * row_stride + row_off + i) * V.
// Every value of the row, and of the row `chk` pairs with it (the draft's q
// row i of an accept, rows i < chk_rows), must be finite.
// It also zeroes the sequence's counter of the decide-and-draw launch that follows.
// Two quads per thread and round, all loaded before the first is used; the
// block's maximum first (the argmax with it), then exponentials relative to it,
// which neither wait for one another nor need merging by further ones.  Bound:
// a block's latency chain (one load round trip, two reductions) for a single
// row; over 16 x 7 rows of 128256 entries (107 MB with the drafts' rows) the
// exponentials and divisions, 43.5 us with one entry per load and an online
// maximum.
__global__ __launch_bounds__(kChunkThreads) void stats_kernel(const float* x, int V, int rows_per_seq, int row_stride,
                                                              int row_off, float T, const float* chk, int chk_rows,
                                                              StatPart* out) {
  __shared__ float sm_m[4], sm_s[4], sm_v[4];
  __shared__ int sm_i[4], sm_b[4];
  const int c = blockIdx.x, r = blockIdx.y, NC = gridDim.x;
  const int b = r / rows_per_seq, i = r % rows_per_seq;
  const float* row = x + ((size_t)b * row_stride + row_off + i) * V;
  const int cs = chunk_size(V), j0 = c * cs, j1 = min(V, j0 + cs);
  const float* crow = chk && i < chk_rows ? chk + ((size_t)b * chk_rows + i) * V : nullptr;
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  constexpr int Q = 2, RND = 4 * Q * kChunkThreads;
  MaxSum st{-INFINITY, 0.f};
  float bv = -INFINITY;
  int bi = 0x7fffffff, bad = 0;
  for (int r0 = j0; r0 < j1; r0 += RND) {  // (block-uniform)
    const int base = r0 + 4 * threadIdx.x;
    float v[Q][4], u[Q][4];
#pragma unroll
    for (int q = 0; q < Q; ++q) load_quad(row, base + 4 * q * kChunkThreads, j1, V, -INFINITY, v[q]);
    if (crow) {  // (block-uniform)
#pragma unroll
      for (int q = 0; q < Q; ++q) load_quad(crow, base + 4 * q * kChunkThreads, j1, V, 0.f, u[q]);
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) bad |= !isfinite(u[q][e]);
    }
    // this thread's maximum, its lowest index, then the wave's (max, then the lowest index that holds it)
    float mv = -INFINITY;
    int mi = 0x7fffffff;
#pragma unroll
    for (int q = 0; q < Q; ++q)
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        const int j = base + 4 * q * kChunkThreads + e;
        bad |= j < j1 && !isfinite(v[q][e]);
        if (v[q][e] > mv) { mv = v[q][e]; mi = j; }
      }
    const float wv = wave_max(mv);
    int wi = mv == wv ? mi : 0x7fffffff;
#pragma unroll
    for (int o = 32; o > 0; o >>= 1) wi = min(wi, __shfl_xor(wi, o, kWave));
    if (wv > bv || (wv == bv && wi < bi)) { bv = wv; bi = wi; }
    if (T > 0.f) {  // (z = v / T grows with v: the wave's maximum z is that of its largest entry)
      const float m = fmaxf(st.m, T == 1.f ? wv : wv / T);
      float sum = 0.f;
#pragma unroll
      for (int q = 0; q < Q; ++q)
#pragma unroll
        for (int e = 0; e < 4; ++e) sum += expf((T == 1.f ? v[q][e] : v[q][e] / T) - m);  // (past the chunk: exp(-inf))
      st.s = (st.m == -INFINITY ? 0.f : st.s * expf(st.m - m)) + sum;
      st.m = m;
    }
  }
  st.s = wave_sum(st.s);  // (st.m and the argmax are the wave's already)
  bad = __any(bad);
  if (lane == 0) { sm_m[w] = st.m; sm_s[w] = st.s; sm_v[w] = bv; sm_i[w] = bi; sm_b[w] = bad; }
  __syncthreads();
  if (threadIdx.x == 0) {
    MaxSum t{sm_m[0], sm_s[0]};
    float tv = sm_v[0];
    int ti = sm_i[0], tb = sm_b[0];
    for (int k = 1; k < kChunkThreads / kWave; ++k) {
      t = ms_merge(t, MaxSum{sm_m[k], sm_s[k]});
      if (sm_v[k] > tv || (sm_v[k] == tv && sm_i[k] < ti)) { tv = sm_v[k]; ti = sm_i[k]; }
      tb |= sm_b[k];
    }
    out[(size_t)r * NC + c] = StatPart{t.m, t.s, tv, ti, tb, 0u, 0, 0};
  }
}

// Merge the chunk statistics of one row across a wave: lane k holds chunk k
// (NC <= 64).  The row's maximum, then each chunk's sum relative to it, added
// by a fixed shuffle tree: every lane ends with the same, deterministic result.
__device__ StatPart wave_merge_stats(const StatPart* parts, int NC) {
  const int lane = threadIdx.x & 63;
  StatPart p{-INFINITY, 0.f, -INFINITY, 0x7fffffff, 0, 0u, 0, 0};
  if (lane < NC) p = parts[lane];
  const float m = wave_max(p.m), v = wave_max(p.amax_v);
  int i = p.amax_v == v ? p.amax_i : 0x7fffffff;
  float s = p.m == -INFINITY ? 0.f : p.s * expf(p.m - m);
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    i = min(i, __shfl_xor(i, o, kWave));
    s += __shfl_xor(s, o, kWave);
  }
  p.m = m;
  p.s = s;
  p.amax_v = v;
  p.amax_i = i;
  p.bad = __any(p.bad);
  return p;
}

// Weight sources of a draw.
enum { W_ACCEPT = 0, W_DRAFT = 1 };

struct DrawArgs {
  int mode, B, V, gamma;
  float T;
  // accept: p rows [B, gamma+1, V] (probabilities or logits), q rows [B, gamma, V], drafts
  const float* p;
  const float* q;
  int logits;
  const int32_t* d;
  int ld_d;
  // draft: logits of the proposing rows (the last of rps per sequence), q output
  const float* lg;
  int rps, slot;
  float* q_out;
  void* scratch;
  int rows;  // rows per sequence in the scratch statistics
  // the words of the draws, the outputs
  const uint32_t* rand;   // accept: [B, gamma+1] (accept words, then the resample word); draft: [B]
  uint64_t seed, step;
  const uint64_t* step_dev;  // or null: read in place of step
  int32_t* n_accepted;    // accept only
  int32_t* out;           // accept: next_token[B]; draft: d_out + slot (stride ld_out)
  int ld_out;
  int32_t* status;
};

// R_j weights of sequence b at the four columns from j (past j1: 0), for the
// residual (res) and the plain row (prob).
__device__ __forceinline__ void weights_quad(const DrawArgs& a, const SeqState& st, int b, int j, int j1, float (&res)[4],
                                             float (&prob)[4]) {
  const bool accept = a.mode == W_ACCEPT;
  const int A = accept ? st.A : 0, g = a.gamma;
  const float* P = accept ? a.p + ((size_t)b * (g + 1) + A) * a.V : a.lg + ((size_t)b * a.rps + a.rps - 1) * a.V;
  const bool resid = accept && A < g;
  float v[4], q[4] = {0.f, 0.f, 0.f, 0.f};
  load_quad(P, j, j1, a.V, 0.f, v);
  if (resid) load_quad(a.q + ((size_t)b * g + A) * a.V, j, j1, a.V, 0.f, q);
  const bool softmax = !accept || a.logits;
  const float2 ms = st.ms[A];
#pragma unroll
  for (int e = 0; e < 4; ++e) {
    const float p = softmax ? expf((a.T == 1.f ? v[e] : v[e] / a.T) - ms.x) / ms.y : v[e];
    prob[e] = j + e < j1 ? p : 0.f;
    res[e] = resid && j + e < j1 ? fmaxf(0.f, __fsub_rn(p, q[e])) : 0.f;
  }
}

// decide-and-draw: grid (NC, B), block 256.  Every block of sequence b first
// takes the sequence's decision itself, from the chunk statistics of the stats
// launch (merged in a fixed order: every block reaches the same result):
//   accept: the row statistics, then the gamma accept tests in parallel lanes,
//           the first event (rejection or error) in draft order wins;
//   draft:  the proposing row's statistics.
// Greedy decisions and errors are written by block 0 and end there.  Otherwise
// block c sums the integer weights of its chunk of the row to draw from (the
// residual and the plain row; the draft's q chunk is written here), publishes
// them with agent-scope stores and counts itself; the last block of the
// sequence finds the chunk holding t (a wave prefix sum over the chunk sums)
// and scans that chunk for the token.  Integer sums: exact in any order.
__global__ __launch_bounds__(kChunkThreads) void decide_draw_kernel(DrawArgs a) {
  __shared__ SeqState st;
  __shared__ int amax[kMaxGamma + 1];
  __shared__ int bad_rows;
  __shared__ unsigned long long sr[4], sp[4], wtot[4];
  __shared__ int last, chunk_sel, use_res, done;
  __shared__ unsigned long long t_in_chunk;
  const int c = blockIdx.x, b = blockIdx.y, V = a.V, NC = gridDim.x, cs = chunk_size(V);
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  Scratch sc = carve(a.scratch, a.B, a.rows, V);
  uint32_t* const count = &sc.stats[(size_t)b * a.rows * NC].count;
  const bool accept = a.mode == W_ACCEPT;
  const int g = accept ? a.gamma : 0;
  const float T = a.T;
  const uint64_t step = a.step_dev ? *a.step_dev : a.step;
  if (threadIdx.x == 0) bad_rows = 0;
  // The accept tests' operands (lane i < g of wave 0: draft position i), on
  // their way while the row statistics are merged.
  int di = 0;
  float pv = 0.f, qv = 0.f;
  if (accept && w == 0 && lane < g) {
    di = a.d[(size_t)b * a.ld_d + lane];
    if (T > 0.f && di >= 0 && di < V) {
      pv = a.p[((size_t)b * (g + 1) + lane) * V + di];
      qv = a.q[((size_t)b * g + lane) * V + di];
    }
  }
  __syncthreads();
  // row statistics (wave w: rows w, w + 4, ...)
  for (int r = w; r <= g; r += kChunkThreads / kWave) {
    const StatPart p = wave_merge_stats(sc.stats + ((size_t)b * a.rows + r) * NC, NC);
    if (lane == 0) {
      amax[r] = p.amax_i;
      st.ms[r] = make_float2(p.m, p.s);
      const bool softmax = accept ? (a.logits && T > 0.f) : T > 0.f;
      if (p.bad || (softmax && (!isfinite(p.m) || !isfinite(p.s)))) atomicOr(&bad_rows, 1);
    }
  }
  __syncthreads();
  if (w == 0) {
    int bad = bad_rows, A = g;
    if (accept && !bad) {
      // lane i < g: event of draft position i (1 = rejection, 2 = error)
      int ev = 0;
      if (lane < g) {
        if (T == 0.f) {
          ev = amax[lane] != di ? 1 : 0;
        } else if (di < 0 || di >= V) {
          ev = 2;
        } else {
          const float pd = a.logits ? expf(pv / T - st.ms[lane].x) / st.ms[lane].y : pv;
          const uint32_t wd = a.rand ? a.rand[(size_t)b * (g + 1) + lane]
                                     : draw_word(a.seed, b, step, SPECDEC_PURPOSE_ACCEPT, lane);
          ev = !isfinite(qv) ? 2 : (!(__fmul_rn(word_to_uniform(wd), qv) < pd) ? 1 : 0);
        }
      }
      const unsigned long long hit = __ballot(ev != 0);
      if (hit) {
        const int first = __ffsll(hit) - 1;
        if (__shfl(ev, first, kWave) == 2) bad = 1;
        else A = first;
      }
    }
    if (lane == 0) {
      const bool greedy = T == 0.f;
      if (c == 0) {  // (one block writes the decision)
        if (bad) set_status(a.status, kStatusNonFinite);
        if (accept) {
          a.n_accepted[b] = bad ? -1 : A;
          if (bad) a.out[b] = -1;
          else if (greedy) a.out[b] = amax[A];
        } else if (bad || greedy) {
          a.out[(size_t)b * a.ld_out] = bad ? 0 : amax[0];
        }
      }
      st.A = bad ? -1 : (greedy ? -2 : (accept ? A : 0));
    }
  }
  __syncthreads();
  if (st.A < 0) return;  // (block-uniform: an error, or a greedy decision already written)

  // this chunk's integer weight sums
  {
    const int j0 = c * cs, j1 = min(V, j0 + cs);
    unsigned long long r_sum = 0, p_sum = 0;
    float* qo = !accept && a.q_out ? a.q_out + ((size_t)b * a.gamma + a.slot) * V : nullptr;
    constexpr int Q = 2;  // quads per thread and round (their loads overlap)
    for (int base = j0 + 4 * threadIdx.x; base < j1; base += 4 * Q * kChunkThreads) {
      float res[Q][4], prob[Q][4];
#pragma unroll
      for (int q = 0; q < Q; ++q) weights_quad(a, st, b, base + 4 * q * kChunkThreads, j1, res[q], prob[q]);
#pragma unroll
      for (int q = 0; q < Q; ++q) {
        const int j = base + 4 * q * kChunkThreads;
        if (qo) {
          if (j + 4 <= j1) *(f32x4_a4*)(qo + j) = f32x4{prob[q][0], prob[q][1], prob[q][2], prob[q][3]};
          else
            for (int e = 0; j + e < j1; ++e) qo[j + e] = prob[q][e];
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
          r_sum += fp_weight(res[q][e]);
          p_sum += fp_weight(prob[q][e]);
        }
      }
    }
    r_sum = wave_sum_u64(r_sum);
    p_sum = wave_sum_u64(p_sum);
    if (lane == 0) { sr[w] = r_sum; sp[w] = p_sum; }
    __syncthreads();
    if (threadIdx.x == 0) {
      unsigned long long dr = 0ull, dp = 0ull;
      for (int k = 0; k < kChunkThreads / kWave; ++k) { dr += sr[k]; dp += sp[k]; }
      DrawPart* dst = sc.draw + (size_t)b * NC + c;
      __hip_atomic_store(&dst->res, dr, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      __hip_atomic_store(&dst->prob, dp, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      // (the stores have completed before the count: the last block reads them with agent-scope loads)
      asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
      const uint32_t old = __hip_atomic_fetch_add(count, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      last = old == (uint32_t)(NC - 1);
      if (last) __hip_atomic_store(count, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
    if (!last) return;
  }

  // the last block: the chunk holding t, then the token inside it
  if (w == 0) {  // lane k holds chunk k
    DrawPart pk{0ull, 0ull};
    if (lane < NC) {
      const DrawPart* src = sc.draw + (size_t)b * NC + lane;
      pk.res = __hip_atomic_load(&src->res, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      pk.prob = __hip_atomic_load(&src->prob, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    const unsigned long long tr = wave_sum_u64(pk.res), tp = wave_sum_u64(pk.prob);
    const bool res = accept && st.A < g && tr != 0;
    const unsigned long long S = res ? tr : tp;
    uint32_t x;
    if (accept)
      x = a.rand ? a.rand[(size_t)b * (g + 1) + g] : draw_word(a.seed, b, step, SPECDEC_PURPOSE_RESAMPLE, 0);
    else
      x = a.rand ? a.rand[b] : draw_word(a.seed, b, step, SPECDEC_PURPOSE_DRAFT, a.slot);
    if (S == 0) {
      if (lane == 0) {
        a.out[(size_t)b * a.ld_out] = -1;
        done = 1;
      }
    } else {
      const unsigned long long t = scale_word(x, S);
      const unsigned long long wk = res ? pk.res : pk.prob;
      unsigned long long incl = wk;
#pragma unroll
      for (int o = 1; o < kWave; o <<= 1) {
        const unsigned long long n = shfl_up_u64(incl, o);
        if (lane >= o) incl += n;
      }
      // the chunk whose share [incl - wk, incl) of the running sum holds t
      const unsigned long long hit = __ballot(t < incl && t >= incl - wk);
      const int csel = __ffsll(hit) - 1;
      if (lane == csel) {
        chunk_sel = csel;
        use_res = res;
        t_in_chunk = t - (incl - wk);
        done = 0;
      }
      if (hit == 0 && lane == 0) {  // (t < S: unreachable)
        a.out[(size_t)b * a.ld_out] = -1;
        done = 1;
      }
    }
  }
  __syncthreads();
  if (done) return;
  // scan the selected chunk: thread k owns 4 consecutive columns
  const int j0 = chunk_sel * cs, j1 = min(V, j0 + cs);
  unsigned long long mine[4], tot = 0;
  for (int base = j0; base < j1; base += 4 * kChunkThreads) {
    const int jj = base + 4 * threadIdx.x;
    float res[4], prob[4];
    weights_quad(a, st, b, jj, j1, res, prob);
#pragma unroll
    for (int e = 0; e < 4; ++e) mine[e] = fp_weight(use_res ? res[e] : prob[e]);
    const unsigned long long sum4 = mine[0] + mine[1] + mine[2] + mine[3];
    unsigned long long incl = sum4;
#pragma unroll
    for (int o = 1; o < kWave; o <<= 1) {
      const unsigned long long n = shfl_up_u64(incl, o);
      if (lane >= o) incl += n;
    }
    __syncthreads();
    if (lane == kWave - 1) wtot[w] = incl;
    __syncthreads();
    unsigned long long wbefore = 0, round_tot = 0;
    for (int k = 0; k < kChunkThreads / kWave; ++k) {
      if (k < w) wbefore += wtot[k];
      round_tot += wtot[k];
    }
    const unsigned long long t = t_in_chunk - tot;  // position inside this round
    unsigned long long cum = wbefore + incl - sum4;
    if (t < round_tot && cum <= t && t < cum + sum4) {
#pragma unroll
      for (int e = 0; e < 4; ++e) {
        cum += mine[e];
        if (cum > t) { a.out[(size_t)b * a.ld_out] = jj + e; break; }
      }
    }
    if (t < round_tot) break;  // uniform: every thread sees the same totals
    tot += round_tot;
  }
}

__global__ void copy_logits_kernel(const float* lg, int rps, int V, float* out) {
  const int b = blockIdx.y;
  const float* src = lg + ((size_t)b * rps + rps - 1) * V;
  for (int j = blockIdx.x * blockDim.x + threadIdx.x; j < V; j += gridDim.x * blockDim.x) out[(size_t)b * V + j] = src[j];
}

// ---------------------------------------------------------------- sampler / philox
__global__ __launch_bounds__(kSampThreads) void sample_kernel(int V, const float* probs, int64_t ld,
                                                              const uint32_t* rand, uint64_t seed, uint64_t step,
                                                              int purpose, int index, int32_t* out) {
  __shared__ SampShared sh;
  const int b = blockIdx.x;
  const float* row = probs + (size_t)b * ld;
  const uint32_t x = rand ? rand[b] : draw_word(seed, b, step, purpose, index);
  const int tok = block_draw([&](int j) { return row[j]; }, V, x, sh);
  if (threadIdx.x == 0) out[b] = tok;
}

__global__ void draw_kernel(int B, uint64_t seed, uint64_t step, int purpose, int index, uint32_t* out) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b < B) out[b] = draw_word(seed, b, step, purpose, index);
}

// ---------------------------------------------------------------- commit
__global__ void commit_kernel(CommitArgs a) {
  for (int b = threadIdx.x; b < a.B; b += blockDim.x) {
    const int A = a.n_accepted[b], g = a.gamma;
    if (A < 0 || A > g) continue;
    const int nxt = a.next_token[b];
    if (a.role == SPECDEC_ROLE_TARGET) {
      a.len[b] += A + 1;
      a.pending[2 * b] = 0;
      a.pending[2 * b + 1] = nxt;
      a.n_pending[b] = 1;
    } else {
      const int np = a.n_pending[b];
      a.len[b] += np + min(A, g - 1);
      if (A == g) {
        a.pending[2 * b] = a.d[(size_t)b * a.ld_d + g - 1];
        a.n_pending[b] = 2;
      } else {
        a.pending[2 * b] = 0;
        a.n_pending[b] = 1;
      }
      a.pending[2 * b + 1] = nxt;
    }
  }
  if (threadIdx.x == 0) *a.counter += 1;
}

}  // namespace

hipError_t launch_rows_embed(int dtype, const RowsArgs& a, hipStream_t s) {
  if (dtype == SPECDEC_BF16)
    hipLaunchKernelGGL((rows_embed_kernel<uint16_t>), dim3(a.M, 2), dim3(256), 0, s, a);
  else
    hipLaunchKernelGGL((rows_embed_kernel<float>), dim3(a.M, 2), dim3(256), 0, s, a);
  return hipGetLastError();
}

size_t sampling_scratch_bytes(int B, int rows, int V) {
  const int NC = n_chunks(V);
  return align256(sizeof(StatPart) * (size_t)B * rows * NC) + align256(sizeof(DrawPart) * (size_t)B * NC);
}

// Two launches: the chunk statistics, then decide-and-draw.
hipError_t launch_draft_finish(const DraftFinishArgs& a, hipStream_t s) {
  const int NC = n_chunks(a.V);
  if (a.logits_out) {
    hipLaunchKernelGGL(copy_logits_kernel, dim3((a.V + 255) / 256, a.B), dim3(256), 0, s, a.logits, a.rps, a.V,
                       a.logits_out);
  }
  Scratch sc = carve(a.scratch, a.B, 1, a.V);
  hipLaunchKernelGGL(stats_kernel, dim3(NC, a.B), dim3(kChunkThreads), 0, s, a.logits, a.V, 1, a.rps, a.rps - 1,
                     a.temperature, nullptr, 0, sc.stats);
  DrawArgs d{};
  d.mode = W_DRAFT;
  d.B = a.B;
  d.V = a.V;
  d.gamma = a.gamma;
  d.T = a.temperature;
  d.lg = a.logits;
  d.rps = a.rps;
  d.slot = a.slot;
  d.q_out = a.q_out;
  d.scratch = a.scratch;
  d.rows = 1;
  d.rand = a.rand;
  d.seed = a.seed;
  d.step = a.step;
  d.step_dev = a.step_dev;
  d.out = a.d_out + a.slot;
  d.ld_out = a.ld_d;
  d.status = a.status;
  hipLaunchKernelGGL(decide_draw_kernel, dim3(NC, a.B), dim3(kChunkThreads), 0, s, d);
  return hipGetLastError();
}

// ---------------------------------------------------------------- static scratch of the no-allocation accept
// Device scratch of specdec_accept_noalloc: a file-scope array each GPU the
// library runs on holds until the process ends.  In host code the array's name
// is not a device address; its address on the current device comes from
// hipGetSymbolAddress, looked up once per device (on that device's first call)
// and kept.  Every call on a GPU shares the array.
static __device__ __align__(256) unsigned char scratch[kStaticAcceptScratchBytes];

hipError_t static_accept_scratch(void** out) {
  constexpr int kMaxDevices = 64;
  static std::mutex mu;
  static void* ptr[kMaxDevices] = {};
  int dev = 0;
  hipError_t e = hipGetDevice(&dev);
  if (e != hipSuccess) return e;
  if (dev < 0 || dev >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(mu);
  if (!ptr[dev]) {
    void* p = nullptr;
    e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    ptr[dev] = p;
  }
  *out = ptr[dev];
  return hipSuccess;
}

// Two launches: the chunk statistics of every row, then decide-and-draw.
hipError_t launch_accept(const AcceptArgs& a, hipStream_t s) {
  if (a.gamma > kMaxGamma) return hipErrorInvalidValue;
  const int NC = n_chunks(a.V);
  Scratch sc = carve(a.scratch, a.B, a.gamma + 1, a.V);
  const bool logits = a.input_kind == SPECDEC_INPUT_LOGITS;
  hipLaunchKernelGGL(stats_kernel, dim3(NC, a.B * (a.gamma + 1)), dim3(kChunkThreads), 0, s, a.p, a.V, a.gamma + 1,
                     a.gamma + 1, 0, logits ? a.temperature : 0.f, a.temperature > 0.f ? a.q : nullptr, a.gamma,
                     sc.stats);
  DrawArgs d{};
  d.mode = W_ACCEPT;
  d.B = a.B;
  d.V = a.V;
  d.gamma = a.gamma;
  d.T = a.temperature;
  d.p = a.p;
  d.q = a.q;
  d.logits = logits;
  d.d = a.d;
  d.ld_d = a.ld_d;
  d.scratch = a.scratch;
  d.rows = a.gamma + 1;
  d.rand = a.rand;
  d.seed = a.seed;
  d.step = a.step;
  d.step_dev = a.step_dev;
  d.n_accepted = a.n_accepted;
  d.out = a.next_token;
  d.ld_out = 1;
  d.status = a.status;
  hipLaunchKernelGGL(decide_draw_kernel, dim3(NC, a.B), dim3(kChunkThreads), 0, s, d);
  return hipGetLastError();
}

hipError_t launch_sample(int B, int V, const float* probs, int64_t ld, const uint32_t* rand, uint64_t seed,
                         uint64_t step, int purpose, int index, int32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(sample_kernel, dim3(B), dim3(kSampThreads), 0, s, V, probs, ld, rand, seed, step, purpose,
                     index, out);
  return hipGetLastError();
}

hipError_t launch_draw(int B, uint64_t seed, uint64_t step, int purpose, int index, uint32_t* out, hipStream_t s) {
  hipLaunchKernelGGL(draw_kernel, dim3((B + 255) / 256), dim3(256), 0, s, B, seed, step, purpose, index, out);
  return hipGetLastError();
}

hipError_t launch_commit(const CommitArgs& a, hipStream_t s) {
  hipLaunchKernelGGL(commit_kernel, dim3(1), dim3(64), 0, s, a);
  return hipGetLastError();
}

}  // namespace specdec
