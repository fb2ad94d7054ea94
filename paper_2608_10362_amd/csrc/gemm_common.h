// Device pieces shared by the GEMM and attention kernel files.
#pragma once

#include "device_common.h"
#include "internal.h"

namespace specdec {

namespace {

__device__ __forceinline__ float silu_f(float z) { return z / (1.0f + expf(-z)); }

// Raw buffer descriptor over `bytes` bytes at `base` (dword 3: the gfx9 raw
// buffer format); loads past `bytes` return zeros.
constexpr uint32_t kOutOfRange = 0x80000000u;
constexpr int kNonTemporal = 2;  // cache-policy bit of a streamed (read-once) load
__device__ __forceinline__ __amdgpu_buffer_rsrc_t make_rsrc(const void* base, uint32_t bytes) {
  return __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(base), (short)0, (int)bytes, 0x00020000);
}

// Waits until at most N of this wave's vector-memory loads are outstanding.
template <int N> __device__ __forceinline__ void wait_vm() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }

// 16 bytes per lane from rsrc at `off` into LDS at dst + 16 * lane, without
// passing the registers.  (Inline asm, so that the compiler does not wait for
// every such load before each LDS read: the kernel counts them itself.  The
// load takes its LDS address from M0, which needs one wait state after a
// scalar write, and the compiler adds none inside an asm block: the s_nop.)
__device__ __forceinline__ void load_lds16(uint32_t dst, uint32_t off, __amdgpu_buffer_rsrc_t rsrc) {
  asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tbuffer_load_dwordx4 %1, %2, 0 offen lds" ::"s"(dst), "v"(off), "s"(rsrc)
               : "memory", "m0");
}

// Segment and local row of row tile t (t < NC/16) of block blk.  A SwiGLU block
// pairs NC/2 gate rows (segment 0) with the up rows of the same columns (1).
__device__ __forceinline__ void tile_segment(const GemmArgs& a, int kind, int blk, int NC, int t, int& seg, int& n,
                                             bool& ok) {
  if (kind == EPI_SWIGLU) {
    const int H = NC / 2;
    seg = 16 * t >= H;
    n = blk * H + 16 * t - seg * H;
    ok = n < a.n_rows;
    if (!ok) n = 0;
  } else {
    n = blk * NC + 16 * t;
    ok = n < a.n_rows;
    if (!ok) n = 0;
    const int b1 = a.n_seg[0], b2 = b1 + a.n_seg[1];
    seg = n < b1 ? 0 : (n < b2 ? 1 : 2);
    n -= seg == 0 ? 0 : (seg == 1 ? b1 : b2);
  }
}
// Base of that tile in the packed bf16 image: sequences of 16-row tiles of
// ceil(K/32) 1 KB fragments.
__device__ __forceinline__ const uint16_t* weight_tile(const GemmArgs& a, int kind, int blk, int NC, int t,
                                                       int KS, bool& ok) {
  int seg, n;
  tile_segment(a, kind, blk, NC, t, seg, n, ok);
  return (const uint16_t*)a.w[seg] + (size_t)(n / 16) * KS * 512;
}

// Four consecutive columns n .. n+3 (n % 4 == 0) of row m of the Q|K|V
// projections, scaled: RoPE on the Q and K columns, then the stores: rotated
// queries to qr, rotated keys and the values into the KV cache at the row's
// position (valid rows).  z: the columns' rotation partners (column ^ 8).  Q
// and K columns come in the packed RoPE order: column c of a head's 16-column
// tile tq is dim 8 tq + c for c < 8, hd/2 + 8 tq + c - 8 otherwise; x1' = x1
// cos - x2 sin, x2' = x2 cos + x1 sin.  The four columns are four consecutive
// dims of one head, which the query row and the K fragment hold side by side.
__device__ __forceinline__ void qkv_store4(const GemmArgs& a, int m, int n, f32x4 y, f32x4 z) {
  const int H = a.n_heads, hd = a.head_dim, half = hd >> 1, cap = a.kv.capacity;
  const int nq = a.n_seg[0], nqk = nq + a.n_seg[1];
  const RowDesc rd = a.rows[m];
  if (n >= nqk) {  // values: natural order
    if (!rd.valid) return;
    const int r = n - nqk, head = r / hd, w = r % hd;
    uint16_t* kvb = k_block<uint16_t>(a.kv, a.layer, rd.b, head);
#pragma unroll
    for (int e = 0; e < 4; ++e) Storage<uint16_t>::store(kvb + KvIndex<uint16_t>::v(rd.pos, w + e, hd, cap), y[e]);
    return;
  }
  const bool is_q = n < nq;
  const int r = n - (is_q ? 0 : nq), head = r / hd, w = r % hd, ec = w & 15, j = 8 * (w >> 4) + (ec & 7);
  const float* cs = a.rope_cs + (size_t)m * hd + j;
  const f32x4 c = *(const f32x4*)cs, sn = *(const f32x4*)(cs + half);
  f32x4 o;
#pragma unroll
  for (int e = 0; e < 4; ++e) o[e] = ec < 8 ? y[e] * c[e] - z[e] * sn[e] : y[e] * c[e] + z[e] * sn[e];
  const int d = ec < 8 ? j : half + j;
  if (is_q) {
    *(f32x4*)(a.qr + ((size_t)m * H + head) * hd + d) = o;
  } else if (rd.valid) {
    uint16_t* kvb = k_block<uint16_t>(a.kv, a.layer, rd.b, head);
    *(u16x4*)(kvb + KvIndex<uint16_t>::k(rd.pos, d, hd, cap)) =
        u16x4{f32_to_bf16_bits(o[0]), f32_to_bf16_bits(o[1]), f32_to_bf16_bits(o[2]), f32_to_bf16_bits(o[3])};
  }
}

}  // namespace

}  // namespace specdec
