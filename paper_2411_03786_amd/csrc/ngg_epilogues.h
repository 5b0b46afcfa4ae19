// Device code that the GEMM kernels share: what becomes of a finished accumulator fragment, and the transfer to LDS.
#pragma once

#include "ngg_internal.h"

namespace ngg {

// ---------------------------------------------------------------------------------------------
// Epilogues, shared by the skinny, the streaming and the single-row kernel.  `sum` is one complete 16x16 accumulator
// fragment: this lane holds column (block row) m and fragment rows 4g .. 4g+3.
// ---------------------------------------------------------------------------------------------

// q/k/v and gate/up: the fragment's rows 0..7 are the first members of 8 output pairs, rows 8..15 the
// second members (rotary pairs (i, i + hd/2) of one head; gate and up of 8 FFN features).  rs: the row's
// 1 / rms times the operand scales.  The caller has checked frag < n_groups; lanes g >= 2 only lend values.
// v: the first members (fragment rows 4g .. 4g+3, g < 2), x2: their partners (rows 8 + 4g ..), both already scaled.
// act_mb: layout of the SwiGLU output; a constant 0 in the kernels whose output gemm_stream_kernel never reads (launch_gemm checks it)
template <typename T, int EPI>
__device__ __forceinline__ void epi_paired_vals(const GemmCore &a, int frag, int m, int M, int g, const float (&v)[4],
                                                const float (&x2)[4], int act_mb) {
  if (m < M && g < 2) {
    if constexpr (EPI == EPI_GATEUP) {
      float o[4];
#pragma unroll
      for (int r = 0; r < 4; ++r) o[r] = silu<T>(v[r]) * x2[r];
      store4((T *)a.act + act_pos<T>(m, frag * 8 + 4 * g, a.Mcap, act_mb), o[0], o[1], o[2], o[3]);   // 4 features lie side by side in either layout
    } else {
      const int half = a.hd / 2, fph = a.hd / 16;    // fragments per head
      const int hh = frag / fph, sub = frag - hh * fph;                 // head over [q heads | k heads | v heads]
      const int kind = hh < a.H ? 0 : (hh < a.H + a.Hkv ? 1 : 2);
      const int head = kind == 0 ? hh : (kind == 1 ? hh - a.H : hh - a.H - a.Hkv);
      const int i0 = sub * 8 + 4 * g;                // dims i0 .. i0+3 and their partners i0 + half ..
      if (kind < 2) {                                // rotary embedding on q and k
        const int pos = (a.n_dev ? *a.n_dev - 1 : a.P) + block_col(m, a.C, a.shared0);
        const float *cs = a.rope_cos + (size_t)pos * half + i0;
        const float *sn = a.rope_sin + (size_t)pos * half + i0;
        float lo[4], hi[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          lo[r] = v[r] * cs[r] - x2[r] * sn[r];
          hi[r] = x2[r] * cs[r] + v[r] * sn[r];
        }
        if (kind == 0) {
          T *dst = (T *)a.q + ((size_t)head * a.Mcap + m) * a.hd + i0;
          store4(dst, lo[0], lo[1], lo[2], lo[3]);
          store4(dst + half, hi[0], hi[1], hi[2], hi[3]);
        } else {                                     // keys: tiles of 32 block positions in operand order
          T *kh = (T *)a.kscr + (size_t)head * a.kv_rows * a.hd;
          store4(kh + k_offset(m, i0, a.hd, (int)sizeof(T)), lo[0], lo[1], lo[2], lo[3]);
          store4(kh + k_offset(m, i0 + half, a.hd, (int)sizeof(T)), hi[0], hi[1], hi[2], hi[3]);
        }
      } else {                                       // values: the transposed tiles
        T *vh = (T *)a.vscr + (size_t)head * a.kv_rows * a.hd;
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          vh[v_offset(m, i0 + r, a.hd, (int)sizeof(T))] = from_f32<T>(v[r]);
          vh[v_offset(m, i0 + half + r, a.hd, (int)sizeof(T))] = from_f32<T>(x2[r]);
        }
      }
    }
  }
}

template <typename T, int EPI>
__device__ __forceinline__ void epi_paired(const GemmCore &a, int frag, int m, int M, int g, float rs, const f32x4 &sum, int act_mb = 0) {
  float v[4], x2[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) { v[r] = sum[r] * rs; x2[r] = other_half(v[r]); }
  epi_paired_vals<T, EPI>(a, frag, m, M, g, v, x2, act_mb);
}

// residual: split ks stores its fp32 partial of output features n0 + 4g .. +4 of block row m
__device__ __forceinline__ void epi_residual(const GemmCore &a, int ks, int m, int n0, int g, const f32x4 &sum) {
  float *dst = a.hpart + ((size_t)ks * a.Mcap + m) * a.N;
  *reinterpret_cast<float4 *>(dst + n0 + 4 * g) =
      float4{sum[0] * a.out_scale, sum[1] * a.out_scale, sum[2] * a.out_scale, sum[3] * a.out_scale};
}

// unembedding: optional logits, and the best (value, id) of block row m over the FN fragments of `group`
// (vocabulary rows nbase[f] ..): ascending ids, so the first maximum stays
template <int FN>
__device__ __forceinline__ void epi_unembed(const GemmCore &a, int group, int m, bool live, int g, float rs,
                                            const int (&nbase)[FN], const f32x4 (&sum)[FN]) {
  float bv = kNegBig;
  int bi = 0x7fffffff;
#pragma unroll
  for (int f = 0; f < FN; ++f)
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const float v = sum[f][r] * rs;
      const int n = nbase[f] + 4 * g + r;
      if (a.logits && live) a.logits[(size_t)m * a.N + n] = v;
      if (v > bv) { bv = v; bi = n; }
    }
#pragma unroll
  for (int off = 16; off < 64; off <<= 1) {
    const float ov = __shfl_xor(bv, off);
    const int oi = __shfl_xor(bi, off);
    if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
  }
  if (live && g == 0) {
    a.pmax_val[(size_t)group * a.Mcap + m] = bv;
    a.pmax_idx[(size_t)group * a.Mcap + m] = bi;
  }
}

// 16 bytes per lane from global memory (uniform base + lane offset) to LDS (lane i: lds + 16 i).  The compiler does not
// see the transfer: the kernel waits for it with its own s_waitcnt before a barrier.  NT: the lines are used once
// (weights that only one workgroup reads), keep them out of the activations' way in the L2.
template <bool NT>
__device__ __forceinline__ void lds_dma16(const void *base, unsigned off, unsigned lds) {
  if constexpr (NT)
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2 nt" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
  else
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds), "v"(off), "s"(base) : "m0", "memory");
}

}  // namespace ngg
