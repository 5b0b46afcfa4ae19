// Streaming GEMM  Y[M x N] = X[M x K] . W[N x K]^T  for blocks of up to 64 rows (q/k/v and gate/up: 128): a verify call is meant to
// stay bound by the one read of W (Section 3), and what a launch costs beyond that read is its start, its barriers and its finish.
//
// A workgroup owns FN fragments (16 rows) of W and all block rows; its NW waves split the steps of 32 contraction elements
// among them, so every element of W and of X is needed by exactly one wave.  Both operands lie in memory in the order the
// matrix instruction takes them (1 KB blocks, act_pos), go from there straight into registers through one ring RING steps
// deep, and the main loop has no LDS and no barrier.  The waves' sums meet in LDS at the end, in the order of the waves.
//
// The RMSNorm in front of a GEMM costs nothing but its row factor here: X holds h * gain, and the sums of squares that the
// producer left per row come by DMA in front of the first operands, are added up while those are on their way, and multiply
// the accumulators in the epilogue.  The RMSNorm behind a residual GEMM is its epilogue: a workgroup takes the whole
// contraction of its output features for all rows, adds the residual stream, writes h and h * gain and leaves one sum of
// squares per row and 16 features.
#include "ngg_epilogues.h"

#include <algorithm>

namespace ngg {

// storage type of the user's weights behind an internal type
template <typename T> struct Stored;
template <> struct Stored<float> { typedef float type; };
template <> struct Stored<half_t> { typedef bf16_t type; };

// column blocks handed over per round: what the LDS holds, and little enough for two workgroups of the unembedding per CU
template <int EPI, int FM, int FN, int NW> constexpr int stream_round() {
  const int most = EPI == EPI_UNEMBED ? 64 / (NW * FN) : 144 / (NW * FN);
  return most < 1 ? 1 : (most < FM ? most : FM);
}

template <typename T, int EPI, int FM, int FN, int NW, int RING>
__global__ __launch_bounds__(64 * NW) void gemm_stream_kernel(const GemmArgs a) {
  constexpr bool PAIRED = EPI == EPI_QKV || EPI == EPI_GATEUP;
  static_assert(EPI != EPI_UNEMBED || FN % 2 == 0, "the unembedding's partial maxima cover two fragments");
  constexpr int LPF = (int)sizeof(T) / 2;                // load instructions per fragment
  constexpr int IN_RING = RING * (FN + FM) * LPF;
  static_assert(IN_RING <= 63, "vmcnt counts to 63");
  constexpr int FMR = stream_round<EPI, FM, FN, NW>(), ROUNDS = (FM + FMR - 1) / FMR;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  __shared__ float rs[16 * FM];                          // 1 / rms of the rows times the operand scales
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int K = a.K, M = a.M, n_steps = K / 32, n_frags = a.n_groups, mb = a.x_mb;
  const int f0 = blockIdx.x * FN;

  // ---- sums of squares of all rows -> LDS, ahead of everything else ---------------------------------
  if constexpr (EPI != EPI_RESIDUAL) {
    if (a.row_ss) {
      const int n = (M * a.ss_segs + 255) / 256;         // 1 KB each; the buffer is padded to whole ones
      const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
      for (int i = wave; i < n; i += NW) lds_dma16<false>(a.row_ss + i * 256, lane * 16, lds0 + i * 1024);
    }
  }

  // ---- operands: uniform bases plus one lane offset per column block --------------------------------
  const T *wbase[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) wbase[f] = (const T *)a.W0 + (size_t)min(f0 + f, n_frags - 1) * n_steps * 512;   // surplus ones repeat the last
  const unsigned wlane = lane * (16 / (unsigned)sizeof(T));
  unsigned xlane[FM];                                    // rows past the block's last one repeat it: no cache lines of their own
#pragma unroll
  for (int fm = 0; fm < FM; ++fm) {
    const int b = min(fm, mb - 1);
    xlane[fm] = (unsigned)(b * 512 + (g * 16 + min(li, M - 1 - b * 16)) * (16 / (int)sizeof(T)));
  }
  Frag<T> wr[RING][FN], xr[RING][FM];
  auto load = [&](int slot, int t) {                     // t-th step of this wave, clamped into the matrix
    const int st = min(wave + NW * t, n_steps - 1);
    const T *xs = (const T *)a.X + (size_t)st * mb * 512;
#pragma unroll
    for (int f = 0; f < FN; ++f) wr[slot][f] = load_frag_stream(wbase[f] + (size_t)st * 512 + wlane);
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) xr[slot][fm] = load_frag_tiled(xs + xlane[fm]);
  };
  f32x4 acc[FN][FM];
#pragma unroll
  for (int f = 0; f < FN; ++f)
#pragma unroll
    for (int fm = 0; fm < FM; ++fm) acc[f][fm] = f32x4{0.f, 0.f, 0.f, 0.f};
  auto mul = [&](int slot) {
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) mma(acc[f][fm], wr[slot][f], xr[slot][fm]);
  };
  const int nt = n_steps > wave ? (n_steps - wave + NW - 1) / NW : 0;
  __builtin_amdgcn_sched_barrier(0);
#pragma unroll
  for (int u = 0; u < RING; ++u) load(u, u);
  __builtin_amdgcn_sched_barrier(0);

  if constexpr (EPI != EPI_RESIDUAL) {
    if (a.row_ss) {
      // the sums were requested first: they have landed once no more than the ring is outstanding
      asm volatile("s_waitcnt vmcnt(%0)" ::"n"(IN_RING) : "memory");
      __builtin_amdgcn_s_barrier();
      // four lanes per row; the 16 rows a wave reads at once start 16 bytes apart, on banks of their own
      const int n4 = a.ss_segs / 4;
      for (int e = tid; e < 64 * FM; e += 64 * NW) {
        const int r = e >> 2, row = min(r, M - 1);
        const f32x4 *src = reinterpret_cast<const f32x4 *>(smem) + (size_t)row * n4;
        const int first = row % n4;
        float t = 0.0f;
        for (int i = e & 3; i < n4; i += 4) {
          const int j = first + i < n4 ? first + i : first + i - n4;
          const f32x4 v = src[j];
          t += (v[0] + v[1]) + (v[2] + v[3]);
        }
        t += __shfl_xor(t, 1);
        t += __shfl_xor(t, 2);
        if ((e & 3) == 0) rs[r] = a.out_scale / sqrtf(t / (float)K + a.ss_eps);
      }
    } else {
      for (int r = tid; r < 16 * FM; r += 64 * NW) rs[r] = a.out_scale;
    }
  }

  // ---- the stream: groups of RING steps; the last two refill only what is still there ---------------
  // Every refill stays behind its own slot's products: left alone the compiler moves the group's products together, which
  // waits for the whole ring before the first refill.  (us so -> pinned: fp32 4096 wide at 33 rows q/k/v 80.5 -> 65.3, gate/up 124 ->
  // 98; 16-bit 5120 wide at 49 rows 34.6 -> 33.4 and 51.4 -> 50.5, 4096 wide at 51 24.8 -> 24.4 and 43.1 -> 43.0.)  Not where one step
  // is in flight (gate/up of 113 rows, 6144 wide 166.9 -> 168.7; fp32 unembedding 117 -> 144), and not in the unembedding, whose
  // two workgroups per CU fill each other's gaps (4096 wide at 51 rows 49.6 -> 51.0).
  constexpr bool PIN = RING > 1 && EPI != EPI_UNEMBED;
  int t0 = 0;
  for (; t0 + 2 * RING <= nt; t0 += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      mul(u);
      load(u, t0 + u + RING);
      if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
    }
  }
#pragma unroll
  for (int u = 0; u < RING; ++u) {
    if (t0 + u < nt) mul(u);                             // (uniform)
    if (t0 + u + RING < nt) load(u, t0 + u + RING);
    if constexpr (PIN) __builtin_amdgcn_sched_barrier(0);
  }
#pragma unroll
  for (int u = 0; u < RING; ++u)
    if (t0 + u + RING < nt) mul(u);

  // ---- hand-over: wave w sums items w, w + NW, ... of the accumulator fragments, waves in order ------
  f32x4 *red = reinterpret_cast<f32x4 *>(smem);          // [NW][FN * cnt][64]
#pragma unroll
  for (int rd = 0; rd < ROUNDS; ++rd) {
    const int cnt = (rd + 1) * FMR <= FM ? FMR : FM - rd * FMR;   // column blocks of this round (constant after unrolling)
    const int items = FN * cnt;                          // item f * cnt + fr covers column block rd * FMR + fr
    f32x4 hv = f32x4{0.f, 0.f, 0.f, 0.f}, gain = hv;
    if constexpr (EPI == EPI_RESIDUAL) {                 // what the first item needs, on its way during the hand-over
      if (a.h && wave < items) {
        const int f = wave / cnt, m = (rd * FMR + wave - f * cnt) * 16 + li, n = min(f0 + f, n_frags - 1) * 16 + 4 * g;
        hv = *reinterpret_cast<const f32x4 *>(a.h + (size_t)min(m, M - 1) * a.N + n);
        const typename Stored<T>::type *gp = (const typename Stored<T>::type *)a.gain + n;
        gain = f32x4{to_f32(gp[0]), to_f32(gp[1]), to_f32(gp[2]), to_f32(gp[3])};
      }
    }
    __syncthreads();                                     // everyone is done with the sums of squares, or the last round's items
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
      for (int fr = 0; fr < FMR; ++fr)
        if (fr < cnt) red[((size_t)wave * items + f * cnt + fr) * 64 + lane] = acc[f][rd * FMR + (fr < cnt ? fr : 0)];
    __syncthreads();
    auto total = [&](int idx) {
      f32x4 t = red[(size_t)idx * 64 + lane];
#pragma unroll
      for (int o = 1; o < NW; ++o) t += red[((size_t)o * items + idx) * 64 + lane];
      return t;
    };
    if constexpr (PAIRED) {
      constexpr int IPW = (FN * FMR + NW - 1) / NW;
      // (unrolled where the items are short or few: eight q/k/v items at once do not fit the registers)
      constexpr int UNR = (EPI == EPI_GATEUP || IPW <= 3) ? IPW : 1;
#pragma unroll UNR
      for (int j = 0; j < IPW; ++j) {
        const int idx = wave + NW * j;
        if (idx >= items) break;
        const int f = idx / cnt, fm = rd * FMR + idx - f * cnt;
        if (f0 + f < n_frags) epi_paired<T, EPI>(a, f0 + f, fm * 16 + li, M, g, rs[fm * 16 + li], total(idx), a.act_mb);   // (uniform)
      }
    } else if constexpr (EPI == EPI_UNEMBED) {
      for (int it = wave; it < items / 2; it += NW) {    // pairs of fragments
        const int p = it / cnt, fr = it - p * cnt, m = (rd * FMR + fr) * 16 + li;
        if (f0 + 2 * p >= n_frags) break;
        const int nbase[2] = {(f0 + 2 * p) * 16, (f0 + 2 * p + 1) * 16};
        const f32x4 sums[2] = {total(2 * p * cnt + fr), total((2 * p + 1) * cnt + fr)};
        epi_unembed<2>(a, (f0 + 2 * p) / 2, m, m < M, g, rs[(rd * FMR + fr) * 16 + li], nbase, sums);
      }
    } else {
      for (int idx = wave; idx < items; idx += NW) {
        const int f = idx / cnt, m = (rd * FMR + idx - f * cnt) * 16 + li, frag = f0 + f;
        if (frag >= n_frags) break;
        const f32x4 sum = total(idx);
        if (!a.h) {
          if (m < M) epi_residual(a, 0, m, frag * 16, g, sum);
          continue;
        }
        const int n = frag * 16 + 4 * g;
        if (idx != wave) {
          hv = *reinterpret_cast<const f32x4 *>(a.h + (size_t)min(m, M - 1) * a.N + n);
          const typename Stored<T>::type *gp = (const typename Stored<T>::type *)a.gain + n;
          gain = f32x4{to_f32(gp[0]), to_f32(gp[1]), to_f32(gp[2]), to_f32(gp[3])};
        }
        const f32x4 x = hv + sum * a.out_scale;
        if (m < M) {
          *reinterpret_cast<f32x4 *>(a.h + (size_t)m * a.N + n) = x;
          store4((T *)a.xn + act_pos<T>(m, n, a.Mcap, a.xn_mb), x[0] * gain[0], x[1] * gain[1], x[2] * gain[2], x[3] * gain[3]);
        }
        const float q = rows_sum((x[0] * x[0] + x[1] * x[1]) + (x[2] * x[2] + x[3] * x[3]));
        const int segs = (a.N / 16 + 3) / 4 * 4;
        if (m < M && g == 0) a.ss_out[(size_t)m * segs + frag] = q;
        if (m < M && g > 0 && frag == n_frags - 1 && frag + g < segs) a.ss_out[(size_t)m * segs + frag + g] = 0.0f;   // read in fours
      }
    }
  }
}

// Steps in flight per wave (16-bit fragments; fp32 ones are twice as large)
template <typename T, int EPI> constexpr int stream_ring(int fm, int fn) {
  if (EPI == EPI_RESIDUAL) return sizeof(T) == 2 ? 6 : 3;
  if (EPI == EPI_UNEMBED) return sizeof(T) == 2 ? (fn == 8 || fm == 4 ? 2 : 3) : 2;
  if (sizeof(T) == 4) return 2;
  if (fm > 4) return fn <= 4 ? (fm == 8 ? (fn == 3 ? 2 : 1) : (fn == 3 ? 3 : 2)) : (fn * fm == 64 ? 1 : 2);
  return fn == 1 ? 3 : (fn == 2 ? 2 : (fn <= 4 ? 4 : (fn * fm <= 28 ? 2 : 1)));   // (2 at 8 x 4 fragments spills)
}

template <typename T, int EPI, int FM, int FN, int NW, int RING = stream_ring<T, EPI>(FM, FN)>
static void launch_stream_cfg(const GemmArgs &a, hipStream_t s) {
  size_t lds = (size_t)NW * FN * stream_round<EPI, FM, FN, NW>() * 1024;
  if (EPI != EPI_RESIDUAL && a.row_ss) lds = std::max(lds, ((size_t)a.M * a.ss_segs * 4 + 1023) / 1024 * 1024);
  static const hipError_t opted = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_stream_kernel<T, EPI, FM, FN, NW, RING>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, 159 * 1024);
  (void)opted;
  hipLaunchKernelGGL((gemm_stream_kernel<T, EPI, FM, FN, NW, RING>), dim3((a.n_groups + FN - 1) / FN), dim3(64 * NW), lds, s, a);
}

// Fragments per workgroup of the 16-bit q/k/v and gate/up: as many as spread the matrix over the 256 CUs in one round, or, above the
// 2048 fragments that eight per workgroup hold, in equal rounds (one workgroup is on a CU: its LDS).  Eight whatever the number left
// the last round partly filled: gate/up 7168 x 20480 (2560 fragments, five instead of eight) at 49 / 121 rows 127 -> 102 / 193 -> 142 us,
// 8192 x 22016 (2752, six) 149 -> 130 / 217 -> 170, 8192 x 28672 (3584, seven) 163 -> 155 / 231 -> 196, 12288 x 36864 (4608, six) 337 -> 296 / 482 -> 383
int stream_paired_frags(int frags) {
  const int rounds = (frags + 2047) / 2048;
  return (frags + 256 * rounds - 1) / (256 * rounds);
}

template <typename T, int EPI, int FM>
static void launch_stream_fm(const GemmArgs &a, hipStream_t s) {
  const bool paired = sizeof(T) == 2 && (EPI == EPI_QKV || EPI == EPI_GATEUP);
  const int fn = paired ? stream_paired_frags(a.n_groups) : (a.n_groups + 255) / 256;
  if constexpr (EPI == EPI_RESIDUAL) launch_stream_cfg<T, EPI, FM, 1, 4>(a, s);
  else if constexpr (EPI == EPI_UNEMBED) {
    if constexpr (sizeof(T) == 2) {
      // (two workgroups of four fragments per CU; contractions from 4096 on take eight, which read X half as often: 5120 wide,
      // 64 rows 64.7 -> 56.3 us, 4096 wide 48.2 -> 47.2, 3072 wide 134 against 137)
      if (fn > 4 && a.K >= 4096) launch_stream_cfg<T, EPI, FM, 8, 4>(a, s);
      else if (fn > 2) launch_stream_cfg<T, EPI, FM, 4, 4>(a, s);
      else launch_stream_cfg<T, EPI, FM, 2, 4>(a, s);
    } else {
      if (fn > 4) launch_stream_cfg<T, EPI, FM, 2, 8, 1>(a, s);   // (2048 wide, 32000 entries, 33 rows: 83 -> 63 us)
      else launch_stream_cfg<T, EPI, FM, 2, 4>(a, s);
    }
  } else if constexpr (sizeof(T) == 4) {
    if (fn <= 1) launch_stream_cfg<T, EPI, FM, 1, 4>(a, s);
    else launch_stream_cfg<T, EPI, FM, 2, 4>(a, s);
  } else if constexpr (FM > 4) {                            // (wide matrices only: stream_takes)
    switch (fn) {
      case 3: launch_stream_cfg<T, EPI, FM, 3, 8>(a, s); break;
      case 4: launch_stream_cfg<T, EPI, FM, 4, 8>(a, s); break;
      case 5: launch_stream_cfg<T, EPI, FM, 5, 4>(a, s); break;
      case 6: launch_stream_cfg<T, EPI, FM, 6, 4>(a, s); break;
      case 7: launch_stream_cfg<T, EPI, FM, 7, 4>(a, s); break;
      default: launch_stream_cfg<T, EPI, FM, 8, 4>(a, s);
    }
  } else {
    switch (fn) {
      case 1: launch_stream_cfg<T, EPI, FM, 1, 4>(a, s); break;
      case 2: launch_stream_cfg<T, EPI, FM, 2, 8>(a, s); break;
      case 3: launch_stream_cfg<T, EPI, FM, 3, 8>(a, s); break;
      case 4: launch_stream_cfg<T, EPI, FM, 4, 8>(a, s); break;
      case 5: launch_stream_cfg<T, EPI, FM, 5, 8>(a, s); break;
      case 6: launch_stream_cfg<T, EPI, FM, 6, 8>(a, s); break;
      case 7: launch_stream_cfg<T, EPI, FM, 7, 8>(a, s); break;
      default: launch_stream_cfg<T, EPI, FM, 8, 8>(a, s);
    }
  }
}

// column blocks (of 16 rows) an instance is built for
static constexpr int stream_blocks(int dtype, int epi) { return dtype == 1 && (epi == EPI_QKV || epi == EPI_GATEUP) ? 8 : 4; }
bool stream_built(int dtype, int epi, int M) { return (M + 15) / 16 <= stream_blocks(dtype, epi); }

template <typename T, int EPI>
static bool launch_stream_epi(const GemmArgs &a, hipStream_t s) {
  switch ((a.M + 15) / 16) {
    case 1: launch_stream_fm<T, EPI, 1>(a, s); return true;
    case 2: launch_stream_fm<T, EPI, 2>(a, s); return true;
    case 3: launch_stream_fm<T, EPI, 3>(a, s); return true;
    case 4: launch_stream_fm<T, EPI, 4>(a, s); return true;
    default: break;
  }
  if constexpr (stream_blocks(sizeof(T) == 2 ? 1 : 0, EPI) == 8) {
    switch ((a.M + 15) / 16) {
      case 5: launch_stream_fm<T, EPI, 5>(a, s); return true;
      case 6: launch_stream_fm<T, EPI, 6>(a, s); return true;
      case 7: launch_stream_fm<T, EPI, 7>(a, s); return true;
      case 8: launch_stream_fm<T, EPI, 8>(a, s); return true;
      default: break;
    }
  }
  return false;
}

template <typename T>
static bool launch_stream_t(int epi, const GemmArgs &a_in, hipStream_t s) {
  GemmArgs a = a_in;
  a.n_groups = epi == EPI_GATEUP ? a.N / 8 : a.N / 16;
  switch (epi) {
    case EPI_QKV: return launch_stream_epi<T, EPI_QKV>(a, s);
    case EPI_GATEUP: return launch_stream_epi<T, EPI_GATEUP>(a, s);
    case EPI_RESIDUAL: return launch_stream_epi<T, EPI_RESIDUAL>(a, s);
    default: return launch_stream_epi<T, EPI_UNEMBED>(a, s);
  }
}

// Which GEMMs of a block run here.  Up to 64 rows, q/k/v, gate/up and the unembedding: all.  Measured against the kernels
// that stage X through LDS, back to back (from 5120 wide and fp32 from 1024: in the call), us at 2 / 17 / 33 / 51 rows:
//   q/k/v    768 wide 5.0 -> 3.9 / 5.6 -> 4.1 / 6.1 -> 4.6 / 6.7 -> 5.3, 2048 7.6 -> 7.0 / 8.1 -> 7.8 / 10.0 -> 8.9 / 11.0 -> 10.0,
//            3072 12.8 -> 11.4 / 13.6 -> 12.7 / 15.5 -> 14.7 / 16.7 -> 16.3, 4096 18.5 -> 17.4 / 19.5 -> 17.9 / 21.4 -> 19.9 / 22.6 -> 21.7
//   gate/up  768 wide 5.0 -> 4.4 / 5.4 -> 4.7 / 6.4 -> 5.2 / 7.1 -> 5.7, 4096 39.6 -> 37.4 / 39.9 -> 37.9 / 41.3 -> 40.2 / 42.5 -> 40.9;
//            3072 wide at 51 rows 19.2 (64 x 64 tiles) against 19.9 here, what q/k/v and the norm give back
//   5120     q/k/v 30.8 -> 29.8 / 31.6 -> 28.6 / 32.3 -> 31.1 / 33.5 -> 33.3, gate/up 49.3 -> 48.3 / 49.3 -> 46.3 / 50.3 -> 48.3 / 51.3 -> 50.5
//   6144     42.4 -> 41.0 / 43.1 -> 41.2 / 43.5 -> 42.0 / 46.5 -> 44.6, 68.5 -> 66.1 / 69.3 -> 66.7 / 68.7 -> 65.6 / 70.1 -> 68.4
//   8192     gate/up of 28672 features 153 -> 146 / 152 -> 143 / 154 -> 147 / 161 -> 154
//   fp32     512 wide q/k/v 5.1 -> 4.1 / 6.5 -> 4.8 / 7.8 -> 5.9 / 9.0 -> 7.0, 1024 10.7 -> 8.9 / 12.1 -> 8.9 / 14.2 -> 10.1 / 16.4 -> 11.3, 4096 44 -> 41 /
//            57 -> 49 / 83 -> 66 / 104 -> 85, its gate/up 67 -> 60 / 83 -> 72 / 112 -> 98 / 154 -> 124
// It loses where long contractions leave CUs idle at 33 rows or more: q/k/v of 576 fragments (192 workgroups), 7168 wide, 30.0 -> 26.5 /
// 28.6 -> 27.9 / 31.5 -> 32.4 / 34.8 -> 36.8, 35.2 -> 38.7 at 64 rows (whole calls 0.94 / 0.97 / 0.99 / 1.00 and 1.01 of their time).
// From 65 to 128 rows q/k/v and gate/up of 16-bit models of more than 512 fragments, at 65 / 81 / 97 / 121 rows: 4096 wide q/k/v
// 27.0 -> 24.9 / 30.1 -> 27.4 / 32.6 -> 30.5 / 34.4 -> 32.9, gate/up 44.4 -> 44.0 / 46.3 and 46.7 / 53.6 -> 50.6 / 61.5 -> 53.5; 3072 wide
// q/k/v 21.1 -> 18.9 / 23.0 -> 20.7 / 25.6 -> 23.6 / 27.3 -> 25.4.  Narrower ones run 128-row tiles there (768 wide gate/up 7.2 at
// 97 rows, 7.7 here); the unembedding stays on the skinny kernel too (128256 entries, 97 rows: 145, 161 here).
// Residual GEMMs: a workgroup reads all of X here, and the launch of the RMSNorm (4 to 5 us) is saved.  Output projection
// and norm 768 wide 7.1 -> 3.2 / 8.3 -> 3.8 / 7.4 -> 4.2 / 7.5 -> 4.6, 4096 11.7 -> 8.5 / 11.8 -> 9.2 / 12.6 -> 11.0 / 13.3 -> 12.5; down
// and norm 768 wide 7.5 -> 5.6 / 8.2 -> 6.6 / 8.6 -> 8.0 / 8.8 and 9.2, 4096 23.4 -> 20.4 / 24.1 and 24.8 / 25.2 and 30.9.  The line:
// the kilobytes a workgroup pulls (its 16 rows of W, and X as if a partly filled column block counted half) against the
// bytes of W, which the splitting kernels stream in that time too (768 x 3072, 4.7 MB: equal at 400 KB; 2048 x 5504, 22 MB:
// at 460; 3072 x 8192, 50 MB: at 680; 4096 x 14336, 117 MB: at 1100; from there on the splitting kernels stream faster: 8192 x 14336,
// 235 MB: at 1600; 7168 x 16384 loses 5 of 47 us at 1820; 8192 x 28672, 470 MB: 4 us faster at 2800, 6 slower at 3190).  More than one
// workgroup per CU share its path to the L2.  fp32 a fifth further: with its norm (4.4) down 512 x 1408 at 17 / 33 / 64 rows 14.7 -> 9.1 /
// 16.9 -> 10.6 / 19.4 -> 12.6, 768 x 3072 at 25 15.8 -> 13.9, 1024 x 4096 at 9 14.5 and 14.4, 4096 x 11008 at 9 and 17 41.4 -> 35.6 and 40.2 -> 39.8,
// the projection 4096 wide at 17 / 41 rows 26.8 -> 18.4 / 31.8 -> 27.5.
bool stream_takes(int dtype, int epi, int M, int frags, int K, int tile_only) {
  if (dtype == 1 && tile_only && M > 1) return false;
  if (M > 64) return dtype == 1 && M <= 128 && (epi == EPI_QKV || epi == EPI_GATEUP) && frags > 512;
  if (epi != EPI_RESIDUAL) return true;
  if (frags > 512 || K <= 64) return false;               // (the sums of squares of 64 rows fit the LDS of the next GEMM)
  const int e = dtype == 1 ? 2 : 4, fm = (M + 15) / 16;
  const float kb = (0.5f * ((float)fm + (float)M / 16.0f) + 1.0f) * (float)(K / 32) * (float)(e / 2) * (float)((frags + 255) / 256);
  const float mb_w = (float)frags * 16.0f * (float)K * (float)e / 1.0e6f;
  const float limit = std::min(390.0f + 6.2f * mb_w, 600.0f + 5.0f * mb_w);
  return kb <= (dtype == 1 ? limit : 1.2f * limit);
}

bool launch_gemm_stream(int dtype, int epi, const GemmArgs &a, hipStream_t s) {
  return dtype == 1 ? launch_stream_t<half_t>(epi, a, s) : launch_stream_t<float>(epi, a, s);
}

}  // namespace ngg
