// Skinny GEMM  Y[M x N] = X[M x K] . W[N x K]^T  for the k*(w+1) block rows of a verify call
// (Section 3: a model call on a (k, w+1) block is meant to stay memory-bound, so the kernel is
// built around streaming W exactly once at HBM speed): every fp32 block above 64 rows, the 16-bit unembedding of 65 to 128, and the
// residual GEMMs of smaller blocks that gemm_stream_kernel (ngg_stream.hip) and gemm_tile_kernel leave.
//
// W rows are the MFMA "row" operand.  The library keeps its own copy of every weight matrix in
// operand order (16 rows x 32 contraction elements per 1 KB block, lane-major), so one load
// instruction of a wave reads 1 KB of contiguous memory, a wave streams one contiguous region, and
// the data goes from global memory straight into MFMA registers (non-temporal loads: read once),
// prefetched RING steps ahead.  X rows are the "column" operand: the workgroup stages X[:, chunk] in LDS (double
// buffered, rows padded by 16 bytes so the 16 lanes of a quarter-wave hit distinct banks) and all
// waves read their fragments from there.  A workgroup has 4 waves arranged WN x WK: WN waves own
// different pairs of 16-row groups of W, WK waves split the steps of a chunk and are summed through
// LDS in a fixed order.  gridDim.y = KS splits the contraction across workgroups; only the
// residual epilogue supports it: every split stores its own fp32 partial, and the RMSNorm kernel
// that follows adds them in split order (deterministic, no atomics).
//
// Epilogues: rotary embedding + KV-scratch write (q, k, v), SwiGLU (gate, up), residual partial,
// and per-position argmax partials for the greedy choice (output embedding).
#include "ngg_epilogues.h"
#include <algorithm>
#include <cmath>

namespace ngg {

template <typename T, int EPI, int FM, int WN, int WK, int RING, int FN>
__global__ __launch_bounds__(64 * WN * WK) void gemm_skinny_kernel(const GemmCore a) {
  constexpr int XD = FM > 4 ? 1 : 2;         // X register stages (chunks fetched ahead); one when the tile is 128 rows
  static_assert(WN * WK == 4 || WN * WK == 8, "four or eight waves per workgroup");
  constexpr bool PAIRED = EPI == EPI_QKV || EPI == EPI_GATEUP;   // fragments that hold both halves of 8 output pairs
  static_assert(PAIRED ? WN == 1 : FN == 2, "paired epilogues: one set of FN fragments per workgroup, waves split K");
  constexpr int NT = 64 * WN * WK;           // threads per workgroup
  constexpr int KC = KChunk<T>::value;
  constexpr int SPC = KC / 32;               // steps per chunk
  constexpr int SPW = SPC / WK;              // steps per wave per chunk
  constexpr int PAD = 16 / (int)sizeof(T);
  constexpr int LDX = KC + PAD;              // LDS row stride in elements
  constexpr int ROWS = 16 * FM;
  constexpr int PIECES = ROWS * KC * (int)sizeof(T) / 16 / NT;    // 16-byte pieces per thread per chunk
  constexpr int PPR = KC * (int)sizeof(T) / 16;                   // pieces per row
  constexpr int UC0 = (RING % SPW == 0) ? RING / SPW : 1;
  constexpr int UC = UC0 % 2 == 0 ? UC0 : 2 * UC0;                // chunks per unrolled iteration (even: two X stages)
  static_assert((UC * SPW) % RING == 0, "ring slots must be static after unrolling");
  static_assert(PIECES >= 1, "chunk too small for the workgroup");

  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T *xs = reinterpret_cast<T *>(smem);       // [2][ROWS][LDX]

  const int tid = threadIdx.x, wave = tid >> 6, lane = tid & 63;
  const int li = lane & 15, g = lane >> 4;
  const int wn = wave % WN, wk = wave / WN;
  const int K = a.K, M = a.M;
  // When X holds h * gain, the RMSNorm kernel left the sums of squares of every row's segments
  // (kNormSegs floats per row, unused ones zero); the epilogue turns them into 1 / rms.
  static_assert(kNormSegs == 4, "one float4 per row");
  auto row_ss_load = [&](int m) {                        // (f32x4, not float4: arrays of the HIP struct go to scratch)
    if (!a.row_ss) return f32x4{0.f, 0.f, 0.f, 0.f};
    return *reinterpret_cast<const f32x4 *>(a.row_ss + (size_t)(m < a.Mcap ? m : a.Mcap - 1) * kNormSegs);
  };
  // ... times the factor that undoes the power-of-two scales of the stored operands (1 for fp32 models)
  auto row_scale = [&](const f32x4 &ss) {
    return (a.row_ss ? 1.0f / sqrtf((((ss[0] + ss[1]) + ss[2]) + ss[3]) / (float)K + a.ss_eps) : 1.0f) * a.out_scale;
  };
  const int n_groups = a.n_groups;
  int group = blockIdx.x * WN + wn;
  const bool group_live = group < n_groups;
  if (!group_live) group = n_groups - 1;     // idle waves still help staging X and hit every barrier

  // ---- the 16-row fragments of W this wave owns (W is stored in operand order: see tile_weights) ----
  // Residual and unembedding: group = 2 consecutive fragments.  q/k/v and gate/up: n_groups counts
  // fragments, the workgroup owns FN consecutive ones, and each fragment holds rows 0..7 = the first
  // members and rows 8..15 = the second members of 8 output pairs (rotary pairs (i, i + hd/2) of one
  // head; gate and up of 8 FFN features), so one accumulator has both halves of every pair it needs.
  const int n_steps = K / 32;
  const T *wblk[FN];                         // this lane's slice of the fragment's first 32-step block
  int nbase[FN];                             // first output feature (residual, unembedding) / fragment index (paired)
  bool frag_live[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) {
    int frag = PAIRED ? blockIdx.x * FN + f : group * FN + f;
    frag_live[f] = PAIRED ? frag < n_groups : group_live;
    if (PAIRED && !frag_live[f]) frag = n_groups - 1;      // the last workgroup repeats a fragment it does not store
    nbase[f] = PAIRED ? frag : frag * 16;
    wblk[f] = tiled_block((const T *)a.W0, frag, n_steps, lane);
  }

  // ---- this workgroup's range of chunks -----------------------------------------------------------
  const int n_chunks = (n_steps + SPC - 1) / SPC;
  const int KS = gridDim.y, ks = blockIdx.y;
  const int c0 = (int)(((long)n_chunks * ks) / KS), c1 = (int)(((long)n_chunks * (ks + 1)) / KS);

  for (int m0 = 0; m0 < M; m0 += ROWS) {
    // X staging: piece p = tid + NT*i covers row p / PPR (= tid / PPR + i * NT / PPR), 16 bytes at column
    // piece p % PPR.
    static_assert(NT % PPR == 0, "row stride of the staging pieces must be constant");
    constexpr int RPI = NT / PPR;                          // rows between a thread's consecutive pieces
    // (rows past the block's last one repeat it: the same cache lines as the threads that stage that row, so they
    // cost no further traffic from L2; what lands in their LDS rows is never stored)
    const T *xsrc0 = (const T *)a.X + (tid % PPR) * PAD;                 // chunk c adds c * Mcap * KC, piece i its row * KC
    const int xrow0 = m0 + tid / PPR, xrow_last = M - 1;
    const int xdst0 = (tid / PPR) * LDX + (tid % PPR) * PAD;
    // X is fetched XD chunks ahead into register stages (an L2 hit takes longer than one chunk of
    // MFMA work), then written to the LDS buffer of its chunk's parity.
    u32x4 stage[XD][PIECES];
    auto stage_load = [&](u32x4 (&st)[PIECES], int c) {
      const int cl = c < n_chunks ? c : n_chunks - 1;      // activation buffers are padded to whole chunks
#pragma unroll
      for (int i = 0; i < PIECES; ++i)
        st[i] = *reinterpret_cast<const u32x4 *>(xsrc0 + ((size_t)cl * a.Mcap + min(xrow0 + i * RPI, xrow_last)) * KC);
    };
    auto stage_store = [&](const u32x4 (&st)[PIECES], int buf) {
#pragma unroll
      for (int i = 0; i < PIECES; ++i) *reinterpret_cast<u32x4 *>(xs + (size_t)buf * ROWS * LDX + xdst0 + i * RPI * LDX) = st[i];
    };

    f32x4 acc[FN][FM];
#pragma unroll
    for (int f = 0; f < FN; ++f)
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) acc[f][fm] = f32x4{0.f, 0.f, 0.f, 0.f};

    // wave-step t is global step (c0 + t/SPW)*SPC + wk + WK*(t % SPW); steps outside the matrix are
    // clamped into it (loaded, never multiplied)
    Frag<T> ring[RING][FN];
    auto load_w = [&](Frag<T> (&slot)[FN], int t) {
      int s = c0 * SPC + (t / SPW) * SPC + wk + WK * (t % SPW);   // t >= 0 here
      s = s < n_steps ? s : n_steps - 1;
#pragma unroll
      for (int f = 0; f < FN; ++f) slot[f] = load_frag_stream(wblk[f] + (size_t)s * 512);
    };

    // The loop has no separate prologue: it starts one unrolled group early (ci = -UC) with the
    // multiplications switched off, so the loads that fill the ring and the X stages are issued by the
    // very instructions that refill them later.  Every trip then enters with the same set of loads
    // outstanding, in the same order, and the compiler's s_waitcnt vmcnt(n) before each use is exact
    // (with a prologue in another order it merged the two states and waited for nearly everything).
    const int n_iter = (c1 - c0 + UC - 1) / UC * UC;       // whole unrolled groups; extra chunks only load
    for (int ci = -UC; ci < n_iter; ci += UC) {
      const bool warm = ci < 0;
#pragma unroll
      for (int cc = 0; cc < UC; ++cc) {
        const int ch = c0 + ci + cc;
        const int buf = cc & 1;                          // UC is even
        if (!warm) stage_store(stage[cc % XD], buf);
        __syncthreads();
        stage_load(stage[cc % XD], max(ch + XD, 0));
        const T *xb = xs + (size_t)buf * ROWS * LDX + li * LDX + g * 8;
        // X fragments are read from LDS one step ahead of the MFMAs that use them (unconditionally:
        // during the warm-up group the buffer holds nothing yet and the values go unused)
        constexpr bool XPRE = FM <= 4;                     // 128-row tiles have no registers to spare
        Frag<T> xf[XPRE ? 2 : 1][FM];
        if constexpr (XPRE) {
#pragma unroll
          for (int fm = 0; fm < FM; ++fm) xf[0][fm] = load_frag(xb + fm * 16 * LDX + wk * 32);
        }
#pragma unroll
        for (int i = 0; i < SPW; ++i) {
          const int slot = (cc * SPW + i) % RING;        // constant after unrolling
          const int ls = wk + WK * i;                    // step inside the chunk
          if constexpr (XPRE) {
            if (i + 1 < SPW) {
#pragma unroll
              for (int fm = 0; fm < FM; ++fm) xf[(i + 1) & 1][fm] = load_frag(xb + fm * 16 * LDX + (ls + WK) * 32);
            }
          } else {
#pragma unroll
            for (int fm = 0; fm < FM; ++fm) xf[0][fm] = load_frag(xb + fm * 16 * LDX + ls * 32);
          }
          if (!warm && ch < c1 && ch * SPC + ls < n_steps) {      // uniform per wave; no global load inside
#pragma unroll
            for (int f = 0; f < FN; ++f)
#pragma unroll
              for (int fm = 0; fm < FM; ++fm) mma(acc[f][fm], ring[slot][f], xf[XPRE ? (i & 1) : 0][fm]);
          }
          load_w(ring[slot], max((ci + cc) * SPW + i + RING, 0));
        }
      }
    }
    __syncthreads();                                     // everyone is done with xs
    // 1 / rms of the pass's block rows, one per thread, left in LDS for the epilogues (fetched only now:
    // the main loop keeps every vector register it can get)
    float *rs_lds = reinterpret_cast<float *>(smem);     // [ROWS]; the hand-over buffers start behind it
    if (tid < ROWS) rs_lds[tid] = row_scale(row_ss_load(m0 + tid));

    // ---- q/k/v and gate/up: every wave hands its partial fragments over through LDS; wave wk then
    //      sums items wk, wk + WK, ... of the FN x FM accumulator fragments (waves in the order 0 .. WK-1)
    //      and runs their epilogue, one item at a time ------------------------------------------------------
    if constexpr (PAIRED) {
      // at most 4 column blocks of every fragment per round, so that the hand-over fits the LDS; the last
      // round of a tile of 5, 6 or 7 column blocks is shorter
      constexpr int FMR = FM < 4 ? FM : 4, ROUNDS = (FM + FMR - 1) / FMR;
      constexpr int IPW = (FN * FMR + WK - 1) / WK;        // items per round and wave, at most
      f32x4 *red = reinterpret_cast<f32x4 *>(smem + ROWS * sizeof(float));   // [WK][FN * cnt][64] lanes x 4 registers
#pragma unroll
      for (int rd = 0; rd < ROUNDS; ++rd) {
      const int cnt = (rd + 1) * FMR <= FM ? FMR : FM - rd * FMR;    // column blocks of this round (constant after unrolling)
      const int items = FN * cnt;                          // item idx = f * cnt + fr covers column block rd * FMR + fr
      if (rd > 0) __syncthreads();                       // the previous round's items were all read
#pragma unroll
      for (int f = 0; f < FN; ++f)
#pragma unroll
        for (int fr = 0; fr < FMR; ++fr)
          if (fr < cnt) red[((size_t)wk * items + f * cnt + fr) * 64 + lane] = acc[f][rd * FMR + (fr < cnt ? fr : 0)];
      __syncthreads();                                   // also: rs_lds is complete
      // unrolled where the items are short (SwiGLU) or few: the q/k/v item (rotary tables, three kinds of
      // stores) times 8 would not fit the registers
      constexpr int UNR = (EPI == EPI_GATEUP || IPW <= 3) ? IPW : 1;
#pragma unroll UNR
      for (int j = 0; j < IPW; ++j) {
        const int idx = wk + WK * j;
        if (idx >= items) break;
        const int f = idx / cnt;
        const int fm = rd * FMR + (idx - f * cnt);
        const int m = m0 + fm * 16 + li;
        const float rs = rs_lds[fm * 16 + li];
        const int frag = blockIdx.x * FN + f;              // fragment index over the whole matrix
        f32x4 sum = red[(size_t)idx * 64 + lane];
#pragma unroll
        for (int o = 1; o < WK; ++o) sum += red[((size_t)o * items + idx) * 64 + lane];
        if (frag < n_groups) epi_paired<T, EPI>(a, frag, m, M, g, rs, sum);   // (uniform per wave)
      }
      }
    }

    // ---- sum the WK waves that share a wn: wave (wn, 0) adds (wn, 1) .. (wn, WK-1) in that order ---
    if constexpr (!PAIRED && WK == 1) __syncthreads();   // rs_lds is complete
    if constexpr (!PAIRED && WK > 1) {
      float *red = reinterpret_cast<float *>(smem) + ROWS;   // [(WK-1)][WN][FN*FM*4][64]
      if (wk > 0) {
        float *dst = red + (size_t)((wk - 1) * WN + wn) * (FN * FM * 4 * 64);
#pragma unroll
        for (int f = 0; f < FN; ++f)
#pragma unroll
          for (int fm = 0; fm < FM; ++fm)
#pragma unroll
            for (int r = 0; r < 4; ++r) dst[((f * FM + fm) * 4 + r) * 64 + lane] = acc[f][fm][r];
      }
      __syncthreads();
      if (wk == 0) {
        for (int o = 1; o < WK; ++o) {
          const float *src = red + (size_t)((o - 1) * WN + wn) * (FN * FM * 4 * 64);
#pragma unroll
          for (int f = 0; f < FN; ++f)
#pragma unroll
            for (int fm = 0; fm < FM; ++fm)
#pragma unroll
              for (int r = 0; r < 4; ++r) acc[f][fm][r] += src[((f * FM + fm) * 4 + r) * 64 + lane];
        }
      }
    }

    // ---- epilogue, waves (wn, 0): lane holds, per group f and column block fm, column
    //      m = m0 + fm*16 + li and output features nbase[f] + 4g .. +4 -----------------------------------
    if (!PAIRED && wk == 0 && group_live) {
#pragma unroll
      for (int fm = 0; fm < FM; ++fm) {
        const int m = m0 + fm * 16 + li;
        const bool live = m < M;
        if constexpr (EPI == EPI_RESIDUAL) {
          if (live) {
#pragma unroll
            for (int f = 0; f < FN; ++f) epi_residual(a, ks, m, nbase[f], g, acc[f][fm]);
          }
        } else {   // EPI_UNEMBED
          f32x4 sums[FN];
#pragma unroll
          for (int f = 0; f < FN; ++f) sums[f] = acc[f][fm];
          epi_unembed<FN>(a, group, m, live, g, rs_lds[fm * 16 + li], nbase, sums);
        }
      }
    }
    __syncthreads();                                       // LDS is reused by the next column block
  }
}


// ---------------------------------------------------------------------------------------------
// Tiled GEMM (16-bit operands): prefill pieces and wide blocks, where a weight meets enough block rows that the
// caches, the LDS and the matrix cores bound the call instead of the stream of W.  A workgroup of WM x WN waves owns
// TM = 32 WM BM block rows and TN = 32 WN BN rows of W; a wave BM x BN blocks of the 32x32x16 MFMA (a loop of nothing
// else runs at 2.1-2.2 PFLOP/s here, 16x16x32 at 1.45-1.55).  Both operands go from global memory straight into LDS
// (16 bytes per lane, no registers in between), in slices of 64 contraction elements, NST slices deep.  Before, W went
// into registers and the two waves that shared a fragment both fetched it: a 128 x 256 tile asked the L2 for 64 KB per
// slice, as much as the path between L2 and CU carries in the slice's MFMA time; a 256 x 256 tile fed through LDS asks
// for half of that per flop.  Measured at the 7B shapes, 2048 rows: gate/up 500 -> 414 us (1.16 PFLOP/s; a library
// GEMM of the same size reaches 1.11-1.18), down 250 -> 217, output projection 85 -> 72; 777 rows: gate/up 256 -> 210,
// q/k/v 194 -> 109, down 186 -> 121, projection 67 -> 38; a 768-wide model at 777 rows: 34 -> 15, 27 -> 13, 20 -> 12.5,
// 22 -> 6.4 (small tiles fill the chip where three 288-row tiles left most CUs idle).  What is left at 2048 rows: the
// matrix cores are busy 54-64 % of the cycles at the 1.8 GHz the card holds under this load, the LDS 22-25 %.
//
// One slice is four multiplication steps of 16 contraction elements.  The fragments of a step are read from LDS under
// the previous step's MFMAs; the barrier that hands over the buffers sits before the last step, whose operands are in
// registers by then: behind it the first fragments of the next slice are read and the DMA of slice s + NST goes out
// between the last step's MFMAs, into the buffer everybody has just finished reading.
//
// LDS images.  W: the 1 KB operand blocks as they are stored (16 rows x 32 elements, lane-major), read without bank
// conflicts.  X: row-major, 128 bytes per row, the 16-byte piece c of row r at position c ^ (r / 2 % 8): a DMA
// instruction covers whole 128-byte lines of 8 rows, and the 16 rows one quarter of the wave reads meet all banks.
// Operand lanes: lane 32 h + r takes row r of a 32-row block and contraction elements 8 h .. 8 h + 7 of the 16.
// Accumulator register 4 j + i of lane (r, h) is W row 8 j + 4 h + i of the 32 at block row r: both halves of an output
// pair (registers of j and j + 1) sit in one lane.
// ---------------------------------------------------------------------------------------------
typedef float f32x16 __attribute__((ext_vector_type(16)));

__device__ __forceinline__ void wave_lds_fence() {       // LDS written by other lanes of this wave is readable behind it
  __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
  __builtin_amdgcn_wave_barrier();
  __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// frag_first, frag_end: 16-row fragments of W this launch covers; MT row tiles, `tiles` tiles in all
template <int EPI, int WM, int WN, int BM, int BN, int NST, bool NT>
__global__ __launch_bounds__(64 * WM * WN) void gemm_tile_kernel(const GemmCore a, int MT, int tiles, int frag_first, int frag_end) {
  typedef half_t T;
  constexpr int NW = WM * WN, TM = 32 * WM * BM, TN = 32 * WN * BN;
  constexpr int KC = KChunk<T>::value, KW = 64;
  constexpr int WI = TN / 8 / NW, XI = TM / 8 / NW;      // DMA instructions (1 KB each) per wave and slice
  static_assert(WI * NW * 8 == TN && XI * NW * 8 == TM, "whole instructions per wave");
  constexpr int PER = WI + XI;
  static_assert((NST - 1) * PER < 64, "vmcnt counts to 63");
  constexpr int BUF = (TM + TN) * KW * 2;                // bytes of one slice
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];

  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int r32 = lane & 31, h = lane >> 5;
  const int wn = wave % WN, wm = wave / WN;
  const int K = a.K, M = a.M;
  const int n_steps = K / 32, n_slices = (n_steps + 1) / 2;
  const int KS = gridDim.y, ks = blockIdx.y;
  // Workgroup b runs on XCD b % 8 and takes that XCD's next tile.  Every XCD has a contiguous share of the tiles, row
  // tiles first: the workgroups that share rows of W run side by side on one L2, which reads them from HBM once.
  const int per = gridDim.x / 8;
  const int tile = (blockIdx.x % 8) * per + blockIdx.x / 8;
  if (tile >= tiles) return;
  const int m0 = tile % MT * TM;
  const int f0 = frag_first + tile / MT * (TN / 16);
  const int c0 = (int)(((long)n_slices * ks) / KS), c1 = (int)(((long)n_slices * (ks + 1)) / KS);   // c1 > c0: KS <= n_slices

  // ---- DMA sources: a wave-uniform base per instruction plus this lane's byte offset ----------------
  // (fragments past the end repeat the last one, rows past the block's last one repeat that row; neither is stored)
  const char *wbase[WI];
  unsigned xoffs[XI];
#pragma unroll
  for (int i = 0; i < WI; ++i) {                         // instruction wave * WI + i: fragment (.. / 2), step (.. % 2)
    const int id = wave * WI + i;
    wbase[i] = (const char *)a.W0 + (size_t)min(f0 + id / 2, frag_end - 1) * n_steps * 1024;
  }
#pragma unroll
  for (int i = 0; i < XI; ++i) {
    const int row = (wave * XI + i) * 8 + (lane >> 3);
    const int piece = (lane & 7) ^ ((row >> 1) & 7);
    xoffs[i] = (unsigned)min(m0 + row, M - 1) * (KC * 2) + piece * 16;
  }
  const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) unsigned char *)smem;
  auto dma = [&](int sl, int buf, int i) {               // i-th of the wave's PER instructions for slice sl (clamped to the last)
    const int s = min(sl, c1 - 1);
    const unsigned base = lds0 + buf * BUF;
    if (i < WI) {
      const int id = wave * WI + i;
      // K % 64 == 32: the last slice's second step repeats the first; X holds zeros there (the padding of its chunk)
      const int st = min(2 * s + (id & 1), n_steps - 1);
      lds_dma16<NT>(wbase[i < WI ? i : 0] + (size_t)st * 1024, lane * 16, base + id * 1024);
    } else {
      const int k0 = s * KW;
      const size_t off = (size_t)(k0 / KC) * a.Mcap * KC + k0 % KC;
      lds_dma16<false>((const char *)a.X + off * 2, xoffs[i < WI ? 0 : i - WI], base + TN * KW * 2 + (wave * XI + i - WI) * 1024);
    }
  };

  f32x16 acc[BN][BM];
#pragma unroll
  for (int p = 0; p < BN; ++p)
#pragma unroll
    for (int b = 0; b < BM; ++b)
#pragma unroll
      for (int r = 0; r < 16; ++r) acc[p][b][r] = 0.f;

  // fragments of step q (the q-th 16 of the slice's 64 contraction elements)
  const int woff = (wn * BN * 2 + (r32 >> 4)) * 2048 + (16 * h + (r32 & 15)) * 16;
  const int xrow = wm * BM * 32 + r32;
  const int xsw = (xrow >> 1) & 7;
  const int xoff = TN * KW * 2 + xrow * 128;
  half8 wf[2][BN], xf[2][BM];
  auto read = [&](int set, int buf, int q) {
    const unsigned char *base = smem + buf * BUF;
#pragma unroll
    for (int p = 0; p < BN; ++p)
      wf[set][p] = *reinterpret_cast<const half8 *>(base + woff + p * 4096 + (q >> 1) * 1024 + (q & 1) * 512);
#pragma unroll
    for (int b = 0; b < BM; ++b)
      xf[set][b] = *reinterpret_cast<const half8 *>(base + xoff + b * 4096 + ((2 * q + h) ^ xsw) * 16);
  };
  constexpr int NMF = BM * BN, NRD = BM + BN;
  auto mul1 = [&](int set, int k) {
    acc[k % BN][k / BN] = __builtin_amdgcn_mfma_f32_32x32x16_f16(wf[set][k % BN], xf[set][k / BN], acc[k % BN][k / BN], 0, 0, 0);
  };

#pragma unroll
  for (int i = 0; i < NST; ++i)
#pragma unroll
    for (int j = 0; j < PER; ++j) dma(c0 + i, i, j);
  asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NST - 1) * PER) : "memory");
  __builtin_amdgcn_s_barrier();
  read(0, 0, 0);
  int buf = 0;
  for (int s = c0; s < c1; ++s) {
    const int nbuf = buf + 1 == NST ? 0 : buf + 1;
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int q = 0; q < 3; ++q) {
      read((q + 1) & 1, buf, q + 1);
#pragma unroll
      for (int k = 0; k < NMF; ++k) mul1(q & 1, k);
#pragma unroll
      for (int k = 0; k < NMF; ++k) {                    // one MFMA, then its share of the LDS reads
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
        __builtin_amdgcn_sched_group_barrier(0x100, (NRD + NMF - 1) / NMF, 0);
      }
      __builtin_amdgcn_sched_barrier(0);
    }
    asm volatile("s_waitcnt vmcnt(%0) lgkmcnt(0)" ::"n"((NST - 2) * PER) : "memory");   // slice s + 1 has landed
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_sched_barrier(0);
    read(0, nbuf, 0);
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int k = 0; k < (NMF > PER ? NMF : PER); ++k) {
      if (k < NMF) mul1(1, k);
      if (k < PER) dma(s + NST, buf, k);
      __builtin_amdgcn_sched_barrier(0);
    }
    buf = nbuf;
  }
  asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)" ::: "memory");
  __syncthreads();                                       // nothing on its way to LDS any more, everyone is done with it

  static_assert(kNormSegs == 4, "one float4 per row");
  float *rs_lds = reinterpret_cast<float *>(smem);       // [TM] 1 / rms times the operand scales
  if constexpr (EPI != EPI_RESIDUAL) {
    for (int r = tid; r < TM; r += 64 * NW) {
      float v = 1.0f;
      if (a.row_ss) {
        const int m = m0 + r;
        const f32x4 ss = *reinterpret_cast<const f32x4 *>(a.row_ss + (size_t)(m < a.Mcap ? m : a.Mcap - 1) * kNormSegs);
        v = 1.0f / sqrtf((((ss[0] + ss[1]) + ss[2]) + ss[3]) / (float)K + a.ss_eps);
      }
      rs_lds[r] = v * a.out_scale;
    }
    __syncthreads();
  }
  const int row0 = wm * BM * 32 + r32;
  const int fw = f0 + wn * BN * 2;                       // first fragment of this wave
  if constexpr (EPI == EPI_QKV) {
    // The scaled accumulators of one 32-row block leave the registers through LDS (every wave its own region) and come
    // back one fragment at a time: all at once, the fragments' table entries and addresses do not fit the registers.
    float *dump = reinterpret_cast<float *>(smem + TM * sizeof(float)) + (size_t)wave * (BN * 4 * 256);
    const int half = a.hd / 2, fph = a.hd / 16;
    const int P = a.n_dev ? *a.n_dev - 1 : a.P;
#pragma unroll
    for (int b = 0; b < BM; ++b) {
      const int row = row0 + b * 32, m = m0 + row;
      const float rs = rs_lds[row];
#pragma unroll
      for (int p = 0; p < BN; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<f32x4 *>(dump + ((p * 4 + j) * 64 + lane) * 4) =
              f32x4{acc[p][b][4 * j] * rs, acc[p][b][4 * j + 1] * rs, acc[p][b][4 * j + 2] * rs, acc[p][b][4 * j + 3] * rs};
      wave_lds_fence();
#pragma unroll 1
      for (int idx = 0; idx < BN * 2; ++idx) {
        const int frag = fw + idx;
        if (frag >= frag_end) break;                     // uniform per wave
        const int hh = frag / fph, sub = frag - hh * fph;  // head over [q heads | k heads | v heads], 8-dim group of its lower half
        if (hh < a.H + a.Hkv) {                          // q and k: rotary embedding, then 8 consecutive dims per lane
          const f32x4 v = *reinterpret_cast<const f32x4 *>(dump + (2 * idx * 64 + lane) * 4);
          const f32x4 x2 = *reinterpret_cast<const f32x4 *>(dump + ((2 * idx + 1) * 64 + lane) * 4);
          const int pos = P + block_col(min(m, M - 1), a.C, a.shared0);
          const f32x4 cs = *reinterpret_cast<const f32x4 *>(a.rope_cos + (size_t)pos * half + sub * 8 + 4 * h);
          const f32x4 sn = *reinterpret_cast<const f32x4 *>(a.rope_sin + (size_t)pos * half + sub * 8 + 4 * h);
          union { half4 v; unsigned u[2]; } lo, hi;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            lo.v[r] = to_half(v[r] * cs[r] - x2[r] * sn[r]);
            hi.v[r] = to_half(x2[r] * cs[r] + v[r] * sn[r]);
          }
          // lanes h = 0 collect the 8 lower dims, lanes h = 1 the 8 upper ones
          const auto w0 = __builtin_amdgcn_permlane32_swap(lo.u[0], hi.u[0], false, false);
          const auto w1 = __builtin_amdgcn_permlane32_swap(lo.u[1], hi.u[1], false, false);
          const u32x4 piece = u32x4{w0[0], w1[0], w0[1], w1[1]};
          const int dim = sub * 8 + (h ? half : 0);
          T *dst = hh < a.H ? (T *)a.q + ((size_t)hh * a.Mcap + m) * a.hd + dim
                            : (T *)a.kscr + (size_t)(hh - a.H) * a.kv_rows * a.hd + k_offset(m, dim, a.hd, 2);
          if (m < M) *reinterpret_cast<u32x4 *>(dst) = piece;
        } else {                                         // values: 8 consecutive positions of one dim per lane
          const int dd = lane >> 2, g8 = lane & 3;       // dim of the fragment (0..7 lower, 8..15 upper), group of 8 positions
          const float *src = dump + ((2 * idx + (dd >> 3)) * 64 + 32 * ((dd >> 2) & 1) + 8 * g8) * 4 + (dd & 3);
          half8 o;
#pragma unroll
          for (int e = 0; e < 8; ++e) o[e] = to_half(src[4 * e]);
          const int mb = m0 + wm * BM * 32 + b * 32 + 8 * g8;
          const int dim = sub * 8 + (dd & 7) + (dd >> 3) * half;
          T *dst = (T *)a.vscr + (size_t)(hh - a.H - a.Hkv) * a.kv_rows * a.hd + v_offset(mb, dim, a.hd, 2);
          if (mb + 8 <= M) *reinterpret_cast<half8 *>(dst) = o;
          else
#pragma unroll
            for (int e = 0; e < 8; ++e)
              if (mb + e < M) dst[e] = o[e];
        }
      }
      wave_lds_fence();
    }
  } else if constexpr (EPI == EPI_GATEUP) {
    // the tile's activations go through LDS, so that a row's features leave in 16-byte pieces side by side (8-byte
    // pieces of 32 rows per instruction cost 3 % more at 2048 rows)
    constexpr int LDO = TN / 2 + 8;                      // LDS row stride in elements
    T *ot = reinterpret_cast<T *>(smem + TM * sizeof(float));
#pragma unroll
    for (int b = 0; b < BM; ++b) {
      const int row = row0 + b * 32;
      const float rs = rs_lds[row];
#pragma unroll
      for (int p = 0; p < BN; ++p)
#pragma unroll
        for (int t = 0; t < 2; ++t) {
          float o[4];
#pragma unroll
          for (int r = 0; r < 4; ++r) o[r] = silu<T>(acc[p][b][8 * t + r] * rs) * (acc[p][b][8 * t + 4 + r] * rs);
          store4(ot + row * LDO + (wn * BN * 2 + 2 * p + t) * 8 + 4 * h, o[0], o[1], o[2], o[3]);
        }
    }
    __syncthreads();
    constexpr int PPR = TN / 16;                         // 16-byte pieces per row: one per fragment
    for (int e = tid; e < TM * PPR; e += 64 * NW) {
      const int row = e / PPR, fr = e % PPR, m = m0 + row;
      if (m < M && f0 + fr < frag_end)
        *reinterpret_cast<u32x4 *>((T *)a.act + act_offset<T>(m, (f0 + fr) * 8, a.Mcap)) = *reinterpret_cast<const u32x4 *>(ot + row * LDO + fr * 8);
    }
  } else if constexpr (EPI == EPI_UNEMBED) {
    // optional logits, and the best (value, id) of a block row over every 32 vocabulary rows; ids ascend with (j, i)
    // inside a lane, the two lanes of a row hold alternate groups of four
#pragma unroll
    for (int b = 0; b < BM; ++b) {
      const int row = row0 + b * 32, m = m0 + row;
      const float rs = rs_lds[row];
#pragma unroll
      for (int p = 0; p < BN; ++p) {
        if (fw + 2 * p >= frag_end) continue;            // uniform per wave
        const int n0 = (fw + 2 * p) * 16 + 4 * h;
        float bv = kNegBig;
        int bi = 0x7fffffff;
#pragma unroll
        for (int j = 0; j < 4; ++j) {
          f32x4 v;
#pragma unroll
          for (int r = 0; r < 4; ++r) {
            v[r] = acc[p][b][4 * j + r] * rs;
            if (v[r] > bv) { bv = v[r]; bi = n0 + 8 * j + r; }
          }
          if (a.logits && m < M) *reinterpret_cast<f32x4 *>(a.logits + (size_t)m * a.N + n0 + 8 * j) = v;
        }
        const float ov = other_half(bv);
        const int oi = __float_as_int(other_half(__int_as_float(bi)));
        if (ov > bv || (ov == bv && oi < bi)) { bv = ov; bi = oi; }
        if (m < M && h == 0) {
          a.pmax_val[(size_t)(fw / 2 + p) * a.Mcap + m] = bv;
          a.pmax_idx[(size_t)(fw / 2 + p) * a.Mcap + m] = bi;
        }
      }
    }
  } else {
    // partials: every wave turns its blocks around in LDS of its own and stores whole row segments (stored straight
    // from the accumulators, 16 bytes per row and instruction: 226 instead of 213 us for down, 92 instead of 74 for O)
    constexpr int LDO = 32 * BN + 4;
    float *ot = reinterpret_cast<float *>(smem) + wave * 32 * LDO;
    constexpr int LPR = 8 * BN;                          // lanes per row segment
    const int n0 = fw * 16;
#pragma unroll
    for (int b = 0; b < BM; ++b) {
#pragma unroll
      for (int p = 0; p < BN; ++p)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          *reinterpret_cast<f32x4 *>(ot + r32 * LDO + p * 32 + 8 * j + 4 * h) =
              f32x4{acc[p][b][4 * j] * a.out_scale, acc[p][b][4 * j + 1] * a.out_scale, acc[p][b][4 * j + 2] * a.out_scale, acc[p][b][4 * j + 3] * a.out_scale};
      wave_lds_fence();
#pragma unroll
      for (int it = 0; it < 32; it += 64 / LPR) {
        const int row = it + lane / LPR, col = lane % LPR * 4, m = m0 + wm * BM * 32 + b * 32 + row;
        const f32x4 v = *reinterpret_cast<const f32x4 *>(ot + row * LDO + col);
        if (m < M && n0 + col < frag_end * 16) *reinterpret_cast<f32x4 *>(a.hpart + ((size_t)ks * a.Mcap + m) * a.N + n0 + col) = v;
      }
      wave_lds_fence();
    }
  }
}

template <int EPI, int WM, int WN, int BM, int BN, int NST>
static void launch_tile_cfg(const GemmCore &a, int KS, int frag_first, int frag_end, hipStream_t s) {
  constexpr int TM = 32 * WM * BM, TN = 32 * WN * BN;
  size_t lds = (size_t)NST * (TM + TN) * 64 * 2;
  if (EPI == EPI_QKV) lds = std::max(lds, (size_t)TM * 4 + (size_t)WM * WN * BN * 4096);
  if (EPI == EPI_GATEUP) lds = std::max(lds, (size_t)TM * 4 + (size_t)TM * (TN / 2 + 8) * 2);
  if (EPI == EPI_RESIDUAL) lds = std::max(lds, (size_t)WM * WN * 32 * (32 * BN + 4) * 4);
  static const hipError_t opted = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_tile_kernel<EPI, WM, WN, BM, BN, NST, false>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  static const hipError_t opted_nt = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_tile_kernel<EPI, WM, WN, BM, BN, NST, true>),
                                                         hipFuncAttributeMaxDynamicSharedMemorySize, 160 * 1024);
  (void)opted; (void)opted_nt;
  const int MT = (a.M + TM - 1) / TM;
  const int tiles = MT * ((frag_end - frag_first + TN / 16 - 1) / (TN / 16));
  const dim3 grid((tiles + 7) / 8 * 8, KS), block(64 * WM * WN);
  if (MT == 1) hipLaunchKernelGGL((gemm_tile_kernel<EPI, WM, WN, BM, BN, NST, true>), grid, block, lds, s, a, MT, tiles, frag_first, frag_end);
  else hipLaunchKernelGGL((gemm_tile_kernel<EPI, WM, WN, BM, BN, NST, false>), grid, block, lds, s, a, MT, tiles, frag_first, frag_end);
}

// Tile shapes of gemm_tile_kernel with what a workgroup costs: microseconds per slice of 64 contraction elements, and
// for its start and epilogue (fitted to launches at the 7B shapes above 128 rows and at 768-wide ones from 97, up to 2048, on
// MI355X; below that it is optimistic for wide models, 29.5 us where q/k/v of 97 rows took 35.3: takes_tile decides there).
// The last two are for 129 to 192 rows as one row tile, where two tiles of 128 rows compute 256 and W is fetched for each of
// them (gate/up, us: 145 rows 67 -> 55, 177 rows 70 -> 60; the kernel before this one took 64 at 145).  The three before them
// are for 257 to 384 rows, which the 256-row tile computes as 512 and the 128-row one as 384 in one and a
// half rounds (7B shapes, us; before them -> with them): gate/up as one row tile of 288 or 384, 257 rows 118 -> 83, 289-384
// rows 118-121 -> 97-100; q/k/v as two of 192 x 96, one full round, 67 -> 50-52.  The 288-row tile runs on four waves of
// nine MFMA blocks: on eight, two of the four SIMDs would have a wave more than the others.
struct TileShape { int tm, tn; float slice_us, fixed_us; };
constexpr TileShape kTileShapes[] = {{256, 256, 1.60f, 10.0f}, {128, 256, 0.98f, 8.0f}, {128, 128, 0.54f, 6.0f}, {128, 64, 0.36f, 4.5f}, {64, 64, 0.30f, 3.5f},
                                     {288, 128, 1.13f, 10.0f}, {384, 128, 1.38f, 10.0f}, {192, 96, 0.65f, 7.0f},
                                     {160, 128, 0.70f, 9.5f}, {192, 128, 0.78f, 10.0f}};
constexpr int kNumTileShapes = 10;

// Which of them a launch chooses among.  Beyond 384 rows the last five only replace equals (7B: gate/up of 513 rows 163
// against 162 us, q/k/v of 641 rows 103 and 103); the residual GEMMs do without them (257 rows: 35.2 us on 128 x 256 with
// five splits, 35.8 on 288 x 128 with eight, and the RMSNorm that adds the splits 7.7 -> 8.9).
static bool shape_fits(int c, int epi, int M) {
  if (c < 5) return true;
  return epi != EPI_RESIDUAL && (c < 8 ? M > 256 && M <= 384 : M > 128 && M <= 192);
}

struct TilePlan { int shape, KS, split, shape2; };        // fragments from `split` on run as a second launch in shape2

static float tile_cost(int shape, int epi, int M, int frags, int K, int KS) {
  const TileShape &t = kTileShapes[shape];
  const int mt = (M + t.tm - 1) / t.tm;
  const float rounds = (float)(mt * ((frags * 16 + t.tn - 1) / t.tn) * KS) / 256.0f;
  // whole rounds of 256 CUs; the last one, partly empty, runs a little faster than a full one (less traffic, higher
  // clocks).  7B shapes: 1.13 rounds cost 1.95, 1.31 cost 1.7, 1.75 cost 1.95, 2.6 cost 3.0, 6.1 cost 6.5
  const float eff = rounds <= 1.0f ? 1.0f : 0.3f * rounds + 0.7f * std::ceil(rounds);
  const float slices = (float)((K + 63) / 64) / (float)KS;
  return eff * (slices * t.slice_us + t.fixed_us + (epi == EPI_QKV ? 2.0f : 0.0f));
}

// The cheapest plan by the costs above.  Splitting the contraction (residual only) fills the chip when there are few
// tiles; every split costs M x N partials written and read again by the RMSNorm.  When the tiles of a launch fill a
// number of rounds and a half, the half round is given smaller tiles in a launch of its own.
// only: 1 + the shape every launch has to take (0: any).
static TilePlan tile_plan(int epi, int M, int frags, int K, int only) {
  const int n_slices = (K + 63) / 64;
  TilePlan best{0, 1, frags, 0};
  float cost = 1e30f;
  for (int c = 0; c < kNumTileShapes; ++c) {
    if (only ? c != only - 1 : !shape_fits(c, epi, M)) continue;
    const TileShape &t = kTileShapes[c];
    if (epi == EPI_RESIDUAL) {
      for (int ks = 1; ks <= kMaxResidualSplits && (ks == 1 || n_slices >= 2 * ks); ++ks) {
        const float x = tile_cost(c, epi, M, frags, K, ks) + (float)M * frags * 64.0f * ks / 6.0e6f;
        if (x < cost) { cost = x; best = {c, ks, frags, c}; }
      }
      continue;
    }
    const float x = tile_cost(c, epi, M, frags, K, 1);
    if (x < cost) { cost = x; best = {c, 1, frags, c}; }
    const int mt = (M + t.tm - 1) / t.tm, cols = (frags * 16 + t.tn - 1) / t.tn;
    const int whole = mt * cols / 256 * 256 / mt;         // columns that fill whole rounds
    if (whole < 1 || whole >= cols) continue;
    const int cut = whole * (t.tn / 16);
    for (int c2 = 0; c2 < kNumTileShapes; ++c2) {
      if (only ? c2 != only - 1 : !shape_fits(c2, epi, M)) continue;
      const float y = tile_cost(c, epi, M, cut, K, 1) + tile_cost(c2, epi, M, frags - cut, K, 1) + 3.0f;
      if (y < cost) { cost = y; best = {c, 1, cut, c2}; }
    }
  }
  return best;
}

template <int EPI>
static void launch_tile_shape(int shape, const GemmCore &a, int KS, int f0, int f1, hipStream_t s) {
  if (f0 >= f1) return;
  switch (shape) {
    case 0: launch_tile_cfg<EPI, 2, 4, 4, 2, 2>(a, KS, f0, f1, s); break;
    case 1: launch_tile_cfg<EPI, 2, 4, 2, 2, 3>(a, KS, f0, f1, s); break;
    case 2: launch_tile_cfg<EPI, 2, 4, 2, 1, 4>(a, KS, f0, f1, s); break;
    case 3: launch_tile_cfg<EPI, 4, 2, 1, 1, 3>(a, KS, f0, f1, s); break;
    case 4: launch_tile_cfg<EPI, 2, 2, 1, 1, 4>(a, KS, f0, f1, s); break;
    case 5: launch_tile_cfg<EPI, 1, 4, 9, 1, 3>(a, KS, f0, f1, s); break;
    case 6: launch_tile_cfg<EPI, 4, 2, 3, 2, 2>(a, KS, f0, f1, s); break;
    case 7: launch_tile_cfg<EPI, 2, 3, 3, 1, 4>(a, KS, f0, f1, s); break;
    case 8: launch_tile_cfg<EPI, 1, 4, 5, 1, 4>(a, KS, f0, f1, s); break;
    default: launch_tile_cfg<EPI, 2, 4, 3, 1, 4>(a, KS, f0, f1, s);
  }
}

template <int EPI>
static void launch_tile(const GemmCore &a, hipStream_t s) {
  const int frags = EPI == EPI_QKV ? (a.H + 2 * a.Hkv) * (a.hd / 16) : (EPI == EPI_GATEUP ? a.N / 8 : a.N / 16);
  const TilePlan p = tile_plan(EPI, a.M, frags, a.K, a.tile_only);
  launch_tile_shape<EPI>(p.shape, a, p.KS, 0, p.split, s);  // residual: p.KS == a.KS (gemm_residual_splits)
  launch_tile_shape<EPI>(p.shape2, a, p.KS, p.split, frags, s);
}
template <typename T, int EPI, int FM, int WN, int WK, int RING, int FN = 2>
void launch_gemm_cfg(const GemmCore &a, int KS, hipStream_t s) {
  constexpr int KC = KChunk<T>::value;
  constexpr int PAD = 16 / (int)sizeof(T);
  constexpr bool PAIRED = EPI == EPI_QKV || EPI == EPI_GATEUP;
  size_t lds = (size_t)2 * 16 * FM * (KC + PAD) * sizeof(T);
  const size_t red = (size_t)(PAIRED ? WK * (FM < 4 ? FM : 4) : (WK - 1) * WN * FM) * FN * 4 * 64 * sizeof(float) +
                     (size_t)16 * FM * sizeof(float);          // + one 1 / rms per block row of the pass
  if (red > lds) lds = red;
  const int blocks = PAIRED ? (a.n_groups + FN - 1) / FN : (a.n_groups + WN - 1) / WN;
  if (lds > 64 * 1024) {                     // more than the default dynamic LDS limit: opt in once
    static const hipError_t opted = hipFuncSetAttribute(
        reinterpret_cast<const void *>(&gemm_skinny_kernel<T, EPI, FM, WN, WK, RING, FN>),
        hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
    (void)opted;
  }
  hipLaunchKernelGGL((gemm_skinny_kernel<T, EPI, FM, WN, WK, RING, FN>), dim3(blocks, KS), dim3(64 * WN * WK), lds, s, a);
}

// residual, unembedding: pairs of 16-row fragments; q/k/v and gate/up: 16-row fragments of 8 output pairs
int gemm_groups(int epi, const GemmCore &a) {
  switch (epi) {
    case EPI_QKV: return (a.H + 2 * a.Hkv) * (a.hd / 16);
    case EPI_GATEUP: return a.N / 8;
    default: return a.N / 32;
  }
}

// The row tile holds the block's rows in 16-row column blocks of the MFMA: as many as the block needs, up
// to 8 (128 rows; more rows take another pass over W).  Every extra column block costs activation traffic
// from L2, LDS reads and MFMA work, so a 40-row block runs on 3 of them, not 4.
static int gemm_row_blocks(int M) { return M >= 128 ? 8 : (M + 15) / 16; }

template <typename T, int EPI, int WN, int WK, int RING>
static void launch_fm(const GemmCore &a, int KS, hipStream_t s) {
  switch (gemm_row_blocks(a.M)) {                            // 16-row column blocks of the tile
    case 5: launch_gemm_cfg<T, EPI, 5, WN, WK, RING>(a, KS, s); return;
    case 6: launch_gemm_cfg<T, EPI, 6, WN, WK, RING>(a, KS, s); return;
    case 7: launch_gemm_cfg<T, EPI, 7, WN, WK, RING>(a, KS, s); return;
    default: break;
  }
  if constexpr (EPI == EPI_RESIDUAL) {                       // (the unembedding of up to 64 rows: gemm_stream_kernel)
    switch (gemm_row_blocks(a.M)) {
      case 1: launch_gemm_cfg<T, EPI, 1, WN, WK, RING>(a, KS, s); return;
      case 2: launch_gemm_cfg<T, EPI, 2, WN, WK, RING>(a, KS, s); return;
      case 3: launch_gemm_cfg<T, EPI, 3, WN, WK, RING>(a, KS, s); return;
      case 4: launch_gemm_cfg<T, EPI, 4, WN, WK, RING>(a, KS, s); return;
      default: break;
    }
  }
  launch_gemm_cfg<T, EPI, 8, WN, WK, RING>(a, KS, s);        // 128-row tiles; more rows loop over W again
}

// q/k/v and gate/up: one workgroup = FN fragments, its four waves split the steps of every chunk (WN = 1, WK = 4).  fp32
// only: the 16-bit ones run on gemm_stream_kernel or the tiled one.
template <typename T, int EPI, int FM>
static void launch_paired_fm(const GemmCore &a, hipStream_t s) {
  if (a.n_groups <= 256) launch_gemm_cfg<T, EPI, FM, 1, 4, 4, 1>(a, 1, s);
  else launch_gemm_cfg<T, EPI, FM, 1, 4, 4, 2>(a, 1, s);
}

template <typename T, int EPI>
static void launch_paired(const GemmCore &a, hipStream_t s) {
  switch (gemm_row_blocks(a.M)) {                            // (up to four: gemm_stream_kernel)
    case 5: launch_paired_fm<T, EPI, 5>(a, s); break;
    case 6: launch_paired_fm<T, EPI, 6>(a, s); break;
    case 7: launch_paired_fm<T, EPI, 7>(a, s); break;
    default: launch_paired_fm<T, EPI, 8>(a, s);
  }
}

// Residual GEMMs: a workgroup takes 64 rows of W (WN = 2, its waves 2 x 2), or 32 rows with all four
// waves splitting the steps (WN = 1) where that measured faster on MI355X: single-token steps, and the
// square output projection (4096 x 4096: 11.0 against 11.7 us at 60 block rows, 8.2 against 9.5 at one;
// down 4096 x 14336: 26.2 against 23.4 at 60 rows, 19.6 against 20.5 at one).  Narrower workgroups need
// half the splits of the contraction, so the RMSNorm that follows adds half the partials.
static bool residual_narrow(int M, int N, int K) { return M <= 16 || K <= N; }

// Workgroups of the skinny kernel for a residual GEMM: about one per CU, as long as each split keeps at least 2 chunks.
static int skinny_residual_blocks(int M, int N, int K) { return residual_narrow(M, N, K) ? N / 32 : (N / 32 + 1) / 2; }
static int skinny_residual_splits(int kc, int M, int N, int K) {
  const int n_chunks = (K + kc - 1) / kc;
  const int blocks = skinny_residual_blocks(M, N, K);
  int ks = (256 + blocks - 1) / blocks;
  ks = ks > kMaxResidualSplits ? kMaxResidualSplits : ks;
  while (ks > 1 && n_chunks / ks < 2) --ks;
  return ks < 1 ? 1 : ks;
}

// Which blocks gemm_tile_kernel takes of those that gemm_stream_kernel leaves (16-bit operands).  Above 128 rows: all.  Up to 128,
// measured on MI355X (skinny -> tiled, us, at 17 / 33 / 51 / 64-65 / 97 rows):
//  * residual GEMMs.  The tiled kernel reads X once per 64 columns of W instead of 32 and splits the contraction where that
//    fills the chip: output projection 4096 x 4096 8.4 -> 8.8 / 9.7 -> 9.0 / 11.0 -> 9.4 / 13.6 -> 12.2 / 16.7 -> 12.8, 768 x 768
//    4.9 -> 4.0 / 5.7 -> 4.1 / 6.6 -> 4.2 / 7.5 -> 3.9 / 9.1 -> 4.0; down 4096 x 14336 20.8 -> 21.6 / 21.8 -> 22.0 / 23.6 -> 22.8 /
//    26.8 -> 27.4 / 32.6 -> 28.4, 2048 x 5504 7.6 -> 7.7 / 8.5 -> 8.0 / 9.8 -> 8.1 / 9.9 -> 8.4 / 12.8 -> 10.1.  Where the skinny
//    kernel's workgroups come to more than one per CU the second round costs it most (3072-wide, 288 workgroups: down
//    16.2 -> 11.7 / 17.7 -> 11.8 / 19.4 -> 12.0 / 20.2 -> 12.3 / 28.3 -> 16.4, projection 8.1 -> 6.9 / 9.8 -> 7.1 / 11.4 -> 7.2).
//    Left to the skinny kernel: down of 65 to 96 rows on models 4096 to 5120 wide, where it computes 80 or 96 rows and a tile
//    128.  The 128 x 128 tiles take 25-26 us there on some cards and 30-33 on others (4096 x 14336; skinny 27-30), so that
//    8-layer steps of 81 to 93 rows came to 0.96-0.97 of the skinny kernel's on four cards and 1.00-1.03 on four.  Wider
//    models run 128 x 256 tiles, faster on all of them (8192 x 28672, 81-93 rows: steps 0.97-0.98).
//  * gate/up and q/k/v of 65 rows or more on narrow models, where one or two fragments per workgroup leave too little in
//    flight (768-wide, 97 rows, against kernels that staged X through LDS: 9.6 -> 7.1 and 9.9 -> 8.0; 65 rows 8.0 -> 7.1, 8.3 -> 8.0); wide
//    ones run gemm_stream_kernel (stream_takes has the figures).
static bool takes_tile(int epi, int M, int frags, int K, int tile_only) {
  if (M > 128 || (tile_only && M > 1)) return true;
  if (epi == EPI_UNEMBED || M <= 16) return false;
  if (epi != EPI_RESIDUAL) return M > 64 && frags <= 512;  // (up to 64 rows: gemm_stream_kernel)
  const int N = frags * 16;
  if (skinny_residual_blocks(M, N, K) * skinny_residual_splits(KChunk<half_t>::value, M, N, K) > 256) return true;
  return M > 24 && !(K > N && frags >= 256 && frags <= 320 && M > 64 && M <= 96);
}

// Split of the contraction across workgroups for the residual GEMMs
int gemm_residual_splits(int dtype, int M, int N, int K, int tile_only) {
  if (dtype == 1 && takes_tile(EPI_RESIDUAL, M, N / 16, K, tile_only)) return tile_plan(EPI_RESIDUAL, M, N / 16, K, tile_only).KS;
  return skinny_residual_splits(dtype == 1 ? KChunk<half_t>::value : KChunk<float>::value, M, N, K);
}

// fp32: the row tile the block needs.  16-bit: takes_tile leaves this kernel the blocks of up to 24 rows (up to 16 always in the
// 1 x 4 layout) and, in the 2 x 2 layout, those of 65 to 96; skinny_built holds what the instances reach.
static bool skinny_built(int dtype, int epi, int M, int N, int K) {
  if (epi == EPI_QKV || epi == EPI_GATEUP) return dtype == 0;
  return dtype == 0 || epi == EPI_UNEMBED || M <= (residual_narrow(M, N, K) ? 32 : 96);
}
template <typename T, int WN, int WK>
static bool launch_residual(const GemmCore &a, hipStream_t s) {
  if (!skinny_built(sizeof(T) == 2 ? 1 : 0, EPI_RESIDUAL, a.M, a.N, a.K)) return false;
  if constexpr (sizeof(T) == 4) launch_fm<T, EPI_RESIDUAL, WN, WK, 4>(a, a.KS, s);
  else if constexpr (WN == 1) {
    if (a.M <= 16) launch_gemm_cfg<T, EPI_RESIDUAL, 1, WN, WK, 4>(a, a.KS, s);
    else launch_gemm_cfg<T, EPI_RESIDUAL, 2, WN, WK, 4>(a, a.KS, s);
  } else {
    if (a.M <= 32) launch_gemm_cfg<T, EPI_RESIDUAL, 2, WN, WK, 4>(a, a.KS, s);
    else if (a.M <= 80) launch_gemm_cfg<T, EPI_RESIDUAL, 5, WN, WK, 4>(a, a.KS, s);
    else launch_gemm_cfg<T, EPI_RESIDUAL, 6, WN, WK, 4>(a, a.KS, s);
  }
  return true;
}

// Workgroup shapes measured on MI355X at the 7B shapes (60 rows).  Unembedding: wide tiles
// (WN = 4) where there are enough row groups to give every CU a workgroup, otherwise two waves per
// pair of groups; residual GEMMs: WN x WK = 2 x 2 or 1 x 4 (residual_narrow) with the contraction split
// across workgroups.
template <typename T>
static bool launch_skinny(int epi, const GemmCore &a_in, hipStream_t s) {
  GemmCore a = a_in;
  a.n_groups = gemm_groups(epi, a);
  const bool wide = a.n_groups >= 4 * 200;
  switch (epi) {
    case EPI_QKV:
      if constexpr (sizeof(T) == 4) { launch_paired<T, EPI_QKV>(a, s); return true; }
      return false;
    case EPI_GATEUP:
      if constexpr (sizeof(T) == 4) { launch_paired<T, EPI_GATEUP>(a, s); return true; }
      return false;
    case EPI_RESIDUAL:
      if (residual_narrow(a.M, a.N, a.K)) return launch_residual<T, 1, 4>(a, s);
      return launch_residual<T, 2, 2>(a, s);
    default:
      if (wide) launch_fm<T, EPI_UNEMBED, 4, 1, 8>(a, 1, s);
      else launch_fm<T, EPI_UNEMBED, 2, 2, 4>(a, 1, s);
      return true;
  }
}

// ---------------------------------------------------------------------------------------------
// One block token (the single-token decode step, and the blocks of one token a table build leaves over).  Such a step is
// a chain of short launches: the stream of W takes 5 to 34 us per GEMM at the 7B shapes and 1 us on a 768-wide model,
// while every launch costs 2 us and a latency chain of its own.  With one row the input of a GEMM is so small that every
// workgroup can build all of it: the kernel takes over the RMSNorm (residual partials, gain, sum of squares) and the merge
// of the attention slices, which as launches took 4.7 us (2.5-3.2 on the small model) each.  The row then sits in LDS
// once and the main loop has no barrier: W fragments stream through a register ring, the four waves split the steps and
// hand their sums over at the end.  Five launches per layer instead of eight; measured on the whole step: 7B, 2K context
// 3.55 -> 3.27 ms; 768 wide, 12 layers 510 -> 380 us.  Per launch at the 7B shapes (before: GEMM + norm or merge):
// q/k/v 18.4 + 4.7 -> 19.1, O 8.2 + 4.6 -> 9.3, gate/up 39.2 + 4.7 -> 39.6, down 19.6 -> 20.2 us.
//   PRO 0: X is row 0 of an activation buffer.  PRO 1: X = (h + residual partials) * gain, 1 / rms in the epilogue;
//   workgroup 0 stores the new residual stream to h_out (not over h: others still read it).  PRO 2: X = the merge of the
//   attention slices; the workgroups with blockIdx.x == 0 store it to attn_out.
// U: storage type of the gain.
// ---------------------------------------------------------------------------------------------
constexpr int kRowThreads = 256;

// q/k/v, gate/up: enough fragments per workgroup that 256 of them cover the matrix; residual: one or two fragments and a
// split contraction; unembedding: pairs
static int row_frags_per_wg(int epi, int frags) {
  if (epi == EPI_RESIDUAL) return frags <= 128 ? 1 : 2;
  int fn = (frags + 255) / 256;
  fn = fn > 8 ? 8 : fn;
  return epi == EPI_UNEMBED ? (fn + 1) / 2 * 2 : fn;
}
int gemm_row_splits(int N, int K) {
  const int wgs = N / 16 / row_frags_per_wg(EPI_RESIDUAL, N / 16);
  int ks = (256 + wgs - 1) / wgs;
  ks = ks > kMaxResidualSplits ? kMaxResidualSplits : ks;
  while (ks > 1 && K / 32 / ks < 8) --ks;                // at least two steps per wave
  return ks;
}
// the normalised row, and the merged attention output's share of a contraction split, have to fit the LDS
bool gemm_row_fits(int dtype, int d_model, int dq) {
  const int e = dtype == 1 ? 2 : 4;
  return (size_t)d_model * e <= 64 * 1024 && ((size_t)dq / gemm_row_splits(d_model, dq) + 64) * e <= 96 * 1024;
}

// NP: residual partials fetched at once (PRO 1), the number itself is r.n_part <= NP
template <typename U, typename T, int EPI, int FN, int RING, int PRO, int NP>
__global__ __launch_bounds__(kRowThreads) void gemm_row_kernel(const GemmCore a, const RowArgs r) {
  constexpr bool PAIRED = EPI == EPI_QKV || EPI == EPI_GATEUP;
  constexpr int KC = KChunk<T>::value, NW = 4;
  extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
  T *xs = reinterpret_cast<T *>(smem);                   // [K of this workgroup] (PRO 1, 2)
  __shared__ float sh[NW];
  const int tid = threadIdx.x, lane = tid & 63;
  const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
  const int li = lane & 15, g = lane >> 4;
  const int K = a.K, n_steps = K / 32, n_frags = a.n_groups;
  const int KS = gridDim.y, ks = blockIdx.y;
  const int s0 = n_steps * ks / KS, s1 = n_steps * (ks + 1) / KS;
  const int k0 = s0 * 32, kr = (s1 - s0) * 32;           // contraction elements of this workgroup
  const int f0 = blockIdx.x * FN;
  const int nt = s1 - s0 > wave ? (s1 - s0 - wave + NW - 1) / NW : 0;   // steps of this wave: s0 + wave, + 4, ...

  const T *wblk[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) wblk[f] = tiled_block((const T *)a.W0, min(f0 + f, n_frags - 1), n_steps, lane);
  Frag<T> ring[RING][FN], xring[PRO == 0 ? RING : 1];
  auto load_w = [&](int slot, int t) {                   // clamped into the matrix: loaded, never multiplied
    const int st = min(s0 + wave + NW * t, n_steps - 1);
#pragma unroll
    for (int f = 0; f < FN; ++f) ring[slot][f] = load_frag_stream(wblk[f] + (size_t)st * 512);
    // an input that is ready as it stands needs no staging: its 64 bytes of the step travel with the weights
    if constexpr (PRO == 0) xring[slot] = load_frag((const T *)a.X + (size_t)(st * 32 / KC) * a.Mcap * KC + st * 32 % KC + g * 8);
  };
  // The row's loads go out first (they come from the L2), the ring's behind them, so that the row can be waited for
  // while the weights are on their way; the scheduling barriers keep that order.
  auto fill_ring = [&]() {
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int u = 0; u < RING; ++u) load_w(u, u);
    __builtin_amdgcn_sched_barrier(0);
  };

  constexpr int J = NP <= 2 ? 4 : 2;                     // PRO 1: float4 groups per thread and round
  f32x4 hx[J];
  const int rounds = (K / 4 + J * kRowThreads - 1) / (J * kRowThreads);
  if constexpr (PRO == 1) {
    float ss = 0.0f;
    for (int rd = 0; rd < rounds; ++rd) {
      f32x4 p[J][NP], gn[J];
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int i = min(tid + (rd * J + j) * kRowThreads, K / 4 - 1);
        hx[j] = *reinterpret_cast<const f32x4 *>(r.h_in + 4 * i);
#pragma unroll
        for (int s = 0; s < NP; ++s)                     // surplus slots repeat the last partial (of none: the first) and are not added
          p[j][s] = *reinterpret_cast<const f32x4 *>(r.hpart + (size_t)max(min(s, r.n_part - 1), 0) * r.part_stride + 4 * i);
        const U *gp = (const U *)r.gain + 4 * i;
        gn[j] = f32x4{to_f32(gp[0]), to_f32(gp[1]), to_f32(gp[2]), to_f32(gp[3])};
      }
      if (rd == 0) fill_ring();
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int i = tid + (rd * J + j) * kRowThreads;
#pragma unroll
        for (int s = 0; s < NP; ++s) {                   // split order
          const bool add = s < r.n_part;
          hx[j] += f32x4{add ? p[j][s][0] : 0.f, add ? p[j][s][1] : 0.f, add ? p[j][s][2] : 0.f, add ? p[j][s][3] : 0.f};
        }
        const f32x4 x = hx[j];
        const float q = x[0] * x[0] + x[1] * x[1] + x[2] * x[2] + x[3] * x[3];
        ss += i < K / 4 ? q : 0.0f;
        if (i < K / 4) {
          store4(xs + 4 * i, x[0] * gn[j][0], x[1] * gn[j][1], x[2] * gn[j][2], x[3] * gn[j][3]);
          if (rd + 1 < rounds && r.n_part > 0 && blockIdx.x == 0) *reinterpret_cast<f32x4 *>(r.h_out + 4 * i) = x;
        }
      }
    }
#pragma unroll
    for (int off = 32; off > 0; off >>= 1) ss += __shfl_xor(ss, off);
    if (lane == 0) sh[wave] = ss;
    __syncthreads();
  } else if constexpr (PRO == 2) {
    // merge of the attention slices: 4 dims per thread and turn, the slices in order, eight at a time
    const int S = r.n_splits, hd = a.hd;
    constexpr int G = 2;                                 // turns whose first eight slices are fetched before the weights
    f32x4 v[G][8];
    float mm[G][8], ll[G][8];
    auto fetch = [&](int gi, int i, int t0) {
      const int k = k0 + 4 * min(i, kr / 4 - 1), h = k / hd, d = k - h * hd;
      const float *po = r.part_o + (size_t)h * S * hd + d, *ml = r.part_ml + (size_t)h * S * 2;
#pragma unroll
      for (int t = 0; t < 8; ++t) {
        const int sc = min(t0 + t, S - 1);
        v[gi][t] = *reinterpret_cast<const f32x4 *>(po + (size_t)sc * hd);
        mm[gi][t] = ml[sc * 2];
        ll[gi][t] = ml[sc * 2 + 1];
      }
    };
#pragma unroll
    for (int gi = 0; gi < G; ++gi) fetch(gi, tid + gi * kRowThreads, 0);
    fill_ring();
    // (the first eight slices apart from the loop over the rest: inside it their loads would be waited for together
    // with everything issued since, the weights included)
    auto finish = [&](int gi, int i) {
      float mrun = kNegBig, l = 0.0f;
      f32x4 o = f32x4{0.f, 0.f, 0.f, 0.f};
      auto add8 = [&](int t0) {
        float mnew = mrun;
#pragma unroll
        for (int t = 0; t < 8; ++t) mnew = fmaxf(mnew, t0 + t < S ? mm[gi][t] : kNegBig);
        const float alpha = part_exp<T>(mrun - mnew);
        l *= alpha;
        o *= alpha;
        mrun = mnew;
#pragma unroll
        for (int t = 0; t < 8; ++t) {
          const float wgt = t0 + t < S ? part_exp<T>(mm[gi][t] - mrun) : 0.0f;   // surplus slots repeat the last slice: weight 0
          l += ll[gi][t] * wgt;
          o += v[gi][t] * wgt;
        }
      };
      add8(0);
      for (int t0 = 8; t0 < S; t0 += 8) {
        fetch(gi, i, t0);
        add8(t0);
      }
      if (i < kr / 4) {
        const float inv = 1.0f / l;
        store4(xs + 4 * i, o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
        if (blockIdx.x == 0) store4((T *)r.attn_out + act_offset<T>(0, k0 + 4 * i, a.Mcap), o[0] * inv, o[1] * inv, o[2] * inv, o[3] * inv);
      }
    };
#pragma unroll
    for (int gi = 0; gi < G; ++gi) finish(gi, tid + gi * kRowThreads);
    for (int i = tid + G * kRowThreads; i < kr / 4; i += kRowThreads) {
      fetch(0, i, 0);
      finish(0, i);
    }
    __syncthreads();
  } else {
    fill_ring();
  }

  // ---- the stream of W; every column of the second operand is the row ---------------------------------
  f32x4 acc[FN];
#pragma unroll
  for (int f = 0; f < FN; ++f) acc[f] = f32x4{0.f, 0.f, 0.f, 0.f};
  for (int t0 = 0; t0 < nt; t0 += RING) {
#pragma unroll
    for (int u = 0; u < RING; ++u) {
      const int t = t0 + u;
      if (t < nt) {                                      // uniform per wave, no global load inside
        Frag<T> xf;
        if constexpr (PRO == 0) xf = xring[u];
        else xf = load_frag(xs + (wave + NW * t) * 32 + g * 8);
#pragma unroll
        for (int f = 0; f < FN; ++f) mma(acc[f], ring[u][f], xf);
      }
      load_w(u, t + RING);
    }
  }
  if constexpr (PRO == 1) {                              // the new residual stream (the last round's share of it), behind the stream of W
    if (r.n_part > 0 && blockIdx.x == 0)
#pragma unroll
      for (int j = 0; j < J; ++j) {
        const int i = tid + ((rounds - 1) * J + j) * kRowThreads;
        if (i < K / 4) *reinterpret_cast<f32x4 *>(r.h_out + 4 * i) = hx[j];
      }
  }
  float rs = a.out_scale;
  if constexpr (PRO == 1) rs *= 1.0f / sqrtf((((sh[0] + sh[1]) + sh[2]) + sh[3]) / (float)K + a.ss_eps);
  __syncthreads();                                       // everyone is done with xs
  f32x4 *red = reinterpret_cast<f32x4 *>(smem);          // [NW][FN][64]
#pragma unroll
  for (int f = 0; f < FN; ++f) red[(wave * FN + f) * 64 + lane] = acc[f];
  __syncthreads();
  auto total = [&](int f) {
    f32x4 t = red[f * 64 + lane];
#pragma unroll
    for (int o = 1; o < NW; ++o) t += red[(o * FN + f) * 64 + lane];
    return t;
  };
  if constexpr (EPI == EPI_UNEMBED) {
    for (int f = 2 * wave; f < FN; f += 2 * NW) {
      if (f0 + f >= n_frags) break;
      const int nbase[2] = {(f0 + f) * 16, (f0 + f + 1) * 16};
      const f32x4 sums[2] = {total(f), total(f + 1)};
      epi_unembed<2>(a, (f0 + f) / 2, li, li == 0, g, rs, nbase, sums);
    }
  } else {
    for (int f = wave; f < FN; f += NW) {
      if (f0 + f >= n_frags) break;                      // uniform per wave
      if constexpr (PAIRED) epi_paired<T, EPI>(a, f0 + f, li, 1, g, rs, total(f));
      else if (li == 0) epi_residual(a, ks, 0, (f0 + f) * 16, g, total(f));
    }
  }
}

template <typename U, int EPI, int FN, int PRO, int NP>
static void launch_row_np(const GemmCore &a, const RowArgs &r, int KS, hipStream_t s) {
  typedef typename Internal<U>::type T;
  // steps in flight per wave: as many 1 KB fragments as the registers hold without spilling (fp32 fragments are 2 KB)
  constexpr int RING = (sizeof(T) == 2 ? (FN >= 5 ? 3 : (FN >= 3 ? 5 : 8)) : (FN >= 5 ? 2 : (FN >= 3 ? 3 : 4)));
  const size_t row = PRO == 0 ? 0 : ((size_t)(a.K / 32 + KS - 1) / KS * 32) * sizeof(T);
  const size_t lds = std::max(row, (size_t)4 * FN * 1024);
  static const hipError_t opted = hipFuncSetAttribute(reinterpret_cast<const void *>(&gemm_row_kernel<U, T, EPI, FN, RING, PRO, NP>),
                                                      hipFuncAttributeMaxDynamicSharedMemorySize, 128 * 1024);
  (void)opted;
  hipLaunchKernelGGL((gemm_row_kernel<U, T, EPI, FN, RING, PRO, NP>), dim3((a.n_groups + FN - 1) / FN, KS), dim3(kRowThreads), lds, s, a, r);
}

template <typename U, int EPI, int FN, int PRO>
static void launch_row_cfg(const GemmCore &a, const RowArgs &r, int KS, hipStream_t s) {
  if constexpr (PRO == 1) {                              // narrow models split the residual GEMMs further (gemm_row_splits)
    if (r.n_part > 2) { launch_row_np<U, EPI, FN, PRO, kMaxResidualSplits>(a, r, KS, s); return; }
  }
  launch_row_np<U, EPI, FN, PRO, 2>(a, r, KS, s);
}

template <typename U, int EPI, int PRO>
static void launch_row_fn(const GemmCore &a, const RowArgs &r, int KS, hipStream_t s) {
  const int fn = row_frags_per_wg(EPI, a.n_groups);
  if constexpr (EPI == EPI_RESIDUAL) {
    if (fn == 1) launch_row_cfg<U, EPI, 1, PRO>(a, r, KS, s);
    else launch_row_cfg<U, EPI, 2, PRO>(a, r, KS, s);
  } else if constexpr (EPI == EPI_UNEMBED) {
    switch (fn) {
      case 2: launch_row_cfg<U, EPI, 2, PRO>(a, r, KS, s); break;
      case 4: launch_row_cfg<U, EPI, 4, PRO>(a, r, KS, s); break;
      case 6: launch_row_cfg<U, EPI, 6, PRO>(a, r, KS, s); break;
      default: launch_row_cfg<U, EPI, 8, PRO>(a, r, KS, s);
    }
  } else {
    switch (fn) {
      case 1: launch_row_cfg<U, EPI, 1, PRO>(a, r, KS, s); break;
      case 2: launch_row_cfg<U, EPI, 2, PRO>(a, r, KS, s); break;
      case 3: launch_row_cfg<U, EPI, 3, PRO>(a, r, KS, s); break;
      case 4: launch_row_cfg<U, EPI, 4, PRO>(a, r, KS, s); break;
      case 5: launch_row_cfg<U, EPI, 5, PRO>(a, r, KS, s); break;
      case 6: launch_row_cfg<U, EPI, 6, PRO>(a, r, KS, s); break;
      case 7: launch_row_cfg<U, EPI, 7, PRO>(a, r, KS, s); break;
      default: launch_row_cfg<U, EPI, 8, PRO>(a, r, KS, s);
    }
  }
}

template <typename U>
static void launch_row_t(int epi, const GemmCore &a_in, const RowArgs &r, hipStream_t s) {
  GemmCore a = a_in;
  a.n_groups = epi == EPI_RESIDUAL || epi == EPI_UNEMBED ? a.N / 16 : gemm_groups(epi, a);
  switch (epi) {
    case EPI_QKV: launch_row_fn<U, EPI_QKV, 1>(a, r, 1, s); break;
    case EPI_GATEUP: launch_row_fn<U, EPI_GATEUP, 1>(a, r, 1, s); break;
    case EPI_RESIDUAL:
      if (r.part_o) launch_row_fn<U, EPI_RESIDUAL, 2>(a, r, a.KS, s);
      else launch_row_fn<U, EPI_RESIDUAL, 0>(a, r, a.KS, s);
      break;
    default: launch_row_fn<U, EPI_UNEMBED, 1>(a, r, 1, s);
  }
}

int gemm_tile_shapes() { return kNumTileShapes; }

GemmPlan gemm_plan(int dtype, int epi, int M, int N, int K) {
  const int frags = epi == EPI_GATEUP ? N / 8 : N / 16;
  GemmPlan p{0, 0, 0, 1, frags, 0, 0};
  const GemmKernel kernel = M > 1 ? gemm_kernel(dtype, epi, M, frags, K, 0) : GEMM_ROW;
  if (kernel == GEMM_STREAM) {
    p.kernel = dtype == 1 && epi == EPI_RESIDUAL ? 3 : 0;
    if (dtype == 1 && (epi == EPI_QKV || epi == EPI_GATEUP)) p.tn = 16 * stream_paired_frags(frags);
    return p;
  }
  if (kernel == GEMM_TILE) {
    const TilePlan t = tile_plan(epi, M, frags, K, 0);
    const TileShape &s = kTileShapes[t.shape], &s2 = kTileShapes[t.shape2];
    return {1, s.tm, s.tn, t.KS, t.split, s2.tm, s2.tn};
  }
  if (epi == EPI_RESIDUAL) p.splits = M == 1 ? gemm_row_splits(N, K) : gemm_residual_splits(dtype, M, N, K);
  p.kernel = kernel;
  return p;
}

void launch_gemm_row(int dtype, int epi, const GemmCore &a, const RowArgs &r, hipStream_t s) {
  if (dtype == 1) launch_row_t<bf16_t>(epi, a, r, s);
  else launch_row_t<float>(epi, a, r, s);
}

GemmKernel gemm_kernel(int dtype, int epi, int M, int frags, int K, int tile_only) {
  if (stream_takes(dtype, epi, M, frags, K, tile_only)) return stream_built(dtype, epi, M) ? GEMM_STREAM : GEMM_NONE;
  if (dtype == 1 && takes_tile(epi, M, frags, K, tile_only)) return GEMM_TILE;
  return skinny_built(dtype, epi, M, frags * 16, K) ? GEMM_SKINNY : GEMM_NONE;
}

bool launch_gemm(int dtype, int epi, const GemmArgs &a, hipStream_t s) {
  const GemmKernel kernel = gemm_kernel(dtype, epi, a.M, epi == EPI_GATEUP ? a.N / 8 : a.N / 16, a.K, a.tile_only);
  // X lies in the other kernels' layout, or the output is asked for in one that only gemm_stream_kernel writes
  if ((kernel == GEMM_STREAM) != (a.x_mb != 0) || (kernel != GEMM_STREAM && a.act_mb)) return false;
  switch (kernel) {
    case GEMM_STREAM: return launch_gemm_stream(dtype, epi, a, s);
    case GEMM_TILE:
      switch (epi) {
        case EPI_QKV: launch_tile<EPI_QKV>(a, s); break;
        case EPI_GATEUP: launch_tile<EPI_GATEUP>(a, s); break;
        case EPI_RESIDUAL: launch_tile<EPI_RESIDUAL>(a, s); break;
        default: launch_tile<EPI_UNEMBED>(a, s);
      }
      return true;
    case GEMM_SKINNY: return dtype == 1 ? launch_skinny<half_t>(epi, a, s) : launch_skinny<float>(epi, a, s);
    default: return false;
  }
}

}  // namespace ngg
