// Skinny-M GEMM for weight-streaming projections: Y[M, N] = A[M, K] W[N, K]^T.
//
// Weights are pre-packed into 1 KB tiles of 16 output columns x KT k values
// (KT = 32 bf16 or 16 fp32) laid out so that lane l of a wavefront loads the
// 16 contiguous bytes W[n0 + l%16][k0 + (l/16)*KL ..] with one dwordx4 load;
// the tiles of one 16-column strip are contiguous along k.  One workgroup owns
// NG strips and the full K range; its waves split K into equal contiguous
// ranges that depend only on (N, K), and the wave partials are summed in LDS
// in wave order.  Every output element therefore sees the same reduction
// order whatever M is, which keeps results batch- and position-invariant.
// Up to SPLIT_MIN_ROWS rows; more rows go to the tiled kernel (gemm_tile.h).
#include <cmath>

#include "common.h"
#include "gemm.h"
#include "gemm_tile.h"

namespace dflow {

template <typename T, int NG, int MT, int EPI, bool NORM>
__global__ void __launch_bounds__(512) gemm_kernel(GemmParams p) {
  constexpr int KL = TT<T>::KL;
  constexpr int KT = TT<T>::KT;
  // k tiles per pipeline stage: 4 fragments of weights per stage and buffer
  constexpr int U = (MT * NG >= 8) ? 1 : 8 / (MT * NG);
  extern __shared__ float lds[];
  const int lane = threadIdx.x & 63;
  // wave index as a scalar: keeps the k-range bounds and the pipeline control uniform
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int nw = blockDim.x >> 6;
  // workgroup (strip group g, K part h): the K parts of a group sit on adjacent workgroups
  const int ks = p.ksplit > 1 ? p.ksplit : 1;
  const int g = blockIdx.x / ks, h = blockIdx.x - g * ks;
  const int nt0 = g * NG;
  const int nvalid = min(NG, p.ntiles - nt0);
  const int kpart = (p.ktiles + ks - 1) / ks;
  const int k0 = min(p.ktiles, h * kpart), k1 = min(p.ktiles, k0 + kpart);
  const int kper = (k1 - k0 + nw - 1) / nw;
  const int kb = min(k1, k0 + w * kper);
  const int ke = min(k1, kb + kper);
  const int M = p.M;
  const int mtiles = (M + 15) >> 4;

  // Explicit global address space: generic (flat) loads would also count
  // against the LDS counter and defeat the load pipelining below.  Weight
  // tiles are read by exactly one wave, once: they are loaded non-temporally,
  // so the weight stream does not evict the A rows, which every workgroup
  // re-reads from L2 (at the 8B down projection this takes a launch from
  // 23.8 to 20.2 us).
  const gu4* Wp = (const gu4*)(p.W);
  const T* Ap = reinterpret_cast<const T*>(p.A);

  f32x4_t acc[MT][NG];
#pragma unroll
  for (int i = 0; i < MT; ++i)
#pragma unroll
    for (int j = 0; j < NG; ++j) acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};

  // Out-of-range strips and rows are clamped to valid addresses instead of
  // being predicated, so the main loop is straight-line code; their results
  // land in columns/rows the epilogue never stores.
  const gu4* wrow[NG];
#pragma unroll
  for (int j = 0; j < NG; ++j) wrow[j] = Wp + (size_t)min(nt0 + j, p.ntiles - 1) * p.ktiles * 64 + lane;
  const gu4* arow[MT];
  // one k tile of A: 16 bytes per lane, 4 apart along a row-major row (16 row
  // pieces per load), or 64 apart in the matrix-core-order copy (1 KB contiguous)
  const int ast = p.Af ? 64 : KT * (int)sizeof(T) / 16;
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if (p.Af) {   // lanes of rows past M read the last row (never stored; few rows then touch few lines)
      const int rt = min(i, mtiles - 1);
      arow[i] = (const gu4*)(p.Af) + (size_t)rt * p.ktiles * 64 + (lane & 48) + min(lane & 15, M - 1 - rt * 16);
    } else {
      const int m = min(i * 16 + (lane & 15), M - 1);
      arow[i] = (const gu4*)(Ap + (size_t)m * p.lda + (lane >> 4) * KL);
    }
  }

  u32x4_t bq[2][U][NG];
  u32x4_t aq[2][U][MT];
#define DFLOW_LOAD(st, kt)                                                             \
  _Pragma("unroll") for (int u = 0; u < U; ++u) {                                       \
    _Pragma("unroll") for (int j = 0; j < NG; ++j) bq[st][u][j] = __builtin_nontemporal_load(&wrow[j][(size_t)((kt) + u) * 64]); \
    _Pragma("unroll") for (int i = 0; i < MT; ++i) aq[st][u][i] = arow[i][(size_t)((kt) + u) * ast]; \
  }                                                                                     \
  __builtin_amdgcn_sched_barrier(0);
#define DFLOW_COMPUTE(st)                                                              \
  _Pragma("unroll") for (int u = 0; u < U; ++u)                                         \
    _Pragma("unroll") for (int i = 0; i < MT; ++i)                                      \
      _Pragma("unroll") for (int j = 0; j < NG; ++j) acc[i][j] = mma_frag(T(), aq[st][u][i], bq[st][u][j], acc[i][j]);

  // RMSNorm row scales.  The norm gain is folded into the packed weight, so
  // the normalised projection is rs[m] * (x W'^T) and the scale is applied in
  // the epilogue.  rs comes from the per-strip sums of squares ssq[m][c] that
  // the producer of x left behind: lane q of a 16-lane group sums strips
  // c = q (mod 16) in increasing c, then a fixed butterfly over the group --
  // the same order for every row, batch and launch shape.  Group g owns rows
  // g + k * ngrp; the partials of strips c < 256 for its first two rows are
  // loaded early (see below) and consumed after the main loop, so the
  // reduction costs no latency on the critical path.
  constexpr int EL = 16;                  // early partials per lane and row
  const int q16 = threadIdx.x & 15, grp = threadIdx.x >> 4, ngrp = blockDim.x >> 4;
  float ea[NORM ? EL : 1], eb[NORM ? EL : 1];
  // The epilogue's own operand -- the residual rows (written by the previous
  // launch, so an L2 miss) or the bias -- for this thread's first PF outputs,
  // loaded early instead of after the main loop.
  constexpr bool EPF = EPI == EPI_RESID || EPI == EPI_BIAS_SILU || EPI == EPI_BIAS_F32;
  constexpr int PF = EPF ? 4 : 1;
  const int ncols = nvalid * 16;
  const int colbase = p.col0 + nt0 * 16;
  float pre[PF];
  // Early operand loads (row-scale partials, epilogue operand).  Loads
  // complete in order, so they are issued after the first matrix-core ops:
  // ahead of them they would hold up the pipeline start (the 8B QKV launch's
  // first stage landed 3.7 instead of 1.6 us after its start).
  auto prefetch = [&]() {
    if constexpr (NORM) {
      // rows of a group are clamped to valid rows and strips read the padded
      // row (ssq_ld >= 256 entries), so every load is unconditional
      gf32* ra = (gf32*)(p.ssq) + (size_t)min(grp, M - 1) * p.ssq_ld + q16;
      gf32* rb = (gf32*)(p.ssq) + (size_t)min(grp + ngrp, M - 1) * p.ssq_ld + q16;
#pragma unroll
      for (int it = 0; it < EL; ++it) {
        ea[it] = ra[16 * it];
        eb[it] = rb[16 * it];
      }
      __builtin_amdgcn_sched_barrier(0);
    }

    if constexpr (EPF) {
#pragma unroll
      for (int it = 0; it < PF; ++it) {
        const int e = threadIdx.x + it * (int)blockDim.x;
        const int m = min(e / ncols, M - 1), col = colbase + e % ncols;   // clamped: never used past M
        pre[it] = EPI == EPI_RESID ? TT<T>::ld(reinterpret_cast<const T*>(p.R), (size_t)m * p.ldr + col)
                                   : TT<T>::ld(reinterpret_cast<const T*>(p.bias), col);
      }
    }
  };

  // Full stages of U tiles, double-buffered.  Inside the steady-state loop
  // every load is unconditional, so the compiler's wait before each compute
  // covers only the stage being consumed, never the prefetch just issued.
  const int nst = (ke - kb) / U;
  int kt = kb;
  if (nst > 2) {
    // first iteration peeled: the early loads go out after its first stage
    DFLOW_LOAD(0, kt);
    DFLOW_LOAD(1, kt + U);
    DFLOW_COMPUTE(0);
    prefetch();
    DFLOW_LOAD(0, kt + 2 * U);
    DFLOW_COMPUTE(1);
    kt += 2 * U;
    int left = nst - 2;
    while (left > 2) {
      DFLOW_LOAD(1, kt + U);
      DFLOW_COMPUTE(0);
      DFLOW_LOAD(0, kt + 2 * U);
      DFLOW_COMPUTE(1);
      kt += 2 * U;
      left -= 2;
    }
    if (left == 2) {
      DFLOW_LOAD(1, kt + U);
      DFLOW_COMPUTE(0);
      DFLOW_COMPUTE(1);
      kt += 2 * U;
    } else {
      DFLOW_COMPUTE(0);
      kt += U;
    }
  } else {   // short range (a few stages)
    prefetch();
    if (nst > 0) {
      DFLOW_LOAD(0, kt);
      if (nst == 2) {
        DFLOW_LOAD(1, kt + U);
        DFLOW_COMPUTE(0);
        DFLOW_COMPUTE(1);
        kt += 2 * U;
      } else {
        DFLOW_COMPUTE(0);
        kt += U;
      }
    }
  }
  // ragged tail (fewer than U tiles)
  for (; kt < ke; ++kt) {
    u32x4_t b1[NG], a1[MT];
#pragma unroll
    for (int j = 0; j < NG; ++j) b1[j] = __builtin_nontemporal_load(&wrow[j][(size_t)kt * 64]);
#pragma unroll
    for (int i = 0; i < MT; ++i) a1[i] = arow[i][(size_t)kt * ast];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
      for (int j = 0; j < NG; ++j) acc[i][j] = mma_frag(T(), a1[i], b1[j], acc[i][j]);
  }
#undef DFLOW_LOAD
#undef DFLOW_COMPUTE

  __shared__ float s_rs[NORM ? MT * 16 : 1];
  if constexpr (NORM) {
    const int np = p.ssq_parts;
    for (int m0 = grp; m0 < MT * 16; m0 += 2 * ngrp) {
      const int ma = min(m0, M - 1), mb = min(m0 + ngrp, M - 1);
      float sa = 0.f, sb = 0.f;
      if (m0 == grp) {
#pragma unroll
        for (int it = 0; it < EL; ++it) {
          const bool ok = q16 + 16 * it < np;
          sa += ok ? ea[it] : 0.f;
          sb += ok ? eb[it] : 0.f;
        }
      } else {
        gf32* ra = (gf32*)(p.ssq) + (size_t)ma * p.ssq_ld + q16;
        gf32* rb = (gf32*)(p.ssq) + (size_t)mb * p.ssq_ld + q16;
        float la[EL], lb[EL];
#pragma unroll
        for (int it = 0; it < EL; ++it) {
          la[it] = ra[16 * it];
          lb[it] = rb[16 * it];
        }
#pragma unroll
        for (int it = 0; it < EL; ++it) {
          const bool ok = q16 + 16 * it < np;
          sa += ok ? la[it] : 0.f;
          sb += ok ? lb[it] : 0.f;
        }
      }
      for (int c = q16 + 16 * EL; c < np; c += 16) {   // strips beyond the early window (d > 4096)
        sa += p.ssq[(size_t)ma * p.ssq_ld + c];
        sb += p.ssq[(size_t)mb * p.ssq_ld + c];
      }
#pragma unroll
      for (int x = 8; x >= 1; x >>= 1) {
        sa += __shfl_xor(sa, x, 16);
        sb += __shfl_xor(sb, x, 16);
      }
      if (q16 == 0) {
        s_rs[m0] = rsqrtf(sa / (float)(np * 16) + p.eps);
        if (m0 + ngrp < MT * 16) s_rs[m0 + ngrp] = rsqrtf(sb / (float)(np * 16) + p.eps);
      }
    }
  }

  // ---- cross-wave reduction in fixed wave order, one m tile at a time
  float* red = lds;                                 // [nw][NG][64][4]
  constexpr int CW = NG * 16 + 1;                   // padded C-tile row
  float* ct = lds + (size_t)nw * NG * 256;          // [MT*16][CW]
#pragma unroll
  for (int i = 0; i < MT; ++i) {
    if (i >= mtiles) break;
#pragma unroll
    for (int j = 0; j < NG; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) red[((w * NG + j) * 64 + lane) * 4 + r] = acc[i][j][r];
    __syncthreads();
    for (int e = threadIdx.x; e < NG * 256; e += blockDim.x) {
      float s = 0.f;
      for (int ww = 0; ww < nw; ++ww) s += red[(size_t)ww * NG * 256 + e];
      const int j = e >> 8, l = (e >> 2) & 63, r = e & 3;
      ct[(i * 16 + 4 * (l >> 4) + r) * CW + j * 16 + (l & 15)] = s;
    }
    __syncthreads();
  }

  // ---- epilogue
  if constexpr (EPI == EPI_ARGMAX) {
    for (int e = threadIdx.x; e < M * ncols; e += blockDim.x) {
      const int m = e / ncols, n = e - m * ncols;
      float v = ct[m * CW + n];
      if constexpr (NORM) ct[m * CW + n] = v = v * s_rs[m];
      if (p.logits) p.logits[(size_t)m * p.ldl + colbase + n] = v;
    }
    __syncthreads();
    for (int m = threadIdx.x; m < M; m += blockDim.x) {
      float best = ct[m * CW];
      int bi = 0;
      for (int n = 1; n < ncols; ++n) {
        const float v = ct[m * CW + n];
        if (v > best) { best = v; bi = n; }
      }
      p.amax[(size_t)g * p.amax_ld + m] = argmax_key(best, colbase + bi);
    }
  } else if constexpr (EPI == EPI_SWIGLU) {
    // each packed strip holds 8 gate columns followed by the matching 8 up columns
    const int half = ncols / 2;
    const int obase = (p.col0 + nt0 * 16) / 2;
    for (int e = threadIdx.x; e < M * half; e += blockDim.x) {
      const int m = e / half, c = e - m * half;
      const int strip = c >> 3, cc = c & 7;
      float gt = ct[m * CW + strip * 16 + cc];
      float up = ct[m * CW + strip * 16 + 8 + cc];
      if constexpr (NORM) {
        gt *= s_rs[m];
        up *= s_rs[m];
      }
      const float y = silu(gt) * up;
      if (p.Y) TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + obase + c, y);
      frag_st<T>(p.yf, m, obase + c, y);
    }
  } else {
    // output e of this thread; x = the residual or bias value of its column
    auto out1 = [&](int e, float x) {
      const int m = e / ncols, n = e - m * ncols;
      const int col = colbase + n;
      float v = ct[m * CW + n];
      if constexpr (NORM) v *= s_rs[m];
      if constexpr (EPI == EPI_STORE_T) {
        TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + col, v);
      } else if constexpr (EPI == EPI_STORE_F32) {
        reinterpret_cast<float*>(p.Y)[(size_t)h * p.y_part + (size_t)m * p.ldy + col] = v;
      } else if constexpr (EPI == EPI_RESID) {
        v = TT<T>::rnd(v + x);
        TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + col, v);
        if (p.Y2) TT<T>::st(reinterpret_cast<T*>(p.Y2), (size_t)m * p.ldy2 + col, v);
        frag_st<T>(p.yf, m, col, v);
        frag_st<T>(p.y2f, m, col, v);
        ct[m * CW + n] = v;
      } else if constexpr (EPI == EPI_BIAS_SILU) {
        v += x;
        if (p.Y) TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + col, silu(v));
        frag_st<T>(p.yf, m, col, silu(v));
      } else if constexpr (EPI == EPI_BIAS_F32) {
        v += x;
        reinterpret_cast<float*>(p.Y)[(size_t)m * p.ldy + col] = v;
      }
    };
    const int nout = M * ncols;
#pragma unroll
    for (int it = 0; it < PF; ++it) {
      const int e = threadIdx.x + it * (int)blockDim.x;
      if (e < nout) out1(e, pre[it]);
    }
    for (int e = threadIdx.x + PF * (int)blockDim.x; e < nout; e += blockDim.x) {
      const int col = colbase + e % ncols;
      float x = 0.f;
      if constexpr (EPI == EPI_RESID)
        x = TT<T>::ld(reinterpret_cast<const T*>(p.R), (size_t)(e / ncols) * p.ldr + col);
      else if constexpr (EPI == EPI_BIAS_SILU || EPI == EPI_BIAS_F32)
        x = TT<T>::ld(reinterpret_cast<const T*>(p.bias), col);
      out1(e, x);
    }
    if constexpr (EPI == EPI_RESID) {
      if (p.ssq_out) {   // sum of squares of the stored values, per row and 16-column strip
        __syncthreads();
        for (int e = threadIdx.x; e < M * nvalid; e += blockDim.x) {
          const int m = e / nvalid, j = e - m * nvalid;
          p.ssq_out[(size_t)m * p.ssq_out_ld + nt0 + j] = strip_sq(ct + m * CW + j * 16);
        }
      }
    }
  }
}

// ------------------------------------------------------------------ large M
// Tile shapes of the many-row GEMM, and a launch's time by how the workgroups
// fall on the compute units.  Measured on the Qwen3 projections (8 x 64 .. 64 x
// 200 k tiles per workgroup, bf16): a workgroup's k tile takes t1 us when it has
// its compute unit to itself and tn when the unit holds several, one after
// another where the tile leaves no room for a second.  (Weights that come from
// HBM for the first time take longer alone: 64 x 64 0.16 to 0.20 us, 128 x 64 0.21
// to 0.23, 128 x 128 0.26 to 0.30.  The table only ranks launches, and those
// figures rank them worse.)
// LDS reads bound full launches: a wave of 64 x 32 reads 6 KB per 8 matrix ops,
// one of 64 x 64 8 KB per 16, so the widest tile takes 0.48 us a k tile for twice the
// work of the 128 x 128 one's 0.28 (8B LM head at 512 rows 695 -> 617 us, gate/up
// at 1024 rows 208 -> 190 us, 1.1 PFLOP/s) where it can fill the chip.  The
// smaller ones are for row counts and widths that would leave units idle (8B
// QKV at 128 rows 18.6 us at 128 x 128, 15.5 at 128 x 64; down at 1024 rows 107 us
// at 128 x 128, 142 at 256 x 128).
typedef TileShape<2, 4, 4, 2, 2> Tile128x128;
typedef TileShape<2, 2, 4, 2, 3> Tile128x64;
typedef TileShape<1, 4, 4, 2, 3> Tile64x128;
typedef TileShape<2, 2, 2, 2, 4> Tile64x64;
typedef TileShape<4, 2, 4, 4, 1> Tile256x128;
// fp32 is bound by the matrix cores (four ops of a quarter of the work per k
// tile), so no tile size saves time and the smallest fills the chip best: 64 x
// 64 takes 0.27 us a k tile alone and 0.24 in turn, where 128 x 128, four times the
// work, takes 0.96 to 1.1 (0.93 to 1.0 in turn).  It was the fastest of the four or
// within 1 % at 56 to 1024 rows of 512 to 32768 columns (400 x 32000 x 512: 112 us,
// 130 at 128 x 128), so fp32 has no other.
struct TileCost { int bm, bs; double t1, tn; };
constexpr TileCost TILES[] = {{128, 8, 0.26, 0.28}, {128, 4, 0.18, 0.165}, {64, 8, 0.19, 0.165}, {64, 4, 0.15, 0.115},
                              {256, 8, 0.38, 0.48}};
constexpr int N_TILES = sizeof(TILES) / sizeof(TILES[0]);
constexpr TileCost TILE_F32 = {64, 4, 0.27, 0.24};

// the fastest tile for M rows x ntiles strips x ktiles in ks K parts, and its time in us
template <typename T>
static int pick_tile(int M, int ntiles, int ktiles, int ks, int cus, double* us) {
  int best = 0;
  double tb = 1e30;
  for (int i = 0; i < (sizeof(T) == 2 ? N_TILES : 1); ++i) {
    const TileCost& c = sizeof(T) == 2 ? TILES[i] : TILE_F32;
    const long long wgs = (long long)((M + c.bm - 1) / c.bm) * ((ntiles + c.bs - 1) / c.bs) * ks;
    const long long n = (wgs + cus - 1) / cus;
    const double t = (double)n * ((ktiles + ks - 1) / ks) * (n == 1 ? c.t1 : c.tn);
    if (t < tb) {
      tb = t;
      best = i;
    }
  }
  *us = tb;
  return best;
}

template <typename T, int EPI, typename S>
static hipError_t launch_tile_shape(const GemmParams& p, int waves, int ks, hipStream_t st) {
  const int mt = (p.M + S::BM - 1) / S::BM, units = (p.ntiles + S::BS - 1) / S::BS * ks;
  const int blocks = (units + 7) / 8 * 8 * mt;
  // the ring needs more than the default dynamic LDS; set once per
  // instantiation (thread-safe static initialisation)
  constexpr size_t lds = S::STAGE * S::NS;
  static const hipError_t attr = hipFuncSetAttribute(reinterpret_cast<const void*>(&gemm_tile_kernel<T, EPI, S>),
                                                     hipFuncAttributeMaxDynamicSharedMemorySize, (int)lds);
  if (attr != hipSuccess) return attr;
  hipLaunchKernelGGL((gemm_tile_kernel<T, EPI, S>), dim3(blocks), dim3(S::NW * 64), lds, st, p, waves, mt, units);
  return hipGetLastError();
}

// K parts each folding `waves` ranges; the arithmetic of an output element does not depend on the tile.
template <typename T, int EPI>
static hipError_t launch_tile(const GemmParams& p, int waves, int ks, hipStream_t st) {
  if (!p.Af || (p.norm && !p.rs)) return hipErrorInvalidValue;
  double us;
  const int tile = pick_tile<T>(p.M, p.ntiles, p.ktiles, ks, p.cus > 0 ? p.cus : 256, &us);
  if constexpr (sizeof(T) == 2)
    switch (tile) {
      case 0: return launch_tile_shape<T, EPI, Tile128x128>(p, waves, ks, st);
      case 1: return launch_tile_shape<T, EPI, Tile128x64>(p, waves, ks, st);
      case 2: return launch_tile_shape<T, EPI, Tile64x128>(p, waves, ks, st);
      case 4: return launch_tile_shape<T, EPI, Tile256x128>(p, waves, ks, st);
    }
  return launch_tile_shape<T, EPI, Tile64x64>(p, waves, ks, st);
}

// Launch shape from (N, K) (and the K parts) only, never from M.  Wide weights (>= 1024
// strips) and the LM head take two 16-column strips per workgroup (the A
// fragments are reused across both); narrower ones take one so that enough
// workgroups exist.  The wave count (the K split) is the smallest power of
// two in 2..8 that puts at least 1024 waves in flight while leaving each wave
// at least 8 k tiles.  Chosen from a sweep over the 8B-shape projections at
// M = 16 with weights streamed from HBM.
GemmShape gemm_shape(int ntiles, int ktiles, int epi, int ksplit) {
  GemmShape s;
  s.ng = (epi == EPI_ARGMAX || ntiles >= 1024) ? 2 : 1;
  s.groups = (ntiles + s.ng - 1) / s.ng * ksplit;   // workgroups: strip groups x K parts
  const int kpart = (ktiles + ksplit - 1) / ksplit;
  int waves = 2;
  while (waves < 8 && (long long)s.groups * waves < 1024 && kpart / (2 * waves) >= 8) waves *= 2;
  s.waves = waves;
  return s;
}

// K parts for a projection whose consumer adds fp32 partial outputs: two when
// that spreads the strip groups more evenly over the compute units (every
// unit streams weights at about the same rate, so the slowest unit sets the
// time), one otherwise.  Depends only on (N, K) and the device.
int gemm_ksplit(int ntiles, int ktiles, int cus) {
  const GemmShape s = gemm_shape(ntiles, ktiles, EPI_STORE_F32, 1);
  if (cus < 1 || ktiles < 8) return 1;
  auto imbalance = [&](int ks) {
    const double per = (double)s.groups * ks / cus;
    return std::ceil(per) / per;
  };
  return imbalance(2) < imbalance(1) - 1e-9 ? 2 : 1;
}

template <typename T, int NG, int EPI, bool NORM>
static hipError_t launch_mtn(const GemmParams& p, const GemmShape& sh, hipStream_t st) {
  const int mt = (p.M + 15) / 16;
  const int cw = NG * 16 + 1;
  auto go = [&](auto kern, int MTv) {
    const size_t lds = ((size_t)sh.waves * NG * 256 + (size_t)MTv * 16 * cw) * sizeof(float);
    if (lds > 65536) return hipErrorInvalidConfiguration;
    hipLaunchKernelGGL(kern, dim3(sh.groups), dim3(sh.waves * 64), lds, st, p);
    return hipGetLastError();
  };
  if (mt <= 1) return go(gemm_kernel<T, NG, 1, EPI, NORM>, 1);
  if (mt <= 2) return go(gemm_kernel<T, NG, 2, EPI, NORM>, 2);
  return go(gemm_kernel<T, NG, 4, EPI, NORM>, 4);
}

// The RMSNorm row scale is instantiated only for the projections that follow a norm.
template <int EPI> struct HasNorm {
  static constexpr bool value = EPI == EPI_STORE_T || EPI == EPI_STORE_F32 || EPI == EPI_SWIGLU || EPI == EPI_ARGMAX;
};

template <typename T, int NG, int EPI>
static hipError_t launch_mt(const GemmParams& p, const GemmShape& sh, hipStream_t st) {
  if constexpr (HasNorm<EPI>::value) {
    if (p.norm) return launch_mtn<T, NG, EPI, true>(p, sh, st);
  } else {
    if (p.norm) return hipErrorInvalidValue;
  }
  return launch_mtn<T, NG, EPI, false>(p, sh, st);
}

template <typename T, int EPI>
static hipError_t launch_ng(const GemmParams& p, const GemmShape& sh, hipStream_t st) {
  return sh.ng == 2 ? launch_mt<T, 2, EPI>(p, sh, st) : launch_mt<T, 1, EPI>(p, sh, st);
}

// ---- K-part folds (launches of more than SPLIT_MIN_ROWS rows)
// The KS parts (KS > 0: all loads in flight at once; KS = 0: a loop over ks)
// of a thread's 16 columns, summed in part order from +0 -- the order in which
// the weight-streaming kernel adds its waves' ranges, so each row is
// bit-identical to that kernel's.
template <int KS>
__device__ inline void sum_parts16(const float* part, size_t part_stride, int ks, size_t off, float (&s)[16]) {
#pragma unroll
  for (int c = 0; c < 16; ++c) s[c] = 0.f;
  if constexpr (KS > 0) {
    float v[KS][16];
#pragma unroll
    for (int h = 0; h < KS; ++h) Row16<float>::load(part + h * part_stride + off, v[h]);
#pragma unroll
    for (int h = 0; h < KS; ++h)
#pragma unroll
      for (int c = 0; c < 16; ++c) s[c] += v[h][c];
  } else {
    for (int h = 0; h < ks; ++h) {
      float v[16];
      Row16<float>::load(part + h * part_stride + off, v);
#pragma unroll
      for (int c = 0; c < 16; ++c) s[c] += v[c];
    }
  }
}

// Residual epilogue: one workgroup per row, a thread per 16-column strip:
// rnd(sum + R) to Y (and Y2), the strip's sum of squares of the stored values
// and, from those in LDS, the row's RMSNorm scale for the next projection.
template <typename T, int KS>
__global__ void __launch_bounds__(256) resid_reduce_kernel(const float* part, size_t part_stride, int ks, int N,
                                                           const T* R, int ldr, T* Y, int ldy, T* Y2, int ldy2,
                                                           float* ssq_out, int ssq_ld, float* rs_out, float eps,
                                                           FragOut yf, FragOut y2f) {
  __shared__ float s_sq[SSQ_LD];
  const int nstrips = N / 16;
  const int m = blockIdx.x;
  for (int j = threadIdx.x; j < nstrips; j += blockDim.x) {
    float r[16], s[16];
    Row16<T>::load(R + (size_t)m * ldr + j * 16, r);
    sum_parts16<KS>(part, part_stride, ks, (size_t)m * N + j * 16, s);
#pragma unroll
    for (int c = 0; c < 16; ++c) s[c] = TT<T>::rnd(s[c] + r[c]);
    const float sq = strip_sq(s);
    Row16<T>::store(Y + (size_t)m * ldy + j * 16, s);
    if (Y2) Row16<T>::store(Y2 + (size_t)m * ldy2 + j * 16, s);
    frag_st_run<T>(yf, m, j * 16, s, 16);
    frag_st_run<T>(y2f, m, j * 16, s, 16);
    ssq_out[(size_t)m * ssq_ld + j] = sq;
    s_sq[j] = sq;
  }
  __syncthreads();
  row_scale_store(s_sq, nstrips, eps, rs_out + m);
}

int split_parts(int epi, int ntiles, int ktiles) { return gemm_shape(ntiles, ktiles, epi, 1).waves; }

// SwiGLU epilogue: one thread per (row, 16-column strip of 8 gate + 8 up
// columns), then the weight-streaming kernel's epilogue (row scale,
// silu(gate) * up, rounding).
template <typename T, int KS>
__global__ void __launch_bounds__(256) swiglu_reduce_kernel(GemmParams p, const float* part, size_t part_stride,
                                                            int ks, int N) {
  const int m = blockIdx.y;
  const int j = blockIdx.x * 256 + threadIdx.x;
  if (j >= N / 16) return;
  const float rs = p.norm ? p.rs[m] : 1.f;
  float s[16];
  sum_parts16<KS>(part, part_stride, ks, (size_t)m * N + j * 16, s);
  float y[8];
#pragma unroll
  for (int c = 0; c < 8; ++c) {
    float gt = s[c], up = s[8 + c];
    if (p.norm) {
      gt *= rs;
      up *= rs;
    }
    y[c] = silu(gt) * up;
    if (p.Y) TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + j * 8 + c, y[c]);
  }
  frag_st_run<T>(p.yf, m, j * 8, y, 8);
}

// Plain, fp32, bias + SiLU and bias epilogues: four columns per thread.
template <typename T, int EPI, int KS>
__global__ void __launch_bounds__(256) range_reduce_kernel(GemmParams p, const float* part, size_t part_stride,
                                                           int nw, int N) {
  const int m = blockIdx.y;
  const int c4 = blockIdx.x * 256 + threadIdx.x;
  if (c4 >= N / 4) return;
  const float rs = p.norm ? p.rs[m] : 1.f;
  float s[4] = {0.f, 0.f, 0.f, 0.f};
  const float* src = part + (size_t)m * N + 4 * c4;
  if constexpr (KS > 0) {   // all parts' loads in flight at once, summed in part order
    float4 v[KS];
#pragma unroll
    for (int w = 0; w < KS; ++w) v[w] = *reinterpret_cast<const float4*>(src + (size_t)w * part_stride);
#pragma unroll
    for (int w = 0; w < KS; ++w) {
      s[0] += v[w].x;
      s[1] += v[w].y;
      s[2] += v[w].z;
      s[3] += v[w].w;
    }
  } else {
    for (int w = 0; w < nw; ++w) {
      const float4 v = *reinterpret_cast<const float4*>(src + (size_t)w * part_stride);
      s[0] += v.x;
      s[1] += v.y;
      s[2] += v.z;
      s[3] += v.w;
    }
  }
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const int col = 4 * c4 + i;
    float v = s[i];
    if (p.norm) v *= rs;
    if constexpr (EPI == EPI_STORE_T) {
      TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + col, v);
    } else if constexpr (EPI == EPI_STORE_F32) {
      reinterpret_cast<float*>(p.Y)[(size_t)m * p.ldy + col] = v;
    } else if constexpr (EPI == EPI_BIAS_SILU) {
      v += TT<T>::ld(reinterpret_cast<const T*>(p.bias), col);
      if (p.Y) TT<T>::st(reinterpret_cast<T*>(p.Y), (size_t)m * p.ldy + col, silu(v));
      frag_st<T>(p.yf, m, col, silu(v));
    } else if constexpr (EPI == EPI_BIAS_F32) {
      v += TT<T>::ld(reinterpret_cast<const T*>(p.bias), col);
      reinterpret_cast<float*>(p.Y)[(size_t)m * p.ldy + col] = v;
    }
  }
}

// A launch's K parts: one (the tiles fold the ranges) or, where that leaves
// compute units idle, one per range (fp32 partial sums to part_ws, folded by a
// reduce kernel), whichever is estimated faster.  A reduce takes about 4 us
// plus its bytes at 6.5 TB/s (measured: four parts of 128 x 4096 5 us, of 1024
// x 4096 14.7 us), and so do the partial sums' writes.  The epilogue of a whole
// residual launch takes 4 us more than a plain store at small outputs and 8 to 22
// at 2 to 5 million (4 us + 3.5 per million); its parts were fitted with it: 6 us
// and 5 TB/s.  On 285 residual launches (56 .. 1024 rows of the Qwen3, small
// and tiny shapes' O and down, both ways measured) the choice is off by 42 us in
// sum, by 9 at most (8B down, 868 rows: 114 us, 105 in parts); charging the
// epilogue 3 us flat it was 217 and 36 (32B down, 640 rows: 219 us whole, 183 in
// parts; 8B O, 512 rows: 40.6 and 35.9).
template <typename T>
static int tile_parts(int epi, const GemmParams& p) {
  const int nw = split_parts(epi, p.ntiles, p.ktiles);
  if (nw < 2 || !p.part_ws || (epi != EPI_RESID && p.M > split_max_rows(epi))) return 1;
  const int cus = p.cus > 0 ? p.cus : 256;
  double whole, split;
  pick_tile<T>(p.M, p.ntiles, p.ktiles, 1, cus, &whole);
  pick_tile<T>(p.M, p.ntiles, p.ktiles, nw, cus, &split);
  const double outputs = (double)p.M * p.ntiles * 16, moved = 2.0 * nw * outputs * 4;   // the sums: written and read
  if (epi == EPI_RESID) return split + 6.0 + moved / 5.0e6 < whole + 4.0 + 3.5e-6 * outputs ? nw : 1;
  return split + 4.0 + moved / 6.5e6 < whole ? nw : 1;
}

// fp32 partial sums of ks parts (each folding `waves` ranges) to part_ws
template <typename T>
static hipError_t launch_parts(const GemmParams& p, int waves, int ks, GemmParams* q_out, hipStream_t st) {
  GemmParams q = p;   // the parts read A's matrix-core-order copy; the reduce writes the outputs
  q.yf = q.y2f = FragOut{nullptr, 0, 0};
  q.ksplit = ks;
  q.norm = 0;
  q.Y = p.part_ws;
  q.ldy = p.ntiles * 16;
  q.y_part = (size_t)p.M * q.ldy;
  q.col0 = 0;
  *q_out = q;
  return launch_tile<T, EPI_STORE_F32>(q, waves, ks, st);
}

// the part count as a template argument where it is a wave count, so all loads are in flight at once
template <typename F>
static hipError_t with_parts(int ks, F&& go) {
  if (ks == 2) return go(std::integral_constant<int, 2>{});
  if (ks == 4) return go(std::integral_constant<int, 4>{});
  if (ks == 8) return go(std::integral_constant<int, 8>{});
  return go(std::integral_constant<int, 0>{});
}

template <typename T, int EPI>
static hipError_t launch_range_reduce(const GemmParams& p, const GemmParams& q, int ks, hipStream_t st) {
  return with_parts(ks, [&](auto k) {
    hipLaunchKernelGGL((range_reduce_kernel<T, EPI, decltype(k)::value>), dim3((q.ldy / 4 + 255) / 256, p.M), dim3(256),
                       0, st, p, p.part_ws, q.y_part, ks, q.ldy);
    return hipGetLastError();
  });
}

template <typename T>
static hipError_t launch_many(int epi, const GemmParams& p, hipStream_t st) {
  const int ks = p.ksplit > 1 ? p.ksplit : 1;
  const int waves = gemm_shape(p.ntiles, p.ktiles, epi, ks).waves;
  if (ks > 1) return epi == EPI_STORE_F32 ? launch_tile<T, EPI_STORE_F32>(p, waves, ks, st) : hipErrorInvalidValue;
  const int parts = epi == EPI_ARGMAX ? 1 : tile_parts<T>(epi, p);
  GemmParams q;
  hipError_t e;
  if (epi == EPI_RESID) {
    if (p.norm || p.col0 || !p.ssq_out || !p.rs_out || !p.arrive) return hipErrorInvalidValue;
    if (parts == 1) return launch_tile<T, EPI_RESID>(p, waves, 1, st);
    if ((e = launch_parts<T>(p, 1, parts, &q, st)) != hipSuccess) return e;
    const int threads = p.ntiles < 256 ? (p.ntiles + 63) / 64 * 64 : 256;
    return with_parts(parts, [&](auto k) {
      hipLaunchKernelGGL((resid_reduce_kernel<T, decltype(k)::value>), dim3(p.M), dim3(threads), 0, st, p.part_ws,
                         q.y_part, parts, q.ldy, reinterpret_cast<const T*>(p.R), p.ldr, reinterpret_cast<T*>(p.Y),
                         p.ldy, reinterpret_cast<T*>(p.Y2), p.ldy2, p.ssq_out, p.ssq_out_ld, p.rs_out, p.eps, p.yf,
                         p.y2f);
      return hipGetLastError();
    });
  }
  if (parts > 1) {
    if ((e = launch_parts<T>(p, 1, parts, &q, st)) != hipSuccess) return e;
    switch (epi) {
      case EPI_STORE_T: return launch_range_reduce<T, EPI_STORE_T>(p, q, parts, st);
      case EPI_STORE_F32: return launch_range_reduce<T, EPI_STORE_F32>(p, q, parts, st);
      case EPI_BIAS_SILU: return launch_range_reduce<T, EPI_BIAS_SILU>(p, q, parts, st);
      case EPI_BIAS_F32: return launch_range_reduce<T, EPI_BIAS_F32>(p, q, parts, st);
      case EPI_SWIGLU:
        return with_parts(parts, [&](auto k) {
          hipLaunchKernelGGL((swiglu_reduce_kernel<T, decltype(k)::value>), dim3((p.ntiles + 255) / 256, p.M),
                             dim3(256), 0, st, p, p.part_ws, q.y_part, parts, q.ldy);
          return hipGetLastError();
        });
    }
    return hipErrorInvalidValue;
  }
  switch (epi) {
    case EPI_STORE_T: return launch_tile<T, EPI_STORE_T>(p, waves, 1, st);
    case EPI_STORE_F32: return launch_tile<T, EPI_STORE_F32>(p, waves, 1, st);
    case EPI_SWIGLU: return launch_tile<T, EPI_SWIGLU>(p, waves, 1, st);
    case EPI_BIAS_SILU: return launch_tile<T, EPI_BIAS_SILU>(p, waves, 1, st);
    case EPI_BIAS_F32: return launch_tile<T, EPI_BIAS_F32>(p, waves, 1, st);
    case EPI_ARGMAX: return launch_tile<T, EPI_ARGMAX>(p, waves, 1, st);
  }
  return hipErrorInvalidValue;
}

template <typename T>
static hipError_t launch_t(int epi, const GemmParams& p, hipStream_t st) {
  if (p.M > SPLIT_MIN_ROWS) return launch_many<T>(epi, p, st);
  const int ks = p.ksplit > 1 ? p.ksplit : 1;
  if (ks > 1 && epi != EPI_STORE_F32) return hipErrorInvalidValue;   // only partial fp32 outputs are split
  const GemmShape sh = gemm_shape(p.ntiles, p.ktiles, epi, ks);
  switch (epi) {
    case EPI_STORE_T: return launch_ng<T, EPI_STORE_T>(p, sh, st);
    case EPI_STORE_F32: return launch_ng<T, EPI_STORE_F32>(p, sh, st);
    case EPI_RESID: return launch_ng<T, EPI_RESID>(p, sh, st);
    case EPI_SWIGLU: return launch_ng<T, EPI_SWIGLU>(p, sh, st);
    case EPI_BIAS_SILU: return launch_ng<T, EPI_BIAS_SILU>(p, sh, st);
    case EPI_BIAS_F32: return launch_ng<T, EPI_BIAS_F32>(p, sh, st);
    case EPI_ARGMAX: return launch_mt<T, 2, EPI_ARGMAX>(p, sh, st);
  }
  return hipErrorInvalidValue;
}

hipError_t launch_gemm(bool bf16, int epi, const GemmParams& p, hipStream_t st) {
  if (p.M <= 0 || p.ntiles <= 0 || p.ktiles <= 0) return hipSuccess;
  return bf16 ? launch_t<dflow::bf16>(epi, p, st) : launch_t<float>(epi, p, st);
}

// ------------------------------------------------------------------ packing
// out tile (nt, kt) lane l element e <- W[src_row(nt, l%16)][kt*KT + (l/16)*KL + e] * gain[col]
// gate_up: W is [2F, K] = [gate; up]; packed strip i holds gate rows 8i..8i+7
// followed by up rows 8i..8i+7, so one strip yields 8 SwiGLU outputs.  The
// optional column gain (the RMSNorm gain of the rows this weight multiplies)
// is applied in fp32 and rounded once to the storage type.
template <typename T>
__global__ void pack_kernel(const T* __restrict__ W, int N, int K, int gate_up, const T* __restrict__ gain,
                            T* __restrict__ out) {
  constexpr int KL = TT<T>::KL, KT = TT<T>::KT;
  const int ktiles = K / KT;
  const size_t total = (size_t)N * K;
  for (size_t o = (size_t)blockIdx.x * blockDim.x + threadIdx.x; o < total; o += (size_t)gridDim.x * blockDim.x) {
    const int e = (int)(o % KL);
    const size_t lt = o / KL;
    const int l = (int)(lt % 64);
    const size_t tile = lt / 64;
    const int kt = (int)(tile % ktiles);
    const int nt = (int)(tile / ktiles);
    const int r16 = l & 15;
    size_t row = (size_t)nt * 16 + r16;
    if (gate_up) row = (r16 < 8) ? (size_t)nt * 8 + r16 : (size_t)N / 2 + (size_t)nt * 8 + (r16 - 8);
    const size_t col = (size_t)kt * KT + (l >> 4) * KL + e;
    if (gain)
      TT<T>::st(out, o, TT<T>::ld(W, row * K + col) * TT<T>::ld(gain, col));
    else
      out[o] = W[row * K + col];
  }
}

hipError_t launch_pack(bool bf16, const void* w, int N, int K, int gate_up, const void* col_gain, void* out,
                       hipStream_t s) {
  const int threads = 256;
  const size_t total = (size_t)N * K;
  int blocks = (int)((total + threads - 1) / threads);
  if (blocks > 65536) blocks = 65536;
  if (bf16)
    hipLaunchKernelGGL(pack_kernel<dflow::bf16>, dim3(blocks), dim3(threads), 0, s, (const dflow::bf16*)w, N, K,
                       gate_up, (const dflow::bf16*)col_gain, (dflow::bf16*)out);
  else
    hipLaunchKernelGGL(pack_kernel<float>, dim3(blocks), dim3(threads), 0, s, (const float*)w, N, K, gate_up,
                       (const float*)col_gain, (float*)out);
  return hipGetLastError();
}

}  // namespace dflow
