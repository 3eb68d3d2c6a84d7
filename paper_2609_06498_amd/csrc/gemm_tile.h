// Tiled GEMM for many rows (included by gemm.hip): Y[M, N] = A[M, K] W[N, K]^T
// with A in its matrix-core-order copy (afrag_off) and W packed.
//
// Workgroup tile: NWM x NWN waves of 16 WM rows x WN strips of 16 columns each
// (1 x 4 to 4 x 2 waves, 64 x 64 to 256 x 128).  A stage is one k tile of both
// operands, a 1 KB tile per 16 rows and per strip, already in fragment order in
// memory, so each goes to LDS with one load-to-LDS instruction of a wave (no
// registers, no LDS writes by the waves).  NS stages sit in an LDS ring.
//
// A step works on stage s, whose fragments are in registers or on their way
// there.  It waits until this wave's loads of stage s + 1 have landed (those of s
// + 2 .. s + NS - 1 stay in flight) and its own LDS reads are done, and meets the
// other waves: every wave has now read stage s and sees s + 1 whole.  The ring
// slot of s takes the loads of stage s + NS, the fragments of s + 1 are read, and
// the matrix cores multiply stage s meanwhile.  One barrier per stage.
//
// Arithmetic: the K loop runs the weight-streaming kernel's wave ranges
// (gemm_shape) in order, each range one matrix-core chain from zero, folded
// into the running sum in range order from +0, so every output element is
// bit-identical to what that kernel computes for it at any M.  The operands
// are swapped (W first): a lane then holds four consecutive columns of one
// row, and the epilogues store vectors straight from registers.
#pragma once
#include "common.h"
#include "gemm.h"

namespace dflow {

// two consecutive values (even column)
template <typename T> __device__ __forceinline__ void pair_st(T* p, float a, float b);
template <> __device__ __forceinline__ void pair_st<bf16>(bf16* p, float a, float b) {
  *reinterpret_cast<uint32_t*>(p) = f2bf2(a, b);
}
template <> __device__ __forceinline__ void pair_st<float>(float* p, float a, float b) {
  *reinterpret_cast<float2*>(p) = make_float2(a, b);
}

constexpr size_t TILE_LDS_CU = 156 * 1024;

// Tile shape: NWM x NWN waves of 16 WM rows x WN strips, OCC workgroups per compute unit.
template <int NWM_, int NWN_, int WM_, int WN_, int OCC_>
struct TileShape {
  static constexpr int NWM = NWM_, NWN = NWN_, WM = WM_, WN = WN_, OCC = OCC_;
  static constexpr int NW = NWM * NWN, BM = 16 * NWM * WM, BS = NWN * WN;   // waves, rows, strips
  static constexpr int AT = NWM * WM, TPS = AT + BS;                        // 1 KB tiles per stage: A, both
  static constexpr int LPW = TPS / NW;                                      // loads per wave and stage
  static constexpr size_t STAGE = (size_t)TPS * 1024;
  static constexpr int FIT = (int)(TILE_LDS_CU / OCC / STAGE), NS = FIT < 8 ? FIT : 8;   // ring depth
  static_assert(TPS % NW == 0 && NS >= 3 && (NS - 1) * LPW < 64, "loads, ring depth, vmcnt range");
};

// Residual epilogue: rnd(sum + R) to Y (and Y2) and the matrix-core-order
// copies, the sum of squares of every 16-column strip, and from those the row's RMSNorm
// scale.  The scale needs the whole row, so the workgroup of a row tile that
// arrives last computes its rows' scales.  The strip sums are written and read
// with device-scope accesses (no cache write-back), each wave waits for its
// writes before the workgroup counts its arrival, and the last one resets the
// counter.  A separate pass over fp32 sums took 17.7 us after the 8B O and down
// projections at 1024 rows; in the epilogue it adds about 10 (O and down 75 ->
// 86 us on average), and at 512 rows of the 1.7B shape O takes 21.5 us in place
// of 19.0 + 5.7.
template <typename T, typename S>
__device__ __forceinline__ void resid_epilogue(const GemmParams& p, const f32x4_t (&tot)[S::WM][S::WN], int rt0,
                                               int nt0, int wm, int wn, int mtile, int arrivals, int* s_last) {
  constexpr int WM = S::WM, WN = S::WN;
  const int lane = threadIdx.x & 63, q = lane >> 4, c16 = lane & 15;
  float r[WM][WN][4];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) {              // (rows and strips past the end: valid ones, not stored)
      const int m = min((rt0 + wm * WM + i) * 16 + c16, p.M - 1);
      const int nt = min(nt0 + wn * WN + j, p.ntiles - 1);
      Run4<T>::load(reinterpret_cast<const T*>(p.R) + (size_t)m * p.ldr + nt * 16 + 4 * q, r[i][j]);
    }
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int m = (rt0 + wm * WM + i) * 16 + c16;
#pragma unroll
    for (int j = 0; j < WN; ++j) {
      const int nt = nt0 + wn * WN + j, col = nt * 16 + 4 * q;
      const bool ok = m < p.M && nt < p.ntiles;
      float v[4];
#pragma unroll
      for (int e = 0; e < 4; ++e) v[e] = TT<T>::rnd(tot[i][j][e] + r[i][j][e]);
      if (ok) {
        Run4<T>::store(reinterpret_cast<T*>(p.Y) + (size_t)m * p.ldy + col, v);
        if (p.Y2) Run4<T>::store(reinterpret_cast<T*>(p.Y2) + (size_t)m * p.ldy2 + col, v);
        if (p.yf.p) frag_st4<T>(p.yf, m, col, v);
        if (p.y2f.p) frag_st4<T>(p.y2f, m, col, v);
      }
      // strip_sq, lane group by lane group
      float sq = 0.f;
#pragma unroll
      for (int g = 0; g < 4; ++g) {
        if (g > 0) sq = __shfl(sq, (g - 1) * 16 + c16, 64);
        if (q == g) {
          sq = g == 0 ? sq_start(v[0], v[1]) : sq_next(sq_next(sq, v[0]), v[1]);
          sq = sq_next(sq_next(sq, v[2]), v[3]);
        }
      }
      if (ok && q == 3)
        __hip_atomic_store(p.ssq_out + (size_t)m * p.ssq_out_ld + nt, sq, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
  }
  asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  __syncthreads();                              // (and no wave reads its operand tiles any more)
  if (threadIdx.x == 0)
    *s_last = __hip_atomic_fetch_add(p.arrive + mtile, 1u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT) ==
              (unsigned)arrivals - 1;
  __syncthreads();
  if (!*s_last) return;                         // uniform
  // row_scale_store's order: lane x of 16 sums strips x, x + 16, ..., then a butterfly.
  // RB rows of a lane group at once, 16 strips each: that many loads in flight.
  constexpr int GROUPS = S::NW * 4, RB = S::BM / GROUPS < 4 ? S::BM / GROUPS : 4, EL = 16;
  const int np = p.ntiles, grp = threadIdx.x >> 4, x = threadIdx.x & 15;
  for (int b0 = grp; b0 < S::BM; b0 += RB * GROUPS) {
    float s[RB];
#pragma unroll
    for (int b = 0; b < RB; ++b) s[b] = 0.f;
    for (int c0 = x; c0 < np; c0 += 16 * EL) {
      float v[RB][EL];
#pragma unroll
      for (int b = 0; b < RB; ++b) {
        const float* row = p.ssq_out + (size_t)min(rt0 * 16 + b0 + b * GROUPS, p.M - 1) * p.ssq_out_ld;
#pragma unroll
        for (int e = 0; e < EL; ++e)
          v[b][e] = __hip_atomic_load(row + min(c0 + 16 * e, np - 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
      }
#pragma unroll
      for (int b = 0; b < RB; ++b)
#pragma unroll
        for (int e = 0; e < EL; ++e)
          if (c0 + 16 * e < np) s[b] += v[b][e];
    }
#pragma unroll
    for (int b = 0; b < RB; ++b) {
#pragma unroll
      for (int o = 8; o >= 1; o >>= 1) s[b] += __shfl_xor(s[b], o, 16);
      const int m = rt0 * 16 + b0 + b * GROUPS;
      if (x == 0 && m < p.M) p.rs_out[m] = rsqrtf(s[b] / (float)(np * 16) + p.eps);
    }
  }
  if (threadIdx.x == 0) __hip_atomic_store(p.arrive + mtile, 0u, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

template <typename T, int EPI, typename S>
__global__ void __launch_bounds__(S::NW * 64, S::OCC * S::NW / 4) gemm_tile_kernel(GemmParams p, int nw, int mt,
                                                                                   int units) {
  constexpr int WM = S::WM, WN = S::WN, NS = S::NS, LPW = S::LPW;
  constexpr uint32_t STAGE = (uint32_t)S::STAGE;
  extern __shared__ __align__(16) unsigned char tile_smem[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int wm = w / S::NWN, wn = w % S::NWN;
  // block -> (m tile, unit = strip tile x K part); the m tiles of a unit share
  // an XCD (round-robin placement, id mod 8), so its weights are fetched once
  const int x8 = blockIdx.x & 7, y = blockIdx.x >> 3;
  const int mtile = y % mt, unit = (y / mt) * 8 + x8;
  if (unit >= units) return;                   // padding of the dispatch grid
  const int ks = p.ksplit > 1 ? p.ksplit : 1;
  const int stile = unit / ks, h = unit - stile * ks;
  const int nt0 = stile * S::BS;
  const int rt0 = mtile * S::AT;               // first 16-row tile
  const int kpart = (p.ktiles + ks - 1) / ks;
  const int k0 = min(p.ktiles, h * kpart), k1 = min(p.ktiles, k0 + kpart);
  const int kper = max(1, (k1 - k0 + nw - 1) / nw);
  const int nst = k1 - k0;                     // stages
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)tile_smem + w * 1024;

  // this wave's loads of a stage: tiles w + NW i of its row tiles, then strips
  // (clamped to valid ones: rows and strips past the end are never stored)
  const char* src[LPW];
#pragma unroll
  for (int i = 0; i < LPW; ++i) {
    const int idx = w + S::NW * i;
    src[i] = idx < S::AT ? (const char*)p.Af + (size_t)min(rt0 + idx, (p.M + 15) / 16 - 1) * p.ktiles * 1024
                         : (const char*)p.W + (size_t)min(nt0 + idx - S::AT, p.ntiles - 1) * p.ktiles * 1024;
  }
  // loads of stage s into the ring slot at LDS offset SLOT * STAGE past `base`
  const uint32_t voff = lane * 16;
  auto issue = [&]<int SLOT>(std::integral_constant<int, SLOT>, int s, uint32_t base) {
    static_for<LPW>([&]<int I>(std::integral_constant<int, I>) {
      load_to_lds<SLOT * (int)STAGE + S::NW * I * 1024>(base, src[I], (uint32_t)(k0 + s) * 1024 + voff);
    });
  };

  f32x4_t acc[WM][WN], tot[WM][WN];
#pragma unroll
  for (int i = 0; i < WM; ++i)
#pragma unroll
    for (int j = 0; j < WN; ++j) acc[i][j] = tot[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  int left = kper;                              // k tiles to the end of the current range
  auto fold = [&]() {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) {
#pragma unroll
        for (int r = 0; r < 4; ++r) tot[i][j][r] += acc[i][j][r];
        acc[i][j] = f32x4_t{0.f, 0.f, 0.f, 0.f};
      }
    left = kper;
  };
  u32x4_t fa[2][WM], fb[2][WN];                 // fragments of the stage being multiplied and of the next one
  auto frags = [&](int slot, int f) {
    const u32x4_t* t = reinterpret_cast<const u32x4_t*>(tile_smem + (size_t)slot * STAGE);
#pragma unroll
    for (int j = 0; j < WN; ++j) fb[f][j] = t[(S::AT + wn * WN + j) * 64 + lane];
#pragma unroll
    for (int i = 0; i < WM; ++i) fa[f][i] = t[(wm * WM + i) * 64 + lane];
  };
  auto mul = [&](int f) {
#pragma unroll
    for (int i = 0; i < WM; ++i)
#pragma unroll
      for (int j = 0; j < WN; ++j) acc[i][j] = mma_frag(T(), fb[f][j], fa[f][i], acc[i][j]);
    if (--left == 0) fold();
  };
  if (nst > 0) {
    constexpr std::integral_constant<int, 0> Z{};
    const int pre = min(nst, NS);
    for (int s = 0; s < pre; ++s) issue(Z, s, lds0 + s * STAGE);
    if (nst >= NS) wait_barrier<(NS - 1) * LPW>();
    else wait_barrier<0>();
    frags(0, 0);
    // steady state, unrolled over the ring (and the two fragment sets)
    constexpr int U = NS % 2 == 0 ? NS : 2 * NS;
    int s = 0;
    for (; s + NS + U - 1 < nst; s += U)
      static_for<U>([&]<int I>(std::integral_constant<int, I>) {
        constexpr int slot = I % NS, nxt = (I + 1) % NS;
        wait_barrier<(NS - 2) * LPW>();
        issue(std::integral_constant<int, slot>{}, s + I + NS, lds0);
        frags(nxt, (I & 1) ^ 1);
        mul(I & 1);
      });
    // the rest, two stages at a time
    int slot = 0;                               // s is a multiple of NS here
    auto advance = [&](int x, int f) {
      if (x + NS <= nst) wait_barrier<(NS - 2) * LPW>();
      else wait_barrier<0>();
      if (x + NS < nst) issue(Z, x + NS, lds0 + slot * STAGE);
      slot = slot + 1 == NS ? 0 : slot + 1;
      frags(slot, f);
    };
    for (; s + 2 < nst; s += 2) {
      advance(s, 1);
      mul(0);
      advance(s + 1, 0);
      mul(1);
    }
    const bool two = s + 1 < nst;
    if (two) advance(s, 1);
    mul(0);
    if (two) mul(1);
    if (left != kper) fold();                   // the last, shorter range
  }
  // (ranges past the end are empty: their partial sums are +0, and adding +0
  // to a sum that started from +0 changes nothing)

  // ---- epilogue: element r of acc tile (i, j) is row 16 i + lane % 16, column 4 (lane / 16) + r of strip j
  const int q = lane >> 4, c16 = lane & 15;
  const int colbase = p.col0;
  if constexpr (EPI == EPI_RESID) {
    resid_epilogue<T, S>(p, tot, rt0, nt0, wm, wn, mtile, units, reinterpret_cast<int*>(tile_smem));
    return;
  }
#pragma unroll
  for (int i = 0; i < WM; ++i) {
    const int m = (rt0 + wm * WM + i) * 16 + c16;
    const bool row = m < p.M;
    const float rs = p.norm ? p.rs[row ? m : p.M - 1] : 1.f;
    if constexpr (EPI == EPI_ARGMAX) {
      // one key per row and group of two strips, as the weight-streaming
      // kernel's workgroups: the largest value, lowest column on ties; a NaN
      // wins only as a group's first column
      static_assert(WN % 2 == 0, "strip pairs within a wave");
#pragma unroll
      for (int j = 0; j < WN; j += 2) {
        const int nt = nt0 + wn * WN + j;
        if (nt >= p.ntiles) break;             // uniform
        const bool pair = nt + 1 < p.ntiles;
        float v[8];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
          v[r] = p.norm ? tot[i][j][r] * rs : tot[i][j][r];
          v[4 + r] = p.norm ? tot[i][j + 1][r] * rs : tot[i][j + 1][r];
        }
        if (p.logits && row) {
          float* o = p.logits + (size_t)m * p.ldl + colbase + nt * 16 + 4 * q;
          // (the caller's buffer: aligned as floats are, not to 16 bytes)
          typedef float run_t __attribute__((ext_vector_type(4), aligned(4)));
          *reinterpret_cast<run_t*>(o) = run_t{v[0], v[1], v[2], v[3]};
          if (pair) *reinterpret_cast<run_t*>(o + 16) = run_t{v[4], v[5], v[6], v[7]};
        }
        const float first = __shfl(v[0], c16, 64);   // the group's first column (lane group 0)
        float best = -INFINITY;
        int bi = 4 * q;
#pragma unroll
        for (int r = 0; r < 8; ++r)
          if ((r < 4 || pair) && v[r] > best) {
            best = v[r];
            bi = 4 * q + (r & 3) + (r >= 4 ? 16 : 0);
          }
#pragma unroll
        for (int x = 16; x <= 32; x <<= 1) {
          const float ob = __shfl_xor(best, x, 64);
          const int oi = __shfl_xor(bi, x, 64);
          if (ob > best || (ob == best && oi < bi)) {
            best = ob;
            bi = oi;
          }
        }
        if (!(first == first)) {
          best = first;
          bi = 0;
        }
        if (q == 0 && row) p.amax[(size_t)(nt / 2) * p.amax_ld + m] = argmax_key(best, colbase + nt * 16 + bi);
      }
    } else if constexpr (EPI == EPI_SWIGLU) {
      // a strip is 8 gate columns (lane groups 0, 1) and the same 8 up columns
      // (2, 3): the partner holds the other half; each lane finishes two outputs
      const bool up = q >= 2;
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int nt = nt0 + wn * WN + j;
        float o[4], t[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) t[r] = p.norm ? tot[i][j][r] * rs : tot[i][j][r];
#pragma unroll
        for (int r = 0; r < 4; ++r) o[r] = __shfl_xor(t[r], 32, 64);
        const float y0 = up ? silu(o[2]) * t[2] : silu(t[0]) * o[0];
        const float y1 = up ? silu(o[3]) * t[3] : silu(t[1]) * o[1];
        if (nt < p.ntiles && row) {
          const int c = (colbase >> 1) + nt * 8 + (q & 1) * 4 + (up ? 2 : 0);
          if (p.Y) pair_st<T>(reinterpret_cast<T*>(p.Y) + (size_t)m * p.ldy + c, y0, y1);
          if (p.yf.p)
            pair_st<T>(reinterpret_cast<T*>(p.yf.p) + afrag_off<T>(m, p.yf.c0 + c, p.yf.ktiles), y0, y1);
        }
      }
    } else {
#pragma unroll
      for (int j = 0; j < WN; ++j) {
        const int nt = nt0 + wn * WN + j;
        if (nt >= p.ntiles) break;             // uniform
        const int col = colbase + nt * 16 + 4 * q;
        float v[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) v[r] = p.norm ? tot[i][j][r] * rs : tot[i][j][r];
        if (!row) continue;
        if constexpr (EPI == EPI_BIAS_SILU || EPI == EPI_BIAS_F32) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] += TT<T>::ld(reinterpret_cast<const T*>(p.bias), col + r);
        }
        if constexpr (EPI == EPI_BIAS_SILU) {
#pragma unroll
          for (int r = 0; r < 4; ++r) v[r] = silu(v[r]);
        }
        if constexpr (EPI == EPI_STORE_F32 || EPI == EPI_BIAS_F32) {
          const size_t part = EPI == EPI_STORE_F32 ? (size_t)h * p.y_part : 0;
          *reinterpret_cast<float4*>(reinterpret_cast<float*>(p.Y) + part + (size_t)m * p.ldy + col) =
              make_float4(v[0], v[1], v[2], v[3]);
        } else {
          if (EPI != EPI_BIAS_SILU || p.Y) {
            T* o = reinterpret_cast<T*>(p.Y) + (size_t)m * p.ldy + col;
            pair_st<T>(o, v[0], v[1]);
            pair_st<T>(o + 2, v[2], v[3]);
          }
          if constexpr (EPI == EPI_BIAS_SILU) {
            if (p.yf.p) {
              T* f = reinterpret_cast<T*>(p.yf.p) + afrag_off<T>(m, p.yf.c0 + col, p.yf.ktiles);
              pair_st<T>(f, v[0], v[1]);
              pair_st<T>(f + 2, v[2], v[3]);
            }
          }
        }
      }
    }
  }
}

}  // namespace dflow
