// Prompt attention (included by attention.hip): causal attention of a prefill
// chunk's query rows over the paged cache, which already holds the chunk's own
// keys and values.
//
// A workgroup takes NW * RG groups of 16 rows (row = (chunk row j, query head g
// of a kv group)) of one kv head and one split of PREFILL_SPLIT keys at fixed
// absolute positions.  K and V pages are in matrix-core fragment order, so they
// go to an LDS ring by load-to-LDS, up to NS - 1 pages ahead; one barrier per page.
// Per page a wave computes S^T = K Q^T, one running-softmax step (log2 units)
// and O^T += V^T P^T: with the operands this way round a lane holds one query
// row throughout, so row maxima, sums and rescales need no exchange beyond the
// four lane groups of the maximum.  The rescale is skipped while no row's
// reference moves (a factor of exactly 1), the row sum is kept per lane and added
// across lane groups once per split, and pages before the wave's rows skip the
// mask.
//
// Reference of a row's exponentials: with bf16 probabilities the page's own
// maximum, so that the largest probability of every page is exactly 1 and free of
// rounding.  The running maximum over a 2048-key split rounds all but one page's;
// the keys and values after it were 0.14 to 0.52 % further from the 64-bit ones
// than with 128-key splits, and are 0.04 to 0.29 % nearer than those now (8B
// and 1.7B prompts).  It falls at most SPAN (log2 units) below the row's largest
// score so far, so the rescales stay below 2^SPAN times what a running maximum
// keeps.  Cost: the rescale is hardly ever skipped, 1.1 % of the attention, 0.1
// to 0.4 % of a whole prompt (1.7B shape, 12288 tokens: 10074 -> 10113 us).  fp32 probabilities are
// not rounded: SPAN 0, the running maximum.
//
// A split's result goes straight to the output when it is the row's only one,
// else as (m, l, O) to the partials that the combine kernel merges in split
// order.  A row's arithmetic depends on its own keys and the fixed split and
// page boundaries only, never on the chunk, the tile or the rows beside it.
//
// Bound: LDS reads (32 KB per page and wave, 256 clocks, shared by its RG row
// groups), the vector unit (64 keys x 16 rows: 16 exponentials per lane and
// their scale, maximum, sum and conversion, about 600 clocks) and the matrix
// cores (32 ops of 16 clocks) are of one size.  Qwen3-1.7B shape, 512 rows
// against 11.8 thousand keys: 82 us (80 with the running maximum) + 8 us combine,
// where 256-key splits of the round kernel with their partials took 150 + 50.
#pragma once
#include "common.h"
#include "kernels.h"

namespace dflow {

// x of the same lane and of lane ^ 16 / lane ^ 32 (vector-unit row swaps: no LDS round trip)
__device__ __forceinline__ void pair16(float x, float& a, float& b) {
  const auto v = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(v[0]);
  b = __uint_as_float(v[1]);
}
__device__ __forceinline__ void pair32(float x, float& a, float& b) {
  const auto v = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
  a = __uint_as_float(v[0]);
  b = __uint_as_float(v[1]);
}

template <typename T, int DH, int NW, int RG, int NS>
__global__ void __launch_bounds__(NW * 64, 2) attn_prefill_kernel(AttnParams p, int tiles) {
  constexpr int KL = TT<T>::KL, KT = TT<T>::KT;
  constexpr int KS = DH / KT, DT = DH / 16;
  constexpr uint32_t PB = PAGE * DH * (uint32_t)sizeof(T);   // bytes of a K (or V) page block
  constexpr int LPW = (int)(2 * PB / 1024) / NW;             // loads per wave and page
  static_assert((2 * PB / 1024) % NW == 0 && (NS - 1) * LPW < 64, "page loads and vmcnt range");
  extern __shared__ __align__(16) unsigned char pf_smem[];
  const int lane = threadIdx.x & 63;
  const int w = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  // block -> (kv head fastest, so a head's pages stay in one XCD's L2; split; row tile, last rows first)
  const int kvh = blockIdx.x % p.Hkv, rest = blockIdx.x / p.Hkv;
  const int split = rest % p.nsplit, tile = tiles - 1 - rest / p.nsplit;
  const int G = p.Hq / p.Hkv, R = p.Bq * G;
  const int rg0 = tile * NW * RG;
  const int t0 = p.start_pos[0];
  const int last = t0 + (min((rg0 + NW * RG) * 16, R) - 1) / G;   // position of the tile's last row
  const int key0 = split * PREFILL_SPLIT;
  if (key0 > last) return;                                        // uniform over the workgroup
  const int cap = p.max_pages * PAGE;
  if (blockIdx.x == 0 && threadIdx.x == 0 && t0 + p.Bq > cap) set_status(p.status, ST_CAPACITY);
  const int np = (min(last + 1 - key0, PREFILL_SPLIT) + PAGE - 1) / PAGE;   // pages of the split the tile sees
  static_assert(PREFILL_SPLIT / PAGE <= 64, "a page id per lane");
  const int pid = p.page_table[min(key0 / PAGE + min(lane, np - 1), p.max_pages - 1)];
  {
    const bool bad = pid < 0 || pid >= p.num_pages;
    if (__builtin_amdgcn_ballot_w64(bad) != 0 && threadIdx.x == 0) set_status(p.status, ST_BAD_PAGE);
  }
  const uint32_t lds0 = (uint32_t)(uintptr_t)(__attribute__((address_space(3))) unsigned char*)pf_smem;
  const uint32_t voff = lane * 16;
  auto page_ok = [&](int i) {                   // uniform
    const int v = __builtin_amdgcn_readlane(pid, i);
    return v >= 0 && v < p.num_pages;
  };
  auto issue = [&](int i, uint32_t base) {      // page i of the split (an invalid id reads page 0 and is not used)
    const int v = page_ok(i) ? __builtin_amdgcn_readlane(pid, i) : 0;
    const size_t off = ((size_t)v * p.Hkv + kvh) * PB;
    const char* kp = (const char*)p.kpool + off + w * 1024;
    const char* vp = (const char*)p.vpool + off + w * 1024;
    const uint32_t l = base + w * 1024;
    static_for<LPW / 2>([&]<int I>(std::integral_constant<int, I>) {
      load_to_lds<NW * 1024 * I>(l, kp + NW * 1024 * I, voff);
    });
    static_for<LPW / 2>([&]<int I>(std::integral_constant<int, I>) {
      load_to_lds<(int)PB + NW * 1024 * I>(l, vp + NW * 1024 * I, voff);
    });
  };

  // the wave's query fragments: row groups rg0 + w * RG + i
  u32x4_t qf[RG][KS];
  int pos[RG];                                  // position of lane%16's row (clamped rows are never stored)
  const int wr0 = (rg0 + w * RG) * 16;
#pragma unroll
  for (int i = 0; i < RG; ++i) {
    const int r = min(wr0 + i * 16 + (lane & 15), R - 1), j = r / G, g = r - j * G;
    pos[i] = t0 + j;
    const T* q = reinterpret_cast<const T*>(p.q) + ((size_t)j * p.Hq + kvh * G + g) * DH;
#pragma unroll
    for (int k = 0; k < KS; ++k) qf[i][k] = *(const gu4*)(q + k * KT + (lane >> 4) * KL);
  }
  const int first = t0 + min(wr0, R - 1) / G;   // position of the wave's first row
  const int wlast = t0 + min(wr0 + RG * 16 - 1, R - 1) / G;
#pragma unroll
  for (int i = 0; i < RG; ++i)
#pragma unroll
    for (int k = 0; k < KS; ++k) asm volatile("" ::"v"(qf[i][k]));   // the rows are in before the page loads are counted

  const float sl2 = rsqrtf((float)DH) * 1.4426950408889634f;   // softmax scale x log2(e)
  // exponentials' reference of the row, its largest score so far (log2 units), this lane's share of its sum
  float m[RG], top[RG], l[RG];
  f32x4_t o[RG][DT];                            // channel 16 dt + 4 (lane / 16) + r of row lane % 16
#pragma unroll
  for (int i = 0; i < RG; ++i) {
    m[i] = top[i] = -INFINITY;
    l[i] = 0.f;
#pragma unroll
    for (int d = 0; d < DT; ++d) o[i][d] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  }

  float sc[RG][16];                             // score of key 16 kt + 4 (lane / 16) + r, then its exponential
  constexpr float SPAN = sizeof(T) == 2 ? 8.f : 0.f;
  auto finish_scores = [&](const f32x4_t (&a)[RG][4], int kp0) {   // mask, running softmax step
#pragma unroll
    for (int i = 0; i < RG; ++i)
#pragma unroll
      for (int e = 0; e < 16; ++e) sc[i][e] = a[i][e >> 2][e & 3];
    if (kp0 + PAGE - 1 > first) {               // uniform: some row of the wave does not see the whole page
#pragma unroll
      for (int i = 0; i < RG; ++i)
#pragma unroll
        for (int e = 0; e < 16; ++e)
          if (kp0 + (e >> 2) * 16 + 4 * (lane >> 4) + (e & 3) > pos[i]) sc[i][e] = -INFINITY;
    }
#pragma unroll
    for (int i = 0; i < RG; ++i) {
      float mx = sc[i][0];
#pragma unroll
      for (int e = 1; e < 16; ++e) mx = fmaxf(mx, sc[i][e]);
      float x0, x1;
      pair16(mx, x0, x1);
      pair32(fmaxf(x0, x1), x0, x1);
      const float pm = fmaxf(x0, x1) * sl2;
      top[i] = fmaxf(top[i], pm);
      const float mn = pm == -INFINITY ? m[i] : fmaxf(pm, top[i] - SPAN);   // (no visible key: as it was)
      if (__builtin_amdgcn_ballot_w64(mn != m[i]) != 0) {   // uniform
        const float f = m[i] == -INFINITY ? 0.f : __builtin_amdgcn_exp2f(m[i] - mn);
        l[i] *= f;
#pragma unroll
        for (int d = 0; d < DT; ++d)
#pragma unroll
          for (int r = 0; r < 4; ++r) o[i][d][r] *= f;
        m[i] = mn;
      }
      // a row with no visible key yet keeps m = -inf; its scores are all -inf and exponentiate to 0
      const float mref = m[i] == -INFINITY ? 0.f : m[i];
      float s = 0.f;
#pragma unroll
      for (int e = 0; e < 16; ++e) {
        sc[i][e] = __builtin_amdgcn_exp2f(fmaf(sc[i][e], sl2, -mref));
        s += sc[i][e];
      }
      l[i] += s;
    }
  };
  constexpr int NB = PAGE / (4 * KL);           // P V steps per page: 4 KL keys each
  constexpr int NKF = 4 * KS, NVF = DT;         // fragments of a page's keys, of a P V step's values
  auto kfrag = [&](int slot, int n) {           // key tile n % 4, k step n / 4
    return reinterpret_cast<const u32x4_t*>(pf_smem + (size_t)slot * 2 * PB)[((n & 3) * KS + (n >> 2)) * 64 + lane];
  };
  auto vfrag = [&](int slot, int h, int d) {
    return reinterpret_cast<const u32x4_t*>(pf_smem + (size_t)slot * 2 * PB + PB)[(h * DT + d) * 64 + lane];
  };
  f32x4_t a[RG][4];
  auto zero_scores = [&]() {
#pragma unroll
    for (int i = 0; i < RG; ++i)
#pragma unroll
      for (int kt = 0; kt < 4; ++kt) a[i][kt] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  };
  auto qk = [&](int n, const u32x4_t& kf) {
#pragma unroll
    for (int i = 0; i < RG; ++i) a[i][n & 3] = mma_frag(T(), kf, qf[i][n >> 2], a[i][n & 3]);
  };
  auto pv = [&](int h, int d, const u32x4_t& vf, const u32x4_t (&pa)[RG]) {
#pragma unroll
    for (int i = 0; i < RG; ++i) o[i][d] = mma_frag(T(), vf, pa[i], o[i][d]);
  };

  const int pre = min(np, NS);
  for (int i = 0; i < pre; ++i) issue(i, lds0 + i * 2 * PB);
  if (np >= NS) wait_barrier<(NS - 1) * LPW>();
  else wait_barrier<0>();
  int slot = 0;
  // page c + 1 is in (c + 2 .. c + NS - 1 may be in flight) and every wave has
  // read page c: its slot takes page c + NS
  auto advance = [&](int c) {
    if (c + NS <= np) wait_barrier<(NS - 2) * LPW>();
    else wait_barrier<0>();
    if (c + NS < np) issue(c + NS, lds0 + slot * 2 * PB);
    slot = slot + 1 == NS ? 0 : slot + 1;
  };
  // uniform: the page holds keys of the wave's rows
  auto used = [&](int c) { return key0 + c * PAGE <= wlast && page_ok(c); };
  if constexpr (sizeof(T) == 2) {
    // All fragments of a page pass through registers ahead of their use: the
    // next page's keys are read under P V, the values under the softmax
    // (left to the compiler, each small batch of reads exposed the LDS latency:
    // 1.5 us a page and wave).
    // With two row groups per wave the registers hold half of the next keys.
    constexpr int KPRE = RG == 1 ? NKF : NKF / 2;
    u32x4_t kf[NKF], vf[NB][NVF];
#pragma unroll
    for (int n = 0; n < KPRE; ++n) kf[n] = kfrag(0, n);
    for (int c = 0; c < np; ++c) {
      const bool on = used(c);
      if (on) {
#pragma unroll
        for (int n = KPRE; n < NKF; ++n) kf[n] = kfrag(slot, n);
        __builtin_amdgcn_sched_barrier(0);
        zero_scores();
#pragma unroll
        for (int n = 0; n < NKF; ++n) qk(n, kf[n]);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
          for (int d = 0; d < NVF; ++d) vf[h][d] = vfrag(slot, h, d);
        __builtin_amdgcn_sched_barrier(0);
        finish_scores(a, key0 + c * PAGE);
      }
      if (c + 1 < np) {
        advance(c);
        // the barrier waited for the values; saying so keeps P V from waiting for the key reads below
#pragma unroll
        for (int h = 0; h < NB; ++h)
#pragma unroll
          for (int d = 0; d < NVF; ++d) asm volatile("" ::"v"(vf[h][d]));
#pragma unroll
        for (int n = 0; n < KPRE; ++n) kf[n] = kfrag(slot, n);
        __builtin_amdgcn_sched_barrier(0);
      }
      if (on) {
#pragma unroll
        for (int h = 0; h < NB; ++h) {
          u32x4_t pa[RG];
#pragma unroll
          for (int i = 0; i < RG; ++i) pa[i] = Chunk<T>::pack(&sc[i][KL * h]);
#pragma unroll
          for (int d = 0; d < NVF; ++d) pv(h, d, vf[h][d], pa);
        }
      }
    }
  } else {
    for (int c = 0; c < np; ++c) {
      if (used(c)) {
        zero_scores();
#pragma unroll
        for (int n = 0; n < NKF; ++n) qk(n, kfrag(slot, n));
        finish_scores(a, key0 + c * PAGE);
#pragma unroll
        for (int h = 0; h < NB; ++h) {          // 16 keys per fragment
          u32x4_t pa[RG];
#pragma unroll
          for (int i = 0; i < RG; ++i) pa[i] = Chunk<T>::pack(&sc[i][KL * h]);
#pragma unroll
          for (int d = 0; d < NVF; ++d) pv(h, d, vfrag(slot, h, d), pa);
        }
      }
      if (c + 1 < np) advance(c);
    }
  }

#pragma unroll
  for (int i = 0; i < RG; ++i) {
    const int r = wr0 + i * 16 + (lane & 15);
    float l0, l1;
    pair16(l[i], l0, l1);
    pair32(l0 + l1, l0, l1);
    const float ls = l0 + l1;
    if (r >= R) continue;
    if (p.nsplit == 1) {
      const int j = r / G, c0 = (kvh * G + r - j * G) * DH;
#pragma unroll
      for (int d = 0; d < DT; ++d) {
        float y[4];
#pragma unroll
        for (int e = 0; e < 4; ++e) y[e] = ls > 0.f ? (0.f + o[i][d][e]) / ls : 0.f;
        frag_st4<T>(p.outf, p.out_row0 + j, c0 + d * 16 + 4 * (lane >> 4), y);
      }
    } else {
      const size_t idx = (((size_t)kvh * p.rg + (r >> 4)) * p.nsplit + split) * 16 + (r & 15);
      float* po = p.part_o + idx * DH + 4 * (lane >> 4);
#pragma unroll
      for (int d = 0; d < DT; ++d)
        *reinterpret_cast<float4*>(po + d * 16) = make_float4(o[i][d][0], o[i][d][1], o[i][d][2], o[i][d][3]);
      if (lane < 16) *reinterpret_cast<float2*>(p.part_ml + 2 * idx) = make_float2(m[i], ls);
    }
  }
}

}  // namespace dflow
