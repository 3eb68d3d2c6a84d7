// Internal launch interface of the weight-streaming and tiled GEMMs.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace dflow {

// Matrix-core-order copy of an activation block (afrag_off): written by the
// producer of a projection's A operand besides its row-major output, read by
// the projection in whole 16-row tiles (buffers hold the launch's rows rounded
// up to 16).  p null: no copy.
struct FragOut {
  void* p;
  int ktiles;   // K / KT of the consuming projection
  int c0;       // first column of the producer's output within that K
};

enum Epi : int {
  EPI_STORE_T = 0,   // Y = acc                       (storage type)
  EPI_STORE_F32,     // Y = acc                       (fp32)
  EPI_RESID,         // Y = R + acc; optional copy Y2 (storage type)
  EPI_SWIGLU,        // Y = silu(gate) * up           (gate/up tiles interleaved)
  EPI_BIAS_SILU,     // Y = silu(acc + bias)          (storage type)
  EPI_BIAS_F32,      // Y = acc + bias                (fp32)
  EPI_ARGMAX,        // per-row best (value, lowest index) over the group's columns
  EPI_COUNT
};

struct GemmParams {
  const void* A; int lda;           // activations [M, lda], storage type
  const void* W;                    // packed weight tiles of this column range
  int M, ntiles, ktiles;            // ntiles = N/16 of the range, ktiles = K/KT
  void* Y; int ldy;                 // null for EPI_SWIGLU and EPI_BIAS_SILU: only the copy yf is written
  const void* R; int ldr;
  void* Y2; int ldy2;
  const void* bias;
  uint64_t* amax; int amax_ld;      // [workgroup][amax_ld] argmax keys
  float* logits; int ldl;           // optional fp32 logits
  int col0;                         // first output column of this range (argmax indices, bias)
  // RMSNorm row scale (norm = 1): A rows are the raw x, the norm gain is
  // folded into W, and every output of row m is scaled by rs[m] =
  // (sum_c ssq[m * ssq_ld + c] / (16 ssq_parts) + eps)^(-1/2).  Rows are
  // padded: ssq_ld >= max(256, ssq_parts) entries are readable.
  int norm;
  const float* ssq; int ssq_ld; int ssq_parts;
  float eps;
  const float* rs;   // [M] the row scales themselves, for launches of more than SPLIT_MIN_ROWS rows
  // EPI_RESID: per-16-column-strip sums of squares of the stored rows, [m * ssq_out_ld + strip]
  float* ssq_out; int ssq_out_ld;
  // EPI_STORE_F32 only: K split into ksplit parts; part h writes its partial
  // sums at Y + h * y_part (floats), and the consumer adds the parts
  int ksplit; size_t y_part;
  float* rs_out;     // EPI_RESID above SPLIT_MIN_ROWS rows: [M] RMSNorm scales of the stored rows (for d = N)
  unsigned* arrive;  // EPI_RESID above SPLIT_MIN_ROWS rows: a counter per 64 rows, zero between launches
  // above SPLIT_MIN_ROWS rows: fp32 scratch of split_parts(epi, ntiles,
  // ktiles) x M x N floats for K-part partial sums (EPI_RESID at any M, the
  // others up to split_max_rows(epi) rows; null: no split)
  float* part_ws;
  int cus;                          // compute units (0: unknown, no balance-driven split)
  // A read from its matrix-core-order copy (afrag_off; null: from A), and
  // copies of the outputs Y / Y2 written in that order for the next
  // projection (every path and epilogue that writes Y / Y2 honours them).
  const void* Af;
  FragOut yf, y2f;
};

// Up to SPLIT_MIN_ROWS rows the weight-streaming kernel; more rows the tiled one.
constexpr int SPLIT_MIN_ROWS = 48;
// Most rows at which a launch may be split into K-part partial sums (beyond,
// the tiles alone fill the compute units, and the scratch would only grow).
inline int split_max_rows(int epi) { return epi == EPI_SWIGLU ? 256 : 512; }

struct GemmShape { int ng; int waves; int groups; };
GemmShape gemm_shape(int ntiles, int ktiles, int epi, int ksplit = 1);
int gemm_ksplit(int ntiles, int ktiles, int cus);
// K parts of a split launch (the weight-streaming kernel's wave count for
// (N, K), so every part is one of its K ranges)
int split_parts(int epi, int ntiles, int ktiles);
hipError_t launch_gemm(bool bf16, int epi, const GemmParams& p, hipStream_t s);
hipError_t launch_pack(bool bf16, const void* w, int N, int K, int gate_up, const void* col_gain, void* out,
                       hipStream_t s);

}  // namespace dflow
