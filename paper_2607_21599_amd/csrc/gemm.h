// Dense bf16 projections: the job description shared by the host code and
// gemm.hip.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

namespace daf {

// One column block of a projection job: C = A W^T (+ bias), with its own
// weights and output. Several segments of one job share A (the Q, K and V
// projections of a layer run as one launch).
struct GemmSeg {
  const void *W;     // [N][K]; gated jobs: [2N][K], the gate rows then the up rows
  const void *bias;  // [N] or null
  void *C;           // [M][N]
  int32_t N;         // multiple of 128 (gated: of 64)
};

constexpr int kMaxGemmSegs = 3;

struct GemmJob {
  const void *A;         // [M][K]
  const void *residual;  // [M][N] or null (may be C itself); one segment only
  int64_t M;
  int32_t K;       // multiple of 64
  int32_t n_segs;
  // gated: C[m][j] = SiLU((A W^T)[m][j]) * (A W^T)[m][N + j], one segment, no
  // bias or residual
  int32_t glu;
  GemmSeg seg[kMaxGemmSegs];
};

// part: workspace for fp32 pieces of tiles cut along k (kGemmPieceBytes is
// always enough), or null: then no tile is cut.
hipError_t launch_gemm_job(const GemmJob &job, float *part, size_t part_bytes, hipStream_t st);
constexpr size_t kGemmPieceBytes = (size_t)256 * 128 * 256 * 4;  // one 128 x 256 piece per CU

// Whether C [M][N] of K, without a workspace, runs in tiles of 128 x 128
// (gemm_small.hip): while these are few and K is short, that kernel's chain is the
// shorter one. With long K and the weights from HBM the other one's copies, issued
// further ahead, decide. Times of the 256-row kernel over its, back to back in a
// graph, 16 to 900 rows (16 / 64 / 128 / 129 / 256 / 500):
//   K  896  HBM 0.98 / 1.06 / 1.18 / 1.03 / 1.17 / 1.15   caches 1.19-1.27
//   K 1024      0.96 / 1.03 / 1.15 / 0.99 / 1.11 / 1.09          1.18-1.27
//   K 1536      0.92 / 1.04 / 1.15 / 0.95 / 1.16 / 1.13          1.15-1.21
//   K 2048      0.86 / 0.95 / 1.07 / 0.89 / 1.05 / 1.01          1.13-1.20
//   K 4864      0.85 / 0.96 / 1.09 / 0.85 / 1.04 / 0.98          0.91-1.13
// and with more tiles, from the caches:
//   up to 512   K 64 1.2-1.3, 256 1.1-1.15, 512 1.01-1.07, 1024 0.9-1.0
//   up to 1024  K 64 1.1-1.25, 256 1.0-1.16, 512 0.92-1.07
constexpr bool small_tiles_pay(int64_t M, int64_t N, int64_t K) {
  const int64_t tiles = (M + 127) / 128 * (N / 128);
  if (tiles > (K <= 256 ? 1024 : K <= 512 ? 512 : 256)) return false;
  return K <= 1024 || (K <= 1536 && M >= 64);
}
hipError_t launch_gemm_small(const GemmJob &job, hipStream_t st);

}  // namespace daf
