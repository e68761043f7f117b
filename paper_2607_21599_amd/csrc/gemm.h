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

}  // namespace daf
