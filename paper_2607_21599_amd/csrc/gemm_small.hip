// Projections of little work: C = A W^T (+ bias) (+ residual) as in gemm.hip, one
// segment, not gated, in tiles of 128 x 128 by workgroups of 4 waves (64 x 64 each,
// 2 x 2 blocks of v_mfma_f32_32x32x16_bf16), two workgroups per CU.
//
// A launch that gives every CU at most a tile or two is a chain: launch, first
// copies, k steps, epilogue. The 256-row kernel of gemm.hip, made for the rate of
// full rounds, has the longer one (more code to fetch, a ring to fill, twice the
// output per workgroup, and half the workgroups), so this one runs where
// small_tiles_pay (gemm.h) says. Graph replays, us, 256-row kernel and this one:
//   500 x 512 x 64 6.6 / 4.3, 500 x 512 x 512 10.2 / 7.6, 1000 x 1024 x 1024 14.9 /
//   11.9, 500 x 2048 x 1536 19.0 / 16.0.
//
// The A and W tiles of a k step (64) are copied global -> LDS with the buffer unit
// (rows of 128 B, 16-byte chunks XOR-swizzled by (row / 2) mod 8: no bank
// conflicts), double-buffered so that the copy of step k + 1 overlaps the MFMAs of
// step k. The accumulators are staged through LDS in fp32 so that bias, residual
// and the stores run on whole 128-byte row segments.
#include "daf_internal.h"
#include "gemm.h"

namespace daf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_u8;

constexpr int kTile = 128, kRowB = 128;  // tile rows; bytes per tile row in LDS (64 k)
constexpr int kTileB = kTile * kRowB;
constexpr int kIpw = kTile / 4 / 8;      // copy instructions (8 rows each) per wave and tile
constexpr int kGroupM = 8;               // M-tiles per group of the tile order
[[maybe_unused]] constexpr int kRsrcWord3 = 0x00020000;  // raw buffer descriptor word 3 (gfx9 family)

struct SmallGemm {
  const unsigned char *A, *W;
  const __bf16 *bias, *residual;
  __bf16 *C;
  int64_t M;
  int32_t N, K, tiles_m, tiles_n;
};

__device__ __forceinline__ int swz(int r) { return (r >> 1) & 7; }

// Copy 128 rows x 64 columns (rows at `base`) into LDS; this wave copies 32 of
// them. Bytes at or past `nrec` read as zero.
__device__ __forceinline__ void copy_tile(const unsigned char *base, int nrec, unsigned char *lds, int wave,
                                          const int (&voff)[kIpw]) {
#if defined(__HIP_DEVICE_COMPILE__)
  const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc((void *)base, 0, nrec, kRsrcWord3);
#pragma unroll
  for (int i = 0; i < kIpw; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(
        r, (void __attribute__((address_space(3))) *)((lds_u8 *)lds + (wave * kIpw + i) * 8 * kRowB), 16, voff[i], 0,
        0, 0);
#endif
}

// One k step on the tiles in (as, bs); the next step's go to (an, bn).
struct Wave {
  f32x16 acc[2][2];  // D^T blocks: rows are output columns, columns output rows
  int voff[kIpw];
  int fa[2][4], fb[2][4];
  const unsigned char *A, *W;
  int a_bytes, w_bytes, wave;

  __device__ __forceinline__ void step(const unsigned char *as, const unsigned char *bs, unsigned char *an,
                                       unsigned char *bn, int kt, bool prefetch) {
    // this wave's copies of step kt have landed; after the barrier every wave's
    // have, and every wave is done reading the other buffers (step kt - 1)
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt left at their maxima
    __syncthreads();
    if (prefetch) {
      const int kb = (kt + 1) * kRowB;
      copy_tile(A + kb, a_bytes - kb, an, wave, voff);
      copy_tile(W + kb, w_bytes - kb, bn, wave, voff);
    }
    // the reads of each half of the step go out before its MFMAs
#pragma unroll
    for (int h = 0; h < 2; ++h) {
      bf16x8 a[2][2], b[2][2];
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int j = 0; j < 2; ++j) {
          a[kk][j] = *reinterpret_cast<const bf16x8 *>(as + fa[j][2 * h + kk]);
          b[kk][j] = *reinterpret_cast<const bf16x8 *>(bs + fb[j][2 * h + kk]);
        }
#pragma unroll
      for (int kk = 0; kk < 2; ++kk)
#pragma unroll
        for (int mb = 0; mb < 2; ++mb)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            acc[mb][nb] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[kk][nb], a[kk][mb], acc[mb][nb], 0, 0, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 8, 0);  // this half's LDS reads
      __builtin_amdgcn_sched_group_barrier(0x008, 8, 0);  // then its MFMAs
    }
  }
};

// The tiles are cut into 8 contiguous ranges, one per XCD (workgroup i runs on XCD
// i mod 8); groups of kGroupM M-tiles sweep the column tiles, so that neighbours
// share A and W rows in that XCD's L2.
__global__ __launch_bounds__(256, 2) void gemm_small_kernel(const SmallGemm p) {
  // two buffers of A and of W tiles, then the epilogue's staging space
  __shared__ __attribute__((aligned(1024))) unsigned char a0[kTileB], b0[kTileB], a1[kTileB], b1[kTileB];
  const int count = p.tiles_m * p.tiles_n, per_xcd = (count + kXcds - 1) / kXcds;
  const int slot = blockIdx.x / kXcds, t = blockIdx.x % kXcds * per_xcd + slot;
  if (slot >= per_xcd || t >= count) return;
  const int span = kGroupM * p.tiles_n, first_m = t / span * kGroupM, gsize = min(p.tiles_m - first_m, kGroupM);
  const int tm = first_m + t % span % gsize, tn = t % span / gsize;

  const int lane = threadIdx.x & 63, l32 = lane & 31, half = lane >> 5;
  const int64_t m0 = (int64_t)tm * kTile;
  const int n0 = tn * kTile, row_bytes = p.K * 2;
  Wave w;
  w.wave = threadIdx.x >> 6;
  const int wm = w.wave & 1, wn = w.wave >> 1;
  w.A = p.A + m0 * row_bytes;
  w.W = p.W + (int64_t)n0 * row_bytes;
  w.a_bytes = (int)min((int64_t)kTile, p.M - m0) * row_bytes;  // rows past M read as zero
  w.w_bytes = kTile * row_bytes;
#pragma unroll
  for (int i = 0; i < kIpw; ++i) {
    const int r = (w.wave * kIpw + i) * 8 + lane / 8;
    w.voff[i] = r * row_bytes + (((lane & 7) ^ swz(r)) << 4);
  }
#pragma unroll
  for (int ks = 0; ks < 4; ++ks)
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int ra = wm * 64 + j * 32 + l32, rb = wn * 64 + j * 32 + l32;
      w.fa[j][ks] = ra * kRowB + (((2 * ks + half) ^ swz(ra)) << 4);
      w.fb[j][ks] = rb * kRowB + (((2 * ks + half) ^ swz(rb)) << 4);
    }
#pragma unroll
  for (int i = 0; i < 4; ++i) w.acc[i >> 1][i & 1] = f32x16{};

  const int KT = p.K / 64;
  copy_tile(w.A, w.a_bytes, a0, w.wave, w.voff);
  copy_tile(w.W, w.w_bytes, b0, w.wave, w.voff);
  for (int kt = 0; kt < KT; kt += 2) {
    w.step(a0, b0, a1, b1, kt, kt + 1 < KT);
    if (kt + 1 < KT) w.step(a1, b1, a0, b0, kt + 1, kt + 2 < KT);
  }

  // every wave is done reading the tiles and no copy is in flight: a wave stages
  // its 64 rows of 64 columns in a tile buffer (rows of 256 B, 16-byte chunks
  // XOR-swizzled by row), then each lane finishes 8 columns of a row
  __syncthreads();
  unsigned char *stg = w.wave == 0 ? a0 : w.wave == 1 ? b0 : w.wave == 2 ? a1 : b1;
  const int cg = lane & 7, n = n0 + wn * 64 + cg * 8;
  bf16x8 bias = bf16x8{};
  if (p.bias) bias = *reinterpret_cast<const bf16x8 *>(p.bias + n);
#pragma unroll
  for (int mb = 0; mb < 2; ++mb)
#pragma unroll
    for (int nb = 0; nb < 2; ++nb)
#pragma unroll
      for (int q = 0; q < 4; ++q) {
        const int row = mb * 32 + l32, c = nb * 8 + 2 * q + half;  // 4-column chunk of the wave's columns
        f32x4 v;
#pragma unroll
        for (int e = 0; e < 4; ++e) v[e] = w.acc[mb][nb][4 * q + e];
        *reinterpret_cast<f32x4 *>(stg + row * 256 + ((c ^ (row & 15)) << 4)) = v;
      }
  // every staged piece and residual before the first store: behind a store, an LDS
  // read waits for it (the compiler counts it with the copies to LDS), and so would
  // a residual load (C may be the residual)
  f32x4 v[8][2];
  bf16x8 res[8];
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int row = it * 8 + (lane >> 3);
    const int64_t m = m0 + wm * 64 + row;
    res[it] = bf16x8{};
    if (p.residual && m < p.M) res[it] = *reinterpret_cast<const bf16x8 *>(p.residual + m * p.N + n);
#pragma unroll
    for (int h = 0; h < 2; ++h)
      v[it][h] = *reinterpret_cast<const f32x4 *>(stg + row * 256 + (((2 * cg + h) ^ (row & 15)) << 4));
  }
#pragma unroll
  for (int it = 0; it < 8; ++it) {
    const int64_t m = m0 + wm * 64 + it * 8 + (lane >> 3);
    if (m >= p.M) continue;
    bf16x8 out;
#pragma unroll
    for (int e = 0; e < 8; ++e) out[e] = (__bf16)(v[it][e >> 2][e & 3] + (float)res[it][e] + (float)bias[e]);
    *reinterpret_cast<bf16x8 *>(p.C + m * p.N + n) = out;
  }
}

}  // namespace

hipError_t launch_gemm_small(const GemmJob &j, hipStream_t st) {
  const GemmSeg &s = j.seg[0];
  const SmallGemm p{static_cast<const unsigned char *>(j.A), static_cast<const unsigned char *>(s.W),
                    static_cast<const __bf16 *>(s.bias), static_cast<const __bf16 *>(j.residual),
                    static_cast<__bf16 *>(s.C), j.M, s.N, j.K, (int32_t)((j.M + kTile - 1) / kTile), s.N / kTile};
  const int per_xcd = (p.tiles_m * p.tiles_n + kXcds - 1) / kXcds;
  gemm_small_kernel<<<dim3(kXcds * per_xcd), dim3(256), 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace daf
