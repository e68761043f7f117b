// Dense bf16 projections around the DAF attention: C = A W^T (+ bias)
// (+ residual), A [M][K] and W [N][K] row-major, fp32 accumulation, bf16 out.
// These are the QKV, output and MLP projections of a decoder layer, which the
// paper's layer runs on the important and question rows only (Sec. 2 item 2:
// the QKV computation phase; Sec. 2 item 3: the fused compact state feeds the
// next layer's projections).
//
// Tile: 256 (M) x 256 (N), k steps of 64, one workgroup of 8 waves per CU. The
// waves form two groups of four (rows 64 wm .. of each 128-row half, wm = wave
// / 4; two waves of different groups share a SIMD) that run half a phase
// apart: while one group issues the MFMAs of a phase, the other reads its LDS
// fragments and issues its global -> LDS copies, with a barrier between, so
// the matrix cores always have one wave's MFMAs and the other wave's loads are
// off their critical path. A k step has four phases, one per quadrant of the
// wave's 128 x 64 block:
//   (rows half 0, columns 0-31), (0, 32-63), (1, 32-63), (1, 0-31)
// so that only one operand fragment set changes per phase.
//
// Both operands are K-contiguous, as the matrix cores take them. All of the LDS
// is a ring of ten 16 KiB regions of 128 rows x 128 bytes (A rows half 0 / half
// 1, W columns 0-31 / 32-63 of every wave), 16-byte chunks XOR-swizzled by
// (row / 2) mod 8: no bank conflicts in the loop. Regions pass
// through it in the order in which they are read. A slot is copied into again
// two phases after its fragments were read (by then both groups have read it),
// eight phases before its new region is, and that copy is waited for with a
// counted s_waitcnt vmcnt, the seven younger ones staying in flight across the
// barriers. (Two k steps of regions and copies six phases ahead: 5-6% slower in
// a decoder layer, where the weights come from HBM.)
//
// What bounds it: the chip's power, then the barriers between phases. At 8192^3
// the matrix cores are busy 84% of the cycles, and the shader clock settles at
// 1.75 GHz of 2.4: 727 us, 1512 TFLOP/s. The instruction that needs less power per
// FLOP runs faster: v_mfma_f32_16x16x32_bf16 reads and writes half the accumulator
// registers per FLOP of v_mfma_f32_32x32x16_bf16 (an early form of this kernel 868
// us with the latter and 732 with the former; the previous two-stage kernel with
// 32x32x16 ~1150 TFLOP/s). 64-byte rows per copy (k steps of 32, four stages)
// doubled the L2 requests: 911 us. With few rows it is HBM latency: 986 x 3584 x
// 18944 without a workspace takes 177 us with the weights in the caches and 231
// from HBM; in the decoder layer, in two k pieces per half, 139 and 10 for the sum.
//
// Work list (plan_job): whole rounds of 256 tiles, one per CU, then the rest:
// row ranges of at most 128 rows and, where that shortens the last round,
// tiles of the last round cut in two 128 x 256 tiles (two phases per k step, copies
// seven and eight regions ahead) and, given a workspace, cut along k, all in the same
// launch after the whole tiles.
#include <algorithm>
#include <type_traits>

#include "daf_internal.h"
#include "gemm.h"

namespace daf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_u8;

constexpr int kTK = 64;          // k step
constexpr int kRegion = 16384;   // LDS region: 128 rows x 128 bytes
constexpr int kGroupM = 8;       // M-tiles per group of the tile order
constexpr int kCus = 256;
constexpr int kSlots = 10;       // regions in LDS (all 160 KiB)
constexpr int kLds = kSlots * kRegion;
[[maybe_unused]] constexpr unsigned kRsrcWord3 = 0x00020000;  // raw buffer descriptor word 3 (gfx9 family)

struct GemmPlan {
  GemmJob j;
  int32_t tn;          // column tiles over all segments
  int32_t seg_tn[kMaxGemmSegs];
  int32_t tiles_m;     // 256-row tiles (the last may hold 129-255 rows)
  int32_t n_full;      // 256-row tiles run whole, in tile order
  int32_t n_cut;       // the tiles after them, run as two halves each
  int32_t n_half;      // 128-row units: 2 n_cut, then one per column tile if <= 128 rows remain
  int32_t k_parts;     // pieces per 128-row unit along k
  float *part;         // k_parts > 1: [unit][piece][128][256] fp32
};

template <int N>
__device__ __forceinline__ void wait_vm() {
  __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);  // vmcnt(N); the other counters at their maxima
}
// A workgroup barrier that neither memory operations nor MFMAs move across;
// unlike __syncthreads it waits for no memory operation.
__device__ __forceinline__ void phase_barrier() {
  __builtin_amdgcn_sched_barrier(0);
  asm volatile("s_barrier" ::: "memory");
  __builtin_amdgcn_sched_barrier(0);
}

// A region copy: buffer descriptor of the source rows and the LDS byte of this
// wave's share.
struct Copy {
  u32x4 r;
  uint32_t lds;
};
__device__ __forceinline__ Copy make_copy(const unsigned char *base, uint32_t nrec, uint32_t lds) {
  const uint64_t a = (uint64_t)base;
  return Copy{{(uint32_t)a, (uint32_t)(a >> 32) & 0xffffu, nrec, kRsrcWord3}, lds};
}
// Issue it: this wave copies rows 16 wave .. 16 wave + 15 (two 1 KiB
// instructions); bytes at or past the descriptor's extent read as zero. In asm,
// so that the compiler does not wait for the copies in flight at each LDS read:
// wait_vm counts them, the phase barriers order them.
__device__ __forceinline__ void issue(const Copy &c, const uint32_t (&voff)[2]) {
#if defined(__HIP_DEVICE_COMPILE__)
  asm volatile(
      "s_mov_b32 m0, %0\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %2, %4, 0 offen lds\n\t"
      "s_mov_b32 m0, %1\n\t"
      "s_nop 0\n\t"
      "buffer_load_dwordx4 %3, %4, 0 offen lds"
      :
      : "s"(c.lds), "s"(c.lds + 1024), "v"(voff[0]), "v"(voff[1]), "s"(c.r)
      : "memory", "m0");
#endif
}

// LDS byte of the slot n after `at`.
template <int N>
__device__ __forceinline__ uint32_t slot_after(uint32_t at) {
  const uint32_t x = at + N * kRegion;
  return x >= (uint32_t)kLds ? x - kLds : x;
}

// Per-wave state of a tile of H 128-row halves.
template <int H>
struct Tile {
  f32x4 acc[H][2][4][2];  // [row half][column half][16 rows][16 columns], D^T blocks: a lane holds 4 columns of a row
  bf16x8 a[4][2];         // fragments of one row half: [16 rows][32 k]
  bf16x8 b[2][2][2];      // fragments of the column halves: [half][16 columns][32 k]
  int fa[2], fb[2];       // LDS read offsets per 32 k
  uint32_t va[2], vb[2];  // copy source offsets
  const unsigned char *A, *W0, *W1;  // tile origin; the two column halves' weight rows
  uint32_t na, nb0, nb1;  // valid bytes from A, W0, W1
  uint32_t a_half;        // bytes from row half 0 to 1
  uint32_t lds0;          // LDS byte of this wave's rows of slot 0
  uint32_t slot;          // slot (LDS byte) of the region to read next
  int kt1;                // k steps of this piece

  __device__ __forceinline__ void read_a(const unsigned char *lds) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int m = 0; m < 4; ++m)
        a[m][ks] = *reinterpret_cast<const bf16x8 *>(lds + (slot + fa[ks]) + m * 16 * 128);
    slot = slot_after<1>(slot);
  }
  template <int C>
  __device__ __forceinline__ void read_b(const unsigned char *lds) {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int n = 0; n < 2; ++n)
        b[C][n][ks] = *reinterpret_cast<const bf16x8 *>(lds + (slot + fb[ks]) + n * 16 * 128);
    slot = slot_after<1>(slot);
  }
  template <int HH, int C>
  __device__ __forceinline__ void mma() {
#pragma unroll
    for (int ks = 0; ks < 2; ++ks)
#pragma unroll
      for (int m = 0; m < 4; ++m)
#pragma unroll
        for (int n = 0; n < 2; ++n)
          acc[HH][C][m][n] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[C][n][ks], a[m][ks], acc[HH][C][m][n], 0, 0, 0);
  }
  // Copies of k step kt into the slot at `to`; steps past the last read
  // nothing and write zeros (no fragment of them is used), which keeps the
  // count of copies in flight. Before that the extents reach past the offset:
  // a 256-row tile has more than 128 valid rows and a tile at least 64 columns.
  template <int HH>
  __device__ __forceinline__ Copy copy_a(int kt, uint32_t to) const {
    const uint32_t off = HH * a_half + (uint32_t)kt * 128;
    return make_copy(A + off, kt < kt1 ? na - off : 0, lds0 + to);
  }
  template <int C>
  __device__ __forceinline__ Copy copy_b(int kt, uint32_t to) const {
    const uint32_t off = (uint32_t)kt * 128;
    return make_copy((C ? W1 : W0) + off, kt < kt1 ? (C ? nb1 : nb0) - off : 0, lds0 + to);
  }
};

// Between a phase's reads and its MFMAs: the region the next phase reads has
// landed (all but the N youngest copies of this wave), then every wave's has;
// the fragments read in this phase are in registers.
template <int N>
__device__ __forceinline__ void enter_mma() {
  wait_vm<N>();
  phase_barrier();
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
  __builtin_amdgcn_sched_barrier(0);
}

// The next phase's copy is prepared (scalar work) between this phase's MFMAs,
// so that a phase starts with its LDS reads: with the descriptor computed before
// them a phase took longer than the other group's MFMAs (2586 x 3584 x 18944,
// 154 workgroups: 327 us, with this 296).
__device__ __forceinline__ void spread_scalar() {
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);  // MFMA
    __builtin_amdgcn_sched_group_barrier(0x004, 2, 0);  // scalar
  }
}

// One k step of a 256-row tile. F is the column half of its first and last
// phase (0 on even steps, 1 on odd ones), whose fragments were read in the
// previous step's last phase. The regions pass through the ring of slots in the
// order in which they are read: A half 0, column half 1 - F, A half 1, column
// half 1 - F of the next step. Phase i copies the region that phase i + 8
// reads, into the slot whose region phase i - 2 read. n: the first phase's copy.
template <int F>
__device__ __forceinline__ void step_full(Tile<2> &s, Copy &n, int kt, const unsigned char *lds) {
  s.read_a(lds);
  issue(n, s.va);
  enter_mma<14>();
  n = s.copy_b<1 - F>(kt + 2, slot_after<8>(s.slot));
  s.mma<0, F>();
  spread_scalar();
  phase_barrier();
  s.read_b<1 - F>(lds);
  issue(n, s.vb);
  enter_mma<14>();
  n = s.copy_a<1>(kt + 2, slot_after<8>(s.slot));
  s.mma<0, 1 - F>();
  spread_scalar();
  phase_barrier();
  s.read_a(lds);
  issue(n, s.va);
  enter_mma<14>();
  n = s.copy_b<1 - F>(kt + 3, slot_after<8>(s.slot));
  s.mma<1, 1 - F>();
  spread_scalar();
  phase_barrier();
  s.read_b<1 - F>(lds);
  issue(n, s.vb);
  enter_mma<14>();
  n = s.copy_a<0>(kt + 3, slot_after<8>(s.slot));
  s.mma<1, F>();
  spread_scalar();
  phase_barrier();
}

// One k step of a 128-row tile: A; column half 1 and the next step's half 0.
__device__ __forceinline__ void step_half(Tile<1> &s, Copy &n, int kt, const unsigned char *lds) {
  s.read_a(lds);
  issue(n, s.vb);
  enter_mma<10>();
  n = s.copy_b<0>(kt + 3, slot_after<7>(s.slot));
  const Copy n2 = s.copy_a<0>(kt + 3, slot_after<8>(s.slot));
  s.mma<0, 0>();
  spread_scalar();
  phase_barrier();
  s.read_b<1>(lds);
  s.read_b<0>(lds);
  issue(n, s.vb);
  issue(n2, s.va);
  enter_mma<12>();
  n = s.copy_b<1>(kt + 3, slot_after<7>(s.slot));
  s.mma<0, 1>();
  spread_scalar();
  phase_barrier();
}

// One tile: rows m0 .. of H 128-row halves, column tile tc, k piece kp.
template <int H, bool GLU>
__device__ __forceinline__ void run_tile(const GemmPlan &p, int64_t m0, int tc, int unit, int kp, int k_parts,
                                         unsigned char *lds) {
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6), lane = threadIdx.x & 63;
  const int l16 = lane & 15, quad = lane >> 4, wm = wave >> 2, wn = wave & 3;
  int si = 0;
  while (si + 1 < p.j.n_segs && tc >= p.seg_tn[si]) tc -= p.seg_tn[si++];
  const GemmSeg &S = p.j.seg[si];
  constexpr int TN = GLU ? 128 : 256;  // output columns per tile
  const int n0 = tc * TN, N = S.N;
  const uint32_t rb = (uint32_t)p.j.K * 2;
  const int KT = p.j.K / kTK, k0 = (int)((int64_t)kp * KT / k_parts), k1 = (int)((int64_t)(kp + 1) * KT / k_parts);
  Tile<H> s;
  s.lds0 = (uint32_t)(uintptr_t)(lds_u8 *)lds + wave * 2048;
  s.slot = 0;
  s.kt1 = k1 - k0;
  const uint32_t ko = (uint32_t)k0 * 128;
  const uint32_t rows = (uint32_t)min((int64_t)128 * H, p.j.M - m0);
  s.A = static_cast<const unsigned char *>(p.j.A) + m0 * rb + ko;
  s.na = rows * rb - ko;
  s.a_half = 128 * rb;
  const unsigned char *W = static_cast<const unsigned char *>(S.W) + ko;
  const uint32_t cols = (uint32_t)min(TN, N - n0);
  if (GLU) {  // column half 0: gate rows, half 1: the matching up rows
    s.W0 = W + (int64_t)n0 * rb;
    s.W1 = W + ((int64_t)N + n0) * rb;
    s.nb0 = s.nb1 = cols * rb - ko;
  } else {    // column half h of wave wn: columns 64 wn + 32 h ..
    s.W0 = W + (int64_t)n0 * rb;
    s.W1 = s.W0 + 32 * (int64_t)rb;
    s.nb0 = cols * rb - ko;
    s.nb1 = s.nb0 - 32 * rb;
  }
#pragma unroll
  for (int i = 0; i < 2; ++i) {
    const uint32_t r = wave * 16 + i * 8 + lane / 8;
    const uint32_t c = ((lane & 7) ^ ((r >> 1) & 7)) << 4;
    s.va[i] = r * rb + c;
    s.vb[i] = (GLU ? r : (r >> 5) * 64 + (r & 31)) * rb + c;
  }
#pragma unroll
  for (int ks = 0; ks < 2; ++ks) {
    const int c = ((4 * ks + quad) ^ ((l16 >> 1) & 7)) << 4;
    s.fa[ks] = (wm * 64 + l16) * 128 + c;
    s.fb[ks] = (wn * 32 + l16) * 128 + c;
  }
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
      for (int m = 0; m < 4; ++m) s.acc[h][j][m][0] = s.acc[h][j][m][1] = f32x4{};

  // The first regions in the order in which they are read. Group 1 then falls
  // half a phase behind; group 0 waits for it at the end.
  int kt = 0;
  auto copy_a = [&](auto h, int k, int slot) { issue(s.template copy_a<decltype(h)::value>(k, slot * kRegion), s.va); };
  auto copy_b = [&](auto c, int k, int slot) { issue(s.template copy_b<decltype(c)::value>(k, slot * kRegion), s.vb); };
  constexpr std::integral_constant<int, 0> c0{};
  constexpr std::integral_constant<int, 1> c1{};
  copy_b(c0, 0, 0);
  copy_a(c0, 0, 1);
  copy_b(c1, 0, 2);
  if constexpr (H == 2) {
    copy_a(c1, 0, 3);
    copy_b(c1, 1, 4);
    copy_a(c0, 1, 5);
    copy_b(c0, 1, 6);
    copy_a(c1, 1, 7);
    copy_b(c0, 2, 8);
    wait_vm<14>();
  } else {
    copy_b(c0, 1, 3);
    copy_a(c0, 1, 4);
    copy_b(c1, 1, 5);
    copy_b(c0, 2, 6);
    copy_a(c0, 2, 7);
    wait_vm<12>();
  }
  phase_barrier();
  s.template read_b<0>(lds);
  __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0): slot 0 is written again in phase 1
  if (wm) phase_barrier();
  if constexpr (H == 2) {
    Copy n = s.template copy_a<0>(2, slot_after<8>(s.slot));
    for (;;) {
      step_full<0>(s, n, kt, lds);
      if (++kt == s.kt1) break;
      step_full<1>(s, n, kt, lds);
      if (++kt == s.kt1) break;
    }
  } else {
    Copy n = s.template copy_b<1>(2, slot_after<7>(s.slot));
    for (; kt < s.kt1; ++kt) step_half(s, n, kt, lds);
  }
  if (!wm) phase_barrier();
  wait_vm<0>();
  __syncthreads();  // no copy in flight, every wave is done with the regions

  // ---- epilogue -------------------------------------------------------------------
  // Each wave stages its 64 rows of a row half in fp32 in a region of its own
  // (rows of 256 B, gated 128 B, 16-byte chunks XOR-swizzled by row), then
  // each lane finishes 8 consecutive columns of a row, so that residual loads
  // and stores are 16 bytes of whole row segments.
  unsigned char *stg = lds + wave * kRegion;
  constexpr int CPR = GLU ? 4 : 8;        // lanes (8 columns each) per row
  const int cg = lane % CPR;
  const int n = n0 + wn * (TN / 4) + cg * 8;
  const bool n_ok = n < N;
  float bias[8];
  {
    bf16x8 bv = bf16x8{};
    if (!GLU && S.bias && k_parts == 1 && n_ok) bv = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(S.bias) + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) bias[e] = (float)bv[e];
  }
  // every residual piece before the first store (C may be the residual, so the
  // compiler cannot move a load over a store: a round trip each otherwise)
  bf16x8 res[H][CPR];
#pragma unroll
  for (int h = 0; h < H; ++h)
#pragma unroll
    for (int it = 0; it < CPR; ++it) {
      const int64_t m = m0 + h * 128 + wm * 64 + it * (64 / CPR) + lane / CPR;
      res[h][it] = bf16x8{};
      if (!GLU && p.j.residual && k_parts == 1 && m < p.j.M && n_ok)
        res[h][it] = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(p.j.residual) + m * N + n);
    }
#pragma unroll
  for (int h = 0; h < H; ++h) {
#pragma unroll
    for (int mb = 0; mb < 4; ++mb) {
      const int row = mb * 16 + l16;
      if (GLU) {
#pragma unroll
        for (int nb = 0; nb < 2; ++nb) {
          f32x4 v;
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const float g = s.acc[h][0][mb][nb][e];
            v[e] = g / (1.0f + __expf(-g)) * s.acc[h][1][mb][nb][e];
          }
          *reinterpret_cast<f32x4 *>(stg + row * 128 + (((nb * 4 + quad) ^ ((row >> 1) & 7)) << 4)) = v;
        }
      } else {
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
          for (int nb = 0; nb < 2; ++nb)
            *reinterpret_cast<f32x4 *>(stg + row * 256 + (((j * 8 + nb * 4 + quad) ^ l16) << 4)) = s.acc[h][j][mb][nb];
      }
    }
#pragma unroll
    for (int it = 0; it < CPR; ++it) {
      const int row = it * (64 / CPR) + lane / CPR;
      const int64_t m = m0 + h * 128 + wm * 64 + row;
      f32x4 v0, v1;
      if (GLU) {
        v0 = *reinterpret_cast<const f32x4 *>(stg + row * 128 + (((2 * cg) ^ ((row >> 1) & 7)) << 4));
        v1 = *reinterpret_cast<const f32x4 *>(stg + row * 128 + (((2 * cg + 1) ^ ((row >> 1) & 7)) << 4));
      } else {
        v0 = *reinterpret_cast<const f32x4 *>(stg + row * 256 + (((2 * cg) ^ (row & 15)) << 4));
        v1 = *reinterpret_cast<const f32x4 *>(stg + row * 256 + (((2 * cg + 1) ^ (row & 15)) << 4));
      }
      if (m >= p.j.M || !n_ok) continue;
      if (H == 1 && k_parts > 1) {
        float *dst = p.part + ((size_t)unit * k_parts + kp) * (128 * 256) + (size_t)(m - m0) * 256 + (n - n0);
        *reinterpret_cast<f32x4 *>(dst) = v0;
        *reinterpret_cast<f32x4 *>(dst + 4) = v1;
        continue;
      }
      float o[8] = {v0[0], v0[1], v0[2], v0[3], v1[0], v1[1], v1[2], v1[3]};
      if (!GLU) {
#pragma unroll
        for (int e = 0; e < 8; ++e) o[e] += (float)res[h][it][e];
      }
      bf16x8 out;
#pragma unroll
      for (int e = 0; e < 8; ++e) out[e] = (__bf16)(o[e] + bias[e]);
      *reinterpret_cast<bf16x8 *>(static_cast<__bf16 *>(S.C) + m * N + n) = out;
    }
  }
}

// 256-row tile t of the tile order: groups of kGroupM M-tiles sweep the
// column tiles.
__device__ __forceinline__ void tile_coords(const GemmPlan &p, int t, int &tm, int &tc) {
  const int span = kGroupM * p.tn;
  const int first_m = (t / span) * kGroupM;
  const int gsize = min(p.tiles_m - first_m, kGroupM);
  tm = first_m + (t % span) % gsize;
  tc = (t % span) / gsize;
}
// 128-row unit u: the halves of the cut tiles, then the last rows.
__device__ __forceinline__ void unit_coords(const GemmPlan &p, int u, int64_t &m0, int &tc) {
  if (u < 2 * p.n_cut) {
    int tm;
    tile_coords(p, p.n_full + u / 2, tm, tc);
    m0 = (int64_t)tm * 256 + (u & 1) * 128;
  } else {
    tc = u - 2 * p.n_cut;
    m0 = (int64_t)p.tiles_m * 256;
  }
}

// Workgroup i runs on XCD i mod 8: the whole tiles, and after them the units
// (piece-major), are cut into 8 contiguous ranges, one per XCD, so that
// neighbours in the order share A and W rows in that XCD's L2.
template <bool GLU>
__global__ __launch_bounds__(512, 2) void gemm_bf16_kernel(const GemmPlan p) {
  __shared__ __attribute__((aligned(1024))) unsigned char lds[kLds];
  const int xcd = blockIdx.x % kXcds, slot = blockIdx.x / kXcds;
  const int full_per = (p.n_full + kXcds - 1) / kXcds;
  if (slot < full_per) {
    const int t = xcd * full_per + slot;
    if (t >= p.n_full) return;
    int tm, tc;
    tile_coords(p, t, tm, tc);
    run_tile<2, GLU>(p, (int64_t)tm * 256, tc, 0, 0, 1, lds);
    return;
  }
  const int jobs = p.n_half * p.k_parts, per = (jobs + kXcds - 1) / kXcds;
  const int i = xcd * per + slot - full_per;
  if (slot - full_per >= per || i >= jobs) return;
  const int u = i % p.n_half;
  int tc;
  int64_t m0;
  unit_coords(p, u, m0, tc);
  run_tile<1, GLU>(p, m0, tc, u, i / p.n_half, p.k_parts, lds);
}

// The cut units' k pieces summed: C = sum of pieces (+ residual) (+ bias), in
// the order of the whole-tile epilogue. One thread per 8 columns of a row.
__global__ __launch_bounds__(256) void gemm_reduce_kernel(const GemmPlan p) {
  const int64_t gid = (int64_t)blockIdx.x * 256 + threadIdx.x;
  const int u = (int)(gid >> 12), row = (int)(gid >> 5) & 127, cg = (int)gid & 31;
  if (u >= p.n_half) return;
  int tc;
  int64_t m0;
  unit_coords(p, u, m0, tc);
  int si = 0;
  while (si + 1 < p.j.n_segs && tc >= p.seg_tn[si]) tc -= p.seg_tn[si++];
  const GemmSeg &S = p.j.seg[si];
  const int64_t m = m0 + row;
  const int n = tc * 256 + cg * 8;
  if (m >= p.j.M || n >= S.N) return;
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  const float *src = p.part + (size_t)u * p.k_parts * (128 * 256) + (size_t)row * 256 + cg * 8;
  for (int k = 0; k < p.k_parts; ++k) {
    const f32x4 a = *reinterpret_cast<const f32x4 *>(src + (size_t)k * (128 * 256));
    const f32x4 b = *reinterpret_cast<const f32x4 *>(src + (size_t)k * (128 * 256) + 4);
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      o[e] += a[e];
      o[4 + e] += b[e];
    }
  }
  if (p.j.residual) {
    const bf16x8 rv = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(p.j.residual) + m * S.N + n);
#pragma unroll
    for (int e = 0; e < 8; ++e) o[e] += (float)rv[e];
  }
  bf16x8 bv = bf16x8{};
  if (S.bias) bv = *reinterpret_cast<const bf16x8 *>(static_cast<const __bf16 *>(S.bias) + n);
  bf16x8 out;
#pragma unroll
  for (int e = 0; e < 8; ++e) out[e] = (__bf16)(o[e] + (float)bv[e]);
  *reinterpret_cast<bf16x8 *>(static_cast<__bf16 *>(S.C) + m * S.N + n) = out;
}

// Which tiles run whole, as halves or in k pieces. Rows beyond the last whole
// 256-row tile take one more 256-row tile if there are more than 128 of them,
// else 128-row units. Whole rounds of 256 tiles always run whole; the r tiles
// of a last, partial round run
//   whole, r + units workgroups:                one tile's time,
//   as 2 r halves if these fit the CUs:         0.6-0.65 of it (a k step of
//     a 128-row tile takes 0.57 us, of a 256-row tile 0.95-1.0 us while part of
//     the CUs is busy and the weights are in the caches, 0.8 and 1.2 us with
//     the weights from HBM, as in a program that goes through its layers),
//   as halves cut into P pieces along k:        1/P of that, plus the fp32
//     pieces written and read back (128 KiB each) and the reduction's launch
//     (10 us in all for 224 pieces, and about 4 us more of the tiles' stores),
// whichever the figures below say is shortest.
void plan_job(GemmPlan &p, size_t part_bytes) {
  const GemmJob &j = p.j;
  const int tn_out = j.glu ? 128 : 256;
  p.tn = 0;
  for (int i = 0; i < j.n_segs; ++i) {
    p.seg_tn[i] = (j.seg[i].N + tn_out - 1) / tn_out;
    p.tn += p.seg_tn[i];
  }
  const int rest = (int)(j.M % 256);
  p.tiles_m = (int)(j.M / 256) + (rest > 128 ? 1 : 0);
  const int edge = rest > 0 && rest <= 128 ? p.tn : 0;  // 128-row units of the last rows
  const int n_tiles = p.tiles_m * p.tn, r = n_tiles % kCus;
  const double kt = j.K / kTK;
  const double whole_us = 1.2 * kt + 8.0;
  auto half_us = [&](double k) { return 0.8 * k + 6.0; };
  p.n_cut = 0;
  p.k_parts = 1;
  const int units = 2 * r + edge;
  double best = r ? whole_us + (r + edge > kCus ? half_us(kt) : 0.0) : half_us(kt) * ((edge + kCus - 1) / kCus);
  if (units > 0 && units <= kCus) {
    for (int parts = 1; parts * units <= kCus && (parts == 1 || 2 * parts <= kt); ++parts) {
      if (parts > 1 && (p.part == nullptr || j.glu || (size_t)units * parts * 128 * 256 * 4 > part_bytes)) break;
      const double us = half_us(kt / parts) + (parts > 1 ? 5.0 + units * parts * 0.04 : 0.0);
      if (us < best) {
        best = us;
        p.n_cut = r;
        p.k_parts = parts;
      }
    }
  }
  p.n_full = n_tiles - p.n_cut;
  p.n_half = 2 * p.n_cut + edge;
}

}  // namespace

hipError_t launch_gemm_job(const GemmJob &job, float *part, size_t part_bytes, hipStream_t st) {
  GemmPlan p{};
  p.j = job;
  p.part = part;
  if (job.M <= 0 || job.n_segs <= 0) return hipSuccess;
  if (!job.glu && part == nullptr && job.n_segs == 1 && small_tiles_pay(job.M, job.seg[0].N, job.K))
    return launch_gemm_small(job, st);
  plan_job(p, part_bytes);
  const int blocks = kXcds * ((p.n_full + kXcds - 1) / kXcds + (p.n_half * p.k_parts + kXcds - 1) / kXcds);
  if (job.glu) gemm_bf16_kernel<true><<<dim3(blocks), dim3(512), 0, st>>>(p);
  else gemm_bf16_kernel<false><<<dim3(blocks), dim3(512), 0, st>>>(p);
  if (p.k_parts > 1) gemm_reduce_kernel<<<dim3(p.n_half * 16), dim3(256), 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace daf
