// bf16 causal GQA flash attention for both DAF attention stages (gfx950).
//
// Same operation and work decomposition as the fp32 kernel in attn.hip (see
// there): query row i of a request sees keys 0 .. i + (n_keys - n_rows), a
// workgroup of 4 waves owns 128 query rows (64 where that fills more CUs) of
// one head and one key split, and the G heads that share a KV head form an
// XCD-local work group.
//
// bf16 data path, per 64-key tile:
//  * K and V tiles are copied global -> LDS by the buffer unit
//    (buffer_load_dwordx4 ... lds): no VGPR staging, no VALU address math in
//    the loop, and rows past the end of the request read as zeros through the
//    buffer range check. Each 1 KiB DMA instruction writes 1024/(2D) whole rows;
//    16-byte chunks are XOR-swizzled within a row so that the two LDS read
//    patterns below are free of bank conflicts. Two tile buffers: the DMA of
//    tile t+1 runs while tile t is consumed, one barrier per tile.
//  * S^T = K Q^T on v_mfma_f32_16x16x32_bf16 (16 keys on M, 16 query rows on N,
//    Q in registers): a lane holds 4 keys of one row.
//  * O^T += V^T P^T: P^T comes straight from the S^T accumulators (contraction
//    slots in the order in which a lane holds its keys); the V^T operand is
//    read from the row-major V tile with ds_read_b64_tr_b16, which transposes
//    16-bit data across each 16-lane group.
//  * Softmax in fp32, base 2, scale folded into one FMA per score, against a
//    running reference per row, so no max of the scores is taken: the half
//    tile's probabilities are formed and rounded, and only if one of them has
//    reached 2^28 (a packed maximum of their bits) is the exact max taken, the
//    reference raised, O and the sum rescaled and the half formed again. A split's
//    first tile and masked tiles take the max of their 64 keys beforehand.
//  * The row sum is one more MFMA per half tile and 16 rows, of the rounded
//    probabilities against ones.
//
// What bounds it: how far a wave's phases (S from K fragments, softmax, P V from
// V fragments) overlap with those of the one other wave of its SIMD (two fit: 256
// VGPRs and 64 KiB of LDS per workgroup), and the clock, which the chip's power
// sets. Stage 1 at n = 4915, 28 heads of 128 (profiles of the standalone call): the
// matrix cores are busy 47% of the cycles and VALU issue 41%; the 32 KiB of
// fragments per tile and wave need 48% of the LDS's 128 bytes per cycle. Copies of
// the kernel with one part taken out (163 us whole): 143 us without the softmax,
// 122 without the fragments' LDS reads, 105 without both, 148 without the copies
// to LDS; the matrix work alone is 83 us at that clock.
//   16x16x32 MFMAs need less power per FLOP than 32x32x16, and beside a wave that
// issues MFMAs back to back a v_dot2 waits about 50 cycles, so 4 MFMAs per tile
// took the place of 16 v_dot2 for the row sums: 173 us with 32x32x16 MFMAs and
// v_dot2, 166 with 16x16x32, 163 with the sum on the matrix cores; 5043 rows at
// positions of 32896 keys: 1122, 1062 and 1045 us.
//
// Launch shape for causal self attention: the heaviest 128 jobs of an XCD (one
// query head of one 128-row block each) are run by its 64 resident workgroups
// in pairs, job u with job 127 - u, so each workgroup gets a heavy and a light
// block of near-equal total; lighter jobs get a workgroup each.
#include <math.h>

#include <algorithm>

#include "daf_internal.h"

namespace daf {
namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;

constexpr int kBN = 64;                  // keys per tile
[[maybe_unused]] constexpr int kRsrcWord3 = 0x00020000;  // raw buffer descriptor word 3 (gfx9 family)
// Probabilities are formed against a running reference per row, the largest
// scaled score at its last raise: 1 there, so that products with values down to
// the smallest normal ones stay normal in fp32. Only if a probability reaches
// 2^28 (kLimit, its bf16 bits; at most 2^32 per 16 keys) is the exact max taken,
// the reference raised and the probabilities formed again.
constexpr unsigned kLimit = (127 + 28) << 7;
// A split of at most kShortSplit tiles (stage 2 with few key tiles per workgroup,
// whose splits would otherwise be half as long) raises it past 2^6: the LSE's error
// against 64 bits (1473 keys, 243 rows, 8 heads of 64) is 1.03e-5 with one tile per
// split, with two 1.05e-5 at 2^28 and 1.01e-5 at 2^6; stage 2 takes 0-2% longer.
constexpr unsigned kShortLimit = (127 + 6) << 7;
constexpr int kShortSplit = 10;
constexpr float kMaskedSlack = 8.0f;    // growth (log2) of a row's max that raises the reference in a masked tile
constexpr float kNoReference = -3e38f;  // before the first key: every visible one's probability is infinite

template <int D>
struct Geo {
  static constexpr int ROWB = D * 2;         // bytes per K/V row in LDS
  static constexpr int CH = D / 8;           // 16-byte chunks per row
  static constexpr int TILE = kBN * ROWB;    // bytes of one K or V tile
  static constexpr int RPI = 64 / CH;        // rows written by one 1 KiB DMA instruction
  static constexpr int IPW = kBN / RPI / 4;  // DMA instructions per wave, per tensor and tile
  static constexpr int DS = D / 32;          // contraction steps of S^T
  static constexpr int DB = D / 16;          // 16-feature output blocks
  static_assert(RPI * ROWB == 1024, "one DMA instruction writes 1 KiB");
};

// chunk swizzles (XOR, so their own inverse), both < CH. K: the 16 lanes of a
// read phase take one chunk of 16 consecutive rows; V: the 32 lanes of a phase
// take a pair of chunks of 8 consecutive rows. 128-byte rows (CH = 8) already
// alternate between the halves of the banks.
__device__ __forceinline__ int swz_k(int r, int ch) { return ch == 16 ? r & 15 : (r >> 1) & 7; }
__device__ __forceinline__ int swz_v(int r, int ch) { return ch == 16 ? (r & 7) << 1 : ((r >> 1) & 3) << 1; }

__device__ __forceinline__ float fast_exp2(float x) { return __builtin_amdgcn_exp2f(x); }

// x and the same register of lane ^ 32: v_permlane32_swap on two copies of x
// leaves {x[l % 32], x[l % 32 + 32]} in the two results. Each result element
// is copied to a scalar before the bit cast (a bit cast of a vector element
// expression reads the vector's first element).
__device__ __forceinline__ void lane_pair(float x, float &a, float &b) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  a = __builtin_bit_cast(float, r0);
  b = __builtin_bit_cast(float, r1);
}
// the same for lane ^ 16
__device__ __forceinline__ void lane_pair16(float x, float &a, float &b) {
  const unsigned u = __builtin_bit_cast(unsigned, x);
  const auto r = __builtin_amdgcn_permlane16_swap(u, u, false, false);
  const unsigned r0 = r[0], r1 = r[1];
  a = __builtin_bit_cast(float, r0);
  b = __builtin_bit_cast(float, r1);
}
// over the four lanes that share a query row (lane mod 16)
__device__ __forceinline__ float row_max(float x) {
  float a, b;
  lane_pair(x, a, b);
  lane_pair16(fmaxf(a, b), a, b);
  return fmaxf(a, b);
}

__device__ __forceinline__ bf16x8 tr_pair(const unsigned char *lds_base, int off_a, int off_b) {
  const lds_u8 *b = (const lds_u8 *)lds_base;
  const bf16x4 a = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(b + off_a));
  const bf16x4 c = __builtin_amdgcn_ds_read_tr16_b64_v4bf16((lds_bf16x4 *)(b + off_b));
  return bf16x8{a[0], a[1], a[2], a[3], c[0], c[1], c[2], c[3]};
}

// Copy one 64-key K tile and V tile global -> LDS with the buffer unit. Each
// wave writes its IPW KiB of each tile; rows at or past n_keys read as zero.
template <int IPW>
__device__ __forceinline__ void dma_tile(const unsigned char *kg, const unsigned char *vg, int kb, int n_keys,
                                         int kv_row_bytes, unsigned char *k_lds, unsigned char *v_lds, int wave,
                                         const int (&dma_k)[IPW], const int (&dma_v)[IPW]) {
  // The buffer->LDS builtin only exists for the GPU target; the host pass of
  // this translation unit only needs the kernel's launch stub.
#if defined(__HIP_DEVICE_COMPILE__)
  const int nrec = (n_keys - kb) * kv_row_bytes;
  const __amdgpu_buffer_rsrc_t rk =
      __builtin_amdgcn_make_buffer_rsrc((void *)(kg + (size_t)kb * kv_row_bytes), 0, nrec, kRsrcWord3);
  const __amdgpu_buffer_rsrc_t rv =
      __builtin_amdgcn_make_buffer_rsrc((void *)(vg + (size_t)kb * kv_row_bytes), 0, nrec, kRsrcWord3);
  lds_u8 *kbase = (lds_u8 *)k_lds + wave * IPW * 1024;
  lds_u8 *vbase = (lds_u8 *)v_lds + wave * IPW * 1024;
#pragma unroll
  for (int i = 0; i < IPW; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rk, (void __attribute__((address_space(3))) *)(kbase + i * 1024), 16,
                                             dma_k[i], 0, 0, 0);
#pragma unroll
  for (int i = 0; i < IPW; ++i)
    __builtin_amdgcn_raw_ptr_buffer_load_lds(rv, (void __attribute__((address_space(3))) *)(vbase + i * 1024), 16,
                                             dma_v[i], 0, 0, 0);
#endif
}

// Output staging: up to 32 rows of ROWB bytes per wave in LDS, the 16-byte chunks of
// a row XOR-swizzled by the row so that both the per-lane writes (pieces of
// every chunk of one row) and the row-contiguous reads spread over the banks.
// stage_put writes v (8 or 16 bytes) at byte `sub` of logical chunk c of row r.
template <int D, typename V>
__device__ __forceinline__ void stage_put(unsigned char *stg, int r, int c, int sub, const V &v) {
  constexpr int CH = Geo<D>::CH;
  *reinterpret_cast<V *>(stg + r * Geo<D>::ROWB + ((c ^ (r & (CH - 1))) << 4) + sub) = v;
}
// Write the wave's staged rows wrow .. wrow+ROWS-1 (those below n_rows): each lane
// moves one 16-byte chunk, CH lanes cover a row, so every store instruction
// writes 64/CH whole rows. dst(r) is the byte address of row r's first chunk.
template <int D, int ROWS, typename F>
__device__ __forceinline__ void store_rows(const unsigned char *stg, int lane, int wrow, int n_rows, F dst) {
  constexpr int CH = Geo<D>::CH, RPL = 64 / CH;
  const int j = lane % CH;
#pragma unroll
  for (int it = 0; it < ROWS / RPL; ++it) {
    const int r = it * RPL + lane / CH;
    const u32x4 v = *reinterpret_cast<const u32x4 *>(stg + r * Geo<D>::ROWB + ((j ^ (r & (CH - 1))) << 4));
    if (wrow + r < n_rows) *reinterpret_cast<u32x4 *>(dst(wrow + r) + j * 16) = v;
  }
}

// Per-wave state of one workgroup tile (lives in registers after inlining). A
// wave has 16 NB rows; a lane works on rows lane % 16 + 16 nb, nb < NB, and the
// four lanes of a row split its keys.
template <int D, int NB>
struct WaveState {
  using Gm = Geo<D>;
  bf16x8 qf[NB][Gm::DS];    // Q rows as the B operand of S^T
  f32x4 oacc[NB][Gm::DB];   // O^T accumulators
  float m_run[NB];          // running reference, scaled base-2 units, equal in a row's four lanes
  f32x4 lacc[NB];           // row sums of the rounded probabilities (four equal elements)
  int koff[Gm::DS];        // K tile read offsets
  int voff[Gm::DB];        // V tile transposed-read offsets
  int dma_k[Gm::IPW], dma_v[Gm::IPW];
  const unsigned char *kg, *vg;
  int n_keys, kv_row_bytes, limit[NB], quad, wave;
  int wave_last_key;       // keys above this are masked for every row of the wave
  int wave_first_limit;    // keys up to this are visible to every row of the wave
  float sl2;
  unsigned p_limit;        // bf16 bits of the probability that raises the reference
};

// Scores of one 32-key half tile: [16-key block][row block], D^T blocks: a
// lane holds 4 consecutive keys of one row.
template <int NB>
using Scores = f32x4[2][NB];

// The larger of three bf16 values, in both halves of a word: bits of values that
// are not negative order alike as fp16, and a pattern of an fp16 NaN (2^121 and
// more) stays one. Two of these per 16 rows and half tile; as four integer
// maxima of two words they cost the 32k layer 1.6% and position_attn at 16k 4%.
__device__ __forceinline__ unsigned max3_pairs(unsigned a, unsigned b, unsigned c) {
  unsigned r;
  asm("v_pk_maximum3_f16 %0, %1, %2, %3" : "=v"(r) : "v"(a), "v"(b), "v"(c));
  return r;
}

// P^T operands (bf16) of one 32-key half, against the running reference m.
// Returns the largest of their bit patterns (which order like the values: none is
// negative), over the even and over the odd ones.
template <int D, int NB>
__device__ __forceinline__ unsigned softmax_half(const WaveState<D, NB> &w, const Scores<NB> &sc, const float (&m)[NB],
                                                 bf16x8 (&pf)[NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int r = 0; r < 8; ++r)
      pf[nb][r] = (__bf16)fast_exp2(__builtin_fmaf(sc[r >> 2][nb][r & 3], w.sl2, -m[nb]));
  const u32x4 a = __builtin_bit_cast(u32x4, pf[0]);
  unsigned top = max3_pairs(max3_pairs(a[0], a[1], a[2]), a[3], a[3]);
  if constexpr (NB == 2) {
    const u32x4 b = __builtin_bit_cast(u32x4, pf[1]);
    top = max3_pairs(max3_pairs(max3_pairs(max3_pairs(a[0], a[1], a[2]), a[3], b[0]), b[1], b[2]), b[3], b[3]);
  }
  return top;
}
__device__ __forceinline__ bool out_of_range(unsigned top, unsigned limit) {
  return __builtin_amdgcn_ballot_w64(top >= limit << 16 || (top & 0xffffu) >= limit) != 0;
}

// O^T += V^T P^T over the 32 keys of one half tile. Contraction slot 8 g + j of
// lane group g is key 4 g + j of the half's first 16 keys (j < 4) or key 4 g +
// j - 4 of its last 16: the keys whose scores that group holds.
template <int D, int NB>
__device__ __forceinline__ void read_v(const WaveState<D, NB> &w, const unsigned char *vs, bf16x8 (&a)[Geo<D>::DB]) {
#pragma unroll
  for (int db = 0; db < Geo<D>::DB; ++db) a[db] = tr_pair(vs, w.voff[db], w.voff[db] + 16 * Geo<D>::ROWB);
}
template <int D, int NB>
__device__ __forceinline__ void pv_half(WaveState<D, NB> &w, const bf16x8 (&a)[Geo<D>::DB], const bf16x8 (&pf)[NB]) {
#pragma unroll
  for (int db = 0; db < Geo<D>::DB; ++db)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
      w.oacc[nb][db] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[db], pf[nb], w.oacc[nb][db], 0, 0, 0);
  const __bf16 one = (__bf16)1.0f;
  const bf16x8 ones = {one, one, one, one, one, one, one, one};
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) w.lacc[nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(ones, pf[nb], w.lacc[nb], 0, 0, 0);
}

// Raise the running references to the rows' maxima mt, rescaling O and the row
// sums.
template <int D, int NB>
__device__ __forceinline__ void raise_to(WaveState<D, NB> &w, const float (&mt)[NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float m_new = fmaxf(w.m_run[nb], mt[nb]);
    const float alpha = fast_exp2(w.m_run[nb] - m_new);
    w.m_run[nb] = m_new;
    w.lacc[nb] *= alpha;
#pragma unroll
    for (int db = 0; db < Geo<D>::DB; ++db) w.oacc[nb][db] *= alpha;
  }
}
template <int D, int NB>
__device__ __forceinline__ void half_max(const WaveState<D, NB> &w, const Scores<NB> &sc, float (&mt)[NB]) {
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    float mx = sc[0][nb][0];
#pragma unroll
    for (int r = 1; r < 8; ++r) mx = fmaxf(mx, sc[r >> 2][nb][r & 3]);
    mt[nb] = row_max(mx) * w.sl2;
  }
}
// Probabilities of a half tile: against the running reference as it stands,
// and again after raising it if one of them is out of range.
template <int D, int NB>
__device__ __forceinline__ void finish_half(WaveState<D, NB> &w, const Scores<NB> &sc, bf16x8 (&pf)[NB], unsigned top) {
  if (out_of_range(top, w.p_limit)) {
    float mt[NB];
    half_max<D, NB>(w, sc, mt);
    raise_to<D, NB>(w, mt);
    softmax_half<D, NB>(w, sc, w.m_run, pf);
  }
}

// One 64-key tile: S^T = K Q^T, online softmax, O^T update. MASK selects the
// variant for diagonal tiles (causal mask, possibly a fully masked second half)
// and for the first tile.
// Full tiles check one 32-key half at a time against the reference, so the S
// MFMAs of half 1 overlap the softmax of half 0 and the P.V MFMAs of half 0 that
// of half 1.
template <int D, int NB, bool MASK>
__device__ __forceinline__ void tile_math(WaveState<D, NB> &w, const unsigned char *ks, const unsigned char *vs, int kb) {
  constexpr int ROWB = Geo<D>::ROWB, DS = Geo<D>::DS;
  if (!MASK) {
    bf16x8 kf[4][DS];
#pragma unroll
    for (int b = 0; b < 4; ++b)
#pragma unroll
      for (int ds = 0; ds < DS; ++ds) kf[b][ds] = *reinterpret_cast<const bf16x8 *>(ks + b * 16 * ROWB + w.koff[ds]);
    Scores<NB> s0 = {}, s1 = {};
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s0[b][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[b][ds], w.qf[nb][ds], s0[b][nb], 0, 0, 0);
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb) s1[b][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[2 + b][ds], w.qf[nb][ds], s1[b][nb], 0, 0, 0);
    bf16x8 pf0[NB], pf1[NB];
    const unsigned top0 = softmax_half<D, NB>(w, s0, w.m_run, pf0);
    // scheduling: K reads of half 0, the S MFMAs of half 0 in pairs beside a K
    // read of half 1, then the S MFMAs of half 1 in pairs beside a share of
    // the softmax of half 0
    __builtin_amdgcn_sched_group_barrier(0x100, 2 * DS, 0);
#pragma unroll
    for (int i = 0; i < 2 * DS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
      __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
    }
#pragma unroll
    for (int i = 0; i < 2 * DS; ++i) {
      __builtin_amdgcn_sched_group_barrier(0x008, NB, 0);
      __builtin_amdgcn_sched_group_barrier(0x002, 3 * NB, 0);
    }
    finish_half<D, NB>(w, s0, pf0, top0);
    bf16x8 v[Geo<D>::DB];
    read_v<D, NB>(w, vs, v);
    pv_half<D, NB>(w, v, pf0);
    const unsigned top1 = softmax_half<D, NB>(w, s1, w.m_run, pf1);
    finish_half<D, NB>(w, s1, pf1, top1);
    read_v<D, NB>(w, vs + 32 * ROWB, v);
    pv_half<D, NB>(w, v, pf1);
    return;
  }
  const bool second = kb + 32 <= w.wave_last_key;
  Scores<NB> sc[2];
#pragma unroll
  for (int h = 0; h < 2; ++h) {
#pragma unroll
    for (int b = 0; b < 2; ++b) for (int nb = 0; nb < NB; ++nb) sc[h][b][nb] = f32x4{};
    if (h == 1 && !second) continue;
    bf16x8 kf[2][DS];
#pragma unroll
    for (int b = 0; b < 2; ++b)
#pragma unroll
      for (int ds = 0; ds < DS; ++ds)
        kf[b][ds] = *reinterpret_cast<const bf16x8 *>(ks + (2 * h + b) * 16 * ROWB + w.koff[ds]);
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          sc[h][b][nb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(kf[b][ds], w.qf[nb][ds], sc[h][b][nb], 0, 0, 0);
  }
  if (kb + kBN - 1 > w.wave_first_limit) {  // not so in most first tiles
#pragma unroll
    for (int h = 0; h < 2; ++h)
#pragma unroll
      for (int b = 0; b < 2; ++b)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int e = 0; e < 4; ++e) {
            const int key = kb + 32 * h + 16 * b + 4 * w.quad + e;
            if (key > w.limit[nb]) sc[h][b][nb][e] = -INFINITY;
          }
  }
  // The max of the whole tile, and the reference raised past a growth of
  // kMaskedSlack: a key that dominates its row from here on has a probability of
  // 1, which bf16 holds exactly, so that its weight in the row's sum is exact
  // too. Against the max of the first tile's first half instead, LSE errors (2-norm
  // against 64 bits) were up to 2% larger in stage 1 and 19% in stage 2 with two
  // tiles per split; the times are level (one layer of 32k tokens 250.9 and 251.4 us).
  float mt[NB], m1[NB];
  half_max<D, NB>(w, sc[0], mt);
  half_max<D, NB>(w, sc[1], m1);
  bool raise = false;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    mt[nb] = fmaxf(mt[nb], m1[nb]);
    raise |= mt[nb] > w.m_run[nb] + kMaskedSlack;
  }
  if (__builtin_amdgcn_ballot_w64(raise) != 0) raise_to<D, NB>(w, mt);
#pragma unroll
  for (int h = 0; h < 2; ++h) {
    if (h == 1 && !second) break;
    bf16x8 pf[NB], v[Geo<D>::DB];
    softmax_half<D, NB>(w, sc[h], w.m_run, pf);
    read_v<D, NB>(w, vs + h * 32 * ROWB, v);
    pv_half<D, NB>(w, v, pf);
  }
}

// One 64-key tile read from buffer `ks`/`vs`; the DMA of the next tile goes to
// `nk`/`nv`. The buffers are distinct LDS objects at each call site.
template <int D, int NB>
__device__ __forceinline__ void tile_step(WaveState<D, NB> &w, const unsigned char *ks, const unsigned char *vs,
                                          unsigned char *nk, unsigned char *nv, int kb, bool first, bool prefetch) {
  // Wait for this wave's DMA of this tile (the only vector-memory work in
  // flight; the compiler does not count LDS DMA as a store to release), then
  // barrier: every wave's DMA has landed and every wave is done reading the
  // other buffer (previous tile). The fences of __syncthreads keep the
  // compiler from moving LDS reads or the next DMA across the barrier.
  __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0); expcnt and lgkmcnt left at their maxima
  __syncthreads();
  if (prefetch) dma_tile<Geo<D>::IPW>(w.kg, w.vg, kb + kBN, w.n_keys, w.kv_row_bytes, nk, nv, w.wave, w.dma_k, w.dma_v);
  if (kb > w.wave_last_key) return;               // the whole tile is masked for this wave
  if (first || kb + kBN - 1 > w.wave_first_limit) tile_math<D, NB, true>(w, ks, vs, kb);
  else tile_math<D, NB, false>(w, ks, vs, kb);
}

// One job: the work of launch slot `slot` of XCD `xcd` (one query head of one
// work group, or one packed stage-2 unit group), run by the whole workgroup.
template <int D, int KIND, int NB>
__device__ __forceinline__ void attn_job(const AttnLaunch &p, const AttnList &l, const int xcd, const int slot, unsigned char *k_lds0,
                                         unsigned char *v_lds0, unsigned char *k_lds1, unsigned char *v_lds1) {
  using Gm = Geo<D>;
  constexpr int ROWB = Gm::ROWB, CH = Gm::CH, TILE = Gm::TILE, IPW = Gm::IPW, DS = Gm::DS, DB = Gm::DB;
  constexpr int RPI = Gm::RPI;
  // ---- which work -----------------------------------------------------------
  // A work group is the G heads that share one KV head, for one entry, query
  // block and key split. When Hkv divides the 8 XCDs, each XCD serves one KV
  // head (8/Hkv XCDs per head, dealt alternately a, b, b, a, ...), so every L2
  // holds the K/V of a single head;
  // otherwise work groups are dealt to the XCDs round-robin. Within an XCD,
  // work groups run heaviest first, and the G heads of a work group are
  // consecutive workgroups of that XCD.
  const int G = p.group, WPG = l.wgs_per_group;
  const int hl = slot % WPG;
  int g, lam;  // KV head, index of the work group among that head's work groups
  if (kXcds % p.hkv == 0) {
    const int xph = kXcds / p.hkv;
    g = xcd / xph;
    // work groups of a head are dealt to its xph XCDs in boustrophedon order
    // (a, b, b, a, ...), so the XCDs get equal shares of the heaviest-first list
    const int q = slot / WPG, r = xcd % xph;
    lam = q * xph + ((q & 1) ? xph - 1 - r : r);
    if (lam * p.hkv >= l.n_groups) return;
  } else {
    const int gamma = (slot / WPG) * kXcds + xcd;
    if (gamma >= l.n_groups) return;
    g = gamma % p.hkv;
    lam = gamma / p.hkv;
  }
  int ei = l.e0;
  while (ei + 1 < l.e0 + l.n_entries && p.e[ei + 1].group0 <= lam * p.hkv) ++ei;
  const AttnEntry &E = p.e[ei];
  const int ll = lam - E.group0 / p.hkv;
  const int s = ll % E.n_splits;
  const int mb = E.mb_hi - ll / E.n_splits;

  const int n_rows = E.n_rows;
  const int n_keys = E.n_keys;
  const int tid = threadIdx.x;
  const int wave = tid >> 6;
  // this wave's query head and first row, and the workgroup's last row
  int h, wrow0, row_last;
  if (KIND == 1 && WPG == 1) {
    // packed units (the split-key kernel always runs packed; with G = 1 the
    // units of a workgroup are 4 consecutive row blocks of one head): unit u = (head hl_u, 32-row block rb_u), u = hl_u * n_rb + rb_u
    const int n_rb = (n_rows + 31) / 32, n_units = G * n_rb;
    const int u = mb * 4 + wave;
    h = g * G + min(u, n_units - 1) / n_rb;
    wrow0 = u < n_units ? (u % n_rb) * 32 : n_rows;  // a wave past the last unit has no rows
    row_last = 0;
    for (int j = 0; j < 4; ++j) {
      const int uj = mb * 4 + j;
      if (uj < n_units) row_last = max(row_last, min((uj % n_rb) * 32 + 31, n_rows - 1));
    }
  } else {
    h = g * G + hl;
    wrow0 = (mb * 4 + wave) * (16 * NB);
    row_last = min((mb + 1) * (64 * NB), n_rows) - 1;
  }
  const int k_begin = s * E.split_keys;
  const int k_end = min(min(k_begin + E.split_keys, n_keys), row_limit(E, row_last) + 1);
  const int n_tiles = k_end > k_begin ? (k_end - k_begin + kBN - 1) / kBN : 0;

  const int lane = tid & 63;
  const int l16 = lane & 15;
  const int quad = lane >> 4;
  const int my_row = wrow0 + l16;  // and my_row + 16 with NB = 2
  // keys above this are masked for the whole wave (a wave past the last row has none)
  const int wave_last_key = wrow0 < n_rows ? row_limit(E, wrow0 + 16 * NB - 1) : -1;

  WaveState<D, NB> w;
  w.kg = static_cast<const unsigned char *>(E.k);
  w.vg = static_cast<const unsigned char *>(E.v);
  w.n_keys = n_keys;
  w.kv_row_bytes = p.hkv * D * 2;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) w.limit[nb] = row_limit(E, my_row + 16 * nb);
  w.wave_last_key = wave_last_key;
  w.wave_first_limit = row_limit(E, wrow0);
  w.quad = quad;
  w.wave = wave;
  w.sl2 = p.scale_log2;
  w.p_limit = KIND == 1 && E.split_keys <= kShortSplit * kBN ? kShortLimit : kLimit;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    w.m_run[nb] = kNoReference;
    w.lacc[nb] = f32x4{};
#pragma unroll
    for (int db = 0; db < DB; ++db) w.oacc[nb][db] = f32x4{};
    const int row = my_row + 16 * nb;
    const __bf16 *qp = static_cast<const __bf16 *>(E.q) + ((size_t)row * p.hq + h) * D + 8 * quad;
#pragma unroll
    for (int ds = 0; ds < DS; ++ds)
      w.qf[nb][ds] = row < n_rows ? *reinterpret_cast<const bf16x8 *>(qp + 32 * ds) : bf16x8{};
  }
#pragma unroll
  for (int i = 0; i < IPW; ++i) {
    const int r = (wave * IPW + i) * RPI + lane / CH;
    const int pc = lane % CH;
    w.dma_k[i] = r * w.kv_row_bytes + g * D * 2 + ((pc ^ swz_k(r, CH)) << 4);
    w.dma_v[i] = r * w.kv_row_bytes + g * D * 2 + ((pc ^ swz_v(r, CH)) << 4);
  }
#pragma unroll
  for (int ds = 0; ds < DS; ++ds) w.koff[ds] = l16 * ROWB + (((4 * ds + quad) ^ swz_k(l16, CH)) << 4);
  {
    // transposed read: lane 4 r + c of a 16-lane group addresses key 4 quad + r,
    // features 4 c .. 4 c + 3 of the block, and receives 4 keys of one feature
    const int key = 4 * quad + (l16 >> 2), sw = swz_v(key, CH);
#pragma unroll
    for (int db = 0; db < DB; ++db)
      w.voff[db] = key * ROWB + (((2 * db + ((l16 & 3) >> 1)) ^ sw) << 4) + 8 * (l16 & 1);
  }

  if (n_tiles > 0) dma_tile<IPW>(w.kg, w.vg, k_begin, n_keys, w.kv_row_bytes, k_lds0, v_lds0, wave, w.dma_k, w.dma_v);
  for (int t = 0; t < n_tiles; t += 2) {
    // even tiles live in buffer 0, odd tiles in buffer 1
    int kb = k_begin + t * kBN;
    tile_step<D, NB>(w, k_lds0, v_lds0, k_lds1, v_lds1, kb, t == 0, t + 1 < n_tiles);
    if (t + 1 < n_tiles) {
      kb += kBN;
      tile_step<D, NB>(w, k_lds1, v_lds1, k_lds0, v_lds0, kb, false, t + 2 < n_tiles);
    }
  }

  // ---- epilogue ---------------------------------------------------------------
  float inv[NB], lse_nat[NB];
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    const float l_tot = w.lacc[nb][0];
    inv[nb] = l_tot > 0.f ? 1.f / l_tot : 0.f;
    lse_nat[nb] = l_tot > 0.f ? (w.m_run[nb] + __log2f(l_tot)) * 0.69314718055994531f : -INFINITY;
  }
  // Rows go out through LDS so that every store is a 16-byte piece of a
  // contiguous row (a lane holds 4-feature pieces of one row, spread over the
  // row). Each wave stages in its own quarter of the stage buffer that did
  // not hold the last tile: every wave finished reading it before the last
  // barrier and no copy targets it any more.
  unsigned char *stg = ((n_tiles & 1) ? (wave < 2 ? k_lds1 : v_lds1) : (wave < 2 ? k_lds0 : v_lds0)) +
                       (wave & 1) * (TILE / 2);
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int db = 0; db < DB; ++db) {
      bf16x4 v;
#pragma unroll
      for (int t = 0; t < 4; ++t) v[t] = (__bf16)(w.oacc[nb][db][t] * inv[nb]);
      stage_put<D>(stg, nb * 16 + l16, 2 * db + (quad >> 1), 8 * (quad & 1), v);
    }
  const int wrow = wrow0;  // first row of this wave
  if (E.n_splits == 1 && E.o != nullptr) {
    store_rows<D, 16 * NB>(stg, lane, wrow, n_rows, [&](int r) {
      return static_cast<unsigned char *>(E.o) + ((size_t)r * p.hq + h) * D * 2;
    });
    if (E.o2 != nullptr)
      store_rows<D, 16 * NB>(stg, lane, wrow, n_rows, [&](int r) {
        const int64_t r2 = E.o2_row0 + (E.o2_idx ? E.o2_idx[r] : r);
        return static_cast<unsigned char *>(E.o2) + ((size_t)r2 * p.hq + h) * D * 2;
      });
    if (E.lse != nullptr && quad == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        if (my_row + 16 * nb < n_rows) E.lse[(size_t)h * E.lse_stride + my_row + 16 * nb] = lse_nat[nb];
    }
  } else {
    // bf16 partials (the normalised split output, like a final output row)
    store_rows<D, 16 * NB>(stg, lane, wrow, n_rows, [&](int r) {
      const size_t prow = (size_t)r * E.n_splits + s;
      return static_cast<unsigned char *>(E.part_o) + (prow * p.hq + h) * D * 2;
    });
    if (quad == 0) {
#pragma unroll
      for (int nb = 0; nb < NB; ++nb)
        if (my_row + 16 * nb < n_rows)
          E.part_lse[((size_t)(my_row + 16 * nb) * E.n_splits + s) * p.hq + h] = lse_nat[nb];
    }
  }
}

// Launch shape: the first pair_wgs workgroups of each XCD each run two jobs,
// slot u and slot 2*pair_wgs-1-u of the XCD's heaviest-first list (a heavy job
// with a light one, so that their sums are nearly equal), and every further
// workgroup runs one of the remaining, lightest slots. With pair_wgs = 0 each
// workgroup runs one slot.
template <int D, int KIND, int NB>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_bf16_kernel(const AttnLaunch p) {
  constexpr int TILE = Geo<D>::TILE;
  // separate objects per stage and tensor: lets the compiler see that the DMA
  // into one buffer does not alias reads of another
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds1[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds1[TILE];
  const int xcd = blockIdx.x % kXcds;
  const int u = blockIdx.x / kXcds;
  const AttnList &l = p.list[0];
  const bool paired = u < l.pair_wgs;
  const int first = paired ? u : u + l.pair_wgs;
  const int second = 2 * l.pair_wgs - 1 - u;
  const int n_jobs = (paired && second < l.slots_per_xcd) ? 2 : 1;
  for (int j = 0; j < n_jobs; ++j) {
    if (j) __syncthreads();  // every wave is done with the LDS buffers of the first job
    attn_job<D, KIND, NB>(p, l, xcd, j ? second : first, k_lds0, v_lds0, k_lds1, v_lds1);
  }
}

// Both stages in one launch, one job per workgroup, each stage's heaviest jobs
// first. QDOC_FIRST: the first workgroups of each XCD run stage 2 and the rest
// stage 1, else the other way round.
template <int D, bool QDOC_FIRST, int NB>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_both_kernel(const AttnLaunch p) {
  constexpr int TILE = Geo<D>::TILE;
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds1[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds1[TILE];
  const int xcd = blockIdx.x % kXcds, u = blockIdx.x / kXcds;
  const int n1 = QDOC_FIRST ? 0 : p.list[0].slots_per_xcd, n2 = QDOC_FIRST ? p.list[1].slots_per_xcd : 0;
  const bool self = QDOC_FIRST ? u >= n2 : u < n1;
  if (self) attn_job<D, 0, NB>(p, p.list[0], xcd, u - n2, k_lds0, v_lds0, k_lds1, v_lds1);
  else attn_job<D, 1, 2>(p, p.list[1], xcd, u - n1, k_lds0, v_lds0, k_lds1, v_lds1);
}

// Rows at given positions where the positions decide the block height: one job
// per workgroup, list[0] (e[0]) in 64-row and list[1] (e[1], the same rows) in
// 128-row blocks; the grid holds the former. The positions ascend, so the middle
// one over the last estimates the chains' mean share of the longest. 28 heads of
// 128, 32768 keys, always 64 rows and now: 1792 rows spread over the keys 481 and
// 491 us, at their end 1039 and 795.
template <int D>
__global__ __launch_bounds__(kAttnThreads, 2) void attn_positions_kernel(const AttnLaunch p) {
  constexpr int TILE = Geo<D>::TILE;
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds0[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char k_lds1[TILE];
  __shared__ __attribute__((aligned(1024))) unsigned char v_lds1[TILE];
  const int xcd = blockIdx.x % kXcds, u = blockIdx.x / kXcds;
  const AttnEntry &E = p.e[0];
  const double share = (double)E.q_pos[E.n_rows / 2] / (E.q_pos[E.n_rows - 1] + 1);
  const bool narrow = narrow_pays(D, (long long)p.list[1].n_groups * p.group, share);
  if (narrow) attn_job<D, 0, 1>(p, p.list[0], xcd, u, k_lds0, v_lds0, k_lds1, v_lds1);
  else if (u < p.list[1].slots_per_xcd) attn_job<D, 0, 2>(p, p.list[1], xcd, u, k_lds0, v_lds0, k_lds1, v_lds1);
}

// Slots per XCD of a list: work groups per XCD times the workgroups of one.
int list_slots(const AttnLaunch &p, const AttnList &l) {
  int per_xcd;
  if (kXcds % p.hkv == 0) {
    const int xph = kXcds / p.hkv, per_head = l.n_groups / p.hkv;
    per_xcd = (per_head + xph - 1) / xph;
  } else {
    per_xcd = (l.n_groups + kXcds - 1) / kXcds;
  }
  return l.wgs_per_group * per_xcd;
}

// The entries of a self-attention list in 64-row blocks.
void narrow_blocks(AttnLaunch &p, AttnList &l) {
  l.n_groups = 0;
  for (int i = l.e0; i < l.e0 + l.n_entries; ++i) {
    AttnEntry &e = p.e[i];
    e.mb_count = (e.n_rows + 63) / 64;
    e.mb_hi = e.mb_count - 1;
    e.group0 = l.n_groups;
    l.n_groups += e.mb_count * p.hkv;
  }
}

// The rule's share of a list (all rows without given positions).
double chain_share(const AttnLaunch &p, const AttnList &l) {
  double work = 0, blocks = 0, longest = 1;
  for (int i = l.e0; i < l.e0 + l.n_entries; ++i) {
    const AttnEntry &e = p.e[i];
    work += e.mb_count * (e.n_keys - 0.5 * e.n_rows);
    blocks += e.mb_count;
    longest = std::max(longest, (double)e.n_keys);
  }
  return blocks > 0 ? work / (blocks * longest) : 0.0;
}

template <int D>
hipError_t launch_positions_t(const AttnLaunch &p0, hipStream_t st) {
  AttnLaunch p = p0;
  p.list[1] = p.list[0];
  p.list[1].e0 = 1;
  p.e[1] = p.e[0];
  narrow_blocks(p, p.list[0]);
  for (AttnList &l : p.list) l.slots_per_xcd = list_slots(p, l);
  attn_positions_kernel<D><<<dim3(kXcds * p.list[0].slots_per_xcd), dim3(kAttnThreads), 0, st>>>(p);
  return hipGetLastError();
}

template <int D>
hipError_t launch_t(AttnKind kind, const AttnLaunch &p0, hipStream_t st) {
  AttnLaunch p = p0;
  AttnList &l = p.list[0];
  // 64-row blocks (16 rows per wave) where the rule says so. Stage 1, n = 512 /
  // 922 / 1500 of 28 heads (112 / 224 / 336 jobs): 14.6 / 21.6 / 33.5 us with 128
  // rows, 10.7 / 17.0 / 27.3 with 64; n = 2000 (448) 43.2 and 42.7, n = 2458 (560)
  // 54.7 and 57.4.
  const long long jobs = (long long)l.n_groups * p.group;
  bool narrow = false;
  if (kind == AttnKind::kSelf) {
    const bool given = p.e[0].q_pos != nullptr;  // one entry
    if (given && jobs > narrow_always(D) && jobs <= narrow_most(D)) return launch_positions_t<D>(p, st);
    narrow = narrow_pays(D, jobs, given ? 1.0 : chain_share(p, l));
  }
  if (narrow) narrow_blocks(p, l);
  const int slots = list_slots(p, l);
  // Causal self attention: the heaviest 2 * kResidentPerXcd slots of an XCD
  // run in heavy/light pairs (see the kernel). Slots are in heaviest-first
  // order within an entry, and entries heaviest request first, so the pairing
  // is used when the first entry alone fills those slots.
  const int xph = kXcds % p.hkv == 0 ? kXcds / p.hkv : 0;
  const int first_groups = xph ? p.e[0].mb_count / xph : p.e[0].mb_count * p.hkv / kXcds;
  l.slots_per_xcd = slots;
  l.pair_wgs = (kind == AttnKind::kSelf && p.e[0].n_splits == 1 &&
                first_groups * l.wgs_per_group >= 2 * kResidentPerXcd)
                   ? kResidentPerXcd
                   : 0;
  const int wgs = l.pair_wgs ? l.pair_wgs + std::max(0, slots - 2 * l.pair_wgs) : slots;
  const dim3 grid(kXcds * wgs), block(kAttnThreads);
  switch (kind) {
    case AttnKind::kSelf:
      if (narrow) attn_bf16_kernel<D, 0, 1><<<grid, block, 0, st>>>(p);
      else attn_bf16_kernel<D, 0, 2><<<grid, block, 0, st>>>(p);
      break;
    default: attn_bf16_kernel<D, 1, 2><<<grid, block, 0, st>>>(p); break;
  }
  return hipGetLastError();
}

template <int D>
hipError_t launch_both_t(const AttnLaunch &p0, hipStream_t st) {
  AttnLaunch p = p0;
  AttnList &l1 = p.list[0], &l2 = p.list[1];
  const bool narrow = narrow_pays(D, (long long)l1.n_groups * p.group, chain_share(p, l1));
  if (narrow) narrow_blocks(p, l1);
  for (AttnList &l : p.list) l.slots_per_xcd = list_slots(p, l);
  // Which stage's jobs go first, from an estimate of the time in key tiles of a
  // 32-row wave (a 16-row wave's takes about 0.6) over the 512 resident
  // workgroups: all the work spread evenly, or stage 1's longest job, which
  // waits for a stage-2 job if those go first and take the slots. Stage 2 first ends with stage
  // 1's lightest blocks, stage 1 first with whole stage-2 jobs (most of one
  // job's time is lost there). Layer, stage 1 / stage 2 first: 16k keys, n =
  // 819, 128 question rows 62.3 / 57.1 us; n = 2458 104.9 / 111.8; 32k, n =
  // 4915 253.9 / 250.7; 6k, n = 922, 64 rows (half the slots) 36.8 / 35.6.
  const double tile1 = narrow ? 0.6 : 1.0;
  const int rows = narrow ? 64 : kAttnBM;
  double work = 0, chain1 = 0, chain2 = 0;
  for (int i = l1.e0; i < l1.e0 + l1.n_entries; ++i) {
    const AttnEntry &e = p.e[i];
    const double tiles = (double)e.n_keys / kBN;
    chain1 = std::max(chain1, tile1 * tiles);
    work += tile1 * p.hq * e.mb_count * 0.5 * (tiles + (double)rows / kBN);
  }
  for (int i = l2.e0; i < l2.e0 + l2.n_entries; ++i) {
    const AttnEntry &e = p.e[i];
    const double tiles = (double)e.split_keys / kBN;
    chain2 = std::max(chain2, tiles);
    work += (double)p.hkv * e.mb_count * e.n_splits * tiles;
  }
  const double even = work / kTargetWorkgroups;
  const double wait = kXcds * l2.slots_per_xcd > kTargetWorkgroups * 3 / 4 ? chain2 : 0.0;
  const bool qdoc_first = std::max(wait + chain1, even) < std::max(chain1, even + 0.75 * chain2);
  const dim3 grid(kXcds * (l1.slots_per_xcd + l2.slots_per_xcd)), block(kAttnThreads);
  if (qdoc_first && narrow) attn_both_kernel<D, true, 1><<<grid, block, 0, st>>>(p);
  else if (qdoc_first) attn_both_kernel<D, true, 2><<<grid, block, 0, st>>>(p);
  else if (narrow) attn_both_kernel<D, false, 1><<<grid, block, 0, st>>>(p);
  else attn_both_kernel<D, false, 2><<<grid, block, 0, st>>>(p);
  return hipGetLastError();
}

// ---- merge of the stage-2 split partials ---------------------------------------
//
// Merge of the bf16 split partials: one wave per (question row, query head).
// Lane = split group * CHN + chunk: each lane accumulates one 8-feature chunk
// over every SG-th split (online log-sum-exp), then the split groups combine
// across lanes.
template <int D>
__global__ __launch_bounds__(256) void qdoc_merge_kernel(const MergeLaunch p) {
  constexpr int CHN = D / 8, SG = 64 / CHN;
  const int item = blockIdx.x * 4 + (threadIdx.x >> 6);
  const int lane = threadIdx.x & 63, c = lane % CHN, sg = lane / CHN;
  const int row = item / p.hq, h = item % p.hq;
  if (row >= p.total_rows) return;  // whole waves leave together
  int ei = 0;
  while (ei + 1 < p.n_entries && p.e[ei + 1].row0 <= row) ++ei;
  const MergeEntry &E = p.e[ei];
  const int r = row - E.row0;
  const int S = E.n_splits;
  const size_t prow0 = (size_t)r * S;
  const float *lse = E.part_lse + prow0 * p.hq + h;
  const __bf16 *src = static_cast<const __bf16 *>(E.part_o) + (prow0 * p.hq + h) * D + 8 * c;
  const size_t sstride = (size_t)p.hq * D;
  constexpr int U = 8;
  float acc[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
  float m = -INFINITY, wsum = 0.f;
  for (int s0 = sg; s0 < S; s0 += SG * U) {
    float ls[U];
    bf16x8 po[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int sx = s0 + u * SG;
      if (sx < S) {
        ls[u] = lse[(size_t)sx * p.hq];
        po[u] = *reinterpret_cast<const bf16x8 *>(src + sx * sstride);
      } else {
        ls[u] = -INFINITY;
        po[u] = bf16x8{};
      }
    }
    float mc = m;
#pragma unroll
    for (int u = 0; u < U; ++u) mc = fmaxf(mc, ls[u]);
    const float a = (m == -INFINITY) ? 0.f : __expf(m - mc);
    wsum *= a;
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] *= a;
    m = mc;
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const float wt = (ls[u] == -INFINITY) ? 0.f : __expf(ls[u] - m);
      wsum += wt;
#pragma unroll
      for (int k = 0; k < 8; ++k) acc[k] += wt * (float)po[u][k];
    }
  }
  // combine the SG split groups (lanes c, c + CHN, c + 2 CHN, ...)
#pragma unroll
  for (int off = CHN; off < 64; off *= 2) {
    const float m2 = __shfl_xor(m, off, 64), w2 = __shfl_xor(wsum, off, 64);
    const float mm = fmaxf(m, m2);
    const float a = (m == -INFINITY) ? 0.f : __expf(m - mm);
    const float b = (m2 == -INFINITY) ? 0.f : __expf(m2 - mm);
#pragma unroll
    for (int k = 0; k < 8; ++k) acc[k] = acc[k] * a + __shfl_xor(acc[k], off, 64) * b;
    wsum = wsum * a + w2 * b;
    m = mm;
  }
  if (sg != 0) return;
  const float inv = wsum > 0.f ? 1.f / wsum : 0.f;
  bf16x8 out;
#pragma unroll
  for (int k = 0; k < 8; ++k) out[k] = (__bf16)(acc[k] * inv);
  *reinterpret_cast<bf16x8 *>(static_cast<__bf16 *>(E.o) + ((size_t)r * p.hq + h) * D + 8 * c) = out;
  if (E.o2 != nullptr)
    *reinterpret_cast<bf16x8 *>(static_cast<__bf16 *>(E.o2) + ((size_t)(E.o2_row0 + r) * p.hq + h) * D + 8 * c) = out;
  if (E.lse != nullptr && c == 0) E.lse[(size_t)h * E.lse_stride + r] = wsum > 0.f ? m + __logf(wsum) : -INFINITY;
}

template <int D>
hipError_t launch_qdoc_merge_t(const MergeLaunch &p, hipStream_t st) {
  const int64_t items = (int64_t)p.total_rows * p.hq;
  qdoc_merge_kernel<D><<<dim3((unsigned)((items + 3) / 4)), dim3(256), 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace

hipError_t launch_attention_bf16(int head_dim, AttnKind kind, const AttnLaunch &p, hipStream_t st) {
  if (p.list[0].n_groups <= 0) return hipSuccess;
  return head_dim == 128 ? launch_t<128>(kind, p, st) : launch_t<64>(kind, p, st);
}

hipError_t launch_attention_both_bf16(int head_dim, const AttnLaunch &p, hipStream_t st) {
  return head_dim == 128 ? launch_both_t<128>(p, st) : launch_both_t<64>(p, st);
}

hipError_t launch_qdoc_merge_bf16(int head_dim, const MergeLaunch &p, hipStream_t st) {
  if (p.total_rows <= 0) return hipSuccess;
  return head_dim == 128 ? launch_qdoc_merge_t<128>(p, st) : launch_qdoc_merge_t<64>(p, st);
}

}  // namespace daf
