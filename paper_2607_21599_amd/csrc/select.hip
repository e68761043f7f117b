// Important-token selection (Sec. 2 item 1): tokens are chosen by the
// deviation of their freshly computed keys from the offline cached keys,
// aggregated over several early layers (typically the 2nd to the 4th). Score of
// a document token = mean over the selection layers of the L2 norm of
// (k_fresh - k_cached) over all its KV heads and features; request b keeps its
// n_b highest-scoring tokens (equal scores: lower index first), listed in
// ascending original order, which is the idx every other entry point takes.
//
// select_score_kernel: one wave per document row, HBM-bound (2 * layers * row
// bytes read per row); every lane loads 16-byte pieces of the row for all
// layers before reducing, fp32 sums of squares, a wave reduction per layer.
//
// select_topn_kernel: one 1024-thread workgroup per request, its keys held in
// LDS (slab by slab beyond 32k tokens), copied there without passing through
// registers. Scores are non-negative floats, so their bit patterns order like
// the values: a radix select finds the key T of the n-th highest score and how
// many tokens scoring exactly T to keep, 8 bits per pass of the keys' distance
// from the lowest one (so the first histogram spreads over the scores' actual
// range), stopping early once a digit's keys are all taken. The histogram is
// kept in 16 copies, one per lane modulo 16 (rows padded to 257 words so that
// one digit's copies sit in different banks): scores cluster, and with a single
// copy the lanes of one instruction that share a digit serialise on its word.
// Each wave owns a contiguous range of tokens; a prefix sum over the waves of
// their kept counts, then ballots within each wave, place every kept index, so
// the output comes out sorted.
//   One CU does a request's work and runs each part of the code once or a few
// times, so it is bound by latencies: of memory (a request's 128 KiB take about
// 4 us to reach the CU), of the LDS behind each key, and of the instructions
// themselves, which is why the loops are rolled. Score and top-n together, us back
// to back, 3 layers of 512 values per token, with the keys in registers and
// straight code before: 1024 tokens 20.0, now 12.7; 8192 27.4 and 19.0; 32768 49.7
// and 47.3; 33000 61.8 and 58.7 (70.8 with uneven slabs, each reloaded by every
// pass); 131072 216 and 206, of one layer 111 and 110 (115). Ranking the last 512
// keys against each other instead of the last passes cost 4 us more at 32768.
#include "daf_internal.h"

namespace daf {
namespace {

typedef unsigned int u32x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

constexpr int kScoreThreads = 256;
constexpr int kTopnThreads = 1024;
constexpr int kTopnWaves = kTopnThreads / 64;
constexpr int kChunk = 8;  // keys per lane read from LDS ahead of their use
constexpr int kHistCopies = 16, kHistStride = 257;

__device__ __forceinline__ float wave_sum(float x) {
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) x += __shfl_xor(x, off, 64);
  return x;
}

// Sum of squared differences of the 16-byte pieces a and b (8 bf16 or 4 fp32).
template <bool BF16>
__device__ __forceinline__ float sq_diff(u32x4 a, u32x4 b) {
  float s = 0.f;
  if (BF16) {
    const bf16x8 x = __builtin_bit_cast(bf16x8, a), y = __builtin_bit_cast(bf16x8, b);
#pragma unroll
    for (int i = 0; i < 8; ++i) {
      const float d = (float)x[i] - (float)y[i];
      s = __builtin_fmaf(d, d, s);
    }
  } else {
    // whole-vector casts: a bit cast of a vector element expression reads the
    // vector's first element
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const float d = x[i] - y[i];
      s = __builtin_fmaf(d, d, s);
    }
  }
  return s;
}

// CPL = 16-byte pieces per lane (row bytes / 1024, rounded up).
template <bool BF16, int CPL>
__global__ __launch_bounds__(kScoreThreads) void select_score_kernel(const SelectLaunch p) {
  const int lane = threadIdx.x & 63;
  const int64_t row = (int64_t)blockIdx.x * (kScoreThreads / 64) + (threadIdx.x >> 6);
  if (row >= p.rows) return;
  const int pieces = p.row_bytes / 16;
  float acc = 0.f;
  for (int l0 = 0; l0 < p.n_layers; l0 += 2) {
    // two layers' loads in flight before their reductions
    u32x4 f[2][CPL], c[2][CPL];
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      const int l = l0 + j;
#pragma unroll
      for (int k = 0; k < CPL; ++k) {
        const int pc = lane + 64 * k;
        f[j][k] = c[j][k] = u32x4{0u, 0u, 0u, 0u};
        if (l < p.n_layers && pc < pieces) {
          const size_t off = (size_t)row * p.row_bytes + (size_t)pc * 16;
          f[j][k] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.fresh[l]) + off);
          c[j][k] = *reinterpret_cast<const u32x4 *>(static_cast<const char *>(p.cached[l]) + off);
        }
      }
    }
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      float s = 0.f;
#pragma unroll
      for (int k = 0; k < CPL; ++k) s += sq_diff<BF16>(f[j][k], c[j][k]);
      s = wave_sum(s);
      if (l0 + j < p.n_layers) acc += sqrtf(s);
    }
  }
  if (lane == 0) p.scores[row] = acc / (float)p.n_layers;
}

// Most keys in LDS at a time (128 KiB); a longer request is reloaded per pass.
constexpr int kSlabKeys = kTopnThreads * 32;

// Exclusive prefix sum over the waves of a wave-uniform value, in wave order;
// also returns the sum over all waves. Unsigned: packed counts reach 2^31. wsum:
// kTopnWaves words of LDS.
__device__ __forceinline__ unsigned wave_scan(unsigned v, unsigned *wsum, unsigned &total) {
  const int wave = threadIdx.x >> 6;
  if ((threadIdx.x & 63) == 0) wsum[wave] = v;
  __syncthreads();
  unsigned before = 0;
  total = 0;
#pragma unroll
  for (int w = 0; w < kTopnWaves; ++w) {
    const unsigned t = wsum[w];
    before += w < wave ? t : 0u;
    total += t;
  }
  __syncthreads();  // wsum is reused by the next call
  return before;
}

// Exclusive prefix sum of v over the threads in thread order.
__device__ __forceinline__ int block_scan(int v, unsigned *wsum) {
  const int lane = threadIdx.x & 63;
  int inc = v;
#pragma unroll
  for (int off = 1; off < 64; off <<= 1) {
    const int t = __shfl_up(inc, off, 64);
    if (lane >= off) inc += t;
  }
  unsigned total;
  return (int)wave_scan((unsigned)__shfl(inc, 63, 64), wsum, total) + inc - v;
}

// Number of set bits of m below this lane.
__device__ __forceinline__ unsigned lanes_below(unsigned long long m) {
  return __builtin_amdgcn_mbcnt_hi((unsigned)(m >> 32), __builtin_amdgcn_mbcnt_lo((unsigned)m, 0u));
}

__device__ __forceinline__ unsigned long long ballot(bool x) { return __builtin_amdgcn_ballot_w64(x); }

__device__ __forceinline__ int uniform(int x) { return __builtin_amdgcn_readfirstlane(x); }

__global__ __launch_bounds__(kTopnThreads) void select_topn_kernel(const SelectLaunch p) {
  __shared__ unsigned s_key[kSlabKeys + (kChunk - 1) * 64];
  __shared__ int hist[kHistCopies * kHistStride];
  __shared__ unsigned wsum[kTopnWaves];
  __shared__ unsigned s_lo[kTopnWaves], s_hi[kTopnWaves], s_base;
  __shared__ int s_remaining, s_top;
  const int b = blockIdx.x;
  const int L = p.req[b].L_d, n = p.req[b].n;
  if (n <= 0 || L <= 0) return;
  const unsigned *key = reinterpret_cast<const unsigned *>(p.scores + p.req[b].doc0);
  int32_t *out = p.idx + p.req[b].imp0;
  const int lane = threadIdx.x & 63, wave = uniform((int)(threadIdx.x >> 6));

  // slabs of equal size (33000 keys as 32768 + 232 took every pass the work of
  // 65536), dealt to the waves in ranges of `steps` * 64, the same in every slab: a
  // wave copies and reads its own range only, so the passes need no barrier around
  // a slab. Passes go over the slabs in turns up and down, so that a pass begins
  // with the slab that the one before ended with.
  const int most = (L - 1) / kSlabKeys + 1, steps = ((L - 1) / most + kTopnThreads) / kTopnThreads;
  const int slab = steps * kTopnThreads, n_slabs = (L - 1) / slab + 1, own = wave * steps * 64;
  int loaded = -1, slab0 = 0, len = 0;  // the loaded slab, its first key and its keys
  auto load = [&](int s) {
    if (s == loaded) return;
    loaded = s;
    slab0 = s * slab;
    len = min(L - slab0, slab);
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");  // every read of the slab before is done
    for (int j = 0; j < steps; ++j) {
      // lanes past the last key copy it again; every use below tests the index
      const unsigned *from = key + slab0 + min(own + j * 64 + lane, len - 1);
      __builtin_amdgcn_global_load_lds((const __attribute__((address_space(1))) void *)from,
                                       (__attribute__((address_space(3))) void *)&s_key[own + j * 64], 4, 0, 0);
    }
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
  };
  bool down = false;
  auto slabs = [&](auto f) {
    for (int t = 0; t < n_slabs; ++t) {
      load(down ? n_slabs - 1 - t : t);
      f();
    }
    down = !down;
  };
  // f(key, its index in the wave's range, whether it is a token), in order. The
  // reads of a chunk are issued together: behind f's LDS atomics and stores each
  // would wait for the one before. Rolled over chunks: every pass runs once or
  // a few times, and straight code would wait for its own instructions.
  auto each = [&](auto f) {
    const int end = min(steps * 64, len - own);
    for (int j = 0; j < steps; j += kChunk) {
      unsigned k[kChunk];
#pragma unroll
      for (int e = 0; e < kChunk; ++e) k[e] = s_key[own + (j + e) * 64 + lane];
#pragma unroll
      for (int e = 0; e < kChunk; ++e) f(k[e], (j + e) * 64 + lane, (j + e) * 64 + lane < end);
    }
  };

  // ---- the keys' range -------------------------------------------------------
  for (int i = threadIdx.x; i < kHistCopies * kHistStride; i += kTopnThreads) hist[i] = 0;
  unsigned lo = 0xffffffffu, hi = 0u;
  slabs([&] {
    each([&](unsigned k, int, bool token) {
      lo = min(lo, token ? k : 0xffffffffu);
      hi = max(hi, token ? k : 0u);
    });
  });
#pragma unroll
  for (int off = 32; off > 0; off >>= 1) {
    lo = min(lo, (unsigned)__shfl_xor((int)lo, off, 64));
    hi = max(hi, (unsigned)__shfl_xor((int)hi, off, 64));
  }
  if (lane == 0) {
    s_lo[wave] = lo;
    s_hi[wave] = hi;
  }
  __syncthreads();
#pragma unroll
  for (int w = 0; w < kTopnWaves; ++w) {
    lo = min(lo, s_lo[w]);
    hi = max(hi, s_hi[w]);
  }
  // the keys that may hold T: base + [0, 2^top); `remaining` of them are to be
  // taken, and every key above them
  unsigned base = (unsigned)uniform((int)lo);
  const unsigned range = (unsigned)uniform((int)hi) - base;
  int top = range == 0u ? 0 : 32 - __builtin_clz(range);
  int remaining = n;

  // ---- radix select of the n-th highest key, 8 bits per pass -------------------
  while (top > 0) {
    const int w = min(8, top), shift = top - w;
    const unsigned last = ~0u >> (32 - top);
    int *mine = &hist[(lane & (kHistCopies - 1)) * kHistStride];
    slabs([&] {
      each([&](unsigned k, int, bool token) {
        const unsigned r = k - base;
        if (token & (r <= last)) atomicAdd(&mine[r >> shift], 1);
      });
    });
    __syncthreads();
    // digits from the highest down: the selected one holds the remaining-th key
    if (threadIdx.x == 0) s_top = 0;  // every pass ends the loop unless a digit is chosen
    const int d = (1 << w) - 1 - (int)threadIdx.x;
    int h = 0;
    if (d >= 0) {
#pragma unroll
      for (int c = 0; c < kHistCopies; ++c) {
        h += hist[c * kHistStride + d];
        hist[c * kHistStride + d] = 0;  // cleared for the next pass
      }
    }
    const int above = block_scan(h, wsum);
    if (d >= 0 && above < remaining && above + h >= remaining) {
      s_base = base + ((unsigned)d << shift);
      // every key in the digit is taken: no lower bits need deciding
      s_top = above + h == remaining ? 0 : shift;
      s_remaining = above + h == remaining ? 0x7fffffff : remaining - above;
    }
    __syncthreads();
    base = (unsigned)uniform((int)s_base);
    top = uniform(s_top);
    remaining = uniform(s_remaining);
  }
  const unsigned T = base;  // keep keys above T and the first `remaining` equal to T

  // ---- ordered compaction, slab by slab ----------------------------------------
  int out_base = 0;  // kept keys of earlier slabs
  for (int s = 0; s < n_slabs; ++s) {
    load(s);
    int n_gt = 0, n_eq = 0;
    each([&](unsigned k, int, bool token) {
      n_gt += __popcll(ballot(token) & ballot(k > T));
      n_eq += __popcll(ballot(token) & ballot(k == T));
    });
    // both counts of a slab are at most 2^15: one scan takes them side by side
    unsigned totals;
    const unsigned before = wave_scan((unsigned)n_gt << 16 | (unsigned)n_eq, wsum, totals);
    const int eq_before = uniform((int)(before & 0xffffu));
    const int eq_keep = max(0, min(n_eq, remaining - eq_before));
    int pos = out_base + uniform((int)(before >> 16)) + min(eq_before, remaining);
    // (a scalar base and a 32-bit lane offset for the stores)
    if (eq_keep == 0 || (eq_keep == n_eq && T > 0u)) {
      // none or all of the wave's keys equal to T (the usual case): one comparison
      const unsigned below = eq_keep == 0 ? T : T - 1u;
      each([&](unsigned k, int i, bool token) {
        const bool keep = token & (k > below);
        const unsigned long long km = ballot(token) & ballot(k > below);
        char *to = reinterpret_cast<char *>(out + pos);
        if (keep) *reinterpret_cast<int32_t *>(to + lanes_below(km) * 4u) = slab0 + own + i;
        pos += __popcll(km);
      });
    } else {
      int eq_left = eq_keep;  // keys equal to T still to take
      each([&](unsigned k, int i, bool token) {
        const unsigned long long eq = ballot(token) & ballot(k == T);
        const bool keep = token & ((k > T) | ((k == T) & ((int)lanes_below(eq) < eq_left)));
        eq_left -= min(eq_left, (int)__popcll(eq));
        const unsigned long long km = ballot(keep);
        char *to = reinterpret_cast<char *>(out + pos);
        if (keep) *reinterpret_cast<int32_t *>(to + lanes_below(km) * 4u) = slab0 + own + i;
        pos += __popcll(km);
      });
    }
    const int eq_total = uniform((int)(totals & 0xffffu));
    out_base += uniform((int)(totals >> 16)) + min(eq_total, remaining);
    remaining -= min(eq_total, remaining);
  }
}

}  // namespace

hipError_t launch_select_scores(const SelectLaunch &p, bool bf16, hipStream_t st) {
  if (p.rows <= 0) return hipSuccess;
  const int64_t blocks = (p.rows + kScoreThreads / 64 - 1) / (kScoreThreads / 64);
  const int cpl = (p.row_bytes / 16 + 63) / 64;  // row_bytes <= 4096: at most 4
  auto go = [&](auto kern) { kern<<<(unsigned)blocks, kScoreThreads, 0, st>>>(p); };
  if (bf16) {
    if (cpl <= 1) go(select_score_kernel<true, 1>);
    else if (cpl <= 2) go(select_score_kernel<true, 2>);
    else go(select_score_kernel<true, 4>);
  } else {
    if (cpl <= 1) go(select_score_kernel<false, 1>);
    else if (cpl <= 2) go(select_score_kernel<false, 2>);
    else go(select_score_kernel<false, 4>);
  }
  return hipGetLastError();
}

hipError_t launch_select_topn(const SelectLaunch &p, hipStream_t st) {
  if (p.n_req <= 0) return hipSuccess;
  select_topn_kernel<<<p.n_req, kTopnThreads, 0, st>>>(p);
  return hipGetLastError();
}

}  // namespace daf
