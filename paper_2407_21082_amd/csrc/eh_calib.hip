// Threshold calibration on the device (arXiv 2407.21082, Section 3.4.1,
// "Calibration of Confidence Thresholds"), entropy as the confidence metric.
//
// For one head and a level epsilon the threshold is the largest entropy v among
// the M calibration tokens such that, of the C(v) tokens with entropy <= v (all
// tokens at least as confident), the R(v) whose prediction equals the model's
// (eq. (2)) make up a proportion R(v)/C(v) >= epsilon.  Tokens of equal entropy are
// taken as a whole (v runs over the distinct entropies), NaN entropies are no
// candidates and are counted nowhere, and "no v qualifies" gives tau = -inf.
//
// R/C is not monotone in v, so there is nothing to bisect; but only the largest
// qualifying v is wanted, and whole ranges of v can be ruled out from counts alone.
// The entropies become order-preserving 32-bit keys, which are cut three times: into 8192
// bins over the range of a sample of the tokens and 8192 more outside it, each of those into
// up to 2048, each of those into up to 512 single keys.  A bin whose tokens number cnt, cor of
// them correct, on top of C0 tokens and R0 correct ones below it, holds
//   - a top candidate (its largest key) with exactly C = C0 + cnt, R = R0 + cor, and
//   - inner candidates whose proportion is at most (R0 + cor) / (C0 + cor)
//     (R0 / (C0 + 1) if cor = 0): the correct tokens first, no wrong one.
// Walking down from the largest keys, a level keeps, for each epsilon, the bins whose
// bound reaches epsilon until the first bin whose top candidate qualifies, that one
// included; everything below it is smaller than a key that qualifies and everything
// else above it cannot qualify.  The next level counts only the tokens of kept bins.
// At the last level the bins are single keys and the first one that qualifies is the
// answer.  All quotients are the correctly rounded double divisions of the section's
// proportion; rounding is monotone, so the bound survives it.
//
// Passes over the tokens: one that reads entropy, prediction and reference (12 bytes),
// packs the correctness bits and counts, one that reads the entropies again (4 bytes) and
// sets the tokens of kept bins aside, and one over the tokens set aside.  2^24 tokens, 11 levels: 141 us
// with a pass of its own for the key range, 111 now; 2^20 96 and 81, 5000 80 and 69 (eight short
// dependent launches and the wait of the host).  The tables are small: 128 kept bins of the first level and 1024 of the second,
// over all epsilon together.  Data that keeps more (a
// proportion that hovers at epsilon over a wide range of thresholds) sets a flag that
// the host reads back, and the call is then served by the full sort below it: rocPRIM's
// radix sort of (key, correctness) pairs, a running sum, and a search of every position.
#include <algorithm>
#include <cstdlib>
#include <cstring>
#include <type_traits>

#include <rocprim/device/device_radix_sort.hpp>
#include <rocprim/device/device_scan.hpp>
#include <rocprim/functional.hpp>

#include "eh_internal.hpp"
#include "eh_kernels.hpp"

namespace eh {

namespace {

constexpr int kMaxEps = 64;
struct EpsList {
  double v[kMaxEps];
  int n;
};

// Order-preserving map of a float to an unsigned key, inverted so that ascending
// keys are descending entropies; NaN -> 0 (sorts first; no finite or infinite
// value maps to 0).
__device__ __forceinline__ uint32_t entropy_key(float h) {
  if (h != h) return 0u;
  if (h == 0.f) h = 0.f;  // -0 and +0 are one value
  const uint32_t u = __float_as_uint(h);
  const uint32_t asc = u ^ ((u >> 31) ? 0xFFFFFFFFu : 0x80000000u);
  return ~asc;
}
__device__ __forceinline__ float key_entropy(uint32_t key) {
  const uint32_t asc = ~key;
  return __uint_as_float(asc ^ ((asc >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

__global__ __launch_bounds__(256) void calib_keys_kernel(const float* __restrict__ H,
                                                         const int* __restrict__ pred,
                                                         const int* __restrict__ ref, int64_t M,
                                                         uint32_t* __restrict__ keys,
                                                         uint32_t* __restrict__ vals) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i >= M) return;
  keys[i] = entropy_key(H[i]);
  vals[i] = pred[i] == ref[i] ? 1u : 0u;
}

__global__ void calib_init_kernel(unsigned* __restrict__ best, int n, unsigned M) {
  if ((int)threadIdx.x < n) best[threadIdx.x] = M;
}

// keys ascending, prefix = inclusive running count of correct tokens in that order.
// Workgroups of 1024 positions.  Only a position before the best one found so far can
// improve it, and positions are visited roughly in ascending order: the workgroup reads
// the current bests once (possibly stale, which only costs a redundant atomic) and skips
// every level that is already settled before its first position.
__global__ __launch_bounds__(1024) void calib_search_kernel(const uint32_t* __restrict__ keys,
                                                            const uint32_t* __restrict__ prefix, int64_t M,
                                                            EpsList eps, unsigned* __restrict__ best) {
  __shared__ unsigned cur[kMaxEps];
  __shared__ unsigned wg_min[kMaxEps];
  if ((int)threadIdx.x < eps.n) {
    cur[threadIdx.x] = __builtin_nontemporal_load(&best[threadIdx.x]);
    wg_min[threadIdx.x] = 0xFFFFFFFFu;
  }
  __syncthreads();
  const int64_t j = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const unsigned wg_first = (unsigned)((int64_t)blockIdx.x * blockDim.x);
  const int lane = threadIdx.x & 63;
  bool cand = false;
  // proportion of correct predictions among the tokens at least as confident as this one:
  // the section's quotient as a correctly rounded double (IEEE division), compared with the
  // levels as it stands, so that exactly p of q tokens meet a level written as the decimal p/q
  double prop = 0.0;
  if (j < M) {
    const uint32_t k = keys[j];
    cand = k != 0u && (j == 0 || keys[j - 1] != k);
    if (cand) {
      const uint32_t total = prefix[M - 1];
      prop = (double)(total - (j ? prefix[j - 1] : 0u)) / (double)(M - j);
    }
  }
  bool any = false;
  for (int e = 0; e < eps.n; ++e) {
    if (cur[e] <= wg_first) continue;  // uniform over the workgroup
    any = true;
    // lanes hold ascending positions: the first lane that qualifies is the wave's minimum
    const unsigned long long q = __ballot(cand && prop >= eps.v[e]);
    if (lane == 0 && q) atomicMin(&wg_min[e], (unsigned)(j + __builtin_ctzll(q)));
  }
  if (!any) return;  // uniform
  __syncthreads();
  if ((int)threadIdx.x < eps.n && wg_min[threadIdx.x] != 0xFFFFFFFFu) atomicMin(&best[threadIdx.x], wg_min[threadIdx.x]);
}

__global__ void calib_read_kernel(const uint32_t* __restrict__ keys, const unsigned* __restrict__ best, int n,
                                  unsigned M, float* __restrict__ tau, long long* __restrict__ n_exit) {
  const int e = threadIdx.x;
  if (e >= n) return;
  const unsigned b = best[e];
  tau[e] = b < M ? key_entropy(keys[b]) : -INFINITY;
  if (n_exit) n_exit[e] = b < M ? (long long)(M - b) : 0;
}


// ---------------------------------------------------------------------------------
// The refinement: three levels of counts instead of a sort.

constexpr int kInner = 8192;       // bins of level 1 over the key range of a sample of the tokens
constexpr int kOuterBits = 20;     // keys outside that range: bins of 2^20 keys
constexpr int kOuter = 1 << (32 - kOuterBits);  // of which there are this many on either side
constexpr int kBins1 = kInner + 2 * kOuter;     // ascending: below the sample's range, inside, above
constexpr int kBins2 = 2048;       // bins of one kept level-1 bin
constexpr int kBins3 = 512;        // single keys of one kept level-2 bin
constexpr int kSampleWgs = 64;     // workgroups that look at kSample tokens for their key range
constexpr int kSample = 65536;
constexpr int kCap1 = 128;         // kept bins of level 1, all epsilon together
constexpr int kCap2 = 1024;        // kept bins of level 2
constexpr int kSegment = 32768;    // tokens behind one row of level-1 partial counts (16-bit counters)
constexpr int64_t kRefineMax = (int64_t)1 << 27;  // larger sets go to the sort (4096 partial rows)

// Ascending key of an entropy (that of the sort above, not inverted): -0 and +0 have one, NaNs lie
// above all others or below them.
__device__ __forceinline__ uint32_t ascending_key(float h) {
  const uint32_t u = __float_as_uint(h + 0.f);
  return u ^ ((uint32_t)((int32_t)u >> 31) | 0x80000000u);
}
__device__ __forceinline__ float ascending_entropy(uint32_t asc) {
  return __uint_as_float(asc ^ ((asc >> 31) ? 0x80000000u : 0xFFFFFFFFu));
}

// Device memory of one call.  Counts are pairs in one 64-bit word: tokens in the low half,
// correct tokens in the high half.
struct CalibWork {
  uint64_t* bits;     // [ceil(M / 256)][4] correctness of token 256 b + 4 i + j in bit i of word [b][j]
  uint32_t* part1;    // [ceil(M / kSegment)][kInner] level-1 counts of a segment, 16 + 16 bits
  uint32_t* kept;     // [M] tokens of kept level-1 bins: correct << 31 | row << 20 | key inside the bin; a
                      // wave's share of a segment has its own part
  int* n_aside;       // [waves] tokens in each part
  uint2* range;       // [kSampleWgs] smallest and largest key of a share of the sample
  int* host_flag;     // host memory: 0 if a table has proved too small
  // preset to 0
  int* n_kept;        // [2] kept bins of level 1, of level 2
  uint64_t* h1;       // [kBins1]
  uint64_t* sel1;     // [kBins1] which epsilon keep the bin
  uint64_t* h2;       // [kCap1][kBins2]
  uint64_t* sel2;     // [kCap1][kBins2]
  uint64_t* h3;       // [kCap2][kBins3]
  // preset to -1
  int* overflow;      // [1] -1, or 0 once a table has proved too small
  int* row_b3;        // [kCap1] Cut::b3 of a row's level-1 bin
  signed char* slot1; // [kBins1] row of a kept bin in h2
  int* slot2;         // [kCap1][kBins2] row of a kept bin in h3
};

// Inclusive prefix sums over the lanes of a wave (of each row of 16 lanes), by cross-lane moves of the vector
// unit (through LDS, as __shfl_up goes, a trip of 60 clocks a step).
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t from_lane(uint32_t v) {
  return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, CTRL, ROWS, 0xf, false);
}
__device__ __forceinline__ uint32_t row_inclusive(uint32_t v) {
  v += from_lane<0x111, 0xf>(v);  // row_shr:1, 2, 4, 8
  v += from_lane<0x112, 0xf>(v);
  v += from_lane<0x114, 0xf>(v);
  v += from_lane<0x118, 0xf>(v);
  return v;
}
__device__ __forceinline__ uint32_t wave_inclusive(uint32_t v) {
  v = row_inclusive(v);
  v += from_lane<0x142, 0xa>(v);  // lane 15 of a row to the next (rows 1 and 3)
  v += from_lane<0x143, 0xc>(v);  // lane 31 to rows 2 and 3
  return v;
}
// The largest value of the wave.
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t max_from_lane(uint32_t v) {
  return max(v, (uint32_t)__builtin_amdgcn_update_dpp((int)v, (int)v, CTRL, ROWS, 0xf, false));
}
__device__ __forceinline__ uint32_t wave_max(uint32_t v) {
  v = max_from_lane<0x111, 0xf>(v);
  v = max_from_lane<0x112, 0xf>(v);
  v = max_from_lane<0x114, 0xf>(v);
  v = max_from_lane<0x118, 0xf>(v);
  v = max_from_lane<0x142, 0xa>(v);
  v = max_from_lane<0x143, 0xc>(v);
  return (uint32_t)__builtin_amdgcn_readlane((int)v, 63);
}

// How the keys are cut.  The range [lo, hi] of the sample has kInner bins of level 1, which take the
// bits above s of a key's distance from lo; the few keys outside it go to the bins of 2^20 keys
// below and above.  Level 2 takes a bin's next (at most 11) bits, level 3 the rest (at most 9).
// The range of all tokens would leave nothing outside, but is known only after a pass over all
// entropies, which then had to be read once more to be counted (17 us of 141 for 2^24).
struct Cut {
  uint32_t lo, hi;
  int s;
  // the short way to an inner bin: the bits of an entropy less lo_bits, if that is below n_plain, are its
  // key's distance from lo (everything else, -0 and NaN too, takes the long way)
  uint32_t lo_bits, n_plain;
  __device__ __forceinline__ int bin(uint32_t key) const {
    return key < lo ? (int)(key >> kOuterBits)
                    : key > hi ? kOuter + kInner + (int)(key >> kOuterBits) : kOuter + (int)((key - lo) >> s);
  }
  __device__ __forceinline__ uint32_t within(uint32_t key) const {  // a key's place inside its bin
    return key < lo || key > hi ? key & ((1u << kOuterBits) - 1u) : (key - lo) & ((1u << s) - 1u);
  }
  __device__ __forceinline__ bool inner(int bin) const { return bin >= kOuter && bin < kOuter + kInner; }
  __device__ __forceinline__ uint32_t start(int bin) const {  // the smallest key of a bin
    return inner(bin) ? lo + ((uint32_t)(bin - kOuter) << s)
                      : (uint32_t)(bin < kOuter ? bin : bin - kOuter - kInner) << kOuterBits;
  }
  __device__ __forceinline__ int bits(int bin) const { return inner(bin) ? s : kOuterBits; }
  __device__ __forceinline__ int b2(int bin) const { return min(bits(bin), 11); }
  __device__ __forceinline__ int b3(int bin) const { return bits(bin) - b2(bin); }
};
// Every lane of the wave must call.
__device__ __forceinline__ Cut cut_of(const CalibWork& w) {
  static_assert(kSampleWgs == 64, "a share per lane");
  const uint2 r = w.range[threadIdx.x & 63];
  Cut c;
  c.lo = ~wave_max(~r.x);
  c.hi = wave_max(r.y);
  if (c.lo > c.hi) c.lo = c.hi = 0;  // no token of the sample has an entropy: all keys are above the range
  const uint32_t span = c.hi - c.lo;
  c.s = 0;
  while ((span >> c.s) >= (uint32_t)kInner) ++c.s;  // at most 19
  const bool plain = c.lo >= 0x80000000u;  // no negative entropy in the range: keys and bits of a float differ by a constant
  c.lo_bits = c.lo ^ 0x80000000u;
  c.n_plain = plain ? span + 1u : 0u;
  return c;
}

struct Pair {
  uint32_t c, r;
};
__device__ __forceinline__ Pair operator+(Pair a, Pair b) { return Pair{a.c + b.c, a.r + b.r}; }
__device__ __forceinline__ Pair pair_of(uint64_t v) { return Pair{(uint32_t)v, (uint32_t)(v >> 32)}; }

// proportion r / c >= eps, by the correctly rounded quotient (c > 0).  The difference r - eps c in 32 bits
// is off by less than 4e-7 c; only where that leaves the answer open is the division worked out.
__device__ __forceinline__ bool reaches(uint32_t r, uint32_t c, double eps, float eps32) {
  const float fc = (float)c;
  const float diff = __builtin_fmaf(-eps32, fc, (float)r);
  bool yes = diff > 0.f;
  if (fabsf(diff) <= 1e-6f * fc) yes = (double)r / (double)c >= eps;
  return yes;
}

// A workgroup barrier that orders LDS traffic only: loads, and counts sent to memory by atomics that
// return nothing, are not waited for.
__device__ __forceinline__ void lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

constexpr int kWalkWaves = 16;  // waves of the workgroups that walk a table

__device__ __forceinline__ Pair wave_inclusive(Pair v) { return Pair{wave_inclusive(v.c), wave_inclusive(v.r)}; }

// Exclusive prefix of one Pair per thread over a workgroup of kWalkWaves waves; *total_c
// receives the sum of the first members.  sh: kWalkWaves entries that no call before has used.
__device__ __forceinline__ Pair block_exclusive(Pair v, Pair* sh, int* total_c = nullptr) {
  static_assert(kWalkWaves == 16, "a row of lanes");
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const Pair inc = wave_inclusive(v);
  if (lane == 63) sh[wave] = inc;
  lds_barrier();
  const Pair own = sh[lane & 15];
  const uint32_t c = row_inclusive(own.c), r = row_inclusive(own.r);
  if (total_c) *total_c = __builtin_amdgcn_readlane((int)c, 15);
  Pair off{0, 0};
  if (wave > 0) off = Pair{(uint32_t)__builtin_amdgcn_readlane((int)c, wave - 1), (uint32_t)__builtin_amdgcn_readlane((int)r, wave - 1)};
  return Pair{off.c + inc.c - v.c, off.r + inc.r - v.r};
}
// The last lane's value of those that are not negative (-1: none has one).
__device__ __forceinline__ int last_of_wave(int v) {
  const unsigned long long any = __ballot(v >= 0);
  return any ? __builtin_amdgcn_readlane(v, 63 - __builtin_clzll(any)) : -1;
}

// What a walk decides on one bin of counts v on top of `run`: whether a candidate inside may
// qualify, and whether its top candidate does (its proportion is at most the bound, and so is the quotient).
struct Verdict {
  bool may, top;
};
__device__ __forceinline__ Verdict judge(Pair run, Pair v, double eps) {
  Verdict d{false, false};
  if (v.c == 0) return d;
  const float e32 = (float)eps;
  const Pair incl = run + v;
  d.may = reaches(v.r ? incl.r : run.r, run.c + (v.r ? v.r : 1u), eps, e32);
  if (d.may) d.top = reaches(incl.r, incl.c, eps, e32);
  return d;
}

// A wave takes blocks of 256 consecutive tokens, four to a lane.  The arrays are only known to be
// aligned to their elements; the hardware loads 16 bytes from there all the same.
typedef float f32x4_any __attribute__((ext_vector_type(4), aligned(4)));
typedef int i32x4_any __attribute__((ext_vector_type(4), aligned(4)));
constexpr int kBlock = 256;
constexpr int kWaveBlocks = kSegment / 16 / kBlock;  // blocks that are a wave's share of a segment
static_assert(kWaveBlocks * 4 <= 64, "a word of correctness bits per lane");

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>)
template <int N, int I = 0, typename F>
__device__ __forceinline__ void unrolled(F&& f) {
  if constexpr (I < N) {
    f(std::integral_constant<int, I>{});
    unrolled<N, I + 1>(static_cast<F&&>(f));
  }
}

// Pass 1: correctness bits, and the level-1 counts.  One workgroup of 1024 per segment of kSegment
// tokens; it counts into 16 + 16 bit bins of its own in LDS (no bin can hold more than the segment),
// writes those inside the sample's range out and adds the others' few tokens to the table of all.
// Bound by its 12 bytes per token (2^24: 35 us, 5.8 TB/s): a wave asks for block u + kAhead before it looks
// at block u.
__global__ __launch_bounds__(1024) void calib_count1_kernel(const float* __restrict__ H, const int* __restrict__ pred,
                                                            const int* __restrict__ ref, int64_t M, CalibWork w) {
  __shared__ uint32_t bins[kBins1];
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  constexpr int kAhead = 2;
  const int64_t g0 = (int64_t)blockIdx.x * 16 * kWaveBlocks + wave;  // its blocks: every 16th of the segment
  f32x4_any h[kWaveBlocks];
  i32x4_any a[kWaveBlocks], b[kWaveBlocks];
  auto load = [&](int u) {
    h[u] = *(const f32x4_any*)(H + (g0 + 16 * u) * kBlock + 4 * lane);
    a[u] = __builtin_nontemporal_load((const i32x4_any*)(pred + (g0 + 16 * u) * kBlock + 4 * lane));
    b[u] = __builtin_nontemporal_load((const i32x4_any*)(ref + (g0 + 16 * u) * kBlock + 4 * lane));
  };
  auto load_some = [&](int u) {
    const int64_t i = (g0 + 16 * u) * kBlock + 4 * lane;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      h[u][j] = i + j < M ? H[i + j] : NAN;
      a[u][j] = i + j < M ? pred[i + j] : 0;
      b[u][j] = i + j < M ? ref[i + j] : 1;
    }
  };
  const bool whole = (int64_t)(blockIdx.x + 1) * kSegment <= M;  // uniform
  const Cut c = cut_of(w);
  if (whole) {
#pragma unroll
    for (int u = 0; u < kAhead; ++u) load(u);
  }
  for (int i = threadIdx.x; i < kBins1; i += 1024) bins[i] = 0;
  lds_barrier();
  uint32_t bits_lo = 0, bits_hi = 0;  // word 4 u + j in lane 4 u + j
  auto count = [&](auto uc) {
    constexpr int u = decltype(uc)::value;
    bool odd = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const bool right = a[u][j] == b[u][j];
      const unsigned long long word = __ballot(right);
      // A vector instruction may read a scalar register only two wait states after another has written it (the
      // ballot's compare has).  The compiler keeps that distance for its own instructions but does not look
      // into inline assembly.
      asm("s_nop 1\n\tv_writelane_b32 %0, %2, %4\n\tv_writelane_b32 %1, %3, %4"
          : "+v"(bits_lo), "+v"(bits_hi) : "s"((uint32_t)word), "s"((uint32_t)(word >> 32)), "n"(4 * u + j));
      const uint32_t off = __float_as_uint(h[u][j]) - c.lo_bits;
      const bool in = off < c.n_plain;
      odd |= !in;
      if (in) atomicAdd(&bins[kOuter + (off >> c.s)], right ? 0x10001u : 1u);
    }
    if (odd) {  // rare
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (__float_as_uint(h[u][j]) - c.lo_bits >= c.n_plain && h[u][j] == h[u][j])
          atomicAdd(&bins[c.bin(ascending_key(h[u][j]))], a[u][j] == b[u][j] ? 0x10001u : 1u);
    }
  };
  if (whole) {
    unrolled<kWaveBlocks>([&](auto uc) {
      constexpr int u = decltype(uc)::value;
      if (u + kAhead < kWaveBlocks) load(u + kAhead);
      __builtin_amdgcn_sched_barrier(0);
      count(uc);
    });
  } else {
    unrolled<kWaveBlocks>([&](auto uc) {
      load_some(decltype(uc)::value);
      count(uc);
    });
  }
  const int64_t block = g0 + 16 * (lane >> 2);
  if (lane < 4 * kWaveBlocks && block * kBlock < M) w.bits[block * 4 + (lane & 3)] = (unsigned long long)bits_hi << 32 | bits_lo;
  lds_barrier();
  uint32_t* out = w.part1 + (size_t)blockIdx.x * kInner;
  for (int i = threadIdx.x; i < kInner; i += 1024) out[i] = bins[kOuter + i];
  for (int i = threadIdx.x; i < 2 * kOuter; i += 1024) {
    const int at = i < kOuter ? i : i + kInner;
    const uint32_t v = bins[at];
    if (v) atomicAdd((unsigned long long*)&w.h1[at], (unsigned long long)(v & 0xFFFFu) | ((unsigned long long)(v >> 16) << 32));
  }
}

// grid (kInner / 256, 16): each thread adds up one bin over a sixteenth of the segments.
__global__ __launch_bounds__(256) void calib_sum1_kernel(CalibWork w, int n_parts) {
  const int b = blockIdx.x * 256 + threadIdx.x;
  const int per = (n_parts + gridDim.y - 1) / gridDim.y;
  const int p0 = blockIdx.y * per, p1 = p0 + per < n_parts ? p0 + per : n_parts;
  uint32_t cnt = 0, cor = 0;
#pragma unroll 8
  for (int p = p0; p < p1; ++p) {
    const uint32_t v = w.part1[(size_t)p * kInner + b];
    cnt += v & 0xFFFFu;
    cor += v >> 16;
  }
  if (cnt) atomicAdd((unsigned long long*)&w.h1[kOuter + b], (unsigned long long)cnt | ((unsigned long long)cor << 32));
}

// table[idx] += (1, ok) for the lanes that are `on`; lanes of a wave that name the same word
// (tokens of one entropy value sit together in the data as often as not) add once for all.
__device__ __forceinline__ void add_counted(uint64_t* __restrict__ table, uint32_t idx, bool on, unsigned ok) {
  unsigned long long pending = __ballot(on);
  const unsigned long long right = __ballot(on && ok);
  const int lane = threadIdx.x & 63;
  while (pending) {  // uniform over the wave
    const int leader = __builtin_ctzll(pending);
    const uint32_t word = __shfl(idx, leader);
    const unsigned long long same = __ballot(on && idx == word);
    if (lane == leader)
      atomicAdd((unsigned long long*)&table[word],
                (unsigned long long)__popcll(same) | ((unsigned long long)__popcll(same & right) << 32));
    pending &= ~same;
  }
}

// Keeps a bin of a level for epsilon `e`; the first to keep it gives it a row in the next table,
// which is returned (-1: it has one already, or there is no room).
__device__ __forceinline__ int keep_bin(uint64_t* sel, int* n_kept, int cap, int* overflow, int e) {
  const uint64_t old = atomicOr((unsigned long long*)sel, 1ull << e);
  if (old != 0) return -1;
  const int row = atomicAdd(n_kept, 1);
  if (row < cap) return row;
  *overflow = 0;
  return -1;
}

// What the levels hand on, per epsilon: the kept bins in the order in which the next level
// walks them, with the counts below each, so that no later kernel has to scan a table again.
constexpr int kList2 = 256;  // kept level-2 bins of one epsilon
struct EpsWalk {
  int n1;                  // kept level-1 bins, ascending
  int bin1[kCap1];
  Pair below1[kCap1];
  int n2;                  // kept level-2 bins, descending: the order of the final walk
  uint32_t at2[kList2];    // index into sel2 / slot2: row of the level-1 bin * kBins2 + bin
  uint32_t start2[kList2]; // smallest key of the bin
  int b3[kList2];          // bits of its keys that level 3 takes
  Pair below2[kList2];
};

// Level 1, one workgroup per epsilon; thread t looks at bins [PER * t, PER * (t + 1)).  Bound by what one CU
// issues and its trips to memory: 9.6 us for twice the bins that took 12.4 with 256 threads and two
// divisions a bin.
__global__ __launch_bounds__(kWalkWaves * 64) void calib_keep1_kernel(CalibWork w, EpsList eps, EpsWalk* __restrict__ walks) {
  __shared__ Pair scan[2][kWalkWaves];
  __shared__ int top_w[kWalkWaves];
  __shared__ int bin[kCap1];
  constexpr int PER = kBins1 / (kWalkWaves * 64);
  static_assert(PER * kWalkWaves * 64 == kBins1 && PER <= 32, "bins per thread");
  const int e = blockIdx.x;
  const double ep = eps.v[e];
  EpsWalk& walk = walks[e];
  const int b0 = threadIdx.x * PER;
  Pair v[PER], sum{0, 0};
#pragma unroll
  for (int j = 0; j < PER; ++j) v[j] = pair_of(w.h1[b0 + j]);
  const Cut c = cut_of(w);
#pragma unroll
  for (int j = 0; j < PER; ++j) sum = sum + v[j];
  const Pair below = block_exclusive(sum, scan[0]);
  Pair run = below;
  unsigned may = 0;
  int top = -1;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const Verdict d = judge(run, v[j], ep);
    may |= (unsigned)d.may << j;
    if (d.top) top = b0 + j;
    run = run + v[j];
  }
  top = last_of_wave(top);
  if ((threadIdx.x & 63) == 0) top_w[threadIdx.x >> 6] = top;
  lds_barrier();
  top = last_of_wave(top_w[threadIdx.x & 15]);  // (every row of lanes sees the waves in order)
  unsigned mine = 0;
#pragma unroll
  for (int j = 0; j < PER; ++j) mine |= (unsigned)((may >> j & 1u) && b0 + j >= top) << j;
  int total;
  int k = (int)block_exclusive(Pair{(uint32_t)__popc(mine), 0u}, scan[1], &total).c;
  run = below;
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    if ((mine >> j & 1u) && k < kCap1) {
      bin[k] = b0 + j;
      walk.bin1[k] = b0 + j;
      walk.below1[k] = run;
      ++k;
    }
    run = run + v[j];
  }
  if (threadIdx.x == 0) {
    walk.n1 = total < kCap1 ? total : kCap1;
    if (total > kCap1) *w.overflow = 0;
  }
  lds_barrier();
  // one bin per thread: the atomics of a workgroup are in flight together
  if ((int)threadIdx.x < total && threadIdx.x < kCap1) {
    const int b = bin[threadIdx.x];
    const int row = keep_bin(&w.sel1[b], &w.n_kept[0], kCap1, w.overflow, e);
    if (row >= 0) {
      w.slot1[b] = (signed char)row;
      w.row_b3[row] = c.b3(b);
    }
  }
}

// Pass 2: tokens of kept level-1 bins are counted by their next b2 bits and set aside for
// pass 3.  One workgroup of 1024 per segment, as in pass 1; a wave asks for all its entropies at once
// and sets tokens aside in a part of `kept` of its own, so that nothing waits for another wave.  2^24 tokens are 256
// groups of 64 for each SIMD of the card, and an instruction on each of them half a microsecond, so a
// token costs little more than its look-up: one of a kept bin (1 in 100 as a rule, but one in every
// other group) is only put into the wave's region of LDS, and what it takes to count it is done for
// full waves of them.  2^24 tokens: 26 us worked out group by group, 23 with full waves, of which 4 were
// the waves' reservation in one list, 20 now: 10 to bring the entropies, 5 to look at the last of them.
constexpr int kStageWave = 512;    // tokens of kept bins a wave holds back
__global__ __launch_bounds__(1024) void calib_count2_kernel(const float* __restrict__ H, int64_t M, CalibWork w) {
  __shared__ __align__(16) signed char slot[kBins1];  // rows are below kCap1 = 128
  __shared__ uint32_t stage_key[16][kStageWave];  // a region per wave: no barrier while the tokens stream
  __shared__ uint16_t stage_row[16][kStageWave];  // row << 6 | word of its correctness bit
  __shared__ unsigned char stage_lane[16][kStageWave];  // the bit
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int64_t wg_wave = (int64_t)blockIdx.x * 16 + wave, g0 = (int64_t)blockIdx.x * 16 * kWaveBlocks + wave;
  static_assert(kBins1 == 1024 * 16, "16 bytes of the table per thread");
  const int4 table = ((const int4*)w.slot1)[threadIdx.x];
  const int ov = *w.overflow;
  const Cut c = cut_of(w);
  unsigned long long bits = 0;
  if (lane < 4 * kWaveBlocks && (g0 + 16 * (lane >> 2)) * kBlock < M) bits = w.bits[(g0 + 16 * (lane >> 2)) * 4 + (lane & 3)];
  f32x4_any h[kWaveBlocks];
  if ((int64_t)(blockIdx.x + 1) * kSegment <= M) {  // uniform
#pragma unroll
    for (int u = 0; u < kWaveBlocks; ++u) h[u] = *(const f32x4_any*)(H + (g0 + 16 * u) * kBlock + 4 * lane);
  } else {
#pragma unroll
    for (int u = 0; u < kWaveBlocks; ++u)
#pragma unroll
      for (int j = 0; j < 4; ++j) {
        const int64_t i = (g0 + 16 * u) * kBlock + 4 * lane + j;
        h[u][j] = i < M ? H[i] : NAN;
      }
  }
  ((int4*)slot)[threadIdx.x] = table;
  lds_barrier();
  if (ov == 0) return;
  uint32_t* keys = stage_key[wave];
  uint16_t* rows = stage_row[wave];
  unsigned char* lanes = stage_lane[wave];
  uint32_t* kept = w.kept + wg_wave * kWaveBlocks * kBlock;
  int n = 0, n_out = 0;  // held back; set aside (uniform over the wave)
  auto count = [&]() {
    for (int i0 = 0; i0 < n; i0 += 64) {
      const bool on = i0 + lane < n;
      const uint32_t key = on ? keys[i0 + lane] : 0u, rk = on ? rows[i0 + lane] : 0u, bit = on ? lanes[i0 + lane] : 0u;
      const uint32_t row = rk >> 6, ok = (uint32_t)(__shfl(bits, rk & 63u) >> bit) & 1u, within = c.within(key);
      add_counted(w.h2, row * kBins2 + (within >> c.b3(c.bin(key))), on, ok);
      if (on) kept[n_out + i0 + lane] = (ok << 31) | (row << 20) | within;
    }
    n_out += n;
    n = 0;
  };
#pragma unroll
  for (int u = 0; u < kWaveBlocks; ++u) {
    if (n + kBlock > kStageWave) count();
    int row[4];
    bool odd = false;
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const uint32_t off = __float_as_uint(h[u][j]) - c.lo_bits;
      const bool in = off < c.n_plain;
      odd |= !in;
      row[j] = in ? slot[kOuter + (off >> c.s)] : -1;
    }
    if (odd) {
#pragma unroll
      for (int j = 0; j < 4; ++j)
        if (__float_as_uint(h[u][j]) - c.lo_bits >= c.n_plain && h[u][j] == h[u][j]) row[j] = slot[c.bin(ascending_key(h[u][j]))];
    }
#pragma unroll
    for (int j = 0; j < 4; ++j) {
      const unsigned long long on = __ballot(row[j] >= 0);
      if (!on) continue;  // uniform over the wave
      if (row[j] >= 0) {
        const int at = n + __popcll(on & ((1ull << lane) - 1ull));
        keys[at] = ascending_key(h[u][j]);
        rows[at] = (uint16_t)((row[j] << 6) | (4 * u + j));
        lanes[at] = (unsigned char)lane;
      }
      n += __popcll(on);
    }
  }
  count();
  if (lane == 0) w.n_aside[wg_wave] = n_out;
}

// One node for one wave: nb <= 64 * PER bins, lane l looks at bins [PER * l, PER * (l + 1)).
// Gives back the mask of the lane's bins that may hold a qualifying candidate and, as the return value, the highest
// bin whose top candidate qualifies (-1: none), with the counts up to and including it in at_top.
template <int PER>
__device__ __forceinline__ int wave_node_scan(const uint64_t* __restrict__ t, int nb, Pair below, double eps,
                                              unsigned& may, Pair& at_top) {
  const int lane = threadIdx.x & 63;
  const int b0 = lane * PER;
  Pair v[PER];
  Pair sum{0, 0};
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    v[j] = b0 + j < nb ? pair_of(t[b0 + j]) : Pair{0, 0};
    sum = sum + v[j];
  }
  const Pair inc = wave_inclusive(sum);
  Pair run{below.c + inc.c - sum.c, below.r + inc.r - sum.r};
  may = 0;
  int top = -1;
  Pair top_incl{0, 0};
#pragma unroll
  for (int j = 0; j < PER; ++j) {
    const Verdict d = judge(run, v[j], eps);
    may |= (unsigned)d.may << j;
    run = run + v[j];
    if (d.top) {
      top = b0 + j;
      top_incl = run;
    }
  }
  const int best = last_of_wave(top);
  const int owner = best >= 0 ? best / PER : 0;
  at_top = Pair{(uint32_t)__shfl((int)top_incl.c, owner), (uint32_t)__shfl((int)top_incl.r, owner)};
  return best;
}

// Level 2, one workgroup per epsilon: down the kept level-1 bins, four at a time (four waves
// each), until a top candidate qualifies.  It does not ask whether a table has proved too small already: the
// workgroups beside it may be finding that out, and its waves, which share barriers, could see different
// answers.  Behind an overflow of level 1 it walks bins without a row or with no counts, and keeps none.
__global__ __launch_bounds__(kWalkWaves * 64) void calib_keep2_kernel(CalibWork w, EpsList eps, EpsWalk* __restrict__ walks) {
  constexpr int kNodes = 4, NW = kWalkWaves / kNodes;  // nodes at a time, waves on each
  __shared__ Pair sum_w[kWalkWaves];
  __shared__ int top_w[kWalkWaves], cnt_w[kWalkWaves];
  __shared__ uint32_t at2[kList2];
  constexpr int PER = kBins2 / (NW * 64);
  const Cut c = cut_of(w);
  const int e = blockIdx.x;
  const double ep = eps.v[e];
  EpsWalk& walk = walks[e];
  const int n1 = walk.n1;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  const int node = wave / NW, b0 = ((wave % NW) * 64 + lane) * PER;
  int n2 = 0;  // uniform over the workgroup
  for (int r = 0; kNodes * r < n1; ++r) {
    const int i = n1 - 1 - (kNodes * r + node);  // uniform over the wave
    int row = 0, bin1 = 0, nb = 0;
    Pair below{0, 0};
    Pair v[PER], sum{0, 0};
    if (i >= 0) {
      bin1 = walk.bin1[i];
      below = walk.below1[i];
      row = w.slot1[bin1];
      nb = row >= 0 ? 1 << c.b2(bin1) : 0;
    }
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      v[j] = b0 + j < nb ? pair_of(w.h2[(size_t)row * kBins2 + b0 + j]) : Pair{0, 0};
      sum = sum + v[j];
    }
    const Pair inc = wave_inclusive(sum);
    if (lane == 63) sum_w[wave] = inc;
    lds_barrier();
    Pair run = below;
    for (int k = node * NW; k < wave; ++k) run = run + sum_w[k];
    run = Pair{run.c + inc.c - sum.c, run.r + inc.r - sum.r};
    const Pair start = run;
    unsigned may = 0;
    int top = -1;
#pragma unroll
    for (int j = 0; j < PER; ++j) {
      const Verdict d = judge(run, v[j], ep);
      may |= (unsigned)d.may << j;
      if (d.top) top = b0 + j;
      run = run + v[j];
    }
    top = last_of_wave(top);
    if (lane == 0) top_w[wave] = top;
    lds_barrier();
    for (int k = 0; k < NW; ++k) top = max(top, top_w[node * NW + k]);
    unsigned keep = 0;
#pragma unroll
    for (int j = 0; j < PER; ++j) keep |= (unsigned)((may >> j & 1u) && b0 + j >= top) << j;
    int before = (int)wave_inclusive((uint32_t)__popc(keep));
    if (lane == 63) cnt_w[wave] = before;
    before -= __popc(keep);
    lds_barrier();
    // the bins of the nodes down to the first one with a qualifying top candidate, each from its top
    int stop = kNodes, first = n2, all = 0, cnt = 0;
    for (int k = kWalkWaves - 1; k >= 0; --k)
      if (top_w[k] >= 0) stop = k / NW;
    for (int k = 0; k < kWalkWaves; ++k) {
      const int q = k / NW, m = cnt_w[k];
      if (q > stop) continue;
      if (q < node) first += m;
      if (q == node) {
        cnt += m;
        if (k < wave) before += m;
      }
      all += m;
    }
    if (i >= 0 && node <= stop) {
      int at = first + cnt - 1 - before;
      run = start;
#pragma unroll
      for (int j = 0; j < PER; ++j) {
        if (keep >> j & 1u) {
          if (at < kList2) {
            at2[at] = (uint32_t)row * kBins2 + b0 + j;
            walk.at2[at] = (uint32_t)row * kBins2 + b0 + j;
            walk.start2[at] = c.start(bin1) + ((uint32_t)(b0 + j) << c.b3(bin1));
            walk.b3[at] = c.b3(bin1);
            walk.below2[at] = run;
          }
          --at;
        }
        run = run + v[j];
      }
    }
    n2 += all;
    lds_barrier();  // the shared words are rewritten in the next round
    if (stop < kNodes) break;  // uniform: every smaller key is below one that qualifies
  }
  if (threadIdx.x == 0) {
    walk.n2 = n2 < kList2 ? n2 : kList2;
    if (n2 > kList2) *w.overflow = 0;
  }
  for (int k = threadIdx.x; k < n2 && k < kList2; k += kWalkWaves * 64) {
    const int row = keep_bin(&w.sel2[at2[k]], &w.n_kept[1], kCap2, w.overflow, e);
    if (row >= 0) w.slot2[at2[k]] = row;
  }
}

// Pass 3: the tokens set aside whose level-2 bin is kept are counted by their last b3 bits,
// that is, by key.  A wave takes the parts of `kept` in turn.
__global__ __launch_bounds__(256) void calib_count3_kernel(CalibWork w, int n_parts) {
  if (*w.overflow == 0) return;
  const int lane = threadIdx.x & 63, n_waves = gridDim.x * 4;
  for (int part = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6); part < n_parts; part += n_waves) {
    const int n = w.n_aside[part];
    const uint32_t* kept = w.kept + (int64_t)part * kWaveBlocks * kBlock;
    for (int i0 = 0; i0 < n; i0 += 64) {  // uniform over the wave
      const bool in = i0 + lane < n;
      const uint32_t v = in ? kept[i0 + lane] : 0u;
      const uint32_t within = v & 0xFFFFFu, row1 = (v >> 20) & 127u;
      const int b3 = in ? w.row_b3[row1] : 0;
      const int row = in ? w.slot2[(size_t)row1 * kBins2 + (within >> b3)] : -1;
      add_counted(w.h3, (uint32_t)row * kBins3 + (within & ((1u << b3) - 1u)), row >= 0, v >> 31);
    }
  }
}

// Level 3, one workgroup per epsilon: the first single key, from the top, that qualifies.
// As many kept level-2 bins at a time as there are waves.  Also tells the host whether the tables were
// large enough (a copy of that word behind the kernel took 4 us).
__global__ __launch_bounds__(kWalkWaves * 64) void calib_pick_kernel(CalibWork w, EpsList eps, const EpsWalk* __restrict__ walks,
                                                                     float* __restrict__ tau, long long* __restrict__ n_exit) {
  __shared__ int top_w[kWalkWaves];
  __shared__ uint32_t cnt_w[kWalkWaves];
  constexpr int PER = kBins3 / 64;
  const int ov = *w.overflow;
  const int e = blockIdx.x;
  const EpsWalk& walk = walks[e];
  const int n2 = walk.n2;
  if (e == 0 && threadIdx.x == 0) __hip_atomic_store(w.host_flag, ov, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_SYSTEM);
  if (ov == 0) return;
  const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  for (int r = 0; kWalkWaves * r < n2; ++r) {
    const int q = kWalkWaves * r + wave;  // uniform over the wave
    int top = -1;
    Pair at_top{0, 0};
    if (q < n2) {
      const int row = w.slot2[walk.at2[q]];
      unsigned may;
      top = wave_node_scan<PER>(w.h3 + (size_t)row * kBins3, 1 << walk.b3[q], walk.below2[q], eps.v[e], may, at_top);
    }
    if (lane == 0) {
      top_w[wave] = top;
      cnt_w[wave] = at_top.c;
    }
    __syncthreads();
    for (int k = 0; k < kWalkWaves; ++k)
      if (top_w[k] >= 0) {  // uniform
        if (threadIdx.x == 0) {
          tau[e] = ascending_entropy(walk.start2[kWalkWaves * r + k] + (uint32_t)top_w[k]);
          if (n_exit) n_exit[e] = (long long)cnt_w[k];
        }
        return;
      }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    tau[e] = -INFINITY;
    if (n_exit) n_exit[e] = 0;
  }
}

// Presets the tables: n0 words of 0 from p0, n1 words of -1 from p1; and the first kSampleWgs workgroups
// find the key range of kSample tokens, one from each of as many equal parts of the set (all tokens if there are
// no more).  Which one of a part is left to a hash: at a fixed stride a set of equally long sequences would
// be seen at the same few positions of each, whose entropies are a kind of their own; most tokens would then be
// outside the range and take the long way (2^24 tokens in sequences of 256 with one entropy at their first
// position: 552 us at a fixed stride, 104 now; the same tokens in no order 107 and 105).
__global__ __launch_bounds__(256) void calib_preset_kernel(int* __restrict__ p0, int64_t n0, int* __restrict__ p1,
                                                           int64_t n1, const float* __restrict__ H, int64_t M,
                                                           uint2* __restrict__ range) {
  const int64_t i = (int64_t)blockIdx.x * 256 + threadIdx.x;
  if (i < n0)
    p0[i] = 0;
  else if (i - n0 < n1)
    p1[i - n0] = -1;
  if (blockIdx.x >= kSampleWgs) return;
  __shared__ uint32_t sh_lo[4], sh_hi[4];
  uint32_t lo = 0xFFFFFFFFu, hi = 0u;
  constexpr int U = kSample / (kSampleWgs * 256);
  const uint32_t part = (uint32_t)(M / kSample);  // tokens to choose from
#pragma unroll
  for (int u = 0; u < U; ++u) {
    const int64_t j = ((int64_t)blockIdx.x * U + u) * 256 + threadIdx.x;
    uint32_t mix = (uint32_t)j * 0x9E3779B1u;
    mix = (mix ^ (mix >> 15)) * 0x85EBCA77u;
    mix ^= mix >> 13;
    const int64_t at = M <= kSample ? j : j * M / kSample + __umulhi(mix, part);
    const float h = at < M ? H[at] : NAN;
    if (h == h) {
      const uint32_t key = ascending_key(h);
      lo = key < lo ? key : lo;
      hi = key > hi ? key : hi;
    }
  }
#pragma unroll
  for (int o = 32; o; o >>= 1) {
    const uint32_t l2 = __shfl_xor(lo, o), h2 = __shfl_xor(hi, o);
    lo = l2 < lo ? l2 : lo;
    hi = h2 > hi ? h2 : hi;
  }
  if ((threadIdx.x & 63) == 0) {
    sh_lo[threadIdx.x >> 6] = lo;
    sh_hi[threadIdx.x >> 6] = hi;
  }
  __syncthreads();
  if (threadIdx.x == 0)
    range[blockIdx.x] = uint2{min(min(sh_lo[0], sh_lo[1]), min(sh_lo[2], sh_lo[3])),
                              max(max(sh_hi[0], sh_hi[1]), max(sh_hi[2], sh_hi[3]))};
}

}  // namespace

namespace {

// Grows the call scratch; an earlier call may still be using the old buffer on some stream.
hipError_t calib_reserve(CalibScratch& sc, size_t need) {
  if (sc.bytes >= need) return hipSuccess;
  hipError_t e = hipDeviceSynchronize();
  if (e != hipSuccess) return e;
  if (sc.buf) (void)hipFree(sc.buf);
  sc.buf = nullptr;
  sc.bytes = 0;
  e = hipMalloc(&sc.buf, need);
  if (e != hipSuccess) return e;
  sc.bytes = need;
  return hipSuccess;
}

// The full sort: always enough, about 60 bytes of traffic per token.
hipError_t calibrate_sort(CalibScratch& sc, const float* H, const int* pred, const int* ref, int64_t M,
                          const EpsList& el, float* tau_out, long long* n_exit_out, hipStream_t s) {
  const int n_eps = el.n;
  size_t tmp_sort = 0, tmp_scan = 0;
  hipError_t e = rocprim::radix_sort_pairs(nullptr, tmp_sort, (uint32_t*)nullptr, (uint32_t*)nullptr,
                                           (uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)M, 0u, 32u, s);
  if (e == hipSuccess)
    e = rocprim::inclusive_scan(nullptr, tmp_scan, (uint32_t*)nullptr, (uint32_t*)nullptr, (size_t)M,
                                rocprim::plus<uint32_t>(), s);
  if (e != hipSuccess) return e;
  const size_t tmp_bytes = ((tmp_sort > tmp_scan ? tmp_sort : tmp_scan) + 255) & ~(size_t)255;
  // one buffer: keys_in, vals_in, keys_out, vals_out, prefix (M words each), bests, primitive scratch
  const size_t words = 5 * (size_t)M + kMaxEps;
  e = calib_reserve(sc, words * sizeof(uint32_t) + 256 + tmp_bytes);
  if (e != hipSuccess) return e;
  uint32_t* buf = (uint32_t*)sc.buf;
  uint32_t *k0 = buf, *v0 = buf + M, *k1 = buf + 2 * M, *v1 = buf + 3 * M, *pf = buf + 4 * M;
  unsigned* best = buf + 5 * M;
  void* tmp = (char*)sc.buf + ((words * sizeof(uint32_t) + 255) & ~(size_t)255);
  const unsigned grid = (unsigned)((M + 255) / 256);
  hipLaunchKernelGGL(calib_keys_kernel, dim3(grid), dim3(256), 0, s, H, pred, ref, M, k0, v0);
  size_t ts = tmp_bytes;
  e = rocprim::radix_sort_pairs(tmp, ts, k0, k1, v0, v1, (size_t)M, 0u, 32u, s);
  ts = tmp_bytes;
  if (e == hipSuccess) e = rocprim::inclusive_scan(tmp, ts, v1, pf, (size_t)M, rocprim::plus<uint32_t>(), s);
  if (e != hipSuccess) return e;
  hipLaunchKernelGGL(calib_init_kernel, dim3(1), dim3(kMaxEps), 0, s, best, n_eps, (unsigned)M);
  hipLaunchKernelGGL(calib_search_kernel, dim3((unsigned)((M + 1023) / 1024)), dim3(1024), 0, s, k1, pf, M, el,
                     best);
  hipLaunchKernelGGL(calib_read_kernel, dim3(1), dim3(kMaxEps), 0, s, k1, best, n_eps, (unsigned)M, tau_out,
                     n_exit_out);
  return hipGetLastError();
}

// The refinement.  *enough comes back false if a table was too small for the data (the
// outputs are then not written).  Waits for the stream: the flag is read on the host.
hipError_t calibrate_refine(CalibScratch& sc, const float* H, const int* pred, const int* ref, int64_t M,
                            const EpsList& el, float* tau_out, long long* n_exit_out, hipStream_t s, bool* enough) {
  hipError_t e;
  if (!sc.host_flag) {
    e = hipHostMalloc((void**)&sc.host_flag, sizeof(int), hipHostMallocDefault);
    if (e != hipSuccess) return e;
  }
  const size_t n_groups = 4 * (size_t)((M + kBlock - 1) / kBlock);  // words of correctness bits
  const size_t n_segments = (size_t)((M + kSegment - 1) / kSegment);
  const size_t kept_cap = n_segments * kSegment;
  const size_t zero_words = 4 + 2 * ((size_t)kBins1 + kBins1 + 2 * (size_t)kCap1 * kBins2 + (size_t)kCap2 * kBins3);
  const size_t ones_words = 4 + (size_t)kCap1 + kBins1 / 4 + (size_t)kCap1 * kBins2;
  e = calib_reserve(sc, (2 * n_groups + 4 + n_segments * (kInner + 16) + kept_cap + 8 + 2 * kSampleWgs + zero_words + ones_words) * 4 + kMaxEps * sizeof(EpsWalk) + 256);
  if (e != hipSuccess) return e;
  CalibWork w;
  uint32_t* p = (uint32_t*)sc.buf;
  w.bits = (uint64_t*)p;
  p += (2 * n_groups + 3) & ~(size_t)3;
  w.part1 = p;
  p += n_segments * kInner;
  w.kept = p;
  p += kept_cap;
  w.n_aside = (int*)p;
  p += n_segments * 16;
  w.range = (uint2*)p;
  p += 2 * kSampleWgs;
  w.host_flag = sc.host_flag;
  uint32_t* zero0 = p;
  w.n_kept = (int*)p;
  p += 4;
  w.h1 = (uint64_t*)p;
  p += 2 * kBins1;
  w.sel1 = (uint64_t*)p;
  p += 2 * kBins1;
  w.h2 = (uint64_t*)p;
  p += 2 * (size_t)kCap1 * kBins2;
  w.sel2 = (uint64_t*)p;
  p += 2 * (size_t)kCap1 * kBins2;
  w.h3 = (uint64_t*)p;
  p += 2 * (size_t)kCap2 * kBins3;
  uint32_t* ones0 = p;
  w.overflow = (int*)p;
  p += 4;  // slot1 is read 16 bytes at a time
  w.row_b3 = (int*)p;
  p += kCap1;
  w.slot1 = (signed char*)p;
  p += kBins1 / 4;
  w.slot2 = (int*)p;
  p += (size_t)kCap1 * kBins2;
  EpsWalk* walks = (EpsWalk*)p;
  hipLaunchKernelGGL(calib_preset_kernel, dim3((unsigned)((zero_words + ones_words + 255) / 256)), dim3(256), 0, s,
                     (int*)zero0, (int64_t)zero_words, (int*)ones0, (int64_t)ones_words, H, M, w.range);
  hipLaunchKernelGGL(calib_count1_kernel, dim3((unsigned)n_segments), dim3(1024), 0, s, H, pred, ref, M, w);
  hipLaunchKernelGGL(calib_sum1_kernel, dim3(kInner / 256, 16), dim3(256), 0, s, w, (int)n_segments);
  hipLaunchKernelGGL(calib_keep1_kernel, dim3(el.n), dim3(kWalkWaves * 64), 0, s, w, el, walks);
  hipLaunchKernelGGL(calib_count2_kernel, dim3((unsigned)n_segments), dim3(1024), 0, s, H, M, w);
  hipLaunchKernelGGL(calib_keep2_kernel, dim3(el.n), dim3(kWalkWaves * 64), 0, s, w, el, walks);
  hipLaunchKernelGGL(calib_count3_kernel, dim3((unsigned)std::min<size_t>(4 * n_segments, 2048)), dim3(256), 0, s, w, (int)(16 * n_segments));
  hipLaunchKernelGGL(calib_pick_kernel, dim3(el.n), dim3(kWalkWaves * 64), 0, s, w, el, walks, tau_out, n_exit_out);
  e = hipGetLastError();
  if (e != hipSuccess) return e;
  e = hipStreamSynchronize(s);
  if (e != hipSuccess) return e;
  *enough = *sc.host_flag != 0;
  return hipSuccess;
}

}  // namespace

hipError_t calibrate_run(CalibScratch& sc, const float* H, const int* pred, const int* ref, int64_t M,
                         const double* eps, int n_eps, float* tau_out, long long* n_exit_out, hipStream_t s) {
  EpsList el;
  el.n = n_eps;
  for (int i = 0; i < n_eps; ++i) el.v[i] = eps[i];
  const char* force = getenv("EH_CALIBRATE_SORT");
  bool enough = false;
  if (!(force && force[0] == '1') && M <= kRefineMax) {
    const hipError_t e = calibrate_refine(sc, H, pred, ref, M, el, tau_out, n_exit_out, s, &enough);
    if (e != hipSuccess) return e;
  }
  if (enough) return hipSuccess;
  ++sc.n_sorted;
  return calibrate_sort(sc, H, pred, ref, M, el, tau_out, n_exit_out, s);
}

}  // namespace eh
