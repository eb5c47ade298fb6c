// Projection with fused softmax statistics for up to 64 rows at a time: the weight stream split
// over k (arXiv 2407.21082, Sections 3.2 and 3.4.1).
//
// Up to 64 rows a head is a pure weight stream (at most 64 flop per byte in bf16), so what
// counts is that the reads never stop.  A workgroup owns a slice of the vocabulary (at most 7
// tiles of 32 rows per pass, one workgroup per CU); its four waves split the slice's k, not its
// rows or tokens: wave w takes the k-steps w, w+4, ...  A wave then shares nothing with the
// others while it streams: weights and activations go straight to registers in matrix-core
// operand order, with no LDS, no barrier and no hand-counted wait in the loop, two k-steps
// (36 KiB of weights and activations with 64 rows) always in flight per wave, 144 KiB per CU, and
// the next pass's (or the next head's) first two k-steps are asked for before this one's are
// finished, so that the stream runs on while the four waves add up their partial logits through
// LDS and work out the statistics (about 3 us).  The activations of a step are read once per
// workgroup, 4 KiB for 64 rows next to 14 KiB of weights; beyond 64 rows the accumulators no
// longer fit and the kernels that share weights through LDS are the better ones.
//
// Measured (one MI355X, V = 50304, us before -> now; before: weights shared through LDS for bf16 and
// fp32, both operands straight from memory without a pipeline for heads with a bias vector):
//   8 heads x 64 rows, d = 2560, bf16    52.8 -> 45.3 per head (4.9 -> 5.7 TB/s of weights)
//   8 heads x 32 rows, d = 1024, bf16    23.7 -> 18.4 per head (4.3 -> 5.6 TB/s)
//   6 heads x 32 rows, d = 512, fp32 cascade                 273 -> 211 (190 with products of bf16 parts)
// (single calls repeated on the same head, whose weights then stay in the 256 MB last-level cache; on
// weights met for the first time a call on 48 rows of d = 768 gains 1.24 times where it gains 1.7 then)
//
// Operands: v_mfma_f32_32x32x16_bf16; fp32 values as three bf16 ones each (ks_split).  Weights stay in the one layout the library has (fragments of 16 rows); the lane
// permutation that turns two of them into a 32-row operand is in the load addresses: lane l reads
// lane (2h + l/32)*16 + l%16 of fragment (l%32)/16, whole 256-byte lines all the same.
#pragma once
#include "eh_internal.hpp"
#include "eh_kernels.hpp"

#include <type_traits>

namespace eh {

typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kKsWaves = 4;
constexpr int kKsThreads = kKsWaves * kWave;
constexpr int kKsMaxMT = 7;      // 32-row tiles per pass
constexpr int kKsGroup = 64;     // rows per token group

#define EH_KS_LDS __attribute__((address_space(3)))
#define EH_KS_GLOBAL __attribute__((address_space(1)))

__device__ __forceinline__ f32x16 ks_mma(const frag_t& a, const frag_t& b, f32x16 c) {
  return __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}

// Eight fp32 values (both halves of a k-step of 16) as the sum of three bf16 values each: the upper 16 bits, the rest
// rounded to nearest even, and what that leaves, which has eight bits.  Exact from 2^-103 on; below that the last part, and then
// the second, may be no normal bf16 number, and less than 2^-125 is lost.  (The upper bits are cut off and not rounded, so that
// a value next to the largest float has no infinite part.)
struct KsSplit {
  frag_t hi, mid, lo;
};
__device__ __forceinline__ KsSplit ks_split(const frag_t& x0, const frag_t& x1) {
  KsSplit s;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const frag_t& x = i < 2 ? x0 : x1;
    const uint32_t a = x[2 * (i & 1)], b = x[2 * (i & 1) + 1];
    s.hi[i] = __builtin_amdgcn_perm(b, a, 0x07060302u);
    const float ra = __uint_as_float(a) - __uint_as_float(a & 0xffff0000u), rb = __uint_as_float(b) - __uint_as_float(b & 0xffff0000u);
    const uint32_t m = bf16_pair(ra, rb);
    s.mid[i] = m;
    s.lo[i] = bf16_pair(ra - __uint_as_float(m << 16), rb - __uint_as_float(m & 0xffff0000u));
  }
  return s;
}

// fp32 on fp32 matrix instructions, for contexts of `wide` values: infinity does not split into parts.
struct DtF32Whole {};
__device__ __forceinline__ f32x16 ks_mma_f32(const frag_t& a, const frag_t& b, f32x16 c) {
#pragma unroll
  for (int i = 0; i < 4; ++i) c = __builtin_amdgcn_mfma_f32_32x32x2f32(__uint_as_float(a[i]), __uint_as_float(b[i]), c, 0, 0, 0);
  return c;
}

// One k-step of all tiles and blocks.  fp32 products as six of bf16 parts, the smallest first (hi*lo, mid*mid, hi*mid,
// hi*hi).  Left out are mid*lo, lo*mid and lo*lo: of 2^-7 and 2^-16 at most, they come to 2^-22 of a product, of either sign, where
// the fp32 instructions round it by 2^-24; over a sum the errors against 64 bits are no larger (a cascade of six heads on 32 rows of
// d = 512, entropies: 4.1e-8 of their norm against 4.9e-8).  192 clocks of the matrix core for a 32 x 32 x 16 tile instead of 512.  Cascade of 6 heads, us, 512 / 192: 32 rows of d = 512 204 / 190, 24 of
// d = 1024 293 / 275; one head on 128 rows of d = 1024 with a bias vector 135 / 92.
template <typename DT, int MT, int NB>
__device__ __forceinline__ void ks_step(const frag_t (&a)[MT][2], const frag_t (&b)[2][2], f32x16 (&acc)[MT][NB]) {
  if constexpr (!std::is_same<DT, DtF32>::value) {
#pragma unroll
    for (int m = 0; m < MT; ++m)
#pragma unroll
      for (int h = 0; h < 2; ++h)
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
          acc[m][nb] = std::is_same<DT, DtBf16>::value ? ks_mma(a[m][h], b[nb][h], acc[m][nb]) : ks_mma_f32(a[m][h], b[nb][h], acc[m][nb]);
  } else {
    KsSplit y[NB];
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) y[nb] = ks_split(b[nb][0], b[nb][1]);
    constexpr int kGroup = NB == 1 ? 4 : 2;  // four accumulators in turn: none waits for its last product
#pragma unroll
    for (int m0 = 0; m0 < MT; m0 += kGroup) {
      KsSplit w[kGroup];
#pragma unroll
      for (int i = 0; i < kGroup; ++i)
        if (m0 + i < MT) w[i] = ks_split(a[m0 + i][0], a[m0 + i][1]);
#define EH_KS_TERM(A_, B_)                                                                              \
  _Pragma("unroll") for (int i = 0; i < kGroup; ++i) _Pragma("unroll") for (int nb = 0; nb < NB; ++nb) \
    if (m0 + i < MT) acc[m0 + i][nb] = ks_mma(w[i].A_, y[nb].B_, acc[m0 + i][nb])
      EH_KS_TERM(lo, hi);
      EH_KS_TERM(hi, lo);
      EH_KS_TERM(mid, mid);
      EH_KS_TERM(mid, hi);
      EH_KS_TERM(hi, mid);
      EH_KS_TERM(hi, hi);
#undef EH_KS_TERM
    }
  }
}

// LDS: partial logits handed between the waves ([destination][source][tile][lane] f32x4, one
// token block at a time), then the waves' statistics ([word][wave][token], the sixth word the second largest logit).
__host__ __device__ constexpr size_t ks_red_bytes() { return (size_t)kKsWaves * kKsWaves * kKsMaxMT * kWave * 16; }
__host__ __device__ constexpr size_t ks_lds_bytes() { return ks_red_bytes() + (size_t)6 * kKsWaves * kKsGroup * 4; }

// Waits for this wave's LDS traffic only: the weights in flight stay in flight.
__device__ __forceinline__ void ks_lds_barrier() { asm volatile("s_waitcnt lgkmcnt(0)\n\ts_barrier" ::: "memory"); }

// Loads go through buffer resources: scalar base and k offset, 32-bit lane offset, so a step's
// addresses cost no vector registers.  Every offset is in range by construction (clamped tiles and
// k-steps); the resource's size is not relied on.
typedef __amdgpu_buffer_rsrc_t ks_buf_t;
__device__ __forceinline__ ks_buf_t ks_buffer(const void* p) {
  const uint64_t v = (uint64_t)p;  // wave-uniform, kept in scalar registers
  const uint32_t lo = __builtin_amdgcn_readfirstlane((uint32_t)v), hi = __builtin_amdgcn_readfirstlane((uint32_t)(v >> 32));
  return __builtin_amdgcn_make_buffer_rsrc((void*)(((uint64_t)hi << 32) | lo), 0, 0xffffffffu, 0x00020000);
}
constexpr int kKsNt = 2;         // cache policy: non-temporal (a weight is read once)
constexpr int kKsCoherent = 16;  // cache policy: device-coherent (sc1)
template <int AUX>
__device__ __forceinline__ frag_t ks_load(ks_buf_t buf, uint32_t lane_off, uint32_t base) {
  return __builtin_bit_cast(frag_t, __builtin_amdgcn_raw_buffer_load_b128(buf, (int)lane_off, (int)base, AUX));
}

// 32-row tiles per pass of a slice of tiles16 tiles of 16: passes of at most kKsMaxMT of about equal size.
__host__ __device__ inline int ks_passes(int tiles16) { return ((tiles16 + 1) / 2 + kKsMaxMT - 1) / kKsMaxMT; }
__host__ __device__ inline int ks_pass_tiles(int tiles16) {
  const int passes = ks_passes(tiles16);
  return passes > 0 ? ((tiles16 + 1) / 2 + passes - 1) / passes : 0;
}

// One wave's view of the slice of a workgroup: 16-row tiles [t0, t1) walked in `passes` passes of
// MT 32-row tiles.
struct KsSlice {
  int t0, t1, passes, mt;
  __device__ __forceinline__ KsSlice(int VT16, int part, int parts) {
    t0 = (int)((long long)VT16 * part / parts);
    t1 = (int)((long long)VT16 * (part + 1) / parts);
    passes = ks_passes(t1 - t0);
    mt = ks_pass_tiles(t1 - t0);
  }
};

// Byte offsets of this lane's operands of the pass's MT tiles from the pass's first fragment; a
// half tile that is missing at the end of the slice repeats the slice's last one (masked later).
template <int MT>
__device__ __forceinline__ void ks_offsets(int tiles16, int KS, int lane, uint32_t (&voff)[MT]) {
#pragma unroll
  for (int m = 0; m < MT; ++m) {
    const int t = min(2 * m + ((lane & 31) >> 4), max(tiles16 - 1, 0));  // (an empty slice: its first tile, unused)
    voff[m] = ((uint32_t)t * (uint32_t)KS << 10) + (((lane >> 5) * 16 + (lane & 15)) << 4);
  }
}

template <int MT>
__device__ __forceinline__ void ks_load_a(frag_t (&a)[MT][2], ks_buf_t w, uint32_t at, const uint32_t (&voff)[MT]) {
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int h = 0; h < 2; ++h) a[m][h] = ks_load<kKsNt>(w, voff[m] + h * 512, at);
}

// byte offset of this wave's i-th k-step in the weights, clamped to the last one there is
__device__ __forceinline__ uint32_t ks_at(int i, int wave, int KS) { return (uint32_t)min(wave + kKsWaves * i, KS - 1) << 10; }

// The first two k-steps of a pass.
template <int MT>
__device__ __forceinline__ void ks_start(frag_t (&a)[2][MT][2], const void* w, int KS, int wave, const uint32_t (&voff)[MT]) {
  const ks_buf_t wu = ks_buffer(w);
#pragma unroll
  for (int j = 0; j < 2; ++j) ks_load_a<MT>(a[j], wu, ks_at(j, wave, KS), voff);
}

// Activations of this wave's i-th k-step: fragment (block nb, 2*ks + h) of 2*KS per block, in 32-row
// operand order.
template <int NB>
__device__ __forceinline__ void ks_load_b(frag_t (&b)[2][2], ks_buf_t y, int i, int KS, int wave, int lane) {
  const uint32_t at = 2 * ks_at(i, wave, KS), lane16 = (uint32_t)lane << 4;
#pragma unroll
  for (int nb = 0; nb < NB; ++nb)
#pragma unroll
    for (int h = 0; h < 2; ++h) b[nb][h] = ks_load<0>(y, lane16 + h * 1024, at + (uint32_t)nb * 2 * KS * 1024);
}
template <int NB>
__device__ __forceinline__ void ks_start_b(frag_t (&b)[2][2][2], const void* y, int KS, int wave, int lane) {
  const ks_buf_t yu = ks_buffer(y);
#pragma unroll
  for (int j = 0; j < 2; ++j) ks_load_b<NB>(b[j], yu, j, KS, wave, lane);
}

// One pass over this wave's share of k.  a and b hold the weights and activations of the pass's first
// two k-steps on entry (asked for, not waited for) and those of the next pass on return: weights
// at w_next (a slice of tiles16_next 16-row tiles, whose offsets replace voff), activations at
// y_next(), which is called in front of the last two k-steps; ask() is called two k-steps earlier
// (not at all if there are only two).  A wave with an odd number of k-steps runs one more on
// zeroed activations so that the two buffers keep their roles.
template <typename DT, int MT, int NB, typename AskFn, typename NextFn>
__device__ __forceinline__ void ks_pass(frag_t (&a)[2][MT][2], frag_t (&b)[2][2][2], const void* w, const void* w_next,
                                        const frag_t* y, int KS, int wave, int lane, uint32_t (&voff)[MT], int tiles16_next,
                                        f32x16 (&acc)[MT][NB], AskFn ask, NextFn y_next) {
  const int n = (KS - wave + kKsWaves - 1) / kKsWaves;
  const int n2 = (n + 1) & ~1;
  const ks_buf_t wu = ks_buffer(w), yu = ks_buffer(y);
#pragma unroll
  for (int m = 0; m < MT; ++m)
#pragma unroll
    for (int nb = 0; nb < NB; ++nb)
#pragma unroll
      for (int i = 0; i < 16; ++i) acc[m][nb][i] = 0.f;
  auto step = [&](frag_t (&aj)[MT][2], frag_t (&bj)[2][2]) { ks_step<DT, MT, NB>(aj, bj, acc); };
  // refills are unconditional: a load under a branch makes the compiler wait for everything
  int i = 0;
  for (; i + 2 < n2; i += 2) {
    if (i + 4 >= n2) ask();
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      step(a[j], b[j]);
      ks_load_a<MT>(a[j], wu, ks_at(i + 2 + j, wave, KS), voff);
      ks_load_b<NB>(b[j], yu, i + 2 + j, KS, wave, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
  const ks_buf_t wx = ks_buffer(w_next), yx = ks_buffer(y_next());
  ks_offsets<MT>(tiles16_next, KS, lane, voff);
  if (i < n2) {  // the last two steps refill with the next pass's first two
#pragma unroll
    for (int j = 0; j < 2; ++j) {
      if (j == 1) {
        const uint32_t keep = i + 1 < n ? 0xffffffffu : 0u;
#pragma unroll
        for (int nb = 0; nb < NB; ++nb)
#pragma unroll
          for (int h = 0; h < 2; ++h) b[1][nb][h] &= keep;
      }
      step(a[j], b[j]);
      ks_load_a<MT>(a[j], wx, ks_at(j, wave, KS), voff);
      ks_load_b<NB>(b[j], yx, j, KS, wave, lane);
      __builtin_amdgcn_sched_barrier(0);
    }
  }
}

// The logits of a pass summed over the four waves and folded into running statistics.  Wave g ends
// up with accumulator registers 4g..4g+3 of every tile, i.e. vocabulary rows row_base + 32m + 8g +
// 4*(lane/32) + i of token lane%32.  bias: NULL or [rows padded to 16].  TOP2: second[nb] is the
// largest logit besides st[nb].zb so far (with multiplicity).  wide: a logit may be -infinity.  n_cols: columns that anybody reads; a second block
// beyond them is left out.  (Between two heads of a persistent cascade of 64 rows this takes 8 us, more than the loads in
// flight last.  16 heads, us, without the second block where nobody reads it: 33 rows of d = 2048 598 -> 581, 40 of d = 1024
// 401 -> 392, 64 of d = 2560 731 -> 725.)
template <int MT, int NB, bool ARGMAX_ONLY, bool TOP2>
__device__ __forceinline__ void ks_finish(const f32x16 (&acc)[MT][NB], EH_KS_LDS char* lds, int wave, int lane,
                                          int row_base, int row_hi, const float* __restrict__ bias, Stats (&st)[NB],
                                          float (&second)[NB], bool wide, int n_cols = 32 * NB) {
  EH_KS_LDS f32x4* red = (EH_KS_LDS f32x4*)lds;
  const int r0 = row_base + 8 * wave + 4 * (lane >> 5);
  const bool ragged = row_base + 32 * MT > row_hi;  // wave-uniform: only the slice's last pass can be
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if (nb > 0 && n_cols <= 32 * nb) break;  // (uniform over the workgroup)
    ks_lds_barrier();  // nobody still reads the previous block's (or pass's) partial logits
#pragma unroll
    for (int g = 0; g < kKsWaves; ++g)
#pragma unroll
      for (int m = 0; m < MT; ++m)
        red[((g * kKsWaves + wave) * MT + m) * kWave + lane] =
            f32x4{acc[m][nb][4 * g], acc[m][nb][4 * g + 1], acc[m][nb][4 * g + 2], acc[m][nb][4 * g + 3]};
    ks_lds_barrier();
    f32x4 z[MT];
#pragma unroll
    for (int m = 0; m < MT; ++m) {
      EH_KS_LDS const f32x4* src = red + (wave * kKsWaves * MT + m) * kWave + lane;
      z[m] = (src[0] + src[MT * kWave]) + (src[2 * MT * kWave] + src[3 * MT * kWave]);
    }
    if (bias) {
#pragma unroll
      for (int m = 0; m < MT; ++m) {
        // (a half tile beyond the slice reads the bias of its last rows; masked below)
        z[m] += *(const f32x4*)(bias + min(r0 + 32 * m, (row_hi - 1) & ~3));
      }
    }
    if (ragged) {
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) z[m][i] = r0 + 32 * m + i < row_hi ? z[m][i] : -INFINITY;
    }
    // one maximum over the lane's 4*MT logits (a NaN is ignored), then independent exponentials
    float zmax = -INFINITY;
#pragma unroll
    for (int m = 0; m < MT; ++m) zmax = fmaxf(zmax, fmaxf(fmaxf(z[m][0], z[m][1]), fmaxf(z[m][2], z[m][3])));
    Stats& s = st[nb];
    if constexpr (TOP2) {
      float z1 = s.zb, z2 = second[nb];
#pragma unroll
      for (int m = 0; m < MT; ++m)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
          z2 = fmaxf(z2, fminf(z[m][i], z1));
          z1 = fmaxf(z1, z[m][i]);
        }
      second[nb] = z2;
    }
    if (zmax > s.zb) {
      int at = 0;
#pragma unroll
      for (int m = MT - 1; m >= 0; --m)
#pragma unroll
        for (int i = 3; i >= 0; --i) at = (z[m][i] == zmax) ? 32 * m + i : at;  // lowest index attaining the maximum
      if (!ARGMAX_ONLY) {
        const float mn = zmax * kLog2e;
        const float dm = s.m - mn;
        const float sc = fast_exp2(dm);
        s.U = sc * (s.U + dm * s.S);
        s.S = sc * s.S;
        s.m = mn;
      }
      s.zb = zmax;
      s.ib = r0 + at;
    }
    if (!ARGMAX_ONLY) {
      float S4[4] = {0.f, 0.f, 0.f, 0.f}, U4[4] = {0.f, 0.f, 0.f, 0.f};
      auto add = [&](bool masked) {
#pragma unroll
        for (int m = 0; m < MT; ++m)
#pragma unroll
          for (int i = 0; i < 4; ++i) {
            // a row beyond the slice, or a masked word (z = -inf), contributes 0 * (finite)
            const float t = masked && z[m][i] == -INFINITY ? -1.0e9f : z[m][i] * kLog2e - s.m;
            const float e = fast_exp2(t);
            S4[i] += e;
            U4[i] += t * e;
          }
      };
      // without the test where nothing is masked: 16 heads of d = 1024 on 64 rows 419 -> 405 us (with one block of
      // rows the second copy costs more than it saves: 8 heads of d = 2048 on 32 rows 263 -> 266)
      if (NB > 1 && !ragged && !wide) add(false);
      else add(true);
      s.S += (S4[0] + S4[1]) + (S4[2] + S4[3]);
      s.U += (U4[0] + U4[1]) + (U4[2] + U4[3]);
    }
    __builtin_amdgcn_sched_barrier(0);
  }
}

// The workgroup's statistics of token t = threadIdx.x < 32*NB, merged over the lanes and waves that
// hold its rows (every thread must call; the result is valid for those threads).
template <int NB, bool TOP2>
__device__ __forceinline__ Stats ks_merge(Stats (&st)[NB], float (&second)[NB], float& second_out, EH_KS_LDS char* lds,
                                          int wave, int lane) {
  EH_KS_LDS float* ws = (EH_KS_LDS float*)(lds + ks_red_bytes());
#pragma unroll
  for (int nb = 0; nb < NB; ++nb) {
    if constexpr (TOP2)  // second largest of a union
      second[nb] = fmaxf(fminf(st[nb].zb, __shfl_xor(st[nb].zb, 32)), fmaxf(second[nb], __shfl_xor(second[nb], 32)));
    st[nb] = stats_merge(st[nb], stats_shfl_xor(st[nb], 32));
    if (lane < 32) {
      const int at = wave * kKsGroup + nb * 32 + lane;
      ws[0 * kKsWaves * kKsGroup + at] = st[nb].m;
      ws[1 * kKsWaves * kKsGroup + at] = st[nb].S;
      ws[2 * kKsWaves * kKsGroup + at] = st[nb].U;
      ws[3 * kKsWaves * kKsGroup + at] = st[nb].zb;
      ws[4 * kKsWaves * kKsGroup + at] = __int_as_float(st[nb].ib);
      if constexpr (TOP2) ws[5 * kKsWaves * kKsGroup + at] = second[nb];
    }
  }
  ks_lds_barrier();
  Stats s;
  stats_init(s);
  second_out = -INFINITY;
  if (threadIdx.x < 32 * NB) {
#pragma unroll
    for (int w = 0; w < kKsWaves; ++w) {
      const int at = w * kKsGroup + (int)threadIdx.x;
      Stats o;
      o.m = ws[0 * kKsWaves * kKsGroup + at];
      o.S = ws[1 * kKsWaves * kKsGroup + at];
      o.U = ws[2 * kKsWaves * kKsGroup + at];
      o.zb = ws[3 * kKsWaves * kKsGroup + at];
      o.ib = __float_as_int(ws[4 * kKsWaves * kKsGroup + at]);
      if constexpr (TOP2)
        second_out = fmaxf(fminf(s.zb, o.zb), fmaxf(second_out, ws[5 * kKsWaves * kKsGroup + at]));
      s = stats_merge(s, o);
    }
  }
  return s;
}

}  // namespace eh
