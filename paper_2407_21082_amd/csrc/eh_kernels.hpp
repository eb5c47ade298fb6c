// General-purpose kernels of libeh: weight re-tiling, LayerNorm + packing,
// the streaming projection with fused softmax statistics, the cross-workgroup
// merge, the exit decision with compaction and the DSSD prefix compare.
// (arXiv 2407.21082: Section 3.2 heads, 3.4.1 entropy/argmax, 3.4.2 exit rule,
// 4.3.1 verification.)
#pragma once
#include "eh_device.hpp"

#include <algorithm>

namespace eh {

// A context's copy of a bias vector, by one workgroup.  Entries that mask a word (-infinity, the lowest float) are raised to
// kBiasSpan below the largest entry: a logit there has probability 0 all the same, and the statistics need no test per
// logit: its share t * 2^t of an entropy's sum is 0 where -infinity * 0 would be NaN, and where a lane holds nothing
// but masked words, t = z log2 e - m stays below 1 (at 10^20 the product's rounding alone is 10^13).  NaN stays.
// Where the largest entry is further from 0 than kBiasTop (a word forced by 10^30, say), a float kBiasSpan below it may
// round back to it: there *wide is set, which selects the kernels that test every logit for -infinity, and that is what
// entries become that lie below the largest by kBiasSpan and by 2^-20 of it.  A vector without a finite largest entry is
// copied as it is.
constexpr float kBiasSpan = 1e6f;
constexpr float kBiasTop = 16777216.f;  // 2^24: a float there is exact to 1
constexpr int kBiasThreads = 1024;
static __global__ __launch_bounds__(kBiasThreads) void copy_bias_kernel(const float* __restrict__ bias, int V, float* __restrict__ out,
                                                                        int* __restrict__ wide) {
  __shared__ float top[kBiasThreads];
  float m = -INFINITY;
  for (int i = threadIdx.x; i < V; i += kBiasThreads) m = fmaxf(m, bias[i]);
  top[threadIdx.x] = m;
  __syncthreads();
  for (int n = kBiasThreads / 2; n > 0; n >>= 1) {
    if ((int)threadIdx.x < n) top[threadIdx.x] = fmaxf(top[threadIdx.x], top[threadIdx.x + n]);
    __syncthreads();
  }
  const bool raise = fabsf(top[0]) <= kBiasTop;
  if (!raise && threadIdx.x == 0) *wide = 1;
  const float span = fmaxf(kBiasSpan, fabsf(top[0]) * 0x1p-20f), lowest = fabsf(top[0]) < INFINITY ? top[0] - span : -INFINITY;
  for (int i = threadIdx.x; i < V; i += kBiasThreads) out[i] = bias[i] < lowest ? (raise ? lowest : -INFINITY) : bias[i];
}

// ---------------------------------------------------------------------------
// Row-major W [V, d] -> fragment-major copy (done once, at context creation).
// One thread per 16-byte chunk of the destination.  *wide is set if a weight, or a value of gamma or beta, is not
// within 2^30.
// ---------------------------------------------------------------------------
constexpr uint32_t kWideBits = 0x4e800000u;  // 2^30
__device__ __forceinline__ bool f32_is_wide(uint32_t bits) { return (bits & 0x7fffffffu) > kWideBits; }
template <typename DT>
__global__ __launch_bounds__(256) void repack_w_kernel(const void* __restrict__ W, int V, int d,
                                                       int VT, int KS, frag_t* __restrict__ Wf, const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, int* __restrict__ wide) {
  if (blockIdx.x == 0)  // (the context's copies, [d])
    for (int i = threadIdx.x; i < d; i += blockDim.x)
      if (f32_is_wide(__float_as_uint(gamma[i])) || f32_is_wide(__float_as_uint(beta[i]))) *wide = 1;
  const int64_t o = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t total = (int64_t)VT * KS * kWave;
  if (o >= total) return;
  const int lane = (int)(o % kWave);
  const int64_t f = o / kWave;
  const int ks = (int)(f % KS);
  const int vt = (int)(f / KS);
  const int r = lane & 15, q = lane >> 4;
  const int row = vt * 16 + r;
  const int k0 = ks * DT::KPF + q * DT::EPL;
  frag_t v = mk_frag(0, 0, 0, 0);
  if (row < V && k0 < d) {
    const char* src = (const char*)W + ((int64_t)row * d + k0) * DT::ESZ;
    v = *(const frag_t*)src;  // d % EPL == 0 and a 16-byte aligned base are checked by the host
    bool out = false;
#pragma unroll
    for (int i = 0; i < 4; ++i) out |= f32_is_wide(v[i]) || (DT::EPL == 8 && f32_is_wide(v[i] << 16));
    if (out) *wide = 1;
  }
  Wf[o] = v;
}

// ---------------------------------------------------------------------------
// LayerNorm of each live row, written as y fragments.  One wave per output
// position p (gathered through row_idx).  Mean and variance are two-pass and
// the whole normalisation runs in fp64: it costs nothing at these sizes and it
// makes the bf16 rounding of y independent of the reduction order.
// Positions >= live rows (up to R_pad) are zero-filled.
// ---------------------------------------------------------------------------
template <typename DT>
__device__ __forceinline__ void load_elems(const void* row, int k0, float (&x)[DT::EPL]);

// 16 bytes of a row -> its EPL elements as float
template <typename DT>
__device__ __forceinline__ void decode_elems(const frag_t& v, float (&x)[DT::EPL]);
template <>
__device__ __forceinline__ void decode_elems<DtBf16>(const frag_t& v, float (&x)[8]) {
  x[0] = bf16_bits_to_f32(v.x & 0xffffu); x[1] = bf16_bits_to_f32(v.x >> 16);
  x[2] = bf16_bits_to_f32(v.y & 0xffffu); x[3] = bf16_bits_to_f32(v.y >> 16);
  x[4] = bf16_bits_to_f32(v.z & 0xffffu); x[5] = bf16_bits_to_f32(v.z >> 16);
  x[6] = bf16_bits_to_f32(v.w & 0xffffu); x[7] = bf16_bits_to_f32(v.w >> 16);
}
template <>
__device__ __forceinline__ void decode_elems<DtF32>(const frag_t& v, float (&x)[4]) {
  x[0] = __uint_as_float(v.x); x[1] = __uint_as_float(v.y);
  x[2] = __uint_as_float(v.z); x[3] = __uint_as_float(v.w);
}
template <>
__device__ __forceinline__ void load_elems<DtBf16>(const void* row, int k0, float (&x)[8]) {
  decode_elems<DtBf16>(*(const frag_t*)((const char*)row + (int64_t)k0 * 2), x);
}
template <>
__device__ __forceinline__ void load_elems<DtF32>(const void* row, int k0, float (&x)[4]) {
  decode_elems<DtF32>(*(const frag_t*)((const char*)row + (int64_t)k0 * 4), x);
}

// EPL outputs -> 16 bytes.  LONG: every element by f64_to_bf16_bits (the decode kernel's call of one row, whose
// timing wants it so: 313.5 us against 315.3; 8 rows 821.8 against 810.1 the other way).
template <typename DT, bool LONG = false>
struct Pack;
template <bool LONG>
struct Pack<DtBf16, LONG> {
  static __device__ __forceinline__ frag_t elems(const double (&y)[8]) {
    uint32_t b[8];
    bool normal = !LONG;
#pragma unroll
    for (int i = 0; i < 8 && !LONG; ++i) b[i] = f64_to_bf16_bits_normal(y[i], normal);
    if (!normal) {  // zeros, tiny and non-finite values: rare
#pragma unroll
      for (int i = 0; i < 8; ++i) b[i] = f64_to_bf16_bits(y[i]);
    }
    return mk_frag(b[0] | (b[1] << 16), b[2] | (b[3] << 16), b[4] | (b[5] << 16), b[6] | (b[7] << 16));
  }
};
template <bool LONG>
struct Pack<DtF32, LONG> {
  static __device__ __forceinline__ frag_t elems(const double (&y)[4]) {
    return mk_frag(__float_as_uint((float)y[0]), __float_as_uint((float)y[1]), __float_as_uint((float)y[2]),
                   __float_as_uint((float)y[3]));
  }
};
template <typename DT, bool LONG = false>
__device__ __forceinline__ frag_t pack_elems(const double (&y)[DT::EPL]) {
  return Pack<DT, LONG>::elems(y);
}

__device__ __forceinline__ double wave_sum(double v) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) v += __shfl_xor(v, o);
  return v;
}

// Rows are normalised by a workgroup of NW waves (kLnWaves in the kernels below; the decode
// kernel has its own single-wave LayerNorm).  Sum over the workgroup: per wave, then over
// the waves' totals in wave order through LDS (`red`, NW doubles, one array per call site
// so that no barrier is needed between consecutive sums).
constexpr int kLnWaves = 4;
constexpr int kLnThreads = kLnWaves * kWave;
template <int NW>
__device__ __forceinline__ double group_sum(double v, double* red, int tid) {
  v = wave_sum(v);
  if (NW == 1) return v;
  if ((tid & (kWave - 1)) == 0) red[tid >> 6] = v;
  __syncthreads();
  double t = red[0];
#pragma unroll
  for (int w = 1; w < NW; ++w) t += red[w];
  return t;
}

// LayerNorm of one row by NW waves (tid = thread in the group); out(c, chunk) receives the
// packed chunk c (EPL consecutive outputs starting at k = c*EPL) for every c < n_chunks.
// red: 2*NW doubles of LDS.
template <typename DT, int NW, typename OutFn>
__device__ __forceinline__ void group_layernorm(const void* row, int d, int n_chunks,
                                                const float* __restrict__ gamma,
                                                const float* __restrict__ beta, float eps, int tid,
                                                double* red, OutFn out) {
  constexpr int NT = NW * kWave;
  const int live_chunks = d / DT::EPL;
  double s = 0.0;
  for (int c = tid; c < live_chunks; c += NT) {
    float x[DT::EPL];
    load_elems<DT>(row, c * DT::EPL, x);
#pragma unroll
    for (int i = 0; i < DT::EPL; ++i) s += (double)x[i];
  }
  const double mu = group_sum<NW>(s, red, tid) / (double)d;
  double v = 0.0;
  for (int c = tid; c < live_chunks; c += NT) {
    float x[DT::EPL];
    load_elems<DT>(row, c * DT::EPL, x);
#pragma unroll
    for (int i = 0; i < DT::EPL; ++i) {
      const double cdev = (double)x[i] - mu;
      v += cdev * cdev;
    }
  }
  const double var = group_sum<NW>(v, red + NW, tid) / (double)d;
  const double rstd = 1.0 / sqrt(var + (double)eps);
  for (int c = tid; c < n_chunks; c += NT) {
    frag_t o = mk_frag(0, 0, 0, 0);
    if (c < live_chunks) {
      float x[DT::EPL];
      load_elems<DT>(row, c * DT::EPL, x);
      double y[DT::EPL];
#pragma unroll
      for (int i = 0; i < DT::EPL; ++i) {
        const int k = c * DT::EPL + i;
        y[i] = (double)gamma[k] * (((double)x[i] - mu) * rstd) + (double)beta[k];
      }
      o = pack_elems<DT>(y);
    }
    out(c, o);
  }
}

// Same arithmetic, in the same order, for rows of at most kLnCache*64 chunks: the row is read
// from memory once and kept in registers for the three sweeps (mean, variance, output).
constexpr int kLnCache = 8;
template <typename DT, int NW, typename OutFn>
__device__ __forceinline__ void group_layernorm_cached(const void* row, int d, int n_chunks,
                                                       const float* __restrict__ gamma,
                                                       const float* __restrict__ beta, float eps, int tid,
                                                       double* red, OutFn out) {
  constexpr int NT = NW * kWave;
  constexpr int NJ = kLnCache / NW;
  static_assert(NJ * NW == kLnCache, "cache split");
  const int live_chunks = d / DT::EPL;
  frag_t raw[NJ];
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int c = tid + j * NT;
    raw[j] = mk_frag(0, 0, 0, 0);
    if (c < live_chunks) raw[j] = *(const frag_t*)((const char*)row + (int64_t)c * 16);
  }
  double s = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (tid + j * NT < live_chunks) {
      float x[DT::EPL];
      decode_elems<DT>(raw[j], x);
#pragma unroll
      for (int i = 0; i < DT::EPL; ++i) s += (double)x[i];
    }
  }
  const double mu = group_sum<NW>(s, red, tid) / (double)d;
  double v = 0.0;
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    if (tid + j * NT < live_chunks) {
      float x[DT::EPL];
      decode_elems<DT>(raw[j], x);
#pragma unroll
      for (int i = 0; i < DT::EPL; ++i) {
        const double cdev = (double)x[i] - mu;
        v += cdev * cdev;
      }
    }
  }
  const double var = group_sum<NW>(v, red + NW, tid) / (double)d;
  const double rstd = 1.0 / sqrt(var + (double)eps);
#pragma unroll
  for (int j = 0; j < NJ; ++j) {
    const int c = tid + j * NT;
    if (c < n_chunks) {
      frag_t o = mk_frag(0, 0, 0, 0);
      if (c < live_chunks) {
        float x[DT::EPL];
        decode_elems<DT>(raw[j], x);
        double y[DT::EPL];
#pragma unroll
        for (int i = 0; i < DT::EPL; ++i) {
          const int k = c * DT::EPL + i;
          y[i] = (double)gamma[k] * (((double)x[i] - mu) * rstd) + (double)beta[k];
        }
        o = pack_elems<DT>(y);
      }
      out(c, o);
    }
  }
}

// One workgroup of kLnWaves waves per row.
// RB = rows per activation block: 16 (fragments of 16 rows x KPF k, the operand
// order of the 16x16 matrix instructions) or 32 (bf16 only: fragments of 32 rows
// x 16 k for v_mfma_f32_32x32x16_bf16; lane l of fragment (block, k16) holds row
// l%32, k = 16*k16 + 8*(l/32) .. +8).  R_pad is a multiple of RB; rows between
// the live rows and R_pad are zero-filled.
// Writes 16-byte chunk c of the row at position p of the activation workspace.
template <int RB>
__device__ __forceinline__ void put_chunk(frag_t* __restrict__ yf, int KS, int p, int c, const frag_t& v) {
  const int nb = p / RB, n = p % RB;
  // a block holds KS*4 chunks of 16 bytes per row either way
  frag_t* dst = yf + (int64_t)nb * KS * kWave * (RB / 16);
  if (RB == 16) dst[(c >> 2) * kWave + (c & 3) * 16 + n] = v;
  else dst[(c >> 1) * kWave + (c & 1) * 32 + n] = v;
}

// LayerNorm of the row at `row` into position p (the whole workgroup of kLnWaves waves; every
// thread of it must call; red: 2*kLnWaves doubles of LDS).
template <typename DT, int RB>
__device__ __forceinline__ void ln_write_row(const void* __restrict__ row, int d, int KS,
                                             const float* __restrict__ gamma,
                                             const float* __restrict__ beta, float eps,
                                             frag_t* __restrict__ yf, int p, int tid, double* red) {
  static_assert(RB == 16 || RB == 32, "row block");
  const int n_chunks = KS * 4;
  auto put = [&](int c, const frag_t& v) { put_chunk<RB>(yf, KS, p, c, v); };
  if (n_chunks <= kLnCache * kWave)
    group_layernorm_cached<DT, kLnWaves>(row, d, n_chunks, gamma, beta, eps, tid, red, put);
  else
    group_layernorm<DT, kLnWaves>(row, d, n_chunks, gamma, beta, eps, tid, red, put);
}

template <typename DT, int RB>
__device__ __forceinline__ void ln_pack_row(const void* __restrict__ h, int64_t row_stride,
                                            const int* __restrict__ row_idx, int n_live, int R_pad, int d,
                                            int KS, const float* __restrict__ gamma,
                                            const float* __restrict__ beta, float eps,
                                            frag_t* __restrict__ yf, int p, int tid, double* red) {
  if (p >= R_pad) return;
  if (p >= n_live) {
    for (int c = tid; c < KS * 4; c += kLnThreads) put_chunk<RB>(yf, KS, p, c, mk_frag(0, 0, 0, 0));
    return;
  }
  const int64_t r = row_idx ? row_idx[p] : p;
  ln_write_row<DT, RB>((const char*)h + r * row_stride * DT::ESZ, d, KS, gamma, beta, eps, yf, p, tid, red);
}

template <typename DT, int RB>
__global__ __launch_bounds__(kLnThreads) void ln_pack_kernel(const void* __restrict__ h, int64_t row_stride,
                                                     const int* __restrict__ row_idx,
                                                     const int* __restrict__ n_rows_dev, int n_rows,
                                                     int R_pad, int d, int KS,
                                                     const float* __restrict__ gamma,
                                                     const float* __restrict__ beta, float eps,
                                                     frag_t* __restrict__ yf) {
  int n_live = n_rows;
  if (n_rows_dev) n_live = min(max(*n_rows_dev, 0), n_rows);
  __shared__ double red[2 * kLnWaves];
  ln_pack_row<DT, RB>(h, row_stride, row_idx, n_live, R_pad, d, KS, gamma, beta, eps, yf, blockIdx.x,
                      threadIdx.x, red);
}

// Two heads' rows in one launch (blockIdx.y = 0 or 1), each with its own hidden states: an exit head and the model's
// for the training objectives (two launches took 14 us of 244).
struct LnRows {
  const void* h;
  int64_t row_stride;
  const float *gamma, *beta;
};
template <typename DT, int RB>
__global__ __launch_bounds__(kLnThreads) void ln_pack_pair_kernel(LnRows a, LnRows b, int n_rows, int R_pad, int d, int KS,
                                                          float eps, frag_t* __restrict__ yf, int64_t y_stride) {
  const LnRows x = blockIdx.y ? b : a;
  __shared__ double red[2 * kLnWaves];
  ln_pack_row<DT, RB>(x.h, x.row_stride, nullptr, n_rows, R_pad, d, KS, x.gamma, x.beta, eps, yf + blockIdx.y * y_stride,
                      blockIdx.x, threadIdx.x, red);
}

// The first launch of a cascade: LayerNorm of all rows for its first head, and the presets of the launches
// behind it (three launches of 4 to 5 us each otherwise): n_clear counters to zero, n_H entropies to NaN.
template <typename DT, int RB>
__global__ __launch_bounds__(kLnThreads) void cascade_init_kernel(const void* __restrict__ h, int64_t row_stride, int n_rows,
                                                          int R_pad, int d, int KS, const float* __restrict__ gamma,
                                                          const float* __restrict__ beta, float eps,
                                                          frag_t* __restrict__ yf, int* __restrict__ clear, int n_clear,
                                                          float* __restrict__ H_out, int64_t n_H) {
  if (blockIdx.x == 0 && (int)threadIdx.x < n_clear) clear[threadIdx.x] = 0;
  if (H_out)
    for (int64_t i = (int64_t)blockIdx.x * kLnThreads + threadIdx.x; i < n_H; i += (int64_t)gridDim.x * kLnThreads) H_out[i] = NAN;
  __shared__ double red[2 * kLnWaves];
  ln_pack_row<DT, RB>(h, row_stride, nullptr, n_rows, R_pad, d, KS, gamma, beta, eps, yf, blockIdx.x, threadIdx.x, red);
}

// Several heads at once and many rows (bf16, blocks of 32 rows, rows of at most kLnCache * 64 chunks): a wave per row, eight rows
// a workgroup, and the rows' chunks put next to each other in LDS before they go out, 128 bytes at a
// time.  A row by four waves, whose chunks go out 16 bytes at a time, left the chip waiting at barriers
// and wrote 64 lines with every store (8 heads x 203 rows of d = 1024 with all metrics 230 -> 226 us, 24 x 512 of
// d = 2048 2296 -> 2278).  grid (R_pad / 8, heads).
constexpr int kLnTeam = 8;
template <typename DT>
__global__ __launch_bounds__(kLnTeam* kWave) void ln_pack_many_kernel(const void* __restrict__ h_layers, int64_t layer_stride,
                                                                      int64_t row_stride, int n_rows, int d, int KS,
                                                                      const float* const* __restrict__ gamma_tab,
                                                                      const float* const* __restrict__ beta_tab, float eps,
                                                                      frag_t* __restrict__ yf, int64_t y_stride) {
  extern __shared__ __attribute__((aligned(16))) char ln_smem[];
  frag_t* tile = (frag_t*)ln_smem;  // [chunk][row], the rows of chunk c rotated by c against bank conflicts
  const int l = blockIdx.y, p0 = blockIdx.x * kLnTeam, r = threadIdx.x >> 6, lane = threadIdx.x & 63, n_chunks = KS * 4;
  auto put = [&](int c, const frag_t& v) { tile[c * kLnTeam + (r ^ (c & (kLnTeam - 1)))] = v; };
  if (p0 + r < n_rows) {
    const char* row = (const char*)h_layers + ((int64_t)l * layer_stride + (int64_t)(p0 + r) * row_stride) * DT::ESZ;
    group_layernorm_cached<DT, 1>(row, d, n_chunks, gamma_tab[l], beta_tab[l], eps, lane, (double*)nullptr, put);
  } else {
    for (int c = lane; c < n_chunks; c += kWave) put(c, mk_frag(0, 0, 0, 0));
  }
  __syncthreads();
  frag_t* dst = yf + (int64_t)l * y_stride + (int64_t)(p0 >> 5) * KS * kWave * 2 + (p0 & 31);
  for (int i = threadIdx.x; i < n_chunks * kLnTeam; i += kLnTeam * kWave) {
    const int c = i / kLnTeam, q = i % kLnTeam;
    dst[(c >> 1) * kWave + (c & 1) * 32 + q] = tile[c * kLnTeam + (q ^ (c & (kLnTeam - 1)))];
  }
}

// The same for several heads at once: blockIdx.y = head (relative to the first),
// whose hidden states start layer_stride elements after the previous head's and
// whose output goes y_stride fragments after it.
template <typename DT, int RB>
__global__ __launch_bounds__(kLnThreads) void ln_pack_heads_kernel(const void* __restrict__ h_layers,
                                                           int64_t layer_stride, int64_t row_stride,
                                                           int n_rows, int R_pad, int d, int KS,
                                                           const float* const* __restrict__ gamma_tab,
                                                           const float* const* __restrict__ beta_tab,
                                                           float eps, frag_t* __restrict__ yf,
                                                           int64_t y_stride) {
  const int l = blockIdx.y;
  const void* h = (const char*)h_layers + (int64_t)l * layer_stride * DT::ESZ;
  __shared__ double red[2 * kLnWaves];
  ln_pack_row<DT, RB>(h, row_stride, nullptr, n_rows, R_pad, d, KS, gamma_tab[l], beta_tab[l], eps,
                      yf + (int64_t)l * y_stride, blockIdx.x, threadIdx.x, red);
}

// ---------------------------------------------------------------------------
// Merge the per-workgroup partials of each live row and finalise:
// H = ln2 (log2 S - U/S), lse = ln2 (m + log2 S), argmax = ib.
// ---------------------------------------------------------------------------
__device__ __forceinline__ void stats_finalize(const Stats& s, float& H, float& lse) {
  const double S = (double)s.S, U = (double)s.U;
  const double l2 = log2(S);
  H = (float)(kLn2d * (l2 - U / S));
  lse = (float)(kLn2d * ((double)s.m + l2));
}

// A workgroup merges the partial statistics of FR rows: thread t takes the records t/FR, t/FR + 256/FR,
// ... of row t%FR, so that neighbouring threads read neighbouring records (one wave per row read
// 20 bytes of every line it fetched: 62 us for 24 heads x 512 rows x 128 records).  FR = 16; 4 for
// calls of at most 128 rows, whose few workgroups would otherwise take up to 16 records a thread one
// batch after the other (a whole call, us, FR = 16 / 4: 48 rows 33.6 / 31.7, 100 rows 32.4 / 30.8,
// 128 rows 33.3 / 31.0, 200 rows 40.9 / 40.6, 300 rows 55.5 / 55.6, 512 rows 64.2 / 65.0; 4 heads x
// 100 rows 59.7 / 58.6, 16 x 100 218 / 222, 16 x 203 312 / 314).  The number of heads does not enter: the order of
// the merge goes with FR, and many heads at once give the bits of one at a time.  TOP2: the second
// largest logit as well (with multiplicity; second of a union = max(min(z1a, z1b), max(z2a, z2b))).
// The result is valid for threads t < FR.
constexpr int kFinThreads = 256;
inline int fin_rows(int n_rows) { return n_rows <= 128 ? 4 : 16; }
template <bool TOP2, int FR>
__device__ __forceinline__ Stats merge_partials(const Stats* __restrict__ partials, const float* __restrict__ second, int n_parts,
                                                int R_pad, int row, float& z2) {
  __shared__ Stats red[kFinThreads / kWave][FR];
  __shared__ float red2[kFinThreads / kWave][FR];
  constexpr int Q = kFinThreads / FR;
  const int tid = threadIdx.x, q = tid / FR;
  Stats s;
  stats_init(s);
  z2 = -INFINITY;
  auto add = [&](const Stats& o, float o2) {
    if (TOP2) z2 = fmaxf(fminf(s.zb, o.zb), fmaxf(z2, o2));
    s = stats_merge(s, o);
  };
  for (int g0 = q; g0 < n_parts; g0 += 4 * Q) {  // four records asked for at a time
    Stats o[4];
    float o2[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int64_t at = (int64_t)min(g0 + i * Q, n_parts - 1) * R_pad + row;
      o[i] = partials[at];
      o2[i] = TOP2 ? second[at] : 0.f;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i)
      if (g0 + i * Q < n_parts) add(o[i], o2[i]);
  }
#pragma unroll
  for (int x = FR; x < kWave; x <<= 1) {
    const float p2 = TOP2 ? __shfl_xor(z2, x) : 0.f;
    add(stats_shfl_xor(s, x), p2);
  }
  if ((tid & (kWave - 1)) < FR) {
    red[tid / kWave][tid & (FR - 1)] = s;
    if (TOP2) red2[tid / kWave][tid & (FR - 1)] = z2;
  }
  __syncthreads();
  if (tid < FR) {
    s = red[0][tid];
    z2 = TOP2 ? red2[0][tid] : -INFINITY;
#pragma unroll
    for (int w = 1; w < kFinThreads / kWave; ++w) add(red[w][tid], TOP2 ? red2[w][tid] : 0.f);
  }
  return s;
}

// blockIdx.x = group of FR rows, blockIdx.y = head (relative): partials advance by part_stride
// records per head, outputs by out_stride elements (both 0 for a single head).
template <int FR>
__global__ __launch_bounds__(kFinThreads) void finalize_kernel(const Stats* __restrict__ partials, PartCount part_count,
                                                      int R_pad, const int* __restrict__ n_rows_dev,
                                                      int n_rows, float* __restrict__ H,
                                                      float* __restrict__ lse, int* __restrict__ argmax,
                                                      int64_t part_stride, int64_t out_stride) {
  const int p = blockIdx.x * FR + (threadIdx.x & (FR - 1));
  int n_live = n_rows;
  if (n_rows_dev) n_live = min(max(*n_rows_dev, 0), n_rows);
  if ((int)blockIdx.x * FR >= n_live) return;
  float z2;
  const Stats s = merge_partials<false, FR>(partials + (int64_t)blockIdx.y * part_stride, nullptr, part_count.of(n_live), R_pad,
                                        min(p, n_live - 1), z2);
  if (threadIdx.x < FR && p < n_live) {
    const int64_t o = (int64_t)blockIdx.y * out_stride + p;
    float h, l;
    stats_finalize(s, h, l);
    if (H) H[o] = h;
    if (lse) lse[o] = l;
    if (argmax) argmax[o] = stats_token(s);
  }
}

// Final merge with the other two confidence metrics of Section 3.4.1:
//   max_prob = p1 = 2^(z1 log2 e - m) / S   (S sums such terms; m is the rounded product, so this one is not quite 1)
//   margin   = p1 - p2 = p1 (1 - e^(z2 - z1)).
template <int FR>
__global__ __launch_bounds__(kFinThreads) void finalize_metrics_kernel(
    const Stats* __restrict__ partials, const float* __restrict__ second, int n_parts, int R_pad, int n_rows,
    float* __restrict__ H, float* __restrict__ lse, int* __restrict__ argmax, float* __restrict__ max_prob,
    float* __restrict__ margin, int64_t part_stride, int64_t out_stride) {
  const int p = blockIdx.x * FR + (threadIdx.x & (FR - 1));
  if ((int)blockIdx.x * FR >= n_rows) return;
  float z2;
  const Stats s = merge_partials<true, FR>(partials + (int64_t)blockIdx.y * part_stride, second + (int64_t)blockIdx.y * part_stride,
                                       n_parts, R_pad, min(p, n_rows - 1), z2);
  if (threadIdx.x < FR && p < n_rows) {
    const int64_t o = (int64_t)blockIdx.y * out_stride + p;
    float h, l;
    stats_finalize(s, h, l);
    if (H) H[o] = h;
    if (lse) lse[o] = l;
    if (argmax) argmax[o] = stats_token(s);
    const float p1 = fast_exp2(fmaf(s.zb, kLog2e, -s.m)) / s.S;  // NaN statistics give NaN metrics
    if (max_prob) max_prob[o] = p1;
    if (margin) margin[o] = p1 * (1.0f - fast_exp2((z2 - s.zb) * kLog2e));
  }
}

// ---------------------------------------------------------------------------
// Cascade step behind a head's projection (Sections 3.4.1, 3.4.2), one workgroup per
// position p of the head's active list: merge the partial statistics of the row,
// apply the exit rule, and for a row that goes on append it to the next head's
// active list and write its LayerNorm for the next head straight into the
// activation workspace at the position it got.  Positions are handed out by an
// atomic counter, so the next list is not in row order (nothing depends on the
// order: rows are independent and every output is indexed by the row).  Positions
// beyond the next head's live count keep whatever an earlier head left there; the
// projection never lets a token column influence another.
// ---------------------------------------------------------------------------
constexpr int kPostDies = 8;  // workgroups go round the dies in turn; the grid is a multiple of this
template <typename DT, int RB>
__global__ __launch_bounds__(kLnThreads) void cascade_post_kernel(
    const Stats* __restrict__ partials, PartCount part_count, int R_pad, const int* __restrict__ row_idx,
    const int* __restrict__ n_rows_dev, int n_rows, float tau, int is_last, int head,
    int* __restrict__ exit_layer,
    int* __restrict__ token, float* __restrict__ H_out, unsigned long long* __restrict__ n_evals,
    int* __restrict__ active_next, int* __restrict__ n_active_next, int* __restrict__ clear,
    const void* __restrict__ h_next, int64_t row_stride, int d, int KS,
    const float* __restrict__ gamma_next, const float* __restrict__ beta_next, float eps,
    frag_t* __restrict__ yf) {
  __shared__ double red[2 * kLnWaves];
  __shared__ Stats wave_stats[kLnWaves];
  __shared__ int pos_s;
  const int tid = threadIdx.x, lane = tid & (kWave - 1);
  if (blockIdx.x == 0 && tid == 0 && clear) *clear = 0;  // the counter of the head after next
  int n_live = n_rows;
  if (n_rows_dev) n_live = min(max(*n_rows_dev, 0), n_rows);
  // Neighbouring positions, whose records share cache lines, go to workgroups eight apart: on one die, whose L2
  // then fetches a line once, and not to every die.  12 heads, us, one after the other / eight apart: 300 rows of d = 512
  // 354.6 / 349.4, 150 of d = 768 350.7 / 347.2, 400 of d = 1024 529.5 / 527.0.
  const int per = (n_live + kPostDies - 1) / kPostDies, at = (int)blockIdx.x / kPostDies;
  const int p = (int)(blockIdx.x % kPostDies) * per + at;
  if (at >= per || p >= n_live) return;
  const int r = row_idx ? row_idx[p] : p;
  const int n_parts = part_count.of(n_live);
  // Everything the workgroup needs from memory is asked for at once: a record per thread, and the
  // row, whose LayerNorm does not depend on the decision (only whether and where it goes does).  One
  // trip to memory after the other the step took 8 to 11 us a head.
  Stats s;
  stats_init(s);
  if (tid < n_parts) s = partials[(int64_t)tid * R_pad + p];
  constexpr int kKeep = kLnCache / kLnWaves;
  frag_t keep[kKeep];
  const void* row = (const char*)h_next + (int64_t)r * row_stride * DT::ESZ;
  const bool ahead = !is_last && KS * 4 <= kLnCache * kWave;
  if (ahead)
    group_layernorm_cached<DT, kLnWaves>(row, d, KS * 4, gamma_next, beta_next, eps, tid, red,
                                         [&](int c, const frag_t& v) { keep[(c - tid) / kLnThreads] = v; });
  for (int g = tid + kLnThreads; g < n_parts; g += kLnThreads) s = stats_merge(s, partials[(int64_t)g * R_pad + p]);
#pragma unroll
  for (int x = 32; x > 0; x >>= 1) s = stats_merge(s, stats_shfl_xor(s, x));
  if (lane == 0) wave_stats[tid >> 6] = s;
  __syncthreads();
  if (tid == 0) {
#pragma unroll
    for (int w = 1; w < kLnWaves; ++w) s = stats_merge(s, wave_stats[w]);
    int pos = -1;
    float H, l;
    stats_finalize(s, H, l);
    if (H_out) H_out[r] = H;
    if (n_evals) atomicAdd(n_evals, 1ull);
    if (is_last || H < tau) {  // NaN never passes the test
      exit_layer[r] = head;
      token[r] = stats_token(s);
    } else {
      pos = atomicAdd(n_active_next, 1);
      active_next[pos] = r;
    }
    pos_s = pos;
  }
  __syncthreads();
  const int pos = pos_s;
  if (pos < 0) return;
  if (ahead) {
#pragma unroll
    for (int j = 0; j < kKeep; ++j) {
      const int c = tid + j * kLnThreads;
      if (c < KS * 4) put_chunk<RB>(yf, KS, pos, c, keep[j]);
    }
  } else {
    ln_write_row<DT, RB>(row, d, KS, gamma_next, beta_next, eps, yf, pos, tid, red);
  }
}

// ---------------------------------------------------------------------------
// Exit rule + stable compaction.  Single workgroup; positions are processed in
// chunks of blockDim.x with a block-wide exclusive scan of the "stays" flags.
// ---------------------------------------------------------------------------
static __global__ __launch_bounds__(256) void decide_kernel(const float* __restrict__ H,
                                                     const int* __restrict__ argmax,
                                                     const int* __restrict__ row_idx,
                                                     const int* __restrict__ n_rows_dev, int n_rows,
                                                     float tau, int is_last, int head,
                                                     int* __restrict__ exit_layer, int* __restrict__ token,
                                                     int* __restrict__ active_out,
                                                     int* __restrict__ n_active_out,
                                                     float* __restrict__ H_out,
                                                     unsigned long long* __restrict__ n_evals) {
  __shared__ int wave_tot[4];
  __shared__ int base_s;
  const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
  int n_live = n_rows;
  if (n_rows_dev) n_live = min(max(*n_rows_dev, 0), n_rows);
  if (tid == 0) base_s = 0;
  __syncthreads();
  for (int start = 0; start < n_live; start += blockDim.x) {
    const int p = start + tid;
    const bool valid = p < n_live;
    int r = 0;
    bool stays = false;
    if (valid) {
      r = row_idx ? row_idx[p] : p;
      const float hp = H[p];
      const bool leaves = is_last || (hp < tau);
      stays = !leaves;
      if (leaves) {
        exit_layer[r] = head;
        token[r] = argmax[p];
      }
      if (H_out) H_out[r] = hp;
    }
    const unsigned long long bal = __ballot(stays);
    const int before = __popcll(bal & ((1ull << lane) - 1ull));
    if (lane == 0) wave_tot[wave] = __popcll(bal);
    __syncthreads();
    int off = base_s;
    for (int w = 0; w < wave; ++w) off += wave_tot[w];
    if (stays) active_out[off + before] = r;
    __syncthreads();
    if (tid == 0) base_s += wave_tot[0] + wave_tot[1] + wave_tot[2] + wave_tot[3];
    __syncthreads();
  }
  if (tid == 0) {
    if (n_active_out) *n_active_out = base_s;
    if (n_evals) *n_evals += (unsigned long long)n_live;
  }
}

// ---------------------------------------------------------------------------
// DSSD: length of the accepted prefix and the token that follows it.
// ---------------------------------------------------------------------------
static __global__ void verify_compare_kernel(const int* __restrict__ draft, const int* __restrict__ draft_len,
                                      const int* __restrict__ target, int B, int k,
                                      int* __restrict__ accepted, int* __restrict__ next_token) {
  const int b = blockIdx.x * blockDim.x + threadIdx.x;
  if (b >= B) return;
  int len = k;
  if (draft_len) len = min(max(draft_len[b], 0), k);
  int n = 0;
  while (n < len && draft[(int64_t)b * k + n] == target[(int64_t)b * (k + 1) + n]) ++n;
  accepted[b] = n;
  next_token[b] = target[(int64_t)b * (k + 1) + n];
}

// The same behind the batched projection in one launch: workgroup b merges the partial
// argmax records of row b's k+1 positions, then its first wave finds the end of the prefix, 64 positions at a
// time.  `target` (nullable) receives the merged argmaxes.
//
// What bounds it is how many cache lines one compute unit can ask for: records lie [part][row], so the lanes of a wave take
// neighbouring positions of a part, and of as many parts as there is room for, and the waves share the parts.  (With a wave to a
// position, whose lanes take a part and a line each, and a prefix walked by one thread, us, verification with V = 50304, all drafts
// accepted: d = 512, one row of 32 / 64 / 200 positions 26.7 / 36.6 / 77.4 against 21.2 / 23.1 / 41.8 this way, d = 2560, 4 rows of 40
// 66.9 / 59.2.)  Up to kVerifyFew positions, where that saves no line, a wave a position is the shorter way: no second
// stage through LDS (d = 512, 64 rows of 2 positions 22.3 / 22.6, 32 of 3 21.6 / 22.2).
constexpr int kVerifyWaves = 16;  // at most
constexpr int kVerifyFew = 4;
// As many waves as ask for all records at once, and as have sixteen lanes for every position of a turn.
inline int verify_waves(int n_parts, int k) {
  if (k < kVerifyFew) return k + 1;
  const int sub = kWave / std::min(kWave, k + 1);
  int waves = 4;
  while (waves < kVerifyWaves && waves * 4 * sub < n_parts) waves *= 2;
  return k < 4 * waves ? waves : kVerifyWaves;
}
__device__ __forceinline__ void argmax_take(float& zb, int& ib, float z, int i) {
  if (z > zb || (z == zb && i < ib)) { zb = z; ib = i; }
}
// The records g0, g0 + step, ... of a position, four asked for at a time.
__device__ __forceinline__ void argmax_records(const Stats* rec, int g0, int step, int n_parts, int R_pad, float& zb, int& ib) {
  for (; g0 < n_parts; g0 += 4 * step) {
    float z[4];
    int i4[4];
#pragma unroll
    for (int i = 0; i < 4; ++i) {  // (the last record again where there are no more: no difference)
      const Stats& q = rec[(int64_t)min(g0 + i * step, n_parts - 1) * R_pad];
      z[i] = q.zb;
      i4[i] = q.ib;
    }
#pragma unroll
    for (int i = 0; i < 4; ++i) argmax_take(zb, ib, z[i], i4[i]);
  }
}
static __global__ __launch_bounds__(kVerifyWaves* kWave) void verify_post_kernel(
    const Stats* __restrict__ partials, int n_parts, int R_pad, const int* __restrict__ draft,
    const int* __restrict__ draft_len, int k, int* __restrict__ target, int* __restrict__ accepted,
    int* __restrict__ next_token) {
  extern __shared__ int verify_tgt[];  // k + 1 entries
  __shared__ float wave_z[kVerifyWaves][kWave];
  __shared__ int wave_i[kVerifyWaves][kWave];
  const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6, waves = (int)blockDim.x / kWave;
  const int64_t p0 = (int64_t)b * (k + 1);
  if (k < kVerifyFew) {
    float zb = -INFINITY;
    int ib = 0x7fffffff;
    argmax_records(partials + p0 + wave, lane, kWave, n_parts, R_pad, zb, ib);
#pragma unroll
    for (int x = kWave / 2; x > 0; x >>= 1) argmax_take(zb, ib, __shfl_xor(zb, x), __shfl_xor(ib, x));
    if (lane == 0) {
      verify_tgt[wave] = argmax_or_none(ib);
      if (target) target[p0 + wave] = argmax_or_none(ib);
    }
    __syncthreads();
  } else {
    for (int c0 = 0; c0 <= k; c0 += kWave) {
      const int n = min(kWave, k + 1 - c0);      // positions of this turn
      const int sub = kWave / n, at = lane / n;  // parts a wave takes at once, and the lane's one
      float zb = -INFINITY;
      int ib = 0x7fffffff;
      // (lanes without a part take the last one's too)
      argmax_records(partials + p0 + c0 + (lane - at * n), wave * sub + min(at, sub - 1), waves * sub, n_parts, R_pad, zb, ib);
      for (int h = kWave / 2; h > 0; h >>= 1) {
        if (h >= sub) continue;  // (the same for all lanes)
        const int from = at + h < sub ? lane + h * n : lane;
        argmax_take(zb, ib, __shfl(zb, from), __shfl(ib, from));
      }
      if (lane < n) {
        wave_z[wave][lane] = zb;
        wave_i[wave][lane] = ib;
      }
      __syncthreads();
      // sixteen neighbouring lanes to a position, the first with a wave's record each
      const int pos = threadIdx.x / kVerifyWaves, of = min((int)threadIdx.x % kVerifyWaves, waves - 1);
      zb = wave_z[of][min(pos, n - 1)];
      ib = wave_i[of][min(pos, n - 1)];
#pragma unroll
      for (int x = kVerifyWaves / 2; x > 0; x >>= 1) {
        if (x >= waves) continue;
        argmax_take(zb, ib, __shfl_xor(zb, x), __shfl_xor(ib, x));
      }
      if (threadIdx.x % kVerifyWaves == 0 && pos < n) {
        verify_tgt[c0 + pos] = argmax_or_none(ib);
        if (target) target[p0 + c0 + pos] = argmax_or_none(ib);
      }
      __syncthreads();
    }
  }
  if (wave == 0) {
    int len = k;
    if (draft_len) len = min(max(draft_len[b], 0), k);
    int n = 0;
    for (;; n += kWave) {  // (ends: the lane at position len stops)
      const int j = n + lane;
      const unsigned long long stop = __ballot(j >= len || draft[(int64_t)b * k + j] != verify_tgt[j]);
      if (stop) {
        n += __ffsll(stop) - 1;
        break;
      }
    }
    if (lane == 0) {
      accepted[b] = n;
      next_token[b] = verify_tgt[n];
    }
  }
}

// ---------------------------------------------------------------------------
// DSSD drafting controller (Section 4.3.1, "Drafting phase"): one thread, run
// behind the cascade of a position.  state = {live, length, reason, fallback}:
// `live` is the device-side row count of the next position's cascade (0 once
// drafting has stopped, which turns the remaining launches into no-ops).
// ---------------------------------------------------------------------------
static __global__ void draft_init_kernel(int* __restrict__ state, int limit, int* __restrict__ exit_layers) {
  if (threadIdx.x == 0) {
    state[0] = limit > 0 ? 1 : 0;
    state[1] = 0;
    state[2] = limit > 0 ? -1 : 0;  // an empty buffer is full at once
    state[3] = -1;
  }
  for (int i = threadIdx.x; i < limit; i += blockDim.x) exit_layers[i] = -1;
}

static __global__ void draft_step_kernel(int* __restrict__ state, const int* __restrict__ exit_layer,
                                         const int* __restrict__ token, int last_head, int limit, int eos,
                                         int* __restrict__ draft, int* __restrict__ exit_layers) {
  if (state[0] == 0) return;
  const int e = *exit_layer, tk = *token;
  if (e < 0) {  // the cascade of this position gave up (reported by eh_check): stop, append nothing
    state[0] = 0;
    state[2] = 3;
    return;
  }
  if (e >= last_head) {  // no exit head was confident: the model's own prediction is the fallback
    state[0] = 0;
    state[2] = 2;
    state[3] = tk;
    return;
  }
  const int n = state[1];
  draft[n] = tk;
  exit_layers[n] = e;
  state[1] = n + 1;
  if (tk == eos) {
    state[0] = 0;
    state[2] = 1;
  } else if (n + 1 == limit) {
    state[0] = 0;
    state[2] = 0;
  }
}

static __global__ void draft_finish_kernel(const int* __restrict__ state, int* __restrict__ draft_len,
                                           int* __restrict__ stop_reason, int* __restrict__ fallback_token) {
  *draft_len = state[1];
  if (stop_reason) *stop_reason = state[2] < 0 ? 3 : state[2];  // still running: the positions ran out
  if (fallback_token) *fallback_token = state[3];
}

// ---------------------------------------------------------------------------
// Verification bookkeeping (Section 4.3.1, verification phase; the quantities
// reported in Section 4.3.2): adds one batch of rounds to the running counters
// {rounds, drafted, accepted, wasted, exit-layer sum}.  One workgroup; lengths
// are clamped to [0, k] and accepted counts to [0, length].
// ---------------------------------------------------------------------------
static __global__ void tally_kernel(const int* __restrict__ draft_len, const int* __restrict__ accepted, int B, int k,
                                    const int* __restrict__ exit_layers, unsigned long long* __restrict__ counters) {
  long long drafted = 0, acc = 0, layers = 0;
  for (int b = threadIdx.x; b < B; b += blockDim.x) {
    int n = draft_len ? draft_len[b] : k;
    n = n < 0 ? 0 : (n > k ? k : n);
    int a = accepted[b];
    a = a < 0 ? 0 : (a > n ? n : a);
    drafted += n;
    acc += a;
    if (exit_layers)
      for (int j = 0; j < n; ++j) layers += exit_layers[(int64_t)b * k + j];
  }
  for (int o = 32; o > 0; o >>= 1) {
    drafted += __shfl_xor(drafted, o);
    acc += __shfl_xor(acc, o);
    layers += __shfl_xor(layers, o);
  }
  if ((threadIdx.x & 63) == 0) {
    atomicAdd(&counters[1], (unsigned long long)drafted);
    atomicAdd(&counters[2], (unsigned long long)acc);
    atomicAdd(&counters[3], (unsigned long long)(drafted - acc));
    atomicAdd(&counters[4], (unsigned long long)layers);
  }
  if (threadIdx.x == 0) atomicAdd(&counters[0], (unsigned long long)B);
}

// ---------------------------------------------------------------------------
// Training objectives (Section 3.3): final merge of a token's partial statistics
// (one wave per token), then the means over the sequence (one workgroup, fixed
// summation order, fp64).
// ---------------------------------------------------------------------------
static __global__ __launch_bounds__(64) void kl_finalize_kernel(const KlStats* __restrict__ partials, int n_parts,
                                                         int R_pad, int n_rows, int V,
                                                         float* __restrict__ rows, float* __restrict__ kl_out,
                                                         float* __restrict__ ce_out) {
  const int p = blockIdx.x, lane = threadIdx.x;
  if (p >= n_rows) return;
  KlStats s;
  kl_init(s, -1);
  for (int g = lane; g < n_parts; g += kWave) {
    const KlStats q = partials[(int64_t)g * R_pad + p];
    const int lab = q.lab;
    s = kl_merge(s, q);
    s.lab = lab;
  }
#pragma unroll
  for (int x = 32; x > 0; x >>= 1) {
    const KlStats o = kl_shfl_xor(s, x);
    const int lab = max(s.lab, o.lab);  // lanes that merged nothing still hold -1
    s = kl_merge(s, o);
    s.lab = lab;
  }
  if (lane == 0) {
    const double Ss = (double)s.Ss, St = (double)s.St;
    const double lse_s = kLn2d * ((double)s.ms + log2(Ss));
    const double lse_t = kLn2d * ((double)s.mt + log2(St));
    const float kl = (float)((double)s.C / Ss - lse_s + lse_t);
    const float ce = (s.lab >= 0 && s.lab < V) ? (float)(lse_s - (double)s.zl) : NAN;
    rows[p] = kl;
    rows[R_pad + p] = ce;
    if (kl_out) kl_out[p] = kl;
    if (ce_out) ce_out[p] = ce;
  }
}

// loss[0] = L_CE, loss[1] = L_KL, loss[2] = alpha * L_CE + (1 - alpha) * L_KL
static __global__ __launch_bounds__(256) void kl_mean_kernel(const float* __restrict__ rows, int R_pad, int n_rows,
                                                      float alpha, float* __restrict__ loss) {
  __shared__ double skl[256], sce[256];
  double a = 0.0, b = 0.0;
  for (int r = threadIdx.x; r < n_rows; r += 256) {
    a += (double)rows[r];
    b += (double)rows[R_pad + r];
  }
  skl[threadIdx.x] = a;
  sce[threadIdx.x] = b;
  __syncthreads();
  for (int o = 128; o > 0; o >>= 1) {
    if ((int)threadIdx.x < o) {
      skl[threadIdx.x] += skl[threadIdx.x + o];
      sce[threadIdx.x] += sce[threadIdx.x + o];
    }
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    const double L_kl = skl[0] / n_rows, L_ce = sce[0] / n_rows;
    loss[0] = (float)L_ce;
    loss[1] = (float)L_kl;
    loss[2] = (float)((double)alpha * L_ce + (1.0 - (double)alpha) * L_kl);
  }
}

static __global__ void fill_f32_kernel(float* p, int64_t n, float v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}
static __global__ void fill_i32_kernel(int* p, int64_t n, int v) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < n) p[i] = v;
}

}  // namespace eh
