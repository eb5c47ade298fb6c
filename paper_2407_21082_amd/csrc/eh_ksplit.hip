// eh_eval and its relatives for a few rows: see eh_ksplit.hpp for the projection.
#include "eh_ksplit.hpp"

namespace eh {

namespace {

__host__ __device__ inline int ks_groups(int n_rows) { return (n_rows + kKsGroup - 1) / kKsGroup; }

// A workgroup walks its slice of the vocabulary (`part`) of n_heads consecutive heads (weights and bias
// vectors from the tables; activations and partial statistics of consecutive heads y_stride fragments /
// part_stride records apart) for the 64 rows from row0 on, without its weight stream stopping between
// the heads.
template <typename DT, int MT, int NB, bool AO, bool TOP2>
__device__ __forceinline__ void ks_heads(const KsSlice& sl, const frag_t* const* __restrict__ Wf, const float* const* __restrict__ bias,
                                         int n_heads, const frag_t* __restrict__ yq, long long y_stride, int KS, int V, bool wide,
                                         int n_live, int row0, int part, int R_pad, Stats* __restrict__ partials, float* __restrict__ second_out, long long part_stride,
                                         EH_KS_LDS char* lds, int wave, int lane) {
  const int row_hi = min(V, sl.t1 * 16);
  const long long slice_at = (long long)sl.t0 * KS * kWave;       // fragments (16 bytes per lane)
  const long long pass_len = (long long)2 * MT * KS * kWave;
  auto tiles_of = [&](int p) { return sl.t1 - sl.t0 - 2 * MT * p; };  // 16-row tiles from pass p on
  uint32_t voff[MT];
  ks_offsets<MT>(tiles_of(0), KS, lane, voff);
  frag_t a[2][MT][2], b[2][2][2];
  ks_start<MT>(a, Wf[0] + slice_at, KS, wave, voff);
  ks_start_b<NB>(b, yq, KS, wave, lane);
  for (int l = 0; l < n_heads; ++l) {
    Stats st[NB];
    float second[NB], z2;
#pragma unroll
    for (int nb = 0; nb < NB; ++nb) {
      stats_init(st[nb]);
      second[nb] = -INFINITY;
    }
    const frag_t* W = Wf[l] + slice_at;
    const frag_t* Wn = Wf[min(l + 1, n_heads - 1)] + slice_at;
    for (int p = 0; p < sl.passes; ++p) {
      const bool last = p + 1 == sl.passes;
      f32x16 acc[MT][NB];
      const frag_t* y = yq + l * y_stride;
      ks_pass<DT, MT, NB>(a, b, W + p * pass_len, last ? Wn : W + (p + 1) * pass_len, y, KS, wave, lane, voff,
                          tiles_of(last ? 0 : p + 1), acc, []() {},
                          [&]() { return last && l + 1 < n_heads ? y + y_stride : y; });
      ks_finish<MT, NB, AO, TOP2>(acc, lds, wave, lane, (sl.t0 + 2 * MT * p) * 16, row_hi, bias ? bias[l] : nullptr, st, second, wide);
    }
    const Stats s = ks_merge<NB, TOP2>(st, second, z2, lds, wave, lane);
    const int t = row0 + threadIdx.x;
    if (threadIdx.x < 32 * NB && t < n_live) {
      partials[l * part_stride + (long long)part * R_pad + t] = s;
      if constexpr (TOP2) second_out[l * part_stride + (long long)part * R_pad + t] = z2;
    }
  }
}

// The groups of 64 rows share the grid: `parts` workgroups over the vocabulary each, those of one slice
// side by side in time and, for a power of two of groups, on one die, whose L2 then fetches the slice
// once (one workgroup taking the groups in turn: 169 us for 512 rows of d = 1024 with a bias vector,
// against 122).  How many rows are live may only be known on the device.  While at least half of the
// groups are, the slices stay as the host's rows give them, and so do a row's sums; below that the
// grid is dealt out anew, or the few live groups would leave most compute units idle (40 live of 512
// rows: 128 us with 32 workgroups, 37 with 256).
template <typename DT, bool AO, bool TOP2>
__global__ __launch_bounds__(kKsThreads, 1) void ksplit_kernel(
    const frag_t* const* __restrict__ Wf, const float* const* __restrict__ bias, int n_heads, const frag_t* __restrict__ yq,
    long long y_stride, int VT16, int KS, int V, int wide, const int* __restrict__ n_rows_dev, int n_rows, int max_parts, int R_pad,
    Stats* __restrict__ partials, float* __restrict__ second, long long part_stride) {
  extern __shared__ __attribute__((aligned(16))) char ks_smem[];
  EH_KS_LDS char* lds = (EH_KS_LDS char*)ks_smem;
  const int lane = threadIdx.x & 63;
  const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
  int n_live = n_rows;
  if (n_rows_dev) n_live = min(max(*n_rows_dev, 0), n_rows);
  const int parts = live_parts(n_live, kKsGroup, ks_groups(n_rows), gridDim.x, max_parts);
  const int group = (int)blockIdx.x / parts, part = (int)blockIdx.x - group * parts, row0 = group * kKsGroup;
  const int mine = n_live - row0;
  if (mine <= 0) return;
  const KsSlice sl(VT16, part, parts);
  yq += (long long)group * (kKsGroup / 32) * 2 * KS * kWave;
#define EH_KS_CASE(MT_)                                                                                                    \
  case MT_:                                                                                                                \
    if (mine <= 32) ks_heads<DT, MT_, 1, AO, TOP2>(sl, Wf, bias, n_heads, yq, y_stride, KS, V, wide != 0, n_live, row0, part, R_pad, partials, second, part_stride, lds, wave, lane); \
    else ks_heads<DT, MT_, 2, AO, TOP2>(sl, Wf, bias, n_heads, yq, y_stride, KS, V, wide != 0, n_live, row0, part, R_pad, partials, second, part_stride, lds, wave, lane);           \
    break
  switch (sl.mt) {
    EH_KS_CASE(7);
    EH_KS_CASE(6);
    EH_KS_CASE(5);
    EH_KS_CASE(4);
    EH_KS_CASE(3);
    EH_KS_CASE(2);
    EH_KS_CASE(1);
    default: break;
  }
#undef EH_KS_CASE
}

template <typename DT, bool AO, bool TOP2>
hipError_t launch_ksplit(dim3 g, hipStream_t s, const frag_t* const* Wf, const float* const* bias, int n_heads, const frag_t* yq,
                         long long y_stride, int VT16, int KS, int V, int wide, const int* n_rows_dev, int n_rows, int max_parts, int R_pad,
                         Stats* partials, float* second, long long part_stride) {
  hipLaunchKernelGGL((ksplit_kernel<DT, AO, TOP2>), g, dim3(kKsThreads), ks_lds_bytes(), s, Wf, bias, n_heads, yq, y_stride, VT16, KS,
                     V, wide, n_rows_dev, n_rows, max_parts, R_pad, partials, second, part_stride);
  return hipGetLastError();
}

}  // namespace

hipError_t ksplit_prepare() {
  for (const void* fn : {(const void*)ksplit_kernel<DtBf16, false, true>, (const void*)ksplit_kernel<DtBf16, true, false>,
                         (const void*)ksplit_kernel<DtBf16, false, false>, (const void*)ksplit_kernel<DtF32, true, false>,
                         (const void*)ksplit_kernel<DtF32, false, false>, (const void*)ksplit_kernel<DtF32Whole, true, false>,
                         (const void*)ksplit_kernel<DtF32Whole, false, false>}) {
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)ks_lds_bytes());
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

int ksplit_pass_tiles(const eh_ctx* c) {
  const int slices = std::min({c->num_cu > 0 ? c->num_cu : 256, kMaxParts, c->VT});
  return ks_pass_tiles((c->VT + slices - 1) / slices);
}

hipError_t ksplit_launch(const eh_ctx* c, int head, int n_heads, const int* n_rows_dev, int n_rows, bool argmax_only,
                         const frag_t* yf, long long y_stride, Stats* partials, float* second, long long part_stride,
                         PartCount* parts, hipStream_t s) {
  const int R_pad = (n_rows + 31) & ~31;
  const int cus = c->num_cu > 0 ? c->num_cu : 256;
  // one workgroup per compute unit, or one per group of rows if that is more; as many partial
  // statistics as there is room for, and no slice without a tile of its own
  const int groups = ks_groups(n_rows), grid = std::max(cus, groups);
  const int max_parts = std::min({cus, kMaxParts, c->VT});  // (as in ksplit_pass_tiles)
  *parts = PartCount{live_parts(n_rows, kKsGroup, groups, grid, max_parts), kKsGroup, groups, n_rows_dev ? grid : 0, max_parts};
  const frag_t* const* W = (const frag_t* const*)(c->d_Wf + head);
  const float* const* bias = c->d_bias ? (const float* const*)(c->d_bias + head) : nullptr;
  const dim3 g(grid);
#define EH_KS_GO(DT, AO_, T2_)                                                                                               \
  return launch_ksplit<DT, AO_, T2_>(g, s, W, bias, n_heads, yf, y_stride, c->VT, c->KS, c->V, c->wide, n_rows_dev, n_rows, max_parts, R_pad, \
                                     partials, second, part_stride)
  if (second) {
    if (argmax_only || c->dtype != EH_BF16) return hipErrorInvalidValue;
    EH_KS_GO(DtBf16, false, true);
  }
  if (c->dtype == EH_BF16) {
    if (argmax_only) EH_KS_GO(DtBf16, true, false);
    EH_KS_GO(DtBf16, false, false);
  }
  if (c->wide) {
    if (argmax_only) EH_KS_GO(DtF32Whole, true, false);
    EH_KS_GO(DtF32Whole, false, false);
  }
  if (argmax_only) EH_KS_GO(DtF32, true, false);
  EH_KS_GO(DtF32, false, false);
#undef EH_KS_GO
}

}  // namespace eh
