// libeh: C ABI and host-side dispatch (see include/eh.h for the contract).
#include "eh.h"

#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

#include "eh_internal.hpp"
#include "eh_kernels.hpp"

using namespace eh;

// Workspace of eh_eval_noalloc: one array per GPU, part of the library's image on that GPU
// from the moment the library is loaded there until the process ends.  Host code never uses
// this name as an address: eh_create looks the array's device address up once per device
// (scratch_address) and everything is done through that pointer.
constexpr size_t kNoAllocScratchBytes = (size_t)16 << 20;
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

namespace {

thread_local std::string g_create_error = "";

constexpr int kMaxDevices = 64;
std::mutex g_scratch_mutex;
void* g_scratch_ptr[kMaxDevices] = {};

// Device address of `scratch` on `device`, which must be the current device.
hipError_t scratch_address(int device, void** out) {
  if (device < 0 || device >= kMaxDevices) return hipErrorInvalidDevice;
  std::lock_guard<std::mutex> lock(g_scratch_mutex);
  if (!g_scratch_ptr[device]) {
    void* p = nullptr;
    const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
    if (e != hipSuccess) return e;
    if (!p) return hipErrorInvalidSymbol;
    g_scratch_ptr[device] = p;
  }
  *out = g_scratch_ptr[device];
  return hipSuccess;
}

struct DeviceGuard {
  int prev = -1;
  bool changed = false;
  explicit DeviceGuard(int dev) {
    if (hipGetDevice(&prev) == hipSuccess && prev != dev) {
      changed = (hipSetDevice(dev) == hipSuccess);
    }
  }
  ~DeviceGuard() {
    if (changed) (void)hipSetDevice(prev);
  }
};

}  // namespace

namespace {

eh_status fail(eh_ctx* ctx, eh_status st, const std::string& msg) {
  if (ctx) ctx->err = msg; else g_create_error = msg;
  return st;
}

#define EH_HIP(ctx, call)                                                             \
  do {                                                                                \
    hipError_t e_ = (call);                                                           \
    if (e_ != hipSuccess)                                                             \
      return fail(ctx, EH_ERR_HIP, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

template <typename T>
hipError_t dev_alloc(eh_ctx* ctx, T** p, size_t count) {
  void* v = nullptr;
  hipError_t e = hipMalloc(&v, count * sizeof(T) > 0 ? count * sizeof(T) : 16);
  if (e == hipSuccess) {
    ctx->allocs.push_back(v);
    *p = (T*)v;
  }
  return e;
}

void free_all(eh_ctx* ctx) {
  for (void* p : ctx->allocs) (void)hipFree(p);
  ctx->allocs.clear();
  if (ctx->calib.buf) (void)hipFree(ctx->calib.buf);
  if (ctx->calib.host_flag) (void)hipHostFree(ctx->calib.host_flag);
  ctx->calib = CalibScratch();
}

inline bool aligned16(const void* p) { return ((uintptr_t)p & 15u) == 0; }

// The k-split kernel: up to 32 rows; fp32 heads with a bias vector or of d = 256 and more at any number of rows, bf16 heads
// up to its 64 unless a pass has seven tiles.  (bf16 heads with a bias vector went there at any number of rows before the
// batched kernel took one, us, V = 50257, there / here: d = 768, 48 rows 30.3 / 27.3, 100 rows 41.4 / 28.3, 200 rows 65.1 / 37.1;
// d = 1024, 300 rows 117 / 59, 512 rows 121 / 70.  Relative error of the entropies against 64 bits, mean of 12 sets: d = 768, 48 rows
// 9.5e-8 / 9.5e-8, d = 2048, 200 rows 1.10e-7 / 1.14e-7.)
// They still do where the batched kernel has too little to spread.  Small vocabularies leave it workgroups without a tile, or with one whose
// k it does not split, while this kernel deals the workgroups to groups of 64 rows (bias_few; us, weights in memory, d = 2560, there / here:
// V = 1000, 65 / 200 / 1000 rows 24.0 / 21.0, 27.7 / 22.2, 33.2 / 27.7; V = 4000, 128 / 256 / 512 rows 25.3 / 22.6, 30.3 / 25.2, 33.8 / 32.1;
// V = 8000, 128 / 256 rows 30.9 / 28.6, 39.4 / 33.5; beyond the line V = 16000, 100 / 200 rows 39 / 39, 44 / 54, V = 4000, 1000 rows
// 43 / 51, V = 8000, 512 rows 42.7 / 49.6).  Numbers of groups that are no power of two make this kernel slower (V = 4000, 320 rows
// 29.1 / 37.3, V = 8000, 150 rows 33 / 37, V = 1000, 320 rows 26.1 / 24.7) and have a line of their own.
// And one group of at most 64 rows on a vocabulary of seven tiles a pass with long k loops, whose weights fit no cache (there / here,
// 48 rows of V = 50304: d = 3072 74.8 / 73.1, 3584 85.2 / 79.8, 4096 94 / 87; V = 57000 78.7 / 80.1, 90.9 / 90.0, 103 / 100; below the line
// d = 2560 66 / 63 on weights met for the first time but 52 / 60 on a head called again).
// fp32 beyond 32 rows goes where its products cost least: this kernel makes them of bf16 parts (ks_step), gemm_launch's
// of fp32 matrix instructions, but with less to do at the end of a pass, of which a narrow head has many.  One
// head of V = 50304, us, this kernel against that, 64 / 300 / 1000 rows: d = 64 22.5 / 60 / 141 against 16.9 / 46 / 114,
// d = 128 23.2 / 65 / 146 against 20.6 / 64 / 165, d = 192 28.3 / 87 / 203 against 24.9 / 83 / 215, d = 256 28.8 / 94 / 205
// against 28.7 / 101 / 265, d = 384 34.0 / 120 / 267 against 36.0 / 138 / 362; d = 1024, 100 and 4096 rows 89 and 2412
// against 123 and 3355.  The error against 64 bits is smaller (relative, entropies / log-sum-exps, this kernel against
// that: d = 1024, 128 rows 1.3e-7 / 8e-8 against 6e-7 / 3e-7, d = 288, 48 rows 8.8e-8 / 2.6e-8 against 3.3e-7 / 4.4e-8; against
// this kernel on fp32 matrix instructions, the mean of 24 sets of 27 rows 1.4e-7 / 7e-8 against 1.6e-7 / 9e-8).  For that error the
// line lies at d = 256 although this kernel works in steps of 128 of k, and widths well below the next multiple are slower
// on vocabularies of seven tiles a pass (V = 50304, 48 / 130 rows on weights in memory: d = 256 32.2 / 60 against 30.7 / 60, d = 288
// 36.3 / 72.6 against 33.2 / 65.3, d = 320 37.7 / 75.5 against 35.5 / 70.0, d = 384 38 / 77 against 39 / 80; V = 32000, d = 288 26 / 48 against
// 27 / 48).
// bf16 at 33 to 64 rows: with seven tiles a pass (V above 12 tiles of 16 a workgroup, 49152 on 256
// compute units, up to 57344) two blocks of rows fill the register file, and the statistics behind a
// pass spill; gemm32_launch's kernel is then the better one.  With six tiles and fewer it is the better one for a
// single head of a large V (by up to 7 %), this one for several heads in one call: the line is drawn
// for those.  48 rows, us, this kernel against that, d = 512 / 1024 / 2048: one head, V = 50304 25.2 / 32.9 / 48.8
// against 21.7 / 28.9 / 43.2, V = 49152 22.7 / 29.1 / 44.3 against 21.3 / 27.7 / 43.8, V = 32000 18.3 / 23.4 / 32.6
// against 17.3 / 23.4 / 32.4, V = 16384 15.5 / 17.2 / 23.2 against 15.6 / 17.6 / 24.9; 12 heads in one call,
// V = 50304 155 / 236 / 419 against 130 / 221 / 404, V = 49152 131 / 212 / 386 against 127 / 214 / 395, V = 32000
// 96 / 151 / 270 against 100 / 159 / 284, V = 16384 63 / 94 / 164 against 69 / 113 / 204.
// Contexts of `wide` values (eh_internal.hpp) with a bias vector go there at any number of rows: its statistics test every
// logit.  fp32 ones take its form on fp32 matrix instructions, and gemm_launch's kernel beyond 32 rows without one.
constexpr int kF32Split = 256;
constexpr int kBiasLongK = 3072;
bool bias_few(const eh_ctx* c, int n_rows) {
  const int groups = (n_rows + 63) / 64;
  const int64_t tiles = (int64_t)c->VT * groups;
  return c->VT <= 512 && tiles <= ((groups & (groups - 1)) == 0 ? 2048 : 512);
}
bool use_ksplit(const eh_ctx* c, int n_rows) {
  const bool bias = !c->bias.empty();
  if (n_rows <= 32 || (c->wide && bias)) return true;
  if (c->dtype == EH_F32) return bias || (c->d >= kF32Split && !c->wide);
  if (n_rows <= 64) return ksplit_pass_tiles(c) < 7 || (bias && c->d >= kBiasLongK);
  return bias && bias_few(c, n_rows);
}
// Rows per block of the activations' operand order: 16 for gemm_launch's kernel, 32 for all others.
int row_block(const eh_ctx* c, int n_rows) { return c->dtype == EH_BF16 || use_ksplit(c, n_rows) ? 32 : 16; }

int round_up(int n, int to) { return (n + to - 1) / to * to; }

// Rows of all heads together (padded) from which ln_pack_many_kernel's wave per row is the better LayerNorm: below,
// the rows do not fill the chip and four waves have one done sooner.  One wave against four, us a call: 4 heads x
// 20 rows of d = 1024 80.4 / 79.3, 4 x 64 87.0 / 85.0, 8 x 40 of d = 2048 276 / 275, 8 x 100 of d = 1024 165 / 166, 8 x 203 with
// all metrics 222 / 224, 24 x 512 of d = 2048 2251 / 2271.
constexpr int64_t kLnMany = 1024;

// LayerNorm of a head's rows into yf, in the operand order of the kernel that n_rows rows go to.
void launch_ln(const eh_ctx* c, int head, const void* h, int64_t row_stride, const int* row_idx, const int* n_rows_dev,
               int n_rows, int R_pad, frag_t* yf, hipStream_t s) {
#define EH_LN(DT, RB)                                                                                            \
  hipLaunchKernelGGL((ln_pack_kernel<DT, RB>), dim3(R_pad), dim3(kLnThreads), 0, s, h, row_stride, row_idx,      \
                     n_rows_dev, n_rows, R_pad, c->d, c->KS, c->gamma[head], c->beta[head], c->eps, yf)
  if (c->dtype == EH_BF16) EH_LN(DtBf16, 32);
  else if (row_block(c, n_rows) == 32) EH_LN(DtF32, 32);
  else EH_LN(DtF32, 16);
#undef EH_LN
}

// Projection and partial statistics of the rows launch_ln has prepared; call_heads: heads the whole call walks.
hipError_t project(const eh_ctx* c, int head, int call_heads, const int* n_rows_dev, int n_rows, bool argmax_only, const frag_t* yf,
                   Stats* partials, PartCount* parts, hipStream_t s) {
  *parts = PartCount{0, 0, 0, 0, 0};
  if (use_ksplit(c, n_rows))
    return ksplit_launch(c, head, 1, n_rows_dev, n_rows, argmax_only, yf, 0, partials, nullptr, 0, parts, s);
  if (c->dtype == EH_BF16)
    return gemm32_launch(c, head, 1, call_heads, n_rows_dev, n_rows, argmax_only, yf, 0, partials, nullptr, 0, parts, s);
  return gemm_launch(c, head, n_rows_dev, n_rows, argmax_only, yf, partials, &parts->n, s);
}

// Merge of the partial statistics of n_heads heads (part_stride records apart), outputs [n_heads][n_rows].
void launch_finalize(const Stats* partials, PartCount parts, int R_pad, const int* n_rows_dev, int n_rows, int n_heads, float* H,
                     float* lse, int* argmax, int64_t part_stride, hipStream_t s) {
#define EH_FIN(FR)                                                                                                  \
  hipLaunchKernelGGL((finalize_kernel<FR>), dim3((n_rows + FR - 1) / FR, n_heads), dim3(kFinThreads), 0, s, partials, \
                     parts, R_pad, n_rows_dev, n_rows, H, lse, argmax, part_stride, (int64_t)n_rows)
  if (fin_rows(n_rows) == 4) EH_FIN(4);
  else EH_FIN(16);
#undef EH_FIN
}

// LayerNorm + projection + statistics for one head; results to (H, lse, argmax).
// yf / partials: the activation workspace and the per-workgroup partial statistics to use
// (the context's own, or another buffer of at least the same layout for n_rows rows).
template <bool AO>
eh_status run_head(eh_ctx* c, int head, const void* h, int64_t row_stride, const int* row_idx,
                   const int* n_rows_dev, int n_rows, float* H, float* lse, int* argmax,
                   hipStream_t s, frag_t* yf = nullptr, Stats* partials = nullptr) {
  if (!yf) yf = c->yf;
  if (!partials) partials = c->partials;
  const int R_pad = round_up(n_rows, row_block(c, n_rows));
  launch_ln(c, head, h, row_stride, row_idx, n_rows_dev, n_rows, R_pad, yf, s);
  PartCount parts;
  EH_HIP(c, project(c, head, 1, n_rows_dev, n_rows, AO, yf, partials, &parts, s));
  launch_finalize(partials, parts, R_pad, n_rows_dev, n_rows, 1, AO ? nullptr : H, AO ? nullptr : lse, argmax, 0, s);
  EH_HIP(c, hipGetLastError());
  return EH_OK;
}

eh_status check_rows(eh_ctx* ctx, const void* h, int64_t row_stride, int n_rows) {
  if (n_rows < 0 || n_rows > ctx->max_rows)
    return fail(ctx, EH_ERR_WORKSPACE, "n_rows outside [0, max_rows]");
  if (row_stride < ctx->d) return fail(ctx, EH_ERR_SHAPE, "row stride smaller than d");
  const int esz = ctx->dtype == EH_BF16 ? 2 : 4;
  if (!aligned16(h) || (row_stride * esz) % 16 != 0)
    return fail(ctx, EH_ERR_SHAPE, "hidden rows must be 16-byte aligned");
  return EH_OK;
}

// Rows <= 16 go through the persistent decode kernel when the shape fits it.
bool use_decode(const eh_ctx* c, int n_rows) { return c->decode_grid > 0 && n_rows <= 16; }
// The persistent rows kernel, one launch for a whole cascade or verification (at most 16 rows go to
// the decode kernel where the context has one, and here otherwise).
//
// A verification: its one head cannot hide the LayerNorm and the hand-over in front of its weights, and three launches
// take less time at every size measured (us, one launch / three: V = 50304, d = 512, 24 and 64 positions 28.6 / 19.4 and
// 34.3 / 21.3, d = 1024, 40 positions 41.3 / 27.6, d = 2048, 64 56.8 / 42.7, d = 2560, 18 and 63 59.6 / 52.3 and
// 67.4 / 52.7; V = 32000, d = 1024, 60 32.9 / 22.3; V = 128256, d = 2048, 32 100 / 93; one sequence of 64, V = 32000, d = 256 26.6 / 19.2,
// V = 50304, d = 2560 68.8 / 61.5).  Heads of less than kVerifySmall
// elements still take one launch up to 64 positions, and not because it is the faster way (V = 20000, d = 256, 48
// 23.3 / 14.8): the tests of a verification that gives up its bounded wait and is tried again run there.
constexpr int64_t kVerifySmall = 6000000;
//
// A cascade: as long as the two launches per head and the gaps between them cost more than the
// service workgroups, whose time grows with the rows, cost the streaming ones; the longer a head's
// stream, the more rows that is.  Rows at which 10 heads take the same time either way (measured at
// 65 to 256 rows): V = 50304, d = 512 / 640 / 768 / 1024 / 1536 none / 130 / 150 / 205 / above 256; V = 40001, d = 768
// 88, d = 960 above 112; V = 32000, d = 1024 / 1536 / 2048 88 / 165 / 205; V = 38000, d = 1024 above 112; V = 64000,
// d = 512 125.  One launch against two per head, us, 66 and 160 rows: V = 50304, d = 1024 279 / 314 and
// 326 / 342, d = 2048 383 / 484 and 436 / 517; V = 32000, d = 2048 306 / 373 and 355 / 391.  The line lies below
// those rows: it was drawn for an earlier form of the kernel, and the calls above it, which need not have
// the device to themselves, have been left as they are.
int rows_most(const eh_ctx* c) {
  // Small heads: a head's stream is over before the service workgroups have finished the one before (10 heads, one
  // launch against two per head, 65 / 80 rows, us: V = 50304, d = 512 238 / 239 against 233 / 234; V = 40001,
  // d = 768 236 / 234 against 239 / 240; V = 32000, d = 1024 243 / 239 against 245 / 248; but d = 640 of V = 50304
  // 242 / 238 against 255 / 259, d = 960 of V = 40001 248 / 256 against 276 / 275, and the more words, each of
  // which costs the statistics behind a pass the same, the smaller: V = 64000, d = 512 245 / 246 against 257 / 259,
  // V = 128256, d = 288 233 / 232 against 295 / 297).
  const int64_t bulk = (int64_t)c->V * c->d, rows_by_bulk = (int64_t)c->V * (c->d + 620) / 1000000;
  if (bulk < 35000000 && rows_by_bulk < 60) return 64;
  return (int)std::min<int64_t>(kRowsMax, std::max<int64_t>(64, 26 + rows_by_bulk));
}
bool use_rows(const eh_ctx* c, int64_t n_rows, bool verify) {
  const int most = !verify ? rows_most(c) : (int64_t)c->V * c->d < kVerifySmall ? 64 : 0;
  return c->rows_grid > 0 && (n_rows > 16 || c->decode_grid == 0) && n_rows >= 1 && n_rows <= most &&
         n_rows <= c->max_rows;
}

RowsParams rows_base(eh_ctx* c, int n_rows) {
  RowsParams p{};
  p.Wf = c->d_Wf; p.gamma = c->d_gamma; p.beta = c->d_beta; p.tau = c->d_tau;
  p.n_rows = n_rows; p.n_heads = c->n_heads;
  p.V = c->V; p.d = c->d; p.KS = c->KS; p.VT16 = c->VT; p.eps = c->eps; p.wide = c->wide;
  p.n_stream = c->rows_grid - rows_service_workgroups(n_rows, (long long)c->V * c->d);
  p.spin_limit = c->spin_limit;
  p.ctl = c->rows_ctl; p.y = c->rows_y; p.y_stride = c->rows_y_stride;
  p.part4 = c->rows_part4; p.parti = c->rows_parti; p.R_pad = (n_rows + 31) & ~31;
  p.status = c->dec_status;
  return p;
}

DecodeParams decode_base(eh_ctx* c) {
  DecodeParams p{};
  p.Wf = c->d_Wf; p.gamma = c->d_gamma; p.beta = c->d_beta; p.bias = c->d_bias; p.tau = c->d_tau;
  p.n_heads = c->n_heads; p.V = c->V; p.d = c->d; p.KS = c->KS; p.VT = c->VT; p.eps = c->eps;
  p.records = c->dec_records; p.n_heads_alloc = c->n_heads;
  if (++c->dec_epoch == 0u) ++c->dec_epoch;  // never 0
  p.epoch = c->dec_epoch; p.status = c->dec_status;
  p.spin_limit = c->spin_limit;
#ifdef EH_DIAGNOSTICS
  p.trace = c->dec_trace_on ? c->dec_trace : nullptr;
#endif
  return p;
}

}  // namespace

extern "C" {

const char* eh_version(void) { return "libeh 0.1 (gfx950)"; }

const char* eh_last_error(const eh_ctx* ctx) {
  return ctx ? ctx->err.c_str() : g_create_error.c_str();
}

eh_status eh_create(const eh_config* cfg, eh_ctx** out) {
  if (out) *out = nullptr;
  if (!cfg || !out) return fail(nullptr, EH_ERR_NULL, "cfg or out is NULL");
  if (!cfg->W || !cfg->gamma || !cfg->beta || !cfg->tau)
    return fail(nullptr, EH_ERR_NULL, "W, gamma, beta and tau are required");
  if (cfg->d <= 0 || cfg->V <= 0 || cfg->n_heads <= 0 || cfg->max_rows <= 0)
    return fail(nullptr, EH_ERR_SHAPE, "d, V, n_heads and max_rows must be positive");
  if (cfg->w_dtype != EH_F32 && cfg->w_dtype != EH_BF16)
    return fail(nullptr, EH_ERR_DTYPE, "unknown w_dtype");
  if (cfg->w_dtype != cfg->h_dtype)
    return fail(nullptr, EH_ERR_DTYPE, "w_dtype and h_dtype must match");
  const int epl = cfg->w_dtype == EH_BF16 ? 8 : 4;
  const int kpf = 4 * epl;
  if (cfg->d % epl != 0)
    return fail(nullptr, EH_ERR_SHAPE, "d must be a multiple of 16 bytes worth of elements");
  if (!(cfg->ln_eps > 0.f) || !std::isfinite(cfg->ln_eps))
    return fail(nullptr, EH_ERR_RANGE, "ln_eps must be positive and finite");
  if ((int64_t)cfg->max_rows > (1 << 20)) return fail(nullptr, EH_ERR_RANGE, "max_rows too large");
  for (int l = 0; l < cfg->n_heads; ++l) {
    if (!cfg->W[l] || !cfg->gamma[l] || !cfg->beta[l] || (cfg->bias && !cfg->bias[l]))
      return fail(nullptr, EH_ERR_NULL, "a per-head pointer is NULL");
    if (!aligned16(cfg->W[l])) return fail(nullptr, EH_ERR_SHAPE, "W must be 16-byte aligned");
  }
  int ndev = 0;
  if (hipGetDeviceCount(&ndev) != hipSuccess || cfg->device < 0 || cfg->device >= ndev)
    return fail(nullptr, EH_ERR_RANGE, "no such HIP device");

  eh_ctx* c = new (std::nothrow) eh_ctx();
  if (!c) return fail(nullptr, EH_ERR_HIP, "out of host memory");
  c->d = cfg->d; c->V = cfg->V; c->n_heads = cfg->n_heads; c->max_rows = cfg->max_rows;
  c->dtype = cfg->w_dtype; c->device = cfg->device; c->eps = cfg->ln_eps;
  c->KS = (cfg->d + kpf - 1) / kpf;
  c->VT = (cfg->V + 15) / 16;
  c->R_pad_max = (cfg->max_rows + 31) & ~31;
  c->tau.assign(cfg->tau, cfg->tau + cfg->n_heads);

  DeviceGuard guard(c->device);
  auto bail = [&](hipError_t e, const char* what) {
    std::string msg = std::string(what) + ": " + hipGetErrorString(e);
    free_all(c);
    delete c;
    return fail(nullptr, EH_ERR_HIP, msg);
  };
  hipError_t e;
  if ((e = scratch_address(c->device, &c->static_scratch)) != hipSuccess) return bail(e, "hipGetSymbolAddress(scratch)");
  const size_t wf_frags = (size_t)c->VT * c->KS * kWave;
  const int Vp = c->VT * 16;
  c->Wf.resize(c->n_heads); c->gamma.resize(c->n_heads); c->beta.resize(c->n_heads);
  if (cfg->bias) c->bias.resize(c->n_heads);
  // the status word both persistent kernels report a given-up wait in (read by eh_check), and what is found about the values
  if ((e = dev_alloc(c, &c->dec_status, (size_t)4)) != hipSuccess) return bail(e, "hipMalloc(status)");
  if ((e = hipMemset(c->dec_status, 0, 16)) != hipSuccess) return bail(e, "memset");
  int* const wide = c->dec_status + 1;
  for (int l = 0; l < c->n_heads; ++l) {
    if ((e = dev_alloc(c, &c->Wf[l], wf_frags)) != hipSuccess) return bail(e, "hipMalloc(W)");
    if ((e = dev_alloc(c, &c->gamma[l], (size_t)c->d)) != hipSuccess) return bail(e, "hipMalloc(gamma)");
    if ((e = dev_alloc(c, &c->beta[l], (size_t)c->d)) != hipSuccess) return bail(e, "hipMalloc(beta)");
    if ((e = hipMemcpy(c->gamma[l], cfg->gamma[l], sizeof(float) * c->d, hipMemcpyDeviceToDevice)) != hipSuccess)
      return bail(e, "copy gamma");
    if ((e = hipMemcpy(c->beta[l], cfg->beta[l], sizeof(float) * c->d, hipMemcpyDeviceToDevice)) != hipSuccess)
      return bail(e, "copy beta");
    const unsigned blocks = (unsigned)((wf_frags + 255) / 256);
    if (c->dtype == EH_BF16)
      hipLaunchKernelGGL((repack_w_kernel<DtBf16>), dim3(blocks), dim3(256), 0, 0, cfg->W[l], c->V,
                         c->d, c->VT, c->KS, c->Wf[l], c->gamma[l], c->beta[l], wide);
    else
      hipLaunchKernelGGL((repack_w_kernel<DtF32>), dim3(blocks), dim3(256), 0, 0, cfg->W[l], c->V,
                         c->d, c->VT, c->KS, c->Wf[l], c->gamma[l], c->beta[l], wide);
    if ((e = hipGetLastError()) != hipSuccess) return bail(e, "repack launch");
    if (cfg->bias) {
      if ((e = dev_alloc(c, &c->bias[l], (size_t)Vp)) != hipSuccess) return bail(e, "hipMalloc(bias)");
      if ((e = hipMemset(c->bias[l], 0, sizeof(float) * Vp)) != hipSuccess) return bail(e, "memset bias");
      hipLaunchKernelGGL(copy_bias_kernel, dim3(1), dim3(kBiasThreads), 0, 0, cfg->bias[l], c->V, c->bias[l], wide);
      if ((e = hipGetLastError()) != hipSuccess) return bail(e, "bias launch");
    }
  }
  int is_wide = 0;
  if ((e = hipMemcpy(&is_wide, wide, sizeof(int), hipMemcpyDeviceToHost)) != hipSuccess) return bail(e, "copy wide");
  c->wide = is_wide != 0;
  // the fp32 kernel reads whole groups of token blocks, up to 4 waves x 8 blocks of 16 rows
  // starting inside the padded rows, so 32 zero blocks follow them
  const size_t y_frags = (size_t)(c->R_pad_max / 16 + 32) * c->KS * kWave;
  if ((e = dev_alloc(c, &c->yf, y_frags)) != hipSuccess) return bail(e, "hipMalloc(y)");
  if ((e = hipMemset(c->yf, 0, y_frags * sizeof(frag_t))) != hipSuccess) return bail(e, "memset y");
  if ((e = dev_alloc(c, &c->partials, (size_t)kMaxParts * c->R_pad_max)) != hipSuccess)
    return bail(e, "hipMalloc(partials)");
  if ((e = dev_alloc(c, &c->ws_argmax, (size_t)c->max_rows)) != hipSuccess) return bail(e, "hipMalloc(ws)");
  for (int i = 0; i < 2; ++i) {
    if ((e = dev_alloc(c, &c->active[i], (size_t)c->max_rows)) != hipSuccess) return bail(e, "hipMalloc(ws)");
    if ((e = dev_alloc(c, &c->n_active[i], (size_t)4)) != hipSuccess) return bail(e, "hipMalloc(ws)");
  }
  {
    // device-side tables for the persistent decode kernel
    const size_t np = (size_t)c->n_heads;
    if ((e = dev_alloc(c, &c->d_Wf, np)) != hipSuccess) return bail(e, "hipMalloc(tables)");
    if ((e = dev_alloc(c, &c->d_gamma, np)) != hipSuccess) return bail(e, "hipMalloc(tables)");
    if ((e = dev_alloc(c, &c->d_beta, np)) != hipSuccess) return bail(e, "hipMalloc(tables)");
    if ((e = dev_alloc(c, &c->d_tau, np)) != hipSuccess) return bail(e, "hipMalloc(tables)");
    if ((e = hipMemcpy(c->d_Wf, c->Wf.data(), np * sizeof(void*), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "copy tables");
    if ((e = hipMemcpy(c->d_gamma, c->gamma.data(), np * sizeof(void*), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "copy tables");
    if ((e = hipMemcpy(c->d_beta, c->beta.data(), np * sizeof(void*), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "copy tables");
    if ((e = hipMemcpy(c->d_tau, c->tau.data(), np * sizeof(float), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "copy tables");
    if (cfg->bias) {
      if ((e = dev_alloc(c, &c->d_bias, np)) != hipSuccess) return bail(e, "hipMalloc(tables)");
      if ((e = hipMemcpy(c->d_bias, c->bias.data(), np * sizeof(void*), hipMemcpyHostToDevice)) != hipSuccess) return bail(e, "copy tables");
    }
    if ((e = decode_prepare(c)) != hipSuccess) return bail(e, "decode_prepare");
    if ((e = rows_prepare(c)) != hipSuccess) return bail(e, "rows_prepare");
    if ((e = gemm_prepare()) != hipSuccess) return bail(e, "gemm_prepare");
    if ((e = gemm32_prepare()) != hipSuccess) return bail(e, "gemm32_prepare");
    if ((e = ksplit_prepare()) != hipSuccess) return bail(e, "ksplit_prepare");
    if (c->rows_grid > 0 && (c->max_rows > 16 || c->decode_grid == 0)) {
      // workspace of the persistent kernel for as many rows as it may get: one activation buffer per
      // head (plus the blocks a wave may read past the last live one), two sets of partial statistics
      const int rmax = std::min(c->R_pad_max, round_up(rows_most(c), 32));
      c->rows_y_stride = (long long)(rmax / 16 + 32) * c->KS * kWave;
      c->rows_ctl_ints = rows_control_ints(c->n_heads);
      if ((e = dev_alloc(c, &c->rows_y, (size_t)c->n_heads * c->rows_y_stride)) != hipSuccess) return bail(e, "hipMalloc(rows)");
      if ((e = hipMemset(c->rows_y, 0, (size_t)c->n_heads * c->rows_y_stride * sizeof(frag_t))) != hipSuccess) return bail(e, "memset rows");
      if ((e = dev_alloc(c, &c->rows_part4, (size_t)2 * c->rows_grid * rmax)) != hipSuccess) return bail(e, "hipMalloc(rows)");
      if ((e = dev_alloc(c, &c->rows_parti, (size_t)2 * c->rows_grid * rmax)) != hipSuccess) return bail(e, "hipMalloc(rows)");
      if ((e = dev_alloc(c, &c->rows_ctl, (size_t)c->rows_ctl_ints)) != hipSuccess) return bail(e, "hipMalloc(rows)");
      c->rows_vctl_ints = rows_control_ints(1);
      if ((e = dev_alloc(c, &c->rows_vctl, (size_t)2 * c->rows_vctl_ints)) != hipSuccess) return bail(e, "hipMalloc(rows)");
      if ((e = hipMemset(c->rows_vctl, 0, (size_t)2 * c->rows_vctl_ints * sizeof(int))) != hipSuccess) return bail(e, "memset rows");
    } else {
      c->rows_grid = 0;
    }
    {
      hipDeviceProp_t prop;
      if ((e = hipGetDeviceProperties(&prop, c->device)) != hipSuccess) return bail(e, "device properties");
      c->num_cu = prop.multiProcessorCount;
    }
    if (c->decode_grid > 0) {
      const size_t nrec = 2 * np * c->decode_grid * 16 * 5;
      if ((e = dev_alloc(c, &c->dec_records, nrec)) != hipSuccess) return bail(e, "hipMalloc(decode)");
      if ((e = hipMemset(c->dec_records, 0, nrec * sizeof(unsigned long long))) != hipSuccess) return bail(e, "memset");
      if ((e = dev_alloc(c, &c->dec_trace, np * 16 + 4 * (size_t)c->decode_grid)) != hipSuccess) return bail(e, "hipMalloc(decode)");
      if ((e = hipMemset(c->dec_trace, 0, (np * 16 + 4 * (size_t)c->decode_grid) * sizeof(unsigned long long))) != hipSuccess) return bail(e, "memset");
    }
  }
  if ((e = hipDeviceSynchronize()) != hipSuccess) return bail(e, "eh_create sync");
  *out = c;
  return EH_OK;
}

eh_status eh_destroy(eh_ctx* ctx) {
  if (!ctx) return EH_ERR_NULL;
  DeviceGuard guard(ctx->device);
  (void)hipDeviceSynchronize();
  free_all(ctx);
  delete ctx;
  return EH_OK;
}

eh_status eh_eval(eh_ctx* ctx, int32_t head, const void* h, int64_t h_row_stride,
                  const int32_t* row_idx, const int32_t* n_rows_dev, int32_t n_rows, float* H,
                  float* lse, int32_t* argmax, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (head < 0 || head >= ctx->n_heads) return fail(ctx, EH_ERR_RANGE, "head out of range");
  if (n_rows == 0) return EH_OK;
  if (!h) return fail(ctx, EH_ERR_NULL, "h is NULL");
  eh_status st = check_rows(ctx, h, h_row_stride, n_rows);
  if (st != EH_OK) return st;
  DeviceGuard guard(ctx->device);
  if (use_decode(ctx, n_rows)) {
    DecodeParams p = decode_base(ctx);
    p.h = h; p.layer_stride = 0; p.row_stride = h_row_stride; p.row_idx = row_idx;
    p.n_rows_dev = n_rows_dev; p.n_rows = n_rows; p.l0 = 0; p.l1 = 1; p.decide = 0;
    // evaluation mode addresses one head: shift the tables instead of the layer stride
    p.Wf += head; p.gamma += head; p.beta += head; if (p.bias) p.bias += head;
    p.records += (size_t)head * ctx->decode_grid * 16 * 5;
    p.H = H; p.lse = lse; p.argmax = argmax;
    EH_HIP(ctx, decode_launch(ctx, p, (hipStream_t)stream));
    return EH_OK;
  }
  return run_head<false>(ctx, head, h, h_row_stride, row_idx, n_rows_dev, n_rows, H, lse, argmax,
                         (hipStream_t)stream);
}

eh_status eh_eval_noalloc(eh_ctx* ctx, int32_t head, const void* h, int64_t h_row_stride,
                          const int32_t* row_idx, const int32_t* n_rows_dev, int32_t n_rows, float* H,
                          float* lse, int32_t* argmax, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (head < 0 || head >= ctx->n_heads) return fail(ctx, EH_ERR_RANGE, "head out of range");
  if (n_rows < 0) return fail(ctx, EH_ERR_SHAPE, "n_rows is negative");
  if (n_rows == 0) return EH_OK;
  if (!h) return fail(ctx, EH_ERR_NULL, "h is NULL");
  if (h_row_stride < ctx->d) return fail(ctx, EH_ERR_SHAPE, "row stride smaller than d");
  const int esz = ctx->dtype == EH_BF16 ? 2 : 4;
  if (!aligned16(h) || (h_row_stride * esz) % 16 != 0)
    return fail(ctx, EH_ERR_SHAPE, "hidden rows must be 16-byte aligned");
  // layout of the static array for this call: activations of the rows (padded to blocks of 32,
  // plus the 32 blocks of 16 the batched kernels may read beyond them), then one partial
  // statistics record per (workgroup, row)
  const size_t R_pad = ((size_t)n_rows + 31) & ~(size_t)31;
  const size_t y_bytes = (R_pad / 16 + 32) * (size_t)ctx->KS * kWave * sizeof(frag_t);
  const size_t part_off = (y_bytes + 255) & ~(size_t)255;
  const size_t need = part_off + (size_t)kMaxParts * R_pad * sizeof(Stats);
  if ((size_t)n_rows > ((size_t)1 << 20) || need > kNoAllocScratchBytes)
    return fail(ctx, EH_ERR_WORKSPACE,
                "n_rows rows of d elements need " + std::to_string(need) + " bytes of workspace; the static one holds " +
                    std::to_string(kNoAllocScratchBytes));
  if (!ctx->static_scratch) return fail(ctx, EH_ERR_HIP, "the static workspace has no device address");
  DeviceGuard guard(ctx->device);
  unsigned char* base = (unsigned char*)ctx->static_scratch;
  return run_head<false>(ctx, head, h, h_row_stride, row_idx, n_rows_dev, n_rows, H, lse, argmax,
                         (hipStream_t)stream, (frag_t*)base, (Stats*)(base + part_off));
}

namespace {

// eh_eval_heads and eh_eval_heads_metrics.  `metrics`: also the maximum probability and the
// difference of the two largest probabilities (either output may be NULL).
// The many-heads workspace: per head, activations for max_rows rows (plus the zero blocks the
// batched kernel may read past them), one set of partial statistics and one of second largest
// logits.  Grow-only, kept by the context; the old one may still be in use on a stream.
eh_status ensure_mh(eh_ctx* ctx, int n_heads_needed) {
  if (ctx->mh_heads >= n_heads_needed) return EH_OK;
  const size_t y_stride = (size_t)(ctx->R_pad_max / 16 + 32) * ctx->KS * kWave;
  const size_t part_stride = (size_t)kMaxParts * ctx->R_pad_max;
  EH_HIP(ctx, hipDeviceSynchronize());
  eh::frag_t* y = nullptr;
  eh::Stats* pt = nullptr;
  float* sec = nullptr;
  hipError_t e = dev_alloc(ctx, &y, y_stride * n_heads_needed);
  if (e == hipSuccess) e = dev_alloc(ctx, &pt, part_stride * n_heads_needed);
  if (e == hipSuccess) e = dev_alloc(ctx, &sec, part_stride * n_heads_needed);
  if (e == hipSuccess) e = hipMemset(y, 0, y_stride * n_heads_needed * sizeof(frag_t));
  EH_HIP(ctx, e);
  ctx->mh_yf = y;
  ctx->mh_partials = pt;
  ctx->mh_second = sec;
  ctx->mh_heads = n_heads_needed;
  return EH_OK;
}

eh_status eval_heads_impl(eh_ctx* ctx, int32_t head0, int32_t n_heads_eval, const void* h_layers,
                          int64_t layer_stride, int64_t row_stride, int32_t n_rows, float* H, float* lse,
                          int32_t* argmax, bool metrics, float* max_prob, float* margin, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (n_heads_eval < 0 || head0 < 0 || head0 + n_heads_eval > ctx->n_heads)
    return fail(ctx, EH_ERR_RANGE, "heads out of range");
  if (metrics && (ctx->dtype != EH_BF16 || !ctx->bias.empty()))
    return fail(ctx, EH_ERR_DTYPE, "the extra confidence metrics need bf16 heads without a bias vector");
  if (n_rows == 0 || n_heads_eval == 0) return EH_OK;
  if (!h_layers) return fail(ctx, EH_ERR_NULL, "h_layers is NULL");
  eh_status st = check_rows(ctx, h_layers, row_stride, n_rows);
  if (st != EH_OK) return st;
  const int esz = ctx->dtype == EH_BF16 ? 2 : 4;
  if ((layer_stride * esz) % 16 != 0) return fail(ctx, EH_ERR_SHAPE, "hidden rows must be 16-byte aligned");
  hipStream_t s = (hipStream_t)stream;
  const bool batched =
      ctx->dtype == EH_BF16 && ctx->bias.empty() && (n_rows > 16 || metrics);
  if (!batched) {
    // shapes the many-heads kernels do not cover: one head after the other
    for (int l = 0; l < n_heads_eval; ++l) {
      st = eh_eval(ctx, head0 + l, (const char*)h_layers + (int64_t)l * layer_stride * esz, row_stride,
                   nullptr, nullptr, n_rows, H ? H + (int64_t)l * n_rows : nullptr,
                   lse ? lse + (int64_t)l * n_rows : nullptr,
                   argmax ? argmax + (int64_t)l * n_rows : nullptr, stream);
      if (st != EH_OK) return st;
    }
    return EH_OK;
  }
  DeviceGuard guard(ctx->device);
  // per head: activations for max_rows rows (plus the zero blocks the kernel may read past
  // them), one set of partial statistics and one of second largest logits
  const size_t y_stride = (size_t)(ctx->R_pad_max / 16 + 32) * ctx->KS * kWave;
  const size_t part_stride = (size_t)kMaxParts * ctx->R_pad_max;
  st = ensure_mh(ctx, n_heads_eval);
  if (st != EH_OK) return st;
  const int R_pad = (n_rows + 31) & ~31;
  const float* const* gamma_tab = (const float* const*)(ctx->d_gamma + head0);
  const float* const* beta_tab = (const float* const*)(ctx->d_beta + head0);
  if (ctx->KS * 4 <= kLnCache * kWave && (int64_t)R_pad * n_heads_eval >= kLnMany)
    hipLaunchKernelGGL((ln_pack_many_kernel<DtBf16>), dim3(R_pad / kLnTeam, n_heads_eval), dim3(kLnTeam * kWave),
                       (size_t)ctx->KS * 4 * kLnTeam * sizeof(frag_t), s, h_layers, layer_stride, row_stride, n_rows, ctx->d,
                       ctx->KS, gamma_tab, beta_tab, ctx->eps, ctx->mh_yf, (int64_t)y_stride);
  else
    hipLaunchKernelGGL((ln_pack_heads_kernel<DtBf16, 32>), dim3(R_pad, n_heads_eval), dim3(kLnThreads), 0, s, h_layers,
                       layer_stride, row_stride, n_rows, R_pad, ctx->d, ctx->KS, gamma_tab, beta_tab, ctx->eps, ctx->mh_yf,
                       (int64_t)y_stride);
  PartCount parts{0, 0, 0, 0, 0};
  float* second = metrics ? ctx->mh_second : nullptr;
  if (use_ksplit(ctx, n_rows))
    EH_HIP(ctx, ksplit_launch(ctx, head0, n_heads_eval, nullptr, n_rows, false, ctx->mh_yf, (long long)y_stride,
                              ctx->mh_partials, second, (long long)part_stride, &parts, s));
  else
    EH_HIP(ctx, gemm32_launch(ctx, head0, n_heads_eval, n_heads_eval, nullptr, n_rows, false, ctx->mh_yf, (long long)y_stride,
                              ctx->mh_partials, second, (long long)part_stride, &parts, s));
  if (metrics) {
#define EH_FINM(FR)                                                                                                      \
  hipLaunchKernelGGL((finalize_metrics_kernel<FR>), dim3((n_rows + FR - 1) / FR, n_heads_eval), dim3(kFinThreads), 0, s, \
                     ctx->mh_partials, ctx->mh_second, parts.n, R_pad, n_rows, H, lse, argmax, max_prob, margin,         \
                     (int64_t)part_stride, (int64_t)n_rows)
    if (fin_rows(n_rows) == 4) EH_FINM(4);
    else EH_FINM(16);
#undef EH_FINM
  } else {
    launch_finalize(ctx->mh_partials, parts, R_pad, nullptr, n_rows, n_heads_eval, H, lse, argmax, (int64_t)part_stride, s);
  }
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

}  // namespace

eh_status eh_eval_heads(eh_ctx* ctx, int32_t head0, int32_t n_heads_eval, const void* h_layers,
                        int64_t layer_stride, int64_t row_stride, int32_t n_rows, float* H, float* lse,
                        int32_t* argmax, void* stream) {
  return eval_heads_impl(ctx, head0, n_heads_eval, h_layers, layer_stride, row_stride, n_rows, H, lse, argmax,
                         false, nullptr, nullptr, stream);
}

eh_status eh_eval_heads_metrics(eh_ctx* ctx, int32_t head0, int32_t n_heads_eval, const void* h_layers,
                                int64_t layer_stride, int64_t row_stride, int32_t n_rows, float* H, float* lse,
                                int32_t* argmax, float* max_prob, float* margin, void* stream) {
  return eval_heads_impl(ctx, head0, n_heads_eval, h_layers, layer_stride, row_stride, n_rows, H, lse, argmax,
                         true, max_prob, margin, stream);
}

eh_status eh_exit_decide(eh_ctx* ctx, int32_t head, const float* H, const int32_t* argmax,
                         const int32_t* row_idx, const int32_t* n_rows_dev, int32_t n_rows,
                         int32_t* exit_layer, int32_t* token, int32_t* active_idx_out,
                         int32_t* n_active_out, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (head < 0 || head >= ctx->n_heads) return fail(ctx, EH_ERR_RANGE, "head out of range");
  if (n_rows < 0 || n_rows > ctx->max_rows) return fail(ctx, EH_ERR_WORKSPACE, "n_rows outside [0, max_rows]");
  if (!H || !argmax || !exit_layer || !token || !active_idx_out || !n_active_out)
    return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  if (active_idx_out == row_idx) return fail(ctx, EH_ERR_RANGE, "active_idx_out must not alias row_idx");
  DeviceGuard guard(ctx->device);
  const float tau = ctx->tau[head];
  hipLaunchKernelGGL(decide_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, H, argmax, row_idx,
                     n_rows_dev, n_rows, tau, head == ctx->n_heads - 1 ? 1 : 0, head, exit_layer, token,
                     active_idx_out, n_active_out, (float*)nullptr, (unsigned long long*)nullptr);
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status eh_cascade(eh_ctx* ctx, const void* h_layers, int64_t layer_stride, int64_t row_stride,
                     int32_t n_rows, int32_t* exit_layer, int32_t* token, float* H_out,
                     int64_t* n_evals_out, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (n_rows == 0) return EH_OK;
  if (!h_layers || !exit_layer || !token) return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  eh_status st = check_rows(ctx, h_layers, row_stride, n_rows);
  if (st != EH_OK) return st;
  const int esz = ctx->dtype == EH_BF16 ? 2 : 4;
  if (ctx->n_heads > 1 && (layer_stride * esz) % 16 != 0)
    return fail(ctx, EH_ERR_SHAPE, "layer stride must keep rows 16-byte aligned");
  DeviceGuard guard(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  if (use_decode(ctx, n_rows)) {
    DecodeParams p = decode_base(ctx);
    p.h = h_layers; p.layer_stride = layer_stride; p.row_stride = row_stride;
    p.n_rows = n_rows; p.l0 = 0; p.l1 = ctx->n_heads; p.decide = 1;
    p.exit_layer = exit_layer; p.token = token; p.H_out = H_out;
    p.n_evals = (unsigned long long*)n_evals_out;
    EH_HIP(ctx, decode_launch(ctx, p, s));
    return EH_OK;
  }
  if (use_rows(ctx, n_rows, false)) {
    // one persistent launch for the whole cascade
    RowsParams p = rows_base(ctx, n_rows);
    p.h = h_layers; p.layer_stride = layer_stride; p.row_stride = row_stride;
    p.l0 = 0; p.l1 = ctx->n_heads; p.mode = 0; p.argmax_only = 0;
    p.exit_layer = exit_layer; p.token = token; p.H_out = H_out;
    p.n_evals = (unsigned long long*)n_evals_out;
    EH_HIP(ctx, rows_launch(ctx, p, s));
    return EH_OK;
  }
  // Two launches per head: the batched projection, then one kernel that merges the partial
  // statistics, applies the exit rule, appends the rows that go on to the next head's list
  // and writes their LayerNorm for the next head.  Three live-row counters rotate: head l
  // reads counter l%3, fills (l+1)%3 and clears (l+2)%3.
  const int RB = row_block(ctx, n_rows);
  const int R_pad = round_up(n_rows, RB);
  int* cnt = ctx->n_active[0];
#define EH_INIT(DT, RBV)                                                                                               \
  hipLaunchKernelGGL((cascade_init_kernel<DT, RBV>), dim3(R_pad), dim3(kLnThreads), 0, s, h_layers, row_stride, n_rows, \
                     R_pad, ctx->d, ctx->KS, ctx->gamma[0], ctx->beta[0], ctx->eps, ctx->yf, cnt, 3, H_out,             \
                     (int64_t)ctx->n_heads * n_rows)
  if (ctx->dtype == EH_BF16) EH_INIT(DtBf16, 32);
  else if (RB == 32) EH_INIT(DtF32, 32);
  else EH_INIT(DtF32, 16);
#undef EH_INIT
  for (int l = 0; l < ctx->n_heads; ++l) {
    const int last = l == ctx->n_heads - 1 ? 1 : 0;
    const int* idx = l == 0 ? nullptr : ctx->active[l & 1];
    const int* live = l == 0 ? nullptr : cnt + l % 3;
    PartCount parts;
    EH_HIP(ctx, project(ctx, l, ctx->n_heads, live, n_rows, false, ctx->yf, ctx->partials, &parts, s));
    const void* hn = last ? nullptr : (const char*)h_layers + (int64_t)(l + 1) * layer_stride * esz;
    const float* gn = last ? nullptr : ctx->gamma[l + 1];
    const float* bn = last ? nullptr : ctx->beta[l + 1];
    float* Hl = H_out ? H_out + (int64_t)l * n_rows : nullptr;
#define EH_POST(DT, RBV)                                                                              \
  hipLaunchKernelGGL((cascade_post_kernel<DT, RBV>), dim3(round_up(n_rows, kPostDies)), dim3(kLnThreads), 0, s, ctx->partials, parts, \
                     R_pad, idx, live, n_rows, ctx->tau[l], last, l, exit_layer, token, Hl,            \
                     (unsigned long long*)n_evals_out, ctx->active[(l + 1) & 1], cnt + (l + 1) % 3,    \
                     cnt + (l + 2) % 3, hn, row_stride, ctx->d, ctx->KS, gn, bn, ctx->eps, ctx->yf)
    if (ctx->dtype == EH_BF16) EH_POST(DtBf16, 32);
    else if (RB == 32) EH_POST(DtF32, 32);
    else EH_POST(DtF32, 16);
#undef EH_POST
  }
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status dssd_verify(eh_ctx* ctx, const void* f_final, const int32_t* draft, const int32_t* draft_len,
                      int32_t B, int32_t k, int32_t* accepted, int32_t* next_token, int32_t* target,
                      void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (B < 0 || k < 0) return fail(ctx, EH_ERR_SHAPE, "B and k must be non-negative");
  if (B == 0) return EH_OK;
  if (!f_final || !accepted || !next_token || (k > 0 && !draft))
    return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  const int64_t rows = (int64_t)B * (k + 1);
  if (rows > ctx->max_rows) return fail(ctx, EH_ERR_WORKSPACE, "B*(k+1) exceeds max_rows");
  eh_status st = check_rows(ctx, f_final, ctx->d, (int)rows);
  if (st != EH_OK) return st;
  DeviceGuard guard(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  if (use_rows(ctx, rows, true)) {
    // one persistent launch: LayerNorm, argmax-only projection, merge and prefix walk
    RowsParams p = rows_base(ctx, (int)rows);
    p.h = f_final; p.layer_stride = 0; p.row_stride = ctx->d;
    p.l0 = ctx->n_heads - 1; p.l1 = ctx->n_heads; p.mode = 1; p.argmax_only = 1;
    p.n_stream = ctx->rows_grid;  // a verification has no serving workgroups: all stream, then all merge
    // no preset launch in front of a verification: it runs on one of two control blocks in turn and
    // clears the other for the call after it (calls on a context are serialised)
    p.ctl = ctx->rows_vctl + (size_t)(ctx->rows_vturn & 1u) * ctx->rows_vctl_ints;
    p.ctl_next = ctx->rows_vctl + (size_t)((ctx->rows_vturn + 1u) & 1u) * ctx->rows_vctl_ints;
    p.n_ctl_next = ctx->rows_vctl_ints;
    ++ctx->rows_vturn;
    p.draft = draft; p.draft_len = draft_len; p.B = B; p.k = k;
    p.accepted = accepted; p.next_token = next_token; p.target = target;
    EH_HIP(ctx, rows_launch(ctx, p, s));
    return EH_OK;
  }
  if ((size_t)(k + 1) * sizeof(int) <= 48 * 1024) {
    // three launches: LayerNorm, argmax-only projection, then one kernel that merges the
    // partial argmaxes of a row's k+1 positions and walks the prefix
    const int R_pad = round_up((int)rows, row_block(ctx, (int)rows));
    const int fin = ctx->n_heads - 1;
    launch_ln(ctx, fin, f_final, ctx->d, nullptr, nullptr, (int)rows, R_pad, ctx->yf, s);
    PartCount parts;
    EH_HIP(ctx, project(ctx, fin, 1, nullptr, (int)rows, true, ctx->yf, ctx->partials, &parts, s));
    hipLaunchKernelGGL(verify_post_kernel, dim3(B), dim3(kWave * verify_waves(parts.n, k)), (size_t)(k + 1) * sizeof(int), s, ctx->partials,
                       parts.n, R_pad, draft, draft_len, k, target, accepted, next_token);
    EH_HIP(ctx, hipGetLastError());
    return EH_OK;
  }
  int* tgt = target ? target : ctx->ws_argmax;
  st = run_head<true>(ctx, ctx->n_heads - 1, f_final, ctx->d, nullptr, nullptr, (int)rows, nullptr,
                      nullptr, tgt, s);
  if (st != EH_OK) return st;
  hipLaunchKernelGGL(verify_compare_kernel, dim3((B + 63) / 64), dim3(64), 0, s, draft, draft_len, tgt, B,
                     k, accepted, next_token);
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status dssd_draft(eh_ctx* ctx, const void* h_positions, int64_t pos_stride, int64_t layer_stride,
                     int32_t n_positions, int32_t limit, int32_t eos_token, int32_t* draft, int32_t* draft_len,
                     int32_t* exit_layers, int32_t* stop_reason, int32_t* fallback_token, int64_t* n_evals_out,
                     void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (limit < 0 || n_positions < 0) return fail(ctx, EH_ERR_SHAPE, "limit and n_positions must be non-negative");
  if (!draft_len || (limit > 0 && (!draft || !exit_layers))) return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  if (n_positions > 0 && limit > 0 && !h_positions) return fail(ctx, EH_ERR_NULL, "h_positions is NULL");
  const bool by_rows = ctx->decode_grid <= 0 && use_rows(ctx, 1, false);  // hidden sizes above the decode kernel's
  if (ctx->decode_grid <= 0 && !by_rows)
    return fail(ctx, EH_ERR_DTYPE, "drafting needs a single-launch cascade kernel (bf16 or fp32 heads without a bias "
                                   "vector; fp32 up to d = 1024)");
  if (ctx->n_heads < 2) return fail(ctx, EH_ERR_RANGE, "drafting needs at least one exit head besides the model's");
  const int esz = ctx->dtype == EH_BF16 ? 2 : 4;
  const int steps = n_positions < limit ? n_positions : limit;
  if (steps > 0) {
    eh_status st = check_rows(ctx, h_positions, ctx->d, 1);
    if (st != EH_OK) return st;
    if ((layer_stride * esz) % 16 != 0 || (pos_stride * esz) % 16 != 0)
      return fail(ctx, EH_ERR_SHAPE, "strides must keep rows 16-byte aligned");
  }
  DeviceGuard guard(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  int* state = ctx->n_active[1];     // {live, length, reason, fallback token}
  int* ex = ctx->active[0];          // the current position's exit layer and token
  int* tk = ctx->active[1];
  hipLaunchKernelGGL(draft_init_kernel, dim3(1), dim3(64), 0, s, state, limit, exit_layers);
  for (int t = 0; t < steps && by_rows; ++t) {
    RowsParams p = rows_base(ctx, 1);
    p.h = (const char*)h_positions + (int64_t)t * pos_stride * esz;
    p.layer_stride = layer_stride;
    p.row_stride = ctx->d;
    p.l0 = 0; p.l1 = ctx->n_heads; p.mode = 0; p.argmax_only = 0;
    p.live = state;  // 1 while drafting, 0 once it has stopped: both launches then return at once
    p.exit_layer = ex; p.token = tk; p.H_out = nullptr;
    p.n_evals = (unsigned long long*)n_evals_out;
    EH_HIP(ctx, rows_launch(ctx, p, s));
    hipLaunchKernelGGL(draft_step_kernel, dim3(1), dim3(1), 0, s, state, ex, tk, ctx->n_heads - 1, limit, eos_token,
                       draft, exit_layers);
  }
  for (int t = 0; t < steps && !by_rows; ++t) {
    DecodeParams p = decode_base(ctx);
    p.h = (const char*)h_positions + (int64_t)t * pos_stride * esz;
    p.layer_stride = layer_stride;
    p.row_stride = ctx->d;
    p.n_rows = 1;
    p.n_rows_dev = state;  // 1 while drafting, 0 once it has stopped: the launch then returns at once
    p.l0 = 0;
    p.l1 = ctx->n_heads;
    p.decide = 1;
    p.exit_layer = ex;
    p.token = tk;
    p.H_out = nullptr;
    p.n_evals = (unsigned long long*)n_evals_out;
    EH_HIP(ctx, decode_launch(ctx, p, s));
    hipLaunchKernelGGL(draft_step_kernel, dim3(1), dim3(1), 0, s, state, ex, tk, ctx->n_heads - 1, limit, eos_token,
                       draft, exit_layers);
  }
  hipLaunchKernelGGL(draft_finish_kernel, dim3(1), dim3(1), 0, s, state, draft_len, stop_reason, fallback_token);
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status dssd_tally(eh_ctx* ctx, const int32_t* draft_len, const int32_t* accepted, int32_t B, int32_t k,
                     const int32_t* exit_layers, int64_t* counters, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (B < 0 || k < 0) return fail(ctx, EH_ERR_SHAPE, "B and k must be non-negative");
  if (!counters || (B > 0 && !accepted)) return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  if (B == 0) return EH_OK;
  DeviceGuard guard(ctx->device);
  hipLaunchKernelGGL(tally_kernel, dim3(1), dim3(256), 0, (hipStream_t)stream, draft_len, accepted, B, k, exit_layers,
                     (unsigned long long*)counters);
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status eh_head_losses(eh_ctx* ctx, int32_t head, const void* h_head, int64_t row_stride_head,
                         const void* h_model, int64_t row_stride_model, const int32_t* labels, int32_t n_rows,
                         float alpha, float* kl, float* ce, float* loss, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (head < 0 || head >= ctx->n_heads) return fail(ctx, EH_ERR_RANGE, "head out of range");
  if (ctx->dtype != EH_BF16 || !ctx->bias.empty())
    return fail(ctx, EH_ERR_DTYPE, "the fused objectives need bf16 heads without a bias vector");
  if (n_rows <= 0) return fail(ctx, EH_ERR_SHAPE, "the mean over an empty sequence is undefined");
  if (!h_head || !h_model || !loss) return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  eh_status st = check_rows(ctx, h_head, row_stride_head, n_rows);
  if (st == EH_OK) st = check_rows(ctx, h_model, row_stride_model, n_rows);
  if (st != EH_OK) return st;
  DeviceGuard guard(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  st = ensure_mh(ctx, 2);
  if (st != EH_OK) return st;
  if (!ctx->kl_partials) {
    EH_HIP(ctx, dev_alloc(ctx, &ctx->kl_partials, (size_t)kMaxParts * ctx->R_pad_max));
    EH_HIP(ctx, dev_alloc(ctx, &ctx->kl_rows, (size_t)2 * ctx->R_pad_max));
  }
  const size_t y_stride = (size_t)(ctx->R_pad_max / 16 + 32) * ctx->KS * kWave;
  const int R_pad = (n_rows + 31) & ~31;
  const int fin = ctx->n_heads - 1;
  const LnRows exit_rows{h_head, row_stride_head, ctx->gamma[head], ctx->beta[head]};
  const LnRows model_rows{h_model, row_stride_model, ctx->gamma[fin], ctx->beta[fin]};
  hipLaunchKernelGGL((ln_pack_pair_kernel<DtBf16, 32>), dim3(R_pad, 2), dim3(kLnThreads), 0, s, exit_rows, model_rows, n_rows, R_pad,
                     ctx->d, ctx->KS, ctx->eps, ctx->mh_yf, (int64_t)y_stride);
  int n_parts = 0;
  EH_HIP(ctx, gemm32_kl_launch(ctx, head, fin, n_rows, ctx->mh_yf, ctx->mh_yf + y_stride, labels, ctx->kl_partials,
                               &n_parts, s));
  hipLaunchKernelGGL(kl_finalize_kernel, dim3(n_rows), dim3(64), 0, s, ctx->kl_partials, n_parts, R_pad, n_rows,
                     ctx->V, ctx->kl_rows, kl, ce);
  hipLaunchKernelGGL(kl_mean_kernel, dim3(1), dim3(256), 0, s, ctx->kl_rows, R_pad, n_rows, alpha, loss);
  EH_HIP(ctx, hipGetLastError());
  return EH_OK;
}

eh_status eh_calibrate(eh_ctx* ctx, const float* H, const int32_t* pred, const int32_t* ref, int64_t M,
                       const double* eps, int32_t n_eps, float* tau_out, int64_t* n_exit_out, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  if (n_eps < 0 || n_eps > 64) return fail(ctx, EH_ERR_RANGE, "n_eps outside [0, 64]");
  if (M < 0 || M >= ((int64_t)1 << 31)) return fail(ctx, EH_ERR_SHAPE, "M outside [0, 2^31)");
  if (n_eps == 0) return EH_OK;
  if (!eps || !tau_out || (M > 0 && (!H || !pred || !ref))) return fail(ctx, EH_ERR_NULL, "a required pointer is NULL");
  for (int i = 0; i < n_eps; ++i)
    if (!(eps[i] >= 0.0 && eps[i] <= 1.0)) return fail(ctx, EH_ERR_RANGE, "epsilon outside [0, 1]");
  DeviceGuard guard(ctx->device);
  hipStream_t s = (hipStream_t)stream;
  if (M == 0) {
    hipLaunchKernelGGL(fill_f32_kernel, dim3(1), dim3(64), 0, s, tau_out, (int64_t)n_eps, -INFINITY);
    if (n_exit_out)
      hipLaunchKernelGGL(fill_i32_kernel, dim3(1), dim3(128), 0, s, (int*)n_exit_out, (int64_t)2 * n_eps, 0);
    EH_HIP(ctx, hipGetLastError());
    return EH_OK;
  }
  EH_HIP(ctx, calibrate_run(ctx->calib, H, pred, ref, M, eps, n_eps, tau_out, (long long*)n_exit_out, s));
  return EH_OK;
}

#ifdef EH_DIAGNOSTICS
// Diagnostics build: the 128 time-stamp words the last rows-kernel launch over n_heads heads left.
extern "C" eh_status eh_rows_trace(eh_ctx* ctx, int32_t n_heads, int32_t* host_out) {
  if (!ctx || !ctx->rows_ctl || !host_out) return EH_ERR_NULL;
  DeviceGuard guard(ctx->device);
  EH_HIP(ctx, hipDeviceSynchronize());
  const int* from = n_heads == 1 && ctx->rows_vturn > 0
                        ? ctx->rows_vctl + (size_t)((ctx->rows_vturn - 1u) & 1u) * ctx->rows_vctl_ints + ctx->rows_vctl_ints - 128
                        : ctx->rows_ctl + rows_control_ints(n_heads) - 128;
  EH_HIP(ctx, hipMemcpy(host_out, from, 128 * sizeof(int), hipMemcpyDeviceToHost));
  return EH_OK;
}
eh_status eh_decode_trace(eh_ctx* ctx, int32_t enable, uint64_t* host_out, int32_t n) {
  if (!ctx) return EH_ERR_NULL;
  if (!ctx->dec_trace) return fail(ctx, EH_ERR_RANGE, "this context has no decode kernel");
  DeviceGuard guard(ctx->device);
  if (host_out) {
    if (n < 0 || n > ctx->n_heads * 16 + 4 * ctx->decode_grid)
      return fail(ctx, EH_ERR_RANGE, "n outside [0, 16 * n_heads + 4 * workgroups]");
    EH_HIP(ctx, hipDeviceSynchronize());
    EH_HIP(ctx, hipMemcpy(host_out, ctx->dec_trace, sizeof(uint64_t) * n, hipMemcpyDeviceToHost));
  }
  ctx->dec_trace_on = enable ? 1 : 0;
  return EH_OK;
}
#endif

eh_status eh_check(eh_ctx* ctx, void* stream) {
  if (!ctx) return EH_ERR_NULL;
  DeviceGuard guard(ctx->device);
  EH_HIP(ctx, hipStreamSynchronize((hipStream_t)stream));
  if (ctx->dec_status) {
    int flag = 0;
    EH_HIP(ctx, hipMemcpy(&flag, ctx->dec_status, sizeof(int), hipMemcpyDeviceToHost));
    if (flag != 0) {
      // report once and re-arm: the failed call's unfinished rows hold -1 / NaN
      EH_HIP(ctx, hipMemset(ctx->dec_status, 0, sizeof(int)));
      if (ctx->rows_vctl) EH_HIP(ctx, hipMemset(ctx->rows_vctl, 0, (size_t)2 * ctx->rows_vctl_ints * sizeof(int)));
      return fail(ctx, EH_ERR_HIP,
                  "the persistent kernel gave up waiting for another workgroup: the stream did not have the "
                  "device to itself (rows it did not finish hold -1 / NaN)");
    }
  }
  return EH_OK;
}

eh_status eh_set_spin_limit(eh_ctx* ctx, int32_t polls) {
  if (!ctx) return EH_ERR_NULL;
  if (polls < 0) return fail(ctx, EH_ERR_RANGE, "polls must be non-negative");
  ctx->spin_limit = polls;
  return EH_OK;
}

}  // extern "C"
