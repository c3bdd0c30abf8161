// Host side of the stress-surrogate C ABI (include/rsur.h): memory layout, marshalling of the
// flat parameter layout to the padded device layout, and the launch sequence of inference and
// of one training step.  The arithmetic runs in the kernels of rsur_device.h.
#include <hip/hip_runtime.h>
#include <rocprofiler-sdk-roctx/roctx.h>

#include <algorithm>
#include <cmath>
#include <cstring>
#include <mutex>
#include <string>
#include <vector>

#include "../../include/rcell.h"
#include "../../include/rsur.h"
#include "rsur_device.h"

using namespace rsur;

namespace {
thread_local std::string g_rsur_create_error;

// A roctx range over a scope (rocprofv3 --marker-trace names each call; a few ns without a profiler)
struct TraceRange {
  explicit TraceRange(const char* name) { roctxRangePush(name); }
  ~TraceRange() { roctxRangePop(); }
  TraceRange(const TraceRange&) = delete;
  TraceRange& operator=(const TraceRange&) = delete;
};
}

// Scratch of rsur_forward_static: every member's output for the rows of one call (K x pad64(B) x
// padded dout floats).  One copy per device, holding the last call's outputs until the process
// ends.  Host code never uses this name as an address: the device address of each device's copy
// comes from hipGetSymbolAddress (static_scratch_ptr).
constexpr long long RSUR_STATIC_FLOATS = 1LL << 21;   // 8 MiB
static __device__ __align__(256) float scratch[RSUR_STATIC_FLOATS];

namespace {
constexpr int MAX_DEVICES = 64;
std::mutex g_scratch_mu;
float* g_scratch_ptr[MAX_DEVICES] = {};

// device address of the current device's scratch, looked up once per device (no allocation)
int static_scratch_ptr(float** out) {
  int dev = 0;
  if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
    (void)hipGetLastError();
    return RCELL_ERR_DEVICE;
  }
  std::lock_guard<std::mutex> lock(g_scratch_mu);
  if (!g_scratch_ptr[dev]) {
    void* q = nullptr;
    if (hipGetSymbolAddress(&q, HIP_SYMBOL(scratch)) != hipSuccess || !q) {
      (void)hipGetLastError();
      return RCELL_ERR_DEVICE;
    }
    g_scratch_ptr[dev] = (float*)q;
  }
  *out = g_scratch_ptr[dev];
  return RCELL_OK;
}
}  // namespace

struct rsur_ctx {
  int din = 0, width = 0, depth = 0, dout = 0, K = 0, maxB = 0, Mp = 0, L = 0;
  std::vector<int> dims, dp;                 // logical and padded layer widths (L + 1)
  std::vector<long long> woff, boff;         // offsets of W_l, b_l inside one member's padded block
  long long P = 0, Pflat = 0;                // padded and flat parameter counts per member
  hipStream_t stream = nullptr;
  bool own_stream = false;
  std::string err;
  float *p = nullptr, *g = nullptr, *m1 = nullptr, *m2 = nullptr;   // K x P
  bf16* pb = nullptr;                                               // K x P (weights used)
  bf16 *pbf = nullptr, *pbt = nullptr;                              // K x P, weights by fragments, and transposed
  std::vector<bf16*> act;                    // act[l]: K x Mp x dp[l] (act[0] shared: Mp x dp[0])
  std::vector<float*> Z;                     // Z[l]: K x Mp x dp[l + 1], hidden layers
  float* out = nullptr;                      // K x Mp x dp[L]
  bf16 *dza = nullptr, *dzb = nullptr;       // output gradients layer by layer: K x Mp x max(dp), two in turn (the
                                             // fused pass keeps them in Z and out)
  float *xmu = nullptr, *xsd = nullptr, *ymu = nullptr, *ysd = nullptr, *loss = nullptr;
  int max_split = 0;                         // most ranges of a split gradient reduction; 0: never split
  float* split = nullptr;                    // max_split x K x P: their partial sums
  float* lpart = nullptr;                    // partial losses, up to K x Mp / 32
  std::vector<long long> t;                  // Adam steps per member
  std::vector<void*> allocs;
};

namespace {

int rfail(rsur_ctx* c, int code, const std::string& m) {
  if (c) c->err = m; else g_rsur_create_error = m;
  return code;
}

#define RCHK(ctx, call)                                                                         \
  do {                                                                                          \
    hipError_t e_ = (call);                                                                     \
    if (e_ != hipSuccess)                                                                       \
      return rfail((ctx), RCELL_ERR_DEVICE, std::string(#call) + ": " + hipGetErrorString(e_)); \
  } while (0)

template <class T>
int ralloc(rsur_ctx* c, T** out, size_t count) {
  void* q = nullptr;
  const size_t bytes = std::max<size_t>(count, 1) * sizeof(T);
  if (hipMalloc(&q, bytes) != hipSuccess) {
    (void)hipGetLastError();
    return rfail(c, RCELL_ERR_OOM, "device allocation of " + std::to_string(bytes) + " bytes failed");
  }
  c->allocs.push_back(q);
  *out = (T*)q;
  return RCELL_OK;
}

int pad64(int v) { return (v + 63) / 64 * 64; }

// shapes that the fused inference kernel takes
bool fused_shape(const rsur_ctx* c) {
  return *std::max_element(c->dp.begin(), c->dp.end()) <= FW && c->L <= MAXL;
}

FragMap frag_map(const rsur_ctx* c) {
  FragMap m{};
  if (!fused_shape(c)) return m;
  m.L = c->L;
  for (int l = 0; l <= c->L; ++l) m.dp[l] = c->dp[l];
  for (int l = 0; l < c->L; ++l) m.woff[l] = c->woff[l];
  return m;
}

// The gradient reductions over the batch (weight gradients, bias column sums) are split into S
// ranges of at least 256 rows (S a power of two up to MAX_SPLIT dividing Mp / 64) so that enough
// blocks work at once; S partial results are then added in order (deterministic).
// S is bounded by the memory of the partial results too: a network whose S copies would be larger than
// SPLIT_FLOATS has blocks enough without (64 x 64 weights each).
constexpr int MAX_SPLIT = 8;
constexpr long long SPLIT_FLOATS = 1LL << 26;
int batch_splits(const rsur_ctx* c, int Mp) {
  int S = 1;
  while (2 * S <= c->max_split && (Mp / 64) % (2 * S) == 0 && Mp / (2 * S) >= 256) S *= 2;
  return S;
}

template <bool AT, bool BT, int EPI>
void gemm(rsur_ctx* c, const GemmArgs& a) {
  GemmArgs b = a;
  b.nmem = c->K;
  if (b.ksplit < 1) b.ksplit = 1;
  hipLaunchKernelGGL((k_gemm<AT, BT, EPI>), dim3(b.N / TN, b.M / TM, c->K * b.ksplit), dim3(256), 0, c->stream, b);
}

// forward of every member for Mp rows already normalised in act[0]; keeps Z and activations
void forward_layers(rsur_ctx* c, int Mp) {
  for (int l = 0; l < c->L; ++l) {
    GemmArgs a{};
    a.A = c->act[l];
    a.lda = c->dp[l];
    a.sA = l == 0 ? 0 : (long long)c->Mp * c->dp[l];
    a.B = c->pb + c->woff[l];
    a.ldb = c->dp[l + 1];
    a.sB = c->P;
    a.M = Mp; a.N = c->dp[l + 1]; a.K = c->dp[l];
    a.bias = c->p + c->boff[l];
    a.sBias = c->P;
    if (l < c->L - 1) {
      a.Z = c->Z[l]; a.ldz = c->dp[l + 1]; a.sZ = (long long)c->Mp * c->dp[l + 1];
      a.O = c->act[l + 1]; a.ldo = c->dp[l + 1]; a.sO = (long long)c->Mp * c->dp[l + 1];
      gemm<false, false, EPI_FWD_HIDDEN>(c, a);
    } else {
      a.Z = c->out; a.ldz = c->dp[l + 1]; a.sZ = (long long)c->Mp * c->dp[l + 1];
      gemm<false, false, EPI_FWD_OUT>(c, a);
    }
  }
}

int check_batch(rsur_ctx* c, int B) {
  if (B < 1 || B > c->maxB) return rfail(c, RCELL_ERR_ARG, "batch size must be in [1, max_batch]");
  return RCELL_OK;
}

void normalise_inputs(rsur_ctx* c, const float* X, int B, int Mp) {
  const long long n = (long long)Mp * c->dp[0];
  hipLaunchKernelGGL(k_norm_in, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, X, B, c->din, Mp,
                     c->dp[0], c->xmu, c->xsd, c->act[0]);
}

void destroy_all(rsur_ctx* c) {
  if (c->stream) (void)hipStreamSynchronize(c->stream);
  for (void* q : c->allocs) (void)hipFree(q);
  c->allocs.clear();
  if (c->own_stream && c->stream) (void)hipStreamDestroy(c->stream);
  c->stream = nullptr;
}

}  // namespace

extern "C" {

int rsur_create(int32_t din, int32_t width, int32_t depth, int32_t dout, int32_t ensemble, int32_t max_batch,
                void* hip_stream, rsur_ctx** out) {
  if (!out) return rfail(nullptr, RCELL_ERR_ARG, "out is NULL");
  *out = nullptr;
  if (din < 1 || dout < 1 || depth < 0 || (depth > 0 && width < 1) || ensemble < 1 || max_batch < 1)
    return rfail(nullptr, RCELL_ERR_ARG, "din, dout, ensemble, max_batch >= 1; depth >= 0; width >= 1 with hidden layers");
  rsur_ctx* c = new (std::nothrow) rsur_ctx();
  if (!c) return rfail(nullptr, RCELL_ERR_OOM, "host allocation failed");
  auto bail = [&](int code) {
    g_rsur_create_error = c->err.empty() ? g_rsur_create_error : c->err;
    destroy_all(c);
    delete c;
    return code;
  };
  c->err.reserve(256);             // short error messages are then assigned without allocating
  {
    float* sp = nullptr;             // the static scratch's address on this device, once per device
    if (static_scratch_ptr(&sp) != RCELL_OK)
      return bail(rfail(c, RCELL_ERR_DEVICE, "no usable HIP device (current device, or the static scratch address)"));
  }
  c->din = din; c->width = width; c->depth = depth; c->dout = dout; c->K = ensemble; c->maxB = max_batch;
  c->Mp = pad64(max_batch);
  c->dims.push_back(din);
  for (int k = 0; k < depth; ++k) c->dims.push_back(width);
  c->dims.push_back(dout);
  c->L = (int)c->dims.size() - 1;
  for (int d : c->dims) c->dp.push_back(pad64(d));
  long long o = 0, of = 0;
  for (int l = 0; l < c->L; ++l) {
    c->woff.push_back(o); o += (long long)c->dp[l] * c->dp[l + 1];
    c->boff.push_back(o); o += c->dp[l + 1];
    of += (long long)c->dims[l] * c->dims[l + 1] + c->dims[l + 1];
  }
  c->P = (o + 63) / 64 * 64;
  c->Pflat = of;
  c->t.assign(ensemble, 0);
  if (hip_stream) c->stream = (hipStream_t)hip_stream;
  else {
    if (hipStreamCreateWithFlags(&c->stream, hipStreamNonBlocking) != hipSuccess)
      return bail(rfail(c, RCELL_ERR_DEVICE, "hipStreamCreate failed"));
    c->own_stream = true;
  }
  const long long KP = (long long)c->K * c->P;
  int ms = 1;
  while (2 * ms <= MAX_SPLIT && c->Mp / (2 * ms) >= 256 && 2 * ms * KP <= SPLIT_FLOATS) ms *= 2;
  c->max_split = ms > 1 ? ms : 0;
  int e;
  if ((e = ralloc(c, &c->p, KP)) || (e = ralloc(c, &c->g, KP)) || (e = ralloc(c, &c->m1, KP)) ||
      (e = ralloc(c, &c->m2, KP)) || (e = ralloc(c, &c->pb, KP)) || (e = ralloc(c, &c->pbf, KP)) ||
      (e = ralloc(c, &c->pbt, KP)))
    return bail(e);
  c->act.resize(c->L);
  c->Z.resize(std::max(c->L - 1, 0));
  for (int l = 0; l < c->L; ++l)
    if ((e = ralloc(c, &c->act[l], (size_t)(l == 0 ? 1 : c->K) * c->Mp * c->dp[l]))) return bail(e);
  for (int l = 0; l < c->L - 1; ++l)
    if ((e = ralloc(c, &c->Z[l], (size_t)c->K * c->Mp * c->dp[l + 1]))) return bail(e);
  const int dmax = *std::max_element(c->dp.begin(), c->dp.end());
  if (!fused_shape(c) &&
      ((e = ralloc(c, &c->dza, (size_t)c->K * c->Mp * dmax)) || (e = ralloc(c, &c->dzb, (size_t)c->K * c->Mp * dmax))))
    return bail(e);
  if ((e = ralloc(c, &c->split, (size_t)c->max_split * KP))) return bail(e);
  if ((e = ralloc(c, &c->out, (size_t)c->K * c->Mp * c->dp[c->L])) ||
      (e = ralloc(c, &c->xmu, din)) || (e = ralloc(c, &c->xsd, din)) || (e = ralloc(c, &c->ymu, dout)) ||
      (e = ralloc(c, &c->ysd, dout)) || (e = ralloc(c, &c->loss, ensemble)) || (e = ralloc(c, &c->lpart, (size_t)ensemble * (c->Mp / 32))))
    return bail(e);
  std::vector<float> zeros(std::max(din, dout), 0.0f), ones(std::max(din, dout), 1.0f);
  if (hipMemsetAsync(c->p, 0, sizeof(float) * KP, c->stream) || hipMemsetAsync(c->g, 0, sizeof(float) * KP, c->stream) ||
      hipMemsetAsync(c->m1, 0, sizeof(float) * KP, c->stream) || hipMemsetAsync(c->m2, 0, sizeof(float) * KP, c->stream) ||
      hipMemsetAsync(c->pb, 0, sizeof(bf16) * KP, c->stream) || hipMemsetAsync(c->pbf, 0, sizeof(bf16) * KP, c->stream) ||
      hipMemsetAsync(c->pbt, 0, sizeof(bf16) * KP, c->stream) ||
      hipMemcpyAsync(c->xmu, zeros.data(), sizeof(float) * din, hipMemcpyHostToDevice, c->stream) ||
      hipMemcpyAsync(c->xsd, ones.data(), sizeof(float) * din, hipMemcpyHostToDevice, c->stream) ||
      hipMemcpyAsync(c->ymu, zeros.data(), sizeof(float) * dout, hipMemcpyHostToDevice, c->stream) ||
      hipMemcpyAsync(c->ysd, ones.data(), sizeof(float) * dout, hipMemcpyHostToDevice, c->stream) ||
      hipStreamSynchronize(c->stream))
    return bail(rfail(c, RCELL_ERR_DEVICE, "initialisation failed"));
  *out = c;
  return RCELL_OK;
}

int rsur_destroy(rsur_ctx* c) {
  if (!c) return RCELL_OK;
  destroy_all(c);
  delete c;
  return RCELL_OK;
}

const char* rsur_last_error(const rsur_ctx* c) { return c ? c->err.c_str() : g_rsur_create_error.c_str(); }

int rsur_num_params(rsur_ctx* c, int64_t* n) {
  if (!c || !n) return RCELL_ERR_ARG;
  *n = c->Pflat;
  return RCELL_OK;
}

int rsur_set_params(rsur_ctx* c, int32_t member, const float* w) {
  if (!c || !w || member < 0 || member >= c->K) return c ? rfail(c, RCELL_ERR_ARG, "bad member or NULL") : RCELL_ERR_ARG;
  std::vector<float> h(c->P, 0.0f);
  long long o = 0;
  for (int l = 0; l < c->L; ++l) {
    for (int i = 0; i < c->dims[l]; ++i)
      for (int j = 0; j < c->dims[l + 1]; ++j) h[c->woff[l] + (long long)i * c->dp[l + 1] + j] = w[o++];
    for (int j = 0; j < c->dims[l + 1]; ++j) h[c->boff[l] + j] = w[o++];
  }
  for (float v : h)
    if (!std::isfinite(v)) return rfail(c, RCELL_ERR_ARG, "non-finite parameter");
  const long long off = (long long)member * c->P;
  RCHK(c, hipMemcpyAsync(c->p + off, h.data(), sizeof(float) * c->P, hipMemcpyHostToDevice, c->stream));
  RCHK(c, hipMemsetAsync(c->m1 + off, 0, sizeof(float) * c->P, c->stream));
  RCHK(c, hipMemsetAsync(c->m2 + off, 0, sizeof(float) * c->P, c->stream));
  hipLaunchKernelGGL(k_to_bf16, dim3((unsigned)((c->P + 255) / 256)), dim3(256), 0, c->stream, (const float*)c->p, c->pb,
                     c->pbf, c->pbt, frag_map(c), c->P, off);
  RCHK(c, hipStreamSynchronize(c->stream));
  c->t[member] = 0;
  return RCELL_OK;
}

static int get_flat(rsur_ctx* c, const float* src_dev, int32_t member, float* w) {
  if (!c || !w || member < 0 || member >= c->K) return c ? rfail(c, RCELL_ERR_ARG, "bad member or NULL") : RCELL_ERR_ARG;
  std::vector<float> h(c->P);
  RCHK(c, hipMemcpyAsync(h.data(), src_dev + (long long)member * c->P, sizeof(float) * c->P, hipMemcpyDeviceToHost,
                         c->stream));
  RCHK(c, hipStreamSynchronize(c->stream));
  long long o = 0;
  for (int l = 0; l < c->L; ++l) {
    for (int i = 0; i < c->dims[l]; ++i)
      for (int j = 0; j < c->dims[l + 1]; ++j) w[o++] = h[c->woff[l] + (long long)i * c->dp[l + 1] + j];
    for (int j = 0; j < c->dims[l + 1]; ++j) w[o++] = h[c->boff[l] + j];
  }
  return RCELL_OK;
}

int rsur_get_params(rsur_ctx* c, int32_t member, float* w) { return c ? get_flat(c, c->p, member, w) : RCELL_ERR_ARG; }
int rsur_get_grads(rsur_ctx* c, int32_t member, float* g) { return c ? get_flat(c, c->g, member, g) : RCELL_ERR_ARG; }

int rsur_set_norm(rsur_ctx* c, const float* x_mu, const float* x_sd, const float* y_mu, const float* y_sd) {
  if (!c || !x_mu || !x_sd || !y_mu || !y_sd) return c ? rfail(c, RCELL_ERR_ARG, "NULL statistics") : RCELL_ERR_ARG;
  for (int k = 0; k < c->din; ++k)
    if (!(x_sd[k] > 0) || !std::isfinite(x_mu[k])) return rfail(c, RCELL_ERR_ARG, "x_sd must be > 0");
  for (int k = 0; k < c->dout; ++k)
    if (!(y_sd[k] > 0) || !std::isfinite(y_mu[k])) return rfail(c, RCELL_ERR_ARG, "y_sd must be > 0");
  RCHK(c, hipMemcpyAsync(c->xmu, x_mu, sizeof(float) * c->din, hipMemcpyHostToDevice, c->stream));
  RCHK(c, hipMemcpyAsync(c->xsd, x_sd, sizeof(float) * c->din, hipMemcpyHostToDevice, c->stream));
  RCHK(c, hipMemcpyAsync(c->ymu, y_mu, sizeof(float) * c->dout, hipMemcpyHostToDevice, c->stream));
  RCHK(c, hipMemcpyAsync(c->ysd, y_sd, sizeof(float) * c->dout, hipMemcpyHostToDevice, c->stream));
  RCHK(c, hipStreamSynchronize(c->stream));
  return RCELL_OK;
}

int rsur_fit_norm(rsur_ctx* c, const void* X_dev, const void* Y_dev, int32_t n) {
  if (!c || !X_dev || !Y_dev || n < 1) return c ? rfail(c, RCELL_ERR_ARG, "bad fit_norm arguments") : RCELL_ERR_ARG;
  hipLaunchKernelGGL(k_fit_norm, dim3(c->din), dim3(FIT_NT), 0, c->stream, (const float*)X_dev, n, c->din, c->xmu, c->xsd);
  hipLaunchKernelGGL(k_fit_norm, dim3(c->dout), dim3(FIT_NT), 0, c->stream, (const float*)Y_dev, n, c->dout, c->ymu,
                     c->ysd);
  RCHK(c, hipGetLastError());
  return RCELL_OK;
}

// inference: every layer in one fused kernel when the padded widths allow it.  128 rows per block read
// the weights least often; small batches take 32 rows per block, four times as many blocks, each done
// sooner.  The two meet at ~4000 rows of 5 members (one call, us, 128 against 32 rows per block: 1024
// rows 33.7 / 19.7, 2048 34.4 / 26.1, 4096 37.9 / 38.8, 8192 56 / 60, 16 384 85 / 109).
constexpr int FUSED_MIN_BLOCKS = 160;

static MlpArgs mlp_args(const rsur_ctx* c, const float* X, int B) {
  MlpArgs g{};
  g.X = X; g.B = B; g.din = c->din; g.xmu = c->xmu; g.xsd = c->xsd;
  g.wf = c->pbf; g.sW = c->P; g.p = c->p; g.sP = c->P;
  g.L = c->L; g.dout = c->dout;
  for (int l = 0; l <= c->L; ++l) g.dp[l] = c->dp[l];
  for (int l = 0; l < c->L; ++l) { g.woff[l] = c->woff[l]; g.boff[l] = c->boff[l]; }
  return g;
}

// the fused forward of every member for B rows into out (K x Mp x dp[L], member stride sOut)
static void forward_fused(rsur_ctx* c, const float* X, int B, float* out, long long sOut) {
  MlpArgs g = mlp_args(c, X, B);
  g.out = out; g.sOut = sOut; g.ldo = c->dp[c->L];
  if ((long long)((B + 127) / 128) * c->K >= FUSED_MIN_BLOCKS)
    hipLaunchKernelGGL((k_mlp_forward<4, 8>), dim3((B + 127) / 128, c->K), dim3(512), 0, c->stream, g);
  else
    hipLaunchKernelGGL((k_mlp_forward<1, 8>), dim3((B + 31) / 32, c->K), dim3(512), 0, c->stream, g);
}

// forward, loss and the output gradients of every layer; returns the partial losses per member
static int train_pass(rsur_ctx* c, const float* X, const float* Y, int B, int Mp) {
  TrainArgs h{};
  h.Y = Y; h.ymu = c->ymu; h.ysd = c->ysd; h.wt = c->pbt;
  for (int l = 0; l < c->L; ++l) { h.act[l] = c->act[l]; h.Z[l] = l < c->L - 1 ? c->Z[l] : c->out; }
  h.lpart = c->lpart; h.Mp = Mp; h.rows = c->Mp; h.inv = 1.0f / ((float)B * (float)c->dout);
  const MlpArgs g = mlp_args(c, X, B);
  // 32 rows per block while two of them per CU hold the whole batch, 64 (the weights read half as often)
  // beyond.  A step of 5 members, us, 32 / 64 / 128 rows per block: 256 rows 56 / 70 / 98, 2048 96 / 102 /
  // 128, 3072 108 / 117 / 143, 4096 151 / 142 / 159, 8192 285 / 298 / 333, 60 000 1840 / 1719 / 2000.
  const bool small = (long long)(Mp / 32) * c->K <= 512;
  const dim3 grid(Mp / (small ? 32 : 64), c->K);
  if (small) hipLaunchKernelGGL((k_mlp_train<1, 8>), grid, dim3(512), 0, c->stream, g, h);
  else hipLaunchKernelGGL((k_mlp_train<2, 8>), grid, dim3(512), 0, c->stream, g, h);
  return (int)grid.x;
}

// the arguments of layer l's weight and bias gradients over Mp rows in S ranges (dz: rows of lddz, members sdz apart)
static GemmArgs dw_args(const rsur_ctx* c, int l, const bf16* dz, int lddz, long long sdz, int Mp, int S, float* grads) {
  GemmArgs w{};                                      // dW_l = act_l^T dZ_l
  w.A = c->act[l]; w.lda = c->dp[l]; w.sA = l == 0 ? 0 : (long long)c->Mp * c->dp[l];
  w.B = dz; w.ldb = lddz; w.sB = sdz;
  w.M = c->dp[l]; w.N = c->dp[l + 1]; w.K = Mp;
  w.Z = grads + c->woff[l]; w.ldz = c->dp[l + 1]; w.sZ = c->P;
  w.nmem = c->K; w.ksplit = S; w.sRange = (long long)c->K * c->P;
  w.colsum = grads + c->boff[l]; w.sCol = c->P;      // and db_l, the column sums of dZ_l
  return w;
}

static void forward_infer(rsur_ctx* c, const float* X, int B, int Mp) {
  if (!fused_shape(c)) {
    normalise_inputs(c, X, B, Mp);
    forward_layers(c, Mp);
    return;
  }
  forward_fused(c, X, B, c->out, (long long)c->Mp * c->dp[c->L]);
}

static int forward_common(rsur_ctx* c, const void* X_dev, int32_t B, float* mean, float* var, float* members) {
  int e = check_batch(c, B);
  if (e) return e;
  const int Mp = pad64(B);
  forward_infer(c, (const float*)X_dev, B, Mp);
  const long long n = (long long)B * c->dout;
  hipLaunchKernelGGL(k_ensemble, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, c->out,
                     (long long)c->Mp * c->dp[c->L], c->dp[c->L], c->K, B, c->dout, c->ymu, c->ysd, mean, var, members);
  RCHK(c, hipGetLastError());
  return RCELL_OK;
}

int rsur_forward(rsur_ctx* c, const void* X_dev, int32_t B, void* mean_dev, void* var_dev) {
  TraceRange tr("rsur_forward");
  if (!c || !X_dev || !mean_dev) return c ? rfail(c, RCELL_ERR_ARG, "NULL pointer") : RCELL_ERR_ARG;
  return forward_common(c, X_dev, B, (float*)mean_dev, (float*)var_dev, nullptr);
}

int rsur_forward_static(rsur_ctx* c, const void* X_dev, int32_t B, void* mean_dev, void* var_dev) {
  TraceRange tr("rsur_forward_static");
  if (!c || !X_dev || !mean_dev) return c ? rfail(c, RCELL_ERR_ARG, "NULL pointer") : RCELL_ERR_ARG;
  if (!fused_shape(c)) return rfail(c, RCELL_ERR_ARG, "static forward: padded widths <= 256, <= 8 layers");
  if (B < 1 || (long long)c->K * pad64(B) * c->dp[c->L] > RSUR_STATIC_FLOATS)
    return rfail(c, RCELL_ERR_ARG, "static forward: B must be >= 1 and K * pad64(B) * pad64(dout) <= 2^21");
  float* out = nullptr;
  if (static_scratch_ptr(&out) != RCELL_OK) return rfail(c, RCELL_ERR_DEVICE, "static scratch address");
  const int Mp = pad64(B);
  const long long sOut = (long long)Mp * c->dp[c->L];
  forward_fused(c, (const float*)X_dev, B, out, sOut);
  const long long n = (long long)B * c->dout;
  hipLaunchKernelGGL(k_ensemble, dim3((unsigned)((n + 255) / 256)), dim3(256), 0, c->stream, out, sOut,
                     c->dp[c->L], c->K, B, c->dout, c->ymu, c->ysd, (float*)mean_dev, (float*)var_dev, (float*)nullptr);
  if (hipGetLastError() != hipSuccess) return rfail(c, RCELL_ERR_DEVICE, "static forward: launch failed");
  return RCELL_OK;
}

int rsur_forward_members(rsur_ctx* c, const void* X_dev, int32_t B, void* out_dev) {
  if (!c || !X_dev || !out_dev) return c ? rfail(c, RCELL_ERR_ARG, "NULL pointer") : RCELL_ERR_ARG;
  return forward_common(c, X_dev, B, nullptr, nullptr, (float*)out_dev);
}

int rsur_train_step(rsur_ctx* c, const void* X_dev, const void* Y_dev, int32_t B, float lr, float* loss) {
  TraceRange tr("rsur_train_step");
  if (!c || !X_dev || !Y_dev || !(lr > 0)) return c ? rfail(c, RCELL_ERR_ARG, "bad train_step arguments") : RCELL_ERR_ARG;
  int e = check_batch(c, B);
  if (e) return e;
  const int Mp = pad64(B), L = c->L;
  const int S = batch_splits(c, Mp);
  const long long n = (long long)c->K * c->P;
  float* grads = S > 1 ? c->split : c->g;            // k_adam adds the ranges up
  int chunks;                                        // partial losses per member
  if (fused_shape(c)) {
    chunks = train_pass(c, (const float*)X_dev, (const float*)Y_dev, B, Mp);
    DwArgs d{};
    for (int l = 0; l < L; ++l) {
      const int ld = 2 * c->dp[l + 1];               // TrainArgs::Z
      d.g[l] = dw_args(c, l, (const bf16*)(l < L - 1 ? c->Z[l] : c->out), ld, (long long)c->Mp * ld, Mp, S, grads);
      d.first[l + 1] = d.first[l] + d.g[l].M / TM * (d.g[l].N / TN);
    }
    hipLaunchKernelGGL(k_dw, dim3(d.first[L], c->K * S), dim3(256), 0, c->stream, d);
  } else {
    normalise_inputs(c, (const float*)X_dev, B, Mp);
    forward_layers(c, Mp);
    const long long sOut = (long long)c->Mp * c->dp[L];
    const long long sdz = (long long)c->Mp * *std::max_element(c->dp.begin(), c->dp.end());
    chunks = Mp / LOSS_ROWS;
    hipLaunchKernelGGL(k_loss, dim3(chunks, c->K), dim3(LOSS_NT), 0, c->stream, c->out, sOut, c->dp[L],
                       (const float*)Y_dev, B, c->dout, c->ymu, c->ysd, c->dza, sdz, c->lpart);
    bf16 *dz = c->dza, *dzn = c->dzb;
    for (int l = L - 1; l >= 0; --l) {
      gemm<true, false, EPI_BWD_DW>(c, dw_args(c, l, dz, c->dp[l + 1], sdz, Mp, S, grads));
      if (l > 0) {                                   // dZ_{l-1} = (dZ_l W_l^T) * SiLU'(Z_{l-1})
        GemmArgs d{};
        d.A = dz; d.lda = c->dp[l + 1]; d.sA = sdz;
        d.B = c->pb + c->woff[l]; d.ldb = c->dp[l + 1]; d.sB = c->P;
        d.M = Mp; d.N = c->dp[l]; d.K = c->dp[l + 1];
        d.Zp = c->Z[l - 1]; d.ldzp = c->dp[l]; d.sZp = (long long)c->Mp * c->dp[l];
        d.O = dzn; d.ldo = c->dp[l]; d.sO = sdz;
        gemm<false, true, EPI_BWD_DA>(c, d);
        std::swap(dz, dzn);
      }
    }
  }
  if (loss)                                          // read by this call alone
    hipLaunchKernelGGL(k_loss_total, dim3(c->K), dim3(64), 0, c->stream, c->lpart, chunks,
                       1.0f / ((float)B * (float)c->dout), c->loss);
  // Adam with per-member bias corrections
  const FragMap map = frag_map(c);
  for (int k0 = 0; k0 < c->K; k0 += ADAM_MEM) {
    AdamBias bias{};
    const int nk = std::min(ADAM_MEM, c->K - k0);
    for (int k = 0; k < nk; ++k) {
      c->t[k0 + k] += 1;
      bias.c1[k] = (float)(1.0 - std::pow(0.9, (double)c->t[k0 + k]));
      bias.c2[k] = (float)(1.0 - std::pow(0.999, (double)c->t[k0 + k]));
    }
    hipLaunchKernelGGL(k_adam, dim3((unsigned)((c->P + 255) / 256), nk), dim3(256), 0, c->stream, c->p, c->g,
                       (const float*)c->split, S, n, c->m1, c->m2, c->pb, c->pbf, c->pbt, map, c->P, k0, bias, lr, 0.9f, 0.999f, 1e-8f);
  }
  RCHK(c, hipGetLastError());
  if (loss) {
    RCHK(c, hipMemcpyAsync(loss, c->loss, sizeof(float) * c->K, hipMemcpyDeviceToHost, c->stream));
    RCHK(c, hipStreamSynchronize(c->stream));
  }
  return RCELL_OK;
}

}  // extern "C"
