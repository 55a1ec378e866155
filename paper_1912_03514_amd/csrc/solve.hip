// Host side of the persistent solve (solve_kernel.hpp): launch shape, workspace layout,
// the gradient pass on its own and the per-XCD row weights.
#include <stdlib.h>

#include "solve_kernel.hpp"

namespace mihs {

namespace {

// The gradient pass of Algorithm 1 on its own: partial A^T (c - A x) of one row
// block per workgroup (c = b, or none), then a fixed-order column sum that adds
// rhs and subtracts lambda x.  Used by drivers whose inner step is not CG.
template <typename TA, int EPT>
__global__ __launch_bounds__(kBlock) void grad_partial_kernel(const TA* A, int64_t n, int64_t lda,
                                                              int d, int dpad, const double* c,
                                                              const double* x, double* part,
                                                              const int* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  extern __shared__ double smem[];
  double* vbuf = smem;
  double* rbuf = smem + dpad;
  for (int k = threadIdx.x; k < dpad; k += kBlock) vbuf[k] = (k < d) ? x[k] : 0.0;
  __syncthreads();
  const int64_t G = gridDim.x, w = blockIdx.x;
  const int64_t r0 = n * w / G, r1 = n * (w + 1) / G;
  if constexpr (EPT == 64) {
    __shared__ double s_part[2 * kQuarterRows * kWavesPerBlock];
    double acc[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.0;
    rowpass_quarters<TA, 16, true, quarter_rows<TA>()>(A, lda, r0, r1, d, vbuf, c, acc, s_part);
    store_quarters<TA, 16>(acc, part + w * dpad, d);
  } else {
    double acc[EPT];
#pragma unroll
    for (int e = 0; e < EPT; ++e) acc[e] = 0.0;
    double ssq = 0.0;
    rowpass<TA, double, EPT, true, RowsInFlight<TA, EPT>::value>(A, lda, r0, r1, d, vbuf, c,
                                                                   acc, ssq);
    wg_store_partial<TA, double, EPT>(acc, rbuf, part + w * dpad, d);
  }
}

// 32 columns per workgroup; the 8 thread rows of a column sum interleaved
// partials (t = q, q + 8, ...) and meet in LDS in a fixed order.
constexpr int kFinCols = 32;
__global__ __launch_bounds__(kBlock) void grad_finish_kernel(const double* part, int G, int dpad,
                                                             int d, const double* rhs,
                                                             const double* x, double lam,
                                                             double* g, const int* skip) {
  if (skip && __hip_atomic_load(skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  __shared__ double red[kBlock / kFinCols][kFinCols];
  constexpr int Q = kBlock / kFinCols;
  const int cl = threadIdx.x % kFinCols, q = threadIdx.x / kFinCols;
  const int k = blockIdx.x * kFinCols + cl;
  double s = 0.0;
  if (k < d)
    for (int t = q; t < G; t += Q) s += part[(int64_t)t * dpad + k];
  red[q][cl] = s;
  __syncthreads();
  if (q == 0 && k < d) {
    double tot = red[0][cl];
    for (int i = 1; i < Q; ++i) tot += red[i][cl];
    if (rhs) tot += rhs[k];
    g[k] = tot - lam * x[k];
  }
}

template <typename TA, int EPT>
int launch_grad_partial(int G, size_t shmem, hipStream_t stream, const TA* A, int64_t n,
                        int64_t lda, int d, int dpad, const double* c, const double* x,
                        double* part, const int* skip) {
  if (hipFuncSetAttribute((const void*)grad_partial_kernel<TA, EPT>,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)shmem) != hipSuccess)
    return MIHS_ERR_HIP;
  hipLaunchKernelGGL((grad_partial_kernel<TA, EPT>), dim3(G), dim3(kBlock), shmem, stream, A, n,
                     lda, d, dpad, c, x, part, skip);
  return MIHS_OK;
}

template <typename TA>
int launch_grad_partial_ept(int ept, int G, size_t shmem, hipStream_t stream, const TA* A,
                            int64_t n, int64_t lda, int d, int dpad, const double* c,
                            const double* x, double* part, const int* skip) {
  switch (ept) {
    case 1:
      return launch_grad_partial<TA, 1>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 2:
      return launch_grad_partial<TA, 2>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 4:
      return launch_grad_partial<TA, 4>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 8:
      return launch_grad_partial<TA, 8>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 16:
      return launch_grad_partial<TA, 16>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 32:
      return launch_grad_partial<TA, 32>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    case 64:
      return launch_grad_partial<TA, 64>(G, shmem, stream, A, n, lda, d, dpad, c, x, part,
                                          skip);
    default: return MIHS_ERR_UNSUPPORTED;
  }
}

__global__ void zero_words(unsigned* p, int count) {
  for (int i = blockIdx.x * blockDim.x + threadIdx.x; i < count; i += gridDim.x * blockDim.x)
    p[i] = 0u;
}

// Mixed precision stores the inner solver's operator (SA, or its Gram matrix)
// in FP32, which halves the bytes every inner step streams, and keeps the CG
// recurrences (vectors, step lengths, dot products) in FP64: FP32 recurrences
// lose their conjugacy on ill-conditioned sub-problems (kappa ~ 6e8: 87k inner
// steps against 27k, measured), and in this latency-bound loop the FP64
// vectors cost about 1% at the headline size.
SolveKernel pick_kernel(int a_f32, int mixed, int ept, bool gram, bool res) {
  if (!a_f32 && !mixed) return pick_kernel_typed<double, double>(ept, gram, res);
  if (!a_f32 && mixed) return pick_kernel_typed<double, float>(ept, gram, res);
  if (a_f32 && !mixed) return pick_kernel_typed<float, double>(ept, gram, res);
  return pick_kernel_typed<float, float>(ept, gram, res);
}

int max_grid(const mihs_handle* h) { return h->num_cu * kMaxBlocksPerCU; }

}  // namespace

// ---- scratch of the entry point without a workspace argument -------------
// mihs_solve_noalloc runs the solve kernels on this array instead of a caller
// workspace: one copy per GPU, held by the loaded code object until the process
// ends.  In host code the name is only a stand-in for the symbol (passing it
// to a kernel would make the kernel fault): every host use goes through the
// device address that noalloc_scratch_address() returns, which differs per GPU.
static __device__ __align__(256) unsigned char scratch[kNoAllocScratchBytes];

int noalloc_scratch_address(void** ptr) {
  // call with the handle's device current: each GPU holds its own copy
  *ptr = nullptr;
  if (hipGetSymbolAddress(ptr, HIP_SYMBOL(scratch)) != hipSuccess || *ptr == nullptr)
    return MIHS_ERR_HIP;
  return MIHS_OK;
}

int ept_for(int64_t d) {
  int e = 1;
  while (64 * (int64_t)e < d) e *= 2;
  return e;
}

size_t solve_workspace_bytes(const mihs_handle* h, int64_t n, int64_t d, int64_t m, int mixed,
                             int no_gram) {
  (void)n;
  return solve_layout_bound(max_grid(h), d, m, mixed ? 4 : 8, no_gram != 0);
}

int grad_partials(const mihs_handle* h, int64_t n, int64_t d) {
  int64_t g = (int64_t)h->num_cu * kMaxBlocksPerCU;
  const int64_t by_rows = (n + 63) / 64;
  if (g > by_rows) g = by_rows < 1 ? 1 : by_rows;
  (void)d;
  return (int)g;
}

size_t grad_workspace_bytes(const mihs_handle* h, int64_t n, int64_t d) {
  return align_up((size_t)grad_partials(h, n, d) * (size_t)dpad_for(d) * 8, 256);
}

int launch_grad(const mihs_handle* h, const void* A, int a_f32, int64_t n, int64_t d,
                int64_t lda, const double* c, const double* rhs, const double* x, double lam,
                double* g, void* ws, size_t ws_bytes, const int* skip, hipStream_t stream) {
  const int ept = ept_for(d);
  if (ept > 64) return MIHS_ERR_UNSUPPORTED;
  if (ws_bytes < grad_workspace_bytes(h, n, d) || ws == nullptr) return MIHS_ERR_WORKSPACE;
  const int dpad = (int)dpad_for(d);
  const size_t shmem = 2 * (size_t)dpad * sizeof(double);
  const int G = grad_partials(h, n, d);
  double* part = (double*)ws;
  const int rc = a_f32 ? launch_grad_partial_ept<float>(ept, G, shmem, stream, (const float*)A, n,
                                                        lda, (int)d, dpad, c, x, part, skip)
                       : launch_grad_partial_ept<double>(ept, G, shmem, stream, (const double*)A,
                                                         n, lda, (int)d, dpad, c, x, part, skip);
  if (rc) return rc;
  hipLaunchKernelGGL(grad_finish_kernel, dim3((unsigned)((d + kFinCols - 1) / kFinCols)),
                     dim3(kBlock), 0, stream, part, G, dpad, (int)d, rhs, x, lam, g, skip);
  return hipGetLastError() == hipSuccess ? MIHS_OK : MIHS_ERR_HIP;
}

int launch_solve(const mihs_handle* h, const SolveDesc& s, void* ws, size_t ws_bytes,
                 hipStream_t stream) {
  const int ept = ept_for(s.d);
  if (ept > 64) return MIHS_ERR_UNSUPPORTED;
  // AAb_Solver needs M v and M^T p separately: it always streams SA
  const bool gram = !s.no_gram && !s.aab && use_gram(s.m, s.d);
  const int64_t dpad = dpad_for(s.d);
  SolveKernel kern = nullptr;
  bool hip_error = false;
  const SolveShape shape = pick_solve_shape(
      s.n, s.d, s.m, s.mixed ? 4 : 8, ept, gram, h->num_cu, [&](bool res, size_t lds) {
        kern = pick_kernel(s.a_f32, s.mixed, ept, gram, res);
        int occ = 0;
        hip_error = !kern ||
                    hipFuncSetAttribute((const void*)kern,
                                        hipFuncAttributeMaxDynamicSharedMemorySize,
                                        (int)lds) != hipSuccess ||
                    hipOccupancyMaxActiveBlocksPerMultiprocessor(&occ, kern, kBlock, lds) !=
                        hipSuccess;
        return hip_error ? -1 : occ;
      });
  if (hip_error) return MIHS_ERR_HIP;
  if (shape.G == 0) return MIHS_ERR_UNSUPPORTED;
  const int G = shape.G, Gc = shape.Gc, cpw = shape.cpw;
  const size_t shmem = shape.lds;
  const SolveTags tags = solve_tags(gram, shape.res, s.mixed ? 4 : 8, ept, Gc, cpw);
  const SolveLayout L = solve_layout(G, Gc, dpad, tags, gram ? gram_bytes(s.d, s.mixed ? 4 : 8) : 0,
                                     s.m);
  if (ws_bytes < L.total || ws == nullptr) return MIHS_ERR_WORKSPACE;

  char* base = (char*)ws;
  SolveArgs a;
  a.A = s.A;
  a.n = s.n;
  a.lda = s.lda;
  a.b = s.b;
  a.rhs = s.rhs;
  a.SA = s.SA;
  a.m = s.m;
  a.ldsa = s.ldsa;
  a.lam = s.lam;
  a.alpha = s.alpha;
  a.beta = s.beta;
  a.eps_sub = s.eps_sub;
  a.step_thr = (s.tol > 0.0 && s.beta > 0.0 && s.beta < 1.0)
                   ? s.tol * (1.0 - sqrt(s.beta)) / sqrt(s.beta)
                   : (s.tol > 0.0 ? s.tol : 0.0);
  a.max_outer = s.max_outer;
  a.max_inner = s.max_inner;
  a.x = s.x;
  a.xp = s.x_prev ? s.x_prev : (double*)(base + L.xp);
  a.xp_from_x = s.x_prev ? 0 : 1;
  a.info = s.info;
  a.partA = (double*)(base + L.partA);
  a.partS = (void*)(base + L.partS);
  a.scal = (double*)(base + L.scal);
  a.r = (void*)(base + L.vecs);
  a.z = (void*)(base + L.vecs + (size_t)dpad * 8);
  a.p0 = (void*)(base + L.vecs + 2 * (size_t)dpad * 8);
  a.p1 = (void*)(base + L.vecs + 3 * (size_t)dpad * 8);
  unsigned* bar = (unsigned*)(base + L.bar);
  a.bar_all = bar;
  a.bar_cg = bar + 9 * 32;
  a.bar_cgh = bar + 12 * 32;
  a.cg_hier = Gc > 128 ? 1 : 0;
  for (int k = 0; k < kXcds; ++k) a.xw[k] = h->row_weight[k];
  a.err = (int*)(bar + 10 * 32);
  a.status = (int*)(bar + 11 * 32);
  a.d = (int)s.d;
  a.dpad = (int)dpad;
  a.G = G;
  a.Gc = Gc;
  a.cpw = cpw;
  a.tags = (tagged_t*)(base + L.tags);
  a.tagw = (tagged_t*)(base + L.tagw);
  a.partT = tags == SolveTags::kStreaming ? (tagged_t*)(base + L.region) : nullptr;
  a.spin_fast = {kBarrierPolls, 1, kTagPolls};
  a.spin_idle = {kIdlePolls, 16, kTagPolls};
  a.H = gram ? (const void*)(base + L.region) : nullptr;
  a.ldh = dpad;
  // One barrier per CG step pays off where the CG is latency-bound (headline,
  // FP64: 32.2 -> 29.4 ms per solve); the two-reduction form keeps fewer steps
  // on very ill-conditioned solves (measured on the CountSketch workload,
  // kappa ~ 6e8: FP64 22k vs 27-38k steps; FP32 breaks down), so the kernel
  // takes the single-reduction form only where trace(H) / lambda is small.
  a.cg1 = 1;
  a.aab = s.aab ? 1 : 0;
  a.yrow = (double*)(base + L.yrow);
  a.skip = s.skip;
  if (gram && !s.gram_ready) {
    const int rc = launch_gram(s.SA, s.mixed, s.m, s.d, s.ldsa, base + L.region, s.mixed, dpad,
                               stream);
    if (rc) return rc;
  }

  // barrier words and tags (contiguous)
  const int zwords = (int)((L.zero_end - L.bar) / 4);
  hipLaunchKernelGGL(zero_words, dim3((unsigned)((zwords + 1023) / 1024)), dim3(256), 0, stream,
                     bar, zwords);
  if (hipGetLastError() != hipSuccess) return MIHS_ERR_HIP;
  void* args[] = {&a};
  if (hipLaunchCooperativeKernel((const void*)kern, dim3(G), dim3(kBlock), args, shmem, stream) !=
      hipSuccess)
    return MIHS_ERR_HIP;
  return MIHS_OK;
}

// ---- per-XCD row weights of the gradient pass --------------------------------
// The gradient pass streams A once per outer iteration in contiguous row ranges,
// one workgroup per CU; its length is that of the slowest workgroup.  XCDs do
// not all stream from HBM at the same rate: on MI355X, with equal shares of an
// FP64 matrix of 2048 columns, the odd-numbered XCDs took 6-8% longer than the
// even ones, on every pass (a plain 16-byte stream shows about half of that, so
// the measurement below runs the gradient pass's own row loop).  The rows are
// shared out by per-XCD weights measured here.

constexpr int kCalCols = 2048;                      // FP64 columns of the timing matrix
constexpr int64_t kCalRows = (int64_t)1 << 17;      // 2 GiB (> the Infinity Cache)
constexpr int kCalWarm = 6;    // untimed passes (the first calibration of a process,
                               // with 2, sometimes saw a 14% spread instead of 10%)
constexpr int kCalPasses = 15;  // timed passes; per XCD the median pass counts
constexpr long kRowWeightStep = 4;                  // weights are multiples of this
constexpr size_t kCalLds = 96 * 1024;               // keeps one workgroup per CU

// One workgroup per CU runs the gradient pass's row loop (x = 0) over its equal
// share of the rows and records its start and end wall clock (clk[2w],
// clk[2w + 1]).
__global__ __launch_bounds__(kBlock) void xcd_rowpass_kernel(const double* __restrict__ M,
                                                             long long* clk, double* sink) {
  extern __shared__ double v[];  // kCalCols zeros, then padding
  for (int c = threadIdx.x; c < kCalCols; c += kBlock) v[c] = 0.0;
  __syncthreads();
  const int G = gridDim.x, w = blockIdx.x;
  const long long t0 = wall_clock64();
  constexpr int EPT = kCalCols / kWave;
  double acc[EPT];
#pragma unroll
  for (int e = 0; e < EPT; ++e) acc[e] = 0.0;
  double ssq = 0.0;
  rowpass<double, double, EPT, true, RowsInFlight<double, EPT>::value>(
      M, kCalCols, kCalRows * w / G, kCalRows * (w + 1) / G, kCalCols, v, nullptr, acc, ssq);
  __syncthreads();
  if (threadIdx.x == 0) {
    clk[2 * w] = t0;
    clk[2 * w + 1] = wall_clock64();
  }
  // keeps the arithmetic (never true: the matrix is zero)
  double t = ssq;
#pragma unroll
  for (int e = 0; e < EPT; ++e) t += acc[e];
  if (t == 1.25e300) sink[w] = t;
}

int calibrate_rows(mihs_handle* h) {
  int prev = 0;
  if (hipGetDevice(&prev) != hipSuccess || hipSetDevice(h->device) != hipSuccess)
    return MIHS_ERR_HIP;
  const int G = h->num_cu;
  char* buf = nullptr;
  const size_t bytes = (size_t)kCalRows * kCalCols * sizeof(double);
  const size_t clk_off = bytes, sink_off = bytes + (size_t)G * 16;
  int rc = MIHS_OK;
  if (G < kXcds || hipMalloc(&buf, sink_off + (size_t)G * 8) != hipSuccess) {
    (void)hipGetLastError();
    (void)hipSetDevice(prev);
    return MIHS_ERR_HIP;
  }
  std::vector<long long> clk((size_t)2 * G);
  std::vector<double> tpass[kXcds];  // per XCD: mean workgroup time of each pass
  if (hipMemset(buf, 0, bytes) != hipSuccess ||
      hipFuncSetAttribute((const void*)xcd_rowpass_kernel,
                          hipFuncAttributeMaxDynamicSharedMemorySize, (int)kCalLds) != hipSuccess)
    rc = MIHS_ERR_HIP;
  for (int pass = 0; pass < kCalWarm + kCalPasses && rc == MIHS_OK; ++pass) {
    hipLaunchKernelGGL(xcd_rowpass_kernel, dim3(G), dim3(kBlock), kCalLds, 0, (const double*)buf,
                       (long long*)(buf + clk_off), (double*)(buf + sink_off));
    if (hipGetLastError() != hipSuccess ||
        hipMemcpy(clk.data(), buf + clk_off, clk.size() * sizeof(long long),
                  hipMemcpyDeviceToHost) != hipSuccess) {
      rc = MIHS_ERR_HIP;
      break;
    }
    if (pass < kCalWarm) continue;
    double sum[kXcds] = {0.0};
    int cnt[kXcds] = {0};
    for (int w = 0; w < G; ++w) {
      sum[w % kXcds] += (double)(clk[2 * w + 1] - clk[2 * w]);
      cnt[w % kXcds] += 1;
    }
    for (int k = 0; k < kXcds; ++k) tpass[k].push_back(sum[k] / (double)cnt[k]);
  }
  (void)hipFree(buf);
  (void)hipSetDevice(prev);
  if (rc != MIHS_OK) return rc;
  // Weight (t_min / t)^(3/4) of the fastest XCD's kRowWeightMax, at most a 2:1
  // spread, in steps of kRowWeightStep.  With equal shares the slow XCDs also
  // stream faster once the fast ones are done, so the time ratio overstates the
  // rate ratio under a balanced load: on the headline solve (odd XCDs 7-9%
  // slower at equal shares) weights 64/60 by XCD parity gave 25.10-25.26 ms
  // per solve, 64/56 25.47 ms, equal weights 25.56-25.67 ms.  The steps keep
  // the 1-2% drift of the means between calibrations from moving the split
  // (64/60 with one even XCD at 63 measured 25.36 ms).
  double tk[kXcds], tmin = 0.0;
  for (int k = 0; k < kXcds; ++k) {
    std::vector<double>& v = tpass[k];
    std::nth_element(v.begin(), v.begin() + v.size() / 2, v.end());
    tk[k] = v[v.size() / 2];
    if (!(tk[k] > 0.0)) return MIHS_ERR_HIP;
    if (k == 0 || tk[k] < tmin) tmin = tk[k];
  }
  for (int k = 0; k < kXcds; ++k) {
    const double t = tk[k];
    const long wk =
        kRowWeightStep * lround((double)(kRowWeightMax / kRowWeightStep) * pow(tmin / t, 0.75));
    h->row_weight[k] = (int32_t)std::min<long>(kRowWeightMax, std::max<long>(kRowWeightMax / 2, wk));
  }
  return MIHS_OK;
}

}  // namespace mihs
