// Gram matrices H = M^T M of sketches (M = SA, m x d row-major) on the FP64
// matrix cores.  The inner CG applies the sub-problem operator (SA)^T SA as
// H p, one d x d product per step instead of two passes over SA.
#include "gemm64.hpp"
#include "internal.hpp"

namespace mihs {

namespace {

// One T x T block (bi <= bj) of H: the FP64 tile product of M's columns [T bi, T bi + T)
// and [T bj, T bj + T).  The block goes through LDS so that it and its mirror image are
// both written along rows (the mirror written straight from the result registers is one
// 8-byte store per row of H).  Entries of index >= d come out zero; entries below hn (the
// padded size of H) are written; off-diagonal blocks are mirrored and the diagonal ones
// mirror their upper half, so H is exactly symmetric.
template <typename TS, typename TH, int T>
__device__ __forceinline__ void gram_block(const TS* __restrict__ M, int64_t m, int64_t ld, int d,
                                           TH* __restrict__ H, int64_t ldh, int hn, int bi, int bj,
                                           double* lds) {
  typedef KRows<TS, T> O;
  constexpr int MB = T / 32;
  if (bj * T >= d) {  // a block of padding only: zeros, and no column of M to read
    for (int e = threadIdx.x; e < T * T; e += kBlock) {
      const int i = bi * T + e / T, j = bj * T + e % T;
      if (i < hn && j < hn) {
        H[(int64_t)i * ldh + j] = TH(0);
        H[(int64_t)j * ldh + i] = TH(0);
      }
    }
    return;
  }
  f64x4 acc[MB][MB];
  gemm64_tile<O, O, T, T>(M, ld, (int64_t)bi * T, d, M, ld, (int64_t)bj * T, d, 0, m, lds, acc);
  const int lane = lane_id(), wave = wave_id();
  constexpr int LD = T + 1;
  static_assert(T * LD <= gemm64_lds<O, O>(), "the block fits the operand buffers");
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < MB; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r)
        lds[((wave >> 1) * (T / 2) + 16 * a + (lane >> 4) + 4 * r) * LD +
            (wave & 1) * (T / 2) + 16 * b + (lane & 15)] = acc[a][b][r];
  __syncthreads();
  for (int e = threadIdx.x; e < T * T; e += kBlock) {
    const int r = e / T, c = e % T;
    const int i = bi * T + r, j = bj * T + c;
    if (i < hn && j < hn && i <= j) H[(int64_t)i * ldh + j] = (TH)lds[r * LD + c];
  }
  for (int e = threadIdx.x; e < T * T; e += kBlock) {
    const int c = e / T, r = e % T;
    const int i = bi * T + r, j = bj * T + c;
    if (i < hn && j < hn && i < j) H[(int64_t)j * ldh + i] = (TH)lds[r * LD + c];
  }
}

template <typename TS>
__global__ __launch_bounds__(kBlock) void gram_jobs_kernel(const GramJob* jobs) {
  typedef KRows<TS, 64> O;
  __shared__ __attribute__((aligned(16))) double lds[gemm64_lds<O, O>()];
  const GramJob J = jobs[blockIdx.x];
  if (J.h_f32)
    gram_block<TS, float, 64>((const TS*)J.M, J.m, J.ld, J.d, (float*)J.H, J.ldh, (int)J.ldh,
                              J.bi, J.bj, lds);
  else
    gram_block<TS, double, 64>((const TS*)J.M, J.m, J.ld, J.d, (double*)J.H, J.ldh, (int)J.ldh,
                               J.bi, J.bj, lds);
}

// One matrix, grid (hn / T, hn / T); blocks below the diagonal return at once.
template <typename TS, typename TH, int T>
__global__ __launch_bounds__(kBlock) void gram_one_kernel(const TS* M, int64_t m, int64_t ld,
                                                          int d, TH* H, int64_t ldh, int hn) {
  typedef KRows<TS, T> O;
  __shared__ __attribute__((aligned(16))) double lds[gemm64_lds<O, O>()];
  const int bi = blockIdx.y, bj = blockIdx.x;
  if (bi > bj) return;
  gram_block<TS, TH, T>(M, m, ld, d, H, ldh, hn, bi, bj, lds);
}

template <typename TS, typename TH>
void launch_one(const void* M, int64_t m, int64_t d, int64_t ld, void* H, int64_t ldh, int hn,
                hipStream_t st) {
  // Up to d = 512 the 64 x 64 blocks on and above the diagonal are fewer than one per seven
  // CUs and every one is a serial chain over m: 32 x 32 blocks 18 against 33 us at
  // 512 x 512, 10 against 19 at 256 x 256; at 1024 x 1024 (136 blocks of 64) 74 against 65.
  if (hn <= 512)
    gram_one_kernel<TS, TH, 32><<<dim3(hn / 32, hn / 32), dim3(kBlock), 0, st>>>(
        (const TS*)M, m, ld, (int)d, (TH*)H, ldh, hn);
  else
    gram_one_kernel<TS, TH, 64><<<dim3(hn / 64, hn / 64), dim3(kBlock), 0, st>>>(
        (const TS*)M, m, ld, (int)d, (TH*)H, ldh, hn);
}

}  // namespace

int launch_gram_jobs(const GramJob* d_jobs, int64_t njobs, int m_f32, hipStream_t st) {
  if (njobs <= 0) return MIHS_OK;
  if (m_f32)
    gram_jobs_kernel<float><<<dim3((unsigned)njobs), dim3(kBlock), 0, st>>>(d_jobs);
  else
    gram_jobs_kernel<double><<<dim3((unsigned)njobs), dim3(kBlock), 0, st>>>(d_jobs);
  return hipGetLastError() == hipSuccess ? MIHS_OK : MIHS_ERR_HIP;
}

int launch_gram(const void* M, int m_f32, int64_t m, int64_t d, int64_t ld, void* H, int h_f32,
                int64_t ldh, hipStream_t st) {
  const int hn = 64 * (int)((d + 63) / 64);
  if (ldh < hn) return MIHS_ERR_INVALID;
  if (m_f32 && h_f32)
    launch_one<float, float>(M, m, d, ld, H, ldh, hn, st);
  else if (m_f32)
    launch_one<float, double>(M, m, d, ld, H, ldh, hn, st);
  else if (h_f32)
    launch_one<double, float>(M, m, d, ld, H, ldh, hn, st);
  else
    launch_one<double, double>(M, m, d, ld, H, ldh, hn, st);
  return hipGetLastError() == hipSuccess ? MIHS_OK : MIHS_ERR_HIP;
}

}  // namespace mihs
