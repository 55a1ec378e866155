// Sketch kernels (Lemma 3): SRHT via a blocked fast Walsh-Hadamard transform,
// CountSketch via a deterministic bucket sort + segmented sums, Gaussian via
// counter-based generation and a matrix-core GEMM (FP64 MFMA for the plain
// path, BF16 MFMA with FP32 accumulation for the mixed path).
#include <math.h>

#include <algorithm>
#include <type_traits>

#include "gemm64.hpp"
#include "internal.hpp"
#include "rng.hpp"

namespace mihs {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

// ---------------------------------------------------------------------------
// BF16 rounding (round to nearest even of the exact value).  A double is first
// narrowed to float with round-to-odd (truncate, then set the sticky bit if
// inexact) so the second rounding to BF16 is a single correct rounding.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint16_t bf16_rne_from_float(float f) {
  uint32_t u = __float_as_uint(f);
  if ((u & 0x7F800000u) == 0x7F800000u) return (uint16_t)((u >> 16) | ((u & 0xFFFFu) ? 0x40u : 0u));
  u += 0x7FFFu + ((u >> 16) & 1u);
  return (uint16_t)(u >> 16);
}
__device__ __forceinline__ uint16_t bf16_rne(double x) {
  float f = __double2float_rz(x);
  if ((double)f != x) f = __uint_as_float(__float_as_uint(f) | 1u);
  return bf16_rne_from_float(f);
}
__device__ __forceinline__ uint16_t bf16_rne(float x) { return bf16_rne_from_float(x); }

// ---------------------------------------------------------------------------
// SRHT:  SA = (1/sqrt(m)) P H D A with H = H_hi (x) H_lo (Sylvester order):
// row index i = i_hi * B + i_lo.  Stage 1 applies D and the length-B transform
// over i_lo inside each block of B consecutive rows (in LDS).  Stage 2 forms
// each sampled row k = (k_hi, k_lo) as sum_{i_hi} (-1)^{popc(k_hi & i_hi)}
// Y[i_hi * B + k_lo], reading each needed row of Y once per column block.
// ---------------------------------------------------------------------------
__global__ void srht_rows_kernel(int* idx, int64_t m, int64_t n, uint32_t seed) {
  const int64_t k = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (k < m) idx[k] = (int)(murmur3_u32((uint32_t)k, seed + kSrhtSampleSeedOffset) & (uint32_t)(n - 1));
}

constexpr int kFwhtW = 16;  // columns per stage-1 tile

template <typename TA, typename TY>
__global__ __launch_bounds__(kBlock) void srht_stage1(const TA* __restrict__ A, int64_t lda,
                                                      int64_t d, int logB, uint32_t seed,
                                                      TY* __restrict__ Y, int64_t ldy) {
  extern __shared__ unsigned char smem_raw[];
  TY* T = (TY*)smem_raw;  // B x kFwhtW
  const int B = 1 << logB;
  const int64_t row0 = (int64_t)blockIdx.y * B;
  const int64_t c0 = (int64_t)blockIdx.x * kFwhtW;
  for (int e = threadIdx.x; e < B * kFwhtW; e += kBlock) {
    const int r = e / kFwhtW, c = e % kFwhtW;
    const int64_t gr = row0 + r, gc = c0 + c;
    TY v = TY(0);
    if (gc < d) {
      v = (TY)A[gr * lda + gc];
      if (murmur3_u32((uint32_t)gr, seed) >> 31) v = -v;
    }
    T[e] = v;
  }
  __syncthreads();
  for (int h = 1; h < B; h <<= 1) {
    for (int p = threadIdx.x; p < (B / 2) * kFwhtW; p += kBlock) {
      const int c = p % kFwhtW, q = p / kFwhtW;
      const int i = (q / h) * 2 * h + (q % h);
      const TY u = T[i * kFwhtW + c], v = T[(i + h) * kFwhtW + c];
      T[i * kFwhtW + c] = u + v;
      T[(i + h) * kFwhtW + c] = u - v;
    }
    __syncthreads();
  }
  for (int e = threadIdx.x; e < B * kFwhtW; e += kBlock) {
    const int r = e / kFwhtW, c = e % kFwhtW;
    const int64_t gc = c0 + c;
    if (gc < d) Y[(row0 + r) * ldy + gc] = T[e];
  }
}

// Stage 1 for blocks of 512 rows: the 9 butterfly levels of H_512 split as
// 4 levels in registers on rows s + 32 i (i = 0..15, bits 5..8 of the row),
// one transpose through LDS, then 5 levels in registers on rows 32 g + i
// (i = 0..31, bits 0..4).  W columns per workgroup (16 for FP64 A, 32 for
// FP32 A, i.e. 128-byte row segments).
template <typename T, int N>
__device__ __forceinline__ void fwht_regs(T (&x)[N]) {
#pragma unroll
  for (int h = 1; h < N; h <<= 1) {
#pragma unroll
    for (int j = 0; j < N; ++j) {
      if ((j & h) == 0) {
        const T a = x[j], b = x[j + h];
        x[j] = a + b;
        x[j + h] = a - b;
      }
    }
  }
}

template <typename TA, typename TY>
__global__ __launch_bounds__(kBlock) void srht_stage1_b512(const TA* __restrict__ A, int64_t lda,
                                                           int64_t d, uint32_t seed,
                                                           TY* __restrict__ Y, int64_t ldy) {
  // 32 columns when the transform runs in FP32 (256-byte row segments of FP64 A),
  // else 16 (the LDS tile stays at ~66 KiB either way)
  constexpr int W = sizeof(TY) == 4 ? 32 : 16;
  constexpr int C1 = W / 8;   // columns per thread, phase 1
  constexpr int C2 = W / 16;  // columns per thread, phase 2
  constexpr int PAD = 1;
  __shared__ TY T[512][W + PAD];
  const int64_t row0 = (int64_t)blockIdx.y * 512;  // column blocks vary fastest, so
  const int64_t c0 = (int64_t)blockIdx.x * W;       // concurrent workgroups cover whole rows
  const int t = threadIdx.x;
  {
    const int cp = t % 8, sl = t / 8;  // column group, row slot 0..31
    TY x[C1][16];
#pragma unroll
    for (int i = 0; i < 16; ++i) {
      const int64_t gr = row0 + sl + 32 * i;
      const TA* src = A + gr * lda + c0 + C1 * cp;
      TA v[C1];
      if (c0 + C1 * cp + C1 <= d) {
        VecLoad<TA, C1, true>::run(src, v);  // one 16-byte load
      } else {
#pragma unroll
        for (int q = 0; q < C1; ++q) v[q] = (c0 + C1 * cp + q < d) ? src[q] : TA(0);
      }
      const bool neg = (murmur3_u32((uint32_t)gr, seed) >> 31) != 0;
#pragma unroll
      for (int q = 0; q < C1; ++q) x[q][i] = neg ? -(TY)v[q] : (TY)v[q];
    }
#pragma unroll
    for (int q = 0; q < C1; ++q) fwht_regs<TY, 16>(x[q]);
#pragma unroll
    for (int i = 0; i < 16; ++i)
#pragma unroll
      for (int q = 0; q < C1; ++q) T[sl + 32 * i][C1 * cp + q] = x[q][i];
  }
  __syncthreads();
  {
    const int c = C2 * (t % 16), g = t / 16;  // first column (C2 adjacent), row group 0..15
    TY y[C2][32];
#pragma unroll
    for (int i = 0; i < 32; ++i)
#pragma unroll
      for (int q = 0; q < C2; ++q) y[q][i] = T[32 * g + i][c + q];
#pragma unroll
    for (int q = 0; q < C2; ++q) fwht_regs<TY, 32>(y[q]);
#pragma unroll
    for (int i = 0; i < 32; ++i) {
      TY* dst = Y + (row0 + 32 * g + i) * ldy + c0 + c;
      if (c0 + c + C2 <= d) {
#pragma unroll
        for (int q = 0; q < C2; ++q) dst[q] = y[q][i];
      } else {
#pragma unroll
        for (int q = 0; q < C2; ++q)
          if (c0 + c + q < d) dst[q] = y[q][i];
      }
    }
  }
}

constexpr int kS2Cols = 64;    // columns per stage-2 workgroup
constexpr int kS2Chunk = 8;    // samples accumulated together
constexpr int kS2Cap = 512;    // sample list capacity

template <typename TY, typename TS>
__global__ __launch_bounds__(kBlock) void srht_stage2(const TY* __restrict__ Y, int64_t ldy,
                                                      int64_t d, int logB, int64_t nhi,
                                                      const int* __restrict__ idx, int64_t m,
                                                      TS* __restrict__ SA, int64_t ldsa,
                                                      double scale) {
  __shared__ int s_list[kS2Cap];
  __shared__ int s_wcnt[kWavesPerBlock];
  __shared__ TY s_red[kWavesPerBlock][kS2Chunk][kS2Cols];
  const int B = 1 << logB;
  const int klo = blockIdx.y;  // column blocks vary fastest (whole rows of Y in flight)
  const int64_t col = (int64_t)blockIdx.x * kS2Cols + (threadIdx.x & (kS2Cols - 1));
  const int rg = threadIdx.x >> 6;  // row group = wave
  const int lane = lane_id();
  int cnt = 0;

  auto process = [&](int count) {
    for (int s0 = 0; s0 < count; s0 += kS2Chunk) {
      const int ns = min(kS2Chunk, count - s0);
      int khi[kS2Chunk];
      TY acc[kS2Chunk];
#pragma unroll
      for (int s = 0; s < kS2Chunk; ++s) {
        khi[s] = (s < ns) ? (idx[s_list[s0 + s]] >> logB) : 0;
        acc[s] = TY(0);
      }
      if (col < d) {
        constexpr int U = 8;  // rows loaded together per thread
        for (int64_t ih0 = rg; ih0 < nhi; ih0 += (int64_t)U * kWavesPerBlock) {
          TY y[U];
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const int64_t ih = ih0 + (int64_t)u * kWavesPerBlock;
            y[u] = (ih < nhi) ? Y[(ih * B + klo) * ldy + col] : TY(0);
          }
#pragma unroll
          for (int u = 0; u < U; ++u) {
            const unsigned ih = (unsigned)(ih0 + (int64_t)u * kWavesPerBlock);
#pragma unroll
            for (int s = 0; s < kS2Chunk; ++s) {
              if (s < ns) {  // uniform: the chunk's sample count
                const int par = __popc((unsigned)khi[s] & ih) & 1;
                acc[s] += par ? -y[u] : y[u];
              }
            }
          }
        }
      }
#pragma unroll
      for (int s = 0; s < kS2Chunk; ++s) s_red[rg][s][lane] = acc[s];
      __syncthreads();
      if (rg == 0 && col < d) {
        for (int s = 0; s < ns; ++s) {
          TY t = s_red[0][s][lane];
#pragma unroll
          for (int g = 1; g < kWavesPerBlock; ++g) t += s_red[g][s][lane];
          SA[(int64_t)s_list[s0 + s] * ldsa + col] = (TS)((double)t * scale);
        }
      }
      __syncthreads();
    }
  };

  for (int64_t w0 = 0; w0 < m; w0 += kBlock) {
    const int64_t k = w0 + threadIdx.x;
    const bool match = (k < m) && ((idx[k] & (B - 1)) == klo);
    const unsigned long long ball = __ballot(match);
    const int before = __popcll(ball & ((1ull << lane) - 1ull));
    if (lane == 0) s_wcnt[rg] = __popcll(ball);
    __syncthreads();
    int off = 0, total = 0;
    for (int g = 0; g < kWavesPerBlock; ++g) {
      if (g < rg) off += s_wcnt[g];
      total += s_wcnt[g];
    }
    if (cnt + total > kS2Cap) {
      process(cnt);
      cnt = 0;
    }
    if (match) s_list[cnt + off + before] = (int)k;
    cnt += total;
    __syncthreads();
  }
  if (cnt > 0) process(cnt);
}

// ---------------------------------------------------------------------------
// SRHT in one read of A.  A workgroup of 512 threads owns a strip of 16
// columns and a range of blocks of B = 2^LOGB consecutive rows.  For each block
// i_hi it applies D and the length-B transform over i_lo (registers, one LDS
// transpose), leaving T[k_lo] = sum_{i_lo} (-1)^{popc(k_lo & i_lo)} (D A)[i_hi B + i_lo]
// in LDS, and then adds every sampled row k = (k_hi, k_lo) with its sign:
//     acc_k += (-1)^{popc(k_hi & i_hi)} T[k_lo],
// so that after all blocks acc_k = ((H D A)[idx_k]) restricted to the strip.
// The transform's threads (c, g), c = t % 16, g = t / 16, hold column c of R rows; the
// accumulation's threads own the 16 bytes of columns from VC (t % (16 / VC)) of NS samples,
// in registers, so that one LDS read of T, one of the sample's word (its row offset in T and
// block index k_hi) and one sign serve VC = 4 (FP32) or 2 (FP64) columns.  The next block's
// rows are loaded while the current one is transformed and accumulated.  The partial
// sums of the workgroup's block range go to P[part] (or, with one range per
// strip, scaled straight to SA).
//
// Bound: the 128-byte row segments' rate from memory and, with many samples, the LDS reads
// and arithmetic of the accumulation (two waves per SIMD).  2^18 x 2048 FP64, m = 2048 in FP32:
// 1065 us with one column per accumulating thread, 880 us now (4.9 TB/s); 2^16 x 4096,
// m = 4096: 555 us (1430 in two stages); 2^17 x 1500 FP32, m = 3000: 1003 us in two stages,
// 420 before neighbouring strips shared an L2, 341 now.
// ---------------------------------------------------------------------------
// Mixed CountSketch -> Gaussian: the FP32 bucket sums CA enter the Gaussian
// stage as three BF16 terms (hi + mid + lo), so that the BF16 products keep
// CA's FP32 accuracy; rounding CA itself to BF16 (2^-9 relative) perturbs
// the sketched Hessian by more than lambda on ill-conditioned problems.
constexpr int kCountGaussTerms = 3;

constexpr int kFusedThreads = 512;
constexpr int kBufferRsrcWord3 = 0x00020000;  // raw 32-bit buffer data (gfx9 family)
constexpr int kBufferNt = 2;                  // cache policy: non-temporal
constexpr int kFusedW = 16;       // columns per strip
// columns per accumulating thread (16 bytes)
template <typename TY>
constexpr int fused_vc() { return 16 / (int)sizeof(TY); }
// Rows of T lie one after the other in LDS with an unused one after every R (R rows per
// thread and phase): both the rows g, g + 1, .. that a wave's first phase stores together and
// the rows R g, R (g + 1), .. of its second phase then fall into different banks.
MIHS_HOST_DEVICE constexpr int fused_row(int r, int R) { return r + r / R; }
// row stride of the partial sums: 16-byte rows in either type
inline int64_t fused_ldp(int64_t d) { return (d + 3) / 4 * 4; }
// threads that share a sample set
template <typename TY>
constexpr int fused_groups() { return kFusedThreads * fused_vc<TY>() / kFusedW; }

// Strip and block range of a workgroup.  A strip's 16 columns of FP32 rows are half a
// 128-byte line, so two neighbouring strips of the same range go to workgroups 8 apart:
// dispatched together to the same XCD, they share the lines in its L2 (apart, every line came
// from memory twice).
template <typename TA>
constexpr int fused_pair() { return sizeof(TA) == 4 ? 2 : 1; }
template <typename TA>
__device__ __forceinline__ bool fused_place(int strips, int nparts, int& strip, int& part) {
  int b = blockIdx.x, sub = 0, n = strips;
  if (fused_pair<TA>() == 2) {
    sub = b / kXcds % 2;
    b = b / (2 * kXcds) * kXcds + b % kXcds;
    n = (strips + 1) / 2;
  }
  strip = b % n * fused_pair<TA>() + sub;
  part = b / n;
  return strip < strips && part < nparts;
}

// sign words: bit j of word w is set iff D_{32 w + j} = -1
__global__ void srht_sign_words_kernel(uint32_t* words, int64_t nwords, uint32_t seed) {
  const int64_t w = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (w >= nwords) return;
  uint32_t v = 0u;
  for (int j = 0; j < 32; ++j)
    v |= (murmur3_u32((uint32_t)(w * 32 + j), seed) >> 31) << j;
  words[w] = v;
}

// WIDE: rows so long that a block spans 2 GiB and more, addressed by 64-bit pointers instead of
// 32-bit offsets into the block.
template <typename TA, typename TY, int LOGB, int NS, typename TS, bool WIDE>
__global__ __launch_bounds__(kFusedThreads) void srht_fused_kernel(
    const TA* __restrict__ A, int64_t lda, int64_t d, const uint32_t* __restrict__ signw,
    const int* __restrict__ idx, int64_t m, int64_t nblk, int nparts, TY* __restrict__ P,
    int64_t ldp, TS* __restrict__ SA, int64_t ldsa, double scale) {
  constexpr int B = 1 << LOGB;
  constexpr int R = B * kFusedW / kFusedThreads;  // rows per thread per phase (16 or 32)
  static_assert(R == 16 || R == 32, "block shape");
  constexpr int VC = fused_vc<TY>(), GS = fused_groups<TY>();
  typedef TY vec_t __attribute__((ext_vector_type(VC)));
  extern __shared__ unsigned char smem_raw[];
  TY* T = (TY*)smem_raw;  // fused_row(B) x kFusedW
  // per sample: k_hi (low 16 bits) and its row's offset in T in 16-byte units (high 16)
  uint32_t* s_smp = (uint32_t*)(T + (size_t)fused_row(B, R) * kFusedW);      // GS * NS
  const int t = threadIdx.x;
  const int c = t % kFusedW, g = t / kFusedW;              // g in [0, 32)
  const int cs = VC * (t % (kFusedW / VC)), gs = t / (kFusedW / VC);  // accumulation
  int strip, part;
  if (!fused_place<TA>((int)((d + kFusedW - 1) / kFusedW), nparts, strip, part)) return;
  const int64_t col = (int64_t)strip * kFusedW + c;
  const bool col_ok = col < d;
  const int64_t b0 = nblk * part / nparts, b1 = nblk * (part + 1) / nparts;

  for (int k = t; k < GS * NS; k += kFusedThreads) {
    const int v = k < m ? idx[k] : 0;
    const uint32_t khi = k < m ? (uint32_t)(v >> LOGB) : 0u;
    s_smp[k] = (uint32_t)(fused_row(v & (B - 1), R) * (kFusedW / VC)) << 16 | khi;
  }
  vec_t acc[NS];
#pragma unroll
  for (int j = 0; j < NS; ++j) acc[j] = (vec_t)(TY(0));

  // rows g + 32 i of block b, this thread's column, as buffer loads: the
  // block's base in a buffer resource, row 32 i's byte offset in a scalar
  // register and one per-lane byte offset, so that the row addresses do not
  // each occupy a pair of vector registers.  Non-temporal for FP64 (each line is
  // read once; two strips share one of FP32).
  // Every offset stays below the block's B rows (checked against num_records).
  TA xa[R];
  const uint32_t lane_off = (uint32_t)(((int64_t)g * lda + (col_ok ? col : 0)) * sizeof(TA));
  const int32_t row32 = (int32_t)(32 * lda * (int64_t)sizeof(TA));  // bytes between rows g + 32 i
  const int32_t blk_bytes = (int32_t)(B * lda * (int64_t)sizeof(TA));
  auto load_block = [&](int64_t b) {
    if constexpr (WIDE) {
      const TA* p = A + (b * B + g) * lda + (col_ok ? col : 0);
#pragma unroll
      for (int i = 0; i < R; ++i)
        xa[i] = sizeof(TA) == 8 ? __builtin_nontemporal_load(p + (int64_t)(32 * i) * lda)
                                : p[(int64_t)(32 * i) * lda];
    } else {
      const __amdgpu_buffer_rsrc_t rs = __builtin_amdgcn_make_buffer_rsrc(
          (void*)(A + b * B * lda), (short)0, blk_bytes, kBufferRsrcWord3);
#pragma unroll
      for (int i = 0; i < R; ++i) {
        if constexpr (sizeof(TA) == 8) {
          const auto v = __builtin_amdgcn_raw_buffer_load_b64(rs, lane_off, i * row32, kBufferNt);
          xa[i] = __builtin_bit_cast(TA, v);
        } else {
          const auto v = __builtin_amdgcn_raw_buffer_load_b32(rs, lane_off, i * row32, 0);
          xa[i] = __builtin_bit_cast(TA, v);
        }
      }
    }
  };
  if (b0 < b1) load_block(b0);
  for (int64_t b = b0; b < b1; ++b) {
    // phase 1: D, then the butterflies of row bits 5 .. LOGB-1 (register index bits)
    TY x[R];
    const uint32_t* sw = signw + b * (B / 32);
#pragma unroll
    for (int i = 0; i < R; ++i) {
      const bool neg = (sw[i] >> g) & 1u;
      x[i] = neg ? -(TY)xa[i] : (TY)xa[i];
    }
    // the next block's rows as soon as this block's are in x, or (FP64 rows beside 96 and
    // more accumulators: the registers would spill) once the transform is done
    constexpr bool kLate = sizeof(TA) == 8 && sizeof(TY) == 4 && NS >= 24;
    if (!kLate && b + 1 < b1) load_block(b + 1);
    fwht_regs<TY, R>(x);
    lds_barrier();  // the previous block's accumulation has read T
#pragma unroll
    for (int i = 0; i < R; ++i) T[fused_row(g + 32 * i, R) * kFusedW + c] = x[i];
    lds_barrier();
    // phase 2: the butterflies of row bits 0 .. log2(R)-1 on rows R g + i
    {
      TY y[R];
#pragma unroll
      for (int i = 0; i < R; ++i) y[i] = T[((R + 1) * g + i) * kFusedW + c];
      fwht_regs<TY, R>(y);
      if constexpr (R == 16) {
        // row bit 4: rows 16 g + i and 16 (g ^ 1) + i live in threads t and t ^ 16
        // (the same wave)
        const bool upper = (g & 1) != 0;
#pragma unroll
        for (int i = 0; i < R; ++i) {
          const TY other = __shfl_xor(y[i], kFusedW, kWave);
          y[i] = upper ? other - y[i] : y[i] + other;
        }
      }
#pragma unroll
      for (int i = 0; i < R; ++i) T[((R + 1) * g + i) * kFusedW + c] = y[i];
    }
    if (kLate && b + 1 < b1) load_block(b + 1);
    lds_barrier();
    // every owned sample: acc_k += (-1)^{popc(k_hi & b)} T[k_lo][cs ..], NG samples
    // at a time (the empty asm keeps the compiler from hoisting every sample's LDS
    // reads at once, which would not fit in the registers).  The sign enters as a
    // factor of exactly +-1, one instruction per column.
    constexpr int NG = NS % 8 == 0 && (NS < 32 || sizeof(TA) == 4) ? 8 : 4;
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const uint32_t bb = (uint32_t)b;
    const char* Tc = (const char*)(T + cs);
    const uint32_t* smp = s_smp + gs * NS;
#pragma unroll
    for (int j0 = 0; j0 < NS; j0 += NG) {
      asm volatile("" ::: "memory");
      uint32_t w[NG];
#pragma unroll
      for (int j = 0; j < NG; j += 4) {
        const u32x4 x = *(const u32x4*)(smp + j0 + j);
#pragma unroll
        for (int i = 0; i < 4; ++i) w[j + i] = x[i];
      }
      vec_t v[NG];
#pragma unroll
      for (int j = 0; j < NG; ++j) v[j] = *(const vec_t*)(Tc + ((w[j] >> 12) & ~15u));
#pragma unroll
      for (int j = 0; j < NG; ++j) {
        const uint32_t neg = (uint32_t)__popc(w[j] & bb) << 31;  // b < 2^16
        TY sgn;
        if constexpr (sizeof(TY) == 4)
          sgn = __uint_as_float(0x3F800000u | neg);
        else
          sgn = __hiloint2double((int)(0x3FF00000u | neg), 0);
#pragma unroll
        for (int q = 0; q < VC; ++q) acc[j0 + j][q] += v[j][q] * sgn;
      }
    }
  }
  // 16 bytes per store (P's rows are padded to them, SA's begin on them): element by element,
  // a wave's store touches 64 places, and at few blocks that cost more than the transform
  // (2^16 x 16 FP64, m = 4096, in FP32: 46 us, 21 now; 4096 x 61, m = 2500: 21 and 11)
  typedef TS out_t __attribute__((ext_vector_type(VC)));
  const int64_t c0 = (int64_t)strip * kFusedW + cs;
  TY* Pp = nparts == 1 ? nullptr : P + (int64_t)part * m * ldp + c0;
#pragma unroll
  for (int j = 0; j < NS; ++j) {
    const int64_t k = (int64_t)gs * NS + j;
    if (k >= m || c0 >= d) continue;
    if (Pp) {
      *(vec_t*)(Pp + k * ldp) = acc[j];
    } else {
      out_t o;
#pragma unroll
      for (int q = 0; q < VC; ++q) o[q] = (TS)((double)acc[j][q] * scale);
      TS* dst = SA + k * ldsa + c0;
      if (c0 + VC <= d) {
        *(out_t*)dst = o;
      } else {
#pragma unroll
        for (int q = 0; q < VC; ++q)
          if (c0 + q < d) dst[q] = o[q];
      }
    }
  }
}

// SA[k][col] = scale * sum_{part} P[part][k][col], parts in order.
template <typename TY, typename TS>
__global__ void srht_parts_sum_kernel(const TY* __restrict__ P, int nparts, int64_t m, int64_t d,
                                      int64_t ldp, TS* __restrict__ SA, int64_t ldsa, double scale) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (e >= m * d) return;
  const int64_t k = e / d, col = e - k * d;
  TY s = P[k * ldp + col];
  for (int q = 1; q < nparts; ++q) s += P[((int64_t)q * m + k) * ldp + col];
  SA[k * ldsa + col] = (TS)((double)s * scale);
}

__global__ void zero_u32_kernel(unsigned* p, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = 0u;
}

// ---------------------------------------------------------------------------
// CountSketch: h = murmur3(i, seed), bucket = h mod m, sign = -1 iff bit 31.
// One kernel hashes the rows into slot lists, one per bucket and range of rows;
// then each (bucket, column block) sorts its lists ascending in LDS, range after
// range, and sums its rows in that order, so the result does not depend on
// scheduling.  A row's sign is hashed again where the row is summed (scalar
// work, one hash per wave and row).
//
// Bound: one read of A.  Slots of a fixed capacity need neither an offset scan
// nor a scatter launch with atomics of its own, and the list comes from LDS,
// so that the rows' 16-byte loads depend on nothing else:
// 500009 x 1000 FP32, m = 4000: 508 us with separate hash, scan, scatter, sort
// and 4-byte-load sum kernels, 400 now.  The work stays proportional to the rows at any number
// per bucket: 2^25 x 16 FP32 into 4500 buckets (7456 rows each, two ranges) 12 ms, 191 when
// every bucket hashed every row; 2^27 x 8 into 17000 46 ms, 2590 so and 1680 with the serial
// sort of long lists before.
// ---------------------------------------------------------------------------
constexpr int64_t kCsMaxMean = 7168;  // rows per list on average, so that a list fits in LDS
constexpr int64_t kCsFewBuckets = 100;  // fewer than this, of more rows, hash every row instead
constexpr int kCsBlock = kBlock;
constexpr int kCsRankSort = 512;      // lists up to this length are sorted by rank

// Row ranges (a multiple of kCsBlock rows each, but for the last) and the slots of a list: the
// mean row count plus seven standard deviations and a few, in fours (a list that overflows is replaced by
// hashing its range again, see cs_accum_kernel).
struct CsLists {
  int64_t ranges, rows, cap;
};
CsLists cs_lists(int64_t n, int64_t m) {
  CsLists c;
  const double mean = (double)n / (double)m;
  // With few buckets, hashing every row once per bucket costs less than the atomics on so few
  // counters and the sorting (8000 rows per bucket, 300 FP32 columns: 64 buckets 1.65 ms, by
  // lists 2.0; 128 buckets 2.28 and 2.06); it grows with the square of their number (4096
  // buckets, 16 columns: 174 and 12 ms).
  if (mean > (double)kCsMaxMean && m < kCsFewBuckets) return {1, n, 0};
  c.ranges = (int64_t)ceil(mean / (double)kCsMaxMean);
  c.rows = ((n + c.ranges - 1) / c.ranges + kCsBlock - 1) / kCsBlock * kCsBlock;
  c.ranges = (n + c.rows - 1) / c.rows;
  const double per = (double)std::min(c.rows, n) / (double)m;
  c.cap = ((int64_t)ceil(per + 7.0 * sqrt(per)) + 6 + 3) / 4 * 4;
  return c;
}
// LDS list length (entries): a power of two for the sort, and room for the rows that the
// hashing form collects between sums.
int64_t cs_list_len(int64_t cap) {
  int64_t p = 4 * kCsBlock;
  while (p < cap) p <<= 1;
  return p;
}

// hist and slots: [range][bucket]; range_blocks workgroups per range (0: one range)
__global__ __launch_bounds__(kCsBlock) void cs_hash_kernel(int64_t n, int64_t m, uint32_t seed,
                                                           unsigned range_blocks, unsigned cap,
                                                           unsigned* hist, unsigned* slots) {
  const int64_t i = (int64_t)blockIdx.x * kCsBlock + threadIdx.x;
  if (i >= n) return;
  const uint32_t h = murmur3_u32((uint32_t)i, seed);
  int64_t list = h % (uint32_t)m;
  if (range_blocks) list += blockIdx.x / range_blocks * m;
  const unsigned pos = atomicAdd(&hist[list], 1u);
  if (pos < cap) slots[list * cap + pos] = (unsigned)i;
}

// acc += the rows of list[0..cnt), in order, this thread's V columns.
template <typename TA, typename TAcc, int V, int U>
__device__ __forceinline__ void cs_add_rows(const TA* __restrict__ A, int64_t lda, int64_t c,
                                            uint32_t seed, const unsigned* list, int cnt,
                                            TAcc (&acc)[V]) {
  auto take = [&](int p, TA (&v)[V]) {
    const unsigned row = (unsigned)__builtin_amdgcn_readfirstlane((int)list[p]);
    VecLoad<TA, V, true>::run(A + (int64_t)row * lda + c, v);
    return (murmur3_u32(row, seed) >> 31) != 0;
  };
  int p = 0;
  for (; p + U <= cnt; p += U) {
    TA v[U][V];
    bool neg[U];
#pragma unroll
    for (int t = 0; t < U; ++t) neg[t] = take(p + t, v[t]);
#pragma unroll
    for (int t = 0; t < U; ++t)
#pragma unroll
      for (int q = 0; q < V; ++q) acc[q] += neg[t] ? -(TAcc)v[t][q] : (TAcc)v[t][q];
  }
  for (; p < cnt; ++p) {
    TA v[V];
    const bool neg = take(p, v);
#pragma unroll
    for (int q = 0; q < V; ++q) acc[q] += neg ? -(TAcc)v[q] : (TAcc)v[q];
  }
}

// One workgroup per (bucket, kCsBlock * V columns); a thread owns the 16 bytes of A's rows
// from column c (rows are 16-byte aligned, so the last chunk stays inside a row's span).
// LDS: 2 * list_len entries.  ONE: a single range of rows (as a loop it costs buckets of a row or
// two up to 10%: 5000 x 4096 FP64 into 4999 buckets 106 us, 118 as a loop).
template <typename TA, typename TAcc, typename TOut, bool ONE>
__global__ __launch_bounds__(kCsBlock) void cs_accum_kernel(
    const TA* __restrict__ A, int64_t lda, int64_t n, int64_t d, int64_t m, uint32_t seed,
    unsigned cap, int list_len, const unsigned* hist, const unsigned* slots,
    TOut* __restrict__ out, int64_t ldo, int ranges, int64_t range_rows) {
  constexpr int V = 16 / (int)sizeof(TA);
  extern __shared__ unsigned cs_lds[];
  unsigned* list = cs_lds;
  unsigned* sorted = cs_lds + list_len;
  __shared__ int s_cnt[kCsBlock / kWave];
  const unsigned bucket = blockIdx.x;
  const int64_t c = ((int64_t)blockIdx.y * kCsBlock + threadIdx.x) * V;
  const bool on = c < d;
  TAcc acc[V];
#pragma unroll
  for (int q = 0; q < V; ++q) acc[q] = TAcc(0);
  auto sum_range = [&](int r) {
    const int64_t which = ONE ? bucket : (int64_t)r * m + bucket;
    const unsigned total = cap ? hist[which] : 0xFFFFFFFFu;
    if (total <= cap) {
      const unsigned* mine = slots + which * cap;
      const int cnt = (int)total;
      if (cnt <= kCsRankSort) {
        // each element's rank is the number of smaller ones (all rows differ)
        for (int i = threadIdx.x; i < cnt; i += kCsBlock) list[i] = mine[i];
        __syncthreads();
        for (int i = threadIdx.x; i < cnt; i += kCsBlock) {
          const unsigned v = list[i];
          int rank = 0;
#pragma unroll 8
          for (int j = 0; j < cnt; ++j) rank += list[j] < v;
          sorted[rank] = v;
        }
        __syncthreads();
      } else {
        // bitonic, padded to a power of two (at most list_len)
        int P = 1;
        while (P < cnt) P <<= 1;
        for (int i = threadIdx.x; i < P; i += kCsBlock) sorted[i] = i < cnt ? mine[i] : 0xFFFFFFFFu;
        __syncthreads();
        for (int k = 2; k <= P; k <<= 1)
          for (int j = k >> 1; j > 0; j >>= 1) {
            for (int i = threadIdx.x; i < P / 2; i += kCsBlock) {
              const int lo = (i / j) * 2 * j + (i % j), hi = lo + j;
              const unsigned a = sorted[lo], b = sorted[hi];
              if ((a > b) == ((lo & k) == 0)) {
                sorted[lo] = b;
                sorted[hi] = a;
              }
            }
            __syncthreads();
          }
      }
      if (on) cs_add_rows<TA, TAcc, V, 8>(A, lda, c, seed, sorted, cnt, acc);
    } else {
      // no list: hash every row of the range, collect this bucket's in ascending order and sum
      // them whenever the list is nearly full
      const int64_t end = ONE ? n : min(n, (r + 1) * range_rows);
      const int wave = wave_id(), lane = lane_id();
      int cnt = 0;
      for (int64_t r0 = r * range_rows; r0 < end; r0 += kCsBlock) {
        const int64_t i = r0 + threadIdx.x;
        const uint32_t h = murmur3_u32((uint32_t)i, seed);
        const bool match = i < end && h % (uint32_t)m == bucket;
        const unsigned long long ball = __ballot(match);
        if (lane == 0) s_cnt[wave] = __popcll(ball);
        __syncthreads();
        int off = cnt, all = cnt;
#pragma unroll
        for (int w = 0; w < kCsBlock / kWave; ++w) {
          if (w < wave) off += s_cnt[w];
          all += s_cnt[w];
        }
        if (match)
          list[off + __popcll(ball & ((1ull << lane) - 1ull))] = (unsigned)i;
        cnt = all;
        __syncthreads();
        if (cnt + kCsBlock > list_len || r0 + kCsBlock >= end) {
          if (on) cs_add_rows<TA, TAcc, V, 16>(A, lda, c, seed, list, cnt, acc);
          cnt = 0;
          __syncthreads();
        }
      }
    }
  };
  if constexpr (ONE) {
    sum_range(0);
  } else {
    for (int r = 0; r < ranges; ++r) {
      if (r > 0) __syncthreads();  // the last range's rows are summed
      sum_range(r);
    }
  }
  if (on) {
    TOut* o = out + (int64_t)bucket * ldo + c;
#pragma unroll
    for (int q = 0; q < V; ++q)
      if (c + q < d) o[q] = (TOut)acc[q];
  }
}

// ---------------------------------------------------------------------------
// Gaussian:  S (M x K) with S_ij = N(0,1) * scale drawn from Philox element
// i*K + j.  FP64 S (plain) is laid out in panels of 16 k (element (i, k) at
// (k / 16) * 16 M + 16 i + k % 16: a step's tile of the product is one
// contiguous range), BF16 bits (mixed) row-major with row stride lds.  Columns
// K .. kpad-1 (kpad = lds, or K rounded up to 16) are zero: the thread that
// draws a row's last entry writes them.
// ---------------------------------------------------------------------------
template <typename TSel>
__global__ void gauss_gen_kernel(TSel* S, int64_t M, int64_t K, int64_t kpad, uint32_t seed,
                                 uint64_t stream, double scale) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;  // one Philox block each
  const int64_t total = M * K;
  const int64_t first = e * 4;
  if (first >= total) return;
  // FP64 draws for the FP64 sketch; FP32 draws for the BF16 sketch (rounded to
  // 8 significant bits anyway)
  double z[4];
  float zf[4];
  if constexpr (sizeof(TSel) == 8)
    gaussian_block(seed, stream, (uint64_t)e, z);
  else
    gaussian_block_f32(seed, stream, (uint64_t)e, zf);
  const float scale_f = (float)scale;
  auto at = [&](int64_t i, int64_t j) {
    return sizeof(TSel) == 8 ? (j / kGemmK) * kGemmK * M + i * kGemmK + j % kGemmK : i * kpad + j;
  };
  // row and column of the first element (one division per thread, 32-bit where the index
  // allows it), then step along the row with wrap-around
  int64_t i, j;
  if (total <= 0xFFFFFFFFll) {
    i = (uint32_t)first / (uint32_t)K;
    j = (uint32_t)first - (uint32_t)i * (uint32_t)K;
  } else {
    i = first / K;
    j = first - i * K;
  }
#pragma unroll
  for (int t = 0; t < 4; ++t) {
    if (first + t < total) {
      if constexpr (sizeof(TSel) == 8) {
        S[at(i, j)] = z[t] * scale;
      } else {
        S[at(i, j)] = bf16_rne(zf[t] * scale_f);
      }
      if (++j == K) {
        for (; j < kpad; ++j) S[at(i, j)] = TSel(0);
        j = 0;
        ++i;
      }
    }
  }
}

// P[z] (M x N) = X[:, kz] Y[kz, :], one 64 x BN tile per workgroup (gemm64.hpp); X by
// operand type (FP64 panels of S, or the rows of A), Y k-major.
template <typename OX, typename OY, int BN, typename TX, typename TY>
__global__ __launch_bounds__(kBlock) void gemm_f64_kernel(const TX* __restrict__ X, int64_t ldx,
                                                          int64_t M, int64_t K,
                                                          const TY* __restrict__ Y, int64_t ldy,
                                                          int64_t N, int64_t kchunk,
                                                          double* __restrict__ P) {
  constexpr int BM = 64;
  __shared__ __attribute__((aligned(16))) double lds[gemm64_lds<OX, OY>()];
  const int64_t m0 = (int64_t)blockIdx.x * BM, n0 = (int64_t)blockIdx.y * BN;
  const int64_t kb = (int64_t)blockIdx.z * kchunk, ke = min(K, kb + kchunk);
  f64x4 acc[BM / 32][BN / 32];
  gemm64_tile<OX, OY, BM, BN>(X, ldx, m0, M, Y, ldy, n0, N, kb, ke, lds, acc);
  const int lane = lane_id(), wave = wave_id();
  double* Pz = P + (int64_t)blockIdx.z * M * N;
#pragma unroll
  for (int a = 0; a < BM / 32; ++a)
#pragma unroll
    for (int b = 0; b < BN / 32; ++b)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = m0 + (wave >> 1) * (BM / 2) + 16 * a + (lane >> 4) + 4 * r;
        const int64_t col = n0 + (wave & 1) * (BN / 2) + 16 * b + (lane & 15);
        if (row < M && col < N) Pz[row * N + col] = acc[a][b][r];
      }
}

// y[r] = A[r, :] . w, four rows per wave: each 16 bytes of w serve four of A.  Bound by
// the one read of A (2^16 x 4096 FP64: 0.35 ms at the ~6 TB/s of a read stream; as a 64-wide
// matrix product with one useful column it took 1.24 ms).
template <typename TA>
__global__ __launch_bounds__(kBlock) void rowdot_kernel(const TA* __restrict__ A, int64_t n,
                                                        int64_t d, int64_t lda,
                                                        const double* __restrict__ w,
                                                        double* __restrict__ y) {
  constexpr int R = 4, V = 16 / (int)sizeof(TA);
  const int lane = lane_id();
  const int64_t r0 = ((int64_t)blockIdx.x * kWavesPerBlock + wave_id()) * R;
  if (r0 >= n) return;
  const TA* row[R];
  double acc[R];
#pragma unroll
  for (int t = 0; t < R; ++t) {
    row[t] = A + min(r0 + t, n - 1) * lda;
    acc[t] = 0.0;
  }
  int64_t c = (int64_t)lane * V;
#pragma unroll 2
  for (; c + V <= d; c += kWave * V) {
    TA a[R][V];
    double wv[V];
#pragma unroll
    for (int t = 0; t < R; ++t) VecLoad<TA, V, true>::run(row[t] + c, a[t]);
#pragma unroll
    for (int q = 0; q < V; ++q) wv[q] = w[c + q];
#pragma unroll
    for (int t = 0; t < R; ++t)
#pragma unroll
      for (int q = 0; q < V; ++q) acc[t] += (double)a[t][q] * wv[q];
  }
#pragma unroll
  for (int q = 0; q < V; ++q)
    if (c + q < d) {
#pragma unroll
      for (int t = 0; t < R; ++t) acc[t] += (double)row[t][c + q] * w[c + q];
    }
#pragma unroll
  for (int t = 0; t < R; ++t) {
    const double s = wave_sum(acc[t]);
    if (lane == 0 && r0 + t < n) y[r0 + t] = s;
  }
}

// Bt (N x ldbt, BF16 bits) = B^T rounded to BF16 (round to nearest even of the
// exact value), zero for k in [K, ldbt): the sketch GEMM's right operand with k
// contiguous, made once per sketch so that the GEMM streams 2-byte values
// instead of re-reading (and re-rounding) B for every 128-row tile of S.
// 64 x 64 tiles through LDS: reads along n, writes along k.
template <typename TB>
__global__ __launch_bounds__(kBlock) void bf16_transpose_kernel(const TB* __restrict__ B,
                                                                int64_t K, int64_t N, int64_t ldb,
                                                                uint16_t* __restrict__ Bt,
                                                                int64_t ldbt) {
  __shared__ uint16_t tile[64][66];
  const int64_t k0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int kk = ty + 4 * i;
    const int64_t gk = k0 + kk, gn = n0 + tx;
    tile[kk][tx] = (gk < K && gn < N) ? bf16_rne(B[gk * ldb + gn]) : (uint16_t)0;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < 16; ++i) {
    const int nn = ty + 4 * i;
    const int64_t gn = n0 + nn, gk = k0 + tx;
    if (gn < N && gk < ldbt) Bt[gn * ldbt + gk] = tile[tx][nn];
  }
}

// The three-term BF16 split of B^T for products that must keep B's FP32
// accuracy: Bt_t (t = 0, 1, 2; stride part_stride) holds hi, mid, lo with
// hi = bf16(v), mid = bf16(v - hi), lo = bf16(v - hi - mid) for v = B[k, n]
// (each difference is exact in FP32), so that hi + mid + lo equals v to about
// 2^-24 relative and S (hi + mid + lo) is S B to FP32 accuracy.
__global__ __launch_bounds__(kBlock) void bf16_split3_transpose_kernel(
    const float* __restrict__ B, int64_t K, int64_t N, int64_t ldb, uint16_t* __restrict__ Bt,
    int64_t ldbt, int64_t part_stride) {
  __shared__ uint16_t tile[3][64][66];
  const int64_t k0 = (int64_t)blockIdx.y * 64, n0 = (int64_t)blockIdx.x * 64;
  const int tx = threadIdx.x % 64, ty = threadIdx.x / 64;
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int kk = ty + 4 * i;
    const int64_t gk = k0 + kk, gn = n0 + tx;
    uint16_t h = 0, mi = 0, lo = 0;
    if (gk < K && gn < N) {
      const float v = B[gk * ldb + gn];
      h = bf16_rne(v);
      const float r1 = v - __uint_as_float((uint32_t)h << 16);
      mi = bf16_rne(r1);
      const float r2 = r1 - __uint_as_float((uint32_t)mi << 16);
      lo = bf16_rne(r2);
    }
    tile[0][kk][tx] = h;
    tile[1][kk][tx] = mi;
    tile[2][kk][tx] = lo;
  }
  __syncthreads();
#pragma unroll 4
  for (int i = 0; i < 16; ++i) {
    const int nn = ty + 4 * i;
    const int64_t gn = n0 + nn, gk = k0 + tx;
    if (gn < N && gk < ldbt) {
      Bt[gn * ldbt + gk] = tile[0][tx][nn];
      Bt[part_stride + gn * ldbt + gk] = tile[1][tx][nn];
      Bt[2 * part_stride + gn * ldbt + gk] = tile[2][tx][nn];
    }
  }
}

// P[z] (M x N) = S[:, kz] B[kz, :] with BF16 inputs and FP32 accumulation, B
// given as Bt = B^T in BF16 (both operands k-contiguous)
// (v_mfma_f32_16x16x32_bf16: lane l holds 8 consecutive k, 8(l/16)..+7, of
// row l%16 (A) / column l%16 (B); result register r of lane l is row
// 4(l/16) + r, column l%16).  128 x 128 tiles, 64 k per step; the global loads
// of step t + 1 are in flight in registers while step t is multiplied from LDS.
__global__ __launch_bounds__(kBlock) void gemm_bf16_kernel(const uint16_t* __restrict__ S,
                                                           int64_t lds, int64_t M, int64_t K,
                                                           const uint16_t* __restrict__ Bt,
                                                           int64_t ldbt, int64_t N,
                                                           int64_t kchunk, float* __restrict__ P) {
  constexpr int BM = 128, BN = 128, BK = 64, PAD = 8;
  constexpr int Q = BM * (BK / 8) / kBlock;  // 16-byte chunks per operand, thread and step
  static_assert(BM == BN && Q == 4, "tile shape");
  __shared__ __attribute__((aligned(16))) uint16_t As[BM][BK + PAD];
  __shared__ __attribute__((aligned(16))) uint16_t Bs[BN][BK + PAD];
  const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
  const int64_t kb = (int64_t)blockIdx.z * kchunk, ke = min(K, kb + kchunk);
  const int lane = lane_id(), wave = wave_id();
  const int wr = wave >> 1, wc = wave & 1;
  f32x4 acc[4][4];
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j) acc[i][j] = (f32x4){0.f, 0.f, 0.f, 0.f};
  uint4 sreg[Q], breg[Q];
  auto gload = [&](int64_t k0) {
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int e = (int)threadIdx.x + t * kBlock;
      const int r = e / (BK / 8), q = e % (BK / 8);
      const int64_t gk = k0 + 8 * q;
      uint4 v = make_uint4(0u, 0u, 0u, 0u), w = make_uint4(0u, 0u, 0u, 0u);
      if (gk < ke) {
        const int64_t gr = m0 + r, gn = n0 + r;
        if (gr < M) {
          v = *(const uint4*)(S + gr * lds + gk);
          if (gk + 8 > ke) {  // zero the k's beyond this split's end (in S only)
            union {
              uint4 u;
              uint16_t h[8];
            } x;
            x.u = v;
#pragma unroll
            for (int u = 0; u < 8; ++u)
              if (gk + u >= ke) x.h[u] = 0;
            v = x.u;
          }
        }
        if (gn < N) w = *(const uint4*)(Bt + gn * ldbt + gk);
      }
      sreg[t] = v;
      breg[t] = w;
    }
  };
  auto lstore = [&]() {
#pragma unroll
    for (int t = 0; t < Q; ++t) {
      const int e = (int)threadIdx.x + t * kBlock;
      const int r = e / (BK / 8), q = e % (BK / 8);
      *(uint4*)&As[r][8 * q] = sreg[t];
      *(uint4*)&Bs[r][8 * q] = breg[t];
    }
  };
  if (kb < ke) gload(kb);
  for (int64_t k0 = kb; k0 < ke; k0 += BK) {
    __syncthreads();  // the previous step's products are done with As / Bs
    lstore();
    __syncthreads();
    if (k0 + BK < ke) gload(k0 + BK);  // in flight during this step's products
#pragma unroll
    for (int kk = 0; kk < BK; kk += 32) {
      bf16x8 a[4], b[4];
#pragma unroll
      for (int i = 0; i < 4; ++i)
        a[i] = *(const bf16x8*)&As[wr * 64 + i * 16 + (lane & 15)][kk + 8 * (lane >> 4)];
#pragma unroll
      for (int j = 0; j < 4; ++j)
        b[j] = *(const bf16x8*)&Bs[wc * 64 + j * 16 + (lane & 15)][kk + 8 * (lane >> 4)];
#pragma unroll
      for (int i = 0; i < 4; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
          acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(a[i], b[j], acc[i][j], 0, 0, 0);
    }
  }
  float* Pz = P + (int64_t)blockIdx.z * M * N;
#pragma unroll
  for (int i = 0; i < 4; ++i)
#pragma unroll
    for (int j = 0; j < 4; ++j)
#pragma unroll
      for (int r = 0; r < 4; ++r) {
        const int64_t row = m0 + wr * 64 + i * 16 + 4 * (lane >> 4) + r;
        const int64_t col = n0 + wc * 64 + j * 16 + (lane & 15);
        if (row < M && col < N) Pz[row * N + col] = acc[i][j][r];
      }
}

// out (M x N, row stride ldo) = sum_z P[z] in order z = 0..splits-1
template <typename TP, typename TOut>
__global__ void splitk_reduce_kernel(const TP* P, int splits, int64_t M, int64_t N, TOut* out,
                                     int64_t ldo) {
  const int64_t e = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  const int64_t MN = M * N;
  if (e >= MN) return;
  double s = 0.0;
#pragma unroll 8
  for (int z = 0; z < splits; ++z) s += (double)P[z * MN + e];
  const int64_t r = MN <= 0xFFFFFFFFll ? (int64_t)((uint32_t)e / (uint32_t)N) : e / N;
  out[r * ldo + (e - r * N)] = (TOut)s;
}

inline int64_t ceil_div(int64_t a, int64_t b) { return (a + b - 1) / b; }
inline bool hip_ok() { return hipGetLastError() == hipSuccess; }

// ---- Gaussian sketch driver -------------------------------------------------
struct GaussPlan {
  int64_t lds;     // padded columns of S (its row stride when BF16)
  int splits;
  int64_t kchunk;
  int64_t ldbt;    // row stride of the BF16 transpose of B (mixed)
  int terms;       // BF16 terms of B (mixed): 1, or 3 for the FP32-accurate split
  size_t s_bytes, p_bytes, bt_bytes;
  size_t total() const { return s_bytes + p_bytes + bt_bytes; }
};

GaussPlan gauss_plan(const mihs_handle* h, int64_t M, int64_t K, int64_t N, int mixed,
                     int terms = 1) {
  GaussPlan g;
  g.terms = mixed ? terms : 1;
  const int BM = mixed ? 128 : 64, BN = mixed ? 128 : 64, BK = mixed ? 64 : kGemmK;
  g.lds = mixed ? (K + 7) / 8 * 8 : (K + kGemmK - 1) / kGemmK * kGemmK;
  const int64_t tiles = ceil_div(M, BM) * ceil_div(N, BN);
  // mixed: two workgroups per CU and >= 8 steps per split.  FP64: four per CU (they fill
  // each other's operand waits: 1400 x 30011 x 700, 242 tiles, 1852 us whole, 1148 in 4
  // splits, 1119 in 8) and >= 4 steps (200 x 1500 x 61, 4 tiles: 14.4 us in 8 splits, 7.1
  // in 24); at most 32, as every split is written and read back once.
  const int64_t most = mixed ? 64 : 32;
  int64_t want = ceil_div((mixed ? 2 : 4) * (int64_t)h->num_cu, tiles);
  const int64_t kmax = ceil_div(K, (mixed ? 8 : 4) * BK);
  if (want > kmax) want = kmax;
  if (want > most) want = most;
  if (want < 1) want = 1;
  g.kchunk = ceil_div(ceil_div(K, want), BK) * BK;
  g.splits = (int)ceil_div(K, g.kchunk);
  g.s_bytes = align_up((size_t)M * g.lds * (mixed ? 2 : 8), 256);
  g.p_bytes = align_up((size_t)g.terms * g.splits * M * N * (mixed ? 4 : 8), 256);
  g.ldbt = (K + 7) / 8 * 8;
  g.bt_bytes = mixed ? align_up((size_t)g.terms * N * g.ldbt * 2, 256) : 0;
  return g;
}

// SA (M x N, row stride ldo, TOut) = G B with G = N(0,1)/sqrt(M) (M x K) from
// Philox stream `stream`; B is K x N (row stride ldb, TB).
template <typename TB>
int run_gauss(const mihs_handle* h, const TB* B, int64_t K, int64_t N, int64_t ldb, int64_t M,
              uint32_t seed, uint64_t stream_id, int mixed, void* out, int64_t ldo, char* ws,
              size_t ws_bytes, hipStream_t st, int terms = 1) {
  const GaussPlan g = gauss_plan(h, M, K, N, mixed, terms);
  if (ws_bytes < g.total()) return MIHS_ERR_WORKSPACE;
  void* S = ws;
  void* P = ws + g.s_bytes;
  const double scale = 1.0 / sqrt((double)M);
  const int64_t nblk = ceil_div(M * K, 4);
  if (mixed)
    hipLaunchKernelGGL(gauss_gen_kernel<uint16_t>, dim3((unsigned)ceil_div(nblk, 256)), dim3(256),
                       0, st, (uint16_t*)S, M, K, g.lds, seed, stream_id, scale);
  else
    hipLaunchKernelGGL(gauss_gen_kernel<double>, dim3((unsigned)ceil_div(nblk, 256)), dim3(256), 0,
                       st, (double*)S, M, K, g.lds, seed, stream_id, scale);
  if (!hip_ok()) return MIHS_ERR_HIP;
  if (mixed) {
    uint16_t* Bt = (uint16_t*)(ws + g.s_bytes + g.p_bytes);
    const dim3 tgrid((unsigned)ceil_div(N, 64), (unsigned)ceil_div(g.ldbt, 64));
    const int64_t part = N * g.ldbt;  // elements of one BF16 term of B^T
    if constexpr (sizeof(TB) == 4) {
      if (g.terms == 3)
        hipLaunchKernelGGL(bf16_split3_transpose_kernel, tgrid, dim3(kBlock), 0, st, B, K, N,
                           ldb, Bt, g.ldbt, part);
      else
        hipLaunchKernelGGL(bf16_transpose_kernel<TB>, tgrid, dim3(kBlock), 0, st, B, K, N, ldb,
                           Bt, g.ldbt);
    } else {
      if (g.terms != 1) return MIHS_ERR_UNSUPPORTED;
      hipLaunchKernelGGL(bf16_transpose_kernel<TB>, tgrid, dim3(kBlock), 0, st, B, K, N, ldb, Bt,
                         g.ldbt);
    }
    // one GEMM per term into its own split-K partials; the reduction adds them
    // all in a fixed order
    dim3 grid((unsigned)ceil_div(N, 128), (unsigned)ceil_div(M, 128), (unsigned)g.splits);
    for (int t = 0; t < g.terms; ++t)
      hipLaunchKernelGGL(gemm_bf16_kernel, grid, dim3(kBlock), 0, st, (const uint16_t*)S, g.lds,
                         M, K, (const uint16_t*)(Bt + t * part), g.ldbt, N, g.kchunk,
                         (float*)P + (int64_t)t * g.splits * M * N);
    hipLaunchKernelGGL((splitk_reduce_kernel<float, float>), dim3((unsigned)ceil_div(M * N, 256)),
                       dim3(256), 0, st, (const float*)P, g.terms * g.splits, M, N, (float*)out,
                       ldo);
  } else {
    dim3 grid((unsigned)ceil_div(M, 64), (unsigned)ceil_div(N, 64), (unsigned)g.splits);
    hipLaunchKernelGGL((gemm_f64_kernel<KPanel<double, 64>, KRows<TB, 64>, 64, double, TB>), grid,
                       dim3(kBlock), 0, st, (const double*)S, M, M, K, B, ldb, N, g.kchunk,
                       (double*)P);
    hipLaunchKernelGGL((splitk_reduce_kernel<double, double>), dim3((unsigned)ceil_div(M * N, 256)),
                       dim3(256), 0, st, (const double*)P, g.splits, M, N, (double*)out, ldo);
  }
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

// ---- CountSketch driver -------------------------------------------------------
struct CsPlan {
  CsLists lists;
  size_t hist, slots, total;
};
CsPlan cs_plan(int64_t n, int64_t m) {
  CsPlan p;
  p.lists = cs_lists(n, m);
  const size_t count = p.lists.cap ? (size_t)p.lists.ranges * m : 0;
  size_t o = 0;
  p.hist = o; o = align_up(o + count * 4, 256);
  p.slots = o; o = align_up(o + count * (size_t)p.lists.cap * 4, 256);
  p.total = o;
  return p;
}

template <typename TA, typename TAcc, typename TOut>
int run_countsketch(const TA* A, int64_t n, int64_t d, int64_t lda, int64_t m, uint32_t seed,
                    TOut* out, int64_t ldo, char* ws, size_t ws_bytes, hipStream_t st) {
  const CsPlan p = cs_plan(n, m);
  if (ws_bytes < p.total) return MIHS_ERR_WORKSPACE;
  unsigned* hist = (unsigned*)(ws + p.hist);
  unsigned* slots = (unsigned*)(ws + p.slots);
  const unsigned cap = (unsigned)p.lists.cap;
  const int list_len = (int)cs_list_len(p.lists.cap);
  if (cap) {
    // the counts start from zero (a kernel, not a memset: a caller may capture
    // this sequence in a graph)
    const int64_t count = p.lists.ranges * m;
    hipLaunchKernelGGL(zero_u32_kernel, dim3((unsigned)ceil_div(count, 256)), dim3(256), 0, st,
                       hist, count);
    hipLaunchKernelGGL(cs_hash_kernel, dim3((unsigned)ceil_div(n, kCsBlock)), dim3(kCsBlock), 0,
                       st, n, m, seed,
                       p.lists.ranges > 1 ? (unsigned)(p.lists.rows / kCsBlock) : 0u, cap, hist,
                       slots);
  }
  const size_t lds = 2 * (size_t)list_len * sizeof(unsigned);
  auto kern = p.lists.ranges == 1 ? cs_accum_kernel<TA, TAcc, TOut, true>
                                  : cs_accum_kernel<TA, TAcc, TOut, false>;
  if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                          (int)lds) != hipSuccess)
    return MIHS_ERR_HIP;
  const int64_t wide = kCsBlock * (16 / (int64_t)sizeof(TA));
  hipLaunchKernelGGL(kern, dim3((unsigned)m, (unsigned)ceil_div(d, wide)), dim3(kCsBlock), lds, st,
                     A, lda, n, d, m, seed, cap, list_len, hist, slots, out, ldo,
                     (int)p.lists.ranges, p.lists.rows);
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

// ---- SRHT driver ----------------------------------------------------------------
int srht_logB(int64_t n) {
  int lb = 0;
  while ((1LL << (lb + 1)) <= n && lb < 9) ++lb;
  return lb;
}

// The one-read SRHT: block size (B = 2^logb rows), samples per thread, and the
// number of block ranges per strip.  Used when n >= B and the samples fit the registers
// (m <= 4096 in FP32, 2048 in FP64); else the two-stage transform below.
struct SrhtFusedPlan {
  bool ok = false;
  int logb = 0, ns = 0, nparts = 1;
  int64_t nblk = 0, strips = 0;
  size_t idx_bytes = 0, sign_bytes = 0, part_bytes = 0;
  size_t total() const { return idx_bytes + sign_bytes + part_bytes; }
};

SrhtFusedPlan srht_fused_plan(const mihs_handle* h, int64_t n, int64_t d, int64_t m, int ty_bytes) {
  SrhtFusedPlan F;
  const bool f32 = ty_bytes == 4;
  F.logb = f32 ? 10 : 9;
  if (n < (1LL << F.logb) || (n & (n - 1)) != 0 || m > (f32 ? 4096 : 2048) || m < 1) return F;
  // a sample's block index k_hi is kept in 16 bits
  if ((n >> F.logb) > 65536) return F;
  F.ok = true;
  const int groups = f32 ? fused_groups<float>() : fused_groups<double>();
  F.ns = m <= 512 ? 512 / groups : m <= 1024 ? 1024 / groups : m <= 2048 ? 2048 / groups
                                             : m <= 3072 ? 3072 / groups : 4096 / groups;
  F.nblk = n >> F.logb;
  F.strips = (d + kFusedW - 1) / kFusedW;
  // Block ranges per strip: one workgroup runs per CU, so strips x ranges workgroups take
  // ceil(that / CUs) rounds of nblk / ranges blocks, and every range writes and reads back
  // its partial sums.  The least of rounds x blocks x ~3 us (a 1024-row FP32 block; twice
  // that from FP64 rows) plus the partials' bytes at ~4 TB/s.  A range's sum runs over its blocks
  // one by one, so fewer ranges mean longer FP32 sums: against the FP64 form the mixed sketch's
  // relative error is 1.4e-7 to 2.3e-7 from 65536 x 100 to 2^22 x 40, within 1% of the even split
  // over the CUs or below it.
  double best = 0.0;
  const int64_t pmax = std::max<int64_t>(32, 2 * ceil_div(h->num_cu, F.strips));
  for (int64_t p = 1; p <= pmax && p <= F.nblk; ++p) {
    const double rounds = (double)ceil_div(F.strips * p, h->num_cu);
    const double us = rounds * (double)ceil_div(F.nblk, p) * 3.0 +
                      (p > 1 ? 2.0 * (double)p * (double)m * (double)d * ty_bytes / 4e6 : 0.0);
    if (p == 1 || us < best) {
      best = us;
      F.nparts = (int)p;
    }
  }
  F.idx_bytes = align_up((size_t)m * 4, 256);
  F.sign_bytes = align_up((size_t)(n / 32) * 4, 256);
  F.part_bytes = F.nparts > 1 ? align_up((size_t)F.nparts * m * fused_ldp(d) * ty_bytes, 256) : 0;
  return F;
}

template <typename TA, typename TY, int LOGB, typename TS>
int launch_srht_fused(const SrhtFusedPlan& F, const TA* A, int64_t lda, int64_t d, int64_t m,
                      const uint32_t* signw, const int* idx, TY* P, TS* SA, int64_t ldsa,
                      double scale, hipStream_t st) {
  int64_t wgs = F.strips * F.nparts;
  if (fused_pair<TA>() == 2)
    wgs = ceil_div((F.strips + 1) / 2 * F.nparts, kXcds) * 2 * kXcds;
  const dim3 grid((unsigned)wgs);
  auto go = [&](auto kern, int ns) -> int {
    const size_t lds = ((size_t)fused_row(1 << LOGB, sizeof(TY) == 4 ? 32 : 16) * kFusedW) *
                           sizeof(TY) + (size_t)fused_groups<TY>() * ns * 4;
    if (hipFuncSetAttribute((const void*)kern, hipFuncAttributeMaxDynamicSharedMemorySize,
                            (int)lds) != hipSuccess)
      return MIHS_ERR_HIP;
    hipLaunchKernelGGL(kern, grid, dim3(kFusedThreads), lds, st, A, lda, d, signw, idx, m,
                       F.nblk, F.nparts, P, fused_ldp(d), SA, ldsa, scale);
    return MIHS_OK;
  };
  int rc = MIHS_ERR_UNSUPPORTED;
  // the 32-bit offsets of a block's rows reach 2 GiB; longer blocks (FP64 rows of 2 MiB and
  // more at 1024 rows) take the addressing by pointers, in one form for all sample counts
  // (1024 x 262144 FP64, m = 3000: 4.8 ms, 16.9 in two stages)
  if ((double)(1LL << LOGB) * (double)lda * sizeof(TA) >= 2147483647.0) {
    rc = go(srht_fused_kernel<TA, TY, LOGB, 32, TS, true>, 32);
  } else if constexpr (sizeof(TY) == 4) {
    switch (F.ns) {
      case 4: rc = go(srht_fused_kernel<TA, TY, LOGB, 4, TS, false>, 4); break;
      case 8: rc = go(srht_fused_kernel<TA, TY, LOGB, 8, TS, false>, 8); break;
      case 16: rc = go(srht_fused_kernel<TA, TY, LOGB, 16, TS, false>, 16); break;
      case 24: rc = go(srht_fused_kernel<TA, TY, LOGB, 24, TS, false>, 24); break;
      case 32: rc = go(srht_fused_kernel<TA, TY, LOGB, 32, TS, false>, 32); break;
    }
  } else {
    switch (F.ns) {
      case 8: rc = go(srht_fused_kernel<TA, TY, LOGB, 8, TS, false>, 8); break;
      case 16: rc = go(srht_fused_kernel<TA, TY, LOGB, 16, TS, false>, 16); break;
      case 32: rc = go(srht_fused_kernel<TA, TY, LOGB, 32, TS, false>, 32); break;
    }
  }
  if (rc) return rc;
  if (F.nparts > 1)
    hipLaunchKernelGGL((srht_parts_sum_kernel<TY, TS>), dim3((unsigned)ceil_div(m * d, 256)),
                       dim3(256), 0, st, P, F.nparts, m, d, fused_ldp(d), SA, ldsa, scale);
  return MIHS_OK;
}

template <typename TA, typename TY, typename TS>
int run_srht(const mihs_handle* h, const TA* A, int64_t n, int64_t d, int64_t lda, int64_t m,
             uint32_t seed, TS* SA, int64_t ldsa, char* ws, size_t ws_bytes, hipStream_t st) {
  // (the workspace query knows no row stride, so the form must not depend on it)
  const SrhtFusedPlan F = srht_fused_plan(h, n, d, m, (int)sizeof(TY));
  if (F.ok) {
    if (ws_bytes < F.total()) return MIHS_ERR_WORKSPACE;
    int* idx = (int*)ws;
    uint32_t* signw = (uint32_t*)(ws + F.idx_bytes);
    TY* P = (TY*)(ws + F.idx_bytes + F.sign_bytes);
    hipLaunchKernelGGL(srht_rows_kernel, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, idx,
                       m, n, seed);
    hipLaunchKernelGGL(srht_sign_words_kernel, dim3((unsigned)ceil_div(n / 32, 256)), dim3(256),
                       0, st, signw, n / 32, seed);
    const double scale = 1.0 / sqrt((double)m);
    int rc;
    if constexpr (sizeof(TY) == 4)
      rc = launch_srht_fused<TA, TY, 10, TS>(F, A, lda, d, m, signw, idx, P, SA, ldsa, scale, st);
    else
      rc = launch_srht_fused<TA, TY, 9, TS>(F, A, lda, d, m, signw, idx, P, SA, ldsa, scale, st);
    if (rc) return rc;
    return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
  }
  const size_t idx_bytes = align_up((size_t)m * 4, 256);
  const int64_t ldy = (d + 3) / 4 * 4;
  const size_t y_bytes = align_up((size_t)n * ldy * sizeof(TY), 256);
  if (ws_bytes < idx_bytes + y_bytes) return MIHS_ERR_WORKSPACE;
  int* idx = (int*)ws;
  TY* Y = (TY*)(ws + idx_bytes);
  const int logB = srht_logB(n);
  const int B = 1 << logB;
  const int64_t nhi = n >> logB;
  hipLaunchKernelGGL(srht_rows_kernel, dim3((unsigned)ceil_div(m, 256)), dim3(256), 0, st, idx, m, n,
                     seed);
  if (logB == 9) {
    constexpr int W = sizeof(TY) == 4 ? 32 : 16;
    hipLaunchKernelGGL((srht_stage1_b512<TA, TY>), dim3((unsigned)ceil_div(d, W), (unsigned)nhi),
                       dim3(kBlock), 0, st, A, lda, d, seed, Y, ldy);
  } else {
    const size_t sh1 = (size_t)B * kFwhtW * sizeof(TY);
    if (hipFuncSetAttribute((const void*)srht_stage1<TA, TY>,
                            hipFuncAttributeMaxDynamicSharedMemorySize, (int)sh1) != hipSuccess)
      return MIHS_ERR_HIP;
    hipLaunchKernelGGL((srht_stage1<TA, TY>), dim3((unsigned)ceil_div(d, kFwhtW), (unsigned)nhi),
                       dim3(kBlock), sh1, st, A, lda, d, logB, seed, Y, ldy);
  }
  hipLaunchKernelGGL((srht_stage2<TY, TS>), dim3((unsigned)ceil_div(d, kS2Cols), (unsigned)B),
                     dim3(kBlock), 0, st, Y, ldy, d, logB, nhi, idx, m, SA, ldsa,
                     1.0 / sqrt((double)m));
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

__global__ __launch_bounds__(kBlock) void neg_dot_kernel(const double* X, const double* W,
                                                         int64_t count, double lam, double* out,
                                                         double* out_log) {
  __shared__ double s_red[kWavesPerBlock];
  double v = 0.0;
  for (int64_t i = threadIdx.x; i < count; i += kBlock) v += X[i] * W[i];
  v = block_sum(v, s_red);
  if (threadIdx.x == 0) {
    *out = -v;
    if (out_log) *out_log = lam * -v;  // chain rule through lambda = exp(log lambda)
  }
}

__global__ void fill_kernel(double* p, double v, int64_t count) {
  const int64_t i = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
  if (i < count) p[i] = v;
}

}  // namespace

int launch_fill(double* p, double value, int64_t count, hipStream_t st) {
  hipLaunchKernelGGL(fill_kernel, dim3((unsigned)ceil_div(count, 256)), dim3(256), 0, st, p, value,
                     count);
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

template <typename TA>
static void apply_rows(const TA* A, int64_t n, int64_t d, int64_t lda, const double* W, int64_t k,
                       double* Y, hipStream_t st) {
  if (k == 1) {
    hipLaunchKernelGGL(rowdot_kernel<TA>, dim3((unsigned)ceil_div(n, 4 * kWavesPerBlock)),
                       dim3(kBlock), 0, st, A, n, d, lda, W, Y);
    return;
  }
  // W's rows start on 16-byte boundaries when k is even and W itself does
  const bool vec = k % 2 == 0 && ((uintptr_t)W & 15) == 0;
  auto go = [&](auto ox, auto oy, auto bn) {
    constexpr int BN = decltype(bn)::value;
    hipLaunchKernelGGL((gemm_f64_kernel<decltype(ox), decltype(oy), BN, TA, double>),
                       dim3((unsigned)ceil_div(n, 64), (unsigned)ceil_div(k, BN), 1), dim3(kBlock),
                       0, st, A, lda, n, d, W, k, k, d, Y);
  };
  const std::integral_constant<int, 32> b32;
  const std::integral_constant<int, 64> b64;
  // up to 32 columns a 32-wide tile multiplies less padding
  if (k <= 32 && vec) go(KCols<TA, 64>(), KRows<double, 32, true>(), b32);
  else if (k <= 32) go(KCols<TA, 64>(), KRows<double, 32, false>(), b32);
  else if (vec) go(KCols<TA, 64>(), KRows<double, 64, true>(), b64);
  else go(KCols<TA, 64>(), KRows<double, 64, false>(), b64);
}

int launch_apply_rows(const mihs_handle* h, const void* A, int a_f32, int64_t n, int64_t d,
                      int64_t lda, const double* W, int64_t k, double* Y, int64_t ldy,
                      hipStream_t st) {
  (void)h;
  if (ldy != k) return MIHS_ERR_UNSUPPORTED;
  if (a_f32)
    apply_rows((const float*)A, n, d, lda, W, k, Y, st);
  else
    apply_rows((const double*)A, n, d, lda, W, k, Y, st);
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

int launch_neg_dot(const double* X, const double* W, int64_t count, double lam, double* out,
                   double* out_log, hipStream_t st) {
  hipLaunchKernelGGL(neg_dot_kernel, dim3(1), dim3(kBlock), 0, st, X, W, count, lam, out,
                     out_log);
  return hip_ok() ? MIHS_OK : MIHS_ERR_HIP;
}

size_t sketch_workspace_bytes(const mihs_handle* h, int64_t n, int64_t d, int64_t m, int64_t m2,
                              int kind, int a_f32, int mixed) {
  (void)a_f32;
  switch (kind) {
    case MIHS_GAUSSIAN: {
      const GaussPlan g = gauss_plan(h, m, n, d, mixed);
      return g.total();
    }
    case MIHS_SRHT: {
      const SrhtFusedPlan F = srht_fused_plan(h, n, d, m, mixed ? 4 : 8);
      if (F.ok) return F.total();
      const int64_t ldy = (d + 3) / 4 * 4;
      return align_up((size_t)m * 4, 256) + align_up((size_t)n * ldy * (mixed ? 4 : 8), 256);
    }
    case MIHS_COUNTSKETCH:
      return cs_plan(n, m).total;
    case MIHS_COUNT_GAUSS: {
      const int64_t ldc = (d + 3) / 4 * 4;
      const size_t ca = align_up((size_t)m * ldc * (mixed ? 4 : 8), 256);
      const GaussPlan g = gauss_plan(h, m2, m, d, mixed, kCountGaussTerms);
      const size_t a = cs_plan(n, m).total, b = g.total();
      return ca + (a > b ? a : b);
    }
    default:
      return 0;
  }
}

int launch_sketch(const mihs_handle* h, const void* A, int a_f32, int64_t n, int64_t d,
                  int64_t lda, int kind, int64_t m, int64_t m2, uint32_t seed, int mixed,
                  void* SA, int64_t ldsa, void* ws, size_t ws_bytes, hipStream_t st) {
  const size_t need = sketch_workspace_bytes(h, n, d, m, m2, kind, a_f32, mixed);
  if (!ws || ws_bytes < need) return MIHS_ERR_WORKSPACE;
  char* w = (char*)ws;
  switch (kind) {
    case MIHS_GAUSSIAN:
      if (a_f32)
        return run_gauss<float>(h, (const float*)A, n, d, lda, m, seed, 0, mixed, SA, ldsa, w, ws_bytes, st);
      return run_gauss<double>(h, (const double*)A, n, d, lda, m, seed, 0, mixed, SA, ldsa, w, ws_bytes, st);
    case MIHS_SRHT:
      if (mixed) {
        if (a_f32)
          return run_srht<float, float, float>(h, (const float*)A, n, d, lda, m, seed, (float*)SA, ldsa, w, ws_bytes, st);
        return run_srht<double, float, float>(h, (const double*)A, n, d, lda, m, seed, (float*)SA, ldsa, w, ws_bytes, st);
      }
      if (a_f32)
        return run_srht<float, double, double>(h, (const float*)A, n, d, lda, m, seed, (double*)SA, ldsa, w, ws_bytes, st);
      return run_srht<double, double, double>(h, (const double*)A, n, d, lda, m, seed, (double*)SA, ldsa, w, ws_bytes, st);
    case MIHS_COUNTSKETCH:
      if (mixed) {
        if (a_f32)
          return run_countsketch<float, float, float>((const float*)A, n, d, lda, m, seed, (float*)SA, ldsa, w, ws_bytes, st);
        return run_countsketch<double, float, float>((const double*)A, n, d, lda, m, seed, (float*)SA, ldsa, w, ws_bytes, st);
      }
      if (a_f32)
        return run_countsketch<float, double, double>((const float*)A, n, d, lda, m, seed, (double*)SA, ldsa, w, ws_bytes, st);
      return run_countsketch<double, double, double>((const double*)A, n, d, lda, m, seed, (double*)SA, ldsa, w, ws_bytes, st);
    case MIHS_COUNT_GAUSS: {
      const int64_t ldc = (d + 3) / 4 * 4;
      const size_t ca_bytes = align_up((size_t)m * ldc * (mixed ? 4 : 8), 256);
      char* rest = w + ca_bytes;
      const size_t rest_bytes = ws_bytes - ca_bytes;
      int rc;
      if (mixed) {
        float* CA = (float*)w;
        rc = a_f32 ? run_countsketch<float, float, float>((const float*)A, n, d, lda, m, seed, CA, ldc, rest, rest_bytes, st)
                   : run_countsketch<double, float, float>((const double*)A, n, d, lda, m, seed, CA, ldc, rest, rest_bytes, st);
        if (rc) return rc;
        return run_gauss<float>(h, CA, m, d, ldc, m2, seed, 1, 1, SA, ldsa, rest, rest_bytes, st,
                                kCountGaussTerms);
      }
      double* CA = (double*)w;
      rc = a_f32 ? run_countsketch<float, double, double>((const float*)A, n, d, lda, m, seed, CA, ldc, rest, rest_bytes, st)
                 : run_countsketch<double, double, double>((const double*)A, n, d, lda, m, seed, CA, ldc, rest, rest_bytes, st);
      if (rc) return rc;
      return run_gauss<double>(h, CA, m, d, ldc, m2, seed, 1, 0, SA, ldsa, rest, rest_bytes, st);
    }
    default:
      return MIHS_ERR_INVALID;
  }
}

}  // namespace mihs
