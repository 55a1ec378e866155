// FP64 matrix-core tile product shared by the Gaussian sketch, A W and the Gram
// matrices: one workgroup of four waves forms a BM x BN tile of sum_k X(k, i) Y(k, j)
// with v_mfma_f64_16x16x4 (A operand: lane l holds row l % 16, k l / 16; B operand:
// column l % 16, k l / 16; result register r of lane l: row l / 16 + 4 r, column l % 16).
//
// The waves form a 2 x 2 grid of (BM / 2) x (BN / 2) quarters.  16 k per step go
// through double-buffered LDS (one barrier per step); the next step's 16-byte global
// loads are in flight in registers while this step is multiplied.  Both operands are
// converted to FP64 on their way into LDS.
//
// Bound: the FP64 matrix pipe (77 TFLOP/s measured with registers only; one wave per
// SIMD and even a single dependent chain of products reach that rate, so operand
// latency is what is left to hide).  A 64 x 64 tile takes 39 KiB of LDS, so four
// workgroups share a CU and fill each other's waits: 4096^3 59-61 TFLOP/s (128 x 128,
// two workgroups per CU: 63; one: 36), 1400 x 30011 x 700 with 8 k ranges 52 against
// 22 for an unpipelined 64 x 64 tile whose left operand was read row-major.
#pragma once

#include "device_util.hpp"

namespace mihs {

typedef double f64x4 __attribute__((ext_vector_type(4)));

constexpr int kGemmK = 16;  // k per step

// The operand types move 16-byte chunks: chunk c of a thread is element e = c * kBlock +
// thread of the tile, consecutive lanes consecutive chunks.  A chunk that begins inside the
// matrix is loaded whole: rows start on 16-byte boundaries (checked by the caller), so it
// stays inside the row's aligned span.  Chunks past an edge load some chunk inside instead,
// and what lies beyond the bounds is zeroed on its way to LDS: loads under a condition of
// their own, or zeroed where they land, wait for one another (4096^3 dropped to 54).

// k runs over rows: element (k, i) at M[k * ld + i].  LDS tile [k][i], row stride W + 16
// doubles, so that the two k rows a half-wave reads lie 32 banks apart.
// VEC: rows are 16-byte aligned; otherwise elements are loaded one by one.
template <typename T, int W, bool VEC = true>
struct KRows {
  static constexpr int V = 16 / (int)sizeof(T);
  static constexpr int CPR = W / V;                // chunks per k row
  static constexpr int TOT = kGemmK * CPR;         // chunks per tile
  static constexpr int N = (TOT + kBlock - 1) / kBlock;  // chunks per thread
  static constexpr int LD = W + 16;
  static constexpr int SIZE = kGemmK * LD;
  static_assert(TOT % kBlock == 0 || TOT < kBlock, "tile shape");
  typedef T vec_t __attribute__((ext_vector_type(V)));
  struct Regs {
    vec_t v[N];
  };
  // a tile of fewer chunks than threads is moved by every thread group alike (the same
  // values to the same places)
  static __device__ __forceinline__ int elem(int c) {
    return TOT < kBlock ? (int)threadIdx.x % TOT : c * kBlock + (int)threadIdx.x;
  }

  // k in [k0, ke), columns [i0, ni) of M
  static __device__ __forceinline__ void load(const T* __restrict__ M, int64_t ld, int64_t k0,
                                              int64_t ke, int64_t i0, int64_t ni, Regs& out) {
    if constexpr (VEC) {
      if (k0 + kGemmK <= ke && i0 + W <= ni) {  // uniform
        const T* p = M + k0 * ld + i0;
#pragma unroll
        for (int c = 0; c < N; ++c) {
          const int e = elem(c);
          out.v[c] = *(const vec_t*)(p + (int64_t)(e / CPR) * ld + (e % CPR) * V);
        }
        return;
      }
    }
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int e = elem(c);
      const int64_t k = min(k0 + e / CPR, ke - 1), i = i0 + (e % CPR) * V;
      if constexpr (VEC) {
        out.v[c] = *(const vec_t*)(M + k * ld + (i < ni ? i : i0));
      } else {
#pragma unroll
        for (int q = 0; q < V; ++q) out.v[c][q] = M[k * ld + min(i + q, ni - 1)];
      }
    }
  }
  static __device__ __forceinline__ void store(const Regs& in, int64_t k0, int64_t ke, int64_t i0,
                                               int64_t ni, double* tile) {
    const bool inside = k0 + kGemmK <= ke && i0 + W <= ni;  // uniform
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int e = elem(c);
      double* p = tile + (e / CPR) * LD + (e % CPR) * V;
      double x[V];
#pragma unroll
      for (int q = 0; q < V; ++q) x[q] = (double)in.v[c][q];
      if (!inside) {
        const int64_t k = k0 + e / CPR, i = i0 + (e % CPR) * V;
#pragma unroll
        for (int q = 0; q < V; ++q) x[q] = (k < ke && i + q < ni) ? x[q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < V; q += 2) *(dbl2*)(p + q) = (dbl2){x[q], x[q + 1]};
    }
  }
  static __device__ __forceinline__ double get(const double* tile, int k, int i) {
    return tile[k * LD + i];
  }
};

// k runs along rows: element (k, i) at M[i * ld + k].  LDS tile [i][k], row stride 18 doubles
// (the 16 rows x 2 k of a half-wave's read hit 32 different bank pairs).
template <typename T, int W>
struct KCols {
  static constexpr int V = 16 / (int)sizeof(T);
  static constexpr int CPR = kGemmK / V;
  static constexpr int N = W * CPR / kBlock;
  static constexpr int LD = kGemmK + 2;
  static constexpr int SIZE = W * LD;
  static_assert(N >= 1 && W * CPR % kBlock == 0, "tile shape");
  typedef T vec_t __attribute__((ext_vector_type(V)));
  struct Regs {
    vec_t v[N];
  };

  static __device__ __forceinline__ void load(const T* __restrict__ M, int64_t ld, int64_t k0,
                                              int64_t ke, int64_t i0, int64_t ni, Regs& out) {
    if (k0 + kGemmK <= ke && i0 + W <= ni) {
      const T* p = M + i0 * ld + k0;
#pragma unroll
      for (int c = 0; c < N; ++c) {
        const int e = c * kBlock + (int)threadIdx.x;
        out.v[c] = *(const vec_t*)(p + (int64_t)(e / CPR) * ld + (e % CPR) * V);
      }
      return;
    }
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int e = c * kBlock + (int)threadIdx.x;
      const int64_t i = min(i0 + e / CPR, ni - 1), k = k0 + (e % CPR) * V;
      out.v[c] = *(const vec_t*)(M + i * ld + (k < ke ? k : k0));
    }
  }
  static __device__ __forceinline__ void store(const Regs& in, int64_t k0, int64_t ke, int64_t i0,
                                               int64_t ni, double* tile) {
    const bool inside = k0 + kGemmK <= ke && i0 + W <= ni;
#pragma unroll
    for (int c = 0; c < N; ++c) {
      const int e = c * kBlock + (int)threadIdx.x;
      double* p = tile + (e / CPR) * LD + (e % CPR) * V;
      double x[V];
#pragma unroll
      for (int q = 0; q < V; ++q) x[q] = (double)in.v[c][q];
      if (!inside) {
        const int64_t i = i0 + e / CPR, k = k0 + (e % CPR) * V;
#pragma unroll
        for (int q = 0; q < V; ++q) x[q] = (i < ni && k + q < ke) ? x[q] : 0.0;
      }
#pragma unroll
      for (int q = 0; q < V; q += 2) *(dbl2*)(p + q) = (dbl2){x[q], x[q + 1]};
    }
  }
  static __device__ __forceinline__ double get(const double* tile, int k, int i) {
    return tile[i * LD + k];
  }
};

// Panels of 16 k: element (k, i) at M[(k / 16) * 16 * ld + 16 i + k % 16], ld rows per panel.
// A step's tile is one contiguous range (row-major rows of 240 KB stride cost 10% at the
// 1400 x 30011 x 700 sketch).  k0 is a multiple of 16.  LDS as KCols.
template <typename T, int W>
struct KPanel : KCols<T, W> {
  typedef KCols<T, W> B;
  static __device__ __forceinline__ void load(const T* __restrict__ M, int64_t ld, int64_t k0,
                                              int64_t ke, int64_t i0, int64_t ni,
                                              typename B::Regs& out) {
    const T* p = M + k0 * ld + i0 * kGemmK;
    const int last = (int)min((int64_t)W, ni - i0) * B::CPR - B::CPR;  // first chunk of the last row
#pragma unroll
    for (int c = 0; c < B::N; ++c) {
      const int e = c * kBlock + (int)threadIdx.x;
      out.v[c] = *(const typename B::vec_t*)(p + min(e, last + e % B::CPR) * B::V);
    }
  }
};

template <typename OX, typename OY>
constexpr int gemm64_lds() { return 2 * (OX::SIZE + OY::SIZE); }  // doubles

// acc[a][b] (16 x 16 blocks of this wave's quarter) = sum over k in [kb, ke), in ascending
// order.  X: rows i0.. of ni, Y: columns j0.. of nj; the tile must hold an element
// (i0 < ni, j0 < nj), as chunks past an edge read the tile's first column or last row.  lds: gemm64_lds doubles, 16-byte aligned.
template <typename OX, typename OY, int BM, int BN, typename TX, typename TY>
__device__ __forceinline__ void gemm64_tile(const TX* __restrict__ X, int64_t ldx, int64_t i0,
                                            int64_t ni, const TY* __restrict__ Y, int64_t ldy,
                                            int64_t j0, int64_t nj, int64_t kb, int64_t ke,
                                            double* lds, f64x4 (&acc)[BM / 32][BN / 32]) {
  constexpr int MB = BM / 32, NB = BN / 32;
  const int lane = lane_id(), wave = wave_id();
  const int wi = (wave >> 1) * (BM / 2) + (lane & 15), wj = (wave & 1) * (BN / 2) + (lane & 15);
  constexpr int S = OX::SIZE + OY::SIZE;
#pragma unroll
  for (int a = 0; a < MB; ++a)
#pragma unroll
    for (int b = 0; b < NB; ++b) acc[a][b] = (f64x4){0.0, 0.0, 0.0, 0.0};
  if (kb >= ke) return;
  typename OX::Regs gx = {};
  typename OY::Regs gy = {};
  OX::load(X, ldx, kb, ke, i0, ni, gx);
  OY::load(Y, ldy, kb, ke, j0, nj, gy);
  OX::store(gx, kb, ke, i0, ni, lds);
  OY::store(gy, kb, ke, j0, nj, lds + OX::SIZE);
  __syncthreads();
  int cur = 0;
  for (int64_t k0 = kb; k0 < ke; k0 += kGemmK) {
    const bool more = k0 + kGemmK < ke;
    if (more) {
      OX::load(X, ldx, k0 + kGemmK, ke, i0, ni, gx);
      OY::load(Y, ldy, k0 + kGemmK, ke, j0, nj, gy);
    }
    // the loads are issued before the products
    __builtin_amdgcn_sched_barrier(0);
    const double* tx = lds + cur * S;
    const double* ty = tx + OX::SIZE;
#pragma unroll
    for (int ks = 0; ks < kGemmK / 4; ++ks) {
      const int k = 4 * ks + (lane >> 4);
      double xv[MB], yv[NB];
#pragma unroll
      for (int a = 0; a < MB; ++a) xv[a] = OX::get(tx, k, wi + 16 * a);
#pragma unroll
      for (int b = 0; b < NB; ++b) yv[b] = OY::get(ty, k, wj + 16 * b);
#pragma unroll
      for (int a = 0; a < MB; ++a)
#pragma unroll
        for (int b = 0; b < NB; ++b)
          acc[a][b] = __builtin_amdgcn_mfma_f64_16x16x4f64(xv[a], yv[b], acc[a][b], 0, 0, 0);
    }
    if (more) {
      cur ^= 1;
      OX::store(gx, k0 + kGemmK, ke, i0, ni, lds + cur * S);
      OY::store(gy, k0 + kGemmK, ke, j0, nj, lds + cur * S + OX::SIZE);
    }
    __syncthreads();
  }
}

}  // namespace mihs
