// Persistent M-IHS solve kernel (Algorithm 1 with a CG inner solver).
//
// One cooperative launch runs the whole outer loop.  All G workgroups stream
// A; a subgroup of the first Gc workgroups runs the inner solve, so the inner
// loop only pays for a small, fast barrier.  Phases:
//
//   A1  (all G)  stage x in LDS; stream this workgroup's contiguous row block
//       of A once: each wave holds whole rows in registers, forms
//       r_i = b_i - A_i x by a wave reduction and accumulates A_i^T r_i into
//       per-lane partial gradients; the four waves combine in LDS and write one
//       partial d-vector.                                   -> barrier (all)
//   A2  (Gc)     column owners add the G partials (fixed order), form
//       g = sum + rhs - lambda x and start CG (z = 0, r = p = g).  -> barrier (Gc)
//   CG  (Gc)     per iteration two barriers:
//       C1  every CG workgroup forms p = r + beta_cg p_prev in LDS (owners
//           also store their slice) and streams its rows of SA:
//           u_j = SA_j p, partial -SA^T u, sum u_j^2.        -> barrier (Gc)
//       C2  p^T q = ||u||^2 + lambda ||p||^2 (scalar partials, fixed order);
//           owners form q = -sum + lambda p and update z, r. -> barrier (Gc)
//       The stop test ||r|| <= eps_sub ||g|| uses sums every CG workgroup
//       computes identically, so they all leave the loop together.
//       Where the group's registers hold the operator's rows (RES) and the vector is
//       short, the exchanges of C1 and C2 are tagged words instead of barriers.
//   U   (Gc)     owners apply x+ = x + alpha z + beta (x - x_prev) and write
//       the relative-step partials.                          -> barrier (all)
//       Every workgroup then evaluates the same stop test.
//
// Every reduction runs in a fixed order, so a solve is bit-reproducible.
#pragma once

#include <math.h>

#include <algorithm>
#include <type_traits>

#include "device_util.hpp"
#include "internal.hpp"
#include "solve_shape.hpp"

namespace mihs {

constexpr int kScal = 8;           // scalar partial slots per workgroup (solve_layout)
constexpr double kCg1MaxCond = 1e5;  // single-reduction CG up to this trace(H)/lambda
// Rows per group in rowpass_quarters: 128 KB of a 4096-wide matrix in flight per CU in
// either type (FP32, 2^20 x 4096: 4 rows with the next group prefetched 3.35 ms a pass,
// 8 without 3.20).
constexpr int kQuarterRows = 8;
template <typename T>
constexpr int quarter_rows() {
  return sizeof(T) == 4 ? 8 : 4;
}

struct SolveArgs {
  const void* A;
  int64_t n;
  int64_t lda;
  const double* b;
  const double* rhs;
  const void* SA;
  int64_t m;
  int64_t ldsa;
  double lam, alpha, beta, eps_sub, step_thr;
  int64_t max_outer, max_inner;
  double* x;
  double* xp;
  int xp_from_x;
  mihs_info_t* info;
  double* partA;   // G x dpad
  void* partS;     // Gc x dpad (TV)
  double* scal;    // G x kScal
  void* r;
  void* z;
  void* p0;
  void* p1;
  unsigned* bar_all;  // 9 lines (hierarchical barrier)
  unsigned* bar_cg;   // 1 line (flat inner-solve barrier)
  unsigned* bar_cgh;  // 9 lines (hierarchical inner-solve barrier)
  int* err;
  int* status;        // decision published by the CG group
  const void* H;      // Gram matrix (SA)^T SA (TS), dpad x dpad, when the CG uses it
  int64_t ldh;
  int cg1;            // Gram path: single-reduction CG (one barrier per step)
  int aab;            // streaming path: AAb_Solver (Algorithm 6) instead of CG
  double* yrow;       // AAb: m doubles, -(M v - theta p) of each row of SA
  const int* skip;    // when set and nonzero the launch returns at once
  int d, dpad, G, Gc, cpw;
  int cg_hier;        // inner-solve group large enough for the two-level barrier
  int32_t xw[kXcds];  // gradient-pass row weight of each XCD (row_split_bound)
  tagged_t* tagw;     // kVectorSlots x dpad tagged vector entries
  tagged_t* tags;     // kScalarSlots x Gc x 2 tagged scalars
  tagged_t* partT;    // Gc x dpad tagged partials of SA^T u (null: by barrier, partS)
  BarrierSpin spin_fast, spin_idle;
};

// Rows loaded per wave step: enough bytes in flight for short rows, one row
// when the row buffer and the EPT accumulators already fill the registers.
template <typename TM, int EPT>
struct RowsInFlight {
  static constexpr int kBytes = EPT * (int)sizeof(TM);   // bytes per lane per row
  static constexpr int value =
      (kBytes >= 512 || (EPT >= 32 && sizeof(TM) < 8)) ? 1 : (kBytes >= 256 ? 2 : 4);
};

// One pass over rows [r0, r1) of M: for each row, u = cs c_row - M_row . v and
// acc += u * M_row (acc in this lane's columns), ssq += u^2; u is also stored
// to uout[row] when uout is set (uout may alias c: each row is read before it
// is written, by the same wave).
template <typename TM, typename TV, int EPT, bool NT, int R>
__device__ __forceinline__ void rowpass(const TM* __restrict__ M, int64_t ld, int64_t r0,
                                        int64_t r1, int d, const TV* __restrict__ v,
                                        const double* c, TV (&acc)[EPT], TV& ssq,
                                        double cs = 1.0, double* uout = nullptr) {
  using L = RowLayout<TM, EPT>;
  const int lane = lane_id();
  constexpr bool CLAMP = EPT < 64;
  // (opaque: the clamped columns are not kept between passes)
  if constexpr (CLAMP) asm volatile("" : "+s"(d));
  for (int64_t row = r0 + (int64_t)wave_id() * R; row < r1; row += (int64_t)kWavesPerBlock * R) {
    // Rows past the range read another one of it; their u is zero.  As an offset from the group's
    // first row their addresses need no product of their own (2^18 x 2048 FP64: 24.9 ms, 25.0
    // with the row number clamped); up to 256 columns the compiler's schedule of the CG loop
    // is the better one with the number clamped (4096 x 256: 4.1 against 4.6 ms).
    TM rv[R][EPT];
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const TM* p = t == 0     ? M + row * ld
                    : EPT >= 8 ? M + row * ld + (row + t < r1 ? t * ld : 0)
                               : M + min(row + t, r1 - 1) * ld;
      load_row<TM, EPT, NT, CLAMP>(p, 0, d, lane, rv[t]);
    }
    if (CLAMP) clear_tail<TM, EPT, R>(0, d, lane, rv);
    TV dot[R];
#pragma unroll
    for (int t = 0; t < R; ++t) dot[t] = TV(0);
#pragma unroll
    for (int j = 0; j < L::J; ++j) {
#pragma unroll
      for (int vv = 0; vv < L::V; ++vv) {
        const TV xv = v[L::col(j, lane, vv)];
#pragma unroll
        for (int t = 0; t < R; ++t) dot[t] += (TV)rv[t][j * L::V + vv] * xv;
      }
    }
#pragma unroll
    for (int t = 0; t < R; ++t) dot[t] = wave_sum(dot[t]);
#pragma unroll
    for (int t = 0; t < R; ++t) {
      TV u = TV(0);
      if (row + t < r1) {
        u = (c ? (TV)(cs * c[row + t]) : TV(0)) - dot[t];
        if (uout && lane == 0) uout[row + t] = (double)u;
      }
      ssq += u * u;
#pragma unroll
      for (int e = 0; e < EPT; ++e) acc[e] += u * (TV)rv[t][e];
    }
  }
}

// The gradient pass for rows too long for one wave's registers (d > 2048): the
// four waves split every row into quarters of 64 * EQ columns, each lane holding
// EQ entries of its wave's quarter.  Per group of R rows every wave forms its
// partial dot products, they meet in LDS (double-buffered, one barrier per
// group), and each wave accumulates u_i * A_i on its own quarter, so no
// cross-wave reduction is needed at the end.  The next group's rows are loaded
// before the current group is processed.  u_i = c_i - A_i . v (c may be null).
template <typename TM, int EQ, bool NT, int R>
__device__ __forceinline__ void rowpass_quarters(const TM* __restrict__ M, int64_t ld, int64_t r0,
                                                 int64_t r1, int d, const double* __restrict__ v,
                                                 const double* __restrict__ c, double (&acc)[EQ],
                                                 double* s_part) {
  using L = RowLayout<TM, EQ>;
  // fetch the next group during this one only while both fit in registers
  constexpr bool PF = R * EQ * (int)sizeof(TM) <= 256;
  const int lane = lane_id(), w = wave_id();
  const int q0 = w * kWave * EQ;  // first column of this wave's quarter
  if (r0 >= r1) return;
  asm volatile("" : "+s"(d));  // (opaque: the clamped columns are not kept between passes)
  double vr[EQ];
#pragma unroll
  for (int j = 0; j < L::J; ++j)
#pragma unroll
    for (int vv = 0; vv < L::V; ++vv) vr[j * L::V + vv] = v[q0 + L::col(j, lane, vv)];
  auto load_group = [&](int64_t row0, TM (&buf)[R][EQ]) {
#pragma unroll
    for (int t = 0; t < R; ++t)
      load_row<TM, EQ, NT>(M + min(row0 + t, r1 - 1) * ld, q0, d, lane, buf[t]);
  };
  TM cur[R][EQ];
  if constexpr (PF) load_group(r0, cur);
  int buf = 0;
  for (int64_t row = r0; row < r1; row += R) {
    TM nxt[R][EQ];
    if constexpr (PF) load_group(row + R, nxt);
    else load_group(row, cur);
    clear_tail<TM, EQ, R>(q0, d, lane, cur);
    double dot[R];
#pragma unroll
    for (int t = 0; t < R; ++t) {
      dot[t] = 0.0;
#pragma unroll
      for (int e = 0; e < EQ; ++e) dot[t] += (double)cur[t][e] * vr[e];
      dot[t] = wave_sum(dot[t]);
    }
    if (lane == 0) {
#pragma unroll
      for (int t = 0; t < R; ++t) s_part[(buf * R + t) * kWavesPerBlock + w] = dot[t];
    }
    lds_barrier();
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const double* sp = s_part + (buf * R + t) * kWavesPerBlock;
      const double total = ((sp[0] + sp[1]) + sp[2]) + sp[3];
      const double u = (row + t < r1) ? ((c ? c[row + t] : 0.0) - total) : 0.0;
#pragma unroll
      for (int e = 0; e < EQ; ++e) acc[e] += u * (double)cur[t][e];
    }
    buf ^= 1;
    if constexpr (PF) {
#pragma unroll
      for (int t = 0; t < R; ++t)
#pragma unroll
        for (int e = 0; e < EQ; ++e) cur[t][e] = nxt[t][e];
    }
  }
}

// Store a wave's quarter of the partial vector (rowpass_quarters layout).
template <typename TM, int EQ>
__device__ __forceinline__ void store_quarters(const double (&acc)[EQ], double* out, int d) {
  using L = RowLayout<TM, EQ>;
  const int lane = lane_id();
  const int q0 = wave_id() * kWave * EQ;
#pragma unroll
  for (int j = 0; j < L::J; ++j)
#pragma unroll
    for (int vv = 0; vv < L::V; ++vv) {
      const int col = q0 + L::col(j, lane, vv);
      if (col < d) co_store(out + col, acc[j * L::V + vv]);
    }
}

// Combine the four waves' per-lane partial vectors (fixed wave order) and
// store them to `out[0..d)`.
template <typename TM, typename TV, int EPT>
__device__ __forceinline__ void wg_store_partial(const TV (&acc)[EPT], TV* red, TV* out, int d) {
  using L = RowLayout<TM, EPT>;
  const int lane = lane_id();
#pragma unroll
  for (int w = 0; w < kWavesPerBlock; ++w) {
    if (wave_id() == w) {
#pragma unroll
      for (int j = 0; j < L::J; ++j)
#pragma unroll
        for (int vv = 0; vv < L::V; ++vv) {
          const int col = L::col(j, lane, vv);
          red[col] = (w == 0 ? TV(0) : red[col]) + acc[j * L::V + vv];
        }
    }
    __syncthreads();
  }
  for (int col = threadIdx.x; col < d; col += kBlock) co_store(out + col, red[col]);
}

template <typename TV>
__device__ __forceinline__ TV wg_sum_ssq(TV ssq, double* s_red) {
  // every lane of a wave holds the same ssq; combine the four waves in order
  __syncthreads();
  if (lane_id() == 0) s_red[wave_id()] = (double)ssq;
  __syncthreads();
  double t = s_red[0];
  for (int w = 1; w < kWavesPerBlock; ++w) t += s_red[w];
  return (TV)t;
}

// Two workgroup sums at once (fixed wave order, the same result as two
// block_sum calls, with one pair of barriers).
__device__ __forceinline__ void block_sum2(double& a, double& b, double* s_red2) {
  a = wave_sum(a);
  b = wave_sum(b);
  __syncthreads();
  if (lane_id() == 0) {
    s_red2[2 * wave_id()] = a;
    s_red2[2 * wave_id() + 1] = b;
  }
  __syncthreads();
  a = s_red2[0];
  b = s_red2[1];
  for (int w = 1; w < kWavesPerBlock; ++w) {
    a += s_red2[2 * w];
    b += s_red2[2 * w + 1];
  }
}

// Two scalar sums over K workgroups' slots (fixed order), returned to every thread.
__device__ __forceinline__ void sum2_slots(const double* scal, int K, int s0, int s1,
                                           double* s_red2, double& o0, double& o1) {
  double a = 0.0, b = 0.0;
  for (int k = threadIdx.x; k < K; k += kBlock) {
    a += co_load(scal + (int64_t)k * kScal + s0);
    b += co_load(scal + (int64_t)k * kScal + s1);
  }
  a = wave_sum(a);
  b = wave_sum(b);
  __syncthreads();
  if (lane_id() == 0) {
    s_red2[2 * wave_id()] = a;
    s_red2[2 * wave_id() + 1] = b;
  }
  __syncthreads();
  o0 = s_red2[0];
  o1 = s_red2[1];
  for (int w = 1; w < kWavesPerBlock; ++w) {
    o0 += s_red2[2 * w];
    o1 += s_red2[2 * w + 1];
  }
}

// Column sums over K partial vectors for this workgroup's owned columns,
// out[i] = sum_k P[k * ldp + c0 + i], with every load of a thread issued before
// any is used (one memory round trip for K <= 16 * threads-per-column).
template <typename T>
__device__ __forceinline__ void owned_column_sums(const T* __restrict__ P, int K, int64_t ldp,
                                                  int c0, int ncols, double* out,
                                                  double* scratch) {
  constexpr int NB = 16;
  for (int cc0 = 0; cc0 < ncols; cc0 += kBlock) {
    const int CC = min(kBlock, ncols - cc0);
    int TPC = 1;
    while (TPC * 2 * CC <= kBlock) TPC *= 2;
    const int t = threadIdx.x;
    const int col = t % CC, ks = t / CC;
    double s = 0.0;
    if (ks < TPC) {
      const T* base = P + c0 + cc0 + col;
      for (int k0 = ks; k0 < K; k0 += NB * TPC) {
        T v[NB];
#pragma unroll
        for (int i = 0; i < NB; ++i) {
          const int k = k0 + i * TPC;
          v[i] = (k < K) ? co_load(base + (int64_t)k * ldp) : T(0);
        }
#pragma unroll
        for (int i = 0; i < NB; ++i) s += (double)v[i];
      }
    }
    __syncthreads();
    scratch[t] = s;
    __syncthreads();
    if (t < CC) {
      double acc = scratch[t];
      for (int i = 1; i < TPC; ++i) acc += scratch[i * CC + t];
      out[cc0 + t] = acc;
    }
    __syncthreads();
  }
}

// out[c - r0] = H[c, :] . v for rows c in [r0, r1), in a fixed order.  Each
// wave loads R rows before using any: a CG workgroup owns few rows, so this is
// usually one round trip.
template <typename TH, typename TV, int EPT, int R>
__device__ __forceinline__ void rowdots_r(const TH* __restrict__ H, int64_t ldh, int r0, int r1,
                                          int d, const TV* __restrict__ v, double* out) {
  using L = RowLayout<TH, EPT>;
  const int lane = lane_id();
  for (int c = r0 + wave_id() * R; c < r1; c += kWavesPerBlock * R) {
    TH rv[R][EPT];
    constexpr bool CLAMP = EPT < 64;
#pragma unroll
    for (int t = 0; t < R; ++t)
      load_row<TH, EPT, false, CLAMP>(H + (int64_t)(R == 1 ? c : min(c + t, r1 - 1)) * ldh, 0, d, lane, rv[t]);
    if (CLAMP) clear_tail<TH, EPT, R>(0, d, lane, rv);
    TV dot[R];
#pragma unroll
    for (int t = 0; t < R; ++t) dot[t] = TV(0);
#pragma unroll
    for (int j = 0; j < L::J; ++j) {
#pragma unroll
      for (int vv = 0; vv < L::V; ++vv) {
        const TV xv = v[L::col(j, lane, vv)];
#pragma unroll
        for (int t = 0; t < R; ++t) dot[t] += (TV)rv[t][j * L::V + vv] * xv;
      }
    }
#pragma unroll
    for (int t = 0; t < R; ++t) {
      const TV sdot = wave_sum(dot[t]);
      if (lane == 0 && c + t < r1) out[c + t - r0] = (double)sdot;
    }
  }
}

// Rows per wave: up to 512 bytes per lane in flight (at most 4 rows), halved
// when the workgroup owns too few rows to give every wave a full set.  Rows of
// 4096 entries keep one row in flight: a second FP32 row spilled the solve
// kernel's registers to scratch (89 VGPRs), which cost more than the extra
// round trip saves.
template <typename TH, typename TV, int EPT>
__device__ __forceinline__ void rowdots(const TH* __restrict__ H, int64_t ldh, int r0, int r1,
                                        int d, const TV* __restrict__ v, double* out) {
  constexpr int RB = (EPT >= 64 ? 256 : 512) / (EPT * (int)sizeof(TH));
  constexpr int R = RB < 1 ? 1 : (RB > 4 ? 4 : RB);
  if constexpr (R > 1) {
    if (r1 - r0 <= kWavesPerBlock * (R / 2)) {
      rowdots_r<TH, TV, EPT, R / 2>(H, ldh, r0, r1, d, v, out);
      return;
    }
  }
  rowdots_r<TH, TV, EPT, R>(H, ldh, r0, r1, d, v, out);
}

// ---- operator rows kept in registers --------------------------------------------
// The inner solvers multiply the same few rows per workgroup (of the Gram matrix, or of SA)
// by a new vector in every step, and what a step costs is the round trip that reloads them:
// 13.4 us of a 21 us CG step on the 64 MB FP32 matrix at d = 4096 (4.8 TB/s from the
// Infinity Cache), 6.7 us of a 24 us AAb step on a 2048 x 2048 FP64 sketch.  One wave per
// SIMD has 512 registers and the inner loop itself needs few, so the rows stay there for the
// whole inner solve (the gradient pass takes the registers back): the 256 CUs hold the
// 64 MB matrix in half of their register files.
//
// The four waves split every row into quarters of 64 * EQ columns, so each reads only its
// quarter of the vector from LDS and, for SA, accumulates only its quarter of SA^T u.

// Sums of N values (N = 1, 2, 4, 8 or 16) over each row of 16 lanes at once: a stage either
// halves the number of values per lane (each lane keeps the half that its lane bit names
// and adds the partner's) or, when one is left, adds the partner's.  Lane l ends with value
// (l % 16) / (16 / N); 7 instructions per kept value and stage instead of a whole reduction
// per value.
template <int N>
__device__ __forceinline__ double row_sums(double (&v)[N]) {
  const int lane = lane_id();
  auto stage = [&](auto ctrl, int bit, int half) {
    constexpr int C = decltype(ctrl)::value;
    if (half >= 1) {
#pragma unroll
      for (int i = 0; i < N; ++i) {
        if (i < half) {
          const double send = bit ? v[i] : v[i + half];
          const double keep = bit ? v[i + half] : v[i];
          v[i] = keep + dpp_row_move<C>(send);
        }
      }
    } else {
      v[0] += dpp_row_move<C>(v[0]);
    }
  };
  // mirrors first: they flip every lower lane bit as well
  stage(std::integral_constant<int, 0x140>(), (lane >> 3) & 1, N / 2);
  stage(std::integral_constant<int, 0x141>(), (lane >> 2) & 1, N / 4);
  stage(std::integral_constant<int, 0x4E>(), (lane >> 1) & 1, N / 8);
  stage(std::integral_constant<int, 0xB1>(), lane & 1, N / 16);
  return v[0];
}

constexpr int kResParts = 4 * kWavesPerBlock;  // partial sums per resident row's product

template <typename TS, int EQ, int NR>
struct ResidentRows {
  using L = RowLayout<TS, EQ>;
  TS h[NR][EQ];

  // rows [r0, min(r1, r0 + NR)) of M (d columns); missing rows are zero
  __device__ __forceinline__ void load(const TS* __restrict__ M, int64_t ld, int64_t r0,
                                       int64_t r1, int d) {
    const int q0 = wave_id() * kWave * EQ;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      if (r0 + r < r1) {
        load_row<TS, EQ, false>(M + (r0 + r) * ld, q0, d, lane_id(), h[r]);
      } else {
#pragma unroll
        for (int e = 0; e < EQ; ++e) h[r][e] = TS(0);
      }
    }
    clear_tail<TS, EQ, NR>(q0, d, lane_id(), h);
  }
  // Entry e of row r.  FP32 rows are widened at each use: hoisted out of the step loop, the
  // conversions would take twice the registers.
  __device__ __forceinline__ double value(int r, int e) const {
    if constexpr (sizeof(TS) == 4) {
      float t = h[r][e];
      asm volatile("" : "+v"(t));
      return (double)t;
    } else {
      return h[r][e];
    }
  }
  // part[p * NR + r], p < kResParts: partial products of row r with v (LDS, dpad entries)
  __device__ __forceinline__ void dots(const double* v, int dpad, double* part) const {
    const int lane = lane_id(), q0 = wave_id() * kWave * EQ;
    double dot[NR];
#pragma unroll
    for (int r = 0; r < NR; ++r) dot[r] = 0.0;
    if (q0 < dpad) {
#pragma unroll
      for (int j = 0; j < L::J; ++j)
#pragma unroll
        for (int vv = 0; vv < L::V; ++vv) {
          const double x = v[q0 + L::col(j, lane, vv)];
#pragma unroll
          for (int r = 0; r < NR; ++r) dot[r] += value(r, j * L::V + vv) * x;
        }
    }
    const double s = row_sums<NR>(dot);
    constexpr int G = 16 / NR;
    if (lane % G == 0) part[(wave_id() * 4 + lane / 16) * NR + (lane % 16) / G] = s;
  }
  static __device__ __forceinline__ double total(const double* part, int r) {
    double s = part[r];
#pragma unroll
    for (int p = 1; p < kResParts; ++p) s += part[p * NR + r];
    return s;
  }
  // put(col, sum_r u[r] h[r][col]) for this wave's quarter of [0, d) (u in LDS)
  template <typename F>
  __device__ __forceinline__ void combine(const double* u, int d, F&& put) const {
    const int lane = lane_id(), q0 = wave_id() * kWave * EQ;
    double acc[EQ];
#pragma unroll
    for (int e = 0; e < EQ; ++e) acc[e] = 0.0;
#pragma unroll
    for (int r = 0; r < NR; ++r) {
      const double ur = u[r];
#pragma unroll
      for (int e = 0; e < EQ; ++e) acc[e] += ur * value(r, e);
    }
#pragma unroll
    for (int j = 0; j < L::J; ++j)
#pragma unroll
      for (int vv = 0; vv < L::V; ++vv) {
        const int col = q0 + L::col(j, lane, vv);
        if (col < d) put(col, acc[j * L::V + vv]);
      }
  }
};

// Barrier of the inner-solve group: one counter for small groups, the two-level
// form (per-XCD counters, then one top counter) from 256 workgroups on, where
// one counter's arrivals queue up (128 workgroups: 2.1 us either way; 256:
// 3.8 us flat against 2.2 us two-level).
__device__ __forceinline__ bool cg_sync(const SolveArgs& a, unsigned& epoch, int* s_flag) {
  return a.cg_hier ? barrier_hier(a.bar_cgh, epoch, a.Gc, a.err, s_flag, a.spin_fast)
                   : barrier_flat(a.bar_cg, epoch, a.Gc, a.err, s_flag, a.spin_fast);
}

// GRAM: the inner CG applies (SA)^T SA through the precomputed H (owners form
// their entries of q directly); otherwise through two passes over SA rows.
//
// Up to 512 columns two workgroups share a CU (256 registers): the gradient pass of a tall
// matrix then has twice the rows in flight (536870 x 500 FP64, 300 rows of SA, 8 outer steps:
// 5.0 ms with one, 2.9 with two).  Only the streaming forms of 257 to 512 columns have to be
// held to it (28 to 44 bytes of spills with an FP32 operator); asked of the narrower ones, which
// need fewer anyway, the bound only costs the CG schedule (4096 x 256: 4.9 against 4.5 ms).
template <typename TA, typename TS, typename TV, int EPT, bool GRAM, bool RES>
__global__ __launch_bounds__(kBlock, EPT == 8 && !GRAM ? 2 : 1) void solve_kernel(SolveArgs a) {
  // a driver that enqueues several solves ahead stops them once it is done
  if (a.skip && __hip_atomic_load(a.skip, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) return;
  extern __shared__ double smem[];
  const int cpw = a.cpw;
  double* vbuf = smem;                 // x (A pass) or p (CG, as TV)
  double* rbuf = vbuf + a.dpad;        // workgroup reduction buffer
  double* colbuf = rbuf + a.dpad;      // owned-column sums
  double* scratch = colbuf + cpw;      // kBlock doubles
  double* own_x = scratch + kBlock;    // owner-private state of the owned columns
  double* own_xp = own_x + cpw;
  double* own_rhs = own_xp + cpw;
  TV* own_r = (TV*)(own_rhs + cpw);
  TV* own_z = (TV*)(own_rhs + 2 * cpw);
  __shared__ double s_red[2 * kWavesPerBlock];
  __shared__ double s_part[2 * kQuarterRows * kWavesPerBlock];  // rowpass_quarters exchange
  constexpr int EQ = EPT >= 4 ? EPT / 4 : 1;
  constexpr int NR = resident_rows(sizeof(TS), EPT, GRAM);
  // (streaming at 2048 columns spilled 100 registers: Primal-Dual 16384 x 4096 59.7 against 54.7
  // ms by barrier)
  constexpr bool TAGGED = GRAM && RES && tagged_gram(sizeof(TS), EPT);
  constexpr bool TAGGED_SA = !GRAM && RES && tagged_streaming(EPT);
  __shared__ double s_res[kResParts * NR];  // resident rows' partial products
  __shared__ double s_u[NR], s_y[NR];       // SA rows: u of this step, y of the last one
  __shared__ int s_flag;

  const int w = blockIdx.x;
  const int G = a.G, Gc = a.Gc;
  const int d = a.d;
  const bool in_cg = w < Gc;
  unsigned ep_all = 0, ep_cg = 0, tag = 0;
  const int c_lo = in_cg ? min(d, w * cpw) : d;
  const int c_hi = in_cg ? min(d, c_lo + cpw) : d;
  const int nown = c_hi - c_lo;
  double* scal_w = a.scal + (int64_t)w * kScal;
  // CG vectors exchanged between the CG workgroups: every access goes through
  // co_store / co_load (agent-scope, global address space)
  TV* r = (TV*)a.r;
  TV* P[2] = {(TV*)a.p0, (TV*)a.p1};
  TV* partS = (TV*)a.partS;
  const TA* A = (const TA*)a.A;
  const TS* SA = (const TS*)a.SA;
  constexpr int RA = RowsInFlight<TA, EPT>::value;
  constexpr int RS = RowsInFlight<TS, EPT>::value;
  constexpr int NPT = EPT >= 4 ? EPT / 4 : 1;  // vector entries per thread (dpad / kBlock)

  for (int i = threadIdx.x; i < nown; i += kBlock) {
    const int c = c_lo + i;
    own_x[i] = a.x[c];
    own_xp[i] = a.xp_from_x ? a.x[c] : a.xp[c];
    own_rhs[i] = a.rhs ? a.rhs[c] : 0.0;
  }
  // this workgroup's rows of the CG operator H: the first NR stay in registers during the
  // inner solve, further ones are read from L2 / Infinity Cache on every step
  const TS* Hrows = (GRAM && in_cg) ? (const TS*)a.H + (int64_t)c_lo * a.ldh : nullptr;
  const int64_t ldhr = a.ldh;
  __syncthreads();

  // Single-reduction CG only where the sub-problem is well conditioned for its
  // precision: trace(H) / lambda bounds kappa(H + lambda I) from above.  Every CG
  // workgroup sums the same diagonal in the same order, so all decide alike.
  bool cg1 = false;
  if (GRAM && a.cg1 && in_cg) {
    const TS* Hm = (const TS*)a.H;
    double tr = 0.0;
    for (int c = threadIdx.x; c < d; c += kBlock) tr += (double)Hm[(int64_t)c * a.ldh + c];
    tr = block_sum(tr, s_red);
    cg1 = tr <= kCg1MaxCond * a.lam;
  }

  const int64_t a_r0 = row_split_bound(a.n, G, a.xw, w);
  const int64_t a_r1 = row_split_bound(a.n, G, a.xw, w + 1);
  const int64_t s_r0 = in_cg ? a.m * w / Gc : 0;
  const int64_t s_r1 = in_cg ? a.m * (w + 1) / Gc : 0;

  int64_t outer = 0, inner_total = 0, inner_max = 0;
  double last_step = 0.0, last_gnorm = 0.0;
  int status = MIHS_MAX_ITER;
  bool alive = true;

  // x in LDS for the first gradient pass; later passes get it at the end of
  // the previous iteration, fetched together with the stop test's sums
  for (int c = threadIdx.x; c < a.dpad; c += kBlock) vbuf[c] = (c < d) ? co_load(a.x + c) : 0.0;
  __syncthreads();
  while (outer < a.max_outer) {
    // ---- A1 (all): partial A^T (b - A x) over this workgroup's rows
    if constexpr (EPT == 64) {
      double acc[16];
#pragma unroll
      for (int e = 0; e < 16; ++e) acc[e] = 0.0;
      rowpass_quarters<TA, 16, true, quarter_rows<TA>()>(A, a.lda, a_r0, a_r1, d, vbuf, a.b, acc, s_part);
      store_quarters<TA, 16>(acc, a.partA + (int64_t)w * a.dpad, d);
      __syncthreads();
    } else {
      double acc[EPT];
#pragma unroll
      for (int e = 0; e < EPT; ++e) acc[e] = 0.0;
      double ssq = 0.0;
      rowpass<TA, double, EPT, true, RA>(A, a.lda, a_r0, a_r1, d, vbuf, a.b, acc, ssq);
      wg_store_partial<TA, double, EPT>(acc, rbuf, a.partA + (int64_t)w * a.dpad, d);
    }
    if (!(alive = barrier_hier(a.bar_all, ep_all, G, a.err, &s_flag, a.spin_fast))) break;

    int decision = 0;  // 0 continue, 1 converged, 2 breakdown
    if (in_cg) {
      ResidentRows<TS, EQ, NR> res;
      if constexpr (RES) {
        // (opaque: as loop invariants the rows' addresses and bounds would be kept, or spilled,
        // across the gradient pass)
        const TS* M = GRAM ? Hrows : SA + s_r0 * a.ldsa;
        int64_t ldm = GRAM ? ldhr : a.ldsa;
        int nrows = GRAM ? nown : (int)(s_r1 - s_r0), dd = d;
        asm volatile("" : "+s"(M), "+s"(ldm), "+s"(nrows), "+s"(dd));
        res.load(M, ldm, 0, nrows, dd);
      }
      // colbuf[i] = row i of H . v for the owned rows (thread i < nown reads its own; the
      // barrier inside orders the rest)
      auto gram_product = [&](const TV* v) {
        if constexpr (RES) {
          res.dots(v, a.dpad, s_res);
          __syncthreads();
          if ((int)threadIdx.x < nown) colbuf[threadIdx.x] = res.total(s_res, threadIdx.x);
        } else {
          rowdots<TS, TV, EPT>(Hrows, ldhr, 0, nown, d, v, colbuf);
          __syncthreads();
        }
      };
      // u = cs y_prev - SA v on this workgroup's rows of SA (keep: y_prev is the last u),
      // partS = SA^T u; returns ||u||^2 over those rows
      auto sa_pass = [&](const TV* v, double cs, bool keep) -> TV {
        if constexpr (RES) {
          res.dots(v, a.dpad, s_res);
          __syncthreads();
          if (threadIdx.x < NR) {
            const double y = keep ? cs * s_y[threadIdx.x] : 0.0;
            const double u = y - res.total(s_res, threadIdx.x);
            s_u[threadIdx.x] = u;
            s_y[threadIdx.x] = u;
          }
          __syncthreads();
          double ss = 0.0;
#pragma unroll
          for (int r = 0; r < NR; ++r) ss += s_u[r] * s_u[r];
          if (TAGGED_SA && a.partT) {
            ++tag;
            res.combine(s_u, d, [&](int col, double v) {
              tagged_put(a.partT + 2 * ((int64_t)w * a.dpad + col), v, tag);
            });
          } else {
            double* out = (double*)partS + (int64_t)w * a.dpad;
            res.combine(s_u, d, [&](int col, double v) { co_store(out + col, v); });
          }
          return ss;
        } else {
          TV ssq = TV(0);
          TV acc[EPT];
#pragma unroll
          for (int e = 0; e < EPT; ++e) acc[e] = TV(0);
          rowpass<TS, TV, EPT, false, RS>(SA, a.ldsa, s_r0, s_r1, d, v, keep ? a.yrow : nullptr,
                                          acc, ssq, cs, a.aab ? a.yrow : nullptr);
          wg_store_partial<TS, TV, EPT>(acc, (TV*)rbuf, partS + (int64_t)w * a.dpad, d);
          return wg_sum_ssq(ssq, s_red);
        }
      };
      // ---- A2: owners form g and start CG (z = 0, r = p = g)
      owned_column_sums(a.partA, G, a.dpad, c_lo, nown, colbuf, scratch);
      double rr_part = 0.0;
      for (int i = threadIdx.x; i < nown; i += kBlock) {
        const TV gt = (TV)(colbuf[i] + own_rhs[i] - a.lam * own_x[i]);
        own_r[i] = gt;
        own_z[i] = TV(0);
        co_store(r + c_lo + i, gt);
        co_store(P[0] + c_lo + i, gt);
        rr_part += (double)gt * (double)gt;
      }
      rr_part = block_sum(rr_part, s_red);
      if (threadIdx.x == 0) co_store(scal_w + 0, rr_part);
      if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;

      // the CG on resident rows and the single-reduction form start from the whole of
      // r = g: its loads are issued before the slot sum
      TV rpre[NPT];
      if (TAGGED || TAGGED_SA || (GRAM && cg1)) {
#pragma unroll
        for (int i = 0; i < NPT; ++i) {
          const int c = threadIdx.x + i * kBlock;
          rpre[i] = (c < d) ? co_load(r + c) : TV(0);
        }
      }
      double rr0, unused;
      sum2_slots(a.scal, Gc, 0, 0, s_red, rr0, unused);
      last_gnorm = sqrt(rr0);
      int64_t k = 0;
      if (!(rr0 > 0.0)) {
        decision = (rr0 == 0.0) ? 1 : 2;  // stationary point, or NaN
      } else {
        const double stop = a.eps_sub * a.eps_sub * rr0;
        bool solved = false;
        const int tid = threadIdx.x, lane = lane_id();
        const bool own = tid < nown;
        const double lt = a.lam;
        bool ok = true;  // this thread met no timeout
        // owned row tid of H v (0 elsewhere)
        auto product = [&](const double* v) {
          res.dots(v, a.dpad, s_res);
          lds_barrier();
          return own ? res.total(s_res, tid) : 0.0;
        };
        // this thread's columns of the vector to multiply go to LDS; false after a timeout
        auto stage = [&](auto&& value) {
#pragma unroll
          for (int i = 0; i < NPT; ++i) {
            const int c = tid + i * kBlock;
            const double v = value(i);
            if (c < a.dpad) vbuf[c] = v;
          }
          if (!ok) s_flag = 0;
          lds_barrier();
          return s_flag != 0;
        };
        auto put_scalars = [&](double s0, double s1) {
          if (tid < 2)
            tagged_put(a.tags + (scalar_slot(tag) * (4u * Gc) + (4u * w + 2u * tid)),
                       tid ? s1 : s0, tag);
        };
        // sums of the workgroups' scalars under the current tag, for this wave (lane l
        // takes workgroups l, l + 64, ..; d <= 2048 in 16 columns each: at most 128)
        constexpr int SL = EPT <= 16 ? 1 : 2;
        auto get_scalars = [&](double& t0, double& t1) {
          const tagged_t* ps[2 * SL];
          bool on[2 * SL];
          double v[2 * SL];
#pragma unroll
          for (int i = 0; i < SL; ++i) {
            const int q = lane + i * kWave;
            on[2 * i] = on[2 * i + 1] = q < Gc;
            ps[2 * i] = a.tags + (scalar_slot(tag) * (4u * Gc) + 4u * (q < Gc ? q : 0));
            ps[2 * i + 1] = ps[2 * i] + 2;
          }
          if (!tagged_get<2 * SL>(ps, on, tag, v, a.err, a.spin_fast)) {
            ok = false;
#pragma unroll
            for (int i = 0; i < 2 * SL; ++i) v[i] = 0.0;
          }
          double a0 = v[0], a1 = v[1];
#pragma unroll
          for (int i = 1; i < SL; ++i) {
            a0 += v[2 * i];
            a1 += v[2 * i + 1];
          }
          t0 = wave_sum(a0);
          t1 = wave_sum(a1);
        };
        // All-gather: the owned entry v and two scalars (first wave) to everybody's x and
        // sums.
        auto exchange = [&](double v, double s0, double s1, double (&x)[NPT], double& t0,
                            double& t1) {
          ++tag;
          tagged_t* tv = a.tagw + vector_slot(tag) * (2u * a.dpad);
          if (own) tagged_put(tv + 2 * (c_lo + tid), v, tag);
          put_scalars(s0, s1);
          // the vector first, then the scalars (polled together: 4096 x 256 5.26 instead of
          // 4.71 ms, every retry repeats all loads)
          const tagged_t* ps[NPT];
          bool on[NPT];
#pragma unroll
          for (int i = 0; i < NPT; ++i) {
            const int c = tid + i * kBlock;
            on[i] = c < d;
            ps[i] = tv + 2 * (on[i] ? c : 0);
          }
          if (!tagged_get<NPT>(ps, on, tag, x, a.err, a.spin_fast)) {
            ok = false;
#pragma unroll
            for (int i = 0; i < NPT; ++i) x[i] = 0.0;
          }
          get_scalars(t0, t1);
        };
        if constexpr (TAGGED) {
          // ---- CG on resident rows of H, d <= 2048.  A step is a chain of latencies, so it has as few
          // links as the recurrences allow: every thread keeps its columns of the full
          // vectors in registers (LDS holds the one that is multiplied), the first wave's
          // lanes i < nown finish the owned rows and their sums without a barrier, the
          // exchanged vector (d <= 2048) and scalars travel as tagged values, and every
          // wave adds the scalars itself.  Each workgroup adds in the same order, so all
          // take the same steps.  4096 x 256: 4.0 us a step with the barrier forms below.
          double z = 0.0, x[NPT];
          if (cg1) {
            // single-reduction CG (Chronopoulos-Gear): s = M p by its own recurrence, one
            // product (w = M r) and one exchange (w, r^T r, w^T r) per step
            double rv[NPT], sv[NPT], mu = rr0, alpha = 0.0, p = 0.0, t0, nu;
            if (!(alive = stage([&](int i) { return rv[i] = rpre[i]; }))) break;
            double rc = own ? vbuf[c_lo + tid] : 0.0;
            double wc = product(vbuf) + lt * rc;
            exchange(wc, 0.0, row16_sum(wc * rc), x, t0, nu);
            alpha = mu / nu;
            if (!(nu > 0.0) || !isfinite(alpha)) decision = 2;
            p = rc;
#pragma unroll
            for (int i = 0; i < NPT; ++i) sv[i] = x[i];
            while (decision == 0) {
              z += alpha * p;
              if (!(alive = stage([&](int i) { return rv[i] -= alpha * sv[i]; }))) break;
              ++k;
              rc = own ? vbuf[c_lo + tid] : 0.0;
              wc = product(vbuf) + lt * rc;
              double mu_n, nu_n;
              exchange(wc, row16_sum(rc * rc), row16_sum(wc * rc), x, mu_n, nu_n);
              if (mu_n <= stop || k >= a.max_inner) break;
              const double bt = mu_n / mu;
              const double den = nu_n - bt * mu_n / alpha;
              const double an = mu_n / den;
              if (!(den > 0.0) || !isfinite(an)) {
                decision = 2;
                break;
              }
              mu = mu_n;
              alpha = an;
#pragma unroll
              for (int i = 0; i < NPT; ++i) sv[i] = x[i] + bt * sv[i];
              p = rc + bt * p;
            }
          } else {
            // CG with two reductions: p . q among the first waves only (the owners need the
            // step length), then the new r and r^T r to everybody
            double pv[NPT], rr = rr0, bc = 0.0, rn = own ? own_r[tid] : 0.0, t1;
            bool first = true;
#pragma unroll
            for (int i = 0; i < NPT; ++i) x[i] = rpre[i];
            while (true) {
              if (!(alive = stage([&](int i) {
                      return pv[i] = first ? x[i] : x[i] + bc * pv[i];
                    })))
                break;
              first = false;
              const double pc = own ? vbuf[c_lo + tid] : 0.0;
              const double h = product(vbuf);
              double rpart = 0.0;
              ++tag;
              if (wave_id() == 0) {
                double pqs;
                put_scalars(row16_sum(pc * (h + lt * pc)), 0.0);
                get_scalars(pqs, t1);
                const double acg = rr / pqs;
                if (!(pqs > 0.0) || !isfinite(acg)) {
                  rpart = -1.0;  // breakdown: a negative r^T r tells everybody
                } else {
                  z += acg * pc;
                  rn -= acg * (h + lt * pc);
                  rpart = row16_sum(rn * rn);
                }
              }
              double rr_new;
              exchange(rn, rpart, 0.0, x, rr_new, t1);
              if (rr_new < 0.0) {
                decision = 2;
                break;
              }
              ++k;
              if (rr_new <= stop || k >= a.max_inner) break;
              bc = rr_new / rr;
              rr = rr_new;
            }
          }
          if (!alive) break;
          if (own) own_z[tid] = z;
          // a timeout in the last exchange
          if (!ok) s_flag = 0;
          lds_barrier();
          if (!(alive = s_flag != 0)) break;
          solved = true;
        }
        if constexpr (TAGGED_SA) {
          if (a.partT) {
            // ---- the streaming solvers on resident rows of SA, exchanged the same way: the
            // workgroups' partial vectors SA^T u go tagged to their columns' owners (a
            // 16 x 16 thread grid, column x workgroup), the owners' new entries and scalars
            // tagged to everybody.  2048 x 2048: 24 us an AAb step with rows from memory
            // and barriers.
            double z = 0.0, x[NPT], t0, t1;
            // owned entry tid of sum_w partT (0 elsewhere)
            auto owned_sum = [&]() {
              constexpr int NB = 4;  // workgroups per thread (Gc <= 16 NB)
              const int col = tid % 16, q = tid / 16;
              const tagged_t* ps[NB];
              bool on[NB];
              double v[NB], sum = 0.0;
#pragma unroll
              for (int i = 0; i < NB; ++i) {
                on[i] = col < nown && q + 16 * i < Gc;
                ps[i] = a.partT +
                        2 * ((int64_t)(on[i] ? q + 16 * i : 0) * a.dpad + (on[i] ? c_lo + col : 0));
              }
              const bool got = tagged_get<NB>(ps, on, tag, v, a.err, a.spin_fast);
              if (!got) ok = false;
#pragma unroll
              for (int i = 0; i < NB; ++i) sum += got && on[i] ? v[i] : 0.0;
              scratch[tid] = sum;
              lds_barrier();
              double s = 0.0;
              if (own)
#pragma unroll
                for (int i = 0; i < 16; ++i) s += scratch[i * 16 + tid];
              return s;
            };
            if (a.aab) {
              // AAb_Solver (Algorithm 6), see the barrier form below
              const double theta1 = sqrt(rr0);
              double theta = 0.0, rho_prev = 1.0, rhobar = 0.0, cs = 0.0, sn = 0.0, phi = 0.0;
              double dv = 0.0, scale = theta1;
              bool first = true;
#pragma unroll
              for (int i = 0; i < NPT; ++i) x[i] = rpre[i];
              while (true) {
                if (!(alive = stage([&](int i) { return x[i] / scale; }))) break;
                const double vc = own ? vbuf[c_lo + tid] : 0.0;
                const double ssq = sa_pass(vbuf, -theta / rho_prev, !first);
                put_scalars(ssq, 0.0);
                const double my = -owned_sum();  // (M^T y) of the owned column
                double rho2, th2;
                get_scalars(rho2, t1);
                const double rho = sqrt(rho2);
                double t;
                if (first) {
                  rhobar = sqrt(rho * rho + a.lam);
                  cs = rho / rhobar;
                  sn = sqrt(a.lam) / rhobar;
                  phi = theta1 / rhobar;
                  dv = vc / rhobar;
                  z = phi * dv;
                  t = INFINITY;
                  first = false;
                } else {
                  const double lbar = sqrt(a.lam + (sn * theta) * (sn * theta));
                  const double thetabar = cs * theta;
                  rhobar = sqrt(rho * rho + lbar * lbar);
                  cs = rho / rhobar;
                  sn = lbar / rhobar;
                  phi = -phi * thetabar / rhobar;
                  dv = (vc - thetabar * dv) / rhobar;
                  z = z + phi * dv;
                  t = fabs(phi * rhobar) / theta1;
                  ++k;
                }
                if (!isfinite(phi) || !isfinite(rhobar)) {
                  decision = 2;
                  break;
                }
                if (!(t >= a.eps_sub) || k >= a.max_inner || !(rho > 0.0)) break;
                // w = M^T p - rho v = (M^T y) / rho - rho v on the owned columns
                const double wc = own ? my / rho - rho * vc : 0.0;
                exchange(wc, row16_sum(wc * wc), 0.0, x, th2, t1);
                theta = sqrt(th2);
                if (!(theta > 0.0)) break;  // w = 0: the iterate is exact
                rho_prev = rho;
                scale = theta;
              }
            } else {
              double pv[NPT], rr = rr0, bc = 0.0, rn = own ? own_r[tid] : 0.0;
              bool first = true;
#pragma unroll
              for (int i = 0; i < NPT; ++i) x[i] = rpre[i];
              while (true) {
                if (!(alive = stage([&](int i) {
                        return pv[i] = first ? x[i] : x[i] + bc * pv[i];
                      })))
                  break;
                first = false;
                const double pc = own ? vbuf[c_lo + tid] : 0.0;
                const double ssq = sa_pass(vbuf, 0.0, false);
                put_scalars(ssq, row16_sum(pc * pc));
                const double mp = -owned_sum();
                double uu, pp, rr_new;
                get_scalars(uu, pp);
                const double pq = uu + a.lam * pp;
                const double acg = rr / pq;
                if (!(pq > 0.0) || !isfinite(acg)) {
                  decision = 2;
                  break;
                }
                z += acg * pc;
                rn -= acg * (mp + lt * pc);
                exchange(rn, row16_sum(rn * rn), 0.0, x, rr_new, t0);
                ++k;
                if (rr_new <= stop || k >= a.max_inner) break;
                bc = rr_new / rr;
                rr = rr_new;
              }
            }
            if (!alive) break;
            if (own) own_z[tid] = z;
            // a timeout in the last exchange
            if (!ok) s_flag = 0;
            lds_barrier();
            if (!(alive = s_flag != 0)) break;
            solved = true;
          }
        }
        if (solved) {
        } else if (!GRAM && a.aab) {
          // AAb_Solver (Algorithm 6) on ((SA)^T SA + lambda I) z = g: Golub-Kahan
          // bidiagonalisation of M = SA started from v = g / ||g||, the
          // sqrt(lambda) I block folded in by Givens rotations.  One pass over
          // the owned rows of M per step gives y = M v - theta p and M^T y
          // together (p = y_prev / rho_prev is never normalised in memory, the
          // scale rides on the next pass), then two barriers: one for rho = ||y||
          // and M^T y, one for theta = ||w||, w = M^T p - rho v.  Every CG
          // workgroup keeps v in LDS and the same scalars; owners keep the
          // direction vector (in own_r) and the iterate z on their columns.
          TV* vp = (TV*)vbuf;
          TV* wv = r;  // w, exchanged through the residual buffer
          TV* dv = own_r;
          const double theta1 = sqrt(rr0);
          for (int c = threadIdx.x; c < a.dpad; c += kBlock)
            vp[c] = (c < d) ? (TV)((double)co_load(r + c) / theta1) : TV(0);
          __syncthreads();
          double theta = 0.0, rho_prev = 1.0, rhobar = 0.0, cs = 0.0, sn = 0.0, phi = 0.0;
          bool first = true;
          while (true) {
            // u = -(M v - theta p) = (-theta / rho_prev) y_prev - M v
            const TV ssq = sa_pass(vp, -theta / rho_prev, !first);
            if (threadIdx.x == 0) co_store(scal_w + 1, (double)ssq);
            if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
            // colbuf = -M^T y on the owned columns; rho = ||y||
            owned_column_sums(partS, Gc, a.dpad, c_lo, nown, colbuf, scratch);
            double rho2, unused2;
            sum2_slots(a.scal, Gc, 1, 1, s_red, rho2, unused2);
            const double rho = sqrt(rho2);
            double t;
            if (first) {
              rhobar = sqrt(rho * rho + a.lam);
              cs = rho / rhobar;
              sn = sqrt(a.lam) / rhobar;
              phi = theta1 / rhobar;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const TV dn = (TV)((double)vp[c_lo + i] / rhobar);
                dv[i] = dn;
                own_z[i] = (TV)(phi * (double)dn);
              }
              t = INFINITY;
              first = false;
            } else {
              const double lbar = sqrt(a.lam + (sn * theta) * (sn * theta));
              const double thetabar = cs * theta;
              rhobar = sqrt(rho * rho + lbar * lbar);
              cs = rho / rhobar;
              sn = lbar / rhobar;
              phi = -phi * thetabar / rhobar;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const TV dn =
                    (TV)(((double)vp[c_lo + i] - thetabar * (double)dv[i]) / rhobar);
                dv[i] = dn;
                own_z[i] = own_z[i] + (TV)(phi * (double)dn);
              }
              t = fabs(phi * rhobar) / theta1;
              ++k;
            }
            if (!isfinite(phi) || !isfinite(rhobar)) {
              decision = 2;
              break;
            }
            // stop on the relative residual of the current iterate; rho = 0
            // ends the Krylov space (the iterate is then exact)
            if (!(t >= a.eps_sub) || k >= a.max_inner || !(rho > 0.0)) break;
            // w = M^T p - rho v = (M^T y) / rho - rho v on the owned columns
            double th_part = 0.0;
            for (int i = threadIdx.x; i < nown; i += kBlock) {
              const TV wc = (TV)(-colbuf[i] / rho - rho * (double)vp[c_lo + i]);
              co_store(wv + c_lo + i, wc);
              th_part += (double)wc * (double)wc;
            }
            th_part = block_sum(th_part, s_red);
            if (threadIdx.x == 0) co_store(scal_w + 2, th_part);
            if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
            double th2;
            sum2_slots(a.scal, Gc, 2, 2, s_red, th2, unused2);
            theta = sqrt(th2);
            if (!(theta > 0.0)) break;  // w = 0: the iterate is exact
            rho_prev = rho;
            for (int c = threadIdx.x; c < a.dpad; c += kBlock)
              vp[c] = (c < d) ? (TV)((double)co_load(wv + c) / theta) : TV(0);
            __syncthreads();
          }
          if (!alive) break;
        } else if (GRAM && cg1) {
          // Single-reduction CG (Chronopoulos-Gear): with s = M p kept by its own
          // recurrence, one matrix product (w = M r on the owned rows) and one
          // fused reduction (r^T r, w^T r) per step, so one barrier per step.
          // Every CG workgroup keeps full copies of r and s in LDS (identical
          // arithmetic everywhere), gathers w from global memory (two buffers,
          // alternating) and owns p and z on its columns.
          TV* rv = (TV*)vbuf;
          TV* sv = (TV*)rbuf;
          const TV lt = (TV)a.lam;
#pragma unroll
          for (int i = 0; i < NPT; ++i) {
            const int c = threadIdx.x + i * kBlock;
            if (c < a.dpad) rv[c] = rpre[i];
          }
          __syncthreads();
          int wb = 0;
          double mu = rr0, alpha = 0.0, unused2;
          {
            gram_product(rv);
            double nu_part = 0.0;
            for (int i = threadIdx.x; i < nown; i += kBlock) {
              const TV rc = rv[c_lo + i];
              const TV wc = (TV)colbuf[i] + lt * rc;
              co_store(P[wb] + c_lo + i, wc);
              nu_part += (double)wc * (double)rc;
            }
            nu_part = block_sum(nu_part, s_red);
            if (threadIdx.x == 0) co_store(scal_w + 1, nu_part);
            if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
              const int c = threadIdx.x + i * kBlock;
              rpre[i] = (c < d) ? co_load(P[wb] + c) : TV(0);  // w, for s below
            }
            double nu;
            sum2_slots(a.scal, Gc, 1, 1, s_red, nu, unused2);
            alpha = mu / nu;
            if (!(nu > 0.0) || !isfinite(alpha)) decision = 2;
          }
          if (decision == 0) {
            // s = w, p = r
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
              const int c = threadIdx.x + i * kBlock;
              if (c < a.dpad) sv[c] = rpre[i];
            }
            for (int i = threadIdx.x; i < nown; i += kBlock) own_r[i] = rv[c_lo + i];
            __syncthreads();
            while (true) {
              const TV at = (TV)alpha;
              for (int i = threadIdx.x; i < nown; i += kBlock) own_z[i] = own_z[i] + at * own_r[i];
              for (int c = threadIdx.x; c < a.dpad; c += kBlock) rv[c] = rv[c] - at * sv[c];
              __syncthreads();
              ++k;
              wb ^= 1;
              gram_product(rv);
              double mu_p = 0.0, nu_p = 0.0;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const TV rc = rv[c_lo + i];
                const TV wc = (TV)colbuf[i] + lt * rc;
                co_store(P[wb] + c_lo + i, wc);
                mu_p += (double)rc * (double)rc;
                nu_p += (double)wc * (double)rc;
              }
              block_sum2(mu_p, nu_p, s_red);
              // the step's scalar slots alternate like w: one barrier separates
              // a step's reads of a slot pair from its next write (two steps on)
              const int sp = 2 + 4 * wb;
              if (threadIdx.x == 0) {
                co_store(scal_w + sp, mu_p);
                co_store(scal_w + sp + 1, nu_p);
              }
              if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
              // fetch w (written by every CG workgroup before the barrier) while
              // the scalar partials are summed
              TV wpre[NPT];
#pragma unroll
              for (int i = 0; i < NPT; ++i) {
                const int c = threadIdx.x + i * kBlock;
                wpre[i] = (c < d) ? co_load(P[wb] + c) : TV(0);
              }
              double mu_n, nu_n;
              sum2_slots(a.scal, Gc, sp, sp + 1, s_red, mu_n, nu_n);
              if (mu_n <= stop || k >= a.max_inner) break;
              const double bt = mu_n / mu;
              const double den = nu_n - bt * mu_n / alpha;
              const double an = mu_n / den;
              if (!(den > 0.0) || !isfinite(an)) {
                decision = 2;
                break;
              }
              mu = mu_n;
              alpha = an;
              // s = w + beta s (full), p = r + beta p (owned)
              const TV btt = (TV)bt;
#pragma unroll
              for (int i = 0; i < NPT; ++i) {
                const int c = threadIdx.x + i * kBlock;
                if (c < a.dpad) sv[c] = wpre[i] + btt * sv[c];
              }
              for (int i = threadIdx.x; i < nown; i += kBlock)
                own_r[i] = rv[c_lo + i] + btt * own_r[i];
              __syncthreads();
            }
          }
          if (!alive) break;
        } else {
          double rr = rr0;
          TV* vp = (TV*)vbuf;
          while (true) {
            // ---- C1: p = r + beta_cg p_prev (k > 0), staged in LDS over p_prev
            // (every CG workgroup holds the whole of p: the same arithmetic on the
            // same values everywhere).  The loads of r and of the residual
            // partials are all issued before use; the first direction is g.
            TV rv[NPT], pv[NPT];
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
              const int c = threadIdx.x + i * kBlock;
              rv[i] = TV(0);
              pv[i] = TV(0);
              if (c < d) {
                if (k == 0) {
                  rv[i] = co_load(P[0] + c);
                } else {
                  rv[i] = co_load(r + c);
                  pv[i] = vp[c];
                }
              }
            }
            TV bc = TV(0);
            if (k > 0) {
              double rr_new;
              sum2_slots(a.scal, Gc, 3, 3, s_red, rr_new, unused);
              if (rr_new <= stop || k >= a.max_inner) break;
              bc = (TV)(rr_new / rr);
              rr = rr_new;
            }
#pragma unroll
            for (int i = 0; i < NPT; ++i) {
              const int c = threadIdx.x + i * kBlock;
              if (c < a.dpad) {
                const TV p = (k == 0) ? rv[i] : (TV)(rv[i] + bc * pv[i]);
                vp[c] = (c < d) ? p : TV(0);
              }
            }
            for (int c = NPT * kBlock + threadIdx.x; c < a.dpad; c += kBlock) vp[c] = TV(0);
            __syncthreads();
            double rpart = 0.0;
            if (GRAM) {
              // q = H p + lambda p on the owned columns (colbuf <- H p)
              gram_product(vp);
              double pq = 0.0;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const double pc = (double)vp[c_lo + i];
                pq += pc * (colbuf[i] + a.lam * pc);
              }
              pq = block_sum(pq, s_red);
              if (threadIdx.x == 0) co_store(scal_w + 1, pq);
              if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
              double pqs, unused2;
              sum2_slots(a.scal, Gc, 1, 1, s_red, pqs, unused2);
              const double acg = rr / pqs;
              if (!(pqs > 0.0) || !isfinite(acg)) {
                decision = 2;
                break;
              }
              const TV at = (TV)acg, lt = (TV)a.lam;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const TV pc = vp[c_lo + i];
                const TV q = (TV)colbuf[i] + lt * pc;
                own_z[i] = own_z[i] + at * pc;
                const TV rn = own_r[i] - at * q;
                own_r[i] = rn;
                co_store(r + c_lo + i, rn);
                rpart += (double)rn * (double)rn;
              }
            } else {
              const TV ssq = sa_pass(vp, 0.0, false);
              double pp = 0.0;
              for (int c = c_lo + threadIdx.x; c < c_hi; c += kBlock)
                pp += (double)vp[c] * (double)vp[c];
              pp = block_sum(pp, s_red);
              if (threadIdx.x == 0) {
                co_store(scal_w + 1, pp);
                co_store(scal_w + 2, (double)ssq);
              }
              if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;

              // ---- C2: step length (p^T q = ||u||^2 + lambda ||p||^2) and owner updates
              owned_column_sums(partS, Gc, a.dpad, c_lo, nown, colbuf, scratch);
              double ppn, uu;
              sum2_slots(a.scal, Gc, 1, 2, s_red, ppn, uu);
              const double pq = uu + a.lam * ppn;
              const double acg = rr / pq;
              if (!(pq > 0.0) || !isfinite(acg)) {
                decision = 2;
                break;
              }
              const TV at = (TV)acg, lt = (TV)a.lam;
              for (int i = threadIdx.x; i < nown; i += kBlock) {
                const TV pc = vp[c_lo + i];
                const TV q = (TV)(-colbuf[i]) + lt * pc;
                own_z[i] = own_z[i] + at * pc;
                const TV rn = own_r[i] - at * q;
                own_r[i] = rn;
                co_store(r + c_lo + i, rn);
                rpart += (double)rn * (double)rn;
              }
            }
            rpart = block_sum(rpart, s_red);
            if (threadIdx.x == 0) co_store(scal_w + 3, rpart);
            if (!(alive = cg_sync(a, ep_cg, &s_flag))) break;
            ++k;
          }

        }
        if (!alive) break;
      }
      inner_total += k;
      if (k > inner_max) inner_max = k;

      // ---- U: heavy-ball update on owned columns
      double s0 = 0.0, s1 = 0.0;
      if (decision == 0) {
        for (int i = threadIdx.x; i < nown; i += kBlock) {
          const double xc = own_x[i];
          const double xn = xc + a.alpha * (double)own_z[i] + a.beta * (xc - own_xp[i]);
          own_xp[i] = xc;
          own_x[i] = xn;
          co_store(a.x + c_lo + i, xn);
          s0 += (xn - xc) * (xn - xc);
          s1 += xn * xn;
        }
      }
      s0 = block_sum(s0, s_red);
      s1 = block_sum(s1, s_red);
      if (threadIdx.x == 0) {
        co_store(scal_w + 4, s0);
        co_store(scal_w + 5, s1);
        if (w == 0) co_store(a.status, decision);
      }
    }
    if (!(alive = barrier_hier(a.bar_all, ep_all, G, a.err, &s_flag,
                               in_cg ? a.spin_fast : a.spin_idle)))
      break;
    // the updated x (owners stored it before the barrier), the decision and the
    // step sums: all loads issued before any is used
    double xpre[NPT];
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int c = threadIdx.x + i * kBlock;
      xpre[i] = (c < d) ? co_load(a.x + c) : 0.0;
    }
    decision = __hip_atomic_load(a.status, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    if (decision == 1) {
      status = MIHS_CONVERGED;
      break;
    }
    if (decision == 2) {
      status = MIHS_BREAKDOWN;
      break;
    }
    double S0, S1;
    sum2_slots(a.scal, Gc, 4, 5, s_red, S0, S1);
    ++outer;
    last_step = S1 > 0.0 ? sqrt(S0 / S1) : 0.0;
    if (!isfinite(last_step)) {
      status = MIHS_BREAKDOWN;
      break;
    }
    if (a.step_thr > 0.0 && last_step <= a.step_thr) {
      status = MIHS_CONVERGED;
      break;
    }
#pragma unroll
    for (int i = 0; i < NPT; ++i) {
      const int c = threadIdx.x + i * kBlock;
      if (c < a.dpad) vbuf[c] = xpre[i];
    }
    __syncthreads();
  }
  if (!alive) status = MIHS_BARRIER_TIMEOUT;
  // publish the momentum state (the iterate before x) of the owned columns
  for (int i = threadIdx.x; i < nown; i += kBlock) a.xp[c_lo + i] = own_xp[i];
  if (w == 0 && threadIdx.x == 0) {
    a.info->outer_iters = outer;
    a.info->inner_iters_total = inner_total;
    a.info->inner_iters_max = inner_max;
    a.info->rel_step = last_step;
    a.info->grad_norm = last_gnorm;
    a.info->status = status;
    a.info->elapsed_us = 0;
  }
}

typedef void (*SolveKernel)(SolveArgs);

template <typename TA, typename TS, bool GRAM, bool RES, int EPT = 1>
SolveKernel pick_by_ept(int ept) {
  if (ept == EPT) {
    if constexpr (solve_instance(sizeof(TS), EPT, GRAM, RES))
      return solve_kernel<TA, TS, double, EPT, GRAM, RES>;
    else
      return nullptr;
  }
  if constexpr (EPT < 64)
    return pick_by_ept<TA, TS, GRAM, RES, 2 * EPT>(ept);
  else
    return nullptr;
}

// The instances are compiled in four files, by the types of A and of the inner operator.
template <typename TA, typename TS>
SolveKernel pick_kernel_typed(int ept, bool gram, bool res);
extern template SolveKernel pick_kernel_typed<double, double>(int, bool, bool);
extern template SolveKernel pick_kernel_typed<double, float>(int, bool, bool);
extern template SolveKernel pick_kernel_typed<float, double>(int, bool, bool);
extern template SolveKernel pick_kernel_typed<float, float>(int, bool, bool);

}  // namespace mihs
