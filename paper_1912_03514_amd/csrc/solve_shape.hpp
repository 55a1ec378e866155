// Launch shape and workspace of the persistent solve (host only, no HIP calls): which form of the
// kernel runs, on how many workgroups, with how much LDS, and where its scratch lies.
#pragma once

#include <stddef.h>
#include <stdint.h>

#include <algorithm>

#include "internal.hpp"

namespace mihs {

constexpr int kMaxBlocksPerCU = 2;
constexpr size_t kSolveLds = 152 * 1024;  // dynamic LDS at most (the kernel has up to 3 KB more)

// Rows of the inner operator that a workgroup keeps in registers (one quarter of each row per
// wave, `ept / 4` entries per lane): 256 registers per lane, at most 16 rows; 8 streamed rows of
// 4096 columns in either type, as SA^T u is accumulated beside them (16 FP32 rows spilled 1.2 KB
// per lane: 16384 x 4096 with 2457 rows of SA, 76 CG steps, 4.4 ms, and 3.2 with rows read in
// every step).
constexpr int resident_rows(int bytes, int ept, bool gram) {
  const int eq = ept >= 4 ? ept / 4 : 1;
  int r = !gram && ept == 64 ? 8 : 16;
  while (r * eq * bytes / 4 > 256) r /= 2;
  return r;
}

// Which forms of the kernel exist.  The streaming operators have both, as a sketch may have any
// number of rows.  Gram matrices are resident wherever 16 rows fit a workgroup's registers (not
// FP64 rows of 4096 entries) and the grid has d / 16 workgroups.  A whole GPU always has; the
// form that reads H in every step is left for the widths that a partition's CUs may not hold
// (the smallest has 32: d > 512).
constexpr bool solve_instance(int bytes, int ept, bool gram, bool res) {
  return !gram || (res ? resident_rows(bytes, ept, true) == 16 : ept >= 16);
}

// Size of the inner-solve subgroup.  With the operator's rows in registers (`res`) it is the
// fewest workgroups that hold them (NR rows each): a step is then bound by its exchange,
// which costs more the more workgroups take part (one barrier and gather, 2048 entries: 2.9
// us among 64, 3.6 among 128, 3.9 among 256).  Otherwise every step streams the operator:
// 256 workgroups for 8 MB and more, fewer below, at least a few rows each.  No workgroup
// owns more than 16 columns unless the grid is that small: the owners add the gradient's
// partial vectors, 16 columns of 256 partials in one round of loads.  Returns 0 when the
// rows do not fit (res).
inline int pick_cg_groups(int64_t m, int64_t d, int sa_bytes, int G, bool gram, bool res, int NR) {
  const int64_t rows = gram ? d : m, by_cols = (d + 15) / 16;
  int64_t gc;
  if (res) {
    gc = std::max((rows + NR - 1) / NR, by_cols);
    if (gc > G) gc = G;
    return gc * NR >= rows ? (int)gc : 0;
  }
  const double mb = (double)rows * (double)d * sa_bytes / (1024.0 * 1024.0);
  gc = mb >= 8.0 ? 256 : (mb >= 4.0 ? 64 : (mb >= 1.0 ? 32 : 16));
  gc = std::max(std::min(gc, (m + 3) / 4), by_cols);
  return (int)std::max<int64_t>(1, std::min<int64_t>(gc, G));
}

struct SolveShape {
  bool res = false;   // the inner operator's rows stay in registers
  int G = 0, Gc = 0;  // workgroups, of which the first Gc run the inner solve (G = 0: none fits)
  int cpw = 0;        // columns owned per inner-solve workgroup
  size_t lds = 0;     // dynamic LDS bytes
};

// occupancy(res, lds): workgroups of that form per CU, or < 0 on an error (then G stays 0).
// Resident rows where they fit; two workgroups per CU, then one.
template <typename Occ>
SolveShape pick_solve_shape(int64_t n, int64_t d, int64_t m, int bytes, int ept, bool gram,
                            int num_cu, Occ&& occupancy) {
  SolveShape S;
  const int64_t dpad = 64 * (int64_t)ept;
  // keep >= 16 rows of A per workgroup (64 left three quarters of the CUs idle in the
  // Primal-Dual dual steps, which pass over 4096 rows: 82 against 71 ms at 16384 x 4096),
  // and >= 64 before a CU takes a second one (more partial vectors to add)
  const int64_t g16 = (n + 15) / 16, g64 = (n + 63) / 64;
  const int64_t g_rows = std::max<int64_t>(1, std::min(g16, std::max<int64_t>(g64, num_cu)));
  const int NR = resident_rows(bytes, ept, gram);
  for (int res = 1; res >= 0; --res) {
    if (!solve_instance(bytes, ept, gram, res != 0)) continue;
    // a Gram matrix is as large as d says, however few rows A has (Primal-Dual solves may have
    // fewer rows than columns): the resident form takes the workgroups that hold it, some
    // without rows of A
    const int64_t need = gram && res ? (d + NR - 1) / NR : 1;
    for (int occ_try = kMaxBlocksPerCU; occ_try >= 1; --occ_try) {
      const int64_t most = (int64_t)num_cu * occ_try;
      const int g = (int)std::min(most, std::max(g_rows, need));
      const int gc = pick_cg_groups(m, d, bytes, g, gram, res != 0, NR);
      if (gc == 0) continue;
      const int cp = (int)((d + gc - 1) / gc);
      const size_t lds = (2 * (size_t)dpad + 6 * (size_t)cp + 256) * sizeof(double);
      if (lds > kSolveLds) continue;
      const int occ = occupancy(res != 0, lds);
      if (occ < 0) return S;
      if (occ >= occ_try || (occ >= 1 && (int64_t)g <= (int64_t)num_cu * occ)) {
        S.res = res != 0;
        S.G = g;
        S.Gc = gc;
        S.cpw = cp;
        S.lds = lds;
        return S;
      }
    }
  }
  return S;
}

// ---- workspace ------------------------------------------------------------------

// The CG goes through the Gram matrix when it is no larger than SA (m >= d).
inline bool use_gram(int64_t m, int64_t d) { return m >= d; }

inline size_t gram_bytes(int64_t d, int bytes) {
  int64_t dp = 64;
  while (dp < d) dp *= 2;
  return (size_t)dp * dp * bytes;
}

// Which exchanges go by tagged words instead of barriers: those of the CG on a resident Gram
// matrix up to 2048 columns (FP64 rows of 2048 entries fill the registers: by barrier; every
// workgroup polls the whole vector at twice its size: 256 workgroups, a round of 2048 values 3.4
// us tagged, 3.9 by barrier; of 4096 5.1 against 4.3), and those of the streaming solvers on
// resident rows up to 1024 columns, at most 16 owned columns and 64 workgroups (what one round of
// the owners' thread grid reads).
enum class SolveTags { kNone, kGram, kStreaming };
constexpr bool tagged_gram(int bytes, int ept) { return ept * bytes < 256; }
constexpr bool tagged_streaming(int ept) { return ept <= 16; }
inline SolveTags solve_tags(bool gram, bool res, int bytes, int ept, int Gc, int cpw) {
  if (!res) return SolveTags::kNone;
  if (gram) return tagged_gram(bytes, ept) ? SolveTags::kGram : SolveTags::kNone;
  return tagged_streaming(ept) && cpw <= 16 && Gc <= 64 ? SolveTags::kStreaming : SolveTags::kNone;
}

struct SolveLayout {
  size_t partA, partS, scal, vecs, xp, bar, tags, tagw, region, yrow, total;
  size_t zero_end;  // every launch clears [bar, zero_end)
};

// Barrier region: line 0 = top counter of the all-workgroup barrier, lines 1-8
// its group counters, line 9 = inner-solve group counter, line 10 = error flag,
// line 11 = status word, lines 12-20 = top and group counters of the two-level
// inner-solve barrier (128-byte lines).
constexpr size_t kBarLines = 21;

// gram: bytes of the Gram matrix (0 when SA is streamed).  Its place is taken by the tagged
// partial vectors of the streaming solvers.
inline SolveLayout solve_layout(int G, int Gc, int64_t dpad, SolveTags tags, size_t gram,
                                int64_t m) {
  SolveLayout L;
  size_t off = 0;
  L.partA = off; off = align_up(off + (size_t)G * dpad * 8, 256);
  L.partS = off; off = align_up(off + (size_t)Gc * dpad * 8, 256);
  L.scal = off;  off = align_up(off + (size_t)G * 8 * 8, 256);
  L.vecs = off;  off = align_up(off + 4 * (size_t)dpad * 8, 256);
  L.xp = off;    off = align_up(off + (size_t)dpad * 8, 256);
  L.bar = off;   off = align_up(off + kBarLines * 128, 256);
  L.tags = off;
  if (tags != SolveTags::kNone) off += kScalarSlots * (size_t)Gc * 2 * 16;
  L.tagw = off;
  if (tags != SolveTags::kNone) off += kVectorSlots * (size_t)dpad * 16;
  off = align_up(off, 256);
  const size_t part = tags == SolveTags::kStreaming ? (size_t)Gc * dpad * 16 : 0;
  L.region = off;
  L.zero_end = off + part;
  off = align_up(off + std::max(gram, part), 256);
  L.yrow = off;  off = align_up(off + (size_t)m * 8, 256);
  L.total = off;
  return L;
}

// Workspace of any launch at these sizes on at most G workgroups, by whichever inner solver and
// from whatever A: without tags the inner group may be the whole grid, with them it is small.
inline size_t solve_layout_bound(int G, int64_t d, int64_t m, int bytes, bool no_gram) {
  int ept = 1;
  while (64 * (int64_t)ept < d) ept *= 2;
  const int64_t dpad = 64 * (int64_t)ept;
  const size_t gram = !no_gram && use_gram(m, d) ? gram_bytes(d, bytes) : 0;
  size_t most = solve_layout(G, G, dpad, SolveTags::kNone, gram, m).total;
  if (gram && tagged_gram(bytes, ept))
    most = std::max(most, solve_layout(G, std::min(G, 128), dpad, SolveTags::kGram, gram, m).total);
  if (tagged_streaming(ept))
    most = std::max(most,
                    solve_layout(G, std::min(G, 64), dpad, SolveTags::kStreaming, gram, m).total);
  return most;
}

}  // namespace mihs
