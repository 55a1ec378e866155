// Launch shapes of the persistent solve (solve_shape.hpp) over sizes, forms and device sizes: every
// call that the entry points accept has one, and what it promises the kernel holds.
#include <stdio.h>

#include "../paper_1912_03514_amd/csrc/solve_shape.hpp"

using namespace mihs;

int main() {
  int failures = 0, found = 0;
  const int64_t ds[] = {1, 16, 17, 64, 65, 97, 200, 256, 500, 512, 513, 800, 1024, 1025, 2000,
                        2048, 2049, 3000, 4096};
  const int64_t ns[] = {1, 40, 96, 100, 129, 300, 1000, 4096, 100000, (int64_t)1 << 24};
  for (int cus : {32, 64, 128, 256})
    for (int occ : {1, 2, 3})
      for (int bytes : {4, 8})
        for (int64_t d : ds)
          for (int64_t n : ns)
            for (int64_t m : {d / 3 + 1, d, 2 * d, 9000 + d})
              for (int streamed : {0, 1}) {
                const bool gram = !streamed && m >= d;
                int ept = 1;
                while (64 * (int64_t)ept < d) ept *= 2;
                const int NR = resident_rows(bytes, ept, gram);
                bool asked_missing = false;
                const SolveShape S = pick_solve_shape(
                    n, d, m, bytes, ept, gram, cus, [&](bool res, size_t) {
                      asked_missing = asked_missing || !solve_instance(bytes, ept, gram, res);
                      return occ;
                    });
                // 4096 columns owned by one or two workgroups (A of at most 32 rows) do not
                // fit the LDS
                const bool must = n > 32 || d <= 2048;
                bool ok = !asked_missing && (S.G > 0 || !must);
                if (S.G > 0) {
                  ++found;
                  ok = ok && S.Gc >= 1 && S.Gc <= S.G && (int64_t)S.Gc * S.cpw >= d &&
                       S.lds <= kSolveLds && S.G <= cus * occ &&
                       solve_instance(bytes, ept, gram, S.res);
                  if (S.res) ok = ok && (int64_t)S.Gc * NR >= (gram ? d : m);
                  // the owned rows of a resident Gram matrix are those that are kept
                  if (S.res && gram) ok = ok && S.cpw <= NR && S.cpw <= 16;
                }
                // the workspace query covers the launch, and on a whole GPU the tagged exchanges
                // fit what the barrier forms take on the largest grid
                const int64_t dpad = 64 * (int64_t)ept;
                const size_t full = gram ? gram_bytes(d, bytes) : 0;
                const size_t bound = solve_layout_bound(cus * kMaxBlocksPerCU, d, m, bytes, streamed);
                if (S.G > 0)
                  ok = ok && solve_layout(S.G, S.Gc, dpad,
                                          solve_tags(gram, S.res, bytes, ept, S.Gc, S.cpw), full,
                                          m).total <= bound;
                if (cus == 256)
                  ok = ok && bound == solve_layout(2 * cus, 2 * cus, dpad, SolveTags::kNone,
                                                   !streamed && m >= d ? full : 0, m).total;
                // a whole GPU keeps every Gram matrix that fits the registers
                if (gram && cus == 256 && solve_instance(bytes, ept, true, true)) ok = ok && S.res;
                if (!ok && ++failures < 20)
                  fprintf(stderr, "cus %d occ %d bytes %d n %lld d %lld m %lld gram %d: G %d Gc %d "
                          "cpw %d res %d\n", cus, occ, bytes, (long long)n, (long long)d,
                          (long long)m, gram, S.G, S.Gc, S.cpw, S.res);
              }
  // the static scratch of 64 MiB holds what it did: d = 2048, FP64, a Gram matrix, and as many
  // rows of SA (8 bytes of scratch each) as fill it
  {
    const size_t scratch = (size_t)64 << 20;
    const size_t base = 2 * (size_t)512 * 2048 * 8 + 512 * 64 + 5 * 2048 * 8 + 21 * 128 + 128 +
                        (size_t)2048 * 2048 * 8;
    const int64_t m = (int64_t)((scratch - base) / 8);
    if (solve_layout_bound(512, 2048, m, 8, false) > scratch) ++failures;
    if (solve_layout_bound(512, 2048, m + 64, 8, false) <= scratch) ++failures;
  }
  // the Primal-Dual dual steps of 100 columns and 200 sketch rows, on a GPU and on a partition
  for (int cus : {32, 256}) {
    const SolveShape S = pick_solve_shape(100, 200, 200, 8, 4, true, cus,
                                          [](bool, size_t) { return 2; });
    if (!S.res || S.G != 13) ++failures;
  }
  printf("%d shapes, %d failures\n", found, failures);
  return failures ? 1 : 0;
}
