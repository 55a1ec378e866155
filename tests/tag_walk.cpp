// Exhaustive walk of the inner solvers' tagged exchanges (solve_kernel.hpp): two workgroups of
// two waves each (the first wave, which puts vector entries and scalars, and one of the others)
// run three steps of every form in every interleaving.  A wave waits until all workgroups'
// words carry its tag at once; a state in which no wave can move and not all have ended is a
// wait that never ends.  Each word is written by one wave, so the words follow from the waves'
// positions.  Usage: tag_walk [scalar slots vector slots] (default: the kernel's).
#include <stdio.h>
#include <stdlib.h>

#include <array>
#include <set>
#include <vector>

#include "../paper_1912_03514_amd/csrc/internal.hpp"

enum Kind { SCAL, VEC, PART, BAR };
struct Op {
  Kind kind;
  bool put;
  unsigned tag;
};
typedef std::vector<Op> Program;
typedef std::array<Program, 2> Waves;  // the first wave, another wave

static unsigned scal_slots, vec_slots;
static unsigned slot(Kind k, unsigned tag) {
  return k == SCAL ? tag % scal_slots : k == VEC ? tag % vec_slots : 0u;
}

// ---- the forms, by what each wave does (barriers are the workgroup's own) ----
static void both(Waves& w, Op o) {
  w[0].push_back(o);
  w[1].push_back(o);
}
static void bar(Waves& w) { both(w, {BAR, false, 0}); }
static void exchange(Waves& w, unsigned tag) {  // vector and scalars, everybody to everybody
  w[0].push_back({VEC, true, tag});
  w[0].push_back({SCAL, true, tag});
  both(w, {VEC, false, tag});
  both(w, {SCAL, false, tag});
}
static Waves single_reduction(int steps) {
  Waves w;
  unsigned tag = 0;
  for (int s = 0; s < steps; ++s) {
    bar(w);  // stage
    bar(w);  // product
    exchange(w, ++tag);
  }
  return w;
}
static Waves two_reductions(int steps) {
  Waves w;
  unsigned tag = 0;
  for (int s = 0; s < steps; ++s) {
    bar(w);
    bar(w);
    ++tag;
    w[0].push_back({SCAL, true, tag});
    w[0].push_back({SCAL, false, tag});
    exchange(w, ++tag);
  }
  return w;
}
static Waves streaming(int steps) {
  Waves w;
  unsigned tag = 0;
  for (int s = 0; s < steps; ++s) {
    bar(w);  // stage
    bar(w);  // partial products
    bar(w);  // u
    ++tag;
    both(w, {PART, true, tag});
    w[0].push_back({SCAL, true, tag});
    both(w, {PART, false, tag});
    bar(w);  // column sums
    both(w, {SCAL, false, tag});
    exchange(w, ++tag);
  }
  return w;
}

typedef std::array<unsigned char, 4> State;  // position of wave v of workgroup g at 2 g + v

// the last tag that wave v put into the slot before position pos (0: none)
static unsigned word(const Program& p, int pos, Kind k, unsigned sl) {
  unsigned t = 0;
  for (int i = 0; i < pos; ++i)
    if (p[i].put && p[i].kind == k && slot(k, p[i].tag) == sl) t = p[i].tag;
  return t;
}
static int bars(const Program& p, int pos) {
  int n = 0;
  for (int i = 0; i < pos; ++i) n += p[i].kind == BAR;
  return n;
}
static bool can_move(const Waves& w, const State& s, int i) {
  const Program& p = w[i % 2];
  if (s[i] >= p.size()) return false;
  const Op o = p[s[i]];
  if (o.kind == BAR) {  // the other wave is at this barrier or past it
    const int o2 = i ^ 1;
    const Program& q = w[o2 % 2];
    const int mine = bars(p, s[i]), other = bars(q, s[o2]);
    return other > mine || (other == mine && s[o2] < q.size() && q[s[o2]].kind == BAR);
  }
  if (o.put) return true;
  for (int g = 0; g < 2; ++g)
    for (int v = 0; v < (o.kind == PART ? 2 : 1); ++v)
      if (word(w[v], s[2 * g + v], o.kind, slot(o.kind, o.tag)) != o.tag) return false;
  return true;
}
static size_t stuck_states(const Waves& w, size_t& seen_count) {
  std::set<State> seen;
  std::vector<State> todo;
  State s0 = {0, 0, 0, 0};
  seen.insert(s0);
  todo.push_back(s0);
  size_t stuck = 0;
  while (!todo.empty()) {
    const State s = todo.back();
    todo.pop_back();
    bool any = false, done = true;
    for (int i = 0; i < 4; ++i) {
      done = done && s[i] == w[i % 2].size();
      if (!can_move(w, s, i)) continue;
      any = true;
      State t = s;
      ++t[i];
      if (seen.insert(t).second) todo.push_back(t);
    }
    if (!any && !done) ++stuck;
  }
  seen_count = seen.size();
  return stuck;
}

// a poll takes about a microsecond: a tagged wait that will not end is given up within ten
// seconds, any other within two minutes
static_assert(mihs::kTagPolls <= 10000000 && mihs::kIdlePolls <= mihs::kBarrierPolls &&
                  mihs::kBarrierPolls <= 120000000,
              "bounds of the waits");

int main(int argc, char** argv) {
  scal_slots = argc > 1 ? (unsigned)atoi(argv[1]) : mihs::kScalarSlots;
  vec_slots = argc > 2 ? (unsigned)atoi(argv[2]) : mihs::kVectorSlots;
  if (argc < 2)
    for (unsigned t = 0; t < 64; ++t)
      if (mihs::scalar_slot(t) != t % scal_slots || mihs::vector_slot(t) != t % vec_slots) {
        printf("slot rule\n");
        return 2;
      }
  const struct {
    const char* name;
    Waves w;
  } forms[] = {{"single reduction", single_reduction(3)},
               {"two reductions", two_reductions(3)},
               {"streaming", streaming(3)}};
  size_t total = 0;
  for (const auto& f : forms) {
    size_t seen = 0;
    const size_t stuck = stuck_states(f.w, seen);
    printf("%s: %zu states, %zu stuck\n", f.name, seen, stuck);
    total += stuck;
  }
  return total ? 1 : 0;
}
