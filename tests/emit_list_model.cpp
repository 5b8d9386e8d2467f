// Host model of the list of slots with a label inside one workgroup of wind_group_vocab_kernel.h: four waves as state machines, of which the first writes
// the next iteration's list, and a scheduler that holds one wave back for as long as any other can move, or picks at random.
//   arguments: wave held back (-1: random order, seeded), seed, 1: lists by the kernel's rule / 0: one list
//   prints: done | wrong (a wave took another iteration's list for its own)
#include <cstdio>
#include <cstdlib>
#include <random>
#include "wind_group_protocol.h"

static const int kWaves = 4, kIters = 200, kSteps = 5;
static int by_rule, list[2] = {0, 0};   // the iteration whose list it is
struct Wave { int it = 0, step = 0; } w[kWaves];
static bool wrong = false;

static int &at(int it) { return list[by_rule ? wind::vocab_emit_list(it) : 0]; }
static bool barrier(int me) {   // everybody has come this far
  for (const Wave &x : w) if (x.it * kSteps + x.step < w[me].it * kSteps + w[me].step) return false;
  return true;
}
static bool move(int me) {
  Wave &x = w[me];
  switch (x.step) {
    case 0: if (!barrier(me)) return false; break;                    // behind the last chunk of rows
    case 1: if (at(x.it) != x.it) wrong = true; break;                // the recurrent sums of the lower tile of slots
    case 2: if (me == 0) at(x.it + 1) = x.it + 1; break;              // the decisions are there: the slots move on
    case 3: if (!barrier(me)) return false; break;
    case 4: if (at(x.it + 1) != x.it + 1) wrong = true; break;        // the new hidden vectors, for the projection
  }
  if (++x.step == kSteps) { x.step = 0; ++x.it; }
  return true;
}
int main(int, char **a) {
  const int held = atoi(a[1]);
  std::mt19937 rng((unsigned)atoi(a[2]));
  by_rule = atoi(a[3]);
  for (bool all = false; !all && !wrong;) {
    bool moved = false;
    if (held >= 0) {
      for (int i = 0; i < kWaves; ++i)
        while (i != held && w[i].it < kIters && move(i)) moved = true;
      if (!moved && w[held].it < kIters) move(held);
    } else {
      const int i = (int)(rng() % kWaves);
      if (w[i].it < kIters) move(i);
    }
    all = true;
    for (const Wave &x : w) all = all && x.it >= kIters;
  }
  puts(wrong ? "wrong" : "done");
}
