// Host model of the exchanges inside one resident group (csrc/wind_group_kernel.h, wind_group_f32_kernel.h): workgroups as state machines, words as
// memory, and a scheduler that holds one workgroup back for as long as any other can move (or picks at random).  Every
// word also carries the iteration it was really written in, which only the model looks at.
//   arguments: workgroups, column parts, row groups, first iteration without rows in the last row group, iterations from one label to the next,
//              workgroup held back (-1: random order, seeded), seed, 1: writers go by the rules / 0: they don't,
//              1: a word is recognised by its tag bit / 0: by its whole iteration
//   prints: done | stuck | wrong (a workgroup took keys of another iteration for its own)
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>
#include "wind_group_protocol.h"

struct Word { int stamp = -1; };   // the iteration it was written in
static int gw, nparts, rg, empty_from, label_every, by_need, by_tag;
static const int kIters = 200;
static std::vector<Word> keys[2], hx, px;   // keys: [row group][part]
static std::vector<int> progress;
struct Group { int it = 0, step = 0; };
static bool wrong = false;

static bool active(int tile, int it) { return tile < rg - 1 || rg == 1 || it < empty_from; }   // whether the row group has rows
static bool own(const Word &w, int it) {   // as the reader sees it
  if (by_tag) return (w.stamp < 0 ? 1 : wind::group_key_tag(w.stamp)) == wind::group_key_tag(it);   // at launch: tag bits set
  return w.stamp == it;
}
// One step of workgroup g; false: it waits.
static bool move(int g, Group &s) {
  const int cg = gw / rg, tile = g / cg, col = g % cg, it = s.it;
  std::vector<Word> &k = keys[wind::group_key_buffer(it)];
  switch (s.step) {
    case 0:   // may the keys of two iterations ago be overwritten?
      if (by_need && !wind::group_keys_suffice(nparts, cg, rg))
        for (int p : progress) if (p < wind::group_keys_need(it)) return false;
      break;
    case 1:   // every row tile of a workgroup writes its parts
      for (int p = col; p < nparts; p += cg) k[tile * nparts + p].stamp = it;
      break;
    case 2: case 3:   // 2: all keys of the rows there are; 3: near-ties look at them again, without asking for the tag
      for (int t = 0; t < rg; ++t)
        for (int p = 0; p < nparts && active(t, it); ++p) {
          const Word &w = k[t * nparts + p];
          if (s.step == 2 && !own(w, it)) return false;
          if (w.stamp != it) wrong = true;
        }
      if (s.step == 3) progress[g] = it + 1;
      break;
    case 4: if (it % label_every == 0) hx[g].stamp = it; break;
    case 5: if (it % label_every == 0) for (Word &w : hx) if (w.stamp != it) return false; break;
    case 6: if (it % label_every == 0) px[g].stamp = it; break;
    case 7: if (it % label_every == 0) for (Word &w : px) if (w.stamp != it) return false; break;
  }
  if (++s.step == 8) { s.step = 0; ++s.it; }
  return true;
}
int main(int, char **a) {
  gw = atoi(a[1]); nparts = atoi(a[2]); rg = atoi(a[3]); empty_from = atoi(a[4]); label_every = atoi(a[5]);
  const int held = atoi(a[6]);
  std::mt19937 rng((unsigned)atoi(a[7]));
  by_need = atoi(a[8]); by_tag = atoi(a[9]);
  for (auto &k : keys) k.resize(rg * nparts);
  hx.resize(gw); px.resize(gw); progress.assign(gw, 0);
  std::vector<Group> s(gw);
  for (;;) {
    bool moved = false, all = true;
    for (const Group &x : s) all = all && x.it >= kIters;
    if (all || wrong) break;
    if (held >= 0) {
      for (int g = 0; g < gw; ++g)
        while (g != held && s[g].it < kIters && move(g, s[g])) moved = true;
      if (!moved && s[held].it < kIters) moved = move(held, s[held]);
    } else {   // a workgroup at a time, some of them far ahead in what the scheduler gives them
      for (int tries = 0; tries < 64 * gw && !moved; ++tries) {
        const int g = (int)(std::min(rng() % gw, rng() % gw));
        if (s[g].it < kIters) moved = move(g, s[g]);
      }
      for (int g = 0; g < gw && !moved; ++g) if (s[g].it < kIters) moved = move(g, s[g]);
    }
    if (!moved) { puts("stuck"); return 0; }
  }
  puts(wrong ? "wrong" : "done");
}
