// Host model of the exchange between the workgroups of the tridiagonal
// reduction (eigh.hip), under the rules of exchange.h, built without a device
// by tests/test_exchange_host.py.  Every workgroup is a sequence of single
// stores and waits on tagged words; a scheduler picks who moves next, with one
// workgroup at a time held back for long stretches.  A reader that finds a
// newer tag than the one it waits for has been overrun, and waits for ever on
// the device.  Prints "ok" and exits 0, or the first failure and exits 1.
#include <cstdio>
#include <cstdlib>
#include <random>
#include <vector>

#include "exchange.h"

namespace {

struct Op {
  bool store;
  int word, tag;
};

// x: word (buffer, row), row buffers after them.  `ahead`: the pivot row is
// published a column early into one of four buffers (a wave per row), instead
// of with x into one of two.
std::vector<Op> program(int g, int n, int G, bool ahead) {
  std::vector<Op> p;
  const int rows = 2 * n;
  for (int k = 0; k + 1 < n; ++k) {
    const int x = (k & 1) * n;
    for (int r = g; r < n; r += G)
      if (tdx::publishes(r, k, n, G)) p.push_back({true, x + r, k + 1});
    if (ahead) {
      if (k + 2 < n && (k + 2) % G == g) p.push_back({true, rows + ((k + 2) & 3), k + 2});
      if (k > 0) p.push_back({false, rows + ((k + 1) & 3), k + 1});
    } else {
      if ((k + 1) % G == g) p.push_back({true, rows + (k & 1), k + 1});
      p.push_back({false, rows + (k & 1), k + 1});
    }
    for (int c = tdx::first_awaited(k, n, G); c < n; ++c) p.push_back({false, x + c, k + 1});
  }
  return p;
}

bool run(int n, int G, bool ahead, unsigned seed) {
  std::mt19937 rng(seed);
  std::vector<std::vector<Op>> prog;
  for (int g = 0; g < G; ++g) prog.push_back(program(g, n, G, ahead));
  std::vector<size_t> pc(G, 0);
  std::vector<int> tag(2 * n + 4, 0);
  int held = 0, idle = 0;
  auto step = [&](int g, bool* failed) {   // one store or satisfied wait
    if (pc[g] == prog[g].size()) return false;
    const Op& o = prog[g][pc[g]];
    if (o.store) {
      tag[o.word] = o.tag;
    } else if (tag[o.word] > o.tag) {
      std::printf("n %d, G %d, %s: workgroup %d waits for tag %d and finds %d\n", n, G, ahead ? "row ahead" : "row with x",
                  g, o.tag, tag[o.word]);
      *failed = true;
      return false;
    } else if (tag[o.word] < o.tag) {
      return false;
    }
    ++pc[g];
    return true;
  };
  while (true) {
    bool all = true, failed = false;
    for (int g = 0; g < G; ++g) all = all && pc[g] == prog[g].size();
    if (all) return true;
    if (rng() % 64 == 0) held = (int)(rng() % G);
    const int g = (int)(rng() % G);
    const bool moved = g != held && step(g, &failed);
    if (failed) return false;
    // nobody else can move: the one held back takes a single step
    idle = moved ? 0 : idle + 1;
    if (idle > 20 * G) {
      bool any = false;
      for (int h = 0; h < G && !any; ++h)
        if (h != held) any = step(h, &failed);
      if (!any && !failed) any = step(held, &failed);
      if (failed) return false;
      if (!any) {
        std::printf("n %d, G %d: nobody can move\n", n, G);
        return false;
      }
      idle = 0;
    }
  }
}

}  // namespace

int main() {
  for (int n = 2; n <= 24; ++n)
    for (int G = 1; G <= n; G += 1 + G / 4)
      for (unsigned seed = 0; seed < 6; ++seed)
        for (int ahead = 0; ahead < 2; ++ahead)
          // a wave per row: at most four rows a workgroup
          if ((!ahead || (n + G - 1) / G <= 4) && !run(n, G, ahead != 0, seed)) return 1;
  std::printf("ok\n");
  return 0;
}
