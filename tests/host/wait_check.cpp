// The hand-over of a wait's outcome to the wavefronts of a workgroup, modelled on the CPU:
// wavefront 0 writes outcome n to a word, all pass a barrier, every wavefront reads the
// word, and the next wait follows without another barrier. All orders of the wavefronts'
// accesses are walked through.
#include <set>
#include <vector>

#include "direct.h"

namespace {

constexpr int kWavefronts = 3, kWaits = 5;

struct State {
  int at[kWavefronts];      // accesses made: 2 n: before wait n, 2 n + 1: at its read
  int word[4];              // outcome held (the number of its wait)
  bool operator<(const State& o) const {
    for (int w = 0; w < kWavefronts; ++w)
      if (at[w] != o.at[w]) return at[w] < o.at[w];
    for (int k = 0; k < 4; ++k)
      if (word[k] != o.word[k]) return word[k] < o.word[k];
    return false;
  }
};

}  // namespace

// Number of reads, over all orders, that see another wait's outcome; `words` words in turn
// (0: as the solver chooses them).
extern "C" int wait_check(int words) {
  std::vector<int> word_of(kWaits);
  int w = 0;
  for (int n = 0; n < kWaits; ++n) {
    word_of[n] = w;
    w = words ? (w + 1) % words : phisft::ds_next_word(w);
  }
  std::set<State> seen, todo;
  State s0{};
  for (int& k : s0.word) k = -1;
  todo.insert(s0);
  int wrong = 0;
  while (!todo.empty()) {
    const State s = *todo.begin();
    todo.erase(todo.begin());
    if (!seen.insert(s).second) continue;
    for (int v = 0; v < kWavefronts; ++v) {
      if (s.at[v] == 2 * kWaits) continue;
      const int n = s.at[v] / 2;
      State t = s;
      ++t.at[v];
      if (s.at[v] % 2 == 0) {
        // into the barrier of wait n, wavefront 0 with its outcome; its write may land
        // before any wavefront's outstanding read
        if (v == 0) t.word[word_of[n]] = n;
      } else {
        // through the barrier once all have entered it
        bool all = true;
        for (int k = 0; k < kWavefronts; ++k) all = all && s.at[k] >= 2 * n + 1;
        if (!all) continue;
        if (s.word[word_of[n]] != n) ++wrong;
      }
      todo.insert(t);
    }
  }
  return wrong;
}
