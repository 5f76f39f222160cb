// Every order in which the workgroups of a row can write their states, count themselves and merge, by the rules the kernel uses
// (csrc/short_count.h): one call behind another on a word that was left at anything, and two calls at once.  CPU only; the test
// beside it compiles and runs this.
//   - a call on its own merges its row once, behind the last of its states, whatever the word was, and leaves it at zero;
//   - of two calls at once each row is its own call's, or has been made NaN with a status that is not zero and stays so;
//   - the call behind them is right.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <unordered_set>
#include <string>
#include <vector>

#include "../paper_2503_23294_amd/csrc/short_count.h"

using namespace cocktail;

constexpr int kMost = 4, kTokens = 7;
// slots of one queue's ring side by side, the same slot of another queue, one far away
constexpr uint64_t kSteps[4] = {short_step(0x500000001040), short_step(0x500000001080), short_step(0x500000801040), short_step(0x4ffffff00000)};

enum Step : uint8_t { kState, kRow, kAdd, kHeal, kAddAgain, kZero, kRead, kDone };
struct World {   // compared byte by byte
  uint64_t word, seen[2][kMost];            // seen: of the word, by the compare-and-swap under way
  Step step[2][kMost];
  uint8_t written[2][kMost];                // the state is this call's
  uint8_t row[2], merges[2];                // 0 as it was, 1 NaN and reported, 2 the call's result, 3 a wrong one
  uint8_t zero[4];
};
static_assert(sizeof(World) == 96, "no padding");
struct Model {
  int calls = 1, groups = 2;
  uint64_t steps[2] = {kSteps[0], kSteps[1]};

  void add(World& w, int c, int i, bool again) const {
    const uint64_t step = steps[c], all = uint64_t(groups) * step, old = w.word;
    w.word += step;
    if (old + step == all) w.step[c][i] = kZero;
    else if (!again && !short_own(old, step)) w.step[c][i] = kHeal, w.seen[c][i] = old + step;
    else w.step[c][i] = kDone;
  }
  void next(World& w, int c, int i) const {
    switch (w.step[c][i]) {
      case kState: w.written[c][i] = 1, w.step[c][i] = i == 0 ? kRow : kAdd; break;
      case kRow: w.row[c] = short_pending(0) && short_pending(kTokens) ? 1 : 3, w.step[c][i] = kAdd; break;
      case kAdd: add(w, c, i, false); break;
      case kAddAgain: add(w, c, i, true); break;
      case kHeal:
        if (!short_own(w.seen[c][i], steps[c]) && w.word != w.seen[c][i]) w.seen[c][i] = w.word;
        else {
          if (!short_own(w.seen[c][i], steps[c])) w.word = 0;
          w.step[c][i] = kAddAgain;
        }
        break;
      case kDone: break;
      case kZero:
        if (w.word == uint64_t(groups) * steps[c]) w.word = 0;
        w.step[c][i] = kRead;
        break;
      case kRead: {   // (what it reads changes no more)
        bool whole = true;
        for (int k = 0; k < groups; ++k) whole = whole && w.written[c][k];
        w.row[c] = whole && w.row[c] == 1 ? 2 : 3, ++w.merges[c], w.step[c][i] = kDone;
        break;
      }
    }
    if (w.step[c][i] == kDone || w.step[c][i] == kAddAgain) w.seen[c][i] = 0;
  }
  // every world in which all workgroups are done
  std::vector<World> ends(const World& start, long& seen) const {
    std::unordered_set<std::string> known;
    std::vector<World> open{start}, done;
    while (!open.empty()) {
      const World w = open.back();
      open.pop_back();
      bool over = true;
      for (int c = 0; c < calls; ++c)
        for (int i = 0; i < groups; ++i) {
          if (w.step[c][i] == kDone) continue;
          over = false;
          World then = w;
          next(then, c, i);
          if (std::memcmp(&then, &w, sizeof(w)) && known.emplace(reinterpret_cast<const char*>(&then), sizeof(then)).second) open.push_back(then);
        }
      if (over) done.push_back(w);
    }
    seen += long(known.size());
    return done;
  }
};

static World begin(uint64_t word) {
  World w;
  std::memset(&w, 0, sizeof(w));
  w.word = word;
  return w;
}
static void require(bool ok, const char* what, int groups, uint64_t word) {
  if (ok) return;
  std::fprintf(stderr, "%s: %d workgroups, the word at 0x%llx\n", what, groups, (unsigned long long)word);
  std::exit(1);
}

int main() {
  long seen = 0, alone = 0, pairs = 0;
  for (int groups = 2; groups <= 4; ++groups) {
    // what calls, aborted ones among them, and damage can leave
    std::vector<uint64_t> words = {0, ~uint64_t(0), 255, 256, uint64_t(1) << 63, kSteps[1] + kSteps[2], 2 * kSteps[1] - kSteps[2], uint64_t(0) - kSteps[1]};
    for (uint64_t n = 1; n <= 2u * groups + 1; ++n)
      for (uint64_t step : {uint64_t(1), kSteps[1], kSteps[2], kSteps[3]}) words.push_back(n * step);
    Model m;
    m.groups = groups;
    for (uint64_t word : words)
      for (const World& e : m.ends(begin(word), seen)) {
        require(e.row[0] == 2 && e.merges[0] == 1, "a call on its own is not right", groups, word);
        require(e.word == 0, "a call on its own leaves the word at something", groups, word);
        ++alone;
      }
    if (groups > 3) continue;
    for (uint64_t word : groups == 2 ? std::vector<uint64_t>{0, 1, kSteps[3]} : std::vector<uint64_t>{0})
      for (const World& both : (m.calls = 2, m).ends(begin(word), seen)) {
        for (int c = 0; c < 2; ++c)
          require(both.merges[c] == (both.row[c] == 2) && (both.row[c] == 1 || both.row[c] == 2), "of two calls at once one is neither right nor reported", groups, word);
        Model behind = m;
        behind.calls = 1, behind.steps[0] = kSteps[2];
        for (const World& e : behind.ends(begin(both.word), seen)) require(e.row[0] == 2 && e.word == 0, "the call behind two at once is not right", groups, both.word);
        ++pairs;
      }
    m.calls = 1;
  }
  std::printf("passed: %ld worlds, %ld ends of a call on its own, %ld of two at once\n", seen, alone, pairs);
  return 0;
}
