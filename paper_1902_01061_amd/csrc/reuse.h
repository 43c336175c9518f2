// What a context remembers of earlier calls to choose how the next one runs
// (host only; the results do not depend on it beyond rounding).
#pragma once
#include <stdint.h>
#include <stdlib.h>

#include <climits>
#include <vector>

namespace sgr {

// Whether a call with the given key runs directly, is captured as a graph, or
// replays the graph that was captured for its key.  A capture costs what four
// runs from its graph save (100 iterations at 1 024 points take 1 593 us with a
// capture, 1 331 launched directly and 1 266 from a graph that exists), so it
// is made when a key comes the fourth time in a row, calls that replay another
// key's graph between them counted as interruptions.
struct CaptureRule {
  enum Act { DIRECT, CAPTURE, REPLAY };
  static constexpr int AT = 4;
  std::vector<uint8_t> key;   // of the captured graph (empty: none)
  std::vector<uint8_t> seen;  // of the last calls that ran directly
  int times = 0;              // how many they were in a row

  Act next(const std::vector<uint8_t>& k) {
    if (!key.empty() && k == key) {
      seen.clear();
      times = 0;
      return REPLAY;
    }
    times = k == seen ? times + 1 : 1;
    seen = k;
    return times < AT ? DIRECT : CAPTURE;
  }
  void captured(const std::vector<uint8_t>& k) {
    key = k;
    seen.clear();
    times = 0;
  }
  void dropped() { key.clear(); }
};

// Whether a registration may run its iterations in one launch, whose blocks
// wait for each other.  When they were not resident together, the call has
// waited its poll limit for nothing and done its work twice; what keeps them
// apart (another context's work on the same card) is likely to last, so the
// next registrations do without.
struct LoopRule {
  static constexpr int SPINS = 200000;  // polls before a loop gives up (0.2 s at an estimated 1 us each)
  static constexpr int REST = 255;
  int spins = SPINS;
  int rest = 0;  // registrations still to do without

  bool use() {
    if (rest == 0) return true;
    --rest;
    return false;
  }
  void stalled() { rest = REST; }

  // The limit from a text: a whole number from 1 up, else (or nullptr) SPINS.
  static int limit(const char* text) {
    if (!text || *text < '0' || *text > '9') return SPINS;
    char* end = nullptr;
    const long v = strtol(text, &end, 10);
    return *end == 0 && v >= 1 && v <= INT_MAX ? (int)v : SPINS;
  }
};

}  // namespace sgr
