// Host harness for the capture rule: reads a line of keys (letters), prints what
// each call does, d(irect), c(apture) or r(eplay).
#include <cstdio>

#include "../../paper_1902_01061_amd/csrc/reuse.h"

int main() {
  sgr::CaptureRule rule;
  for (int c = std::getchar(); c > ' '; c = std::getchar()) {
    const std::vector<uint8_t> key(3, (uint8_t)c);
    const auto act = rule.next(key);
    if (act == sgr::CaptureRule::CAPTURE) {
      rule.dropped();
      rule.captured(key);
    }
    std::putchar("dcr"[act]);
  }
}
