// Host harness for csrc/reuse.h.
//   reuse_check capture KEYS   what a call with each key (letter) does:
//                              d(irect), c(apture) or r(eplay)
//   reuse_check loop CALLS     a call per letter: s if its loop stalls; prints
//                              l(oop) or i(teration by iteration)
//   reuse_check limit [TEXT]   the poll limit from the text
#include <cstdio>
#include <cstring>

#include "../../paper_1902_01061_amd/csrc/reuse.h"

int main(int argc, char** argv) {
  const char* text = argc > 2 ? argv[2] : nullptr;
  if (!std::strcmp(argv[1], "limit")) {
    std::printf("%d", sgr::LoopRule::limit(text));
  } else if (!std::strcmp(argv[1], "loop")) {
    sgr::LoopRule rule;
    for (; *text; ++text) {
      const bool loop = rule.use();
      if (loop && *text == 's') rule.stalled();
      std::putchar(loop ? 'l' : 'i');
    }
  } else {
    sgr::CaptureRule rule;
    for (; *text; ++text) {
      const std::vector<uint8_t> key(3, (uint8_t)*text);
      const auto act = rule.next(key);
      if (act == sgr::CaptureRule::CAPTURE) {
        rule.dropped();
        rule.captured(key);
      }
      std::putchar("dcr"[act]);
    }
  }
}
