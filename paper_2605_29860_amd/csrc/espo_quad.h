// Which four positions of an array a lane loads at once where a row starts or ends (plain C++, for the host's tests too).
#ifndef ESPO_QUAD_H_
#define ESPO_QUAD_H_

#include <stdint.h>

namespace espo {

struct Quad {
  int at;       // the first of the four
  uint32_t in;  // bit j: position at + j is one of this lane's
};

// A lane owns what lies in [lo, hi) of positions t .. t + 3.  Of a span of at least four it loads four that all lie in there, those of its
// own among them: moved in from an end if need be, and then not at a multiple of four.  (A shorter span starts at `at`, and is read by single
// loads of what `in` names.)
constexpr Quad quad_of(int t, int lo, int hi) {
  int at = t < hi - 4 ? t : hi - 4;
  at = at < lo ? lo : at;
  const int from = (t < lo ? lo : t) - at, to = (t + 4 > hi ? hi : t + 4) - at;  // 0 <= from, to <= 4 where there are any
  return Quad{at, from < to ? (0xfu >> (4 - to)) & (0xfu << from) : 0u};
}

}  // namespace espo
#endif  // ESPO_QUAD_H_
