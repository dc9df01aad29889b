// The value bounds that ModDown's forward pass is compiled for, against the
// values it is given: the bounds of every stage (Bounds) follow from the one on
// entry, and on doubles they are what keeps the transform exact.
#include <cstdint>
#include <cstdio>

#include "ntt_core.h"

using namespace hck;

// The largest value on entry, in units of q / 1024 and rounded up.  On doubles:
// a converted value (a word below q where the conversion ran on whole words,
// else within 1/2 and a reduction's rounding) plus a reduced rounding term.
constexpr int entry(bool is_float, bool s30) {
  return is_float ? (s30 ? ArF::kReduced : 1024) + ArF::kReduced : 2 * 1024;
}

template <class Ar, bool S30, int LOGR>
constexpr bool holds() {
  constexpr int x0 = moddown_bound<Ar, S30>();
  constexpr Bounds<Ar, LOGR, false> planned(x0);
  return x0 >= entry(Ar::kFloat, S30) && Ar::fits(planned.x[LOGR]);
}

// strided passes of the rings 2^11 .. 2^17: 2^6 .. 2^9 points
template <class Ar, bool S30>
constexpr bool all() {
  return holds<Ar, S30, 6>() && holds<Ar, S30, 7>() && holds<Ar, S30, 8>() && holds<Ar, S30, 9>();
}

int main() {
  bool ok = true;
  auto check = [&](bool good, const char *what) {
    if (!good) std::printf("bound too small: %s\n", what);
    ok = ok && good;
  };
  check(all<ArF, true>(), "doubles, converted in doubles");
  check(all<ArF, false>(), "doubles, converted on whole words");
  check(all<ArI<16>, true>(), "integers below 2^60, halves");
  check(all<ArI<16>, false>(), "integers below 2^60, whole words");
  check(all<ArI<8>, false>(), "integers from 2^60 on");
  if (ok) std::printf("all checks passed\n");
  return ok ? 0 : 1;
}
