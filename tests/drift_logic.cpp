// Host check of the fp32 drift bounds (drift_add, slack_less) against 64 bits over many steps, with the steps at which
// a plain sum loses most.  Built and run by tests/test_drift.py; prints the number of failed checks.
#include "sf_internal.h"

#include <cmath>
#include <cstdio>

int main() {
  int fails = 0;
  // steps in units in the last place of 1: less than half, just under one and a half, and many
  for (double ulps : {0.01, 0.49, 1.0, 1.49, 7.49, 1000.49}) {
    const float step = (float)(ulps * std::ldexp(1.0, -24));
    float sum = 0.5f, slack = 1.0f, plain = 0.5f;
    double exact = 0.5, left = 1.0;
    for (int i = 0; i < 2000000 && exact < 1.0 && left > 0.5; ++i) {
      sum = sf::drift_add(sum, step);
      slack = sf::slack_less(slack, step);
      plain += step;
      exact += step;
      left -= step;
    }
    // (a step and a sum each round once: 2^-23 of them at most)
    if (!(sum >= exact * (1.0 - std::ldexp(1.0, -23)))) {
      std::printf("FAIL sum, %g units: %.9g below %.9g (plain %.9g)\n", ulps, sum, exact, plain);
      ++fails;
    }
    if (!(slack <= left * (1.0 + std::ldexp(1.0, -23)))) {
      std::printf("FAIL slack, %g units: %.9g above %.9g\n", ulps, slack, left);
      ++fails;
    }
  }
  // what is not a number stays one, and is not below any margin
  const float nan = std::nanf("");
  if (sf::drift_add(nan, 1.0f) <= 1e30f || sf::drift_add(0.0f, nan) <= 1e30f) ++fails;
  if (sf::slack_less(nan, 1.0f) > -1e30f || sf::slack_less(1.0f, nan) > -1e30f) ++fails;
  std::printf("%d\n", fails);
  return fails != 0;
}
