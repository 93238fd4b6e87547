// The append's launch: every head row of every token has its wave, once, and up to the 2^26 tokens that 64 threads per
// token allow no launch has more than 2^32 - 1 threads along x.
#include <cstdio>
#include <random>
#include "efim_internal.h"

using namespace efim;
int main() {
  std::mt19937_64 rng(3);
  long whole = 0, held_back = 0;
  for (int iter = 0; iter < 200000; ++iter) {
    const int d = rng() & 1 ? 64 : 128, rows = 2 + (int)(rng() % 200);
    int64_t tokens = 1 + (int64_t)(rng() >> (38 + rng() % 26));
    if (tokens >= (int64_t)1 << 26) tokens = ((int64_t)1 << 26) - 1 - (int64_t)(rng() % 1000);
    const AppendShape s = append_shape(tokens, rows, d);
    const int64_t threads = (int64_t)64 * s.parts << s.tok_shift;
    if (threads > kAppendThreads || (int64_t)s.x * threads >= (int64_t)1 << 32 || s.y > 65535) {
      printf("%lld tokens of %d rows of %d: %u x %u workgroups of %lld threads\n", (long long)tokens, rows, d, s.x, s.y, (long long)threads);
      return 1;
    }
    const int64_t covered = (int64_t)s.x << s.tok_shift, waves = (int64_t)s.y * s.parts, per_wave = kAppendPasses * 1024 / d;
    if (covered < tokens || covered - tokens >= 1 << s.tok_shift || waves * per_wave < rows || (waves - s.parts) * per_wave >= rows) {
      printf("%lld tokens of %d rows of %d: covered %lld, waves %lld\n", (long long)tokens, rows, d, (long long)covered, (long long)waves);
      return 1;
    }
    const bool large = tokens * rows * d * 2 >= (int64_t)1 << 29;
    whole += large && s.y < (rows + per_wave - 1) / per_wave;
    held_back += large && s.parts == 1 && s.y > 1;
  }
  if (!whole || !held_back) { printf("%ld of whole tokens, %ld held back\n", whole, held_back); return 1; }
  printf("append shape ok, %ld of whole tokens, %ld held back\n", whole, held_back);
  return 0;
}
