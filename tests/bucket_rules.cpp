// Prints, for lines "key_words n_max m" on standard input: the default log2 buckets (default block
// shape), then variant and log2 buckets of every choice of the autotuner.
#include <cstdio>

#include "../paper_2407_07718_amd/csrc/kc_rules.hpp"

int main() {
  int kw, m;
  unsigned long long n;
  while (scanf("%d %llu %d", &kw, &n, &m) == 3) {
    printf("%d", default_log_b(n, m, hash_slots(kw, DEFAULT_VARIANT)));
    for (const TuneChoice& c : TUNE_CHOICES) printf(" %u %d", c.variant, tuned_log_b(n, m, kw, c));
    printf("\n");
  }
}
