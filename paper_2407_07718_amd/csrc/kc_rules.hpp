// Rules on sizes, in plain host code.
#pragma once
#include <stdint.h>

#include <algorithm>

// On-chip shapes of the bucket count, as slots of the block's hash table (half as many for
// 128-bit keys): 1 = 4,096 (the default: the most that leaves three blocks of 512 threads per
// CU), 2 = 8,192, 3 = 2,048.
constexpr uint32_t DEFAULT_VARIANT = 1;
inline uint32_t hash_slots(int key_words, uint32_t variant) {
  return (variant == 2 ? 8192u : variant == 3 ? 2048u : 4096u) >> (key_words - 1);
}
// Buckets of a count of n_max k-mers: a mean of at most the table's slots, but for small
// inputs up to 1,024 buckets of 512 k-mers, so that every CU has some.  Larger buckets would
// suit repeated k-mers (1 Gbp at 20x: 15.1 ms with 3,800 k-mers per bucket, 14.7 ms with 7,600),
// but where nearly all are distinct they overflow the table and are counted in classes
// (400 Mbp at 0.8x: 12.2 ms with 3,050, 13.2 ms with 6,100).
inline int auto_log_b(uint64_t n_max, uint64_t slots) {
  int lb = 1, few = 1;
  while (lb < 20 && (n_max >> lb) > slots) ++lb;
  while (few < 10 && (n_max >> few) > 512) ++few;
  return std::max(lb, few);
}
// The same where minimizers of at least 9 bases (2^17 of them) spread the k-mers evenly over few
// buckets: from 64 buckets on only as many as bring the mean to half the slots, because each costs
// its share of an empty table.  (240,000 k-mers of 31 bases, 6x: 87 us of kernels in 128 buckets,
// 100 in 512; 500,000: 103 us in 256, 120 in 1,024; 800,000 in 64 210 us, in 128 123.  With
// minimizers of 5 bases 500,000 k-mers seen once take 1.33 ms in 256 buckets, 0.79 in 1,024, with 8
// bases 240,000 of 51 bases 158 us in 256 and 147 in 512.)
inline int even_log_b(uint64_t n_max, uint64_t slots) {
  int lb = auto_log_b(n_max, slots), few = 6;
  while (few < lb && (n_max >> few) > slots / 2) ++few;
  return std::min(lb, few);
}
// log2 of the buckets of a count with minimizers of m bases.
inline int default_log_b(uint64_t n_max, int m, uint64_t slots) {
  return m >= 9 ? even_log_b(n_max, slots) : auto_log_b(n_max, slots);
}

// What the autotuner chooses from: a block shape, and buckets around the rule's number.
struct TuneChoice {
  uint32_t variant;
  int log_b_delta;
};
constexpr TuneChoice TUNE_CHOICES[] = {{1, -1}, {1, 0}, {1, 1}, {2, -1}, {2, 0}, {2, 1}, {3, -1}, {3, 0}, {3, 1}};
inline int tuned_log_b(uint64_t n_max, int m, int key_words, TuneChoice c) {
  return std::min(20, std::max(1, default_log_b(n_max, m, hash_slots(key_words, c.variant)) + c.log_b_delta));
}
