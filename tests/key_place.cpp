// Prints key_top32 and key_place of the keys read from standard input: lines of
// "words nbits hi lo" (hexadecimal words), for tests/test_key_place.py.
#include <cstdio>

#include "../paper_2407_07718_amd/csrc/kc_segsort.hpp"

int main() {
  unsigned words, nbits;
  unsigned long long hi, lo;
  while (scanf("%u %u %llx %llx", &words, &nbits, &hi, &lo) == 4) {
    if (words == 1)
      printf("%u %u %u\n", key_top32((u64)lo, (int)nbits), key_place((u64)lo, (int)nbits, 0), key_place((u64)lo, (int)nbits, 1));
    else {
      const k128 k{lo, hi};
      printf("%u %u %u\n", key_top32(k, (int)nbits), key_place(k, (int)nbits, 0), key_place(k, (int)nbits, 1));
    }
  }
}
