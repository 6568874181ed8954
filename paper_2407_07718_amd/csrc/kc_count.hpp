// Stage 3 of the pipeline: per bucket, expand supermers into canonical k-mer keys and count
// them in a hash table on chip; keys whose count lies in [min_freq, max_freq] survive, every
// distinct key feeds the frequency histogram.  Large buckets are cut into chunks whose
// (k-mer, count) lists are merged (kc_segsort.hpp).
//
// Paper mapping: k-mers are extracted from the supermers of a task and counted (there by a sort
// and a linear scan over the sorted array, Section 3.5, heavy-hitter transform; Section 3.1), and
// the scan records the histogram or copies the k-mers that meet the frequency requirement to
// another array (Section 3.1).  A bucket is a task (Section 3.4): independent of all others because
// equal k-mers never span two buckets.
#pragma once
#include <type_traits>

#include "kc_common.hpp"
#include "kc_sort.hpp"

struct DevTotals {
  u64 n_pairs;        // survivors (pairs in [min_freq, max_freq])
  u64 n_windows;      // valid k-mer windows
  u64 n_distinct;     // runs = distinct canonical k-mers
  u64 overflow_sum;   // sum of counts that fall into the last histogram bin
  u64 max_count;
  u64 n_records;      // supermer records written
  u64 flags;          // bit 0: bad offsets, bit 1: record buffer overflow, bit 2: survivor overflow;
                      // rounds: bit 3: a bucket group exceeds a round, bit 4: survivors exceed the pool
  u64 large_keys;     // k-mers of large buckets
  u64 tiny_buckets, tiny_kmers, small_buckets, small_kmers, large_buckets, chunks, list_entries, buckets;
  u64 n_occ;          // extension version: occurrences of the reported k-mers
};

struct CountArgs {
  const u32* rec;          // bucket-ordered supermer records
  const u32* rec_off;      // [B+1]
  const u64* bcnt;         // per bucket (records << 32) | k-mers
  const u32* large_list;
  const u64* chunk_start;  // chunks of large buckets: first key in lkeys ...
  const u32* chunk_len;    // ... and length (<= cap)
  const u64* meta;         // see plan_meta
  const u64* kall_off;     // per bucket: first k-mer slot (prefix of k-mers over all buckets)
  int k;
  int rec_words;
  u32 min_freq, max_freq;
  u64 hist_len;
  u64* hist;               // [hist_len]
  DevTotals* tot;
  void* surv_k;            // survivors of bucket b at slots kall_off[b] + i: keys ...
  u32* surv_c;             // ... and counts
  u32* surv_cnt;           // survivors per bucket
  u32* late;               // buckets left to the second launch: bucket | class depth << 24 ...
  u32* late_n;             // ... and their number
  const void* lkeys;       // expanded keys of the large buckets, at their buckets' k-mer slots
  void* kl_k;              // (k-mer, count) list of chunk c at slots chunk_start[c] + i (an array of
                           // its own: a chunk counted in classes reads its keys several times)
  u32* kl_c;
  u32* kl_cnt;             // list length per chunk
  // several read sets in one count: bucket b belongs to set bset[b], and hist / tot are
  // arrays over the sets ([n_sets][hist_len] bins, [n_sets] totals)
  const u32* bset;
  u32 n_sets;
  // rounds: only the buckets of coarse groups [rng[0], rng[1]) hold k-mers (null: all)
  const u32* rng;
  int log_f;
};

// ---------------------------------------------------------------------------- key mixing
// The classes of a bucket that overflows its table, and the sorts that bring equal keys of a large
// bucket's lists together (whatever their order), go by the keys' images
// under a bijection whose low bits depend on every key bit: y = b ^ (b >> 32) with
// b = a * C mod 2^64 and a = x ^ (x >> 32).  Both xor-shifts are involutions and C is
// odd, so the map is undone exactly by the same steps in reverse with C^-1.  K-mers that
// differ in one base (sequencing errors) then differ in their low bits with
// probability about 1 - 2^-32, so a sort over the low digits alone already separates
// distinct keys (checked, and completed by the remaining passes when it did not).
// 128-bit keys mix their low word and fold in a mix of the high word (a Feistel step).
constexpr u64 MIX_C = 0x9e3779b97f4a7c15ull;
constexpr u64 mod_inverse64(u64 c) {
  u64 x = c;                                      // correct to 3 bits for odd c
  for (int i = 0; i < 5; ++i) x *= 2ull - c * x;  // Newton step doubles the correct bits
  return x;
}
constexpr u64 MIX_CINV = mod_inverse64(MIX_C);
static_assert(MIX_C * MIX_CINV == 1ull, "modular inverse");

__device__ __forceinline__ u64 mix64(u64 x) {
  x ^= x >> 32;
  x *= MIX_C;
  return x ^ (x >> 32);
}
__device__ __forceinline__ u64 unmix64(u64 y) {
  y ^= y >> 32;
  y *= MIX_CINV;
  return y ^ (y >> 32);
}
__device__ __forceinline__ u64 mix_key(u64 x) { return mix64(x); }
__device__ __forceinline__ u64 unmix_key(u64 y) { return unmix64(y); }
__device__ __forceinline__ k128 mix_key(k128 x) { return k128{mix64(x.lo) ^ mix64(x.hi ^ MIX_C), x.hi}; }
__device__ __forceinline__ k128 unmix_key(k128 y) { return k128{unmix64(y.lo ^ mix64(y.hi ^ MIX_C)), y.hi}; }

// ---------------------------------------------------------------------------- expand
// The canonical k-mer whose first base is bit q of a record's base field (k <= 31: a
// u64; k >= 32: a 128-bit key), read with funnel shifts from the record words at rec.
__device__ __forceinline__ u64 rec_bits64(const u32* p, u32 q) {   // 64 bits from bit q of p
  const u32 w = q >> 5, sh = q & 31;
  return ((u64)__builtin_amdgcn_alignbit(p[w + 2], p[w + 1], sh) << 32) | __builtin_amdgcn_alignbit(p[w + 1], p[w], sh);
}
template <typename K> __device__ __forceinline__ K canon_at(const u32* rec, u32 q, int k);
template <> __device__ __forceinline__ u64 canon_at<u64>(const u32* rec, u32 q, int k) {
  const u64 kmask = (1ull << (2 * k)) - 1;
  const u64 V = rec_bits64(rec, q) & kmask;
  const u64 F = rev2_64(V) >> (64 - 2 * k);
  const u64 RC = ~V & kmask;
  return F < RC ? F : RC;
}
template <> __device__ __forceinline__ k128 canon_at<k128>(const u32* rec, u32 q, int k) {
  const int hb = 2 * k - 64;                      // bits in the high word, 0..62
  const u64 mhi = hb ? ((1ull << hb) - 1) : 0ull;
  const u64 vlo = rec_bits64(rec, q), vhi = rec_bits64(rec, q + 64) & mhi;
  const u64 rlo = rev2_64(vhi), rhi = rev2_64(vlo);
  const int s = 128 - 2 * k;                      // 2..64
  k128 F, RC;
  if (s == 64) { F.lo = rhi; F.hi = 0; }
  else { F.lo = (rlo >> s) | (rhi << (64 - s)); F.hi = rhi >> s; }
  RC.lo = ~vlo;
  RC.hi = ~vhi & mhi;
  return key_lt(F, RC) ? F : RC;
}


// ---------------------------------------------------------------------------- run output
// One run (distinct key with count c): histogram, extremes and the filtered output.
struct RunSink {
  u32* hist_s;             // LDS bins [0, 256)
  u64 hist_len;
  u64* hist;
  DevTotals* tot;
  u32* lmax;               // LDS running max
  unsigned long long* lover;   // LDS sum of counts in the last bin
};

// Runs held by the lanes with `act` set; every lane of the wave calls it (converged).
// Runs seen once -- most error k-mers -- are counted with one ballot, and the running
// maximum is only raised by lanes above the value already recorded, so that the LDS
// atomics of a wave rarely pile up on one address.
__device__ __forceinline__ void run_stats_lanes(const RunSink& S, u64 c, bool act) {
  const u64 last = S.hist_len - 1;
  const u64 bin = c < last ? c : last;
  const u64 ones = __ballot(act && bin == 1);
  if (ones && lane_id() == 0) atomicAdd(&S.hist_s[1], (u32)__popcll(ones));
  if (act && bin != 1) {
    if (bin < 256) atomicAdd(&S.hist_s[bin], 1u);
    else atomicAdd((unsigned long long*)&S.hist[bin], 1ull);
  }
  if (act && c >= last) atomicAdd(S.lover, (unsigned long long)c);
  const u32 c32 = (u32)min(c, (u64)0xFFFFFFFFu);
  if (act && c32 > *(volatile u32*)S.lmax) atomicMax(S.lmax, c32);
}

// Several read sets in one count: the sink's global targets become those of set s.
__device__ __forceinline__ void sink_to_set(RunSink& S, u64* hist, DevTotals* tot, u32 s) {
  S.hist = hist + (u64)s * S.hist_len;
  S.tot = tot + s;
}

__device__ __forceinline__ void flush_stats(const RunSink& S, u64 ndist) {
  const u32 H = (u32)min(S.hist_len, (u64)256);
  for (u32 i = threadIdx.x; i < H; i += blockDim.x) {
    const u32 v = S.hist_s[i];
    if (v) atomicAdd((unsigned long long*)&S.hist[i], (unsigned long long)v);
  }
  if (threadIdx.x == 0) {
    // (each guard keeps empty blocks off these shared addresses: same-address atomics
    // serialize, and many blocks of a persistent grid finish together)
    if (*S.lmax) atomicMax((unsigned long long*)&S.tot->max_count, (unsigned long long)*S.lmax);
    if (*S.lover) atomicAdd((unsigned long long*)&S.tot->overflow_sum, *S.lover);
    if (ndist) atomicAdd((unsigned long long*)&S.tot->n_distinct, (unsigned long long)ndist);
  }
}

// ---------------------------------------------------------------------------- on-chip count
// A bucket is counted in a hash table in LDS: its supermers are expanded key by key, each
// key finds or claims its slot and adds one there, and the occupied slots are the bucket's
// distinct k-mers with their counts.  (The survivors are sorted by key at the end, so the
// order inside a bucket is free.)
//
// Table of SLOTS keys with 16-bit counts (an item holds at most 65,535 keys), probed by
// aligned pairs: one 16-byte read sees two slots, a free slot is claimed by a compare and
// swap, and a key whose pair is full goes on to the next pair.  A slot never becomes free
// again and a key takes the first slot of its probe sequence that no other key holds, so a
// key has one slot whatever the order of the lanes.  After PROBES full pairs the table is
// given up as too full, and the item is counted in two halves, by the next bit of the
// keys' mixed images (DFS over the bits; the images are a bijection, so a class at full
// depth holds one key), or, where that would take four passes over a bucket and more, in as many
// classes by other blocks.  Only the distinct keys count against the table, so an item may
// hold many times SLOTS keys.
// One wave's scratch: the records it expands, one bit per unit of them (a unit is up to U
// consecutive k-mers of one record, expanded by one lane) at each record's first unit, and
// keys waiting for a slot; after the insertion, the list of its occupied slots.
template <typename K>
struct HashWave {
  static constexpr int RW = sizeof(K) == 8 ? 4 : 8;
  static constexpr u32 RECS = sizeof(K) == 8 ? 48 : 24, QUEUE = 64;
  alignas(16) u32 rec[RECS * RW + 4];   // (+ words read past the last record)
  u64 mark[16];
  K queue[QUEUE];
};
template <typename K, int T, u32 SLOTS>
struct HashSmem {
  static constexpr int W = T / 64;
  alignas(16) u64 lo[SLOTS];
  alignas(16) u64 hi[sizeof(K) == 8 ? 2 : SLOTS];
  u32 cnt[SLOTS / 2];              // two 16-bit counts per word, one word per pair
  HashWave<K> w[W];
  u32 hist_s[256];
  u32 lmax, kept, full, seen, dist[2];   // (dist: of this item and the next)
  unsigned long long lover, ndist;
};
// No canonical k-mer has these words: 2k <= 62 bits for k <= 31; for k >= 32 a low word of
// 32 T's has a smaller reverse complement, and the high word has at most 62 bits.
constexpr u64 HASH_FREE = ~0ull;
constexpr u32 HASH_PROBES = 16;

// 24-bit products run at the full rate (32-bit ones at a quarter); the top bits of the sum
// depend on every key bit.
__device__ __forceinline__ u32 mul24(u32 a, u32 c) { return (a & 0xFFFFFFu) * c; }
__device__ __forceinline__ u32 key_hash(u64 k) {
  const u32 l = (u32)k, h = (u32)(k >> 32);
  return mul24(l, 0x9E3779u) + mul24(__builtin_amdgcn_alignbit(h, l, 24), 0x85EBCBu) + mul24(h >> 16, 0xC2B2AFu);
}
__device__ __forceinline__ u32 key_hash(k128 k) {
  const u32 l = (u32)k.hi, h = (u32)(k.hi >> 32);
  return key_hash(k.lo) + mul24(l, 0x27D4EBu) + mul24(__builtin_amdgcn_alignbit(h, l, 24), 0x165667u) +
         mul24(h >> 16, 0xB5297Bu);
}

// Classes of the DFS: keys whose mixed image has the low d bits p (d = 0: all keys).
template <typename K> struct HashClass;
template <> struct HashClass<u64> {
  u32 d = 0;
  u64 p = 0;
  __device__ __forceinline__ bool has(u64 k) const {
    const u64 y = mix_key(k);
    return (d >= 64 ? y : y & ((1ull << d) - 1)) == p;
  }
  __device__ __forceinline__ bool bit() const { return (p >> (d - 1)) & 1; }
  __device__ __forceinline__ void flip() { p ^= 1ull << (d - 1); }
  __device__ __forceinline__ void set(u32 d_, u32 p_) { d = d_, p = p_; }
};
template <> struct HashClass<k128> {
  u32 d = 0;
  k128 p = {0, 0};
  __device__ __forceinline__ bool has(k128 k) const {
    const k128 y = mix_key(k);
    if (d < 64) return (y.lo & ((1ull << d) - 1)) == p.lo;
    return y.lo == p.lo && (d >= 128 ? y.hi == p.hi : (y.hi & ((1ull << (d - 64)) - 1)) == p.hi);
  }
  __device__ __forceinline__ bool bit() const { return d <= 64 ? (p.lo >> (d - 1)) & 1 : (p.hi >> (d - 65)) & 1; }
  __device__ __forceinline__ void flip() {
    if (d <= 64) p.lo ^= 1ull << (d - 1);
    else p.hi ^= 1ull << (d - 65);
  }
  __device__ __forceinline__ void set(u32 d_, u32 p_) { d = d_, p = k128{p_, 0}; }
};
// The next class after c, of those that share its low d0 bits; false when all are counted.
template <typename K>
__device__ __forceinline__ bool next_class(HashClass<K>& c, u32 d0) {
  while (c.d > d0 && c.bit()) {
    c.flip();
    --c.d;
  }
  if (c.d == d0) return false;
  c.flip();
  return true;
}

// The two words of a pair, read together.
struct HashPair {
  u64 x, y;
};
__device__ __forceinline__ HashPair hash_pair(const u64* p) {
  typedef u32 u32x4 __attribute__((ext_vector_type(4)));
  const u32x4 v = *reinterpret_cast<const u32x4*>(p);
  return HashPair{((u64)v.y << 32) | v.x, ((u64)v.w << 32) | v.z};
}

// Each lane with `act` counts its key; false for a lane whose key found no slot.
template <int T, u32 SLOTS>
__device__ __forceinline__ bool hash_add(HashSmem<u64, T, SLOTS>& S, u64 key, bool act) {
  constexpr int SH = 32 - __builtin_ctz(SLOTS / 2);
  u32 i = (key_hash(key) >> SH) * 2;
  u32 left = HASH_PROBES;
  while (act) {
    const HashPair t = hash_pair(&S.lo[i]);
    u32 s = i + (t.x == key ? 0u : 1u);
    bool done = t.x == key || t.y == key;
    if (!done) {
      if (t.x == HASH_FREE || t.y == HASH_FREE) {   // claim it, or look at the pair again
        s = i + (t.x == HASH_FREE ? 0u : 1u);
        const u64 old = atomicCAS((unsigned long long*)&S.lo[s], HASH_FREE, key);
        done = old == HASH_FREE || old == key;
      } else {
        i = (i + 2) & (SLOTS - 1);
        if (--left == 0) return false;
      }
    }
    if (done) {
      atomicAdd(&S.cnt[s >> 1], 1u << ((s & 1) * 16));
      act = false;
    }
  }
  return true;
}
// 128-bit keys claim a slot with their low word and then write its high word; a lane that
// meets its low word in a slot whose high word is not there yet looks again (the claiming
// lane writes it with its next instruction).
template <int T, u32 SLOTS>
__device__ __forceinline__ bool hash_add(HashSmem<k128, T, SLOTS>& S, k128 key, bool act) {
  constexpr int SH = 32 - __builtin_ctz(SLOTS / 2);
  u32 i = (key_hash(key) >> SH) * 2;
  u32 left = HASH_PROBES;
  while (act) {
    const HashPair t = hash_pair(&S.lo[i]);
    u32 s = i;
    bool done = false, again = false;
    if (t.x == key.lo) {
      const u64 h = __hip_atomic_load(&S.hi[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      done = h == key.hi;
      again = h == HASH_FREE;
    }
    if (!done && !again && t.y == key.lo) {
      s = i + 1;
      const u64 h = __hip_atomic_load(&S.hi[s], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
      done = h == key.hi;
      again = h == HASH_FREE;
    }
    if (!done && !again) {
      if (t.x == HASH_FREE || t.y == HASH_FREE) {
        s = i + (t.x == HASH_FREE ? 0u : 1u);
        if (atomicCAS((unsigned long long*)&S.lo[s], HASH_FREE, key.lo) == HASH_FREE) {
          __hip_atomic_store(&S.hi[s], key.hi, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_WORKGROUP);
          done = true;
        }
      } else {
        i = (i + 2) & (SLOTS - 1);
        if (--left == 0) return false;
      }
    }
    if (done) {
      atomicAdd(&S.cnt[s >> 1], 1u << ((s & 1) * 16));
      act = false;
    }
  }
  return true;
}

// Whether the key sits in the first / second slot of pair p.
template <int T, u32 SLOTS>
__device__ __forceinline__ void hash_find(const HashSmem<u64, T, SLOTS>& S, u64 key, u32 p, bool& in0, bool& in1) {
  const HashPair t = hash_pair(&S.lo[2 * p]);
  in0 = t.x == key;
  in1 = t.y == key;
}
template <int T, u32 SLOTS>
__device__ __forceinline__ void hash_find(const HashSmem<k128, T, SLOTS>& S, k128 key, u32 p, bool& in0, bool& in1) {
  const HashPair t = hash_pair(&S.lo[2 * p]), h = hash_pair(&S.hi[2 * p]);
  in0 = ((t.x ^ key.lo) | (h.x ^ key.hi)) == 0;
  in1 = ((t.y ^ key.lo) | (h.y ^ key.hi)) == 0;
}

// The canonical k-mers at bases o and o + 1 of the record at rec.  One window of 64 (128)
// bits holds both; it is read with funnel shifts, and its 2-bit reversal, brought down so
// that the second k-mer's forward value starts at bit 0, gives the forward values.
__device__ __forceinline__ void canon_two(const u32* rec, u32 o, int k, u64 (&out)[2]) {
  const u64 mask = (1ull << (2 * k)) - 1;
  const u64 V = rec_bits64(rec, 2 * o), R = rev2_64(V) >> (62 - 2 * k);
  const u64 f0 = (R >> 2) & mask, c0 = ~V & mask, f1 = R & mask, c1 = ~(V >> 2) & mask;
  out[0] = f0 < c0 ? f0 : c0;
  out[1] = f1 < c1 ? f1 : c1;
}
__device__ __forceinline__ void canon_two(const u32* rec, u32 o, int k, k128 (&out)[2]) {
  const u64 mhi = (1ull << (2 * k - 64)) - 1;
  const u64 vl = rec_bits64(rec, 2 * o), vh = rec_bits64(rec, 2 * o + 64);
  const u64 rl = rev2_64(vh), rh = rev2_64(vl);
  const int s = 126 - 2 * k;                      // 0 .. 62
  const u64 fl = (rl >> s) | ((rh << 1) << (63 - s)), fh = rh >> s;
  const k128 f0{(fl >> 2) | (fh << 62), (fh >> 2) & mhi}, c0{~vl, ~vh & mhi};
  const k128 f1{fl, fh & mhi}, c1{~((vl >> 2) | (vh << 62)), ~(vh >> 2) & mhi};
  out[0] = key_lt(f0, c0) ? f0 : c0;
  out[1] = key_lt(f1, c1) ? f1 : c1;
}

// Blocks take buckets (REST = false), or in a second launch (REST) the chunks of large buckets
// (whose keys are already expanded in HBM) and the classes of the buckets that the first one left
// to it, in turn.  A bucket's slots are final counts: statistics, and the
// survivors to the bucket's own k-mer slots; a chunk's are the (k-mer, count) list of its
// slots -- the paper's kmerlist form of a heavy-hitter task (Section 3.5) -- merged later
// through HBM.  Several read sets (MS): a contiguous range of buckets per block (they are
// numbered set by set), whose statistics are flushed when the set changes.
//
// Bound by VALU issue and LDS round trips (on the 1 Gbp long reads, k = 31: 68% of the VALU slots, 46%
// of the LDS cycles; HBM is idle): about 97 vector instructions per 64 k-mers, half of them the
// expansion.  Hence two k-mers per lane from one window of bits, 24-bit hash products, full
// rows of 64 units, and a queue for the keys that need more than one look (10% there, but
// nearly every row of 64 has some).  512 threads on 4,096 slots: 53 KB and at most 80 VGPRs, so
// three blocks and 24 waves share a CU.  Measured there against the LSD radix passes in LDS
// that it replaces (one wave per bucket up to 896 k-mers, one block up to 2,048, longer ones
// expanded into HBM, cut and merged): 12.4 -> 3.7 ms at k = 31 (998 M k-mers), and at k = 51
// 10.8 -> 3.2 ms (398 M).  256 threads on 2,048 slots: 4.0 ms; one key per lane, rows cut at
// every 48 records and no queue: 5.7 ms.
// Neighbouring buckets share a table while their distinct keys fill about a quarter of it,
// which spares barriers and table scans (2^18 buckets: 4.15 -> 3.67 ms); at half full the first
// pair misses too often (4.8 ms), at a tenth the scans show again (4.3 ms).
// A bucket of more k-mers than slots whose table overflows is given up at once: the share of its
// records that filled the table tells how many classes it takes.  Two are counted by the
// block; four to 16 are left to the second launch, where they run side by side.  (With all classes one
// after the other in the bucket's block: 5 Mbp at 0.7x, k = 21, minimizers of 6 bases 4.2 ms, 1.9 so;
// 9 Mbp of reads with 80 % A and T, k = 21, minimizers of 11 bases 2.9 and 1.1.  With buckets above two
// tables cut into chunks and merged, for any input: 2.0 and 1.9, but 400 Mbp of long reads, k = 51,
// 7.9 instead of 6.7 ms.)
constexpr u32 LATE_DEPTH = 4;      // classes of a bucket left over: 2^2 to 2^4
template <typename K, int T, u32 SLOTS, bool REST, bool MS>
__global__ __launch_bounds__(T, T <= 512 ? 6 : 4) void k_hash_count(CountArgs A, u32 B, u32 cap) {
  using SM = HashSmem<K, T, SLOTS>;
  using HW = HashWave<K>;
  constexpr int W = SM::W, RW = HW::RW, U = 2;
  constexpr u32 ROWS = SLOTS / T, SH = 32 - __builtin_ctz(SLOTS / 2);
  static_assert(sizeof(HW) >= 2 * 64 * ROWS, "the list of a wave's occupied slots");
  __shared__ SM S;
  const u32 tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6);
  // second launch: the chunks, then the classes, class by class over the buckets left over
  const u32 n_chunks = REST ? (u32)A.meta[4] : 0u, n_late = REST ? *A.late_n : 0u;
  const u32 n_rest = n_chunks + (n_late << LATE_DEPTH);
  if (REST && blockIdx.x >= n_rest) return;
  HW& H = S.w[wave];
  auto clear_table = [&]() {
    for (u32 i = tid; i < SLOTS; i += T) {
      S.lo[i] = HASH_FREE;
      if (sizeof(K) == 16) S.hi[i] = HASH_FREE;
    }
    for (u32 i = tid; i < SLOTS / 2; i += T) S.cnt[i] = 0;
  };
  clear_table();
  for (u32 i = tid; i < 256; i += T) S.hist_s[i] = 0;
  if (lane < 4) H.rec[HW::RECS * RW + lane] = 0;
  if (tid == 0) {
    S.lmax = 0;
    S.lover = 0;
    S.ndist = 0;
    S.kept = 0;
    S.full = 0;
    S.seen = 0;
    S.dist[0] = S.dist[1] = 0;
  }
  // the marks hold 1,024 units: records of up to 32 k-mers RECS at a time, longer ones 24
  const u32 step = (RW == 4 && 52 - A.k <= 32) ? HW::RECS : 24u;
  static_assert(HW::RECS >= 24 && HW::RECS <= 64, "one record per lane");
  RunSink sink{S.hist_s, A.hist_len, A.hist, A.tot, &S.lmax, &S.lover};
  const u64 lemask = lane == 63 ? ~0ull : ((2ull << lane) - 1);   // lanes <= this lane
  const K* lkeys = reinterpret_cast<const K*>(A.lkeys);
  // Many buckets per block: consecutive ones are counted together while they fit.  (Equal
  // k-mers share a bucket, and the records and k-mer slots of neighbouring buckets adjoin.)
  const u32 b0 = A.rng ? A.rng[0] << A.log_f : 0u, nb = (A.rng ? A.rng[1] << A.log_f : B) - b0;
  const bool merge = !REST && nb >= 8 * gridDim.x;
  const u32 stride = MS || merge ? 1u : gridDim.x;
  u32 room = 0, parity = 0;
  u32 learned = 0;   // class depth that the last full item ended at
  u32 ndist = 0;     // distinct keys this wave saw
  auto flush = [&]() {
    if (lane == 0 && ndist) atomicAdd(&S.ndist, (unsigned long long)ndist);
    ndist = 0;
    __syncthreads();
    flush_stats(sink, S.ndist);
  };
  // An item: its size and place, this wave's share of its records [ra, rb), the item after it.
  struct Item {
    u64 base;
    u32 n, ra, rb, after;
  };
  // The plan's figures of the buckets from b on, one bucket per lane, loaded an item ahead.
  struct Ahead {
    u64 c, ko;
    u32 ro, st;
  };
  auto load_ahead = [&](u32 b, u32 end) {
    Ahead R{0, 0, 0, 0};
    if (b < end) {
      const u32 i = merge ? min(b + lane, end - 1) : b;
      R.c = A.bcnt[i];
      R.ko = A.kall_off[i];
      R.ro = A.rec_off[i];
      if constexpr (MS) R.st = A.bset[i];
    }
    return R;
  };
  // The item that starts at bucket b: as many buckets up to `end` as hold at most `room`
  // k-mers together, but one at least (a large bucket is an item with nothing to do).
  auto look_up = [&](const Ahead& R, u32 b, u32 end) {
    Item I{0, 0, 0, 0, b + stride};
    if (b >= end) return I;
    const u32 nk = (u32)R.c, nr = (u32)(R.c >> 32);
    I.base = uniform(R.ko);
    I.n = uniform(nk);
    u32 m = 1;
    if (merge) {
      const bool fits =
          b + lane < end && nk <= cap && R.ko + nk - I.base <= room && (!MS || R.st == uniform(R.st));
      m = max(1u, (u32)__builtin_ctzll(~__ballot(fits) | (1ull << 63)));
      I.after = b + m;
    }
    const u32 r0 = uniform(R.ro), r1 = lane_read(R.ro + nr, (int)m - 1), per = (r1 - r0 + W - 1) / W;
    I.n = I.n > cap ? 0u : lane_read((u32)(R.ko - I.base) + nk, (int)m - 1);
    if (I.n) {
      I.ra = min(r1, r0 + wave * per);
      I.rb = min(r1, I.ra + per);
    }
    return I;
  };
  // The first records of an item are on their way while the item before it is counted.
  uint4 v[RW / 4];
  auto load_records = [&](u32 c0, u32 rb) {
#pragma unroll
    for (int q = 0; q < RW / 4; ++q)
      v[q] = lane < step && c0 + lane < rb ? reinterpret_cast<const uint4*>(A.rec)[(u64)(c0 + lane) * (RW / 4) + q]
                                           : make_uint4(0u, 0u, 0u, 0u);
  };
  // (REST: `chunk` tells chunks from classes of a bucket; of the latter, the class p at depth d0)
  auto do_item = [&](u32 item, const Item& I, const Item& next, bool chunk, u32 d0, u32 p) {
    const u32 n = I.n;
    const u64 base = I.base;
    if (n == 0) {
      load_records(next.ra, next.rb);
      return;
    }
    K* const out_k = reinterpret_cast<K*>(chunk ? A.kl_k : A.surv_k) + base;
    u32* const out_c = (chunk ? A.kl_c : A.surv_c) + base;
    const u32 n_buckets = merge ? I.after - item : 1u;
    // whether the item may be left to the second launch (not once a class of it is counted)
    bool may_leave = !REST && n > SLOTS && n_buckets == 1;
    HashClass<K> cls;
    if (REST && !chunk) cls.set(d0, p);
    else cls.d = !may_leave && n > SLOTS / 2 ? learned : 0u;
    u32 deepest = cls.d;
    for (;;) {
      bool ok = true;
      u32 queued = 0;   // keys in the wave's queue
      // The queue's keys claim their slots, one per lane.
      auto drain = [&]() {
        __builtin_amdgcn_wave_barrier();
        const K key = H.queue[lane];
        ok &= hash_add(S, key, lane < queued);
        __builtin_amdgcn_wave_barrier();
        queued = 0;
      };
      // One key per lane: counted at once where it sits in its first pair (the common case);
      // the others wait in the queue until most lanes have one, because claiming a slot takes
      // several LDS round trips whatever the number of lanes.
      auto add_keys = [&](const K (&key)[U], const bool (&on)[U]) {
        u32 p[U];
        bool in0[U], in1[U];
#pragma unroll
        for (int j = 0; j < U; ++j) {
          p[j] = key_hash(key[j]) >> SH;
          hash_find(S, key[j], p[j], in0[j], in1[j]);
        }
#pragma unroll
        for (int j = 0; j < U; ++j)
          if (on[j] & (in0[j] | in1[j])) atomicAdd(&S.cnt[p[j]], in0[j] ? 1u : 0x10000u);
#pragma unroll
        for (int j = 0; j < U; ++j) {
          const bool pend = on[j] & !(in0[j] | in1[j]);
          const u64 m = __ballot(pend);
          const u32 c = (u32)__popcll(m);
          if (c > 24) {
            ok &= hash_add(S, key[j], pend);
          } else if (c) {
            if (pend) H.queue[queued + mbcnt64(m)] = key[j];
            queued += c;
            if (queued >= 40) drain();
          }
        }
      };
      u32 seen = I.rb - I.ra;   // records that the wave has added
      if (chunk) {
        for (u32 i0 = wave * 64 * U; i0 < n; i0 += T * U) {
          K key[U];
          bool on[U];
#pragma unroll
          for (int j = 0; j < U; ++j) {
            const u32 i = i0 + 64 * j + lane;
            key[j] = i < n ? lkeys[base + i] : key_zero<K>();
            on[j] = i < n && (cls.d == 0 || cls.has(key[j]));
          }
          add_keys(key, on);
        }
      } else {
        // each wave expands its records `step` at a time: lanes take the units in turn and find
        // their record by the marks of the records' first units; the units past the last full
        // row of 64 are left to the next step, which starts with their record (`skip` units of
        // it done)
        auto expand = [&](auto filtered, auto leaving) {
          constexpr bool LEAVING = decltype(leaving)::value;
          if (I.ra >= I.rb) load_records(next.ra, next.rb);
          u32 skip = 0;
          for (u32 c0 = I.ra; c0 < I.rb;) {
            if constexpr (LEAVING) {   // (the table is too full: nothing of this pass is of use)
              if (uniform(*(volatile u32*)&S.full)) {
                seen = c0 - I.ra;
                break;
              }
            }
            const u32 cnt = min(step, I.rb - c0);
            const u32 g = lane < cnt ? (v[RW / 4 - 1].w >> 26) + 1u : 0u;
            const u32 units = (g + U - 1) / U - (lane == 0 ? skip : 0u);
            const u32 inc = wave_scan_u32(units), rel = inc - units;
            const u32 G = lane_read(inc, 63);
            const u32 full = c0 + cnt == I.rb || G < 64 ? G : G & ~63u;
            const u32 before0 = skip ? 1u : 0u, first0 = 0u - skip;
            u32 c1 = c0 + cnt;
            skip = 0;
            if (full < G) {   // unit `full` is in record c1
              const u32 l = (u32)__popcll(__ballot(lane < cnt && rel <= full)) - 1u;
              skip = full - lane_read(rel, (int)l) - (l == 0 ? first0 : 0u);
              c1 = c0 + l;
            }
            __builtin_amdgcn_wave_barrier();
            if (lane < HW::RECS) {
#pragma unroll
              for (int q = 0; q < RW / 4; ++q) *reinterpret_cast<uint4*>(&H.rec[RW * lane + 4 * q]) = v[q];
            }
            if (lane < 16) H.mark[lane] = 0;
            if (g && lane >= before0) atomicOr((unsigned long long*)&H.mark[rel >> 6], 1ull << (rel & 63));
            __builtin_amdgcn_wave_barrier();
            if (c1 < I.rb) load_records(c1, I.rb);
            else load_records(next.ra, next.rb);
            const u64 mk = H.mark[lane & 15];   // lane j: the marks of units [64 j, 64 j + 64)
            u32 first = first0, before = before0;   // records before this row, the last one's first unit
            for (u32 q0 = 0, j = 0; q0 < full; q0 += 64, ++j) {
              const u64 m = ((u64)lane_read((u32)(mk >> 32), (int)j) << 32) | lane_read((u32)mk, (int)j);
              const u64 le = m & lemask;
              const u32 q = q0 + lane;
              const u32 st = le ? q0 + 63u - (u32)__clzll(le) : first;
              const u32 o = U * (q - st);   // (lanes past the last unit read on inside H)
              const u32* rec = &H.rec[RW * (before + (u32)__popcll(le) - 1u)];
              const u32 left = (rec[RW - 1] >> 26) + 1u - o;   // k-mers from o on
              K key[U];
              canon_two(rec, o, A.k, key);
              bool on[U] = {q < full, q < full && left > 1};
              if constexpr (decltype(filtered)::value) {
#pragma unroll
                for (int u = 0; u < U; ++u) on[u] = on[u] && cls.has(key[u]);
              }
              add_keys(key, on);
              before += (u32)__popcll(m);
              if (m) first = q0 + 63u - (u32)__clzll(m);
            }
            c0 = c1;
            if (LEAVING && !__all(ok)) S.full = 1;
          }
        };
        if (cls.d) expand(std::true_type(), std::false_type());
        else if (may_leave) expand(std::false_type(), std::bool_constant<!REST>());
        else expand(std::false_type(), std::false_type());
      }
      if (queued) drain();
      if (!ok) S.full = 1;
      __syncthreads();
      if (__builtin_expect(uniform(S.full), 0)) {
        if (may_leave && lane == 0) atomicAdd(&S.seen, seen);
        __syncthreads();
        // a table takes about nine tenths of its slots of distinct keys; a class is to have no more
        // than seven
        u32 depth = cls.d + 1;
        if (may_leave) {
          const u32 all = (u32)(A.bcnt[item] >> 32), part = max(1u, uniform(S.seen));
          while (depth < LATE_DEPTH && (u64)part << (depth - cls.d) < all + all / 4) ++depth;
        }
        clear_table();
        const bool leave = may_leave && depth >= 2;
        __syncthreads();
        if (tid == 0) {
          S.full = 0;
          S.seen = 0;
          if (leave) A.late[atomicAdd(A.late_n, 1u)] = item | depth << 24;
        }
        __syncthreads();
        if (leave) {
          load_records(next.ra, next.rb);
          return;
        }
        ++cls.d;   // the class's first half
        deepest = max(deepest, cls.d);
        load_records(I.ra, I.rb);
        continue;
      }
      may_leave = false;
      // (lanes of the first wave: the item's buckets' first k-mer slots and k-mers)
      u32 place = 0, size = 0;
      if constexpr (!REST) {
        if (wave == 0 && lane < n_buckets) {
          place = (u32)(A.kall_off[item + lane] - base);
          size = (u32)A.bcnt[item + lane];
        }
      }
      // each wave lists the occupied slots of its rows, then counts, reports and frees them
      u16* const list = reinterpret_cast<u16*>(&H);
      u32 dist = 0;
      {
        u32 c[ROWS];
#pragma unroll
        for (u32 j = 0; j < ROWS; ++j) c[j] = reinterpret_cast<const u16*>(S.cnt)[j * T + tid];
#pragma unroll
        for (u32 j = 0; j < ROWS; ++j) {
          const u64 occ = __ballot(c[j] != 0);
          if (c[j]) list[dist + mbcnt64(occ)] = (u16)(j * T + tid);
          dist += (u32)__popcll(occ);
        }
      }
      __builtin_amdgcn_wave_barrier();
      for (u32 e0 = 0; e0 < dist; e0 += 64) {
        const bool act = e0 + lane < dist;
        const u32 s = act ? list[e0 + lane] : 0u;
        u16* const cs = reinterpret_cast<u16*>(S.cnt) + s;
        const u32 c = act ? *cs : 0u;
        bool emit = act;
        if (!chunk) {
          emit = c >= A.min_freq && c <= A.max_freq;   // (min_freq >= 1)
          run_stats_lanes(sink, c, act);
        }
        const u64 em = __ballot(emit);
        if (em) {
          u32 at = 0;
          if (lane == 0) at = atomicAdd(REST && !chunk ? &A.surv_cnt[item] : &S.kept, (u32)__popcll(em));
          at = lane_read(at, 0) + mbcnt64(em);
          if (emit) {
            if constexpr (sizeof(K) == 8) out_k[at] = S.lo[s];
            else out_k[at] = K{S.lo[s], S.hi[s]};
            out_c[at] = c;
          }
        }
        if (act) {
          *cs = 0;
          S.lo[s] = HASH_FREE;
          if (sizeof(K) == 16) S.hi[s] = HASH_FREE;
        }
      }
      if (lane < 4) H.rec[HW::RECS * RW + lane] = 0;
      if (!chunk) ndist += dist;   // (a list's k-mers are counted where the lists are merged)
      if (lane == 0) atomicAdd(&S.dist[parity], dist);
      if (tid == 0) S.dist[parity ^ 1] = 0;
      __syncthreads();
      if (!next_class(cls, d0)) {
        // each bucket of the item gets what lies at its own slots (the next item adds to S.kept
        // after its first barrier)
        if (!REST && wave == 0) {
          const u32 kept = S.kept;
          if (lane < n_buckets) A.surv_cnt[item + lane] = min(max(kept, place) - place, size);
          if (lane == 0) S.kept = 0;
        }
        break;
      }
      load_records(I.ra, I.rb);
    }
    // what this item teaches: the class depth to start with, and how many k-mers fill about a
    // quarter of a table
    const u32 d = uniform(S.dist[parity]);
    parity ^= 1;
    if (!REST || chunk) learned = deepest && (d >> deepest) <= SLOTS / 4 ? deepest - 1 : deepest;
    if (merge) room = (u32)min((float)cap, (float)n * (SLOTS / 4) / (float)max(d, 1u));
    if (chunk && tid == 0) {   // (the next item adds to S.kept after its first barrier)
      A.kl_cnt[item] = S.kept;
      S.kept = 0;
    }
  };
  __syncthreads();
  u32 cur = ~0u;
  // several sets: the statistics are those of the set of bucket b from here on
  auto to_set = [&](u32 b) {
    if constexpr (MS) {
      const u32 st = A.bset[b];
      if (st == cur) return;
      if (cur != ~0u) {
        flush();
        __syncthreads();
        for (u32 i = tid; i < 256; i += T) S.hist_s[i] = 0;
        if (tid == 0) {
          S.lmax = 0;
          S.lover = 0;
          S.ndist = 0;
        }
        __syncthreads();
      }
      sink_to_set(sink, A.hist, A.tot, st);
      cur = st;
    }
  };
  if constexpr (REST) {
    const Item none{0, 0, 0, 0, 0};
    bool stats = false;
    for (u32 r = blockIdx.x; r < n_rest; r += gridDim.x) {
      Item I = none;
      if (r < n_chunks) {
        I.base = A.chunk_start[r];
        I.n = A.chunk_len[r];
        do_item(r, I, none, true, 0u, 0u);
        continue;
      }
      const u32 e = A.late[(r - n_chunks) % n_late], p = (r - n_chunks) / n_late, b = e & 0xFFFFFFu, d = e >> 24;
      if (p >> d) continue;
      const u64 c = A.bcnt[b];
      const u32 r0 = A.rec_off[b], r1 = r0 + (u32)(c >> 32), per = (r1 - r0 + W - 1) / W;
      I.base = A.kall_off[b];
      I.n = (u32)c;
      I.ra = min(r1, r0 + wave * per);
      I.rb = min(r1, I.ra + per);
      to_set(b);
      load_records(I.ra, I.rb);
      do_item(b, I, none, false, d, p);
      stats = true;
    }
    if (stats) flush();
  } else {
    const bool ranges = MS || merge;
    u32 item = b0 + (ranges ? (u32)((u64)nb * blockIdx.x / gridDim.x) : blockIdx.x);
    const u32 end = b0 + (ranges ? (u32)((u64)nb * (blockIdx.x + 1) / gridDim.x) : nb);
    Item I = look_up(load_ahead(item, end), item, end);
    load_records(I.ra, I.rb);
    Ahead ahead = load_ahead(I.after, end);
    while (item < end) {
      to_set(item);
      const Item next = look_up(ahead, I.after, end);
      ahead = load_ahead(next.after, end);
      do_item(item, I, next, false, 0u, 0u);
      item = I.after;
      I = next;
    }
    flush();
  }
}

// ---------------------------------------------------------------------------- LDS radix passes
// Key above every canonical k-mer (which uses only the low 2k bits): pads a bucket to
// whole waves.  Its digit is 0xFF in every pass, so a stable sort keeps the padding
// after all real keys and the padded lanes need no masking.
template <typename K> __device__ __forceinline__ K key_pad();
template <> __device__ __forceinline__ u64 key_pad<u64>() { return ~0ull; }
template <> __device__ __forceinline__ k128 key_pad<k128>() { return k128{~0ull, ~0ull}; }

// Lanes of a fully active wave that share digit d with this lane, as a lane mask.  Every
// lane ORs its bit into the wave's table entry of its digit and reads the entry back;
// when neighbouring lanes hold equal digits (frequent once equal keys cluster) only the
// first lane of each such run ORs the bits of the whole run, so that the LDS atomics of
// a wave do not pile up on one address.
__device__ __forceinline__ u64 digit_peers_full(u64* tbl, u32 d, u64 ge_mask) {
  const u32 lane = lane_id();
  const bool same = lane_prev(d, d ^ 1u) == d;   // lane 0 never matches
  const u64 S = __ballot(same);
  u64 bits = 1ull << lane;
  if (S != 0) {
    // run of this lane: up to (not including) the next lane that starts a run
    const u64 starts_after = ~S & (ge_mask << 1);
    bits = ((starts_after & (0ull - starts_after)) - 1ull) & ge_mask;
  }
  if (!same) atomicOr((unsigned long long*)&tbl[d], (unsigned long long)bits);
  return tbl[d];
}

// LSD radix passes [p_begin, p_end) over 8-bit digits of keys[0, n_pad) in LDS (with
// vals moving alongside when HASV).  Per pass: each item is ranked among the equal
// digits of its wave (digit_peers_full + mbcnt; the lowest lane adds the group size to
// the wave's running count); then threads 0..255 turn the counts into per-wave offsets
// -- prefix over waves within a digit, wave scan over 64 digits, and a 4-entry prefix
// over digit groups applied at the scatter.  tbl is [W][256], cnt is [2][W][256] (one
// table per pass parity), gtot has 4 entries.  With `clear` the tables are zeroed first;
// otherwise they must be as a previous call left them (tbl zero, the table of parity
// p_begin zero).  n_pad is a multiple of 64 * W.  Block-wide: barriers inside.
template <typename K, int T, int ITEMS, bool HASV, typename CntT = u32>
__device__ __forceinline__ void lds_sort_passes(K* keys, u32* vals, u64* tbl, CntT* cnt, u32* gtot, u32 n_pad,
                                                int p_begin, int p_end, bool clear) {
  constexpr int W = T / 64;
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const u64 ge = ~((1ull << lane) - 1ull);
  if (clear) {
    for (u32 i = tid; i < W * 256; i += T) {
      tbl[i] = 0;
      cnt[i] = 0;
      cnt[W * 256 + i] = 0;
    }
    __syncthreads();
  }
  const int per = (int)(n_pad / (64u * W));
  u64* wtbl = tbl + wave * 256;
  for (int p = p_begin; p < p_end; ++p) {
    CntT* C = cnt + (p & 1) * (W * 256);
    K kr[ITEMS];
    u32 vr[HASV ? ITEMS : 1];
    u32 rk[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 at = (wave * (u32)per + (u32)j) * 64u + lane;
        kr[j] = keys[at];
        if (HASV) vr[HASV ? j : 0] = vals[at];
      }
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 d = key_digit(kr[j], 8 * p);
        const u64 mask = digit_peers_full(wtbl, d, ge);
        const u32 base = C[wave * 256 + d];
        const u32 lr = mbcnt64(mask);
        if (lr == 0) {
          C[wave * 256 + d] = (CntT)(base + (u32)__popcll(mask));
          wtbl[d] = 0;
        }
        rk[j] = base + lr;
      }
    }
    __syncthreads();
    if (tid < 256) {
      // prefix over waves within digit tid, then over the 64 digits of this wave
      u32 col = 0;
#pragma unroll
      for (int v = 0; v < W; ++v) {
        const u32 x = C[v * 256 + tid];
        C[v * 256 + tid] = (CntT)col;
        col += x;
      }
      const u32 inc = wave_scan_u32(col);
      const u32 ex = inc - col;
#pragma unroll
      for (int v = 0; v < W; ++v) C[v * 256 + tid] = (CntT)(C[v * 256 + tid] + ex);
      if (lane == 63) gtot[wave] = inc;
    }
    __syncthreads();
    const u32 g1 = gtot[0], g2 = g1 + gtot[1], g3 = g2 + gtot[2];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 d = key_digit(kr[j], 8 * p);
        const u32 gb = d < 128 ? (d < 64 ? 0u : g1) : (d < 192 ? g2 : g3);
        const u32 at = C[wave * 256 + d] + gb + rk[j];
        keys[at] = kr[j];
        if (HASV) vals[at] = vr[HASV ? j : 0];
      }
    }
    // the other count table is free again: clear it for the next pass
    CntT* nxt = cnt + ((p + 1) & 1) * (W * 256);
    for (u32 i = tid; i < W * 256; i += T) nxt[i] = 0;
    __syncthreads();
  }
}

// Merging lists needs equal keys adjacent, not ascending order (the survivors of all buckets
// are sorted by key at the end).  After the LSD passes over the low `bits` bits the
// keys are ordered by those bits, so equal keys already share one group of equal low
// bits; if no two neighbours in [0, n) have equal low bits but different keys, every
// such group holds one distinct key and each key's copies are contiguous.  Otherwise the
// remaining passes complete the sort.  (Padding keys follow all real keys after any
// number of passes: their digits are all 0xFF and the sort is stable.)
__device__ __forceinline__ bool low_eq(u64 a, u64 b, int bits) { return ((a ^ b) & ((1ull << bits) - 1ull)) == 0; }
__device__ __forceinline__ bool low_eq(k128 a, k128 b, int bits) { return low_eq(a.lo, b.lo, bits); }

template <typename K>
__device__ __forceinline__ bool mixed_pair(const K* keys, u32 idx, u32 n, int bits) {
  if (idx == 0 || idx >= n) return false;
  const K a = keys[idx], b = keys[idx - 1];
  return low_eq(a, b, bits) && !key_eq(a, b);
}

// Passes that order the keys in full; keys of at most 32 bits are not mixed.
template <typename K> __device__ __forceinline__ int sort_passes(int k);
template <> __device__ __forceinline__ int sort_passes<u64>(int k) { return 2 * k <= 32 ? (2 * k + 7) / 8 : 8; }
template <> __device__ __forceinline__ int sort_passes<k128>(int k) { return (2 * k + 7) / 8; }

// ---------------------------------------------------------------------------- large buckets
// Expand the records of every large bucket into one HBM key array.  Equal k-mers share
// a bucket, so sorting that array as a whole still groups each k-mer's copies.
// Key-parallel: after the block scan of record sizes, each wave writes the keys
// of its 64 records as consecutive 64-key rows.  The wave's records and their offsets go
// to its LDS slice with a map from output position to record; each lane then takes one
// output position and computes that k-mer directly from its record's bases (funnel
// shifts, a 2-bit reversal, the smaller of the two strands), so the stores are coalesced
// and no lane waits for a longer record of its wave.  RW = record words (4: k <= 31,
// u64 keys; 8: k >= 32, 128-bit keys).
template <typename K, int T>
__global__ __launch_bounds__(T) void k_expand_large(CountArgs A, K* __restrict__ lkeys) {
  constexpr int W = T / 64, RW = sizeof(K) == 8 ? 4 : 8;
  __shared__ u64 scr[17];
  __shared__ u32 s_rec[W][64 * RW + 4];  // the wave's records (+ words read past the last one)
  __shared__ u16 s_ex[W][64];            // each record's first key, relative to the wave's first
  __shared__ u8 s_rid[W][64 * 64];       // record of each output position (g <= 64)
  const u64 n_large = A.meta[1];
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const int k = A.k;
  u32* const rec_w = s_rec[wave];
  u16* const ex_w = s_ex[wave];
  u8* const rid_w = s_rid[wave];
  if (lane < 4) rec_w[64 * RW + lane] = 0;
  for (u64 item = blockIdx.x; item < n_large; item += gridDim.x) {
    const u32 b = A.large_list[item];
    const u32 r0 = A.rec_off[b], nr = A.rec_off[b + 1] - r0;
    u64 base = A.kall_off[b];
    for (u32 c0 = 0; c0 < nr; c0 += T) {
      const u32 r = c0 + tid;
      uint4 v[RW / 4];
#pragma unroll
      for (int i = 0; i < RW / 4; ++i)
        v[i] = r < nr ? reinterpret_cast<const uint4*>(A.rec)[((u64)r0 + r) * (RW / 4) + i] : make_uint4(0u, 0u, 0u, 0u);
      const u32 g = r < nr ? (v[RW / 4 - 1].w >> 26) + 1u : 0u;
      u64 tot;
      const u64 ex = block_exclusive_scan<u64>((u64)g, scr, &tot);
      // the wave's keys are [wb, wb + G) of this round's keys
      const u64 wb = ((u64)lane_read((u32)(ex >> 32), 0) << 32) | lane_read((u32)ex, 0);
      const u32 rel = (u32)(ex - wb);
      const u32 G = lane_read(rel + g, 63);
#pragma unroll
      for (int i = 0; i < RW / 4; ++i) {
        rec_w[RW * lane + 4 * i] = v[i].x;
        rec_w[RW * lane + 4 * i + 1] = v[i].y;
        rec_w[RW * lane + 4 * i + 2] = v[i].z;
        rec_w[RW * lane + 4 * i + 3] = v[i].w;
      }
      ex_w[lane] = (u16)rel;
      for (u32 t = 0; t < g; ++t) rid_w[rel + t] = (u8)lane;
      for (u32 o0 = 0; o0 < G; o0 += 64) {
        const u32 o = o0 + lane;
        if (o < G) {
          const u32 rr = rid_w[o];
          lkeys[base + wb + o] = canon_at<K>(rec_w + RW * rr, 2u * (o - ex_w[rr]), k);
        }
      }
      base += tot;
    }
  }
}

// ---------------------------------------------------------------------------- gather
// Gather of sparse segments into one dense array: segment i holds cnt[i] entries at
// src + base[i] and lands at dst + off[i] (after *dst_base entries), off being the exclusive scan
// of cnt.  One wave per segment.
template <typename K>
__global__ __launch_bounds__(256) void k_gather_segments(const K* __restrict__ src_k, const u32* __restrict__ src_c,
                                                         const u64* __restrict__ base, const u32* __restrict__ cnt,
                                                         const u32* __restrict__ off, u64 n_seg,
                                                         K* __restrict__ dst_k, u32* __restrict__ dst_c,
                                                         const u64* __restrict__ dst_base, u64 dst_cap) {
  const u64 db = *dst_base;   // rounds: the pool's fill so far
  const u64 wave = (blockIdx.x * (u64)blockDim.x + threadIdx.x) >> 6;
  const u64 n_waves = ((u64)gridDim.x * blockDim.x) >> 6;
  const u32 lane = lane_id();
  for (u64 i = wave; i < n_seg; i += n_waves) {
    const u32 c = cnt[i];
    if (!c) continue;
    const u64 from = base[i], o = db + off[i];
    for (u32 j = lane; j < c; j += 64) {
      if (o + j < dst_cap) {
        dst_k[o + j] = src_k[from + j];
        dst_c[o + j] = src_c[from + j];
      }
    }
  }
}

// ---------------------------------------------------------------------------- several sets
// Several read sets in one count: survivors are sorted once by (set, k-mer) as 128-bit
// "wide" keys, set << 2k | k-mer (2k plus the set's bits at most 128).
__device__ __forceinline__ k128 wide_of(u64 key, u32 s, int k) {
  const int sh = 2 * k;   // < 64
  return k128{key | ((u64)s << sh), (u64)s >> (64 - sh)};
}
__device__ __forceinline__ k128 wide_of(k128 key, u32 s, int k) {
  return k128{key.lo, key.hi | ((u64)s << (2 * k - 64))};
}
__device__ __forceinline__ u32 wide_set(k128 w, int k) {
  const int sh = 2 * k;
  return sh < 64 ? (u32)((w.lo >> sh) | (w.hi << (64 - sh))) : (u32)(w.hi >> (sh - 64));
}
__device__ __forceinline__ void wide_key(k128 w, int k, u64* out) { out[0] = w.lo & ((1ull << (2 * k)) - 1ull); }
__device__ __forceinline__ void wide_key(k128 w, int k, k128* out) {
  *out = k128{w.lo, 2 * k == 64 ? 0ull : (w.hi & ((1ull << (2 * k - 64)) - 1ull))};
}

// k_gather_segments for several sets: the same segments, of set bset[i], written as wide keys.
template <typename K>
__global__ __launch_bounds__(256) void k_gather_wide(const K* __restrict__ src_k, const u32* __restrict__ src_c,
                                                     const u64* __restrict__ base, const u32* __restrict__ bset,
                                                     const u32* __restrict__ cnt, const u32* __restrict__ off,
                                                     u64 n_seg, int k, k128* __restrict__ dst_k,
                                                     u32* __restrict__ dst_c, u64 dst_cap) {
  const u64 wave = (blockIdx.x * (u64)blockDim.x + threadIdx.x) >> 6;
  const u64 n_waves = ((u64)gridDim.x * blockDim.x) >> 6;
  const u32 lane = lane_id();
  for (u64 i = wave; i < n_seg; i += n_waves) {
    const u32 c = cnt[i];
    if (!c) continue;
    const u64 from = base[i];
    const u32 st = bset[i];
    const u64 o = off[i];
    for (u32 j = lane; j < c; j += 64) {
      if (o + j < dst_cap) {
        dst_k[o + j] = wide_of(src_k[from + j], st, k);
        dst_c[o + j] = src_c[from + j];
      }
    }
  }
}

// k_gather_segments for several sets when count and set share the 32-bit value:
// value = count | set << cbits (the count is at most max_freq < 2^cbits).
template <typename K>
__global__ __launch_bounds__(256) void k_gather_packed(const K* __restrict__ src_k, const u32* __restrict__ src_c,
                                                       const u64* __restrict__ base, const u32* __restrict__ bset,
                                                       const u32* __restrict__ cnt, const u32* __restrict__ off,
                                                       u64 n_seg, int cbits, K* __restrict__ dst_k,
                                                       u32* __restrict__ dst_c, u64 dst_cap) {
  const u64 wave = (blockIdx.x * (u64)blockDim.x + threadIdx.x) >> 6;
  const u64 n_waves = ((u64)gridDim.x * blockDim.x) >> 6;
  const u32 lane = lane_id();
  for (u64 i = wave; i < n_seg; i += n_waves) {
    const u32 c = cnt[i];
    if (!c) continue;
    const u64 from = base[i];
    const u32 st = bset[i];
    const u64 o = off[i];
    for (u32 j = lane; j < c; j += 64) {
      if (o + j < dst_cap) {
        dst_k[o + j] = src_k[from + j];
        dst_c[o + j] = src_c[from + j] | (st << cbits);
      }
    }
  }
}

// Sorted wide pairs -> each set's pairs in the caller's buffers (set by set, back to
// back) and first[s] = index of set s's first pair (first[n_sets] = all pairs).
template <typename K>
__global__ __launch_bounds__(256) void k_split_wide(const k128* __restrict__ wk, const u32* __restrict__ wc,
                                                    const u64* __restrict__ n_ptr, u64 cap, int k, u32 n_sets,
                                                    K* __restrict__ out_k, u32* __restrict__ out_c,
                                                    u64* __restrict__ first) {
  const u64 n = min(*n_ptr, cap);
  if (n == 0) {
    for (u64 t = blockIdx.x * (u64)blockDim.x + threadIdx.x; t <= n_sets; t += (u64)gridDim.x * blockDim.x)
      first[t] = 0;
    return;
  }
  for (u64 i = blockIdx.x * (u64)blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
    const k128 w = wk[i];
    const u32 st = wide_set(w, k);
    wide_key(w, k, &out_k[i]);
    out_c[i] = wc[i];
    const u32 prev = i ? wide_set(wk[i - 1], k) + 1u : 0u;
    for (u32 t = prev; t <= st && t < n_sets; ++t) first[t] = i;
    if (i == n - 1)
      for (u32 t = st + 1; t <= n_sets; ++t) first[t] = n;
  }
}

// Per-set totals of a count over several sets: one block per set sums its buckets'
// records and k-mers (windows) and bucket classes; pairs from the split; n_distinct,
// overflow_sum and max_count were accumulated by the counting kernels.  Chunk and list
// figures are not split by set (0).
__global__ __launch_bounds__(256) void k_finalize_sets(DevTotals* __restrict__ tot, const u64* __restrict__ bcnt,
                                                       const u32* __restrict__ set_bbase, const u32* __restrict__ set_lb,
                                                       const u64* __restrict__ first, u32 cap_tiny, u32 cap_small,
                                                       const u32* __restrict__ flags, const u64* __restrict__ counters,
                                                       u64 rec_cap, const u64* __restrict__ surv_n, u64 surv_cap) {
  __shared__ u64 red[8][256];
  const u32 st = blockIdx.x;
  const u32 b0 = set_bbase[st], nb = 1u << set_lb[st];
  u64 q[8] = {0, 0, 0, 0, 0, 0, 0, 0};   // records, windows, tiny b, tiny k, small b, small k, large b, large k
  for (u32 i = threadIdx.x; i < nb; i += blockDim.x) {
    const u64 c = bcnt[b0 + i];
    const u64 nk = (u32)c, nr = c >> 32;
    q[0] += nr;
    q[1] += nk;
    if (nk == 0) continue;
    const int cl = nk > cap_small ? 3 : nk > cap_tiny ? 2 : 1;
    q[2 * cl] += 1;
    q[2 * cl + 1] += nk;
  }
  for (int j = 0; j < 8; ++j) red[j][threadIdx.x] = q[j];
  __syncthreads();
  for (u32 w = 128; w > 0; w >>= 1) {
    if (threadIdx.x < w)
      for (int j = 0; j < 8; ++j) red[j][threadIdx.x] += red[j][threadIdx.x + w];
    __syncthreads();
  }
  if (threadIdx.x == 0) {
    DevTotals* t = tot + st;
    t->n_records = red[0][0];
    t->n_windows = red[1][0];
    t->tiny_buckets = red[2][0];
    t->tiny_kmers = red[3][0];
    t->small_buckets = red[4][0];
    t->small_kmers = red[5][0];
    t->large_buckets = red[6][0];
    t->large_keys = red[7][0];
    t->n_pairs = first[st + 1] - first[st];
    t->buckets = nb;
    t->chunks = 0;
    t->list_entries = 0;
    t->n_occ = 0;
    u64 f = *flags & 1u;
    if (counters[0] > rec_cap) f |= 2u;
    if (*surv_n > surv_cap) f |= 4u;   // survivors beyond the sort's capacity
    t->flags = f;
  }
}

// ---------------------------------------------------------------------------- output
template <typename K>
__global__ __launch_bounds__(256) void k_copy_pairs(const K* __restrict__ sk, const u32* __restrict__ sc,
                                                    const u64* __restrict__ n_ptr, u64 cap, K* __restrict__ ok,
                                                    u32* __restrict__ oc) {
  const u64 n = min(*n_ptr, cap);
  for (u64 i = blockIdx.x * (u64)blockDim.x + threadIdx.x; i < n; i += (u64)gridDim.x * blockDim.x) {
    ok[i] = sk[i];
    oc[i] = sc[i];
  }
}

// Memory-bounded counting: after each round its figures join the running totals
// (acc: windows, records, large k-mers, tiny buckets, tiny k-mers, small buckets, small
// k-mers, large buckets, chunks, list entries) and its survivors, gathered behind the
// previous rounds' in the pool, advance the pool's fill.  Flag bit 1: a round's records
// overflowed; bit 4: the survivors outgrew the pool.
__global__ void k_round_end(const u64* counters, const u64* meta, const u64* surv_n, const u64* kl_n, u64 rec_cap,
                            u64* acc, u64* pool_n, u64 pool_cap, u32* flags) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  acc[0] += meta[2] + meta[6] + meta[7];
  acc[1] += counters[0];
  acc[2] += meta[2];
  acc[3] += meta[5];
  acc[4] += meta[6];
  acc[5] += meta[0];
  acc[6] += meta[7];
  acc[7] += meta[1];
  acc[8] += meta[4];
  acc[9] += *kl_n;
  if (counters[0] > rec_cap) *flags |= 2u;
  *pool_n += *surv_n;
  if (*pool_n > pool_cap) *flags |= 16u;
}

// *out = min(*in, cap).
__global__ void k_clamp_u64(const u64* in, u64 cap, u64* out) {
  if (threadIdx.x == 0 && blockIdx.x == 0) *out = min(*in, cap);
}

// Totals of a count in rounds, from the running totals.
__global__ void k_finalize_rounds(DevTotals* tot, const u64* acc, const u64* pool_n, const u32* flags, u32 B) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  tot->n_windows = acc[0];
  tot->n_records = acc[1];
  tot->n_pairs = *pool_n;
  tot->flags = *flags;
  tot->large_keys = acc[2];
  tot->tiny_buckets = acc[3];
  tot->tiny_kmers = acc[4];
  tot->small_buckets = acc[5];
  tot->small_kmers = acc[6];
  tot->large_buckets = acc[7];
  tot->chunks = acc[8];
  tot->list_entries = acc[9];
  tot->buckets = B;
}

// Totals of a count, with the bucket-plan figures (meta: small, large, large k-mers,
// records, chunks, tiny, tiny k-mers, small k-mers).
__global__ void k_finalize(DevTotals* tot, const u64* counters, const u64* surv_n, u64 rec_cap, u64 surv_cap,
                           const u32* flags, const u64* meta, const u64* kl_n, u32 B) {
  if (threadIdx.x != 0 || blockIdx.x != 0) return;
  tot->n_windows = meta[2] + meta[6] + meta[7];   // every valid window is in one record
  tot->n_records = counters[0];
  tot->n_pairs = *surv_n;
  u64 f = *flags & 1u;
  if (counters[0] > rec_cap) f |= 2u;
  if (*surv_n > surv_cap) f |= 4u;
  tot->flags = f;
  tot->large_keys = meta[2];
  tot->tiny_buckets = meta[5];
  tot->tiny_kmers = meta[6];
  tot->small_buckets = meta[0];
  tot->small_kmers = meta[7];
  tot->large_buckets = meta[1];
  tot->chunks = meta[4];
  tot->list_entries = *kl_n;
  tot->buckets = B;
}
