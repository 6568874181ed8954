// Segmented sorts of (key, value) pairs, used where a stage needs keys in order but the
// keys already fall into independent segments:
//   * the (k-mer, count) lists of one heavy bucket (Section 3.5: lists are sorted and
//     merged again) -- equal k-mers never span two buckets, so each bucket's lists are
//     sorted on their own and summed per run;
//   * the survivors, split by their top key bits into key ranges (two scatter passes),
//     each range then sorted on its own -- ascending order of the whole output.
// A segment that fits on chip is sorted there in one read and one write, by one digit of about
// log2(length) bits and a ranking inside the digit's bin: keys of a segment spread over the
// bins, so a bin holds one or two keys and each key's rank is its bin's start plus the smaller
// keys of its bin.  Where a bin holds more than SEG_BIN_MAX (keys that share their leading 32 bits:
// reads with a primer or an insert in common), a block sorts the segment by LSD passes in LDS.  A
// longer segment is sorted by its block through HBM (stable LSD passes over LDS tiles).
#pragma once
#include "kc_common.hpp"
#include "kc_count.hpp"

// Bits [sh, sh + nb) of a key, nb <= 16 (may straddle the words of a 128-bit key).
__device__ __forceinline__ u32 key_field(u64 k, int sh, int nb) {
  return nb ? (u32)(k >> sh) & ((1u << nb) - 1u) : 0u;
}
__device__ __forceinline__ u32 key_field(k128 k, int sh, int nb) {
  if (!nb) return 0u;
  u64 v;
  if (sh >= 64) v = k.hi >> (sh - 64);
  else if (sh == 0) v = k.lo;
  else v = (k.lo >> sh) | (k.hi << (64 - sh));
  return (u32)v & ((1u << nb) - 1u);
}

constexpr u32 MSD_NB = 1024;   // blocks of the coarse pass at most

// The leading 32 bits of a key of nbits bits (fewer bits: moved up).
__host__ __device__ __forceinline__ u32 key_top32(u64 k, int nbits) {
  return nbits >= 32 ? (u32)(k >> (nbits - 32)) : (u32)k << (32 - nbits);
}
// (wide keys, set << 2k | k-mer, may have as few bits as a set and a base)
__host__ __device__ __forceinline__ u32 key_top32(k128 k, int nbits) {
  const int sh = nbits - 32;
  if (sh < 0) return (u32)k.lo << -sh;
  if (sh <= 32) return (u32)(k.lo >> sh);
  return sh >= 64 ? (u32)(k.hi >> (sh - 64)) : (u32)(k.lo >> sh) | (u32)(k.hi << (64 - sh));
}
// Where a key falls among all keys, as a 32-bit fraction that never decreases with the key.
// Canonical k-mers are the smaller of two strands, so their density falls linearly from twice
// the mean to nothing and the share of keys below x is 1 - (1 - x)^2: that spreads them
// evenly over ranges and bins (split by their leading bits the first ranges hold twice the
// mean, which a third of the blocks then waits for).  Wide keys start with the set: as they are.
template <typename K>
__host__ __device__ __forceinline__ u32 key_place(K k, int nbits, int canonical) {
  const u32 t = key_top32(k, nbits);
  return canonical ? ~(u32)(((u64)~t * ~t) >> 32) : t;
}

// Survivors where the count left them: bucket i's s_cnt[i] from its first k-mer slot s_base[i] of
// (s_k, s_c) on, at most as many as it has slots (see plan_meta for `meta`).
struct SurvSegs {
  const void* s_k;
  const u32* s_c;
  const u64* s_base;
  const u32* s_cnt;
  u32 n_buckets;
  const u64* meta;
};
struct MsdArgs {
  const void* in_k;        // dense survivors ...
  const u32* in_v;
  SurvSegs sv;             // ... or as the count left them
  const u64* n_ptr;        // survivors
  void* mid_k;             // grouped by the top 8 bits of their places
  u32* mid_v;
  void* out_k;             // grouped by the top 8 + g2 bits
  u32* out_v;
  u32* hist;               // [256][nb] counts -> offsets
  u32 nb;                  // blocks of the coarse pass (<= MSD_NB)
  u64* seg;                // [(256 << g2) + 1] range starts
  u64* n_seg;              // ranges
  int nbits;               // key bits (2k)
  int canonical;           // see key_place
  u32 target;              // keys per range wanted
};

// Fine field width: the fewest bits that bring a range to `target` keys on average.
constexpr int MSD_G2_MAX = 10;
__host__ __device__ __forceinline__ int msd_g2(u64 n, u32 target) {
  int g2 = 0;
  while (g2 < MSD_G2_MAX && (n >> (8 + g2)) > (u64)target) ++g2;
  return g2;
}

struct SegArgs {
  void* keys;              // input pairs; also the first ping-pong buffer of long segments
  u32* vals;
  void* tmp_k;             // second ping-pong buffer (same positions)
  u32* tmp_v;
  void* out_k;             // sorted output (may equal keys); positions >= out_cap are dropped
  u32* out_v;
  u64 out_cap;
  u64* seg;                // segment i = [seg[i], seg[i + 1]); SEG_CROWDED: left to k_seg_sort
  const u64* n_seg_ptr;    // number of segments
  int nbits;               // key bits (2k)
  int canonical;           // see key_place
  const u64* msd_n;        // when set: segments are key ranges of k_msd_fine over *msd_n keys
  u32 msd_target;
  u32 wave_cap;            // segments of at most this many pairs are left to k_seg_wave
};

// A ranking compares each key with its whole bin.  60,000 reads of 150 bases with one of 20 inserts of
// 100 bases (795,000 k-mers of 31 bases, 500 and more of which share 16): 4.26 ms for the output of
// all k-mers where any bin is ranked, 0.44 by LSD passes in LDS alone, 0.68 with this limit.
constexpr u32 SEG_BIN_MAX = 64;
constexpr u64 SEG_CROWDED = 1ull << 63;   // set in a segment's start by k_seg_wave
__device__ __forceinline__ u64 seg_start(const SegArgs& A, u64 i) { return A.seg[i] & ~SEG_CROWDED; }

// Bits of the keys' places that a segment's keys share: those of its range.
__device__ __forceinline__ int seg_place_bits(const SegArgs& A) {
  return A.msd_n ? 8 + msd_g2(*A.msd_n, A.msd_target) : 0;
}

// Bins of a segment of m keys: a power of two of at least m and 64.
__device__ __forceinline__ int seg_bin_bits(u32 m) { return max(6, 32 - __builtin_clz((m - 1) | 1)); }
// The bin of a key: the bits of its place below its segment's.
template <typename K>
__device__ __forceinline__ u32 seg_bin(const SegArgs& A, K key, int pbits, int db) {
  return (key_place(key, A.nbits, A.canonical) << pbits) >> (32 - db);
}
// Keys of the bin [b0, b1) that come before the key at slot `at` (equal keys by their slot).
template <typename K>
__device__ __forceinline__ u32 seg_rank(const K* keys, K key, u32 at, u32 b0, u32 b1) {
  u32 r = b0;
  if (b1 - b0 > 1)
    for (u32 i = b0; i < b1; ++i) {
      const K x = keys[i];
      r += (key_lt(x, key) || (key_eq(x, key) && i < at)) ? 1u : 0u;
    }
  return r;
}

template <typename K, int T, int ITEMS>
struct SegSmem {
  static constexpr int W = T / 64, CAP = T * ITEMS;
  K keys[CAP];
  union {
    u32 bins[CAP + 4];                // counts, then first slots; [bins] = keys
    u32 vals[CAP];
  } b;
  // long segments
  u64 tbl[W * 256];
  u32 cnt[2 * W * 256];
  u32 gtot[4];
  u32 dcnt[256], dstart[256], drun[256];
  u64 scr[17];
  u16 lng[T];                         // the long ones among T segments
  u32 n_long;
};

// The block's m pairs (kr, vr; thread t holds pairs t, t + T, ...) sorted into S.keys and
// S.b.vals by bin(key), below 2^db, then by key.  db: 2^db of at least T and m.  With CHECK false,
// and nothing done, where a bin holds more than SEG_BIN_MAX.
template <int T, int ITEMS, bool CHECK, typename K, typename SM, typename Bin>
__device__ __forceinline__ bool seg_sort_chip(SM& S, u32 m, int db, const K (&kr)[ITEMS], const u32 (&vr)[ITEMS], Bin bin) {
  const u32 tid = threadIdx.x, per = (1u << db) / T;   // bins per thread
  for (u32 i = tid; i < 1u << db; i += T) S.b.bins[i] = 0;
  __syncthreads();
  u32 rk[ITEMS];
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (tid + (u32)j * T < m) rk[j] = atomicAdd(&S.b.bins[bin(kr[j])], 1u);
  __syncthreads();
  u32 most = 0;
  {
    u64 sum = 0, tot;
    for (u32 q = 0; q < per; ++q) sum += S.b.bins[tid * per + q];
    u32 run = (u32)block_exclusive_scan<u64>(sum, S.scr, &tot);
    for (u32 q = 0; q < per; ++q) {
      const u32 c = S.b.bins[tid * per + q];
      S.b.bins[tid * per + q] = run;
      run += c;
      if constexpr (CHECK) most = max(most, c);
    }
    if (tid == 0) S.b.bins[1u << db] = m;
  }
  if constexpr (CHECK) {
    if (__syncthreads_or(most > SEG_BIN_MAX)) return false;
  } else {
    __syncthreads();
  }
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (tid + (u32)j * T < m) {
      rk[j] += S.b.bins[bin(kr[j])];
      S.keys[rk[j]] = kr[j];
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (tid + (u32)j * T < m) {
      const u32 d = bin(kr[j]);
      rk[j] = seg_rank(S.keys, kr[j], rk[j], S.b.bins[d], S.b.bins[d + 1]);
    }
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j)
    if (tid + (u32)j * T < m) {
      S.keys[rk[j]] = kr[j];
      S.b.vals[rk[j]] = vr[j];
    }
  __syncthreads();
  return true;
}

// A segment [s0, s0 + n) longer than a block holds: stable LSD passes through HBM, ping-pong
// between src and dst (which end with the sorted pairs in src).  With `mixed` (keys of more than
// 32 bits), where equal keys
// need only be adjacent, the keys are mixed as they are first read, the low 8 * p0 bits are
// sorted first (p0 from the length, so that two distinct keys share those bits with a chance of
// about 1%), and the remaining passes run only if some group of equal low bits holds two keys;
// the keys stay mixed.
template <int T, int ITEMS, typename K, typename SM>
__device__ __forceinline__ void seg_sort_long(SM& S, K*& src_k, u32*& src_v, K*& dst_k, u32*& dst_v, u64 s0, u64 n,
                                              int nbits, bool mixed) {
  constexpr u32 CAP = SM::CAP, WB = 64u * (T / 64);
  const u32 tid = threadIdx.x;
  auto ld = [&](const K* src, u64 i, int p) { return (mixed && p == 0) ? mix_key(src[i]) : src[i]; };
  auto pass = [&](int p) {
    for (u32 d = tid; d < 256; d += T) S.dcnt[d] = 0;
    __syncthreads();
    for (u64 i = tid; i < n; i += T) atomicAdd(&S.dcnt[key_digit(ld(src_k, s0 + i, p), 8 * p)], 1u);
    __syncthreads();
    {
      u64 tot;
      const u64 v = tid < 256 ? (u64)S.dcnt[tid] : 0ull;
      const u64 ex = block_exclusive_scan<u64>(v, S.scr, &tot);
      if (tid < 256) S.drun[tid] = (u32)ex;
    }
    __syncthreads();
    for (u64 t0 = 0; t0 < n; t0 += CAP) {
      const u32 m = (u32)min((u64)CAP, n - t0), m_pad = (m + WB - 1) / WB * WB;
      for (u32 i = tid; i < m_pad; i += T) {
        S.keys[i] = i < m ? ld(src_k, s0 + t0 + i, p) : key_pad<K>();
        S.b.vals[i] = i < m ? src_v[s0 + t0 + i] : 0u;
      }
      for (u32 d = tid; d < 256; d += T) S.dcnt[d] = 0;
      __syncthreads();
      // one stable pass on digit p orders the tile by that digit (padding last)
      lds_sort_passes<K, T, ITEMS, true>(S.keys, S.b.vals, S.tbl, S.cnt, S.gtot, m_pad, p, p + 1, true);
      for (u32 i = tid; i < m; i += T) {
        const u32 d = key_digit(S.keys[i], 8 * p);
        if (i == 0 || key_digit(S.keys[i - 1], 8 * p) != d) S.dstart[d] = i;
        atomicAdd(&S.dcnt[d], 1u);
      }
      __syncthreads();
      for (u32 i = tid; i < m; i += T) {
        const u32 d = key_digit(S.keys[i], 8 * p);
        const u64 at = s0 + S.drun[d] + (i - S.dstart[d]);
        dst_k[at] = S.keys[i];
        dst_v[at] = S.b.vals[i];
      }
      __syncthreads();
      for (u32 d = tid; d < 256; d += T) S.drun[d] += S.dcnt[d];
      __syncthreads();
    }
    K* tk = src_k;
    src_k = dst_k;
    dst_k = tk;
    u32* tv = src_v;
    src_v = dst_v;
    dst_v = tv;
  };
  const int np = mixed ? sort_passes<K>(nbits / 2) : (nbits + 7) / 8;
  // 8 * p0 >= 2 log2(n) + 7 bits (one pass loop, so that the pass is inlined once)
  int p_end = mixed ? min((2 * (64 - __builtin_clzll(n)) + 14) / 8, np) : np;
  bool checked = !mixed;
  for (int p = 0;;) {
    const int p0 = p_end;
    for (; p < p_end; ++p) pass(p);
    if (checked) break;
    checked = true;
    bool bad = false;
    for (u64 i = tid; i < n; i += T) bad |= mixed_pair(src_k + s0, (u32)i, (u32)n, 8 * p0);
    if (!__syncthreads_or(bad)) break;
    p_end = np;
  }
}

// (128-bit keys: LDS holds two blocks per CU, so the registers have to)
template <typename K, int T, int ITEMS>
__global__ __launch_bounds__(T, sizeof(K) == 16 ? 4 : 2) void k_seg_sort(SegArgs A) {
  using SM = SegSmem<K, T, ITEMS>;
  constexpr u32 CAP = SM::CAP;
  __shared__ SM S;
  const u32 tid = threadIdx.x;
  const u64 n_seg = *A.n_seg_ptr;
  const int pbits = seg_place_bits(A);
  K* in_k = reinterpret_cast<K*>(A.keys);
  K* tmp_k = reinterpret_cast<K*>(A.tmp_k);
  K* out_k = reinterpret_cast<K*>(A.out_k);
  // the block's segments (block, + grid, ...) are looked through T at a time: most are short
  for (u64 c0 = blockIdx.x; c0 < n_seg; c0 += (u64)gridDim.x * T) {
   __syncthreads();
   if (tid == 0) S.n_long = 0;
   __syncthreads();
   {
    const u64 sgi = c0 + (u64)tid * gridDim.x;
    if (sgi < n_seg && (A.seg[sgi] >= SEG_CROWDED || seg_start(A, sgi + 1) > seg_start(A, sgi) + A.wave_cap))
      S.lng[atomicAdd(&S.n_long, 1u)] = (u16)tid;
   }
   __syncthreads();
   const u32 n_long = S.n_long;
   // those that a block holds, where their bins allow it; the others stay in the list (in two loops:
   // in one the registers of both would halve the blocks per CU)
   u32 rest = 0;
   for (u32 li = 0; li < n_long; ++li) {
    const u32 at = S.lng[li];
    const u64 sgi = c0 + (u64)at * gridDim.x;
    const u64 s0 = seg_start(A, sgi), n = seg_start(A, sgi + 1) - s0;
    __syncthreads();                             // LDS of the previous segment is free
    bool done = false;
    if (n <= CAP && A.seg[sgi] < SEG_CROWDED) {
      const u32 m = (u32)n;
      const int db = max(__builtin_ctz(T), seg_bin_bits(m));
      K kr[ITEMS];
      u32 vr[ITEMS];
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        const u32 i = tid + (u32)j * T;
        kr[j] = i < m ? in_k[s0 + i] : key_zero<K>();
        vr[j] = i < m ? A.vals[s0 + i] : 0u;
      }
      done = seg_sort_chip<T, ITEMS, true>(S, m, db, kr, vr, [&](K k) { return seg_bin(A, k, pbits, db); });
      for (u32 i = tid; done && i < m; i += T) {
        if (s0 + i < A.out_cap) {
          out_k[s0 + i] = S.keys[i];
          A.out_v[s0 + i] = S.b.vals[i];
        }
      }
    }
    if (!done) {
      if (tid == 0) S.lng[rest] = (u16)at;
      ++rest;
    }
   }
   for (u32 li = 0; li < rest; ++li) {
    __syncthreads();
    const u64 sgi = c0 + (u64)S.lng[li] * gridDim.x;
    const u64 s0 = seg_start(A, sgi), n = seg_start(A, sgi + 1) - s0;
    if (n <= CAP) {
      constexpr u32 WB = 64u * (T / 64);
      const u32 m = (u32)n, m_pad = (m + WB - 1) / WB * WB;
      for (u32 i = tid; i < m_pad; i += T) {
        S.keys[i] = i < m ? in_k[s0 + i] : key_pad<K>();
        S.b.vals[i] = i < m ? A.vals[s0 + i] : 0u;
      }
      __syncthreads();
      lds_sort_passes<K, T, ITEMS, true>(S.keys, S.b.vals, S.tbl, S.cnt, S.gtot, m_pad, 0, (A.nbits + 7) / 8, true);
      for (u32 i = tid; i < m; i += T) {
        if (s0 + i < A.out_cap) {
          out_k[s0 + i] = S.keys[i];
          A.out_v[s0 + i] = S.b.vals[i];
        }
      }
      continue;
    }
    K *src_k = in_k, *dst_k = tmp_k;
    u32 *src_v = A.vals, *dst_v = A.tmp_v;
    seg_sort_long<T, ITEMS>(S, src_k, src_v, dst_k, dst_v, s0, n, A.nbits, false);
    if (src_k != out_k) {
      for (u64 i = tid; i < n; i += T)
        if (s0 + i < A.out_cap) out_k[s0 + i] = src_k[s0 + i];
    }
    if (src_v != A.out_v) {
      for (u64 i = tid; i < n; i += T)
        if (s0 + i < A.out_cap) A.out_v[s0 + i] = src_v[s0 + i];
    }
   }
  }
}

// ---------------------------------------------------------------------------- heavy buckets
// A large bucket's chunks left (k-mer, count) lists with distinct k-mers each; one block brings a
// bucket's lists together, sorts them so that equal k-mers adjoin, adds up each run's counts and
// leaves the bucket's survivors, like any other's, at its k-mer slots.  (The steps by kernels of
// their own, over all buckets' lists at once, were seven launches, which most counts made for
// nothing: a count of 240 kbp took 188 us with them, 166 without.)
struct MergeArgs {
  CountArgs c;
  const u32* ch0;          // first chunk of each large bucket
  u64 chunk_cap;
  void *k0, *k1;           // two buffers for lists that a block does not hold, at the k-mer slots
  u32 *v0, *v1;
  u64* n_entries;          // list entries, added up
};

template <typename K, int T, int ITEMS, bool MS>
__global__ __launch_bounds__(T) void k_merge_lists(MergeArgs M) {
  using SM = SegSmem<K, T, ITEMS>;
  constexpr u32 CAP = SM::CAP;
  __shared__ SM S;
  __shared__ u32 hist_s[256], lmax, cursor, kept;
  __shared__ unsigned long long lover, nd;
  const CountArgs& A = M.c;
  const u32 tid = threadIdx.x, lane = lane_id(), wave = uniform(tid >> 6);
  const u64 n_large = A.meta[1], n_chunks = min(A.meta[4], M.chunk_cap);
  if (blockIdx.x >= n_large) return;
  auto clear_stats = [&]() {
    for (u32 i = tid; i < 256; i += T) hist_s[i] = 0;
    if (tid == 0) {
      lmax = 0;
      lover = 0;
      nd = 0;
      kept = 0;
    }
  };
  clear_stats();
  RunSink sink{hist_s, A.hist_len, A.hist, A.tot, &lmax, &lover};
  const K* lists_k = reinterpret_cast<const K*>(A.kl_k);
  const bool mixed = 2 * A.k > 32;
  u64 entries = 0;
  u32 cur = ~0u;
  for (u64 b = blockIdx.x; b < n_large; b += gridDim.x) {
    const u32 bucket = A.large_list[b];
    const u64 base = A.kall_off[bucket];
    const u64 c0 = min((u64)M.ch0[b], n_chunks), c1 = b + 1 < n_large ? min((u64)M.ch0[b + 1], n_chunks) : n_chunks;
    __syncthreads();                             // (the previous bucket is done with LDS)
    if constexpr (MS) {
      const u32 st = A.bset[bucket];
      if (st != cur) {
        if (cur != ~0u) {
          flush_stats(sink, nd);
          __syncthreads();
          clear_stats();
        }
        sink_to_set(sink, A.hist, A.tot, st);
        cur = st;
      }
    }
    if (tid == 0) cursor = 0;
    u64 n;
    {
      u64 sum = 0;
      for (u64 c = c0 + tid; c < c1; c += T) sum += A.kl_cnt[c];
      block_exclusive_scan<u64>(sum, S.scr, &n);
    }
    entries += n;
    // the lists into LDS or the first buffer, 64 chunks per wave at a time: short ones one per
    // lane, others one after the other
    const bool chip = n <= CAP;
    K* src_k = reinterpret_cast<K*>(M.k0);
    u32* src_v = M.v0;
    auto bring = [&](auto put) {
      for (u64 g = c0 + wave * 64; g < c1; g += T) {
        const u32 cnt = g + lane < c1 ? A.kl_cnt[g + lane] : 0u;
        const u64 from = g + lane < c1 ? A.chunk_start[g + lane] : 0ull;
        const u32 inc = wave_scan_u32(cnt);
        u32 at = 0;
        if (lane == 63) at = atomicAdd(&cursor, inc);
        at = lane_read(at, 63) + inc - cnt;
        if (!__ballot(cnt > 8)) {
          for (u32 j = 0; j < cnt; ++j) put(at + j, from + j);
        } else {
          for (u64 left = __ballot(cnt != 0); left; left &= left - 1) {
            const int l = __builtin_ctzll(left);
            const u32 cl = lane_read(cnt, l), al = lane_read(at, l);
            const u64 fl = ((u64)lane_read((u32)(from >> 32), l) << 32) | lane_read((u32)from, l);
            for (u32 j = lane; j < cl; j += 64) put(al + j, fl + j);
          }
        }
      }
    };
    if (chip)
      bring([&](u32 at, u64 from) {
        S.keys[at] = lists_k[from];
        S.b.vals[at] = A.kl_c[from];
      });
    else
      bring([&](u32 at, u64 from) {
        src_k[base + at] = lists_k[from];
        src_v[base + at] = A.kl_c[from];
      });
    __syncthreads();
    // equal k-mers together
    if (chip) {
      const u32 m = (u32)n;
      const int db = max(__builtin_ctz(T), seg_bin_bits(m));
      K kr[ITEMS];
      u32 vr[ITEMS];
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        const u32 i = tid + (u32)j * T;
        kr[j] = i < m ? S.keys[i] : key_zero<K>();
        vr[j] = i < m ? S.b.vals[i] : 0u;
      }
      __syncthreads();
      // (bins of mixed keys: a crowded one holds copies of one k-mer, from that many chunks)
      seg_sort_chip<T, ITEMS, false>(S, m, db, kr, vr, [&](K k) { return key_field(mix_key(k), 0, db); });
    } else {
      K* dst_k = reinterpret_cast<K*>(M.k1);
      u32* dst_v = M.v1;
      seg_sort_long<T, ITEMS>(S, src_k, src_v, dst_k, dst_v, base, n, 2 * A.k, mixed);
    }
    // Runs, a block's hold of entries at a time (up to the last run that may go on behind it): the
    // thread of a run's first entry adds up its counts.
    K* const out_k = reinterpret_cast<K*>(A.surv_k) + base;
    u32* const out_c = A.surv_c + base;
    u32 distinct = 0;
    auto report = [&](K key, u64 c, bool head) {
      run_stats_lanes(sink, c, head);
      distinct += (u32)__popcll(__ballot(head));
      const bool emit = head && c >= A.min_freq && c <= A.max_freq;
      const u64 em = __ballot(emit);
      if (!em) return;
      u32 at = 0;
      if (lane == 0) at = atomicAdd(&kept, (u32)__popcll(em));
      at = lane_read(at, 0) + mbcnt64(em);
      if (emit) {
        out_k[at] = chip || !mixed ? key : unmix_key(key);
        out_c[at] = (u32)c;
      }
    };
    for (u64 t0 = 0; t0 < n;) {
      const u32 m = (u32)min((u64)CAP, n - t0);
      if (!chip) {
        __syncthreads();
        for (u32 i = tid; i < m; i += T) {
          S.keys[i] = src_k[base + t0 + i];
          S.b.vals[i] = src_v[base + t0 + i];
        }
        if (tid == 0) cursor = 0;
        __syncthreads();
      }
      u32 last = m;
      if (t0 + m < n) {
        u32 h = 0;
        for (u32 i = tid; i < m; i += T)
          if (i && !key_eq(S.keys[i], S.keys[i - 1])) h = i;
        if (h) atomicMax(&cursor, h);
        __syncthreads();
        last = cursor;
      }
      if (last == 0) {   // one run, all of it and more
        const K key = S.keys[0];
        u64 sum = 0, c, pos = t0;
        for (;;) {
          const u64 i = pos + tid;
          const bool on = i < n && key_eq(src_k[base + i], key);
          sum += on ? src_v[base + i] : 0u;
          const u32 got = (u32)__syncthreads_count(on);
          pos += got;
          if (got < T) break;
        }
        block_exclusive_scan<u64>(sum, S.scr, &c);
        report(key, c, tid == 0);
        t0 = pos;
        continue;
      }
      for (u32 r0 = 0; r0 < last; r0 += T) {
        const u32 i = r0 + tid;
        const K key = S.keys[min(i, last - 1)];
        const bool head = i < last && (i == 0 || !key_eq(key, S.keys[i - 1]));
        u64 c = 0;
        if (head)
          for (u32 j = i; j < last && key_eq(S.keys[j], key); ++j) c += S.b.vals[j];
        report(key, c, head);
      }
      t0 += last;
    }
    if (lane == 0 && distinct) atomicAdd(&nd, (unsigned long long)distinct);
    __syncthreads();
    if (tid == 0) {
      A.surv_cnt[bucket] = kept;
      kept = 0;
    }
  }
  __syncthreads();
  flush_stats(sink, nd);
  if (tid == 0) atomicAdd((unsigned long long*)M.n_entries, (unsigned long long)entries);
}

// ---------------------------------------------------------------------------- short segments
// Segments of at most WCAP pairs are sorted by one wave each in its own slice of LDS, with no
// block barriers (the waves of a block are independent).  Bound by LDS round trips: per pair
// one counter, one staged key, the one or two keys of its bin and the output staging, against
// nine operations in each of the 5 to 12 LSD passes it replaces.
// Measured, survivors' segment sorts (all kernels): 43 M u64 pairs 1.24 -> 0.46 ms, 18.6 M 128-bit
// pairs 1.25 -> 0.35 ms; with LSD passes the longer half of the ranges (split by leading bits)
// also went to k_seg_sort.
template <typename K, int WCAP>
struct SegWaveSmem {
  static constexpr int BINS = WCAP <= 512 ? 512 : 1024;
  static_assert(WCAP <= 1024, "bins");
  K keys[WCAP];
  union {
    u32 bins[BINS + 4];               // counts, then first slots; [bins] = keys
    u32 vals[WCAP];
  } b;
};

// Waves take segments in turn (segment = global wave index, + all waves of the grid, ...);
// a segment longer than WCAP, or with a crowded bin, is left to k_seg_sort.
template <typename K, int WCAP, int WPB>
__global__ __launch_bounds__(WPB * 64) void k_seg_wave(SegArgs A) {
  constexpr int ITEMS = WCAP / 64;
  __shared__ SegWaveSmem<K, WCAP> WS[WPB];
  const u32 lane = lane_id(), wave = uniform(threadIdx.x >> 6);
  SegWaveSmem<K, WCAP>& S = WS[wave];
  const u64 n_seg = *A.n_seg_ptr;
  const int pbits = seg_place_bits(A);
  const K* in_k = reinterpret_cast<const K*>(A.keys);
  K* out_k = reinterpret_cast<K*>(A.out_k);
  for (u64 sgi = (u64)blockIdx.x * WPB + wave; sgi < n_seg; sgi += (u64)gridDim.x * WPB) {
    const u64 s0 = uniform(seg_start(A, sgi)), s1 = uniform(seg_start(A, sgi + 1));
    if (s1 <= s0 || s1 - s0 > WCAP) continue;    // uniform over the wave
    const u32 m = (u32)(s1 - s0), rows = (m + 63) / 64;
    const int db = seg_bin_bits(m);
    const u32 per = (1u << db) / 64;             // bins per lane, a power of two
    K kr[ITEMS];
    u32 vr[ITEMS], rk[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      const u32 i = (u32)j * 64 + lane;
      if ((u32)j < rows && i < m) {
        kr[j] = in_k[s0 + i];
        vr[j] = A.vals[s0 + i];
      }
    }
    for (u32 q = 0; q < per; ++q) S.b.bins[q * 64 + lane] = 0;
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
      if ((u32)j < rows && (u32)j * 64 + lane < m) rk[j] = atomicAdd(&S.b.bins[seg_bin(A, kr[j], pbits, db)], 1u);
    __builtin_amdgcn_wave_barrier();
    u32 most = 0;
    {
      u32 sum = 0;
      for (u32 q = 0; q < per; ++q) sum += S.b.bins[lane * per + q];
      u32 run = wave_scan_u32(sum) - sum;
      for (u32 q = 0; q < per; ++q) {
        const u32 c = S.b.bins[lane * per + q];
        S.b.bins[lane * per + q] = run;
        run += c;
        most = max(most, c);
      }
      if (lane == 0) S.b.bins[1u << db] = m;
    }
    __builtin_amdgcn_wave_barrier();
    if (__any(most > SEG_BIN_MAX)) {             // (uniform; other waves may read the start just now)
      if (lane == 0) atomicOr((unsigned long long*)&A.seg[sgi], (unsigned long long)SEG_CROWDED);
      continue;
    }
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
      if ((u32)j < rows && (u32)j * 64 + lane < m) {
        rk[j] += S.b.bins[seg_bin(A, kr[j], pbits, db)];
        S.keys[rk[j]] = kr[j];
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
      if ((u32)j < rows && (u32)j * 64 + lane < m) {
        const u32 d = seg_bin(A, kr[j], pbits, db);
        rk[j] = seg_rank(S.keys, kr[j], rk[j], S.b.bins[d], S.b.bins[d + 1]);
      }
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int j = 0; j < ITEMS; ++j)
      if ((u32)j < rows && (u32)j * 64 + lane < m) {
        S.keys[rk[j]] = kr[j];
        S.b.vals[rk[j]] = vr[j];
      }
    __builtin_amdgcn_wave_barrier();
    for (u32 i = lane; i < m; i += 64) {
      if (s0 + i < A.out_cap) {
        out_k[s0 + i] = S.keys[i];
        A.out_v[s0 + i] = S.b.vals[i];
      }
    }
    __builtin_amdgcn_wave_barrier();
  }
}

// ---------------------------------------------------------------------------- key ranges
// The survivors are split into key ranges by their top bits: a coarse pass on the top 8
// bits (per-block LDS histograms, one scan, a scatter staged through LDS) and a fine
// pass, one block per coarse group, on the next g2 bits, g2 chosen from the survivor
// count so that a range averages at most `target` keys.  The fine pass writes the range
// table in key order.
//
// The coarse pass of a one-pass count reads the survivors from where the count left them: a
// block takes an equal share of the k-mer slots, whatever the buckets' sizes, and its waves the rows
// of up to 64 survivors in it in turn; where a share has more than four times 64 buckets, fewer waves
// read the same ones (300 kbp in 2^18 buckets, 215 times 64 a share: the count takes 415 us where
// all waves look at all of them, 212 so).  (Gathered into one dense array first, 1 Gbp with 43 M
// survivors took 13.19 ms instead of 12.87, 60 Mbp with 20 M 1.76 instead of 1.65, and every count
// five launches more.  With shares by buckets, a wave reads a long segment alone: 300 kbp in one
// bucket (minimizers of one base) had an output stage of 1.94 ms, 0.08 so.  With a share of the slots
// for each wave, whose rows differ in number, 60 Mbp with 20 M survivors took 211 us in
// k_msd_scatter, with the rows in turn 163.)
template <typename K, u32 NW>
struct SegRows {
  const SurvSegs& V;
  u64 w0, w1;          // the block's slots
  u32 i0;              // 64 buckets: i0 + lane
  u32 c;               // lane: survivors of its segment in these slots ...
  u32 at;              // ... and the first one's slot, from w0
  u32 inc;             // rows of the lanes' segments up to it
  u32 r, rows;         // the wave's next row, all rows of these buckets
  u32 nw;              // waves that share them ...
  u32 step;            // ... and the buckets from these to the wave's next
  bool last;           // no buckets after these

  __device__ __forceinline__ SegRows(const SurvSegs& v, u32 n_blk) : V(v) {
    // 64 buckets that hold the share's first slot: 64 probes at a time
    u32 lo = 0, hi = v.n_buckets;
    u64 n = 0;
    for (bool first = true; first || hi - lo > 64; first = false) {
      const u32 step = (hi - lo + 63) / 64, i = lo + lane_id() * step;
      const u64 x = i < hi ? v.s_base[i] : ~0ull;
      if (first) {
        n = uniform(v.meta[2] + v.meta[6] + v.meta[7]);   // k-mer slots
        const u64 per = (n + n_blk - 1) / n_blk;
        w0 = min(n, blockIdx.x * per);
        w1 = min(n, w0 + per);
        if (hi <= 64) break;
      }
      lo += (63u - (u32)__clzll(__ballot(lane_id() == 0 || x <= w0))) * step;
      hi = min(hi, lo + step);
    }
    r = uniform(threadIdx.x >> 6);
    i0 = lo;
    nw = NW;
    step = 64;
    while (nw > 1 && v.n_buckets > 4 * step * n_blk) {
      nw >>= 1;
      if (r & nw) i0 += step;
      step <<= 1;
    }
    r &= nw - 1;
    load();
  }
  // Buckets whose slots are full up to the next one's (those counted together, but the last of them)
  // are one segment with it: the lane of the first holds it.
  __device__ __forceinline__ void load() {
    const u32 i = i0 + lane_id();
    const bool in = i < V.n_buckets;
    const u64 s = in ? V.s_base[i] : w1, e = in ? s + V.s_cnt[i] : w1;
    at = (u32)(min(max(s, w0), w1) - w0);
    const u32 end = (u32)(min(max(e, w0), w1) - w0);
    const u64 goes_on = __ballot(at == lane_prev(end, ~0u));     // (never of lane 0)
    const u64 after = lane_id() == 63 ? 0ull : goes_on >> (lane_id() + 1);
    const int l = (int)lane_id() + __builtin_ctzll(~after);
    c = __shfl(end, l, 64) - at;
    if ((goes_on >> lane_id()) & 1) c = 0;
    inc = wave_scan_u32((c + 63) / 64);
    rows = lane_read(inc, 63);
    last = __any(s >= w1);
  }
  // The next row's keys, one per lane: true where the lane has one.  (Past the last row: none.)
  __device__ __forceinline__ bool row(const K** k, const u32** v) {
    while (r >= rows) {
      if (last) return false;
      r -= rows;
      i0 += step;
      load();
    }
    const int l = (int)__popcll(__ballot(inc <= r));
    const u32 cl = lane_read(c, l), o = (r - (lane_read(inc, l) - (cl + 63) / 64)) * 64 + lane_id();
    const u64 slot = w0 + lane_read(at, l);
    *k = reinterpret_cast<const K*>(V.s_k) + slot + o;
    *v = V.s_c + slot + o;
    r += nw;
    return o < cl;
  }
  __device__ __forceinline__ bool done() const { return r >= rows && last; }
};

template <typename K, bool SEGS>
__global__ __launch_bounds__(256) void k_msd_hist(MsdArgs A) {
  __shared__ u32 h[256];
  h[threadIdx.x] = 0;
  __syncthreads();
  if constexpr (SEGS) {
    constexpr int U = 8;   // rows in flight
    SegRows<K, 4> S(A.sv, A.nb);
    while (!S.done()) {
      K k[U];
      bool on[U];
#pragma unroll
      for (int u = 0; u < U; ++u) {
        const K* pk;
        const u32* pv;
        on[u] = S.row(&pk, &pv);
        k[u] = on[u] ? *pk : key_zero<K>();
      }
#pragma unroll
      for (int u = 0; u < U; ++u)
        if (on[u]) atomicAdd(&h[key_place(k[u], A.nbits, A.canonical) >> 24], 1u);
    }
  } else {
    const u64 n = *A.n_ptr;
    const u64 per = (n + A.nb - 1) / A.nb;
    const u64 a = min(n, blockIdx.x * per), b = min(n, a + per);
    const K* in = reinterpret_cast<const K*>(A.in_k);
    for (u64 i = a + threadIdx.x; i < b; i += 256) atomicAdd(&h[key_place(in[i], A.nbits, A.canonical) >> 24], 1u);
  }
  __syncthreads();
  A.hist[(u64)threadIdx.x * A.nb + blockIdx.x] = h[threadIdx.x];
}

// Pairs for msd_rounds, up to IT per thread at a time: those of [a, b) of an array ...
template <typename K, u32 T, u32 IT>
struct DensePairs {
  const K* in;
  const u32* in_v;
  u64 r0, b;
  __device__ __forceinline__ bool more() const { return r0 < b; }
  __device__ __forceinline__ void get(K (&k)[IT], u32 (&v)[IT], bool (&on)[IT]) {
#pragma unroll
    for (u32 j = 0; j < IT; ++j) {
      const u64 i = r0 + threadIdx.x + j * T;
      on[j] = i < b;
      k[j] = on[j] ? in[i] : key_zero<K>();
      v[j] = on[j] ? in_v[i] : 0u;
    }
    r0 += (u64)IT * T;
  }
};
// ... or the block's share of the survivors as the count left them.
template <typename K, u32 T, u32 IT>
struct SegPairs {
  SegRows<K, T / 64> S;
  __device__ __forceinline__ bool more() const { return __syncthreads_or(!S.done()); }
  __device__ __forceinline__ void get(K (&k)[IT], u32 (&v)[IT], bool (&on)[IT]) {
#pragma unroll
    for (u32 j = 0; j < IT; ++j) {
      const K* pk;
      const u32* pv;
      on[j] = S.row(&pk, &pv);
      k[j] = on[j] ? *pk : key_zero<K>();
      v[j] = on[j] ? *pv : 0u;
    }
  }
};

// The pairs of `in` moved to out in rounds of at most R staged through LDS: each round is
// ranked by its field (fb bits of its place below the leading `pb`, 2^fb <= F) with LDS counters,
// staged in field order and written so that consecutive threads write consecutive slots
// of a field's range; gpos[f] is the next output slot of field f (advanced per round).
// cnt, lbase and gpos have F <= T entries.  Block-wide (barriers inside).
template <typename K, u32 T, u32 F, u32 IT, typename In>
__device__ __forceinline__ void msd_rounds(In& in, const MsdArgs& A, int pb, int fb, K* __restrict__ out,
                                           u32* __restrict__ out_v, K* sk, u32* sv, u32* cnt, u32* lbase, u32* gpos,
                                           u64* scr) {
  const u32 tid = threadIdx.x;
  auto field = [&](K k) { return fb ? (key_place(k, A.nbits, A.canonical) << pb) >> (32 - fb) : 0u; };
  while (in.more()) {
    K kr[IT];
    u32 vr[IT], cc[IT], rk[IT];
    bool on[IT];
    in.get(kr, vr, on);
#pragma unroll
    for (u32 j = 0; j < IT; ++j) {
      if (on[j]) {
        cc[j] = field(kr[j]);
        rk[j] = atomicAdd(&cnt[cc[j]], 1u);
      }
    }
    __syncthreads();
    u64 tot;
    static_assert(F <= T, "one thread per field");
    const u32 ex = (u32)block_exclusive_scan<u64>(tid < F ? (u64)cnt[tid] : 0ull, scr, &tot);
    if (tid < F) lbase[tid] = ex;
    __syncthreads();
#pragma unroll
    for (u32 j = 0; j < IT; ++j) {
      if (on[j]) {
        const u32 at = lbase[cc[j]] + rk[j];
        sk[at] = kr[j];
        sv[at] = vr[j];
      }
    }
    __syncthreads();
    for (u32 i = tid; i < (u32)tot; i += T) {
      const u32 c = field(sk[i]);
      const u64 d = (u64)gpos[c] + (i - lbase[c]);
      out[d] = sk[i];
      out_v[d] = sv[i];
    }
    __syncthreads();
    if (tid < F) {
      gpos[tid] += cnt[tid];
      cnt[tid] = 0;
    }
    __syncthreads();
  }
}

// Coarse scatter: the block's range in rounds staged through LDS, written group by group.  At most 80
// VGPRs where the survivors' rows are read, so that three blocks share a CU, as their LDS allows: a count
// of 12 Mbp has 519 blocks, seven more than two each would hold (17.2 us, 13.2 so).
template <typename K, bool SEGS>
__global__ __launch_bounds__(512, SEGS ? 6 : 1) void k_msd_scatter(MsdArgs A) {
  constexpr u32 T = 512, R = sizeof(K) == 8 ? 4096u : 2048u;
  __shared__ K sk[R];
  __shared__ u32 sv[R];
  __shared__ u32 cnt[256], lbase[256], gpos[256];
  __shared__ u64 scr[17];
  const u32 tid = threadIdx.x;
  if (tid < 256) {
    cnt[tid] = 0;
    gpos[tid] = A.hist[(u64)tid * A.nb + blockIdx.x];
  }
  __syncthreads();
  auto move = [&](auto& in) {
    msd_rounds<K, T, 256, R / T>(in, A, 0, 8, reinterpret_cast<K*>(A.mid_k), A.mid_v, sk, sv, cnt, lbase, gpos, scr);
  };
  if constexpr (SEGS) {
    SegPairs<K, T, R / T> in{SegRows<K, T / 64>(A.sv, A.nb)};
    move(in);
  } else {
    const u64 n = *A.n_ptr;
    const u64 per = (n + A.nb - 1) / A.nb;
    const u64 a = min(n, blockIdx.x * per), b = min(n, a + per);
    DensePairs<K, T, R / T> in{reinterpret_cast<const K*>(A.in_k), A.in_v, a, b};
    move(in);
  }
}

// Fine pass (43 M pairs: 0.69 ms with groups by leading bits, the first twice as long as the
// mean; 0.50 ms by place): one block per coarse group; counts its sub-ranges, writes the range table,
// then moves the group's elements into their sub-ranges in staged rounds.
template <typename K>
__global__ __launch_bounds__(1024) void k_msd_fine(MsdArgs A) {
  constexpr u32 T = 1024, R = sizeof(K) == 8 ? 4096u : 2048u;
  __shared__ K sk[R];
  __shared__ u32 sv[R];
  __shared__ u32 cnt[1 << MSD_G2_MAX], lbase[1 << MSD_G2_MAX], cur[1 << MSD_G2_MAX];
  __shared__ u64 scr[17];
  const u32 g = blockIdx.x, tid = threadIdx.x;
  const u64 n = *A.n_ptr;
  const int g2 = msd_g2(n, A.target);
  const u32 F = 1u << g2;
  const u64 a = A.hist[(u64)g * A.nb];
  const u64 b = g + 1 < 256 ? (u64)A.hist[(u64)(g + 1) * A.nb] : n;
  const K* mid = reinterpret_cast<const K*>(A.mid_k);
  cnt[tid] = 0;
  __syncthreads();
  for (u64 i = a + tid; i < b; i += T) atomicAdd(&cnt[g2 ? (key_place(mid[i], A.nbits, A.canonical) << 8) >> (32 - g2) : 0u], 1u);
  __syncthreads();
  {
    u64 tot;
    const u32 run = (u32)block_exclusive_scan<u64>(tid < F ? (u64)cnt[tid] : 0ull, scr, &tot);
    if (tid < F) {
      cur[tid] = (u32)a + run;
      A.seg[((u64)g << g2) + tid] = a + run;
    }
  }
  if (g == 0 && tid == 0) {
    A.seg[(u64)256 << g2] = n;
    *A.n_seg = (u64)256 << g2;
  }
  __syncthreads();
  cnt[tid] = 0;
  __syncthreads();
  DensePairs<K, T, R / T> in{mid, A.mid_v, a, b};
  msd_rounds<K, T, 1u << MSD_G2_MAX, R / T>(in, A, 8, g2, reinterpret_cast<K*>(A.out_k), A.out_v, sk, sv, cnt, lbase,
                                            cur, scr);
}
