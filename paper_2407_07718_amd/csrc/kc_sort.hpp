// LSD radix sort of canonical k-mer keys (u64 for k <= 31, k128 for k <= 63), digits of
// DB bits (8 or 9) over the low 2k bits.
//
// Paper mapping: the k-mers are sorted so that equal values become adjacent (Section
// 3.1); the paper uses the CPU radix sorts RADULS (out of place) and PARADIS (in place)
// with O(n*d) work (Section 2.3, Section 3.1).  Here the sort is a stable LSD radix
// sort written for wave64: each pass ranks a tile of keys by digit with
//  * a per-wave table of lane masks in LDS: every lane ORs its lane bit into the entry
//    of its digit, then reads the entry back, so each lane learns which lanes of its
//    wave share its digit (an order-free way to get the wave's match masks);
//  * mbcnt over that mask for the lane's rank among equal digits (stable by lane);
//  * per-wave running digit counts in LDS across the wave's batches, and one block
//    scan over (digit, wave) for the tile offsets.
// Buckets that fit on chip are sorted entirely in LDS (lds_sort); larger key arrays go
// through HBM passes: per-block digit counts (upsweep), one scan, then a downsweep that
// ranks each tile, stages it in LDS in digit order and writes runs per digit.
#pragma once
#include "kc_common.hpp"

// Radix digit of DB bits starting at bit sh; for 128-bit keys a digit may straddle the
// two words.
template <int DB> __device__ __forceinline__ u32 key_digit_w(u64 k, int sh) {
  return (u32)(k >> sh) & ((1u << DB) - 1u);
}
template <int DB> __device__ __forceinline__ u32 key_digit_w(k128 k, int sh) {
  const u64 v = sh >= 64 ? (k.hi >> (sh - 64)) : sh == 0 ? k.lo : ((k.lo >> sh) | (k.hi << (64 - sh)));
  return (u32)v & ((1u << DB) - 1u);
}

template <int DB> __device__ __forceinline__ u32 key_digit_w(u32 k, int sh) { return (k >> sh) & ((1u << DB) - 1u); }

// The digit of a pass: the DB bits from bit `sh` on, or, for 32-bit keys, the pass-th of
// `passes` equal digits (of at most DB bits) of an index below *n_idx.
struct DigitSel {
  int sh = 0;
  const u64* n_idx = nullptr;
  int pass = 0, passes = 1;
};
struct Digit {
  int sh;
  u32 mask;
};
template <typename K, int DB> __device__ __forceinline__ Digit digit_of(const DigitSel& D) {
  if constexpr (sizeof(K) != 4) return Digit{D.sh, (1u << DB) - 1u};
  const u64 n = max(*D.n_idx, (u64)2) - 1;       // the largest index
  const int w = (64 - __builtin_clzll(n) + D.passes - 1) / D.passes;
  return Digit{min(31, w * D.pass), (1u << min(w, DB)) - 1u};
}
// Where a downsweep's pairs go: two arrays.
template <typename K>
struct StorePairs {
  K* k;
  u32* v;
  __device__ __forceinline__ void key(u64 i, K x) const { k[i] = x; }
  __device__ __forceinline__ void val(u64 i, u32 x) const { v[i] = x; }
};

template <int W, int DB = 8>
struct RankSmem {
  static constexpr int NB = 1 << DB;
  u64 tbl[W][NB];    // lane masks per digit; all zero between uses
  u32 cnt[W][NB];    // per-wave digit counts, then the items' base offsets
  u32 dstart[NB + 1];   // per-digit exclusive start within the tile; [NB] = tile size
  u64 scr[17];       // block-scan scratch
};

// Rank the active items of a tile by digit.  Item j of lane l of wave v is tile element
// (v*per + j)*64 + l; it is active iff that index is < n.  On return rk[j] holds the
// item's stable position in digit order and S.dstart the per-digit starts.
// Every thread of the block must call this (it contains barriers).
template <int T, int ITEMS, int DB = 8>
__device__ __forceinline__ void rank_by_digit(const u32 (&dg)[ITEMS], u32 (&rk)[ITEMS], int per, u32 n,
                                              RankSmem<T / 64, DB>& S) {
  constexpr int W = T / 64, NB = 1 << DB;
  static_assert(NB <= T, "one thread per digit in the offsets step");
  const u32 tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  u32* cntf = &S.cnt[0][0];
  for (u32 i = tid; i < W * NB; i += T) cntf[i] = 0;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (j < per) {
      const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
      const bool act = idx < n;
      const u32 d = dg[j];
      u64 mask = 0;
      if (act) {
        atomicOr((unsigned long long*)&S.tbl[wave][d], (unsigned long long)(1ull << lane));
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      if (act) mask = S.tbl[wave][d];
      const u32 lr = mbcnt64(mask);
      const u32 base = act ? S.cnt[wave][d] : 0u;
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      if (act && lr == 0) {
        S.cnt[wave][d] = base + (u32)__popcll(mask);
        S.tbl[wave][d] = 0;
      }
      __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
      rk[j] = base + lr;
    }
  }
  __syncthreads();
  u32 tot = 0;
  if (tid < NB) {
#pragma unroll
    for (int v = 0; v < W; ++v) {
      u32 c = S.cnt[v][tid];
      S.cnt[v][tid] = tot;
      tot += c;
    }
  }
  u64 all;
  const u64 start = block_exclusive_scan<u64>((u64)tot, S.scr, &all);
  if (tid < NB) {
    S.dstart[tid] = (u32)start;
#pragma unroll
    for (int v = 0; v < W; ++v) S.cnt[v][tid] += (u32)start;
  }
  if (tid == 0) S.dstart[NB] = (u32)all;
  __syncthreads();
#pragma unroll
  for (int j = 0; j < ITEMS; ++j) {
    if (j < per) rk[j] += S.cnt[wave][dg[j]];
  }
}

// ---------------------------------------------------------------------------- HBM passes
// Block b of nb owns elements [b*per, min(n, (b+1)*per)), per = ceil(n / nb).
__device__ __forceinline__ void block_range(u64 n, u32 nb, u64* s, u64* e) {
  const u64 per = (n + nb - 1) / nb;
  *s = min(n, (u64)blockIdx.x * per);
  *e = min(n, *s + per);
}

// counts[d * nb + b] = number of keys of block b with digit d (DB-bit digits).
template <typename K, int DB = 8>
__global__ __launch_bounds__(256) void k_radix_upsweep(const K* __restrict__ keys, const u64* __restrict__ n_ptr,
                                                       u32* __restrict__ counts, DigitSel D) {
  constexpr u32 NB = 1u << DB;
  const Digit dg = digit_of<K, DB>(D);
  __shared__ u32 h[4][NB];
  const u32 nb = gridDim.x, tid = threadIdx.x, wave = tid >> 6;
  for (u32 i = tid; i < 4 * NB; i += 256) (&h[0][0])[i] = 0;
  __syncthreads();
  u64 s, e;
  block_range(*n_ptr, nb, &s, &e);
  // batches of eight keys per thread, the next batch's loads issued before this
  // batch's counts
  constexpr u32 U = 8;
  K ka[U], kb[U];
  auto load = [&](K (&kx)[U], u64 i0) {
#pragma unroll
    for (u32 u = 0; u < U; ++u) {
      const u64 i = i0 + (u64)u * 256;
      if (i < e) kx[u] = keys[i];
    }
  };
  load(ka, s + tid);
  for (u64 i0 = s + tid; i0 < e; i0 += 256 * U) {
    if (i0 + 256 * U < e) load(kb, i0 + 256 * U);
#pragma unroll
    for (u32 u = 0; u < U; ++u)
      if (i0 + (u64)u * 256 < e) atomicAdd(&h[wave][key_digit_w<DB>(ka[u], dg.sh) & dg.mask], 1u);
#pragma unroll
    for (u32 u = 0; u < U; ++u) ka[u] = kb[u];
  }
  __syncthreads();
  for (u32 d = tid; d < NB; d += 256) counts[(u64)d * nb + blockIdx.x] = h[0][d] + h[1][d] + h[2][d] + h[3][d];
}

// ---------------------------------------------------------------------------- scan
// Exclusive scans out[i] = sum of in[0, i) for i < n; n = min(*n_ptr, n_max) when n_ptr is given,
// else n_max; *total = sum, *clamped = min(sum, cap) (where non-null).  in and out may be the
// same array; it starts and, padded, ends at 256-byte boundaries.
//
// Four consecutive values from element i of n on (i a multiple of 4; those past the end: 0), and
// the same to be written.
__device__ __forceinline__ uint4 load4(const u32* __restrict__ p, u64 i, u64 n) {
  if (i >= n) return make_uint4(0u, 0u, 0u, 0u);
  uint4 v = *reinterpret_cast<const uint4*>(p + i);
  if (i + 1 >= n) v.y = 0;
  if (i + 2 >= n) v.z = 0;
  if (i + 3 >= n) v.w = 0;
  return v;
}
__device__ __forceinline__ void store4(u32* __restrict__ p, u64 i, u64 n, uint4 v) {
  if (i + 3 < n) {
    *reinterpret_cast<uint4*>(p + i) = v;
  } else {
    if (i < n) p[i] = v.x;
    if (i + 1 < n) p[i + 1] = v.y;
    if (i + 2 < n) p[i + 2] = v.z;
  }
}
__device__ __forceinline__ u64 sum4(uint4 v) { return (u64)v.x + v.y + v.z + v.w; }

// ROWS rows of 256 values from element i0 on, one wave: their exclusive prefixes after `base`
// (sums modulo 2^32, as the array holds them).
template <int ROWS>
__device__ __forceinline__ void wave_scan_rows(const uint4 (&v)[ROWS], u32 base, u32* __restrict__ out, u64 i0, u64 n) {
#pragma unroll
  for (int r = 0; r < ROWS; ++r) {
    if (i0 + 256 * r >= n) break;   // (the same in all lanes)
    const u32 s = v[r].x + v[r].y + v[r].z + v[r].w, inc = wave_scan_u32(s), a = base + inc - s;
    store4(out, i0 + 256 * r + 4 * lane_id(), n, make_uint4(a, a + v[r].x, a + v[r].x + v[r].y, a + v[r].x + v[r].y + v[r].z));
    base += lane_read(inc, 63);
  }
}

// By one block, n_max at most SCAN_ONE_MAX: each wave holds its share, a whole number of rows of
// 256, in registers.  (10,000 values: 5 us; thread by
// thread over consecutive values, read twice, 9.)
constexpr u32 SCAN_ONE_T = 1024, SCAN_ONE_ROWS = 8;
constexpr u64 SCAN_ONE_MAX = SCAN_ONE_T / 64 * SCAN_ONE_ROWS * 256;
__global__ __launch_bounds__(SCAN_ONE_T) void k_scan_u32(const u32* __restrict__ in, u32* __restrict__ out,
                                                         const u64* __restrict__ n_ptr, u64 n_max,
                                                         u64* __restrict__ total, u64* __restrict__ clamped = nullptr,
                                                         u64 cap = 0) {
  constexpr u32 W = SCAN_ONE_T / 64;
  __shared__ u64 wsum[W];
  const u64 n = n_ptr ? min(*n_ptr, n_max) : n_max;
  const u32 lane = lane_id(), wave = uniform(threadIdx.x >> 6);
  const u32 rows = (u32)((n + W * 256 - 1) / (W * 256));   // of each wave
  const u64 i0 = (u64)wave * rows * 256, end = min(n, i0 + (u64)rows * 256);
  uint4 v[SCAN_ONE_ROWS];
  u64 sum = 0;
#pragma unroll
  for (u32 r = 0; r < SCAN_ONE_ROWS; ++r) v[r] = make_uint4(0u, 0u, 0u, 0u);
#pragma unroll
  for (u32 r = 0; r < SCAN_ONE_ROWS; ++r) {
    if (i0 + 256 * r >= end) break;
    v[r] = load4(in, i0 + 256 * r + 4 * lane, end);
    sum += sum4(v[r]);
  }
  sum = wave_sum(sum);
  if (lane == 0) wsum[wave] = sum;
  __syncthreads();
  // (the first 16 lanes hold the waves' sums)
  u64 base = lane < W ? wsum[lane] : 0ull;
  const u64 all = wave_sum(base);
  base = wave_sum(lane < wave ? base : 0ull);
  wave_scan_rows<SCAN_ONE_ROWS>(v, (u32)base, out, i0, end);
  if (threadIdx.x == 0 && total) *total = all;
  if (threadIdx.x == 0 && clamped) *clamped = min(all, cap);
}

// Larger arrays (up to 1024 * SCAN_BLOCK), in two launches: each block's sum, then each block's
// prefixes after the sum of the blocks before it, which it adds up itself (at most 1023: less
// than a third launch).  The last block writes the total.  (A count of 6 Mbp, with the plan's sums
// the same way: 325 us with the third launches and values read one by one, 288 so.)
constexpr u32 SCAN_T = 256, SCAN_ROWS = 4, SCAN_BLOCK = SCAN_T / 64 * SCAN_ROWS * 256;
__device__ __forceinline__ u64 scan_wave_load(const u32* __restrict__ in, u64 i0, u64 n, uint4 (&v)[SCAN_ROWS]) {
  u64 sum = 0;
#pragma unroll
  for (u32 r = 0; r < SCAN_ROWS; ++r) {
    v[r] = load4(in, i0 + 256 * r + 4 * lane_id(), n);
    sum += sum4(v[r]);
  }
  return wave_sum(sum);
}
__global__ __launch_bounds__(SCAN_T) void k_scan_reduce(const u32* __restrict__ in, const u64* __restrict__ n_ptr,
                                                        u64 n_max, u64* __restrict__ bsum) {
  __shared__ u64 wsum[SCAN_T / 64];
  const u64 n = n_ptr ? min(*n_ptr, n_max) : n_max;
  const u32 wave = uniform(threadIdx.x >> 6);
  uint4 v[SCAN_ROWS];
  const u64 sum = scan_wave_load(in, (u64)blockIdx.x * SCAN_BLOCK + (u64)wave * SCAN_ROWS * 256, n, v);
  if (lane_id() == 0) wsum[wave] = sum;
  __syncthreads();
  if (threadIdx.x == 0) {
    u64 t = 0;
    for (u32 w = 0; w < SCAN_T / 64; ++w) t += wsum[w];
    bsum[blockIdx.x] = t;
  }
}
__global__ __launch_bounds__(SCAN_T) void k_scan_apply(const u32* __restrict__ in, u32* __restrict__ out,
                                                       const u64* __restrict__ n_ptr, u64 n_max,
                                                       const u64* __restrict__ bsum, u64* __restrict__ total,
                                                       u64* __restrict__ clamped, u64 cap) {
  __shared__ u64 wsum[SCAN_T / 64], wbefore[SCAN_T / 64];
  const u64 n = n_ptr ? min(*n_ptr, n_max) : n_max;
  const u32 wave = uniform(threadIdx.x >> 6);
  const u64 i0 = (u64)blockIdx.x * SCAN_BLOCK + (u64)wave * SCAN_ROWS * 256;
  u64 before = 0;
  for (u32 i = threadIdx.x; i < blockIdx.x; i += SCAN_T) before += bsum[i];
  uint4 v[SCAN_ROWS];
  const u64 sum = scan_wave_load(in, i0, n, v);
  before = wave_sum(before);
  if (lane_id() == 0) {
    wsum[wave] = sum;
    wbefore[wave] = before;
  }
  __syncthreads();
  u64 base = 0, all = 0;
  for (u32 w = 0; w < SCAN_T / 64; ++w) {
    base += wbefore[w] + (w < wave ? wsum[w] : 0ull);
    all += wbefore[w] + wsum[w];
  }
  wave_scan_rows<SCAN_ROWS>(v, (u32)base, out, i0, n);
  if (blockIdx.x + 1 == gridDim.x && threadIdx.x == 0) {
    if (total) *total = all;
    if (clamped) *clamped = min(all, cap);
  }
}

// Row d of counts (one digit over all nb blocks) -> exclusive prefix over blocks, and
// totals[d] = the row sum.  One block per digit.
__global__ __launch_bounds__(256) void k_radix_rowscan(u32* __restrict__ counts, u32 nb, u32* __restrict__ totals) {
  __shared__ u64 scr[17];
  u32* row = counts + (u64)blockIdx.x * nb;
  const u32 per = (nb + 255) / 256;
  const u32 s = min(nb, threadIdx.x * per), e = min(nb, s + per);
  u64 sum = 0;
  for (u32 i = s; i < e; ++i) sum += row[i];
  u64 all;
  u64 run = block_exclusive_scan<u64>(sum, scr, &all);
  for (u32 i = s; i < e; ++i) {
    const u32 v = row[i];
    row[i] = (u32)run;
    run += v;
  }
  if (threadIdx.x == 0) totals[blockIdx.x] = (u32)all;
}

// Stable scatter of one pass.  Each tile of T*ITEMS keys is ranked by digit, staged in
// LDS in digit order and written out as one run per digit.  With SHARED the values are
// staged after the keys in the same LDS buffer (less LDS per block, one more barrier).
template <typename K, bool HASV, int T, int ITEMS, bool SHARED, int DB, typename Out>
__global__ __launch_bounds__(T) void k_radix_downsweep(const K* __restrict__ kin, const u32* __restrict__ vin, Out out,
                                                       const u64* __restrict__ n_ptr, const u32* __restrict__ counts,
                                                       const u32* __restrict__ totals, DigitSel D) {
  constexpr int W = T / 64, TILE = T * ITEMS, NB = 1 << DB;
  static_assert(NB <= T, "one thread per digit");
  const Digit digit = digit_of<K, DB>(D);
  __shared__ RankSmem<W, DB> S;
  __shared__ K stage_k[TILE];
  __shared__ u32 stage_v[(HASV && !SHARED) ? TILE : 1];
  __shared__ u32 run_base[NB];
  const u32 nb = gridDim.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  for (u32 i = tid; i < W * NB; i += T) (&S.tbl[0][0])[i] = 0;
  {
    // digit d of this block starts at (sum of all smaller digits) + (digit d in earlier blocks)
    const u64 t = tid < (u32)NB ? totals[tid] : 0u;
    u64 all;
    const u64 dbase = block_exclusive_scan<u64>(t, S.scr, &all);
    if (tid < (u32)NB) run_base[tid] = (u32)dbase + counts[(u64)tid * nb + blockIdx.x];
  }
  __syncthreads();
  u64 s, e;
  block_range(*n_ptr, nb, &s, &e);
  // Tiles are loaded one ahead into registers: the next tile's loads stay in flight
  // while this tile is ranked, staged and written (barriers wait on LDS only).
  K kn[ITEMS];
  u32 vn[ITEMS];
  auto load_tile = [&](u64 t0) {
    const u32 nt = (u32)min((u64)TILE, e - t0);
    const int per = (int)((nt + 64u * W - 1) / (64u * W));
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
        if (idx < nt) {
          kn[j] = kin[t0 + idx];
          if (HASV) vn[j] = vin[t0 + idx];
        } else {
          kn[j] = key_zero<K>();
          vn[j] = 0;
        }
      }
    }
  };
  if (s < e) load_tile(s);
  for (u64 t0 = s; t0 < e; t0 += TILE) {
    const u32 nt = (u32)min((u64)TILE, e - t0);
    const int per = (int)((nt + 64u * W - 1) / (64u * W));
    K kr[ITEMS];
    u32 vr[ITEMS], dg[ITEMS], rk[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      kr[j] = kn[j];
      vr[j] = vn[j];
    }
    if (t0 + TILE < e) load_tile(t0 + TILE);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) dg[j] = key_digit_w<DB>(kr[j], digit.sh) & digit.mask;
    }
    rank_by_digit<T, ITEMS, DB>(dg, rk, per, nt, S);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
        if (idx < nt) {
          stage_k[rk[j]] = kr[j];
          if (HASV && !SHARED) stage_v[rk[j]] = vr[j];
        }
      }
    }
    __syncthreads();
    if (HASV && SHARED) {
      // keys out, remembering each staged slot's destination; then the values
      u32 dsts[ITEMS];
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        const u32 i = tid + (u32)j * T;
        if (i < nt) {
          const K key = stage_k[i];
          const u32 d = key_digit_w<DB>(key, digit.sh) & digit.mask;
          dsts[j] = run_base[d] + (i - S.dstart[d]);
          out.key(dsts[j], key);
        }
      }
      __syncthreads();
      u32* sv = reinterpret_cast<u32*>(stage_k);
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        if (j < per) {
          const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
          if (idx < nt) sv[rk[j]] = vr[j];
        }
      }
      __syncthreads();
#pragma unroll
      for (int j = 0; j < ITEMS; ++j) {
        const u32 i = tid + (u32)j * T;
        if (i < nt) out.val(dsts[j], sv[i]);
      }
    } else {
      for (u32 i = tid; i < nt; i += T) {
        const K key = stage_k[i];
        const u32 d = key_digit_w<DB>(key, digit.sh) & digit.mask;
        const u64 dst = (u64)run_base[d] + (i - S.dstart[d]);
        out.key(dst, key);
        if (HASV) out.val(dst, stage_v[i]);
      }
    }
    __syncthreads();
    if (tid < (u32)NB) run_base[tid] += S.dstart[tid + 1] - S.dstart[tid];
    __syncthreads();
  }
}

// ---------------------------------------------------------------------------- pass by set
// One stable pass that orders (key, value) pairs by the set held in the value's bits above
// cbits (sets < 512), keeping their order within each set; the values leave with the set
// bits cleared.  k_set_hist counts the sets of each block's range (counts[s * nb + b]),
// k_radix_rowscan turns the counts into offsets (totals = pairs per set), and
// k_set_scatter ranks each tile by set in LDS, stages it in set order and writes one run
// per set.
constexpr int SET_DB = 9;

__global__ __launch_bounds__(256) void k_set_hist(const u32* __restrict__ vals, const u64* __restrict__ n_ptr,
                                                  u32* __restrict__ counts, int cbits) {
  constexpr u32 NB = 1u << SET_DB;
  __shared__ u32 h[4][NB];
  const u32 nb = gridDim.x, tid = threadIdx.x, wave = tid >> 6;
  for (u32 i = tid; i < 4 * NB; i += 256) (&h[0][0])[i] = 0;
  __syncthreads();
  u64 s, e;
  block_range(*n_ptr, nb, &s, &e);
  for (u64 i = s + tid; i < e; i += 256) atomicAdd(&h[wave][(vals[i] >> cbits) & (NB - 1)], 1u);
  __syncthreads();
  for (u32 d = tid; d < NB; d += 256) counts[(u64)d * nb + blockIdx.x] = h[0][d] + h[1][d] + h[2][d] + h[3][d];
}

template <typename K, int T, int ITEMS>
__global__ __launch_bounds__(T) void k_set_scatter(const K* __restrict__ kin, K* __restrict__ kout,
                                                   const u32* __restrict__ vin, u32* __restrict__ vout,
                                                   const u64* __restrict__ n_ptr, const u32* __restrict__ counts,
                                                   const u32* __restrict__ totals, int cbits) {
  constexpr int W = T / 64, TILE = T * ITEMS, NB = 1 << SET_DB;
  static_assert(NB <= T, "one thread per set");
  __shared__ RankSmem<W, SET_DB> S;
  __shared__ K stage_k[TILE];
  __shared__ u32 stage_v[TILE];
  __shared__ u16 stage_d[TILE];
  __shared__ u32 run_base[NB];
  const u32 nb = gridDim.x, tid = threadIdx.x, lane = lane_id(), wave = tid >> 6;
  const u32 cmask = cbits >= 32 ? ~0u : ((1u << cbits) - 1u);
  for (u32 i = tid; i < W * NB; i += T) (&S.tbl[0][0])[i] = 0;
  {
    const u64 t = tid < (u32)NB ? totals[tid] : 0u;
    u64 all;
    const u64 dbase = block_exclusive_scan<u64>(t, S.scr, &all);
    if (tid < (u32)NB) run_base[tid] = (u32)dbase + counts[(u64)tid * nb + blockIdx.x];
  }
  __syncthreads();
  u64 s, e;
  block_range(*n_ptr, nb, &s, &e);
  for (u64 t0 = s; t0 < e; t0 += TILE) {
    const u32 nt = (u32)min((u64)TILE, e - t0);
    const int per = (int)((nt + 64u * W - 1) / (64u * W));
    K kr[ITEMS];
    u32 vr[ITEMS], dg[ITEMS], rk[ITEMS];
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
        if (idx < nt) {
          kr[j] = kin[t0 + idx];
          vr[j] = vin[t0 + idx];
        } else {
          kr[j] = key_zero<K>();
          vr[j] = 0;
        }
        dg[j] = (vr[j] >> cbits) & (NB - 1);
      }
    }
    rank_by_digit<T, ITEMS, SET_DB>(dg, rk, per, nt, S);
#pragma unroll
    for (int j = 0; j < ITEMS; ++j) {
      if (j < per) {
        const u32 idx = (wave * (u32)per + (u32)j) * 64u + lane;
        if (idx < nt) {
          stage_k[rk[j]] = kr[j];
          stage_v[rk[j]] = vr[j] & cmask;
          stage_d[rk[j]] = (u16)dg[j];
        }
      }
    }
    __syncthreads();
    for (u32 i = tid; i < nt; i += T) {
      const u32 d = stage_d[i];
      const u64 dst = (u64)run_base[d] + (i - S.dstart[d]);
      kout[dst] = stage_k[i];
      vout[dst] = stage_v[i];
    }
    __syncthreads();
    if (tid < (u32)NB) run_base[tid] += S.dstart[tid + 1] - S.dstart[tid];
    __syncthreads();
  }
}

// first[s] = pairs of the sets before s (exclusive scan of the per-set totals), s <= n_sets.
__global__ __launch_bounds__(512) void k_set_first(const u32* __restrict__ totals, u32 n_sets,
                                                   u64* __restrict__ first) {
  __shared__ u64 scr[17];
  const u32 tid = threadIdx.x;
  const u64 v = tid < n_sets ? (u64)totals[tid] : 0ull;
  u64 all;
  const u64 ex = block_exclusive_scan<u64>(v, scr, &all);
  if (tid < n_sets) first[tid] = ex;
  if (tid == 0) first[n_sets] = all;
}

