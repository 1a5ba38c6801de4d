// Split-mask generation on gfx950: which Gaussians the next Long-Axis-Split
// takes (the selection that feeds it; Sec. 2.1's edge scores moved to the
// Gaussians, Sec. 3's gradient threshold and warm-up, and a budget).
//
//   sel_clear   : scores[0, N) = 0, the histograms and the lists' lengths = 0
//                 (fill kernels, so the call can be captured)
//   sel_scatter : per contribution (Gaussian g, view v, pixel p, weight w):
//                 scores[g] += floor(fl32(E_v[p] * w) * 2^32); each
//                 work-group sums a chunk of the contributions per Gaussian
//                 (runs on consecutive lanes, then an LDS hash table) and
//                 adds each sum with one 64-bit atomic; fixed
//                 point makes the sum exact and independent of the order
//                 the additions land in
//   sel_hist    : the candidates' keys (score + 1) counted by their leading
//                 bits: exponent and 6 more, so keys below 128 exactly
//   sel_collect : every work-group finds K = min(candidates, max(0, budget -
//                 N)) and the bin of the K-th largest key from that histogram;
//                 rows above the bin are selected, rows inside it listed (or,
//                 where the bin is one exact key shared by more rows than are
//                 still to take, counted per tile)
//   sel_refine  : (three times) where that list would be long, because most
//                 scores lie within 1.6% of each other, the next 12 bits are
//                 counted instead, by all work-groups, and the rows of the K-th
//                 key's digit listed (or counted on); nothing to do otherwise
//   sel_finish  : one work-group: exact selection among the listed keys, ties
//                 by lower index; or all of them: the rows of one shared key, up
//                 to the last one taken, found from the tile counts
#include "igsp_internal.h"

namespace igsp {
namespace {

__device__ __forceinline__ int64_t live_count(const SelLaunch& S) {
  const int64_t n = *S.count;
  return n < 0 ? 0 : (n > S.capacity ? S.capacity : n);
}

__device__ __forceinline__ bool candidate(const SelLaunch& S, int64_t g) {
  return S.warmup || S.grad[g] >= S.grad_threshold;
}

__device__ __forceinline__ uint64_t key_of(const SelLaunch& S, int64_t g) {
  return candidate(S, g) ? (uint64_t)S.scores[g] + 1ull : 0ull;
}

__global__ __launch_bounds__(kSelThreads) void sel_clear_kernel(SelLaunch S) {
  const int64_t N = live_count(S);
  for (int64_t g = (int64_t)blockIdx.x * kSelThreads + threadIdx.x; g < N; g += (int64_t)gridDim.x * kSelThreads)
    S.scores[g] = 0;
  if (blockIdx.x == 0) {
    for (int i = threadIdx.x; i < kSelLevels * kSelBins / 4; i += kSelThreads)
      reinterpret_cast<uint4*>(S.hist)[i] = uint4{0u, 0u, 0u, 0u};
    if (threadIdx.x < kSelLevels) S.state[threadIdx.x].listed = 0;
  }
}

// Contributions arrive in image order, so neighbouring entries often name the
// same Gaussian, and a Gaussian's entries recur a few image rows later. The
// grid sweeps the list in order, one chunk of `rounds` x kSelThreads
// contributions per work-group at a time (so the map reads of neighbouring
// chunks stay close). Each wavefront first sums the runs of equal Gaussian
// index on consecutive lanes (a prefix sum over the lanes by DPP, whose
// difference over a run is exact modulo 2^64; a segmented sum by shuffles
// kept the LDS pipe busy with 18 of them a round: 3.5M entries 30.7 -> 26.6 us;
// 106M, bound by memory, the same); a run's
// first lane then adds the run's sum into the work-group's LDS hash table
// (open addressing, kScatterProbes linear probes; a run that finds no slot
// goes straight to its global atomic); at the end of the chunk every used
// slot issues one 64-bit atomic and is cleared.
constexpr int kScatterSlots = 1024;  // 12 KB of LDS: keys and 64-bit sums
constexpr int kScatterProbes = 16;
static_assert(kScatterSlots == 1 << 10, "the slot hash keeps the top 10 bits");

// LDS_VIEWS: the view table is copied into (dynamic) LDS first, so each
// contribution's map read waits on one global load fewer.
constexpr int kSelLdsViews = 512;  // at most this many views go to LDS (8 KB)

// Inclusive sum over a wavefront's lanes (mod 2^64).
__device__ __forceinline__ uint64_t wave_incl_sum(uint64_t v) {
#define IGSP_SUM_STEP(ctrl, rows)                                                                  \
  {                                                                                                \
    const uint32_t lo = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)v, ctrl, rows, 0xf, false);          \
    const uint32_t hi = (uint32_t)__builtin_amdgcn_update_dpp(0, (int)(uint32_t)(v >> 32), ctrl, rows, 0xf, false);  \
    v += ((uint64_t)hi << 32) | lo;                                                                \
  }
  IGSP_SUM_STEP(0x111, 0xf)  // row_shr:1
  IGSP_SUM_STEP(0x112, 0xf)  // row_shr:2
  IGSP_SUM_STEP(0x114, 0xf)  // row_shr:4
  IGSP_SUM_STEP(0x118, 0xf)  // row_shr:8
  IGSP_SUM_STEP(0x142, 0xa)  // row_bcast:15 into rows 1 and 3
  IGSP_SUM_STEP(0x143, 0xc)  // row_bcast:31 into rows 2 and 3
#undef IGSP_SUM_STEP
  return v;
}

template <class T, bool NT>
__device__ __forceinline__ T stream_load(const T* p) {
  if constexpr (NT) return __builtin_nontemporal_load(p);
  else return *p;
}

template <bool LDS_VIEWS, bool NT>
__global__ __launch_bounds__(kSelThreads) void sel_scatter_kernel(SelLaunch S, int rounds) {
  __shared__ int32_t keys[kScatterSlots];
  __shared__ unsigned long long sums[kScatterSlots];
  extern __shared__ SelView lviews[];
  const int64_t chunk = (int64_t)rounds * kSelThreads;
  const int64_t N = live_count(S);
  const int lane = threadIdx.x & 63;
  for (int i = threadIdx.x; i < kScatterSlots; i += kSelThreads) {
    keys[i] = -1;
    sums[i] = 0ull;
  }
  if constexpr (LDS_VIEWS)
    for (int i = threadIdx.x; i < S.n_views; i += kSelThreads) lviews[i] = S.views[i];
  __syncthreads();
  for (int64_t b0 = (int64_t)blockIdx.x * chunk; b0 < S.n_contrib; b0 += (int64_t)gridDim.x * chunk) {
    const int64_t b1 = b0 + chunk < S.n_contrib ? b0 + chunk : S.n_contrib;
    // software pipeline over the chunk's rounds: while round r's values are
    // scattered, round r + 1's map value and round r + 2's entries are in
    // flight (entries past the chunk read as ignored)
    auto load_entry = [&](int64_t c, int32_t& gi, int32_t& v, int32_t& p, float& w) {
      gi = -1;
      if (c < b1) {
        gi = stream_load<int32_t, NT>(S.gauss + c);
        v = stream_load<int32_t, NT>(S.view + c);
        p = stream_load<int32_t, NT>(S.pixel + c);
        w = stream_load<float, NT>(S.weight + c);
      }
    };
    // the contribution's map value (0 for an ignored entry) and its Gaussian (-1)
    auto map_value = [&](int32_t gi, int32_t v, int32_t p, float w, int32_t& g) -> float {
      g = -1;
      if (gi >= 0 && gi < N && v >= 0 && v < S.n_views) {                 // else outside the live set: ignored
        const SelView sv = LDS_VIEWS ? lviews[v] : S.views[v];
        if (p >= 0 && (int64_t)p < sv.pixels) {
          g = gi;
          return S.maps[sv.out_offset + p] * w;                            // one FP32 product
        }
      }
      return 0.0f;
    };
    int32_t gi1 = -1, v1 = 0, p1 = 0, gi2 = -1, v2 = 0, p2 = 0, g1 = -1;
    float w1 = 0.0f, w2 = 0.0f;
    load_entry(b0 + threadIdx.x, gi1, v1, p1, w1);
    load_entry(b0 + kSelThreads + threadIdx.x, gi2, v2, p2, w2);
    float e1 = map_value(gi1, v1, p1, w1, g1);
    for (int64_t c0 = b0; c0 < b1; c0 += kSelThreads) {
      const int32_t g = g1;
      const float e = e1;
      e1 = map_value(gi2, v2, p2, w2, g1);                                 // round r + 1
      load_entry(c0 + 2 * kSelThreads + threadIdx.x, gi2, v2, p2, w2);    // round r + 2
      uint64_t q = 0;
      if (e > 0.0f) q = (uint64_t)floorf(e * 4294967296.0f);               // exact: a power-of-two scale
      int32_t gp = __builtin_amdgcn_mov_dpp(g, 0x138, 0xf, 0xf, true);     // wave_shr:1
      asm volatile("" : "+v"(gp));  // kept a plain move (a wave shift folded into its use is not exact here)
      const bool head = lane == 0 || gp != g;
      const uint64_t heads = __ballot(head);
      const uint64_t incl = wave_incl_sum(q), excl = incl - q;
      // the run's last lane: the one before the next head
      const uint64_t later = (heads >> lane) >> 1;
      const int last = later ? lane + __builtin_ctzll(later) : 63;
      q = (uint64_t)__shfl((unsigned long long)incl, last, 64) - excl;
      if (head && g >= 0 && q != 0) {
        uint32_t h = ((uint32_t)g * 2654435761u) >> (32 - 10);         // 10 bits: kScatterSlots
        bool placed = false;
        for (int k = 0; k < kScatterProbes && !placed; ++k) {
          const int32_t prev = atomicCAS(&keys[h], -1, g);
          if (prev == -1 || prev == g) {
            atomicAdd(&sums[h], (unsigned long long)q);
            placed = true;
          }
          h = (h + 1) & (kScatterSlots - 1);
        }
        if (!placed) atomicAdd(reinterpret_cast<unsigned long long*>(S.scores + g), (unsigned long long)q);
      }
    }
    __syncthreads();
    for (int i = threadIdx.x; i < kScatterSlots; i += kSelThreads) {
      const int32_t g = keys[i];
      if (g >= 0) {
        const unsigned long long q = sums[i];
        if (q != 0ull) atomicAdd(reinterpret_cast<unsigned long long*>(S.scores + g), q);
        keys[i] = -1;
        sums[i] = 0ull;
      }
    }
    __syncthreads();
  }
}

// Exclusive scan over the work-group (kSelThreads threads).
__device__ __forceinline__ uint32_t sel_scan(uint32_t v, uint32_t* wsum, uint32_t& total) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t before = 0, tot = 0;
#pragma unroll
  for (int k = 0; k < kSelThreads / 64; ++k) {
    const uint32_t t = wsum[k];
    if (k < w) before += t;
    tot += t;
  }
  total = tot;
  __syncthreads();
  return before + x - v;
}

// Bin of a key by its leading bits (monotone): keys below 128 by themselves,
// larger ones by exponent and the 6 bits after the leading one.
__device__ __forceinline__ int key_bin(uint64_t key) {
  const int e = 63 - __clzll((long long)(key | 1ull));
  return e <= 6 ? (int)key : (e - 5) * 64 + (int)((key >> (e - 6)) & 63u);
}
// Low bits of the keys of a bin that the bin leaves open (0: one exact key).
__device__ __forceinline__ int open_bits(int bin) { return bin < 128 ? 0 : bin / 64 - 1; }

// Rows' keys in flight per thread in the row passes: independent loads, a
// row's two arrays each.
constexpr int kSelUnroll = 8;
static_assert(kSelTile == kSelUnroll * kSelThreads, "one step per tile");

__device__ __forceinline__ void tile_keys(const SelLaunch& S, int64_t t, int64_t N, uint64_t key[kSelUnroll]) {
  float gr[kSelUnroll];
  int64_t sc[kSelUnroll];
#pragma unroll
  for (int k = 0; k < kSelUnroll; ++k) {
    const int64_t g = min(t * kSelTile + k * kSelThreads + threadIdx.x, N - 1);  // (past the end: the last row, dropped below)
    gr[k] = S.grad[g];
    sc[k] = S.scores[g];
  }
#pragma unroll
  for (int k = 0; k < kSelUnroll; ++k) {
    const int64_t g = t * kSelTile + k * kSelThreads + threadIdx.x;
    key[k] = g < N && (S.warmup || gr[k] >= S.grad_threshold) ? (uint64_t)sc[k] + 1ull : 0ull;
  }
}

// The candidates' keys counted by bin.
__global__ __launch_bounds__(kSelThreads) void sel_hist_kernel(SelLaunch S) {
  __shared__ uint32_t h[kSelBins];
  const int64_t N = live_count(S);
  const int64_t nt = (N + kSelTile - 1) / kSelTile;
  if ((int64_t)blockIdx.x >= nt) return;
  for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) h[i] = 0;
  __syncthreads();
  for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
    uint64_t key[kSelUnroll];
    tile_keys(S, t, N, key);
#pragma unroll
    for (int k = 0; k < kSelUnroll; ++k)
      if (key[k]) atomicAdd(&h[key_bin(key[k])], 1u);
  }
  __syncthreads();
  for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) {
    const uint32_t c = h[i];
    if (c) atomicAdd(&S.hist[i], c);
  }
}

// What is left to select once a histogram is known; every work-group takes
// this step alike.
struct SelPick {
  int64_t k;       // Gaussians to select from the whole histogram
  int64_t need;    // of them, inside the bin
  int64_t in_bin;  // candidates inside the bin
  int bin;
};

// The bin of the K-th largest entry; K = want, or (want < 0) what the budget
// leaves room for.
__device__ __forceinline__ SelPick pick_bin(const SelLaunch& S, const uint32_t* hist, int64_t N, int64_t want,
                                            uint32_t* wsum, SelPick* s_pick) {
  constexpr int PER = kSelBins / kSelThreads;
  static_assert(kSelBins % kSelThreads == 0 && PER % 4 == 0, "whole 16-byte words of bins per thread");
  // descending order: thread t holds the bins from kSelBins - 1 - t PER down
  uint32_t c[PER];
  const int lo = kSelBins - (threadIdx.x + 1) * PER;
  uint32_t sum = 0;
#pragma unroll
  for (int j = 0; j < PER / 4; ++j) {
    const uint4 q = reinterpret_cast<const uint4*>(hist + lo)[j];
    c[4 * j] = q.x; c[4 * j + 1] = q.y; c[4 * j + 2] = q.z; c[4 * j + 3] = q.w;
    sum += q.x + q.y + q.z + q.w;
  }
  uint32_t total = 0;
  int64_t above = sel_scan(sum, wsum, total);
  const int64_t room = want >= 0 ? want : (S.budget > N ? S.budget - N : 0);
  const int64_t K = (int64_t)total < room ? (int64_t)total : room;
  if (K == 0) {
    if (threadIdx.x == 0) *s_pick = SelPick{0, 0, 0, kSelBins};
  } else if (above < K && K <= above + sum) {
    int bin = lo;
    uint32_t in = 0;
    int64_t up = above;
#pragma unroll
    for (int j = PER - 1; j >= 0; --j) {
      if (up + c[j] >= K) { bin = lo + j; in = c[j]; break; }
      up += c[j];
    }
    *s_pick = SelPick{K, K - up, in, bin};
  }
  __syncthreads();
  return *s_pick;
}

// How the rest of a group of rows is selected: its keys share the bits above
// `shift`, `need` of its `in` rows are taken. A list is finished by one
// work-group, so a long one is refined first.
constexpr int64_t kSelLongList = 8192;

__device__ __forceinline__ int group_mode(int64_t need, int64_t in, int shift, int level) {
  if (need == in) return kSelDone;
  if (shift == 0) return kSelTie;
  if (in <= kSelLongList) return kSelList;
  return level + 1 < kSelLevels ? kSelWide : kSelLast;
}

// Work-group state of a pass over the rows: a tile's listed rows, or the
// digit histogram of the work-group's tiles.
struct SelLds {
  union {
    uint64_t key[kSelTile];
    uint32_t hist[kSelBins];
  };
  int32_t row[kSelTile];
  SelRange range[kSelThreads / 64];
  uint32_t n, base;
};
static_assert(kSelBins * sizeof(uint32_t) <= kSelTile * sizeof(uint64_t), "the histogram fits the keys");

constexpr int kSelDigit = 12;
static_assert((1 << kSelDigit) == kSelBins, "a digit is a bin");

// The smallest and the largest of the NT threads' keys, in every thread of the
// work-group. (A work-group's range is stored, and all are read by every
// work-group of the next launch, 16 KB at most: minima and maxima taken by
// atomics on one address follow one another at about 11 ns.)
template <int NT>
__device__ __forceinline__ SelRange wg_range(SelRange r, SelRange* wave /* [NT / 64] */) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) {
    const uint64_t a = (uint64_t)__shfl_xor((unsigned long long)r.least, o, 64);
    const uint64_t b = (uint64_t)__shfl_xor((unsigned long long)r.most, o, 64);
    r.least = a < r.least ? a : r.least;
    r.most = b > r.most ? b : r.most;
  }
  if ((threadIdx.x & 63) == 0) wave[threadIdx.x >> 6] = r;
  __syncthreads();
#pragma unroll
  for (int k = 0; k < NT / 64; ++k) {
    r.least = wave[k].least < r.least ? wave[k].least : r.least;
    r.most = wave[k].most > r.most ? wave[k].most : r.most;
  }
  return r;
}

// The smallest and largest key of a level's group, from the work-groups of the
// pass over its nt tiles.
template <int NT>
__device__ __forceinline__ SelRange group_range(const SelLaunch& S, int level, int64_t nt, SelRange* wave) {
  SelRange r = {~0ull, 0ull};
  const int n = nt < S.grid ? (int)nt : S.grid;
  for (int i = threadIdx.x; i < n; i += NT) {
    const SelRange q = S.ranges[level * kSelGrid + i];
    r.least = q.least < r.least ? q.least : r.least;
    r.most = q.most > r.most ? q.most : r.most;
  }
  return wg_range<NT>(r, wave);
}

// A pass over the rows: `above(key)` rows are selected (the mask is written
// for every row, or only for those: WRITE), rows of the group (key >> shift ==
// prefix) counted or listed as `mode` says, for level `level`.
template <bool WRITE, class Above>
__device__ __forceinline__ void sel_pass(const SelLaunch& S, int64_t N, int level, int mode, uint64_t prefix, int shift,
                                         SelLds& l, uint32_t* wsum, Above above) {
  SelState* const st = S.state + level;
  const int64_t nt = (N + kSelTile - 1) / kSelTile;
  const int bits = shift < kSelDigit ? shift : kSelDigit;
  uint64_t least = ~0ull, most = 0;
  const bool ranged = mode == kSelWide || mode == kSelLast, counted = ranged || mode == kSelTie;
  if (mode == kSelWide)
    for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) l.hist[i] = 0;
  if (threadIdx.x == 0) l.n = 0;
  __syncthreads();
  for (int64_t t = blockIdx.x; t < nt; t += gridDim.x) {
    uint64_t key[kSelUnroll];
    tile_keys(S, t, N, key);
    uint32_t ties = 0;
#pragma unroll
    for (int k = 0; k < kSelUnroll; ++k) {
      const int64_t g = t * kSelTile + k * kSelThreads + threadIdx.x;
      const bool up = key[k] && above(key[k]);
      if (g < N && (WRITE || up)) S.mask[g] = (uint8_t)up;
      if (mode == kSelDone || !key[k] || (key[k] >> shift) != prefix) continue;
      ++ties;
      if (ranged) {
        least = key[k] < least ? key[k] : least;
        most = key[k] > most ? key[k] : most;
      }
      if (mode == kSelWide) atomicAdd(&l.hist[(uint32_t)(key[k] >> (shift - bits)) & ((1u << bits) - 1u)], 1u);
      if (mode == kSelList || mode == kSelLast) {
        const uint32_t at = atomicAdd(&l.n, 1u);
        l.key[at] = key[k];
        l.row[at] = (int32_t)g;
      }
    }
    if (mode == kSelDone) continue;  // uniform, here and below
    if (counted) {
      uint32_t total = 0;
      (void)sel_scan(ties, wsum, total);
      if (threadIdx.x == 0) S.tile_counts[t] = total;
      if (mode != kSelLast) continue;
    }
    __syncthreads();
    if (threadIdx.x == 0 && l.n) l.base = atomicAdd(&st->listed, l.n);
    __syncthreads();
    const uint32_t n = l.n;
    for (uint32_t i = threadIdx.x; i < n; i += kSelThreads) {
      S.ckeys[l.base + i] = l.key[i];
      S.crows[l.base + i] = l.row[i];
    }
    __syncthreads();
    if (threadIdx.x == 0) l.n = 0;
    __syncthreads();
  }
  if (mode == kSelWide) {
    __syncthreads();
    for (int i = threadIdx.x; i < kSelBins; i += kSelThreads) {
      const uint32_t c = l.hist[i];
      if (c) atomicAdd(&S.hist[(level + 1) * kSelBins + i], c);
    }
  }
  if (ranged) {
    const SelRange r = wg_range<kSelThreads>(SelRange{least, most}, l.range);
    if (threadIdx.x == 0) S.ranges[level * kSelGrid + blockIdx.x] = r;
  }
}

__device__ __forceinline__ void put_group(SelState* st, int64_t need, int64_t in, uint64_t prefix, int shift, int mode) {
  st->need = need;
  st->in = in;
  st->prefix = prefix;
  st->shift = shift;
  st->mode = mode;
}

__global__ __launch_bounds__(kSelThreads) void sel_collect_kernel(SelLaunch S) {
  __shared__ uint32_t wsum[kSelThreads / 64];
  __shared__ SelPick s_pick;
  __shared__ SelLds l;
  const int64_t N = live_count(S);
  const int64_t nt = (N + kSelTile - 1) / kSelTile;
  if ((int64_t)blockIdx.x >= nt && blockIdx.x > 0) return;
  const SelPick p = pick_bin(S, S.hist, N, -1, wsum, &s_pick);
  const int shift = open_bits(p.bin);
  const uint64_t prefix = p.bin < 128 ? (uint64_t)p.bin : (uint64_t)(64 + (p.bin & 63));
  const int mode = group_mode(p.need, p.in_bin, shift, 0);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    put_group(S.state, p.need, p.in_bin, prefix, shift, mode);
    if (S.n_selected) *S.n_selected = p.k;
  }
  const int least = mode == kSelDone ? p.bin : p.bin + 1;              // bins selected as a whole
  sel_pass<true>(S, N, 0, mode, prefix, shift, l, wsum, [&](uint64_t key) { return key_bin(key) >= least; });
}

// The next digit of a group whose list would be long. A group of one key is a
// tie at once, and bits that all of a group's keys share are passed over, so
// that equal scores and ones that differ in their last bits alone take one and
// three passes. All work-groups take part: the selection by one of them (as
// below) of 3M scores, all equal but for one that is 3 units larger, took 12.7 ms
// a call where this takes 0.19; all equal, 286 and 156 us; within 1%, 7.4 ms and
// 180 us (3M different scores: 155 us).
__global__ __launch_bounds__(kSelThreads) void sel_refine_kernel(SelLaunch S, int level) {
  __shared__ uint32_t wsum[kSelThreads / 64];
  __shared__ SelPick s_pick;
  __shared__ SelLds l;
  const SelState* const from = S.state + level - 1;
  const int old = from->mode;
  if (old != kSelWide) {
    if (blockIdx.x == 0 && threadIdx.x == 0) {
      put_group(S.state + level, from->need, from->in, from->prefix, from->shift, old);
      S.state[level].listed = from->listed;
    }
    return;
  }
  const int64_t N = live_count(S);
  const int64_t nt = (N + kSelTile - 1) / kSelTile;
  if ((int64_t)blockIdx.x >= nt && blockIdx.x > 0) return;
  const SelRange range = group_range<kSelThreads>(S, level - 1, nt, l.range);
  if (range.least == range.most) {  // counted per tile by the pass before
    if (blockIdx.x == 0 && threadIdx.x == 0) put_group(S.state + level, from->need, from->in, range.least, 0, kSelTie);
    return;
  }
  const uint64_t prefix0 = from->prefix;
  const int shift0 = from->shift, bits = shift0 < kSelDigit ? shift0 : kSelDigit;
  const SelPick p = pick_bin(S, S.hist + level * kSelBins, N, from->need, wsum, &s_pick);
  int shift = shift0 - bits;
  uint64_t prefix = (prefix0 << bits) | (uint64_t)p.bin;
  const int open = 64 - __clzll((long long)(range.least ^ range.most));  // bits in which the old group's keys differ
  if (open < shift) {  // then the digit is one bin: the group is as it was
    shift = open;
    prefix = range.least >> open;
  }
  const int mode = group_mode(p.need, p.in_bin, shift, level);
  if (blockIdx.x == 0 && threadIdx.x == 0) put_group(S.state + level, p.need, p.in_bin, prefix, shift, mode);
  const uint64_t least = mode == kSelDone ? prefix : prefix + 1;
  sel_pass<false>(S, N, level, mode, prefix, shift, l, wsum,
                  [&](uint64_t key) { return (key >> shift0) == prefix0 && (key >> shift) >= least; });
}

// Work-groups of kFinThreads threads; a list's digit of kFinBits bits per pass.
constexpr int kFinThreads = 1024;
constexpr int kFinBits = 11;
constexpr int kFinBins = 1 << kFinBits;
static_assert(kFinBins == 2 * kFinThreads, "two bins per thread");

// Exclusive sum over the work-group's threads.
__device__ __forceinline__ uint32_t fin_scan(uint32_t v, uint32_t* wsum) {
  const int lane = threadIdx.x & 63, w = threadIdx.x >> 6;
  uint32_t x = v;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) wsum[w] = x;
  __syncthreads();
  uint32_t before = 0;
#pragma unroll
  for (int k = 0; k < kFinThreads / 64; ++k) before += k < w ? wsum[k] : 0;
  __syncthreads();
  return before + x - v;
}

// One radix pass over the n listed entries that match(i): their digit(i)
// counted, then the digit that holds rank `need` found, from the top
// (DESCENDING) or from the bottom. On return `need` is the rank inside that
// digit and `in` its entries.
template <bool DESCENDING, class Match, class Digit>
__device__ __forceinline__ uint32_t fin_pass(uint32_t n, Match match, Digit digit, int64_t& need, uint32_t& in,
                                             uint32_t* h, uint32_t* wsum, int64_t* pick) {
  h[threadIdx.x] = h[threadIdx.x + kFinThreads] = 0;
  __syncthreads();
  for (uint32_t i = threadIdx.x; i < n; i += kFinThreads)
    if (match(i)) atomicAdd(&h[digit(i)], 1u);
  __syncthreads();
  const int d0 = DESCENDING ? kFinBins - 1 - 2 * (int)threadIdx.x : 2 * (int)threadIdx.x;
  const int d1 = DESCENDING ? d0 - 1 : d0 + 1;
  const uint32_t c0 = h[d0], c1 = h[d1];
  const int64_t before = fin_scan(c0 + c1, wsum);
  if (before < need && need <= before + c0 + c1) {
    const bool second = need > before + c0;
    pick[0] = second ? d1 : d0;
    pick[1] = need - before - (second ? c0 : 0);
    pick[2] = second ? c1 : c0;
  }
  __syncthreads();
  const uint32_t d = (uint32_t)pick[0];
  need = pick[1];
  in = (uint32_t)pick[2];
  __syncthreads();
  return d;
}

// The rest of the selection. A list is one work-group's: the candidates of
// 1/64 of an octave of scores (about 5,000 for 1.2M of 3M Gaussians), or at
// most kSelLongList, bound by latency (4 to 10 us). It is longer only where
// more rows than that agree in the 43 bits that the histogram and three digits
// resolve (keys of 44 bits and more: scores of 2048 and above) and still differ;
// then a pass over it takes about 0.8 ms for each million of its rows. The rows
// of one key are taken by all work-groups, each of which finds the last one
// from the tile counts (1,465 words for 3M rows).
constexpr int kFinGrid = 256;

__global__ __launch_bounds__(kFinThreads) void sel_finish_kernel(SelLaunch S) {
  __shared__ uint32_t h[kFinBins];
  __shared__ uint32_t wsum[kFinThreads / 64];
  __shared__ int64_t pick[3];
  const SelState* const st = S.state + kSelLevels - 1;
  int mode = st->mode;
  int64_t need = st->need;
  uint64_t key = st->prefix;  // kSelTie: the one key
  if (mode == kSelLast) {
    __shared__ SelRange wave[kFinThreads / 64];
    const SelRange r = group_range<kFinThreads>(S, kSelLevels - 1, (live_count(S) + kSelTile - 1) / kSelTile, wave);
    mode = r.least == r.most ? kSelTie : kSelList;
    if (mode == kSelTie) key = r.least;
  }
  if (mode == kSelList) {
    if (blockIdx.x > 0) return;
    const uint32_t n = st->listed;
    const uint64_t* keys = S.ckeys;
    const int32_t* rows = S.crows;
    int shift = st->shift;
    uint64_t prefix = key;  // the bits that every key of the list shares
    uint32_t in = n;
    while (shift > 0 && need < (int64_t)in) {
      const int bits = min(shift, kFinBits), s = shift - bits;
      const uint32_t d = fin_pass<true>(
          n, [&](uint32_t i) { return (keys[i] >> shift) == prefix; },
          [&](uint32_t i) { return (uint32_t)(keys[i] >> s) & ((1u << bits) - 1u); }, need, in, h, wsum, pick);
      prefix = (prefix << bits) | d;
      shift = s;
    }
    // `in` entries share the prefix, `need` of them are taken: all, or (equal
    // keys) those of the lowest rows
    uint32_t last = 0xFFFFFFFFu;
    if (need < (int64_t)in) {
      uint32_t rp = 0;
      int rs = 33;
      while (rs > 0) {
        rs -= kFinBits;
        const uint32_t d = fin_pass<false>(
            n, [&](uint32_t i) { return keys[i] == prefix && (rs >= 22 || ((uint32_t)rows[i] >> (rs + kFinBits)) == rp); },
            [&](uint32_t i) { return ((uint32_t)rows[i] >> rs) & (kFinBins - 1u); }, need, in, h, wsum, pick);
        rp = (rp << kFinBits) | d;
      }
      last = rp;
    }
    for (uint32_t i = threadIdx.x; i < n; i += kFinThreads) {
      const uint64_t q = keys[i] >> shift;
      if (q > prefix || (q == prefix && (uint32_t)rows[i] <= last)) S.mask[rows[i]] = 1;
    }
  } else if (mode == kSelTie) {
    // the row of the last tie taken: its tile from the counts, then the tile
    const int64_t N = live_count(S);
    const int64_t nt = (N + kSelTile - 1) / kSelTile;
    const int64_t per = (nt + kFinThreads - 1) / kFinThreads, t0 = threadIdx.x * per;
    uint32_t c = 0;
    for (int64_t k = 0; k < per; ++k)
      if (t0 + k < nt) c += S.tile_counts[t0 + k];
    int64_t before = fin_scan(c, wsum);
    if (before < need && need <= before + c) {
      for (int64_t k = 0; k < per; ++k) {
        const uint32_t tc = t0 + k < nt ? S.tile_counts[t0 + k] : 0;
        if (need <= before + tc) {
          pick[0] = t0 + k;
          pick[1] = need - before;
          break;
        }
        before += tc;
      }
    }
    __syncthreads();
    static_assert(kSelTile == 2 * kFinThreads, "two rows of the tile per thread");
    const int64_t g0 = pick[0] * kSelTile + 2 * threadIdx.x;
    const bool a = g0 < N && key_of(S, g0) == key, b = g0 + 1 < N && key_of(S, g0 + 1) == key;
    const int64_t r = (int64_t)fin_scan((a ? 1u : 0u) + (b ? 1u : 0u), wsum), want = pick[1];
    if (a && r + 1 == want) pick[2] = g0;
    if (b && r + (a ? 2 : 1) == want) pick[2] = g0 + 1;
    __syncthreads();
    const int64_t last = pick[2];
    for (int64_t g = (int64_t)blockIdx.x * kFinThreads + threadIdx.x; g <= last; g += (int64_t)gridDim.x * kFinThreads)
      if (key_of(S, g) == key) S.mask[g] = 1;
  }
}

}  // namespace

// Shape of the contribution sweep. More rounds of kSelThreads entries per
// chunk let the LDS table merge more of a Gaussian's image rows, fewer give
// short lists enough work-groups (2048 fit the chip). Entries beyond half the
// 256 MB Infinity Cache are read past it (non-temporal), which leaves it to
// the map lines; smaller lists may still be in it. Whole call, rounds 4 / 8 /
// 16 / 32: 0.7M entries 28.6 / 30.2 / 35.9 / 50.6 us, 3.5M 46.5 / 44.0 / 45.6
// / 58.1, 10.5M (non-temporal) 85 / 83 / 89 / 86, 35M 259 / 252 / 245 / 252,
// 106M 792 / 764 / 739 / 717; plain loads at the best: 3.5M 44.0 (44.5
// non-temporal), 10.5M 88, 35M 260, 106M 784. A work-group per chunk instead
// of 2048 sweeping work-groups: 106M 717 -> 696, 10.5M 83 -> 87.
struct ScatterShape {
  int rounds;
  bool nt;
  int64_t grid;
};

ScatterShape scatter_shape(int64_t n) {
  const int64_t m = int64_t(1) << 20;
  return ScatterShape{n < 2 * m ? 4 : (n < 16 * m ? 8 : (n < 64 * m ? 16 : 32)), n >= 8 * m,
                      n < 16 * m ? (int64_t)kSelScatterGrid : m};
}

hipError_t launch_select(const SelLaunch& S, hipStream_t s) {
  const int grid = S.grid;
  hipLaunchKernelGGL(sel_clear_kernel, dim3(grid), dim3(kSelThreads), 0, s, S);
  if (S.n_contrib > 0) {
    const ScatterShape sh = scatter_shape(S.n_contrib);
    const int rounds = sh.rounds;
    const bool nt = sh.nt;
    const int64_t chunks = (S.n_contrib + rounds * kSelThreads - 1) / (rounds * kSelThreads);
    const dim3 g((unsigned)(chunks < sh.grid ? chunks : sh.grid)), b(kSelThreads);
    const bool lds = S.n_views <= kSelLdsViews;
    const size_t bytes = lds ? (size_t)S.n_views * sizeof(SelView) : 0;
    if (lds && nt) hipLaunchKernelGGL((sel_scatter_kernel<true, true>), g, b, bytes, s, S, rounds);
    else if (lds) hipLaunchKernelGGL((sel_scatter_kernel<true, false>), g, b, bytes, s, S, rounds);
    else if (nt) hipLaunchKernelGGL((sel_scatter_kernel<false, true>), g, b, 0, s, S, rounds);
    else hipLaunchKernelGGL((sel_scatter_kernel<false, false>), g, b, 0, s, S, rounds);
  }
  hipLaunchKernelGGL(sel_hist_kernel, dim3(grid < kSelHistGrid ? grid : kSelHistGrid), dim3(kSelThreads), 0, s, S);
  hipLaunchKernelGGL(sel_collect_kernel, dim3(grid), dim3(kSelThreads), 0, s, S);
  for (int level = 1; level < kSelLevels; ++level)
    hipLaunchKernelGGL(sel_refine_kernel, dim3(grid), dim3(kSelThreads), 0, s, S, level);
  hipLaunchKernelGGL(sel_finish_kernel, dim3(grid < kFinGrid ? grid : kFinGrid), dim3(kFinThreads), 0, s, S);
  return hipGetLastError();
}

}  // namespace igsp
