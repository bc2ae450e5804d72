// k_emit.hip -- the end of a selection: from the staged keys of the k-th key's bin to the ascending
// index list and, in the fused steps, the exact values and the reset, in one kernel.
//
// Each workgroup owns a range of coordinates and needs nothing from another one: the keys above the
// bin are known from the digit pass (a bit in the output bitmap and
// a count per range, whose sum over the ranges before its own is the workgroup's output offset), and
// every workgroup finds the cut inside the bin by itself, since the bin holds about a hundred keys:
//   1. A key and its coordinate make one 64-bit word, key first and the lower coordinate larger,
//      so the words are distinct and the selection is the k largest of them. The bin's words (in
//      LDS) are cut down by 10-bit histograms until at most 256 are left, and ranked against each
//      other: the need-th largest is the cut.
//   2. The range's bitmap words; the bin's words at or above the cut set their bit if they are in the
//      range and are counted if before it.
//   3. Bits become indices; the workgroup's own indices are gathered and reset.
// One kernel instead of four (digit 3 in one workgroup, marking, emission with a look-back,
// gather), at about 4.6 us each however little they do.
// When the bin does not fit the LDS (ties: a zero sketch, a diverged one), or the pruned pass fell
// short of k candidates and the list is every coordinate's keys, the workgroups first settle the list together
// (settle_list): every pass reads it once, so its time grows with the list alone. Ties of nearly all
// coordinates, r = 1, pruned: 0.58 ms at 14.7M, 3.1 at 140M, 21 at 537M, where every workgroup reading the
// whole list took 8.8, 162 and 1,556; 113 us at 100,003 (107 so).
// Short of k the first pass estimates the keys: the selection takes 1,318 us at 14.7M, r = 5, c = 1.47M and
// 933 at 25.6M, c = 256,000 (the full estimate read directly: 1,065 and 695).
#include <algorithm>

#include "gs_internal.hpp"
#include "gs_select.hpp"

namespace gs {
namespace {

#define GS_FOR_ROWS(M) \
  M(1) M(2) M(3) M(4) M(5) M(6) M(7) M(8) M(9) M(10) M(11) M(12) M(13) M(14) M(15) M(16)

constexpr int kBlock = 1024;
constexpr int kBucketCap = 8192;   // words of the k-th key's bin kept in LDS
constexpr int kRankCap = 256;      // words ranked against each other

struct EmitArgs {
  const uint32_t* list_key;   // staged keys of the bin
  const int32_t* list_idx;    // and their coordinates
  const uint32_t* list0_key;  // those of the first digit's bin
  const int32_t* list0_idx;
  uint32_t* bitmap;
  uint32_t* counts;
  SelectCtl* ctl;
  uint32_t* hist;             // histograms cleared here for the next call
  uint32_t* hist2;
  const float* merged;
  uint32_t* all_keys;         // short of k: every coordinate's key (list0_key)
  const uint32_t* rnd;        // HEAVYMIX: the draws, or null
  int32_t* out;
  int64_t* n_heavy;
  double* l2sq;
  int64_t d, range;
  uint32_t k;
  int level;
};

__device__ __forceinline__ uint64_t word_of(uint32_t key, uint32_t ix) {
  return ((uint64_t)key << 32) | (0xffffffffu - ix);
}

struct Shared {
  union {
    uint64_t bucket[kBucketCap];
    float rows[kBlock * kMaxRows];  // estimate_any's, where no bucket is held
  };
  uint64_t fin[kRankCap];
  uint32_t h[1024];
  uint32_t shw[kBlock / 64];
  uint32_t res[2];
  uint64_t cut;
  SettlePass pass;
  uint32_t n, before, last, item;
};

// The `need`-th largest of the n words in the bucket, all of them in [lo, hi].
__device__ __forceinline__ uint64_t nth_largest(Shared& sh, uint64_t lo, uint64_t hi, uint32_t need, uint32_t n) {
  auto each = [&](auto f) {  // f(a word?, word), in the same number of rounds for every thread
    for (uint32_t t0 = 0; t0 < n; t0 += kBlock) {
      const uint32_t t = t0 + threadIdx.x;
      f(t < n, t < n ? sh.bucket[t] : 0ull);
    }
  };
  uint32_t n_in = n;
  while (n_in > (uint32_t)kRankCap) {  // the words are distinct, so the interval is wider than 2^8
    const int bits = 64 - __clzll((long long)(hi - lo));
    const int shift = bits > 10 ? bits - 10 : 0;
    for (int b = threadIdx.x; b < 1024; b += kBlock) sh.h[b] = 0u;
    __syncthreads();
    each([&](bool ok, uint64_t w) {
      const bool in = ok && w >= lo && w <= hi;
      hist_add(sh.h, in, in ? (uint32_t)((w - lo) >> shift) : 0u);
    });
    __syncthreads();
    find_bucket<kBlock, 1024>(sh.h, true, need, sh.shw, sh.res);
    const uint64_t b = sh.res[0];
    n_in = sh.h[b];
    need -= sh.res[1];
    lo += b << shift;
    const uint64_t top = lo + ((1ull << shift) - 1ull);
    hi = top < hi ? top : hi;
    __syncthreads();
  }
  if (threadIdx.x == 0) sh.n = 0u;
  __syncthreads();
  each([&](bool ok, uint64_t w) {
    if (ok && w >= lo && w <= hi) {
      const uint32_t pos = atomicAdd(&sh.n, 1u);
      if (pos < (uint32_t)kRankCap) sh.fin[pos] = w;
    }
  });
  __syncthreads();
  const uint32_t nf = min(sh.n, (uint32_t)kRankCap);  // == n_in
  if (threadIdx.x < nf) {
    const uint64_t w = sh.fin[threadIdx.x];
    uint32_t rank = 0;
    for (uint32_t b = 0; b < nf; ++b) rank += sh.fin[b] > w ? 1u : 0u;
    if (rank == need - 1) sh.cut = w;
  }
  __syncthreads();
  return sh.cut;
}

// ------------------------------------------------------------------------------------
// A list too long for the LDS is settled by all workgroups together, in passes over it: 10 bits of
// the words a pass until the cut is known, then a pass that marks what is selected in the output bitmap
// and counts it per range. A pass is cut into items that the workgroups claim; the one whose items
// complete a pass finds the digit and opens the next. A workgroup that finds no item left waits
// for that, so only for items that running workgroups hold: those not yet launched are not needed (they find
// the passes done, or help), and no wait depends on them. The waits are bounded all the same.
constexpr int kSettleUnroll = 8;                           // entries per thread and round
constexpr int64_t kSettleRound = kSettleUnroll * kBlock;
constexpr uint32_t kMaxPolls = 1u << 20;                   // about a second

template <typename T>
__device__ __forceinline__ T load_agent(const T* p) {
  return __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

// The word of an entry: the key's distance from klo, then the coordinate from the last one down,
// in as many bits (ib) as coordinates have.
struct List {
  const uint32_t* key;
  const int32_t* idx;  // null: entry t is coordinate t
  int64_t n;
  uint32_t klo, width;  // entries with keys in [klo, klo + width] count
  uint32_t last;        // d - 1
  int ib;
  __device__ __forceinline__ uint64_t word(uint32_t k, uint32_t ix) const {
    return ((uint64_t)(k - klo) << ib) | (last - ix);
  }
};

// Items of `chunk` entries (a multiple of 64): some for every workgroup, none short of a round.
__device__ __forceinline__ int64_t settle_chunk(int64_t n) {
  const int64_t per = n / 2048;
  return (per / kSettleRound + 1) * kSettleRound;
}

// f(a listed entry?, word, coordinate) for the entries of item `it`, in as many rounds for every thread.
template <class F>
__device__ __forceinline__ void each_entry(const List& l, int64_t it, F f) {
  const int64_t chunk = settle_chunk(l.n), end = min(l.n, (it + 1) * chunk);
  for (int64_t t0 = it * chunk; t0 < end; t0 += kSettleRound) {
    uint32_t kk[kSettleUnroll], ii[kSettleUnroll];
#pragma unroll
    for (int m = 0; m < kSettleUnroll; ++m) {
      const int64_t t = min(t0 + (int64_t)m * kBlock + threadIdx.x, l.n - 1);
      kk[m] = l.key[t];
      ii[m] = l.idx ? (uint32_t)l.idx[t] : (uint32_t)t;
    }
    __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the adds
#pragma unroll
    for (int m = 0; m < kSettleUnroll; ++m) {
      const bool in = t0 + (int64_t)m * kBlock + threadIdx.x < end && kk[m] - l.klo <= l.width;
      f(in, l.word(kk[m], ii[m]), ii[m]);
    }
  }
}

// The same for a list that is not there yet, every coordinate's keys: they are estimated, with all R cell
// loads of kEstimate coordinates in flight per thread, and written.
template <int R, class F>
__device__ __forceinline__ void each_estimate(const EmitArgs& a, const HashSet& hs, const List& l, int64_t it, F f) {
  constexpr int kEstimate = R <= 8 ? 2 : 1;
  RowConst kr[R];
#pragma unroll
  for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
  const double theta = a.rnd ? a.ctl->theta : 0.0;
  const int64_t chunk = settle_chunk(l.n), end = min(l.n, (it + 1) * chunk);
  for (int64_t t0 = it * chunk; t0 < end; t0 += kEstimate * kBlock) {
    float e[kEstimate];
#pragma unroll
    for (int m = 0; m < kEstimate; ++m)  // a column is valid for any hash value
      e[m] = estimate_val<R>(kr, a.merged, (uint32_t)(t0 + m * kBlock + threadIdx.x));
#pragma unroll
    for (int m = 0; m < kEstimate; ++m) {
      const int64_t t = t0 + m * kBlock + threadIdx.x;
      const bool in = t < end;
      uint32_t key = abs_key(e[m]);
      if (a.rnd) key = (double)e[m] * (double)e[m] >= theta ? 0x80000000u | key : a.rnd[min(t, l.n - 1)] >> 1;
      if (in) a.all_keys[t] = key;
      f(in, l.word(key, (uint32_t)t), (uint32_t)t);
    }
  }
}

// The selection's `need` largest words of the list marked in the bitmap and counted per range.
// False when a wait ran out (the control block in use by a call that overlaps this one).
// R > 0: without indices, the list is every coordinate's keys, which the first pass estimates.
template <int R>
__device__ __forceinline__ bool settle_list(const EmitArgs& a, const HashSet& hs, Shared& sh, const List& l,
                                            uint32_t need) {
  SelectCtl* const ctl = a.ctl;
  Settle& g = ctl->settle;
  const int64_t items = (l.n + settle_chunk(l.n) - 1) / settle_chunk(l.n);
  const int nr = (int)gridDim.x;
  for (int p = 0; p < kSettlePasses; ++p) {
    if (threadIdx.x == 0) {
      sh.pass = SettlePass{0, (((uint64_t)l.width + 1) << l.ib) - 1, need, kSettleDigit};
      if (p > 0) {
        uint32_t polls = 0;
        while (load_agent(&g.open) < (uint32_t)p && ++polls < kMaxPolls) __builtin_amdgcn_s_sleep(4);
        if (polls >= kMaxPolls) {
          sh.pass.kind = kSettleFailed;
        } else {
          __threadfence();  // what the pass before wrote
          const SettlePass* q = &g.pass[p];
          sh.pass = SettlePass{load_agent(&q->lo), load_agent(&q->hi), load_agent(&q->need), load_agent(&q->kind)};
        }
      }
    }
    for (int b = threadIdx.x; b < 1024; b += kBlock) sh.h[b] = 0u;
    __syncthreads();
    const SettlePass q = sh.pass;
    if (q.kind == kSettleFailed) return false;
    if (q.kind == kSettleDone) return true;
    const int bits = 64 - __clzll((long long)(q.hi - q.lo));
    const int shift = bits > 10 ? bits - 10 : 0;
    uint32_t mine = 0;  // items taken (block-uniform)
    for (;;) {
      if (threadIdx.x == 0) sh.item = atomicAdd(&g.claim[p], 1u);
      __syncthreads();
      const int64_t it = sh.item;
      __syncthreads();
      if (it >= items) break;
      ++mine;
      if (q.kind == kSettleDigit) {
        auto add = [&](bool in, uint64_t w, uint32_t) {
          const bool take = in && w >= q.lo && w <= q.hi;
          hist_add(sh.h, take, take ? (uint32_t)((w - q.lo) >> shift) : 0u);
        };
        bool listed = true;
        if constexpr (R > 0) {
          if (p == 0 && !l.idx) {
            listed = false;
            each_estimate<R>(a, hs, l, it, add);
          }
        }
        if (listed) each_entry(l, it, add);
      } else {
        each_entry(l, it, [&](bool in, uint64_t w, uint32_t ix) {
          const bool take = in && w >= q.lo;
          if (l.idx) {
            if (take) atomicOr(&a.bitmap[ix >> 5], 1u << (ix & 31u));
          } else if (const uint64_t bal = __ballot(take)) {  // 64 coordinates from a multiple of 64
            const uint32_t half = threadIdx.x & 1 ? (uint32_t)(bal >> 32) : (uint32_t)bal;
            const uint32_t first = __shfl(ix, 0) >> 5;
            if ((threadIdx.x & 63) < 2 && half) atomicOr(&a.bitmap[first + (threadIdx.x & 1)], half);
          }
          const uint32_t b = take ? ix / (uint32_t)a.range : 0u;
          if (nr <= 1024)
            hist_add(sh.h, take, b);
          else if (take)
            atomicAdd(&a.counts[b], 1u);
        });
      }
    }
    if (mine == 0) continue;
    __syncthreads();
    uint32_t* const to = q.kind == kSettleDigit ? g.hist : a.counts;
    for (int b = threadIdx.x; b < (q.kind == kSettleDigit || nr > 1024 ? 1024 : nr); b += kBlock)
      if (const uint32_t c = sh.h[b]) atomicAdd(&to[b], c);
    __syncthreads();
    if (threadIdx.x == 0) {
      __threadfence();
      sh.last = atomicAdd(&g.done[p], mine) + mine == (uint32_t)items ? 1u : 0u;
      __threadfence();
    }
    __syncthreads();
    if (!sh.last) continue;
    SettlePass next{q.lo, q.hi, q.need, kSettleDone};
    if (q.kind == kSettleDigit) {
      for (int b = threadIdx.x; b < 1024; b += kBlock) {
        sh.h[b] = load_agent(&g.hist[b]);
        g.hist[b] = 0u;
      }
      __syncthreads();
      find_bucket<kBlock, 1024>(sh.h, true, q.need, sh.shw, sh.res);
      const uint64_t b = sh.res[0];
      next.need -= sh.res[1];
      next.lo += b << shift;
      next.hi = min(q.hi, next.lo + ((1ull << shift) - 1ull));
      // all of the bin is taken (or it is one word): its first word is the cut
      next.kind = next.need == sh.h[b] ? kSettleMark : kSettleDigit;
    }
    if (threadIdx.x == 0 && p + 1 < kSettlePasses) {
      g.pass[p + 1] = next;
      __threadfence();
      __hip_atomic_store(&g.open, (uint32_t)(p + 1), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    }
    __syncthreads();
  }
  return false;
}

__device__ __forceinline__ uint32_t wave_sum(uint32_t x) {
#pragma unroll
  for (int o = 32; o > 0; o >>= 1) x += __shfl_xor(x, o, 64);
  return x;
}

// Entries idx[t0], idx[t0 + step], ... below n, a lane group of ga.gl threads each.
__device__ __forceinline__ void gather_range(const GatherArgs& ga, const HashSet& hs, const float* __restrict__ merged,
                                             const int32_t* __restrict__ idx, int64_t t0, int64_t step, int64_t n,
                                             float* rows) {
  const int sub = (int)(threadIdx.x & (unsigned)(ga.gl - 1));
  for (int64_t t = t0; t < n; t += step) {
    const int32_t i = idx[t];
    if (ga.op != kGatherSketch) {
      gather_entry(ga, i, t, sub);
      continue;
    }
    ga.values[t] = estimate_any(hs, merged, (uint32_t)i, rows + threadIdx.x * kMaxRows);
#pragma nounroll
    for (int j = 0; j < hs.r; ++j) {
      uint32_t col, sflip;
      hash_ij(hs, j, (uint32_t)i, col, sflip);
      const int64_t cell = (int64_t)j * hs.c + col;
      ga.acc[cell] = 0.0;
      atomicAnd(&ga.claim[cell >> 5], ~(1u << (cell & 31)));
    }
  }
}

// Entries [p0, p0 + n) of the index list, written by this block.
__device__ __forceinline__ void gather_own(const EmitArgs& a, const HashSet& hs, const GatherArgs& ga, Shared& sh,
                                           int64_t p0, uint32_t n) {
  if (ga.op == kGatherNone) return;
  __syncthreads();
  gather_range(ga, hs, a.merged, a.out, p0 + threadIdx.x / (unsigned)ga.gl, kBlock / (unsigned)ga.gl, p0 + n,
               sh.rows);
}

constexpr int kGatherBlock = 256;
__global__ void __launch_bounds__(kGatherBlock) k_gather_reset(const int32_t* __restrict__ idx, int64_t k, HashSet hs,
                                                               const float* __restrict__ merged, GatherArgs ga) {
  __shared__ float rows[kGatherBlock * kMaxRows];  // sketch-space values only
  const int64_t per = kGatherBlock / (unsigned)ga.gl;
  gather_range(ga, hs, merged, idx, (int64_t)blockIdx.x * per + threadIdx.x / (unsigned)ga.gl,
               (int64_t)gridDim.x * per, k, rows);
}

// Many coordinates of a worker-major state: one lane per coordinate, so that the lanes of a wave read
// one worker's row at neighbouring places, and the workers of a coordinate in groups of at most 16, a
// group's loads in flight together. NP: P up to 16; 0: any P.
template <int NP>
__global__ void __launch_bounds__(kGatherBlock) k_gather_columns(const int32_t* __restrict__ idx, int64_t k,
                                                                 GatherArgs ga) {
  constexpr int G = NP ? NP : 16, B = NP ? 1 : kMaxWorkers / G;
  const int P = NP ? NP : ga.P;
  const int64_t qs = ga.sv.qs, stride = (int64_t)gridDim.x * kGatherBlock;
  for (int64_t t = (int64_t)blockIdx.x * kGatherBlock + threadIdx.x; t < k; t += stride) {
    const int64_t i = idx[t];
    float sum[B];
#pragma unroll
    for (int b = 0; b < B; ++b) {
      const int n = P - G * b;
      if (n <= 0) break;
      float* const v = ga.v + G * b * qs + i;
      float* const u = ga.u + G * b * qs + i;
      float x[G];
#pragma unroll
      for (int q = 0; q < G; ++q) x[q] = q < n ? v[q * qs] : 0.f;
      sum[b] = tree_sum_upto<G>(x, n);
#pragma unroll
      for (int q = 0; q < G; ++q) {
        if (q >= n) break;
        v[q * qs] = 0.f;
        if (ga.reset_u) u[q * qs] = 0.f;
      }
    }
    ga.values[t] = tree_sum_upto<B>(sum, (P + G - 1) / G);
  }
}

// R: rows, where a pruned pass may have fallen short of k candidates; 0 for the full estimate's.
template <int R>
__global__ void __launch_bounds__(kBlock) k_emit(EmitArgs a, HashSet hs, GatherArgs ga) {
  extern __shared__ uint32_t bits[];  // [range / 32]
  __shared__ Shared sh;
  const int64_t lo = (int64_t)blockIdx.x * a.range, hi = min(a.d, lo + a.range);
  const uint32_t nb = a.ctl->n_stage[a.level];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (a.n_heavy) *a.n_heavy = (int64_t)a.ctl->n_heavy;
    if (a.l2sq) *a.l2sq = a.ctl->l2sq;
  }
  // the bound admitted too little: the digit pass marked nothing, and every coordinate is estimated
  const bool few = R > 0 && a.ctl->n_cand < a.k;
  const uint32_t l32 = (uint32_t)lo, width = (uint32_t)(hi - lo);
  const int nw = (int)(a.range / 32);
  const uint32_t klo = few ? 0u : a.ctl->lo[a.level], khi = few ? ~0u : a.ctl->hi[a.level];
  const uint32_t need = few ? a.k : a.ctl->need[a.level];
  const bool in_lds = !few && nb <= (uint32_t)kBucketCap;
  uint32_t before = 0;
  const int64_t words = (a.d + 31) / 32, word0 = lo / 32;
  auto load_own = [&](bool ok) {
    before = 0;
    for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kBlock) before += a.counts[t];
    for (int w = threadIdx.x; w < nw; w += kBlock) bits[w] = ok && word0 + w < words ? a.bitmap[word0 + w] : 0u;
  };
  load_own(true);
  if (threadIdx.x == 0) sh.before = 0u;
  bool ok = true;
  if (!in_lds) {
    const uint32_t last = (uint32_t)(a.d - 1);
    const List l{a.list0_key, few ? nullptr : a.list0_idx, few ? a.d : (int64_t)a.ctl->n_stage[0],
                 klo, khi - klo, last, 32 - __clz((int)(last | 1u))};
    ok = settle_list<R>(a, hs, sh, l, need);
    load_own(ok);
  }
  const int per = (nw + kBlock - 1) / kBlock, w0 = threadIdx.x * per;
  if (in_lds) {
    for (uint32_t t = threadIdx.x; t < nb; t += kBlock) sh.bucket[t] = word_of(a.list_key[t], (uint32_t)a.list_idx[t]);
    __syncthreads();
    const uint64_t cut = nth_largest(sh, (uint64_t)klo << 32, ((uint64_t)khi << 32) | 0xffffffffull, need, nb);
    for (uint32_t t = threadIdx.x; t < nb; t += kBlock) {
      const uint64_t w = sh.bucket[t];
      const uint32_t ix = 0xffffffffu - (uint32_t)w;
      if (w >= cut) {
        if (ix < l32)
          ++before;
        else if (ix - l32 < width)
          atomicOr(&bits[(ix - l32) >> 5], 1u << ((ix - l32) & 31u));
      }
    }
  } else {
    __syncthreads();
  }
  before = wave_sum(before);
  if ((threadIdx.x & 63) == 0 && before) atomicAdd(&sh.before, before);
  __syncthreads();
  uint32_t cnt = 0;
  for (int m = 0; m < per; ++m)
    if (w0 + m < nw) cnt += (uint32_t)__popc(bits[w0 + m]);
  uint32_t total;
  const uint32_t p0 = sh.before;
  uint32_t pos = p0 + block_scan_incl<kBlock>(cnt, sh.shw, total) - cnt;
  for (int m = 0; m < per; ++m) {
    uint32_t x = w0 + m < nw ? bits[w0 + m] : 0u;
    while (x) {
      const int bit = __ffs(x) - 1;
      if (pos < a.k) a.out[pos] = (int32_t)(lo + 32 * (w0 + m) + bit);
      ++pos;
      x &= x - 1u;
    }
  }
  gather_own(a, hs, ga, sh, p0, total);
  // the last workgroup to get here clears what the next call needs zero
  __syncthreads();
  if (threadIdx.x == 0) sh.last = atomicAdd(&a.ctl->emit_ticket, 1u) == gridDim.x - 1 ? 1u : 0u;
  __syncthreads();
  if (!sh.last) return;
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) a.hist[b] = 0u;
  for (int b = threadIdx.x; b < kDigitBins; b += kBlock) a.hist2[b] = 0u;
  for (unsigned b = threadIdx.x; b < gridDim.x; b += kBlock) a.counts[b] = 0u;
  if (threadIdx.x == 0) {
    a.ctl->n_stage[0] = a.ctl->n_stage[1] = 0u;
    a.ctl->emit_ticket = 0u;
  }
  if (in_lds) return;
  Settle& g = a.ctl->settle;
  if (threadIdx.x < kSettlePasses) g.claim[threadIdx.x] = g.done[threadIdx.x] = 0u;
  if (threadIdx.x == 0) g.open = 0u;
  if (!ok)
    for (int b = threadIdx.x; b < 1024; b += kBlock) g.hist[b] = 0u;
}

}  // namespace

// The emit gathers what each workgroup has written, unless one could have so much of it (the selection
// in one part of d, a layer's gradients) that it would work alone: more than 12 passes of its threads,
// in a selection of at most d/8. With all large estimates within d/256, 66M x 16 takes 10.9 ms so, 10.1
// with a gather of its own, 25.6M x 8 worker-major 1,968 and 1,662 us, 14.7M x 4 712 and 675; where they
// are spread the kernel more costs 2 us (14.7M x 4 659 and 661; 1.2M x 6, 12 passes at most, 119
// and 122). Beyond d/8 no workgroup has more than 8 times the mean (14.7M x 4, k = d/4: spread
// 1,402 and 1,437 us, in one quarter of d 1,431 and 1,454).
bool emit_gathers(int64_t d, int num_cus, int64_t k, const GatherArgs& ga) {
  return std::min(k, emit_range(d, num_cus)) * ga.gl <= 12 * kBlock || 8 * k > d;
}

hipError_t launch_emit(const HashSet& hs, int64_t d, int num_cus, const SelectBufs& b, hipStream_t s,
                       const float* merged, const uint32_t* rnd, int64_t k, int pruned, int level, int32_t* idx,
                       int64_t* n_heavy, double* l2sq, const GatherArgs* ga) {
  EmitArgs a{};
  a.range = emit_range(d, num_cus);
  a.list_key = level ? b.stage2 : b.keys;
  a.list_idx = level ? reinterpret_cast<const int32_t*>(b.stage2 + kStage2Cap) : b.stage_idx;
  a.list0_key = b.keys;
  a.list0_idx = b.stage_idx;
  a.bitmap = b.bitmap;
  a.counts = b.counts;
  a.ctl = b.ctl;
  a.hist = pruned ? b.hist_c : b.hist;
  a.hist2 = b.hist2;
  a.merged = merged;
  a.all_keys = b.keys;
  a.rnd = rnd;
  a.out = idx;
  a.n_heavy = n_heavy;
  a.l2sq = l2sq;
  a.d = d;
  a.k = (uint32_t)k;
  a.level = level;
  const unsigned blocks = (unsigned)((d + a.range - 1) / a.range);
  const size_t lds = (size_t)(a.range / 32) * sizeof(uint32_t);
  const GatherArgs g = ga ? *ga : GatherArgs{};
  switch (pruned ? hs.r : 0) {
#define GS_EMIT(R) \
  case R: hipLaunchKernelGGL(k_emit<R>, dim3(blocks), dim3(kBlock), lds, s, a, hs, g); break;
    GS_EMIT(0) GS_FOR_ROWS(GS_EMIT)
#undef GS_EMIT
    default: return hipErrorInvalidValue;
  }
  return hipGetLastError();
}

hipError_t prepare_emit() {
#define GS_EMIT(R) reinterpret_cast<const void*>(&k_emit<R>),
  for (const void* f : {GS_FOR_ROWS(GS_EMIT) reinterpret_cast<const void*>(&k_emit<0>)}) {
#undef GS_EMIT
    const hipError_t e = hipFuncSetAttribute(f, hipFuncAttributeMaxDynamicSharedMemorySize, kRangeMax / 8);
    if (e != hipSuccess) return e;
  }
  return hipSuccess;
}

hipError_t launch_gather(int num_cus, hipStream_t s, const HashSet& hs, const float* merged, const int32_t* idx,
                         int64_t k, const GatherArgs& ga) {
  // A lane per (coordinate, worker) is worth its scattered accesses only while there are too few coordinates
  // to fill the chip: at 32,768 the two cost the same (P = 4, 8, 16 at 2M, k = 20,000: 10 us, 10 and 12,
  // 15 and 19 by columns; k = 65,000: 12, 18, 34 us both; 20M, k = 65,000, P = 16: 68 us, 44 by columns; 2M,
  // k = 400,000, P = 3, 8, 16, 64: 16, 42, 93 and 1,012 us, 14, 36, 68 and 420 by columns).
  const bool columns = ga.op == kGatherWorkers && ga.sv.is == 1 && ga.P > 1 && k >= 32768;
  const int64_t per = columns ? kGatherBlock : kGatherBlock / ga.gl;
  const int64_t blocks = std::min<int64_t>((k + per - 1) / per, (columns ? 4 : 8) * num_cus);
  const dim3 grid((unsigned)blocks), block(kGatherBlock);
  if (!columns) {
    hipLaunchKernelGGL(k_gather_reset, grid, block, 0, s, idx, k, hs, merged, ga);
    return hipGetLastError();
  }
  switch (ga.P) {
#define GS_COLUMNS(P) \
  case P: hipLaunchKernelGGL(k_gather_columns<P>, grid, block, 0, s, idx, k, ga); break;
    GS_COLUMNS(2) GS_COLUMNS(3) GS_COLUMNS(4) GS_COLUMNS(5) GS_COLUMNS(6) GS_COLUMNS(7) GS_COLUMNS(8) GS_COLUMNS(9)
    GS_COLUMNS(10) GS_COLUMNS(11) GS_COLUMNS(12) GS_COLUMNS(13) GS_COLUMNS(14) GS_COLUMNS(15) GS_COLUMNS(16)
#undef GS_COLUMNS
    default: hipLaunchKernelGGL(k_gather_columns<0>, grid, block, 0, s, idx, k, ga); break;
  }
  return hipGetLastError();
}

GatherArgs gather_args(const gs_ctx* x, float* u, float* v, float* values) {
  GatherArgs a{};
  const bool rows = x->state_layout == GS_STATE_INTERLEAVED && ((((uintptr_t)u | (uintptr_t)v) & 15u) == 0);
  a.op = rows ? kGatherRows : kGatherWorkers;
  const int lanes = rows ? x->state_stride / 4 : x->P;  // at most 16 or 64
  a.gl = 1;
  while (a.gl < lanes) a.gl *= 2;
  a.P = x->P;
  a.PP = x->state_stride;
  a.reset_u = x->reset_momentum ? 1 : 0;
  a.u = u;
  a.v = v;
  a.values = values;
  a.sv = state_view(x);
  return a;
}

}  // namespace gs
