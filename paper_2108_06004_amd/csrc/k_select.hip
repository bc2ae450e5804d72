// k_select.hip -- HEAVYMIX estimate and selection (Alg. 2): the deterministic top-k and
// HEAVYMIX as printed.
//
// Estimate: est_i = median over rows of s_j(i) * S[j][h_j(i)] (register sorting network).
// Selection: the k largest keys, ties toward the lower index, output ascending. For the
// top-k the keys are the bit patterns of |est_i| (non-negative floats order like unsigned
// integers); for HEAVYMIX, heavy coordinates get 0x80000000 | bits(|est_i|) and the others
// their fill draw. The k-th key is found by a most-significant-digit radix select entirely
// on the device (no host synchronisation inside the call):
//   1. candidates: either every coordinate whose key reaches the pruned pass's sampled bound
//      (k_sample, k_heavy, then k_pruned or k_planes and k_combine: bound, heavy-cell map, survivor
//      estimates, with the candidates' histogram in fine bins), or every coordinate, from the full
//      estimate (k_unsketch, k_unsketch_hm, or k_push by tile and k_median);
//   2. k_digit2 (many blocks): each block finds the bin of the k-th key in the candidates'
//      histogram; candidates above it are taken and set their bit in the output bitmap; the bin is
//      compacted (keys and coordinates), twice where a large dense selection's bin is crowded;
//   3. k_emit (k_emit.hip): the cut inside the bin, the ascending indices, the values and the reset.
#include <algorithm>
#include <cmath>
#include <type_traits>

#include "gs_internal.hpp"
#include "gs_select.hpp"

namespace gs {
namespace {

constexpr int kBlock = 256;
constexpr int kSelBlock = 1024;

int grid_for(int64_t work_items, int per_block, int cap) {
  int64_t b = (work_items + per_block - 1) / per_block;
  if (b < 1) b = 1;
  if (b > cap) b = cap;
  return (int)b;
}

// ------------------------------------------------------------------------------------
// Step 1, full path: every coordinate is a candidate ("dense" candidates: candidate t is
// coordinate t, so no index array). The estimate, its key in cand_key[i], the digit-1
// histogram in hist, and the output bitmap cleared.

// k_unsketch's grid. Each block adds its LDS histogram into the global one with an atomic
// per non-empty bin, and the atomics of many blocks on the few well-filled bins queue at one
// address each. Up to kUnsketchSmall * kBlock * (CUs) coordinates that queue costs more than
// the blocks' parallelism gains: at most one block per CU then, each thread taking two
// coordinates per pass with all their cell loads in flight. Beyond it, four blocks per CU,
// one coordinate per thread per pass.
constexpr int kUnsketchSmall = 8;

template <int R, int U>
__global__ void __launch_bounds__(kBlock) k_unsketch(HashSet hs, const float* __restrict__ merged, int64_t d,
                                                     float* __restrict__ est, uint32_t* __restrict__ keys,
                                                     uint32_t* __restrict__ hist) {
  __shared__ uint32_t h[kDigit1Bins];
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) h[b] = 0u;
  RowConst kr[R];
#pragma unroll
  for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  const int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  uint32_t hb[R], hsg[R], db[R], dsg[R];  // raw hashes of the current i and their per-stride steps
#pragma unroll
  for (int j = 0; j < R; ++j) {
    hb[j] = mod_mersenne_affine(kr[j].a, kr[j].b, (uint32_t)i0);
    hsg[j] = mod_mersenne_affine(kr[j].a2, kr[j].b2, (uint32_t)i0);
    db[j] = mod_mersenne_affine(kr[j].a, 0u, (uint32_t)stride);
    dsg[j] = mod_mersenne_affine(kr[j].a2, 0u, (uint32_t)stride);
  }
  // U coordinates (i, i + stride, ...) per pass with all their cell loads in flight; a cell
  // column is valid for any hash value, so the loads past d need no guard
  for (int64_t ib = i0; ib < d; ib += U * stride) {
    float val[U][R];
#pragma unroll
    for (int u = 0; u < U; ++u) {
#pragma unroll
      for (int j = 0; j < R; ++j) {
        const uint32_t col = mod_c(hb[j], kr[j].c, kr[j].magic, kr[j].shift);
        val[u][j] = apply_sign(merged[(int64_t)j * hs.c + col], sign_flip_of(hsg[j]));
        hb[j] = add_mod_mersenne(hb[j], db[j]);
        hsg[j] = add_mod_mersenne(hsg[j], dsg[j]);
      }
    }
#pragma unroll
    for (int u = 0; u < U; ++u) {
      const int64_t i = ib + u * stride;
      if (i >= d) break;
      sort_net<R>(val[u]);
      const float e = median_sorted<R>(val[u]);
      if (est) est[i] = e;
      const uint32_t key = abs_key(e);
      keys[i] = key;
      atomicAdd(&h[key >> 19], 1u);  // cand_bin's coarse bins
    }
  }
  __syncthreads();
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) {
    const uint32_t n = h[b];
    if (n) atomicAdd(&hist[b], n);
  }
}

// The full estimate from k_push's row values, four coordinates per thread and pass; the rows from
// `pushed` on (no scratch for them) are read from the table. keys may be rows.p[0]: a
// thread reads its coordinates' values before it writes their keys.
constexpr int kMedianBlock = 1024;
template <int R, bool HM>
__global__ void __launch_bounds__(kMedianBlock) k_median(HashSet hs, const float* __restrict__ merged, int64_t d,
                                                         RowValues rows, int pushed, const uint32_t* __restrict__ rnd,
                                                         float* __restrict__ est, uint32_t* keys,
                                                         uint32_t* __restrict__ hist, SelectCtl* __restrict__ ctl) {
  __shared__ uint32_t h[kDigit1Bins];
  __shared__ uint32_t nh;
  for (int b = threadIdx.x; b < kDigit1Bins; b += kMedianBlock) h[b] = 0u;
  if (threadIdx.x == 0) nh = 0u;
  const double theta = HM ? ctl->theta : 0.0;
  __syncthreads();
  uint32_t mine = 0;
  constexpr int U = 4;
  for (int64_t b0 = (int64_t)blockIdx.x * kMedianBlock * U; b0 < d; b0 += (int64_t)gridDim.x * kMedianBlock * U) {
    float val[U][R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      if (j < pushed) {
#pragma unroll
        for (int m = 0; m < U; ++m) {
          const int64_t i = b0 + m * kMedianBlock + threadIdx.x;
          val[m][j] = i < d ? rows.p[j][i] : 0.f;
        }
      } else {
        const RowConst k = row_const(hs, j);
#pragma unroll
        for (int m = 0; m < U; ++m) {  // a column is valid for any hash value
          uint32_t col, sflip;
          hash_row(k, (uint32_t)(b0 + m * kMedianBlock + threadIdx.x), col, sflip);
          val[m][j] = apply_sign(merged[(int64_t)j * k.c + col], sflip);
        }
      }
    }
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int64_t i = b0 + m * kMedianBlock + threadIdx.x;
      if (i >= d) break;
      sort_net<R>(val[m]);
      const float e = median_sorted<R>(val[m]);
      if (est) est[i] = e;
      uint32_t key = abs_key(e);
      if constexpr (HM) {
        const bool heavy = (double)e * (double)e >= theta;
        key = heavy ? 0x80000000u | key : rnd[i] >> 1;
        mine += heavy ? 1u : 0u;
      }
      keys[i] = key;
      atomicAdd(&h[key >> (HM ? 20 : 19)], 1u);  // cand_bin's coarse bins
    }
  }
  if (HM && mine) atomicAdd(&nh, mine);
  __syncthreads();
  for (int b = threadIdx.x; b < kDigit1Bins; b += kMedianBlock) {
    const uint32_t n = h[b];
    if (n) atomicAdd(&hist[b], n);
  }
  if (HM && threadIdx.x == 0 && nh) atomicAdd(&ctl->n_heavy, (unsigned long long)nh);
}

// ------------------------------------------------------------------------------------
// Step 2: the digit pass. Candidates are either the pruned pass's (keys in cand_key, coordinates in
// cand_idx, fine bins in hist_c) or dense (after the full estimate: every coordinate, key in
// cand_key, coarse bins in hist).

constexpr int kDigit2Block = 1024;           // threads per k_digit2 block
constexpr int kStageBuf = 8 * kDigit2Block;  // per-block LDS buffer of k_digit2 (keys and coordinates)
constexpr int64_t kTwoMinK = 16384;          // dense selections beyond this k take a second digit pass
constexpr int kCountMax = 1024;              // emit ranges counted in LDS: all of them up to d = 2^29

struct DigitArgs {
  const uint32_t* key;   // [n] candidate keys; dense: key of coordinate t at t
  const int32_t* idx;    // [n] their coordinates; dense: null
  SelectCtl* ctl;
  const uint32_t* hist;  // [kDigit1Bins] level 0, [kDigitBins] level 1
  uint32_t* hist_next;   // [kDigitBins] next digit of the staged keys, or null
  uint32_t* out_key;     // staged keys of the bin
  int32_t* out_idx;
  int64_t cap;           // room in out_key and out_idx
  uint32_t* bitmap;      // keys above the bin set their bit (dense: every word is written)
  uint32_t* counts;      // and are counted per emit range
  int64_t d, range;
  int64_t slice;         // dense: keys per block (a multiple of 64)
  uint32_t slices;       // and blocks per emit range
  uint32_t k;
  int pruned, hm, level;
};

// Many blocks: every block finds the bin of the k-th key in the histogram (block 0 records it);
// keys above it are taken (their bit in the output bitmap: an atomic each, or for dense candidates a
// ballot per 64 coordinates; and the count of their emit range; a kernel of its own for each: 1.3 us
// less at d = 4.1M than one that tests); the bin is compacted, key and coordinate, through an LDS buffer per
// block and one global atomic per flush, with a histogram of the next ten bits on request. Level 1
// runs the same over the keys staged by level 0, by that next digit: a dense bin holds percents
// of d, too many for the emit's workgroups to read one by one.
// When the pruned pass left fewer than k candidates there is nothing to find here: the emit estimates
// every coordinate.
template <bool DENSE>
__global__ void __launch_bounds__(kDigit2Block) k_digit2(DigitArgs a) {
  __shared__ uint32_t buf_key[kStageBuf];
  __shared__ int32_t buf_idx[kStageBuf];
  __shared__ uint32_t h[kDigitBins];
  __shared__ uint32_t cnt[DENSE ? 1 : kCountMax];
  __shared__ uint32_t shw[kDigit2Block / 64];
  __shared__ uint32_t res[2];
  __shared__ uint32_t bn, gbase;
  SelectCtl* const ctl = a.ctl;
  const int64_t grid = gridDim.x;
  if (!DENSE && a.pruned && ctl->n_cand < a.k) return;
  int64_t n;
  uint32_t need = a.k, klo, khi;
  if (a.level == 0) {
    n = DENSE ? a.d : (int64_t)ctl->n_cand;
    find_bucket<kDigit2Block, kDigit1Bins>(a.hist, true, need, shw, res);
    const CandBins bins = cand_bins(a.pruned ? ctl->tau0 : 0u, a.hm != 0, a.hm ? ctl->theta : 0.0, a.pruned != 0);
    klo = (uint32_t)cand_bin_lo(bins, res[0]);
    khi = (uint32_t)(cand_bin_lo(bins, res[0] + 1u) - 1ull);
  } else {
    n = (int64_t)ctl->n_stage[0];
    need = ctl->need[0];
    const uint32_t lo0 = ctl->lo[0], w = ctl->hi[0] - lo0;  // level 0's bin is 2^19 or 2^20 keys wide
    const int sh = 32 - __clz(w) - 10;
    find_bucket<kDigit2Block, kDigitBins>(a.hist, true, need, shw, res);
    klo = lo0 + (res[0] << sh);
    khi = klo + ((1u << sh) - 1u);
  }
  need -= res[1];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->need[a.level] = need;
    ctl->lo[a.level] = klo;
    ctl->hi[a.level] = khi;
  }
  const uint32_t kw = khi - klo;
  const int nsh = 32 - __clz(kw | 1u) - 10;  // shift of the next digit (with hist_next: kw is 2^19 - 1 or 2^20 - 1)
  const int lane = threadIdx.x & 63;
  const int nr = DENSE ? 1 : (int)((a.d + a.range - 1) / a.range);
  for (int b = threadIdx.x; b < kDigitBins; b += kDigit2Block) h[b] = 0u;
  for (int b = threadIdx.x; b < (DENSE ? 1 : kCountMax); b += kDigit2Block) cnt[b] = 0u;
  if (threadIdx.x == 0) bn = 0u;
  __syncthreads();
  const uint32_t range = (uint32_t)a.range;
  // a dense slice lies in one emit range, and its words of the bitmap are its own
  const int64_t per = DENSE ? a.slice : (n + grid - 1) / grid;
  const int64_t r0 = DENSE ? (int64_t)(blockIdx.x / a.slices) * a.range : 0;
  const int64_t lo = DENSE ? r0 + blockIdx.x % a.slices * per : blockIdx.x * per;
  const int64_t hi = min(DENSE ? min(n, r0 + a.range) : n, lo + per);
  uint32_t mine = 0;  // dense: this wave's keys above the bin
  constexpr int V = 4;
  for (int64_t c0 = lo; c0 < hi; c0 += (int64_t)V * kDigit2Block) {  // block-uniform
    uint32_t key[V], ix[V];
#pragma unroll
    for (int m = 0; m < V; ++m) {
      const int64_t t = c0 + (int64_t)m * kDigit2Block + threadIdx.x;
      key[m] = t < hi ? a.key[t] : 0u;
      ix[m] = !DENSE && t < hi ? (uint32_t)a.idx[t] : (uint32_t)t;
    }
#pragma unroll
    for (int m = 0; m < V; ++m) {
      const int64_t t = c0 + (int64_t)m * kDigit2Block + threadIdx.x;
      const bool above = t < hi && key[m] > khi;
      if constexpr (DENSE) {
        const uint64_t bal = __ballot(above);
        mine += (uint32_t)__popcll(bal);
        const int64_t w = (t - lane) / 32 + lane;  // slices are multiples of 64 coordinates
        if (lane < 2 && t - lane + 32 * lane < hi) a.bitmap[w] = (uint32_t)(lane ? bal >> 32 : bal);
      } else {
        if (above) atomicOr(&a.bitmap[ix[m] >> 5], 1u << (ix[m] & 31u));
        if (nr <= kCountMax)
          hist_add(cnt, above, above ? ix[m] / range : 0u);
        else if (above)
          atomicAdd(&a.counts[ix[m] / range], 1u);
      }
      const bool take = t < hi && key[m] - klo <= kw;
      if (a.hist_next) hist_add(h, take, take ? (key[m] - klo) >> nsh : 0u);
      const uint64_t bal = __ballot(take);
      uint32_t wbase = 0u;
      if (lane == 0 && bal) wbase = atomicAdd(&bn, (uint32_t)__popcll(bal));
      wbase = __shfl(wbase, 0);
      if (take) {
        const uint32_t pos = wbase + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        buf_key[pos] = key[m];
        buf_idx[pos] = (int32_t)ix[m];
      }
    }
    __syncthreads();
    const uint32_t nb = bn;  // < kStageBuf / 2 + V * kDigit2Block <= kStageBuf
    if (nb >= (uint32_t)(kStageBuf / 2) || (c0 + (int64_t)V * kDigit2Block >= hi && nb > 0)) {
      if (threadIdx.x == 0) gbase = atomicAdd(&ctl->n_stage[a.level], nb);
      __syncthreads();
      const int64_t g0 = gbase;
      for (uint32_t t = threadIdx.x; t < nb; t += kDigit2Block) {
        if (g0 + t < a.cap) {
          a.out_key[g0 + t] = buf_key[t];
          a.out_idx[g0 + t] = buf_idx[t];
        }
      }
      __syncthreads();
      if (threadIdx.x == 0) bn = 0u;
    }
    __syncthreads();
  }
  if (a.hist_next)
    for (int b = threadIdx.x; b < kDigitBins; b += kDigit2Block) {
      const uint32_t c = h[b];
      if (c) atomicAdd(&a.hist_next[b], c);
    }
  if constexpr (DENSE) {
    if (lane == 0 && mine) atomicAdd(&cnt[0], mine);
    __syncthreads();
    if (threadIdx.x == 0 && cnt[0]) atomicAdd(&a.counts[blockIdx.x / a.slices], cnt[0]);
    return;
  }
  for (int b = threadIdx.x; b < min(nr, kCountMax); b += kDigit2Block) {
    const uint32_t c = cnt[b];
    if (c) atomicAdd(&a.counts[b], c);
  }
}

// ------------------------------------------------------------------------------------
// Pruned estimate (used when no estimate vector is requested). A coordinate whose median
// over rows has |est| >= tau0 has at least ceil(r/2) cells with |cell| >= tau0 (odd r: the
// median and the values beyond it; even r: the upper (or lower) half, since
// fl(fl(m1 + m2) * 0.5) never exceeds m2 in magnitude). So with tau0 no larger than the
// k-th |est|, only coordinates with ceil(r/2) "heavy" cells can be selected, and a bitmap
// of heavy cells replaces most table reads. tau0 is the rho-th largest of M sampled exact
// estimates, rho ~ 1.2 M k / d plus a margin; if fewer than k coordinates reach tau0 the emit's
// workgroups estimate every coordinate (settle_list), so the result is exact either way.

template <int R>
__device__ __forceinline__ uint32_t estimate_key(const RowConst (&kr)[R], const float* __restrict__ merged,
                                                 uint32_t i) {
  return abs_key(estimate_val<R>(kr, merged, i));
}

// Sampled keys at M evenly spaced coordinates: |est| keys, or (HEAVYMIX) the fill keys
// rnd >> 1, whose rho-th largest bounds the fill from below. Their digit-1 histogram is
// added into hist_s for k_heavy's bound.
template <int R, bool HM>
__global__ void __launch_bounds__(kBlock) k_sample(HashSet hs, const float* __restrict__ merged, int64_t d, int M,
                                                   const uint32_t* __restrict__ rnd, uint32_t* __restrict__ out,
                                                   uint32_t* __restrict__ hist_s) {
  __shared__ uint32_t h[kDigit1Bins];
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) h[b] = 0u;
  __syncthreads();
  const int s = blockIdx.x * kBlock + threadIdx.x;
  const bool ok = s < M;
  uint32_t key = 0u;
  if (ok) {
    const uint32_t i = (uint32_t)(((int64_t)s * d) / M);
    if constexpr (HM) {
      key = rnd[i] >> 1;
    } else {
      RowConst kr[R];
#pragma unroll
      for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
      key = estimate_key<R>(kr, merged, i);
    }
    out[s] = key;
  }
  hist_add(h, ok, key >> kDigit1Shift);
  __syncthreads();
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) {
    const uint32_t c = h[b];
    if (c) atomicAdd(&hist_s[b], c);
  }
}

// tau0 = the rho-th largest sampled key, found by one block of BS threads: digit 1 from
// k_sample's histogram hist_s, digits 2 and 3 over the sampled keys held in registers. h is
// an LDS histogram of kDigitBins words. All threads must call it; each gets tau0.
template <int BS>
__device__ uint32_t sampled_bound(const uint32_t* __restrict__ sample, int M, uint32_t rho,
                                  const uint32_t* __restrict__ hist_s, uint32_t* h, uint32_t* shw, uint32_t* res) {
  constexpr int kPer = kSampleMax / BS;
  uint32_t key[kPer];
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    const int t = m * BS + threadIdx.x;
    key[m] = t < M ? sample[t] : 0u;
  }
  for (int b = threadIdx.x; b < kDigitBins; b += BS) h[b] = 0u;
  find_bucket<BS, kDigit1Bins>(hist_s, true, rho, shw, res);
  const uint32_t b1 = res[0], need2 = rho - res[1];
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    const bool take = m * BS + (int)threadIdx.x < M && (key[m] >> kDigit1Shift) == b1;
    hist_add(h, take, (key[m] >> 10) & 1023u);
  }
  __syncthreads();
  find_bucket<BS, kDigitBins>(h, true, need2, shw, res);
  const uint32_t pre = (b1 << 10) | res[0], need3 = need2 - res[1];
  for (int b = threadIdx.x; b < kDigitBins; b += BS) h[b] = 0u;
  __syncthreads();
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    const bool take = m * BS + (int)threadIdx.x < M && (key[m] >> 10) == pre;
    hist_add(h, take, key[m] & 1023u);
  }
  __syncthreads();
  find_bucket<BS, kDigitBins>(h, true, need3, shw, res);
  return (pre << 10) | res[0];
}

// Heavy-cell bitmap: bit j * hrow + col (rows padded to hrow bits, a multiple of 128, so a
// row starts on a word) is |merged[j][col]| >= tau0, or (HEAVYMIX,
// hm = 1) merged[j][col]^2 >= theta in fp64 (one ballot per 64 cells); with hm the sampled fill
// bound tau0 is still found here, for the pruned pass. A coordinate with
// est^2 >= theta has ceil(r/2) cells with |cell| >= |est| (see the pruned pass), and the
// squares of fp32 values are exact in fp64, so those cells pass the same test.
// Every block first finds tau0 itself (the sampled keys are read from L2; block 0 records
// it and resets the selection counters), so no single-block kernel runs in between.
constexpr int kHeavyUnroll = 8;  // 64-cell groups per wave and pass of k_heavy
__global__ void __launch_bounds__(kSelBlock) k_heavy(const float* __restrict__ merged, int64_t c, int64_t hrow,
                                                  int r,
                                                  SelectCtl* __restrict__ ctl, uint32_t* __restrict__ heavy,
                                                  int hm, const uint32_t* __restrict__ sample, int M,
                                                  uint32_t rho, const uint32_t* __restrict__ hist_s) {
  __shared__ uint32_t h[kDigitBins];
  __shared__ uint32_t shw[kSelBlock / 64];
  __shared__ uint32_t res[2];
  const uint32_t tau0 = sampled_bound<kSelBlock>(sample, M, rho, hist_s, h, shw, res);
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    ctl->tau0 = tau0;
    ctl->n_cand = 0u;
  }
  const double theta = ctl->theta;
  // The map in groups of 64 cells (one ballot, two words each; hrow is a multiple of 64, so a
  // group lies in one row). A wave takes UH consecutive groups per pass with all their loads
  // in flight together. r <= 16 and hrow <= 2^31 keep group indices below 2^29.
  constexpr int UH = kHeavyUnroll;
  const uint32_t gpr = (uint32_t)(hrow >> 6);  // groups per row
  const int64_t ng = ((int64_t)r * hrow) >> 6;
  const int lane = threadIdx.x & 63;
  // wave index, the same in every lane (a scalar)
  const int64_t wv = __builtin_amdgcn_readfirstlane((uint32_t)(((int64_t)blockIdx.x * kSelBlock + threadIdx.x) >> 6));
  const int64_t nwv = ((int64_t)gridDim.x * kSelBlock) >> 6;
  for (int64_t g0 = wv * UH; g0 < ng; g0 += nwv * UH) {
    float x[UH];
    bool in[UH];
    // row j and group-in-row rr of group g0 + q, advanced one group at a time
    uint32_t j = (uint32_t)g0 / gpr, rr = (uint32_t)g0 - j * gpr;
#pragma unroll
    for (int q = 0; q < UH; ++q) {
      const int64_t col = (int64_t)rr * 64 + lane;
      in[q] = g0 + q < ng && col < c;
      x[q] = in[q] ? merged[(int64_t)j * c + col] : 0.f;
      if (++rr == gpr) {
        rr = 0;
        ++j;
      }
    }
#pragma unroll
    for (int q = 0; q < UH; ++q) {
      const bool hv = in[q] && (hm ? (double)x[q] * (double)x[q] >= theta : abs_key(x[q]) >= tau0);
      const uint64_t m = __ballot(hv);
      if (lane == 0 && g0 + q < ng) {
        heavy[2 * (g0 + q)] = (uint32_t)m;
        heavy[2 * (g0 + q) + 1] = (uint32_t)(m >> 32);
      }
    }
  }
}

// Coarse heavy-cell map: coarse word w covers fine words [w*G, w*G + G) (G = 2^log2g <= 32);
// each fine word contributes 32/G bits, bit q set when any of its cells q*G .. q*G+G-1 is.
__global__ void __launch_bounds__(kBlock) k_coarse(const uint32_t* __restrict__ fine, int64_t fine_words,
                                                   int log2g, uint32_t* __restrict__ coarse, int64_t coarse_words) {
  const int G = 1 << log2g;
  const int per = 32 / G;  // coarse bits from one fine word
  const uint32_t mask = G == 32 ? 0xffffffffu : ((1u << G) - 1u);
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  for (int64_t w = (int64_t)blockIdx.x * kBlock + threadIdx.x; w < coarse_words; w += stride) {
    uint32_t out = 0u;
    for (int f = 0; f < G; ++f) {
      const int64_t fw = w * G + f;
      const uint32_t x = fw < fine_words ? fine[fw] : 0u;
      for (int q = 0; q < per; ++q)
        if ((x >> (q * G)) & mask) out |= 1u << (f * per + q);
    }
    coarse[w] = out;
  }
}

// The pruned pass (k_pruned), in two phases per workgroup.
// 1. Every coordinate of the workgroup checks its r heavy bits (bitmap in LDS when it fits); the
//    survivors (ceil(r/2) heavy cells; for HEAVYMIX also every coordinate whose fill key
//    rnd[i] >> 1 reaches tau0) are queued, through an LDS buffer, in the workgroup's own part of
//    the queue (as many entries as it has coordinates, so no counter is shared).
// 2. The workgroup's survivors, two per thread with every lane busy, get their exact estimate;
//    those with key >= tau0 (for HEAVYMIX the heavy ones always, key 0x80000000 | bits(|est|),
//    the others by their fill key) are appended to the candidates and counted in their
//    histogram, and |H| is counted.
// Estimating a survivor where it is found stalled whole waves for a few lanes (159 us at
// 25.6M x 8); a second kernel for the estimates cost its launch and drained the chip in between
// (73 + 14 us, against 78 us in one kernel).
// dynamic LDS of k_pruned: [map words?][buf indices]
constexpr int kPruneBlock = 1024;  // 16 waves per CU; the heavy bitmap fills the LDS

// Where the pruned pass finds a cell's heavy bit. The map's address space is fixed at
// compile time so that LDS lookups are LDS instructions, not generic ones.
constexpr int kMapFine = 0;    // the fine map (one bit per cell), copied into LDS
constexpr int kMapCoarse = 1;  // a coarse map in LDS (one bit per 2^coarse_log2 cells, set when
                               // any of them is heavy); a set bit is confirmed in the fine map
                               // in global memory, so the count equals the fine map's
constexpr int kMapGlobal = 2;  // the fine map read from global memory

constexpr int kPruneLdsWords = 160 * 1024 / 4;  // the whole LDS of a CU (one workgroup per CU)
constexpr int kSurvBuf = 4 * kPruneBlock;       // candidate buffer of the second phase
static_assert(kDigit1Bins + 2 * kSurvBuf + 3 <= kPruneLdsWords, "second phase of k_pruned");

template <int MAP>
__device__ __forceinline__ int64_t map_words_in_lds(int64_t map_words) {
  return MAP == kMapGlobal ? 0 : map_words;
}

// Bit e & 31 of word w (the hardware takes the low five bits of the offset).
__device__ __forceinline__ uint32_t bit_at(uint32_t w, uint32_t e) { return __builtin_amdgcn_ubfe(w, e, 1u); }

// Phase 2: exact estimates of the workgroup's survivors queue[0, qn), candidates appended and
// binned. sm: kSurvWords words of LDS, free (a barrier before). kPruneBlock threads.
constexpr int kSurvWords = kDigit1Bins + 2 * kSurvBuf + 3;
template <int R, bool HM>
__device__ __forceinline__ void estimate_survivors(uint32_t* sm, const RowConst (&kr)[R],
                                                   const float* __restrict__ merged, SelectCtl* __restrict__ ctl,
                                                   uint32_t tau0, const uint32_t* queue, int64_t qn,
                                                   const uint32_t* __restrict__ rnd, uint32_t* __restrict__ cand_key,
                                                   int32_t* __restrict__ cand_idx, uint32_t* __restrict__ hist_c,
                                                   const uint32_t* __restrict__ confirm = nullptr,
                                                   int64_t hrow = 0) {
  constexpr int V = 2;  // survivors per thread and pass, all their cell loads in flight
  uint32_t* const h = sm;
  uint32_t* const bkey = sm + kDigit1Bins;
  int32_t* const bidx = reinterpret_cast<int32_t*>(bkey + kSurvBuf);
  uint32_t& cn = sm[kDigit1Bins + 2 * kSurvBuf];
  uint32_t& cbase = sm[kDigit1Bins + 2 * kSurvBuf + 1];
  uint32_t& nheavy = sm[kDigit1Bins + 2 * kSurvBuf + 2];
  for (int b = threadIdx.x; b < kDigit1Bins; b += kPruneBlock) h[b] = 0u;
  if (threadIdx.x == 0) {
    cn = 0u;
    nheavy = 0u;
  }
  __syncthreads();
  const double theta = HM ? ctl->theta : 0.0;
  const CandBins bins = cand_bins(tau0, HM, theta, true);
  const int lane = threadIdx.x & 63;
  uint32_t mine = 0;
  for (int64_t t0 = 0; t0 < qn; t0 += V * kPruneBlock) {  // block-uniform
    uint32_t ii[V], key[V];
    float e[V];
    bool cand[V];
#pragma unroll
    for (int m = 0; m < V; ++m) {
      const int64_t t = t0 + m * kPruneBlock + threadIdx.x;
      cand[m] = t < qn;
      ii[m] = cand[m] ? queue[t] : 0u;  // coordinate 0 stands in past the end (in range)
    }
    if (confirm) {
      // folded heavy bits let coordinates through that have too few heavy cells: their cells' own
      // bits (a map that stays in the L2s) are read first, and only what passes reads the table
#pragma unroll
      for (int m = 0; m < V; ++m) {
        uint32_t n = 0u;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          uint32_t col, sflip;
          hash_row(kr[j], ii[m], col, sflip);
          n += bit_at(confirm[j * (hrow >> 5) + (col >> 5)], col);
        }
        bool pass = n >= (uint32_t)(R + 1) / 2;
        if constexpr (HM) pass = pass || rnd[ii[m]] >> 1 >= tau0;
        cand[m] = cand[m] && pass;
      }
#pragma unroll
      for (int m = 0; m < V; ++m) e[m] = cand[m] ? estimate_val<R>(kr, merged, ii[m]) : 0.f;
    } else {
#pragma unroll
      for (int m = 0; m < V; ++m) e[m] = estimate_val<R>(kr, merged, ii[m]);
    }
#pragma unroll
    for (int m = 0; m < V; ++m) {
      if constexpr (HM) {
        const bool hv = cand[m] && (double)e[m] * (double)e[m] >= theta;
        key[m] = hv ? (0x80000000u | abs_key(e[m])) : (cand[m] ? rnd[ii[m]] >> 1 : 0u);
        cand[m] = hv || (cand[m] && key[m] >= tau0);
        mine += hv ? 1u : 0u;
      } else {
        key[m] = abs_key(e[m]);
        cand[m] = cand[m] && key[m] >= tau0;
      }
      hist_add(h, cand[m], cand_bin(bins, key[m]));
      // one LDS atomic per wave; at most V * kPruneBlock entries a pass, and the buffer, flushed
      // whenever it is half full, holds twice that
      const uint64_t bal = __ballot(cand[m]);
      uint32_t wbase = 0u;
      if (lane == 0 && bal) wbase = atomicAdd(&cn, (uint32_t)__popcll(bal));
      wbase = __shfl(wbase, 0);
      if (cand[m]) {
        const uint32_t pos = wbase + (uint32_t)__popcll(bal & ((1ull << lane) - 1ull));
        bkey[pos] = key[m];
        bidx[pos] = (int32_t)ii[m];
      }
    }
    __syncthreads();
    const uint32_t nb = cn;
    if (nb >= (uint32_t)(kSurvBuf / 2) || (t0 + V * kPruneBlock >= qn && nb > 0)) {
      if (threadIdx.x == 0) cbase = atomicAdd(&ctl->n_cand, nb);
      __syncthreads();
      const int64_t g0 = cbase;
      for (uint32_t t = threadIdx.x; t < nb; t += kPruneBlock) {
        cand_key[g0 + t] = bkey[t];
        cand_idx[g0 + t] = bidx[t];
      }
      __syncthreads();
      if (threadIdx.x == 0) cn = 0u;
    }
    __syncthreads();
  }
  if constexpr (HM) {
    if (mine) atomicAdd(&nheavy, mine);
    __syncthreads();
    if (threadIdx.x == 0 && nheavy) atomicAdd(&ctl->n_heavy, (unsigned long long)nheavy);
  }
  for (int b = threadIdx.x; b < kDigit1Bins; b += kPruneBlock) {
    const uint32_t c = h[b];
    if (c) atomicAdd(&hist_c[b], c);
  }
}

template <int R, bool HM, int MAP>
__global__ void __launch_bounds__(kPruneBlock) k_pruned(HashSet hs, int64_t d, SelectCtl* __restrict__ ctl,
                                                   const uint32_t* __restrict__ heavy,
                                                   const uint32_t* __restrict__ lmap, int64_t map_words,
                                                   int64_t hrow, int coarse_log2, int buf_cap,
                                                   uint32_t* __restrict__ queue,
                                                   uint32_t* __restrict__ bitmap, const uint32_t* __restrict__ rnd,
                                                   uint32_t* __restrict__ hist_s, const float* __restrict__ merged,
                                                   uint32_t* __restrict__ cand_key, int32_t* __restrict__ cand_idx,
                                                   uint32_t* __restrict__ hist_c) {
  // coordinates per lane per pass: independent hash chains in flight (two registers each per
  // row, so fewer with many rows, where four would spill); six with the map in LDS and few
  // rows (d = 25.6M x 8, r = 5: 71 -> 68.5 us; with the coarse map six measured no better)
  constexpr int U = (MAP == kMapFine && R <= 6) ? 6 : R <= 8 ? 4 : R <= 12 ? 2 : 1;
  // map index j * hrow + col of a cell; below 2^32 whenever a map fits in LDS
  using Cell = typename std::conditional<MAP == kMapGlobal, uint64_t, uint32_t>::type;
  // LDS: [map words][buf_cap queue entries][counter], one static array, so a lookup's
  // address is known at compile time to need no base added
  __shared__ uint32_t sm[kPruneLdsWords];
  uint32_t& bn = sm[map_words_in_lds<MAP>(map_words) + buf_cap];
  if (blockIdx.x == 0)  // the samples' histogram, read by k_heavy, cleared for the next call
    for (int b = threadIdx.x; b < kDigit1Bins; b += kPruneBlock) hist_s[b] = 0u;
  uint32_t* buf = sm;
  if constexpr (MAP != kMapGlobal) {
    // map_words is even and the map 8-byte aligned: copy 16 bytes per lane, 8 loads in flight
    const int64_t n4 = map_words / 4;
    const uint4* src = reinterpret_cast<const uint4*>(lmap);
    uint4* dst = reinterpret_cast<uint4*>(sm);
    int64_t w = threadIdx.x;
    for (; w + 7 * kPruneBlock < n4; w += 8 * kPruneBlock) {
      uint4 t[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) t[m] = src[w + m * kPruneBlock];
#pragma unroll
      for (int m = 0; m < 8; ++m) dst[w + m * kPruneBlock] = t[m];
    }
    for (; w < n4; w += kPruneBlock) dst[w] = src[w];
    for (int64_t x = 4 * n4 + threadIdx.x; x < map_words; x += kPruneBlock) sm[x] = lmap[x];
    buf = sm + map_words;
  }
  RowConst kr[R];
#pragma unroll
  for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
  const uint32_t tau0 = ctl->tau0;
  constexpr int need = (R + 1) / 2;
  if (threadIdx.x == 0) bn = 0;
  __syncthreads();
  const int64_t stride = (int64_t)gridDim.x * kPruneBlock * U;
  const int64_t base0 = (int64_t)blockIdx.x * kPruneBlock * U;
  // this workgroup's part of the queue: as long as the number of its coordinates, after the
  // parts of the workgroups before it (d / stride whole passes and a share of the rest)
  const int64_t passes = d / stride;
  queue += passes * base0 + min(d - passes * stride, base0);
  int64_t qn = 0;  // survivors in it (block-uniform)
  // Raw bucket hashes and columns of this lane's U coordinates, advanced by one stride per
  // pass without a multiply: the raw hash moves by db = (a * stride) mod p, less p when it
  // passes p, so the column moves by dc1 = db mod c, or by dc2 = (db - p) mod c after such a
  // wrap, and is brought back below c by one subtraction. The raw hash is kept biased by
  // kBias = 2^32 - p, so that passing p is the carry out of the 32-bit add.
  constexpr uint32_t kBias = 0x80000001u;
  uint32_t hb[R][U], cb[R][U], db[R], dc1[R], dc2[R];
  const uint32_t pc = mod_c(kMersenne, kr[0].c, kr[0].magic, kr[0].shift);  // p mod c
#pragma unroll
  for (int j = 0; j < R; ++j) {
    db[j] = mod_mersenne_affine(kr[j].a, 0u, (uint32_t)stride);
    dc1[j] = mod_c(db[j], kr[j].c, kr[j].magic, kr[j].shift);
    dc2[j] = dc1[j] >= pc ? dc1[j] - pc : dc1[j] + (kr[j].c - pc);
    // the select between the two steps takes one operand from a vector register: keep both
    // there for the whole kernel rather than copying them in every pass
    asm volatile("" : "+v"(dc1[j]), "+v"(dc2[j]));
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const uint32_t raw =
          mod_mersenne_affine(kr[j].a, kr[j].b, (uint32_t)(base0 + threadIdx.x + (int64_t)m * kPruneBlock));
      hb[j][m] = raw + kBias;  // < 2^32: raw < p
      cb[j][m] = mod_c(raw, kr[j].c, kr[j].magic, kr[j].shift);
    }
  }
  auto advance = [&](int j, int m) {
    const uint32_t t = hb[j][m] + db[j];
    const bool wrap = t < db[j];  // carry out: raw + db >= p
    hb[j][m] = wrap ? t + kBias : t;  // on a carry t is the new raw hash itself
    const uint32_t cn = cb[j][m] + (wrap ? dc2[j] : dc1[j]);
    cb[j][m] = min(cn, cn - kr[j].c);  // cn < 2c: one subtraction, unsigned
  };
  // words per map row (rows padded to hrow bits, hrow a multiple of 64)
  const uint32_t hrow32 = (uint32_t)(hrow >> 5);
  for (int64_t base = base0; base < d; base += stride) {  // block-uniform
    // HEAVYMIX: the draws are loaded first, so their memory latency overlaps the lookups
    uint32_t fill[U];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int64_t i = base + threadIdx.x + (int64_t)m * kPruneBlock;
      fill[m] = HM && i < d ? rnd[i] >> 1 : 0u;
    }
    // all U * R lookups first (independent), then the appends
    uint32_t cnt[U];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      cnt[m] = 0u;
      if constexpr (MAP == kMapCoarse) {
        // a coarse bit covers its cells' heavy bits, so a coordinate with fewer than `need`
        // coarse-set rows is out without a global read; the others confirm their set rows in
        // the fine map (global reads, the cost here: L2 requests) while `need` is in reach
        Cell ev[R];
        uint32_t cset = 0u, nset = 0u;
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const uint32_t col = cb[j][m];
          advance(j, m);
          ev[j] = (Cell)j * (Cell)hrow + col;
          const uint32_t cbit = ev[j] >> coarse_log2;
          const uint32_t bit = bit_at(sm[cbit >> 5], cbit);
          cset |= bit << j;
          nset += bit;
        }
        if (nset >= (uint32_t)need) {
          uint32_t left = nset;  // coarse-set rows not yet confirmed, this one included
#pragma unroll
          for (int j = 0; j < R; ++j) {
            if ((cset >> j) & 1u) {
              if (cnt[m] + left >= (uint32_t)need) cnt[m] += (heavy[ev[j] >> 5] >> (ev[j] & 31)) & 1u;
              --left;
            }
          }
        }
      } else if constexpr (MAP == kMapFine) {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const uint32_t col = cb[j][m];
          advance(j, m);
          cnt[m] += bit_at(sm[(uint32_t)j * hrow32 + (col >> 5)], col);
        }
      } else {
#pragma unroll
        for (int j = 0; j < R; ++j) {
          const uint32_t col = cb[j][m];
          advance(j, m);
          const Cell e = (Cell)j * (Cell)hrow + col;
          // global reads are the cost here (L2 requests): skip a row once the coordinate
          // cannot reach `need` with the rows left, which leaves the keep decision unchanged
          if (cnt[m] + (uint32_t)(R - j) >= (uint32_t)need) cnt[m] += (heavy[e >> 5] >> (e & 31)) & 1u;
        }
      }
    }
    // keep the lookups together, ahead of the appends (the compiler would otherwise sink
    // each coordinate's into its own guarded block and wait once per coordinate)
#pragma unroll
    for (int m = 0; m < U; ++m) asm volatile("" : "+v"(cnt[m]));
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int64_t i = base + threadIdx.x + (int64_t)m * kPruneBlock;
      bool keep = i < d && cnt[m] >= (uint32_t)need;
      if constexpr (HM) keep = keep || (i < d && fill[m] >= tau0);
      if (keep) {
        const uint32_t pos = atomicAdd(&bn, 1u);
        if (pos < (uint32_t)buf_cap)
          buf[pos] = (uint32_t)i;
        else
          queue[qn + pos] = (uint32_t)i;  // buffer full within this pass (dense survivors)
      }
      if (i < d && (i & 31) == 0) bitmap[i >> 5] = 0u;
    }
    __syncthreads();
    const uint32_t n = bn;
    const bool last = base + stride >= d;
    if (n >= (uint32_t)(buf_cap / 2) || (last && n > 0)) {
      const uint32_t nb = min(n, (uint32_t)buf_cap);
      for (uint32_t t = threadIdx.x; t < nb; t += kPruneBlock) queue[qn + t] = buf[t];
      qn += n;
      __syncthreads();
      if (threadIdx.x == 0) bn = 0;
    }
    __syncthreads();
  }

  estimate_survivors<R, HM>(sm, kr, merged, ctl, tau0, queue, qn, rnd, cand_key, cand_idx, hist_c);
}

// The pruned pass where the heavy bits of all rows outgrow a CU's LDS (1.3M cells): k_planes looks
// up one row per workgroup (the workgroups are dealt over the rows), whose bits do fit or nearly,
// and writes the row's bit of every coordinate as a bit plane (d/8 bytes); k_combine counts the r
// bits of 32 coordinates at a time and estimates the survivors. A row of more than kPlaneBits cells
// keeps its first `fine` cells one bit each and folds the rest, two cells to a bit that is set
// when either is heavy, so that the row fits exactly: a folded bit can only add survivors,
// whose estimate decides. Each workgroup folds its row as it loads it, 16 bytes a lane (bit by
// bit that cost more than the lookups: 4M, r = 4, c = 2.4M, the selection 133 us, so 77).
// Against k_pruned with all rows folded 8 to 32 cells to a bit, where most coordinates have
// to confirm their set bits in the global map and the pass is bound by L2 requests (66M x 16,
// r = 7: 69% of the folded bits set, 161M requests): the selection takes 448 against 891 us there,
// 138 against 158 at 14.7M x 4 (c = 1.47M), 120 against 166 at 20M x 2 (c = 600,000), 262 against 314 at
// 22M x 12 (c = 2.05M, k = 0.5%); over d of 1M to 30M, c of 1.25M to 2.4M, r = 4 and 7, a folded row takes
// 0.64 to 1.05 of it (the largest ratio at 1M, c = 1.25M, r = 4: 66 against 63 us). It is used while a row is folded by two at most and for four rows or
// more: folded by four it lost (50M x 2, r = 7, c = 5M: 1,571 against 1,237 us), and with three rows it
// gained nothing (15M x 4, c = 1.5M: 136 against 131 us).
constexpr int64_t kPlaneBits = (kPruneLdsWords - 64) / 4 * 4 * 32ll;

// Bit q of the result: bit 2 q or 2 q + 1 of x.
__device__ __forceinline__ uint32_t pair_bits(uint32_t x) {
  x = (x | (x >> 1)) & 0x55555555u;
  x = (x | (x >> 1)) & 0x33333333u;
  x = (x | (x >> 2)) & 0x0f0f0f0fu;
  x = (x | (x >> 4)) & 0x00ff00ffu;
  return (x | (x >> 8)) & 0x0000ffffu;
}

template <bool FOLD>
__global__ void __launch_bounds__(kPruneBlock) k_planes(HashSet hs, int64_t d, const uint32_t* __restrict__ heavy,
                                                        int64_t hrow, int64_t fine,
                                                        uint64_t* __restrict__ planes, int64_t plane_words,
                                                        uint32_t* __restrict__ hist_s) {
  constexpr int U = 8;  // coordinates per lane per pass
  __shared__ uint32_t sm[kPruneLdsWords];
  if (blockIdx.x == 0)  // the samples' histogram, read by k_heavy, cleared for the next call
    for (int b = threadIdx.x; b < kDigit1Bins; b += kPruneBlock) hist_s[b] = 0u;
  const int j = blockIdx.x % hs.r;
  const int64_t part = blockIdx.x / hs.r, parts = gridDim.x / hs.r;
  const uint32_t* src = heavy + j * (hrow >> 5);  // 16-byte aligned: rows are padded to 128 cells
  const int64_t f4 = fine >> 7;                   // fine is a multiple of 128
  for (int64_t w0 = 0; w0 < f4; w0 += 8 * kPruneBlock) {
    uint4 t[8];
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int64_t w = w0 + m * kPruneBlock + threadIdx.x;
      if (w < f4) t[m] = reinterpret_cast<const uint4*>(src)[w];
    }
#pragma unroll
    for (int m = 0; m < 8; ++m) {
      const int64_t w = w0 + m * kPruneBlock + threadIdx.x;
      if (w < f4) reinterpret_cast<uint4*>(sm)[w] = t[m];
    }
  }
  if constexpr (FOLD) {
    // the rest in pairs of cells: four source words make two folded ones
    const uint4* const rest = reinterpret_cast<const uint4*>(src) + f4;
    uint2* const out2 = reinterpret_cast<uint2*>(sm + (fine >> 5));
    const int64_t n4 = (hrow - fine) >> 7;
    for (int64_t w0 = 0; w0 < n4; w0 += 8 * kPruneBlock) {
      uint4 t[8];
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int64_t w = w0 + m * kPruneBlock + threadIdx.x;
        if (w < n4) t[m] = rest[w];
      }
#pragma unroll
      for (int m = 0; m < 8; ++m) {
        const int64_t w = w0 + m * kPruneBlock + threadIdx.x;
        if (w < n4)
          out2[w] = make_uint2(pair_bits(t[m].x) | pair_bits(t[m].y) << 16, pair_bits(t[m].z) | pair_bits(t[m].w) << 16);
      }
    }
  }
  const RowConst k = row_const(hs, j);
  const int64_t stride = parts * kPruneBlock * U;
  // columns advanced by one stride per pass without a multiply (as in k_pruned)
  constexpr uint32_t kBias = 0x80000001u;
  const uint32_t pc = mod_c(kMersenne, k.c, k.magic, k.shift);
  const uint32_t db = mod_mersenne_affine(k.a, 0u, (uint32_t)stride);
  uint32_t dc1 = mod_c(db, k.c, k.magic, k.shift);
  uint32_t dc2 = dc1 >= pc ? dc1 - pc : dc1 + (k.c - pc);
  asm volatile("" : "+v"(dc1), "+v"(dc2));
  const int64_t base0 = part * kPruneBlock * U;
  uint32_t hb[U], cb[U];
#pragma unroll
  for (int m = 0; m < U; ++m) {
    const uint32_t raw = mod_mersenne_affine(k.a, k.b, (uint32_t)(base0 + threadIdx.x + (int64_t)m * kPruneBlock));
    hb[m] = raw + kBias;
    cb[m] = mod_c(raw, k.c, k.magic, k.shift);
  }
  const int lane = threadIdx.x & 63;
  uint64_t* const out = planes + j * plane_words;
  __syncthreads();
  for (int64_t base = base0; base < d; base += stride) {  // block-uniform
    uint32_t bit[U];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      uint32_t e = cb[m];
      if constexpr (FOLD) {
        const int32_t over = max((int32_t)(e - (uint32_t)fine), 0);  // cells beyond the fine ones
        e = e - (uint32_t)over + ((uint32_t)over >> 1);
      }
      bit[m] = bit_at(sm[e >> 5], e);
      const uint32_t t = hb[m] + db;
      const bool wrap = t < db;
      hb[m] = wrap ? t + kBias : t;
      const uint32_t cn = cb[m] + (wrap ? dc2 : dc1);
      cb[m] = min(cn, cn - k.c);
    }
    // the 64 bits of a wave's coordinates are one word of the plane; lane m stores word m
    uint64_t mine = 0;
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const uint64_t w = __ballot(bit[m] != 0u);
      mine = lane == m ? w : mine;
    }
    const int64_t i = base + (threadIdx.x & ~63) + (int64_t)lane * kPruneBlock;
    if (lane < U && i < d) out[i >> 6] = mine;
  }
}

// Bits whose count over the R planes reaches `need`, by a bit-sliced counter.
template <int R>
__device__ __forceinline__ uint32_t count_reaches(const uint32_t (&x)[R], int need) {
  uint32_t c[5] = {0u, 0u, 0u, 0u, 0u};  // counts up to 16
#pragma unroll
  for (int j = 0; j < R; ++j) {
    uint32_t carry = x[j];
#pragma unroll
    for (int b = 0; b < 5; ++b) {
      const uint32_t t = c[b] & carry;
      c[b] ^= carry;
      carry = t;
    }
  }
  uint32_t ge = 0u, eq = ~0u;
#pragma unroll
  for (int b = 4; b >= 0; --b) {
    const uint32_t n = (need >> b) & 1 ? ~0u : 0u;
    ge |= eq & c[b] & ~n;
    eq &= ~(c[b] ^ n);
  }
  return ge | eq;
}

template <int R, bool HM>
__global__ void __launch_bounds__(kPruneBlock) k_combine(HashSet hs, int64_t d, SelectCtl* __restrict__ ctl,
                                                         const uint32_t* __restrict__ planes, int64_t plane_words,
                                                         uint32_t* __restrict__ queue, uint32_t* __restrict__ bitmap,
                                                         const uint32_t* __restrict__ rnd,
                                                         const float* __restrict__ merged,
                                                         uint32_t* __restrict__ cand_key,
                                                         int32_t* __restrict__ cand_idx,
                                                         uint32_t* __restrict__ hist_c,
                                                         const uint32_t* __restrict__ confirm, int64_t hrow) {
  __shared__ uint32_t sm[kSurvWords];
  __shared__ uint32_t qs;
  constexpr int need = (R + 1) / 2;
  RowConst kr[R];
#pragma unroll
  for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
  const uint32_t tau0 = ctl->tau0;
  // Chunks of words, a wave's pass, are dealt to the workgroups in turn, so that survivors crowded
  // in one part of d (one layer's coordinates) still spread over the chip: with a contiguous
  // part per workgroup, survivors within d/256 were all estimated by one (14.7M x 4: 530 us, 66M x 16:
  // 2,630 us). A workgroup's part of the queue has room for its coordinates, after those of
  // the workgroups before it.
  constexpr int kWaves = kPruneBlock / 64;
  constexpr int kWords = HM ? 16 : 64;  // HEAVYMIX: smaller chunks, more waves for the draws' loads
  constexpr int64_t kChunk = kWords * 32;  // coordinates
  const int64_t words = (d + 31) / 32, chunks = (words + kWords - 1) / kWords, grid = gridDim.x, wg = blockIdx.x;
  const int64_t mine = chunks / grid + (wg < chunks % grid ? 1 : 0);
  int64_t q0 = (wg * (chunks / grid) + min(wg, chunks % grid)) * kChunk;
  if (wg > (chunks - 1) % grid) q0 -= chunks * kChunk - d;  // the last chunk may be short
  queue += q0;
  if (threadIdx.x == 0) qs = 0u;
  __syncthreads();
  const int lane = threadIdx.x & 63;
  const int64_t row_words = 2 * plane_words;  // 32-bit words per plane
  for (int64_t t = threadIdx.x >> 6; t < mine; t += kWaves) {  // one word per lane
    const int64_t chunk = wg + t * grid, w = lane < kWords ? chunk * kWords + lane : words;
    uint32_t x[R];
#pragma unroll
    for (int j = 0; j < R; ++j) x[j] = w < words ? planes[j * row_words + w] : 0u;
    uint32_t m = count_reaches<R>(x, need);
    if (w < words) bitmap[w] = 0u;
    if (w >= words) m = 0u;
    if (w == words - 1 && (d & 31)) m &= (1u << (d & 31)) - 1u;
    if constexpr (HM) {
      // the chunk's draws, 64 coordinates a load: their ballots are the words of lanes 2 q and 2 q + 1
      // (a coordinate per lane, which reads each word of the planes 32 times: 15M x 4 51 us, so 27, 1M 13, so
      // 12; chunks of 64 words: 36 and 19 us)
      constexpr int D = kWords / 2;
      uint32_t draw[D];
#pragma unroll
      for (int q = 0; q < D; ++q) draw[q] = rnd[min(chunk * kChunk + q * 64 + lane, d - 1)] >> 1;
#pragma unroll
      for (int q = 0; q < D; ++q) {
        const uint64_t bal = __ballot(chunk * kChunk + q * 64 + lane < d && draw[q] >= tau0);
        if ((lane >> 1) == q) m |= (uint32_t)(lane & 1 ? bal >> 32 : bal);
      }
    }
    // the wave's survivors take consecutive places: one LDS atomic per wave
    uint32_t before = (uint32_t)__popc(m);
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(before, o, 64);
      if (lane >= o) before += y;
    }
    uint32_t base = 0u;
    if (lane == 63 && before) base = atomicAdd(&qs, before);
    base = __shfl(base, 63) + before - (uint32_t)__popc(m);
    while (m) {
      queue[base++] = (uint32_t)(32 * w + __ffs(m) - 1);
      m &= m - 1u;
    }
  }
  __syncthreads();
  estimate_survivors<R, HM>(sm, kr, merged, ctl, tau0, queue, qs, rnd, cand_key, cand_idx, hist_c, confirm,
                            hrow);
}

// ------------------------------------------------------------------------------------
// HEAVYMIX as printed (Alg. 2). The l2-norm-squared estimate is the median over rows of
// sum_col S[j][col]^2 in fp64, each row summed in one fixed order (a pairwise tree over
// the squares padded with zeros to a power of two, adjacent pairs level by level), so the
// heavy test est_i^2 >= l2sq / k is a function of S alone. Keys then rank the heavy set
// above the fill: heavy i gets 0x80000000 | bits(|est_i|), the others their draw
// rnd[i] >> 1, and the radix selection above takes the k largest, ties to the lower index:
// all of H (or its k largest |est| when |H| >= k) plus the l = k - |H| non-heavy
// coordinates with the largest draws.

constexpr int kTreeLeaves = 2048;  // leaves per block of one tree pass (1024 threads)

// One tree pass: block b reduces the aligned group of G leaves (G a power of two, at most
// kTreeLeaves) of row j = b / (n / G) to one value, adding adjacent pairs level by level.
// First pass (sq != nullptr): leaf t of row j is sq[j][t]^2 for t < c, else 0 (n = padded
// width). Later passes: leaf t is in[j * n + t].
__global__ void __launch_bounds__(kTreeLeaves / 2) k_sq_tree(const float* __restrict__ sq,
                                                            const double* __restrict__ in, int64_t c, int64_t n,
                                                            int64_t G, double* __restrict__ out) {
  __shared__ double t2[kTreeLeaves / 2];
  const int64_t groups = n / G;
  const int64_t j = blockIdx.x / groups, base = (blockIdx.x - j * groups) * G;
  const int tid = threadIdx.x;
  auto leaf = [&](int64_t t) -> double {
    if (sq) {
      if (t >= c) return 0.0;
      const double x = (double)sq[j * c + t];
      return x * x;
    }
    return in[j * n + t];
  };
  if (G == 1) {
    if (tid == 0) out[blockIdx.x] = leaf(base);
    return;
  }
  int64_t w = G / 2;
  if (tid < w) t2[tid] = leaf(base + 2 * tid) + leaf(base + 2 * tid + 1);
  __syncthreads();
  for (; w > 1; w /= 2) {
    double a = 0.0;
    if (tid < w / 2) a = t2[2 * tid] + t2[2 * tid + 1];
    __syncthreads();
    if (tid < w / 2) t2[tid] = a;
    __syncthreads();
  }
  if (tid == 0) out[blockIdx.x] = t2[0];
}

// Median of the r row sums (insertion sort; even r: fl(fl(m1 + m2) * 0.5)), the threshold
// theta = l2sq / k, and the heavy counter reset. One thread.
__global__ void k_theta(const double* __restrict__ rows, int r, int64_t k, SelectCtl* __restrict__ ctl) {
  if (threadIdx.x != 0) return;
  double v[kMaxRows];
  for (int j = 0; j < r; ++j) v[j] = rows[j];
  for (int a = 1; a < r; ++a) {
    const double x = v[a];
    int b = a - 1;
    while (b >= 0 && v[b] > x) {
      v[b + 1] = v[b];
      --b;
    }
    v[b + 1] = x;
  }
  const double med = (r & 1) ? v[r / 2] : 0.5 * (v[r / 2 - 1] + v[r / 2]);
  ctl->l2sq = med;
  ctl->theta = med / (double)k;
  ctl->n_heavy = 0ull;
}

// Estimate + HEAVYMIX key + digit-1 histogram + |H|.
template <int R>
__global__ void __launch_bounds__(kBlock) k_unsketch_hm(HashSet hs, const float* __restrict__ merged, int64_t d,
                                                        const uint32_t* __restrict__ rnd, float* __restrict__ est,
                                                        uint32_t* __restrict__ keys, uint32_t* __restrict__ hist,
                                                        SelectCtl* __restrict__ ctl) {
  __shared__ uint32_t h[kDigit1Bins];
  __shared__ uint32_t nh;
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) h[b] = 0u;
  if (threadIdx.x == 0) nh = 0u;
  RowConst kr[R];
#pragma unroll
  for (int j = 0; j < R; ++j) kr[j] = row_const(hs, j);
  const double theta = ctl->theta;
  __syncthreads();
  uint32_t mine = 0;
  const int64_t stride = (int64_t)gridDim.x * kBlock;
  const int64_t i0 = (int64_t)blockIdx.x * kBlock + threadIdx.x;
  uint32_t hb[R], hsg[R], db[R], dsg[R];
#pragma unroll
  for (int j = 0; j < R; ++j) {
    hb[j] = mod_mersenne_affine(kr[j].a, kr[j].b, (uint32_t)i0);
    hsg[j] = mod_mersenne_affine(kr[j].a2, kr[j].b2, (uint32_t)i0);
    db[j] = mod_mersenne_affine(kr[j].a, 0u, (uint32_t)stride);
    dsg[j] = mod_mersenne_affine(kr[j].a2, 0u, (uint32_t)stride);
  }
  for (int64_t i = i0; i < d; i += stride) {
    float val[R];
#pragma unroll
    for (int j = 0; j < R; ++j) {
      const uint32_t col = mod_c(hb[j], kr[j].c, kr[j].magic, kr[j].shift);
      val[j] = apply_sign(merged[(int64_t)j * hs.c + col], sign_flip_of(hsg[j]));
      hb[j] = add_mod_mersenne(hb[j], db[j]);
      hsg[j] = add_mod_mersenne(hsg[j], dsg[j]);
    }
    sort_net<R>(val);
    const float e = median_sorted<R>(val);
    if (est) est[i] = e;
    const double ed = (double)e;
    const bool heavy = ed * ed >= theta;
    const uint32_t key = heavy ? (0x80000000u | abs_key(e)) : (rnd[i] >> 1);
    mine += heavy ? 1u : 0u;
    keys[i] = key;
    atomicAdd(&h[key >> 20], 1u);  // cand_bin's coarse bins
  }
  if (mine) atomicAdd(&nh, mine);
  __syncthreads();
  for (int b = threadIdx.x; b < kDigit1Bins; b += kBlock) {
    const uint32_t n = h[b];
    if (n) atomicAdd(&hist[b], n);
  }
  if (threadIdx.x == 0 && nh) atomicAdd(&ctl->n_heavy, (unsigned long long)nh);
}

template <int R>
void launch_unsketch_r(const HashSet& hs, int64_t d, int num_cus, const SelectBufs& b, hipStream_t s,
                       const float* merged, float* est) {
  if (d <= (int64_t)kUnsketchSmall * kBlock * num_cus)
    hipLaunchKernelGGL((k_unsketch<R, 2>), dim3(grid_for(d, 2 * kBlock, num_cus)), dim3(kBlock), 0, s, hs, merged, d,
                       est, b.cand_key, b.hist);
  else
    hipLaunchKernelGGL((k_unsketch<R, 1>), dim3(grid_for(d, kBlock, 4 * num_cus)), dim3(kBlock), 0, s, hs, merged, d,
                       est, b.cand_key, b.hist);
}

// Every coordinate's estimate of a context: by tile for large d, else directly.
template <int R, bool HM>
hipError_t launch_full_r(gs_ctx* x, hipStream_t s, const float* merged, const uint32_t* rnd, float* est) {
  const SelectBufs b = select_bufs(x);
  if (x->push) {
    RowValues rows{};
    const int n = push_rows(x, &rows);
    const hipError_t e = launch_push(x, s, merged, rows, n);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((k_median<R, HM>), dim3(grid_for(x->d, 4 * kMedianBlock, 2 * x->num_cus)), dim3(kMedianBlock), 0,
                       s, x->hs, merged, x->d, rows, n, rnd, est, b.cand_key, b.hist, x->ctl);
  } else if constexpr (HM) {
    hipLaunchKernelGGL(k_unsketch_hm<R>, dim3(grid_for(x->d, kBlock, 4 * x->num_cus)), dim3(kBlock), 0, s, x->hs,
                       merged, x->d, rnd, est, x->cand_key, x->hist, x->ctl);
  } else {
    launch_unsketch_r<R>(x->hs, x->d, x->num_cus, b, s, merged, est);
  }
  return hipGetLastError();
}

template <int R, bool HM>
void launch_prune_r(gs_ctx* x, hipStream_t s, const float* merged, int64_t k, const uint32_t* rnd) {
  const int M = (int)(x->d < kSampleMax ? x->d : kSampleMax);
  const double mk = (double)M * (double)k / (double)x->d;
  // expected sampled keys above the k-th key: mk (sd ~ sqrt(mk)); the margin is ~8 sd
  double rho_d = std::ceil(1.2 * mk + 5.0 * std::sqrt(mk) + 8.0);
  if (rho_d > M) rho_d = M;
  if (rho_d < 1) rho_d = 1;
  hipLaunchKernelGGL((k_sample<R, HM>), dim3((M + kBlock - 1) / kBlock), dim3(kBlock), 0, s, x->hs, merged, x->d, M,
                     rnd, x->sample_keys, x->hist_s);
  const int64_t nbits = (int64_t)x->r * x->heavy_row;  // heavy-cell map bits (padded rows)
  hipLaunchKernelGGL(k_heavy, dim3(grid_for(nbits, kSelBlock * kHeavyUnroll, x->num_cus)), dim3(kSelBlock), 0, s,
                     merged, x->c, x->heavy_row, x->r, x->ctl, x->heavy, HM ? 1 : 0, x->sample_keys, M,
                     (uint32_t)rho_d, x->hist_s);
  if (x->planes) {
    const int64_t plane_words = (x->d + 63) / 64;
    const int wgs = std::max(1, x->num_cus / x->r) * x->r;
    if (x->plane_fold)
      hipLaunchKernelGGL(k_planes<true>, dim3(wgs), dim3(kPruneBlock), 0, s, x->hs, x->d, x->heavy, x->heavy_row,
                         x->plane_fine, x->planes, plane_words, x->hist_s);
    else
      hipLaunchKernelGGL(k_planes<false>, dim3(wgs), dim3(kPruneBlock), 0, s, x->hs, x->d, x->heavy, x->heavy_row,
                         x->plane_fine, x->planes, plane_words, x->hist_s);
    hipLaunchKernelGGL((k_combine<R, HM>), dim3(x->num_cus), dim3(kPruneBlock), 0, s, x->hs, x->d, x->ctl,
                       reinterpret_cast<const uint32_t*>(x->planes), plane_words, x->keys, x->bitmap, rnd, merged,
                       x->cand_key, x->cand_idx, x->hist_c, x->plane_fold ? x->heavy : nullptr, x->heavy_row);
    return;
  }
  // with the bitmap in LDS one block fits a CU: launch one per CU so the map is loaded once
  const int pgrid = grid_for(x->d, 4 * kPruneBlock, x->prune_map_in_lds ? x->num_cus : 2 * x->num_cus);
#define GS_PRUNED(MAP, LMAP, COARSE)                                                                              \
  hipLaunchKernelGGL((k_pruned<R, HM, MAP>), dim3(pgrid), dim3(kPruneBlock), 0, s, x->hs, x->d, x->ctl, x->heavy, \
                     LMAP, x->prune_map_words, x->heavy_row, COARSE, x->prune_buf_cap, x->keys, x->bitmap, rnd,   \
                     x->hist_s, merged, x->cand_key, x->cand_idx, x->hist_c)
  if (!x->prune_map_in_lds) {
    GS_PRUNED(kMapGlobal, x->heavy, 0);
  } else if (x->prune_coarse_log2 > 0) {
    hipLaunchKernelGGL(k_coarse, dim3(grid_for(x->prune_map_words, kBlock, 4 * x->num_cus)), dim3(kBlock), 0, s,
                       x->heavy, nbits / 32, x->prune_coarse_log2, x->coarse, x->prune_map_words);
    GS_PRUNED(kMapCoarse, x->coarse, x->prune_coarse_log2);
  } else {
    GS_PRUNED(kMapFine, x->heavy, 0);
  }
#undef GS_PRUNED
}

// digit2 (twice for a large dense selection) -> emit over the candidates: the pruned pass's or the
// full estimate's dense ones.
hipError_t launch_select_tail(const HashSet& hs, int64_t d, int num_cus, const SelectBufs& b, hipStream_t s,
                              const float* merged, const uint32_t* rnd, int64_t k, int pruned, int hm, int32_t* idx,
                              int64_t* n_heavy, double* l2sq, const GatherArgs* ga) {
  DigitArgs a{};
  a.key = b.cand_key;
  a.idx = pruned ? b.cand_idx : nullptr;
  a.ctl = b.ctl;
  a.hist = pruned ? b.hist_c : b.hist;
  a.out_key = b.keys;
  a.out_idx = b.stage_idx;
  a.cap = d;
  a.bitmap = b.bitmap;
  a.counts = b.counts;
  a.d = d;
  a.range = emit_range(d, num_cus);
  a.k = (uint32_t)k;
  a.pruned = pruned;
  a.hm = hm;
  // the k-th key's coarse bin holds about k/2 keys (a sixteenth of an octave of a Gaussian's tail);
  // Up to 8,192 the emit's workgroups keep them in LDS and beyond they read them a few times, so a
  // second digit pass (8 us) pays from there on: full estimate and selection of 1.1M at k = 5,500 and
  // 55,000, r = 5: 52.8 and 59 us, against 57 with a second pass and 62 without
  const bool two = !pruned && k > kTwoMinK;
  if (two) a.hist_next = b.hist2;
  // one block (of 1,024 threads) per four CUs for the pruned candidates (a few times k: fewer
  // blocks add their counts with fewer atomics), more where k is large; the full estimate's dense
  // ones take slices of up to 16,384 keys
  int64_t g2 = std::max<int64_t>(std::max(1, num_cus / 4), std::min<int64_t>(2 * num_cus, k / 4096));
  if (!pruned) {
    const int64_t parts = (a.range + 16383) / 16384;
    a.slice = ((a.range + parts - 1) / parts + 63) / 64 * 64;
    a.slices = (uint32_t)parts;
    g2 = (d + a.range - 1) / a.range * parts;
  }
  if (pruned)
    hipLaunchKernelGGL(k_digit2<false>, dim3((unsigned)g2), dim3(kDigit2Block), 0, s, a);
  else
    hipLaunchKernelGGL(k_digit2<true>, dim3((unsigned)g2), dim3(kDigit2Block), 0, s, a);
  if (two) {
    DigitArgs a1 = a;
    a1.key = b.keys;
    a1.idx = b.stage_idx;
    a1.hist = b.hist2;
    a1.hist_next = nullptr;
    a1.out_key = b.stage2;
    a1.out_idx = reinterpret_cast<int32_t*>(b.stage2 + kStage2Cap);
    a1.cap = kStage2Cap;
    a1.level = 1;
    hipLaunchKernelGGL(k_digit2<false>, dim3(num_cus), dim3(kDigit2Block), 0, s, a1);
  }
  return launch_emit(hs, d, num_cus, b, s, merged, rnd, k, pruned, two ? 1 : 0, idx, n_heavy, l2sq, ga);
}

}  // namespace

hipError_t prepare_prune(gs_ctx* x) {
  const int64_t rc = (int64_t)x->r * x->heavy_row;  // bits of the heavy-cell map (padded rows)
  const int64_t words = rc / 32;
  const int64_t lds_max = 160 * 1024 - 256;
  // the fine map of all rows in LDS if it fits beside a 512-entry queue buffer; else row by row (see
  // k_planes); else the coarsest-needed coarse map (2 .. 32 cells per bit); else the fine map from
  // global memory
  int64_t map_words = words;
  int log2g = 0;
  while ((lds_max - map_words * 4) / 4 < 512 && log2g < 5) {
    ++log2g;
    map_words = (rc + (32ll << log2g) - 1) / (32ll << log2g);
    map_words += map_words & 1;
  }
  if (log2g > 0 && x->r >= 4 && x->heavy_row <= 2 * (kPlaneBits - 128)) {
    x->plane_fold = x->heavy_row > kPlaneBits;
    // folded by two: `fine` cells as they are and (row - fine) / 2 bits after them fill kPlaneBits - 128
    x->plane_fine = x->plane_fold ? (2 * (kPlaneBits - 128) - x->heavy_row) / 128 * 128 : x->heavy_row;
    const hipError_t e =
        hipMalloc(reinterpret_cast<void**>(&x->planes), (size_t)(x->r * ((x->d + 63) / 64)) * sizeof(uint64_t));
    if (e != hipSuccess) return e;
  }
  const int64_t buf = std::min<int64_t>((lds_max - map_words * 4) / 4, 8192);
  x->prune_map_in_lds = buf >= 512 ? 1 : 0;
  x->prune_coarse_log2 = buf >= 512 ? log2g : 0;
  x->prune_map_words = buf >= 512 ? map_words : words;
  x->prune_buf_cap = buf >= 512 ? (int)buf : 8192;
  if (x->prune_coarse_log2 > 0 && !x->planes) {
    const hipError_t e = hipMalloc(reinterpret_cast<void**>(&x->coarse), (size_t)map_words * sizeof(uint32_t));
    if (e != hipSuccess) return e;
  }
  // the map (when in LDS), the queue buffer and a counter share the pass's LDS array
  if ((x->prune_map_in_lds ? x->prune_map_words : 0) + x->prune_buf_cap + 1 > kPruneLdsWords)
    return hipErrorInvalidValue;
  return hipSuccess;
}

// Whether a selection without an estimate vector prunes.
static bool prunes(const gs_ctx* x, const float* est, int64_t k, bool hm) {
  return est == nullptr && x->d * x->r > x->prune_min_cells && k * x->prune_max_density[hm ? 1 : 0] <= x->d;
}

hipError_t launch_unsketch_topk(gs_ctx* x, hipStream_t s, const float* merged, int64_t k, float* est, int32_t* idx,
                                const GatherArgs* ga) {
  // With an estimate vector requested, or a sketch small enough (d*r at most
  // prune_min_cells) that the full estimate is the cheaper chain, every coordinate is
  // estimated. Otherwise the pruned path runs (and the digit pass estimates every coordinate if its
  // candidates fell short of k).
  const bool prune = prunes(x, est, k, false);
  hipError_t e = hipSuccess;
  switch (x->r) {
#define GS_R_CASE(RR)                                                \
  case RR:                                                           \
    if (prune)                                                       \
      launch_prune_r<RR, false>(x, s, merged, k, nullptr);           \
    else                                                             \
      e = launch_full_r<RR, false>(x, s, merged, nullptr, est);      \
    break;
    GS_R_CASE(1) GS_R_CASE(2) GS_R_CASE(3) GS_R_CASE(4) GS_R_CASE(5) GS_R_CASE(6) GS_R_CASE(7) GS_R_CASE(8)
    GS_R_CASE(9) GS_R_CASE(10) GS_R_CASE(11) GS_R_CASE(12) GS_R_CASE(13) GS_R_CASE(14) GS_R_CASE(15) GS_R_CASE(16)
#undef GS_R_CASE
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  return launch_select_tail(x->hs, x->d, x->num_cus, select_bufs(x), s, merged, nullptr, k, prune ? 1 : 0, 0, idx,
                            nullptr, nullptr, ga);
}

hipError_t launch_unsketch_topk_dense(const HashSet& hs, int64_t d, int num_cus, const SelectBufs& b, hipStream_t s,
                                      const float* merged, int64_t k, float* est, int32_t* idx,
                                      const GatherArgs* ga) {
  switch (hs.r) {
#define GS_R_CASE(RR) \
  case RR: launch_unsketch_r<RR>(hs, d, num_cus, b, s, merged, est); break;
    GS_R_CASE(1) GS_R_CASE(2) GS_R_CASE(3) GS_R_CASE(4) GS_R_CASE(5) GS_R_CASE(6) GS_R_CASE(7) GS_R_CASE(8)
    GS_R_CASE(9) GS_R_CASE(10) GS_R_CASE(11) GS_R_CASE(12) GS_R_CASE(13) GS_R_CASE(14) GS_R_CASE(15) GS_R_CASE(16)
#undef GS_R_CASE
    default: return hipErrorInvalidValue;
  }
  return launch_select_tail(hs, d, num_cus, b, s, merged, nullptr, k, 0, 0, idx, nullptr, nullptr, ga);
}

hipError_t launch_heavymix_topk(gs_ctx* x, hipStream_t s, const float* merged, int64_t k, const uint32_t* rnd,
                                float* est, int32_t* idx, int64_t* n_heavy, double* l2sq, const GatherArgs* ga) {
  // row sums of squares, pass by pass (each reduces aligned groups of up to 2048 values)
  const int64_t npad = l2_pad(x->c);
  int64_t n = npad;
  const double* in = nullptr;
  double* out = x->l2buf;
  bool first = true;
  while (first || n > 1) {
    const int64_t G = n < kTreeLeaves ? n : kTreeLeaves;
    const int64_t groups = n / G;
    hipLaunchKernelGGL(k_sq_tree, dim3((unsigned)(x->r * groups)), dim3(kTreeLeaves / 2), 0, s,
                       first ? merged : nullptr, in, x->c, n, G, out);
    in = out;
    out = (out == x->l2buf) ? x->l2buf + x->l2_half : x->l2buf;
    n = groups;
    first = false;
  }
  hipLaunchKernelGGL(k_theta, dim3(1), dim3(64), 0, s, in, x->r, k, x->ctl);
  // As in launch_unsketch_topk: the full estimate with an estimate vector or a small sketch,
  // else the pruned pass, with the full one acting only if its candidates fell short of k.
  const bool prune = prunes(x, est, k, true);
  hipError_t e = hipSuccess;
  switch (x->r) {
#define GS_R_CASE(RR)                                                                                                \
  case RR:                                                                                                           \
    if (prune)                                                                                                       \
      launch_prune_r<RR, true>(x, s, merged, k, rnd);                                                                \
    else                                                                                                             \
      e = launch_full_r<RR, true>(x, s, merged, rnd, est);                                                           \
    break;
    GS_R_CASE(1) GS_R_CASE(2) GS_R_CASE(3) GS_R_CASE(4) GS_R_CASE(5) GS_R_CASE(6) GS_R_CASE(7) GS_R_CASE(8)
    GS_R_CASE(9) GS_R_CASE(10) GS_R_CASE(11) GS_R_CASE(12) GS_R_CASE(13) GS_R_CASE(14) GS_R_CASE(15) GS_R_CASE(16)
#undef GS_R_CASE
    default: return hipErrorInvalidValue;
  }
  if (e != hipSuccess) return e;
  return launch_select_tail(x->hs, x->d, x->num_cus, select_bufs(x), s, merged, rnd, k, prune ? 1 : 0, 1, idx,
                            n_heavy, l2sq, ga);
}

int64_t l2_pad(int64_t c) {
  int64_t n = 1;
  while (n < c) n *= 2;
  return n;
}

}  // namespace gs