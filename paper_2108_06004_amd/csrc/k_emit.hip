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
// short of k candidates and the list holds every key, every workgroup reads the whole list: its
// histograms give the k-th key, and one more pass the marks of the own range and the entries before
// it; ties at the k-th key are taken in coordinate order (a zero sketch of 14.7M: 9 ms, and 60 ms
// by one workgroup alone). No workgroup ever waits for another.
#include <algorithm>

#include "gs_internal.hpp"
#include "gs_select.hpp"

namespace gs {
namespace {

constexpr int kBlock = 1024;
constexpr int kBucketCap = 8192;   // words of the k-th key's bin kept in LDS
constexpr int kRankCap = 256;      // words ranked against each other

struct EmitArgs {
  const uint32_t* list_key;   // staged keys of the bin
  const int32_t* list_idx;    // and their coordinates
  const uint32_t* list0_key;  // those of the first digit's bin (complete; or every key by coordinate)
  const int32_t* list0_idx;
  uint32_t* bitmap;
  uint32_t* counts;
  SelectCtl* ctl;
  uint32_t* hist;             // histograms cleared here for the next call
  uint32_t* hist2;
  const float* merged;
  int32_t* out;
  int64_t* n_heavy;
  double* l2sq;
  int64_t d, range;
  uint32_t k;
  int pruned, level;
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
  uint32_t n, before, ties, last;
};
static_assert(kRangeMax <= (int64_t)kBucketCap * 64, "the ties of a range have a bit each in the bucket");

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

// A list too long for the LDS: the selection is its keys above T and the first need of those equal
// to T (sets need and returns T). Only the keys in [klo, khi] are read as its entries. 10 bits of
// the key range a pass; 16 loads per thread in flight, since one workgroup fills a CU.
__device__ __forceinline__ uint32_t nth_key(Shared& sh, const uint32_t* __restrict__ key, int64_t n, uint32_t klo,
                                            uint32_t khi, uint32_t& need) {
  constexpr int U = 16;
  while (khi > klo) {
    const int bits = 32 - __clz((int)(khi - klo));
    const int shift = bits > 10 ? bits - 10 : 0;
    for (int b = threadIdx.x; b < 1024; b += kBlock) sh.h[b] = 0u;
    __syncthreads();
    for (int64_t t0 = 0; t0 < n; t0 += (int64_t)U * kBlock) {  // block-uniform
      uint32_t kk[U];
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const int64_t t = t0 + (int64_t)m * kBlock + threadIdx.x;
        kk[m] = key[min(t, n - 1)];
      }
      __builtin_amdgcn_sched_barrier(0);  // the loads stay ahead of the adds
#pragma unroll
      for (int m = 0; m < U; ++m) {
        const bool in = t0 + (int64_t)m * kBlock + threadIdx.x < n && kk[m] - klo <= khi - klo;
        hist_add(sh.h, in, in ? (kk[m] - klo) >> shift : 0u);
      }
    }
    __syncthreads();
    find_bucket<kBlock, 1024>(sh.h, true, need, sh.shw, sh.res);
    const uint32_t b = sh.res[0];
    need -= sh.res[1];
    klo += b << shift;
    khi = min(khi, klo + ((1u << shift) - 1u));
    __syncthreads();
  }
  return klo;
}

// The entries of that list in [T, khi]: their bit in `above` or `ties` if they are in [lo, lo + width),
// and their number before lo.
__device__ __forceinline__ void mark_list(const uint32_t* __restrict__ key, const int32_t* __restrict__ idx, int64_t n,
                                          uint32_t T, uint32_t khi, uint32_t lo, uint32_t width, uint32_t* above,
                                          uint32_t* ties, uint32_t& above_before, uint32_t& ties_before) {
  constexpr int U = 8;
  for (int64_t t0 = 0; t0 < n; t0 += (int64_t)U * kBlock) {
    uint32_t kk[U], ii[U];
#pragma unroll
    for (int m = 0; m < U; ++m) {
      const int64_t t = min(t0 + (int64_t)m * kBlock + threadIdx.x, n - 1);
      kk[m] = key[t];
      ii[m] = idx ? (uint32_t)idx[t] : (uint32_t)t;
    }
    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int m = 0; m < U; ++m) {
      if (t0 + (int64_t)m * kBlock + threadIdx.x >= n || kk[m] < T || kk[m] > khi) continue;
      if (ii[m] < lo)
        ++(kk[m] == T ? ties_before : above_before);
      else if (ii[m] - lo < width)
        atomicOr(&(kk[m] == T ? ties : above)[(ii[m] - lo) >> 5], 1u << ((ii[m] - lo) & 31u));
    }
  }
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

__global__ void __launch_bounds__(kBlock) k_emit(EmitArgs a, HashSet hs, GatherArgs ga) {
  extern __shared__ uint32_t bits[];  // [range / 32]
  __shared__ Shared sh;
  const int64_t lo = (int64_t)blockIdx.x * a.range, hi = min(a.d, lo + a.range);
  const uint32_t nb = a.ctl->n_stage[a.level];
  if (blockIdx.x == 0 && threadIdx.x == 0) {
    if (a.n_heavy) *a.n_heavy = (int64_t)a.ctl->n_heavy;
    if (a.l2sq) *a.l2sq = a.ctl->l2sq;
  }
  // the bound admitted too little: the digit pass left every key in the list, and marked nothing
  const bool few = a.pruned && a.ctl->n_cand < a.k;
  const uint32_t l32 = (uint32_t)lo, width = (uint32_t)(hi - lo);
  const int nw = (int)(a.range / 32);
  uint32_t before = 0;
  for (uint32_t t = threadIdx.x; t < blockIdx.x; t += kBlock) before += a.counts[t];
  const int64_t words = (a.d + 31) / 32, word0 = lo / 32;
  for (int w = threadIdx.x; w < nw; w += kBlock) bits[w] = word0 + w < words ? a.bitmap[word0 + w] : 0u;
  if (threadIdx.x == 0) sh.before = sh.ties = 0u;
  uint32_t need = few ? a.k : a.ctl->need[a.level];
  const uint32_t klo = few ? 0u : a.ctl->lo[a.level], khi = few ? ~0u : a.ctl->hi[a.level];
  const int per = (nw + kBlock - 1) / kBlock, w0 = threadIdx.x * per;
  if (!few && nb <= (uint32_t)kBucketCap) {
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
    before = wave_sum(before);
    if ((threadIdx.x & 63) == 0 && before) atomicAdd(&sh.before, before);
    __syncthreads();
  } else {
    uint32_t* const ties = reinterpret_cast<uint32_t*>(sh.bucket);
    for (int w = threadIdx.x; w < nw; w += kBlock) ties[w] = 0u;
    __syncthreads();
    const int64_t n = few ? a.d : (int64_t)a.ctl->n_stage[0];
    const int32_t* const idx = few ? nullptr : a.list0_idx;
    const uint32_t T = nth_key(sh, a.list0_key, n, klo, khi, need);
    uint32_t ties_before = 0;
    mark_list(a.list0_key, idx, n, T, khi, l32, width, bits, ties, before, ties_before);
    before = wave_sum(before);
    ties_before = wave_sum(ties_before);
    if ((threadIdx.x & 63) == 0) {
      atomicAdd(&sh.before, before);
      atomicAdd(&sh.ties, ties_before);
    }
    __syncthreads();
    const uint32_t gone = min(sh.ties, need);  // ties taken by the ranges before
    uint32_t cnt = 0, total;
    for (int m = 0; m < per; ++m)
      if (w0 + m < nw) cnt += (uint32_t)__popc(ties[w0 + m]);
    uint32_t pos = gone + block_scan_incl<kBlock>(cnt, sh.shw, total) - cnt;
    for (int m = 0; m < per; ++m) {
      uint32_t x = w0 + m < nw ? ties[w0 + m] : 0u;
      for (; x && pos < need; ++pos, x &= x - 1u) bits[w0 + m] |= x & (0u - x);
    }
    if (threadIdx.x == 0) sh.before += gone;
    __syncthreads();
  }
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
}

}  // namespace

hipError_t launch_emit(const HashSet& hs, int64_t d, int num_cus, const SelectBufs& b, hipStream_t s,
                       const float* merged, int64_t k, int pruned, int level, int32_t* idx, int64_t* n_heavy,
                       double* l2sq, const GatherArgs* ga) {
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
  a.out = idx;
  a.n_heavy = n_heavy;
  a.l2sq = l2sq;
  a.d = d;
  a.k = (uint32_t)k;
  a.pruned = pruned;
  a.level = level;
  const unsigned blocks = (unsigned)((d + a.range - 1) / a.range);
  // The emit gathers what each workgroup has written, unless one could have so much of it (the selection
  // in one part of d, a layer's gradients) that it would work alone: more than 12 passes of its threads,
  // in a selection of at most d/8. With all large estimates within d/256, 66M x 16 takes 10.9 ms so, 10.1
  // with a gather of its own, 25.6M x 8 worker-major 1,968 and 1,662 us, 14.7M x 4 712 and 675; where they
  // are spread the kernel more costs 2 us (14.7M x 4 659 and 661; 1.2M x 6, 12 passes at most, 119
  // and 122). Beyond d/8 no workgroup has more than 8 times the mean (14.7M x 4, k = d/4: spread
  // 1,402 and 1,437 us, in one quarter of d 1,431 and 1,454).
  const bool own = !ga || std::min(k, a.range) * ga->gl <= 12 * kBlock || 8 * k > d;
  hipLaunchKernelGGL(k_emit, dim3(blocks), dim3(kBlock), (size_t)(a.range / 32) * sizeof(uint32_t), s, a, hs,
                     ga && own ? *ga : GatherArgs{});
  const hipError_t e = hipGetLastError();
  if (e != hipSuccess || own) return e;
  return launch_gather(num_cus, s, hs, merged, idx, k, *ga);
}

hipError_t prepare_emit() {
  return hipFuncSetAttribute(reinterpret_cast<const void*>(&k_emit), hipFuncAttributeMaxDynamicSharedMemorySize,
                             kRangeMax / 8);
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
