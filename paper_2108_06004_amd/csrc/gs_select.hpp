// gs_select.hpp -- block-level building blocks of the selection kernels (gfx950), the order in
// which candidate keys are binned, and the exact-value gather that a selection kernel may run on
// the indices it has just written.
#pragma once
#include "gs_device.hpp"
#include "gs_internal.hpp"

namespace gs {

// Inclusive prefix sum of x over the threads of a block of BS threads (BS a multiple of 64,
// at most 64 waves). sh must hold BS/64 words. All threads must call it.
template <int BS>
__device__ __forceinline__ uint32_t block_scan_incl(uint32_t x, uint32_t* sh, uint32_t& total) {
  constexpr int kWaves = BS / 64;
  const int lane = threadIdx.x & 63, wid = threadIdx.x >> 6;
#pragma unroll
  for (int o = 1; o < 64; o <<= 1) {
    const uint32_t y = __shfl_up(x, o, 64);
    if (lane >= o) x += y;
  }
  if (lane == 63) sh[wid] = x;
  __syncthreads();
  if (wid == 0) {
    uint32_t w = lane < kWaves ? sh[lane] : 0u;
#pragma unroll
    for (int o = 1; o < 64; o <<= 1) {
      const uint32_t y = __shfl_up(w, o, 64);
      if (lane >= o) w += y;
    }
    if (lane < kWaves) sh[lane] = w;
  }
  __syncthreads();
  total = sh[kWaves - 1];
  const uint32_t add = wid ? sh[wid - 1] : 0u;
  __syncthreads();
  return x + add;
}

// Scan the histogram h[NB] (LDS or global; NB a multiple of BS, at most 16 bins per
// thread) in descending or ascending bin order and find the first bin at which the running
// count reaches `need` (1 <= need <= total). res[0] = that bin, res[1] = count in the bins
// before it (in scan order). Each thread reads its bins once. All threads must call it.
template <int BS, int NB>
__device__ __forceinline__ void find_bucket(const uint32_t* h, bool descending, uint32_t need, uint32_t* shw, uint32_t* res) {
  constexpr int kPer = NB / BS;
  static_assert(kPer >= 1 && kPer * BS == NB && kPer <= 16, "bins per thread");
  uint32_t cnt[kPer];
  uint32_t sum = 0;
#pragma unroll
  for (int m = 0; m < kPer; ++m) {
    const int pos = threadIdx.x * kPer + m;
    cnt[m] = h[descending ? NB - 1 - pos : pos];
    sum += cnt[m];
  }
  uint32_t total;
  const uint32_t incl = block_scan_incl<BS>(sum, shw, total);
  const uint32_t excl = incl - sum;
  if (excl < need && need <= incl) {
    uint32_t run = excl;
    for (int m = 0; m < kPer; ++m) {
      if (run + cnt[m] >= need) {
        const int pos = threadIdx.x * kPer + m;
        res[0] = (uint32_t)(descending ? NB - 1 - pos : pos);
        res[1] = run;
        break;
      }
      run += cnt[m];
    }
  }
  __syncthreads();
}

// Adds 1 to the LDS histogram bin `bin` of every lane with `take` set; every lane of the
// wave must call it. The lanes whose bin equals that of the first taking lane add with one
// atomic, so runs of equal keys (all-zero estimates, say) do not serialise on one address.
__device__ __forceinline__ void hist_add(uint32_t* h, bool take, uint32_t bin) {
  const uint64_t act = __ballot(take);
  if (act == 0ull) return;
  const int first = __builtin_ctzll(act);
  const uint32_t b0 = __shfl(bin, first, 64);
  const uint64_t same = __ballot(take && bin == b0);
  if (take && bin != b0) atomicAdd(&h[bin], 1u);
  if ((int)(threadIdx.x & 63) == first) atomicAdd(&h[b0], (uint32_t)__popcll(same));
}

// Bins of the candidates' histogram, monotone in the key. Coarse bins, for the full estimate's keys,
// are key bits 30..19 (a sixteenth of an octave of |est|), or bits 31..20 with HEAVYMIX. Near the
// k-th key such a bin can hold as many keys as are selected. Fine bins, for the pruned pass's
// candidates, start at the sampled bound tau0, just below the k-th key, and are
// narrow there, so that the bin of the k-th key holds about a hundred keys:
//   top-k:    2,048 bins of 2^12 keys (one octave above tau0), then 2,048 of 2^16 (16 octaves);
//   HEAVYMIX: 2,048 equal bins for the fill keys in [tau0, 2^31); for the heavy ones, from the
//             smallest key est^2 >= theta allows, 1,024 of 2^12 and 1,024 of 2^17.
struct CandBins {
  uint32_t base0, sh0, base1;
  int hm, fine;
};
__device__ __forceinline__ CandBins cand_bins(uint32_t tau0, bool hm, double theta, bool fine) {
  CandBins c{tau0, hm ? 20u : 19u, 0u, hm ? 1 : 0, fine ? 1 : 0};
  if (hm && fine) {
    const uint32_t last = 0x7fffffffu - tau0;  // tau0 < 2^31 (a 31-bit draw)
    const int bits = 32 - __clz(last | 1u);
    c.sh0 = bits > 11 ? (uint32_t)(bits - 11) : 0u;
    // at most the key of any |est| with est^2 >= theta (any value here keeps the bins monotone)
    const uint32_t root = __float_as_uint((float)sqrt(theta)) & 0x7fffffffu;
    c.base1 = 0x80000000u | (root > 0u ? root - 1u : 0u);
  }
  return c;
}
__device__ __forceinline__ uint32_t cand_bin(const CandBins& c, uint32_t key) {
  if (!c.fine) return key >> c.sh0;
  if (!c.hm) {
    const uint32_t o = key > c.base0 ? key - c.base0 : 0u;
    return o < (1u << 23) ? o >> 12 : 2048u + min((o - (1u << 23)) >> 16, 2047u);
  }
  if (key < 0x80000000u) return min((key > c.base0 ? key - c.base0 : 0u) >> c.sh0, 2047u);
  const uint32_t o = key > c.base1 ? key - c.base1 : 0u;
  return o < (1u << 22) ? 2048u + (o >> 12) : 3072u + min((o - (1u << 22)) >> 17, 1023u);
}
// The smallest key of bin b that is not in bin b - 1 (2^32 for b = kDigit1Bins).
__device__ __forceinline__ uint64_t cand_bin_lo(const CandBins& c, uint32_t b) {
  if (b == 0) return 0;
  if (!c.fine) return (uint64_t)b << c.sh0;
  if (b >= (uint32_t)kDigit1Bins) return 1ull << 32;
  if (!c.hm) return c.base0 + (b < 2048u ? (uint64_t)b << 12 : (1ull << 23) + ((uint64_t)(b - 2048u) << 16));
  uint64_t lo;
  if (b < 2048u) {
    lo = c.base0 + ((uint64_t)b << c.sh0);
    return lo < (1ull << 31) ? lo : 1ull << 31;
  }
  if (b == 2048u) return 1ull << 31;
  lo = c.base1 + (b < 3072u ? (uint64_t)(b - 2048u) << 12 : (1ull << 22) + ((uint64_t)(b - 3072u) << 17));
  return lo < (1ull << 32) ? lo : 1ull << 32;
}

// Median estimate with r rows at run time, sorted by insertion in the thread's own kMaxRows floats
// of LDS: small code for the few values of the sketch-space state. Unrolled over kMaxRows in registers, the
// rows' hash constants crowded the scalar registers of the whole kernel.
__device__ __forceinline__ float estimate_any(const HashSet& hs, const float* __restrict__ merged, uint32_t i,
                                              float* val) {
  const int r = hs.r;
#pragma nounroll
  for (int j = 0; j < r; ++j) {
    uint32_t col, sflip;
    hash_ij(hs, j, i, col, sflip);
    const float x = apply_sign(merged[(int64_t)j * hs.c + col], sflip);
    int b = j;
#pragma nounroll
    for (; b > 0 && val[b - 1] > x; --b) val[b] = val[b - 1];
    val[b] = x;
  }
  if (r & 1) return val[r / 2];
  const float s = val[r / 2 - 1] + val[r / 2];
  return s * 0.5f;
}

// The exact values of selected coordinates and their reset (Alg. 2, second round), by the
// threads of one block or of a whole grid: entry t of idx[0, n) goes to lane group (first +
// t's turn). A group of gl lanes (a power of two) shares a coordinate.
//   rows:    the interleaved state, 16-byte aligned: lane sub holds the row's piece of workers
//            4 sub .. 4 sub + 3, so a row is one coalesced access (4 gl >= PP)
//   workers: any strides and alignment: lane sub holds worker sub (gl >= P)
// The tree runs in the lane's own four (strides 1, 2), then across lanes; an element absorbs its
// partner only if that worker exists, so the sums are those of tree_sum.
__device__ __forceinline__ void gather_entry(const GatherArgs& a, int64_t i, int64_t t, int sub) {
  if (a.op == kGatherRows) {
    typedef float f4 __attribute__((ext_vector_type(4)));
    const int nw = a.P - 4 * sub;  // workers from this lane's first one on
    const int64_t o = i * a.PP + 4 * sub;
    f4 x = {0.f, 0.f, 0.f, 0.f};
    if (nw > 0) x = *reinterpret_cast<const f4*>(a.v + o);
    if (nw > 1) x.x = x.x + x.y;
    if (nw > 3) x.z = x.z + x.w;
    float y = nw > 2 ? x.x + x.z : x.x;
    for (int s = 1; s < a.gl; s <<= 1) {
      const float z = __shfl_down(y, s, a.gl);
      if (nw > 4 * s) y = y + z;
    }
    if (sub == 0) a.values[t] = y;
    const f4 zero = {0.f, 0.f, 0.f, 0.f};
    if (nw >= 4) {
      *reinterpret_cast<f4*>(a.v + o) = zero;
      if (a.reset_u) *reinterpret_cast<f4*>(a.u + o) = zero;
    } else {
      for (int q = 0; q < nw; ++q) {  // the row's padding is not written
        a.v[o + q] = 0.f;
        if (a.reset_u) a.u[o + q] = 0.f;
      }
    }
  } else {
    const bool mine = sub < a.P;
    const int64_t o = a.sv.at(sub, i);
    float y = mine ? a.v[o] : 0.f;
    for (int s = 1; s < a.gl; s <<= 1) {
      const float z = __shfl_down(y, s, a.gl);
      if (sub + s < a.P) y = y + z;
    }
    if (sub == 0) a.values[t] = y;
    if (mine) {
      a.v[o] = 0.f;
      if (a.reset_u) a.u[o] = 0.f;
    }
  }
}

}  // namespace gs
