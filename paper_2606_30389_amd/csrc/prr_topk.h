// Exact top-K of up to 16384 pages by one 256-thread workgroup, from keys in memory: the
// selection of Section 2.1 / Appendix A.1 and the predicted set of Section 4.1 for the
// separate kernels, whose pages are scored by many workgroups (the last to finish selects).
//
// The one selecting workgroup is bound by its instructions per key and by the loads one CU
// can make, so it looks at few keys.  The scoring workgroups also publish the largest key of
// every group of 4 (above 8192 pages: 8) consecutive pages; the K-th largest of those bounds
// the threshold from below (K groups hold a key that large), only the groups that reach it are
// loaded, and the keys at or above it (about 1.1 K of them) are compacted to LDS in page order
// and ranked.  A load costs a memory round trip, so the loads of a step are issued together:
// the groups' keys, up to eight per thread, then theirs.
//
// rank_keys() finds the bin that holds a rank: one histogram over 1024 bins linear in the
// value (the scores of a head share their leading key bits, so bins over key bits would hold
// most of them), then, only where that bin still holds many keys (outliers, infinities),
// further passes over key bits.  Every wave owns a contiguous range of pages and a segment of
// the list of its own, so lists are in page order without a scan over the workgroup.
#pragma once

#include "prr_device.h"
#include "prr_launch.h"

namespace prr {

constexpr int kTopkThreads = 256;
constexpr int kTopkWaves = kTopkThreads / kWave;
constexpr int kTopkLog2Bins = 10;
constexpr int kTopkBins = 1 << kTopkLog2Bins;
constexpr int kTopkPasses = (32 + kTopkLog2Bins - 1) / kTopkLog2Bins;
constexpr int kTopkSmall = 64;      // keys of the boundary bin ranked directly by one wave
constexpr int kTopkSeg = 512;       // list entries of a wave
constexpr int kTopkEntRegs = kTopkSeg / kWave;  // of a lane
constexpr int kTopkForced = 1 << 30;  // flag of a listed page
constexpr int kTopkMaxGroups = 2048;
constexpr int kTopkGroupRegs = kTopkMaxGroups / kTopkThreads;  // groups of a thread
constexpr int kTopkDirect = kTopkWaves * kTopkSeg;             // pages listed without a bound
static_assert(kTopkMaxGroups * 8 >= PRR_MAX_PAGES_DEV, "groups of eight pages cover every page");

struct __align__(16) TopkLds {
  uint32_t ck[kTopkWaves][kTopkSeg];  // the listed keys
  uint16_t cp[kTopkWaves][kTopkSeg];  // their pages (bit 15: forced)
  uint16_t glist[kTopkMaxGroups];     // the groups that reach the bound, per wave
  uint32_t hist[kTopkBins];
  uint32_t forceb[PRR_MAX_PAGES_DEV / 32];
  uint32_t small[kTopkSmall];
  uint32_t kred[2][kTopkWaves];
  int nsmall;
  int red[4][kTopkWaves];
  int res[6];
};

// log2 of the pages per group for a select among n pages; 0 = every key is listed (up to 2048
// pages, eight per thread, one load of all keys is cheaper than the groups' and then theirs).
__host__ __device__ inline int topk_group_shift(int n) {
  return n <= kTopkDirect ? 0 : n <= 4 * kTopkMaxGroups ? 2 : 3;
}

// Whether a select of k of n pages with n_forced more always taken leaves the bound too low:
// with fewer than twice as many groups as it counts (a budget of more than an eighth of the
// pages) most keys may reach it.
inline bool topk_crowded(int n, int k, int n_forced) {
  const int s = topk_group_shift(n);
  return s > 0 && 2 * (k + n_forced) > (n + (1 << s) - 1) >> s;
}

// the float whose score_key is k
__device__ __forceinline__ float topk_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

// One wave: the bin (from the top) of `hist` that holds rank `rank`, the count above it and
// its own count, to res[0..2].  Where fewer keys than that were counted (see rank_keys): the
// lowest bin.
template <int BINS>
__device__ __forceinline__ void scan_bins(const uint32_t* hist, int rank, int* res) {
  constexpr int PL = BINS / kWave;  // bins per lane
  static_assert(PL % 4 == 0 && PL <= kWave, "bins per lane");
  const int lane = lane_id();
  const uint4* hb = reinterpret_cast<const uint4*>(hist + BINS - PL * (lane + 1));
  int sum = 0;
#pragma unroll
  for (int v = 0; v < PL / 4; ++v) {
    const uint4 x = hb[v];
    sum += (int)(x.x + x.y + x.z + x.w);
  }
  const int incl = wave_inclusive_scan(sum);
  const int excl = incl - sum;
  const uint64_t hit = __ballot(excl < rank && rank <= incl);
  const int ls = hit != 0ull ? __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1) : kWave - 1;
  const int ex = __builtin_amdgcn_readlane(excl, ls);
  const int lbase = BINS - PL * (ls + 1);
  const int cj = lane < PL ? (int)hist[lbase + PL - 1 - lane] : 0;
  const int cinc = wave_inclusive_scan(cj);
  const uint64_t hit2 = __ballot(lane < PL && ex + cinc >= rank);
  const int js = hit2 != 0ull ? __builtin_amdgcn_readfirstlane(__ffsll((long long)hit2) - 1) : PL - 1;
  if (lane == js) {
    res[0] = lbase + PL - 1 - js;
    res[1] = ex + cinc - cj;
    res[2] = cj;
  }
}

__device__ __forceinline__ void topk_clear_hist(TopkLds& S) {
  for (int b = threadIdx.x; b < kTopkBins / 4; b += kTopkThreads)
    reinterpret_cast<uint4*>(S.hist)[b] = make_uint4(0, 0, 0, 0);
}

struct TopkBin {
  // value bins (narrowed == false): the boundary bin is `bin` of the values' linear map;
  // otherwise it is the keys in [lo, hi]
  bool narrowed;
  int bin;
  float vlo, scale;
  uint32_t lo, hi;
  int above, count;  // keys in higher bins; keys of the boundary bin

  __device__ __forceinline__ int bin_of(uint32_t k) const {
    return min(kTopkBins - 1, (int)fmaxf((topk_value(k) - vlo) * scale, 0.0f));
  }
  __device__ __forceinline__ bool in(uint32_t k) const { return narrowed ? k >= lo && k <= hi : bin_of(k) == bin; }
  __device__ __forceinline__ bool at_least(uint32_t k) const { return narrowed ? k >= lo : bin_of(k) >= bin; }
  // A key no larger than any of the boundary bin's.  Of a value bin: the lower edge of the bin
  // below it (its width covers the rounding of the map, at most 2^-22 of 1024 bins), less two
  // units for the rounding of the edge itself.
  __device__ __forceinline__ uint32_t bound() const {
    if (narrowed) return lo;
    if (bin == 0) return lo;
    return max(lo, score_key(vlo + (float)(bin - 1) / scale) - 2u);
  }
};

// The smallest and largest key for which in(k) holds to lo, hi (one barrier, after which
// S.kred is read; it is next written behind two more).
template <class EACH, class IN>
__device__ __forceinline__ void topk_range(const EACH& each, const IN& in, uint32_t& lo, uint32_t& hi, TopkLds& S) {
  uint32_t l = 0xffffffffu, h = 0u;
  each([&](uint32_t k) {
    if (in(k)) {
      l = min(l, k);
      h = max(h, k);
    }
  });
  l = wave_umin(l);
  h = wave_umax(h);
  if (lane_id() == 0) {
    S.kred[0][threadIdx.x / kWave] = l;
    S.kred[1][threadIdx.x / kWave] = h;
  }
  __syncthreads();
#pragma unroll
  for (int i = 0; i < kTopkWaves; ++i) {
    l = min(l, S.kred[0][i]);
    h = max(h, S.kred[1][i]);
  }
  lo = l;
  hi = h;
}

// The boundary bin of rank `rank` among the keys that `each(f)` hands to f (this thread's;
// all of them in [lo, hi], at least `rank` over the workgroup), narrowed until it holds at
// most `slack` keys or one value.  The histogram is zero on entry and, behind the caller's
// next barrier, on return.
// Both holds only as long as the keys and the group maxima in memory belong together; where a
// caller lets them be overwritten, the result is unspecified but this still ends: a pass over
// key bits leaves at most 2^-10 of its range (kTopkPasses cover 32 bits), and a bin that holds
// none of the keys ends it, as its range is empty.
template <class EACH>
__device__ __forceinline__ TopkBin rank_keys(const EACH& each, int rank, int slack, uint32_t lo, uint32_t hi,
                                             TopkLds& S) {
  TopkBin b;
  b.vlo = topk_value(lo);
  const float span = topk_value(hi) - b.vlo;
  b.scale = (float)kTopkBins / span;
  b.lo = lo;
  b.hi = hi;
  b.above = 0;
  b.count = 0x7fffffff;
  b.bin = 0;
  b.narrowed = !(span > 0.0f && __builtin_isfinite(span) && __builtin_isfinite(b.scale));
  if (!b.narrowed) {
    each([&](uint32_t k) { atomicAdd(&S.hist[b.bin_of(k)], 1u); });
    __syncthreads();
    if (threadIdx.x < kWave) scan_bins<kTopkBins>(S.hist, rank, S.res);
    __syncthreads();
    b.bin = S.res[0];
    b.above = S.res[1];
    b.count = S.res[2];
    topk_clear_hist(S);
    if (b.count <= slack) return b;
    topk_range(each, [&](uint32_t k) { return b.bin_of(k) == b.bin; }, b.lo, b.hi, S);
    b.narrowed = true;
  }
  for (int pass = 0; pass < kTopkPasses && b.count > slack && b.lo < b.hi; ++pass) {
    const uint32_t klo = b.lo, khi = b.hi;
    const int bits = 32 - __clz(khi - klo), shift = bits > kTopkLog2Bins ? bits - kTopkLog2Bins : 0;
    each([&](uint32_t k) {
      if (k >= klo && k <= khi) atomicAdd(&S.hist[(k - klo) >> shift], 1u);
    });
    __syncthreads();
    if (threadIdx.x < kWave) scan_bins<kTopkBins>(S.hist, rank - b.above, S.res);
    __syncthreads();
    const uint32_t bs = (uint32_t)S.res[0];
    b.above += S.res[1];
    b.count = S.res[2];
    topk_clear_hist(S);
    topk_range(each, [&](uint32_t k) { return k >= klo && k <= khi && (k - klo) >> shift == bs; }, b.lo, b.hi, S);
  }
  return b;
}

// The exact top-kextra of pages [0, n) (key descending, page ascending) and the forced pages,
// in page order, to out[0, cap) with the count to *out_count.  key_of(p): the key of page p;
// gmax_of(g): the largest key of pages [g << gshift, (g + 1) << gshift) (not called when
// gshift is 0).  Called by every thread of a workgroup of 256.
template <class GMAX, class KEY>
__device__ __forceinline__ void topk_select(int n, int gshift, int kextra, const int32_t* forced, int n_forced,
                                            const GMAX& gmax_of, const KEY& key_of,
                                            int32_t* __restrict__ out, int cap,
                                            int32_t* __restrict__ out_count, TopkLds& S) {
  const int t = threadIdx.x, lane = lane_id(), w = __builtin_amdgcn_readfirstlane(t / kWave);
  if (kextra <= 0 || kextra >= n - n_forced) {  // only the forced pages, or every page
    const int total = kextra <= 0 ? n_forced : n;
    if (kextra > 0) {
      for (int i = t; i < min(n, cap); i += kTopkThreads) out[i] = i;
    } else if (t < n_forced) {
      int r = 0;
      for (int i = 0; i < n_forced; ++i) r += forced[i] < forced[t] ? 1 : 0;
      if (r < cap) out[r] = forced[t];
    }
    if (t == 0) *out_count = min(total, cap);
    return;
  }
  topk_clear_hist(S);
  if (t == 0) S.nsmall = 0;
  if (n_forced > 0) {
    for (int i = t; i < (n + 31) / 32; i += kTopkThreads) S.forceb[i] = 0u;
    __syncthreads();
    if (t < n_forced) atomicOr(&S.forceb[forced[t] >> 5], 1u << (forced[t] & 31));
    __syncthreads();
  }
  const auto is_forced = [&](int p) { return n_forced > 0 && ((S.forceb[p >> 5] >> (p & 31)) & 1u); };
  constexpr int kBatch = 10;  // key loads of a lane in flight
  int c = 0;                  // entries of this wave
  uint32_t ek[kTopkEntRegs];  // entry 64 r + lane: its key ..
  int ep[kTopkEntRegs];       // .. and page (bit 30: forced; -1: none)
  uint32_t lo = 0xffffffffu, hi = 0u;
  if (gshift > 0) {
    // this wave's groups: gbase + 64 r + lane, below gend
    const int ng = (n + (1 << gshift) - 1) >> gshift;
    const int gw = ((ng + kTopkWaves - 1) / kTopkWaves + kWave - 1) / kWave * kWave;
    const int gbase = w * gw, gend = min(ng, gbase + gw);
    uint32_t gm[kTopkGroupRegs];
#pragma unroll
    for (int r = 0; r < kTopkGroupRegs; ++r) gm[r] = gmax_of(min(gbase + r * kWave + lane, ng - 1));
#pragma unroll
    for (int r = 0; r < kTopkGroupRegs; ++r) {
      if (gbase + r * kWave + lane < gend) {
        lo = min(lo, gm[r]);
        hi = max(hi, gm[r]);
      }
    }
    lo = wave_umin(lo);
    hi = wave_umax(hi);
    if (lane == 0) {
      S.red[0][w] = (int)lo;
      S.red[1][w] = (int)hi;
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < kTopkWaves; ++i) {
      lo = min(lo, (uint32_t)S.red[0][i]);
      hi = max(hi, (uint32_t)S.red[1][i]);
    }
    // forced pages may be among the groups' largest: the bound counts that many more
    const int want = kextra + n_forced;
    const TopkBin b = rank_keys(
        [&](const auto& f) {
#pragma unroll
          for (int r = 0; r < kTopkGroupRegs; ++r)
            if (gbase + r * kWave + lane < gend) f(gm[r]);
        },
        min(want, ng), max(kTopkSmall, want / 4), lo, hi, S);
    const uint32_t bound = want <= ng ? b.bound() : 0u;
    // this wave's groups that reach the bound (or hold a forced page), then their keys that do
    int cg = 0;
#pragma unroll
    for (int r = 0; r < kTopkGroupRegs; ++r) {
      const int g = gbase + r * kWave + lane, p = min(g, ng - 1) << gshift;
      const bool pass = g < gend && (gm[r] >= bound ||
                                     (n_forced > 0 && ((S.forceb[p >> 5] >> (p & 31)) & ((1u << (1 << gshift)) - 1u)) != 0u));
      const uint64_t bm = __ballot(pass);
      if (pass) S.glist[gbase + cg + lanes_below(bm)] = (uint16_t)g;
      cg += __popcll(bm);
    }
    __builtin_amdgcn_wave_barrier();
    const int items = cg << gshift;
    int ceq = 0;  // keys equal to the bound: ties are taken in page order, so the first kextra do
    for (int i0 = 0; i0 < items; i0 += kBatch * kWave) {
      uint32_t k[kBatch];
      int pg[kBatch];
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        const int i = i0 + u * kWave + lane;
        const int p = ((int)S.glist[gbase + (min(i, items - 1) >> gshift)] << gshift) + (i & ((1 << gshift) - 1));
        pg[u] = i < items && p < n ? p : -1;
        k[u] = key_of(max(pg[u], 0));
      }
#pragma unroll
      for (int u = 0; u < kBatch; ++u) {
        if (i0 + u * kWave >= items) break;
        const bool f = pg[u] >= 0 && is_forced(pg[u]);
        bool pass = pg[u] >= 0 && (f || k[u] >= bound);
        uint64_t bm = __ballot(pass);
        const uint64_t em = __ballot(pass && !f && k[u] == bound);
        if (em != 0ull) {
          pass = pass && !(((em >> lane) & 1ull) && ceq + lanes_below(em) >= kextra);
          ceq += __popcll(em);
          bm = __ballot(pass);
        }
        const int pos = c + lanes_below(bm);
        if (pass && pos < kTopkSeg) {
          S.ck[w][pos] = k[u];
          S.cp[w][pos] = (uint16_t)(pg[u] | (f ? 0x8000 : 0));
        }
        c += __popcll(bm);
      }
    }
    lo = bound;  // (the smallest listed key or below it; hi: the largest)
    __builtin_amdgcn_wave_barrier();
#pragma unroll
    for (int r = 0; r < kTopkEntRegs; ++r) {
      const int i = r * kWave + lane;
      const int pv = i < c ? (int)S.cp[w][i] : -1;
      ek[r] = i < c ? S.ck[w][i] : 0u;
      ep[r] = pv < 0 ? -1 : (pv & 0x7fff) | ((pv & 0x8000) ? kTopkForced : 0);
    }
  } else {
    const int pw = ((n + kTopkWaves - 1) / kTopkWaves + kWave - 1) / kWave * kWave;
    const int pbase = w * pw, pend = min(n, pbase + pw);
#pragma unroll
    for (int r = 0; r < kTopkEntRegs; ++r) ek[r] = key_of(min(pbase + r * kWave + lane, n - 1));
#pragma unroll
    for (int r = 0; r < kTopkEntRegs; ++r) {
      const int p = pbase + r * kWave + lane;
      ep[r] = p < pend ? p | (is_forced(p) ? kTopkForced : 0) : -1;
      if (ep[r] >= 0 && ep[r] < kTopkForced) {
        lo = min(lo, ek[r]);
        hi = max(hi, ek[r]);
      }
    }
    c = max(0, pend - pbase);
    lo = wave_umin(lo);
    hi = wave_umax(hi);
  }
  if (lane == 0) {
    S.red[2][w] = c;
    if (gshift == 0) {
      S.red[0][w] = (int)lo;
      S.red[1][w] = (int)hi;
    }
  }
  __syncthreads();
  int most = 0;
#pragma unroll
  for (int i = 0; i < kTopkWaves; ++i) {
    most = max(most, S.red[2][i]);
    if (gshift == 0) {
      lo = min(lo, (uint32_t)S.red[0][i]);
      hi = max(hi, (uint32_t)S.red[1][i]);
    }
  }
  if (most <= kTopkSeg) {
    const TopkBin b = rank_keys(
        [&](const auto& f) {
#pragma unroll
          for (int r = 0; r < kTopkEntRegs; ++r) {
            if (r * kWave >= c) break;
            if ((uint32_t)ep[r] < (uint32_t)kTopkForced) f(ek[r]);
          }
        },
        kextra, kTopkSmall, lo, hi, S);
    const int rank = kextra - b.above;  // among the boundary bin's keys
    uint32_t T = b.lo;
    int need_eq = rank, eq_total = b.count;  // (one value, or the whole bin is taken)
    const bool whole = rank == b.count;
    if (!whole && !(b.narrowed && b.lo == b.hi)) {
      // the few keys of the boundary bin, ranked directly by one wave
#pragma unroll
      for (int r = 0; r < kTopkEntRegs; ++r) {
        if (r * kWave >= c) break;
        if ((uint32_t)ep[r] < (uint32_t)kTopkForced && b.in(ek[r])) {
          const int i = atomicAdd(&S.nsmall, 1);
          if (i < kTopkSmall) S.small[i] = ek[r];
        }
      }
      __syncthreads();
      if (w == 0) {
        const int nb = min(b.count, kTopkSmall);
        const uint32_t kx = S.small[lane < nb ? lane : 0];
        int gt = 0, ge = 0;
        for (int x = 0; x < nb; ++x) {
          const uint32_t ky = (uint32_t)__builtin_amdgcn_readlane((int)kx, x);
          gt += ky > kx ? 1 : 0;
          ge += ky >= kx ? 1 : 0;
        }
        const uint64_t hit = __ballot(lane < nb && gt < rank && rank <= ge);
        const int ls = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
        if (lane == ls) {
          S.res[3] = (int)kx;
          S.res[4] = rank - gt;
          S.res[5] = ge - gt;
        }
      }
      __syncthreads();
      T = (uint32_t)S.res[3];
      need_eq = S.res[4];
      eq_total = S.res[5];
    }
    const bool cut = !whole && need_eq < eq_total;  // the first need_eq keys equal to T, in page order
    uint64_t inm[kTopkEntRegs], eqm[kTopkEntRegs];
    int ci = 0, ce = 0;
#pragma unroll
    for (int r = 0; r < kTopkEntRegs; ++r) {
      inm[r] = eqm[r] = 0ull;
      if (r * kWave >= c) continue;
      const bool f = ep[r] >= kTopkForced, e = !f && ep[r] >= 0;
      inm[r] = __ballot(f || (e && (whole ? b.at_least(ek[r]) : cut ? ek[r] > T : ek[r] >= T)));
      eqm[r] = cut ? __ballot(e && ek[r] == T) : 0ull;
      ci += __popcll(inm[r]);
      ce += __popcll(eqm[r]);
    }
    if (cut) {
      if (lane == 0) S.red[3][w] = ce;
      __syncthreads();
      int run = 0;
      for (int i = 0; i < w; ++i) run += S.red[3][i];
#pragma unroll
      for (int r = 0; r < kTopkEntRegs; ++r) {
        if (r * kWave >= c) break;
        const bool e = (eqm[r] >> lane) & 1ull;
        const uint64_t taken = __ballot(e && run + lanes_below(eqm[r]) < need_eq);
        run += __popcll(eqm[r]);
        inm[r] |= taken;
        ci += __popcll(taken);
      }
    }
    if (lane == 0) S.red[0][w] = ci;  // (last read before the barriers of rank_keys)
    __syncthreads();
    int pos = 0, total = 0;
#pragma unroll
    for (int i = 0; i < kTopkWaves; ++i) {
      const int x = S.red[0][i];
      pos += i < w ? x : 0;
      total += x;
    }
#pragma unroll
    for (int r = 0; r < kTopkEntRegs; ++r) {
      if (r * kWave >= c) break;
      const int q = pos + lanes_below(inm[r]);
      if (((inm[r] >> lane) & 1ull) && q < cap) out[q] = ep[r] & (kTopkForced - 1);
      pos += __popcll(inm[r]);
    }
    if (t == 0) *out_count = min(total, cap);
    return;
  }
  // More keys reach the bound than the list holds (large clusters of pages): an exact radix
  // select over all keys in memory, eight key bits per pass.
  uint32_t prefix = 0u, mask = 0u;
  int rank = kextra, eq_total = 0;
  constexpr int kSlow = 16;
  for (int shift = 24; shift >= 0; shift -= 8) {
    for (int p0 = 0; p0 < n; p0 += kSlow * kTopkThreads) {
      uint32_t k[kSlow];
#pragma unroll
      for (int u = 0; u < kSlow; ++u) k[u] = key_of(min(p0 + u * kTopkThreads + t, n - 1));
#pragma unroll
      for (int u = 0; u < kSlow; ++u) {
        const int p = p0 + u * kTopkThreads + t;
        if (p < n && (k[u] & mask) == prefix && !is_forced(p)) atomicAdd(&S.hist[(k[u] >> shift) & 255u], 1u);
      }
    }
    __syncthreads();
    if (w == 0) scan_bins<256>(S.hist, rank, S.res);
    __syncthreads();
    prefix |= (uint32_t)S.res[0] << shift;
    mask |= 255u << shift;
    rank -= S.res[1];
    eq_total = S.res[2];
    topk_clear_hist(S);
    __syncthreads();
  }
  const int pw = ((n + kTopkWaves - 1) / kTopkWaves + kWave - 1) / kWave * kWave;
  const int pbase = w * pw, pend = min(n, pbase + pw);
  uint64_t gtm = 0, eqm = 0;  // bit r: page pbase + r * 64 + lane
  for (int r0 = 0; pbase + r0 * kWave < pend; r0 += kSlow) {
    uint32_t k[kSlow];
#pragma unroll
    for (int u = 0; u < kSlow; ++u) k[u] = key_of(min(pbase + (r0 + u) * kWave + lane, n - 1));
#pragma unroll
    for (int u = 0; u < kSlow; ++u) {
      const int p = pbase + (r0 + u) * kWave + lane;
      if (p < pend) {
        const bool f = is_forced(p);
        if (f || k[u] > prefix) gtm |= 1ull << (r0 + u);
        if (!f && k[u] == prefix) eqm |= 1ull << (r0 + u);
      }
    }
  }
  const int ce = wave_isum(__popcll(eqm));
  if (lane == 0) S.red[3][w] = ce;
  __syncthreads();
  int run = 0;
  for (int i = 0; i < w; ++i) run += S.red[3][i];
  for (int r = 0; pbase + r * kWave < pend; ++r) {
    const bool e = (eqm >> r) & 1ull;
    const uint64_t bm = __ballot(e);
    if (e && run + lanes_below(bm) < rank) gtm |= 1ull << r;
    run += __popcll(bm);
  }
  (void)eq_total;
  const int ci = wave_isum(__popcll(gtm));
  if (lane == 0) S.red[0][w] = ci;
  __syncthreads();
  int pos = 0, total = 0;
#pragma unroll
  for (int i = 0; i < kTopkWaves; ++i) {
    const int x = S.red[0][i];
    pos += i < w ? x : 0;
    total += x;
  }
  for (int r = 0; pbase + r * kWave < pend; ++r) {
    const bool in = (gtm >> r) & 1ull;
    const uint64_t bm = __ballot(in);
    const int q = pos + lanes_below(bm);
    if (in && q < cap) out[q] = pbase + r * kWave + lane;
    pos += __popcll(bm);
  }
  if (t == 0) *out_count = min(total, cap);
}

}  // namespace prr
