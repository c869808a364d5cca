// gfx950 (CDNA4) kernels of the speculate-reuse-repair decode path.
//
//   meta_minmax / meta_mean   page metadata (Appendix A.1; block means)
//   predict                   EMA update and prediction (Section 4.1, Eqs. (2)-(3)) + top-|P|
//                             by one workgroup per KV head, without scratch
//   merge_states              stand-alone merge of partial states
//
// (score + select, speculate and repair: prr_sep.h.)  Wave64 throughout.
#include <algorithm>

#include "prr_device.h"
#include "prr_launch.h"
#include "prr_select.h"

namespace prr {


// =====================================================================================
// epoch of captured fused steps: one thread advances the word (skipping 0)
// =====================================================================================

__global__ void epoch_advance_kernel(uint32_t* p) {
  if (threadIdx.x == 0) {
    const uint32_t v = *p + 1u;
    *p = v == 0u ? 1u : v;
  }
}

hipError_t launch_epoch_advance(uint32_t* epoch_dev, hipStream_t stream) {
  void* args[] = {&epoch_dev};
  return hipLaunchKernel((const void*)epoch_advance_kernel, dim3(1), dim3(64), args, 0, stream);
}

// =====================================================================================
// workspace fill
// =====================================================================================

// An empty kernel: the launch floor of a grid of a given shape.
__global__ void empty_kernel() {}

hipError_t launch_empty(int grid, int threads, hipStream_t stream) {
  return hipLaunchKernel((const void*)empty_kernel, dim3(grid), dim3(threads), nullptr, 0, stream);
}

// Read-stream rate: every 16-byte word of the buffer read once (eight loads in flight
// per thread, consecutive lanes on consecutive words), folded into one word per
// workgroup so that the loads stay live.
__global__ void __launch_bounds__(256) read_stream_kernel(const u32x4_t* __restrict__ p, size_t n16,
                                                          uint32_t* __restrict__ sink) {
  constexpr int kU = 8;
  const size_t stride = (size_t)gridDim.x * 256;
  uint32_t acc = 0;
  size_t i = (size_t)blockIdx.x * 256 + threadIdx.x;
  for (; i + (kU - 1) * stride < n16; i += kU * stride) {
    u32x4_t v[kU];
#pragma unroll
    for (int u = 0; u < kU; ++u) v[u] = __builtin_nontemporal_load(p + i + u * stride);
#pragma unroll
    for (int u = 0; u < kU; ++u) acc ^= v[u].x ^ v[u].y ^ v[u].z ^ v[u].w;
  }
  for (; i < n16; i += stride) {
    const u32x4_t v = p[i];
    acc ^= v.x ^ v.y ^ v.z ^ v.w;
  }
  __shared__ uint32_t red[4];
  for (int o = 32; o > 0; o >>= 1) acc ^= __shfl_xor(acc, o);
  if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = acc;
  __syncthreads();
  if (threadIdx.x == 0) sink[blockIdx.x] = red[0] ^ red[1] ^ red[2] ^ red[3];
}

hipError_t launch_read_stream(const void* p, size_t bytes, uint32_t* sink, int grid, hipStream_t stream) {
  read_stream_kernel<<<grid, 256, 0, stream>>>(static_cast<const u32x4_t*>(p), bytes / 16, sink);
  return hipGetLastError();
}

__global__ void fill_zero_kernel(u32x4_t* __restrict__ p, size_t n16) {
  const size_t stride = (size_t)gridDim.x * blockDim.x;
  for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < n16; i += stride) p[i] = u32x4_t{0, 0, 0, 0};
}

hipError_t launch_fill_zero(void* p, size_t bytes, hipStream_t stream) {
  const size_t n16 = bytes / 16;
  if (n16 == 0) return hipSuccess;
  size_t nb = (n16 + 255) / 256;
  const unsigned grid = (unsigned)(nb < 1024 ? nb : 1024);
  u32x4_t* ptr = reinterpret_cast<u32x4_t*>(p);
  size_t n = n16;
  void* args[] = {&ptr, &n};
  return hipLaunchKernel((const void*)fill_zero_kernel, dim3(grid), dim3(256), args, 0, stream);
}

// =====================================================================================
// page metadata
// =====================================================================================
// A wave takes kPages consecutive pages (two of 16 tokens, one from 32 on).  Lane l covers
// channels 8*(l%16) .. +8 of token rows l/16, l/16+4, .. of each page (16-byte loads, a wave
// load covers 4 full rows); the loads of all its pages are issued before any is reduced (8
// per lane in flight for 16- and 32-token pages, batches of 16 from 64 tokens on), then the
// four row groups are combined by swaps of rows between pairs of registers, each of which
// reduces two values at once and leaves every lane with its share of the page's metadata to
// store (12 swaps for the minima and maxima of a page; a shuffle per value, row group and
// extreme is 32 trips through the LDS crossbar, as long as the page's own loads).  K is read
// once, with non-temporal loads.  The stores are
// non-temporal too (a layer's metadata is read again only after the other layers').  Two KV heads x
// 8192 pages of 16 tokens: 16.9 us per layer with shuffles, 16.4 now; 8 x 4096: 32.4 -> 28.3;
// 100003 tokens: 15.65 -> 13.6.  One page per wave instead of two: 17.6 / 30.1 / 12.8 us, four:
// 18.3 / 34.4 / 17.3.
template <int PS>
struct MetaShape {
  static constexpr int kPages = PS >= 32 ? 1 : 32 / PS;  // pages per wave
  static constexpr int kRows = PS / 4;                   // row loads per lane and page
  static constexpr int kBatch = kRows < 16 ? kRows : 16; // row loads per lane issued together
};

// Pages per metadata workgroup (four waves).
template <int PS>
constexpr int meta_pages_per_block() {
  return 4 * MetaShape<PS>::kPages;
}

// Rows 1 and 3 of x for rows 0 and 2 of y, and the upper half of x for the lower half of y.
__device__ __forceinline__ void swap_odd_rows(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}
__device__ __forceinline__ void swap_halves(float& x, float& y) {
  const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(y), false, false);
  x = __uint_as_float(r[0]);
  y = __uint_as_float(r[1]);
}

// The pages of this wave: source rows (lane's channels), valid tokens, and whether the
// page exists (in range, with a physical page inside the cache).
template <int PS>
__device__ __forceinline__ void meta_pages(const uint16_t* k, const int32_t* ptab, int num_tokens, int page_end,
                                           int max_pages, int h, int first, int cg,
                                           const uint16_t* (&src)[MetaShape<PS>::kPages],
                                           int (&valid)[MetaShape<PS>::kPages], bool (&ok)[MetaShape<PS>::kPages]) {
#pragma unroll
  for (int j = 0; j < MetaShape<PS>::kPages; ++j) {
    const int page = first + j;
    int phys = -1;
    if (page < page_end) phys = ptab ? ptab[page] : page;
    ok[j] = phys >= 0 && phys < max_pages;
    valid[j] = ok[j] ? min(PS, num_tokens - page * PS) : 0;
    src[j] = k + ((size_t)h * max_pages + (ok[j] ? phys : 0)) * PS * kHeadDim + cg * 8;
  }
}

template <bool BF16, int PS>
__global__ __launch_bounds__(256) void meta_minmax_kernel(const uint16_t* __restrict__ k, const int32_t* __restrict__ ptab,
                                                          int num_tokens, int page_begin, int page_end, int max_pages,
                                                          uint16_t* __restrict__ meta) {
  using S = MetaShape<PS>;
  const int h = blockIdx.y;
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int first = page_begin + (blockIdx.x * 4 + w) * S::kPages;
  if (first >= page_end) return;
  const int cg = lane & 15, rg = lane >> 4;
  const uint16_t* src[S::kPages];
  int valid[S::kPages];
  bool ok[S::kPages];
  meta_pages<PS>(k, ptab, num_tokens, page_end, max_pages, h, first, cg, src, valid, ok);
  float mn[S::kPages][8], mx[S::kPages][8];
#pragma unroll
  for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      mn[j][e] = __builtin_inff();
      mx[j][e] = -__builtin_inff();
    }
  }
#pragma unroll
  for (int b = 0; b < S::kRows; b += S::kBatch) {
    u32x4_t v[S::kPages][S::kBatch];
#pragma unroll
    for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
      for (int i = 0; i < S::kBatch; ++i) {
        const int r = (b + i) * 4 + rg;
        v[j][i] = r < valid[j] ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src[j] + (size_t)r * kHeadDim))
                               : u32x4_t{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
      for (int i = 0; i < S::kBatch; ++i) {
        if ((b + i) * 4 + rg < valid[j]) {
          const uint4 u = make_uint4(v[j][i].x, v[j][i].y, v[j][i].z, v[j][i].w);
#pragma unroll
          for (int e = 0; e < 8; ++e) {
            const float f = u4_elem<BF16>(u, e);
            mn[j][e] = fminf(mn[j][e], f);
            mx[j][e] = fmaxf(mx[j][e], f);
          }
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < S::kPages; ++j) {
    // rows 0 and 2 get the minima of two row groups, rows 1 and 3 the negated maxima; then the
    // lower half all of elements 0..3, the upper half of 4..7
    float z[8];
#pragma unroll
    for (int e = 0; e < 8; ++e) {
      float x = mn[j][e], y = -mx[j][e];
      swap_odd_rows(x, y);
      z[e] = fminf(x, y);
    }
    uint32_t b[4];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = z[e], y = z[e + 4];
      swap_halves(x, y);
      const float v = fminf(x, y);
      b[e] = f2h_exact<BF16>((rg & 1) ? -v : v);
    }
    if (ok[j]) {
      uint16_t* dst = meta + (((size_t)h * max_pages + first + j) * 2 + (rg & 1)) * kHeadDim + cg * 8 + (rg >> 1) * 4;
      __builtin_nontemporal_store((uint64_t)(b[0] | (b[1] << 16)) | ((uint64_t)(b[2] | (b[3] << 16)) << 32), reinterpret_cast<uint64_t*>(dst));
    }
  }
}

template <bool BF16, int PS>
__global__ __launch_bounds__(256) void meta_mean_kernel(const uint16_t* __restrict__ k, const int32_t* __restrict__ ptab,
                                                        int num_tokens, int page_begin, int page_end, int max_pages,
                                                        float* __restrict__ meta) {
  using S = MetaShape<PS>;
  const int h = blockIdx.y;
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const int first = page_begin + (blockIdx.x * 4 + w) * S::kPages;
  if (first >= page_end) return;
  const int cg = lane & 15, rg = lane >> 4;
  const uint16_t* src[S::kPages];
  int valid[S::kPages];
  bool ok[S::kPages];
  meta_pages<PS>(k, ptab, num_tokens, page_end, max_pages, h, first, cg, src, valid, ok);
  float sm[S::kPages][8];
#pragma unroll
  for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
    for (int e = 0; e < 8; ++e) sm[j][e] = 0.0f;
  }
#pragma unroll
  for (int b = 0; b < S::kRows; b += S::kBatch) {
    u32x4_t v[S::kPages][S::kBatch];
#pragma unroll
    for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
      for (int i = 0; i < S::kBatch; ++i) {
        const int r = (b + i) * 4 + rg;
        v[j][i] = r < valid[j] ? __builtin_nontemporal_load(reinterpret_cast<const u32x4_t*>(src[j] + (size_t)r * kHeadDim))
                               : u32x4_t{0, 0, 0, 0};
      }
    }
#pragma unroll
    for (int j = 0; j < S::kPages; ++j) {
#pragma unroll
      for (int i = 0; i < S::kBatch; ++i) {
        if ((b + i) * 4 + rg < valid[j]) {
          const uint4 u = make_uint4(v[j][i].x, v[j][i].y, v[j][i].z, v[j][i].w);
#pragma unroll
          for (int e = 0; e < 8; ++e) sm[j][e] += u4_elem<BF16>(u, e);
        }
      }
    }
  }
#pragma unroll
  for (int j = 0; j < S::kPages; ++j) {
    const float inv = 1.0f / (float)valid[j];
    // (s0 + s1) + (s2 + s3) of the four row groups: rows 0 and 2 get elements 0..3 of two of
    // them, rows 1 and 3 elements 4..7; then each half two of the four
    float z[4], o[2];
#pragma unroll
    for (int e = 0; e < 4; ++e) {
      float x = sm[j][e], y = sm[j][e + 4];
      swap_odd_rows(x, y);
      z[e] = x + y;
    }
#pragma unroll
    for (int e = 0; e < 2; ++e) {
      float x = z[e], y = z[e + 2];
      swap_halves(x, y);
      o[e] = (x + y) * inv;
    }
    if (ok[j]) {
      float* dst = meta + ((size_t)h * max_pages + first + j) * kHeadDim + cg * 8 + (rg & 1) * 4 + (rg >> 1) * 2;
      *reinterpret_cast<float2*>(dst) = make_float2(o[0], o[1]);
    }
  }
}

// The instance of a kernel template for a page size (16, 32, 64, 128 or 256 tokens), or
// NULL for another size (the C ABI admits only these).
template <typename K>
const void* by_page_size(int ps) {
  switch (ps) {
    case 16: return K::template get<16>();
    case 32: return K::template get<32>();
    case 64: return K::template get<64>();
    case 128: return K::template get<128>();
    case 256: return K::template get<256>();
    default: return nullptr;
  }
}

template <bool BF16>
struct MetaMeanK {
  template <int PS>
  static const void* get() { return (const void*)meta_mean_kernel<BF16, PS>; }
};
template <bool BF16>
struct MetaMinmaxK {
  template <int PS>
  static const void* get() { return (const void*)meta_minmax_kernel<BF16, PS>; }
};

hipError_t launch_meta(const MetaLaunch& a, hipStream_t stream) {
  const int np = a.page_end - a.page_begin;
  if (np <= 0) return hipSuccess;
  int ppb = 0;  // pages per workgroup
  switch (a.page_size) {
    case 16: ppb = meta_pages_per_block<16>(); break;
    case 32: ppb = meta_pages_per_block<32>(); break;
    case 64: ppb = meta_pages_per_block<64>(); break;
    case 128: ppb = meta_pages_per_block<128>(); break;
    case 256: ppb = meta_pages_per_block<256>(); break;
    default: return hipErrorInvalidValue;
  }
  dim3 grid((np + ppb - 1) / ppb, a.num_kv_heads);
  const uint16_t* k = static_cast<const uint16_t*>(a.k_cache);
  const int32_t* ptab = a.page_table;
  int nt = a.num_tokens, pb = a.page_begin, pe = a.page_end, mp = a.max_pages;
  void* meta = a.meta;
  void* args[] = {&k, &ptab, &nt, &pb, &pe, &mp, &meta};
  const void* f = a.meta_mean ? (a.bf16 ? by_page_size<MetaMeanK<true>>(a.page_size) : by_page_size<MetaMeanK<false>>(a.page_size))
                              : (a.bf16 ? by_page_size<MetaMinmaxK<true>>(a.page_size)
                                        : by_page_size<MetaMinmaxK<false>>(a.page_size));
  if (!f) return hipErrorInvalidValue;
  return hipLaunchKernel(f, grid, dim3(256), args, 0, stream);
}

// =====================================================================================
// block top-K select (score_topk_block, predict)
// =====================================================================================
// 1024 threads; thread (wave w, lane) owns pages w*J*64 + j*64 + lane, j < J, with their
// keys in registers, so that (w, j, lane) is ascending page order.  Candidates have their
// bit set in `cand`, pages in `force` are always selected.
//
// All pages of a KV head are candidates here, so their keys span the whole range of the
// scores (negative and positive), and radix bins over the key bits put most keys into a
// few bins, whose LDS atomics then serialise.  The first pass therefore bins the values
// linearly between the smallest and the largest candidate (a non-decreasing map, so a
// higher bin holds only larger values); the key-space radix select of prr_select.h then
// ranks the keys of the one bin that holds rank kextra.  Keys of NaN or infinite values
// fall back to the key-space select.  The selection is emitted in ascending page order
// by ballot compaction.

constexpr int kSelThreads = 1024;

struct __align__(16) SelectScratch {
  Sel2Lds sel;
  uint32_t forceb[PRR_MAX_PAGES_DEV / 32];
  int wcnt[kSelThreads / kWave];  // selected pages per wave
};

__host__ __device__ inline int select_j(int n) { return sel2_j(n, kSelThreads); }

// the float whose score_key is k
__device__ __forceinline__ float key_value(uint32_t k) {
  return __uint_as_float((k & 0x80000000u) ? (k & 0x7fffffffu) : ~k);
}

template <int J>
__device__ __forceinline__ void select_topk_regs(const uint32_t (&key)[J], uint64_t cand, uint64_t force, int kextra,
                                                 int32_t* __restrict__ out, int cap, int32_t* __restrict__ out_count,
                                                 SelectScratch& ss) {
  constexpr int NT = kSelThreads, NW = NT / kWave;
  Sel2Lds& S = ss.sel;
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  int page[J];
#pragma unroll
  for (int j = 0; j < J; ++j) page[j] = sel2_page<J>(j);

  int cnt = __popcll(cand);
  uint32_t lo = 0xffffffffu, hi = 0u;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    if ((cand >> j) & 1ull) {
      lo = min(lo, key[j]);
      hi = max(hi, key[j]);
    }
  }
  cnt = wave_isum(cnt);
  lo = wave_umin(lo);
  hi = wave_umax(hi);
  for (int b = t; b < kSel2Bins / 4; b += NT) reinterpret_cast<uint4*>(S.hist[0])[b] = make_uint4(0, 0, 0, 0);
  if (t == 0) S.nsmall = 0;
  if (lane == 0) {
    S.red[0][w] = cnt;
    S.red[1][w] = (int)lo;
    S.red[2][w] = (int)hi;
  }
  __syncthreads();
  cnt = 0;
  lo = 0xffffffffu;
  hi = 0u;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    cnt += S.red[0][i];
    lo = min(lo, (uint32_t)S.red[1][i]);
    hi = max(hi, (uint32_t)S.red[2][i]);
  }
  const float vlo = key_value(lo), span = key_value(hi) - vlo;
  const float scale = (float)kSel2Bins / span;

  // S.red is next written by the list compaction (after the barriers of the passes below)
  // or, on the key-space path, right at its start, hence the barrier there
  uint64_t in;
  int eq_cut = -1;
  if (kextra <= 0 || cnt == 0) {
    in = force;
  } else if (kextra >= cnt) {
    in = cand | force;
  } else if (!(span > 0.0f) || !__builtin_isfinite(span) || !__builtin_isfinite(scale)) {
    __syncthreads();
    const SelThreshold th = sel2_threshold<NT, J>(key, cand, kextra, S);
    in = sel2_membership<NT, J>(key, page, cand, force, th, &eq_cut, S);
  } else {
    int bin[J];
#pragma unroll
    for (int j = 0; j < J; ++j) {
      bin[j] = min(kSel2Bins - 1, (int)((key_value(key[j]) - vlo) * scale));
      if ((cand >> j) & 1ull) atomicAdd(&S.hist[0][bin[j]], 1u);
    }
    __syncthreads();
    if (w == 0) {
      // lane l owns bins [2048 - 32(l+1), 2048 - 32l); the lane holding rank kextra, then
      // its bin (the scan of prr_select.h's first pass)
      const int base = kSel2Bins - 32 * (lane + 1);
      const uint4* hb = reinterpret_cast<const uint4*>(S.hist[0] + base);
      int sum = 0;
#pragma unroll
      for (int v = 0; v < 8; ++v) {
        const uint4 x = hb[v];
        sum += (int)(x.x + x.y + x.z + x.w);
      }
      const int incl = wave_inclusive_scan(sum);
      const int excl = incl - sum;
      const uint64_t hit = __ballot(excl < kextra && kextra <= incl);
      const int ls = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
      const int ex = __builtin_amdgcn_readlane(excl, ls);
      const int lbase = kSel2Bins - 32 * (ls + 1);
      const int cj = lane < 32 ? (int)S.hist[0][lbase + 31 - lane] : 0;
      const int cinc = wave_inclusive_scan(cj);
      const uint64_t hit2 = __ballot(lane < 32 && ex + cinc >= kextra);
      const int js = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit2) - 1);
      if (lane == js) {
        S.res[0] = lbase + 31 - js;
        S.res[1] = ex + cinc - cj;
        S.res[2] = cj;
      }
    }
    __syncthreads();
    const int bstar = S.res[0], above = S.res[1], cbin = S.res[2];
    const int rank = kextra - above;  // of the threshold among the boundary bin's keys
    uint64_t inbin = 0, upper = 0;
#pragma unroll
    for (int j = 0; j < J; ++j) {
      if ((cand >> j) & 1ull) {
        if (bin[j] == bstar) inbin |= 1ull << j;
        if (bin[j] > bstar) upper |= 1ull << j;
      }
    }
    // every value in a higher bin is larger than every value of the boundary bin, and
    // keys equal to the threshold share its bin, so the tie cut is the boundary bin's
    SelThreshold th;
    if (cbin <= kSel2Small) {
      // the few keys of the boundary bin, ranked directly by one wave
      const int mine = __popcll(inbin);
      if (mine) {
        int slot = atomicAdd(&S.nsmall, mine);
#pragma unroll
        for (int j = 0; j < J; ++j)
          if ((inbin >> j) & 1ull) S.small[slot++] = key[j];
      }
      __syncthreads();
      if (w == 0) {
        const uint32_t kx = S.small[lane < cbin ? lane : 0];
        int gt = 0, ge = 0;
        for (int x = 0; x < cbin; ++x) {
          const uint32_t ky = (uint32_t)__builtin_amdgcn_readlane((int)kx, x);
          gt += ky > kx ? 1 : 0;
          ge += ky >= kx ? 1 : 0;
        }
        const uint64_t hit = __ballot(lane < cbin && gt < rank && rank <= ge);
        const int ls = __builtin_amdgcn_readfirstlane(__ffsll((long long)hit) - 1);
        if (lane == ls) {
          S.res[3] = (int)kx;
          S.res[4] = rank - gt;
          S.res[5] = ge - gt;
        }
      }
      __syncthreads();
      th.mode = 2;
      th.T = (uint32_t)S.res[3];
      th.need_eq = S.res[4];
      th.eq_total = S.res[5];
    } else {
      __syncthreads();  // S.res and the histogram are reused by the select of the boundary bin
      th = sel2_threshold<NT, J>(key, inbin, rank, S);
    }
    in = sel2_membership<NT, J>(key, page, inbin, force | upper, th, &eq_cut, S);
  }
  // ascending page order: the waves before this one, then ballot ranks within the wave
  // (ss.wcnt is not read before this point, so one barrier suffices)
  const int c = wave_isum(__popcll(in));
  if (lane == 0) ss.wcnt[w] = c;
  __syncthreads();
  int run = 0, total = 0;
#pragma unroll
  for (int i = 0; i < NW; ++i) {
    const int ci = ss.wcnt[i];
    run += i < w ? ci : 0;
    total += ci;
  }
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const bool sel = (in >> j) & 1ull;
    const uint64_t bm = __ballot(sel);
    if (sel) {
      const int pos = run + lanes_below(bm);
      if (pos < cap) out[pos] = page[j];
    }
    run += __popcll(bm);
  }
  if (t == 0) *out_count = min(total, cap);
}

// Forced pages as a bitmap in LDS; returns this thread's J-bit mask.
template <int J>
__device__ __forceinline__ uint64_t forced_mask(const int32_t* forced, int n_forced, int n, uint32_t* forceb) {
  if (n_forced == 0) return 0;
  const int nw = (n + 31) / 32;
  for (int i = threadIdx.x; i < nw; i += kSelThreads) forceb[i] = 0u;
  __syncthreads();
  if ((int)threadIdx.x < n_forced) {
    const int p = forced[threadIdx.x];
    atomicOr(&forceb[p >> 5], 1u << (p & 31));
  }
  __syncthreads();
  uint64_t m = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int pj = sel2_page<J>(j);
    const int p = min(pj, n - 1);
    if (pj < n && ((forceb[p >> 5] >> (p & 31)) & 1u)) m |= 1ull << j;
  }
  return m;
}

// =====================================================================================
// score + top-K, every key ranked by one block-wide select
// =====================================================================================
// For the sizes where ranking every key is the quicker select (the rule stands in prr_sep.h).
// grid (ceil(num_pages / 64), Hkv), 1024 threads.  Wave w of a workgroup scores pages
// base + w*4 + (lane/16); lane%16 covers channels 8*(lane%16)..+8.
constexpr int kScorePagesPerWg = 64;

// The selecting workgroup: this KV head's scores (published by every workgroup with
// device-coherent stores) into registers, then the block select.
template <int J>
__device__ __forceinline__ void select_scores(const float* scores, int n, const ScoreLaunch& a, int h,
                                              SelectScratch& ss) {
  uint32_t key[J];
  uint64_t cand = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int p = sel2_page<J>(j);
    key[j] = score_key(ld_dev(&scores[min(p, n - 1)]));
    if (p < n) cand |= 1ull << j;
  }
  const uint64_t force = forced_mask<J>(a.forced, a.n_forced, n, ss.forceb);
  cand &= ~force;
  select_topk_regs<J>(key, cand, force, a.kextra, a.selected + (size_t)h * a.cap, a.cap, a.selected_count + h, ss);
}

template <bool BF16, bool MEAN>
__global__ __launch_bounds__(1024) void score_topk_block_kernel(const ScoreLaunch a) {
  __shared__ SelectScratch ss;
  __shared__ float qbar[kHeadDim];
  __shared__ float qpart[16][kHeadDim];
  __shared__ int s_last;
  const int h = blockIdx.y;
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const int G = a.group;
  const uint16_t* q = static_cast<const uint16_t*>(a.q);

  {
    // thread t < 16G loads 8 channels of query head t/16 of this group (one 16-byte load);
    // the group mean is then summed in head order from LDS
    const int g = t >> 4, c8 = (t & 15) * 8;
    if (g < G) {
      const uint4 v = *reinterpret_cast<const uint4*>(q + (size_t)(h * G + g) * kHeadDim + c8);
#pragma unroll
      for (int e = 0; e < 8; ++e) qpart[g][c8 + e] = u4_elem<BF16>(v, e);
    }
    __syncthreads();
    if (t < kHeadDim) {
      float s = 0.0f;
      for (int gg = 0; gg < G; ++gg) s += qpart[gg][t];
      qbar[t] = s / (float)G;
    }
    __syncthreads();
  }

  const int cg = lane & 15, pi = lane >> 4;
  float qb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) qb[e] = qbar[cg * 8 + e];

  const int page = blockIdx.x * kScorePagesPerWg + w * 4 + pi;
  float* scores = a.scores + (size_t)h * a.max_pages;
  float s = 0.0f;
  if constexpr (!MEAN) {
    if (page < a.num_pages) {
      const uint16_t* row = static_cast<const uint16_t*>(a.meta) + ((size_t)h * a.max_pages + page) * 2 * kHeadDim + cg * 8;
      const uint4 mn = *reinterpret_cast<const uint4*>(row);
      const uint4 mx = *reinterpret_cast<const uint4*>(row + kHeadDim);
#pragma unroll
      for (int e = 0; e < 8; ++e) s += fmaxf(qb[e] * u4_elem<BF16>(mn, e), qb[e] * u4_elem<BF16>(mx, e));
    }
  } else {
    if (page < a.num_pages) {
      const float4* row = reinterpret_cast<const float4*>(static_cast<const float*>(a.meta) +
                                                          ((size_t)h * a.max_pages + page) * kHeadDim + cg * 8);
      const float4 m0 = row[0], m1 = row[1];
      s = qb[0] * m0.x;
      s += qb[1] * m0.y;
      s += qb[2] * m0.z;
      s += qb[3] * m0.w;
      s += qb[4] * m1.x;
      s += qb[5] * m1.y;
      s += qb[6] * m1.z;
      s += qb[7] * m1.w;
    }
  }
  s = sum16(s);
  if (cg == 0 && page < a.num_pages) st_dev(&scores[page], s);

  // the last workgroup of this KV head selects: scores are published with device-coherent
  // stores, completed before the counter is bumped, and read back the same way
  stores_complete();
  __syncthreads();
  if (t == 0) {
    const uint32_t old = counter_add(&a.counters[h * a.cnt_stride], 1u);
    s_last = (old == (uint32_t)(gridDim.x - 1));
  }
  __syncthreads();
  if (!s_last) return;

  const int n = a.num_pages;
  switch (select_j(n)) {
    case 1:  // (not launched for up to 512 pages; 513 to 1024 take a key per thread)
      select_scores<1>(scores, n, a, h, ss);
      break;
    case 2: select_scores<2>(scores, n, a, h, ss); break;
    case 4: select_scores<4>(scores, n, a, h, ss); break;
    case 8: select_scores<8>(scores, n, a, h, ss); break;
    default: select_scores<16>(scores, n, a, h, ss); break;
  }
  if (t == 0) atomicExch(&a.counters[h * a.cnt_stride], 0u);
}

// =====================================================================================
// EMA predictor
// =====================================================================================

template <int J>
__device__ __forceinline__ void predict_head(const PredictLaunch& a, int h, SelectScratch& ss) {
  const int lane = lane_id();
  const int n = a.num_pages;
  const int nwmax = (a.max_pages + 31) / 32;
  float* level = a.level + (size_t)h * a.max_pages;
  float* trend = a.trend + (size_t)h * a.max_pages;
  uint32_t* bits = a.init_bits + (size_t)h * nwmax;
  const float* scores = a.scores ? a.scores + (size_t)h * a.max_pages : nullptr;
  // all loads first (clamped addresses; a wave covers 64 consecutive pages = two bit words per j)
  float lv[J], tv[J], sc[J];
  uint32_t bw[J];
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int p = min(sel2_page<J>(j), n - 1);
    lv[j] = level[p];
    tv[j] = trend[p];
    sc[j] = scores ? scores[p] : 0.0f;
    bw[j] = bits[p >> 5];
  }
  uint32_t key[J];
  uint64_t cand = 0;
#pragma unroll
  for (int j = 0; j < J; ++j) {
    const int p = sel2_page<J>(j);
    const bool inr = p < n;
    bool has = inr && ((bw[j] >> (p & 31)) & 1u);
    float l = lv[j], v = tv[j];
    if (inr && scores) {
      const float s = sc[j];
      if (has) {
        v = a.beta * (s - l) + (1.0f - a.beta) * v;  // Eq. (3): the trend reads the previous level
        l = a.alpha * s + (1.0f - a.alpha) * l;
      } else {
        l = s;
        v = 0.0f;
        has = true;
      }
      level[p] = l;
      trend[p] = v;
    }
    key[j] = score_key(l + a.gamma * v);  // Eq. (2)
    if (has) cand |= 1ull << j;
    const uint64_t hm = __ballot(has);
    const uint64_t vm = __ballot(inr);
    if (scores && (lane == 0 || lane == 32)) {
      const uint32_t hbits = (uint32_t)(lane == 0 ? hm : (hm >> 32));
      const uint32_t vbits = (uint32_t)(lane == 0 ? vm : (vm >> 32));
      if (vbits) bits[p >> 5] = (bw[j] & ~vbits) | hbits;
    }
  }
  const uint64_t force = forced_mask<J>(a.forced, a.n_forced, n, ss.forceb);
  cand &= ~force;
  select_topk_regs<J>(key, cand, force, a.kextra, a.predicted + (size_t)h * a.cap, a.cap, a.predicted_count + h,
                      ss);
}

__global__ __launch_bounds__(1024) void predict_kernel(const PredictLaunch a) {
  __shared__ SelectScratch ss;
  const int h = blockIdx.x;
  switch (select_j(a.num_pages)) {
    case 1: predict_head<1>(a, h, ss); break;
    case 2: predict_head<2>(a, h, ss); break;
    case 4: predict_head<4>(a, h, ss); break;
    case 8: predict_head<8>(a, h, ss); break;
    default: predict_head<16>(a, h, ss); break;
  }
}

// =====================================================================================
// merge of arbitrary partial states
// =====================================================================================

// Latency-bound (64 states x 32 rows x 128 channels are 1 MB): a workgroup takes 64 channels
// of one row, so a small merge still spreads over rows x d / 64 compute units, and its eight
// waves take every eighth state.  A wave issues the output loads of up to 16 of its states
// before the weights are known, so (m, l) and the outputs cost one memory round trip
// together; the weights go through LDS and the eight partial sums are added at the end.
// Tiles of 128 states are folded online (running maximum).  64 states of 32 rows: 28.7 us a
// call with one workgroup per row that walked the states three times, 7.9 us now.
constexpr int kMergeThreads = 512;
constexpr int kMergeWaves = kMergeThreads / kWave;
constexpr int kMergeBatch = 16;                       // states of a wave per tile
constexpr int kMergeTile = kMergeWaves * kMergeBatch;  // states per tile

__global__ __launch_bounds__(kMergeThreads) void merge_states_kernel(int n_states, int rows, int d,
                                                                     const float* __restrict__ o,
                                                                     const float* __restrict__ m,
                                                                     const float* __restrict__ l,
                                                                     float* __restrict__ out_o, float* __restrict__ out_m,
                                                                     float* __restrict__ out_l) {
  static_assert(kMergeTile == 2 * kWave, "each wave reduces a tile's (m, l) with two states per lane");
  __shared__ float wt[kMergeTile];  // weight of each state of the tile; -1: an empty state
  __shared__ float part[kMergeWaves][kWave];
  const int row = blockIdx.x;
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const int c = blockIdx.y * kWave + lane;
  const float kNegInf = -__builtin_inff();
  float M = kNegInf, Lsum = 0.f, acc = 0.f;
  for (int s0 = 0; s0 < n_states; s0 += kMergeTile) {
    float ov[kMergeBatch];
#pragma unroll
    for (int k = 0; k < kMergeBatch; ++k) {
      const int s = s0 + w + kMergeWaves * k;
      ov[k] = s < n_states && c < d ? o[((size_t)s * rows + row) * d + c] : 0.f;
    }
    // every wave reduces the tile's (m, l) for itself: no barrier before the weights
    float mv[2], lv[2];
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      const int s = s0 + lane + kWave * k;
      mv[k] = s < n_states ? m[(size_t)s * rows + row] : kNegInf;
      lv[k] = s < n_states ? l[(size_t)s * rows + row] : 0.f;
    }
    float mx = M;
#pragma unroll
    for (int k = 0; k < 2; ++k)
      if (lv[k] > 0.f) mx = fmaxf(mx, mv[k]);
    mx = wave_max(mx);
    float wk[2], ls = 0.f;
#pragma unroll
    for (int k = 0; k < 2; ++k) {
      wk[k] = lv[k] > 0.f ? lv[k] * exp2f((mv[k] - mx) * kLog2e) : -1.f;
      ls += lv[k] > 0.f ? wk[k] : 0.f;
    }
    ls = wave_sum(ls);
    const float sc = Lsum != 0.f ? exp2f((M - mx) * kLog2e) : 0.f;
    Lsum = Lsum * sc + ls;
    acc *= sc;
    M = mx;
    __syncthreads();  // the weights of the previous tile have been read
    if (w == 0) {
      wt[lane] = wk[0];
      wt[kWave + lane] = wk[1];
    }
    __syncthreads();
#pragma unroll
    for (int k = 0; k < kMergeBatch; ++k) {
      const float x = wt[w + kMergeWaves * k];
      acc = x == -1.f ? acc : acc + x * ov[k];  // (an empty state's output may hold anything)
    }
  }
  part[w][lane] = acc;
  __syncthreads();
  if (w == 0 && c < d) {
    float sum = 0.f;
#pragma unroll
    for (int k = 0; k < kMergeWaves; ++k) sum += part[k][lane];
    out_o[(size_t)row * d + c] = Lsum > 0.f ? sum / Lsum : 0.f;
  }
  if (t == 0 && blockIdx.y == 0) {
    out_m[row] = Lsum > 0.f ? M : kNegInf;
    out_l[row] = Lsum;
  }
}

// A thread per V output channels of a row, the states one after another in batches of B whose
// loads are issued together: for few states, and for so many rows that they fill the chip
// whatever a row costs (a workgroup per row and 64 channels costs 3.8 ns however few its states
// are: 32768 rows x 128 channels of two states 254 us, 41 with a workgroup per row as before
// that, 12 here).
constexpr int kMergeRowThreads = 256;
constexpr uint64_t kMergeRowMaxBlocks = 1 << 22;

template <int V, int B>
__global__ __launch_bounds__(kMergeRowThreads) void merge_rows_kernel(int n_states, int rows, int d,
                                                                      const float* __restrict__ o,
                                                                      const float* __restrict__ m,
                                                                      const float* __restrict__ l,
                                                                      float* __restrict__ out_o, float* __restrict__ out_m,
                                                                      float* __restrict__ out_l) {
  struct __align__(4 * V) Vec {
    float x[V];
  };
  const uint32_t per = (uint32_t)d / V;  // elements of a row
  const uint64_t n = (uint64_t)rows * per;
  const float kNegInf = -__builtin_inff();
  for (uint64_t x = (uint64_t)blockIdx.x * kMergeRowThreads + threadIdx.x; x < n;
       x += (uint64_t)gridDim.x * kMergeRowThreads) {
    const uint32_t row = n <= 0xffffffffull ? (uint32_t)x / per : (uint32_t)(x / per);
    float M = kNegInf, Lsum = 0.f;
    Vec acc;
#pragma unroll
    for (int i = 0; i < V; ++i) acc.x[i] = 0.f;
    for (int s0 = 0; s0 < n_states; s0 += B) {
      Vec ov[B];
      float mv[B], lv[B];
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const size_t s = min(s0 + k, n_states - 1);
        ov[k] = reinterpret_cast<const Vec*>(o)[s * n + x];
        mv[k] = m[s * rows + row];
        lv[k] = s0 + k < n_states ? l[s * rows + row] : 0.f;
      }
      float mx = M;
#pragma unroll
      for (int k = 0; k < B; ++k)
        if (lv[k] > 0.f) mx = fmaxf(mx, mv[k]);
      const float sc = Lsum != 0.f ? exp2f((M - mx) * kLog2e) : 0.f;
      M = mx;
      // the batch is summed by halves: hundreds of states lose no more than its few additions
#pragma unroll
      for (int k = 0; k < B; ++k) {
        const bool some = lv[k] > 0.f;
        lv[k] = some ? lv[k] * exp2f((mv[k] - mx) * kLog2e) : 0.f;
#pragma unroll
        for (int i = 0; i < V; ++i) ov[k].x[i] = some ? lv[k] * ov[k].x[i] : 0.f;  // (it may hold anything)
      }
#pragma unroll
      for (int half = B / 2; half >= 1; half /= 2) {
#pragma unroll
        for (int k = 0; k < half; ++k) {
          lv[k] += lv[k + half];
#pragma unroll
          for (int i = 0; i < V; ++i) ov[k].x[i] += ov[k + half].x[i];
        }
      }
      Lsum = Lsum * sc + lv[0];
#pragma unroll
      for (int i = 0; i < V; ++i) acc.x[i] = acc.x[i] * sc + ov[0].x[i];
    }
#pragma unroll
    for (int i = 0; i < V; ++i) acc.x[i] = Lsum > 0.f ? acc.x[i] / Lsum : 0.f;
    reinterpret_cast<Vec*>(out_o)[x] = acc;
    if (x == (uint64_t)row * per) {
      out_m[row] = Lsum > 0.f ? M : kNegInf;
      out_l[row] = Lsum;
    }
  }
}

// =====================================================================================
// launchers
// =====================================================================================

hipError_t launch_score_topk_block(const ScoreLaunch& a, hipStream_t stream) {
  dim3 grid((a.num_pages + kScorePagesPerWg - 1) / kScorePagesPerWg, a.num_kv_heads);
  const void* f = a.bf16 ? (a.meta_mean ? (const void*)score_topk_block_kernel<true, true> : (const void*)score_topk_block_kernel<true, false>)
                         : (a.meta_mean ? (const void*)score_topk_block_kernel<false, true> : (const void*)score_topk_block_kernel<false, false>);
  void* args[] = {const_cast<ScoreLaunch*>(&a)};
  return hipLaunchKernel(f, grid, dim3(kSelThreads), args, 0, stream);
}

hipError_t launch_predict(const PredictLaunch& a, hipStream_t stream) {
  void* args[] = {const_cast<PredictLaunch*>(&a)};
  return hipLaunchKernel((const void*)predict_kernel, dim3(a.num_kv_heads), dim3(kSelThreads), args, 0, stream);
}

hipError_t launch_merge_states(int n_states, int rows, int d, const float* o, const float* m, const float* l,
                               float* out_o, float* out_m, float* out_l, hipStream_t stream) {
  void* args[] = {&n_states, &rows, &d, &o, &m, &l, &out_o, &out_m, &out_l};
  // The tiles where there are many states for few workgroups of them: 64 states of 32 rows x 128
  // channels 5.4 us against 9 (in batches of eight), of 4096 rows 42 against 27; 16 states of 32
  // rows take 5.5 either way.
  const int64_t tiles = (int64_t)rows * ((d + kWave - 1) / kWave);
  if (n_states > 16 && tiles <= std::min<int64_t>(1024, 16 * (int64_t)n_states))
    return hipLaunchKernel((const void*)merge_states_kernel, dim3(rows, (d + kWave - 1) / kWave), dim3(kMergeThreads),
                           args, 0, stream);
  const bool vec = d % 4 == 0 && ((reinterpret_cast<uintptr_t>(o) | reinterpret_cast<uintptr_t>(out_o)) & 15) == 0;
  const uint64_t n = (uint64_t)rows * (vec ? d / 4 : d), blocks = (n + kMergeRowThreads - 1) / kMergeRowThreads;
  const void* f = n_states <= 2   ? (vec ? (const void*)merge_rows_kernel<4, 2> : (const void*)merge_rows_kernel<1, 2>)
                  : n_states <= 8 ? (vec ? (const void*)merge_rows_kernel<4, 8> : (const void*)merge_rows_kernel<1, 8>)
                                  : (vec ? (const void*)merge_rows_kernel<4, 16> : (const void*)merge_rows_kernel<1, 16>);
  return hipLaunchKernel(f, dim3((uint32_t)std::min(blocks, kMergeRowMaxBlocks)), dim3(kMergeRowThreads), args, 0,
                         stream);
}

}  // namespace prr
