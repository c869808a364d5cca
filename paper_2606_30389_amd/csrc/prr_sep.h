// The separate kernels of the decode step: score + select, EMA + predict, speculate, repair.
// Each is written as a role of 256-thread workgroups, so that one launch can hold two roles
// that need nothing from each other: the two-stream step runs select beside speculate, then
// repair beside predict, as two launches per layer.
//
// Included by one translation unit per 16-bit type (they compile in parallel).
#pragma once

#include <stddef.h>

#include <type_traits>

#include "prr_device.h"
#include "prr_launch.h"
#include "prr_topk.h"

namespace prr {

namespace {

// =====================================================================================
// score + top-K
// =====================================================================================
// Wave w of a workgroup scores pages base + w*4*IT + 4*it + (lane/16), it < IT; lane%16 covers
// channels 8*(lane%16)..+8.  The metadata loads are issued before the mean query is formed.
// Wave 0 then publishes the workgroup's scores, 64 per store instruction (whole lines), with
// the largest key of each group of pages, and counts the workgroup in; the last one of a KV
// head selects (prr_topk.h).  IT = 8 (eight or sixteen 16-byte loads per lane in flight, 128
// pages per workgroup) once that gives two workgroups per CU; IT = 4 spreads a smaller cache
// over more of them (fewer pages yet would cost more in the arrival counter, about 12 ns a
// workgroup, than the shorter scan gains).  Whole call, every head (8 KV heads x 16384 pages,
// 256 selected): 40.9 us with 64 pages per 1024-thread workgroup and a select over all keys in
// registers, 21.1 now; 8 x 4096: 14.0 -> 10.8.
constexpr int kScorePagesPerIt = 4 * kTopkWaves;

template <int IT>
struct ScoreLds {
  union {
    struct {
      float qpart[16][kHeadDim];
      float qbar[kHeadDim];
      float sc[IT * kScorePagesPerIt];
    };
    TopkLds top;
  };
  int last;
};

// The largest key of each group of 1 << gshift pages (lanes of a row hold consecutive pages)
// to the group array, by the first lane of each group; key: 0 past the last page.
__device__ __forceinline__ void publish_groups(uint32_t key, int page, int n, int gshift, uint32_t* gmax) {
  const int lane = lane_id();
  uint32_t m = max(key, dpp_u32<kDppXor1>(key));
  m = max(m, dpp_u32<kDppXor2>(m));
  if (gshift == 3) m = max(m, dpp_u32<kDppHalfMirror>(m));
  if (page < n && (lane & ((1 << gshift) - 1)) == 0) st_dev(&gmax[page >> gshift], m);
}

template <bool BF16, int IT>
__device__ __forceinline__ void role_score_topk(const ScoreLaunch& a, int blk, int h, ScoreLds<IT>& S) {
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const int G = a.group, n = a.num_pages;
  const uint16_t* q = static_cast<const uint16_t*>(a.q);
  const int cg = lane & 15, pi = lane >> 4;
  const int base = blk * (IT * kScorePagesPerIt);
  const int page0 = base + w * 4 * IT + pi;

  // the query first (loads complete in issue order), then this thread's metadata
  // (addresses clamped to the last page)
  const int g16 = t >> 4, c8 = (t & 15) * 8;
  uint4 qv = make_uint4(0, 0, 0, 0);
  if (g16 < G) qv = *reinterpret_cast<const uint4*>(q + (size_t)(h * G + g16) * kHeadDim + c8);
  uint4 m0[IT], m1[IT];  // min and max row, or the two halves of the mean
  const int rowb = a.meta_mean ? 32 : 16, next = a.meta_mean ? 16 : 2 * kHeadDim;  // bytes
#pragma unroll
  for (int it = 0; it < IT; ++it) {
    const size_t row = (size_t)h * a.max_pages + min(page0 + 4 * it, n - 1);
    const char* src = static_cast<const char*>(a.meta) + row * (4 * kHeadDim) + cg * rowb;
    m0[it] = *reinterpret_cast<const uint4*>(src);
    m1[it] = *reinterpret_cast<const uint4*>(src + next);
  }
  // the group mean, summed in head order from LDS
  if (g16 < G) {
#pragma unroll
    for (int e = 0; e < 8; ++e) S.qpart[g16][c8 + e] = u4_elem<BF16>(qv, e);
  }
  __syncthreads();
  if (t < kHeadDim) {
    // (loads issued together; s is never -0, so adding 0 past the last head changes nothing)
    float x[16], s = 0.0f;
#pragma unroll
    for (int gg = 0; gg < 16; ++gg) x[gg] = S.qpart[gg][t];
#pragma unroll
    for (int gg = 0; gg < 16; ++gg) s += gg < G ? x[gg] : 0.0f;
    S.qbar[t] = s / (float)G;
  }
  __syncthreads();
  float qb[8];
#pragma unroll
  for (int e = 0; e < 8; ++e) qb[e] = S.qbar[cg * 8 + e];

#pragma unroll
  for (int it = 0; it < IT; ++it) {
    float s = 0.0f;
    if (!a.meta_mean) {
#pragma unroll
      for (int e = 0; e < 8; ++e) s += fmaxf(qb[e] * u4_elem<BF16>(m0[it], e), qb[e] * u4_elem<BF16>(m1[it], e));
    } else {
      s = qb[0] * __uint_as_float(m0[it].x);
      s += qb[1] * __uint_as_float(m0[it].y);
      s += qb[2] * __uint_as_float(m0[it].z);
      s += qb[3] * __uint_as_float(m0[it].w);
      s += qb[4] * __uint_as_float(m1[it].x);
      s += qb[5] * __uint_as_float(m1[it].y);
      s += qb[6] * __uint_as_float(m1[it].z);
      s += qb[7] * __uint_as_float(m1[it].w);
    }
    s = sum16(s);
    if (cg == 0) S.sc[w * 4 * IT + 4 * it + pi] = s;
  }
  __syncthreads();
  // scores and group keys are published with device-coherent stores, completed before the
  // counter is bumped, and read back the same way
  float* scores = a.scores + (size_t)h * a.max_pages;
  uint32_t* gmax = a.gmax + (size_t)h * a.gmax_stride;  // (used only with groups)
  if (w == 0) {
    constexpr int kPages = IT * kScorePagesPerIt;
#pragma unroll
    for (int r = 0; r < (kPages + kWave - 1) / kWave; ++r) {
      const int x = r * kWave + lane, p = base + x;
      const bool ok = x < kPages && p < n;
      const float s = S.sc[min(x, kPages - 1)];
      if (ok) st_dev(&scores[p], s);
      if (a.gshift) publish_groups(ok ? score_key(s) : 0u, ok ? p : n, n, a.gshift, gmax);
    }
    stores_complete();
    if (lane == 0) S.last = counter_add(&a.counters[h * a.cnt_stride], 1u) == (uint32_t)(a.nblk - 1);
  }
  __syncthreads();
  if (!S.last) return;

  const auto key_of = [&](int p) { return score_key(ld_dev(&scores[p])); };
  topk_select(n, a.gshift, a.kextra, a.forced, a.n_forced, [&](int g) { return ld_dev(&gmax[g]); }, key_of,
              a.selected + (size_t)h * a.cap, a.cap, a.selected_count + h, S.top);
  if (t == 0) atomicExch(&a.counters[h * a.cnt_stride], 0u);
}

template <bool BF16, int IT>
__global__ __launch_bounds__(kTopkThreads) void score_topk_kernel(const ScoreLaunch a) {
  __shared__ ScoreLds<IT> S;
  role_score_topk<BF16, IT>(a, blockIdx.x, blockIdx.y, S);
}

// =====================================================================================
// EMA + predict, with scores in hand and scratch for keys
// =====================================================================================
// One page per thread (the update of thousands of pages would hold a single workgroup for
// longer than the whole selection: 19 us for 16384 pages); the keys of Eq. (2) and their group
// maxima are published and the last workgroup of a KV head selects P.
struct EmaLds {
  TopkLds top;
  int last;
};

__device__ __forceinline__ void role_ema_topk(const PredictLaunch& a, int blk, int h, EmaLds& S) {
  const int t = threadIdx.x, lane = lane_id();
  const int n = a.num_pages, nwmax = (a.max_pages + 31) / 32;
  const int p0 = blk * kTopkThreads + t, p = min(p0, n - 1);
  const bool inr = p0 < n;
  float* level = a.level + (size_t)h * a.max_pages;
  float* trend = a.trend + (size_t)h * a.max_pages;
  uint32_t* bits = a.init_bits + (size_t)h * nwmax;
  uint32_t* keys = a.keys + (size_t)h * a.max_pages;
  uint32_t* gmax = a.gmax + (size_t)h * a.gmax_stride;
  float l = level[p], v = trend[p];
  const float s = a.scores[(size_t)h * a.max_pages + p];
  const uint32_t bw = bits[p >> 5];
  if ((bw >> (p & 31)) & 1u) {
    v = a.beta * (s - l) + (1.0f - a.beta) * v;  // Eq. (3): the trend reads the previous level
    l = a.alpha * s + (1.0f - a.alpha) * l;
  } else {
    l = s;
    v = 0.0f;
  }
  const uint32_t key = score_key(l + a.gamma * v);  // Eq. (2)
  if (inr) {
    level[p] = l;
    trend[p] = v;
    st_dev(&keys[p], key);
  }
  const uint64_t vm = __ballot(inr);
  if (lane == 0 || lane == 32) {
    const uint32_t vbits = (uint32_t)(lane == 0 ? vm : (vm >> 32));
    if (vbits) bits[p >> 5] = bw | vbits;
  }
  if (a.gshift) publish_groups(inr ? key : 0u, inr ? p : n, n, a.gshift, gmax);
  stores_complete();
  __syncthreads();
  if (t == 0) S.last = counter_add(&a.counters[h * a.cnt_stride], 1u) == (uint32_t)(a.nblk - 1);
  __syncthreads();
  if (!S.last) return;
  topk_select(n, a.gshift, a.kextra, a.forced, a.n_forced, [&](int g) { return ld_dev(&gmax[g]); },
              [&](int x) { return ld_dev(&keys[x]); }, a.predicted + (size_t)h * a.cap, a.cap, a.predicted_count + h,
              S.top);
  if (t == 0) atomicExch(&a.counters[h * a.cnt_stride], 0u);
}

// =====================================================================================
// attention over a short page list (one workgroup, four waves)
// =====================================================================================
// A list holds at most 16 tiles of 16 tokens (chunk_pages * page_size / 16 <= 16), four per
// wave.  Pages of 16 and 32 tokens are whole to one wave (wave w takes list entries w, w+4,
// ..); the tiles of a larger page go to the waves in turn, so that a chunk of one or two such
// pages keeps all four waves busy (one 128-token page: two tiles per wave, not four on two
// waves).  Each wave runs an online softmax over its tiles; the four wave states are merged
// in LDS.
//
// q.k^T per tile: S^T (16 tokens x 16 heads) = K (16 x 128) . Q^T (128 x 16) as four
// 16x16x32 MFMAs.  The contraction index is permuted so that each lane reads 64
// contiguous bytes of its key row: for k-step s, lane 16j+r supplies channels
// 32j+8s .. +8 of token r (A operand) and lane 16j+n channels 32j+8s .. +8 of query head n
// (B operand).  The result gives lane 16j+n the logits of tokens 4j..4j+3 for head n.
//
// p.V per tile, transposed: O^T (128 channels x 16 heads) += V^T . P^T by pv_tile
// (prr_device.h): lane 16j+m supplies channel 8m+cb of V rows 4j..4j+3 (from one 16-byte
// row load per row) and the weights of head m for tokens 4j..4j+3 (its own logit
// registers).  Accumulator cb, register i of lane 16j+n then holds O[head n][32j + 8i + cb]:
// each lane owns 32 contiguous channels of the same head whose logits it holds, so the
// online rescale is lane-local.

struct AttnCtx {
  const uint16_t* q;  // q + h*G*128
  const uint16_t* k;  // k_cache + h*max_pages*PS*128
  const uint16_t* v;
  const int32_t* ptab;
  int max_pages, num_pages, num_tokens, G;
};

template <class A>
__device__ __forceinline__ AttnCtx attn_ctx(const A& a, int h) {
  AttnCtx c;
  c.q = static_cast<const uint16_t*>(a.q) + (size_t)h * a.group * kHeadDim;
  c.k = static_cast<const uint16_t*>(a.k_cache) + (size_t)h * a.max_pages * a.page_size * kHeadDim;
  c.v = static_cast<const uint16_t*>(a.v_cache) + (size_t)h * a.max_pages * a.page_size * kHeadDim;
  c.ptab = a.page_table;
  c.max_pages = a.max_pages;
  c.num_pages = a.num_pages;
  c.num_tokens = a.num_tokens;
  c.G = a.group;
  return c;
}

constexpr int kOPad = kHeadDim + 4;  // LDS row stride of a head's partial output

struct __align__(16) UnitLds {  // (rows are read and written 16 bytes at a time)
  float wo[4][16][kOPad];
  float wm[4][16];
  float wl[4][16];
  float wpm[4][4][16];  // [page][wave] page maxima (pages whose tiles are spread over the waves)
};

template <bool BF16>
__device__ __forceinline__ f32x4_t mfma_qk(const u32x4_t& a, const u32x4_t& b, f32x4_t c) {
  if constexpr (BF16) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf16x8_t, a), __builtin_bit_cast(bf16x8_t, b), c,
                                                   0, 0, 0);
  } else {
    return __builtin_amdgcn_mfma_f32_16x16x32_f16(__builtin_bit_cast(f16x8_t, a), __builtin_bit_cast(f16x8_t, b), c, 0,
                                                  0, 0);
  }
}

// Result for thread t: head t/16, channels 8*(t%16)..+8: normalised o, m, l.
struct UnitResult {
  float o[8];
  float m, l;
};

template <bool BF16, int PS>
__device__ void attend_unit(const AttnCtx& c, const int32_t* pages, int cnt, float* page_m_out, UnitLds& sm,
                            uint32_t* flags, UnitResult& res) {
  static_assert(PS == 16 || PS == 32 || PS == 64 || PS == 128 || PS == 256, "page size");
  constexpr int TPP = PS / 16;
  constexpr int NTL = 16 / 4;                       // tiles per wave at most (16 tiles per unit)
  constexpr bool SHARED = TPP >= 4;                 // a page's tiles are spread over the four waves
  constexpr int NPW = SHARED ? 16 / TPP : NTL / TPP;  // list entries seen by a wave at most
  constexpr int TPW = SHARED ? TPP / 4 : TPP;       // tiles of one entry that a wave takes
  const float kNegInf = -__builtin_inff();
  const float scale = 0.08838834764831845f;  // 1/sqrt(128)
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const int j = lane >> 4, n = lane & 15;
  const int G = c.G;

  u32x4_t qf[4];
  if (n < G) {
    const u32x4_t* src = reinterpret_cast<const u32x4_t*>(c.q + (size_t)n * kHeadDim + 32 * j);
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = src[s];
  } else {
#pragma unroll
    for (int s = 0; s < 4; ++s) qf[s] = u32x4_t{0, 0, 0, 0};
  }

  // the wave's list entries: ids first, then page-table entries (wave-uniform values)
  const int wu = __builtin_amdgcn_readfirstlane(w);
  const auto entry = [&](int kk) { return SHARED ? kk : wu + 4 * kk; };
  const auto tile = [&](int x) { return SHARED ? 4 * x + wu : x; };  // tile of its page, x < TPW
  int pg[NPW], ph[NPW];
#pragma unroll
  for (int kk = 0; kk < NPW; ++kk) pg[kk] = entry(kk) < cnt ? pages[entry(kk)] : -1;
#pragma unroll
  for (int kk = 0; kk < NPW; ++kk) {
    pg[kk] = __builtin_amdgcn_readfirstlane(pg[kk]);
    const bool in_list = entry(kk) < cnt;
    const bool valid = pg[kk] >= 0 && pg[kk] < c.num_pages;
    if (in_list && !valid && flags && lane == 0) atomicOr(flags, kFlagBadListEntry);
    if (!valid) pg[kk] = -1;
  }
#pragma unroll
  for (int kk = 0; kk < NPW; ++kk) ph[kk] = (pg[kk] >= 0 && c.ptab) ? c.ptab[pg[kk]] : pg[kk];
  size_t off[NPW];
  int tok0[NPW];
  bool ok[NPW];
#pragma unroll
  for (int kk = 0; kk < NPW; ++kk) {
    const int phys = __builtin_amdgcn_readfirstlane(ph[kk]);
    ok[kk] = pg[kk] >= 0 && phys >= 0 && phys < c.max_pages;
    if (pg[kk] >= 0 && !ok[kk] && flags && lane == 0) atomicOr(flags, kFlagBadListEntry);
    off[kk] = ok[kk] ? (size_t)phys * PS * kHeadDim : 0;
    tok0[kk] = ok[kk] ? pg[kk] * PS : 0;
  }

  f32x4_t acc[8];
#pragma unroll
  for (int cb = 0; cb < 8; ++cb) acc[cb] = f32x4_t{0.f, 0.f, 0.f, 0.f};
  float m_run = kNegInf, l_run = 0.0f;

  // every tile of the wave is loaded up front (at most 4 tiles: 32 registers each)
  u32x4_t kf[NTL][4], vf[NTL][4];
#pragma unroll
  for (int f = 0; f < NTL; ++f) {
    const int kk = f / TPW, tt = tile(f % TPW);
    if (ok[kk]) {
      const uint16_t* kt = c.k + off[kk] + (size_t)tt * 16 * kHeadDim;
      const uint16_t* vt = c.v + off[kk] + (size_t)tt * 16 * kHeadDim;
      const u32x4_t* ks = reinterpret_cast<const u32x4_t*>(kt + (size_t)n * kHeadDim + 32 * j);
#pragma unroll
      for (int s = 0; s < 4; ++s) kf[f][s] = ks[s];
#pragma unroll
      for (int tg = 0; tg < 4; ++tg)
        vf[f][tg] = *reinterpret_cast<const u32x4_t*>(vt + (size_t)(4 * j + tg) * kHeadDim + 8 * n);
    }
  }

  float pm = kNegInf;  // max logit of the current page (this wave's tiles of it), head n
#pragma unroll
  for (int f = 0; f < NTL; ++f) {
    const int kk = f / TPW, tt = tile(f % TPW);
    if constexpr (SHARED) {
      if (f % TPW == 0 && j == 0) sm.wpm[kk][w][n] = kNegInf;
    }
    if (!ok[kk]) continue;
    if (f % TPW == 0) pm = kNegInf;
    f32x4_t st = f32x4_t{0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int s = 0; s < 4; ++s) st = mfma_qk<BF16>(kf[f][s], qf[s], st);
    float sv[4];
    float mx = kNegInf;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
      const int tok = tok0[kk] + tt * 16 + 4 * j + i;
      sv[i] = tok < c.num_tokens ? st[i] * scale : kNegInf;
      mx = fmaxf(mx, sv[i]);
    }
    mx = max_rows(mx);
    pm = fmaxf(pm, mx);
    const float mnew = fmaxf(m_run, mx);
    float alpha = 1.0f;
    float p[4] = {0.f, 0.f, 0.f, 0.f};
    if (mnew != kNegInf) {
      alpha = exp2f((m_run - mnew) * kLog2e);
#pragma unroll
      for (int i = 0; i < 4; ++i) p[i] = exp2f((sv[i] - mnew) * kLog2e);
    }
    const float ls = sum_rows((p[0] + p[1]) + (p[2] + p[3]));
    l_run = l_run * alpha + ls;
    m_run = mnew;
    if (tok0[kk] + PS > c.num_tokens) {
      // a partial last page: the values of tokens at or past num_tokens are zeroed, not
      // only weighted by 0 (0 x NaN or Inf from an unwritten cache tail would poison o)
#pragma unroll
      for (int tg = 0; tg < 4; ++tg)
        if (tok0[kk] + tt * 16 + 4 * j + tg >= c.num_tokens) vf[f][tg] = u32x4_t{0, 0, 0, 0};
    }
#pragma unroll
    for (int cb = 0; cb < 8; ++cb) {
#pragma unroll
      for (int i = 0; i < 4; ++i) acc[cb][i] *= alpha;
    }
    pv_tile<BF16>(acc, vf[f], p);
    if (f % TPW == TPW - 1 && j == 0) {
      if constexpr (SHARED) sm.wpm[kk][w][n] = pm;
      else if (page_m_out && n < G) page_m_out[(size_t)entry(kk) * G + n] = pm;
    }
  }

  // merge the four wave states: lane 16j+n holds channels 32j + 8i + cb of head n
  if (j == 0) {
    sm.wm[w][n] = m_run;
    sm.wl[w][n] = l_run;
  }
  float* row = &sm.wo[w][n][32 * j];
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    *reinterpret_cast<float4*>(row + 8 * i) = make_float4(acc[0][i], acc[1][i], acc[2][i], acc[3][i]);
    *reinterpret_cast<float4*>(row + 8 * i + 4) = make_float4(acc[4][i], acc[5][i], acc[6][i], acc[7][i]);
  }
  __syncthreads();
  if constexpr (SHARED) {
    // page e's maximum over the waves (thread e * 16 + head)
    const int e = t >> 4, hd = t & 15;
    if (page_m_out && e < NPW && e < cnt && hd < G) {
      float m = kNegInf;
#pragma unroll
      for (int x = 0; x < 4; ++x) m = fmaxf(m, sm.wpm[e][x][hd]);
      page_m_out[(size_t)e * G + hd] = m;
    }
  }
  const int hh = t >> 4, c0 = (t & 15) * 8;
  float mw[4], fw[4];
  float ms = kNegInf;
#pragma unroll
  for (int ww = 0; ww < 4; ++ww) {
    mw[ww] = sm.wm[ww][hh];
    if (sm.wl[ww][hh] > 0.0f) ms = fmaxf(ms, mw[ww]);
  }
  float L = 0.0f;
#pragma unroll
  for (int ww = 0; ww < 4; ++ww) {
    const float lw = sm.wl[ww][hh];
    fw[ww] = lw > 0.0f ? exp2f((mw[ww] - ms) * kLog2e) : 0.0f;
    L += lw * fw[ww];
  }
  const float inv = L > 0.0f ? 1.0f / L : 0.0f;
  float o[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
  for (int ww = 0; ww < 4; ++ww) {
    const float4 a = *reinterpret_cast<const float4*>(&sm.wo[ww][hh][c0]);
    const float4 b = *reinterpret_cast<const float4*>(&sm.wo[ww][hh][c0 + 4]);
    o[0] += a.x * fw[ww];
    o[1] += a.y * fw[ww];
    o[2] += a.z * fw[ww];
    o[3] += a.w * fw[ww];
    o[4] += b.x * fw[ww];
    o[5] += b.y * fw[ww];
    o[6] += b.z * fw[ww];
    o[7] += b.w * fw[ww];
  }
#pragma unroll
  for (int e = 0; e < 8; ++e) res.o[e] = o[e] * inv;
  res.m = L > 0.0f ? ms : kNegInf;
  res.l = L;
  __syncthreads();
}

template <bool BF16, int PS>
__device__ __forceinline__ void role_spec_attn(const SpecLaunch& a, int c, int h, UnitLds& sm, int32_t* ids) {
  const int start = c * a.chunk;
  // the chunk's page ids (at most 16) are loaded together with the count, clamped to the
  // capacity, so that the count costs no round trip of its own
  int id = -1;
  if ((int)threadIdx.x < a.chunk) id = a.pages[(size_t)h * a.cap + min(start + (int)threadIdx.x, a.cap - 1)];
  const int total = min(max(a.page_count[h], 0), a.cap);
  if (start >= total) return;
  const int cnt = min(a.chunk, total - start);
  if ((int)threadIdx.x < a.chunk) ids[threadIdx.x] = id;
  __syncthreads();
  const int G = a.group;
  UnitResult r;
  float* pmo = a.page_m ? a.page_m + ((size_t)h * a.cap + start) * G : nullptr;
  attend_unit<BF16, PS>(attn_ctx(a, h), ids, cnt, pmo, sm, nullptr, r);
  const int t = threadIdx.x, hh = t >> 4, c0 = (t & 15) * 8;
  if (hh < G) {
    const size_t row = ((size_t)h * a.nchunks + c) * G + hh;
    float4* dst = reinterpret_cast<float4*>(a.part_o + row * kHeadDim + c0);
    dst[0] = make_float4(r.o[0], r.o[1], r.o[2], r.o[3]);
    dst[1] = make_float4(r.o[4], r.o[5], r.o[6], r.o[7]);
    if ((t & 15) == 0) {
      a.part_m[row] = r.m;
      a.part_l[row] = r.l;
    }
  }
}

struct SpecLds {
  UnitLds unit;
  int32_t ids[16];
};
static_assert(offsetof(SpecLds, unit) % 16 == 0, "16-byte rows in LDS");

template <bool BF16, int PS>
__global__ __launch_bounds__(256) void spec_attn_kernel(const SpecLaunch a) {
  __shared__ SpecLds S;
  role_spec_attn<BF16, PS>(a, blockIdx.x, blockIdx.y, S.unit, S.ids);
}

// Select beside speculate: the scoring workgroups first (the longer chain).  8 KV heads x 1024
// pages of 128 tokens, 32 of them attended: 10.3 us, against 8.5 and 8.8 us one after the other.
template <bool BF16, int PS, int IT>
__global__ __launch_bounds__(256) void select_spec_kernel(const ScoreLaunch a, const SpecLaunch b) {
  __shared__ union {
    ScoreLds<IT> score;
    SpecLds spec;
  } S;
  const int ns = a.num_kv_heads * a.nblk, x = blockIdx.x;
  if (x < ns) role_score_topk<BF16, IT>(a, x % a.nblk, x / a.nblk, S.score);
  else role_spec_attn<BF16, PS>(b, (x - ns) % b.nchunks, (x - ns) / b.nchunks, S.spec.unit, S.spec.ids);
}

// =====================================================================================
// repair
// =====================================================================================
// Grid: Hkv * nwork work workgroups, then Hkv * G merge workgroups (one query head each).
// Without a prediction (the serial path) work unit u attends list entries [uC, uC+C) of A.
// With one, every workgroup first builds the plan of its KV head in LDS (bitmaps of A and P,
// the missed list in A's order, the chunks of P that hold a wasted page).
// Work unit u < ceil(|M|/C): attend missed pages [uC, uC+C).
// Work unit u >= that (exact mode): one contaminated chunk c of P: attend its wasted
//   pages W; if they carry at most kMaxWastedShare of the chunk's softmax mass for every
//   head, subtract them from the chunk's speculative state (the clean part's maximum
//   comes from the per-page maxima of the speculation); otherwise attend the chunk's
//   pages of A afresh.  Either way the unit's state replaces chunk c.
// A unit's outputs are published with device-coherent stores and, once those have completed,
// two words per query head: m and l, each below the call's tag.  A merge workgroup waits
// (bounded spin) for the tag on the words of its head, reads the outputs, and clears the words:
// no counter between the last state and the merge.  Nothing else kept in a workspace looks like
// a tag (see RepairLaunch), so the words need not hold anything in particular before a call and
// may lie where calls of other shapes keep other data, and a state that a merge gave up waiting
// for does not pass for one of a later call.  Serial call, 128 of the 32-token pages of 8 KV
// heads: 17.7 -> 10.7 us (without the plan, the unit counter and a merge of two heads per
// workgroup).

constexpr float kMaxWastedShare = 0.875f;
constexpr int kSpinLimit = 1 << 24;

struct __align__(16) MergeLds {  // each wave's running state
  float acc[4][kHeadDim];
  float ml[4][2];
};

struct RepairLds {
  uint32_t bitA[PRR_MAX_PAGES_DEV / 32];
  uint32_t bitP[PRR_MAX_PAGES_DEV / 32];
  int32_t listP[PRR_MAX_CAP_DEV];
  int32_t missed[PRR_MAX_CAP_DEV];
  int32_t contam[PRR_MAX_CAP_DEV];
  uint32_t contam_bits[PRR_MAX_CAP_DEV / 32];
  uint8_t wflag[PRR_MAX_CAP_DEV];
  int cnt_m[4][4], cnt_w[4][4], cnt_c[4][4];
  int32_t wpages[16];
  int32_t xpages[16];
  int32_t xslots[16];
  int nWp, nXp;
  union {
    UnitLds unit;    // work workgroups
    MergeLds merge;  // merge workgroups
  };
};
static_assert(offsetof(RepairLds, unit) % 16 == 0 && offsetof(RepairLds, merge) % 16 == 0 && kOPad % 4 == 0,
              "16-byte rows in LDS");

// Folds of a merge wave: the states i = w, w + 4, .. < n of one query head into the running
// (M, L, ax, ay), where ml(i, m, l) gives state i's (m, l) and out(i) its outputs at columns
// 2 lane and 2 lane + 1.  A batch issues the loads of up to 16 states before using any of them.
template <class ML, class OUT>
__device__ __forceinline__ void fold_states(int n, int w, const ML& ml, const OUT& out, float& M, float& L, float& ax,
                                            float& ay) {
  constexpr int kB = 16;
  const float kNegInf = -__builtin_inff();
  const int lane = lane_id();
  const int nk = n > w ? (n - w + 3) / 4 : 0;
  for (int k0 = 0; k0 < nk; k0 += kB) {
    const int nb = min(kB, nk - k0);
    float mi = kNegInf, li = 0.0f;
    ml(w + 4 * (k0 + min(lane, nb - 1)), lane < nb, mi, li);
    float2 ov[kB];
#pragma unroll
    for (int r = 0; r < kB; ++r) ov[r] = out(w + 4 * (k0 + min(r, nb - 1)));
    li = lane < nb ? li : 0.0f;
    mi = li > 0.0f ? mi : kNegInf;
    const float Mn = fmaxf(M, wave_max(mi));
    if (Mn == kNegInf) continue;  // no state of this batch holds anything
    const float sc = L > 0.0f ? exp2f((M - Mn) * kLog2e) : 0.0f;
    const float wi = li > 0.0f ? li * exp2f((mi - Mn) * kLog2e) : 0.0f;
    ax *= sc;
    ay *= sc;
    L = L * sc + wave_sum(wi);
    M = Mn;
#pragma unroll
    for (int r = 0; r < kB; ++r) {
      const float wr = __int_as_float(__builtin_amdgcn_readlane(__float_as_int(wi), r));
      ax += wr * ov[r].x;
      ay += wr * ov[r].y;
    }
  }
}

// A unit's state (thread t holds head t / 16, channels 8 (t % 16) .. + 8) to the merge
// workgroups: staged through LDS so that each store instruction writes 256 contiguous bytes.
__device__ __forceinline__ void publish_unit(const RepairLaunch& a, int h, int u, const UnitResult& r, UnitLds& L) {
  const int t = threadIdx.x, hh = t >> 4, c0 = (t & 15) * 8, G = a.group;
  float* tile = &L.wo[0][0][0];  // [16][128], free after the unit's last barrier
  if (hh < G) {
#pragma unroll
    for (int e = 0; e < 8; ++e) tile[hh * kHeadDim + c0 + e] = r.o[e];
    if ((t & 15) == 0) {
      L.wm[0][hh] = r.m;
      L.wl[0][hh] = r.l;
    }
  }
  __syncthreads();
  const size_t row0 = ((size_t)h * a.nwork + u) * G;
  uint64_t* dst = reinterpret_cast<uint64_t*>(a.ws_o + row0 * kHeadDim);
  for (int i = t; i < G * kHeadDim / 2; i += 256)
    __hip_atomic_store(dst + i, reinterpret_cast<const uint64_t*>(tile)[i], __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
  stores_complete();
  __syncthreads();
  if (t < 2 * G) {
    const float x = (t & 1) ? L.wl[0][t >> 1] : L.wm[0][t >> 1];
    __hip_atomic_store(a.ws_ml + row0 * 2 + t, ((uint64_t)a.tag << 32) | __float_as_uint(x), __ATOMIC_RELAXED,
                       __HIP_MEMORY_SCOPE_AGENT);
  }
}

// The unit states of query head g of KV head h into a merge wave's running state: waits for
// the words with this call's tag, then reads the outputs and clears the words.
__device__ __forceinline__ void fold_units(const RepairLaunch& a, int h, int g, int n, int w, float& M, float& L,
                                           float& ax, float& ay) {
  const int lane = lane_id();
  const size_t row0 = (size_t)h * a.nwork * a.group + g;
  fold_states(
      n, w,
      [&](int u, bool mine, float& m, float& l) {
        uint64_t* p = a.ws_ml + (row0 + (size_t)u * a.group) * 2;
        uint64_t vm = 0, vl = 0;
        bool ready = false;
        int it = 0;
        for (;;) {
          vm = __hip_atomic_load(p, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          vl = __hip_atomic_load(p + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          ready = (uint32_t)(vm >> 32) == a.tag && (uint32_t)(vl >> 32) == a.tag;
          if (__ballot(!ready) == 0ull) break;
          __builtin_amdgcn_s_sleep(1);
          if (++it > kSpinLimit) {
            if (lane == 0) atomicOr(a.flags, kFlagSpinTimeout);
            break;
          }
        }
        if (mine) {
          __hip_atomic_store(p, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
          __hip_atomic_store(p + 1, (uint64_t)0, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        m = __uint_as_float((uint32_t)vm);
        l = ready ? __uint_as_float((uint32_t)vl) : 0.0f;
        // the outputs are loaded only now that their state is complete
        asm volatile("" ::: "memory");
      },
      [&](int u) {
        const uint64_t v = __hip_atomic_load(
            reinterpret_cast<uint64_t*>(a.ws_o + (row0 + (size_t)u * a.group) * kHeadDim) + lane, __ATOMIC_RELAXED,
            __HIP_MEMORY_SCOPE_AGENT);
        return make_float2(__uint_as_float((uint32_t)v), __uint_as_float((uint32_t)(v >> 32)));
      },
      M, L, ax, ay);
}

// The four waves' running states combined into the output row of query head g.
template <bool BF16>
__device__ __forceinline__ void merge_write(const RepairLaunch& a, int h, int g, float M, float L, float ax, float ay,
                                            MergeLds& S) {
  const int lane = lane_id(), w = threadIdx.x / kWave;
  const float kNegInf = -__builtin_inff();
  *reinterpret_cast<float2*>(&S.acc[w][2 * lane]) = make_float2(ax, ay);
  if (lane == 0) {
    S.ml[w][0] = M;
    S.ml[w][1] = L;
  }
  __syncthreads();
  if (w != 0) return;
  float ms = kNegInf;
#pragma unroll
  for (int i = 0; i < 4; ++i)
    if (S.ml[i][1] > 0.f) ms = fmaxf(ms, S.ml[i][0]);
  float Ls = 0.f, ox = 0.f, oy = 0.f;
#pragma unroll
  for (int i = 0; i < 4; ++i) {
    const float li = S.ml[i][1];
    const float f = li > 0.f ? exp2f((S.ml[i][0] - ms) * kLog2e) : 0.f;
    const float2 o = *reinterpret_cast<const float2*>(&S.acc[i][2 * lane]);
    Ls += li * f;
    ox += o.x * f;
    oy += o.y * f;
  }
  const float inv = Ls > 0.f ? 1.0f / Ls : 0.f;
  ox *= inv;
  oy *= inv;
  const size_t orow = (size_t)h * a.group + g;
  *reinterpret_cast<float2*>(a.out_o32 + orow * kHeadDim + 2 * lane) = make_float2(ox, oy);
  if (a.out_o)
    reinterpret_cast<uint32_t*>(a.out_o)[(orow * kHeadDim) / 2 + lane] = f2h_rne<BF16>(ox) | (f2h_rne<BF16>(oy) << 16);
  if (lane == 0) {
    a.out_m[orow] = Ls > 0.f ? ms : kNegInf;
    a.out_l[orow] = Ls;
  }
}

// Repair without a prediction: attend every page of A.
template <bool BF16, int PS>
__device__ __forceinline__ void repair_serial(const RepairLaunch& a, bool is_merge, int h, int u, RepairLds& S) {
  const int t = threadIdx.x, C = a.chunk;
  if (!is_merge) {
    const int start = u * C;
    int id = -1;
    if (t < C) id = a.selected[(size_t)h * a.cap + min(start + t, a.cap - 1)];
    const int nA = min(max(a.selected_count[h], 0), a.cap);
    if (start >= nA) return;
    if (t < C) S.xpages[t] = id;
    __syncthreads();
    UnitResult r;
    attend_unit<BF16, PS>(attn_ctx(a, h), S.xpages, min(C, nA - start), nullptr, S.unit, a.flags, r);
    publish_unit(a, h, u, r, S.unit);
    return;
  }
  const int nA = min(max(a.selected_count[h], 0), a.cap);
  const int g = u;
  if (g == 0) {
    // the missed count: the valid entries of A
    int c = 0;
    for (int i = t; i < nA; i += 256) {
      const int p = a.selected[(size_t)h * a.cap + i];
      c += p >= 0 && p < a.num_pages ? 1 : 0;
    }
    c = wave_isum(c);
    if (lane_id() == 0) S.cnt_m[0][t / kWave] = c;
    __syncthreads();
    if (t == 0) {
      if (a.missed_count) a.missed_count[h] = S.cnt_m[0][0] + S.cnt_m[0][1] + S.cnt_m[0][2] + S.cnt_m[0][3];
      if (a.wasted_count) a.wasted_count[h] = 0;
    }
  }
  float M = -__builtin_inff(), L = 0.f, ax = 0.f, ay = 0.f;
  fold_units(a, h, g, (nA + C - 1) / C, t / kWave, M, L, ax, ay);
  merge_write<BF16>(a, h, g, M, L, ax, ay, S.merge);
}

template <bool BF16, int PS>
__device__ __forceinline__ void role_repair(const RepairLaunch& a, int bid, RepairLds& S) {
  const int t = threadIdx.x, lane = lane_id(), w = t / kWave;
  const int G = a.group, C = a.chunk;
  const int work_wgs = a.num_kv_heads * a.nwork;
  const bool is_merge = bid >= work_wgs;
  const int per = is_merge ? G : a.nwork, x = is_merge ? bid - work_wgs : bid;
  const int h = x / per, u = x % per;  // work unit, or query head of a merge
  if (!a.predicted) {
    repair_serial<BF16, PS>(a, is_merge, h, u, S);
    return;
  }
  const bool exact = a.mode == PRR_EXACT_SELECTED;
  const int n = a.num_pages;
  const int nwords = (n + 31) / 32;
  const int nA = min(max(a.selected_count[h], 0), a.cap);
  const int nP = min(max(a.predicted_count[h], 0), a.cap);
  const int rounds = (a.cap + 255) / 256;  // of 256 list entries
  const float kNegInf = -__builtin_inff();

  // ---- plan.  List entry i is handled by thread i % 256 in round i / 256, so a wave
  // covers 64 consecutive entries and every compaction is a ballot.
  for (int i = t; i < nwords; i += 256) {
    S.bitA[i] = 0u;
    S.bitP[i] = 0u;
  }
  // the list entries are loaded together with the counts (clamped to the capacity) and
  // masked afterwards, so the plan costs one memory round trip
  int ea[4], ep[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const size_t ic = (size_t)h * a.cap + min(r * 256 + t, a.cap - 1);
    ea[r] = r < rounds ? a.selected[ic] : -1;
    ep[r] = r < rounds ? a.predicted[ic] : -1;
  }
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = r * 256 + t;
    ea[r] = i < nA ? ea[r] : -1;
    ep[r] = i < nP ? ep[r] : -1;
  }
  __syncthreads();
  bool bad_entry = false;
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = r * 256 + t;
    if (i < nA) {
      if (ea[r] >= 0 && ea[r] < n) atomicOr(&S.bitA[ea[r] >> 5], 1u << (ea[r] & 31));
      else bad_entry = true;
    }
    if (i < nP) {
      S.listP[i] = ep[r];
      if (ep[r] >= 0 && ep[r] < n) atomicOr(&S.bitP[ep[r] >> 5], 1u << (ep[r] & 31));
      else bad_entry = true;
    }
  }
  if (bad_entry && bid == 0) atomicOr(a.flags, kFlagBadListEntry);
  __syncthreads();
  uint64_t bm[4], bw[4];
#pragma unroll
  for (int r = 0; r < 4; ++r) {
    const int i = r * 256 + t;
    const int pa = ea[r], pp = ep[r];
    const bool missed = i < nA && pa >= 0 && pa < n && !((S.bitP[pa >> 5] >> (pa & 31)) & 1u);
    const bool wasted = i < nP && pp >= 0 && pp < n && !((S.bitA[pp >> 5] >> (pp & 31)) & 1u);
    if (i < nP) S.wflag[i] = wasted ? 1 : 0;
    bm[r] = __ballot(missed);
    bw[r] = __ballot(wasted);
    if (lane == 0) {
      S.cnt_m[r][w] = __popcll(bm[r]);
      S.cnt_w[r][w] = __popcll(bw[r]);
    }
  }
  __syncthreads();
  int nM = 0, nW = 0;
  {
    int base[4] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const int c = S.cnt_m[r][ww];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
          if (r < rr || (r == rr && ww < w)) base[rr] += c;
        nM += c;
        nW += S.cnt_w[r][ww];
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r)
      if ((bm[r] >> lane) & 1ull) S.missed[base[r] + lanes_below(bm[r])] = ea[r];
  }
  const int nch = (nP + C - 1) / C;
  int nCont = 0;
  if (exact) {
    // chunk c (of C consecutive entries of P) holds a wasted page: thread c % 256, round c / 256
    uint64_t bc[4];
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      const int c = r * 256 + t;
      bool dirty = false;
      if (c < nch) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
          const int i = c * C + e;
          if (e < C && i < nP) dirty |= S.wflag[i] != 0;
        }
      }
      bc[r] = __ballot(dirty);
      if (lane == 0) S.cnt_c[r][w] = __popcll(bc[r]);
    }
    for (int i = t; i < PRR_MAX_CAP_DEV / 32; i += 256) S.contam_bits[i] = 0u;
    __syncthreads();
    int base[4] = {0, 0, 0, 0};
#pragma unroll
    for (int r = 0; r < 4; ++r) {
#pragma unroll
      for (int ww = 0; ww < 4; ++ww) {
        const int c = S.cnt_c[r][ww];
#pragma unroll
        for (int rr = 0; rr < 4; ++rr)
          if (r < rr || (r == rr && ww < w)) base[rr] += c;
        nCont += c;
      }
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
      if ((bc[r] >> lane) & 1ull) {
        const int c = r * 256 + t;
        S.contam[base[r] + lanes_below(bc[r])] = c;
        atomicOr(&S.contam_bits[c >> 5], 1u << (c & 31));
      }
    }
  }
  __syncthreads();
  const int nMU = (nM + C - 1) / C;

  const AttnCtx ctx = attn_ctx(a, h);
  const int hh = t >> 4, c0 = (t & 15) * 8;

  if (!is_merge) {
    // ---- work
    UnitResult r;
    bool have = false;
    if (u < nMU) {
      const int start = u * C;
      attend_unit<BF16, PS>(ctx, S.missed + start, min(C, nM - start), nullptr, S.unit, a.flags, r);
      have = true;
    } else if (exact && u - nMU < nCont) {
      const int ch = S.contam[u - nMU];
      if (t == 0) {
        int nw = 0, nx = 0;
        for (int i = ch * C; i < min(nP, ch * C + C); ++i) {
          const int p = S.listP[i];
          if (p < 0 || p >= n) continue;
          if ((S.bitA[p >> 5] >> (p & 31)) & 1u) {
            S.xpages[nx] = p;
            S.xslots[nx] = i;
            ++nx;
          } else {
            S.wpages[nw++] = p;
          }
        }
        S.nWp = nw;
        S.nXp = nx;
      }
      __syncthreads();
      const int nwp = S.nWp, nxp = S.nXp;
      bool recompute = true;
      if (a.page_m && nxp > 0 && nwp > 0) {
        // the chunk's speculative state and its kept pages' maxima are loaded before the
        // wasted pages are attended, so that their round trip overlaps the attention's
        const size_t crow = ((size_t)h * a.nchunks + ch) * G;
        float mx = kNegInf, mc = 0.f, lc = 0.f;
        float4 o0 = make_float4(0.f, 0.f, 0.f, 0.f), o1 = o0;
        if (hh < G) {
          mc = a.part_m[crow + hh];
          lc = a.part_l[crow + hh];
          const float4* oc = reinterpret_cast<const float4*>(a.part_o + (crow + hh) * kHeadDim + c0);
          o0 = oc[0];
          o1 = oc[1];
          for (int x = 0; x < nxp; ++x) mx = fmaxf(mx, a.page_m[((size_t)h * a.cap + S.xslots[x]) * G + hh]);
        }
        attend_unit<BF16, PS>(ctx, S.wpages, nwp, nullptr, S.unit, a.flags, r);
        bool bad = false;
        if (hh < G) {
          const float share = (lc > 0.f && r.l > 0.f) ? r.l * exp2f((r.m - mc) * kLog2e) / lc : (r.l > 0.f ? 2.f : 0.f);
          bad = !(share <= kMaxWastedShare);
        }
        bad = __syncthreads_or(bad);
        if (!bad) {
          recompute = false;
          if (hh < G) {
            const float ec = lc * exp2f((mc - mx) * kLog2e);
            const float ew = r.l > 0.f ? r.l * exp2f((r.m - mx) * kLog2e) : 0.f;
            const float lx = ec - ew;
            const float inv = 1.0f / lx;
            const float ocv[8] = {o0.x, o0.y, o0.z, o0.w, o1.x, o1.y, o1.z, o1.w};
#pragma unroll
            for (int e = 0; e < 8; ++e) r.o[e] = (ec * ocv[e] - ew * r.o[e]) * inv;
            r.m = mx;
            r.l = lx;
          }
        }
      }
      if (recompute) attend_unit<BF16, PS>(ctx, S.xpages, nxp, nullptr, S.unit, a.flags, r);
      have = true;
    }
    if (have) publish_unit(a, h, u, r, S.unit);
    return;
  }

  // ---- merge of query head u: wave w folds every fourth of the clean speculative chunks,
  // which are ready at launch (while the work workgroups run), then of the unit states
  const int nUnits = nMU + (exact ? nCont : 0);
  const int g = u;
  const size_t crow0 = ((size_t)h * a.nchunks) * G + g;
  float Mw = kNegInf, Lw = 0.f, ax = 0.f, ay = 0.f;
  fold_states(
      nch, w,
      [&](int c, bool, float& m, float& l) {
        const size_t row = crow0 + (size_t)c * G;
        const bool clean = !(exact && ((S.contam_bits[c >> 5] >> (c & 31)) & 1u));
        m = a.part_m[row];
        l = clean ? a.part_l[row] : 0.0f;
      },
      [&](int c) {
        return *reinterpret_cast<const float2*>(a.part_o + (crow0 + (size_t)c * G) * kHeadDim + 2 * lane);
      },
      Mw, Lw, ax, ay);
  fold_units(a, h, g, nUnits, w, Mw, Lw, ax, ay);
  merge_write<BF16>(a, h, g, Mw, Lw, ax, ay, S.merge);
  if (g == 0 && t == 0) {
    if (a.missed_count) a.missed_count[h] = nM;
    if (a.wasted_count) a.wasted_count[h] = nW;
  }
}

__global__ __launch_bounds__(kTopkThreads) void ema_topk_kernel(const PredictLaunch a) {
  __shared__ EmaLds S;
  role_ema_topk(a, blockIdx.x, blockIdx.y, S);
}

template <bool BF16, int PS>
__global__ __launch_bounds__(256) void repair_kernel(const RepairLaunch a) {
  __shared__ RepairLds S;
  role_repair<BF16, PS>(a, blockIdx.x, S);
}

// Repair beside predict (its workgroups last: the repair is the longer chain).  The same
// shape: 14.3 us, against 19.6 and 6.7 us as separate kernels before.
template <bool BF16, int PS>
__global__ __launch_bounds__(256) void repair_predict_kernel(const RepairLaunch a, const PredictLaunch b) {
  __shared__ union {
    RepairLds repair;
    EmaLds ema;
  } S;
  const int nr = a.num_kv_heads * (a.nwork + a.group), x = blockIdx.x;
  if (x < nr) role_repair<BF16, PS>(a, x, S.repair);
  else role_ema_topk(b, (x - nr) % b.nblk, (x - nr) / b.nblk, S.ema);
}

// =====================================================================================
// launches
// =====================================================================================

template <typename... A>
hipError_t launch(const void* f, dim3 grid, hipStream_t stream, const A&... arg) {
  void* args[] = {const_cast<A*>(&arg)...};
  return hipLaunchKernel(f, grid, dim3(kTopkThreads), args, 0, stream);
}

// f<PS> for a page size (the C ABI admits only these)
template <class F>
hipError_t by_page_size(int ps, const F& f) {
  switch (ps) {
    case 16: return f(std::integral_constant<int, 16>());
    case 32: return f(std::integral_constant<int, 32>());
    case 64: return f(std::integral_constant<int, 64>());
    case 128: return f(std::integral_constant<int, 128>());
    case 256: return f(std::integral_constant<int, 256>());
    default: return hipErrorInvalidValue;
  }
}

constexpr int kScoreItMany = 8, kScoreItFew = 4;

// the launch's pages per workgroup and groups (see the comment at the score role)
int plan_score(ScoreLaunch& a) {
  const int many = kScoreItMany * kScorePagesPerIt;
  const int it = (a.num_pages + many - 1) / many * a.num_kv_heads >= 512 ? kScoreItMany : kScoreItFew;
  a.nblk = (a.num_pages + it * kScorePagesPerIt - 1) / (it * kScorePagesPerIt);
  a.gshift = topk_group_shift(a.num_pages);
  return it;
}

void plan_predict(PredictLaunch& b) {
  b.nblk = (b.num_pages + kTopkThreads - 1) / kTopkThreads;
  b.gshift = topk_group_shift(b.num_pages);
}

bool no_groups(const ScoreLaunch& a) { return topk_group_shift(a.num_pages) > 0 && !a.gmax; }

// Whether the scoring workgroups of this file and the select of prr_topk.h are quicker than the
// block-wide ones (score_topk_block_kernel), whose scan of the metadata takes longer, by heads x
// pages, and whose select of registers is quicker, above all for large budgets and up to 8192
// pages.  Over 1 to 16 KV heads x 64 to 16384 pages x budgets of 16 to n / 8 (us, here / block):
// 1 x 256 pages 7.2 / 7.6; 1 x 4096, 256 selected 11.1 / 9.1; 2 x 8192, 256: 12.4 / 11.5; 2 x
// 16384, 512: 19.1 / 19.7; 4 x 8192, 256: 14.3 / 15.9; 8 x 2048, 128: 10.3 / 8.7; 8 x 4096, 512:
// 14.8 / 14.3; 8 x 8192, 256: 16.1 / 21.1; 16 x 2500, 156: 13.1 / 15.0.  By this rule the worst of
// them takes 6 % longer than the better of the two.  Without scratch for the groups' keys the
// block-wide ones are (static entry, 8 x 2500, 156: 19.1 / 12.7).
bool score_spread(const ScoreLaunch& a) {
  const int n = a.num_pages;
  if (n <= 2 * kTopkThreads) return true;
  if (no_groups(a) || topk_crowded(n, a.kextra, a.n_forced)) return false;
  return (int64_t)a.num_kv_heads * n + (n > 8192 ? 8000 : 0) >= 16400 + 40 * (int64_t)(a.kextra + a.n_forced);
}

// The same for the EMA update and prediction with scratch, against predict_kernel's one workgroup
// per KV head (2 KV heads, us here / there: 256 pages, 32 predicted 4.2 / 4.9; 1024, 64: 5.5 / 4.9;
// 4096, 256: 8.2 / 6.2; 8192, 256: 8.8 / 8.9; 8192, 1024: 13.3 / 9.7; 16384, 512: 12.2 / 14.9).
bool predict_spread(const PredictLaunch& a) {
  const int n = a.num_pages;
  return n <= kTopkThreads || (n > 4096 && 20 * (a.kextra + a.n_forced) <= n);
}

// Beside the repair the update costs no launch of its own, which pays for more: 8 KV heads, us a
// layer with it / with predict_kernel after the repair: 2048 pages, 512 predicted 38.0 / 42.5;
// 6000, 1024: 62.5 / 67.0; 4096, 1024: 79.6 / 73.5; 2500, 625: 60.5 / 56.9.
bool predict_alone(const PredictLaunch& a) {
  return topk_group_shift(a.num_pages) > 0 && 5 * (a.kextra + a.n_forced) > a.num_pages;
}

}  // namespace

template <bool BF16>
hipError_t launch_score_topk_t(ScoreLaunch a, hipStream_t stream) {
  if (!score_spread(a)) return launch_score_topk_block(a, stream);
  const int it = plan_score(a);
  const dim3 grid(a.nblk, a.num_kv_heads);
  return it == kScoreItMany ? launch((const void*)score_topk_kernel<BF16, kScoreItMany>, grid, stream, a)
                            : launch((const void*)score_topk_kernel<BF16, kScoreItFew>, grid, stream, a);
}

template <bool BF16>
hipError_t launch_spec_attn_t(const SpecLaunch& a, hipStream_t stream) {
  return by_page_size(a.page_size, [&](auto ps) {
    return launch((const void*)spec_attn_kernel<BF16, ps()>, dim3(a.nchunks, a.num_kv_heads), stream, a);
  });
}

template <bool BF16>
hipError_t launch_select_spec_t(ScoreLaunch a, const SpecLaunch& b, hipStream_t stream) {
  if (no_groups(a) || topk_crowded(a.num_pages, a.kextra, a.n_forced)) {
    const hipError_t e = launch_score_topk_block(a, stream);
    return e != hipSuccess ? e : launch_spec_attn_t<BF16>(b, stream);
  }
  const int it = plan_score(a);
  const dim3 grid(a.num_kv_heads * (a.nblk + b.nchunks));
  return by_page_size(b.page_size, [&](auto ps) {
    return it == kScoreItMany ? launch((const void*)select_spec_kernel<BF16, ps(), kScoreItMany>, grid, stream, a, b)
                              : launch((const void*)select_spec_kernel<BF16, ps(), kScoreItFew>, grid, stream, a, b);
  });
}

template <bool BF16>
hipError_t launch_repair_t(const RepairLaunch& a, hipStream_t stream) {
  return by_page_size(a.page_size, [&](auto ps) {
    return launch((const void*)repair_kernel<BF16, ps()>, dim3(a.num_kv_heads * (a.nwork + a.group)), stream, a);
  });
}

template <bool BF16>
hipError_t launch_repair_predict_t(const RepairLaunch& a, PredictLaunch b, hipStream_t stream) {
  if (predict_alone(b)) {
    const hipError_t e = launch_repair_t<BF16>(a, stream);
    return e != hipSuccess ? e : launch_predict(b, stream);
  }
  plan_predict(b);
  return by_page_size(a.page_size, [&](auto ps) {
    return launch((const void*)repair_predict_kernel<BF16, ps()>, dim3(a.num_kv_heads * (a.nwork + a.group + b.nblk)),
                  stream, a, b);
  });
}

}  // namespace prr
