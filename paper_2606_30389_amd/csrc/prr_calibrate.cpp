// Online calibration of the EMA predictor (Section 4.2): the score-weighted hit rate of
// Eq. (4) for every candidate theta = (alpha, beta, gamma) of a grid, simulated over
// prefill score trajectories, and its argmax (Eq. (5)).  Host code: it runs on the CPU
// cores while the device finishes the prefill, one grid point per task.
#include <math.h>
#include <string.h>

#include <algorithm>
#include <atomic>
#include <limits>
#include <thread>
#include <vector>

#include "prr_launch.h"

namespace {

// Order-preserving float -> uint32 map of the selection keys (-0 == +0); the decision
// values are rounded to float32 first, as on the device.
inline uint32_t key_of(double v) {
  float f = (float)v;
  if (f == 0.0f) f = 0.0f;
  uint32_t u;
  memcpy(&u, &f, 4);
  return (u & 0x80000000u) ? ~u : (u | 0x80000000u);
}

// Membership (0/1 by block index) of the k largest of the candidates (keys key[j] of
// blocks idx[j]; ties: lower index first): two 11-bit radix passes narrow the rank-k key
// to one bin, whose few members are ordered exactly.
struct TopK {
  std::vector<uint32_t> hist;
  std::vector<uint64_t> tie;
  std::vector<int> sub;
  TopK() : hist(2048), tie(), sub() {}
};

inline uint64_t pack(uint32_t key, int index) { return ((uint64_t)key << 32) | (uint32_t)~(uint32_t)index; }

void top_k(const uint32_t* key, const int* idx, int n, int k, std::vector<uint8_t>& in, TopK& s) {
  std::fill(in.begin(), in.end(), 0);
  if (k <= 0 || n == 0) return;
  if (k >= n) {
    for (int j = 0; j < n; ++j) in[idx[j]] = 1;
    return;
  }
  // pass 1: bins of the top 11 bits; find the bin b1 holding rank k (from the top)
  std::fill(s.hist.begin(), s.hist.end(), 0u);
  for (int j = 0; j < n; ++j) ++s.hist[key[j] >> 21];
  int b1 = 2047, above = 0;
  while (above + (int)s.hist[b1] < k) above += s.hist[b1--];
  s.sub.clear();
  for (int j = 0; j < n; ++j) {
    const uint32_t b = key[j] >> 21;
    if ((int)b > b1) in[idx[j]] = 1;
    else if ((int)b == b1) s.sub.push_back(j);
  }
  // pass 2 within b1: the next 11 bits
  std::fill(s.hist.begin(), s.hist.end(), 0u);
  for (int j : s.sub) ++s.hist[(key[j] >> 10) & 2047u];
  int b2 = 2047;
  while (above + (int)s.hist[b2] < k) above += s.hist[b2--];
  s.tie.clear();
  for (int j : s.sub) {
    const int b = (int)((key[j] >> 10) & 2047u);
    if (b > b2) in[idx[j]] = 1;
    else if (b == b2) s.tie.push_back(pack(key[j], idx[j]));
  }
  // the members of the last bin: exact order by (key desc, index asc)
  const int need = k - above;
  if (need < (int)s.tie.size())
    std::nth_element(s.tie.begin(), s.tie.begin() + (need - 1), s.tie.end(), std::greater<uint64_t>());
  for (int j = 0; j < need; ++j) in[~(uint32_t)s.tie[j] & 0xffffffffu] = 1;
}

// A_phi of every row phi >= 1 of every trajectory (independent of theta): its blocks
// and their scores, and the denominator of Eq. (4).  Block i exists from row born[i] on.
struct RowSets {
  std::vector<std::vector<int>> idx;
  std::vector<std::vector<double>> w;
  std::vector<double> all;
};

void row_set(const float* scores, int T, int N, const int32_t* born, int k, int task, RowSets& R,
             std::vector<uint32_t>& ck, std::vector<int>& ci, std::vector<uint8_t>& inA, TopK& tk) {
  const int phi = task % T;
  if (phi == 0) return;
  const float* row = scores + (size_t)task * N;
  int nc = 0;
  for (int i = 0; i < N; ++i) {
    if (born[i] <= phi) {
      ck[nc] = key_of(row[i]);
      ci[nc++] = i;
    }
  }
  top_k(ck.data(), ci.data(), nc, k, inA, tk);
  for (int i = 0; i < N; ++i) {
    if (inA[i]) {
      R.idx[task].push_back(i);
      R.w[task].push_back(row[i]);
      R.all[task] += row[i];
    }
  }
}

// The two passes of a row over every block, written for the vector units: the host's baseline
// instruction set holds two doubles per register, AVX2 four (no contraction into fused
// multiply-adds either way, so both give the same values).
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
#define PRR_VECTOR __attribute__((target("avx2")))
#else
#define PRR_VECTOR
#endif

// Eq. (2) as signed keys in the order of key_of: sign-magnitude to two's complement, -0 as +0.
#define PRR_KEYS_BODY                                                  \
  for (int i = 0; i < n; ++i) {                                        \
    const float f = (float)(level[i] + gamma * trend[i]) + 0.0f;       \
    int32_t u;                                                         \
    memcpy(&u, &f, 4);                                                 \
    key[i] = u ^ ((u >> 31) & 0x7fffffff);                             \
  }
// Eq. (3): the trend reads the previous level
#define PRR_EMA_BODY                                                   \
  for (int i = 0; i < n; ++i) {                                        \
    const double x = row[i], l = level[i];                             \
    trend[i] = beta * (x - l) + (1.0 - beta) * trend[i];               \
    level[i] = alpha * x + (1.0 - alpha) * l;                          \
  }
// Blocks of 32 whose largest key reaches the bound are looked at one by one.
#define PRR_COLLECT_BODY                                               \
  int m = 0;                                                           \
  for (int i0 = 0; i0 < n; i0 += 32) {                                 \
    const int e = n - i0 < 32 ? n - i0 : 32;                           \
    int any = 0;                                                       \
    for (int i = 0; i < e; ++i) any |= key[i0 + i] >= bound ? 1 : 0;   \
    if (!any) continue;                                                \
    for (int i = 0; i < e; ++i) {                                      \
      out[m] = i0 + i;                                                 \
      m += key[i0 + i] >= bound ? 1 : 0;                               \
    }                                                                  \
  }                                                                    \
  return m;

// A key that at least `rank` and little more of the sampled keys reach, or the smallest of them
// (by halving the range: nth_element takes five times as long).
#define PRR_SAMPLE_BODY                                                \
  int32_t lo = key[0], hi = key[0];                                    \
  for (int i = 0; i < n; ++i) {                                        \
    lo = lo < key[i] ? lo : key[i];                                    \
    hi = hi > key[i] ? hi : key[i];                                    \
  }                                                                    \
  while (lo < hi) {                                                    \
    const int32_t mid = (int32_t)(((int64_t)lo + hi + 1) >> 1);        \
    int c = 0;                                                         \
    for (int i = 0; i < n; ++i) c += key[i] >= mid ? 1 : 0;            \
    if (c < rank) hi = mid - 1;                                        \
    else lo = mid;                                                     \
    if (c >= rank && c <= rank + rank / 8) break;                      \
  }                                                                    \
  return lo;

PRR_VECTOR int32_t sample_bound_avx2(const int32_t* key, int n, int rank) { PRR_SAMPLE_BODY }
int32_t sample_bound_base(const int32_t* key, int n, int rank) { PRR_SAMPLE_BODY }
PRR_VECTOR void keys_avx2(const double* level, const double* trend, double gamma, int n, int32_t* key) { PRR_KEYS_BODY }
void keys_base(const double* level, const double* trend, double gamma, int n, int32_t* key) { PRR_KEYS_BODY }
PRR_VECTOR void ema_avx2(const float* row, double alpha, double beta, int n, double* level, double* trend) { PRR_EMA_BODY }
void ema_base(const float* row, double alpha, double beta, int n, double* level, double* trend) { PRR_EMA_BODY }
PRR_VECTOR int collect_avx2(const int32_t* key, int n, int32_t bound, int* out) { PRR_COLLECT_BODY }
int collect_base(const int32_t* key, int n, int32_t bound, int* out) { PRR_COLLECT_BODY }

bool have_avx2() {
#if !defined(__HIP_DEVICE_COMPILE__) && defined(__x86_64__)
  static const bool have = __builtin_cpu_supports("avx2");
  return have;
#else
  return false;
#endif
}

constexpr int kSampled = 512;  // keys sampled per row

inline uint32_t ranked(int32_t key) { return (uint32_t)key ^ 0x80000000u; }  // as key_of orders them

// Eq. (4) for one theta over B trajectories of T rows of N scores, averaged over B.  Block
// i exists from row born[i] on (Section 4.1: its state starts there as level = its score,
// trend = 0); P_phi ranks the predictions of the blocks that had a state before row phi,
// A_phi (precomputed) the blocks that exist at row phi.  Rows phi >= 1 (those with a
// prediction) are averaged.
//
// The time goes to passes over all blocks, so a row makes three plain ones (keys, collect,
// EMA) and ranks few: keys taken at a stride give a bound that about 2p blocks reach, and those
// are ordered exactly.  Rows where fewer than p or more than half of the blocks reach it,
// and budgets too large for that, rank every block by top_k.  The bound is each row's own: the
// scores of a row move as a whole with the query, so that a key kept from the row before misses
// the range on half of the rows of real trajectories.  64 rows x 8192 blocks, 80
// grid points, 8 threads; one scalar pass that ranks every block, a bound from the row before,
// this: rows of fixed mean 56-71, 22-27, 23-25 ms; Quest scores of 16 query heads (correlation 0.95 between rows)
// 61-75, 65-70, 22; of 4 (0.85) 64-72, 82-90, 24.
double objective(const float* scores, int B, int T, int N, const int32_t* born, const std::vector<int>& late,
                 const RowSets& R, int p, const float theta[3]) {
  const double alpha = theta[0], beta = theta[1], gamma = theta[2];
  const bool vec = have_avx2();
  std::vector<double> level(N), trend(N);
  std::vector<uint8_t> inP(N);
  std::vector<int32_t> key(N);
  std::vector<uint32_t> ck(N);
  std::vector<int> ci(N + 32);
  std::vector<uint64_t> order;
  TopK tk;
  // the sampled keys, and the rank among them that p blocks reach, four standard deviations
  // and two more on top
  const int stride = std::max(1, N / kSampled), n_sample = N / stride;
  const double mean = (double)p * n_sample / N;
  const int srank = (int)std::min(2.0 * kSampled, mean + 4.0 * sqrt(mean) + 2.0);
  std::vector<int32_t> sample(n_sample);
  double sum_b = 0.0;
  for (int b = 0; b < B; ++b) {
    const float* traj = scores + (size_t)b * T * N;
    // `late` holds the blocks that form after row 0, by row; those up to `formed` have
    size_t formed = 0;
    int nhas = 0;
    double sum_t = 0.0;
    int rows = 0;
    for (int phi = 0; phi < T; ++phi) {
      const float* row = traj + (size_t)phi * N;
      if (phi >= 1) {
        (vec ? keys_avx2 : keys_base)(level.data(), trend.data(), gamma, N, key.data());
        for (size_t j = formed; j < late.size(); ++j) key[late[j]] = std::numeric_limits<int32_t>::min();
        int m = -1;
        std::fill(inP.begin(), inP.end(), 0);
        if (srank < n_sample / 2 && p > 0 && p < nhas) {
          for (int j = 0; j < n_sample; ++j) sample[j] = key[j * stride];
          const int32_t bound = (vec ? sample_bound_avx2 : sample_bound_base)(sample.data(), n_sample, srank);
          // (a block that has no state yet is below any bound but the lowest key)
          if (bound != std::numeric_limits<int32_t>::min()) {
            m = (vec ? collect_avx2 : collect_base)(key.data(), N, bound, ci.data());
            if (m < p || m > N / 2) m = -1;
          }
        }
        if (m < 0) {
          m = 0;
          for (int i = 0; i < N; ++i) {
            if (born[i] < phi) {
              ck[m] = ranked(key[i]);
              ci[m++] = i;
            }
          }
          top_k(ck.data(), ci.data(), m, p, inP, tk);
        } else {
          order.clear();
          for (int j = 0; j < m; ++j) order.push_back(pack(ranked(key[ci[j]]), ci[j]));
          std::nth_element(order.begin(), order.begin() + (p - 1), order.end(), std::greater<uint64_t>());
          for (int j = 0; j < p; ++j) inP[~(uint32_t)order[j] & 0xffffffffu] = 1;
        }
        const size_t r = (size_t)b * T + phi;
        double hit = 0.0;
        const std::vector<int>& ia = R.idx[r];
        const std::vector<double>& wa = R.w[r];
        for (size_t j = 0; j < ia.size(); ++j)
          if (inP[ia[j]]) hit += wa[j];
        sum_t += R.all[r] != 0.0 ? hit / R.all[r] : 0.0;
        ++rows;
        (vec ? ema_avx2 : ema_base)(row, alpha, beta, N, level.data(), trend.data());
      } else {
        for (int i = 0; i < N; ++i) {
          level[i] = born[i] <= 0 ? row[i] : 0.0;
          trend[i] = 0.0;
        }
        nhas = N - (int)late.size();
      }
      for (; formed < late.size() && born[late[formed]] <= phi; ++formed) {  // blocks that form at this row
        level[late[formed]] = row[late[formed]];
        trend[late[formed]] = 0.0;
        ++nhas;
      }
      for (size_t j = formed; j < late.size(); ++j) level[late[j]] = trend[late[j]] = 0.0;
    }
    sum_b += rows ? sum_t / rows : 0.0;
  }
  return sum_b / B;
}

}  // namespace

namespace prr {

// Arguments were validated by the C ABI (prr_calibrate).
void calibrate_grid(const float* scores, int n_traj, int n_rows, int n_blocks, const int32_t* form_row, int k_select,
                    int p_select, const float* grid, int n_grid, int n_threads, float* best_theta,
                    double* objective_out) {
  const int p = p_select > 0 ? p_select : k_select;
  std::vector<int32_t> born(n_blocks, 0);
  if (form_row) born.assign(form_row, form_row + n_blocks);
  std::vector<int> late;
  for (int i = 0; i < n_blocks; ++i)
    if (born[i] > 0) late.push_back(i);
  std::stable_sort(late.begin(), late.end(), [&](int x, int y) { return born[x] < born[y]; });
  std::vector<double> obj(n_grid, 0.0);
  unsigned hw = std::thread::hardware_concurrency();
  const int nt_all = std::max(1, n_threads > 0 ? n_threads : (int)(hw ? hw : 1));
  const int n_sets = n_traj * n_rows;
  RowSets R;
  R.idx.resize(n_sets);
  R.w.resize(n_sets);
  R.all.assign(n_sets, 0.0);
  // one set of threads for both parts: the rows' sets, then (once the last of them is done) the
  // grid points
  const int nt = std::max(1, std::min(nt_all, std::max(n_grid, n_sets)));
  std::atomic<int> next_set(0), sets_done(0), next(0);
  auto work = [&]() {
    std::vector<uint32_t> ck(n_blocks);
    std::vector<int> ci(n_blocks);
    std::vector<uint8_t> inA(n_blocks);
    TopK tk;
    for (int task = next_set++; task < n_sets; task = next_set++) {
      row_set(scores, n_rows, n_blocks, born.data(), k_select, task, R, ck, ci, inA, tk);
      ++sets_done;
    }
    while (sets_done.load() < n_sets) std::this_thread::yield();
    for (int g = next++; g < n_grid; g = next++)
      obj[g] = objective(scores, n_traj, n_rows, n_blocks, born.data(), late, R, p, grid + 3 * g);
  };
  std::vector<std::thread> pool;
  for (int i = 1; i < nt; ++i) pool.emplace_back(work);
  work();
  for (auto& th : pool) th.join();
  int best = 0;
  for (int g = 1; g < n_grid; ++g)
    if (obj[g] > obj[best]) best = g;  // the first grid point on ties
  for (int i = 0; i < 3; ++i) best_theta[i] = grid[3 * best + i];
  if (objective_out)
    for (int g = 0; g < n_grid; ++g) objective_out[g] = obj[g];
}

}  // namespace prr
