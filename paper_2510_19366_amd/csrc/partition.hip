// Partition solver (Sec. 3.2.1, "Partition Optimization Solver"; objective Eq. 4).  Host code
// only, offline: splits an expert's C intermediate neurons into S equal groups so that each
// calibration token's activation mass concentrates in few groups.  Greedy initialiser by
// calibration-wide L1 norm, then simulated annealing over swaps between groups.
#ifndef __HIP_DEVICE_COMPILE__  // nothing here is for the device pass of the compiler
#include <immintrin.h>

#include <algorithm>
#include <cmath>
#include <cstdint>
#include <new>
#include <numeric>
#include <vector>

#include "../../include/moe_prism.h"

namespace {

inline uint64_t splitmix64(uint64_t x) {
  x += 0x9E3779B97F4A7C15ull;
  uint64_t z = x;
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

// ---------------------------------------------------------------- Eq. 4, eight tokens at a time
// The annealer spends its time on one thing: the loss of a partition that differs from the current
// one by a swap, i.e. for every token the sum of its S - k_in smallest group sums.  Group sums are
// kept group-major (L[n][b]) and activations neuron-major (|A| transposed once per call), so that 8
// tokens are one vector: a sorting network of vector minima and maxima replaces one sort per token.
// Every token's arithmetic, and the order in which the tokens' losses are added up, is that of the
// plain definition, so the decisions do not depend on the vector width.
// Measured for 256 tokens, 768 neurons, S = 4: 4.1 us a proposal with one sort per token, 0.11 us so, 0.07 us with most
// proposals decided in binary32.
constexpr int V = 8;
typedef double vd __attribute__((vector_size(V * sizeof(double))));
typedef float vf __attribute__((vector_size(V * sizeof(float))));
constexpr int MAX_SUB = 64;

#define MP_INLINE inline __attribute__((always_inline))

template <class Vec>
MP_INLINE void order(Vec& a, Vec& b) {
  const Vec lo = b < a ? b : a, hi = b < a ? a : b;
  a = lo;
  b = hi;
}
// Batcher's odd-even merge sort of S vectors (S = 0: of n)
template <int S, class Vec>
MP_INLINE void sort_vectors(Vec* v, int n) {
  auto merge = [&](int m, int p, int k, int j) {
    for (int i = 0; i < k; ++i)
      if (i + j + k < m && (i + j) / (2 * p) == (i + j + k) / (2 * p)) order(v[i + j], v[i + j + k]);
  };
  if constexpr (S > 0) {
#pragma unroll
    for (int p = 1; p < S; p *= 2)
#pragma unroll
      for (int k = p; k >= 1; k /= 2)
#pragma unroll
        for (int j = k % p; j + k < S; j += 2 * k) merge(S, p, k, j);
  } else {
    for (int p = 1; p < n; p *= 2)
      for (int k = p; k >= 1; k /= 2)
        for (int j = k % p; j + k < n; j += 2 * k) merge(n, p, k, j);
  }
}

// The vectors of B tokens, the last one padded with zeros: loops in binary64 run to n64, arrays have rows of `stride`
// elements, to which the loops in binary32 run.
constexpr int VF = 16;
typedef float vf16 __attribute__((vector_size(VF * sizeof(float))));
struct Span {
  int n64, stride;
};
// (one vector of either kind has them all, so the sums in binary32 cost as much as those they are to replace)
constexpr bool worth_screening(int B) { return B > V; }
constexpr Span span_of(int B) {
  return {(B + V - 1) / V * V, worth_screening(B) ? (B + VF - 1) / VF * VF : V};
}

// One proposal: neurons of |A| columns ci, cj move between groups gi and gj, whose sums become ri, rj.
struct Swap {
  const float *ci, *cj;
  int gi, gj;
  double *ri, *rj;
};
// tok[b] = sum of the k smallest group sums of token b after the swap (ci == nullptr: as they are).  With tok == nullptr
// (a swap, finite sums) nothing of that is written: the tok[b] added up in any order are *plain, the |tok[b]| the result.
template <int S>
MP_INLINE double swap_losses_t(const double* L, Span rows, int n, int k, const Swap& w, double* tok, double* plain) {
  const int m = S > 0 ? S : n;
  const double* row[S > 0 ? S : MAX_SUB];
  vd v[S > 0 ? S : MAX_SUB];
  auto smallest = [&] {
    sort_vectors<S>(v, n);
    vd s = {};
    if constexpr (S > 0) {  // (an index known to the compiler, or v lives in memory)
#pragma unroll
      for (int i = 0; i < S; ++i)
        if (i < k) s += v[i];
    } else {
      for (int i = 0; i < k; ++i) s += v[i];
    }
    return s;
  };
  const double *li = L + (size_t)w.gi * rows.stride, *lj = L + (size_t)w.gj * rows.stride;
  auto swapped = [&](int b, vd& ri, vd& rj) {
    const vd ai = __builtin_convertvector(*reinterpret_cast<const vf*>(w.ci + b), vd);
    const vd aj = __builtin_convertvector(*reinterpret_cast<const vf*>(w.cj + b), vd);
    ri = *reinterpret_cast<const vd*>(li + b) - ai + aj;
    rj = *reinterpret_cast<const vd*>(lj + b) - aj + ai;
  };
  if (tok != nullptr) {
    for (int g = 0; g < m; ++g) row[g] = L + (size_t)g * rows.stride;
    if (w.ci != nullptr) {
      for (int b = 0; b < rows.n64; b += V) {
        vd ri, rj;
        swapped(b, ri, rj);
        *reinterpret_cast<vd*>(w.ri + b) = ri;
        *reinterpret_cast<vd*>(w.rj + b) = rj;
      }
      row[w.gi] = w.ri;
      row[w.gj] = w.rj;
    }
    for (int b = 0; b < rows.n64; b += V) {
      for (int g = 0; g < m; ++g) v[g] = *reinterpret_cast<const vd*>(row[g] + b);
      *reinterpret_cast<vd*>(tok + b) = smallest();
    }
    return 0.0;
  }
  // finite sums: which value is whose does not matter, so the two that change come last
  int kept = 0;
  for (int g = 0; g < m; ++g)
    if (g != w.gi && g != w.gj) row[kept++] = L + (size_t)g * rows.stride;
  vd sum = {}, sum_abs = {};
  for (int b = 0; b < rows.n64; b += V) {
    for (int g = 0; g < m - 2; ++g) v[g] = *reinterpret_cast<const vd*>(row[g] + b);
    swapped(b, v[m - 2], v[m - 1]);
    const vd s = smallest();
    sum += s;
    sum_abs += s < 0.0 ? -s : s;
  }
  double total = 0.0, total_abs = 0.0;
  for (int i = 0; i < V; ++i) total += sum[i], total_abs += sum_abs[i];
  *plain = total;
  return total_abs;
}
MP_INLINE double swap_losses_any(const double* L, Span rows, int S, int k, const Swap& w, double* tok, double* plain) {
  switch (S) {
    case 2: return swap_losses_t<2>(L, rows, S, k, w, tok, plain);
    case 4: return swap_losses_t<4>(L, rows, S, k, w, tok, plain);
    case 8: return swap_losses_t<8>(L, rows, S, k, w, tok, plain);
    default: return swap_losses_t<0>(L, rows, S, k, w, tok, plain);
  }
}
// The same sum in binary32, sixteen tokens at a time, from the group sums rounded to it (Lf): a bound of it decides most
// proposals.  At most RUN vectors are added up before a lane goes on in binary64.
constexpr int RUN = 16;
template <int S>
MP_INLINE double screen_t(const float* Lf, Span rows, int n, int k, const Swap& w) {
  const int m = S > 0 ? S : n;
  const float* row[S > 0 ? S : MAX_SUB];
  int kept = 0;
  for (int g = 0; g < m; ++g)
    if (g != w.gi && g != w.gj) row[kept++] = Lf + (size_t)g * rows.stride;
  const float *li = Lf + (size_t)w.gi * rows.stride, *lj = Lf + (size_t)w.gj * rows.stride;
  auto at = [](const float* p) { return *reinterpret_cast<const vf16*>(p); };
  vd total = {};
  for (int b0 = 0; b0 < rows.stride; b0 += RUN * VF) {
    vf16 sum = {};
    for (int b = b0; b < std::min(rows.stride, b0 + RUN * VF); b += VF) {
      vf16 v[S > 0 ? S : MAX_SUB];
      for (int g = 0; g < m - 2; ++g) v[g] = at(row[g] + b);
      const vf16 ai = at(w.ci + b), aj = at(w.cj + b);
      v[m - 2] = at(li + b) - ai + aj;
      v[m - 1] = at(lj + b) - aj + ai;
      sort_vectors<S>(v, n);
      vf16 s = {};
      if constexpr (S > 0) {
#pragma unroll
        for (int i = 0; i < S; ++i)
          if (i < k) s += v[i];
      } else {
        for (int i = 0; i < k; ++i) s += v[i];
      }
      sum += s;
    }
    const vf* half = reinterpret_cast<const vf*>(&sum);
    total += __builtin_convertvector(half[0], vd) + __builtin_convertvector(half[1], vd);
  }
  double r = 0.0;
  for (int i = 0; i < V; ++i) r += total[i];
  return r;
}
MP_INLINE double screen_any(const float* Lf, Span rows, int S, int k, const Swap& w) {
  switch (S) {
    case 2: return screen_t<2>(Lf, rows, S, k, w);
    case 4: return screen_t<4>(Lf, rows, S, k, w);
    case 8: return screen_t<8>(Lf, rows, S, k, w);
    default: return screen_t<0>(Lf, rows, S, k, w);
  }
}
// row += column
MP_INLINE void add_column_t(double* row, const float* column, Span rows) {
  for (int b = 0; b < rows.n64; b += V)
    *reinterpret_cast<vd*>(row + b) += __builtin_convertvector(*reinterpret_cast<const vf*>(column + b), vd);
}
// the group sums after a swap that is taken, and what is kept of them in binary32 (Lf == nullptr: nothing)
MP_INLINE void apply_t(double* L, float* Lf, Span rows, const Swap& w) {
  double *li = L + (size_t)w.gi * rows.stride, *lj = L + (size_t)w.gj * rows.stride;
  for (int b = 0; b < rows.n64; b += V) {
    const vd ai = __builtin_convertvector(*reinterpret_cast<const vf*>(w.ci + b), vd);
    const vd aj = __builtin_convertvector(*reinterpret_cast<const vf*>(w.cj + b), vd);
    vd &ri = *reinterpret_cast<vd*>(li + b), &rj = *reinterpret_cast<vd*>(lj + b);
    ri = ri - ai + aj;
    rj = rj - aj + ai;
    if (Lf != nullptr) {
      *reinterpret_cast<vf*>(Lf + (size_t)w.gi * rows.stride + b) = __builtin_convertvector(ri, vf);
      *reinterpret_cast<vf*>(Lf + (size_t)w.gj * rows.stride + b) = __builtin_convertvector(rj, vf);
    }
  }
}

// The loops over the tokens for the widest vectors of this CPU.
struct Loops {
  double (*losses)(const double* L, Span rows, int S, int k, const Swap& w, double* tok, double* plain);
  double (*screen)(const float* Lf, Span rows, int S, int k, const Swap& w);
  void (*add_column)(double* row, const float* column, Span rows);
  void (*apply)(double* L, float* Lf, Span rows, const Swap& w);
};
#define MP_LOOPS(WIDTH, TARGET)                                                                                            \
  TARGET double losses_##WIDTH(const double* L, Span rows, int S, int k, const Swap& w, double* tok, double* plain) {        \
    return tok != nullptr ? swap_losses_any(L, rows, S, k, w, tok, plain) : swap_losses_any(L, rows, S, k, w, nullptr, plain); \
  }                                                                                                                        \
  TARGET double screen_##WIDTH(const float* Lf, Span rows, int S, int k, const Swap& w) { return screen_any(Lf, rows, S, k, w); } \
  TARGET void add_column_##WIDTH(double* row, const float* column, Span rows) { add_column_t(row, column, rows); }              \
  TARGET void apply_##WIDTH(double* L, float* Lf, Span rows, const Swap& w) { apply_t(L, Lf, rows, w); }                         \
  constexpr Loops loops_##WIDTH{losses_##WIDTH, screen_##WIDTH, add_column_##WIDTH, apply_##WIDTH};
MP_LOOPS(512, __attribute__((target("avx512f"))))
MP_LOOPS(256, __attribute__((target("avx2"))))
MP_LOOPS(128, )
#undef MP_LOOPS
const Loops& pick_loops() {
  __builtin_cpu_init();
  if (__builtin_cpu_supports("avx512f")) return loops_512;
  if (__builtin_cpu_supports("avx2")) return loops_256;
  return loops_128;
}

// memory for vectors of 64 bytes
template <class T>
struct Aligned {
  T* p;
  explicit Aligned(size_t n) : p(static_cast<T*>(::operator new(n * sizeof(T), std::align_val_t(64)))) {
    std::fill(p, p + n, T(0));
  }
  ~Aligned() { ::operator delete(p, std::align_val_t(64)); }
  Aligned(const Aligned&) = delete;
  Aligned& operator=(const Aligned&) = delete;
};

// |A| neuron-major, tokens padded with zeros to whole vectors, and the group sums of a partition
struct Problem {
  int B, C, S;
  Span rows;
  Aligned<float> cols;   // [C][stride]
  Aligned<double> L;     // [S][stride]: neurons added in ascending index order
  Problem(const Loops& loops, int B_, int C_, int S_, const float* A, const int32_t* g)
      : B(B_), C(C_), S(S_), rows(span_of(B_)), cols((size_t)C_ * rows.stride), L((size_t)S_ * rows.stride) {
    // |A| turned over in blocks of 4 x 4, 16 neurons (whole lines) of 4 tokens at a time
    const int B4 = B / 4 * 4, C4 = C / 4 * 4;
    const __m128 magnitude = _mm_castsi128_ps(_mm_set1_epi32(0x7fffffff));
    for (int c0 = 0; c0 < C4; c0 += 16)
      for (int b = 0; b < B4; b += 4)
        for (int c = c0; c < std::min(C4, c0 + 16); c += 4) {
          __m128 r[4];
          for (int i = 0; i < 4; ++i) r[i] = _mm_and_ps(_mm_loadu_ps(A + (size_t)(b + i) * C + c), magnitude);
          _MM_TRANSPOSE4_PS(r[0], r[1], r[2], r[3]);
          for (int i = 0; i < 4; ++i) _mm_store_ps(column(c + i) + b, r[i]);
        }
    for (int c = 0; c < C; ++c)
      for (int b = c < C4 ? B4 : 0; b < B; ++b) column(c)[b] = std::fabs(A[(size_t)b * C + c]);
    for (int c = 0; c < C; ++c) loops.add_column(L.p + (size_t)g[c] * rows.stride, column(c), rows);
  }
  float* column(int c) const { return cols.p + (size_t)c * rows.stride; }
};

bool args_ok(int32_t B, int32_t C, int32_t S, const float* A, const int32_t* g) {
  return B > 0 && C > 0 && S > 0 && S <= 64 && C % S == 0 && A != nullptr && g != nullptr;
}

bool partition_ok(int32_t C, int32_t S, const int32_t* g) {
  std::vector<int> size(S, 0);
  for (int c = 0; c < C; ++c) {
    if (g[c] < 0 || g[c] >= S) return false;
    ++size[g[c]];
  }
  for (int n = 0; n < S; ++n)
    if (size[n] != C / S) return false;
  return true;
}

}  // namespace

extern "C" int moe_prism_partition_greedy(int32_t B, int32_t C, int32_t S, const float* A,
                                          int32_t* group_of) {
  if (!args_ok(B, C, S, A, group_of)) return MOE_PRISM_ERR_INVALID_ARG;
  std::vector<double> norm(C, 0.0);
  for (int b = 0; b < B; ++b)
    for (int c = 0; c < C; ++c) norm[c] += std::fabs((double)A[(size_t)b * C + c]);
  std::vector<int32_t> order(C);
  std::iota(order.begin(), order.end(), 0);
  std::sort(order.begin(), order.end(), [&](int32_t a, int32_t b) {
    if (norm[a] != norm[b]) return norm[a] > norm[b];
    return a < b;
  });
  std::vector<double> acc(S, 0.0);
  std::vector<int> size(S, 0);
  for (int32_t c : order) {
    int best = -1;
    for (int n = 0; n < S; ++n)
      if (size[n] < C / S && (best < 0 || acc[n] < acc[best])) best = n;
    group_of[c] = best;
    acc[best] += norm[c];
    ++size[best];
  }
  return MOE_PRISM_OK;
}

extern "C" int moe_prism_partition_objective(int32_t B, int32_t C, int32_t S, int32_t k_in,
                                             const float* A, const int32_t* group_of,
                                             double* loss) {
  if (!args_ok(B, C, S, A, group_of) || loss == nullptr || k_in < 0 || k_in > S ||
      !partition_ok(C, S, group_of))
    return MOE_PRISM_ERR_INVALID_ARG;
  const Loops& loops = pick_loops();
  const Problem P(loops, B, C, S, A, group_of);
  Aligned<double> tok(P.rows.stride);
  double unused;
  loops.losses(P.L.p, P.rows, S, S - k_in, Swap{nullptr, nullptr, 0, 0, nullptr, nullptr}, tok.p, &unused);
  double total = 0.0;
  for (int b = 0; b < B; ++b) total += tok.p[b];
  *loss = total;
  return MOE_PRISM_OK;
}

namespace {

// moe_prism_partition_anneal on checked arguments; returns the loss
double anneal(const Loops& loops, int32_t B, int32_t C, int32_t S, int32_t k_in, const float* A, int32_t* group_of, int64_t steps,
              double t0, double t1, uint64_t seed) {
  const int k_drop = S - k_in;
  Problem P(loops, B, C, S, A, group_of);
  const Span rows = P.rows;
  const size_t all = (size_t)S * rows.stride;
  // A loss is its tokens' losses added up in order, one long chain of additions.  A decision rarely needs it: the sum in
  // any order (eight tokens at a time) is within a bound of it, and inside the bounds of a proposal's loss and the
  // current one nearly every decision is the same.  The others, and the final loss, are evaluated as the definition says.
  // 256 tokens, 768 neurons in 4 groups, 3000 steps: 316 us, with the ordered sums of four proposals side by side 536; with
  // the binary32 sums below in front (1 % of the proposals stay open behind them) 215.
  Aligned<double> tok(rows.stride), moved((size_t)2 * rows.stride);
  auto ordered = [&](const Swap& w) {
    double unused, sum = 0.0;
    loops.losses(P.L.p, rows, S, k_drop, w, tok.p, &unused);
    for (int b = 0; b < B; ++b) sum += tok.p[b];
    return sum;
  };
  const Swap none{nullptr, nullptr, 0, 0, nullptr, nullptr};
  double loss = ordered(none), loss_err = 0.0;  // the current loss is within loss_err of `loss`
  bool exact = true;                            // and equal to it
  constexpr double ULP = 1.0 / 9007199254740992.0, SLACK = 1.0 + 1e-9;  // (SLACK: exp and pow are not monotone to the last bit)
  double temp_most = std::max(t0, t1) * SLACK;  // no later step is hotter
  const bool cooling = t1 <= t0;
  bool finite = true;  // (not: what a comparison makes of a NaN depends on the order of the groups)
  for (size_t b = 0; b < all; ++b) finite = finite && std::isfinite(P.L.p[b]);
  // Binary32 first.  With m the sum of all activations, which no swap changes and no group sum, partial or not, exceeds:
  // the group sums are off by a rounding (together 2^-24 m), the two that change by two more each (of at most 2 m together,
  // 4 2^-24 m), the k smallest of a token by no more than that in all, their sum by k - 1 roundings of it, and the sum of
  // RUN vectors by RUN.  That is below (k + RUN + 5) 2^-24 m; a rounding below the normal numbers, also to zero, is off by
  // 2^-126.  Everything stays finite where m does with room to spare.
  double m = 0.0;
  for (size_t b = 0; b < all; ++b) m += std::fabs(P.L.p[b]);
  bool screened = worth_screening(B) && finite && m < 1e37 && k_drop > 0 && k_drop < S;  // (no sum or all of them: nothing to tell apart)
  // Given up where it costs more than it saves.  It takes half as long as the binary64 sum that a decision saves; a
  // proposal it leaves open costs that half, and the ordered sum of the current loss if that is known by the binary32 sum of a
  // taken swap only and too wide for binary64 to decide: the time of both and more.  Against binary64 alone, 768 neurons in 4 | 16
  // groups, half of them in: 9 tokens 1.07 | 1.75 times as fast, 256 1.4 | 1.9; 1408 in 8 at a constant temperature, all but one in,
  // 2048 tokens 0.97 to 1.03 (with the ordered sum before the binary64 one 0.86 to 1.02), 8192 1.00 to 1.04.
  int credit = 16;
  constexpr int MOST_CREDIT = 64, ORDERED_COST = 3;
  const double screen_err = (k_drop + RUN + 8.0) / 16777216.0 * m + (double)rows.stride * (4.0 * S + 4.0) * 1.2e-38;
  Aligned<float> Lf(screened ? all : 0);
  if (screened)
    for (size_t b = 0; b < all; ++b) Lf.p[b] = (float)P.L.p[b];
  for (int64_t step = 0; step < steps; ++step) {
    const int i = (int)(splitmix64(seed + 3ull * (uint64_t)step) % (uint64_t)C);
    const int j = (int)(splitmix64(seed + 3ull * (uint64_t)step + 1ull) % (uint64_t)C);
    const int gi = group_of[i], gj = group_of[j];
    if (gi == gj) continue;
    const Swap w{P.column(i), P.column(j), gi, gj, moved.p, moved.p + rows.stride};
    double sum = 0.0, sum_err = 0.0;
    double u = -1.0, temp = 0.0;
    auto draw = [&] {
      const uint64_t r2 = splitmix64(seed + 3ull * (uint64_t)step + 2ull);
      u = (double)(r2 >> 11) * ULP;
    };
    auto heat = [&] {
      temp = steps > 1 ? t0 * std::pow(t1 / t0, (double)step / (double)(steps - 1)) : t0;
      if (cooling) temp_most = std::min(temp_most, temp * SLACK);
    };
    // the proposal by bounds of the loss's increase
    enum { REFUSED, TAKEN, OPEN };
    auto decide = [&]() __attribute__((always_inline)) {
      const double slack = 1.001 * (sum_err + loss_err + 4.0 * ULP * (std::fabs(sum) + std::fabs(loss)));
      const double least = sum - loss - slack, most = sum - loss + slack;
      if (most <= 0.0) return TAKEN;
      if (!(least > 0.0)) return OPEN;
      if (u < 0.0) draw();
      if (u > 0.0 && least > 40.0 * temp_most) return REFUSED;  // u is at least ULP > e^-37
      if (temp == 0.0) heat();
      if (u >= std::exp(-least / temp) * SLACK) return REFUSED;
      return u * SLACK < std::exp(-most / temp) ? TAKEN : OPEN;
    };
    auto verdict = OPEN;
    if (screened) {
      sum = loops.screen(Lf.p, rows, S, k_drop, w);
      sum_err = screen_err;
      verdict = decide();
      credit = std::min(credit + (verdict == OPEN ? -1 : 1), MOST_CREDIT);
    }
    if (finite && verdict == OPEN) {
      const double mass = loops.losses(P.L.p, rows, S, k_drop, w, nullptr, &sum);
      // either order is within (B - 1) ULP of the sum of the |tok| of the real sum, to first order
      sum_err = (2.0 * B + 8.0) * ULP * mass;
      verdict = decide();
      if (verdict == OPEN && loss_err > 4.0 * sum_err) {  // the current loss is what makes the bounds wide
        loss = ordered(none);
        loss_err = 0.0;
        exact = true;
        credit -= ORDERED_COST;
        verdict = decide();
      }
    }
    screened = screened && credit > 0;
    if (verdict == REFUSED) continue;
    const bool sure = verdict == TAKEN;
    bool take = sure;
    if (!sure) {
      if (!exact) loss = ordered(none);
      exact = true;
      loss_err = 0.0;
      sum = ordered(w);
      sum_err = 0.0;
      const double delta = sum - loss;
      take = delta <= 0.0;
      if (!take) {
        if (u < 0.0) draw();
        if (temp == 0.0) heat();
        take = u < std::exp(-delta / temp);
      }
    }
    if (!take) continue;
    loops.apply(P.L.p, screened ? Lf.p : nullptr, rows, w);
    group_of[i] = gj;
    group_of[j] = gi;
    loss = sum;
    loss_err = sum_err;
    exact = !sure;
  }
  if (!exact) loss = ordered(none);
  return loss;
}

}  // namespace

extern "C" int moe_prism_partition_anneal(int32_t B, int32_t C, int32_t S, int32_t k_in,
                                          const float* A, int32_t* group_of, int64_t steps,
                                          double t0, double t1, uint64_t seed, double* loss_out) {
  if (!args_ok(B, C, S, A, group_of) || k_in < 0 || k_in > S || steps < 0 || !(t0 > 0.0) ||
      !(t1 > 0.0) || !partition_ok(C, S, group_of))
    return MOE_PRISM_ERR_INVALID_ARG;
  const double loss = anneal(pick_loops(), B, C, S, k_in, A, group_of, steps, t0, t1, seed);
  if (loss_out) *loss_out = loss;
  return MOE_PRISM_OK;
}
#endif
