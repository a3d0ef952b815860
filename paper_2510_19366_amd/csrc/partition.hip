// Partition solver (Sec. 3.2.1, "Partition Optimization Solver"; objective Eq. 4).  Host code
// only, offline: splits an expert's C intermediate neurons into S equal groups so that each
// calibration token's activation mass concentrates in few groups.  Greedy initialiser by
// calibration-wide L1 norm, then simulated annealing over swaps between groups.
#ifndef __HIP_DEVICE_COMPILE__  // nothing here is for the device pass of the compiler
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
// Measured for 256 tokens, 768 neurons, S = 4: 4.1 us a proposal with one sort per token, 0.4 us now.
constexpr int V = 8;
typedef double vd __attribute__((vector_size(V * sizeof(double))));
typedef float vf __attribute__((vector_size(V * sizeof(float))));
constexpr int MAX_SUB = 64;

#define MP_INLINE inline __attribute__((always_inline))

MP_INLINE void order(vd& a, vd& b) {
  const vd lo = b < a ? b : a, hi = b < a ? a : b;
  a = lo;
  b = hi;
}
// Batcher's odd-even merge sort of S vectors (S = 0: of n)
template <int S>
MP_INLINE void sort_vectors(vd* v, int n) {
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

// One proposal: neurons of |A| columns ci, cj move between groups gi and gj, whose sums become ri, rj.
struct Swap {
  const float *ci, *cj;
  int gi, gj;
  double *ri, *rj;
};
// tok[b] = sum of the k smallest group sums of token b after the swap (ci == nullptr: as they are)
template <int S>
MP_INLINE void swap_losses_t(const double* L, int Bp, int n, int k, const Swap& w, double* tok) {
  const int m = S > 0 ? S : n;
  const double* row[S > 0 ? S : MAX_SUB];
  for (int g = 0; g < m; ++g) row[g] = L + (size_t)g * Bp;
  if (w.ci != nullptr) {
    const double *li = row[w.gi], *lj = row[w.gj];
    for (int b = 0; b < Bp; b += V) {
      const vd ai = __builtin_convertvector(*reinterpret_cast<const vf*>(w.ci + b), vd);
      const vd aj = __builtin_convertvector(*reinterpret_cast<const vf*>(w.cj + b), vd);
      *reinterpret_cast<vd*>(w.ri + b) = *reinterpret_cast<const vd*>(li + b) - ai + aj;
      *reinterpret_cast<vd*>(w.rj + b) = *reinterpret_cast<const vd*>(lj + b) - aj + ai;
    }
    row[w.gi] = w.ri;
    row[w.gj] = w.rj;
  }
  vd v[S > 0 ? S : MAX_SUB];
  for (int b = 0; b < Bp; b += V) {
    for (int g = 0; g < m; ++g) v[g] = *reinterpret_cast<const vd*>(row[g] + b);
    sort_vectors<S>(v, n);
    vd s = {};
    for (int i = 0; i < k; ++i) s += v[i];
    *reinterpret_cast<vd*>(tok + b) = s;
  }
}
MP_INLINE void swap_losses_any(const double* L, int Bp, int S, int k, const Swap& w, double* tok) {
  switch (S) {
    case 2: return swap_losses_t<2>(L, Bp, S, k, w, tok);
    case 4: return swap_losses_t<4>(L, Bp, S, k, w, tok);
    case 8: return swap_losses_t<8>(L, Bp, S, k, w, tok);
    default: return swap_losses_t<0>(L, Bp, S, k, w, tok);
  }
}
__attribute__((target("avx512f"))) void swap_losses_512(const double* L, int Bp, int S, int k, const Swap& w, double* tok) {
  swap_losses_any(L, Bp, S, k, w, tok);
}
__attribute__((target("avx2"))) void swap_losses_256(const double* L, int Bp, int S, int k, const Swap& w, double* tok) {
  swap_losses_any(L, Bp, S, k, w, tok);
}
void swap_losses_128(const double* L, int Bp, int S, int k, const Swap& w, double* tok) {
  swap_losses_any(L, Bp, S, k, w, tok);
}
typedef void (*SwapLosses)(const double*, int, int, int, const Swap&, double*);
SwapLosses pick_swap_losses() {
  __builtin_cpu_init();
  if (__builtin_cpu_supports("avx512f")) return swap_losses_512;
  if (__builtin_cpu_supports("avx2")) return swap_losses_256;
  return swap_losses_128;
}

// memory for vectors of 8 doubles
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
  int B, C, S, Bp;
  Aligned<float> cols;   // [C][Bp]
  Aligned<double> L;     // [S][Bp]: neurons added in ascending index order
  Problem(int B_, int C_, int S_, const float* A, const int32_t* g)
      : B(B_), C(C_), S(S_), Bp((B_ + V - 1) / V * V), cols((size_t)C_ * Bp), L((size_t)S_ * Bp) {
    constexpr int TB = 16, TC = 64;  // tiles of the transposition
    for (int b0 = 0; b0 < B; b0 += TB)
      for (int c0 = 0; c0 < C; c0 += TC)
        for (int c = c0; c < std::min(C, c0 + TC); ++c)
          for (int b = b0; b < std::min(B, b0 + TB); ++b) cols.p[(size_t)c * Bp + b] = std::fabs(A[(size_t)b * C + c]);
    for (int c = 0; c < C; ++c) {
      const float* a = column(c);
      double* l = L.p + (size_t)g[c] * Bp;
      for (int b = 0; b < Bp; ++b) l[b] += (double)a[b];
    }
  }
  const float* column(int c) const { return cols.p + (size_t)c * Bp; }
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
  const Problem P(B, C, S, A, group_of);
  Aligned<double> tok(P.Bp);
  pick_swap_losses()(P.L.p, P.Bp, S, S - k_in, Swap{nullptr, nullptr, 0, 0, nullptr, nullptr}, tok.p);
  double total = 0.0;
  for (int b = 0; b < B; ++b) total += tok.p[b];
  *loss = total;
  return MOE_PRISM_OK;
}

extern "C" int moe_prism_partition_anneal(int32_t B, int32_t C, int32_t S, int32_t k_in,
                                          const float* A, int32_t* group_of, int64_t steps,
                                          double t0, double t1, uint64_t seed, double* loss_out) {
  if (!args_ok(B, C, S, A, group_of) || k_in < 0 || k_in > S || steps < 0 || !(t0 > 0.0) ||
      !(t1 > 0.0) || !partition_ok(C, S, group_of))
    return MOE_PRISM_ERR_INVALID_ARG;
  const int k_drop = S - k_in;
  Problem P(B, C, S, A, group_of);
  const SwapLosses losses = pick_swap_losses();
  const int Bp = P.Bp;
  // Proposals are numbered, so the next few can be evaluated against the current partition before
  // it is known whether the one before them is taken: rejections leave it as it is, and behind an
  // acceptance the rest are evaluated again.  It pays because the tokens' losses are added up in
  // order, one long chain of additions per proposal: WAYS chains run side by side.  How many are
  // tried follows the rejections seen.
  constexpr int WAYS = 4;
  Aligned<double> tok((size_t)WAYS * Bp), moved((size_t)WAYS * 2 * Bp);
  losses(P.L.p, Bp, S, k_drop, Swap{nullptr, nullptr, 0, 0, nullptr, nullptr}, tok.p);
  double loss = 0.0;
  for (int b = 0; b < B; ++b) loss += tok.p[b];
  int64_t step = 0;
  int ways = 1;
  while (step < steps) {
    int64_t at[WAYS];
    int ni[WAYS], nj[WAYS], n = 0;
    Swap w[WAYS];
    int64_t next = step;
    for (; next < steps && n < ways; ++next) {
      const int i = (int)(splitmix64(seed + 3ull * (uint64_t)next) % (uint64_t)C);
      const int j = (int)(splitmix64(seed + 3ull * (uint64_t)next + 1ull) % (uint64_t)C);
      if (group_of[i] == group_of[j]) continue;
      at[n] = next;
      ni[n] = i;
      nj[n] = j;
      w[n] = Swap{P.column(i), P.column(j), group_of[i], group_of[j], moved.p + (size_t)(2 * n) * Bp,
                  moved.p + (size_t)(2 * n + 1) * Bp};
      ++n;
    }
    double sum[WAYS] = {0.0, 0.0, 0.0, 0.0};
    for (int k = 0; k < n; ++k) losses(P.L.p, Bp, S, k_drop, w[k], tok.p + (size_t)k * Bp);
    if (n == 1) {
      for (int b = 0; b < B; ++b) sum[0] += tok.p[b];
    } else {
      for (int b = 0; b < B; ++b)
        for (int k = 0; k < WAYS; ++k) sum[k] += tok.p[(size_t)k * Bp + b];  // k >= n: not looked at
    }
    bool taken = false;
    for (int k = 0; k < n && !taken; ++k) {
      const double delta = sum[k] - loss;
      bool take = delta <= 0.0;
      if (!take) {
        const uint64_t r2 = splitmix64(seed + 3ull * (uint64_t)at[k] + 2ull);
        const double temp = steps > 1 ? t0 * std::pow(t1 / t0, (double)at[k] / (double)(steps - 1)) : t0;
        const double u = (double)(r2 >> 11) * (1.0 / 9007199254740992.0);
        take = u < std::exp(-delta / temp);
      }
      if (!take) continue;
      std::copy(w[k].ri, w[k].ri + Bp, P.L.p + (size_t)w[k].gi * Bp);
      std::copy(w[k].rj, w[k].rj + Bp, P.L.p + (size_t)w[k].gj * Bp);
      group_of[ni[k]] = w[k].gj;
      group_of[nj[k]] = w[k].gi;
      loss = sum[k];
      step = at[k] + 1;
      taken = true;
    }
    if (!taken) step = next;
    ways = taken ? 1 : std::min(WAYS, 2 * ways);
  }
  if (loss_out) *loss_out = loss;
  return MOE_PRISM_OK;
}
#endif
