// What the annealer spends on a problem, counted in vectors of 64 bytes, against what it spends with the binary64 sums alone.
#include "../paper_2510_19366_amd/csrc/partition.hip"

#include <cstdio>
#include <random>

namespace {

long g_vectors, g_screens, g_passes, g_longest;
bool g_undecided;  // the binary32 sums tell nothing, so that they are given up and the rest is binary64 alone

double counted_losses(const double* L, Span rows, int S, int k, const Swap& w, double* tok, double* plain) {
  g_vectors += (long)S * rows.n64 / V * (tok != nullptr ? 2 : 1);  // (as long again for the chain of additions that follows)
  g_passes += 1;
  g_longest = std::max(g_longest, (long)rows.n64);
  return pick_loops().losses(L, rows, S, k, w, tok, plain);
}
double counted_screen(const float* Lf, Span rows, int S, int k, const Swap& w) {
  if (g_undecided) return std::nan("");
  g_vectors += (long)S * rows.stride / VF;
  g_screens += 1;
  return pick_loops().screen(Lf, rows, S, k, w);
}

struct Result {
  std::vector<int32_t> groups;
  double loss;
  long vectors, screens, passes, longest;
};
struct Case {
  int B, C, S, k_in;
  double t0, t1;
};
Result solve(const Case& c, const std::vector<float>& A, bool undecided) {
  g_vectors = g_screens = g_passes = g_longest = 0;
  g_undecided = undecided;
  const Loops counted{counted_losses, counted_screen, pick_loops().add_column, pick_loops().apply};
  Result r{std::vector<int32_t>(c.C), 0.0, 0, 0, 0, 0};
  for (int n = 0; n < c.C; ++n) r.groups[n] = n % c.S;
  r.loss = anneal(counted, c.B, c.C, c.S, c.k_in, A.data(), r.groups.data(), 1500, c.t0, c.t1, 7);
  r.vectors = g_vectors, r.screens = g_screens, r.passes = g_passes, r.longest = g_longest;
  return r;
}

}  // namespace

int main() {
  std::vector<Case> cases;
  for (int B : {1, 2, 7, 8, 9, 16, 17, 24, 25, 64, 100, 256})
    for (int S : {2, 4, 8, 16})
      for (int k_in : {1, S / 2, S - 1})
        for (double t : {0.01, 1.0, 20.0})
          for (bool cooling : {false, true}) cases.push_back({B, 96, S, k_in, t, cooling ? 1e-3 * t : t});
  // many tokens, all of whose sum the binary32 bound grows with
  for (int k_in : {1, 4, 7})
    for (double t : {0.01, 20.0, 200.0}) cases.push_back({2048, 1408, 8, k_in, t, t}), cases.push_back({4096, 512, 4, k_in / 2, t, t});
  int bad = 0;
  for (const Case& c : cases) {
    std::mt19937 rng(c.B + c.S);
    std::normal_distribution<float> normal;
    std::vector<int> block(c.C);
    for (int& b : block) b = rng() % c.S;
    std::vector<float> A((size_t)c.B * c.C);
    for (int b = 0; b < c.B; ++b) {
      const int hot = rng() % c.S;
      for (int n = 0; n < c.C; ++n) A[(size_t)b * c.C + n] = normal(rng) * (block[n] == hot ? 1.0f : 0.1f);
    }
    const Result plain = solve(c, A, true), r = solve(c, A, false);
    const char* wrong = nullptr;
    if (r.groups != plain.groups || r.loss != plain.loss) wrong = "other result";
    if (c.B <= V && r.screens != 0) wrong = "binary32 sums where one vector has all tokens";
    if (r.longest != (c.B + V - 1) / V * V) wrong = "binary64 sums of tokens that are not there";
    // what trying costs before it is given up: some 16 sums of half the vectors, or ordered sums that go with a few of them
    if (r.vectors > plain.vectors + plain.vectors / 50 + 12L * c.S * (c.B + V - 1) / V) wrong = "more work than without binary32 sums";
    std::printf("%.3f %ld B %d C %d S %d k_in %d t %g..%g: %s (%ld passes, %ld; %ld screens)\n", (double)r.vectors / plain.vectors, (r.vectors - plain.vectors) * V / (c.S * c.B),
                c.B, c.C, c.S, c.k_in, c.t0, c.t1, wrong ? wrong : "ok", r.passes, plain.passes, r.screens);
    bad += wrong != nullptr;
  }
  return bad != 0;
}
