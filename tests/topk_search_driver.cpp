// The search of the top-k kernel on the host: picks against a sort, and the number of steps it takes on
// rows with masks, infinities, NaN, equal and clustered logits.  Prints the largest number of steps by kind of row.
#include <algorithm>
#include <cfloat>
#include <cmath>
#include <cstdio>
#include <cstdlib>
#include <numeric>
#include <random>
#include <vector>

#include "../paper_2510_19366_amd/csrc/topk_search.h"

using namespace mp;

int main() {
  std::mt19937 gen(7);
  std::normal_distribution<float> normal(0.0f, 1.0f);
  const char* kinds[] = {"normal", "one masked", "half masked", "all but k masked", "half -inf", "lognormal", "small",
                         "few values", "all equal", "nan", "clustered"};
  for (int kind = 0; kind < 11; ++kind) {
    int most = 0;
    for (int E : {5, 64, 100, 512})
      for (int k : {1, 2, 3, 4, 5, 8, 9, 16, 17, 32, 33, 64, 65, 200})
        for (int rep = 0; rep < 40 && k <= E; ++rep) {
          std::vector<float> v(E);
          for (int i = 0; i < E; ++i) {
            float f = normal(gen);
            if ((kind == 1 && i == 3) || (kind == 2 && i % 2) || (kind == 3 && i >= k)) f = -FLT_MAX;
            if (kind == 4 && i % 2) f = -INFINITY;
            if (kind == 5) f = std::exp(8 * f);
            if (kind == 6) f *= 1e-38f;
            if (kind == 7) f = (float[]){0.0f, -0.0f, 1.0f, -1e-30f, INFINITY, -INFINITY}[gen() % 6];
            if (kind == 8) f = -2.5f;
            if (kind == 9 && i % 7 == 0) f = bits_float(i % 2 ? -1 : INT32_MAX);
            if (kind == 10) f = 1e3f + 1e-4f * f;
            v[i] = f;
          }
          std::vector<int> key(E);
          for (int i = 0; i < E; ++i) key[i] = topk_key(v[i]);
          // the kernel's lower bound: the smallest of the sets' best keys
          int sets = 64;
          while (sets > 4 && sets >= 4 * k) sets /= 2;
          std::vector<int> best(sets, INT32_MIN);
          for (int i = 0; i < E; ++i) best[i % 64 * sets / 64] = std::max(best[i % 64 * sets / 64], key[i]);
          const int lo = k <= 64 ? *std::min_element(best.begin(), best.end()) : INT32_MIN;
          const int hi = *std::max_element(key.begin(), key.end()) + 1;
          int steps = 0;
          const TopkCut cut = topk_cut(lo, hi, k, [](int m) { return m; }, [&](int m) {
            ++steps;
            return (int)std::count_if(key.begin(), key.end(), [&](int x) { return x >= m; });
          });
          most = std::max(most, steps);
          std::vector<int> picks, order(E);
          int rem = cut.rem;
          for (int i = 0; i < E; ++i)
            if (key[i] > cut.thr || (key[i] == cut.thr && rem-- > 0)) picks.push_back(i);
          std::iota(order.begin(), order.end(), 0);
          std::stable_sort(order.begin(), order.end(), [&](int a, int b) { return key[a] > key[b]; });
          order.resize(k);
          std::sort(order.begin(), order.end());
          if (picks != order) {
            std::printf("wrong picks: kind %d E %d k %d rep %d\n", kind, E, k, rep);
            return 1;
          }
        }
    std::printf("%d %s\n", most, kinds[kind]);
  }
  return 0;
}
