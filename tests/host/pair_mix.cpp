// Errors of the symmetry check's mix: shares of keys under which sets of
// unpaired entries sum to zero.  Prints one line per measurement:
// <word bits> <chosen key or -> <set> <misses> <keys tried>
#include <cstdio>
#include <string>
#include <vector>

#define __host__
#define __device__
#define __forceinline__ inline
#include "dpo_pair.h"

struct Entry {
  uint32_t u, v;
};
struct Set {
  std::string name;
  std::vector<Entry> e;
};

// q: an id that others lie near
static std::vector<Set> sets(uint32_t q) {
  return {{"single", {{5, q}}},
          {"twice", {{5, q}, {5, q}}},
          {"row2", {{5, q}, {q + 1, 5}}},
          {"row2far", {{5, q}, {q + 50, 5}}},
          {"col2", {{5, q}, {q, 6}}},
          {"col2far", {{2, q}, {q, 33}}},
          {"shift2", {{5, q}, {q - 1, 6}}},
          {"row4", {{5, q}, {q + 1, 5}, {q + 2, 5}, {5, q + 3}}},
          {"col4", {{q, q + 60}, {q + 60, q + 1}, {q + 60, q + 2}, {q + 3, q + 60}}},
          {"shift4", {{5, q}, {q - 1, 6}, {q + 4, 10}, {9, q + 5}}},
          {"rect", {{5, q}, {q + 1, 5}, {q, 6}, {6, q + 1}}},
          {"rect2", {{5, q}, {q + 2, 5}, {q, 7}, {7, q + 2}}},
          {"row8", {{5, q}, {q + 1, 5}, {q + 2, 5}, {5, q + 3}, {q + 4, 5}, {5, q + 5}, {5, q + 6}, {q + 7, 5}}},
          {"cycle3", {{5, q}, {q, q + 50}, {q + 50, 5}}},
          {"cycle4", {{5, q}, {q, q + 50}, {q + 50, q + 51}, {q + 51, 5}}},
          {"hub", {{5, q}, {5, q + 1}, {q + 2, 5}, {q + 3, 5}}}};
}

static uint64_t next(uint64_t& s) {
  uint64_t z = (s += 0x9E3779B97F4A7C15ull);
  z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
  z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
  return z ^ (z >> 31);
}

template <typename W, typename D>
static void measure(const Set& s, long keys, const char* chosen, int at, uint32_t value) {
  uint64_t seed = 1;
  long miss = 0, paired = 0;
  for (long i = 0; i < keys; ++i) {
    W k[dpo::PAIR_KEYS];
    for (int j = 0; j < dpo::PAIR_KEYS; ++j) k[j] = (W)(next(seed) >> 20);
    if (at >= 0) k[at] = (W)value;
    D sum = 0, both = 0;
    for (const Entry& e : s.e) {
      const W u = (W)(e.u + k[0]), v = (W)(e.v + k[0]);
      sum = dpo::add_pair<W, D>(sum, u, v, k);
      both = dpo::add_pair<W, D>(dpo::add_pair<W, D>(both, u, v, k), v, u, k);
      both = dpo::add_pair<W, D>(both, u, u, k);  // a loop
    }
    miss += sum == 0;
    paired += both != 0;
  }
  if (paired) printf("PAIRED %s\n", s.name.c_str());
  printf("%zu %s %s %ld %ld\n", 8 * sizeof(W), chosen, s.name.c_str(), miss, keys);
}

int main() {
  for (const Set& s : sets(60)) measure<uint8_t, uint16_t>(s, 1l << 20, "-", -1, 0);
  for (const Set& s : sets(5000)) measure<uint16_t, uint32_t>(s, 1l << 22, "-", -1, 0);
  for (const Set& s : sets(5000)) {
    // a factor of the first product 0, 1 or -1: each has a probability of 2^-32
    for (uint32_t id : {5u, 5000u})
      for (uint32_t f : {0u, 1u, ~0u}) {
        const std::string c = std::to_string(id) + "->" + std::to_string((int)f);
        measure<uint32_t, uint64_t>(s, 1l << 18, c.c_str(), 0, f - id);
      }
    for (int at = 1; at < dpo::PAIR_KEYS; ++at) measure<uint32_t, uint64_t>(s, 1l << 16, "0", at, 0);
  }
}
