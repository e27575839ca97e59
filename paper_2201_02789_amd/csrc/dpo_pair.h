// The symmetry check's keyed mix of an entry's two ids.  Plain C++ but for the
// function qualifiers, so that its errors can be measured on the CPU too, with
// smaller words.
#pragma once
#include <stdint.h>

#include <type_traits>

namespace dpo {

constexpr int PAIR_KEYS = 4;

struct PairKey {
  uint32_t k[PAIR_KEYS];
};

// +-h of the entry (u, v) with the order of its ids as the sign, added to `sum`;
// nothing for a loop.  Both ids come with k[0] added (modulo the word, where any
// order will do).  W is a word, D two of them.  h depends on the smaller and the
// larger of them, A and B:
//   x = A * B + (B : A)
//   y = a * b + (b : a)    a, b: x's low half under a key, its halves folded
//   h = c * d              c, d: y's halves under a key each, made odd
// Adding the factors to the product keeps them where the other factor is 0 or
// another value that the product says little of, and costs nothing (one
// multiply-add).  h is odd: no number of unpaired copies of one entry, and no odd
// number of unpaired entries, sums to zero.
//
// Shares of the keys under which sets of 2 to 8 unpaired entries in neighbouring
// rows and columns sum to zero, with words of 8 and of 16 bits: two entries 2^-11
// and 2^-25, runs of four or eight in one row or column 2^-12 and 2^-24,
// rectangles, chains of one-way entries and hubs 2^-13 and below 2^-26.
// Extrapolated to 32 bits that is some 2^-47 for the worst of them.  (Of a product
// c * d of the bare halves of A * B, either of them possibly zero, 2^-31 for a
// single entry.)
template <typename W, typename D>
__host__ __device__ __forceinline__ D add_pair(D sum, W u, W v, const W (&k)[PAIR_KEYS]) {
  using S = std::make_signed_t<W>;
  using SD = std::make_signed_t<D>;
  constexpr int N = 8 * sizeof(W);
  const W A = u < v ? u : v, B = u < v ? v : u;
  const D x = (D)((D)A * B + ((D)B << N | A));
  const W a = (W)((W)x ^ k[1]), b = (W)((W)(x >> N) ^ (W)x);
  const D y = (D)((D)a * b + ((D)b << N | a));
  S c = (S)(((W)y ^ k[2]) | 1u), d = (S)(((W)(y >> N) ^ k[3]) | 1u);
  c = u > v ? (S)-c : c;  // (odd: never the one value without a negative)
  c = u == v ? (S)0 : c;
  return (D)(sum + (D)((SD)c * (SD)d));
}

}  // namespace dpo
