// The symmetry check's keyed mix of an entry's two ids.  Plain C++ but for the
// function qualifiers, so that its errors can be measured on the CPU too, with
// smaller words.
#pragma once
#include <stdint.h>

#include <type_traits>

namespace dpo {

constexpr int PAIR_KEYS = 6;

struct PairKey {
  uint32_t k[PAIR_KEYS];
};

// +-h of the entry (u, v) with the order of its ids as the sign, added to `sum`;
// nothing for a loop.  W is a word, D two of them; ids are below half of W's
// range.  h depends on the smaller and the larger id:
//   x = A * B + (B : A)    A, B the ids under a key each
//   y = a * b + (b : a)    a, b from x's low half and from its high half folded
//                          with the low one, under a key each
//   h = c * d              c, d y's halves under a key each, made odd
// Adding the factors to the product keeps them where the other factor is 0 or
// another value that the product says little of; the first of the two additions
// is free (one multiply-add), as is the second.  h is odd: no number of unpaired
// copies of one entry, and no odd number of unpaired entries, sums to zero.
//
// Sets of 2 to 8 unpaired entries in neighbouring rows and columns, as words of
// 8 and 16 bits (shares of the keys that miss them): two entries 2^-11 and 2^-26,
// runs of four in one row 2^-12 and 2^-23, rectangles, chains of one-way entries
// and hubs 2^-13 and below 2^-25: extrapolated to 32 bits, some 2^-46 for the worst
// of them.  (The product c * d of unkept, unfolded halves of A * B that
// this replaces missed one entry in 2^31 and some runs of four as often.)
template <typename W, typename D>
__host__ __device__ __forceinline__ D add_pair(D sum, W u, W v, const W (&k)[PAIR_KEYS]) {
  using S = std::make_signed_t<W>;
  using SD = std::make_signed_t<D>;
  constexpr int N = 8 * sizeof(W);
  const W A = (W)((u < v ? u : v) + k[0]), B = (W)((u < v ? v : u) + k[1]);
  const D x = (D)((D)A * B + ((D)B << N | A));
  const W a = (W)((W)x ^ k[2]), b = (W)((W)(x >> N) ^ (W)x ^ k[3]);
  const D y = (D)((D)a * b + ((D)b << N | a));
  S c = (S)(((W)y ^ k[4]) | 1u), d = (S)(((W)(y >> N) ^ k[5]) | 1u);
  c = u > v ? (S)-c : c;  // (odd: never the one value without a negative)
  c = u == v ? (S)0 : c;
  return (D)(sum + (D)((SD)c * (SD)d));
}

}  // namespace dpo
