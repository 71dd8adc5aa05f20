// Internal: how the row-major kernel cuts A into bands and which addresses it reads (plain constants and
// arithmetic, also built without HIP).
#pragma once
#include <stdint.h>

namespace twg {

constexpr int MK_KC = 768;             // columns of A per band, at most
template <int TM>
constexpr int MK_KC_LONG = TM == 32 ? MK_KC : 512;   // columns per band when K needs several: one block per wave
template <int TM>
constexpr int MK_KB = TM == 64 ? 64 : 128;           // columns of A a wave turns round at a time

// First column of the 16-byte chunk that lane chunk kc of block kb reads in the band that starts at column
// k0.  Chunks past K (their columns are never referenced) repeat the one that holds column K - 1: the last
// row of A may end the caller's buffer there, also where lda is larger.
template <int TM>
constexpr int mk_chunk(int k0, int kb, int kc, int K) {
  const int kg = k0 + kb * MK_KB<TM> + kc * 8, last = (K - 1) & ~7;
  return kg < last ? kg : last;
}

// Byte offset of column kg of a row (0 .. 63) inside a band of rows of lda elements.  WIDE: lda above
// MK_LDA_32, where 32 bits do not hold it.
constexpr int MK_LDA_32 = 1 << 25;
template <bool WIDE>
constexpr auto mk_offset(int row, int lda, int kg) {
  if constexpr (WIDE) return (uint64_t)(uint32_t)row * ((uint32_t)lda * 2u) + (uint32_t)kg * 2u;
  else return (uint32_t)row * ((uint32_t)lda * 2u) + (uint32_t)kg * 2u;
}

}  // namespace twg
