// The rules by which the BATCHED schedule chooses the kernel of the ungapped extension
// (plain C++).  They count words, not codes: a bank of fragments is more than half
// separators, and its keys have as many fewer occurrences.
#pragma once

#include <stdint.h>

namespace plast {

constexpr double kRouteKeys = 8800;   // seed keys
constexpr int64_t kRoutePad = 20;     // separators before, between and after the sequences

// Words of a bank whose sequences have 3 letters or more (a shorter one has none, as if
// it were a little longer).
inline double bank_words(int64_t n_padded, int32_t n_seqs) {
  const int64_t w = n_padded - kRoutePad * ((int64_t)n_seqs + 1) - 3 * (int64_t)n_seqs;
  return w > 0 ? (double)w : 0.0;
}

// Whether, in the kernel of an item per wavefront, each XCD takes the columns of its
// eighth of bank b, as the bank's codes say: from the size that a few L2s hold (100 x
// 10,000 proteins, 3.2M codes, 103 us, shared 126; 100 x 30,000, 9.5M, 216 and 198; 30 x
// 300,000 fragments, 10.8M, 80 and 71), and while an eighth about fits one (3 x 100,000,
// 32M, 112 and 88; 3 x 1M 1126 and 1398).  A launch of fewer workgroups than XCDs would
// have none for some eighths.
constexpr int64_t kXcdMinCodes = 4500000, kXcdMaxCodes = 64000000;
constexpr int kXcds = 8;
inline bool columns_shared(int64_t codes2, int64_t workgroups) {
  return codes2 >= kXcdMinCodes && codes2 <= kXcdMaxCodes && workgroups >= kXcds;
}

enum class Route {
  kWave,    // an item per wavefront
  kGroup,   // an item per workgroup, on the VALU
  kMatrix,  // an item per workgroup, on the matrix cores
};

// Whether a threshold is so low that a quarter and more of ordinary pairs are hits: below
// three and a half times the matrix's mean score of equal letters (20.3 for BLOSUM62;
// equal: their sum over the 20 letters).
inline bool low_threshold(int32_t s1, int equal) { return 40 * (int64_t)s1 < 7 * (int64_t)equal; }

// words1 and words2: of banks a and b; codes2: of bank b; matrix: the matrix cores hold
// the scores; low: of the threshold.
//
// An item per wavefront where there are few pairs in all, as the product of the words
// says, and more of them where a key has few columns (us there, and on a workgroup per
// item): 30 x 2000 proteins 28 and 72, 200 x 2000 63 and 162, 400 x 5000 130 and 216, 200 x
// 10,000 141 and 202, 1000 x 2000 176 and 313; 1000 x 5000 266, and 264 on the matrix cores;
// and, whatever the pairs, where a key has few rows: against 100,000 proteins,
// 3.1 rows a key 523 us, 651 by workgroup and 666 on the matrix cores; 6.9 739, 785
// and 818; 10.0 953, 954 and 932; against 45,000 401, 400 and 436, and 496, 482 and 498.
// With a bank b that the L2s do not hold, 3.1 rows against 300,000 2154, 2375 and 2290,
// 6.9 2544, 2623 and 2448.  The same by words with fragments as bank a: 4.6 rows against
// 60,000 proteins 371, 410 and 455, 9.2 566, 565 and 575.
//
// Not at a low threshold, unless there are few pairs or rows: a wavefront there writes its
// hits out by the 256, each time with an atomic on their one counter (200 x 10,000
// proteins at thresholds of 20, 16 and 12: 443, 941 and 1252 us, by workgroup 419, 570 and
// 645; 200 x 2000 at 12 360 and 249; 1000 x 2000 at 16 1061, 489 and on the matrix cores
// 601; but 30 x 100,000, where a workgroup's tile has no more rows, 2029 and 3044).
//
// The matrix cores from 12 rows a key on (against 30,000 proteins 10.0 rows 360 and 378,
// 11.9 396 and 397, 16 484 and 456), and from fewer where bank b is large and its windows
// are the bound, which the 64 rows of an item share (10.0 rows against 80,000 proteins
// 773 and 766, 150,000 1421 and 1365).
constexpr double kWavePairs = 2.15e11, kWaveMorePairs = 3.4e11, kWaveMoreCols = 185;
constexpr double kFewRows = 8, kFewRowsLarge = 4.5, kManyRows = 12;
constexpr int64_t kLargeCodes = 24000000;
constexpr double kLowRows = 4, kLowPairs = 2e10;
inline Route ungapped_route(double words1, double words2, int64_t codes2, bool matrix, bool low) {
  const double rows = words1 / kRouteKeys, cols = words2 / kRouteKeys, pairs = words1 * words2;
  const double few = codes2 > kXcdMaxCodes ? kFewRowsLarge : kFewRows;
  if (rows < few || pairs <= kWavePairs || (pairs <= kWaveMorePairs && cols < kWaveMoreCols))
    return low && rows >= kLowRows && pairs >= kLowPairs ? Route::kGroup : Route::kWave;
  return matrix && (rows >= kManyRows || codes2 >= kLargeCodes) ? Route::kMatrix : Route::kGroup;
}

}  // namespace plast
