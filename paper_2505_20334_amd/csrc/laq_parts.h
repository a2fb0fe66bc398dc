// How decode attention cuts the caches of a call into parts, a workgroup each.  Plain C++, so that the rule can be checked on the host.
//
// Parts: for three workgroups per compute unit, which is what it holds of most kernels here (110 to 136 registers: three or four)
// and fewer than make the folding long, but no parts shorter than a turn of the workgroup's lane groups; at most DEC_MOST_PARTS of
// one cache, since one workgroup folds them.  The least length with which the call keeps to that, last parts counted too, and a
// cache's parts as even as their steps allow: a fourth workgroup on some compute units, or parts of a few rows beside full ones,
// leave the others idle at the end.  Length from the rows of the call alone, the rest of a cache a part of its own : this, us, 8
// heads: 32 caches of 2048 to 128 rows 36.0 : 31.8; 60 of them 58.0 : 53.7; 90 x 200 27.0 : 15.9; 90 x 2048 159 : 117; fp32, two
// query heads a KV head 455 : 300.  The same with 512, 640, 896, 1024 workgroups: 32 caches of 2048 to 128 rows 1024 32.8; grids of
// 319 calls by rows a part, over 768: 896 and 1024 .88-1.12 (.89-.95 for parts of 128 rows), 640 and 512 .87-1.09.  Shares of one
// length that end in one cache and go on in the next, 768 of them: 34.3, and shares of up to 512 rows .78-.96 of these (a second sum
// to merge, a longer kernel).
//
// Not where that would make parts of more than MOST_OF_EVEN times the rows that each of 768 workgroups has of the call: a few long
// caches among short ones would be read by a few workgroups long after the others have ended.  Then the parts have those rows, however
// many workgroups they make.  The least length : those rows, us, by the ratio of the two, bf16, 8 heads unless said:
//   1.17 32 caches of 2048 to 128 rows 31.8 : 33.4;  1.12 20 of 8192 to 64 (even logarithms) 41.8 : 46.1;  1.22 255 x 1 head 59.0 : 65.4
//   1.45 60 of 2048 to 128 53.7 : 52.5, 120 90.9 : 94.8;  1.69 60 of 8192 to 64 79.7 : 79.4;  1.78 10 x 4096 and 50 x 256 45.0 : 42.9,
//   96 of 2048 to 128 76.7 : 77.2, 4 heads, 200 of them 92.6 : 100.6
//   2.13 20 x 2048 and 90 x 512 69.4 : 70.0;  2.16 4 heads, 150 of 8192 to 64 202 : 151;  2.33 32 heads, 20 of these 57.6 : 53.6
//   2.44 80 of 8192 to 64 132 : 122;  3.4 105 of 2048 to 64 56.7 : 50.8;  3.9 100 of 8192 to 64 203 : 129;  36 one of 32768 and 94 x 64 356 : 39
#ifndef LAQ_PARTS_H
#define LAQ_PARTS_H

#include <stdint.h>

namespace laq {

constexpr long long DEC_WORKGROUPS = 768;
constexpr int DEC_PART_STEP = 64;
constexpr int DEC_MOST_PARTS = 128;
constexpr long long DEC_WHOLE_FROM = 1024;       // with that many workgroups without parts there are no parts
constexpr int MOST_OF_EVEN = 2;

// Rows of each of `parts` parts of a cache (the last one may have less): steps of DEC_PART_STEP, unless it is one part.
constexpr int even_rows(int bk, int parts) {
  const int steps = (bk + DEC_PART_STEP - 1) / DEC_PART_STEP;
  return (steps + parts - 1) / parts * DEC_PART_STEP;
}
// The parts of a cache, as even as their steps allow: at most as many as parts of `limit` rows would be, and never more for a longer limit.
constexpr int parts_of(int bk, int limit) {
  const int steps = (bk + DEC_PART_STEP - 1) / DEC_PART_STEP, each = even_rows(bk, (bk + limit - 1) / limit) / DEC_PART_STEP;
  return (steps + each - 1) / each;
}

inline int longest_cache(int n, int L, const int32_t* budget) {
  int most = 0;
  for (int i = 0; i < n; ++i) most = most > budget[i] ? most : budget[i];
  return most < L ? most : L;
}

// The limit of the parts' rows, before they are evened out and rounded to steps.  columns: workgroups of one part.
inline int limit_of_parts(int n, int L, long long columns, const int32_t* budget) {
  const int most = longest_cache(n, L, budget);
  if (n * columns >= DEC_WHOLE_FROM) return most;
  long long rows = 0;
  for (int i = 0; i < n; ++i) rows += budget[i] < L ? budget[i] : L;
  int even = (int)(rows * columns / DEC_WORKGROUPS / DEC_PART_STEP + 1) * DEC_PART_STEP;
  const int least = (most + DEC_MOST_PARTS - 1) / DEC_MOST_PARTS;
  if (even < least) even = least;
  if (even >= most) return most;
  const long long limit = (long long)even * MOST_OF_EVEN < most ? (long long)even * MOST_OF_EVEN : most;
  const auto fits = [&](int rows_of_a_part) {
    long long parts = 0;
    for (int i = 0; i < n; ++i) parts += parts_of(budget[i] < L ? budget[i] : L, rows_of_a_part);
    return parts * columns <= DEC_WORKGROUPS;
  };
  // whole caches that are more workgroups than that anyway
  if (n * columns > DEC_WORKGROUPS) return limit == most ? most : even;
  // Longer parts are never more, so the least number of steps is found by halving (one by one 8.6 us of the host's time for 96
  // caches of 2048 to 128 rows, so 1.8; a call asks up to three times).
  int few = 0, many = (int)((limit - even) / DEC_PART_STEP) + 1;      // (that many steps: beyond the limit)
  while (few < many) {
    const int mid = (few + many) / 2;
    if (fits(even + mid * DEC_PART_STEP)) many = mid;
    else few = mid + 1;
  }
  const long long part = even + (long long)many * DEC_PART_STEP;
  if (part > limit) return limit == most ? most : even;               // (whole caches fit)
  return (int)part;
}

}  // namespace laq

#endif  // LAQ_PARTS_H
