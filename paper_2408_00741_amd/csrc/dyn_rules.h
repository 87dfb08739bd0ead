// Rules of the host side that depend on sizes and tables only, in plain C++: tests/test_rules.py compiles them on the CPU.
#ifndef DYN_RULES_H_
#define DYN_RULES_H_

#include <algorithm>
#include <cstddef>
#include <cstdint>

// Evenly spaced load points: buckets a little narrower than the spacing, of which every point opens its own and fills at most the first
// 2^-10 (the points' own roundings and the 2^-40 take far less).  A product by a constant is monotone, so only loads in that part of a
// bucket can lie below its point: one wave in sixteen meets one.  Points anywhere in their buckets do as well for the result, but with points 0.3 to 0.9 of a
// spacing late most loads are asked twice; with the buckets' index instead they cost what room it takes in LDS (10 bytes a bucket, three
// buckets to the least spacing).  us a call by the index, by the even form (36 000 cells; 12 ticks; mixed pools; evaluation; hierarchy):
//   64 points, 0.3 late, 269 buckets:   464 572   239 291   134 141    97 101       33 points, 0.9 late, 960 buckets:  461 544   235 265   153 160    96 100
//   64 points, 0.8 late, 945 buckets:   522 576   263 291   133 140    98 100       33 points, 0.95, 1920 buckets:     524 544   260 265   158 160   107 100
//   64 points, 0.9 late, 1890 buckets:  586 577   296 291   140 138   109 100       64 points, 0.95, 3780 buckets:     944 577   379 292   154 137   112 100
//   128 points, 0.6 late, 952 buckets:  700 824   314 406   191 180   102 106      128 points, 0.8, 1905 buckets:      942 826   402 406   198 179   112 105
// So beyond DYN_EVEN_BUCKETS buckets the points may lie anywhere in theirs.  Returns buckets per unit of the load axis, 0 where the points do not lie so.
#define DYN_EVEN_BUCKETS 1500
inline double dyn_even_scale(const double* rho, int32_t n_rho, int32_t n_bucket /* of the index */) {
  const double scale = (double)(n_rho - 1) / rho[n_rho - 1] * (1.0 + 0x1p-40);
  const double late = n_bucket > DYN_EVEN_BUCKETS ? 1.0 : 0x1p-10;
  for (int32_t q = 1; q < n_rho; ++q) {
    const double x = rho[q] * scale - (double)q;
    if (!(x >= 0.0 && x < late)) return 0.0;
  }
  return scale;
}

#define DYN_MAX_WIN_PER_BLOCK 32  // windows one block of the space kernel walks

#define DYN_SPACE_IN_FLIGHT 224   // (wave, window) pairs of a compute unit

// Windows one block of the evaluation kernel walks.  Long runs amortise the staging of the table rows in LDS, but
// the blocks a chip holds at a time then write that many more separate streams; and no run should leave the chip with fewer than ~8192
// blocks in all.  What decides is how many rows of 64 results a compute unit writes over a block's life, its resident waves times the windows of a block: about
// 224.  us by windows a block, even load points (GB of results; candidates in tiles of, resident waves):
//   2 GB, 256, 32 waves:  6 365, 7 366, 8 385, 10 403      2 GB, 256, 24 waves:  6 370, 7 365, 8 365, 9 376, 10 395
//   4 GB, 256, 32 waves:  6 708, 7 700, 8 700, 10 744      4 GB, 256, 24 waves:  6 725, 8 691, 9 694, 10 700, 12 738
//   8 GB, 256, 32 waves:  6 1391, 7 1361, 8 1368, 10 1435  10.3 GB and 10^8 requests, 32 waves:  6 2034, 7 1997, 8 2054, 10 2220
//   4 GB, 192, 24 waves:  6 802, 8 744, 9 740, 10 783      1 GB, 192, 24 waves:  6 223, 8 211, 9 216, 10 225
//   4 GB, 128, 22 waves:  5 887, 8 760, 9 755, 10 737, 12 715    4 GB, 64, 20 waves:  4 1002, 8 789, 9 765, 10 748, 12 750
// The former rule counted 64 rows of blocks a compute unit whatever their width: 5 and 4 windows in the last line, and with uneven points (64 wide, 10 waves
// beside their bucket index) 2 GB in 1218 us, 634 now.
// How much a block stages moves that: up to 7 table values a thread leave little to amortise, more than 14 much.  Over 50 traces of 300 000
// requests (13 000 to 313 000 tiles of cells, 0.4 to 40 million results) at 1 to 16 windows, the call is 8.8 % above its best without these two
// lines, 6.4 % with them.  Up to 7, 4 windows in place of 5 to 8: 128 us 121, 113 100, 86 76, 79 76, 64 56, 139 127, 107 105, 58 58 and 61 66 (50 400
// cells of 1152 candidates, beyond 250 000 tiles, 314 at 6, 338); beyond 14, 8 in place of 4: 107 80, 77 66, 71 63, 79 75, 76 74 and 79 81 (the fewest
// tiles 91 000; 31 800 at 4 and 6 windows 66, 61).  Between, 4 in place of 6 is as often better as worse: 237 195, 341 317, 94 89, 125 123, 68 73, 241 279; the
// one-day workload stages 12.  Blocks that stage nothing keep the first rule.  dyn_eval_tune replaces the rule's value by a measured one.
inline int32_t dyn_space_windows(int64_t cell_tiles, int32_t tile, int64_t staged /* table values of a block */, int32_t waves /* of a compute unit */) {
  int64_t w = std::max<int64_t>(1, std::min<int64_t>(DYN_MAX_WIN_PER_BLOCK, (cell_tiles + 8191) / 8192));
  if (waves > 0) w = std::min<int64_t>(w, std::max<int64_t>(4, DYN_SPACE_IN_FLIGHT / waves));
  if (staged > 0 && staged <= 7 * (int64_t)tile && cell_tiles <= 250000) w = std::min<int64_t>(w, 4);
  else if (staged > 14 * (int64_t)tile && cell_tiles >= 8 * 4096) w = std::max<int64_t>(w, 8);   // at least 4096 blocks
  return (int32_t)w;
}

// Whether the hierarchy's frequency kernel keeps a block's copy of the load axis (`axis_lds` of the block's `lds` bytes) in LDS or reads it
// from global memory.  A copy of up to 40 KB, which leaves room for three blocks, is quicker (64 even points: 95 us a call of 1440 blocks, 103);
// a longer one only while all blocks are resident at once: 1000 uneven points (46 KB) 35 us and 38 with 60 blocks, 52 and 60 with 360, 145 and 139 with
// 1440; 4000 (72 KB) 179 and 149 with 1440.
inline bool dyn_freq_axis_staged(size_t axis_lds, size_t lds, int64_t blocks, int32_t n_cu) {
  return axis_lds <= 40 * 1024 || (lds <= 160 * 1024 && blocks <= (int64_t)(160 * 1024 / lds) * n_cu);
}

// How the hierarchy's frequency kernel is cut: blocks of `wins` windows and `run` classes, `chunk` ticks in LDS at a time.  A block's chain (layouts, capacities, four
// rounds of look-ups, sums) is 9 us whatever it holds, so a block takes the windows that give its threads work, as long as every compute unit has a
// block: 20 160 windows of one class and 12 ticks 50 us a call, a window a block 150; 2016 windows 42.6, 50.8; 10 000 windows of 4 classes and 5 ticks 60, 107.
// Classes beyond one run are cut into runs alike: 100 classes (300 windows, 12 ticks) by 34, 34, 32 78 us, by 47, 47, 6 84.  A round of a block's threads is
// 4.8 us: where twice as many blocks as compute units or fewer hold every look-up in one round, classes are cut for that, though the totals are then a launch of
// their own.  An hour of 25 classes and 12 ticks 37.1 us a call (one run, two rounds 40.5), 30 ticks 34.6 (43.8), 90 classes 36.7 (47.5), 240 windows of 25
// 40.3 (44.4).  Larger blocks do as well alone, but those of more than four waves wait for the end of another stream's kernel: beside an
// element-wise one the hour takes 160 us, 2000 to 3000 by blocks of 320 threads.
struct DynFreqShape {
  int32_t wins, run, n_run, chunk;
  bool tabled, staged;           // capacities tabled; load axis in LDS
  int64_t blocks;
  size_t lds;
};
#define DYN_FREQ_THREADS 256
#define DYN_FREQ_CHUNK 64
#define DYN_FREQ_TABLED 128      // frequencies up to which the capacities are tabled
#define DYN_FREQ_LDS (16 * 1024) // of results and capacities: blocks beside another stream's kernel find room
inline DynFreqShape dyn_freq_shape(int32_t n_window, int32_t G, int32_t n_tick, int32_t n_f, size_t axis_lds, int32_t n_cu) {
  DynFreqShape f;
  f.chunk = std::min(n_tick, DYN_FREQ_CHUNK);
  f.tabled = n_f <= DYN_FREQ_TABLED;
  const size_t per_cell = (size_t)f.chunk * 12 + (f.tabled ? (size_t)n_f * 16 : 0) + 20;
  int32_t most = std::min(DYN_FREQ_THREADS, (int32_t)std::max<size_t>(1, DYN_FREQ_LDS / per_cell));   // cells
  const int32_t one = DYN_FREQ_THREADS / f.chunk;            // cells of one round
  if ((int64_t)n_window * ((G + one - 1) / one) <= 2 * (int64_t)n_cu) most = std::min(most, one);
  f.n_run = (G + most - 1) / most;
  f.run = (G + f.n_run - 1) / f.n_run;                       // alike: the last block is as full as the others
  const int32_t items = f.run * f.chunk;
  f.wins = 1;
  if (f.n_run == 1) f.wins = std::max(1, std::min({most / G, DYN_FREQ_THREADS / items, n_window / std::max(1, n_cu)}));
  f.blocks = (int64_t)((n_window + f.wins - 1) / f.wins) * f.n_run;
  f.lds = (size_t)f.wins * f.run * per_cell;
  f.staged = f.tabled && dyn_freq_axis_staged(axis_lds, f.lds + axis_lds, f.blocks, n_cu);
  if (f.staged) f.lds += axis_lds;
  return f;
}

#endif  // DYN_RULES_H_
