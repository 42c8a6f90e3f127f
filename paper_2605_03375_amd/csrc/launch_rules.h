// Rules that decide by sizes alone how a call is run.  Plain C++, so that they can be tested without a GPU; the kernels
// use the ones that need device values themselves.
#pragma once

#include <stdint.h>

#include "layer_call.h"

namespace tutti {

// Workgroups of a whole-GPU launch that fills every place: what its grid, the wavefronts that the rules count and the entry
// writers' share are all cut off at, so that a rule never counts on a wavefront that the grid has not got.  (More than a chip
// holds at once are asked for by the measurement build's knob only.)
constexpr uint32_t full_grid(uint32_t cus, uint32_t wgs_per_cu) {
  return static_cast<uint64_t>(cus) * wgs_per_cu < kMostWgs ? cus * wgs_per_cu : kMostWgs;
}

// Whether a save of several requests gives each wavefront one slice at most and reads it under the scan (store_pack moves no
// second one): up to 3/4 of the chip's wavefronts.
constexpr bool one_slice_saves(uint64_t items, uint64_t chip_waves) { return 4 * items <= 3 * chip_waves; }

// A whole-GPU restore reads its first slices, up to 32 MiB, in one burst; stores that start among those reads cost more
// (the memory turns between reading and writing) than the same stores a little later.  So a wavefront that has read
// ahead holds its first stores back, for the returned number of 512 clocks (0.21 us each): only if the launch gives
// most of the chip's `chip_waves` wavefronts an item and no wavefront more than two, by the items the requests really
// have (the table may be longer); a launch that read nothing ahead sleeps for nothing.  Only the longest scan (six steps,
// beyond 32 requests) delays the stores by itself, by about one step.
// Restore of 32 KiB blocks, graph replay of 16 layers, us, pause 0 / 2 / 5 / 6 / 7 / 8 / 9 / 10 (items / chip_waves in brackets):
//   1 request    384 blocks (0.75)  10.5 /  9.3 /  9.3 /  9.6 /  9.5 /  9.4 /  9.6 /  9.8
//                448 (0.88)         12.2 / 12.4 / 10.5 / 10.2 / 10.3 / 10.4 / 10.7 / 10.6
//                464 (0.91)         12.8 / 13.1 / 13.2 / 13.0 / 11.8 / 11.1 / 11.0 / 11.2
//                512 (1.00)         13.8 / 14.0 / 14.4 / 14.2 / 13.5 / 12.2 / 11.6 / 11.6
//                560 (1.09)         15.4 / 15.0 / 15.4 / 15.1 / 13.6 / 12.9 / 12.9 / 13.0
//                640 (1.25)         17.0 / 16.7 / 17.1 / 16.3 / 15.0 / 14.8 / 14.9 / 15.2
//   8 requests   384                10.4 /  9.1 /  9.6 /  9.6 /  9.6 /  9.7 / 10.0 / 10.1
//                448                12.6 / 12.7 / 10.6 / 10.4 / 10.5 / 10.8 / 10.9 / 10.8
//                464                13.1 / 13.3 / 13.3 / 12.2 / 11.2 / 11.0 / 11.1 / 11.1
//                512                13.9 / 14.2 / 14.4 / 13.7 / 12.6 / 11.9 / 11.6 / 11.7
//                640                17.1 / 17.0 / 17.1 / 15.6 / 15.2 / 15.0 / 15.1 / 15.4
//   64 requests  384                10.1 /  9.1 /  9.7 /  9.6 /  9.6 /  9.7 / 10.0 / 10.2
//                448                12.6 / 12.6 / 10.5 / 10.4 / 10.9 / 10.7 / 10.8 / 10.9
//                464                13.0 / 13.3 / 13.2 / 12.0 / 11.2 / 11.2 / 11.3 / 11.3
//                512                14.2 / 14.5 / 14.4 / 13.2 / 12.0 / 11.6 / 11.9 / 12.0
//                640                17.0 / 17.1 / 16.4 / 15.4 / 15.1 / 15.1 / 15.3 / 15.6
// and 0 / 2 / 5 / 7 at 320 blocks (0.63), 1 request, 7.6 / 7.9 / 7.9 / 8.3, at 1024 (2.0) 23.7 / 23.8 / 23.7 / 23.5, at 2048
// (4.0), 8 requests, 44.1 / 44.1 / 44.2 / 44.4, 64 requests 43.9 / 43.9 / 44.1 / 44.3.
// Where the time falls off a step, the pause stands behind it.
// `file`: a retrieve of one request reads ahead behind two more loads and starts later.  In a train, pause 2 / 5 / 6 / 7 / 8:
// 384 blocks 9.6 / 9.9 / 10.0 / 10.2 / 10.4, 448  12.6 / 11.1 / 11.2 / 11.2 / 11.3, 512  14.6 / 14.7 / 13.9 / 12.9 / 12.5, 640
// 16.8 / 15.7 / 15.4 / 15.5 / 15.7; a call each the same and 1.4 more.
constexpr uint32_t hold_back_pause(uint32_t items, uint32_t chip_waves, uint32_t n_req, bool file) {
  if (items > 2 * chip_waves || 32 * items <= 21 * chip_waves) return 0;
  if (file) return 32 * items <= 25 * chip_waves ? 2 : 32 * items <= 29 * chip_waves ? 5 : 5 * items <= 6 * chip_waves ? 8 : 6;
  if (32 * items <= 25 * chip_waves) return 2;
  if (32 * items <= 28 * chip_waves) return 6;
  return n_req <= 32 && 10 * items <= 11 * chip_waves ? 9 : 8;
}

// Slice of a CU-budgeted copy of `blocks` blocks (K and V each), in pieces of 1 KiB.  What a compute unit moves depends on
// the length of a wavefront's run of loads and of stores, not on the bytes in flight: a plain cold copy of 256 MiB on 8 / 32 /
// 64 compute units (1024 threads each) reaches 61 / 52 / 45 GB/s per unit with 8 KiB runs, with one item in flight as with
// two, and 75 / 63 / 56 with 16 KiB (of 32 MiB 61 / 51 / 43 and 75 / 60 / 49).  But a longer run also ends later: up to about
// 1024 items, in a working set that the last-level cache holds, 8 KiB are the better where the launch reads its first slices
// ahead (`ahead`), and without that unless every wavefront gets one item at most or the compute units are many.  16 / 8 KiB,
// us, 32 KiB blocks:
//   restore of 4 requests   64 blocks on 32 units 6.5 / 5.1    128 on 64  7.9 / 5.7    128 on 8  31.0 / 30.4
//                          256 on 32  20.2 / 20.5             384 on 8  90.9 / 92.4   1024 on 32  71.5 / 79.4
//   save of 4 requests      64 on 8  14.2 / 15.4               64 on 32  6.3 / 7.0     128 on 8  32.4 / 29.2
//                          256 on 8  64.0 / 60.9              384 on 8  95.1 / 93.8   1024 on 32  72.8 / 80.4
//                          256 on 64  12.9 / 13.2
// 8 KiB slices lie in neighbouring wavefronts (first_item), so a last round that is nearly empty falls to a few compute
// units: 34 blocks, 272 slices of 8 KiB, on 8 / 16 units restore in 7.7 / 5.8 as 16 KiB and 9.7 / 7.6 as 8 KiB slices.
// Blocks that are no whole number of slices: slices of 8 KiB if those fit (8 KiB blocks, 4096 on 8 units, restore 261 us
// as pieces, 256 as slices; but saves on many units: 256 of 40 KiB on 64 16.8 and 19.1), pieces otherwise (16 at a time);
// a visiting order keeps slices, of 8 KiB.
// `short_rows`: a head-major pool whose rows are shorter than a cache line: the longer run wins at every size (rows of 64
// bytes, 16 KiB blocks, as line tiles: 256 on 8 units restore 25.3 / 35.6, save 29.6 / 38.0; 192 on 32 8.2 / 11.3, 8.8 / 12.7;
// 320 on 64 9.5 / 12.7, 9.6 / 13.9; moved directly: 300 on 8 32 / 51, 39 / 57).
constexpr uint32_t budget_units(bool ahead, uint32_t block_bytes, uint32_t blocks, uint32_t cu_budget, bool ordered,
                                bool short_rows) {
  if (block_bytes % 8192 != 0) return ordered ? 8 : 16;
  const uint64_t items = 2ull * blocks * (block_bytes / 8192) / 2;
  if (short_rows && block_bytes % 16384 == 0) return 16;
  if (block_bytes % 16384 != 0) return !ordered && !ahead && cu_budget > 32 && items > 1024 ? 16 : 8;
  if (items > 1024 || cu_budget == 0) return 16;
  const uint64_t waves = 16ull * cu_budget, rest = 2 * items % waves;
  const bool even = rest == 0 || 4 * rest >= 3 * waves;
  if (ahead) return 2 * items <= waves || even ? 8 : 16;
  const uint32_t one_each = cu_budget > 16 ? 16 * cu_budget : 256;
  return items <= one_each || cu_budget > 32 || !even ? 16 : 8;
}

// The launch shapes that have kernels for blocks that are no whole number of slices (pieces): under a budget the one that
// budget_units asks for then.  In any other shape the kernel of whole slices would read and write beyond the blocks.
constexpr bool pieces_shape(bool whole_gpu, uint32_t units) { return whole_gpu || units == 16; }

// Blocks that are no whole number of 4 KiB slices, token-major, of a fused launch on the whole GPU: pieces (move_pieces), or equal
// slices of whole 128-byte lines, as few as there can be (cut_slice; 0: none).  Slices read ahead, and save one request's or a few
// requests' blocks without a scan, like those of other blocks; pieces need a search and a table load in each lane first, but put
// several blocks into an item and fill its accesses.  So it goes by the items (cuts_blocks): up to one for each of the chip's
// wavefronts, twice that for a save of one request, which reads behind a single load, and half of it for a restore of blocks that
// are a whole number of pieces.  A slice of up to 2 KiB uses half of its accesses or less: only where a wavefront would do nothing
// else.  Graph replay, us, pieces / slices, by payload:
//                              0.5 MiB        2            4            8           12           16           32          128
//   12.5 KiB  restore of 1   3.86 / 2.85  4.20 / 3.29  4.45 / 3.81  5.79 / 4.86  7.09 / 6.29  8.40 / 8.28  14.0 / 14.1  46.5 / 46.8
//   blocks    of 8 requests  4.15 / 3.48  4.46 / 3.96  4.81 / 4.37  6.17 / 5.57  7.49 / 6.91  8.81 / 8.25  14.2 / 14.2  46.2 / 45.9
//             of 200                                                7.89 / 7.53  8.60 / 7.99  10.2 / 9.7   15.2 / 15.6  46.7 / 46.2
//             save of 1      3.88 / 2.85  4.36 / 3.34  4.63 / 3.83  5.88 / 4.71  7.18 / 6.20  8.56 / 7.58  14.0 / 13.4  48.7 / 47.6
//             of 8           4.31 / 3.46  4.55 / 3.63  4.91 / 3.87  6.08 / 4.48  7.60 / 5.48  8.86 / 7.25  14.5 / 14.5  48.6 / 48.8
//             of 200                                                8.26 / 5.63  9.05 / 6.05  10.5 / 7.3   16.2 / 16.0  50.6 / 50.3
//   10 KiB    restore of 1   3.70 / 2.90  4.04 / 3.31  4.27 / 3.80  5.16 / 5.05  6.66 / 6.80  8.11 / 8.24  13.9 / 13.8  45.4 / 47.0
//             save of 8      4.16 / 3.30  4.49 / 3.62  4.72 / 3.93  5.59 / 4.44  7.19 / 5.70  8.31 / 8.20  14.0 / 14.1  47.3 / 48.6
//   1 KiB     restore of 1   3.64 / 2.77  3.79 / 3.14  4.06 / 4.31  5.19 / 6.26
//             of 200         6.37 / 5.64  6.45 / 5.78  6.56 / 5.97  7.62 / 7.97
//             save of 8      4.11 / 3.45  4.18 / 3.73  4.62 / 4.41  5.61 / 6.25
constexpr uint32_t cut_slice(uint32_t block_bytes) {
  if (block_bytes % 128 != 0 || block_bytes < 1024 || block_bytes > (512u << 10)) return 0;
  const uint32_t lines = block_bytes / 128, least = lines / 32 + (lines % 32 != 0 ? 1 : 0);
  for (uint32_t n = least; n == least || n < 2 * least; ++n)
    if (lines % n == 0) return 128 * (lines / n);
  return 0;
}
constexpr bool cuts_blocks(bool unpack, uint32_t n_req, uint32_t block_bytes, uint32_t slice, uint64_t items,
                           uint32_t chip_waves) {
  if (slice <= 2048) return (unpack ? 4 : 2) * items <= chip_waves;
  if (unpack) return (block_bytes % 1024 == 0 ? 2 : 1) * items <= chip_waves;
  return items <= (n_req == 1 ? 2ull : 1ull) * chip_waves;
}

// Whether the submission entries (or the contexts) of a whole-GPU launch of up to 64 requests are written by workgroups of
// their own, in front of the `copy_wgs` that move blocks, instead of riding along with the first of those.  Riding along a
// small launch is as long as the scan with the entries' divisions, the copy and the entry one behind the other; a larger one
// hides that behind its other items, and the workgroups in front then only come first.  Graph replay, us, along / apart:
//   1 request     restore of 2 blocks of 32 KiB 3.3 / 2.7, 64 3.35 / 3.1, 100 3.5 / 3.4, 128 (512 workgroups) 3.9 / 3.8; save 3.0 /
//                 2.7, 3.8 / 3.6; retrieve of 64 6.1 / 5.5, 100 6.2 / 5.5; 16 layers of 64: retrieves 64.6 / 59.4, stores 72.9 / 59.5
//                 200 (800): restore 5.9 / 5.9, retrieve 8.5 / 8.5, store 8.6 / 8.6
//   several       restore of 64 in 8 4.3 / 4.0, 128 in 30 4.8 / 4.5, 160 in 8 (640) 4.95 / 4.9; save 4.1 / 3.8, 4.6 / 4.2, 4.7 / 4.6;
//                 retrieve 6.8 / 6.2, 7.6 / 7.4, 8.6 / 8.1; 16 layers of 20 in 5: retrieves 78 / 60, stores 66 / 56
//                 200 in 8 (800): store 7.7 / 8.2; 1500 blocks of 4 KiB (750) 7.2 / 8.6
// (What loses: a train of 3 stores of 100 blocks in 8, 15.4 / 16.2, of retrieves of 120 in one request, 15.7 / 16.2.)
constexpr bool entries_apart(uint32_t copy_wgs, uint32_t cus, uint32_t n_req) {
  return 2 * copy_wgs <= (n_req == 1 ? 4 : 5) * cus;
}

// Whether a save of several requests reads its `items` (slices of the table's blocks) at once, or when it has counted the
// requests' blocks (PackItem).  What lies behind the requests' blocks in the table is read for nothing then: with all of it, a
// quarter of the chip's wavefronts (128 blocks of 32 KiB, 8 MiB) is the most at which that costs no more than it gains.  Graph
// replay, us, 2 blocks in 2 requests with a table of 96 / 128 / 160 / 200: in staging order 3.6 / 3.6 / 3.8 / 3.8, read at once
// 3.2 / 3.4 / 3.9 / 4.8, counted first 3.1 / 3.3 / 3.1 / 3.6.
// Up to 64 requests counting costs nothing.  For more it takes a barrier, and the stores then start among the reads; a table of
// up to 8 blocks a request (saves behind a decode step) is taken to be theirs, a longer one for a fixed capacity.  Beyond 1024
// requests reading the counts again behind the data is the longer way.  At once / counted first:
//   all owned   8 KiB blocks, 1280 in 512 9.7 / 10.8, 1024 in 256 7.2 / 8.4, 1024 in 128 7.2 / 8.3; 32 KiB, 300 in 200 8.2 / 9.3;
//               4 KiB, 3000 in 1000 12.2 / 12.9, in 250 11.2 / 11.8, in 2000 22.6 / 18.7
//   half owned  7.9 / 7.6, 6.6 / 6.5, 6.4 / 6.0; 7.9 / 6.3; 10.7 / 9.8, 9.1 / 6.7, 20.1 / 16.8
//   few owned   7.3 / 5.1, 6.0 / 4.4, 5.9 / 4.3; 6.1 / 4.4; 9.8 / 7.5, 7.0 / 4.7, 18.4 / 15.7
constexpr bool pack_at_once(uint64_t items, uint32_t chip_waves, uint32_t n_req, uint32_t table_len) {
  return 4 * items <= chip_waves || (n_req > 64 && n_req <= 1024 && table_len <= 8 * n_req);
}

// The same pause as hold_back_pause for a save of more than 64 requests that has read its slices at once, by the items of 4 KiB
// that the requests have: more than half of the chip's wavefronts.  Us, graph replay and eager calls on warm data, pause 0 / 1 / 2 / 3:
//   1280 of 8 KiB in 512   8.7 8.5 / 8.5 8.3 / 8.5 8.3 / 8.7 8.5    350 of 32 KiB in 100   10.2 9.7 / 10.1 9.3 / 9.8 9.3 / 9.8 9.1
//   3000 of 4 KiB in 1000  12.0 11.3 / 11.9 11.3 / 11.8 11.2 / 11.6 10.9
//   1500 of 8 KiB in 300   10.1 9.6 / 10.5 10.1 / 9.9 9.4 / 10.1 9.6
//   300 of 32 KiB in 200   7.2 7.2 / 7.2 7.1 / 7.3 7.1 / 7.6 7.3
// and with half of the chip's, 1024 of 8 KiB in 256, 6.3 6.3 / 6.5 6.4 / 6.8 6.6; 150 of 32 KiB in 70 5.5 5.3 / 5.7 5.5 / 5.9 5.7.
constexpr uint32_t pack_pause(uint32_t items, uint32_t chip_waves) { return 2 * items > chip_waves ? 2 : 0; }

// The same pause where it was missing: for one request's restore on the path of its own, which has no scan to delay its stores
// and takes up to half of the chip's wavefronts, and for saves of up to 64 requests that read a slice for each wavefront.  By
// the items there are, of 4 KiB (full_slices), and about as long as their reads take; the scan delays the stores by itself, by
// three or four steps.  Blocks of 32 KiB, graph replay, us, by the pause (items / chip_waves in brackets):
//                                      0      2      4      6      8     10     12     14
//   restore of 1      112 (0.22)     4.62   4.33   4.28   4.65   5.09              (3: 4.15; 96 blocks 3.29, with any pause more)
//                     160 (0.31)     5.50   5.41   5.29   5.03   5.43
//                     200 (0.39)     6.52   6.52   5.79   5.74   5.78   6.18       (7: 5.61)
//                     240 (0.47)     7.24   6.88   6.85   6.15   6.28   6.63       (7: 6.10)
//   save of 1         144 (0.28)     5.53   5.45   5.42   5.43   5.07   5.45   5.89
//                     200 (0.39)     7.18   7.19   7.03   7.06   6.47   6.12   6.55   7.01
//                     260 (0.51)     8.02   8.37   7.90   8.21   8.86   7.65   7.47   7.66
//                     320 (0.63)     9.05   9.55   9.20   9.03   9.55   9.44   8.07   8.33
//                     360 (0.70)    10.06  10.60  10.37  10.28  10.22  10.39  11.11   9.83
//                     380 (0.74)    10.48  10.99  10.64  10.81  11.05  10.65  11.44  10.90
//   save of 9         144 (0.28)     5.17   4.99   5.02   5.42
//                     200 (0.39)     6.81   6.49   6.24   6.08   6.46
//                     240 (0.47)     7.55   7.31   6.43   7.09   6.78   7.18       (3: 6.70, 5: 7.39)
//                     260 (0.51)     7.87   8.04   8.33   8.25   7.52   7.51   8.07
//                     320 (0.63)     9.30   9.20   8.98   9.75   9.49   8.01   8.38   9.08
//                     380 (0.74)    11.01  10.81  10.48  10.65  11.47  11.15  10.22  10.05
//   save of 40        144 (0.28)     4.62   4.70   5.09                             (1: 4.50)
//                     240 (0.47)     6.76   6.56   6.11   6.54   6.90   7.26       (3: 6.16)
//                     320 (0.63)     8.73   8.36   8.45   9.08   8.63   7.95   8.67
// Runs fall into one of two modes, 5 to 10 % apart, by where their buffers lie; over block sizes, requests and 0.2 to 0.75 of the
// chip saves gain 3.5 % in the geometric mean, up to 16 %.  Head-major blocks that are moved row by row (rows of 80 bytes) lose
// with it, saves of 432 to 592 blocks of 20 KiB up to 15 %, and one request's restores of cut slices (307 blocks of 12.5 KiB 4.8 / 5.0):
// none there.  Cut slices count as the 4 KiB slices that they make up here, in pack_pause and in hold_back_pause: restores of 2 to
// 40 requests at 0.7 to 1.0 of the chip take the same time with either unit and without a pause, saves of 563 blocks of 12.5 KiB in
// 100 / 300 requests, by slices / so, 7.6 7.6 / 7.8 7.7 and 8.2 8.2 / 8.0 8.0, larger ones the same.
constexpr uint32_t one_restore_pause(uint32_t items, uint32_t chip_waves) {
  const uint32_t i = 32 * items, c = chip_waves;
  if (items > chip_waves || i < 7 * c || c == 0) return 0;
  return 3 + (i >= 8 * c) + (i >= 9 * c) + (i >= 10 * c) + (i >= 12 * c);
}
// `lines`: a head-major pool moved as line tiles, whose reads take longer.  Rows of 64 bytes, 16 heads / rows of 32 bytes, 32 heads,
// 16 tokens, by the part of the chip, without / with the pause of the others (three processes each, medians):
//                      0.36        0.40        0.45        0.50        0.55        0.60        0.63         0.66         0.70
//   save of 1                               8.1 / 7.5   8.5 / 8.0   9.1 / 9.0   9.6 / 9.2  10.5 / 9.7   10.8 / 11.0  10.8 / 11.3
//                                           8.2 / 7.6   8.6 / 8.0   9.2 / 9.1   9.6 / 9.1  10.6 / 10.0  10.9 / 11.1  11.2 / 12.1
//   save of 9        7.1 / 6.8   7.9 / 8.1   8.1 / 8.1   8.7 / 9.0   9.5 / 9.6   9.8 / 9.5  (0.65) 10.9 / 10.2
//                    7.1 / 6.9   8.0 / 8.2   8.2 / 8.1   8.8 / 9.2   9.7 / 9.7   9.9 / 9.6         11.0 / 10.4
//   save of 40       7.2 / 6.8   8.0 / 8.2   8.3 / 8.7   8.7 / 9.2   9.5 / 9.7   9.8 / 9.6         11.0 / 10.2
//                    7.3 / 7.0   8.0 / 8.5   8.3 / 8.6   8.7 / 9.3   9.6 / 9.8   9.9 / 9.7         11.0 / 10.5
// and restores of one request 5.7 / 5.3 at 0.25, 7.6 / 6.6 at 0.4, 8.1 / 6.9 at 0.48.
// `early_end`: none from 2/3 on, which is what the kernels ask for with any blocks: with the buffers elsewhere than for the table
// above, saves of token-major 32 KiB blocks, without / with it, 320 of them (0.63) 9.5 / 8.9, but 360 (0.70) 10.8 / 12.1.
constexpr uint32_t one_save_pause(uint32_t items, uint32_t chip_waves, bool early_end = false) {
  const uint32_t i = 32 * items, c = chip_waves;
  if (items > chip_waves || i < 9 * c || 2 * i > (early_end ? 41 : 45) * c || c == 0) return 0;
  return i < 12 * c ? 8 : i < 16 * c ? 10 : i < 17 * c ? 12 : 14;
}
constexpr uint32_t few_save_pause(uint32_t items, uint32_t chip_waves, uint32_t n_req, bool lines = false) {
  const uint32_t i = 32 * items, c = chip_waves;
  if (items > chip_waves || i < 9 * c || c == 0) return 0;
  if (lines && i >= 12 * c && i <= 16 * c) return 0;
  if (i < 13 * c) return (i < 11 * c ? 2u : 3u) - (n_req > 32 ? 1u : 0u);
  return i < 16 * c ? 3 : i < 17 * c ? 8 : i < 21 * c ? 10 : 12;
}

// Whether a head-major pool goes through LDS tiles or is moved directly, where it is not moved as line tiles
// (as_line_tiles); where this holds an ordered restore keeps staging order.  On the whole GPU it pays while a row is shorter
// than a 128-byte line.  Under a CU budget a workgroup has one tile in flight at a time, and only rows of 16 bytes on more
// than 16 compute units are worth that.  Through LDS / direct, us, save and restore of 16 KiB blocks:
//   rows of 16 bytes   300 blocks on 8 units 85 / 69, 75 / 64   500 on 16  78 / 73, 73 / 64   1000 on 32  87 / 99, 83 / 90
//                      2000 on 64  94 / 122, 89 / 139
//   rows of 32 bytes   300 on 8  82 / 50, 75 / 44   500 on 16  78 / 57, 73 / 48   1000 on 32  87 / 69, 83 / 56
//                      2000 on 64  94 / 79, 89 / 66
//   rows of 64 bytes   300 on 8  81 / 38, 75 / 31   500 on 16  78 / 43, 74 / 37   1000 on 32  87 / 51, 82 / 45
//                      2000 on 64  94 / 57, 89 / 51
constexpr bool hnd_through_lds(uint32_t row_bytes, uint32_t cu_budget) {
  return row_bytes < (cu_budget == 0 ? 128u : cu_budget > 16 ? 32u : 16u);
}

// Whether a head-major pool is moved as line tiles (row size, tokens and heads are powers of two).  While a row is shorter
// than a 128-byte line and the block a whole number of whole-GPU slices they are: the other way is the object's order, in
// which a piece of 1 KiB holds 1024 / heads bytes of every head: whole lines too for up to 8 heads, and its loads of a
// restore need no offsets.  Us, object's order / line tiles, rows of 64 bytes, 8 heads, 16 KiB blocks: restore of 1536 on 32
// units 57.3 / 59.3, of 256 on 8 22.4 / 22.9, of 4096 on the whole GPU 43.5 / 43.6; save of 1536 on 32 units 60.3 / 60.6, of
// 512 21.5 / 20.9, of 384 on the whole GPU 5.5 / 5.3, of 64 in one request 3.6 / 3.4; 4 heads, rows of 16 bytes, 4 KiB blocks,
// restore of 1536 on the whole GPU 6.5 / 6.2 (on 32 units of blocks of any size the same).
// Rows of a line or more, up to 512 bytes, are whole lines in the object's order as well, but there each offset takes two
// divisions: `half_empty`, whole-GPU launches with items for half of the chip's wavefronts at most, where that shows.  Rows of
// 256 bytes, 8 heads: save of 16 blocks of 32 KiB 3.16 / 2.89, 64 3.71 / 3.53, 64 in 33 requests 4.22 / 4.04; restore 2.96 /
// 2.89, 3.33 / 3.27, 4.38 / 4.33; beyond, save of 384 in 8 10.25 / 10.5, 2048 47.6 / 47.5, restore 9.0 / 8.9, 43.5 / 43.9.
constexpr bool as_line_tiles(uint32_t row_bytes, uint32_t block_bytes, uint32_t heads, uint32_t cu_budget, bool unpack,
                             bool half_empty) {
  if (row_bytes >= 128) return cu_budget == 0 && half_empty && row_bytes <= 512 && block_bytes >= 4096;
  return row_bytes >= 16 && block_bytes >= 4096 &&
         !(unpack && cu_budget != 0 && heads <= 8 && row_bytes > 16);
}

// log2 of the tokens of a line tile, from the logarithms of row size, heads and tokens: the runs of both sides about the
// same length (never below a line, and no run is split that could stay whole where there are fewer heads or tokens).
// 2 / 4 tokens, rows of 64 bytes, us: save of 1536 blocks of 16 KiB on 32 units 60.7 / 59.2, restore 61.8 / 60.1.
constexpr uint32_t line_tile_shift(uint32_t row_shift, uint32_t head_shift, uint32_t token_shift) {
  uint32_t t = (10 - row_shift) / 2;
  if (t + head_shift < 10 - row_shift) t = 10 - row_shift - head_shift;
  return t < token_shift ? t : token_shift;
}

}  // namespace tutti
