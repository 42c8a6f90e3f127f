// Rules that decide by sizes alone how a call is run.  Plain C++, so that they can be tested without a GPU; the kernels
// use the ones that need device values themselves.
#pragma once

#include <stdint.h>

namespace tutti {

// A whole-GPU restore reads its first slices, up to 32 MiB, in one burst; stores that start among those reads cost more
// (the memory turns between reading and writing) than the same stores a little later.  So a wavefront that has read
// ahead holds its first stores back, for the returned number of 512 clocks (0.21 us each): only if the launch gives
// most of the chip's `chip_waves` wavefronts an item and no wavefront more than two, by the items the requests really
// have (the table may be longer); a launch that read nothing ahead sleeps for nothing.  Every step of the scan in front
// delays the stores as well, so more requests wait less.
// Restore of 32 KiB blocks, cold, us, pause 0 / 2 / 4 / 6 / 7 (items / chip_waves in brackets):
//   1 request    320 blocks (0.63)  7.7 / 8.0 / 8.0 / 8.2 / 8.4    384 (0.75) 10.5 / 9.1 / 9.1 / 9.5 / 9.4
//                448 (0.88)  12.1 / 12.3 / 11.4 / 10.4 / 10.4      512 (1.00) 13.9 / 13.8 / 13.9 / 13.8 / 12.6
//                640 (1.25)  16.2 / 16.0 / 16.6 / 15.9 / 15.0      1024 (2.0) 23.7 / 23.8 / 23.8 / 23.5 / 23.5
//   8 requests   384  9.0 / 8.8 / 9.3 / 9.1 / 9.2    448  11.8 / 11.3 / 10.1 / 10.3 / 10.4    512  13.1 / 13.3 / 13.2 / 11.3 / 11.2
//                640  15.6 / 16.1 / 14.6 / 14.2 / 14.4    1024  23.7 / 23.7 / 23.4 / 23.4 / 23.5    2048  44.2 / 44.1 / 44.3 / 44.6 / 44.8
//   64 requests  384  8.7 / 9.2 / 9.2 / 9.4 / 9.5    448  11.7 / 10.3 / 10.3 / 10.4 / 10.3    512  13.2 / 13.4 / 11.9 / 11.3 / 11.6
//                640  15.8 / 14.5 / 14.2 / 14.7 / 15.0    1024  23.6 / 23.3 / 23.3 / 23.7 / 23.9    2048  43.9 / 44.1 / 44.4 / 44.8 / 45.0
// `file`: a retrieve of one request reads ahead behind two more loads and starts later.  One call / in a train, pause 0 /
// 7: 320 blocks 10.6 / 11.2 and 9.3 / 9.4, 384  12.5 / 11.8 and 11.1 / 10.3, 448  14.6 / 13.3 and 13.2 / 11.7, 640  18.3
// / 16.8 and 16.9 / 15.8.
constexpr uint32_t hold_back_pause(uint32_t items, uint32_t chip_waves, uint32_t n_req, bool file) {
  if (items > 2 * chip_waves || 32 * items <= 21 * chip_waves) return 0;
  if (file) return 7;
  const uint32_t steps = n_req > 1 ? 32u - static_cast<uint32_t>(__builtin_clz(n_req - 1)) : 0u;
  if (32 * items > 29 * chip_waves) return 7 - steps / 3;
  if (32 * items > 25 * chip_waves) return 6 - (steps + 1) / 2;
  return steps < 4 ? 2 - steps / 2 : 0;
}

}  // namespace tutti
