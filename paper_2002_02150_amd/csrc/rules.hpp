// rules.hpp -- the choices between ways of running a call that depend on its
// sizes alone: plain host functions, so that the tests read them too.
#pragma once

#include <stddef.h>

namespace fcas {

// How pass 1 stores the rows that pass 2 reads (PassArgs::nt).
enum StorePolicy {
  kStoreCached = 0,      // through the L2
  kStoreStreamed = 1,    // non-temporal
  kStoreBySegments = 2,  // non-temporal if the launch holds more than one segment
};

// The policy of a launch that writes `bytes`.  Rows stored through the L2 are
// found there or in the 256 MiB memory-side cache by pass 2, but they displace
// the segment data, which pass 1 reads again wherever a work-group's next point
// is of another segment.  Measured, us per call (through the L2 / non-temporal):
//   one segment:     65536 x 324 (340 MB) 132 / 141, 32768 x 648 132 / 139,
//                    131072 x 238 (500 MB) 193 / 190, 131072 x 2048 (4.3 GB) 1510 / 1475
//   several, 230 MB: 65536 x 219 in 43 segments 116 / 114, 131072 x 109 in 21 118 / 119
//   several, more:   131072 x 320 in 64 346 / 292, in 8 303 / 273, 65536 x 381 in 76
//                    212 / 185, 262144 x 190 in 4 (800 MB) 379 / 334
inline StorePolicy store_policy(size_t bytes) {
  return bytes > ((size_t)1 << 30) ? kStoreStreamed : bytes >= ((size_t)1 << 28) ? kStoreBySegments : kStoreCached;
}

}  // namespace fcas
