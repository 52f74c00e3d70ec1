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

// Whether pass 1 sets the points of a call up itself (k_pass1_direct, which
// gives every tile of every point a work-group): it saves the set-up kernel's
// launch and the reads of its results, about 3 us, and repeats the set-up in
// every work-group, which costs about as much once they no longer all start
// together (16 wavefronts a CU for float and for double of one or two
// detectors, 12 for double of more, and never more than four groups), or once
// more points than these add to one counter.  Measured, direct / set-up kernel,
// four detectors unless said: float 131072 (256 threads) 0.88 at 256
// work-groups, 0.96 at 1024; 262144 (512 threads) 0.91 at 512, 1.02 at 640; 16384
// 0.93 at 1024, 0.99 at 1280; double 131072 (256 threads) 0.95 at 768, 1.02 at
// 896 (two detectors 0.90 at 1024, 0.99 at 1152); 98304 (128 threads) 0.95 at
// 1024, 1.05 at 1152; 2048 (a work-group a point) 0.96 at 384 points, 1.00 at
// 512, 1.21 at 1024 (double 0.98, 1.05, 1.07); 4096 0.87 at 256 points, 0.98 at 512.
inline bool direct_call(int points, int tiles, int threads, bool fp64, int n_det, int n_cu) {
  const long long groups = (long long)points * tiles;
  return groups * (threads / 64) <= (fp64 && n_det > 2 ? 12 : 16) * n_cu && groups <= 4 * n_cu && 4 * points <= 7 * n_cu;
}

// Whether the fused schedule takes a two-pass plan of so many work items
// (tiles of both passes) a point in one persistent launch.  Every item signals,
// and every second one waits, at device scope, so its launch grows with the
// items: us for 320 points, fused / separate launches: 8192 (8 items) 104 / 34,
// 16384 (16) 331 / 48, 32768 (32) 1450 / 81, 131072 (96) 1920 / 270.  It is kept
// where it costs least; longer points run as separate launches, same bits.
inline bool fused_takes(int items) { return items <= 8; }

// Work-groups of a three-pass plan's middle pass: at most one per item, and the
// last pass's number for double.  Float takes at most 4096: beyond, the more
// numerous work-groups of the last pass, which suit that one, cost it up to 12%
// (us for 32 points of 3686400, 4096 / 16384 work-groups: middle 806 / 905, last
// 296 / 280; 8 points of 7372800 451 / 478; double, 4 points, 455 / 423).
inline int middle_groups(long long items, int grid2, bool fp64) {
  const int most = fp64 || grid2 < 4096 ? grid2 : 4096;
  return items < most ? (int)items : most;
}

// Parts that a point's adjoint sums are split into, a work-group each: enough
// work-groups for the chip (1024) in small batches, but at least 64 bins to a
// thread of a long segment and otherwise at most 64 parts, which the chain
// rule reads one after the other.  `groups`: detector groups of a point, each
// with work-groups of its own; `bins` of the longest segment.  Gradient of one
// point, us per call, 64 parts / this many: 7372800 samples (3.5 million bins,
// 213 parts) 322 / 214, 3686400 (106) 179 / 148.
inline int adjoint_parts(int n, int groups, long long bins) {
  const long long most = bins / (64 * 256) < 64 ? 64 : bins / (64 * 256) < 256 ? bins / (64 * 256) : 256;
  const long long want = (1024 + (long long)n * groups - 1) / ((long long)n * groups);
  return (int)(want < 1 ? 1 : want < most ? want : most);
}

}  // namespace fcas
