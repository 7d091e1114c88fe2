// step_rules.h -- where blocks of steps on the moment field pay.
//
// Both routes of a call of several steps at tau = 1 give the same bits: pass 1
// and pass 2 of every step, or pass 1, steps from moments to moments, pass 2.
// The two passes stream the populations, so their time follows the sites and
// the bytes of the storage; a moment step computes the rims of its columns
// again and is bound by latency and vector instructions, whatever the storage.
// In 16 bits the two passes move a quarter of what they move in FP64, and there
// the routes cross.  The first moment step and the pass 2 that follows it also
// read what the passes have not left in the same caches: a block costs about
// 3 us on top from some 80 000 sites on, which the steps between must earn.
#pragma once

#include <stdint.h>

namespace scmc {

enum StorageWidth { WIDE_64, WIDE_32, WIDE_16 };

// D2Q9.  us per step of long calls, two passes against moment steps: FP16 psi =
// n, E4 448^2 10.9, 8.9; 512^2 11.8, 12.0; 600^2 13.5, 16.9; 1024^2 25.2, 36.3;
// 2048^2 80.8, 132; E6 512^2 12.3, 12.1; 600^2 14.3, 18.0.  With psi, E4 600^2
// 18.2, 16.6; 724^2 22.1, 24.8; 2048^2 120, 147; E8 600^2 28.1, 27.8; 1024^2 59,
// 71.  FP32 psi = n, E6 1448^2 72, 68; 2048^2 124, 130; E8 2048^2 128, 142; E4
// 2048^2 126, 125; E8 with psi 850^2 49.7, 46.2; 1024^2 65.6, 68.9.  FP64 gains at
// every size (2048^2 E8 324, 152).  Calls of two steps: FP16 E4 128 x 1024 9.1,
// 10.7; 512^2 11.8, 14.0 (three 14.1); FP32 E4 512^2 13.4, 14.9 (three 14.1; four
// and more gain).
inline bool mom2_steps_pay(StorageWidth w, int order, bool psi, int64_t sites, int64_t steps) {
    if (w == WIDE_64 || sites <= 120000) return true;
    if (w == WIDE_32)
        return steps >= 3 &&
               (order == 4 || sites <= (order == 8 && psi ? 900000 : 2500000));
    return steps >= 4 && sites <= (psi ? 400000 : 240000);
}

}  // namespace scmc
