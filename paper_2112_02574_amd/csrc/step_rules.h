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

#include <algorithm>

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
// and more gain); of three, FP16 E4 384^2 9.5, 8.2, with psi 12.0, 9.5, 448^2 13.8,
// 12.5.
inline bool mom2_steps_pay(StorageWidth w, int order, bool psi, int64_t sites, int64_t steps) {
    if (w == WIDE_64 || sites <= 120000) return true;
    if (w == WIDE_32)
        return steps >= 3 &&
               (order == 4 || sites <= (order == 8 && psi ? 900000 : 2500000));
    return steps >= (sites <= (psi ? 210000 : 150000) ? 3 : 4) && sites <= (psi ? 400000 : 240000);
}

// D3Q19.  sites: of the lattice, or of the members that step together; ragged:
// how many of them lie in rows that are not a multiple of 16; us: the launch
// model's time of a moment step (mom_shape).
//
// FP64 and FP32 gain at all sizes but two: E6 with psi in FP64, whose moment step
// keeps part of its registers in memory (40^3 21.1 against 22.3 us per step of
// long calls, 8 x 64 x 64 17.1 against 19.3; 52^3 37, 33), and calls of two steps
// in FP32 (44^3 E6 11.7, 12.6; 48^3 12.8, 13.7; four of 32^3 12.2, 13.5; 52^3 gains).
// 16 bits, psi = n: the time of the two passes is modelled from long calls, E4 /
// E6: 48^3 10.8 / 12.0, 64^3 14.4 / 16.0, 64 x 64 x 128 23.6 / 26.3, 96^3 38.1 /
// 41.5, 48 of 32^3 58.6 / 65.7; E6 takes 1.1 times E4's, as it does in a moment
// step, so the order cancels; ragged rows take about 9 % more (60^3 15.5 / 17.3).
// Against moment steps: 64^3 15.7 / 17.5, 16 x 128 x 128 17.0 / 18.9, 68^3 17.9 /
// 19.7 against 18.9 / 21.1, 48 of 32^3 68.4 / 75.5, but 60^3 13.7 / 15.0, 80^3 24.2
// / 26.7 against 21.6 / 26.4, 96^3 34.5 / 37.6.  Node storage takes 1.17 times the
// two passes' time (64^3 18.3, 16.4), psi = exp(-1/n) in the model's terms 1.17
// times at E4 (six members of 32^3 17.7 against 18.5, 128 x 128 x 16 21.5, 19.2) and
// 1.35 times at E6 (128 x 128 x 16 27.5, 28.3; 96 x 32 x 96 32.9, 26.6), and from
// 300 000 sites on always gains (48^3 x 4 31.7, 26.2).  Below 80 000 sites moment
// steps gain (32^3 8.8, 6.8).  Short calls, FP16 48^3 E6: two steps 11.8, 13.1;
// four 11.8, 12.4; 56^3 E4 two 13.3, 14.8, sixteen 13.2, 13.1; 60^3 E6 four 18.3,
// 16.9; with psi 64^3 two 21.0, 21.9, four 20.4, 20.4.
// A group of more members than a launch takes makes several launches per step,
// each of which fills the chip by itself: all types then weigh the model against
// the two passes, FP64 and FP32 with a tenth to spare (E6 FP32, us per step: 65
// members of 24^3 60, 42; 129 of them 112, 75; 100 of 25^3 137, 69; 70 of 30^3 150,
// 83; FP64 70 of 16^3 39, 29, with psi, at twice the model's time, 59, 70; FP16
// with psi 129 of 24^3 148, 117; 130 of 16^3 54, 70).
inline bool mom_steps_pay(StorageWidth w, bool node, int order, bool psi, int64_t sites,
                          int64_t ragged, double us, int launches, int64_t steps) {
    if (w != WIDE_16 && launches > 1 &&
        us * (w == WIDE_64 && order == 6 && psi ? 2 : 1) >
            0.9 * (7 + (w == WIDE_64 ? 11.5e-5 : 6e-5) * (double)sites))
        return false;
    if (w == WIDE_64) return !(order == 6 && psi && sites < 120000);
    if (w == WIDE_32) return steps >= 3 || sites < 80000 || sites > 135000;
    if (launches == 1 && (sites < 80000 || (psi && sites >= 300000))) return true;
    if (sites < 300000 && steps < (psi || node || sites > 200000 ? 4 : 8)) return false;
    const double n = (double)sites;
    const double passes = std::max(5.5 + 3.5e-5 * n, 9.3 + 2.2e-5 * n) *
                          (1 + 0.09 * (double)ragged / n) * (node ? 1.17 : 1) *
                          (!psi ? 1 : order == 4 ? 1.17 : 1.35);
    return us < passes;
}

}  // namespace scmc
