// Which lane holds which sum after a halving exchange over the lanes of a wave
// (sum_values in np_eigen.hip).  Plain C++, so that the host can check it.
#pragma once

namespace np {

struct LaneSum {
    int slot;       // the value whose sum the lane ends with
    bool first;     // the one lane that stores it
};

// n <= w values per lane, summed over groups of w lanes (w a power of two):
// over each lane bit, from w / 2 down, the lanes with the bit clear keep the
// first (n + 1) / 2 of their values and the others the rest, until one is left,
// which all further exchanges add up.  An odd count leaves the upper lanes a
// padding zero as their last value.  Halving the rest numbers it like a value
// of the next group, so `real` counts the values that are no padding: lanes
// left with padding alone are never first.
constexpr LaneSum lane_sum(int w, int n, int lane) {
    int slot = 0, real = n;
    bool first = true;
    for (int bit = w / 2; bit > 0; bit /= 2) {
        const bool up = (lane & bit) != 0;
        if (n == 1) {
            first = first && !up;
            continue;
        }
        const int h = (n + 1) / 2;
        slot += up ? h : 0;
        real = up ? real - h : (real < h ? real : h);
        n = h;
    }
    return {slot, first && real > 0};
}

// Every value is stored by exactly one lane of the group.
constexpr bool lane_sum_complete(int w, int n) {
    for (int s = 0; s < n; ++s) {
        int owners = 0;
        for (int lane = 0; lane < w; ++lane) {
            const LaneSum o = lane_sum(w, n, lane);
            owners += o.first && o.slot == s ? 1 : 0;
        }
        if (owners != 1) return false;
    }
    for (int lane = 0; lane < w; ++lane) {
        const LaneSum o = lane_sum(w, n, lane);
        if (o.first && (o.slot < 0 || o.slot >= n)) return false;
    }
    return true;
}

}  // namespace np
