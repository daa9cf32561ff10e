// Host emulation of the halving exchange of sum_values: lane l of a wave starts
// with n values, exchanges them bit by bit, and stores what it is left with at
// lane_sum's slot.  Every sum must be stored once, by a lane that holds it.
#include <cstdio>
#include <vector>

#include "np_lanes.h"

static int check(int w, int n) {
    std::vector<std::vector<double>> v(64, std::vector<double>(n));
    for (int l = 0; l < 64; ++l)
        for (int i = 0; i < n; ++i) v[l][i] = (double)((l + 1) * (i + 3) % 97 + 1);
    std::vector<std::vector<double>> x = v;
    for (int bit = w / 2; bit > 0; bit /= 2) {
        const int c = (int)x[0].size(), h = (c + 1) / 2;
        std::vector<std::vector<double>> r(64, std::vector<double>(h));
        for (int l = 0; l < 64; ++l)
            for (int i = 0; i < h; ++i) {
                const int j = c > 1 && (l & bit) ? i + h : i;
                r[l][i] = j < c ? x[l][j] + x[l ^ bit][j] : 0.0;
            }
        x = r;
    }
    int bad = 0;
    for (int g = 0; g < 64; g += w) {
        std::vector<int> stores(n, 0);
        for (int l = g; l < g + w; ++l) {
            const np::LaneSum o = np::lane_sum(w, n, l & (w - 1));
            if (!o.first) continue;
            if (o.slot < 0 || o.slot >= n) { ++bad; continue; }
            double want = 0.0;
            for (int k = g; k < g + w; ++k) want += v[k][o.slot];
            bad += x[l][0] != want;
            ++stores[o.slot];
        }
        for (int s = 0; s < n; ++s) bad += stores[s] != 1;
    }
    if (bad) std::printf("w %d n %d: %d wrong or missing sums\n", w, n, bad);
    return bad;
}

int main() {
    int bad = 0;
    for (int w : {32, 64})
        for (int n = 1; n <= 16; ++n) bad += check(w, n);
    std::printf("%d failure(s)\n", bad);
    return bad != 0;
}
