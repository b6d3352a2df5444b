// Every LDS access of the two-step D3Q19 kernel's lanes, host code: reads wc, rh,
// whole, xlo, xhi and the workgroup's threads per line and prints the least and the
// greatest position that any lane pulls from, and how many of the lanes that hold a
// node pull a moving value from a place other than the neighbour's.
#include <algorithm>
#include <cstdio>

#include "lbm_d3q19.h"

int main() {
    int wc, rh, whole, walls, threads;
    while (std::scanf("%d %d %d %d %d", &wc, &rh, &whole, &walls, &threads) == 5) {
        const int rw = whole ? wc : wc + 2;
        int lo = 0, hi = 0, wrong = 0;
        for (int th = 0; th < threads; ++th) {
            int ry = th / wc, rx = th % wc;
            bool in = ry < rh;
            if (!in && !whole) {
                const int q = th - rh * wc;
                ry = q >> 1;
                rx = q & 1 ? wc : -1;
                in = ry < rh;
            }
            const int t = in ? ry * rw + rx + (whole ? 0 : 1) : 0;
            const bool xlo = walls && whole && rx == 0, xhi = walls && whole && rx == wc - 1;
            const lbm::TileOffsets o = lbm::tile_offsets(in, whole != 0, rx, ry, wc, rh, xlo, xhi);
            for (int i = 0; i < 19; ++i) {
                const int at = t + (lbm::E3X[i] > 0 ? o.om : lbm::E3X[i] < 0 ? o.op : 0) +
                               (lbm::E3Y[i] > 0 ? o.od : lbm::E3Y[i] < 0 ? o.ou : 0);
                lo = std::min(lo, at);
                hi = std::max(hi, at);
                if (!in) continue;
                int cx = rx - lbm::E3X[i], cy = ry - lbm::E3Y[i];  // where the value comes from
                if (whole && !walls) cx = (cx + wc) % wc;
                const bool held = cx >= (whole ? 0 : -1) && cx < (whole ? wc : wc + 1) && cy >= 0 && cy < rh;
                if (held && at != cy * rw + cx + (whole ? 0 : 1)) ++wrong;
            }
        }
        std::printf("%d %d %d\n", lo, hi, wrong);
    }
    return 0;
}
