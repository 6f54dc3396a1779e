// Every record that is taken from the queue fits a lane's part of the stack,
// at the smallest part that the host lays out, and every frame of a search
// is taken.
#include <cstdio>
#include <initializer_list>

#include "mcs_layout.h"

int main() {
    int bad = 0;
    for (int word : {4, 8, 16, 32})
        for (int m = 1; m <= 254 && m <= 8 * word; m++) {
            const int cap = mcs::lane_hdr_entries(word) + m, frames = m + 1;
            for (int x = 0; x <= 255; x++) {
                const bool k = mcs::record_fits(0, x, 0, 1, frames), d = mcs::record_fits(0, 0, x, 1, frames);
                bad += k && mcs::lane_hdr_entries(word) + x > cap;
                bad += d && (x + 3) / 4 * 8 > mcs::lane_map_bytes_for(m);
                bad += x <= m && !(k && d);
            }
            bad += mcs::record_fits(3, 1, 1, 3, frames) || mcs::record_fits(-1, 1, 1, 3, frames);
        }
    std::printf("bad %d\n", bad);
    return bad != 0;
}
