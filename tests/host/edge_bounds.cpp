// Every load that a partial chunk's lanes make (sl_partial_load_at), over matrices and runs of many shapes: none leaves its
// tensor, and the elements that exist are where the lane looks for them.  Prints the first violation.
#include <algorithm>
#include <cstdio>

#include "sl_internal.h"

static bool check(long long rows, long long cols, long long offset, bool tile)
{
    const long long n = rows * cols;
    long long local = 0;
    auto chunk = [&](SlChunkDesc d) {
        d.local_chunk = (int)local++;
        if (d.rows == 64 && d.cols == 64 && d.last_cols == 64) return true;
        for (int lane = 0; lane < 64; ++lane) {
            const int lr = lane >> 4, lc = (lane & 15) * 4, room = sl_partial_room(d);
            for (int i = 0; i < 16; ++i) {
                const int e = sl_partial_exist(d, lr, lc, i);
                const unsigned place = sl_partial_origin(d, lr, lc, room) + (unsigned)i * 16u * (unsigned)d.stride;
                const unsigned at = sl_partial_load_at(e, place, room);
                const long long first = d.base - room + (at >> 2), want = d.base + (4 * i + lr) * (long long)d.stride + lc;
                bool ok = (at & 3) == 0 && first >= offset && first + 4 <= offset + n;
                if (e >= 4) ok = ok && first == want;
                else if (e > 0) ok = ok && first + sl_partial_back(e, place) == want && sl_partial_back(e, place) + e <= 4;
                if (!ok) {
                    std::printf("%lld x %lld at %lld, %s: chunk %d lane %d access %d loads from %lld\n", rows, cols, offset,
                                tile ? "tiles" : "runs", d.local_chunk, lane, i, first - offset);
                    return false;
                }
            }
        }
        return true;
    };
    SlChunkDesc d{};
    if (!tile) {
        for (long long a = 0; a < n; a += SL_CHUNK) {
            const long long nv = std::min<long long>(SL_CHUNK, n - a);
            if (nv < 4) return true;                     // (no plan takes such a chunk)
            d.base = offset + a, d.stride = 64, d.rows = (unsigned char)((nv + 63) / 64), d.cols = 64;
            d.last_cols = (unsigned char)(nv - (d.rows - 1) * 64);
            if (!chunk(d)) return false;
        }
        return true;
    }
    for (long long a = 0; a < rows; a += 64)
        for (long long b = 0; b < cols; b += 64) {
            const long long rv = std::min<long long>(64, rows - a), cv = std::min<long long>(64, cols - b);
            if (rv * cv < 4) return true;
            d.base = offset + a * cols + b, d.stride = (int)cols, d.rows = (unsigned char)rv;
            d.cols = d.last_cols = (unsigned char)cv;
            if (!chunk(d)) return false;
        }
    return true;
}

int main()
{
    for (long long offset : {0ll, 4ll, 64ll, (1ll << 33) + 4}) {
        for (long long rows : {1, 2, 3, 4, 5, 7, 63, 64, 65, 66, 127, 128, 130})
            for (long long cols = 1; cols <= 200; ++cols)
                if (!check(rows, cols, offset, true)) return 1;
        for (long long n = 4; n <= 4500; ++n)
            if (!check(1, n, offset, false)) return 1;
        for (long long n = 8190; n <= 8200; ++n)
            if (!check(1, n, offset, false)) return 1;
    }
    std::puts("ok");
    return 0;
}
