// The threshold searches of the selection (sl_search.h) on whole chunks of keys, as a wave calls them: by the sample's
// bracket where it serves and holds the threshold, else by the leading bits.  Keys of values, ties, zeros, infinities, NaNs of
// every payload, positions outside the tensor (-1).  The result has to be the k-th largest key, or, where no other lies between,
// a smaller value that exactly k keys reach.
#include <algorithm>
#include <cmath>
#include <cstdio>
#include <cstring>
#include <functional>
#include <random>
#include <vector>

#include "sl_search.h"

typedef std::vector<int> Keys;      // key of register r of lane l at 64 r + l

static int used_sample = 0, calls = 0;

static int threshold(const Keys &key, int k, int margin)
{
    auto all = [&](int x) { return (int)std::count_if(key.begin(), key.end(), [&](int v) { return v >= x; }); };
    const int hi = *std::max_element(key.begin(), key.end()), ks = (k + 4) >> 3;
    bool exact = false;
    ++calls;
    if (margin > 0 && sl_sample_serves(hi)) {
        int start = hi;
        for (int l = 0; l < 64; ++l) {
            int most = -1;
            for (int r = 0; r < 64; ++r) most = std::max(most, key[64 * r + l]);
            start = std::min(start, most);
        }
        auto sample = [&](int x) {
            int n = 0;
            for (int s = 0; s < 8; ++s)
                for (int l = 0; l < 64; ++l) n += key[64 * 9 * s + l] >= x;
            return n;
        };
        int from, upto;
        sl_sample_bracket(start, hi, ks, margin, sample, from, upto);
        if (from < -1 || upto <= from) return -2;
        int n_lo = all(from), n_hi = all(upto);
        if (n_lo >= k && n_hi < k) {
            ++used_sample;
            return sl_find_kth(from, upto, n_lo, n_hi, k, all, exact);
        }
    }
    if (hi <= 0) return 0;
    const int top = 31 - __builtin_clz((unsigned)hi), last = top - 11;
    if (last < 3) return sl_bisect_kth(0, hi, k, all, exact);
    const int T = sl_bisect_kth(0, hi, k, all, exact, 12);
    return exact ? T : sl_bisect_kth(T, T | ((1 << last) - 1), k, all, exact);
}

int main()
{
    std::mt19937 rng(1);
    auto key_of = [](float x) {
        int b;
        std::memcpy(&b, &x, 4);
        return b & 0x7FFFFFFF;
    };
    std::normal_distribution<float> gauss(0.f, 1e-3f);
    std::function<int()> value = [&] { return key_of(gauss(rng)); };
    std::function<int()> zero = [] { return 0; }, tiny = [&] { return (int)(rng() % 64); };
    std::function<int()> tie = [&] { return key_of((float)(rng() % 5)); }, inf = [] { return 0x7F800000; };
    std::function<int()> quiet = [] { return 0x7FC00000; }, nan = [&] { return 0x7F800001 + (int)(rng() % 0x7FFFFF); };
    std::function<int()> top = [&] { return 0x7FE00001 + (int)(rng() % 0x1FFFFE); };
    std::function<int()> last = [] { return 0x7FFFFFFE; }, outside = [] { return -1; };
    const std::function<int()> kinds[] = {value, zero, tiny, tie, inf, quiet, nan, top, last, outside};
    const int ks[] = {516, 520, 640, 1024, 1424, 2048, 3000, 4000, 4032};
    for (int k : ks) {
        const double share = k / 4096.0;
        int margin = (int)(2.5 * std::sqrt(512.0 * share * (1.0 - share))) + 1;
        if (k / 8 + margin >= 511) margin = 0;
        for (const auto &a : kinds)
            for (const auto &b : kinds)
                for (double part : {0.0, 0.02, 0.13, 0.5, 0.9})
                    for (int where = 0; where < 3; ++where) {       // b's share anywhere, in the sample, in some lanes
                        Keys key(4096);
                        for (int p = 0; p < 4096; ++p) {
                            const int r = p / 64, l = p % 64;
                            const bool is_b = where == 0 ? rng() % 10000 < part * 10000 : where == 1 ? r % 9 == 0 : l < 64 * part;
                            key[p] = is_b ? b() : a();
                        }
                        if (std::count_if(key.begin(), key.end(), [](int v) { return v >= 0; }) < k) continue;
                        const int T = threshold(key, k, margin);
                        Keys sorted = key;
                        std::nth_element(sorted.begin(), sorted.begin() + (k - 1), sorted.end(), std::greater<int>());
                        const int want = sorted[k - 1];
                        const int n = (int)std::count_if(key.begin(), key.end(), [&](int v) { return v >= T; });
                        if (T != want && !(T <= want && n == k)) {
                            std::printf("k %d: threshold %d (%d keys reach it), want %d\n", k, T, n, want);
                            return 1;
                        }
                    }
    }
    if (used_sample < calls / 20) std::printf("the sample served %d of %d chunks only\n", used_sample, calls);
    else std::puts("ok");
    return 0;
}
