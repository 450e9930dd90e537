// The searches for a chunk's threshold, the k-th largest of its keys, by counts of the keys that reach a value: plain integer
// code, which a wave runs on uniform values; the host tests compile it as it stands.
#pragma once

#ifdef __HIPCC__
#include "sl_device.h"
#define SL_SEARCH SL_DEV
#define SL_SEARCH_UNIFORM(v) sl_uniform(v)
#define SL_SEARCH_RCP(v) __builtin_amdgcn_rcpf(v)
#else
#define SL_SEARCH inline
#define SL_SEARCH_UNIFORM(v) (v)
#define SL_SEARCH_RCP(v) (1.0f / (v))
#endif

// A threshold T in [lo, hi] with count_ge(T) >= k, given count_ge(lo) >= k and 0 <= lo <= hi: the first one met that
// exactly k keys reach (`exact`; among n keys that takes about log2(n) steps, not one per bit), else, with ties, the
// largest with count_ge(T) >= k.  All values are wave-uniform.
// With `steps` > 0 only that many bits below the highest one in which lo and hi differ are
// decided and the rest left zero: a value that is not above the exact answer and still has
// count_ge >= k.
template <class CountGE>
SL_SEARCH int sl_bisect_kth(int lo, int hi, int k, CountGE count_ge, bool &exact, int steps = 0)
{
    exact = false;
    if (lo >= hi) return lo;
    const int top = 31 - __builtin_clz((unsigned)(lo ^ hi));
    const int last = steps > 0 ? (top >= steps ? top - steps + 1 : 0) : 0;
    int T = hi & ~(int)((2u << top) - 1u);
    for (int b = top; b >= last; --b) {
        const int cand = T | (1 << b), n = count_ge(cand);
        if (n >= k) T = cand;
        if (n == k) {
            exact = true;
            break;
        }
    }
    return T;
}

// A threshold T that exactly k keys reach, or, with ties, the largest that at least k reach (`exact` says which), given
// count_ge(lo) = n_lo >= k > n_hi = count_ge(hi) and lo < hi; afterwards hi and n_hi are the next value tried above
// T (T + 1, unless `exact`) and its count.  Steps go to where k would lie if the keys between lo and hi were spread evenly -
// three or four of them reach it among hundreds of keys - and every third one to the middle, which bounds their number
// whatever the keys.  With `steps` > 0 only that many are taken.  All values are wave-uniform.
template <class CountGE>
SL_SEARCH int sl_find_kth(int lo, int &hi, int &n_lo, int &n_hi, int k, CountGE count_ge, bool &exact, int steps = 0)
{
    exact = n_lo == k;
    for (int it = 1; !exact && hi - lo > 1 && it != steps; ++it) {
        int mid = lo + ((hi - lo) >> 1);
        if (it % 3) {
            const float part = (float)(2 * (n_lo - k) + 1) * SL_SEARCH_RCP((float)(2 * (n_lo - n_hi)));
            mid = SL_SEARCH_UNIFORM(lo + (int)((float)(hi - lo) * part));
            mid = mid < hi ? mid : hi - 1;
            mid = mid > lo ? mid : lo + 1;
        }
        const int n = count_ge(mid);
        exact = n == k;
        if (n >= k) lo = mid, n_lo = n;
        else hi = mid, n_hi = n;
    }
    return lo;
}

// Does the sample serve a chunk whose largest key is hi?  Up to infinity's key: above that - NaN, whose keys reach 2^31 - 1 -
// the bracket's growing steps and its bounds could pass what an int holds.
SL_SEARCH bool sl_sample_serves(int hi) { return hi > 0 && hi <= 0x7F800000; }

// Keys [from, upto) between which the chunk's k-th largest probably lies, from the counts of a sample in which its rank is about
// ks: the sample's keys of rank ks + margin and ks - margin, found in a few steps each.  `start`: where the search begins, at most hi.
template <class CountGE>
SL_SEARCH void sl_sample_bracket(int start, int hi, int ks, int margin, CountGE count_sample, int &from, int &upto)
{
    // the bracket's lower end: the lanes' largest keys are about the chunk's upper 64th, their smallest a start that
    // outliers do not move; from there down by growing steps, then between the last two
    from = start;
    int to = hi + 1, n_to = 0, n_from = count_sample(from);
    for (int d = 1 << 22; n_from < ks + margin && from > 0; d <<= 1) {
        to = from, n_to = n_from;
        from = d < from ? from - d : 0;
        n_from = count_sample(from);
    }
    bool exact = false;
    if (n_from >= ks + margin) from = sl_find_kth(from, to, n_from, n_to, ks + margin, count_sample, exact, 8);
    // its upper end, up from there in the same way
    upto = from;
    int n_upto = n_from, beyond = hi + 1, n_beyond = 0;
    for (int d = 1 << 21; d < hi - upto; d <<= 1) {
        const int n = count_sample(upto + d);
        if (n < ks - margin) {
            beyond = upto + d, n_beyond = n;
            break;
        }
        upto += d, n_upto = n;
    }
    if (beyond > upto) upto = sl_find_kth(upto, beyond, n_upto, n_beyond, ks - margin, count_sample, exact, 8);
    if (upto <= from) upto = beyond;
}
