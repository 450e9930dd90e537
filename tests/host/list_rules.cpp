// The rules on a list's length that choose between the forms of a kernel, at calls that were measured on both sides of every line: a
// call that a form is slower for keeps the other one.  Prints the first row that goes the wrong way.
#include <cstdio>
#include <vector>

#include "sl_internal.h"

static int failures = 0;
static void expect(const char *what, long long n, int k, int got, int want)
{
    if (got == want) return;
    std::printf("%s, %lld chunks, k = %d: %d, want %d\n", what, n, k, got, want);
    ++failures;
}

// waves per chunk of the selection; streams: 1 frozen or Sub-k, 2 deferred, 3 with the update or from parameters
static void selection()
{
    const struct { int n, k, streams, ragged, want; } rows[] = {
        {64, 64, 1, 0, 8}, {512, 4096, 1, 0, 8}, {512, 64, 2, 0, 8}, {512, 256, 3, 0, 8}, {512, 256, 1, 1, 8},
        {1280, 64, 1, 0, 4}, {1281, 64, 1, 0, 1}, {1280, 16, 1, 0, 4}, {2048, 16, 1, 0, 1}, {1280, 136, 1, 0, 4}, {768, 256, 1, 0, 4}, {769, 256, 1, 0, 1}, {768, 512, 1, 0, 4}, {1024, 512, 1, 0, 1},
        {1280, 1024, 1, 0, 4}, {1281, 1024, 1, 0, 1}, {2220, 2048, 1, 0, 4}, {3073, 4096, 1, 0, 1},
        {6144, 64, 2, 0, 4}, {6145, 64, 2, 0, 1}, {1536, 136, 2, 0, 4}, {1537, 136, 2, 0, 1}, {1536, 256, 2, 0, 4}, {1537, 256, 2, 0, 1}, {768, 512, 2, 0, 4}, {1024, 512, 2, 0, 1},
        {2560, 1024, 2, 0, 4}, {2561, 520, 2, 0, 1}, {3072, 2048, 2, 0, 4}, {3073, 4096, 2, 0, 1},
        {6144, 128, 3, 0, 4}, {6145, 4, 3, 0, 1}, {2048, 256, 3, 0, 4}, {2049, 136, 3, 0, 1}, {768, 264, 3, 0, 4}, {769, 512, 3, 0, 1}, {3072, 1024, 3, 0, 4}, {3073, 1024, 3, 0, 1},
        {3120, 32, 1, 1, 4}, {6145, 32, 1, 1, 1}, {1360, 200, 2, 1, 4}, {916, 256, 1, 1, 4}, {2049, 256, 2, 1, 1}, {769, 512, 1, 1, 1}, {3072, 1024, 2, 1, 4},
    };
    for (const auto &r : rows) expect(r.ragged ? "selection, ragged" : "selection", r.n, r.k, sl_select_waves(r.n, r.k, r.streams, r.ragged != 0), r.want);
}

// the eager accumulate without the streaming hint
static void kept()
{
    const struct { int n, k, params, want; } rows[] = {
        {2048, 64, 0, 0}, {4096, 16, 0, 0}, {4096, 256, 0, 0}, {8192, 128, 0, 0}, {9216, 4, 0, 0}, {3072, 512, 0, 0}, {4096, 512, 0, 1}, {9216, 1024, 0, 1},
        {9217, 1024, 0, 0}, {8192, 1536, 0, 1}, {6144, 2048, 0, 0}, {4096, 512, 1, 0}, {9216, 1024, 1, 0}, {6144, 64, 1, 0},
    };
    for (const auto &r : rows) expect(r.params ? "kept, parameters" : "kept", r.n, r.k, sl_update_kept(r.n, r.k, r.params), r.want);
}

// shares of unaligned chunks from which the streaming hint is left out
static void unaligned()
{
    const struct { int n, percent, k, streams, update, params, select, apply, mom, direction, dense; } rows[] = {
        {1920, 24, 64, 2, 0, 0, 0, 0, 0, 0, 0}, {1920, 35, 64, 2, 0, 0, 0, 0, 0, 0, 1}, {1920, 50, 64, 2, 0, 0, 1, 1, 1, 1, 1},
        {5120, 25, 64, 2, 0, 0, 0, 0, 1, 0, 0}, {5120, 39, 128, 3, 1, 0, 0, 0, 1, 0, 0}, {5120, 40, 128, 3, 1, 0, 0, 0, 1, 1, 1},
        {9600, 24, 512, 3, 1, 0, 0, 0, 0, 0, 0}, {9600, 25, 512, 3, 1, 0, 1, 1, 1, 0, 0}, {9600, 25, 512, 3, 1, 1, 0, 1, 1, 0, 0}, {9600, 25, 256, 3, 1, 0, 0, 1, 1, 0, 0},
        {9600, 50, 1024, 3, 1, 1, 1, 1, 1, 1, 1}, {9600, 100, 64, 1, 0, 0, 0, 1, 1, 1, 1}, {25600, 25, 64, 2, 0, 0, 0, 1, 1, 0, 0}, {25600, 50, 64, 2, 0, 0, 1, 1, 1, 1, 1},
        {25600, 50, 256, 3, 0, 1, 1, 1, 1, 1, 1}, {12288, 50, 512, 3, 1, 0, 1, 1, 1, 1, 1}, {25600, 50, 512, 3, 1, 0, 0, 1, 1, 1, 1}, {25600, 75, 512, 3, 1, 1, 1, 1, 1, 1, 1},
    };
    for (const auto &r : rows) {
        sl_plan p{};
        p.k = r.k, p.n_chunks = r.n, p.n_unaligned = (int64_t)r.n * r.percent / 100;
        expect("unaligned, selection", r.n, r.k, sl_select_unaligned(&p, r.streams, r.update != 0, r.params != 0), r.select);
        expect("unaligned, aggregate", r.n, r.k, sl_rows_unaligned(&p, sl_apply_kept_from(&p, false)), r.apply);
        expect("unaligned, momentum", r.n, r.k, sl_rows_unaligned(&p, sl_apply_kept_from(&p, true)), r.mom);
        expect("unaligned, direction", r.n, r.k, sl_rows_unaligned(&p, SL_DIRECTION_KEPT_FROM), r.direction);
        expect("unaligned, dense", r.n, r.k, sl_rows_unaligned(&p, sl_dense_kept_from(&p)), r.dense);
    }
}

// whole pieces written back by Sub-k
static void pieces()
{
    const struct { int n, k, want; } rows[] = {{16383, 64, 0}, {16384, 64, 1}, {16384, 4, 0}, {98304, 8, 0}, {49152, 14, 0}, {16384, 16, 1}, {98304, 4096, 1}};
    for (const auto &r : rows) expect("pieces", r.n, r.k, sl_subk_pieces(r.n, r.k), r.want);
}

// waves per chunk of the aggregates
static void aggregates()
{
    const struct { int n, k, bits, R, coded, mom, want; } rows[] = {
        {64, 64, 2, 4, 0, 0, 8}, {512, 256, 2, 8, 0, 0, 8}, {513, 256, 2, 5, 0, 0, 1}, {1024, 256, 2, 8, 0, 0, 1}, {1024, 256, 2, 4, 0, 0, 4}, {1024, 256, 2, 8, 0, 1, 4},
        {1024, 256, 4, 8, 0, 0, 4}, {1024, 256, 32, 8, 0, 0, 4}, {1024, 248, 2, 8, 0, 0, 4}, {1025, 256, 2, 4, 0, 0, 4}, {1025, 256, 2, 5, 0, 1, 1}, {2048, 64, 2, 8, 0, 0, 4},
        {2049, 64, 2, 1, 0, 0, 1}, {64, 264, 2, 1, 0, 0, 1}, {64, 16, 2, 9, 0, 0, 1}, {256, 128, 2, 8, 1, 0, 8}, {257, 64, 2, 8, 1, 0, 1}, {1024, 64, 2, 4, 1, 1, 4}, {1025, 64, 2, 1, 1, 0, 1},
    };
    for (const auto &r : rows) {
        sl_plan p{};
        p.k = r.k, p.bits = r.bits, p.n_chunks = r.n;
        expect(r.coded ? "aggregate, coded" : "aggregate, plain", r.n, r.k, sl_apply_waves(&p, r.R, r.coded != 0, r.mom != 0), r.want);
    }
}

// pieces whose sums a launch of their own takes: those of the large tensors, and no others
static void tensor_pieces()
{
    std::vector<SlTensorDev> list;
    long long chunk0 = 0;
    for (long long n : {3ll, 25152ll, 4096ll, 10240ll, 10241ll, 10496ll, 1ll}) {
        SlTensorDev t{};
        t.chunk0 = chunk0, t.n_chunks = n;
        list.push_back(t);
        chunk0 += n;
    }
    std::vector<SlPiece> got;
    sl_make_pieces(list, got);
    size_t at = 0;
    for (const SlTensorDev &t : list) {
        const bool split = t.n_chunks > 10240;
        expect("first piece", t.n_chunks, 0, (int)t.piece0, split ? (int)at : -1);
        for (long long c = 0; split && c < t.n_chunks; c += 256, ++at) {
            const bool there = at < got.size();
            expect("piece begins", t.n_chunks, 0, there ? got[at].chunk0 : -1, (int)(t.chunk0 + c));
            expect("piece holds", t.n_chunks, 0, there ? got[at].n_chunks : -1, (int)(t.n_chunks - c < 256 ? t.n_chunks - c : 256));
        }
    }
    expect("pieces", chunk0, 0, (int)got.size(), 99 + 41 + 41);
}

int main()
{
    selection();
    kept();
    unaligned();
    pieces();
    tensor_pieces();
    aggregates();
    if (failures) return 1;
    std::puts("ok");
    return 0;
}
