// The rules that size launches (internal.h), which need no device: exit status 0 when every case holds.
#include <cstdio>

#include "internal.h"

using namespace sellcs;

static int failures = 0;

static void expect(bool ok, const char *what, int64_t a, int64_t b) {
    if (ok) return;
    std::fprintf(stderr, "FAIL %s (%lld, %lld)\n", what, (long long)a, (long long)b);
    ++failures;
}

// `count` matrices of n rows of len entries, chunks of 32 rows, one tile per chunk, b columns (a power
// of two from 4 on, or 1) on 256 compute units with one or two workgroups of 512 threads each
static void batch(int count, int64_t n, int64_t len, int b, int per_cu) {
    const int64_t tiles = count * ((n + 31) / 32), resident = 256 * per_cu;
    const int32_t rows = pass_rows(b, b >= 4 ? 4 : b, kPathFixed, 512);
    const int64_t passes = count * ((n + rows - 1) / rows);
    const int64_t G = batch_workgroups(tiles, std::min(resident, tiles), 16 * resident, double(passes) * index_batches(n * len, n));
    expect(G >= std::min(tiles, resident), "workgroups for the device", G, std::min(tiles, resident));
    expect(G <= std::min(tiles, 16 * resident), "workgroups at most", G, tiles);
    // no workgroup has more than three passes of one index batch per row, or one wave or one tile of work
    const double each = double(passes) * index_batches(n * len, n) / double(G);
    expect(each <= 6.0 || G == tiles || G == 16 * resident, "work per workgroup", int64_t(each), G);
    // short rows in numbers: three passes each, not one tile each
    if (len <= 8 && passes > 3 * resident && passes < 48 * resident)
        expect(G <= passes / 3, "passes per workgroup", G, passes);
}

int main() {
    for (int per_cu : {1, 2})
        for (int b : {1, 4, 8, 16, 32})
            for (int count : {1, 3, 8, 64, 1000})
                for (int64_t n : {1, 31, 33, 500, 2000, 20000, 1000000})
                    for (int64_t len : {1, 7, 9, 60, 500, 2000}) batch(count, n, len, b, per_cu);
    expect(batch_workgroups(0, 0, 4096, 0.0) == 1, "empty batch", 0, 0);
    expect(batch_workgroups(int64_t(1) << 40, 256, int64_t(1) << 20, 1e300) == 1 << 20, "bound", 0, 0);
    // lanes per row of narrow products: columns of their own on few long rows only
    expect(few_long_rows(3, 2000, 2000 * 300) && few_long_rows(7, 8192, 64 * 8192), "few long rows", 0, 0);
    expect(!few_long_rows(8, 2000, 2000 * 300) && !few_long_rows(3, 8193, 8193 * 300) && !few_long_rows(3, 2000, 2000 * 64 - 1),
           "few long rows", 1, 0);
    // cache policy: (matrix MB, vectors MB, columns, bytes of a vector element) either side of its lines
    const struct { double matrix, vectors; int b, esize, keep; } policy[] = {
        {90, 5, 8, 8, 2}, {90, 7, 8, 8, 1}, {84, 256, 16, 8, 1}, {84, 512, 32, 8, 0}, {127, 195, 8, 8, 1}, {127, 389, 16, 8, 0},
        {61, 373, 32, 8, 1}, {65, 373, 32, 8, 0}, {117, 268, 16, 4, 1}, {129, 268, 16, 4, 0}, {84, 768, 48, 8, 1},
        {176, 140, 4, 8, 1}, {176, 150, 4, 8, 0}};
    for (const auto &p : policy)
        expect(keep_in_cache(p.matrix * 1e6, p.vectors * 1e6, p.b, p.esize) == p.keep, "cache policy", int64_t(p.matrix), p.b);
    // the gradient's grid: a launch of fewer than 2^32 threads at any number of rows, all of them in one
    // pass where they are few
    for (int ll = 0; ll <= 4; ++ll)
        for (int64_t n = 1; n <= int64_t(1) << 31; n = 2 * n + 1) {
            const int64_t g = grad_grid(n, ll), per = 256 >> ll;
            expect(g >= 1 && g * 256 < (int64_t(1) << 32), "gradient threads", g, n);
            expect(n > per << 18 || (g * per >= n && (g - 1) * per < n), "gradient workgroups", g, n);
        }
    // value updates: long rows shared by workgroups until the device is busy, never more than their pieces
    for (int64_t n : {1, 255, 2000, 300000, 100000000})
        for (int64_t len : {0, 1, 8, 9, 100, 2000}) {
            const int64_t g = (n + 255) / 256, parts = update_parts(n, n * len, g);
            expect(parts >= 1 && parts <= std::max<int64_t>(1, (len + 7) / 8), "update parts", parts, len);
            expect(parts == 1 || g * parts <= 1024, "update workgroups at most", parts, n);
            expect(g * parts >= std::min<int64_t>(513, g * ((len + 7) / 8)), "update workgroups", parts, n);
        }
    if (failures) return 1;
    std::puts("launch rules ok");
    return 0;
}
