// Host-only checks of the evaluation plan (eval_plan.hpp): chunk sizes, units and
// workspace layouts over element counts, copies, columns, point counts and workspace
// sizes.  Exit status 1 on any failure.
#include <cstdio>
#include <vector>

#include "eval_plan.hpp"

using namespace nebem;

static int failures = 0;
#define CHECK(c)                                                  \
    do {                                                          \
        if (!(c)) {                                               \
            std::printf("FAIL line %d: %s\n", __LINE__, #c);      \
            ++failures;                                           \
        }                                                         \
    } while (0)

static const size_t kRecord = 8832;
static const size_t kScratch = size_t(64) << 20;  // of the allocation-free evaluation

// the sort's scratch grows with the points, in no round numbers
static size_t sort_bytes(int64_t c) { return 3001 + 17 * (size_t)c; }

static EvalShape shape(int64_t n, int ring, int ncol, bool fp64 = true)
{
    const int64_t copies = (int64_t)(2 * ring + 1) * (2 * ring + 1);
    return eval_shape(seg_plan(n, copies), fp64 && grouping_pays(n, copies), 2 * ring + 1, ncol, kRecord);
}

// every part of a layout behind the one before, 256-aligned and large enough
static void sound(const EvalShape &sh, int64_t c, size_t limit)
{
    ChunkLayout L;
    CHECK(chunk_layout(sh, c, limit, sort_bytes, L));
    const size_t u = (size_t)32 * sh.kc * (size_t)c, g = (size_t)sh.ngroup, f = (size_t)sh.nrec;
    const size_t need[] = {sh.group_bytes, L.ordered ? sort_bytes(c) : 0, L.ordered ? 4 * (size_t)c : 0,
                           L.ordered ? 24 * (size_t)c : 0, L.ordered ? u : 0, sh.part_pp * (size_t)c,
                           !L.fsplit ? 0 : !sh.grouped ? u * g * kNearParts : L.fsplit == 2 ? u * f * sh.rows : u * f,
                           !L.nsplit ? 0 : L.nsplit == 2 ? u * g * kNearRuns : u * g, L.fsplit == 2 ? u * f : 0,
                           L.nsplit == 2 ? u * g : 0};
    const size_t at[] = {L.groups, L.sort, L.perm, L.pts, L.res, L.part, L.far, L.near, L.ffold, L.nfold};
    for (int k = 0; k < 10; ++k) {
        CHECK(at[k] % 256 == 0);
        CHECK(at[k] + need[k] <= (k < 9 ? at[k + 1] : L.total));
    }
    CHECK(L.groups == 0);
    CHECK((L.nsplit > 0) == (L.fsplit > 0 && sh.grouped));
    CHECK(L.total <= limit || !L.fsplit);  // whole segments are the least there is
}

int main()
{
    const int64_t ns[] = {1, 100, 542, 1648, 8064, 19776, 41600, 74656, 300000, 3000000};
    const int64_t ms[] = {1, 64, 65, 500, 1000, 2003, 6000, 20000, 40000, 100003, 700001, 30000000};
    for (int64_t n : ns)
        for (int ring : {0, 1, 5})
            for (int ncol : {1, 3, 9})
                for (bool fp64 : {true, false})
                    for (int64_t m : ms) {
                        const EvalShape sh = shape(n, ring, ncol, fp64);
                        ChunkLayout least;
                        CHECK(chunk_layout(sh, std::min<int64_t>(m, 256), 0, sort_bytes, least) && !least.fsplit);
                        for (size_t limit : {size_t(SIZE_MAX), size_t(1) << 30, kScratch, least.total}) {
                            const int64_t c = chunk_points(sh, m, limit, sort_bytes);
                            CHECK((c > 0) == (least.total <= limit));
                            if (!c) continue;
                            CHECK(c <= m || c <= 256);
                            CHECK(c == m || c % 256 == 0);
                            ChunkLayout L;
                            CHECK(chunk_layout(sh, c, limit, sort_bytes, L) && L.total <= limit);
                            sound(sh, c, limit);
                            if (m % c) sound(sh, m % c, limit);
                            // the device is idle in whole segments only if no fewer points have room for
                            // units that fill it
                            if (L.fsplit || (c + 63) / 64 * sh.sp.nseg >= kFullWaves) continue;
                            for (int64_t d = c; d >= 256; d = d > 256 ? std::max<int64_t>(256, (d / 2) & ~(int64_t)255) : 0) {
                                ChunkLayout D;
                                CHECK(chunk_layout(sh, d, limit, sort_bytes, D));
                                const int64_t units = sh.grouped ? sh.nrec : sh.sp.nseg * eval_subunits(sh.sp);
                                CHECK(!D.fsplit || d / 64 * units < kFullWaves || d == c);
                            }
                        }
                    }
    // unit sums that do not fit are given up step by step: a GEM cell in 64 MiB
    ChunkLayout L;
    const EvalShape gem = shape(8064, 5, 1);
    for (int64_t m : {1000, 2003, 6000}) {
        CHECK(chunk_points(gem, m, kScratch, sort_bytes) == m);
        CHECK(chunk_layout(gem, m, kScratch, sort_bytes, L) && L.fsplit == 1);
    }
    // many elements, few copies: fewer points at a time instead of one wave per 64
    const EvalShape flat = shape(74656, 0, 1);
    for (size_t limit : {size_t(SIZE_MAX), kScratch}) {
        const int64_t c = chunk_points(flat, 20000, limit, sort_bytes);
        CHECK(c < 20000 && chunk_layout(flat, c, limit, sort_bytes, L) && L.fsplit);
    }
    // a device with less room than a call would like: half as much, down to the least
    for (size_t room : {size_t(0), size_t(999), size_t(1000), size_t(50000), size_t(1) << 40}) {
        const size_t got = take_workspace(900000, 1000, [&](size_t b) { return b <= room; });
        CHECK(got == (room < 1000 ? 0 : room < 50000 ? 1000 : room < 900000 ? got : 900000));
        CHECK(got <= room && (got == 0 || got >= 1000));
        if (room == 50000) CHECK(got > 25000);
    }
    // and there is a plan for every such size
    for (int64_t m : {100, 2003, 20000, 300000}) {
        ChunkLayout least;
        CHECK(chunk_layout(gem, std::min<int64_t>(m, 256), 0, sort_bytes, least));
        const int64_t c = chunk_points(gem, m, SIZE_MAX, sort_bytes);
        CHECK(chunk_layout(gem, c, SIZE_MAX, sort_bytes, L));
        for (size_t b = L.total; b > least.total; b = std::max(least.total, b / 2)) CHECK(chunk_points(gem, m, b, sort_bytes) > 0);
    }
    std::printf("%s\n", failures ? "FAIL" : "checks passed");
    return failures != 0;
}
