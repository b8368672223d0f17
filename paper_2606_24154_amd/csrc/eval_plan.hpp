// eval_plan.hpp -- how an evaluation is cut up: element segments, groups, the
// points taken at a time, the units of a launch and the workspace they need (host
// code and sizes shared with the kernels, no HIP calls).
#pragma once

#include <algorithm>
#include <cstddef>
#include <cstdint>

#if defined(__HIPCC__)
#define NEBEM_HD __host__ __device__
#else
#define NEBEM_HD
#endif

namespace nebem {

constexpr int kMultiCols = 4;  // density columns per evaluation launch

// Element segments of an evaluation: nseg contiguous ranges of segsz elements
// (the last may be shorter), about kSegWork interactions per point each.  Every
// evaluation path (stateless, session, ordered, several-column, serving) splits a
// geometry's elements into the same segments, evaluates each (point, segment)
// pair as an independent unit and adds the segments' partial sums in segment
// order.  The plan depends on the element count and the copies only, so a point's
// result does not depend on how many other points share its launch; and a launch of
// a few hundred thousand points over tens of thousands of elements still has ~10^5
// workgroups, so its last round of waves is a small share of it (one workgroup per
// 256 points over all elements would leave a 200 000-point launch at 1.5 rounds).
constexpr double kSegWork = 1.2e5;
constexpr int kMaxSeg = 64;
struct SegPlan {
    int nseg, segsz;
};
inline SegPlan seg_plan(int64_t n, int64_t copies)
{
    SegPlan p = {1, (int)(n > 0 ? n : 1)};
    if (n <= 0) return p;
    const double per_pt = (double)n * (double)copies;
    int nseg = (int)(per_pt / kSegWork + 0.5);
    nseg = nseg < 1 ? 1 : (nseg > kMaxSeg ? kMaxSeg : nseg);
    if (nseg > n) nseg = (int)n;
    p.segsz = (int)((n + nseg - 1) / nseg);
    p.nseg = (int)((n + p.segsz - 1) / p.segsz);
    return p;
}

// Groups of an FP64 evaluation (group_kernels.hip, group_far.hpp): runs of
// kGroupElems consecutive elements of a segment, groups_per_seg of them per
// segment (fewer in a short last one).
constexpr int kGroupElems = 64;
constexpr int kNearParts = 4;  // runs of 16 elements per group, units of an ungrouped split evaluation
constexpr int kNearRuns = 8;   // runs of 8 elements per group, units of a split near pass
inline int groups_per_seg(const SegPlan &sp) { return (sp.segsz + kGroupElems - 1) / kGroupElems; }
inline int eval_subunits(const SegPlan &sp) { return groups_per_seg(sp) * kNearParts; }
// Far expansions of a segment: one per group, then one per kSuper consecutive
// groups for the copies far from all of them, and in geometries of many groups
// (far_levels) one per kSuper of those.
constexpr int kSuper = 4;
NEBEM_HD inline int parents_of(int n) { return (n + kSuper - 1) / kSuper; }
NEBEM_HD inline int records_of(int groups, int levels)
{
    return groups + parents_of(groups) + (levels > 1 ? parents_of(parents_of(groups)) : 0);
}
// With 650 groups (double THGEM, 40 000 points) the second level takes 59 ms to 52; with
// 126 (GEM cell) it saves 1 % of 200 000 points and costs 64 points 6 %.
inline int far_levels(const SegPlan &sp) { return (int64_t)sp.nseg * groups_per_seg(sp) >= 256 ? 2 : 1; }
inline int records_per_seg(const SegPlan &sp) { return records_of(groups_per_seg(sp), far_levels(sp)); }

// Whether an FP64 evaluation (without a hole in its lattice) takes far copies of
// whole groups by their expansions.  Grouping pays when a point meets many copies far
// from it: from about 65 000 element copies (a GEM cell with its first two rings of
// copies has 200 000) the moments' launch is a small share even of a 64-point call.
// Below, and for geometries without copies and fewer elements, nearly every group is
// near and the plain kernels do the same work without the tests.
inline bool grouping_pays(int64_t n, int64_t copies) { return (double)n * (double)copies >= 65536.0; }

struct EvalShape {
    SegPlan sp;
    int kc;       // columns per launch
    bool grouped;  // FP64 with far copies of whole groups
    int64_t ngroup, nrec, rows;  // groups of the plan, far expansions, lattice rows of one
    size_t part_pp;    // partial-sum bytes per point (0: one segment, no partials)
    size_t group_bytes;  // the groups' records
};

// rows: lattice rows (reflections x translations along a1); record_bytes: of one group
inline EvalShape eval_shape(const SegPlan &sp, bool grouped, int64_t rows, int ncol, size_t record_bytes)
{
    EvalShape sh;
    sh.sp = sp;
    sh.kc = ncol < kMultiCols ? ncol : kMultiCols;
    sh.grouped = grouped;
    sh.ngroup = (int64_t)sp.nseg * groups_per_seg(sp);
    sh.nrec = (int64_t)sp.nseg * records_per_seg(sp);
    sh.rows = rows;
    sh.part_pp = sp.nseg > 1 || grouped ? (size_t)32 * sh.kc * sp.nseg : 0;
    // behind the records, the order of the segments
    sh.group_bytes = grouped ? (size_t)sh.nrec * record_bytes * sh.kc + (size_t)((sp.nseg + 1) / 2) * 8 : 0;
    return sh;
}

// Units of an evaluation of c points: whole segments once these alone are several
// rounds of waves (8 segments of a GEM cell: from 65 536 points), groups below that,
// and rows / runs of groups when even the groups leave SIMDs without a wave (1024
// SIMDs; 64 points of a GEM cell have 160 expansions, 1760 row waves; at 2003 points,
// 5120 and 56 320 waves, the call takes 3.14 ms by expansions and 2.96 by rows).  No
// result bit depends on the choice.  A split needs its unit sums in memory: at most
// kSplitBudget (kPartBudget where nothing is grouped).
constexpr size_t kPartBudget = size_t(512) << 20;  // preferred bytes of segment partial sums per chunk
constexpr size_t kSplitBudget = size_t(384) << 20;
constexpr int64_t kMaxUnits = 65535;  // grid y
constexpr int64_t kFullWaves = 2048;  // two waves on each of 1024 SIMDs
inline void pick_splits(const EvalShape &sh, int64_t c, int &far, int &near)
{
    const int64_t waves = (c + 63) / 64;
    far = near = 0;
    if (waves * sh.sp.nseg >= 4 * kFullWaves) return;
    const int64_t pp = (int64_t)32 * sh.kc * c;
    const int64_t most = (int64_t)(sh.grouped ? kSplitBudget : kPartBudget);
    auto fits = [&](int64_t units) { return units <= kMaxUnits && units * pp <= most; };
    if (!sh.grouped) {
        far = fits((int64_t)sh.sp.nseg * eval_subunits(sh.sp)) ? 1 : 0;
        return;
    }
    if (!fits(sh.nrec)) return;
    far = waves * sh.nrec < 8 * kFullWaves && fits(sh.nrec * sh.rows) ? 2 : 1;
    near = waves * sh.ngroup < 4 * kFullWaves && fits(sh.ngroup * kNearRuns) ? 2 : 1;
}

// Workspace layout of one chunk of c points: the groups' records (at 0 in every
// chunk, so that they are computed once), [sort scratch | perm | sorted points |
// sorted results (kc columns)] when ordered, then the partial sums and the finer
// units' sums.
constexpr int64_t kOrderMin = 65;  // points are taken in Morton order: more than one wave
struct ChunkLayout {
    bool ordered;
    int fsplit, nsplit;
    size_t groups, sort, sort_ws, perm, pts, res, part, far, near, ffold, nfold, total;
};

// `limit`: bytes at hand.  Unit sums that do not fit are given up in steps: the
// rows of expansions, the runs of groups, then both passes' groups.  sort_bytes(c):
// scratch of the sort of c points (0: error, and chunk_layout returns false).
template <class SortBytes>
bool chunk_layout(const EvalShape &sh, int64_t c, size_t limit, SortBytes &&sort_bytes, ChunkLayout &L)
{
    size_t off = 0;
    auto take = [&](size_t b) {
        const size_t o = off;
        off += (b + 255) & ~size_t(255);
        return o;
    };
    L.ordered = c >= kOrderMin;
    L.groups = take(sh.group_bytes);
    L.sort_ws = 0;
    if (L.ordered && !(L.sort_ws = sort_bytes(c))) return false;
    L.sort = take(L.sort_ws);
    L.perm = take(L.ordered ? 4 * (size_t)c : 0);
    L.pts = take(L.ordered ? 24 * (size_t)c : 0);
    L.res = take(L.ordered ? 32 * (size_t)sh.kc * (size_t)c : 0);
    L.part = take(sh.part_pp * (size_t)c);
    const size_t base = off;
    pick_splits(sh, c, L.fsplit, L.nsplit);
    for (;;) {
        const size_t unit = (size_t)32 * sh.kc * (size_t)c, g = (size_t)sh.ngroup, f = (size_t)sh.nrec;
        L.far = take(!L.fsplit ? 0 : !sh.grouped ? unit * g * kNearParts : unit * f * (L.fsplit == 2 ? sh.rows : 1));
        L.near = take(L.nsplit ? unit * g * (L.nsplit == 2 ? kNearRuns : 1) : 0);
        L.ffold = take(L.fsplit == 2 ? unit * f : 0);
        L.nfold = take(L.nsplit == 2 ? unit * g : 0);
        L.total = off;
        if (off <= limit || !L.fsplit) return true;
        off = base;
        if (L.fsplit == 2)
            L.fsplit = 1;
        else if (L.nsplit == 2)
            L.nsplit = 1;
        else
            L.fsplit = L.nsplit = 0;
    }
}

// Points taken at a time (of m), and their layout within `limit` bytes: the most
// whose partial sums stay within kPartBudget and whose workspace fits, in chunks of
// equal size (a short last chunk would be a launch too small to fill the device).
// Fewer where whole segments of that many points would leave most of the device
// idle and the finer units' sums only fit for fewer: 20 000 points at 74 656
// elements without copies are 313 waves of one segment (106 ms), or four times 120 000
// waves of expansions (12 ms), whose 1532 sums would be 0.98 GB at once; 40 000 points at
// 19 776 elements x 9 copies 74 -> 11 ms.  From kFullWaves on the two come out alike
// (140 000 points, 93 ms in whole segments).  0: no chunk fits (or the sort's size is
// not known).
template <class SortBytes>
int64_t chunk_points(const EvalShape &sh, int64_t m, size_t limit, SortBytes &&sort_bytes)
{
    int64_t c = m;
    if (sh.part_pp) {
        const int64_t lim = (int64_t)(kPartBudget / sh.part_pp) & ~(int64_t)255;
        c = std::min<int64_t>(m, std::max<int64_t>(lim, 256));
    }
    auto half = [](int64_t v) { return std::max<int64_t>(256, (v / 2) & ~(int64_t)255); };
    ChunkLayout L;
    for (;; c = half(c)) {
        if (!chunk_layout(sh, c, limit, sort_bytes, L)) return 0;
        if (L.total <= limit) break;
        if (c <= 256) return 0;
    }
    if (!L.fsplit && (c + 63) / 64 * sh.sp.nseg < kFullWaves)
        for (int64_t d = c; d > 256;) {
            d = half(d);
            if (!chunk_layout(sh, d, limit, sort_bytes, L)) return 0;
            if (L.fsplit) {
                const int64_t units = sh.grouped ? sh.nrec : sh.sp.nseg * eval_subunits(sh.sp);
                if (d / 64 * units >= kFullWaves) c = d;
                break;
            }
        }
    const int64_t nch = (m + c - 1) / c;
    const int64_t even = ((m + nch - 1) / nch + 255) & ~(int64_t)255;
    return even < c ? even : c;
}

// Workspace of a call: `want` bytes, or where the device has no room for them
// half as many and so on, at least `least` (a call then takes coarser units and fewer
// points at a time).  The finer units' sums are most of what a mid-sized call wants:
// 20 000 points of a GEM cell 0.2 GB, its partial sums alone 5 MB.  alloc(bytes):
// whether it was given.  Returns the bytes, 0 if there is no room for `least`.
template <class Alloc>
size_t take_workspace(size_t want, size_t least, Alloc &&alloc)
{
    for (size_t b = want;; b = std::max(least, b / 2)) {
        if (alloc(b)) return b;
        if (b <= least) return 0;
    }
}

}  // namespace nebem
