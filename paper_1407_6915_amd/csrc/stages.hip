// Kernels and planner of the run-time radix schedules (stages.hpp).
//
// A workgroup holds a tile of transforms in LDS and walks the schedule's
// stages: each thread takes the butterflies g = tid, tid + threads, .. of
// the whole tile, reads them into registers (from HBM in the first stage),
// waits until every thread has read, and writes the results where the
// Stockham order wants them (to HBM in the last stage).  The radix of a
// stage is a uniform switch, so one kernel serves every length.
//
// Bound by HBM: 16 B/sample in one pass, 32 in two, where one launch per
// radix moved 16 B/sample per stage with scattered stores.  What keeps a
// pass below the copy rate of 5.8 TB/s is the LDS exchange between stages
// (about 10 % of a pass each) and, above 10000 points or in tiles of more
// than half a CU's LDS, that little of a tile's loads overlaps another's
// stages: 4.1 to 5.0 TB/s up to 125 points, 5.3 to 5.7 with two stages, 4.4 to 5.0
// with three, 3.4 to 4.0 from 10000 points on; two passes move 4.4 to 5.4 with
// tiles of two workgroups a CU and 2.8 to 4.2 with larger ones (2^26 samples).  The
// bytes are the compulsory ones: partial lines add 0 to 2 % to a pass (12 % to the
// writes of 2048-point rows in 8-row tiles).
//
// Products fuse into additions within an expression, as the source has them, and not
// across: a segment's bits then do not depend on the copy of an unrolled loop, or
// on the form of the kernel, that a butterfly falls to.
#pragma clang fp contract(on)
#include "stages.hpp"

#include <algorithm>
#include <cmath>
#include <cstring>

#include "runtime.hpp"
#include "stages_device.hpp"

namespace fftseg {
namespace {

using namespace stages;

template <int D, int F>
__global__ void STAGES_KERNEL(F, false)
    stages_segments_kernel(const c32 *in, c32 *out, const c32 *__restrict__ tw, LdsSched s,
                           int segs, uint64_t batch, uint64_t hop,
                           const float *__restrict__ window)
{
    const uint64_t seg = (uint64_t)blockIdx.x * (unsigned)segs;
    const int have = (int)(batch - seg < (uint64_t)segs ? batch - seg : (uint64_t)segs);
    const SegmentIo io{in + seg * hop, out + seg * (unsigned)s.n, window, hop, s.n, have};
    run_stages<D, F>(io, s, stage_lds, tw);
}

// Segments of one stage (3 and 5 points; 2 and 4 have compiled tiles): a segment a
// thread, no LDS.  Bound by HBM; in the kernel above, whose registers are those of a
// 25-point butterfly, four waves a SIMD were too few for the short loads (2^24
// samples of 3 points 45 us, here 40; of 5 points 60 and 43).  The grid is bounded, and
// the threads walk: a launch holds fewer than 2^32 threads.
template <int R, int D>
__global__ void __launch_bounds__(256)
    stages_short_kernel(const c32 *in, c32 *out, uint64_t batch, uint64_t hop,
                        const float *__restrict__ window)
{
    for (uint64_t seg = (uint64_t)blockIdx.x * 256 + threadIdx.x; seg < batch;
         seg += (uint64_t)gridDim.x * 256) {
        const c32 *x = in + seg * hop;
        c32 v[R];
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = x[r];
        if (window)
#pragma unroll
            for (int r = 0; r < R; ++r)
                v[r] = c32{v[r].x * window[r], v[r].y * window[r]};
        dft<R, D>(v);
        c32 *y = out + seg * R;
#pragma unroll
        for (int r = 0; r < R; ++r)
            y[r] = v[r];
    }
}

template <int D, int F>
__global__ void STAGES_KERNEL(F, true)
    stages_columns_kernel(const c32 *in, c32 *ybuf, const c32 *__restrict__ tw,
                          const c64 *__restrict__ tl, const c64 *__restrict__ th, int sh,
                          LdsSched s, int n2, int lc, int lr, unsigned blocks, uint64_t tiles,
                          uint64_t ysamples, uint64_t hop, const float *__restrict__ window)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const int first = (int)(t - seg * blocks) << lc;
    ColumnIo<false, false> io{in + seg * hop, ybuf + seg * ysamples, window, tl, th, nullptr, sh,
                              n2, first, lc, lr, (unsigned)s.n};
    io.ws = column_factors(io, s);
    run_stages<D, F>(io, s, stage_lds, tw);
}

template <int D, int F>
__global__ void STAGES_KERNEL(F, true)
    stages_middle_columns_kernel(c32 *ybuf, const c32 *__restrict__ tw,
                                 const c64 *__restrict__ tl, const c64 *__restrict__ th, int sh,
                                 LdsSched s, int n1, int n3, int lr, unsigned blocks,
                                 uint64_t tiles, uint64_t ysamples)
{
    // (tile = (segment, row block, column j), j fastest)
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t q = t / (unsigned)n3, seg = q / blocks;
    const int j = (int)(t - q * (unsigned)n3), blk = (int)(q - seg * blocks);
    const MiddleIo io{ybuf + seg * ysamples +
                          (((uint64_t)blk * (unsigned)s.n * (unsigned)n3 + (unsigned)j) << lr),
                      tl, th,
                      two_level_root(tl, th, sh, (unsigned)j * (unsigned)s.st[s.ns - 1].nb),
                      sh, n3, j, n1 - (blk << lr), lr};
    run_stages<D, F>(io, s, stage_lds, tw);
}

// n2: rows of s.n points that a row of Y consists of (1 in two passes)
template <int D, int F>
__global__ void STAGES_KERNEL(F, false)
    stages_rows_kernel(const c32 *ybuf, c32 *out, const c32 *__restrict__ tw, LdsSched s, int n1,
                       int n2, int lr, unsigned blocks, uint64_t tiles, uint64_t ysamples)
{
    // (tile = (segment, k2, row block), the block fastest: neighbours share
    // the output's lines where n1 is no multiple of 16)
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t q = t / blocks, seg = q / (unsigned)n2;
    const unsigned blk = (unsigned)(t - q * blocks), k2 = (unsigned)(q - seg * (unsigned)n2);
    const RowIo<false> io{
        ybuf + seg * ysamples + (((uint64_t)blk * (unsigned)n2 + k2) << lr) * (unsigned)s.n,
        out + seg * ((uint64_t)n1 * (unsigned)n2 * (unsigned)s.n) + (uint64_t)k2 * (unsigned)n1,
        n1, (int)(blk << lr), lr, n1 * n2};
    run_stages<D, F>(io, s, stage_lds, tw);
}

// ---------------------------------------------------------------------------
// planner

constexpr int kRadixList[] = {32, 30, 27, 25, 24, 20, 18, 16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2};

// fewest stages, then the smallest sum of radices (the work of a stage grows
// with neither, its registers and idle threads do)
void best_radices(int n, int from, bool wide, std::vector<int> &cur, std::vector<int> &best)
{
    if (n == 1) {
        auto sum = [](const std::vector<int> &v) {
            int s = 0;
            for (int r : v)
                s += r;
            return s;
        };
        if (best.empty() || cur.size() < best.size() ||
            (cur.size() == best.size() && sum(cur) < sum(best)))
            best = cur;
        return;
    }
    // (radices do not increase: at least this many more)
    size_t need = 0;
    for (int left = n; left > 1; left = (left + kRadixList[from] - 1) / kRadixList[from])
        ++need;
    if (!best.empty() && cur.size() + need > best.size())
        return;
    for (int i = from; i < (int)(sizeof(kRadixList) / sizeof(kRadixList[0])); ++i) {
        // (one stage of a composite length would put the lanes of a load n
        // samples apart: two stages ran at 4.6 TB/s where one ran at 2.8)
        if (n % kRadixList[i] || (!wide && kRadixList[i] > 16 && kRadixList[i] != 25) ||
            (cur.empty() && n == kRadixList[i] && n > 5))
            continue;
        cur.push_back(kRadixList[i]);
        best_radices(n / kRadixList[i], i, wide, cur, best);
        cur.pop_back();
    }
}

}  // namespace

bool lds_schedule(int n, LdsSched *s, bool wide, int group)
{
    std::vector<int> cur, best;
    best_radices(n, 0, wide, cur, best);
    if (best.empty() || (int)best.size() > kMaxLdsStages)
        return false;
    // the smallest odd radix first: the first stage writes LDS at a stride of
    // its radix, which odd strides spread over all banks.  Whole segments without an
    // odd radix: the one with the fewest factors of two (20480 points as 20 32 32
    // in place of 32 32 20: one segment 20.2 us to 14.0, 2^24 samples 94 to 77)
    std::sort(best.begin(), best.end(), std::greater<int>());
    int first = -1;
    for (int i = (int)best.size() - 1; i >= 0; --i) {
        const int two = best[i] & -best[i];
        if ((two == 1 || group == 0) && (first < 0 || two < (best[first] & -best[first])))
            first = i;
    }
    if (first >= 0)
        std::rotate(best.begin(), best.begin() + first, best.begin() + first + 1);
    if (group > 1) {
        size_t last = best.size() - 1;
        double fill = 0;
        for (size_t i = best.size(); i-- > 0;) {
            const int nb = n / best[i];
            const double f = (double)nb / ((nb + group - 1) / group * group);
            if (f > fill) {
                fill = f;
                last = i;
            }
        }
        std::rotate(best.begin() + last, best.begin() + last + 1, best.end());
    }
    *s = LdsSched{};
    s->n = n;
    s->ns = (int)best.size();
    int l = 1, tw = 0;
    for (int i = 0; i < s->ns; ++i) {
        const int r = best[i];
        if (lds_powers(r))
            tw = (tw + 1) & ~1;
        s->st[i] = LdsStage{r, l, n / r, tw, reciprocal(l), reciprocal(n / r)};
        if (l > 1)
            tw += (lds_powers(r) ? 2 : r - 1) * l;
        l *= r;
    }
    return true;
}

int lds_threads(const LdsSched &s, int tiles, int group, int form, bool column)
{
    const int most = form_threads(form, column);
    group = std::max(group, 1);
    long long t = 64;
    for (int i = 0; i < s.ns; ++i) {
        int nb = s.st[i].nb;
        if (i + 1 == s.ns)
            nb = (nb + group - 1) / group * group;
        const long long total = (long long)nb * tiles;
        if ((total + lds_units(s.st[i].r, form) - 1) / lds_units(s.st[i].r, form) > most)
            return 0;
        // (kMost: as many threads as the other forms would take, if they fit)
        const int u = lds_units(s.st[i].r, form == kMost ? kNarrow : form);
        t = std::max(t, std::min<long long>(most, (total + u - 1) / u));
    }
    return (int)((t + 63) / 64 * 64);
}

int lds_table_size(const LdsSched &s)
{
    if (s.ns < 2)
        return 0;
    const LdsStage &st = s.st[s.ns - 1];
    return (st.tw + (lds_powers(st.r) ? 2 : st.r - 1) * st.l + 1) & ~1;
}

std::vector<c32> lds_table(const LdsSched &s)
{
    std::vector<c32> t((size_t)std::max(lds_table_size(s), 1));
    const RootProducts w((uint64_t)s.n, (uint64_t)s.n);
    for (int i = 1; i < s.ns; ++i) {
        const LdsStage &st = s.st[i];
        c32 *to = &t[(size_t)st.tw];
        const int step = s.n / (st.l * st.r);
        if (lds_powers(st.r)) {
            for (int k = 0; k < st.l; ++k, to += 2) {
                const c64 v = w.wide((uint64_t)k * step);
                std::memcpy(to, &v, sizeof v);
            }
            continue;
        }
        for (int j = 1; j < st.r; ++j)
            for (int k = 0; k < st.l; ++k)
                *to++ = w[(uint64_t)j * k * step];  // (< n)
    }
    return t;
}

void lds_radices(const LdsSched &s, std::vector<int> *out)
{
    for (int i = 0; i < s.ns; ++i) {
        switch (s.st[i].r) {
        case 9: out->insert(out->end(), {3, 3}); break;
        case 18: out->insert(out->end(), {2, 3, 3}); break;
        case 24: out->insert(out->end(), {4, 6}); break;
        case 27: out->insert(out->end(), {3, 3, 3}); break;
        case 30: out->insert(out->end(), {2, 15}); break;
        default: out->push_back(s.st[i].r); break;
        }
    }
}

namespace {

struct Tile {
    LdsSched s{};
    int form = kNarrow, threads = 0, l = 0;
};

// The schedule, form and threads of a workgroup for `tiles` transforms of n
// points: the wide form where its radices save a stage (2^26 samples: 360
// points 229 us to 194, 600 224 to 192, 8000 273 to 226, 20000 442 in two
// passes to 272 in one), except in tiles of half a CU's LDS and more with
// several transforms (two rows of 8192: 406 us to 550).
bool choose_form(int n, int tiles, int group, bool column, Tile *t)
{
    LdsSched narrow, wide;
    if (!lds_schedule(n, &narrow, false, group))
        return false;
    if ((tiles == 1 || (size_t)n * tiles * sizeof(c32) <= (size_t)kLdsBytes / 2) &&
        lds_schedule(n, &wide, true, group) && wide.ns < narrow.ns &&
        (t->threads = lds_threads(wide, tiles, group, kWide, column))) {
        t->s = wide;
        t->form = kWide;
        return true;
    }
    t->s = narrow;
    for (t->form = kNarrow; t->form <= kMost; ++t->form)
        if ((t->threads = lds_threads(narrow, tiles, group, t->form, column)))
            return true;
    return false;
}

// The same schedule and form for a tile of 2^l transforms, fewer than they were chosen
// for
bool refit(Tile *t, int l, int group, bool column)
{
    t->l = l;
    t->threads = lds_threads(t->s, 1 << l, group, t->form, column);
    return t->threads > 0;
}

// threads for a tile of `samples`, `each` a thread
int spread(uint64_t samples, int each, int threads, int form, bool column)
{
    const int most = form_threads(form, column);
    const int want =
        (int)std::min<uint64_t>((samples / (unsigned)each + 63) / 64 * 64, (uint64_t)most);
    return std::max(threads, want);
}

size_t tile_bytes(uint64_t n, int l, bool column)
{
    return n * ((1u << l) + (column ? 1 : 0)) * sizeof(c32);
}
// What a tile counts for in the choice: a column tile its samples and a factor (c32)
// for each output of its last stage's butterflies, more than it holds.  With what it
// holds, 600- and 1200-point columns would come 16 wide, slower in 25 of the 90
// plans that this changes (real inverse, 2^24 samples of 9 10^6: 56 us to 62).
size_t tile_lds(const Tile &t, bool column)
{
    if (!column)
        return rows_lds(t.s, t.l);
    return ((size_t)t.s.n * ((1u << t.l) + 1) + ((size_t)t.s.st[t.s.ns - 1].r << t.l)) *
           sizeof(c32);
}

// A tile of 2^l columns or rows of n points: the widest of 16 and 8 that
// leaves room for two workgroups on a CU (one loads while the other
// computes: 1000-point columns 325 us per 2^26 samples with 8, 356 with 16),
// else the widest that fits.  A paired tile's runs are half as long: 16 slots
// wherever they fit.
bool choose_tile(int n, bool column, int group, bool paired, Tile *t)
{
    for (int fill : {2, 1})
        for (t->l = 4; t->l >= (fill == 1 ? (paired ? 1 : 0) : paired ? 4 : 3); --t->l)
            if (tile_bytes(n, t->l, column) <= (size_t)kLdsBytes / fill &&
                choose_form(n, 1 << t->l, group, column, t) &&
                tile_lds(*t, column) <= (size_t)kLdsBytes / fill)
                return true;
    return false;
}

// n = n1 n2 n3 with tiles of 16 that leave room for two workgroups a CU in
// all three passes, if that costs less than `best` (the units of
// stages_choose; the factors fit the sum to whole transforms)
void choose_three(uint64_t n, double best, StagesPlan *p)
{
    // lengths near the cube root: 85 to 435 points at 2^24
    const double third = std::cbrt((double)n);
    const uint64_t least = (uint64_t)(third / 3), most = (uint64_t)(third * 1.7);
    struct Known {
        uint64_t n;
        Tile column, row;
        bool ok;
    };
    std::vector<Known> known;
    for (uint64_t m = std::max<uint64_t>(least, 32); m <= most; ++m) {
        if (n % m)
            continue;
        Known k{m, {}, {}, false};
        k.column.l = k.row.l = 4;
        k.ok = choose_form((int)m, 16, 16, true, &k.column) && k.column.s.ns >= 2 &&
               choose_form((int)m, 16, 1, false, &k.row) && k.row.s.ns >= 2;
        known.push_back(k);
    }
    for (const Known &a : known)
        for (const Known &c : known) {
            if (!a.ok || !c.ok || n / a.n % c.n)
                continue;
            const uint64_t n2 = n / a.n / c.n;
            for (const Known &m : known) {
                if (m.n != n2 || !m.ok)
                    continue;
                const double cost =
                    ((a.column.s.st[a.column.s.ns - 1].nb % 16 ? 1.25 : 1) *
                         (n / a.n % 16 ? 1.08 : 1) +
                     0.95 + 0.9 * (a.n % 16 ? 1.15 : 1) +
                     0.12 * (a.column.s.ns + m.row.s.ns + c.row.s.ns) +
                     0.1 * std::log2((double)std::max({a.n, c.n, n2}) / 256.0 + 1)) *
                    (a.n % 16 ? 0.95 : 0.85);
                if (cost >= best)
                    continue;
                Tile mid;
                if (!choose_form((int)n2, 16, 1, true, &mid) || mid.s.ns < 2)
                    continue;
                best = cost;
                p->passes = 3;
                p->a = a.column.s;
                p->form_a = a.column.form;
                p->threads_a = a.column.threads;
                p->mid = mid.s;
                p->form_mid = mid.form;
                p->threads_mid = mid.threads;
                p->b = c.row.s;
                p->form_b = c.row.form;
                p->threads_b = c.row.threads;
                p->lc = p->lr = 4;
            }
        }
}

}  // namespace

bool stages_choose(uint64_t n, uint64_t batch, int cus, StagesPlan *p, int real)
{
    *p = StagesPlan{};
    p->real = real;
    Tile t;
    if (n * sizeof(c32) <= (uint64_t)kLdsBytes) {
        // 3072 samples a workgroup (24 KB of LDS, six workgroups a CU; 4096
        // and 2048 were up to 30 % and 10 % slower: 1200 points 158 and 113 us
        // against 115, 60 points 112 and 116 against 110, each 2^25 samples),
        // fewer where the batch would leave CUs without work; where there is
        // one stage (3 or 5 points) one butterfly a thread
        const bool one = n == 2 || n == 3 || n == 4 || n == 5;
        int segs = one ? 256 : std::max(1, 3072 / (int)n);
        while (!one && segs > 1 && (batch + segs - 1) / segs < 2 * (uint64_t)cus)
            segs = (segs + 1) / 2;
        if (choose_form((int)n, segs, 0, false, &t)) {
            p->passes = 1;
            p->a = t.s;
            p->form_a = t.form;
            p->segs = segs;
            p->threads_a = one ? segs : t.threads;
            return true;
        }
    }
    // two passes: of every n1 n2 whose tiles fit, the one that the measured
    // rates of the two passes (2^26 samples, relative to a column pass of
    // 240 x 200 at 5 TB/s) make cheapest
    // [log2 width][two workgroups a CU]: whole 128-byte lines at 16
    static const double column[5][2] = {{4, 4}, {2.7, 2.7}, {2, 1.65}, {1.5, 1.45}, {1.6, 1}};
    static const double row[5][2] = {{3, 3}, {1.85, 1.85}, {1.6, 1.25}, {1.2, 1.2}, {1.25, 0.9}};
    constexpr size_t kHalf = (size_t)kLdsBytes / 2;
    std::vector<uint64_t> sizes;  // the divisors, the most balanced first
    for (uint64_t x = 1; n % x == 0; x *= 2)
        for (uint64_t y = x; n % y == 0; y *= 3)
            for (uint64_t z = y; n % z == 0; z *= 5)
                if (z >= 26 && z <= 16384 && n / z >= 2 && n / z <= 16384)
                    sizes.push_back(z);
    std::sort(sizes.begin(), sizes.end(), [n](uint64_t a, uint64_t b) {
        return std::max(a, n / a) < std::max(b, n / b) ||
               (std::max(a, n / a) == std::max(b, n / b) && a < b);
    });
    double best = 1e30;
    Tile ta, tb;
    for (uint64_t n1 : sizes) {
        const uint64_t n2 = n / n1;
        auto score = [&](int lc, int lr, bool lc2, bool lr2, bool groups, int stages) {
            lc -= real > 0 && lc > 0;
            lr -= real < 0 && lr > 0;
            return column[lc][lc2] * (groups ? 1 : 1.25) * (n2 % 16 ? 1.08 : 1) +
                   row[lr][lr2] * (n1 % 16 ? 1.15 : 1) + 0.12 * stages;
        };
        // what the sizes alone allow, before any schedule is looked for
        auto widest = [](uint64_t m, bool column, bool paired) {
            for (int l = 4; l >= (paired ? 4 : 3); --l)
                if (tile_bytes(m, l, column) <= kHalf)
                    return l;
            for (int l = 4; l >= 0; --l)
                if (tile_bytes(m, l, column) <= (size_t)kLdsBytes)
                    return l;
            return -1;
        };
        const int lc0 = widest(n1, true, real > 0), lr0 = widest(n2, false, real < 0);
        if (lr0 < 0 || lc0 < 0 ||
            score(lc0, lr0, tile_bytes(n1, lc0, true) <= kHalf,
                  tile_bytes(n2, lr0, false) <= kHalf, true, 4) >= best)
            continue;
        Tile a, b;
        if (!choose_tile((int)n2, false, 1, real < 0, &b) ||
            !choose_tile((int)n1, true, 1 << b.l, real > 0, &a) || a.s.ns < 2)
            continue;
        const double cost =
            score(a.l, b.l, tile_lds(a, true) <= kHalf, tile_lds(b, false) <= kHalf,
                  a.s.st[a.s.ns - 1].nb % (1 << b.l) == 0, a.s.ns + b.s.ns);
        if (cost >= best)
            continue;
        best = cost;
        ta = a;
        tb = b;
        p->passes = 2;
        p->a = a.s;
        p->b = b.s;
        p->lc = a.l;
        p->lr = b.l;
    }
    // three passes of short tiles, where the long tiles of two cost more: 2^24
    // as 256 x 256 x 256 moves half as much again at twice the rate (2^26
    // samples: 870 us to 648, 2^23 816 to 653, 12 10^6 738 to 609; not where
    // the two lengths are odd or near 2000: 8 10^6 636 us against 669).  Two
    // passes are a fifth faster than their sum says where the strides are no
    // multiples of 8 KB.
    if (!real && best > 3.2) {
        const bool far = p->a.n % 1024 == 0 && p->b.n % 1024 == 0;
        choose_three(n, best * (far ? 1 : 0.8), p);
    }
    if (p->passes == 3) {
        const uint64_t n1 = (uint64_t)p->a.n, m = n / n1;
        p->blocks_a = (unsigned)((m + (1u << p->lc) - 1) >> p->lc);
        p->blocks_b = (unsigned)((n1 + (1u << p->lr) - 1) >> p->lr);
        p->y_samples = ((uint64_t)p->blocks_b << p->lr) * m;
        return true;
    }
    if (p->passes != 2)
        return false;
    // few segments: narrower tiles until every CU has one, of the same schedules (a
    // segment's spectrum is the same bits in any batch)
    const uint64_t n1 = (uint64_t)ta.s.n, n2 = (uint64_t)tb.s.n;
    // (paired tiles of 4 slots move runs of 2: only where 8 slots leave more than half of
    // the CUs without one; two real segments of 2^21 samples forward 38.9 us and 35.6)
    auto few = [&](uint64_t of, int l, bool paired) {
        const uint64_t tiles = batch * ((of + (1u << l) - 1) >> l);
        return l > 2 && tiles < (uint64_t)cus / (paired && l == 3 ? 2 : 1);
    };
    while (few(n2, p->lc, real > 0))
        --p->lc;
    while (few(n1, p->lr, real < 0))
        --p->lr;
    if (!refit(&ta, p->lc, 1 << p->lr, true) || !refit(&tb, p->lr, 1, false))
        return false;
    p->a = ta.s;
    p->form_a = ta.form;
    p->threads_a = ta.threads;
    p->b = tb.s;
    p->form_b = tb.form;
    p->threads_b = tb.threads;
    // paired tiles: the columns or rows up to the middle one, half a tile's
    // slots each
    const uint64_t rows = real < 0 ? 2 * (n1 / 2 + 1) : n1;
    const uint64_t columns = real > 0 ? 2 * (n2 / 2 + 1) : n2;
    p->blocks_a = (unsigned)((columns + (1u << p->lc) - 1) >> p->lc);
    p->blocks_b = (unsigned)((rows + (1u << p->lr) - 1) >> p->lr);
    p->y_samples = ((uint64_t)p->blocks_b << p->lr) * n2;
    // a pass with at most two tiles a CU waits for each tile's own chain of loads, stages
    // and stores: a thread for every 4 samples of a tile that has a CU to itself (one
    // real segment of 2^19 samples forward, tiles of 64 threads 21.2 us, of 512 15.2;
    // of 2^18 17.6 and 13.1), for every 16 of two (with 4 there, 2^18-sample segments
    // forward 16 of them 34 us against 26)
    auto each = [&](uint64_t tiles) { return tiles <= (uint64_t)cus ? 4 : 16; };
    const uint64_t tiles_a = batch * p->blocks_a, tiles_b = batch * p->blocks_b;
    if (tiles_a <= 2 * (uint64_t)cus)
        p->threads_a = spread(n1 << p->lc, each(tiles_a), p->threads_a, p->form_a, true);
    if (tiles_b <= 2 * (uint64_t)cus)
        p->threads_b = spread(n2 << p->lr, each(tiles_b), p->threads_b, p->form_b, false);
    return true;
}

namespace {

template <int D, int F>
hipError_t launch_segments(const StagesPlan &p, const c32 *in, c32 *out, const c32 *tw,
                           uint64_t batch, uint64_t hop, const float *window, hipStream_t s)
{
    // the lanes' offsets within a workgroup's segments are 32-bit byte counts
    const int segs = hop < (1ull << 28) / (unsigned)p.segs ? p.segs : 1;
    const size_t lds = (size_t)segs * p.a.n * sizeof(c32);
    const hipError_t e = allow_lds(stages_segments_kernel<D, F>, lds);
    if (e != hipSuccess)
        return e;
    const uint64_t groups = (batch + segs - 1) / segs;
    hipLaunchKernelGGL((stages_segments_kernel<D, F>), dim3((unsigned)groups),
                       dim3(p.threads_a), (unsigned)lds, s, in, out, tw, p.a, segs, batch, hop,
                       window);
    return hipGetLastError();
}

template <int R>
hipError_t launch_short(int dir, const c32 *in, c32 *out, uint64_t batch, uint64_t hop,
                        const float *window, hipStream_t s)
{
    const dim3 grid((unsigned)std::min<uint64_t>((batch + 255) / 256, 1u << 20));
    if (dir < 0)
        hipLaunchKernelGGL((stages_short_kernel<R, -1>), grid, dim3(256), 0, s, in, out, batch,
                           hop, window);
    else
        hipLaunchKernelGGL((stages_short_kernel<R, 1>), grid, dim3(256), 0, s, in, out, batch,
                           hop, window);
    return hipGetLastError();
}

template <int D, int F>
hipError_t launch_columns(const StagesPlan &p, const c32 *in, c32 *y, const c32 *tw,
                          const c64 *tl, const c64 *th, int sh, uint64_t batch, uint64_t hop,
                          const float *window, hipStream_t s)
{
    const size_t lds = columns_lds(p.a, p.lc);
    const hipError_t e = allow_lds(stages_columns_kernel<D, F>, lds);
    if (e != hipSuccess)
        return e;
    const unsigned blocks = p.blocks_a;
    const int n2 = p.passes == 3 ? p.mid.n * p.b.n : p.b.n;
    hipLaunchKernelGGL((stages_columns_kernel<D, F>), dim3(xcd_grid(batch * blocks)),
                       dim3(p.threads_a), (unsigned)lds, s, in, y, tw, tl, th, sh, p.a, n2,
                       p.lc, p.lr, blocks, batch * blocks, p.y_samples, hop, window);
    return hipGetLastError();
}

template <int D, int F>
hipError_t launch_rows(const StagesPlan &p, const c32 *y, c32 *out, const c32 *tw,
                       uint64_t batch, hipStream_t s)
{
    const size_t lds = rows_lds(p.b, p.lr);
    const hipError_t e = allow_lds(stages_rows_kernel<D, F>, lds);
    if (e != hipSuccess)
        return e;
    const unsigned blocks = p.blocks_b;
    const int n2 = p.passes == 3 ? p.mid.n : 1;
    const uint64_t tiles = batch * blocks * (unsigned)n2;
    hipLaunchKernelGGL((stages_rows_kernel<D, F>), dim3(xcd_grid(tiles)), dim3(p.threads_b),
                       (unsigned)lds, s, y, out, tw, p.b, p.a.n, n2, p.lr, blocks, tiles,
                       p.y_samples);
    return hipGetLastError();
}

template <int D, int F>
hipError_t launch_middle(const StagesPlan &p, c32 *y, const c32 *tw, const c64 *tl,
                         const c64 *th, int sh, uint64_t batch, hipStream_t s)
{
    const size_t lds = rows_lds(p.mid, p.lr);
    const hipError_t e = allow_lds(stages_middle_columns_kernel<D, F>, lds);
    if (e != hipSuccess)
        return e;
    const uint64_t tiles = batch * p.blocks_b * (unsigned)p.b.n;
    hipLaunchKernelGGL((stages_middle_columns_kernel<D, F>), dim3(xcd_grid(tiles)),
                       dim3(p.threads_mid), (unsigned)lds, s, y, tw, tl, th, sh, p.mid, p.a.n,
                       p.b.n, p.lr, p.blocks_b, tiles, p.y_samples);
    return hipGetLastError();
}

}  // namespace

hipError_t stages_one_pass(const StagesPlan &p, int dir, const void *in, void *out,
                           const void *tw, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s)
{
    if (p.a.n == 3 || p.a.n == 5)
        return (p.a.n == 3 ? launch_short<3> : launch_short<5>)(dir, (const c32 *)in, (c32 *)out,
                                                                batch, hop, window, s);
    static constexpr auto f = {launch_segments<-1, kNarrow>, launch_segments<-1, kMost>,
                               launch_segments<-1, kWide>,   launch_segments<1, kNarrow>,
                               launch_segments<1, kMost>,    launch_segments<1, kWide>};
    return f.begin()[p.form_a + (dir < 0 ? 0 : 3)](p, (const c32 *)in, (c32 *)out,
                                                   (const c32 *)tw, batch, hop, window, s);
}

hipError_t stages_rows(const StagesPlan &p, int dir, const void *y, void *out, const void *tw,
                       uint64_t batch, hipStream_t s)
{
    static constexpr auto f = {launch_rows<-1, kNarrow>, launch_rows<-1, kMost>,
                               launch_rows<-1, kWide>,   launch_rows<1, kNarrow>,
                               launch_rows<1, kMost>,    launch_rows<1, kWide>};
    return f.begin()[p.form_b + (dir < 0 ? 0 : 3)](p, (const c32 *)y, (c32 *)out,
                                                   (const c32 *)tw, batch, s);
}

hipError_t stages_two_pass(const StagesPlan &p, int dir, const void *in, void *out, void *y,
                           const StagesTables &t, uint64_t batch, uint64_t hop,
                           const float *window, hipStream_t s)
{
    static constexpr auto f = {launch_columns<-1, kNarrow>, launch_columns<-1, kMost>,
                               launch_columns<-1, kWide>,   launch_columns<1, kNarrow>,
                               launch_columns<1, kMost>,    launch_columns<1, kWide>};
    static constexpr auto fm = {launch_middle<-1, kNarrow>, launch_middle<-1, kMost>,
                                launch_middle<-1, kWide>,   launch_middle<1, kNarrow>,
                                launch_middle<1, kMost>,    launch_middle<1, kWide>};
    hipError_t e = f.begin()[p.form_a + (dir < 0 ? 0 : 3)](
        p, (const c32 *)in, (c32 *)y, (const c32 *)t.a, (const c64 *)t.tl, (const c64 *)t.th,
        t.sh, batch, hop, window, s);
    if (e == hipSuccess && p.passes == 3)
        e = fm.begin()[p.form_mid + (dir < 0 ? 0 : 3)](p, (c32 *)y, (const c32 *)t.mid,
                                                       (const c64 *)t.tl2, (const c64 *)t.th2,
                                                       t.sh2, batch, s);
    return e == hipSuccess ? stages_rows(p, dir, y, out, t.b, batch, s) : e;
}

}  // namespace fftseg
