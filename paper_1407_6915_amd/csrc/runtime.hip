// Planner, twiddle tables, argument checks and the C entry points of the
// batched segment FFT (declared in fftseg.h).
#include "fftseg.h"
#include "runtime.hpp"

#include <algorithm>
#include <cmath>
#include <cstdarg>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <mutex>
#include <new>
#include <string>
#include <vector>

namespace fftseg {

// ---------------------------------------------------------------------------
// per-thread status
namespace {
thread_local int t_status = FFT_OK;
thread_local char t_msg[512] = "";
}  // namespace

int set_ok()
{
    t_status = FFT_OK;
    t_msg[0] = 0;
    return FFT_OK;
}

int set_error(int status, const char *fmt, ...)
{
    t_status = status;
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(t_msg, sizeof(t_msg), fmt, ap);
    va_end(ap);
    return status;
}

int hip_error(hipError_t e, const char *what)
{
    return set_error(FFT_ERR_HIP, "%s: %s", what, hipGetErrorString(e));
}

int last_status() { return t_status; }
const char *last_message() { return t_msg; }

// ---------------------------------------------------------------------------
// twiddles: exp(-2 pi i m / n) in FP64 with the angle folded to the first
// octant in exact integer arithmetic, rounded once to float32
static c64 root_forward64(uint64_t m, uint64_t n)
{
    m %= n;
    // angle 2 pi m / n = (pi/4) (o + r/n) with 8m = o*n + r; quadrant
    // j = floor((o + 1) / 2) and x = (pi/4) (o - 2j + r/n) in [-pi/4, pi/4)
    // (n <= 2^24: 8 m fits)
    const uint64_t m8 = m * 8u;
    const uint64_t o = m8 / n;
    const uint64_t r = m8 - o * n;
    const uint64_t j = (o + 1) / 2;
    const double quarter_pi = 0.78539816339744830961566084581987572;
    const double x = ((double)((long long)o - 2 * (long long)j) + (double)r / (double)n) *
                     quarter_pi;
    double cx, sx;
    sincos(x, &sx, &cx);
    double c, s;
    switch (j & 3) {
    case 0: c = cx; s = sx; break;
    case 1: c = -sx; s = cx; break;
    case 2: c = -cx; s = -sx; break;
    default: c = sx; s = -cx; break;
    }
    return c64{c, -s};
}

c32 root_forward(uint64_t m, uint64_t n)
{
    const c64 w = root_forward64(m, n);
    return c32{(float)w.x, (float)w.y};
}

RootProducts::RootProducts(uint64_t n, uint64_t count) : low(128), high(count / 128 + 1)
{
    for (uint64_t j = 0; j < low.size(); ++j)
        low[j] = root_forward64(j, n);
    for (uint64_t j = 0; j < high.size(); ++j)
        high[j] = root_forward64(128 * j, n);
}

std::vector<c32> root_products(uint64_t n, uint64_t count)
{
    const RootProducts w(n, count);
    std::vector<c32> t(count);
    for (uint64_t m = 0; m < count; ++m)
        t[m] = w[m];
    return t;
}

std::vector<c32> wide_root_products(uint64_t n, uint64_t count)
{
    const RootProducts w(n, count);
    std::vector<c32> t(2 * count);
    for (uint64_t m = 0; m < count; ++m) {
        const c64 v = w.wide(m);
        std::memcpy(&t[2 * m], &v, sizeof v);
    }
    return t;
}

std::vector<c32> root_table(uint64_t n)
{
    // the upper half is the lower half's conjugates
    std::vector<c32> t(n);
    for (uint64_t m = 0; m <= n / 2; ++m)
        t[m] = root_forward(m, n);
    for (uint64_t m = n / 2 + 1; m < n; ++m)
        t[m] = c32{t[n - m].x, -t[n - m].y};
    return t;
}

namespace {

int ilog2_ceil(uint64_t v)
{
    int k = 0;
    while ((1ull << k) < v)
        ++k;
    return k;
}

}  // namespace

int two_level_shift(uint64_t n) { return ilog2_ceil(n) / 2 + (ilog2_ceil(n) & 1); }

namespace {

// the two-level table of W_n: low entries W_n^j, j < 2^sh, and high ones
// W_n^{j 2^sh}, in float32 or (run-time schedules) in FP64, whose product is
// rounded once
template <class Entry>
std::vector<c32> two_level(uint64_t n, uint64_t count, int shift, Entry root)
{
    using E = decltype(root(0, n));
    std::vector<c32> t((size_t)(count * sizeof(E) / sizeof(c32)));
    for (uint64_t j = 0; j < count; ++j) {
        const E w = root(j << shift, n);
        std::memcpy((char *)t.data() + j * sizeof(E), &w, sizeof(E));
    }
    return t;
}

struct TwoLevel {
    std::vector<c32> low, high;
    int sh;
    TwoLevel(uint64_t n, bool wide) : sh(two_level_shift(n))
    {
        const uint64_t lo = 1ull << sh, hi = (n + lo - 1) >> sh;
        low = wide ? two_level(n, lo, 0, root_forward64) : two_level(n, lo, 0, root_forward);
        high = wide ? two_level(n, hi, sh, root_forward64) : two_level(n, hi, sh, root_forward);
    }
};

bool is_pow2(uint64_t v) { return v && !(v & (v - 1)); }

bool smooth235(uint64_t n)
{
    if (n == 0)
        return false;
    for (uint64_t p : {2ull, 3ull, 5ull})
        while (n % p == 0)
            n /= p;
    return n == 1;
}

// greedy radix list of a two-pass length as a whole (fft_plan_factorize)
std::vector<int> generic_radices(uint64_t n)
{
    std::vector<int> r;
    for (int p : {16, 8, 4, 2, 5, 3}) {
        while (n % p == 0 && n > 1) {
            r.push_back(p);
            n /= p;
        }
    }
    return r;
}

// The plan's tables in one allocation (p->tables), each from a 256-byte
// boundary on, uploaded in one copy; `dev` receives the table's address.
struct HostTable {
    const std::vector<c32> &host;
    void **dev;
};

int upload_tables(Plan *p, std::initializer_list<HostTable> set)
{
    constexpr size_t kAlign = 256 / sizeof(c32);
    std::vector<c32> all;
    size_t total = 0;
    for (const HostTable &t : set)
        total += (t.host.size() + kAlign - 1) / kAlign * kAlign;
    hipError_t e = hipMalloc(&p->tables, total * sizeof(c32));
    if (e != hipSuccess) {
        p->tables = nullptr;
        (void)hipGetLastError();
        return e == hipErrorOutOfMemory ? set_error(FFT_ERR_OUT_OF_MEMORY, "twiddles")
                                        : hip_error(e, "twiddle upload");
    }
    if (set.size() > 1)
        all.reserve(total);
    size_t at = 0;
    for (const HostTable &t : set) {
        *t.dev = (c32 *)p->tables + at;
        at += (t.host.size() + kAlign - 1) / kAlign * kAlign;
        if (set.size() > 1) {
            all.insert(all.end(), t.host.begin(), t.host.end());
            all.resize(at);
        }
    }
    const std::vector<c32> &src = set.size() > 1 ? all : set.begin()->host;
    e = hipMemcpy(p->tables, src.data(), src.size() * sizeof(c32), hipMemcpyHostToDevice);
    // (on failure plan_free releases the allocation)
    return e == hipSuccess ? set_ok() : hip_error(e, "twiddle upload");
}

// the tuning table: preferred single-pass variant and grid per length
std::mutex g_tune_mu;
std::vector<TunedChoice> g_tuned;

}  // namespace

int tuned_variant(uint64_t n)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == n)
            return p.keep ? -1 : p.variant;
    return -1;
}

int tuned_grid_mult(uint64_t n, int variant, int fallback)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == n && p.variant == variant && !p.keep)
            return p.grid_mult;
    return fallback;
}

bool tuned_split_variants(uint64_t n, int *col_variant, int *row_variant, uint64_t *n1)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == n && p.variant == -1 && !p.keep) {
            *col_variant = p.col_variant;
            *row_variant = p.row_variant;
            *n1 = p.n1;
            return true;
        }
    return false;
}

int tuned_wl_route(uint64_t n, int *grid)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == n) {
            if (grid)
                *grid = p.wl_grid;
            return p.wl_route;
        }
    return -1;
}

void set_tuned(const TunedChoice &c)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == c.n) {
            p = c;
            return;
        }
    g_tuned.push_back(c);
}

void set_tuned_wl_route(uint64_t n, int route, int grid, double us)
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    for (auto &p : g_tuned)
        if (p.n == n) {
            p.wl_route = route;
            p.wl_grid = grid;
            p.wl_us = us;
            return;
        }
    TunedChoice c{n, -2, 0, 0, 0, 0, 0};  // variant -2: no plan choice
    c.wl_route = route;
    c.wl_grid = grid;
    c.wl_us = us;
    g_tuned.push_back(c);
}

void clear_tuned()
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    g_tuned.clear();
}

std::vector<TunedChoice> tuned_snapshot()
{
    std::lock_guard<std::mutex> lk(g_tune_mu);
    return g_tuned;
}

const SinglePassDesc *find_single(uint64_t n, int variant)
{
    int cnt = 0;
    const SinglePassDesc *t = single_pass_table(&cnt);
    for (int i = 0; i < cnt; ++i)
        if ((uint64_t)t[i].n == n && t[i].variant == variant)
            return &t[i];
    return nullptr;
}

// the variant of length n that carries the frame and real-input kernels
static const SinglePassDesc *find_small_batch(uint64_t n)
{
    int cnt = 0;
    const SinglePassDesc *t = single_pass_table(&cnt);
    for (int i = 0; i < cnt; ++i)
        if ((uint64_t)t[i].n == n && t[i].small_batch)
            return &t[i];
    return nullptr;
}

const SinglePassDesc *find_frames(uint64_t n)
{
    int cnt = 0;
    const SinglePassDesc *t = single_pass_table(&cnt);
    for (int i = 0; i < cnt; ++i)
        if ((uint64_t)t[i].n == n && t[i].launch_strided)
            return &t[i];
    return nullptr;
}

const SinglePassDesc *find_aux(uint64_t n)
{
    int cnt = 0;
    const SinglePassDesc *t = single_pass_table(&cnt);
    for (int i = 0; i < cnt; ++i)
        if ((uint64_t)t[i].n == n && t[i].launch_strided && t[i].launch_real)
            return &t[i];
    return nullptr;
}

int variant_count(uint64_t n)
{
    int cnt = 0, k = 0;
    const SinglePassDesc *t = single_pass_table(&cnt);
    for (int i = 0; i < cnt; ++i)
        k += (uint64_t)t[i].n == n;
    return k;
}

// best four-step split n = n1 * n2 with compiled column and row tiles;
// the split is chosen on the default tiles, then the requested variants of
// those lengths are used (default where a variant does not exist)
bool find_split(uint64_t n, const ColumnDesc **col, const RowDesc **row, int col_variant,
                int row_variant, uint64_t want_n1)
{
    int nc = 0, nr = 0;
    const ColumnDesc *ct = column_table(&nc);
    const RowDesc *rt = row_table(&nr);
    double best = 1e30;
    *col = nullptr;
    *row = nullptr;
    for (int i = 0; i < nc; ++i) {
        if (ct[i].variant != 0 || n % (uint64_t)ct[i].n1 ||
            (want_n1 && (uint64_t)ct[i].n1 != want_n1))
            continue;
        const uint64_t n2 = n / (uint64_t)ct[i].n1;
        for (int j = 0; j < nr; ++j) {
            if (rt[j].variant != 0 || (uint64_t)rt[j].n2 != n2)
                continue;
            // prefer balanced splits, then the smaller column length
            const double score =
                std::fabs(std::log2((double)ct[i].n1) - std::log2((double)n2)) * 2.0 +
                (ct[i].n1 > (int)n2 ? 1.0 : 0.0);
            if (score < best) {
                best = score;
                *col = &ct[i];
                *row = &rt[j];
            }
        }
    }
    if (!*col)
        return false;
    const uint64_t n1 = (uint64_t)(*col)->n1, n2 = n / n1;
    auto fits = [&](const ColumnDesc &c, const RowDesc &r) {
        return n2 % (uint64_t)c.cols == 0 && n1 % (uint64_t)r.rows == 0;
    };
    for (int i = 0; i < nc; ++i)
        if ((uint64_t)ct[i].n1 == n1 && ct[i].variant == col_variant && fits(ct[i], **row))
            *col = &ct[i];
    for (int j = 0; j < nr; ++j)
        if ((uint64_t)rt[j].n2 == n2 && rt[j].variant == row_variant && fits(**col, rt[j]))
            *row = &rt[j];
    return fits(**col, **row);
}

std::vector<uint64_t> split_candidates(uint64_t n)
{
    std::vector<uint64_t> out;
    int nc = 0;
    const ColumnDesc *ct = column_table(&nc);
    for (int i = 0; i < nc; ++i) {
        const ColumnDesc *c = nullptr;
        const RowDesc *r = nullptr;
        if (ct[i].variant == 0 && n % (uint64_t)ct[i].n1 == 0 &&
            find_split(n, &c, &r, 0, 0, (uint64_t)ct[i].n1))
            out.push_back((uint64_t)ct[i].n1);
    }
    return out;
}

const ColumnDesc *find_column_shifted(uint64_t n1)
{
    int nc = 0;
    const ColumnDesc *ct = column_table(&nc);
    for (int i = 0; i < nc; ++i)
        if ((uint64_t)ct[i].n1 == n1 && ct[i].launch_shifted)
            return &ct[i];
    return nullptr;
}

const RowDesc *find_row_shifted(uint64_t n2)
{
    int nr = 0;
    const RowDesc *rt = row_table(&nr);
    for (int j = 0; j < nr; ++j)
        if ((uint64_t)rt[j].n2 == n2 && rt[j].launch_shifted)
            return &rt[j];
    return nullptr;
}

int split_variant_counts(uint64_t n, int *ncol, int *nrow)
{
    const ColumnDesc *c = nullptr;
    const RowDesc *r = nullptr;
    *ncol = *nrow = 0;
    if (!find_split(n, &c, &r, 0, 0))
        return 0;
    int nc = 0, nr = 0;
    const ColumnDesc *ct = column_table(&nc);
    const RowDesc *rt = row_table(&nr);
    for (int i = 0; i < nc; ++i)
        *ncol += ct[i].n1 == c->n1;
    for (int j = 0; j < nr; ++j)
        *nrow += rt[j].n2 == r->n2;
    return 1;
}

// The row tile of an untuned two-pass plan by its batch: where the default's
// 16-row tiles would be at most a quarter of the CUs (half for 2048 points,
// which 1024 threads hold), the length's narrow tile (one segment of 2^19
// points 17.8 us to 14.7, of 2^21 45.7 to 29.6; at more tiles the 64-byte
// runs cost more: four of 2^18 15.1 us to 15.9), else up to 2^26 samples the
// length's tile for that range (1024 points: streamed loads and stores, both tiles
// on their own grids (tile_grid): segments of 2^20, 2^24 samples 114 us to 102, 2^25
// 236 to 206, 2^26 438 to 419, 2^27 847 to 837, 2^28 1678 to 1691; of 2^19, 2^25 238
// to 228, 2^26 432 to 431, 2^26.5 566 to 575, 2^27 807 to 817).
static const RowDesc *row_for_batch(const RowDesc *row, uint64_t n1, uint64_t batch, int cus)
{
    constexpr uint64_t kMidSamples = 1ull << 26;
    const uint64_t tiles = batch * (n1 / (uint64_t)row->rows);
    const bool few = tiles <= (uint64_t)cus / (row->n2 >= 2048 ? 2 : 4);
    const bool mid = !few && batch * n1 * (uint64_t)row->n2 <= kMidSamples;
    int nr = 0;
    const RowDesc *rt = row_table(&nr);
    for (int j = 0; (few || mid) && j < nr; ++j)
        if (rt[j].n2 == row->n2 && (few ? rt[j].few_tiles : rt[j].mid_size) &&
            n1 % (uint64_t)rt[j].rows == 0)
            return &rt[j];
    return row;
}

// CU count per device and resident workgroups per CU per kernel, cached:
// both are fixed for the life of the process and the queries are slow.
namespace {
std::mutex g_occ_mu;
std::vector<std::pair<int, int>> g_cus;                      // (device, CUs)
std::vector<std::pair<std::pair<const void *, int>, int>> g_occ;  // ((kernel, dev), per CU)
}  // namespace

static int device_cus(int dev)
{
    std::lock_guard<std::mutex> lk(g_occ_mu);
    for (auto &c : g_cus)
        if (c.first == dev)
            return c.second;
    int n = 0;
    if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess ||
        n <= 0) {
        (void)hipGetLastError();
        n = 256;
    }
    g_cus.emplace_back(dev, n);
    return n;
}

static int resident_per_cu(const void *kernel, int threads, int dev)
{
    {
        std::lock_guard<std::mutex> lk(g_occ_mu);
        for (auto &o : g_occ)
            if (o.first.first == kernel && o.first.second == dev)
                return o.second;
    }
    int per_cu = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, kernel, threads, 0) != hipSuccess ||
        per_cu <= 0) {
        (void)hipGetLastError();
        per_cu = 1;
    }
    std::lock_guard<std::mutex> lk(g_occ_mu);
    g_occ.push_back({{kernel, dev}, per_cu});
    return per_cu;
}

// Workgroups of a persistent kernel: grid_mult resident waves at most (0: one
// per group).  Kernels that keep their twiddles in registers across groups are
// bound by reading them when a workgroup takes only one or two groups, so those
// with walk > 1 get fewer waves, whole ones, where grid_mult waves would have
// fewer than `walk` groups each (at 2^25 samples, whose groups are 5 to 16 waves,
// every group used to be a workgroup of its own).  Four measured best: 4096
// points at 2^27 samples 402 -> 364 us (2 groups each 379, 8 each 369); 1000
// points 517 -> 395; real forward of 4096 255 -> 211, inverse 303 -> 224, of
// 16384 431 -> 323 and 556 -> 415; frames of 4096 every 4096 560 -> 379, every
// 1024 488 -> 355; at 2^23 samples 33.3 -> 31.0, 28.0 -> 25.2, 23.1 -> 20.0.  One-
// pass lengths whose kernels read few twiddles or reload them per group lose
// (at 2^27 samples 256 points 9 %, 512 and 1024 2 %, 8192 6 %, 16384 8 %) and have walk = 1.
unsigned grid_for(const void *kernel, int threads, uint64_t work_groups, int dev,
                  int grid_mult, int walk)
{
    uint64_t g = work_groups;
    if (grid_mult > 0) {
        const uint64_t wave =
            (uint64_t)resident_per_cu(kernel, threads, dev) * (uint64_t)device_cus(dev);
        uint64_t waves = (uint64_t)grid_mult;
        if (walk > 1)
            waves = std::min<uint64_t>(waves, std::max<uint64_t>(g / (wave * (uint64_t)walk), 1));
        g = std::min<uint64_t>(g, wave * waves);
    }
    g = std::min<uint64_t>(g, 0x7fffffffull);
    return (unsigned)std::max<uint64_t>(g, 1);
}

// Persistent grid: this many resident workgroup waves per CU (each
// workgroup walks tiles with a grid-stride loop, so twiddles loaded once
// stay in registers); FFTSEG_GRID_MULT=0 gives one workgroup per tile.
constexpr int kDefaultGridMult = 8;
constexpr int kTwoPassGridMult = 32;  // four-step passes without a measured choice

// Four-step passes: the measured best grid by column-tile length (sweeps at
// 8 GiB; 128 resident waves per CU is one workgroup per tile of a 4 GiB
// sub-batch from 128- to 2048-point columns, which beat the persistent
// grids of 16-64 once the tiles' twiddle reads were cut: 2^15 points
// 6.21 ms against 6.45 at 32, 2^20 6.42-6.44 against 6.50-6.78 at 64,
// 2^22 9.40 against 9.63 at 32)
int two_pass_grid_mult(uint64_t n1)
{
    switch (n1) {
    case 128:
    case 256:
    case 512:
    case 1024:
    case 2048:
        return 128;
    default:
        return kTwoPassGridMult;
    }
}

// A four-step pass of columns of 1024 points or rows of 1024 or 2048 takes one
// resident wave of workgroups that walk four tiles or more each:
// neighbouring tiles then stay in step on an XCD and find the lines that they
// share, where launching a workgroup per tile lets them drift (2^20 points, 2^24
// to 2^28 samples: 120 -> 107, 250 -> 208, 473 -> 412, 944 -> 851, 1.77 -> 1.69 ms;
// an output base off a line, 2^25 samples: 293 -> 238; frames every 2^20: 255 ->
// 210; 2^21 points, 2^25 samples 289 -> 274; 2^22, rows alone 339 -> 320).  Longer
// walks lose it again: 64 tiles a workgroup for 2^20 points (at 128, 3.39 ms
// against 3.35), 16 above (2^21 at 64: 1.93 ms against 1.89), where 4 gain nothing
// sure either (2^24 samples, frames every n/4: 126.6 us against 123.3).  Shorter columns
// lose at any size (512 by 512 at 2^27 samples 743 -> 819), 2048-point ones from 2^26.
unsigned tile_grid(const Plan *p, const void *kernel, int threads, uint64_t tiles,
                   bool one_wave)
{
    if (p->own_grid && one_wave) {
        const unsigned g = grid_for(kernel, threads, tiles, p->device, 1);
        const bool longer = p->n > (1u << 20);
        if (tiles >= (longer ? 8ull : 4ull) * g && tiles <= (longer ? 16ull : 64ull) * g)
            return g;
    }
    return grid_for(kernel, threads, tiles, p->device, p->grid_mult);
}

bool one_wave_columns(uint64_t n1)
{
    return n1 == 1024;
}

bool one_wave_rows(uint64_t n2)
{
    return n2 == 1024 || n2 == 2048;
}

int env_grid_mult()
{
    const char *e = getenv("FFTSEG_GRID_MULT");
    return e ? atoi(e) : kDefaultGridMult;
}

// ---------------------------------------------------------------------------
// plan construction: the choice of kernels, split and sub-batch (host only),
// then the device tables and scratch
int plan_choose(Plan *p, uint64_t n, uint64_t batch, int dir, int forced_variant,
                int forced_split_variants, uint64_t forced_n1, uint64_t max_sub_samples)
{
    p->n = n;
    p->batch = batch;
    p->dir = dir;
    if (hipGetDevice(&p->device) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FFT_ERR_HIP, "no HIP device available");
    }
    p->grid_mult = env_grid_mult();
    if (n == 1) {
        p->kind = Plan::COPY;
        return set_ok();
    }
    const int tuned = forced_variant >= 0 || p->untuned ? -1 : tuned_variant(n);
    int variant = forced_variant >= 0 ? forced_variant : tuned;
    if (variant < 0)
        variant = 0;
    p->sp = find_single(n, variant);
    if (!p->sp && forced_variant < 0)
        p->sp = find_single(n, 0);
    if (p->sp && p->by_batch && forced_variant < 0 && tuned < 0) {
        // a batch that gives the default kernel few workgroups (two per CU,
        // or one per eight) takes the length's small-batch kernel, if it has
        // one
        const SinglePassDesc *alt = find_small_batch(n);
        const uint64_t groups =
            (batch + (uint64_t)p->sp->segs_per_wg - 1) / (uint64_t)p->sp->segs_per_wg;
        if (alt && 8 * groups < (uint64_t)alt->small_batch * (uint64_t)device_cus(p->device))
            p->sp = alt;
    }
    if (forced_variant >= 0 && !p->sp)
        return set_error(FFT_ERR_INVALID_ARG, "length %llu has no variant %d",
                         (unsigned long long)n, forced_variant);
    if (p->sp) {
        p->kind = Plan::SINGLE;
        if (!getenv("FFTSEG_GRID_MULT")) {
            const int g = p->untuned ? -1 : tuned_grid_mult(n, p->sp->variant, -1);
            p->own_grid = g < 0;
            p->grid_mult = p->own_grid ? p->sp->grid_mult : g;
        }
        return set_ok();
    }
    p->sh = two_level_shift(n);
    int cv = 0, rv = 0;
    uint64_t n1 = forced_n1;
    bool tuned_tiles = false;
    if (forced_split_variants >= 0) {
        cv = forced_split_variants & 0xff;
        rv = (forced_split_variants >> 8) & 0xff;
    } else if (!forced_n1 && !p->untuned) {
        tuned_tiles = tuned_split_variants(n, &cv, &rv, &n1);
    }
    bool split = find_split(n, &p->col, &p->row, cv, rv, n1);
    if (split && p->by_batch && forced_split_variants < 0 && !forced_n1 && !tuned_tiles)
        p->row = row_for_batch(p->row, (uint64_t)p->col->n1, batch, device_cus(p->device));
    if (!split && n1 && !forced_n1)
        split = find_split(n, &p->col, &p->row, 0, 0, 0);  // a tuned split the library lacks
    if (!split && forced_n1)
        return set_error(FFT_ERR_INVALID_ARG, "length %llu has no split with %llu columns",
                         (unsigned long long)n, (unsigned long long)forced_n1);
    if (!getenv("FFTSEG_GRID_MULT")) {
        const int g = p->untuned ? -1 : tuned_grid_mult(n, -1, -1);
        p->own_grid = g < 0;
        p->grid_mult = !p->own_grid ? g
                       : split      ? two_pass_grid_mult((uint64_t)p->col->n1)
                                    : kTwoPassGridMult;
    }
    if (split) {
        p->kind = Plan::FOURSTEP;
        p->n1 = (uint64_t)p->col->n1;
        p->n2 = (uint64_t)p->row->n2;
        // Y in blocks of 16 columns where both tiles have that form
        // (FFTSEG_Y_LAYOUT=plain keeps the input's layout, for comparison)
        const char *yl = getenv("FFTSEG_Y_LAYOUT");
        p->y_blocked = p->col->launch_yblocked && p->row->launch_yblocked &&
                       !(yl && strcmp(yl, "plain") == 0);
        // (one line more: Y may start at the input's offset within a line)
        p->sub_batch = std::min<uint64_t>(batch, max_sub_samples / n);
        p->scratch_bytes = (p->sub_batch * n + kLineSamples) * sizeof(c32);
    } else {
        p->kind = Plan::GENERIC;
        if (!stages_choose(n, batch, device_cus(p->device), &p->stages))
            return set_error(FFT_ERR_UNSUPPORTED_LENGTH, "no schedule for length %llu",
                             (unsigned long long)n);
        p->sub_batch = std::min<uint64_t>(batch, max_sub_samples / n);
        if (p->stages.passes > 1) {
            // Y pads the last row tile of a segment
            if (p->sub_batch > 1)
                p->sub_batch = std::max<uint64_t>(
                    1, std::min(p->sub_batch, max_sub_samples / p->stages.y_samples));
            p->scratch_bytes = p->sub_batch * p->stages.y_samples * sizeof(c32);
        }
    }
    if (p->sub_batch == 0)
        return set_error(FFT_ERR_INVALID_ARG,
                         "one %llu-point segment needs more scratch than %llu samples",
                         (unsigned long long)n, (unsigned long long)max_sub_samples);
    return set_ok();
}

// 4 GiB of complex64 per scratch buffer; FFTSEG_SUB_SAMPLES caps a
// sub-batch at fewer samples
static uint64_t max_scratch_samples()
{
    uint64_t max_sub = 1ull << 29;
    if (const char *e = getenv("FFTSEG_SUB_SAMPLES"))
        max_sub = std::max<uint64_t>(1, std::min<uint64_t>(max_sub, strtoull(e, nullptr, 10)));
    return max_sub;
}

int plan_build(Plan *p, uint64_t n, uint64_t batch, int dir, int forced_variant,
               int forced_split_variants, uint64_t forced_n1)
{
    int st = plan_choose(p, n, batch, dir, forced_variant, forced_split_variants, forced_n1,
                         max_scratch_samples());
    if (st != FFT_OK || p->kind == Plan::COPY)
        return st;
    const bool four = p->kind == Plan::FOURSTEP;
    if (p->kind == Plan::SINGLE)
        return upload_tables(p, {{root_table(n), &p->tw}});
    if (!four && p->stages.passes == 1)
        return upload_tables(p, {{lds_table(p->stages.a), &p->tw}});
    const TwoLevel w(n, !four);
    p->sh = w.sh;
    if (!four && p->stages.passes == 3) {
        const TwoLevel w2(n / (uint64_t)p->stages.a.n, true);
        p->sh2 = w2.sh;
        if (upload_tables(p, {{lds_table(p->stages.a), &p->tw},
                              {lds_table(p->stages.b), &p->tw2},
                              {lds_table(p->stages.mid), &p->w1},
                              {w.low, &p->tl},
                              {w.high, &p->th},
                              {w2.low, &p->tl2},
                              {w2.high, &p->th2}}) != FFT_OK)
            return last_status();
    } else if (upload_tables(p, {{four ? root_table(p->n1) : lds_table(p->stages.a), &p->tw},
                          {four ? root_table(p->n2) : lds_table(p->stages.b), &p->tw2},
                          {w.low, &p->tl},
                          {w.high, &p->th}}) != FFT_OK)
        return last_status();
    hipError_t e = hipMalloc(&p->scratch, p->scratch_bytes);
    if (e != hipSuccess) {
        p->scratch = nullptr;
        (void)hipGetLastError();
        return set_error(FFT_ERR_OUT_OF_MEMORY, "scratch of %zu bytes", p->scratch_bytes);
    }
    return set_ok();
}

int plan_build_real(Plan *p, uint64_t n, uint64_t batch, int dir)
{
    p->n = n;
    p->batch = batch;
    p->dir = dir;
    if (hipGetDevice(&p->device) != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FFT_ERR_HIP, "no HIP device available");
    }
    const uint64_t m = n / 2;
    p->sp = find_aux(m);
    if (p->sp && p->sp->launch_real) {
        // the split fused into the m-point one-pass kernel
        p->kind = Plan::REAL;
        p->own_grid = !getenv("FFTSEG_GRID_MULT");
        p->grid_mult = p->own_grid ? p->sp->grid_mult : env_grid_mult();
        return upload_tables(p, {{root_table(m), &p->tw}, {root_products(n, m + 1), &p->tw2}});
    }
    // a run-time schedule of the m-point transform, the split fused into it
    p->sp = nullptr;
    p->kind = Plan::REAL_STAGES;
    if (!stages_choose(m, batch, device_cus(p->device), &p->stages, dir))
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH, "no schedule for length %llu",
                         (unsigned long long)m);
    // (a cap below one segment is refused as for a plan of m points, also in one pass)
    if (max_scratch_samples() < m)
        return set_error(FFT_ERR_INVALID_ARG,
                         "a %llu-point segment is above the cap of %llu samples on a sub-batch",
                         (unsigned long long)m, (unsigned long long)max_scratch_samples());
    if (p->stages.passes == 1) {
        p->sub_batch = batch;
        return upload_tables(
            p, {{lds_table(p->stages.a), &p->tw}, {root_products(n, m / 2 + 1), &p->w1}});
    }
    // 2 GiB of complex64, before Y's padding, or what FFTSEG_SUB_SAMPLES allows
    const uint64_t max_sub_samples = std::min<uint64_t>(max_scratch_samples(), 1ull << 28);
    p->sub_batch = std::min<uint64_t>(batch, max_sub_samples / m);
    const uint64_t n1 = (uint64_t)p->stages.a.n, n2 = (uint64_t)p->stages.b.n;
    const TwoLevel w(m, true);
    p->sh = w.sh;
    if (upload_tables(p, {{lds_table(p->stages.a), &p->tw},
                          {lds_table(p->stages.b), &p->tw2},
                          {w.low, &p->tl},
                          {w.high, &p->th},
                          {wide_root_products(n, (dir < 0 ? n1 : n2) / 2 + 1), &p->w1},
                          {wide_root_products(2 * (dir < 0 ? n2 : n1), dir < 0 ? n2 : n1),
                           &p->w2}}) != FFT_OK)
        return last_status();
    p->scratch_bytes = p->sub_batch * p->stages.y_samples * sizeof(c32);
    if (hipMalloc(&p->scratch, p->scratch_bytes) != hipSuccess) {
        p->scratch = nullptr;
        (void)hipGetLastError();
        return set_error(FFT_ERR_OUT_OF_MEMORY, "scratch of %zu bytes", p->scratch_bytes);
    }
    return set_ok();
}

int reject_real(const Plan *p, const char *what)
{
    if (p && is_real(p))
        return set_error(FFT_ERR_INVALID_ARG, "%s takes complex plans; real plans run through"
                         " fft_exec_segments", what);
    return FFT_OK;
}

void plan_free(Plan *p)
{
    if (p->used && p->last_stream_valid)
        (void)hipStreamSynchronize(p->last_stream);
    for (void *q : {p->tables, p->scratch})
        if (q)
            (void)hipFree(q);
    stream_state_free(p);
    if (p->graph_exec)
        (void)hipGraphExecDestroy(p->graph_exec);
    if (p->graph)
        (void)hipGraphDestroy(p->graph);
    if (p->capture_stream)
        (void)hipStreamDestroy(p->capture_stream);
    p->graph_exec = nullptr;
    p->graph = nullptr;
    p->capture_stream = nullptr;
    p->tables = p->tw = p->tw2 = p->tl = p->th = p->w1 = p->w2 = p->tl2 = p->th2 =
        p->scratch = nullptr;
}

// ---------------------------------------------------------------------------
// argument checks before any device work
int check_device_range(const void *ptr, uint64_t bytes, const char *name)
{
    void *base = nullptr;
    size_t size = 0;
    hipError_t e = hipMemGetAddressRange(&base, &size, const_cast<void *>(ptr));
    if (e == hipSuccess && base) {
        const uintptr_t b = (uintptr_t)base, q = (uintptr_t)ptr;
        if (q < b || q - b > size || bytes > size - (q - b))
            return set_error(FFT_ERR_BOUNDS,
                             "%s: %llu bytes from %p exceed its allocation [%p, +%zu)", name,
                             (unsigned long long)bytes, ptr, base, size);
        return FFT_OK;
    }
    (void)hipGetLastError();
    hipPointerAttribute_t attr;
    std::memset(&attr, 0, sizeof(attr));
    e = hipPointerGetAttributes(&attr, ptr);
    if (e != hipSuccess) {
        (void)hipGetLastError();
        return set_error(FFT_ERR_INVALID_ARG, "%s (%p) is not device memory", name, ptr);
    }
    if (attr.type != hipMemoryTypeDevice && attr.type != hipMemoryTypeManaged)
        return set_error(FFT_ERR_INVALID_ARG, "%s (%p) is not device memory", name, ptr);
    return FFT_OK;
}

int check_io(const void *in, const void *out, uint64_t bytes)
{
    if (!in || !out)
        return set_error(FFT_ERR_INVALID_ARG, "in/out must not be NULL");
    if (((uintptr_t)in & 7u) || ((uintptr_t)out & 7u))
        return set_error(FFT_ERR_ALIGNMENT, "in/out must be 8-byte aligned");
    if (in != out) {
        const uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
        if (a < b + bytes && b < a + bytes)
            return set_error(FFT_ERR_OVERLAP, "in and out overlap without being equal");
    }
    int st = check_device_range(in, bytes, "in");
    if (st != FFT_OK)
        return st;
    if (in != out && (st = check_device_range(out, bytes, "out")) != FFT_OK)
        return st;
    return FFT_OK;
}

// ---------------------------------------------------------------------------
// Identity transform (segment length 1) as a streaming copy.  Each
// workgroup moves one tile of 256 x K accesses, all loads issued before the
// stores, non-temporal; 16-byte accesses when both pointers allow them and
// the sample count is even, else 8-byte ones.  The dynamic LDS of each
// launch is not used: it holds residency at 3 workgroups per CU, which
// measured faster (5.8 TB/s) than the 8 the registers allow (5.4 TB/s) or
// a device-to-device hipMemcpyAsync (4.3 TB/s).
typedef float f4v __attribute__((ext_vector_type(4)));
typedef float f2v __attribute__((ext_vector_type(2)));
constexpr unsigned kCopyLds = 48 * 1024;

template <class T, int K>
__global__ void __launch_bounds__(256)
    identity_copy_kernel(const T *__restrict__ in, T *__restrict__ out, uint64_t n)
{
    extern __shared__ float unused_lds[];
    const uint64_t tile = 256ull * K;
    for (uint64_t base = (uint64_t)blockIdx.x * tile; base < n; base += (uint64_t)gridDim.x * tile) {
        T v[K];
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t i = base + threadIdx.x + 256ull * k;
            if (i < n)
                v[k] = __builtin_nontemporal_load(in + i);
        }
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t i = base + threadIdx.x + 256ull * k;
            if (i < n)
                __builtin_nontemporal_store(v[k], out + i);
        }
    }
    if (n == UINT64_MAX)  // never true: keeps the (unused) allocation referenced
        unused_lds[threadIdx.x] = 0.f;
}

template <class T, int K>
int identity_copy(const void *in, void *out, uint64_t n, hipStream_t s)
{
    const uint64_t tiles = (n + 256ull * K - 1) / (256ull * K);
    const unsigned grid = (unsigned)std::max<uint64_t>(1, std::min<uint64_t>(tiles, 0x7fffffffull));
    hipLaunchKernelGGL((identity_copy_kernel<T, K>), dim3(grid), dim3(256), kCopyLds, s,
                       (const T *)in, (T *)out, n);
    const hipError_t e = hipGetLastError();
    return e == hipSuccess ? FFT_OK : hip_error(e, "identity copy");
}

// GENERIC plans: segment s starts at in + s * hop, times window (or null)
hipError_t stages_enqueue(const Plan *p, const void *in, void *out, uint64_t batch, uint64_t hop,
                          const float *window, hipStream_t s)
{
    if (p->stages.passes == 1)
        return stages_one_pass(p->stages, p->dir, in, out, p->tw, batch, hop, window, s);
    for (uint64_t s0 = 0; s0 < batch; s0 += p->sub_batch) {
        const hipError_t e = stages_two_pass(
            p->stages, p->dir, (const c32 *)in + s0 * hop, (c32 *)out + s0 * p->n, p->scratch,
            {p->tw, p->tw2, p->w1, p->tl, p->th, p->sh, p->tl2, p->th2, p->sh2},
            std::min(p->sub_batch, batch - s0), hop, window, s);
        if (e != hipSuccess)
            return e;
    }
    return hipSuccess;
}

// the grid of a one-pass plan whose output starts out_m samples into a line
static unsigned single_grid(const Plan *p, uint64_t batch, uint64_t out_m)
{
    // (streamed stores that split 64-byte blocks: consecutive workgroups
    // close together write the halves in time; 1536 points, 2^25 samples
    // at an output base of 24 bytes 118 us against 130 walking)
    const SinglePassDesc *d = p->sp;
    return grid_for(d->kernel[p->dir > 0], d->threads * d->segs_per_wg,
                    (batch + d->segs_per_wg - 1) / d->segs_per_wg, p->device, p->grid_mult,
                    p->own_grid && !(d->nontemporal && out_m % 8) ? d->walk : 1);
}

static unsigned real_grid(const Plan *p, uint64_t batch)
{
    const SinglePassDesc *d = p->sp;
    return grid_for(d->kernel_real[p->dir > 0], d->threads * d->segs_per_wg,
                    (batch + d->segs_per_wg - 1) / d->segs_per_wg, p->device, p->grid_mult,
                    p->own_grid ? d->walk_aux : 1);
}

// the grids of a two-pass plan's passes over sb segments
static unsigned column_grid(const Plan *p, uint64_t sb)
{
    const ColumnDesc *d = p->col;
    return tile_grid(p, d->kernel[p->dir > 0], d->threads * d->cols,
                     sb * (p->n2 / (uint64_t)d->cols), one_wave_columns(p->n1));
}

static unsigned row_grid(const Plan *p, uint64_t sb)
{
    const RowDesc *d = p->row;
    return tile_grid(p, d->kernel[p->dir > 0], d->threads * d->rows,
                     sb * (p->n1 / (uint64_t)d->rows), one_wave_rows(p->n2));
}

// enqueue the transform of `batch` segments (arguments already checked)
int plan_enqueue(Plan *p, const void *in, void *out, uint64_t batch, hipStream_t s)
{
    const uint64_t n = p->n;
    const int dir = p->dir;
    switch (p->kind) {
    case Plan::COPY:
        if (in != out) {
            const bool wide = ((((uintptr_t)in | (uintptr_t)out) & 15u) == 0) && !(batch & 1);
            const int st = wide ? identity_copy<f4v, 8>(in, out, batch / 2, s)
                                : identity_copy<f2v, 16>(in, out, batch, s);
            if (st != FFT_OK)
                return st;
        }
        break;
    case Plan::SINGLE: {
        const SinglePassDesc *d = p->sp;
        const uint64_t groups = (batch + d->segs_per_wg - 1) / d->segs_per_wg;
        // an output base inside a 128-byte line: the kernel with rotated
        // lanes puts each wave's stores back on line boundaries
        const uint64_t out_m = ((uintptr_t)out / sizeof(c32)) % kLineSamples;
        if (out_m) {
            int rv = -1;
            const void *rk[2] = {nullptr, nullptr};
            const sp_rotated_launch_fn rl = rotated_launcher(n, &rv, rk);
            if (rl && rv == d->variant) {
                const unsigned grid = grid_for(rk[dir > 0], d->threads * d->segs_per_wg, groups,
                                               p->device, p->grid_mult,
                                               p->own_grid ? d->walk : 1);
                rl(dir, in, out, p->tw, batch, (int)((kLineSamples - out_m) % kLineSamples),
                   grid, s);
                break;
            }
        }
        d->launch(dir, in, out, p->tw, batch, single_grid(p, batch, out_m), s);
        break;
    }
    case Plan::REAL: {
        p->sp->launch_real(dir, in, out, p->tw, p->tw2, batch, real_grid(p, batch), s);
        break;
    }
    case Plan::REAL_STAGES: {
        const uint64_t m = n / 2;
        if (p->stages.passes == 1) {
            const hipError_t e =
                stages_real_one_pass(p->stages, in, out, p->tw, p->w1, batch, s);
            if (e != hipSuccess)
                return hip_error(e, "real-input launch");
            break;
        }
        // rows of m complex values (n floats) and of m + 1 bins
        const uint64_t ir = dir < 0 ? m : m + 1, orow = dir < 0 ? m + 1 : m;
        for (uint64_t s0 = 0; s0 < batch; s0 += p->sub_batch) {
            const hipError_t e = stages_real_two_pass(
                p->stages, (const c32 *)in + s0 * ir, (c32 *)out + s0 * orow, p->scratch, p->tw,
                p->tw2, p->tl, p->th, p->sh, p->w1, p->w2, std::min(p->sub_batch, batch - s0),
                s);
            if (e != hipSuccess)
                return hip_error(e, "real-input launch");
        }
        break;
    }
    case Plan::FOURSTEP: {
        const ColumnDesc *cd = p->col;
        const RowDesc *rd = p->row;
        // Segments that start inside a 128-byte line (a base pointer off a
        // line boundary): column blocks start at the first line-aligned
        // column and wrap round, Y sits at the input's offset within a
        // line, and row blocks start where the output's lines do, so both
        // passes move whole lines.  The shifted forms exist for each
        // length's default tiles.
        const uint64_t in_m = ((uintptr_t)in / sizeof(c32)) % kLineSamples,
                       out_m = ((uintptr_t)out / sizeof(c32)) % kLineSamples;
        if (in_m || out_m) {
            const ColumnDesc *cs = cd->launch_shifted ? cd : find_column_shifted(p->n1);
            const RowDesc *rs = rd->launch_shifted ? rd : find_row_shifted(p->n2);
            if (cs && rs && p->n2 % (uint64_t)cs->cols == 0 && p->n1 % (uint64_t)rs->rows == 0) {
                const int sa = (int)((kLineSamples - in_m) % kLineSamples);
                const int sb = (int)((kLineSamples - out_m) % kLineSamples);
                c32 *ybuf = (c32 *)p->scratch + in_m;
                for (uint64_t s0 = 0; s0 < batch; s0 += p->sub_batch) {
                    const uint64_t sbat = std::min(p->sub_batch, batch - s0);
                    const uint64_t ta = sbat * (p->n2 / (uint64_t)cs->cols);
                    const uint64_t tb = sbat * (p->n1 / (uint64_t)rs->rows);
                    const unsigned ga = tile_grid(p, cs->kernel_shifted[dir > 0],
                                                  cs->threads * cs->cols, ta,
                                                  one_wave_columns(p->n1));
                    const unsigned gb = tile_grid(p, rs->kernel_shifted[dir > 0],
                                                  rs->threads * rs->rows, tb,
                                                  one_wave_rows(p->n2));
                    cs->launch_shifted(dir, (const c32 *)in + s0 * n, ybuf, p->tw, p->tl, p->th,
                                       p->sh, (int)p->n2, sbat, sa, ga, s);
                    rs->launch_shifted(dir, ybuf, (c32 *)out + s0 * n, p->tw2, (int)p->n1, sbat,
                                       sb, gb, s);
                }
                break;
            }
        }
        for (uint64_t s0 = 0; s0 < batch; s0 += p->sub_batch) {
            const uint64_t sb = std::min(p->sub_batch, batch - s0);
            const c32 *x = (const c32 *)in + s0 * n;
            c32 *y = (c32 *)out + s0 * n;
            const unsigned ga = column_grid(p, sb), gb = row_grid(p, sb);
            (p->y_blocked ? cd->launch_yblocked : cd->launch)(dir, x, p->scratch, p->tw, p->tl,
                                                              p->th, p->sh, (int)p->n2, sb,
                                                              ga, s);
            (p->y_blocked ? rd->launch_yblocked : rd->launch)(dir, p->scratch, y, p->tw2,
                                                              (int)p->n1, sb, gb, s);
        }
        break;
    }
    case Plan::GENERIC: {
        const hipError_t e = stages_enqueue(p, in, out, batch, n, nullptr, s);
        if (e != hipSuccess)
            return hip_error(e, "schedule launch");
        break;
    }
    }
    hipError_t e = hipGetLastError();
    if (e != hipSuccess)
        return hip_error(e, "kernel launch");
    p->used = true;
    p->last_stream = s;
    p->last_stream_valid = true;
    return set_ok();
}

int plan_describe(const Plan *p, std::string &js)
{
    char buf[1024];
    auto rad = [](const int *r, int n) {
        std::string s = "[";
        for (int i = 0; i < n; ++i)
            s += (i ? "," : "") + std::to_string(r[i]);
        return s + "]";
    };
    switch (p->kind) {
    case Plan::COPY:
        snprintf(buf, sizeof buf, "{\"kind\":\"copy\",\"n\":%llu,\"batch\":%llu}",
                 (unsigned long long)p->n, (unsigned long long)p->batch);
        break;
    case Plan::SINGLE:
        snprintf(buf, sizeof buf,
                 "{\"kind\":\"single_pass\",\"n\":%llu,\"batch\":%llu,\"direction\":%d,"
                 "\"variant\":%d,\"radices\":%s,\"threads_per_segment\":%d,"
                 "\"segments_per_workgroup\":%d,\"lds_pad_shift\":%d,\"nontemporal\":%d,"
                 "\"lds_bytes\":%d,\"shuffle_exchange\":%d,\"grid_mult\":%d,"
                 "\"workgroups\":%u,\"scratch_bytes\":0}",
                 (unsigned long long)p->n, (unsigned long long)p->batch, p->dir,
                 p->sp->variant, rad(p->sp->radices, p->sp->nrad).c_str(), p->sp->threads,
                 p->sp->segs_per_wg, p->sp->pad_shift, p->sp->nontemporal,
                 p->sp->lds_bytes, p->sp->shuffle, p->grid_mult, single_grid(p, p->batch, 0));
        break;
    case Plan::FOURSTEP:
        snprintf(buf, sizeof buf,
                 "{\"kind\":\"four_step\",\"n\":%llu,\"batch\":%llu,\"direction\":%d,"
                 "\"n1\":%llu,\"n2\":%llu,\"radices_n1\":%s,\"radices_n2\":%s,"
                 "\"columns_per_workgroup\":%d,\"rows_per_workgroup\":%d,"
                 "\"column_variant\":%d,\"row_variant\":%d,\"grid_mult\":%d,"
                 "\"lds_bytes\":[%d,%d],\"sub_batch\":%llu,\"scratch_bytes\":%zu,"
                 "\"y_blocked\":%d,\"workgroups\":[%u,%u]}",
                 (unsigned long long)p->n, (unsigned long long)p->batch, p->dir,
                 (unsigned long long)p->n1, (unsigned long long)p->n2,
                 rad(p->col->radices, p->col->nrad).c_str(),
                 rad(p->row->radices, p->row->nrad).c_str(), p->col->cols, p->row->rows,
                 p->col->variant, p->row->variant, p->grid_mult,
                 p->col->lds_bytes, p->row->lds_bytes, (unsigned long long)p->sub_batch,
                 p->scratch_bytes, (int)p->y_blocked, column_grid(p, p->sub_batch),
                 row_grid(p, p->sub_batch));
        break;
    case Plan::REAL:
        snprintf(buf, sizeof buf,
                 "{\"kind\":\"real\",\"n\":%llu,\"batch\":%llu,\"direction\":%d,"
                 "\"complex_length\":%llu,\"radices\":%s,\"threads_per_segment\":%d,"
                 "\"segments_per_workgroup\":%d,\"grid_mult\":%d,"
                 "\"workgroups\":%u,\"scratch_bytes\":0}",
                 (unsigned long long)p->n, (unsigned long long)p->batch, p->dir,
                 (unsigned long long)(p->n / 2), rad(p->sp->radices, p->sp->nrad).c_str(),
                 p->sp->threads, p->sp->segs_per_wg, p->grid_mult, real_grid(p, p->batch));
        break;
    case Plan::REAL_STAGES: {
        // ("separate_split" is 1 where the plan takes two passes, the split in one of
        // them; it once had a pass of its own)
        std::vector<int> r;
        const StagesPlan &g = p->stages;
        lds_radices(g.a, &r);
        if (g.passes == 2)
            lds_radices(g.b, &r);
        snprintf(buf, sizeof buf,
                 "{\"kind\":\"real\",\"n\":%llu,\"batch\":%llu,\"direction\":%d,"
                 "\"complex_length\":%llu,\"separate_split\":%d,\"radices\":%s,\"passes\":%d,"
                 "\"n1\":%d,\"n2\":%d,\"threads\":[%d,%d],\"sub_batch\":%llu,"
                 "\"scratch_bytes\":%zu}",
                 (unsigned long long)p->n, (unsigned long long)p->batch, p->dir,
                 (unsigned long long)(p->n / 2), g.passes == 2,
                 rad(r.data(), (int)r.size()).c_str(), g.passes, g.a.n,
                 g.passes == 2 ? g.b.n : 1, g.threads_a, g.threads_b,
                 (unsigned long long)p->sub_batch, p->scratch_bytes);
        break;
    }
    case Plan::GENERIC: {
        std::vector<int> r;
        const StagesPlan &g = p->stages;
        lds_radices(g.a, &r);
        if (g.passes == 3)
            lds_radices(g.mid, &r);
        if (g.passes > 1)
            lds_radices(g.b, &r);
        snprintf(buf, sizeof buf,
                 "{\"kind\":\"radix_stages\",\"n\":%llu,\"batch\":%llu,\"direction\":%d,"
                 "\"radices\":%s,\"passes\":%d,\"n1\":%d,\"n2\":%d,\"n3\":%d,"
                 "\"segments_per_workgroup\":%d,\"columns_per_workgroup\":%d,"
                 "\"rows_per_workgroup\":%d,\"threads\":[%d,%d],\"sub_batch\":%llu,"
                 "\"scratch_bytes\":%zu}",
                 (unsigned long long)p->n, (unsigned long long)p->batch, p->dir,
                 rad(r.data(), (int)r.size()).c_str(), g.passes, g.a.n,
                 g.passes == 3 ? g.mid.n : g.passes == 2 ? g.b.n : 1, g.passes == 3 ? g.b.n : 1,
                 g.passes == 1 ? g.segs : 0, g.passes > 1 ? 1 << g.lc : 0,
                 g.passes > 1 ? 1 << g.lr : 0, g.threads_a, g.threads_b,
                 (unsigned long long)p->sub_batch, p->scratch_bytes);
        break;
    }
    }
    js = buf;
    return FFT_OK;
}

int validate_create(uint64_t n, uint64_t batch, int dir)
{
    if (n == 0)
        return set_error(FFT_ERR_INVALID_ARG, "segment_len must be > 0");
    if (batch == 0)
        return set_error(FFT_ERR_INVALID_ARG, "batch must be > 0");
    if (dir != FFT_FORWARD && dir != FFT_INVERSE)
        return set_error(FFT_ERR_INVALID_ARG, "direction must be -1 or +1 (got %d)", dir);
    if (n > (1ull << 24))
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH, "segment_len %llu exceeds 2^24",
                         (unsigned long long)n);
    if (!smooth235(n))
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH,
                         "segment_len %llu has a prime factor other than 2, 3, 5",
                         (unsigned long long)n);
    if (batch > SIZE_MAX / 8 / n)
        return set_error(FFT_ERR_INVALID_ARG, "batch * segment_len * 8 overflows size_t");
    return FFT_OK;
}

int factorize(uint64_t n, int *radices, int max)
{
    if (n == 0)
        return set_error(FFT_ERR_INVALID_ARG, "n must be > 0");
    if (n > (1ull << 24) || !smooth235(n))
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH, "unsupported length %llu",
                         (unsigned long long)n);
    std::vector<int> r;
    int v = tuned_variant(n);
    const SinglePassDesc *d = find_single(n, v < 0 ? 0 : v);
    if (!d)
        d = find_single(n, 0);
    const ColumnDesc *cd = nullptr;
    const RowDesc *rd = nullptr;
    StagesPlan g;
    if (d) {
        r.assign(d->radices, d->radices + d->nrad);
    } else if (n > 1 && !find_split(n, &cd, &rd, 0, 0) && stages_choose(n, 1, 1, &g)) {
        lds_radices(g.a, &r);
        if (g.passes == 3)
            lds_radices(g.mid, &r);
        if (g.passes > 1)
            lds_radices(g.b, &r);
    } else {
        r = generic_radices(n);
    }
    if (!radices && max != 0)
        return set_error(FFT_ERR_INVALID_ARG, "radices is NULL");
    for (int i = 0; i < (int)r.size() && i < max; ++i)
        radices[i] = r[i];
    set_ok();
    return (int)r.size();
}

}  // namespace fftseg

// ===========================================================================
// C entry points
using namespace fftseg;

#define FFT_GUARD_BEGIN try {
#define FFT_GUARD_END(ret)                                                         \
    }                                                                              \
    catch (const std::bad_alloc &)                                                 \
    {                                                                              \
        set_error(FFT_ERR_OUT_OF_MEMORY, "host allocation failed");                \
        return ret;                                                                \
    }                                                                              \
    catch (...)                                                                    \
    {                                                                              \
        set_error(FFT_ERR_INVALID_ARG, "internal error");                          \
        return ret;                                                                \
    }

static fft_plan_t create_impl(size_t segment_len, size_t batch, int direction, int variant,
                              int split = -1)
{
    if (validate_create(segment_len, batch, direction) != FFT_OK)
        return nullptr;
    Plan *p = new Plan();
    if (plan_build(p, segment_len, batch, direction, variant, split) != FFT_OK) {
        const int st = last_status();
        std::string msg = last_message();
        plan_free(p);
        delete p;
        set_error(st, "%s", msg.c_str());
        return nullptr;
    }
    return reinterpret_cast<fft_plan_t>(p);
}

extern "C" fft_plan_t fft_plan_create(size_t segment_len, size_t batch, int direction)
{
    FFT_GUARD_BEGIN
    return create_impl(segment_len, batch, direction, -1);
    FFT_GUARD_END(nullptr)
}

extern "C" fft_plan_t fft_plan_create_variant(size_t segment_len, size_t batch,
                                              int direction, int variant)
{
    FFT_GUARD_BEGIN
    if (variant < 0) {
        set_error(FFT_ERR_INVALID_ARG, "variant must be >= 0");
        return nullptr;
    }
    return create_impl(segment_len, batch, direction, variant);
    FFT_GUARD_END(nullptr)
}

extern "C" fft_plan_t fft_plan_create_real(size_t segment_len, size_t batch, int direction)
{
    FFT_GUARD_BEGIN
    if (validate_create(segment_len, batch, direction) != FFT_OK)
        return nullptr;
    if (segment_len < 4 || segment_len % 2) {
        set_error(FFT_ERR_UNSUPPORTED_LENGTH, "real segments need an even length >= 4 (got %zu)",
                  segment_len);
        return nullptr;
    }
    Plan *p = new Plan();
    if (plan_build_real(p, segment_len, batch, direction) != FFT_OK) {
        const int st = last_status();
        std::string msg = last_message();
        plan_free(p);
        delete p;
        set_error(st, "%s", msg.c_str());
        return nullptr;
    }
    return reinterpret_cast<fft_plan_t>(p);
    FFT_GUARD_END(nullptr)
}

extern "C" int fft_split_info(size_t n, size_t *n1, size_t *n2, int *ncol, int *nrow)
{
    FFT_GUARD_BEGIN
    int c = 0, r = 0;
    const ColumnDesc *cd = nullptr;
    const RowDesc *rd = nullptr;
    const bool two = n > 0 && variant_count(n) == 0 && find_split(n, &cd, &rd, 0, 0);
    if (two)
        split_variant_counts(n, &c, &r);
    if (n1)
        *n1 = two ? (size_t)cd->n1 : 0;
    if (n2)
        *n2 = two ? (size_t)rd->n2 : 0;
    if (ncol)
        *ncol = c;
    if (nrow)
        *nrow = r;
    set_ok();
    return two ? 1 : 0;
    FFT_GUARD_END(FFT_ERR_INVALID_ARG)
}

extern "C" fft_plan_t fft_plan_create_split(size_t segment_len, size_t batch, int direction,
                                            int column_variant, int row_variant)
{
    FFT_GUARD_BEGIN
    int c = 0, r = 0;
    if (validate_create(segment_len, batch, direction) != FFT_OK)
        return nullptr;
    if (variant_count(segment_len) != 0 || !split_variant_counts(segment_len, &c, &r)) {
        set_error(FFT_ERR_INVALID_ARG, "length %zu is not a two-pass length", segment_len);
        return nullptr;
    }
    if (column_variant < 0 || column_variant >= c || row_variant < 0 || row_variant >= r) {
        set_error(FFT_ERR_INVALID_ARG, "tile variants (%d, %d) outside [0, %d) x [0, %d)",
                  column_variant, row_variant, c, r);
        return nullptr;
    }
    return create_impl(segment_len, batch, direction, -1, column_variant | (row_variant << 8));
    FFT_GUARD_END(nullptr)
}

extern "C" int fft_variant_count(size_t n)
{
    set_ok();
    return variant_count(n);
}

extern "C" int fft_exec_segments_n(fft_plan_t plan, const void *in, void *out,
                                   size_t batch, void *stream)
{
    FFT_GUARD_BEGIN
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (!p)
        return set_error(FFT_ERR_INVALID_ARG, "plan is NULL");
    if (batch == 0 || batch > p->batch)
        return set_error(FFT_ERR_INVALID_ARG, "batch %zu outside [1, %llu]", batch,
                         (unsigned long long)p->batch);
    int st;
    if (is_real(p)) {
        // forward: n floats in, n/2+1 complex out; inverse the other way round
        const uint64_t rb = (uint64_t)batch * p->n * sizeof(float);
        const uint64_t cb = (uint64_t)batch * (p->n / 2 + 1) * sizeof(c32);
        const uint64_t ib = p->dir < 0 ? rb : cb, ob = p->dir < 0 ? cb : rb;
        if (!in || !out)
            return set_error(FFT_ERR_INVALID_ARG, "in/out must not be NULL");
        if (((uintptr_t)in & 7u) || ((uintptr_t)out & 7u))
            return set_error(FFT_ERR_ALIGNMENT, "in/out must be 8-byte aligned");
        const uintptr_t a = (uintptr_t)in, b = (uintptr_t)out;
        if (a < b + ob && b < a + ib)
            return set_error(FFT_ERR_OVERLAP, "real transforms run out of place: in and out"
                             " overlap");
        if ((st = check_device_range(in, ib, "in")) != FFT_OK ||
            (st = check_device_range(out, ob, "out")) != FFT_OK)
            return st;
    } else {
        const uint64_t bytes = (uint64_t)batch * p->n * sizeof(c32);
        st = check_io(in, out, bytes);
        if (st != FFT_OK)
            return st;
    }
    int cur = -1;
    if (hipGetDevice(&cur) != hipSuccess)
        return hip_error(hipGetLastError(), "hipGetDevice");
    if (cur != p->device && hipSetDevice(p->device) != hipSuccess)
        return hip_error(hipGetLastError(), "hipSetDevice");
    st = plan_enqueue(p, in, out, batch, (hipStream_t)stream);
    if (cur != p->device)
        (void)hipSetDevice(cur);
    return st;
    FFT_GUARD_END(FFT_ERR_INVALID_ARG)
}

extern "C" int fft_exec_segments(fft_plan_t plan, const void *in, void *out, void *stream)
{
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (!p)
        return set_error(FFT_ERR_INVALID_ARG, "plan is NULL");
    return fft_exec_segments_n(plan, in, out, p->batch, stream);
}

extern "C" int fft_plan_destroy(fft_plan_t plan)
{
    FFT_GUARD_BEGIN
    Plan *p = reinterpret_cast<Plan *>(plan);
    if (!p)
        return set_ok();
    plan_free(p);
    delete p;
    return set_ok();
    FFT_GUARD_END(FFT_ERR_INVALID_ARG)
}

extern "C" int fft_last_status(void) { return last_status(); }
extern "C" const char *fft_last_error(void) { return last_message(); }

extern "C" int fft_plan_factorize(size_t n, int *radices, int max)
{
    FFT_GUARD_BEGIN
    return factorize(n, radices, max);
    FFT_GUARD_END(FFT_ERR_INVALID_ARG)
}

extern "C" int fft_plan_describe(fft_plan_t plan, char *buf, size_t len)
{
    FFT_GUARD_BEGIN
    const Plan *p = reinterpret_cast<const Plan *>(plan);
    if (!p)
        return set_error(FFT_ERR_INVALID_ARG, "plan is NULL");
    std::string js;
    plan_describe(p, js);
    if (buf && len) {
        const size_t k = std::min(len - 1, js.size());
        std::memcpy(buf, js.data(), k);
        buf[k] = 0;
    }
    set_ok();
    return (int)js.size();
    FFT_GUARD_END(FFT_ERR_INVALID_ARG)
}

extern "C" size_t fft_plan_scratch_bytes(fft_plan_t plan)
{
    const Plan *p = reinterpret_cast<const Plan *>(plan);
    if (!p) {
        set_error(FFT_ERR_INVALID_ARG, "plan is NULL");
        return 0;
    }
    set_ok();
    return p->scratch_bytes;
}
