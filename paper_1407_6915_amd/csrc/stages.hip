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
// radix moved 16 B/sample per stage with scattered stores (30011 segments
// of 360 points: 152 us before, 46 now; 1001 of 15625: 290 and 82; 16 of
// 3 x 2^20: 1188 and 575; 2 of 2^24: 1028 and 492).
#include "stages.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>

#include "runtime.hpp"

namespace fftseg {
namespace {

__device__ __forceinline__ int fast_div(int x, uint32_t m)
{
    return m ? (int)__umulhi((unsigned)x, m) : x;
}

// One stage of the tile.  Io maps a butterfly number g to butterfly b of
// transform c, gives the LDS slots of a transform's elements, and does the
// first stage's loads (gl) and the last stage's stores (gs).
template <int R, int D, class Io>
__device__ __forceinline__ void lds_stage(const Io &io, const LdsStage &st, bool gl, bool gs,
                                          c32 *lds, const c32 *__restrict__ tw)
{
    constexpr int U = lds_units(R, true);
    c32 v[U][R];
    int bb[U], cc[U];
    bool ok[U];
#pragma unroll
    for (int u = 0; u < U; ++u) {
        ok[u] = io.map(st, gs, (int)threadIdx.x + u * (int)blockDim.x, bb[u], cc[u]);
        if (ok[u]) {
            if (gl) {
                io.template load<R>(v[u], bb[u], cc[u], st.nb);
            } else {
                const c32 *p = lds + io.slot(bb[u], cc[u]);
                const int d = st.nb * io.step();
#pragma unroll
                for (int r = 0; r < R; ++r)
                    v[u][r] = p[r * d];
            }
        }
    }
    if (!gl && !gs)
        __syncthreads();
#pragma unroll
    for (int u = 0; u < U; ++u) {
        if (ok[u]) {
            const int b = bb[u];
            int q = b, k = 0;
            if (st.l > 1) {
                q = fast_div(b, st.ml);
                k = b - q * st.l;
                const c32 *t = tw + st.tw + k;
#pragma unroll
                for (int r = 1; r < R; ++r)
                    v[u][r] = twiddle<D>(v[u][r], t[(r - 1) * st.l]);
            }
            dft<R, D>(v[u]);
            if (gs) {
                io.template store<R, D>(v[u], b, cc[u], st.nb);
            } else {
                c32 *p = lds + io.slot(q * st.l * R + k, cc[u]);
                const int d = st.l * io.step();
#pragma unroll
                for (int r = 0; r < R; ++r)
                    p[r * d] = v[u][r];
            }
        }
    }
    if (!gs)
        __syncthreads();
}

template <int D, class Io>
__device__ __forceinline__ void run_stages(const Io &io, const LdsSched &s, bool first_lds,
                                           bool last_lds, c32 *lds, const c32 *__restrict__ tw)
{
    for (int i = 0; i < s.ns; ++i) {
        const LdsStage &st = s.st[i];
        const bool gl = i == 0 && !first_lds, gs = i + 1 == s.ns && !last_lds;
        switch (st.r) {
        case 2: lds_stage<2, D>(io, st, gl, gs, lds, tw); break;
        case 3: lds_stage<3, D>(io, st, gl, gs, lds, tw); break;
        case 4: lds_stage<4, D>(io, st, gl, gs, lds, tw); break;
        case 5: lds_stage<5, D>(io, st, gl, gs, lds, tw); break;
        case 6: lds_stage<6, D>(io, st, gl, gs, lds, tw); break;
        case 8: lds_stage<8, D>(io, st, gl, gs, lds, tw); break;
        case 9: lds_stage<9, D>(io, st, gl, gs, lds, tw); break;
        case 10: lds_stage<10, D>(io, st, gl, gs, lds, tw); break;
        case 12: lds_stage<12, D>(io, st, gl, gs, lds, tw); break;
        case 15: lds_stage<15, D>(io, st, gl, gs, lds, tw); break;
        case 16: lds_stage<16, D>(io, st, gl, gs, lds, tw); break;
        default: lds_stage<25, D>(io, st, gl, gs, lds, tw); break;
        }
    }
}

// Whole segments: transform c is segment c of the tile, its elements in
// consecutive slots; butterflies of a segment on consecutive lanes, so the
// first stage loads and the last stage stores runs of nb samples.
struct SegmentIo {
    const c32 *x;
    c32 *y;
    const float *window;
    uint64_t hop;
    int n, segs;  // segments the tile holds
    __device__ __forceinline__ bool map(const LdsStage &st, bool, int g, int &b, int &c) const
    {
        c = fast_div(g, st.mnb);
        b = g - c * st.nb;
        return c < segs;
    }
    __device__ __forceinline__ int slot(int i, int c) const { return c * n + i; }
    __device__ __forceinline__ int step() const { return 1; }
    template <int R>
    __device__ __forceinline__ void load(c32 *v, int b, int c, int nb) const
    {
        const c32 *p = x + (uint64_t)c * hop + b;
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = p[r * nb];
        if (window) {
            const float *w = window + b;
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float f = w[r * nb];
                v[r] = c32{v[r].x * f, v[r].y * f};
            }
        }
    }
    template <int R, int D>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        c32 *p = y + c * n + b;
#pragma unroll
        for (int r = 0; r < R; ++r)
            p[r * nb] = v[r];
    }
};

extern __shared__ c32 stage_lds[];

template <int D>
__global__ void __launch_bounds__(1024)
    stages_segments_kernel(const c32 *in, c32 *out, const c32 *__restrict__ tw, LdsSched s,
                           int segs, int staged, uint32_t mn, uint64_t batch, uint64_t hop,
                           const float *__restrict__ window)
{
    const uint64_t seg = (uint64_t)blockIdx.x * (unsigned)segs;
    const int have = (int)(batch - seg < (uint64_t)segs ? batch - seg : (uint64_t)segs);
    const SegmentIo io{in + seg * hop, out + seg * (unsigned)s.n, window, hop, s.n, have};
    if (staged) {
        for (int e = threadIdx.x; e < have * s.n; e += blockDim.x) {
            const int c = fast_div(e, mn), i = e - c * s.n;
            c32 a = io.x[(uint64_t)c * hop + i];
            if (window)
                a = c32{a.x * window[i], a.y * window[i]};
            stage_lds[e] = a;
        }
        __syncthreads();
    }
    run_stages<D>(io, s, staged != 0, staged != 0, stage_lds, tw);
    if (staged)
        for (int e = threadIdx.x; e < have * s.n; e += blockDim.x)
            io.y[e] = stage_lds[e];
}

// Four-step column pass: transform c is column first + c of the segment
// (elements n2 samples apart), columns on consecutive lanes, slots of one
// element row 2^lc + 1 apart.  The last stage instead puts 2^lr consecutive
// outputs k1 on consecutive lanes, then the columns: Y keeps the rows of one
// row tile together,
//     Y[(k1 >> lr)][n2][k1 mod 2^lr],
// so that a wave stores one run here and the row pass loads its tile as one.
struct ColumnIo {
    const c32 *x;
    c32 *y;
    const float *window;
    const c32 *__restrict__ tl;
    const c32 *__restrict__ th;
    int sh, n2, first, lc, lr;
    __device__ __forceinline__ bool map(const LdsStage &st, bool gs, int g, int &b, int &c) const
    {
        if (gs) {
            c = (g >> lr) & ((1 << lc) - 1);
            b = ((g >> (lr + lc)) << lr) | (g & ((1 << lr) - 1));
        } else {
            c = g & ((1 << lc) - 1);
            b = g >> lc;
        }
        return b < st.nb && first + c < n2;
    }
    __device__ __forceinline__ int step() const { return (1 << lc) + 1; }
    __device__ __forceinline__ int slot(int i, int c) const { return i * step() + c; }
    template <int R>
    __device__ __forceinline__ void load(c32 *v, int b, int c, int nb) const
    {
        const c32 *p = x + (b * n2 + first + c);
        const int d = nb * n2;
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = p[r * d];
        if (window) {
            const float *w = window + (b * n2 + first + c);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float f = w[r * d];
                v[r] = c32{v[r].x * f, v[r].y * f};
            }
        }
    }
    template <int R, int D>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        const unsigned col = (unsigned)(first + c), mask = (1u << sh) - 1u;
#pragma unroll
        for (int r = 0; r < R; ++r) {
            const unsigned k1 = (unsigned)(b + r * nb), m = col * k1;
            const c32 w = cmul(th[m >> sh], tl[m & mask]);
            y[((((k1 >> lr) * (unsigned)n2 + col) << lr) | (k1 & ((1u << lr) - 1u)))] =
                twiddle<D>(v[r], w);
        }
    }
};

// Four-step row pass: transform c is row first + c of Y (one contiguous tile,
// the rows on consecutive lanes), stored transposed as X[k1 + n1 k2].
struct RowIo {
    const c32 *x;  // the tile
    c32 *y;        // segment output
    int n1, first, lr;
    __device__ __forceinline__ bool map(const LdsStage &st, bool, int g, int &b, int &c) const
    {
        c = g & ((1 << lr) - 1);
        b = g >> lr;
        return b < st.nb && first + c < n1;
    }
    __device__ __forceinline__ int step() const { return 1 << lr; }
    __device__ __forceinline__ int slot(int i, int c) const { return (i << lr) + c; }
    template <int R>
    __device__ __forceinline__ void load(c32 *v, int b, int c, int nb) const
    {
        const c32 *p = x + slot(b, c);
        const int d = nb << lr;
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = p[r * d];
    }
    template <int R, int D>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        c32 *p = y + (b * n1 + first + c);
        const int d = nb * n1;
#pragma unroll
        for (int r = 0; r < R; ++r)
            p[r * d] = v[r];
    }
};

// Tile w of a grid of 8 * per workgroups, dealt so that each XCD (workgroup
// mod 8) takes consecutive tiles: neighbours share cache lines where the
// lengths are no multiple of 16.
__device__ __forceinline__ uint64_t xcd_tile()
{
    return (uint64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

template <int D>
__global__ void __launch_bounds__(1024)
    stages_columns_kernel(const c32 *in, c32 *ybuf, const c32 *__restrict__ tw,
                          const c32 *__restrict__ tl, const c32 *__restrict__ th, int sh,
                          LdsSched s, int n2, int lc, int lr, unsigned blocks, uint64_t tiles,
                          uint64_t ysamples, uint64_t hop, const float *__restrict__ window)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const int first = (int)(t - seg * blocks) << lc;
    const ColumnIo io{in + seg * hop, ybuf + seg * ysamples, window, tl, th, sh, n2, first, lc,
                      lr};
    run_stages<D>(io, s, false, false, stage_lds, tw);
}

template <int D>
__global__ void __launch_bounds__(1024)
    stages_rows_kernel(const c32 *ybuf, c32 *out, const c32 *__restrict__ tw, LdsSched s, int n1,
                       int lr, unsigned blocks, uint64_t tiles, uint64_t ysamples)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const unsigned blk = (unsigned)(t - seg * blocks);
    const RowIo io{ybuf + seg * ysamples + ((uint64_t)blk << lr) * (unsigned)s.n,
                   out + seg * ((uint64_t)n1 * (unsigned)s.n), n1, (int)(blk << lr), lr};
    run_stages<D>(io, s, false, false, stage_lds, tw);
}

// ---------------------------------------------------------------------------
// planner

constexpr int kRadixList[] = {25, 16, 15, 12, 10, 9, 8, 6, 5, 4, 3, 2};

// fewest stages, then the smallest sum of radices (the work of a stage grows
// with neither, its registers and idle threads do)
void best_radices(int n, int from, std::vector<int> &cur, std::vector<int> &best)
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
    if (!best.empty() && cur.size() + 1 > best.size())
        return;
    for (int i = from; i < (int)(sizeof(kRadixList) / sizeof(kRadixList[0])); ++i) {
        if (n % kRadixList[i])
            continue;
        cur.push_back(kRadixList[i]);
        best_radices(n / kRadixList[i], i, cur, best);
        cur.pop_back();
    }
}

uint32_t reciprocal(int d)
{
    return d <= 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d + 1);
}

constexpr int kLdsBytes = 160 * 1024;

}  // namespace

bool lds_schedule(int n, LdsSched *s)
{
    std::vector<int> cur, best;
    best_radices(n, 0, cur, best);
    if (best.empty() || (int)best.size() > kMaxLdsStages)
        return false;
    // the smallest odd radix first: the first stage writes LDS at a stride of
    // its radix, which odd strides spread over all banks
    std::sort(best.begin(), best.end(), std::greater<int>());
    for (int i = (int)best.size() - 1; i >= 0; --i)
        if (best[i] & 1) {
            std::rotate(best.begin(), best.begin() + i, best.begin() + i + 1);
            break;
        }
    *s = LdsSched{};
    s->n = n;
    s->ns = (int)best.size();
    int l = 1, tw = 0;
    for (int i = 0; i < s->ns; ++i) {
        const int r = best[i];
        s->st[i] = LdsStage{r, l, n / r, tw, reciprocal(l), reciprocal(n / r)};
        if (l > 1)
            tw += (r - 1) * l;
        l *= r;
    }
    return true;
}

int lds_threads(const LdsSched &s, int tiles, int group)
{
    int t = 64;
    for (int i = 0; i < s.ns; ++i) {
        int nb = s.st[i].nb;
        if (i + 1 == s.ns)
            nb = (nb + group - 1) / group * group;
        const long long total = (long long)nb * tiles;
        const int un = lds_units(s.st[i].r, false), um = lds_units(s.st[i].r, true);
        if ((total + um - 1) / um > 1024)
            return 0;
        t = std::max<int>(t, (int)std::min<long long>(1024, (total + un - 1) / un));
    }
    return (t + 63) / 64 * 64;
}

int lds_table_size(const LdsSched &s)
{
    return s.ns > 1 ? s.n - s.st[0].r : 0;
}

std::vector<c32> lds_table(const LdsSched &s)
{
    std::vector<c32> t((size_t)std::max(lds_table_size(s), 1));
    const std::vector<c32> w = root_table((uint64_t)s.n);
    for (int i = 1; i < s.ns; ++i) {
        const LdsStage &st = s.st[i];
        c32 *to = &t[(size_t)st.tw];
        for (int j = 1; j < st.r; ++j) {
            const int step = j * (s.n / (st.l * st.r));  // j k step < n
            for (int k = 0; k < st.l; ++k)
                *to++ = w[(size_t)k * step];
        }
    }
    return t;
}

void lds_radices(const LdsSched &s, std::vector<int> *out)
{
    for (int i = 0; i < s.ns; ++i) {
        if (s.st[i].r == 9)
            out->insert(out->end(), {3, 3});
        else
            out->push_back(s.st[i].r);
    }
}

bool stages_choose(uint64_t n, uint64_t batch, int cus, StagesPlan *p)
{
    *p = StagesPlan{};
    if (n * sizeof(c32) <= (uint64_t)kLdsBytes && lds_schedule((int)n, &p->a)) {
        // 4096 samples a workgroup (32 KB of LDS, several workgroups a CU),
        // fewer where the batch would leave CUs without work
        int segs = std::max(1, 4096 / (int)n);
        while (segs > 1 && (batch + segs - 1) / segs < 2 * (uint64_t)cus)
            segs = (segs + 1) / 2;
        p->segs = segs;
        p->staged = n < 256;
        p->threads_a = lds_threads(p->a, segs, 1);
        if (p->threads_a) {
            p->passes = 1;
            return true;
        }
    }
    // two passes: every n1 n2 whose tiles fit, the cheapest by the traffic
    // that partial lines add
    double best = 1e30;
    for (uint64_t n1 = 26; n1 <= n / 2 && n1 <= 16384; ++n1) {
        if (n % n1 || n / n1 > 16384)
            continue;
        const uint64_t n2 = n / n1;
        LdsSched a, b;
        if (!lds_schedule((int)n1, &a) || !lds_schedule((int)n2, &b) || a.ns < 2)
            continue;
        auto widest = [&](const LdsSched &s, bool column, int other) {
            for (int l = 4; l >= 0; --l) {
                const uint64_t pitch = (1u << l) + (column ? 1 : 0);
                if (s.n * pitch * sizeof(c32) <= (uint64_t)kLdsBytes &&
                    lds_threads(s, 1 << l, column ? 1 << other : 1))
                    return l;
            }
            return -1;
        };
        int lr = widest(b, false, 0);
        if (lr < 0)
            continue;
        int lc = widest(a, true, lr);
        if (lc < 0)
            continue;
        const double width[] = {8.0, 4.0, 1.8, 1.15, 1.0};
        const double score = width[lc] * (n2 % 16 ? 1.1 : 1.0) + width[lr] * (n1 % 16 ? 1.1 : 1.0) +
                             0.04 * (a.ns + b.ns) +
                             0.02 * std::fabs(std::log2((double)n1 / (double)n2));
        if (score >= best)
            continue;
        best = score;
        p->passes = 2;
        p->a = a;
        p->b = b;
        p->lc = lc;
        p->lr = lr;
    }
    if (p->passes != 2)
        return false;
    // few segments: narrower tiles until every CU has one
    const uint64_t n1 = (uint64_t)p->a.n, n2 = (uint64_t)p->b.n;
    while (p->lc > 2 && batch * ((n2 + (1u << p->lc) - 1) >> p->lc) < (uint64_t)cus)
        --p->lc;
    while (p->lr > 2 && batch * ((n1 + (1u << p->lr) - 1) >> p->lr) < (uint64_t)cus)
        --p->lr;
    p->threads_a = lds_threads(p->a, 1 << p->lc, 1 << p->lr);
    p->threads_b = lds_threads(p->b, 1 << p->lr, 1);
    p->y_samples = ((n1 + (1u << p->lr) - 1) >> p->lr << p->lr) * n2;
    return p->threads_a && p->threads_b;
}

namespace {

// the workgroup's LDS goes past the runtime's default limit
template <class K>
hipError_t allow_lds(K kernel, size_t bytes)
{
    if (bytes <= 64 * 1024)
        return hipSuccess;
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kLdsBytes);
}

template <int D>
hipError_t one_pass(const StagesPlan &p, const c32 *in, c32 *out, const c32 *tw, uint64_t batch,
                    uint64_t hop, const float *window, hipStream_t s)
{
    const size_t lds = (size_t)p.segs * p.a.n * sizeof(c32);
    const hipError_t e = allow_lds(stages_segments_kernel<D>, lds);
    if (e != hipSuccess)
        return e;
    const uint64_t groups = (batch + p.segs - 1) / p.segs;
    hipLaunchKernelGGL(stages_segments_kernel<D>, dim3((unsigned)groups), dim3(p.threads_a),
                       (unsigned)lds, s, in, out, tw, p.a, p.segs, p.staged,
                       reciprocal(p.a.n), batch, hop, window);
    return hipGetLastError();
}

unsigned xcd_grid(uint64_t tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

template <int D>
hipError_t two_pass(const StagesPlan &p, const c32 *in, c32 *out, c32 *y, const c32 *tw_a,
                    const c32 *tw_b, const c32 *tl, const c32 *th, int sh, uint64_t batch,
                    uint64_t hop, const float *window, hipStream_t s)
{
    const int n1 = p.a.n, n2 = p.b.n;
    const size_t lds_a = (size_t)n1 * ((1u << p.lc) + 1) * sizeof(c32);
    const size_t lds_b = (size_t)n2 * (1u << p.lr) * sizeof(c32);
    hipError_t e = allow_lds(stages_columns_kernel<D>, lds_a);
    if (e == hipSuccess)
        e = allow_lds(stages_rows_kernel<D>, lds_b);
    if (e != hipSuccess)
        return e;
    const unsigned ba = (unsigned)((n2 + (1 << p.lc) - 1) >> p.lc);
    const unsigned bb = (unsigned)((n1 + (1 << p.lr) - 1) >> p.lr);
    hipLaunchKernelGGL(stages_columns_kernel<D>, dim3(xcd_grid(batch * ba)), dim3(p.threads_a),
                       (unsigned)lds_a, s, in, y, tw_a, tl, th, sh, p.a, n2, p.lc, p.lr, ba,
                       batch * ba, p.y_samples, hop, window);
    hipLaunchKernelGGL(stages_rows_kernel<D>, dim3(xcd_grid(batch * bb)), dim3(p.threads_b),
                       (unsigned)lds_b, s, y, out, tw_b, p.b, n1, p.lr, bb, batch * bb,
                       p.y_samples);
    return hipGetLastError();
}

}  // namespace

hipError_t stages_one_pass(const StagesPlan &p, int dir, const void *in, void *out,
                           const void *tw, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s)
{
    return (dir < 0 ? one_pass<-1> : one_pass<1>)(p, (const c32 *)in, (c32 *)out, (const c32 *)tw,
                                                  batch, hop, window, s);
}

hipError_t stages_two_pass(const StagesPlan &p, int dir, const void *in, void *out, void *y,
                           const void *tw_a, const void *tw_b, const void *tl, const void *th,
                           int sh, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s)
{
    return (dir < 0 ? two_pass<-1> : two_pass<1>)(
        p, (const c32 *)in, (c32 *)out, (c32 *)y, (const c32 *)tw_a, (const c32 *)tw_b,
        (const c32 *)tl, (const c32 *)th, sh, batch, hop, window, s);
}

}  // namespace fftseg
