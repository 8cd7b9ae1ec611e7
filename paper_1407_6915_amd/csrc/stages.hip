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
// of 360 points: 152 us before, 45 now; 1001 of 15625: 290 and 78; 16 of
// 3 x 2^20: 1188 and 478; 2 of 2^24: 1028 and 492).  One pass moves 4.4 to
// 5.1 TB/s up to 4096 points and 3.0 to 4.0 above, where one or two
// workgroups fill a CU's LDS and little of a tile's loads overlaps another's
// stages; two passes 4.2 to 5.3 with tiles of two workgroups a CU, 2.5 to
// 3.9 with larger ones (2^26 samples).
#include "stages.hpp"

#include <algorithm>
#include <cmath>
#include <mutex>

#include "runtime.hpp"
#include "tile.hpp"

namespace fftseg {
namespace {

__device__ __forceinline__ int fast_div(int x, uint32_t m)
{
    return m ? (int)__umulhi((unsigned)x, m) : x;
}

// Memory seen through a buffer descriptor: an access is at a uniform
// offset (in samples) plus a lane's offset (in bytes).  The element strides
// of a butterfly are uniform, so its R accesses share one offset register
// and take the rest from scalar ones.  Offsets stay below 2^31 bytes.
struct Buffer {
    __amdgpu_buffer_rsrc_t r;
    __device__ __forceinline__ explicit Buffer(const void *p)
        : r(__builtin_amdgcn_make_buffer_rsrc(const_cast<void *>(p), 0, 0x7fffffff, 0x00027000))
    {
    }
    __device__ __forceinline__ c32 load(unsigned lane, int uniform) const
    {
        return __builtin_bit_cast(c32,
                                  __builtin_amdgcn_raw_buffer_load_b64(r, lane, 8 * uniform, 0));
    }
    __device__ __forceinline__ float load_float(unsigned lane, int uniform) const
    {
        return __builtin_bit_cast(float,
                                  __builtin_amdgcn_raw_buffer_load_b32(r, lane, 4 * uniform, 0));
    }
    __device__ __forceinline__ void store(unsigned lane, int uniform, c32 v) const
    {
        typedef unsigned u2v __attribute__((ext_vector_type(2)));
        __builtin_amdgcn_raw_buffer_store_b64(__builtin_bit_cast(u2v, v), r, lane, 8 * uniform, 0);
    }
};

// One stage of the tile.  Io maps a butterfly number g to butterfly b of
// transform c, gives the LDS slots of a transform's elements, and does the
// first stage's loads (gl) and the last stage's stores (gs).
template <int R, int D, bool Most, class Io>
__device__ __forceinline__ void lds_stage(const Io &io, const LdsStage &st, bool gl, bool gs,
                                          c32 *lds, const Buffer &tw)
{
    constexpr int U = lds_units(R, Most);
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
                // radices from 12 on read theirs in pairs (tw_pair_low)
                constexpr int R1 = tw_pair_low(R);
                if constexpr (R1 > 0) {
                    c32 wl[R1];
#pragma unroll
                    for (int j = 1; j < R1; ++j) {
                        wl[j] = tw.load(8u * k, st.tw + (j - 1) * st.l);
                        v[u][j] = twiddle<D>(v[u][j], wl[j]);
                    }
#pragma unroll
                    for (int h = 1; h < R / R1; ++h) {
                        const c32 wh = tw.load(8u * k, st.tw + (h * R1 - 1) * st.l);
                        v[u][h * R1] = twiddle<D>(v[u][h * R1], wh);
#pragma unroll
                        for (int j = 1; j < R1; ++j)
                            v[u][h * R1 + j] = twiddle<D>(v[u][h * R1 + j], cmul(wh, wl[j]));
                    }
                } else {
#pragma unroll
                    for (int r = 1; r < R; ++r)
                        v[u][r] = twiddle<D>(v[u][r], tw.load(8u * k, st.tw + (r - 1) * st.l));
                }
            }
            dft<R, D>(v[u]);
            if (gs) {
                io.template finish<R, D>(v[u], b, cc[u], st.nb);
                io.template store<R>(v[u], b, cc[u], st.nb);
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

template <int D, bool Most, class Io>
__device__ __forceinline__ void run_stages(const Io &io, const LdsSched &s, c32 *lds,
                                           const c32 *table)
{
    const Buffer tw(table);
    for (int i = 0; i < s.ns; ++i) {
        const LdsStage &st = s.st[i];
        const bool gl = i == 0, gs = i + 1 == s.ns;
        switch (st.r) {
        case 2: lds_stage<2, D, Most>(io, st, gl, gs, lds, tw); break;
        case 3: lds_stage<3, D, Most>(io, st, gl, gs, lds, tw); break;
        case 4: lds_stage<4, D, Most>(io, st, gl, gs, lds, tw); break;
        case 5: lds_stage<5, D, Most>(io, st, gl, gs, lds, tw); break;
        case 6: lds_stage<6, D, Most>(io, st, gl, gs, lds, tw); break;
        case 8: lds_stage<8, D, Most>(io, st, gl, gs, lds, tw); break;
        case 9: lds_stage<9, D, Most>(io, st, gl, gs, lds, tw); break;
        case 10: lds_stage<10, D, Most>(io, st, gl, gs, lds, tw); break;
        case 12: lds_stage<12, D, Most>(io, st, gl, gs, lds, tw); break;
        case 15: lds_stage<15, D, Most>(io, st, gl, gs, lds, tw); break;
        case 16: lds_stage<16, D, Most>(io, st, gl, gs, lds, tw); break;
        default: lds_stage<25, D, Most>(io, st, gl, gs, lds, tw); break;
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
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *, int, int, int) const
    {
    }
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
        // (the launch keeps segs * hop below 2^28 samples)
        const Buffer xb(x);
        const unsigned at = 8u * ((unsigned)c * (unsigned)hop + (unsigned)b);
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = xb.load(at, r * nb);
        if (window) {
            const Buffer w(window);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float f = w.load_float(4u * b, r * nb);
                v[r] = c32{v[r].x * f, v[r].y * f};
            }
        }
    }
    template <int R>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        const Buffer yb(y);
        const unsigned at = 8u * (unsigned)(c * n + b);
#pragma unroll
        for (int r = 0; r < R; ++r)
            yb.store(at, r * nb, v[r]);
    }
};

extern __shared__ c32 stage_lds[];

template <int D, bool Most>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
    stages_segments_kernel(const c32 *in, c32 *out, const c32 *__restrict__ tw, LdsSched s,
                           int segs, uint64_t batch, uint64_t hop,
                           const float *__restrict__ window)
{
    const uint64_t seg = (uint64_t)blockIdx.x * (unsigned)segs;
    const int have = (int)(batch - seg < (uint64_t)segs ? batch - seg : (uint64_t)segs);
    const SegmentIo io{in + seg * hop, out + seg * (unsigned)s.n, window, hop, s.n, have};
    run_stages<D, Most>(io, s, stage_lds, tw);
}

// Four-step column pass: transform c is column first + c of the segment
// (elements n2 samples apart), columns on consecutive lanes, slots of one
// element row 2^lc + 1 apart.  The last stage instead puts 2^lr consecutive
// outputs k1 on consecutive lanes, then the columns: Y keeps the rows of one
// row tile together,
//     Y[(k1 >> lr)][n2][k1 mod 2^lr],
// so that a wave stores one run here and the row pass loads its tile as one
// W_N^{n2 k1} of output k1 = b + r nb is W_N^{n2 b}, looked up once per
// butterfly, times W_N^{n2 r nb}, looked up once per tile into LDS: a lookup
// is two gathers from tables of a few thousand entries, and one per output
// held the pass to half its rate (20000 points: 606 us per 2^26 samples).
struct ColumnIo {
    const c32 *x;
    c32 *y;
    const float *window;
    const c32 *__restrict__ tl;
    const c32 *__restrict__ th;
    const c32 *wr;  // LDS: W_N^{n2 r nb} of the last stage's outputs, [r][column]
    int sh, n2, first, lc, lr;
    __device__ __forceinline__ c32 root(unsigned m) const
    {
        return cmul(th[m >> sh], tl[m & ((1u << sh) - 1u)]);
    }
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
        const Buffer xb(x);
        const unsigned at = 8u * (unsigned)(b * n2 + first + c);
        const int d = nb * n2;
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = xb.load(at, r * d);
        if (window) {
            const Buffer w(window);
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const float f = w.load_float(at / 2, r * d);
                v[r] = c32{v[r].x * f, v[r].y * f};
            }
        }
    }
    template <int R>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        const unsigned col = (unsigned)(first + c);
        const Buffer yb(y);
        if ((nb & ((1 << lr) - 1)) == 0) {
            const unsigned at = 8u * y_at((unsigned)b, col);
#pragma unroll
            for (int r = 0; r < R; ++r)
                yb.store(at, r * nb * n2, v[r]);
        } else {
#pragma unroll
            for (int r = 0; r < R; ++r)
                yb.store(8u * y_at((unsigned)(b + r * nb), col), 0, v[r]);
        }
    }
    __device__ __forceinline__ unsigned y_at(unsigned k1, unsigned col) const
    {
        return (((k1 >> lr) * (unsigned)n2 + col) << lr) | (k1 & ((1u << lr) - 1u));
    }
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *v, int b, int c, int) const
    {
        const c32 wb = root((unsigned)(first + c) * (unsigned)b);
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = twiddle<D>(v[r], cmul(wb, wr[(r << lc) + c]));
    }
};

// Four-step row pass: transform c is row first + c of Y (one contiguous tile,
// the rows on consecutive lanes), stored transposed as X[k1 + n1 k2].
struct RowIo {
    const c32 *x;  // the tile
    c32 *y;        // segment output
    int n1, first, lr;
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *, int, int, int) const
    {
    }
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
        const Buffer xb(x);
        const unsigned at = 8u * (unsigned)slot(b, c);
        const int d = nb << lr;
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = xb.load(at, r * d);
    }
    template <int R>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        const Buffer yb(y);
        const unsigned at = 8u * (unsigned)(b * n1 + first + c);
        const int d = nb * n1;
#pragma unroll
        for (int r = 0; r < R; ++r)
            yb.store(at, r * d, v[r]);
    }
};

// Tile w of a grid of 8 * per workgroups, dealt so that each XCD (workgroup
// mod 8) takes consecutive tiles: neighbours share cache lines where the
// lengths are no multiple of 16.
__device__ __forceinline__ uint64_t xcd_tile()
{
    return (uint64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

template <int D, bool Most>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
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
    c32 *wr = stage_lds + s.n * ((1 << lc) + 1);
    const ColumnIo io{in + seg * hop, ybuf + seg * ysamples, window, tl, th, wr, sh, n2, first,
                      lc,             lr};
    // (read after the barriers of the first exchange)
    const LdsStage &last = s.st[s.ns - 1];
    for (int e = threadIdx.x; e < last.r << lc; e += blockDim.x) {
        const int r = e >> lc, col = first + (e & ((1 << lc) - 1));
        if (col < n2)
            wr[e] = io.root((unsigned)col * (unsigned)(r * last.nb));
    }
    run_stages<D, Most>(io, s, stage_lds, tw);
}

template <int D, bool Most>
__global__ void __launch_bounds__(1024) __attribute__((amdgpu_waves_per_eu(4, 4)))
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
    run_stages<D, Most>(io, s, stage_lds, tw);
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
        // (one stage of a composite length would put the lanes of a load n
        // samples apart: two stages ran at 4.6 TB/s where one ran at 2.8)
        if (n % kRadixList[i] || (cur.empty() && n == kRadixList[i] && n > 5))
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

// LDS of a column tile (with the last stage's W_N factors) and of a row tile
size_t columns_lds(const LdsSched &s, int lc)
{
    return ((size_t)s.n * ((1u << lc) + 1) + ((size_t)s.st[s.ns - 1].r << lc)) * sizeof(c32);
}
size_t rows_lds(const LdsSched &s, int lr) { return ((size_t)s.n << lr) * sizeof(c32); }

// log2 of a tile's columns or rows: the widest of 16 and 8 that leaves room
// for two workgroups on a CU (one loads while the other computes: 1000-point
// columns 325 us per 2^26 samples with 8, 356 with 16), else the widest that
// fits; -1 if none does
template <class Lds>
int widest(Lds lds)
{
    for (int l = 4; l >= 3; --l)
        if (lds(l) <= (size_t)kLdsBytes / 2)
            return l;
    for (int l = 4; l >= 0; --l)
        if (lds(l) <= (size_t)kLdsBytes)
            return l;
    return -1;
}

}  // namespace

bool lds_schedule(int n, LdsSched *s, int group)
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
        s->st[i] = LdsStage{r, l, n / r, tw, reciprocal(l), reciprocal(n / r)};
        if (l > 1)
            tw += (r - 1) * l;
        l *= r;
    }
    return true;
}

int lds_threads(const LdsSched &s, int tiles, int group, bool *most)
{
    int t = 64;
    *most = false;
    for (int i = 0; i < s.ns; ++i) {
        int nb = s.st[i].nb;
        if (i + 1 == s.ns)
            nb = (nb + group - 1) / group * group;
        const long long total = (long long)nb * tiles;
        const int un = lds_units(s.st[i].r, false), um = lds_units(s.st[i].r, true);
        if ((total + um - 1) / um > 1024)
            return 0;
        *most |= (total + un - 1) / un > 1024;
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
        // 3072 samples a workgroup (24 KB of LDS, six workgroups a CU; 4096
        // and 2048 were up to 30 % and 10 % slower: 1200 points 158 and 113 us
        // against 115, 60 points 112 and 116 against 110, each 2^25 samples),
        // fewer where the batch would leave CUs without work; where there is
        // one stage (3 or 5 points) one butterfly a thread
        int segs = p->a.ns == 1 ? 256 : std::max(1, 3072 / (int)n);
        while (p->a.ns > 1 && segs > 1 && (batch + segs - 1) / segs < 2 * (uint64_t)cus)
            segs = (segs + 1) / 2;
        p->segs = segs;
        p->threads_a = p->a.ns == 1 ? segs : lds_threads(p->a, segs, 1, &p->most_a);
        if (p->threads_a) {
            p->passes = 1;
            return true;
        }
    }
    // two passes: of every n1 n2 whose tiles fit, the one that the measured
    // rates of the two passes (2^26 samples, relative to a column pass of
    // 240 x 200 at 5 TB/s) make cheapest
    double best = 1e30;
    for (uint64_t n1 = 26; n1 <= n / 2 && n1 <= 16384; ++n1) {
        if (n % n1 || n / n1 > 16384)
            continue;
        const uint64_t n2 = n / n1;
        LdsSched a, b;
        bool most;
        if (!lds_schedule((int)n2, &b))
            continue;
        const int lr = widest([&](int l) {
            return lds_threads(b, 1 << l, 1, &most) ? rows_lds(b, l) : SIZE_MAX;
        });
        if (lr < 0 || !lds_schedule((int)n1, &a, 1 << lr) || a.ns < 2)
            continue;
        const int lc = widest([&](int l) {
            return lds_threads(a, 1 << l, 1 << lr, &most) ? columns_lds(a, l) : SIZE_MAX;
        });
        if (lc < 0)
            continue;
        // [log2 width][two workgroups a CU]: whole 128-byte lines at 16
        static const double column[5][2] = {{4, 4}, {2.7, 2.7}, {2, 1.65}, {1.5, 1.45}, {1.6, 1}};
        static const double row[5][2] = {{3, 3}, {1.85, 1.85}, {1.6, 1.25}, {1.2, 1.2}, {1.25, 0.9}};
        const double score =
            column[lc][columns_lds(a, lc) <= (size_t)kLdsBytes / 2] *
                (a.st[a.ns - 1].nb % (1 << lr) ? 1.25 : 1) * (n2 % 16 ? 1.08 : 1) +
            row[lr][rows_lds(b, lr) <= (size_t)kLdsBytes / 2] * (n1 % 16 ? 1.15 : 1) +
            0.03 * (a.ns + b.ns);
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
    p->threads_a = lds_threads(p->a, 1 << p->lc, 1 << p->lr, &p->most_a);
    p->threads_b = lds_threads(p->b, 1 << p->lr, 1, &p->most_b);
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

template <int D, bool Most>
hipError_t launch_segments(const StagesPlan &p, const c32 *in, c32 *out, const c32 *tw,
                           uint64_t batch, uint64_t hop, const float *window, hipStream_t s)
{
    // the lanes' offsets within a workgroup's segments are 32-bit byte counts
    const int segs = hop < (1ull << 28) / (unsigned)p.segs ? p.segs : 1;
    const size_t lds = (size_t)segs * p.a.n * sizeof(c32);
    const hipError_t e = allow_lds(stages_segments_kernel<D, Most>, lds);
    if (e != hipSuccess)
        return e;
    const uint64_t groups = (batch + segs - 1) / segs;
    hipLaunchKernelGGL((stages_segments_kernel<D, Most>), dim3((unsigned)groups),
                       dim3(p.threads_a), (unsigned)lds, s, in, out, tw, p.a, segs, batch, hop, window);
    return hipGetLastError();
}

unsigned xcd_grid(uint64_t tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

template <int D, bool Most>
hipError_t launch_columns(const StagesPlan &p, const c32 *in, c32 *y, const c32 *tw,
                          const c32 *tl, const c32 *th, int sh, uint64_t batch, uint64_t hop,
                          const float *window, hipStream_t s)
{
    const size_t lds = columns_lds(p.a, p.lc);
    const hipError_t e = allow_lds(stages_columns_kernel<D, Most>, lds);
    if (e != hipSuccess)
        return e;
    const unsigned blocks = (unsigned)((p.b.n + (1 << p.lc) - 1) >> p.lc);
    hipLaunchKernelGGL((stages_columns_kernel<D, Most>), dim3(xcd_grid(batch * blocks)),
                       dim3(p.threads_a), (unsigned)lds, s, in, y, tw, tl, th, sh, p.a, p.b.n,
                       p.lc, p.lr, blocks, batch * blocks, p.y_samples, hop, window);
    return hipGetLastError();
}

template <int D, bool Most>
hipError_t launch_rows(const StagesPlan &p, const c32 *y, c32 *out, const c32 *tw,
                       uint64_t batch, hipStream_t s)
{
    const size_t lds = rows_lds(p.b, p.lr);
    const hipError_t e = allow_lds(stages_rows_kernel<D, Most>, lds);
    if (e != hipSuccess)
        return e;
    const unsigned blocks = (unsigned)((p.a.n + (1 << p.lr) - 1) >> p.lr);
    hipLaunchKernelGGL((stages_rows_kernel<D, Most>), dim3(xcd_grid(batch * blocks)),
                       dim3(p.threads_b), (unsigned)lds, s, y, out, tw, p.b, p.a.n, p.lr, blocks,
                       batch * blocks, p.y_samples);
    return hipGetLastError();
}

}  // namespace

hipError_t stages_one_pass(const StagesPlan &p, int dir, const void *in, void *out,
                           const void *tw, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s)
{
    const auto f = dir < 0 ? (p.most_a ? launch_segments<-1, true> : launch_segments<-1, false>)
                           : (p.most_a ? launch_segments<1, true> : launch_segments<1, false>);
    return f(p, (const c32 *)in, (c32 *)out, (const c32 *)tw, batch, hop, window, s);
}

hipError_t stages_two_pass(const StagesPlan &p, int dir, const void *in, void *out, void *y,
                           const void *tw_a, const void *tw_b, const void *tl, const void *th,
                           int sh, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s)
{
    const auto fc = dir < 0 ? (p.most_a ? launch_columns<-1, true> : launch_columns<-1, false>)
                            : (p.most_a ? launch_columns<1, true> : launch_columns<1, false>);
    const auto fr = dir < 0 ? (p.most_b ? launch_rows<-1, true> : launch_rows<-1, false>)
                            : (p.most_b ? launch_rows<1, true> : launch_rows<1, false>);
    const hipError_t e = fc(p, (const c32 *)in, (c32 *)y, (const c32 *)tw_a, (const c32 *)tl,
                            (const c32 *)th, sh, batch, hop, window, s);
    return e == hipSuccess ? fr(p, (const c32 *)y, (c32 *)out, (const c32 *)tw_b, batch, s) : e;
}

}  // namespace fftseg
