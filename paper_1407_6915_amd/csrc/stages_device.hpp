// Device side of the run-time radix schedules: the stage engine and the
// accessors of its tiles (whole segments, columns, rows).
#pragma once

#include "stages.hpp"
#include "tile.hpp"

// (a register budget of four waves per SIMD)
#define STAGES_KERNEL(F, COLUMN)               \
    __launch_bounds__(form_threads(F, COLUMN)) \
        __attribute__((amdgpu_waves_per_eu(4, 4)))

namespace fftseg {
namespace stages {

__device__ __forceinline__ int fast_div(int x, uint32_t m)
{
    return m ? (int)__umulhi((unsigned)x, m) : x;
}

__device__ __forceinline__ c64 cmul(c64 a, c64 b)
{
    return {a.x * b.x - a.y * b.y, a.x * b.y + a.y * b.x};
}
__device__ __forceinline__ c32 rounded(c64 a) { return {(float)a.x, (float)a.y}; }

// v[r] times first step^r, r < R: a stage's twiddles W^{r k} (from r = 1 on) or
// the factors W^{m (b + r nb)} between two passes.  The powers run on in FP64, where
// a step costs what one in float32 does, and each factor is rounded once;
// products of two rounded factors in float32 left 2^24 points 2.03e-7 off where
// this is 1.86e-7 (twiddles from pairs of table entries 1.99e-7), 48000 1.42e-7
// and 1.40e-7.  One entry to read or keep in LDS in place of up to R also leaves the
// kernels fewer registers: 2^24 samples of 48000 points 111 -> 104 us, of 2^24
// 156 -> 152; one pass of 15625 points, whose stages wait for the chain, 80.7 ->
// 82.8 (once-rounded products of FP64 pairs 84.7, an entry each 83.9).
template <int R, int D>
__device__ __forceinline__ void twiddle_powers(c32 *v, c64 first, c64 step)
{
    if constexpr (D > 0) {
        first.y = -first.y;
        step.y = -step.y;
    }
    // (two chains: half the dependent products)
    c64 even = first, odd = cmul(first, step);
    const c64 two = cmul(step, step);
#pragma unroll
    for (int r = 0; r < R; r += 2) {
        v[r] = cmul(v[r], rounded(even));
        if (r + 1 < R)
            v[r + 1] = cmul(v[r + 1], rounded(odd));
        if (r + 2 < R)
            even = cmul(even, two);
        if (r + 3 < R)
            odd = cmul(odd, two);
    }
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
    __device__ __forceinline__ c64 load_wide(unsigned lane, int uniform) const
    {
        return __builtin_bit_cast(c64,
                                  __builtin_amdgcn_raw_buffer_load_b128(r, lane, 8 * uniform, 0));
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
// first stage's loads (gl) and the last stage's stores (gs), unless the
// tile is filled before (kFirstLds) or read after (kLastLds) through LDS.
template <int R, int D, int F, class Io>
__device__ __forceinline__ void lds_stage(const Io &io, const LdsStage &st, bool gl, bool gs,
                                          c32 *lds, const Buffer &tw)
{
    constexpr int U = lds_units(R, F);
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
                if constexpr (lds_powers(R)) {
                    const c64 w = tw.load_wide(16u * k, st.tw);
                    twiddle_powers<R - 1, D>(v[u] + 1, w, w);
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

template <int D, int F, class Io>
__device__ __forceinline__ void run_stages(const Io &io, const LdsSched &s, c32 *lds,
                                           const c32 *table)
{
    const Buffer tw(table);
    for (int i = 0; i < s.ns; ++i) {
        const LdsStage &st = s.st[i];
        const bool gl = i == 0 && !Io::kFirstLds, gs = i + 1 == s.ns && !Io::kLastLds;
        switch (st.r) {
        case 2: lds_stage<2, D, F>(io, st, gl, gs, lds, tw); break;
        case 3: lds_stage<3, D, F>(io, st, gl, gs, lds, tw); break;
        case 4: lds_stage<4, D, F>(io, st, gl, gs, lds, tw); break;
        case 5: lds_stage<5, D, F>(io, st, gl, gs, lds, tw); break;
        case 6: lds_stage<6, D, F>(io, st, gl, gs, lds, tw); break;
        case 8: lds_stage<8, D, F>(io, st, gl, gs, lds, tw); break;
        case 9: lds_stage<9, D, F>(io, st, gl, gs, lds, tw); break;
        case 10: lds_stage<10, D, F>(io, st, gl, gs, lds, tw); break;
        case 12: lds_stage<12, D, F>(io, st, gl, gs, lds, tw); break;
        case 15: lds_stage<15, D, F>(io, st, gl, gs, lds, tw); break;
        case 16: lds_stage<16, D, F>(io, st, gl, gs, lds, tw); break;
        default:
            if constexpr (F == kWide) {
                switch (st.r) {
                case 18: lds_stage<18, D, F>(io, st, gl, gs, lds, tw); break;
                case 20: lds_stage<20, D, F>(io, st, gl, gs, lds, tw); break;
                case 24: lds_stage<24, D, F>(io, st, gl, gs, lds, tw); break;
                case 27: lds_stage<27, D, F>(io, st, gl, gs, lds, tw); break;
                case 30: lds_stage<30, D, F>(io, st, gl, gs, lds, tw); break;
                case 32: lds_stage<32, D, F>(io, st, gl, gs, lds, tw); break;
                default: lds_stage<25, D, F>(io, st, gl, gs, lds, tw); break;
                }
            } else {
                lds_stage<25, D, F>(io, st, gl, gs, lds, tw);
            }
            break;
        }
    }
}

// W^m from its two-level table
__device__ __forceinline__ c64 two_level_root(const c64 *tl, const c64 *th, int sh, unsigned m)
{
    return cmul(th[m >> sh], tl[m & ((1u << sh) - 1u)]);
}

// Whole segments: transform c is segment c of the tile, its elements in
// consecutive slots; butterflies of a segment on consecutive lanes, so the
// first stage loads and the last stage stores runs of nb samples.
struct SegmentIo {
    static constexpr bool kFirstLds = false, kLastLds = false;
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

// Four-step column pass: transform c is column first + c of the segment
// (elements n2 samples apart), columns on consecutive lanes, slots of one
// element row 2^lc + 1 apart.  The last stage instead puts 2^lr consecutive
// outputs k1 on consecutive lanes, then the columns: Y keeps the rows of one
// row tile together,
//     Y[(k1 >> lr)][n2][k1 mod 2^lr],
// so that a wave stores one run here and the row pass loads its tile as one
// W_N^{n2 k1} of output k1 = b + r nb is W_N^{n2 b}, looked up once per
// butterfly, times the r-th power of W_N^{n2 nb}, looked up once per column
// into LDS (twiddle_powers): a lookup is two gathers from tables of a few
// thousand entries, and one per output held the pass to half its rate (20000
// points: 606 us per 2^26 samples).
// PairRows (real segments, forward): a row tile holds rows k1 and n1 - k1,
// the first half of its slots and the second, so Y groups the rows so.
// PairColumns (real segments, inverse): the tile holds columns n2' and
// n2 - n2' in the same way, and LDS is filled before the first stage.
template <bool PairRows, bool PairColumns>
struct ColumnIo {
    static constexpr bool kFirstLds = PairColumns, kLastLds = false;
    const c32 *x;
    c32 *y;
    const float *window;
    const c64 *__restrict__ tl;
    const c64 *__restrict__ th;
    const c64 *ws;  // LDS: W_N^{n2 nb} of the columns, nb the last stage's
    int sh, n2, first, lc, lr;
    unsigned n1;
    __device__ __forceinline__ c64 root(unsigned m) const
    {
        return two_level_root(tl, th, sh, m);
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
        return b < st.nb && has(c);
    }
    // column of slot c, and whether the slot holds one
    __device__ __forceinline__ int column(int c) const
    {
        if constexpr (PairColumns)
            if (const int half = 1 << (lc - 1); c >= half)
                return n2 - (first + c - half);
        return first + c;
    }
    __device__ __forceinline__ bool has(int c) const
    {
        if constexpr (!PairColumns)
            return first + c < n2;
        const int half = 1 << (lc - 1), p = first + c - half;
        return c < half ? 2 * (first + c) <= n2 : p > 0 && 2 * p < n2;
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
        const unsigned col = (unsigned)column(c);
        const Buffer yb(y);
        if (!PairRows && (nb & ((1 << lr) - 1)) == 0) {
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
        unsigned at = k1;
        if constexpr (PairRows) {
            const unsigned half = 1u << (lr - 1), high = 2 * k1 > n1 ? 1u : 0u;
            const unsigned p = high ? n1 - k1 : k1;
            at = ((p >> (lr - 1)) << lr) | (high ? half : 0u) | (p & (half - 1u));
        }
        return (((at >> lr) * (unsigned)n2 + col) << lr) | (at & ((1u << lr) - 1u));
    }
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *v, int b, int c, int) const
    {
        twiddle_powers<R, D>(v, root((unsigned)column(c) * (unsigned)b), ws[c]);
    }
};

// Four-step row pass: transform c is row first + c of Y (one contiguous tile,
// the rows on consecutive lanes), stored transposed as X[k1 + n1 k2].
// Row k2 of the n2 that a three-pass row consists of starts k2 n1 samples
// into the output (y), with outputs n1 n2 apart (`stride`; n1 in two passes).
// Pair: the tile of rows first + c and n1 - (first + c) (see ColumnIo), left
// in LDS by the last stage.
template <bool Pair>
struct RowIo {
    static constexpr bool kFirstLds = false, kLastLds = Pair;
    const c32 *x;  // the tile
    c32 *y;        // segment output
    int n1, first, lr, stride;
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *, int, int, int) const
    {
    }
    __device__ __forceinline__ bool map(const LdsStage &st, bool, int g, int &b, int &c) const
    {
        c = g & ((1 << lr) - 1);
        b = g >> lr;
        return b < st.nb && has(c);
    }
    __device__ __forceinline__ bool has(int c) const
    {
        if constexpr (!Pair)
            return first + c < n1;
        const int half = 1 << (lr - 1), p = first + c - half;
        return c < half ? 2 * (first + c) <= n1 : p > 0 && 2 * p < n1;
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
        const unsigned at = 8u * (unsigned)(b * stride + first + c);
        const int d = nb * stride;
#pragma unroll
        for (int r = 0; r < R; ++r)
            yb.store(at, r * d, v[r]);
    }
};

// Middle pass of a three-pass transform n = n1 n2 n3: the row k1 of Y is
// transformed as n2 x n3, its n2-point columns here.  Y keeps 2^lr rows
// together, Y[(k1 >> lr)][i n3 + j][k1 mod 2^lr], so the tile of one column j
// of those rows moves whole runs of 2^lr samples, and goes back in place.
struct MiddleIo {
    static constexpr bool kFirstLds = false, kLastLds = false;
    c32 *y;  // row block, column j
    const c64 *__restrict__ tl;
    const c64 *__restrict__ th;
    c64 ws;                   // W_{n2 n3}^{j nb}, nb the last stage's
    int sh, n3, j, rows, lr;  // rows the block holds
    __device__ __forceinline__ c64 root(unsigned m) const
    {
        return two_level_root(tl, th, sh, m);
    }
    __device__ __forceinline__ bool map(const LdsStage &st, bool, int g, int &b, int &c) const
    {
        c = g & ((1 << lr) - 1);
        b = g >> lr;
        return b < st.nb && c < rows;
    }
    __device__ __forceinline__ int step() const { return 1 << lr; }
    __device__ __forceinline__ int slot(int i, int c) const { return (i << lr) + c; }
    template <int R>
    __device__ __forceinline__ void load(c32 *v, int b, int c, int nb) const
    {
        const Buffer yb(y);
        const unsigned at = 8u * (unsigned)(((b * n3) << lr) + c);
#pragma unroll
        for (int r = 0; r < R; ++r)
            v[r] = yb.load(at, (r * nb * n3) << lr);
    }
    template <int R>
    __device__ __forceinline__ void store(const c32 *v, int b, int c, int nb) const
    {
        const Buffer yb(y);
        const unsigned at = 8u * (unsigned)(((b * n3) << lr) + c);
#pragma unroll
        for (int r = 0; r < R; ++r)
            yb.store(at, (r * nb * n3) << lr, v[r]);
    }
    template <int R, int D>
    __device__ __forceinline__ void finish(c32 *v, int b, int, int) const
    {
        twiddle_powers<R, D>(v, root((unsigned)j * (unsigned)b), ws);
    }
};

// Tile w of a grid of 8 * per workgroups, dealt so that each XCD (workgroup
// mod 8) takes consecutive tiles: neighbours share cache lines where the
// lengths are no multiple of 16.
__device__ __forceinline__ uint64_t xcd_tile()
{
    return (uint64_t)(blockIdx.x & 7u) * (gridDim.x >> 3) + (blockIdx.x >> 3);
}

extern __shared__ __attribute__((aligned(16))) c32 stage_lds[];

// Factors W_N^{n2 nb} of a column tile into LDS behind the tile (read after
// the barriers of the first exchange; a workgroup has at least 64 threads)
template <class Io>
__device__ __forceinline__ c64 *column_factors(const Io &io, const LdsSched &s)
{
    c64 *ws = reinterpret_cast<c64 *>(stage_lds + column_slots(s.n, io.lc));
    const int c = threadIdx.x;
    if (c < 1 << io.lc && io.has(c))
        ws[c] = io.root((unsigned)io.column(c) * (unsigned)s.st[s.ns - 1].nb);
    return ws;
}

}  // namespace stages
}  // namespace fftseg
