// Real-input segments of length N = 2M whose M has no compiled one-pass
// kernel, through the run-time radix schedules of the M-point transform, the
// even/odd split fused into them.  With z[m] = x[2m] + i x[2m+1] and
// Z = DFT_M(z):
//   forward  X[k] = E + T, X[M - k] = conj(E - T) with A = Z[k mod M],
//            B = conj Z[(M - k) mod M], E = (A + B)/2, T = -i W_N^k (A - B)/2
//   inverse  Z[k] = S + T, Z[M - k] = conj(S - T) with A = X[k],
//            B = conj X[M - k], S = A + B, T = i W_N^{-k} (A - B); the
//            imaginary parts of X[0] and X[M] are dropped, and the
//            unnormalised inverse M-point transform of Z is x[2m] + i x[2m+1].
// One pass: the split walks the pairs of the tile in LDS, after the last
// stage (forward) or before the first (inverse).  Two passes: Z[k1 + n1 k2]
// and its partner sit in rows k1 and n1 - k1, so a row tile holds rows of
// both kinds (forward); Z[i n2 + j] and its partner sit in columns j and
// n2 - j, so a column tile does (inverse); W_N^k there is the product of a
// factor of the pair of rows (columns) and one of the place in them, in FP64 and
// rounded once.  HBM sees 8 B per real sample in
// one pass and 16 in two; a split pass of its own was 8 more.
// (products fuse into additions within an expression, as the source has them, and not
// across: a segment's bits then do not depend on the copy of an unrolled loop, or
// on the form of the kernel, that a butterfly falls to)
#pragma clang fp contract(on)
#include "runtime.hpp"
#include "stages_device.hpp"

#include <algorithm>

namespace fftseg {
namespace {

using namespace stages;

__device__ __forceinline__ c32 conj(c32 a) { return {a.x, -a.y}; }

// the bins k and M - k of Z's elements k and M - k
__device__ __forceinline__ void split_forward(c32 a, c32 z, c32 w, c32 &lo, c32 &hi)
{
    const c32 e = {0.5f * (a.x + z.x), 0.5f * (a.y - z.y)};
    const c32 d = {0.5f * (a.x - z.x), 0.5f * (a.y + z.y)};
    const c32 t = cmul(mul_di<-1>(d), w);
    lo = cadd(e, t);
    hi = conj(csub(e, t));
}
// Z's elements k and M - k of the bins k and M - k
__device__ __forceinline__ void split_inverse(c32 a, c32 z, c32 w, c32 &lo, c32 &hi)
{
    const c32 b = conj(z);
    const c32 s = cadd(a, b);
    const c32 t = mul_di<1>(cmulc(csub(a, b), w));
    lo = cadd(s, t);
    hi = conj(csub(s, t));
}

// The split walks `total` pairs of the tile, kAhead per thread and turn: all
// of a turn's loads are issued before the first is used.  load(e, i) reads
// pair e into slot i of the caller's registers (or notes that e is none),
// use(i) works on it.
constexpr int kAhead = 4;
template <class Load, class Use>
__device__ __forceinline__ void walk_pairs(int total, Load &&load, Use &&use)
{
    for (int e0 = threadIdx.x; e0 < total; e0 += kAhead * (int)blockDim.x) {
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            load(e0 + i * (int)blockDim.x, i);
#pragma unroll
        for (int i = 0; i < kAhead; ++i)
            use(i);
    }
}

template <int D>
struct RealSegmentIo : SegmentIo {
    static constexpr bool kFirstLds = D > 0, kLastLds = D < 0;
};

// mp: reciprocal of M/2 + 1, the pairs of a segment
template <int D, int F>
__global__ void STAGES_KERNEL(F, false)
    stages_real_segments_kernel(const c32 *in, c32 *out, const c32 *__restrict__ tw,
                                const c32 *__restrict__ hw, LdsSched s, int segs, uint32_t mp,
                                uint64_t batch)
{
    const uint64_t seg = (uint64_t)blockIdx.x * (unsigned)segs;
    const int have = (int)(batch - seg < (uint64_t)segs ? batch - seg : (uint64_t)segs);
    const int m = s.n, pairs = m / 2 + 1;
    RealSegmentIo<D> io;
    io.x = in + seg * (unsigned)(D < 0 ? m : m + 1);
    io.y = out + seg * (unsigned)(D < 0 ? m + 1 : m);
    io.window = nullptr;
    io.hop = (uint64_t)m;
    io.n = m;
    io.segs = have;
    const int total = have * pairs;
    c32 va[kAhead], vz[kAhead], vw[kAhead];
    int vc[kAhead], vk[kAhead];  // (segment, k); k < 0: none
    auto pair = [&](int e, int i) {
        vc[i] = fast_div(e, mp);
        vk[i] = e < total ? e - vc[i] * pairs : -1;
        if (vk[i] >= 0)
            vw[i] = hw[vk[i]];
    };
    if constexpr (D > 0) {
        walk_pairs(
            total,
            [&](int e, int i) {
                pair(e, i);
                if (vk[i] >= 0) {
                    const c32 *x = io.x + vc[i] * (m + 1);
                    va[i] = x[vk[i]];
                    vz[i] = x[m - vk[i]];
                }
            },
            [&](int i) {
                const int k = vk[i];
                if (k < 0)
                    return;
                if (k == 0)
                    va[i].y = vz[i].y = 0.f;
                c32 lo, hi;
                split_inverse(va[i], vz[i], vw[i], lo, hi);
                c32 *p = stage_lds + vc[i] * m;
                p[k] = lo;
                if (k > 0 && 2 * k < m)
                    p[m - k] = hi;
            });
        __syncthreads();
    }
    run_stages<D, F>(io, s, stage_lds, tw);
    if constexpr (D < 0)
        walk_pairs(total, pair, [&](int i) {
            const int k = vk[i];
            if (k < 0)
                return;
            const c32 *p = stage_lds + vc[i] * m;
            c32 lo, hi;
            split_forward(p[k], p[k == 0 ? 0 : m - k], vw[i], lo, hi);
            c32 *y = io.y + vc[i] * (m + 1);
            y[k] = lo;
            if (2 * k < m)
                y[m - k] = hi;
        });
}

// Columns of a forward transform: the complex pass with Y's rows in pairs.
template <int F>
__global__ void STAGES_KERNEL(F, true)
    stages_real_columns_kernel(const c32 *in, c32 *ybuf, const c32 *__restrict__ tw,
                               const c64 *__restrict__ tl, const c64 *__restrict__ th, int sh,
                               LdsSched s, int n2, int lc, int lr, unsigned blocks,
                               uint64_t tiles, uint64_t ysamples)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const int first = (int)(t - seg * blocks) << lc;
    ColumnIo<true, false> io{in + seg * ((uint64_t)s.n * (unsigned)n2), ybuf + seg * ysamples,
                             nullptr, tl, th, nullptr, sh, n2, first, lc, lr, (unsigned)s.n};
    io.ws = column_factors(io, s);
    run_stages<-1, F>(io, s, stage_lds, tw);
}

// Rows of a forward transform and the split: bin k = k1 + n1 k2 of row k1
// pairs with bin n1 - k1 + n1 (n2 - 1 - k2) of row n1 - k1; row 0 and (n1
// even) row n1/2 pair within themselves.
template <int F>
__global__ void STAGES_KERNEL(F, false)
    stages_real_rows_kernel(const c32 *ybuf, c32 *out, const c32 *__restrict__ tw,
                            const c64 *__restrict__ w1, const c64 *__restrict__ w2, LdsSched s,
                            int n1, int lr, unsigned blocks, uint64_t tiles, uint64_t ysamples)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const unsigned blk = (unsigned)(t - seg * blocks);
    const int n2 = s.n, m = n1 * n2, half = 1 << (lr - 1);
    const RowIo<true> io{ybuf + seg * ysamples + ((uint64_t)blk << lr) * (unsigned)n2,
                         out + seg * (uint64_t)(m + 1), n1, (int)blk * half, lr, n1};
    run_stages<-1, F>(io, s, stage_lds, tw);
    c64 wb[kAhead];
    int vk[kAhead], va[kAhead], vz[kAhead];  // k (< 0: none), slots of the pair
    // (a workgroup is whole waves, so a thread stays with one row pair)
    const int c = (int)threadIdx.x & (half - 1), k1 = io.first + c;
    const bool zero = k1 == 0, self = zero || 2 * k1 == n1, row = 2 * k1 <= n1;
    const c64 wa = row ? w1[k1] : c64{0., 0.};
    walk_pairs(
        n2 << (lr - 1),
        [&](int e, int i) {
            const int k2 = e >> (lr - 1);
            const int p2 = zero ? (k2 == 0 ? 0 : n2 - k2) : n2 - 1 - k2;
            const bool none = k2 >= n2 || !row ||
                              (self && k2 != 0 && p2 < k2);  // (the partner's)
            vk[i] = none ? -1 : k1 + n1 * k2;
            if (!none) {
                wb[i] = w2[k2];
                va[i] = io.slot(k2, c);
                vz[i] = io.slot(p2, self ? c : half + c);
            }
        },
        [&](int i) {
            const int k = vk[i];
            if (k < 0)
                return;
            c32 lo, hi;
            split_forward(stage_lds[va[i]], stage_lds[vz[i]], rounded(cmul(wa, wb[i])), lo, hi);
            io.y[k] = lo;
            if (2 * k != m)
                io.y[m - k] = hi;
        });
}

// Columns of an inverse transform and the split before them: bin i n2 + j of
// column j pairs with bin (n1 - 1 - i) n2 + n2 - j of column n2 - j; column
// 0 and (n2 even) column n2/2 pair within themselves.
template <int F>
__global__ void STAGES_KERNEL(F, true)
    stages_real_inverse_columns_kernel(const c32 *in, c32 *ybuf, const c32 *__restrict__ tw,
                                       const c64 *__restrict__ tl, const c64 *__restrict__ th,
                                       int sh, const c64 *__restrict__ w1,
                                       const c64 *__restrict__ w2, LdsSched s, int n2, int lc,
                                       int lr, unsigned blocks, uint64_t tiles,
                                       uint64_t ysamples)
{
    const uint64_t t = xcd_tile();
    if (t >= tiles)
        return;
    const uint64_t seg = t / blocks;
    const int n1 = s.n, m = n1 * n2, half = 1 << (lc - 1);
    const int first = (int)(t - seg * blocks) * half;
    ColumnIo<false, true> io{in + seg * (uint64_t)(m + 1), ybuf + seg * ysamples, nullptr, tl, th,
                             nullptr, sh, n2, first, lc, lr, (unsigned)n1};
    io.ws = column_factors(io, s);
    c32 va[kAhead], vz[kAhead];
    c64 wb[kAhead];
    int vk[kAhead], sa[kAhead], sz[kAhead];  // k (< 0: none), slots of the pair
    // (a workgroup is whole waves, so a thread stays with one column pair)
    const int c = (int)threadIdx.x & (half - 1), j = first + c;
    const bool zero = j == 0, self = zero || 2 * j == n2, column = 2 * j <= n2;
    const c64 wa = column ? w1[j] : c64{0., 0.};
    walk_pairs(
        n1 << (lc - 1),
        [&](int e, int q) {
            const int i = e >> (lc - 1);
            const int pi = zero ? (i == 0 ? 0 : n1 - i) : n1 - 1 - i;
            const bool none = i >= n1 || !column ||
                              (self && i != 0 && pi < i);  // (the partner's)
            const int k = i * n2 + j;
            vk[q] = none ? -1 : k;
            if (!none) {
                va[q] = io.x[k];
                vz[q] = io.x[m - k];
                wb[q] = w2[i];
                sa[q] = io.slot(i, c);
                sz[q] = io.slot(pi, self ? c : half + c);
            }
        },
        [&](int q) {
            const int k = vk[q];
            if (k < 0)
                return;
            if (k == 0)
                va[q].y = vz[q].y = 0.f;
            c32 lo, hi;
            split_inverse(va[q], vz[q], rounded(cmul(wa, wb[q])), lo, hi);
            stage_lds[sa[q]] = lo;
            if (k != 0 && 2 * k != m)
                stage_lds[sz[q]] = hi;
        });
    __syncthreads();
    run_stages<1, F>(io, s, stage_lds, tw);
}

template <int D, int F>
hipError_t launch_segments(const StagesPlan &p, const c32 *in, c32 *out, const c32 *tw,
                           const c32 *hw, uint64_t batch, hipStream_t s)
{
    const size_t lds = (size_t)p.segs * p.a.n * sizeof(c32);
    const hipError_t e = allow_lds(stages_real_segments_kernel<D, F>, lds);
    if (e != hipSuccess)
        return e;
    // (a launch holds fewer than 2^32 threads: more segments of 6 samples fit the memory)
    const uint64_t most = ((1ull << 31) / (unsigned)p.threads_a) * (unsigned)p.segs;
    const uint64_t ir = (uint64_t)p.a.n + (D > 0), orow = (uint64_t)p.a.n + (D < 0);
    for (uint64_t s0 = 0; s0 < batch; s0 += most) {
        const uint64_t sb = std::min(most, batch - s0);
        hipLaunchKernelGGL((stages_real_segments_kernel<D, F>),
                           dim3((unsigned)((sb + p.segs - 1) / p.segs)), dim3(p.threads_a),
                           (unsigned)lds, s, in + s0 * ir, out + s0 * orow, tw, hw, p.a, p.segs,
                           reciprocal(p.a.n / 2 + 1), sb);
    }
    return hipGetLastError();
}

template <int F>
hipError_t launch_columns(const StagesPlan &p, const c32 *in, c32 *y, const c32 *tw,
                          const c64 *tl, const c64 *th, int sh, const c64 *w1, const c64 *w2,
                          uint64_t batch, hipStream_t s)
{
    const size_t lds = columns_lds(p.a, p.lc);
    const dim3 grid(xcd_grid(batch * p.blocks_a)), threads(p.threads_a);
    hipError_t e = p.real < 0 ? allow_lds(stages_real_columns_kernel<F>, lds)
                              : allow_lds(stages_real_inverse_columns_kernel<F>, lds);
    if (e != hipSuccess)
        return e;
    if (p.real < 0)
        hipLaunchKernelGGL(stages_real_columns_kernel<F>, grid, threads, (unsigned)lds, s, in,
                           y, tw, tl, th, sh, p.a, p.b.n, p.lc, p.lr, p.blocks_a,
                           batch * p.blocks_a, p.y_samples);
    else
        hipLaunchKernelGGL(stages_real_inverse_columns_kernel<F>, grid, threads, (unsigned)lds,
                           s, in, y, tw, tl, th, sh, w1, w2, p.a, p.b.n, p.lc, p.lr, p.blocks_a,
                           batch * p.blocks_a, p.y_samples);
    return hipGetLastError();
}

template <int F>
hipError_t launch_rows(const StagesPlan &p, const c32 *y, c32 *out, const c32 *tw, const c64 *w1,
                       const c64 *w2, uint64_t batch, hipStream_t s)
{
    const size_t lds = rows_lds(p.b, p.lr);
    const hipError_t e = allow_lds(stages_real_rows_kernel<F>, lds);
    if (e != hipSuccess)
        return e;
    hipLaunchKernelGGL(stages_real_rows_kernel<F>, dim3(xcd_grid(batch * p.blocks_b)),
                       dim3(p.threads_b), (unsigned)lds, s, y, out, tw, w1, w2, p.b, p.a.n, p.lr,
                       p.blocks_b, batch * p.blocks_b, p.y_samples);
    return hipGetLastError();
}

}  // namespace

hipError_t stages_real_one_pass(const StagesPlan &p, const void *in, void *out, const void *tw,
                                const void *hw, uint64_t batch, hipStream_t s)
{
    static constexpr auto f = {launch_segments<-1, kNarrow>, launch_segments<-1, kMost>,
                               launch_segments<-1, kWide>,   launch_segments<1, kNarrow>,
                               launch_segments<1, kMost>,    launch_segments<1, kWide>};
    return f.begin()[p.form_a + (p.real < 0 ? 0 : 3)](p, (const c32 *)in, (c32 *)out,
                                                      (const c32 *)tw, (const c32 *)hw, batch, s);
}

hipError_t stages_real_two_pass(const StagesPlan &p, const void *in, void *out, void *y,
                                const void *tw_a, const void *tw_b, const void *tl,
                                const void *th, int sh, const void *w1, const void *w2,
                                uint64_t batch, hipStream_t s)
{
    static constexpr auto fc = {launch_columns<kNarrow>, launch_columns<kMost>,
                                launch_columns<kWide>};
    static constexpr auto fr = {launch_rows<kNarrow>, launch_rows<kMost>, launch_rows<kWide>};
    const hipError_t e = fc.begin()[p.form_a](p, (const c32 *)in, (c32 *)y, (const c32 *)tw_a,
                                              (const c64 *)tl, (const c64 *)th, sh,
                                              (const c64 *)w1, (const c64 *)w2, batch, s);
    if (e != hipSuccess)
        return e;
    if (p.real > 0)
        return stages_rows(p, 1, y, out, tw_b, batch, s);
    return fr.begin()[p.form_b](p, (const c32 *)y, (c32 *)out, (const c32 *)tw_b,
                                (const c64 *)w1, (const c64 *)w2, batch, s);
}

}  // namespace fftseg
