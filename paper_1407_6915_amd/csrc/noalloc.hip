// fft_exec_segments_noalloc: the batched transform without a plan and
// without any device allocation.
//
// For callers that cannot allocate device memory (code under stream
// capture, serving loops, harnesses that forbid it).  Everything the
// kernels need beyond the caller's in/out buffers -- the twiddle tables and
// the Y buffer between the two passes of long segments -- lives in one
// file-scope device array of fixed size.  Each call recomputes the tables on
// the device (a small kernel, so that a captured call carries them), then
// runs the same kernels fft_exec_segments runs, long segments in
// sub-batches whose Y fits the array.  The array is this GPU's, shared by
// every call on it: calls that overlap in time on one GPU race.
#include "fftseg.h"
#include "runtime.hpp"

#include <cmath>
#include <mutex>

namespace fftseg {
namespace {

// tables: W_N or a schedule's (one pass); W_N1, W_N2 or the schedules', and the
// two-level tables (two and three passes)
constexpr uint64_t kTableSamples = 1ull << 15;
// Y: 2^24 samples plus two lines: one sub-batch of a two-pass length with
// compiled tiles (up to 2^22 points, so at least 4 segments), or of a
// run-time schedule (lengths up to 2^23, at least one segment: its Y is less
// than twice the segment)
constexpr uint64_t kYSamples = (1ull << 24) + 2 * kLineSamples;
constexpr uint64_t kScratchBytes = (kTableSamples + kYSamples) * sizeof(c32);

static __device__ __align__(256) unsigned char scratch[kScratchBytes];

// the array's device address, per device (taken once, with that device
// current; the host-side name `scratch` is not a device address)
constexpr int kMaxDevices = 64;
std::mutex g_mu;
void *g_ptr[kMaxDevices] = {};

int scratch_ptr(int dev, void **out)
{
    if (dev < 0 || dev >= kMaxDevices)
        return set_error(FFT_ERR_INVALID_ARG, "device %d outside [0, %d)", dev, kMaxDevices);
    std::lock_guard<std::mutex> lk(g_mu);
    if (!g_ptr[dev]) {
        void *p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || !p) {
            (void)hipGetLastError();
            return set_error(FFT_ERR_HIP, "hipGetSymbolAddress(scratch): %s",
                             hipGetErrorString(e));
        }
        g_ptr[dev] = p;
    }
    *out = g_ptr[dev];
    return FFT_OK;
}

// exp(-2 pi i m / n), m < n <= 2^24, in FP64, the angle folded to the first
// octant in exact integer arithmetic
__device__ c64 device_root(uint32_t m, uint32_t n)
{
    const uint32_t m8 = m * 8u;
    const uint32_t o = m8 / n, r = m8 - o * n;
    const uint32_t j = (o + 1) / 2;
    const double quarter_pi = 0.78539816339744830961566084581987572;
    const double x = ((double)((int)o - 2 * (int)j) + (double)r / (double)n) * quarter_pi;
    double sx, cx;
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

// Table t of a set: the entries up to end[t] of all, W_{mod[t]}^{j step[t]} of
// its entry j, or, with rows of l[t] > 0 entries (the twiddles of one stage of a
// run-time schedule), W_{mod[t]}^{(1 + j / l[t]) (j mod l[t])}; from at[t] (in
// float32 entries) on, rounded once to float32 or, if bit t of `wide` is set,
// in FP64.
constexpr int kMaxTables = 4 + 3 * kMaxLdsStages;
template <int T>
struct TableSet {
    uint32_t end[T], at[T], mod[T], step[T], l[T];
    uint64_t wide;
};
static_assert(kMaxTables <= 64, "a bit of `wide` each");

// Lengths with compiled tiles have four tables at most and no rows: a set of
// that size costs their calls no more than the tables themselves (the kernel for
// any set: 4096 x 64 13.6 us against 12.1, 65536 x 1 13.1 against 12.2).
constexpr int kPlainTables = 4;

template <int T>
__global__ void __launch_bounds__(256) static_tables_kernel(c32 *tables, TableSet<T> ts,
                                                            uint32_t total)
{
    for (uint32_t i = blockIdx.x * 256 + threadIdx.x; i < total; i += gridDim.x * 256) {
        int t = 0;
        while (t + 1 < T && i >= ts.end[t])
            ++t;
        const uint32_t j = i - (t ? ts.end[t - 1] : 0u);
        uint32_t m = j * ts.step[t];
        if constexpr (T > kPlainTables)
            if (const uint32_t l = ts.l[t]; l)
                m = (1 + j / l) * (j % l);
        const c64 w = device_root(m, ts.mod[t]);
        c32 *to = tables + ts.at[t];
        if (T > kPlainTables && (ts.wide >> t & 1))
            reinterpret_cast<c64 *>(to)[j] = w;
        else
            to[j] = c32{(float)w.x, (float)w.y};
    }
}

// The tables of a call, each after the one before
struct Tables {
    TableSet<kMaxTables> ts{};
    int n = 0;
    uint32_t total = 0, room = 0;  // entries; in float32 entries
    // where the table starts, in float32 entries
    uint32_t add(uint64_t count, uint64_t mod, uint64_t step, bool wide, uint64_t l = 0)
    {
        if (wide)
            room = (room + 1) & ~1u;
        const uint32_t at = room;
        ts.end[n] = total += (uint32_t)count;
        ts.at[n] = at;
        ts.mod[n] = (uint32_t)mod;
        ts.step[n] = (uint32_t)step;
        ts.l[n] = (uint32_t)l;
        ts.wide |= (uint64_t)wide << n;
        room += (uint32_t)count * (wide ? 2 : 1);
        ++n;
        return at;
    }
    // the table of a schedule (LdsStage), from an even entry on
    uint32_t add(const LdsSched &s)
    {
        const uint32_t base = room = (room + 1) & ~1u;
        for (int i = 1; i < s.ns; ++i) {
            const uint64_t l = (uint64_t)s.st[i].l, r = (uint64_t)s.st[i].r;
            if (lds_powers(s.st[i].r)) {
                add(l, r * l, 1, true);
            } else {
                add((r - 1) * l, r * l, 0, false, l);
            }
        }
        return base;
    }
    void launch(c32 *tables, hipStream_t s)
    {
        const dim3 grid(std::min<uint32_t>((total + 255) / 256, 1024));
        for (int t = n; t < kMaxTables; ++t)
            ts.end[t] = total;
        bool plain = n <= kPlainTables && !ts.wide;
        TableSet<kPlainTables> few{};
        for (int t = 0; t < kPlainTables; ++t) {
            plain = plain && !ts.l[t];
            few.end[t] = ts.end[t];
            few.at[t] = ts.at[t];
            few.mod[t] = ts.mod[t];
            few.step[t] = ts.step[t];
        }
        if (plain)
            hipLaunchKernelGGL(static_tables_kernel<kPlainTables>, grid, dim3(256), 0, s, tables,
                               few, total);
        else
            hipLaunchKernelGGL(static_tables_kernel<kMaxTables>, grid, dim3(256), 0, s, tables,
                               ts, total);
    }
};

int noalloc_enqueue(uint64_t n, uint64_t batch, int dir, const void *in, void *out,
                    hipStream_t s)
{
    Plan p;  // host-side description only: its pointers go into `scratch`
    int st = plan_choose(&p, n, batch, dir, -1, -1, 0, kYSamples - kLineSamples);
    if (st != FFT_OK)
        return st;
    if (p.kind == Plan::GENERIC)
        p.sub_batch = std::min<uint64_t>(batch, kYSamples / 2 / n);
    if (p.kind != Plan::COPY && p.kind != Plan::SINGLE && p.sub_batch == 0)
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH,
                         "length %llu needs up to %llu samples of scratch; the static "
                         "scratch holds %llu",
                         (unsigned long long)n, (unsigned long long)(2 * n),
                         (unsigned long long)kYSamples);
    Tables tabs;
    // (offsets from the array, then the array's address added)
    uint64_t tw = 0, tw2 = 0, w1 = 0, tl = 0, th = 0, tl2 = 0, th2 = 0;
    const bool two = p.kind == Plan::FOURSTEP || (p.kind == Plan::GENERIC && p.stages.passes > 1);
    auto two_level = [&](uint64_t m, int sh, bool wide, uint64_t *low, uint64_t *high) {
        const uint64_t lo = 1ull << sh;
        *low = tabs.add(lo, m, 1, wide);
        *high = tabs.add((m + lo - 1) / lo, m, lo, wide);
    };
    switch (p.kind) {
    case Plan::COPY: break;
    case Plan::SINGLE: tw = tabs.add(n, n, 1, false); break;
    case Plan::FOURSTEP:
        two_level(n, p.sh, false, &tl, &th);
        tw = tabs.add(p.n1, p.n1, 1, false);
        tw2 = tabs.add(p.n2, p.n2, 1, false);
        break;
    case Plan::GENERIC:
        if (two)
            two_level(n, p.sh, true, &tl, &th);
        if (p.stages.passes == 3) {
            const uint64_t m = n / (uint64_t)p.stages.a.n;
            p.sh2 = two_level_shift(m);
            two_level(m, p.sh2, true, &tl2, &th2);
        }
        tw = tabs.add(p.stages.a);
        tw2 = tabs.add(p.stages.b);
        w1 = tabs.add(p.stages.mid);
        break;
    default:
        return set_error(FFT_ERR_INVALID_ARG, "real plans are not served here");
    }
    if (tabs.room > kTableSamples)
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH,
                         "the tables of length %llu (%llu entries) exceed the %llu of static "
                         "scratch", (unsigned long long)n, (unsigned long long)tabs.room,
                         (unsigned long long)kTableSamples);
    void *base = nullptr;
    if ((st = scratch_ptr(p.device, &base)) != FFT_OK)
        return st;
    c32 *tables = (c32 *)base;
    if (tabs.total)
        tabs.launch(tables, s);
    p.tw = tables + tw;
    p.tw2 = tables + tw2;
    p.w1 = tables + w1;
    p.tl = tables + tl;
    p.th = tables + th;
    p.tl2 = tables + tl2;
    p.th2 = tables + th2;
    p.scratch = two ? tables + kTableSamples : nullptr;
    st = plan_enqueue(&p, in, out, batch, s);
    // nothing of the description is device memory: keep plan_free's hands off
    p.tw = p.tw2 = p.w1 = p.tl = p.th = p.tl2 = p.th2 = p.scratch = nullptr;
    return st;
}

}  // namespace
}  // namespace fftseg

using namespace fftseg;

extern "C" int fft_exec_segments_noalloc(size_t segment_len, size_t batch, int direction,
                                         const void *in, void *out, void *stream)
{
    try {
        if (validate_create(segment_len, batch, direction) != FFT_OK)
            return last_status();
        int st = check_io(in, out, (uint64_t)batch * segment_len * sizeof(c32));
        if (st != FFT_OK)
            return st;
        return noalloc_enqueue(segment_len, batch, direction, in, out, (hipStream_t)stream);
    } catch (...) {
        return set_error(FFT_ERR_INVALID_ARG, "internal error");
    }
}
