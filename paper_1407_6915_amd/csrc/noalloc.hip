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

// tables: W_N (one pass) or W_N1, W_N2 and the two-level W_N (two passes)
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

// exp(-2 pi i m / n) in FP64, the angle folded to the first octant in exact
// integer arithmetic (8 m < 2^28 here)
__device__ c64 device_root(uint64_t m, uint64_t n)
{
    m %= n;
    const uint64_t m8 = m * 8u;
    const uint64_t o = m8 / n, r = m8 - o * n;
    const uint64_t j = (o + 1) / 2;
    const double quarter_pi = 0.78539816339744830961566084581987572;
    const double x = ((double)((long long)o - 2 * (long long)j) + (double)r / (double)n) *
                     quarter_pi;
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

// Consecutive tables: table t holds count[t] entries W_{mod[t]}^{j step[t]},
// j < count[t], or, with rows of l[t] entries (the twiddles of one stage of
// a run-time schedule), W_{mod[t]}^{(1 + j / l[t]) (j mod l[t])}.  The first
// `wide` tables are in FP64, the others rounded once to float32.
constexpr int kMaxTables = 4 + 3 * kMaxLdsStages;
struct TableSet {
    uint64_t count[kMaxTables], mod[kMaxTables], step[kMaxTables], l[kMaxTables];
    int wide;
};

// the tables of a schedule's stages from table t on; returns the next table
int add_schedule(TableSet &ts, int t, const LdsSched &s)
{
    for (int i = 1; i < s.ns; ++i, ++t) {
        ts.l[t] = (uint64_t)s.st[i].l;
        ts.count[t] = (uint64_t)(s.st[i].r - 1) * ts.l[t];
        ts.mod[t] = (uint64_t)s.st[i].r * ts.l[t];
    }
    return t;
}

__global__ void __launch_bounds__(256) static_tables_kernel(c32 *tables, TableSet ts,
                                                            uint64_t total)
{
    for (uint64_t i = (uint64_t)blockIdx.x * 256 + threadIdx.x; i < total;
         i += (uint64_t)gridDim.x * 256) {
        uint64_t j = i;
        uint64_t at = 0;  // in float32 entries
        int t = 0;
        while (t + 1 < kMaxTables && j >= ts.count[t]) {
            at += ts.count[t] * (t < ts.wide ? 2 : 1);
            j -= ts.count[t];
            ++t;
        }
        const uint64_t l = ts.l[t];
        const c64 w = device_root(l ? (1 + j / l) * (j % l) : j * ts.step[t], ts.mod[t]);
        if (t < ts.wide)
            reinterpret_cast<c64 *>(tables + at)[j] = w;
        else
            tables[at + j] = c32{(float)w.x, (float)w.y};
    }
}

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
    TableSet ts{};
    uint64_t total = 0;
    switch (p.kind) {
    case Plan::COPY: break;
    case Plan::SINGLE:
        ts.count[0] = n; ts.mod[0] = n; ts.step[0] = 1;
        break;
    case Plan::FOURSTEP:
    case Plan::GENERIC: {
        if (p.kind == Plan::GENERIC && p.stages.passes == 1) {
            add_schedule(ts, 0, p.stages.a);
            break;
        }
        const uint64_t lo = 1ull << p.sh;
        ts.count[0] = lo; ts.mod[0] = n; ts.step[0] = 1;                  // tl
        ts.count[1] = (n + lo - 1) / lo; ts.mod[1] = n; ts.step[1] = lo;  // th
        if (p.kind == Plan::FOURSTEP) {
            ts.count[2] = p.n1; ts.mod[2] = p.n1; ts.step[2] = 1;         // W_N1
            ts.count[3] = p.n2; ts.mod[3] = p.n2; ts.step[3] = 1;         // W_N2
        } else {
            // the two-level tables, in FP64, before the schedules'
            int t = 2;
            if (p.stages.passes == 3) {
                const uint64_t m = n / (uint64_t)p.stages.a.n;
                p.sh2 = two_level_shift(m);
                const uint64_t lo2 = 1ull << p.sh2;
                ts.count[2] = lo2; ts.mod[2] = m; ts.step[2] = 1;                     // tl2
                ts.count[3] = (m + lo2 - 1) / lo2; ts.mod[3] = m; ts.step[3] = lo2;  // th2
                t = 4;
            }
            ts.wide = t;
            add_schedule(ts, add_schedule(ts, add_schedule(ts, t, p.stages.a), p.stages.b),
                         p.stages.mid);
        }
        break;
    }
    default:
        return set_error(FFT_ERR_INVALID_ARG, "real plans are not served here");
    }
    for (int t = 0; t < kMaxTables; ++t)
        total += ts.count[t];
    uint64_t room = total;  // in float32 entries
    for (int t = 0; t < ts.wide; ++t)
        room += ts.count[t];
    if (room > kTableSamples)
        return set_error(FFT_ERR_UNSUPPORTED_LENGTH,
                         "the tables of length %llu (%llu entries) exceed the %llu of static "
                         "scratch", (unsigned long long)n, (unsigned long long)room,
                         (unsigned long long)kTableSamples);
    void *base = nullptr;
    if ((st = scratch_ptr(p.device, &base)) != FFT_OK)
        return st;
    c32 *tables = (c32 *)base;
    c32 *y = tables + kTableSamples;
    if (total) {
        const unsigned grid = (unsigned)std::min<uint64_t>((total + 255) / 256, 1024);
        hipLaunchKernelGGL(static_tables_kernel, dim3(grid), dim3(256), 0, s, tables, ts, total);
    }
    switch (p.kind) {
    case Plan::SINGLE: p.tw = tables; break;
    case Plan::FOURSTEP:
        p.tl = tables;
        p.th = tables + ts.count[0];
        p.tw = tables + ts.count[0] + ts.count[1];
        p.tw2 = tables + ts.count[0] + ts.count[1] + ts.count[2];
        p.scratch = y;
        break;
    case Plan::GENERIC:
        if (p.stages.passes == 1) {
            p.tw = tables;
            break;
        }
        {
            c32 *at = tables;
            void **wide[4] = {&p.tl, &p.th, &p.tl2, &p.th2};
            for (int t = 0; t < ts.wide; ++t) {
                *wide[t] = at;
                at += 2 * ts.count[t];
            }
            p.tw = at;
            p.tw2 = at + lds_table_size(p.stages.a);
            p.w1 = (c32 *)p.tw2 + lds_table_size(p.stages.b);
        }
        p.scratch = y;
        break;
    default: break;
    }
    st = plan_enqueue(&p, in, out, batch, s);
    // nothing of the description is device memory: keep plan_free's hands off
    p.tw = p.tw2 = p.tl = p.th = p.scratch = nullptr;
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
