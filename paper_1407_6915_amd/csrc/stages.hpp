// Run-time radix schedules: LDS-resident Stockham transforms of any length
// with prime factors 2, 3 and 5, for the lengths without a compiled tile
// (tile.hpp), as one pass over whole segments or as the two passes of a
// four-step split n = n1 n2.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <vector>

#include "radix.hpp"

namespace fftseg {

constexpr int kMaxLdsStages = 8;

// Radices whose stages form their twiddles as powers of one FP64 entry
// (twiddle_powers); the others read an entry for each (from 12 on 0.9 % and from 5
// on 0.2 % slower over 150 lengths).
constexpr bool lds_powers(int r) { return r >= 8; }

// One stage: nb butterflies of radix r at stride l (the product of the
// radices before it); its twiddles W_{l r}^{j k}, 1 <= j < r, k < l, sit at
// tw + (j - 1) l + k of the schedule's table, or, where lds_powers(r), W_{l r}^k
// alone in FP64 from tw on (counted in float32 entries, even).  ml, mnb:
// reciprocals for fast_div by l and nb.
struct LdsStage {
    int r, l, nb, tw;
    uint32_t ml, mnb;
};
struct LdsSched {
    int n, ns;
    LdsStage st[kMaxLdsStages];
};

// The kernels come in three forms.  kNarrow: radices up to 16 (and 25), near
// 16 values a thread.  kMost: the same radices with more butterflies a
// thread, for tiles that 1024 threads hold only so.  kWide: radices up to 32
// and near 32 values a thread (column tiles: at most 512 threads, for their
// registers): one LDS exchange where the others need two.
enum StagesForm { kNarrow, kMost, kWide };

// Butterflies of one stage that a thread may own.
constexpr int lds_units(int r, int form)
{
    if (form == kWide)
        return r <= 4 ? 8 : r == 5 ? 6 : r == 6 ? 5 : r == 8 ? 4 : r <= 10 ? 3 : r <= 16 ? 2 : 1;
    switch (r) {
    case 2: return 8;
    case 3: return 6;
    case 4: return 4;
    case 5: return 4;
    case 6: return 3;
    case 8: case 9: case 10: return 2;
    case 12: case 15: case 16: return form == kMost ? 2 : 1;
    default: return 1;  // 25
    }
}
constexpr int form_threads(int form, bool column)
{
    return form == kWide && column ? 512 : 1024;
}

// The schedule of an n-point transform (n >= 2, prime factors 2, 3, 5);
// false if it would take more than kMaxLdsStages stages.  group > 1: the
// last stage's lanes take butterflies in groups of `group` (column pass), so
// the last radix is the one that fills them best.  group 0: whole segments, a
// segment's butterflies on consecutive lanes.  wide: radices above 16.
bool lds_schedule(int n, LdsSched *s, bool wide, int group = 1);
// Threads of a workgroup whose tile holds `tiles` transforms of the
// schedule (the last stage's butterflies of each in groups of `group`);
// 0 if the form's largest workgroup cannot hold it.
int lds_threads(const LdsSched &s, int tiles, int group, int form, bool column);
// float32 entries of the schedule's twiddle table (an FP64 entry is two), even
int lds_table_size(const LdsSched &s);
std::vector<c32> lds_table(const LdsSched &s);
// the radices as the planner reports them: radix 9, 18, 24, 27 and 30 stages
// as their in-register steps
void lds_radices(const LdsSched &s, std::vector<int> *out);

// The plan of a length without compiled tiles.
struct StagesPlan {
    // 1: whole segments in LDS; 2: columns, then rows; 3: columns, then the
    // rows themselves in two passes
    int passes = 0;
    LdsSched a{}, b{};       // the pass (or column pass), the row pass
    LdsSched mid{};          // three passes: the one between
    int segs = 1;            // one pass: segments per workgroup
    int lc = 0, lr = 0;      // two passes: log2 of the columns / rows per workgroup
    int threads_a = 0, threads_b = 0;
    int form_a = kNarrow, form_b = kNarrow, form_mid = kNarrow, threads_mid = 0;
    unsigned blocks_a = 0, blocks_b = 0;  // two passes: tiles of a segment
    int real = 0;            // real segments of 2n samples: -1 forward (the row tiles pair
                             // rows k1 and n1 - k1), +1 inverse (the column tiles pair
                             // columns)
    uint64_t y_samples = 0;  // two and three passes: samples of Y per segment
};
// false if the length has no plan (none of the supported lengths)
bool stages_choose(uint64_t n, uint64_t batch, int cus, StagesPlan *p, int real = 0);
// Launches of `batch` segments: segment s starts at in + s * hop and is
// multiplied by window[0..n) if that is not null; its spectrum goes to
// out + s * n.
hipError_t stages_one_pass(const StagesPlan &p, int dir, const void *in, void *out,
                           const void *tw, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s);
struct StagesTables {          // device addresses
    const void *a, *b, *mid;   // the schedules' twiddles
    const void *tl, *th;       // two-level W_n (c64)
    int sh;
    const void *tl2, *th2;     // three passes: two-level W_{n / n1}
    int sh2;
};
hipError_t stages_two_pass(const StagesPlan &p, int dir, const void *in, void *out, void *y,
                           const StagesTables &t, uint64_t batch, uint64_t hop,
                           const float *window, hipStream_t s);

hipError_t stages_rows(const StagesPlan &p, int dir, const void *y, void *out, const void *tw,
                       uint64_t batch, hipStream_t s);
// Real segments of N = 2n samples (plans of stages_choose with `real`): the
// batch's rows of N float32 (n complex values) and of n + 1 bins.  One pass:
// hw = W_N^k, k <= n/2.  Two, in FP64: w1 = W_N^j for the first half of the paired
// rows (columns) j, w2 = W_{2 n2}^k, k < n2 (forward) or W_{2 n1}^i, i < n1
// (inverse).
hipError_t stages_real_one_pass(const StagesPlan &p, const void *in, void *out, const void *tw,
                                const void *hw, uint64_t batch, hipStream_t s);
hipError_t stages_real_two_pass(const StagesPlan &p, const void *in, void *out, void *y,
                                const void *tw_a, const void *tw_b, const void *tl,
                                const void *th, int sh, const void *w1, const void *w2,
                                uint64_t batch, hipStream_t s);

constexpr int kLdsBytes = 160 * 1024;

// LDS of a column tile: its samples, from an even slot on one W_N factor (c64) a
// column; of a row tile
constexpr int column_slots(int n, int lc) { return (n * ((1 << lc) + 1) + 1) & ~1; }
inline size_t columns_lds(const LdsSched &s, int lc)
{
    return column_slots(s.n, lc) * sizeof(c32) + (sizeof(c64) << lc);
}
inline size_t rows_lds(const LdsSched &s, int lr) { return ((size_t)s.n << lr) * sizeof(c32); }

// fast_div's multiplier for a division by d: exact for x d < 2^32
inline uint32_t reciprocal(int d)
{
    return d <= 1 ? 0u : (uint32_t)((1ull << 32) / (uint64_t)d + 1);
}

// a workgroup's LDS may go past the runtime's default limit
template <class K>
hipError_t allow_lds(K kernel, size_t bytes)
{
    if (bytes <= 64 * 1024)
        return hipSuccess;
    return hipFuncSetAttribute((const void *)kernel, hipFuncAttributeMaxDynamicSharedMemorySize,
                               kLdsBytes);
}

// grid of `tiles` workgroups for xcd_tile
inline unsigned xcd_grid(uint64_t tiles) { return (unsigned)((tiles + 7) / 8 * 8); }

}  // namespace fftseg
