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

// One stage: nb butterflies of radix r at stride l (the product of the
// radices before it); its twiddles W_{l r}^{j k}, 1 <= j < r, k < l, sit at
// tw + (j - 1) l + k of the schedule's table.  ml, mnb: reciprocals for
// fast_div by l and nb.
struct LdsStage {
    int r, l, nb, tw;
    uint32_t ml, mnb;
};
struct LdsSched {
    int n, ns;
    LdsStage st[kMaxLdsStages];
};

// Butterflies of one stage that a thread may own.  `most`: in the kernels
// for tiles that 1024 threads hold only so; the others keep to the smaller
// count, near 16 values, and to fewer registers.
constexpr int lds_units(int r, bool most)
{
    switch (r) {
    case 2: return 8;
    case 3: return 6;
    case 4: return 4;
    case 5: return 4;
    case 6: return 3;
    case 8: case 9: case 10: return 2;
    case 12: case 15: case 16: return most ? 2 : 1;
    default: return 1;  // 25
    }
}

// The schedule of an n-point transform (n >= 2, prime factors 2, 3, 5);
// false if it would take more than kMaxLdsStages stages.  group > 1: the
// last stage's lanes take butterflies in groups of `group` (column pass), so
// the last radix is the one that fills them best.
bool lds_schedule(int n, LdsSched *s, int group = 1);
// Threads of a workgroup whose tile holds `tiles` transforms of the
// schedule (the last stage's butterflies of each in groups of `group`);
// 0 if 1024 threads cannot hold it.  *most: it needs the kernels compiled
// for lds_units(r, true).
int lds_threads(const LdsSched &s, int tiles, int group, bool *most);
// entries of the schedule's twiddle table (s.n - first radix)
int lds_table_size(const LdsSched &s);
std::vector<c32> lds_table(const LdsSched &s);
// the radices as the planner reports them: a radix-9 stage as its two
// radix-3 steps
void lds_radices(const LdsSched &s, std::vector<int> *out);

// The plan of a length without compiled tiles.
struct StagesPlan {
    int passes = 0;          // 1: whole segments in LDS; 2: columns, then rows
    LdsSched a{}, b{};       // the pass (or column pass), the row pass
    int segs = 1;            // one pass: segments per workgroup
    int lc = 0, lr = 0;      // two passes: log2 of the columns / rows per workgroup
    int threads_a = 0, threads_b = 0;
    bool most_a = false, most_b = false;  // see lds_threads
    uint64_t y_samples = 0;  // two passes: samples of Y per segment
};
// false if the length has no plan (none of the supported lengths)
bool stages_choose(uint64_t n, uint64_t batch, int cus, StagesPlan *p);
// Launches of `batch` segments: segment s starts at in + s * hop and is
// multiplied by window[0..n) if that is not null; its spectrum goes to
// out + s * n.
hipError_t stages_one_pass(const StagesPlan &p, int dir, const void *in, void *out,
                           const void *tw, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s);
hipError_t stages_two_pass(const StagesPlan &p, int dir, const void *in, void *out, void *y,
                           const void *tw_a, const void *tw_b, const void *tl, const void *th,
                           int sh, uint64_t batch, uint64_t hop, const float *window,
                           hipStream_t s);

}  // namespace fftseg
