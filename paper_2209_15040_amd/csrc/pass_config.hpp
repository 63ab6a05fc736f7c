// Launch geometry of the pencil passes.
//
//   T  threads per pencil          P  pencils (contiguous layout) or
//   K  LDS exchange rounds            columns (strided layout) per workgroup
//
// Rules for the lengths that the measured tables below (kStrided*, kContig*) do
// not list, and for the tuner's radix variant:
// * strided tiles of 32 columns: 256-byte rows for complex64, 128-byte rows
//   for the 4-byte types; 64 columns up to 64 points;
// * strided complex64 tiles take radix <= 16 stages (plan 1), the 4-byte types
//   the fewest stages (plan 0);
// * up to 32 elements per thread, the exchange split into rounds of up to ~72
//   KB of LDS, so two workgroups stay resident per CU and one's transform and
//   store drain overlap the other's loads;
// * contiguous pencils: N/16 threads each where the widest stage leaves
//   every thread a butterfly, 256-thread workgroups (one wave for the 4-byte
//   types and for 1024-point complex64), and paired (two-element) first-stage
//   loads where the stage allows them;
// * non-temporal (streaming) loads and stores, unless the cache policies of
//   wsfft_api.hip choose others.
// FP16 storage with FP16 arithmetic (4-byte register and LDS values, argument
// vb = 4) holds half the state per element: strided tiles of 64 columns
// (256-byte rows) for powers of two with twice the elements per thread,
// exchange rounds of at most ~36 KB, and 256-thread contiguous tiles.
#pragma once
#include "fft_device.hpp"

namespace wsfft {

constexpr int kLdsBytesMax = 160 * 1024;   // LDS per CU on gfx950
constexpr int kLdsRoundBudget = 36 * 1024; // LDS per exchange round, 256-thread strided tiles
constexpr int kPassFlags = kFlagNontemporal;

// Radix plan of the default contiguous kernel: the fewest stages, except
// that pencils of up to 32 points take radix <= 8 stages so that 4 threads
// share a pencil (cfg_T_contig), and the 4-byte storage types take radix
// <= 16 stages (512 points: 8 x 8 x 8 with 16 elements per thread, 185-188
// us per GiB against 197-208 us for 16 x 32).
constexpr int cfg_plan_contig(int N, int bytes = 8) { return N <= 32 ? 2 : (bytes == 4 ? 1 : 0); }

// Radix plan of the default strided kernel (see make_radices).
constexpr int cfg_plan_strided(int N, int bytes) {
    (void)N;
    return bytes == 8 ? 1 : 0;
}

// At least 4 threads per pencil where the radix plan allows: with one
// thread per pencil a wave's 64 lanes read 64 pencils, 64 cache lines per
// access.
constexpr int cfg_T_contig(int N, int plan = 0) {
    int t = N / 16;
    if (t < 4) t = 4;
    // every thread must own at least one butterfly of the widest stage
    const int tmax = N / max_radix(make_radices(N, plan));
    if (tmax >= 1 && t > tmax) t = tmax;
    return t > 1024 ? 1024 : t;
}
// Contiguous tiles: 256-thread workgroups for complex64; one wave for the
// 4-byte types, whose tiles carry half the bytes, so more workgroups (and
// more bytes in flight) fit per CU within the same FP32 LDS budget.  The
// 1024-point complex64 tile is one wave as well (two pencils, 17 KB of LDS:
// 355 us per GiB against 363-390 us for eight pencils in 256 threads).
constexpr int cfg_P_contig(int N, int plan = 0, int bytes = 8, int vb = 8) {
    const int p = ((bytes == 8 && N != 1024) || vb == 4 ? 256 : 64) / cfg_T_contig(N, plan);
    return p < 1 ? 1 : p;
}

constexpr bool is_pow2(int n) { return n > 0 && (n & (n - 1)) == 0; }
constexpr int pow2_floor(int n) {
    int p = 1;
    while (p * 2 <= n) p *= 2;
    return p;
}

// Elements per thread in the strided layout: 32 for powers of two (16 up to
// N = 128, so that tiles of these short lengths still have 256 threads and
// a CU holds 16 waves); radix-3 stages leave some threads idle, so fewer
// there to stay within registers.
// Past 512 threads per tile (32 columns x 16 threads) the elements per thread
// double instead: 1024-thread workgroups are held to 128 VGPRs and spill.
constexpr int cfg_T_strided(int N, int bytes, int plan = 0, int vb = 8) {
    (void)bytes;
    int e = is_pow2(N) ? (N <= 128 ? 16 : 32) : 24;
    if ((N + e - 1) / e > 16) e *= 2;
    if (vb == 4 && is_pow2(N) && N <= 512) e *= 2;   // longer or radix-3 pencils would spill
    int t = (N + e - 1) / e;
    const int tmax = N / max_radix(make_radices(N, plan));
    if (tmax >= 1 && t > tmax) t = tmax;
    return t < 1 ? 1 : t;
}
constexpr int cfg_P_strided(int N, int bytes, int plan = 0, int vb = 8) {
    (void)bytes;
    int p = 32;
    if (N <= 64 || (vb == 4 && is_pow2(N))) p = 64;   // one full wave of columns at least
    const int cap = pow2_floor(1024 / cfg_T_strided(N, bytes, plan, vb));
    return p > cap ? cap : p;
}
// Smallest K dividing N whose exchange round fits the LDS budget (twice the
// per-round budget for workgroups of up to 512 threads, two of which still
// fit per CU; four times at 1024 points); when that takes more than 8
// rounds, accept up to twice the budget instead.
constexpr int cfg_K_strided(int N, int bytes, int plan = 0, int vb = 8) {
    const int p = cfg_P_strided(N, bytes, plan, vb);
    // 1024-point tiles run best with two rounds and one workgroup per CU
    const int budget = vb == 4 ? kLdsRoundBudget
                       : N >= 1024 ? 4 * kLdsRoundBudget
                       : cfg_T_strided(N, bytes, plan) * p <= 512 ? 2 * kLdsRoundBudget : kLdsRoundBudget;
    int first = 0;
    for (int k = 1; k <= N && !first; ++k)
        if (N % k == 0 && (N / k) * (p + 1) * vb <= budget) first = k;
    if (first && first <= 8) return first;
    for (int k = 1; k <= N; ++k)
        if (N % k == 0 && (N / k) * (p + 1) * vb <= 2 * kLdsRoundBudget) return k;
    return first ? first : N;
}

// Measured geometry of the default strided kernel, for the lengths where the
// rules above are not the best choice.  The rules count elements per thread;
// what bounds these tiles is how much of a CU stays busy: a thread count that
// does not divide every stage's butterflies leaves lanes idle in each stage,
// radix-3 lengths take a third and fourth stage (one more LDS exchange each)
// under radix <= 16, and tiles of 24 .. 48 elements per thread hold one
// workgroup per CU at 150-210 VGPRs, or spill.  So: the two-stage schedule
// with radices up to 32 (plan 0) where it exists and keeps a butterfly per
// thread in both stages, T a divisor of the butterfly counts or near one, and
// from 432 points on 16-column tiles (128-byte rows of complex64) with two or
// more workgroups per CU.  Every (T, P, K, plan) with at most 16% idle lanes was
// timed over a y-like (columns of one plane) and a z-like array of 256 and 64
// MiB; an entry is the best of the four together and stands where it gains 2%
// or more.  GB/s (y / z, 256 MiB complex64), rule -> entry: 162 4806/4433 ->
// 5688/4979, 216 4769/4514 -> 5313/5062, 243 4710/4519 -> 5161/4972, 288
// 4926/4576 -> 5512/5052, 324 4680/4404 -> 4896/4497, 432 3188/3013 ->
// 4733/4609, 486 3120/3050 -> 4700/4521, 576 3673/3465 -> 4914/4460, 648
// 3440/3348 -> 4742/4682, 729 3545/3403 -> 4593/4560, 768 3861/3685 ->
// 4915/4764, 864 2799/2713 -> 4407/4084, 972 2581/2538 -> 4167/4170, 1024
// 4567/3733 -> 4786/4019 (half width 5077/3948, cfg_half).
// No complex64 entry rounds more than the rule's radix schedule: the relative
// error of single passes against FP64 (2^21 values per length, 0.2% between
// seeds) grew by 3.4% at 576 points in four stages instead of three, 2.4% at 864
// in 27 x 32 and 2.1% at 324 in 18 x 18, so these keep the rule's radices
// (5019/4481, 4781/4348 and 5510/4968 GB/s without that condition; 1024 in
// 32 x 32 instead of 4 x 16 x 16 is level, see PencilPass::FINE).  Storage of 16 bits
// rounds far more than any schedule: its entries may take other stages (768
// points 8 x 8 x 12 instead of 24 x 32).
// 256 points keep the rule's tile with the exchange in two rounds, four
// workgroups per CU instead of two: 5499/5142 -> 5436/5145 at 256 MiB,
// 5071/4802 -> 5512/5317 at 64.  (Complex64 tiles of 128 and 256 points in 64
// columns gained 4-7% there but leave the chip short of workgroups on 128^3 and
// the half spectra of 256^3, which lost 2-6%.)  The 4-byte types gain 3-40%
// (864: 2.7x) the same way; FP16 values hold half the state and keep the wider
// tiles.  (Launches of few 64-column tiles take half-width ones, wsfft_api.hip.)
struct StridedGeo {
    int n, T, P, K, plan;
};
constexpr StridedGeo kStrided8[] = {   // complex64
    {72, 9, 32, 1, 0},   {81, 9, 32, 1, 0},   {162, 9, 32, 1, 0},  {216, 6, 32, 2, 0},
    {243, 9, 32, 3, 0},  {256, 8, 32, 2, 1},  {288, 18, 32, 1, 0}, {324, 12, 16, 2, 1},
    {432, 12, 16, 2, 1}, {486, 27, 16, 2, 1}, {576, 16, 16, 3, 1}, {648, 27, 16, 2, 0}, {729, 27, 16, 3, 0},
    {768, 32, 16, 3, 1}, {864, 24, 16, 3, 1}, {972, 27, 16, 2, 0}, {1024, 16, 32, 2, 0}};
constexpr StridedGeo kStrided4[] = {   // 4-byte storage, FP32 values
    {48, 8, 32, 1, 0},   {64, 8, 64, 1, 0},   {72, 9, 32, 1, 0},   {81, 9, 64, 1, 0},
    {96, 4, 64, 2, 0},   {108, 12, 32, 1, 0},  {128, 8, 64, 2, 0},  {144, 12, 64, 1, 0},  {162, 9, 64, 2, 0},
    {192, 8, 32, 2, 0},  {216, 6, 32, 2, 0},  {243, 9, 64, 3, 0},  {256, 8, 64, 2, 0},  {288, 18, 32, 1, 0},
    {324, 18, 32, 2, 0}, {432, 16, 32, 2, 1}, {486, 18, 32, 2, 0}, {576, 16, 32, 2, 2}, {648, 27, 32, 3, 0},
    {729, 27, 32, 3, 0}, {768, 32, 32, 3, 1}, {864, 32, 32, 3, 0}, {972, 27, 32, 4, 0}};
constexpr StridedGeo kStrided4m[] = {   // 4-byte storage, FP16 values
    {72, 9, 64, 1, 0},   {81, 9, 64, 1, 0},   {96, 8, 64, 1, 0},   {108, 12, 64, 1, 0}, {144, 4, 64, 1, 0},
    {162, 9, 64, 1, 0},  {192, 4, 64, 1, 0},  {216, 6, 64, 1, 0},  {288, 8, 64, 1, 0},  {324, 18, 32, 1, 0},
    {384, 8, 64, 3, 0},  {432, 24, 32, 1, 0}, {486, 18, 32, 1, 0}, {576, 24, 32, 1, 0}, {648, 14, 32, 2, 0},
    {729, 27, 32, 3, 0}, {768, 16, 32, 2, 1}, {864, 16, 32, 2, 0}, {972, 27, 32, 2, 0}, {1024, 16, 64, 4, 0}};

// Half-width tile of the default strided kernel (variant 2): the same with half
// the columns, or the measured one.  The 1024-point complex64 tile holds a CU by
// itself (135 KB of LDS), two of its half-width ones of 32 threads share one.
// Where the rows of an array are less than kNearRows bytes apart those are
// faster, beyond that their 128-byte rows cost more (GB/s, full / half width, by the
// distance of the rows over 2 GiB and 256 MiB: 8 KB 4963/5254 and 4869/5072, 16
// KB 5076/5135 and 4989/4838, 32 KB 4843/5014 and 4773/4994, 48 KB of 6144 x
// 1024 x 16, y and the cached x together 924/882 us, 64 KB 4830/4428 and 4897/4545, 256 KB 3955/3758 and 4028/3926, 8 MB over 8 GiB 4393/3859; the
// rule's tile at 8 MB 3961).
constexpr int kNearRows = 64 * 1024;
constexpr StridedGeo cfg_half(StridedGeo g, int bytes) {
    if (bytes == 8 && g.n == 1024) return {1024, 32, 16, 2, 0};
    if (g.P > 1) g.P /= 2;
    return g;
}
// Whether a tile holds a CU by itself and halves to whole cache lines, and
// whether a launch may halve it (set_narrow).
constexpr bool cfg_alone(int lds, int P, int bytes) { return lds > kLdsBytesMax / 2 && P / 2 * bytes >= 128; }
constexpr bool cfg_halves(int lds, int P, int bytes) { return P >= 64 || cfg_alone(lds, P, bytes); }

// Exchange rounds of a split axis's first pass: its FP64 twiddle recurrence
// restarts in every round, so powers of two take the fewest rounds that leave
// two workgroups per CU (256 points, 65536 x 1024: one round 414 us, two 439).
constexpr int cfg_K_four_step(int N, int P, int K, int vb) {
    if (!is_pow2(N)) return K;
    for (int k = 1; k < K; ++k)
        if (N % k == 0 && (N / k) * (P + 1) * vb <= 2 * kLdsRoundBudget) return k;
    return K;
}

// Exchange rounds of the strided kernel that streams past the caches: 256
// points of complex64 take one (second pass of 65536 x 1024: 184.7 us, two
// rounds 194.5; y axis of 512x256x512: 186.8 and 194.1), where the cached and
// fused kernels of smaller arrays take the two of the table (256^3 Poisson 331
// us, one round 345).  Both sides are measured; the cause is not resolved: two
// rounds hold four workgroups per CU instead of two and wait at one barrier
// more.
constexpr int cfg_K_stream(int N, int bytes, int K) { return N == 256 && bytes == 8 ? 1 : K; }

// Geometry of the default strided kernel: the measured entry, else the rules.
constexpr StridedGeo cfg_strided(int N, int bytes, int vb) {
    if (bytes == 8) {
        for (const StridedGeo& g : kStrided8)
            if (g.n == N) return g;
    } else if (vb == 8) {
        for (const StridedGeo& g : kStrided4)
            if (g.n == N) return g;
    } else {
        for (const StridedGeo& g : kStrided4m)
            if (g.n == N) return g;
    }
    const int plan = cfg_plan_strided(N, bytes);
    return {N, cfg_T_strided(N, bytes, plan, vb), cfg_P_strided(N, bytes, plan, vb), cfg_K_strided(N, bytes, plan, vb),
            plan};
}

// Measured geometry of the default contiguous kernel, for the lengths where
// the rules above are not the best choice.  A direct tile reads and writes
// T-element pieces of pencils: pieces shorter than a cache line, or of
// pencils that are no whole lines apart, make streaming accesses fetch and
// write the same line several times (27 points 1.2 TB/s, 81 points 1.3, 108
// points 1.2, 32 points 3.5).  Staged tiles (kFlagStage) move the tile's rows
// as one contiguous range through LDS, whole lines per wave, for two more LDS
// trips per element; the rest of an entry is as in the strided tables.  Direct and staged
// tiles of every (T, P, plan) were timed at 256 and 32 MiB; staged wins on
// short and radix-3 lengths, direct from about 500 points on where pencils
// are whole lines.  GB/s at 256 MiB of complex64, rule -> entry: 16 3236 ->
// 6281, 27 1191 -> 5823, 32 3546 -> 6235, 36 1290 -> 5849, 64 5903 -> 6183,
// 81 1296 -> 5880, 96 5299 -> 6096, 108 1175 -> 5870, 144 1908 -> 6034, 192
// 4237 -> 5899, 216 3898 -> 5919, 243 3782 -> 5418, 288 4440 -> 5781, 324
// 4617 -> 5829, 384 4845 -> 5796, 432 3950 -> 5253, 486 3939 -> 5392, 512
// 5792 -> 6104, 576 5281 -> 5902, 648 4048 -> 5305, 768 4548 -> 5889, 864
// 3911 -> 5404, 972 3891 -> 5459, 1296 4174 -> 5744, 1728 4014 -> 5628, 4096
// 5361 -> 5853, 7776 2704 -> 4073, 8192 4714 -> 4925, 15552 3496 -> 3820.  As
// in the strided table, no entry rounds more than the rule's radix schedule:
// more or narrower stages raised the error by 6.1% at 576 points, 5.6% at 1296,
// 4.8% at 1728, 4.2% at 108, 0.5-2.1% at 486, 648, 729, 972, 2187, 3888, 4374,
// 6561, 7776 and 8748 (FP16 arithmetic: 1.2% at 729), which keep the rule's
// radices; 2187, 3888, 4374 and 8748 then have no better geometry than the
// rule's.
struct ContigGeo {
    int n, T, P, plan;
    bool stage;
};
constexpr ContigGeo kContig8[] = {   // complex64
    {2, 1, 256, 0, true}, {3, 1, 256, 0, true}, {4, 1, 128, 0, true}, {6, 1, 128, 0, true}, {8, 1, 256, 0, true},
    {9, 1, 256, 0, true}, {12, 1, 64, 2, true}, {16, 1, 64, 2, true}, {18, 2, 64, 1, true}, {24, 2, 32, 1, true},
    {27, 1, 128, 0, true}, {32, 2, 64, 1, true}, {36, 3, 42, 0, true}, {48, 2, 32, 0, true},
    {54, 6, 21, 0, true}, {64, 4, 32, 0, true}, {72, 9, 28, 0, true}, {81, 9, 28, 0, true}, {96, 8, 16, 0, true},
    {108, 9, 14, 0, true}, {128, 8, 16, 0, true}, {144, 12, 10, 0, true}, {162, 27, 9, 2, true},
    {192, 16, 8, 0, true}, {216, 12, 10, 0, true}, {243, 27, 18, 1, true}, {256, 16, 16, 0, true},
    {288, 16, 16, 0, true}, {324, 18, 14, 0, true}, {384, 16, 4, 0, true}, {432, 24, 5, 0, true},
    {486, 18, 7, 0, true}, {512, 32, 4, 1, false}, {576, 24, 10, 0, true}, {648, 24, 5, 0, true},
    {729, 27, 4, 0, true}, {768, 32, 2, 1, false}, {864, 32, 4, 0, false}, {972, 81, 3, 0, true},
    {1296, 108, 2, 0, true}, {1458, 81, 3, 0, true}, {1728, 72, 3, 0, false}, {1944, 122, 1, 1, true},
    {2304, 192, 1, 2, false}, {2592, 144, 1, 0, true}, {2916, 162, 1, 0, true}, {3456, 192, 1, 1, false},
    {4096, 256, 1, 2, false}, {4608, 288, 1, 1, false}, {5184, 192, 1, 1, false}, {6561, 243, 1, 0, false},
    {7776, 216, 1, 0, false}, {8192, 512, 1, 0, false}, {9216, 256, 1, 1, false}, {12288, 384, 1, 1, false},
    {15552, 648, 1, 0, false}};
constexpr ContigGeo kContig4[] = {   // 4-byte storage, FP32 values
    {2, 1, 256, 0, true},    {3, 1, 256, 0, true},    {6, 1, 64, 0, true},     {8, 1, 64, 0, true},
    {9, 1, 64, 0, true},     {12, 1, 64, 0, true},    {16, 1, 64, 0, true},    {18, 3, 42, 1, true},
    {24, 4, 16, 1, true},    {27, 1, 128, 0, true},   {32, 1, 64, 0, true},    {36, 3, 42, 0, true},
    {48, 4, 16, 0, true},    {54, 6, 42, 0, true},    {64, 8, 8, 0, true},     {72, 9, 7, 0, true},
    {81, 9, 28, 0, true},    {96, 8, 8, 0, true},     {108, 9, 14, 2, false},  {128, 8, 8, 2, false},
    {144, 12, 5, 0, true},   {162, 18, 14, 1, true},  {192, 16, 4, 0, true},   {216, 18, 7, 1, false},
    {243, 27, 18, 1, false}, {256, 16, 4, 2, false},  {288, 18, 7, 0, true},   {324, 18, 7, 0, true},
    {384, 16, 4, 1, false},  {432, 24, 10, 0, false}, {486, 54, 9, 1, false},  {576, 24, 10, 0, false},
    {648, 27, 9, 0, false},  {729, 81, 3, 1, false},  {768, 32, 2, 1, false},  {864, 32, 4, 0, false},
    {972, 81, 3, 2, false},  {1024, 32, 2, 0, false}, {2048, 128, 1, 2, false}};
constexpr ContigGeo kContig4m[] = {   // 4-byte storage, FP16 values
    {2, 1, 256, 0, true},    {3, 1, 256, 0, true},    {6, 1, 256, 0, true},    {8, 1, 128, 0, true},
    {9, 1, 64, 0, true},     {12, 1, 64, 0, true},    {16, 1, 64, 0, true},    {18, 1, 128, 0, true},
    {24, 2, 32, 1, true},    {27, 1, 64, 0, true},    {32, 4, 32, 1, true},    {36, 3, 21, 0, true},
    {48, 4, 16, 0, true},    {54, 6, 42, 0, true},    {64, 8, 16, 0, true},    {72, 4, 16, 0, true},
    {81, 9, 28, 0, true},    {96, 8, 8, 0, true},     {108, 12, 10, 0, true},  {128, 8, 32, 0, true},
    {144, 12, 10, 0, true},  {162, 9, 14, 0, true},   {192, 16, 8, 0, true},   {216, 12, 10, 0, true},
    {243, 9, 28, 0, true},   {256, 16, 16, 0, true},  {288, 18, 7, 0, true},   {324, 18, 7, 0, true},
    {384, 16, 4, 1, false},  {432, 24, 5, 0, true},   {486, 27, 18, 1, true},  {648, 36, 7, 1, true},
    {729, 81, 3, 1, false},  {768, 32, 2, 1, false},  {864, 32, 2, 0, false},  {1024, 32, 8, 0, false},
    {2048, 64, 1, 0, false}};

// Exchange rounds of the default contiguous complex64 kernel.  From 5184 points
// on a whole pencil's LDS (8 bytes a point and padding) lets one to three
// workgroups share a CU; where the registers would let more, and the kernel
// needs no more of them for it, the exchange runs in rounds of a part of the
// pencil.  GB/s, one round -> two: 5184 4601 -> 5415, 9216 4828 -> 5461, 10368
// 3755 -> 4508, 11664 3640 -> 4083, 12288 3788 -> 4396, 13122 3600 -> 3969 (1
// GiB), and three, 6561 being odd: 4158 -> 4517.  Where the registers hold as
// few workgroups as the LDS, rounds gain nothing or spend more registers: 7776
// 4073 -> 3604 (135 -> 174 VGPRs), 4374 4333 -> 4241 (256 MiB).  The
// half-spectrum passes need their whole pencil in LDS and keep the rules'
// geometry at these lengths.
constexpr int cfg_K_contig(int N, int bytes) {
    if (bytes == 8 && N == 6561) return 3;
    return bytes == 8 && (N == 5184 || N == 9216 || N == 10368 || N == 11664 || N == 12288 || N == 13122) ? 2 : 1;
}

// Geometry of the default contiguous kernel: the measured entry, else the rules.
constexpr ContigGeo cfg_contig(int N, int bytes, int vb) {
    if (bytes == 8) {
        for (const ContigGeo& g : kContig8)
            if (g.n == N) return g;
    } else if (vb == 8) {
        for (const ContigGeo& g : kContig4)
            if (g.n == N) return g;
    } else {
        for (const ContigGeo& g : kContig4m)
            if (g.n == N) return g;
    }
    const int plan = cfg_plan_contig(N, bytes);
    return {N, cfg_T_contig(N, plan), cfg_P_contig(N, plan, bytes, vb), plan, false};
}

// Longest pencil a single pass handles in each layout.
constexpr int kMaxContigN = 16384;   // one pencil of 16384 complex in LDS
constexpr int kMaxStridedN = 1024;

}  // namespace wsfft
