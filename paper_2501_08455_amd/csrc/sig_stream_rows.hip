// Launch of the stream-mode kernel that writes rows straight from registers (sig_stream_rows.h): compiled shapes, which calls
// take it, and how a call is cut.
#include "sig_stream_rows.h"

namespace sig {
namespace rows {

constexpr int kMostSegments = 32;
constexpr int kMostTileSteps = 256;
constexpr int kBlockSteps = 64;     // ... of what lies before: a block of its fold
constexpr int kLeastTileSteps = 24;

// What the rules below need to know of a compiled shape
struct Shape {
    int d, depth;
    int lanes, slots_per_wave, waves_per_slot;
    int64_t D;
    hipError_t (*launch)(const Args &, int threads, size_t lds, hipStream_t);

    int slots(int threads) const { return threads / kWave / waves_per_slot * slots_per_wave; }
    int threads(int slots) const { return (slots + slots_per_wave - 1) / slots_per_wave * waves_per_slot * kWave; }
};

template <int d, int N>
hipError_t launch(const Args &A, int threads, size_t lds, hipStream_t st)
{
    const dim3 grid((unsigned)((A.B + A.groups - 1) / A.groups * A.segs));
    if (A.steps > kPlainSteps) hipLaunchKernelGGL((sig_stream_rows_kernel<d, N, true>), grid, dim3(threads), lds, st, A);
    else hipLaunchKernelGGL((sig_stream_rows_kernel<d, N, false>), grid, dim3(threads), lds, st, A);
    return hipGetLastError();
}

// Eight lanes a slot and more: with fewer a step's row is a few scattered pieces per store ((2,3), (3,2), 64 paths of 256 points:
// 7.9 and 7.5 us against 7.0 and 6.3 for the register kernels).
#define SIG_ROWS_SHAPES(X)                                                                                              \
    X(8, 2) X(9, 2) X(10, 2) X(11, 2) X(12, 2) X(13, 2) X(14, 2) X(15, 2) X(16, 2) X(17, 2) X(18, 2) X(19, 2) X(20, 2)  \
    X(3, 3) X(4, 3) X(5, 3) X(6, 3) X(7, 3) X(8, 3) X(9, 3) X(10, 3) X(11, 3) X(12, 3)                                  \
    X(2, 4) X(3, 4) X(4, 4) X(5, 4) X(6, 4) X(7, 4) X(8, 4) X(2, 5) X(3, 5) X(4, 5) X(2, 6) X(3, 6)
#define SIG_ROWS_ENTRY(d, N) {d, N, Geo<d, N>::Q, Geo<d, N>::SPW, Geo<d, N>::WPS, Geo<d, N>::D, &launch<d, N>},
const Shape kShapes[] = {SIG_ROWS_SHAPES(SIG_ROWS_ENTRY){0, 0, 0, 0, 0, 0, nullptr}};

const Shape *find(int d, int depth)
{
    for (const Shape *s = kShapes; s->launch; ++s)
        if (s->d == d && s->depth == depth) return s;
    return nullptr;
}

int64_t lds_floats(const Shape &s, const Args &A) { return tile_floats(A, s.d) + (int64_t)A.groups * lds_rows(A.slots, A.segs) * lds_row(s.d, s.D); }

// wavefronts of a launch that does not cut the paths
int64_t uncut_waves(const Shape &s, int64_t B)
{
    return B > INT32_MAX ? INT32_MAX : (B + s.slots_per_wave - 1) / s.slots_per_wave * s.waves_per_slot;
}

// How a call is cut.  forced_segs > 0: into that many workgroups a path (the path's length may leave the last ones without steps:
// then fewer).  False if the launch would not fit the limits.
bool cut(const Shape &s, int64_t B, int64_t L, int forced_segs, int cus, Args *args, int *threads, size_t *lds)
{
    const int64_t K = L - 1;
    Args A{};
    A.B = B;
    A.L = L;
    // Pieces side by side: eight wavefronts hold them (four pieces at least, where sixteen do: (3,6), 64 paths of 256 points 32.0
    // with two and 30.6 us with four), a dozen steps each, and no more than give every SIMD four wavefronts.
    int most = s.slots(512);
    if (most < 4) most = s.slots(kMaxThreads) < 4 ? s.slots(kMaxThreads) : 4;
    int64_t C = (4 * 4 * (int64_t)cus + uncut_waves(s, B) - 1) / uncut_waves(s, B);
    if (C > most) C = most;
    if (C > K / 12) C = K / 12;
    if (C < 1) C = 1;
    for (;; --C) {   // rows that do not fit LDS: fewer pieces
        // a workgroup per compute unit, two steps a piece at least; short rows do not pay for a path's second workgroup, which
        // folds the first one's stretch again ((2,4), 64 paths of 256 points, one and four 7.8 and 9.6 us; (4,4), two and
        // four 12.8 and 12.1)
        int64_t W = forced_segs;
        if (W < 1) {
            W = cus / B;
            if (W > kMostSegments) W = kMostSegments;
            if (W > K / (2 * C)) W = K / (2 * C);
            if (W > (K / C * s.D + 1999) / 2000) W = (K / C * s.D + 1999) / 2000;
            if (W < 1) W = 1;
        }
        if (C * W > K) {
            if (C == 1) return false;
            continue;
        }
        const int64_t T = (K + C * W - 1) / (C * W);
        if (T > INT32_MAX) return false;
        A.slots = (int32_t)C;
        A.steps = (int32_t)T;
        A.segs = (int32_t)((K + C * T - 1) / (C * T));
        *threads = s.threads((int)C);
        // whole paths side by side in 256 threads once there are more than the chip has wavefronts for
        A.groups = 1;
        if (A.segs == 1 && B > 4 * (int64_t)cus && s.slots(256) / C > 1) {
            A.groups = (int32_t)(s.slots(256) / C);
            *threads = s.threads((int)(A.groups * C));
        }
        const int64_t room = kMaxLdsBytes / (int64_t)sizeof(float) - A.groups * lds_rows((int)C, A.segs) * lds_row(s.d, s.D);
        const int64_t behind = (int64_t)(A.segs - 1) * T;
        const int64_t fit = (room / (A.segs > 1 ? 2 : 1) / (A.groups * C) - 1) / s.d - level1_from_points(s.d);
        // tiles of less than two dozen steps cost more than the pieces they make room for
        const int64_t wanted = T > behind ? T : behind;
        if (fit < (wanted < kLeastTileSteps ? wanted : kLeastTileSteps)) {
            if (C == 1) return false;
            continue;
        }
        const int64_t cap = fit < kMostTileSteps ? fit : kMostTileSteps;
        A.tile = (int32_t)(T < cap ? T : cap);
        A.behind = (int32_t)(behind < 1 ? 1 : behind < cap && behind < kBlockSteps ? behind : cap < kBlockSteps ? cap : kBlockSteps);
        break;
    }
    *lds = (size_t)lds_floats(s, A) * sizeof(float);
    const int64_t grid = (B + A.groups - 1) / A.groups * A.segs;
    if (*lds > (size_t)kMaxLdsBytes || grid > INT32_MAX || grid >= ((int64_t)1 << 32) / *threads) return false;
    *args = A;
    return true;
}

}  // namespace rows

// Which stream-mode calls take it.  `held_p`: prefix depth of the register kernel for stream mode that the planner would take, -1 if
// it would take one launch per level.  Microseconds without and with it in brackets.
//  - Against the launches per level: everywhere but on a few paths of hundreds of points whose rows take long to store while the joins
//    stride LDS by a multiple of four [(12,3), one of 488 points 44 and 52; (8,4), four of 470 0.88x, two of 1,415 122 and 191; (7,4), one of 1,356
//    0.86x, but of 1,614 1.48x, (9,3) two of 1,180 124 and 40, (20,2) two of 3,000 1.4x], and, at depth 2 (two launches), on few paths that those
//    launches still hold in one tile, 512 increments [(20,2), two of 490 21 and 28; (17,2), two of 405 19 and 22; (16,2), whose lanes
//    stride LDS by 16, ten of 230 16 and 20].
//  - Against the register kernels, whose rows stop in LDS and reach memory in longer runs: batches that leave the chip below a
//    wavefront per SIMD uncut and rows of some hundred megabytes at most [(4,4), 1,024 paths of 256 points 93 and 79, 4,096 284 and
//    295; (3,5), 500 of 1,000 173 and 275].  At depth 3 the crossing lies lower [(5,3), 1,000 of 100 17.6 and 18.7;
//    (8,3), 600 of 64 20.4 and 22.9; (9,3), 400 of 60 0.97x, but (10,3) 1.02 to 1.06x], and slots of fewer than 16 lanes, whose stores are
//    short pieces, pay for short paths or few [(3,3), 500 of 1,000 points 23 and 34, of 12 5.3 and 3.8; 100 of 64 ... 180 0.97x].  Register
//    kernels with the same lanes (a word of length N - 1 each) in several wavefronts a path lose only where the paths are cut
//    [(6,4), 200 of 73 19.5 and 24.7, of 8 0.97x; 30 of 200 48 and 24], those with fewer lanes than that where a path has two
//    wavefronts and rows of some hundred floats here [(5,4), more than 170 of 128 points and more 0.91 to 1.01x].
int stream_rows_wanted(int d, int depth, int64_t B, int64_t L, int cus, int held_p)
{
    const rows::Shape *s = rows::find(d, depth);
    if (!s || B < 1 || L < 2) return 0;
    const int64_t K = L - 1;
    rows::Args A{};
    int threads = 0;
    size_t lds = 0;
    if (held_p >= 0) {
        if (rows::uncut_waves(*s, B) > 4 * (int64_t)cus) return 0;
        const double bytes = 4.0 * (double)B * (double)K * (double)s->D;
        if (bytes > (s->waves_per_slot > 1 ? 2e8 : 4e8)) return 0;
        if (depth == 3 && B > cus && B * K > (s->lanes >= 64 && s->lanes < 100 ? 10000 : 50000)) return 0;
        if (s->lanes < 16 && B > (K > 32 ? 1 : 4) * (int64_t)cus) return 0;
        if (s->lanes < 9 && K > 32 && (K < 500 || B > cus / 2)) return 0;
        if (depth == 3 && s->lanes < 10 && K > 60 && K < 180) return 0;
        if (held_p < depth - 1 && s->waves_per_slot == 2 && s->D > 700 && 3 * B > 2 * (int64_t)cus) return 0;
        if (held_p == depth - 1 && s->lanes > 128 && (B >= cus / 2 || K < 16)) return 0;
    }
    if (!rows::cut(*s, B, L, 0, cus, &A, &threads, &lds)) return 0;
    if (held_p < 0) {
        const bool one_tile = K < 512;
        if (B < 5 && s->D > 4000 && K / A.slots > 250) return 0;
        if (B < 3 && s->D > 2500 && K > 1000 && K < 1536) return 0;
        if (depth == 2 && one_tile && (d % 16 ? d > 13 && B < 16 && K * d * d * d > 900000 : K > 110 && (B < 32 || (B < 64 && K < 250)))) return 0;
        if (depth > 2 && d % 4 == 0 && s->D > 1800 && (one_tile ? B < 3 + s->D / 2000 && K > 380 : B < 3 && K > 590 && K < 1024)) return 0;
    }
    return A.segs;
}

int stream_rows_segments(int d, int depth, int64_t B, int64_t L, int cus)
{
    const rows::Shape *s = rows::find(d, depth);
    rows::Args A{};
    int threads = 0;
    size_t lds = 0;
    return s && B >= 1 && L >= 2 && rows::cut(*s, B, L, 0, cus, &A, &threads, &lds) ? A.segs : 0;
}

bool stream_rows_geometry(int d, int depth, int64_t B, int64_t L, int segs, int cus, int64_t *lds_bytes, int64_t *workgroups, int *threads)
{
    const rows::Shape *s = rows::find(d, depth);
    rows::Args A{};
    size_t lds = 0;
    if (!s || B < 1 || L < 2 || segs < 1 || segs > rows::kMostSegments || segs > L - 1) return false;
    if (!rows::cut(*s, B, L, segs, cus, &A, threads, &lds)) return false;
    *lds_bytes = (int64_t)lds;
    *workgroups = (B + A.groups - 1) / A.groups * A.segs;
    return true;
}

hipError_t launch_stream_rows(const float *path, float *out, int64_t B, int64_t L, int d, int depth, int segs, int cus, hipStream_t st)
{
    const rows::Shape *s = rows::find(d, depth);
    rows::Args A{};
    int threads = 0;
    size_t lds = 0;
    if (!s || B < 1 || L < 2 || segs < 1 || segs > rows::kMostSegments || segs > L - 1) return hipErrorInvalidValue;
    if (!rows::cut(*s, B, L, segs, cus, &A, &threads, &lds)) return hipErrorInvalidValue;
    A.path = path;
    A.out = out;
    return s->launch(A, threads, lds, st);
}

}  // namespace sig
