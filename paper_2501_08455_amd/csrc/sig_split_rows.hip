// Launch of the stream-mode kernel whose rows are split across workgroups (sig_split_rows.h): compiled shapes, which calls take
// it, and how a call is cut.  (Depth 2 has its own, in sig_depth2_rows.hip.)
#include "sig_split_rows.h"

namespace sig {
namespace split {

constexpr int kMostSegments = 32;
constexpr int64_t kMostPieces = (int64_t)1 << 27;   // floats of the pieces that the planner asks for

struct Shape {
    int d, depth, words;
    int64_t D;
    int (*lds_floats)(int threads);
    hipError_t (*launch)(const Args &, int threads, size_t lds, hipStream_t);
};

template <int d, int N>
hipError_t launch(const Args &A, int threads, size_t lds, hipStream_t st)
{
    if (A.segs > 1 && A.pieces) {
        hipLaunchKernelGGL((sig_split_rows_kernel<d, N, true>), dim3((unsigned)(A.B * (A.segs - 1) * A.slices)), dim3(threads), lds, st, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sig_split_rows_kernel<d, N, false>), dim3((unsigned)(A.B * A.segs * A.slices)), dim3(threads), lds, st, A);
    return hipGetLastError();
}

#define SIG_SPLIT_SHAPES(X) X(10, 3) X(8, 4) X(9, 4) X(10, 4) X(5, 5) X(6, 5) X(4, 6)
#define SIG_SPLIT_ENTRY(d, N) {d, N, Geo<d, N>::Q, Geo<d, N>::D, &lds_floats<d, N>, &launch<d, N>},
const Shape kShapes[] = {SIG_SPLIT_SHAPES(SIG_SPLIT_ENTRY){0, 0, 0, 0, nullptr, nullptr}};

const Shape *find(int d, int depth)
{
    for (const Shape *s = kShapes; s->launch; ++s)
        if (s->d == d && s->depth == depth) return s;
    return nullptr;
}

// The launch with W stretches a path (fewer where it is too short for that) and workgroups of at most `most` threads.  False where it
// would hold 2^32 threads.
struct Cut {
    Args args;
    int threads;
    size_t lds;
};
bool cut(const Shape &s, int64_t B, int64_t L, int W, int most, Cut *c)
{
    const int64_t K = L - 1;
    if (K > INT32_MAX - 2 * kTile) return false;
    Args &A = c->args;
    A = Args{};
    A.B = B;
    A.L = L;
    const int64_t rows = ((K + W - 1) / W + kTile - 1) / kTile * kTile;
    A.rows = (int32_t)rows;
    A.segs = (int32_t)((K + rows - 1) / rows);
    A.slices = (s.words + most - 1) / most;
    A.lanes = (s.words + A.slices - 1) / A.slices;
    c->threads = (A.lanes + kWave - 1) / kWave * kWave;
    c->lds = (size_t)s.lds_floats(c->threads) * sizeof(float);
    const int64_t all = ((int64_t)1 << 32) / ((int64_t)A.segs * A.slices * c->threads);
    return B < all && c->lds <= (size_t)kMaxLdsBytes;
}

// Microseconds, fitted to 4,800 calls of twelve shapes (4 to 2,001 points, 1 to 10,000 paths; 16 % off in the mean).  A step of a
// wavefront takes the same time whether one or four share a SIMD, and a unit holds sixteen; the pieces cost two fifths of the
// rows' steps, joining one 0.8 us.  The choice costs 1.024 times the best one in the mean: a whole path in lockstep in one
// workgroup writes its rows at the rate of a plain fill, but with few paths, or one more than the units hold at once, smaller ones
// lead ((9,4), 154 paths of 631 points 612 us with 256 threads and 536 with 768; (10,4), one of 1,423, in 16 stretches 79 and 124).
double microseconds(const Shape &s, int64_t B, int64_t L, int cus, const Cut &c)
{
    const Args &A = c.args;
    const int waves = c.threads / kWave, per_unit = waves < 16 ? 16 / waves : 1;
    const double work = 1.0 + 1.6 * s.d + 0.4 * s.depth * s.depth;
    const double rounds = (double)B * A.segs * A.slices / (cus * (double)per_unit);
    const double whole = (double)(int64_t)(rounds + 0.999999);
    double load = waves <= 4 ? 1.12 * rounds : rounds < 3.0 ? whole : rounds + 0.5;
    if (load < 1.0) load = 1.0;
    double us = 1.0 + A.rows * 0.0227 * work * load;
    const double bytes = (double)B * (double)(L - 1) * (double)s.D * sizeof(float) * 1e-6 / 5.2 * 256.0 / cus + 4.2;
    if (us < bytes) us = bytes;
    if (A.segs > 1) {
        const double pieces = (double)B * (A.segs - 1) * A.slices / (cus * (double)per_unit);
        const double busy = 0.74 * (pieces < 1.0 ? pieces : 1.0) * waves * per_unit / 4.0;
        us += 2.2 + A.rows * 0.0095 * work * (busy > 1.0 ? busy : 1.0) * (pieces > 1.0 ? pieces : 1.0) +
              (A.segs - 1) * 0.82 * (rounds > 2.0 ? 0.5 * rounds : 1.0);
    }
    return us;
}

// the faster workgroup size for W stretches a path
bool best_cut(const Shape &s, int64_t B, int64_t L, int W, int cus, Cut *best, double *us)
{
    bool found = false;
    for (int most = 256; most <= kMaxThreads; most *= 4) {
        Cut c;
        if (!cut(s, B, L, W, most, &c)) continue;
        const double t = microseconds(s, B, L, cus, c);
        if (found && t >= *us) continue;
        found = true;
        *best = c;
        *us = t;
    }
    return found;
}

}  // namespace split

// Which stream-mode calls take it.  `held_chunks`: of the register kernel that the planner would take, 0 for one launch per level;
// `held_rows`: the call would write its rows from registers by sig_stream_rows.h.  The shapes that kernel is not compiled for: every
// call (2,815 of 4 to 2,001 points and 1 to 10,000 paths: 1.7 (4,6) to 2.4 times (6,5) as fast in the mean, sixteen slower by up to
// 9 %).  (8,4): against the register kernel until its own rows fill the chip (1,000 paths of 120 points 443 us and 463, 130 of 60
// 2.6 times as fast), against the others from 160 increments on (55 of 1,379 491 and 340; 2 of 60 0.8 times as fast).  (10,3):
// against the register kernel with two and a half paths a unit (1,721 of 61 123 and 110, but 421 of 174 88 and 110).
int split_rows_wanted(int d, int depth, int64_t B, int64_t L, int cus, int held_chunks, bool held_rows)
{
    const bool registers = held_chunks > 0 && !held_rows;
    if (depth == 2) return depth2_rows_wanted(d, B, L, cus, registers ? held_chunks : 0);
    const split::Shape *s = split::find(d, depth);
    if (!s || B < 1 || L < 2) return 0;
    const int64_t K = L - 1;
    if (d == 10 && depth == 3 && (!registers || 2 * B < 5 * (int64_t)cus)) return 0;
    if (d == 8 && (registers ? B > 60000 * (int64_t)cus / 256 / K : K < 160)) return 0;
    int best = 0;
    double least = 0.0;
    for (int W = 1; W <= split::kMostSegments; W *= 2) {
        if (W > 1 && (K / W < split::kTile || B > 1500 * (int64_t)cus / 256 / W || B * (W - 1) * s->D > split::kMostPieces)) break;
        split::Cut c;
        double us = 0.0;
        if (!split::best_cut(*s, B, L, W, cus, &c, &us) || (best && us >= least)) continue;
        best = W;
        least = us;
    }
    return best;
}

bool split_rows_geometry(int d, int depth, int64_t B, int64_t L, int segs, int cus, bool registers, SplitRowsCut *cut)
{
    if (depth == 2) return depth2_rows_geometry(d, B, L, segs, cus, registers, cut);
    const split::Shape *s = split::find(d, depth);
    split::Cut c;
    double us = 0.0;
    if (!s || B < 1 || L < 2 || segs < 1 || segs > split::kMostSegments || segs > L - 1) return false;
    if (!split::best_cut(*s, B, L, segs, cus, &c, &us)) return false;
    const split::Args &A = c.args;
    *cut = SplitRowsCut{(int64_t)c.lds, B * A.segs * A.slices, B * (A.segs - 1) * s->D, c.threads, A.segs, A.rows, A.slices, A.lanes, 1, 1};
    return true;
}

hipError_t launch_split_rows(const float *path, float *out, float *scratch, int64_t B, int64_t L, int d, int depth, int segs, bool sticky,
                             bool registers, int cus, hipStream_t st)
{
    if (depth == 2) return launch_depth2_rows(path, out, B, L, d, segs, sticky, registers, cus, st);
    const split::Shape *s = split::find(d, depth);
    split::Cut c;
    double us = 0.0;
    if (!s || B < 1 || L < 2 || segs < 1 || segs > split::kMostSegments || segs > L - 1) return hipErrorInvalidValue;
    if (!split::best_cut(*s, B, L, segs, cus, &c, &us)) return hipErrorInvalidValue;
    c.args.path = path;
    c.args.out = out;
    c.args.pieces = scratch;
    c.args.sticky = sticky;
    return s->launch(c.args, c.threads, c.lds, st);
}

}  // namespace sig
