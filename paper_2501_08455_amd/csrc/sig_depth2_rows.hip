// Every-prefix signature at depth 2 (stream mode; two to twenty channels).
//
// With S1_k = X_k - X_0 the second level is a plain sum over the steps,
//     S2_{k+1}[ab] = S2_k[ab] + (S1_k[a] + v[a] / 2) v[b],     v = X_{k+1} - X_k,
// so that a path can be cut anywhere and the parts need nothing of each other but a sum of d * d floats.
//
// Lanes.  Lane a of d holds row a of S2; a wavefront keeps 64 / d slots and stages R rows of each in LDS, as they lie in memory, which
// then go out in runs of R d (d + 1) floats.  Whole paths side by side (UNCUT), or stretches of a path side by side in a workgroup
// (CUT): each slot sums its steps, a scan in LDS adds what lies before, and the rows are written on a second walk; reading the path
// twice costs next to nothing beside its rows.  Few paths also span W workgroups, each of which sums all that lies before its own
// rows; no workgroup waits for another.
//
// Bound by the stores where the batch fills the chip: the rows are written once (1.00 to 1.05 times their bytes by the counters) at 4.1 to 4.5 MB a
// us of all that moves, the wavefronts wait for memory half of their time and more, the LDS is busy a third (a third of that conflicts).  Else by
// one wave's steps.  Tiles: 6,400 floats a wavefront whole (longer runs; five or six wavefronts a unit hold the rows
// of the others' stores), 1,600 cut (sixteen wavefronts, whose scans overlap; twelve with more points in LDS, see cut()).  Before (one launch
// per level, or register kernels) and now, us, one MI355X, both in turn: (20,2) 1,177 paths of 1,386 points 1,315 and 708, (2,2) 20,000
// of 500 180 and 117, (12,2) 1,024 of 100 26.8 and 20.8.
//
// Rounding: the steps of a tile are summed from zero and what their addition to the sum rounds off goes into the next tile's; level 1
// is the distance between two points.  Error against 64 bits 0.2 to 1.0 times that of the kernels that took these calls (14,300 calls;
// without the carried part 1.1 to 1.5 times where few paths span workgroups).
#include <cmath>
#include <type_traits>

#include "sig_internal.h"

namespace sig {
namespace depth2_rows {

typedef float vec4f_u __attribute__((ext_vector_type(4), aligned(4)));

struct Args {
    const float *path;   // [B][L][d]
    float *out;          // [B][K][d + d * d]
    int64_t B;
    int32_t L;
    int32_t chunks;      // C: stretches of a path side by side in a workgroup
    int32_t segs;        // W: workgroups of a path
    int32_t groups;      // paths in a workgroup
    int32_t steps;       // T: steps of a stretch; W * C * T >= K
    int32_t sticky;      // a point that is not a number spoils level 1 of the rows behind it too
};

enum Mode { UNCUT, CUT, LONG };      // LONG: CUT with the points of eight rows' steps staged together
constexpr int kLongChannels = 14;    // the least that LONG is compiled for (one row a tile)

constexpr int threads_of(int mode) { return mode == UNCUT ? kWave : 4 * kWave; }
constexpr int slots_of(int mode, int d) { return threads_of(mode) / kWave * (kWave / d); }
constexpr int tile_rows(int mode, int d)
{
    const int fit = (mode == UNCUT ? 6400 : 1600) / (kWave / d * (d + d * d));
    return fit < 1 ? 1 : fit > 16 ? 16 : fit;
}

template <int d, int MODE>
struct Tile {
    static constexpr int D = d + d * d, SLOTS = kWave / d, R = tile_rows(MODE, d);
    static constexpr int VECS = (R * D + 3) / 4, NV = (SLOTS * VECS + kWave - 1) / kWave;
    static constexpr int P = MODE == LONG ? 8 * R : R;     // steps whose points are staged together
    static constexpr int PX = (P + 1) * d, NX = (SLOTS * PX + kWave - 1) / kWave;
    // (slots begin some d banks apart, and at whole vectors)
    static constexpr int STRIDE = VECS * 4 + ((d + 3) / 4 * 4 + 64 - VECS * 4 % 32) % 32;
    static constexpr int XS = (d + 3) / 4 * 4;
    static constexpr int FLOATS = SLOTS * (STRIDE + (P + 1) * XS);
    static constexpr int M = d * d + d;               // a slot's sums
    static constexpr int LDS = threads_of(MODE) / kWave * FLOATS + (MODE == UNCUT ? 0 : (slots_of(MODE, d) + 1) * M);
};

extern __shared__ __align__(16) float sig_depth2_rows_smem[];

// sum += part; what that rounded off is left in `part` (infinities and NaN leave nothing)
__device__ __forceinline__ void carry(float &sum, float &part)
{
    const float to = sum + part, off = part - (to - sum);
    sum = to;
    part = fabsf(off) < __builtin_huge_valf() ? off : 0.0f;
}

__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int d, int MODE>
__global__ __launch_bounds__(threads_of(MODE)) __attribute__((amdgpu_waves_per_eu(MODE == LONG ? 3 : 2))) void sig_depth2_rows_kernel(Args A)
{
    using Tl = Tile<d, MODE>;
    constexpr int NT = threads_of(MODE), WSLOTS = Tl::SLOTS, M = Tl::M, D = Tl::D, R = Tl::R, P = Tl::P, XS = Tl::XS;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int K = A.L - 1;
    const int C = MODE == UNCUT ? 1 : A.chunks, W = MODE == UNCUT ? 1 : A.segs, T = MODE == UNCUT ? K : A.steps;
    const int64_t b0 = W > 1 ? blockIdx.x / W : (int64_t)blockIdx.x * A.groups;
    const int k0 = W > 1 ? (int)(blockIdx.x - b0 * W) * C * T : 0;       // first step of the workgroup
    const int npaths = W > 1 ? 1 : A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;
    const int wslot = lane / d, a = lane - wslot * d;
    const int slot = wave * WSLOTS + wslot;
    const int group = slot / C, chunk = slot - group * C;
    const bool active = wslot < WSLOTS && group < npaths;
    const int mine = active ? group : 0;
    const float *points = A.path + b0 * A.L * d;
    float *rows = A.out + b0 * K * D;
    const int last = npaths * A.L * d - 1;            // of the workgroup's points

    float *otile = sig_depth2_rows_smem + wave * Tl::FLOATS, *xtile = otile + WSLOTS * Tl::STRIDE;
    float *myo = otile + (active ? wslot : 0) * Tl::STRIDE;
    const float *myx = xtile + (active ? wslot : 0) * (P + 1) * XS;
    float *sums = sig_depth2_rows_smem + NT / kWave * Tl::FLOATS, *base = sums + NT / kWave * WSLOTS * M;

    // the points around the P steps from `step` on of every slot of the wavefront (beyond the path's end: floats that nothing uses)
    float xv[Tl::NX];
    auto fetch = [&](int step) __attribute__((always_inline)) {
        const int point = mine * A.L + (step < K ? step : K);
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::PX, x = i - ws * Tl::PX;
            const int at = __shfl(point, ws * d) * d + x;
            xv[j] = points[at < last ? at : last];
        }
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::PX, x = i - ws * Tl::PX;
            if (ws < WSLOTS) xtile[(ws * (P + 1) + x / d) * XS + x % d] = xv[j];
        }
    };

    const float first = points[(int64_t)mine * A.L * d + a];
    float s2[d];             // row a of S2 before the steps in `sum`
    float spoilt = 0.0f;     // not a number behind a point that is none (sticky; infinite points too, but the first: the distance from that stays infinite)
#pragma unroll
    for (int b = 0; b < d; ++b) s2[b] = 0.0f;
    // `count` steps of every slot from `from` on, those below `to`; EMIT: and their rows
    // (held: the only tile's points are in LDS already)
    auto walk = [&](int from, int to, int count, bool held, auto emit) __attribute__((always_inline)) {
        constexpr bool EMIT = decltype(emit)::value;
        if (!held) fetch(from);
        float sum[d];
#pragma unroll
        for (int b = 0; b < d; ++b) sum[b] = 0.0f;
        constexpr int S = EMIT ? R : P, TILES = (16 + S - 1) / S;      // steps of a round; rounds whose steps are summed from zero
        float before[XS], here = 0.0f;
        for (int t0 = 0; t0 < count; t0 += S) {
            const int in = P == S ? 0 : t0 % P;       // of the points' tile
            wave_sync();
            if (in == 0) {
                if (!held) put();
                wave_sync();
                if (count - t0 > P) fetch(from + t0 + P);
            }
            const int left = to - from - t0, own = count - t0 < S ? count - t0 : S;
            const int n = !active || left < 1 ? 0 : left < own ? left : own;     // of the slot's steps in this tile
            if (in == 0) {
#pragma unroll
                for (int b = 0; b < XS; b += 4) {
                    const float4 v = *reinterpret_cast<const float4 *>(myx + b);
                    before[b] = v.x; before[b + 1] = v.y; before[b + 2] = v.z; before[b + 3] = v.w;
                }
                here = myx[a];
            }
#pragma unroll 2
            for (int r = 0; r < n; ++r) {
                const float *x = myx + (in + r + 1) * XS;
                float at[XS];
#pragma unroll
                for (int b = 0; b < XS; b += 4) {
                    const float4 v = *reinterpret_cast<const float4 *>(x + b);
                    at[b] = v.x; at[b + 1] = v.y; at[b + 2] = v.z; at[b + 3] = v.w;
                }
                const float next = x[a], va = next - here;
                const float h = fmaf(0.5f, va, here - first + spoilt);
#pragma unroll
                for (int b = 0; b < d; ++b) sum[b] = fmaf(h, at[b] - before[b], sum[b]);
                if constexpr (EMIT) {
                    float *o = myo + r * D;
                    o[a] = next - first + spoilt;
                    constexpr int V = d % 4 == 0 ? 4 : d % 2 == 0 ? 2 : 1;
                    typedef float vec __attribute__((ext_vector_type(V)));
#pragma unroll
                    for (int b = 0; b < d; b += V) {
                        vec v;
#pragma unroll
                        for (int e = 0; e < V; ++e) v[e] = s2[b + e] + sum[b + e];
                        *reinterpret_cast<vec *>(o + d + a * d + b) = v;
                    }
                }
                if (A.sticky) spoilt = fmaf(0.0f, next, spoilt);
                here = next;
#pragma unroll
                for (int b = 0; b < XS; ++b) before[b] = at[b];
            }
            if ((t0 / S + 1) % TILES == 0 || count - t0 <= S) {
#pragma unroll
                for (int b = 0; b < d; ++b) carry(s2[b], sum[b]);
            }
            if constexpr (EMIT) {
                wave_sync();
                const int row = mine * K + from + t0, have = n * D;
#pragma unroll
                for (int j = 0; j < Tl::NV; ++j) {
                    const int i = lane + j * kWave, ws = i / Tl::VECS, at = 4 * (i - ws * Tl::VECS);
                    const int to_row = __shfl(row, ws * d), theirs = __shfl(have, ws * d), floats = ws < WSLOTS ? theirs : 0;   // (all lanes take part)
                    const float *src = otile + (ws < WSLOTS ? ws : 0) * Tl::STRIDE + at;
                    const float4 v = *reinterpret_cast<const float4 *>(src);
                    float *dst = rows + (int64_t)to_row * D + at;
                    if (at + 4 <= floats) *reinterpret_cast<vec4f_u *>(dst) = vec4f_u{v.x, v.y, v.z, v.w};
                    else if (at < floats) {
                        dst[0] = v.x;
                        if (at + 1 < floats) dst[1] = v.y;
                        if (at + 2 < floats) dst[2] = v.z;
                    }
                }
            }
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    if constexpr (MODE == UNCUT) {
        walk(0, K, K, false, yes);
    } else {
        // a slot's sums into LDS, and from each path's the sums of what lies before its slots
        auto leave = [&]() __attribute__((always_inline)) {
            if (active) {
#pragma unroll
                for (int b = 0; b < d; ++b) sums[slot * M + a * d + b] = s2[b];
                sums[slot * M + d * d + a] = spoilt;
            }
            __syncthreads();
        };
        auto clear = [&]() __attribute__((always_inline)) {
#pragma unroll
            for (int b = 0; b < d; ++b) s2[b] = 0.0f;
            spoilt = 0.0f;
        };
        for (int e = tid; e < M; e += NT) base[e] = 0.0f;
        if (k0 > 0) {
            const int count = (k0 + C - 1) / C;
            walk(chunk * count, k0, count, false, no);
            leave();
            for (int e = tid; e < M; e += NT) {
                float sum = 0.0f, off = 0.0f;
#pragma unroll 4
                for (int c = 0; c < C; ++c) {
                    off += sums[c * M + e];
                    carry(sum, off);
                }
                base[e] = sum;
            }
            clear();
        }
        const int from = k0 + chunk * T;
        __syncthreads();                              // (base is written, sums are read)
        if (C > 1) walk(from, K, T, false, no);
        leave();
        for (int i = tid; i < npaths * M; i += NT) {
            const int g = i / M, e = i - g * M;
            float *s = sums + g * C * M + e;
            float sum = W > 1 ? base[e] : 0.0f, off = 0.0f;
#pragma unroll 4
            for (int c = 0; c < C; ++c) {
                off += s[c * M];
                s[c * M] = sum;
                carry(sum, off);
            }
        }
        __syncthreads();
        clear();
        if (active) {
#pragma unroll
            for (int b = 0; b < d; ++b) s2[b] = sums[slot * M + a * d + b];
            spoilt = sums[slot * M + d * d + a];
        }
        walk(from, K, T, C > 1 && T <= P, yes);
    }
}

struct Cut {
    int mode, chunks, segs, groups, steps;
    int64_t grid;
};

template <int d>
size_t lds_bytes(int mode)
{
    return (size_t)(mode == UNCUT ? Tile<d, UNCUT>::LDS : mode == LONG ? Tile<d, LONG>::LDS : Tile<d, CUT>::LDS) * sizeof(float);
}

template <int d>
hipError_t launch(const Args &A0, const Cut &c, hipStream_t st)
{
    Args A = A0;
    A.chunks = c.chunks;
    A.segs = c.segs;
    A.groups = c.groups;
    A.steps = c.steps;
    static_assert(Tile<d, CUT>::LDS * sizeof(float) <= (size_t)kMaxLdsBytes, "the tiles and sums of a workgroup's slots fit its LDS");
    static_assert(d < kLongChannels || Tile<d, LONG>::LDS * sizeof(float) <= (size_t)kMaxLdsBytes, "these too");
    const dim3 grid((unsigned)c.grid), threads(threads_of(c.mode));
    if (c.mode == UNCUT) hipLaunchKernelGGL((sig_depth2_rows_kernel<d, UNCUT>), grid, threads, lds_bytes<d>(UNCUT), st, A);
    else if (c.mode == CUT) hipLaunchKernelGGL((sig_depth2_rows_kernel<d, CUT>), grid, threads, lds_bytes<d>(CUT), st, A);
    else if constexpr (d >= kLongChannels) hipLaunchKernelGGL((sig_depth2_rows_kernel<d, LONG>), grid, threads, lds_bytes<d>(LONG), st, A);
    return hipGetLastError();
}

struct Shape {
    size_t (*lds)(int mode);
    hipError_t (*launch)(const Args &, const Cut &, hipStream_t);
};
#define SIG_DEPTH2_CHANNELS(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)
#define SIG_DEPTH2_ENTRY(d) {&lds_bytes<d>, &launch<d>},
constexpr int kLeastChannels = 2, kMostChannels = 20;
const Shape kShapes[] = {SIG_DEPTH2_CHANNELS(SIG_DEPTH2_ENTRY)};
static_assert(sizeof(kShapes) / sizeof(kShapes[0]) == kMostChannels - kLeastChannels + 1, "one entry a channel count");

constexpr int kMostSegments = 32;
constexpr int kShortSteps = 31;      // fewer steps are not cut

// W == 0: UNCUT; else W workgroups a path and at most `most_chunks` stretches side by side in each.  False where it would hold 2^32
// threads, or a workgroup's rows 2^31 floats.
bool cut(int d, int64_t B, int64_t L, int64_t W, int64_t most_chunks, int cus, Cut *c)
{
    const int64_t K = L - 1, D = d + d * d, slots = slots_of(W > 0 ? CUT : UNCUT, d);
    c->mode = W > 0 ? CUT : UNCUT;
    c->chunks = c->segs = 1;
    if (L > INT32_MAX / (slots * D)) return false;
    c->steps = (int)K;
    c->groups = (int)slots;
    if (W > 0) {
        const int64_t rows = (K + W - 1) / W;
        int64_t C = rows < slots ? rows : slots;
        if (C > most_chunks) C = most_chunks;
        const int64_t T = (rows + C - 1) / C;
        c->chunks = (int)C;
        c->steps = (int)T;
        c->segs = (int)((K + C * T - 1) / (C * T));
        c->groups = c->segs > 1 ? 1 : (int)(slots / C);
    }
    const int64_t most = (((int64_t)1 << 32) - 1) / threads_of(c->mode);
    if (B > most / c->segs * c->groups) return false;
    c->grid = c->segs > 1 ? B * c->segs : (B + c->groups - 1) / c->groups;
    // A tile's points arrive only once the stores before them are through: eight steps' at a time where a stretch has four or more,
    // unless that leaves a round of workgroups (four a unit) more than the chip then holds (three).  Before and with
    // it, us, the same bits: (15,2) 1,493 paths of 1,885 points 1,060 and 696, (18,2) 15 of 1,481 56.4 and 37.1, (20,2) 1,177 of 1,386 971 and 708; none of
    // 2,000 calls slower by more than 4 %.  Stretches of two or three steps are up to a quarter slower with it, and eight to thirteen
    // channels, which stage two and three rows, gain 1.1 to 1.2 on long ones and lose as much on the others.
    if (W > 0 && d >= kLongChannels && c->steps >= 4 && (c->grid <= 3 * (int64_t)cus || c->grid > 4 * (int64_t)cus)) c->mode = LONG;
    return true;
}

// Microseconds, fitted to 20,300 calls (2 to 20 channels, 4 to 2,000 points, 1 to 60,000 paths) with all their cuts, 107,000 launches: 7 (whole paths)
// and 9 % off in the mean.  The workgroups' rounds, and the bytes: within 240 MB the last-level cache takes the stores of whole paths as fast as
// they come; beyond, several paths cut side by side in a workgroup cost the memory a third.  The choice costs 1.014 times the best cut in the mean (1.037
// before it knew of rounds: 1,445 workgroups of whole paths where the chip holds 1,280, 14,441 paths of 79 points of six channels, were
// priced as many of a larger batch, 68 us, the best cut 54).
double microseconds(int d, int64_t B, int64_t L, int cus, const Cut &c)
{
    const double K = (double)(L - 1), mb = (double)B * K * (d + d * d) * 4e-6, cache = 240.0, chip = cus / 256.0;
    const int by_lds = held_by_lds(kShapes[d - kLeastChannels].lds(c.mode)), held = c.mode != UNCUT && by_lds > 4 ? 4 : by_lds;   // (four by their registers)
    const double load = rounds_of(c.grid, cus, held, c.mode == UNCUT ? 0.110 : 0.166);
    if (c.mode == UNCUT) {
        const double work = 4.14 + 0.1152 * (1.0 + 0.26 * d) * K * load, bytes = mb / (mb > cache ? 3.95 : 9.61) / chip;
        return std::sqrt(std::sqrt(work * work * work * work + bytes * bytes * bytes * bytes));
    }
    const double step = 1.0 + 0.0973 * d, before = (double)(c.segs - 1) * c.steps;
    const int R = tile_rows(c.mode, d);
    const double tiles = c.mode == LONG ? 4.01 * ((c.steps + 7) / 8) - 0.88 : 0.829 * ((c.steps + R - 1) / R);
    const double work = 1.81 + load * (0.217 * step * c.steps + tiles + 0.58 + 0.0356 * c.chunks + 0.0913 * step * before);
    const double bytes = 2.64 + ((mb < cache ? mb : cache) / 5.26 + (mb > cache ? mb - cache : 0.0) / 3.0 * (c.groups > 1 ? 1.3 : 1.0)) / chip;
    // (beyond the cache a path to each workgroup unless several are clearly faster: their stores lie closer together)
    return std::sqrt(work * work + bytes * bytes) * (c.groups > 1 && mb > cache ? 1.05 : 1.0) + (c.segs > 1 ? 1.18 : 0.0);
}

// Where the register kernels are the alternative, whole paths of five, six and eight channels lead from a hundred increments on (0.7 to 1.1 times as
// fast before: rows that the last-level cache takes as fast as a register kernel writes them), and stretches side by side in a workgroup
// never with up to four channels and seven (0.8 to 1.1).
constexpr int kLeastSteps = 47;      // fewer stay with the register kernels
bool leads(int d, int64_t K, const Cut &c)
{
    if (c.mode == UNCUT) return (d != 5 && d != 6 && d != 8) || K >= 100;
    return c.segs > 1 || (d > 4 && d != 7);
}

// The fastest launch with `segs` workgroups a path (1: or less than one).  registers: of those that lead on the register kernels, where any do.
// of_all: is lowered to the least time of all of them.
bool choose(int d, int64_t B, int64_t L, int segs, int cus, bool registers, Cut *best, double *least, double *of_all = nullptr)
{
    const int64_t K = L - 1;
    const bool leading = registers && d <= 10 && K >= kLeastSteps;
    bool found = false, behind = true;      // behind: none that leads so far
    auto take = [&](int W, int most_chunks) {
        Cut c;
        if (!cut(d, B, L, W, most_chunks, cus, &c)) return;
        const bool leads_here = !leading || leads(d, K, c);
        if (!leads_here && !behind && !of_all) return;
        const double us = microseconds(d, B, L, cus, c);
        if (of_all && us < *of_all) *of_all = us;
        if (leads_here ? !behind && us >= *least : !behind || (found && us >= *least)) return;
        found = true;
        behind = !leads_here;
        *best = c;
        *least = us;
    };
    const int slots = slots_of(CUT, d);
    if (segs > 1) take(segs, slots);
    else {
        take(0, 1);
        if (K >= kShortSteps) {
            take(1, slots);
            for (int C = 32; C >= 8; C /= 2)
                if (C < slots) take(1, C);
        }
    }
    return found;
}

}  // namespace depth2_rows

// Which calls take it.  Shorter calls: the same launch count and more work to begin with.  More than ten channels, against
// one launch per level and sig_stream_rows.h: 1.37 to 1.54 times as fast, and from 4 steps on where the rows exceed 64 MB.
// Up to ten channels against sig_stream_rows.h: 1.2 (ten) to 1.8 times (eight).  Against the register kernels (chunks: of their plan, 0
// where the call would not take them) by what leads there (see leads()): 1.31 times as fast in the mean over 6,700 calls of four to ten
// channels, two thirds of them from the bands where the two lie close, 100 slower by more than a twentieth (0.82 at worst).  Not taken: short paths
// that a register kernel walks whole, in one pass ((8,2), 20,000 paths of 60 points 92 us and 104); few paths (the launch decides); four
// channels across workgroups under 600 increments (1,000 from a quarter of the units' number of paths on); six side by side in batches that keep the chip busy (5,000 to 20,000 paths of 50 to 190 points
// 0.8 to 1.1); up to four channels and seven where the cuts that do not lead are the faster ones by the
// model (on long paths by a tenth and a quarter: there whole paths lead by more than the model is off).
int depth2_rows_wanted(int d, int64_t B, int64_t L, int cus, int chunks)
{
    using namespace depth2_rows;
    if (d < kLeastChannels || d > kMostChannels || B < 1 || L < 2) return 0;
    const int64_t K = L - 1;
    const double mb = (double)B * K * (d + d * d) * 4e-6;
    const bool registers = chunks > 0;
    if (d > 10 ? K < kShortSteps && (K < 4 || mb < 64.0) : registers ? K < kLeastSteps || (d <= 3 && mb < 4.0) : K < kShortSteps) return 0;
    const bool narrow = registers && (d <= 4 || d == 7);
    Cut best;
    int W = 0;
    double least = 0.0, least_of_all = HUGE_VAL;
    for (int segs = 1; segs <= kMostSegments; segs *= 2) {
        if (segs > 1 && (K < kShortSteps || K / segs < 2 || B > 600 * (int64_t)cus / 256 / segs)) break;
        Cut c;
        double us = 0.0;
        if (!choose(d, B, L, segs, cus, registers, &c, &us, narrow ? &least_of_all : nullptr) || (W && us >= least)) continue;
        if (narrow && segs > 1 && (d <= 3 || (d == 4 && K < (B > cus / 4 ? 1000 : 600)))) continue;
        best = c;
        W = segs;
        least = us;
    }
    if (W == 0 || d > 10 || !registers) return W;
    if (narrow) return least <= (best.segs > 1 || K < 100 ? 1.0 : K < 300 ? 1.1 : 1.25) * least_of_all ? W : 0;
    if ((d == 5 || d == 6 || d == 8) && K < 100 && chunks == 1) return 0;
    if (best.mode != UNCUT && best.segs == 1 && ((B < 16 && K < 200) || (d == 6 && K < 190 && B > 5000 * (int64_t)cus / 256))) return 0;
    return W;
}

bool depth2_rows_geometry(int d, int64_t B, int64_t L, int segs, int cus, bool registers, SplitRowsCut *cut)
{
    using namespace depth2_rows;
    Cut c;
    double us = 0.0;
    if (d < kLeastChannels || d > kMostChannels || B < 1 || L < 2 || segs < 1 || segs > kMostSegments || segs > L - 1) return false;
    if (!choose(d, B, L, segs, cus, registers, &c, &us)) return false;
    *cut = SplitRowsCut{(int64_t)kShapes[d - kLeastChannels].lds(c.mode), c.grid, 0, threads_of(c.mode), c.segs,
                        (int64_t)c.chunks * c.steps, 1, slots_of(c.mode, d), c.chunks, c.groups};
    return true;
}

hipError_t launch_depth2_rows(const float *path, float *out, int64_t B, int64_t L, int d, int segs, bool sticky, bool registers, int cus, hipStream_t st)
{
    using namespace depth2_rows;
    Cut c;
    double us = 0.0;
    if (B == 0) return hipSuccess;
    if (d < kLeastChannels || d > kMostChannels || !choose(d, B, L, segs, cus, registers, &c, &us)) return hipErrorInvalidValue;
    Args A{};
    A.path = path;
    A.out = out;
    A.B = B;
    A.L = (int32_t)L;
    A.sticky = sticky;
    return kShapes[d - kLeastChannels].launch(A, c, st);
}

}  // namespace sig
