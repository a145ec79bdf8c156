// Stream mode, rows written straight from registers and few paths cut across workgroups (compiled per (d, depth N)).
//
// A slot of Q = d^{N-1} lanes folds a piece of a path with the fused step of sig_onchip.h at prefix depth N - 1: a lane owns
// one word of length N - 1 and its d children.  Consecutive lanes then hold consecutive floats of a row's two longest
// levels, so that a step's row goes from the registers to memory in whole runs, without a stop in LDS.
//
// Workgroup w of the W that share a path emits the C * T rows from step w C T on, a slot T of them.  What lies before is not
// handed over by other workgroups (that would take a second launch): every workgroup folds it again, w T steps a slot, side by
// side in its C slots, and joins the pieces by a tree of Eq. 4 products in LDS while the slots' own pieces go through a scan.
//
// Bound by latency on few paths (a launch, K / C steps of the fold, log2 C rounds of the scan, T steps that each store a row) and
// by the stores on many.  Measured against what these calls took before (the register kernels of sig_onchip.h, one workgroup per
// path, their rows staged in LDS; or one launch per level), us: (4,4) 64 paths of 256 points 24.3 and 12.3, 4 of 1,075 62 and 19;
// (5,4) 16 of 100 17.5 and 8.5; (12,3) 1,024 of 100 487 and 228, 128 of 1,000 635 and 363.
//
// Rounding: a sum of T terms, one after the other, is off by about sqrt(T) roundings of its last value.  Pieces of more than
// kPlainSteps steps are therefore summed in blocks (BLOCKS below), level 1 at a piece's start comes from the points, and with more
// than ten channels level 1 of every row does.  Error against 64 bits over 34,000 random calls of 4 to 4,000 points, relative to
// what these calls took before: 0.75 in the mean beyond 64 points (0.58 ... 0.90 by shape), 0.95 below; with plain sums 0.93, but
// 1.1 to 1.5 on batches of 64 paths and more of hundreds of points ((12,3) 128 of 1,000 points 1.4, (20,2) 64 ... 256 of 2,000 1.5).
// The blocks cost up to 7 % ((3,5), 93 paths of 949 points 54.4 and 56.6 us; (4,4), 84 of 939 27.5 and 29.1).
#ifndef SIG_STREAM_ROWS_H
#define SIG_STREAM_ROWS_H

#include "sig_onchip.h"

namespace sig {
namespace rows {

using onchip::cpow;

struct Args {
    const float *path;   // [B][L][d]
    float *out;          // [B][L-1][D]
    int64_t B, L;
    int32_t slots;       // C: pieces of a path side by side in a workgroup
    int32_t segs;        // W: workgroups of a path
    int32_t groups;      // G: paths of a workgroup (1 unless segs is)
    int32_t steps;       // T: rows a slot emits; W * C * T >= L - 1
    int32_t tile;        // steps of a slot that are staged in LDS together, of its own piece
    int32_t behind;      // ... and of what lies before (segs > 1)
};

// a row in LDS: an odd stride where lanes and rows would otherwise all start in every 16th bank ((16,2), 200 paths of 200 points 35 and 31
// us; elsewhere it costs the wide accesses a little: (8,3), 30 of 200, 14.4 and 15.0)
__host__ __device__ constexpr int lds_row(int d, int64_t D) { return (int)(d % 16 == 0 ? D | 1 : D); }

template <int d_, int N_>
struct Geo {
    static constexpr int d = d_, N = N_, P = N - 1;
    static constexpr int Q = cpow(d, P);
    static constexpr int D = onchip::Shape<d, N, P>::D;
    static constexpr int DS = lds_row(d, D);
    static constexpr int SPW = Q <= kWave ? kWave / Q : 1;       // slots of a wavefront
    static constexpr int WPS = (Q + kWave - 1) / kWave;          // wavefronts of a slot
};
constexpr int kMaxThreads = 1024;
// (the shapes whose slots are small: cut() gives them half of that)
__host__ __device__ constexpr int most_threads(int d, int N) { return N == 2 ? 512 : kMaxThreads; }

// a slot's increments in LDS: an odd stride puts the slots of a wavefront into different banks
__host__ __device__ constexpr int tile_stride(int steps, int d) { return (steps * d) | 1; }
// rows of a path in LDS: the slots' own pieces but for the last (twice where the scan takes rounds), and what lies before
__host__ __device__ constexpr int lds_rows(int C, int W) { return (C - 1) * (C > 2 ? 2 : 1) + (W > 1 ? C : 0); }
// More than ten channels: a slot's tile holds points, and level 1 of a row is the point's distance from the path's first one, as the
// launches per level that these shapes took before give it.  A point that is not a number then spoils level 1 of its own row only.
__host__ __device__ constexpr bool level1_from_points(int d) { return d > 10; }
__host__ __device__ constexpr int tile_floats(const Args &A, int d)
{
    return (A.groups * A.slots * (tile_stride(A.tile + level1_from_points(d), d) + (A.segs > 1 ? tile_stride(A.behind, d) : 0)) + 3) / 4 * 4;
}

constexpr int kPlainSteps = 16;    // pieces of more steps than this are summed in blocks of as many (see BLOCKS)

// out = a + b, word by word
template <int d, int N, int P>
__device__ __forceinline__ void add_state(onchip::Lane<d, N, P> &out, const onchip::Lane<d, N, P> &a, const onchip::Lane<d, N, P> &b)
{
    using Sh = onchip::Shape<d, N, P>;
#pragma unroll
    for (int i = 0; i < Sh::SZ; ++i) out.s[i] = a.s[i] + b.s[i];
#pragma unroll
    for (int i = 0; i < Sh::NPRE; ++i) out.pre[i] = a.pre[i] + b.pre[i];
}

// Level 1 of what lies before a piece: the distance `exact` of two points (one rounding), but where one of the two is no finite
// number, what adding the increments up gave (sticky).  An infinite point leaves level 1 infinite in its own row and NaN behind it, and one
// at the path's start leaves it infinite in all rows.
__device__ __forceinline__ float level1_of(float exact, float added, bool sticky)
{
    return !sticky || fabsf(exact - added) < __builtin_huge_valf() ? exact : added;
}

// The fused step of sig_onchip.h for lanes that own a word of length N - 1, with what it adds to the signature `now` summed in `sum`
template <int d, int N>
__device__ __forceinline__ void summed_step(onchip::Lane<d, N, N - 1> &sum, const onchip::Lane<d, N, N - 1> &now, const onchip::Inc<d, N - 1> &inc)
{
    constexpr int P = N - 1;
    onchip::static_for<1, N + 1>([&](auto nc) __attribute__((always_inline)) {
        constexpr int n = decltype(nc)::value;
        float g = 1.0f;
#pragma unroll
        for (int m = 1; m < n; ++m) g = fmaf(g, inc.du[m - 1] * (1.0f / (float)(n - m + 1)), m < P ? now.pre[m - 1] : now.s[0]);
        if constexpr (n < P) {
            sum.pre[n - 1] = fmaf(g, inc.du[n - 1], sum.pre[n - 1]);
        } else if constexpr (n == P) {
            sum.s[0] = fmaf(g, inc.du[n - 1], sum.s[0]);
        } else {
#pragma unroll
            for (int a = 0; a < d; ++a) sum.s[1 + a] = fmaf(g, inc.v[a], sum.s[1 + a]);
        }
    });
}

// A slot's steps, one after the other: increments as they lie in the tile, or the differences of its points.  KEEP: the point behind a
// step stays in registers for the next one; else it is read again.  (Beside the block sums of 17 letters and more it would take the kernel past 128
// registers, and every unit's second workgroup with them: (19,2), 373 paths of 589 points 217 us and 187.)
template <int d, int P, bool POINTS, bool KEEP>
struct Steps {
    const float *row;
    const int *letter;
    onchip::Inc<d, P> last;   // POINTS: the point of `row`; without KEEP only at the lane's letters

    __device__ __forceinline__ Steps(const float *row_, const int *letter_) : row(row_), letter(letter_)
    {
        if constexpr (POINTS && KEEP) onchip::load_inc<d, P>(last, row, letter);
    }
    __device__ __forceinline__ void next(onchip::Inc<d, P> &inc)
    {
        if constexpr (POINTS && KEEP) {
            onchip::Inc<d, P> here;
            row += d;
            onchip::load_inc<d, P>(here, row, letter);
#pragma unroll
            for (int a = 0; a < d; ++a) inc.v[a] = here.v[a] - last.v[a];
#pragma unroll
            for (int m = 0; m < P; ++m) inc.du[m] = here.du[m] - last.du[m];
            last = here;
        } else if constexpr (POINTS) {
#pragma unroll
            for (int m = 0; m < P; ++m) {
                last.du[m] = row[d + letter[m]];
                inc.du[m] = last.du[m] - row[letter[m]];
            }
#pragma unroll
            for (int a = 0; a < d; ++a) {
                if (a == d / 2) __builtin_amdgcn_sched_barrier(0);   // half the letters' reads at a time, for the registers
                inc.v[a] = row[d + a] - row[a];
            }
            row += d;
        } else {
            onchip::load_inc<d, P>(inc, row, letter);
            row += d;
        }
    }
};

extern __shared__ __align__(16) float sig_rows_smem[];

// BLOCKS: the steps of a slot's own piece are summed in blocks of kPlainSteps, each from zero, and a row is the signature at the block's
// start plus that sum (blocks of 8 to 32 give the same error).  The steps go two a round, or the copies from one to the next show: (20,2), 2
// paths of 51 points 11.4 and 10.2 us, (3,5), 93 of 949 60 and 56.6.
// Four wavefronts a SIMD: two workgroups of 512 threads on a unit, or one of 1,024.
template <int d, int N, bool BLOCKS>
__global__ __launch_bounds__((most_threads(d, N))) __attribute__((amdgpu_waves_per_eu(4))) void sig_stream_rows_kernel(Args A)
{
    using G = Geo<d, N>;
    constexpr int P = G::P, Q = G::Q, D = G::D, DS = G::DS;
    constexpr bool POINTS = level1_from_points(d);
    using Lane = onchip::Lane<d, N, P>;
    const int tid = threadIdx.x, nthr = blockDim.x;
    const int wave = tid / kWave, lw = tid - wave * kWave, waves = nthr / kWave;
    const int64_t K = A.L - 1;
    const int C = A.slots, T = A.steps;
    const unsigned unit = blockIdx.x / (unsigned)A.segs;
    const int w = (int)(blockIdx.x - unit * (unsigned)A.segs);
    const int64_t b0 = (int64_t)unit * A.groups;
    const int paths = A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;
    const int64_t k0 = (int64_t)w * C * T;          // first row of the workgroup
    const int64_t before = (int64_t)w * T;          // steps of a slot of what lies before

    int slot;
    unsigned u;
    bool active;
    if constexpr (Q <= kWave) {
        const int sw = lw / Q;
        slot = wave * G::SPW + sw;
        u = (unsigned)(lw - sw * Q);
        active = sw < G::SPW && slot < paths * C;
    } else {
        slot = wave / G::WPS;
        u = (unsigned)((wave - slot * G::WPS) * kWave + lw);
        active = u < (unsigned)Q && slot < paths * C;
    }
    if (!active) { slot = 0; u = 0; }
    const int p = slot / C, c = slot - p * C;       // path and piece
    const int64_t k = k0 + (int64_t)c * T;          // first row of the piece
    int letter[P];
    {
        unsigned rest = u;
#pragma unroll
        for (int m = P - 1; m >= 0; --m) { letter[m] = (int)(rest % d); rest /= d; }
    }

    // level 1 at the path's first point and at the piece's
    float first1 = 0.0f, here1 = 0.0f;
    if (active && k < K) {
        const float *x = A.path + (b0 + p) * A.L * d + letter[0];
        first1 = x[0];
        here1 = x[k * d];
    }

    const int own_stride = tile_stride(A.tile + POINTS, d), old_stride = tile_stride(A.behind, d);
    float *own = sig_rows_smem;                     // [slots][own_stride]
    float *old = own + A.groups * C * own_stride;   // [slots][old_stride]
    float *rows = sig_rows_smem + tile_floats(A, d) + p * lds_rows(C, A.segs) * DS;

    // `count` increments of every slot from step first + c * stride on, zeros beyond the path's end
    auto stage = [&](float *tile, int row, int64_t first, int64_t stride, int count) __attribute__((always_inline)) {
        for (int s = wave; s < paths * C; s += waves) {
            const int sp = s / C;
            const int64_t at = (first + (s - sp * C) * stride) * d;
            const float *X = A.path + (b0 + sp) * A.L * d + at;
            float *dst = tile + s * row;
#pragma unroll 4
            for (int r = lw; r < count * d; r += kWave) dst[r] = at + r < K * d ? X[r + d] - X[r] : 0.0f;
        }
    };
    // the tile of the slots' own pieces: increments, or the points that they lie between, the last one repeated beyond the path's end
    auto stage_own = [&](int t0, int count) __attribute__((always_inline)) {
        if constexpr (POINTS) {
            for (int s = wave; s < paths * C; s += waves) {
                const int sp = s / C;
                const int64_t at = (k0 + t0 + (int64_t)(s - sp * C) * T) * d;
                const float *path = A.path + (b0 + sp) * A.L * d;
                float *dst = own + s * own_stride;
#pragma unroll 4
                for (int r = lw; r < (count + 1) * d; r += kWave) dst[r] = path[at + r < A.L * d ? at + r : K * d + r % d];
            }
        } else {
            stage(own, own_stride, k0 + t0, T, count);
        }
    };
    // `count` steps of the slot's own piece, f after each of them; exact: with level 1 from the points (POINTS)
    auto own_steps = [&](Lane &ln, const float *row, int count, auto exact, auto &&f) __attribute__((always_inline)) {
        Steps<d, P, POINTS, d <= 16 || !BLOCKS> steps(row, letter);
        onchip::Inc<d, P> inc;
        auto level1 = [&](Lane &now) __attribute__((always_inline)) {
            if constexpr (POINTS && decltype(exact)::value) (P > 1 ? now.pre[0] : now.s[0]) = steps.last.du[0] - first1;
        };
        if constexpr (BLOCKS) {
            for (int t0 = 0; t0 < count; t0 += kPlainSteps) {
                const int end = count - t0 < kPlainSteps ? count : t0 + kPlainSteps;
                Lane sum, now = ln;
                onchip::identity_state<d, N, P>(sum);
#pragma unroll 2
                for (int t = t0; t < end; ++t) {
                    steps.next(inc);
                    summed_step<d, N>(sum, now, inc);
                    add_state<d, N, P>(now, ln, sum);
                    level1(now);
                    f(now, t);
                }
                add_state<d, N, P>(ln, ln, sum);   // (not ln = now: the words that no chain reads would stay in registers beside the sum)
                if constexpr (POINTS && decltype(exact)::value) (P > 1 ? ln.pre[0] : ln.s[0]) = P > 1 ? now.pre[0] : now.s[0];
            }
        } else {
#pragma unroll 2
            for (int t = 0; t < count; ++t) {
                steps.next(inc);
                onchip::fused_step<d, N, P>(ln, inc);
                level1(ln);
                f(ln, t);
            }
        }
    };
    // (two steps a round, both increments read first: one wait for the pair; (4,4), 4 paths of 1,075 points 18.5 -> 17.1 us)
    auto fold = [&](Lane &ln, const float *row, int count) __attribute__((always_inline)) {
        int t = 0;
        for (; t + 1 < count; t += 2, row += 2 * d) {
            onchip::Inc<d, P> inc, inc2;
            onchip::load_inc<d, P>(inc, row, letter);
            onchip::load_inc<d, P>(inc2, row + d, letter);
            onchip::fused_step<d, N, P>(ln, inc);
            onchip::fused_step<d, N, P>(ln, inc2);
        }
        if (t < count) {
            onchip::Inc<d, P> inc;
            onchip::load_inc<d, P>(inc, row, letter);
            onchip::fused_step<d, N, P>(ln, inc);
        }
    };
    // the slot's own piece, tile by tile (staged once and for all where one tile holds it)
    auto own_tiles = [&](auto &&f) __attribute__((always_inline)) {
        for (int t0 = 0; t0 < T; t0 += A.tile) {
            const int count = T - t0 < A.tile ? T - t0 : A.tile;
            if (T > A.tile) {
                __syncthreads();
                stage_own(t0, count);
                __syncthreads();
            }
            f(own + slot * own_stride, t0, count);
        }
    };

    Lane ln, bl;   // the slot's own piece, and what lies before it
    onchip::identity_state<d, N, P>(bl);
    if (T <= A.tile) stage_own(0, T);
    // Folded block by block, a tile each, and the blocks multiplied: the rounding of a fold grows with the square root of its
    // steps ((5,4), 16 paths of 2,000 points: error of blocks of 64 steps 1.8e-7, of the 500 steps of a piece in one go 3.7e-7, of one launch per
    // level 2.2e-7).
    float *join = rows + lds_rows(C, 1) * DS;
    for (int64_t t0 = 0; t0 < before; t0 += A.behind) {
        const int count = before - t0 < A.behind ? (int)(before - t0) : A.behind;
        if (t0 > 0) __syncthreads();
        stage(old, old_stride, t0, before, count);
        __syncthreads();
        const float *row = old + slot * old_stride;
        if (t0 == 0) {
            fold(bl, row, count);
        } else {
            onchip::identity_state<d, N, P>(ln);
            fold(ln, row, count);
            if (active) onchip::store_state<d, N, P>(join + c * DS, u, ln);
            __syncthreads();
            if (active) onchip::reg_product<d, N, P>(bl, join + c * DS, u);
        }
    }
    if (before == 0 || before > A.behind) __syncthreads();   // the own tile; the last block's rows have been read
    if (C > 1) {
        float *cur = rows, *nxt = C > 2 ? cur + (C - 1) * DS : cur;
        onchip::identity_state<d, N, P>(ln);
        own_tiles([&](const float *row, int, int count) __attribute__((always_inline)) {
            if constexpr (BLOCKS || POINTS) own_steps(ln, row, count, std::false_type{}, [](const Lane &, int) {});
            else fold(ln, row, count);
        });
        if (active) {
            if (c < C - 1) onchip::store_state<d, N, P>(cur + c * DS, u, ln);
            if (before > 0) onchip::store_state<d, N, P>(join + c * DS, u, bl);
        }
        __syncthreads();
        // Round with stride st.  Scan: the lanes of piece c multiply their value by the row of piece c + st and leave the product
        // as that piece's new row (nobody needs the last one's).  Tree: piece c, a multiple of 2 st, absorbs piece c + st.
        for (int st = 1; st < (before > 0 ? C : C - 1); st <<= 1) {
            const bool scan = st < C - 1;
            if (active) {
                if (before > 0 && (c & (2 * st - 1)) == 0 && c + st < C) {
                    onchip::reg_product<d, N, P>(bl, join + (c + st) * DS, u);
                    onchip::store_state<d, N, P>(join + c * DS, u, bl);
                }
                if (scan) {
                    if (c < st) onchip::store_state<d, N, P>(nxt + c * DS, u, ln);
                    if (c + st < C - 1) {
                        onchip::reg_product<d, N, P>(ln, cur + (c + st) * DS, u);
                        onchip::store_state<d, N, P>(nxt + (c + st) * DS, u, ln);
                    }
                }
            }
            __syncthreads();
            if (scan) {
                if (active && c < C - 1) onchip::load_state<d, N, P>(nxt + c * DS, u, ln);
                float *t = cur; cur = nxt; nxt = t;
            }
        }
        if (before > 0) {
            onchip::load_state<d, N, P>(join, u, bl);
            if (c > 0) onchip::reg_product<d, N, P>(bl, cur + (c - 1) * DS, u);
        } else if (c > 0) {
            onchip::load_state<d, N, P>(cur + (c - 1) * DS, u, bl);
        }
    }

    if (k > 0) {
        float &s1 = P > 1 ? bl.pre[0] : bl.s[0];
        s1 = level1_of(here1 - first1, s1, !POINTS);
    }
    const int mine = !active || k >= K ? 0 : K - k < T ? (int)(K - k) : T;
    float *dst = A.out + ((b0 + p) * K + k) * D;
    own_tiles([&](const float *row, int t0, int count) __attribute__((always_inline)) {
        own_steps(bl, row, count, std::true_type{}, [&](const Lane &now, int t) __attribute__((always_inline)) {
            if (t0 + t < mine) onchip::store_state<d, N, P>(dst, u, now);
            dst += D;
        });
    });
}

}  // namespace rows
}  // namespace sig

#endif  // SIG_STREAM_ROWS_H
