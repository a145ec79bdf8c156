// Gradient of the every-prefix signature with respect to the path at depth 2 (stream mode; two to twenty channels).
//
// With loss gradients G_j of row j = 1 .. K (levels G1_j and the d x d matrix M_j), the loss as a function of an element
// inserted after step k is the sum over the rows behind it (file comment of sig_bracket.h, one F per row), so that with
//     A_j = sum_{i >= j} (M_i - M_i^T),     H_j[b] = G1_j[b] + sum_a (X_j - X_0)[a] M_j[a b]
// the gradient of the points is
//     d(loss)/dX_j[b] = H_j[b] - 1/2 sum_a (v_{j+1}[a] A_{j+1}[a b] + v_j[a] A_j[a b]),      v_j = X_j - X_{j-1},
// the missing step's term left out at j = K, and -sum_j (G1_j[b] + sum_a (X_j - X_0)[a] M_j[b a]) in place of H_0 at j = 0.  A is a
// plain sum over the rows behind a step: no prefix signature is undone, no adjoint is carried, and the rows of S are not read.
//
// Lanes.  Lane b of d holds column b of A and settles channel b; it reads column b and row b of M_j from LDS, where a wavefront
// stages the next few rows of its slots (d lanes each) as they lie in memory while it uses the last ones (read straight from
// memory, 4 bytes a lane and d apart, the address unit took 40 cycles a load).  Whole paths side by side in wavefronts, walked
// from their last row (UNCUT), or stretches of a path side by side in a workgroup (CUT): each slot sums its own rows, a scan in
// LDS adds what lies behind it, and it walks its rows once more.  Few paths also span W workgroups, whose sums a first launch
// (TOTALS) leaves in scratch.  Bound by the rows' bytes where uncut wavefronts fill the chip, by a row's 0.2 to 0.7 us of LDS
// and dependent multiply-adds elsewhere.  Measured, the sweep on signatures against this: 128 paths of 150 points of 16 channels
// (the general sweep) 577 -> 19.5 us, one of 100 of 12 358 -> 9; 20,591 of 79 of 9 248 -> 168 (126 at the rate of a copy), 2,040
// of 1,777 of 9 5,440 -> 493, 55,774 of 446 of 2 786 -> 386, one of 1,445 of 10 55 -> 16; over 4,013 calls 2.9 times as fast in
// the mean.  Rounding against 64 bits: 3e-8 to 1.7e-6 of the gradient's norm, 0.1 to 1.0 times the sweep's (its A is undone
// and carried as well).
#include <type_traits>

#include "sig_internal.h"

namespace sig {
namespace stream_gradient {

typedef float vec4f_u __attribute__((ext_vector_type(4), aligned(4)));
typedef float vec4f_8 __attribute__((ext_vector_type(4), aligned(8)));

struct Args {
    const float *path;      // [B][L][d]
    const float *grad_out;  // [B][K][d + d * d]
    float *grad_path;       // [B][L][d]
    float *totals;          // [B][W][d * d + d]: the sums over a workgroup's rows (W > 1)
    int64_t B;
    int32_t L;
    int32_t chunks;         // C: stretches of a path side by side in a workgroup
    int32_t segs;           // W: workgroups of a path
    int32_t groups;         // paths in a workgroup (one where W > 1 or a path takes several blocks)
    int32_t steps;          // T: rows of a stretch; C * T are a block, and a workgroup walks its blocks one after the other
    int32_t rows;           // of a workgroup: a multiple of C * T where W > 1
};

enum Mode { UNCUT, CUT, TOTALS };

constexpr int kMostChannels = 20;
constexpr int64_t kBlockBytes = 96 * 1024;

constexpr int threads_of(int mode) { return mode == UNCUT ? kWave : 4 * kWave; }
constexpr int slots_of(int mode, int d) { return threads_of(mode) / kWave * (kWave / d); }
constexpr int sums_of(int d) { return d * d + d; }   // A, and a slot's share of the sums that settle point 0

// Rows of each slot that a wavefront stages at a time: some 1,600 floats in all, whole 16-byte vectors (a row is of even length)
constexpr int tile_rows(int d)
{
    const int row = d + d * d, unit = row % 4 == 0 ? 1 : 2;
    const int fit = 1600 / (kWave / d * row * unit);
    return unit * (fit < 1 ? 1 : fit > 16 / unit ? 16 / unit : fit);
}

// A wavefront's tile: R rows of each of its slots, as they lie in memory, and the R + 1 points around them
template <int d>
struct Tile {
    static constexpr int D = d + d * d, SLOTS = kWave / d;
    static constexpr int R = tile_rows(d);
    static constexpr int VECS = R * D / 4;                        // vectors of a slot
    static constexpr int NV = (SLOTS * VECS + kWave - 1) / kWave; // ... that a lane brings
    static constexpr int PX = (R + 1) * d;                        // floats of a slot's points
    static constexpr int NX = (SLOTS * PX + kWave - 1) / kWave;
    // a slot's rows begin some d banks behind its neighbour's, so that the slots' lanes read their columns from different banks
    static constexpr int STRIDE = R * D + ((d + 3) / 4 * 4 + 64 - R * D % 32) % 32;
    static constexpr int XS = (d + 3) / 4 * 4;
    static constexpr int FLOATS = SLOTS * (STRIDE + (R + 1) * XS);
};
template <int d>
constexpr int tiles_floats(int mode) { return threads_of(mode) / kWave * Tile<d>::FLOATS; }
template <int d>
constexpr int lds_floats(int mode) { return tiles_floats<d>(mode) + (mode == UNCUT ? 0 : (slots_of(mode, d) + 1) * sums_of(d)); }

extern __shared__ __align__(16) float sig_stream_gradient_smem[];

// CNT floats of LDS, in the widest pieces that a multiple of CNT floats is aligned to
template <int CNT>
__device__ __forceinline__ void read_floats(float (&dst)[CNT], const float *src)
{
    constexpr int V = CNT % 4 == 0 ? 4 : CNT % 2 == 0 ? 2 : 1;
    typedef float vec __attribute__((ext_vector_type(V)));
#pragma unroll
    for (int i = 0; i < CNT; i += V) {
        const vec v = *reinterpret_cast<const vec *>(src + i);
        if constexpr (V == 1) dst[i] = v[0];
        else {
#pragma unroll
            for (int j = 0; j < V; ++j) dst[i + j] = v[j];
        }
    }
}

// Lanes of a wavefront that exchange data through LDS: the hardware keeps their order, the compiler has to as well
__device__ __forceinline__ void wave_sync()
{
    __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
    __builtin_amdgcn_wave_barrier();
}

template <int d, int MODE>
__global__ __launch_bounds__(threads_of(MODE)) __attribute__((amdgpu_waves_per_eu(2))) void sig_stream_depth2_kernel(Args A)
{
    using Tl = Tile<d>;
    constexpr int NT = threads_of(MODE), WSLOTS = Tl::SLOTS, M = sums_of(d), D = Tl::D, R = Tl::R, XS = Tl::XS;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int K = A.L - 1;
    const int C = MODE == UNCUT ? 1 : A.chunks, W = MODE == UNCUT ? 1 : A.segs, T = MODE == UNCUT ? K : A.steps;
    const int64_t b0 = W > 1 ? blockIdx.x / W : (int64_t)blockIdx.x * A.groups;
    const int seg = W > 1 ? (int)(blockIdx.x - b0 * W) : 0;
    const int k0 = W > 1 ? seg * A.rows : 0;                             // the workgroup's rows are k0 + 1 .. k1
    const int k1 = W > 1 && K - k0 > A.rows ? k0 + A.rows : K;
    const int npaths = W > 1 ? 1 : A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;
    const int wslot = lane / d, b = lane - wslot * d;
    const int slot = wave * WSLOTS + wslot;
    const int group = slot / C, chunk = slot - group * C;
    const bool active = wslot < WSLOTS && group < npaths;
    const float *points = A.path + b0 * A.L * d, *grads = A.grad_out + b0 * K * D;   // (of all its paths: below 2^31 floats)
    const float *X = A.path + (b0 + (active ? group : 0)) * A.L * d;
    float *dX = A.grad_path + (b0 + (active ? group : 0)) * A.L * d;

    float *gtile = sig_stream_gradient_smem + wave * Tl::FLOATS, *xtile = gtile + WSLOTS * Tl::STRIDE;
    const float *myg = gtile + (active ? wslot : 0) * Tl::STRIDE, *myx = xtile + (active ? wslot : 0) * (R + 1) * XS;
    float *sums = sig_stream_gradient_smem + NT / kWave * Tl::FLOATS, *base = sums + NT / kWave * WSLOTS * M;

    // The last row of a slot's stretch of the block that ends with row hi, and the lowest row of the R that begin t0 below it.  Row
    // numbers count from 1; where fewer than R rows are left the tile reaches back up, and below R rows in all beyond K.
    auto top_of = [&](int hi, int c) __attribute__((always_inline)) {
        const int64_t top = (int64_t)hi - (int64_t)(C - 1 - c) * T;
        return top < K ? (int)top : K;
    };
    auto low_of = [&](int top, int t0) __attribute__((always_inline)) { return top - t0 > R ? top - t0 - R + 1 : 1; };

    // A tile's rows and points on their way to LDS: the lane that holds a slot's first letter says where its tile begins
    vec4f_u gv[Tl::NV];
    float xv[Tl::NX];
    const int last = ((K < R ? K : R) * D) - 4;       // of a slot's vectors, where the path has fewer than R rows
    auto fetch = [&](int low) __attribute__((always_inline)) {
        const int row = active ? group * K + low - 1 : 0, point = row + (active ? group : 0);
#pragma unroll
        for (int j = 0; j < Tl::NV; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::VECS, at = 4 * (i - ws * Tl::VECS);
            gv[j] = *reinterpret_cast<const vec4f_u *>(grads + (__shfl(row, ws * d) * D + (at < last ? at : last)));
        }
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::PX, at = i - ws * Tl::PX;
            xv[j] = points[__shfl(point, ws * d) * d + (at < (last / D + 2) * d ? at : 0)];
        }
    };
    auto put = [&]() __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Tl::NV; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::VECS, at = 4 * (i - ws * Tl::VECS);
            if (ws < WSLOTS) *reinterpret_cast<vec4f_8 *>(gtile + ws * Tl::STRIDE + (at < last ? at : last)) = gv[j];
        }
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = lane + j * kWave, ws = i / Tl::PX, x = i - ws * Tl::PX;
            if (ws < WSLOTS) xtile[(ws * (R + 1) + x / d) * XS + x % d] = xv[j];
        }
    };
    // use(j, row j, point j - 1; point j lies XS floats behind it) for the rows of the slot's stretch, from the last one down
    // (held: the only tile is in LDS already)
    auto walk = [&](int hi, bool held, auto &&use) __attribute__((always_inline)) {
        const int top = top_of(hi, chunk);
        const int64_t below = (int64_t)hi - (int64_t)(C - chunk) * T;    // the row under the stretch
        const int least = below > 0 ? (int)below + 1 : 1;
        if (!held) fetch(low_of(top, 0));
        for (int t0 = 0; t0 < T; t0 += R) {
            if (!held) {
                wave_sync();
                put();
                wave_sync();
            }
            if (T - t0 > R) fetch(low_of(top, t0 + R));
            const int low = low_of(top, t0);
#pragma unroll 2
            for (int r = R - 1; r >= 0; --r) {
                const int j = low + r;
                if (active && j >= least && j <= top - t0) use(j, myg + r * D, myx + r * XS);
            }
        }
    };

    float m[d];              // column b of A
    float start = 0.0f;      // what becomes -d(loss)/dX_0
    float x0[d];
#pragma unroll
    for (int a = 0; a < d; ++a) {
        m[a] = 0.0f;
        x0[a] = X[a];
    }
    // a row's share of the sums (SUM) and the gradient of its point (SETTLE)
    float above = 0.0f;      // sum_a v_{j+1}[a] A_{j+1}[a b]
    auto row_of = [&](int j, const float *g, const float *x, auto sum, auto settle) __attribute__((always_inline)) {
        constexpr bool SUM = decltype(sum)::value, SETTLE = decltype(settle)::value;
        float row[d], at[XS], before[XS];
        read_floats<d>(row, g + d + b * d);
        read_floats<XS>(at, x + XS);
        float h = g[b], below = 0.0f;
        if constexpr (SUM) start += h;
        if constexpr (SETTLE) read_floats<XS>(before, x);
#pragma unroll
        for (int a = 0; a < d; ++a) {
            const float col = g[d + a * d + b], s = at[a] - x0[a];
            m[a] += col - row[a];
            if constexpr (SUM) start = fmaf(s, row[a], start);
            if constexpr (SETTLE) {
                h = fmaf(s, col, h);
                below = fmaf(at[a] - before[a], m[a], below);
            }
        }
        if constexpr (SETTLE) {
            dX[(int64_t)j * d + b] = fmaf(-0.5f, above + below, h);
            above = below;
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    if constexpr (MODE == UNCUT) {
        walk(K, false, [&](int j, const float *g, const float *x) __attribute__((always_inline)) { row_of(j, g, x, yes, yes); });
        if (active) dX[b] = fmaf(-0.5f, above, -start);
    } else {
        // what lies behind the workgroup's rows
        for (int e = tid; e < M; e += NT) {
            float sum = 0.0f;
            if constexpr (MODE == CUT)
                for (int w = W - 1; w > seg; --w) sum += A.totals[(b0 * W + w) * M + e];
            base[e] = sum;
        }
        const int span = C * T < k1 - k0 ? C * T : k1 - k0, blocks = (k1 - k0 + span - 1) / span;
        for (int blk = blocks - 1; blk >= 0; --blk) {
            const int hi = k0 + blk * span + C * T;                      // (may lie beyond K in the last block)
            start = 0.0f;
#pragma unroll
            for (int a = 0; a < d; ++a) m[a] = 0.0f;
            walk(hi, false, [&](int j, const float *g, const float *x) __attribute__((always_inline)) { row_of(j, g, x, yes, no); });
            __syncthreads();                                             // (of the block before: base is written, sums are read)
            if (active) {
#pragma unroll
                for (int a = 0; a < d; ++a) sums[slot * M + a * d + b] = m[a];
                sums[slot * M + d * d + b] = start;
            }
            __syncthreads();
            for (int i = tid; i < npaths * M; i += NT) {
                const int g = i / M, e = i - g * M;
                float *s = sums + g * C * M + e;
                float sum = npaths == 1 ? base[e] : 0.0f;
#pragma unroll 4
                for (int c = C - 1; c >= 0; --c) {
                    const float own = s[c * M];
                    s[c * M] = sum;
                    sum += own;
                }
                if (npaths == 1) base[e] = sum;
            }
            __syncthreads();
            if constexpr (MODE == CUT) {
                if (active) {
#pragma unroll
                    for (int a = 0; a < d; ++a) m[a] = sums[slot * M + a * d + b];
                    start += sums[slot * M + d * d + b];
                }
                const int top = top_of(hi, chunk);
                above = 0.0f;
                if (active && top < K && top > 0) {
#pragma unroll
                    for (int a = 0; a < d; ++a)
                        above = fmaf(X[(int64_t)(top + 1) * d + a] - X[(int64_t)top * d + a], m[a], above);
                }
                walk(hi, T <= R, [&](int j, const float *g, const float *x) __attribute__((always_inline)) { row_of(j, g, x, no, yes); });
                if (active && chunk == 0 && hi - C * T == 0) dX[b] = fmaf(-0.5f, above, -start);
            }
        }
        if constexpr (MODE == TOTALS) {
            __syncthreads();
            for (int e = tid; e < M; e += NT) A.totals[(b0 * W + seg) * M + e] = base[e];
        }
    }
}

struct Cut {
    int mode;               // UNCUT or CUT
    int chunks, segs, groups, steps, rows;
    int tile;               // rows of a slot that a wavefront stages at a time
    int64_t grid;
};

template <int d>
hipError_t launch(const Args &A0, const Cut &c, hipStream_t st)
{
    Args A = A0;
    A.chunks = c.chunks;
    A.segs = c.segs;
    A.groups = c.groups;
    A.steps = c.steps;
    A.rows = c.rows;
    const dim3 grid((unsigned)c.grid);
    if (c.mode == UNCUT) {
        constexpr size_t lds = (size_t)lds_floats<d>(UNCUT) * sizeof(float);
        static_assert(lds <= (size_t)kMaxLdsBytes, "a wavefront's tile fits its workgroup's LDS");
        hipLaunchKernelGGL((sig_stream_depth2_kernel<d, UNCUT>), grid, dim3(threads_of(UNCUT)), lds, st, A);
        return hipGetLastError();
    }
    constexpr size_t lds = (size_t)lds_floats<d>(CUT) * sizeof(float);
    static_assert(lds <= (size_t)kMaxLdsBytes, "the tiles and sums of a workgroup's slots fit its LDS");
    if (c.segs > 1) {
        hipLaunchKernelGGL((sig_stream_depth2_kernel<d, TOTALS>), grid, dim3(threads_of(TOTALS)), lds, st, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL((sig_stream_depth2_kernel<d, CUT>), grid, dim3(threads_of(CUT)), lds, st, A);
    return hipGetLastError();
}

// UNCUT (W == 0) or CUT with W workgroups a path and at most `most_chunks` stretches side by side; false where a launch would hold 2^32 threads or an offset 2^31 floats.
bool cut(int d, int64_t B, int64_t L, int64_t W, int most_chunks, Cut *c)
{
    const int64_t K = L - 1, D = d + d * d, slots = slots_of(W > 0 ? CUT : UNCUT, d);
    if (L > INT32_MAX / D) return false;
    c->chunks = c->segs = 1;
    c->tile = tile_rows(d);
    c->steps = c->rows = (int)K;
    if (W == 0) {
        c->mode = UNCUT;
        c->groups = (int)slots;
        c->grid = (B + slots - 1) / slots;
        return slots * L <= INT32_MAX / D && c->grid * threads_of(UNCUT) < (int64_t)1 << 32;
    }
    c->mode = CUT;
    int64_t rows = (K + W - 1) / W;                       // of a workgroup
    int64_t C = rows < slots ? rows : slots;
    if (C > most_chunks) C = most_chunks;
    int64_t T = (rows + C - 1) / C;
    // a block's rows are read twice, the second time from the caches
    int64_t most = kBlockBytes / (C * D * (int64_t)sizeof(float));
    if (most < 8) most = 8;
    const int64_t blocks = (T + most - 1) / most;
    T = (T + blocks - 1) / blocks;
    if (W > 1) {
        rows = (rows + C * T - 1) / (C * T) * (C * T);
        W = (K + rows - 1) / rows;                        // no workgroup is left without rows
    }
    c->chunks = (int)C;
    c->steps = (int)T;
    c->rows = (int)rows;
    c->segs = (int)W;
    c->groups = W > 1 || C * T < K ? 1 : (int)(slots / C);
    c->grid = W > 1 ? B * W : (B + c->groups - 1) / c->groups;
    return C * T <= INT32_MAX && c->grid * threads_of(CUT) < (int64_t)1 << 32;
}

// Microseconds of a launch, fitted to 3,450 calls (2 to 20 channels, 1 to 20,000 paths of 2 to 2,000 points, every cut; 12 and
// 13 % off in the mean).  Uncut, a row follows the other in 0.1 (1 + 0.3 d) us until the wavefronts or the bytes set the pace; cut, a
// block costs its steps (twice), the scan over its stretches and their barriers, less where a stretch is one tile that stays in
// LDS.  The choice costs 1.03 times the best cut in the mean: tens of thousands of short paths uncut (16,294 of 135 points of 4
// channels 46 us, the best cut 58), thousands in a few stretches each (1,719 of 97 of 2: uncut 19, 16 stretches 6.3, 96 of them 25),
// one path of 1,445 of 10 across 16 workgroups (uncut 687, one workgroup 72, 16 of them 16).
double microseconds(int d, int64_t B, int64_t L, int cus, const Cut &c)
{
    const double K = (double)(L - 1), chip = cus / 256.0;
    const double thousands = (double)c.grid / 1000.0 / chip;
    const double gigabytes = (double)B * K * sums_of(d) * sizeof(float) * 1e-9;
    if (c.mode == UNCUT) {
        const double chain = 0.105 * (1 + 0.32 * d) * K, waves = 0.1 * (1 - 0.04 * (d < 16 ? d : 16)) * thousands * K;
        const double bytes = gigabytes / 4.2e-3 / chip;
        return 3.0 + (chain > waves ? (chain > bytes ? chain : bytes) : waves > bytes ? waves : bytes);
    }
    const double span = (double)c.chunks * c.steps;
    const double blocks = c.segs > 1 ? c.rows / span : K > span ? K / span : 1.0;
    const double walk = c.steps * (1 + 0.2 * d), held = c.steps <= c.tile ? 1.0 : 0.0;
    const double alone = 2.7 + blocks * (0.3 * walk + 0.93 + 0.033 * c.chunks - 1.03 * held);
    const double full = 4.9 + thousands * blocks * (0.51 * walk + 5.95 + 0.06 * c.chunks - 3.6 * held);
    const double bytes = gigabytes / 1.9e-3 / chip;
    const double least = c.chunks > 1 ? 5.2 : 3.5;
    const double us = alone > full ? (alone > bytes ? alone : bytes) : full > bytes ? full : bytes;
    return (us > least ? us : least) + (c.segs > 1 ? 3.5 + 0.19 * c.segs : 0.0);
}

bool choose(int d, int64_t B, int64_t L, int cus, bool scratch, Cut *best)
{
    bool found = false;
    double least = 0.0;
    auto consider = [&](int64_t W, int most_chunks) {
        Cut c;
        if (!cut(d, B, L, W, most_chunks, &c)) return;
        const double us = microseconds(d, B, L, cus, c);
        if (found && us >= least) return;
        found = true;
        least = us;
        *best = c;
    };
    const int slots = slots_of(CUT, d);
    consider(0, 1);
    for (int C = slots; C >= 4; C = C == slots ? (slots > 64 ? 64 : slots > 32 ? 32 : slots > 16 ? 16 : slots > 8 ? 8 : 4) : C / 2) {
        consider(1, C);
        if (C == 4) break;
    }
    for (int W = 2; W <= 32 && scratch && B * W <= cus; W *= 2) consider(W, slots);
    return found;
}

}  // namespace stream_gradient

bool stream_gradient_geometry(int d, int64_t B, int64_t L, int cus, bool scratch, int64_t *scratch_floats, int64_t *grid, int64_t *segs,
                              int64_t *groups, int64_t *chunks, int64_t *steps, int64_t *rows)
{
    stream_gradient::Cut c;
    if (d < 2 || d > stream_gradient::kMostChannels || B <= 0 || L < 2 || !stream_gradient::choose(d, B, L, cus, scratch, &c)) return false;
    *scratch_floats = c.segs > 1 ? B * c.segs * stream_gradient::sums_of(d) : 0;
    *grid = c.grid;
    *segs = c.segs;
    *groups = c.groups;
    *chunks = c.chunks;
    *steps = c.steps;
    *rows = c.rows;
    return true;
}

int64_t stream_gradient_scratch_floats(int d, int64_t B, int64_t L, int cus)
{
    stream_gradient::Cut c;
    if (d < 2 || d > stream_gradient::kMostChannels || !stream_gradient::choose(d, B, L, cus, true, &c)) return -1;
    return c.segs > 1 ? B * c.segs * stream_gradient::sums_of(d) : 0;
}

hipError_t launch_stream_gradient(const float *path, const float *grad_out, float *grad_path, float *scratch, int64_t B, int64_t L,
                                  int d, int cus, hipStream_t st)
{
    using namespace stream_gradient;
    Cut c;
    if (B <= 0 || L < 2 || !choose(d, B, L, cus, scratch != nullptr, &c)) return hipErrorInvalidValue;
    Args A{};
    A.path = path;
    A.grad_out = grad_out;
    A.grad_path = grad_path;
    A.totals = scratch;
    A.B = B;
    A.L = (int32_t)L;
    switch (d) {
#define SIG_STREAM_GRADIENT(d_) case d_: return launch<d_>(A, c, st);
    SIG_STREAM_GRADIENT(2) SIG_STREAM_GRADIENT(3) SIG_STREAM_GRADIENT(4) SIG_STREAM_GRADIENT(5) SIG_STREAM_GRADIENT(6)
    SIG_STREAM_GRADIENT(7) SIG_STREAM_GRADIENT(8) SIG_STREAM_GRADIENT(9) SIG_STREAM_GRADIENT(10) SIG_STREAM_GRADIENT(11)
    SIG_STREAM_GRADIENT(12) SIG_STREAM_GRADIENT(13) SIG_STREAM_GRADIENT(14) SIG_STREAM_GRADIENT(15) SIG_STREAM_GRADIENT(16)
    SIG_STREAM_GRADIENT(17) SIG_STREAM_GRADIENT(18) SIG_STREAM_GRADIENT(19) SIG_STREAM_GRADIENT(20)
#undef SIG_STREAM_GRADIENT
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sig
