// Gradient of the every-prefix signature with respect to the path at depth 2 (stream mode; two to twenty channels), and at depth 3
// for eleven and twelve channels (second part).
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
// (TOTALS) leaves in scratch.  Bound by the rows' bytes where the batch fills the chip (uncut they are read once, at 3.0 to 3.7 TB/s of all
// that moves; cut twice, from memory where the blocks that run together exceed the caches: (9,2) 2,040 paths of 1,777 points read 3.1 GB, 1.3
// of them rows, at 6.3 TB/s), by a row's 0.2 to 0.7 us of LDS and dependent multiply-adds elsewhere.  Measured, the sweep on
// signatures against this, one MI355X, both in turn: 128 paths of 150 points of 16 channels
// (the general sweep) 577 -> 19.5 us, one of 100 of 12 358 -> 9; 20,591 of 79 of 9 248 -> 168 (126 at the rate of a copy), 2,040
// of 1,777 of 9 5,440 -> 493, 55,774 of 446 of 2 786 -> 386, one of 1,445 of 10 55 -> 16; over 4,013 calls 2.9 times as fast in
// the mean.  Rounding against 64 bits: 3e-8 to 1.7e-6 of the gradient's norm, 0.1 to 1.0 times the sweep's (its A is undone
// and carried as well).
#include <cmath>
#include <type_traits>

#include "sig_internal.h"

namespace sig {
namespace stream_gradient {

typedef float vec4f_u __attribute__((ext_vector_type(4), aligned(4)));
typedef float vec4f_8 __attribute__((ext_vector_type(4), aligned(8)));

struct Args {
    const float *path;      // [B][L][d]
    const float *sig;       // depth 3: [B][K][D], level 2 is read
    const float *grad_out;  // [B][K][D]
    float *reduced;         // depth 3: [B][K][2 d + d * d], what it leaves for the sweep of depth 2
    float *grad_path;       // [B][L][d]
    float *totals;          // [B][W][d * d + d] (depth 3: [d * d * d]): the sums over a workgroup's rows (W > 1)
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

// Rows of each slot that a wavefront stages at a time: some 1,600 floats in all, whole 16-byte vectors
constexpr int row_floats(int d, bool given) { return (given ? 2 : 1) * d + d * d; }
constexpr int tile_rows(int d, bool given)
{
    const int row = row_floats(d, given), unit = row % 4 == 0 ? 1 : row % 2 == 0 ? 2 : 4;
    const int fit = 1600 / (kWave / d * row * unit);
    return unit * (fit < 1 ? 1 : fit > 16 / unit ? 16 / unit : fit);
}

// Floats between a slot's rows and the next one's, and between its points: rows begin some d banks behind the neighbour's, so that the slots'
// lanes read their columns from different banks
constexpr int rows_stride(int d, bool given)
{
    const int floats = tile_rows(d, given) * row_floats(d, given);
    return floats + ((d + 3) / 4 * 4 + 64 - floats % 32) % 32;
}
constexpr int point_stride(int d) { return (d + 3) / 4 * 4; }
constexpr int lds_floats(int d, bool given, int mode)
{
    const int tile = kWave / d * (rows_stride(d, given) + (tile_rows(d, given) + 1) * point_stride(d));
    return threads_of(mode) / kWave * tile + (mode == UNCUT ? 0 : (slots_of(mode, d) + 1) * sums_of(d));
}

// A wavefront's tile: R rows of each of its slots, as they lie in memory, and the R + 1 points around them
// (GIVEN: rows that the kernel of depth 3 left, of d (2 + d) floats)
template <int d, bool GIVEN>
struct Tile {
    static constexpr int D = row_floats(d, GIVEN), SLOTS = kWave / d;
    static constexpr int MAT = D - d * d;                         // where a row's matrix begins
    static constexpr int R = tile_rows(d, GIVEN);
    static constexpr int VECS = R * D / 4;                        // vectors of a slot
    static constexpr int NV = (SLOTS * VECS + kWave - 1) / kWave; // ... that a lane brings
    static constexpr int PX = (R + 1) * d;                        // floats of a slot's points
    static constexpr int NX = (SLOTS * PX + kWave - 1) / kWave;
    static constexpr int STRIDE = rows_stride(d, GIVEN), XS = point_stride(d);
    static constexpr int FLOATS = SLOTS * (STRIDE + (R + 1) * XS);
};

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

template <int d, int MODE, bool GIVEN>
__global__ __launch_bounds__(threads_of(MODE)) __attribute__((amdgpu_waves_per_eu(2))) void sig_stream_depth2_kernel(Args A)
{
    using Tl = Tile<d, GIVEN>;
    using vec_lds = std::conditional_t<Tl::D % 2 == 0, vec4f_8, vec4f_u>;   // (the last vector of fewer than R rows)
    constexpr int NT = threads_of(MODE), WSLOTS = Tl::SLOTS, M = sums_of(d), D = Tl::D, R = Tl::R, XS = Tl::XS;
    const int tid = threadIdx.x, lane = tid % kWave, wave = tid / kWave;
    const int C = MODE == UNCUT ? 1 : A.chunks, W = MODE == UNCUT ? 1 : A.segs, T = MODE == UNCUT ? A.L - 1 : A.steps;
    const int64_t b0 = W > 1 ? blockIdx.x / W : (int64_t)blockIdx.x * A.groups;
    const int seg = W > 1 ? (int)(blockIdx.x - b0 * W) : 0;
    // The workgroup's rows are k0 + 1 .. k1.  Row and point numbers count from `under`, which a stretch's last tile may reach: offsets take 32 bits
    // where those of the whole path do not.
    const int under = W > 1 && seg * A.rows > R ? seg * A.rows - R : 0;
    const int K = A.L - 1 - under;
    const int k0 = W > 1 ? seg * A.rows - under : 0;
    const int k1 = W > 1 && K - k0 > A.rows ? k0 + A.rows : K;
    const int npaths = W > 1 ? 1 : A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;
    const int wslot = lane / d, b = lane - wslot * d;
    const int slot = wave * WSLOTS + wslot;
    const int group = slot / C, chunk = slot - group * C;
    const bool active = wslot < WSLOTS && group < npaths;
    const float *points = A.path + (b0 * A.L + under) * d, *grads = (GIVEN ? A.reduced : A.grad_out) + (b0 * (A.L - 1) + under) * D;
    const float *first = A.path + (b0 + (active ? group : 0)) * A.L * d, *X = first + (int64_t)under * d;
    float *dX = A.grad_path + ((b0 + (active ? group : 0)) * A.L + under) * d;

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
            if (ws < WSLOTS) *reinterpret_cast<vec_lds *>(gtile + ws * Tl::STRIDE + (at < last ? at : last)) = gv[j];
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
        x0[a] = first[a];
    }
    // a row's share of the sums (SUM) and the gradient of its point (SETTLE)
    float above = 0.0f;      // sum_a v_{j+1}[a] A_{j+1}[a b]
    auto row_of = [&](int j, const float *g, const float *x, auto sum, auto settle) __attribute__((always_inline)) {
        constexpr bool SUM = decltype(sum)::value, SETTLE = decltype(settle)::value;
        float row[d], at[XS], before[XS];
        read_floats<d>(row, g + Tl::MAT + b * d);
        read_floats<XS>(at, x + XS);
        float h = g[b], below = 0.0f;
        if constexpr (SUM) start += GIVEN ? g[d + b] : h;
        if constexpr (SETTLE) read_floats<XS>(before, x);
#pragma unroll
        for (int a = 0; a < d; ++a) {
            const float col = g[Tl::MAT + a * d + b], s = at[a] - x0[a];
            m[a] += col - row[a];
            if constexpr (SUM && !GIVEN) start = fmaf(s, row[a], start);
            if constexpr (SETTLE) {
                if constexpr (!GIVEN) h = fmaf(s, col, h);
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

// ------------------------------------------------------------------------------------------
// Depth 3.  With T_j[abc] = sum_{i >= j} G3_i[abc] and v = v_j,
//     P_j[ab] = sum_c v[c] (T_j[cab] - T_j[abc]),      Z_j[b] = sum_a v[a] (P_j[ab] - P_j[ba]),
// the level above adds to the gradient what a problem of depth 2 with the rows
//     e1_j = H_j + Z_{j+1} / 3 + Z_j / 6,      E2_j = G2_j + sum_u S1_j[u] G3_j[u ab] - P_{j+1}
// adds in place of its own (moving a functional from step j + 1 to j conjugates by exp(v_{j+1}); the derivative of the exponential
// brings the rest), with H_j[b] = <G_j, S_j (x) e_b> of all levels and f0_j[b] = <G_j, e_b (x) S_j> (less Z_1 / 3 at j = 1) for point 0.  This kernel
// leaves the rows [e1, f0, E2]; the one above sweeps them.  T is a plain sum over the rows behind as well, so that paths are cut as there.
//
// For eleven and twelve channels, which had the general sweep: (12,3) 46 paths of 71 points 544 -> 60 us, one of 2,000 17,340 -> 154,
// 1,000 of 100 1,096 -> 644; rounding 1.7e-7 to 3.2e-7 of the gradient's norm where that had 2.9e-7 to 4.1e-6.  Bound by latency,
// 0.8 us a row in three barriers.  With fewer channels the sweep on signatures is the faster one on batches ((6,3), 2,011 paths
// of 421 points 374 us and 690; (10,3), 40 of 266 68 and 119).
//
// Lanes.  Lane (a, b) of d * d holds m[c] = T[cab] - T[abc]; a workgroup's slots stage their next R rows of G, level 2 of the rows of
// S (1 / d of the bytes) and their points in LDS.  The sums over a or b of a step go through LDS, R steps at a time.
template <int d>
struct Tile3 {
    static constexpr int Q = d * d, D = d + d * d + d * d * d, MAT = 2 * d + d * d;
    static constexpr int NT = (2 * Q + kWave - 1) / kWave * kWave;             // two slots
    static constexpr int SLOTS = NT / Q;
    static constexpr int R = 2;                                                 // (what LDS holds beside the sums)
    static constexpr int VECS = (R * D + 3) / 4, NV = (SLOTS * VECS + NT - 1) / NT;
    static constexpr int NS = (SLOTS * R * Q + NT - 1) / NT;                   // floats of level 2 of S that a lane brings
    static constexpr int PX = (R + 1) * d, NX = (SLOTS * PX + NT - 1) / NT;
    static constexpr int XS = (d + 3) / 4 * 4;
    static constexpr int STRIDE = VECS * 4, SSTRIDE = (R * Q + 3) / 4 * 4, XSTRIDE = (R + 1) * XS;
    static constexpr int PARK = R * 3 * Q + 2 * Q;
    static constexpr int M = Q * d;
    static constexpr int tile_floats = (SLOTS * (STRIDE + SSTRIDE + XSTRIDE + PARK + 2) + 3) / 4 * 4;
    static constexpr int lds_floats(int mode) { return tile_floats + (mode == UNCUT ? 0 : (SLOTS + 1) * M); }
};

template <int d, int MODE>
__global__ __launch_bounds__((Tile3<d>::NT)) __attribute__((amdgpu_waves_per_eu(2))) void sig_stream_depth3_kernel(Args A)
{
    using Tl = Tile3<d>;
    constexpr int NT = Tl::NT, SLOTS = Tl::SLOTS, Q = Tl::Q, M = Tl::M, D = Tl::D, R = Tl::R, XS = Tl::XS;
    const int tid = threadIdx.x;
    const int K = A.L - 1;
    const int C = MODE == UNCUT ? 1 : A.chunks, W = MODE == UNCUT ? 1 : A.segs, T = MODE == UNCUT ? K : A.steps;
    const int64_t b0 = W > 1 ? blockIdx.x / W : (int64_t)blockIdx.x * A.groups;
    const int seg = W > 1 ? (int)(blockIdx.x - b0 * W) : 0;
    const int k0 = W > 1 ? seg * A.rows : 0;
    const int k1 = W > 1 && K - k0 > A.rows ? k0 + A.rows : K;
    const int npaths = W > 1 ? 1 : A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;
    const int slot = tid / Q, ab = tid - slot * Q, a = ab / d, b = ab - a * d;
    const int group = slot / C, chunk = slot - group * C;
    const bool active = slot < SLOTS && group < npaths;
    const int sl = active ? slot : 0;
    const float *points = A.path + b0 * A.L * d, *grads = A.grad_out + b0 * K * D, *sigs = A.sig + b0 * K * D;
    const float *X = points + (active ? group : 0) * A.L * d;
    float *rows = A.reduced + b0 * K * Tl::MAT;

    float *gtile = sig_stream_gradient_smem, *stile = gtile + SLOTS * Tl::STRIDE, *xtile = stile + SLOTS * Tl::SSTRIDE;
    float *parks = xtile + SLOTS * Tl::XSTRIDE;
    int *tops = reinterpret_cast<int *>(parks + SLOTS * Tl::PARK);   // [SLOTS]: last row of the slot's stretch; then the first one
    float *sums = sig_stream_gradient_smem + Tl::tile_floats, *base = sums + SLOTS * M;
    float *park = parks + sl * Tl::PARK;
    const int have = (K < R ? K : R) * D;              // floats of a slot's rows

    auto low_of = [&](int top, int t0) __attribute__((always_inline)) { return top - t0 > R ? top - t0 - R + 1 : 1; };
    auto row_of = [&](int s, int low) __attribute__((always_inline)) { return s / C < npaths ? s / C * K + low - 1 : 0; };

    vec4f_u gv[Tl::NV];
    float sv[Tl::NS], xv[Tl::NX];
    auto fetch = [&](int t0, auto level2) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Tl::NV; ++j) {
            const int i = tid + j * NT, s = i / Tl::VECS, at = 4 * (i - s * Tl::VECS);
            if (s < SLOTS) {
                const float *src = grads + row_of(s, low_of(tops[s], t0)) * D;
                if (at + 4 <= have) gv[j] = *reinterpret_cast<const vec4f_u *>(src + at);
                else {
#pragma unroll
                    for (int e = 0; e < 4; ++e) gv[j][e] = src[at + e < have ? at + e : 0];
                }
            }
        }
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = tid + j * NT, s = i / Tl::PX, at = i - s * Tl::PX;
            if (s < SLOTS) xv[j] = points[(row_of(s, low_of(tops[s], t0)) + (s / C < npaths ? s / C : 0)) * d + (at < have / D * d + d ? at : 0)];
        }
        if constexpr (decltype(level2)::value) {
#pragma unroll
            for (int j = 0; j < Tl::NS; ++j) {
                const int i = tid + j * NT, s = i / (R * Q), x = i - s * (R * Q), r = x / Q;
                if (s < SLOTS) sv[j] = sigs[(row_of(s, low_of(tops[s], t0)) + (r < K ? r : 0)) * D + d + (x - r * Q)];
            }
        }
    };
    auto put = [&](auto level2) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < Tl::NV; ++j) {
            const int i = tid + j * NT, s = i / Tl::VECS, at = 4 * (i - s * Tl::VECS);
            if (s < SLOTS) *reinterpret_cast<float4 *>(gtile + s * Tl::STRIDE + at) = make_float4(gv[j][0], gv[j][1], gv[j][2], gv[j][3]);
        }
#pragma unroll
        for (int j = 0; j < Tl::NX; ++j) {
            const int i = tid + j * NT, s = i / Tl::PX, x = i - s * Tl::PX;
            if (s < SLOTS) xtile[(s * (R + 1) + x / d) * XS + x % d] = xv[j];
        }
        if constexpr (decltype(level2)::value) {
#pragma unroll
            for (int j = 0; j < Tl::NS; ++j) {
                const int i = tid + j * NT, s = i / (R * Q), x = i - s * (R * Q);
                if (s < SLOTS) stile[s * Tl::SSTRIDE + x] = sv[j];
            }
        }
    };

    float m[d], x0[d];
#pragma unroll
    for (int c = 0; c < d; ++c) {
        m[c] = 0.0f;
        x0[c] = X[c];
    }
    float above = 0.0f, above_a = 0.0f, above_b = 0.0f;   // P_{j+1}[ab], and times v_{j+1}[a], v_{j+1}[b]
    auto first_of = [&](int hi, int c) __attribute__((always_inline)) {
        const int64_t below = (int64_t)hi - (int64_t)(C - c) * T;
        return below > 0 ? (int)below + 1 : 1;
    };
    // the rows of a block, from the last one of every slot down: their sums, or (SETTLE) what they leave for depth 2 as well
    auto walk = [&](int hi, auto settle) __attribute__((always_inline)) {
        constexpr bool SETTLE = decltype(settle)::value;
        __syncthreads();
        if (tid < SLOTS) {
            const int c = tid - tid / C * C;
            const int64_t top = (int64_t)hi - (int64_t)(C - 1 - c) * T;
            tops[tid] = top < K ? (int)top : K;
            tops[SLOTS + tid] = first_of(hi, c);
        }
        __syncthreads();
        const int top = tops[sl], least = tops[SLOTS + sl];
        fetch(0, settle);
        for (int t0 = 0; t0 < T; t0 += R) {
            __syncthreads();
            put(settle);
            __syncthreads();
            if (T - t0 > R) fetch(t0 + R, settle);
            const int low = low_of(top, t0);
#pragma unroll 1
            for (int r = R - 1; r >= 0; --r) {
                const int j = low + r;
                if (!active || j < least || j > top - t0) continue;
                const float *g = gtile + slot * Tl::STRIDE + r * D, *g3 = g + d + Q;
                const float *x = xtile + slot * Tl::XSTRIDE + r * XS;
                float row[d];
                read_floats<d>(row, g3 + ab * d);
                if constexpr (!SETTLE) {
#pragma unroll
                    for (int c = 0; c < d; ++c) m[c] += g3[c * Q + ab] - row[c];
                } else {
                    const float *s2 = stile + slot * Tl::SSTRIDE + r * Q;
                    float at[XS], before[XS];
                    read_floats<XS>(at, x + XS);
                    read_floats<XS>(before, x);
                    const float g2 = g[d + ab], va = x[XS + a] - x[a], vb = x[XS + b] - x[b];
                    float e2 = g2 - above, into_b = (x[XS + a] - X[a]) * g2, from_a = (x[XS + b] - X[b]) * g2, P = 0.0f;
#pragma unroll
                    for (int c = 0; c < d; ++c) {
                        const float col = g3[c * Q + ab];
                        e2 = fmaf(at[c] - x0[c], col, e2);
                        into_b = fmaf(s2[c * d + a], col, into_b);
                        from_a = fmaf(s2[b * d + c], row[c], from_a);
                        m[c] += col - row[c];
                        P = fmaf(at[c] - before[c], m[c], P);
                    }
                    const float pa = va * P, pb = vb * P;
                    park[(r * 3 + 0) * Q + ab] = into_b + fmaf(above_a, 1.0f / 3.0f, pa * (1.0f / 6.0f));
                    park[(r * 3 + 1) * Q + ab] = -fmaf(above_b, 1.0f / 3.0f, pb * (1.0f / 6.0f));
                    park[(r * 3 + 2) * Q + ab] = from_a;
                    if (j == 1) {
                        park[R * 3 * Q + ab] = pa;
                        park[R * 3 * Q + Q + ab] = pb;
                    }
                    rows[(group * K + j - 1) * Tl::MAT + 2 * d + ab] = e2;
                    above = P;
                    above_a = pa;
                    above_b = pb;
                }
            }
            if constexpr (SETTLE) {
                __syncthreads();
                for (int i = tid; i < npaths * C * R * 2 * d; i += NT) {
                    const int s = i / (R * 2 * d), x = i - s * (R * 2 * d), r = x / (2 * d), o = x - r * (2 * d);
                    const int end = tops[s], j = low_of(end, t0) + r;
                    if (j < tops[SLOTS + s] || j > end - t0) continue;
                    const float *p = parks + s * Tl::PARK + r * 3 * Q, *z = parks + s * Tl::PARK + R * 3 * Q;
                    const int e = o < d ? o : o - d;
                    float sum = gtile[s * Tl::STRIDE + r * D + e];
                    if (o < d) {
#pragma unroll
                        for (int c = 0; c < d; ++c) sum += p[c * d + e] + p[Q + e * d + c];
                    } else {
#pragma unroll
                        for (int c = 0; c < d; ++c) sum += p[2 * Q + e * d + c];
                        if (j == 1) {
                            float z1 = 0.0f;
#pragma unroll
                            for (int c = 0; c < d; ++c) z1 += z[c * d + e] - z[Q + e * d + c];
                            sum = fmaf(z1, -1.0f / 3.0f, sum);
                        }
                    }
                    rows[(s / C * K + j - 1) * Tl::MAT + o] = sum;
                }
            }
        }
    };
    constexpr std::true_type yes{};
    constexpr std::false_type no{};

    if constexpr (MODE == UNCUT) {
        walk(K, yes);
    } else {
        for (int e = tid; e < M; e += NT) {
            float sum = 0.0f;
            if constexpr (MODE == CUT)
                for (int w = W - 1; w > seg; --w) sum += A.totals[(b0 * W + w) * M + e];
            base[e] = sum;
        }
        const int span = C * T < k1 - k0 ? C * T : k1 - k0, blocks = (k1 - k0 + span - 1) / span;
        for (int blk = blocks - 1; blk >= 0; --blk) {
            const int hi = k0 + blk * span + C * T;
#pragma unroll
            for (int c = 0; c < d; ++c) m[c] = 0.0f;
            walk(hi, no);
            __syncthreads();
            if (active) {
#pragma unroll
                for (int c = 0; c < d; ++c) sums[slot * M + c * Q + ab] = m[c];
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
                const int top = tops[sl];
                above = above_a = above_b = 0.0f;
                if (active) {
#pragma unroll
                    for (int c = 0; c < d; ++c) m[c] = sums[slot * M + c * Q + ab];
                    if (top < K && top > 0) {
                        const float *x = X + (int64_t)top * d;
#pragma unroll
                        for (int c = 0; c < d; ++c) above = fmaf(x[d + c] - x[c], m[c], above);
                        above_a = (x[d + a] - x[a]) * above;
                        above_b = (x[d + b] - x[b]) * above;
                    }
                }
                walk(hi, yes);
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
    int threads;
    size_t lds;             // bytes of a workgroup
    int64_t grid;
};

// The launches of a cut: whole paths, or (several workgroups a path) their sums first
using Kernel = void (*)(Args);
hipError_t launch_cut(Kernel uncut, Kernel totals, Kernel cut, const Args &A0, const Cut &c, hipStream_t st)
{
    Args A = A0;
    A.chunks = c.chunks;
    A.segs = c.segs;
    A.groups = c.groups;
    A.steps = c.steps;
    A.rows = c.rows;
    const dim3 grid((unsigned)c.grid), threads((unsigned)c.threads);
    if (c.segs > 1) {
        hipLaunchKernelGGL(totals, grid, threads, c.lds, st, A);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    hipLaunchKernelGGL(c.mode == UNCUT ? uncut : cut, grid, threads, c.lds, st, A);
    return hipGetLastError();
}

template <int d, bool GIVEN>
hipError_t launch(const Args &A, const Cut &c, hipStream_t st)
{
    static_assert(lds_floats(d, GIVEN, UNCUT) * sizeof(float) <= (size_t)kMaxLdsBytes, "a wavefront's tile fits its workgroup's LDS");
    static_assert(lds_floats(d, GIVEN, CUT) * sizeof(float) <= (size_t)kMaxLdsBytes, "the tiles and sums of a workgroup's slots fit its LDS");
    return launch_cut(&sig_stream_depth2_kernel<d, UNCUT, GIVEN>, &sig_stream_depth2_kernel<d, TOTALS, GIVEN>, &sig_stream_depth2_kernel<d, CUT, GIVEN>, A, c, st);
}

// Whole paths of K rows of D floats side by side in the slots of a workgroup (W == 0), or W workgroups a path and at most `most_chunks` stretches
// side by side in each.  False where the launch would hold 2^32 threads.
bool cut_rows(int64_t B, int64_t K, int64_t D, int64_t slots, int threads, int64_t W, int64_t most_chunks, Cut *c)
{
    c->threads = threads;
    c->chunks = c->segs = 1;
    c->steps = c->rows = (int)K;
    c->groups = (int)slots;
    if (W == 0) {
        c->mode = UNCUT;
        c->grid = (B + slots - 1) / slots;
        return c->grid * threads < (int64_t)1 << 32;
    }
    c->mode = CUT;
    int64_t rows = (K + W - 1) / W;                       // of a workgroup
    int64_t C = rows < slots ? rows : slots;
    if (C > most_chunks) C = most_chunks;
    int64_t T = (rows + C - 1) / C;
    // a block's rows are read twice, the second time from the caches while few workgroups run together
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
    return c->grid * threads < (int64_t)1 << 32;
}

// UNCUT (W == 0) or CUT; false also where a path has 2^30 points, or a workgroup's rows 2^31 floats
bool cut(int d, bool given, int64_t B, int64_t L, int64_t W, int most_chunks, Cut *c)
{
    const int64_t K = L - 1, D = row_floats(d, given);
    const int mode = W == 0 ? UNCUT : CUT;
    if (L > INT32_MAX / 2 || !cut_rows(B, K, D, slots_of(mode, d), threads_of(mode), W, most_chunks, c)) return false;
    c->tile = tile_rows(d, given);
    c->lds = (size_t)lds_floats(d, given, mode) * sizeof(float);
    return c->groups * (c->segs > 1 ? (int64_t)c->rows + c->tile : mode == UNCUT ? L : K) <= INT32_MAX / D;
}

// Microseconds of a launch, fitted to 16,500 calls (2 to 20 channels, 4 to 2,000 points, 1 to 60,000 paths) with all their cuts, 99,000
// launches: 8 (uncut) and 11 % off in the mean.  The rounds of workgroups, and the bytes, which come a second time from memory where the
// blocks of the workgroups that run together exceed the caches near the units; a stretch that is one tile stays in LDS.  Long stretches cost
// more than the fit has them, hence the last factor.  The choice costs 1.011
// times the best cut in the mean (1.047 before it knew of rounds: 2,631 paths of 255 points of 8 channels uncut 115 us, in eight stretches 67):
// tens of thousands of short paths uncut (16,294 of 135 points of 4
// channels 46 us, the best cut 58), thousands in a few stretches each (1,719 of 97 of 2: uncut 19, 16 stretches 6.3, 96 of them 25),
// one path of 1,445 of 10 across 16 workgroups (uncut 687, one workgroup 72, 16 of them 16).
double microseconds(int d, bool given, int64_t B, int64_t L, int cus, const Cut &c)
{
    const double K = (double)(L - 1), row = row_floats(d, given) * 4e-6, mb = (double)B * K * row, cache = 240.0, chip = cus / 256.0;
    const double within = mb < cache ? mb : cache, beyond = mb - within;
    const int by_lds = held_by_lds(c.lds), by_registers = c.mode != UNCUT ? 3 : d <= 10 ? 16 : 12, held = by_lds < by_registers ? by_lds : by_registers;
    if (c.mode == UNCUT) {
        const double work = 2.22 + 0.1244 * (1.0 + 0.264 * d) * K * rounds_of(c.grid, cus, held, 0.120);
        const double bytes = (within / 5.03 + beyond / 3.47) / chip;
        return std::sqrt(std::sqrt(work * work * work * work + bytes * bytes * bytes * bytes));
    }
    const int64_t span = (int64_t)c.chunks * c.steps, blocks = c.segs > 1 ? c.rows / span : (L - 1 + span - 1) / span;
    const bool stays = c.steps <= c.tile && blocks == 1;
    const double walk = stays ? 0.83 : 0.316 * (1.0 + 0.171 * d) * c.steps;
    const double work = 1.56 + rounds_of(c.grid, cus, held, 0.155) * (double)blocks * (walk + 2.09 + 0.0166 * c.chunks);
    const double together = (double)(c.grid < (int64_t)cus * held ? c.grid : (int64_t)cus * held) * c.groups * (double)span * row;
    const double again = stays || together < 63.0 ? 0.0 : 1.0 - 63.0 / together;
    const double bytes = 1.85 + (within / 3.68 + beyond / 3.40) * (1.0 + 0.60 * again) / chip;
    const double us = std::sqrt(work * work + bytes * bytes) + (c.segs > 1 ? 4.3 + 0.215 * c.segs : 0.0);
    return us * (1.05 + (c.segs == 1 && c.steps > 8 ? 0.084 * std::log2(c.steps / 8.0) : 0.0));
}

bool choose(int d, bool given, int64_t B, int64_t L, int cus, bool scratch, Cut *best)
{
    bool found = false;
    double least = 0.0;
    auto consider = [&](int64_t W, int most_chunks) {
        Cut c;
        if (!cut(d, given, B, L, W, most_chunks, &c)) return;
        const double us = microseconds(d, given, B, L, cus, c);
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

// The same for depth 3
template <int d>
hipError_t launch3(const Args &A, const Cut &c, hipStream_t st)
{
    static_assert(Tile3<d>::lds_floats(CUT) * sizeof(float) <= (size_t)kMaxLdsBytes, "the tiles, parked sums and sums of a workgroup's slots fit its LDS");
    return launch_cut(&sig_stream_depth3_kernel<d, UNCUT>, &sig_stream_depth3_kernel<d, TOTALS>, &sig_stream_depth3_kernel<d, CUT>, A, c, st);
}

int threads3(int d) { return d == 11 ? Tile3<11>::NT : Tile3<12>::NT; }

bool cut3(int d, int64_t B, int64_t L, int64_t W, Cut *c)
{
    const int64_t D = d + d * d + (int64_t)d * d * d, slots = threads3(d) / (d * d);
    const int mode = W == 0 ? UNCUT : CUT;
    c->lds = (size_t)(d == 11 ? Tile3<11>::lds_floats(mode) : Tile3<12>::lds_floats(mode)) * sizeof(float);
    return L <= INT32_MAX / D / slots &&                  // (offsets in the rows of a workgroup's paths)
           cut_rows(B, L - 1, D, slots, threads3(d), W, slots, c);
}

// Workgroups of a path: as many as give every unit one, four rows a workgroup at least ((12,3), 46 paths of 71 points: one 107 us, four 60,
// sixteen 94; one of 2,000 points: one 2,537, 32 of them 154).  Whole batches of tens of thousands of paths are not cut.
bool choose3(int d, int64_t B, int64_t L, int cus, Cut *c)
{
    if (B >= 16 * (int64_t)cus * (threads3(d) / (d * d))) return cut3(d, B, L, 0, c);
    int64_t W = 1;
    while (W < 32 && B * W * 2 <= cus && (L - 1) / (2 * W) >= 4) W *= 2;
    return cut3(d, B, L, W, c);
}

}  // namespace stream_gradient

bool stream_gradient_geometry(int d, int64_t B, int64_t L, int cus, bool scratch, int64_t *scratch_floats, int64_t *grid, int64_t *segs,
                              int64_t *groups, int64_t *chunks, int64_t *steps, int64_t *rows)
{
    stream_gradient::Cut c;
    if (d < 2 || d > stream_gradient::kMostChannels || B <= 0 || L < 2 || !stream_gradient::choose(d, false, B, L, cus, scratch, &c)) return false;
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
    if (d < 2 || d > stream_gradient::kMostChannels || !stream_gradient::choose(d, false, B, L, cus, true, &c)) return -1;
    return c.segs > 1 ? B * c.segs * stream_gradient::sums_of(d) : 0;
}

int stream_gradient_segments(int d, int depth, int64_t B, int64_t L, int cus)
{
    using namespace stream_gradient;
    Cut c;
    if (B <= 0 || L < 2 || d < 2) return 0;
    if (depth == 2) return d <= kMostChannels && choose(d, false, B, L, cus, true, &c) ? c.segs : 0;
    return depth == 3 && stream_gradient3_scratch_floats(d, B, L, cus) >= 0 && choose3(d, B, L, cus, &c) ? c.segs : 0;
}

int64_t stream_gradient3_scratch_floats(int d, int64_t B, int64_t L, int cus)
{
    using namespace stream_gradient;
    Cut c3, c2;
    if (d < 11 || d > 12 || B < 1 || L < 2 || !choose3(d, B, L, cus, &c3) || !choose(d, true, B, L, cus, true, &c2)) return -1;
    const int64_t D = row_floats(d, true), rows = B * (L - 1);
    if (rows > INT64_MAX / 16 / D) return -1;
    const int64_t sums3 = c3.segs > 1 ? B * c3.segs * d * d * d : 0, sums2 = c2.segs > 1 ? B * c2.segs * sums_of(d) : 0;
    return (rows * D + 3) / 4 * 4 + (sums3 > sums2 ? sums3 : sums2);
}

hipError_t launch_stream_gradient3(const float *path, const float *sig, const float *grad_out, float *grad_path, float *scratch, int64_t B,
                                   int64_t L, int d, int cus, hipStream_t st)
{
    using namespace stream_gradient;
    Cut c3, c2;
    if (!scratch || d < 11 || d > 12 || B < 1 || L < 2 || !choose3(d, B, L, cus, &c3) || !choose(d, true, B, L, cus, true, &c2)) return hipErrorInvalidValue;
    Args A{};
    A.path = path;
    A.sig = sig;
    A.grad_out = grad_out;
    A.grad_path = grad_path;
    A.reduced = scratch;
    A.totals = scratch + (B * (L - 1) * row_floats(d, true) + 3) / 4 * 4;
    A.B = B;
    A.L = (int32_t)L;
    const hipError_t e = d == 11 ? launch3<11>(A, c3, st) : launch3<12>(A, c3, st);
    if (e != hipSuccess) return e;
    return d == 11 ? launch<11, true>(A, c2, st) : launch<12, true>(A, c2, st);
}

hipError_t launch_stream_gradient(const float *path, const float *grad_out, float *grad_path, float *scratch, int64_t B, int64_t L,
                                  int d, int cus, hipStream_t st)
{
    using namespace stream_gradient;
    Cut c;
    if (B <= 0 || L < 2 || d < 2 || d > kMostChannels) return hipErrorInvalidValue;
    if (!choose(d, false, B, L, cus, scratch != nullptr, &c)) return hipErrorNotSupported;
    Args A{};
    A.path = path;
    A.grad_out = grad_out;
    A.grad_path = grad_path;
    A.totals = scratch;
    A.B = B;
    A.L = (int32_t)L;
    switch (d) {
#define SIG_STREAM_GRADIENT(d_) case d_: return launch<d_, false>(A, c, st);
    SIG_STREAM_GRADIENT(2) SIG_STREAM_GRADIENT(3) SIG_STREAM_GRADIENT(4) SIG_STREAM_GRADIENT(5) SIG_STREAM_GRADIENT(6)
    SIG_STREAM_GRADIENT(7) SIG_STREAM_GRADIENT(8) SIG_STREAM_GRADIENT(9) SIG_STREAM_GRADIENT(10) SIG_STREAM_GRADIENT(11)
    SIG_STREAM_GRADIENT(12) SIG_STREAM_GRADIENT(13) SIG_STREAM_GRADIENT(14) SIG_STREAM_GRADIENT(15) SIG_STREAM_GRADIENT(16)
    SIG_STREAM_GRADIENT(17) SIG_STREAM_GRADIENT(18) SIG_STREAM_GRADIENT(19) SIG_STREAM_GRADIENT(20)
#undef SIG_STREAM_GRADIENT
    default: return hipErrorInvalidValue;
    }
}

}  // namespace sig
