// Stream mode of shapes whose words of length N - 1 do not fit a workgroup (compiled per (d, depth N)).
//
// A lane owns one word of length N - 1 and its d children, as in sig_stream_rows.h, and a step needs nothing from other lanes: the
// words of a path are split into slices, a workgroup each, which fold the path's increments one after the other and write their part
// of every row.  A path is also cut into W stretches: a first launch leaves the signatures of all but the last in scratch, and
// a workgroup of the second one multiplies those before its own into its lanes (Eq. 4 with the left factor in registers needs no
// other lane either).  Where scratch cannot be had, it folds what lies before its stretch again.
//
// Bound by the stores where the batch fills the chip.  What decides their rate is how close in time neighbouring lines are
// written: a wavefront's run of the longest level (64 d floats) goes through LDS so that it is stored in whole lines, all
// slices of a stretch run on one XCD, and the wavefronts of a workgroup meet at a barrier every kTile steps ((9,4), 154 paths of
// 631 points, 521 us at the rate of a copy: kTile 32, 256 threads 841 us; slices on one XCD 707; kTile 16 661, 8 569; a whole
// path in one workgroup 530).  Bound by latency on few paths (0.4 us a row, 0.16 a step of a piece, 0.8 a product).
// By the counters the rows are written once, at 4.8 to 5.8 TB/s of all that moves, with the LDS busy a quarter.
// Measured against what these calls took before (the register kernels, or one launch per level), us, one MI355X, both in turn: (10,4) 319 paths of 203
// points 1,000 and 618, 9 of 1,693 657 and 190, one of 1,423 250 and 57; (6,5) 24 of 1,591 1,830 and 355, 218 of 177 431 and
// 279; (5,5) 178 of 514 527 and 302; (4,6) 202 of 650 760 and 569.
//
// Rounding: steps are summed in blocks of kTile, each from zero, and level 1 is the distance between two points: 1.0e-7 to 1.7e-7 where
// those calls had 1.4e-7 to 6.6e-7 (20 calls of 100 to 1,700 points, against 64 bits).
#ifndef SIG_SPLIT_ROWS_H
#define SIG_SPLIT_ROWS_H

#include "sig_stream_rows.h"

namespace sig {
namespace split {

using onchip::cpow;
using onchip::vec4f_u;
using rows::add_state;
using rows::level1_of;
using rows::summed_step;

struct Args {
    const float *path;   // [B][L][d]
    float *out;          // [B][L-1][D]
    int64_t B, L;
    float *pieces;       // [B][W - 1][D]: signatures of the stretches but for the last; null: every workgroup folds what lies before it
    int32_t segs;        // W: stretches of a path, each a workgroup for every slice
    int32_t rows;        // of a stretch, a multiple of kTile; W * rows >= L - 1
    int32_t slices;      // workgroups that the words of a path are split across
    int32_t lanes;       // words of each of them
    int32_t sticky;      // a point that is not a number spoils level 1 of the rows behind it too
};

constexpr int kTile = 8;         // steps staged in LDS together, and summed from zero
constexpr int kMaxThreads = 1024;
constexpr unsigned kXcds = 8;

template <int d_, int N_>
struct Geo {
    static constexpr int d = d_, N = N_, P = N - 1;
    static constexpr int Q = cpow(d, P);
    static constexpr int D = onchip::Shape<d, N, P>::D;
    static constexpr bool LINEAR = d != 4;                               // (four children are one 16-byte store)
    static constexpr int RUN = kWave * d;                                // floats of a wavefront's run
    static constexpr int TILE = (kTile + 1) * d;
    static constexpr int TS = (TILE + 3) / 4 * 4;
};
template <int d, int N>
constexpr int lds_floats(int threads) { return 2 * Geo<d, N>::TS + (Geo<d, N>::LINEAR ? threads / kWave * Geo<d, N>::RUN : 0); }

extern __shared__ __align__(16) float sig_split_smem[];

// PIECES: the signatures of the stretches, into A.pieces, instead of their rows
template <int d, int N, bool PIECES>
__global__ __launch_bounds__(kMaxThreads) __attribute__((amdgpu_waves_per_eu(4))) void sig_split_rows_kernel(Args A)
{
    using G = Geo<d, N>;
    using Lane = onchip::Lane<d, N, N - 1>;
    using Sh = onchip::Shape<d, N, N - 1>;
    constexpr int P = G::P, D = G::D, TS = G::TS;
    float *const smem = sig_split_smem;
    const int tid = threadIdx.x, nthr = blockDim.x, lane = tid % kWave, wave = tid / kWave;
    const int64_t K = A.L - 1;
    // The slices of a stretch run on one XCD (workgroups go to the eight of them in turn), so that the lines that two slices share
    // meet in one L2: (10,4), 319 paths of 203 points 822 -> 654 us.
    const unsigned slices = (unsigned)A.slices;
    const int W = PIECES ? A.segs - 1 : A.segs;
    const unsigned units = gridDim.x / slices, full = units / kXcds * kXcds;
    unsigned unit = blockIdx.x / slices, slice = blockIdx.x - unit * slices;
    if (unit < full) {
        const unsigned turn = blockIdx.x / kXcds;
        unit = turn / slices * kXcds + blockIdx.x % kXcds;
        slice = turn % slices;
    }
    const int64_t b = unit / (unsigned)W;
    const int w = (int)(unit - (unsigned)b * (unsigned)W);
    const int64_t k0 = (int64_t)w * A.rows, k1 = K - k0 < A.rows ? K : k0 + A.rows;   // rows k0 .. k1 - 1
    const int first = (int)slice * A.lanes, last = first + A.lanes < G::Q ? first + A.lanes : G::Q;
    const int mine = first + tid;
    const bool active = mine < last;
    const unsigned u = active ? (unsigned)mine : (unsigned)(last - 1);
    int letter[P];
    {
        unsigned rest = u;
#pragma unroll
        for (int m = P - 1; m >= 0; --m) { letter[m] = (int)(rest % d); rest /= d; }
    }
    const float *X = A.path + b * A.L * d;
    const float first1 = X[(PIECES ? k0 * d : 0) + letter[0]];   // level 1 is the distance from this point,
    float spoilt = 0.0f;   // not a number behind a point that is none (sticky; infinite points too, but that first one: the distance from it stays infinite)

    constexpr int NV = (G::TILE + kWave - 1) / kWave;   // (of a wavefront alone)
    float next[NV];
    auto fetch = [&](int64_t k) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int64_t at = k * d + tid + j * nthr;
            if (tid + j * nthr < G::TILE) next[j] = X[at < A.L * d ? at : 0];
        }
    };
    // The run of this wavefront's lanes in the longest level goes through LDS: a row's is read back while the next step is worked out
    // and stored behind it.  (wave_order: LDS keeps the order of a wavefront's accesses, and so has the compiler to.)
    constexpr int RV = (G::RUN / 4 + kWave - 1) / kWave;
    float *run = smem + 2 * TS + wave * G::RUN;
    const int from = first + wave * kWave, total = (last - from < kWave ? last - from : kWave) * d;   // (below 0: a wavefront without lanes)
    auto wave_order = [&]() __attribute__((always_inline)) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
    };
    vec4f_u held[G::LINEAR ? RV : 1];
    auto read_back = [&]() __attribute__((always_inline)) {
        if constexpr (G::LINEAR) {
#pragma unroll
            for (int j = 0; j < RV; ++j) {
                const int i = 4 * (lane + j * kWave);
                held[j] = *reinterpret_cast<const vec4f_u *>(run + (i < G::RUN ? i : 0));
            }
        }
    };
    auto write_back = [&](float *row) __attribute__((always_inline)) {
        if constexpr (G::LINEAR) {
            float *dst = row + Sh::row_off(N) + from * d;
#pragma unroll
            for (int j = 0; j < RV; ++j) {
                const int i = 4 * (lane + j * kWave);
                if (i + 4 <= total) *reinterpret_cast<vec4f_u *>(dst + i) = held[j];
                else if (i < total)
                    for (int e = 0; e < total - i; ++e) dst[i + e] = held[j][e];
            }
        }
    };
    auto put = [&](float *row, const Lane &now) __attribute__((always_inline)) {
        if constexpr (!G::LINEAR) {
            if (active) onchip::store_state<d, N, P>(row, u, now);
        } else {
            constexpr int V = d % 4 == 0 ? 4 : d % 2 == 0 ? 2 : 1;
            typedef float vec __attribute__((ext_vector_type(V)));
            wave_order();
#pragma unroll
            for (int a = 0; a < d; a += V) {
                if constexpr (V == 1) run[lane * d + a] = now.s[1 + a];
                else {
                    vec v;
#pragma unroll
                    for (int j = 0; j < V; ++j) v[j] = now.s[1 + a + j];
                    *reinterpret_cast<vec *>(run + lane * d + a) = v;
                }
            }
            wave_order();
            if (active) {
                row[Sh::row_off(P) + u] = now.s[0];
                onchip::static_for<1, P>([&](auto mc) __attribute__((always_inline)) {
                    constexpr int m = decltype(mc)::value;
                    constexpr unsigned span = cpow(d, P - m);
                    if (u % span == 0) row[Sh::row_off(m) + u / span] = now.pre[m - 1];
                });
            }
        }
    };

    Lane ln;
    onchip::identity_state<d, N, P>(ln);
    // the stretches before: their signatures one after the other, or folded again
    const bool refold = !PIECES && !A.pieces;
    if (!PIECES && A.pieces && w > 0) {
        const float *piece = A.pieces + b * (W - 1) * D;
        onchip::load_state<d, N, P>(piece, u, ln);
        for (int s = 1; s < w; ++s) onchip::reg_product<d, N, P>(ln, piece + (int64_t)s * D, u);
        const float here1 = X[k0 * d + letter[0]];
        if (A.sticky) spoilt = fmaf(0.0f, here1, ln.pre[0] != ln.pre[0] ? ln.pre[0] : 0.0f);
        ln.pre[0] = level1_of(here1 - first1, ln.pre[0], A.sticky);
    }
    float *const rows0 = PIECES ? nullptr : A.out + (b * K + k0) * D;
    float *out = rows0;
    const int64_t start = refold ? 0 : k0;
    fetch(start);
    int buf = 0;
    for (int64_t k = start; k < k1; k += kTile) {
        float *tile = smem + buf * TS;
        buf ^= 1;
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (tid + j * nthr < G::TILE) tile[tid + j * nthr] = next[j];
        if (k + kTile < k1) fetch(k + kTile);
        __syncthreads();
        const int count = k1 - k < kTile ? (int)(k1 - k) : kTile;
        auto steps = [&](auto emit) __attribute__((always_inline)) {
            rows::Steps<d, P, true, true> it(tile, letter);
            onchip::Inc<d, P> inc;
            Lane sum, now = ln;
            onchip::identity_state<d, N, P>(sum);
#pragma unroll 2
            for (int t = 0; t < count; ++t) {
                if constexpr (decltype(emit)::value) read_back();
                it.next(inc);
                summed_step<d, N>(sum, now, inc);
                add_state<d, N, P>(now, ln, sum);
                now.pre[0] = it.last.du[0] - first1 + spoilt;
                if (A.sticky) spoilt = fmaf(0.0f, it.last.du[0], spoilt);
                if constexpr (decltype(emit)::value) {
                    if (out != rows0) write_back(out - D);
                    put(out, now);
                    out += D;
                }
            }
            add_state<d, N, P>(ln, ln, sum);
            ln.pre[0] = now.pre[0];
        };
        if (!PIECES && k >= k0) steps(std::true_type{});
        else steps(std::false_type{});
    }
    if constexpr (!PIECES) {
        read_back();
        write_back(out - D);
    } else {
        if (active) onchip::store_state<d, N, P>(A.pieces + (b * W + w) * D, u, ln);
    }
}

}  // namespace split
}  // namespace sig

#endif  // SIG_SPLIT_ROWS_H
