// Launch of the final-mode gradient on Lie brackets (sig_bracket.h): compiled shapes, and how a call is cut.
#include "sig_bracket.h"

namespace sig {
namespace bracket {

// bytes of LDS a launch of these kernels asks for at most: two workgroups of the largest rows still share a compute unit
constexpr int kMaxLds = kCuLdsBytes / 2;
constexpr int kMaxChunks = 64;
constexpr int kMinChunkSteps = 4;

template <typename Kernel>
hipError_t allow_lds(Kernel kernel, size_t bytes)
{
    if (bytes <= (size_t)kMaxLdsBytes) return hipSuccess;
    return hipFuncSetAttribute(reinterpret_cast<const void *>(kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
}

// Whole paths packed into wavefronts, or a workgroup per path?  Packed, a path costs a third of the instructions, but its
// steps follow one another, 0.2 us each; cut into chunks it is done in 8 to 30 us, of one of some thousand resident
// workgroups.  Microseconds fitted to both kernels on 18 shapes x 9 ... 100 points x 1,024 ... 32,768 paths; they cross at
// some 3,000 paths of 100 points ((5,4): 1,024 paths 26 and 13 us, 8,192 paths 37 and 88).  Rows of more than 3,000 floats
// leave a wavefront's LDS room for few others on the compute unit: they stay cut ((8,4): 1.0-1.3x at every batch).
template <class G>
bool packed_wanted(const Args &A)
{
    const double K = (double)(A.L - 1), thousands = (double)A.B / 1000.0;
    const double cut_step = G::N == 3 ? 0.002 + 0.0008 * G::LQ : G::N == 4 ? 0.01 + 0.003 * G::LQ : 0.02 + 0.005 * G::LQ;
    const double cut = 4.0 + thousands * (2.0 + G::D / 250.0 + cut_step * K);
    const double packed = 3.0 + G::D / 250.0 + 0.2 * K + thousands * (G::D / 650.0 + 0.0016 * G::LQ * K);
    return packed < cut && A.L * G::PG * G::d <= INT32_MAX;
}

// chunks the threads and the LDS of a workgroup hold
template <class G>
int most_chunks()
{
    int C = G::CT / G::LQ;
    if (C > kMaxChunks) C = kMaxChunks;
    while (C > 1 && chunked_lds_floats<G>(C) * (int64_t)sizeof(float) > kMaxLds) --C;
    return C;
}

// Slots that fold what lies behind a workgroup: two dozen steps each, as far as the threads hold them and their rows leave as
// many workgroups resident as before.  (6,5), one path of 2,000 points: 2 slots 281 us, 13 slots 80.
template <class G>
int fold_slots(int C, int64_t K)
{
    if constexpr (G::FN <= 2) return C;
    else {
        const int64_t now = chunked_lds_floats<G>(C) * (int64_t)sizeof(float);
        int64_t most = kCuLdsBytes / (kCuLdsBytes / now) - 2048;   // (short of the step in which LDS is handed out)
        if (most > kMaxLds) most = kMaxLds;
        int64_t slots = G::CT / G::QF;
        if (slots > kMaxChunks) slots = kMaxChunks;
        if (slots > K / 24) slots = K / 24;
        while (slots > C && chunked_lds_floats<G>(C, (int)slots) * (int64_t)sizeof(float) > most) --slots;
        return slots > C ? (int)slots : C;
    }
}

template <int d, int N, int P>
hipError_t launch(const Args &A0, int cus, hipStream_t st)
{
    using G = Geo<d, N, P>;
    Args A = A0;
    if (A.B <= 0 || A.L < 2) return hipErrorInvalidValue;
    const int64_t K = A.L - 1;
    if constexpr (G::LQ <= kWave && G::D <= 3000) {
        if (packed_wanted<G>(A)) {
            constexpr size_t lds = (size_t)packed_lds_floats<G>() * sizeof(float);
            static_assert(lds <= (size_t)kMaxLdsBytes, "a wavefront's paths fit its workgroup's LDS");
            // as many paths per wavefront as leave every SIMD two wavefronts (the paths' bracket values follow one another:
            // (2,6), 20 points, 8,192 paths 23 us with full wavefronts, 12.6 with four paths each)
            int64_t groups = (A.B + 8 * cus - 1) / (8 * cus);
            if (groups > G::PG) groups = G::PG;
            A.groups = (int32_t)groups;
            const int64_t grid = (A.B + groups - 1) / groups;
            if (grid > INT32_MAX) return hipErrorInvalidValue;
            hipLaunchKernelGGL((sig_bracket_packed_kernel<d, N, P>), dim3((unsigned)grid), dim3(kWave), lds, st, A);
            return hipGetLastError();
        }
    }
    const int W = A.segs < 1 ? 1 : A.segs;
    constexpr int threads = G::CT;
    // chunks of at least four steps: below that the scan over the chunks costs more than the steps it saves
    int64_t C = most_chunks<G>();
    if (C * W * kMinChunkSteps > K) C = K / (W * kMinChunkSteps);
    if (C < 1) C = 1;
    if (K / (C * W) > INT32_MAX - 1024) return hipErrorInvalidValue;
    A.chunks = (int32_t)C;
    A.steps = (int32_t)((K + C * W - 1) / (C * W));
    A.segs = (int32_t)((K + C * A.steps - 1) / (C * A.steps));   // no workgroup is left without steps
    A.fold_slots = A.segs > 1 ? fold_slots<G>((int)C, K) : (int32_t)C;
    const size_t lds = (size_t)chunked_lds_floats<G>((int)C, A.fold_slots) * sizeof(float);
    if (lds > (size_t)kMaxLds || C * G::LQ > threads || A.B * A.segs > INT32_MAX) return hipErrorInvalidValue;
    hipError_t e = allow_lds(&sig_bracket_chunked_kernel<d, N, P>, lds);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL((sig_bracket_chunked_kernel<d, N, P>), dim3((unsigned)(A.B * A.segs)), dim3(threads), lds, st, A);
    return hipGetLastError();
}

// How a depth-2 launch is cut: a point per thread, twice over where the batch fills the chip anyway; whole short paths side
// by side, as far as 16 KB of LDS hold their matrices.  A launch holds fewer than 2^32 threads: beyond, more points each.
template <int d>
bool cut_depth2(Args &A, int cus, int64_t *grid)
{
    constexpr int64_t kMostWorkgroups = ((int64_t)1 << 32) / kDepth2Threads - 1;
    int64_t want = A.B * A.L >= (int64_t)cus * 8 * kDepth2Threads * 4 ? 2 * kDepth2Threads : kDepth2Threads;
    for (; want <= (int64_t)1 << 24; want *= 2) {
        A.segs = 1;
        A.groups = 1;
        if (A.L >= want) {
            const int64_t segs = (A.L + want - 1) / want;
            if (segs > kMostWorkgroups / A.B) continue;
            A.steps = (int32_t)want;
            A.segs = (int32_t)segs;
            *grid = A.B * segs;
        } else {
            int64_t paths = want / A.L;
            const int64_t by_lds = 16384 / (depth2_floats<d>(1) * (int64_t)sizeof(float));
            if (paths > by_lds) paths = by_lds;
            if (paths < 1) paths = 1;
            A.groups = (int32_t)paths;
            *grid = (A.B + paths - 1) / paths;
        }
        if (*grid <= kMostWorkgroups) return true;
    }
    return false;
}

template <int d>
hipError_t launch_depth2(const Args &A0, int cus, hipStream_t st)
{
    Args A = A0;
    int64_t grid = 0;
    if (A.B <= 0 || A.L < 2 || !cut_depth2<d>(A, cus, &grid)) return hipErrorInvalidValue;
    const size_t lds = (size_t)depth2_floats<d>(A.groups) * sizeof(float);
    hipLaunchKernelGGL((sig_bracket_depth2_kernel<d>), dim3((unsigned)grid), dim3(kDepth2Threads), lds, st, A);
    return hipGetLastError();
}

template <int d>
bool depth2_geometry(Args &A, int cus, int64_t *grid, int64_t *lds_bytes)
{
    if (!cut_depth2<d>(A, cus, grid)) return false;
    *lds_bytes = depth2_floats<d>(A.groups) * (int64_t)sizeof(float);
    return true;
}

struct Entry {
    int d, depth;
    int chunks;      // of a workgroup (0: the kernel of depth 2, which is not cut this way)
    int64_t row;     // D
    hipError_t (*launch)(const Args &, int, hipStream_t);
};
#define SIG_BRACKET_SHAPES(X)                                                                                          \
    X(2, 3, 2) X(3, 3, 2) X(4, 3, 2) X(5, 3, 2) X(6, 3, 2) X(7, 3, 2) X(8, 3, 2) X(9, 3, 2) X(10, 3, 2)                \
    X(11, 3, 2) X(12, 3, 2) X(13, 3, 2) X(14, 3, 2) X(15, 3, 2) X(16, 3, 2)                                            \
    X(2, 4, 2) X(3, 4, 2) X(4, 4, 2) X(5, 4, 2) X(6, 4, 2) X(7, 4, 2) X(8, 4, 2) X(9, 4, 2) X(10, 4, 2)                \
    X(2, 5, 3) X(3, 5, 2) X(4, 5, 3) X(5, 5, 3) X(6, 5, 3) X(2, 6, 3) X(3, 6, 3) X(4, 6, 3)
#define SIG_BRACKET_ENTRY(d, N, P) {d, N, most_chunks<Geo<d, N, P>>(), Geo<d, N, P>::D, &launch<d, N, P>},
#define SIG_BRACKET_DEPTH2(X) X(2) X(3) X(4) X(5) X(6) X(7) X(8) X(9) X(10) X(11) X(12) X(13) X(14) X(15) X(16) X(17) X(18) X(19) X(20)
#define SIG_BRACKET_DEPTH2_ENTRY(d) {d, 2, 0, d + d * d, &launch_depth2<d>},
#define SIG_BRACKET_DEPTH2_GEOMETRY(d_) case d_: return depth2_geometry<d_>(A, cus, grid, lds_bytes);
const Entry kEntries[] = {SIG_BRACKET_DEPTH2(SIG_BRACKET_DEPTH2_ENTRY) SIG_BRACKET_SHAPES(SIG_BRACKET_ENTRY){0, 0, 0, 0, nullptr}};

bool depth2_geometry_of(int d, Args &A, int cus, int64_t *grid, int64_t *lds_bytes)
{
    switch (d) {
        SIG_BRACKET_DEPTH2(SIG_BRACKET_DEPTH2_GEOMETRY)
    default: return false;
    }
}

const Entry *find(int d, int depth)
{
    if (!bracket_compiled(d, depth)) return nullptr;
    for (const Entry *e = kEntries; e->launch; ++e)
        if (e->d == d && e->depth == depth) return e;
    return nullptr;
}

}  // namespace bracket

// Cutting a path across workgroups shortens the walk of its chunks, but every workgroup forms the bracket values again and
// folds everything behind it: from two dozen steps a chunk on while there are few paths, twice that for more than 32, at
// most four workgroups per compute unit, and not where the rows that are read again exceed four megabytes.  Uncut and cut:
// (9,3), five paths of 1,221 points 32.5 and 6.4 us; (10,4), one path of 1,000 points 123 and 47; (5,4), 128 paths of 2,000
// points 45 and 36; (6,5), 112 paths of 500 points 153 and 96.
int bracket_segments(int d, int depth, int64_t B, int64_t L, int cus)
{
    const bracket::Entry *e = bracket::find(d, depth);
    if (!e || e->chunks <= 0 || B <= 0 || B * e->row > ((int64_t)1 << 20)) return 1;
    const int64_t steps = (L - 1 + e->chunks - 1) / e->chunks;
    int64_t W = steps / (B > 32 ? 27 : 12);
    if (W > 4 * (int64_t)cus / B) W = 4 * (int64_t)cus / B;
    if (W > 32) W = 32;
    return W < 2 ? 1 : (int)W;
}

// the launch of the depth-2 gradient, for tests of the host side: workgroups, stretches and paths of each, bytes of LDS
bool bracket_depth2_geometry(int d, int64_t B, int64_t L, int cus, int64_t *grid, int64_t *segs, int64_t *steps, int64_t *groups,
                             int64_t *lds_bytes)
{
    bracket::Args A{};
    A.B = B;
    A.L = L;
    const bool ok = B > 0 && L >= 2 && bracket::depth2_geometry_of(d, A, cus, grid, lds_bytes);
    *segs = A.segs;
    *steps = A.steps;
    *groups = A.groups;
    return ok;
}

hipError_t launch_bracket(const float *path, const float *sig, const float *grad_out, float *grad_path, int64_t B, int64_t L,
                          int d, int depth, int segs, int cus, hipStream_t st)
{
    const bracket::Entry *e = bracket::find(d, depth);
    if (!e) return hipErrorInvalidValue;
    bracket::Args A{};
    A.path = path;
    A.sig = sig;
    A.grad_out = grad_out;
    A.grad_path = grad_path;
    A.B = B;
    A.L = L;
    A.segs = segs;
    return e->launch(A, cus, st);
}

}  // namespace sig
