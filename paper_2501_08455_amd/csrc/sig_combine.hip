// Batched truncated product of Eq. 4 on dense rows, compiled per (d, depth N).
//
// Number the words of a row by their place in the d-ary tree of words: the root is node 0 and the children of node h are
// the nodes h d + 1 ... h d + d, so the children of h are the d consecutive floats at h d of the row (level 0 is not
// stored), the last letter of h is (h - 1) mod d and its parent (h - 1) / d.  One work item is a node h of levels 0 .. N-1
// with its d children; the children's words
//     c[h k] = a[h k] + b[h k] + sum over splits h = u x, u not empty, of a[u] b[x k],   k = 0 .. d-1,
// share a[u] and read d consecutive floats of b, and going from one split to the next is a constant division: some 10
// instructions per word in place of 40 for finding every split of every word by itself.  Rows follow each other without a
// gap, so item i of a batch owns the floats i d ... i d + d - 1 of the batch whatever row they are in.
//
// Bound by reading a and b and writing c once.  a + b and c therefore move in fours of consecutive floats, whatever the
// row length, and are turned into items in LDS, where an item's own floats are read and written by its thread alone
// (in place, no barrier between).  The levels below the top one of a and b are staged beside them, through the cache.
// Measured, a thread per word (sig_streaming.hip) against this: 65,536 products of (5,4) rows 171 -> 117 us (5.3 TB/s of what
// must move), 30,000 of (12,3) 166 -> 122 (5.6), 8,000 of (10,4) 279 -> 205, 5,000 of (6,5) 172 -> 114, 20,000 of (2,6) 21 -> 9.6,
// 65,536 of (20,2) 78 -> 64.
#include "sig_internal.h"
#include "sig_onchip.h"

namespace sig {
namespace combine {

using onchip::cpow;
using onchip::geom;
using onchip::vec4f_u;

template <int d_, int N_>
struct Geo {
    static_assert(N_ >= 2 && d_ >= 2, "a row has levels below its top one");
    static constexpr int d = d_, N = N_;
    static constexpr int NODES = geom(d, N);      // items of a row
    static constexpr int LOW = NODES - 1;         // floats of levels 1 .. N-1
    static constexpr int D = NODES * d;
    static constexpr int threads = D > 3584 ? 512 : 256;
    // Rows of a workgroup, within 3,584 floats: the number whose items leave the fewest threads idle in the last pass, the
    // larger of two equals.
    static constexpr int pick_rows()
    {
        int best = 1;
        double best_use = 0.0;
        for (int r = 1; r * D <= 3584; ++r) {
            const int items = r * NODES, passes = (items + threads - 1) / threads;
            const double use = (double)items / (double)(passes * threads);
            if (r * D >= 1536 && use >= best_use) { best = r; best_use = use; }
            else if (r * D < 1536) best = r;
        }
        return best;
    }
    static constexpr int R = pick_rows();
    // x / d for x < NODES by a 24-bit multiply: exact while x (M d - 2^18) < 2^18
    static constexpr uint32_t M = ((1u << 18) + d - 1) / d;
    static_assert((int64_t)NODES * (int64_t)(M * d - (1u << 18)) < (1 << 18) && (int64_t)NODES * M < ((int64_t)1 << 32),
                  "division by a multiply");
    static constexpr int lds_s = (R * D + 3) & ~3, lds_low = (R * LOW + 3) & ~3;
    static_assert((lds_s + 2 * lds_low) * (int)sizeof(float) <= 64 * 1024, "two workgroups on a compute unit at least");
};

// d consecutive floats of LDS whose index is a multiple of d
template <int d>
__device__ __forceinline__ void read_group(float (&v)[d], const float *s)
{
    if constexpr (d % 4 == 0) {
#pragma unroll
        for (int i = 0; i < d / 4; ++i) {
            const float4 q = reinterpret_cast<const float4 *>(s)[i];
            v[4 * i] = q.x; v[4 * i + 1] = q.y; v[4 * i + 2] = q.z; v[4 * i + 3] = q.w;
        }
    } else if constexpr (d % 2 == 0) {
#pragma unroll
        for (int i = 0; i < d / 2; ++i) {
            const float2 q = reinterpret_cast<const float2 *>(s)[i];
            v[2 * i] = q.x; v[2 * i + 1] = q.y;
        }
    } else {
#pragma unroll
        for (int i = 0; i < d; ++i) v[i] = s[i];
    }
}

template <int d>
__device__ __forceinline__ void write_group(float *s, const float (&v)[d])
{
    if constexpr (d % 4 == 0) {
#pragma unroll
        for (int i = 0; i < d / 4; ++i)
            reinterpret_cast<float4 *>(s)[i] = make_float4(v[4 * i], v[4 * i + 1], v[4 * i + 2], v[4 * i + 3]);
    } else if constexpr (d % 2 == 0) {
#pragma unroll
        for (int i = 0; i < d / 2; ++i) reinterpret_cast<float2 *>(s)[i] = make_float2(v[2 * i], v[2 * i + 1]);
    } else {
#pragma unroll
        for (int i = 0; i < d; ++i) s[i] = v[i];
    }
}

template <int d, int N>
__global__ __launch_bounds__((Geo<d, N>::threads)) void sig_combine_tree_kernel(const float *__restrict__ a, const float *__restrict__ b,
                                                                              float *__restrict__ out, int64_t rows, int per_wg)
{
    using G = Geo<d, N>;
    constexpr int T = G::threads;
    __shared__ __attribute__((aligned(16))) float sum[G::lds_s];     // a + b, then the product
    __shared__ __attribute__((aligned(16))) float la[G::lds_low];    // levels 1 .. N-1 of a
    __shared__ __attribute__((aligned(16))) float lb[G::lds_low];    // ... of b
    const int tid = threadIdx.x;
    const int64_t row0 = (int64_t)blockIdx.x * per_wg;
    const int nr = rows - row0 < per_wg ? (int)(rows - row0) : per_wg;
    const int n = nr * G::D, n4 = n >> 2;
    a += row0 * G::D;
    b += row0 * G::D;
    out += row0 * G::D;
#pragma unroll 4
    for (int q = tid; q < n4; q += T) {
        const vec4f_u x = *reinterpret_cast<const vec4f_u *>(a + 4 * q), y = *reinterpret_cast<const vec4f_u *>(b + 4 * q);
        reinterpret_cast<float4 *>(sum)[q] = make_float4(x.x + y.x, x.y + y.y, x.z + y.z, x.w + y.w);
    }
    if (tid < (n & 3)) sum[4 * n4 + tid] = a[4 * n4 + tid] + b[4 * n4 + tid];
#pragma unroll 4
    for (int i = tid; i < nr * G::LOW; i += T) {
        const int r = i / G::LOW, x = r * G::D + (i - r * G::LOW);
        la[i] = a[x];
        lb[i] = b[x];
    }
    __syncthreads();
    const int items = nr * G::NODES;
    for (int it = tid; it < items; it += T) {
        const int r = it / G::NODES;
        int h = it - r * G::NODES;
        const float *ra = la + r * G::LOW, *rb = lb + r * G::LOW;
        float c[d];
        read_group<d>(c, sum + it * d);
        int x = 0;   // the split's second factor but for k, as a node
#pragma unroll
        for (int j = 1; j < N; ++j) {
            if (h > 0) {
                const float u = ra[h - 1];
                float v[d];
                read_group<d>(v, rb + x * d);
#pragma unroll
                for (int k = 0; k < d; ++k) c[k] = fmaf(u, v[k], c[k]);
                const int up = (int)(__umul24((uint32_t)(h - 1), G::M) >> 18);
                x += (h - up * d) * cpow(d, j - 1);   // the last letter of h, plus one, in front of the factor
                h = up;
            }
        }
        write_group<d>(sum + it * d, c);
    }
    __syncthreads();
#pragma unroll 4
    for (int q = tid; q < n4; q += T) {
        const float4 s = reinterpret_cast<const float4 *>(sum)[q];
        vec4f_u v = {s.x, s.y, s.z, s.w};
        *reinterpret_cast<vec4f_u *>(out + 4 * q) = v;
    }
    if (tid < (n & 3)) out[4 * n4 + tid] = sum[4 * n4 + tid];
}

template <int d, int N>
hipError_t launch(const float *a, const float *b, float *out, int64_t B, hipStream_t st)
{
    using G = Geo<d, N>;
    int64_t per_wg = B / 1024;   // at least four workgroups for every compute unit
    if (per_wg > G::R) per_wg = G::R;
    if (per_wg < 1) per_wg = 1;
    const int64_t grid = (B + per_wg - 1) / per_wg;
    if (B <= 0 || grid > INT32_MAX) return hipErrorInvalidValue;
    hipLaunchKernelGGL((sig_combine_tree_kernel<d, N>), dim3((unsigned)grid), dim3(G::threads), 0, st, a, b, out, B, (int)per_wg);
    return hipGetLastError();
}

struct Entry {
    int d, depth;
    hipError_t (*launch)(const float *, const float *, float *, int64_t, hipStream_t);
};
// rows of at most 12,000 floats
#define SIG_COMBINE_SHAPES(X)                                                                                          \
    X(2, 2) X(3, 2) X(4, 2) X(5, 2) X(6, 2) X(7, 2) X(8, 2) X(9, 2) X(10, 2) X(11, 2) X(12, 2) X(13, 2) X(14, 2)       \
    X(15, 2) X(16, 2) X(17, 2) X(18, 2) X(19, 2) X(20, 2)                                                              \
    X(2, 3) X(3, 3) X(4, 3) X(5, 3) X(6, 3) X(7, 3) X(8, 3) X(9, 3) X(10, 3) X(11, 3) X(12, 3) X(13, 3) X(14, 3)       \
    X(15, 3) X(16, 3)                                                                                                  \
    X(2, 4) X(3, 4) X(4, 4) X(5, 4) X(6, 4) X(7, 4) X(8, 4) X(9, 4) X(10, 4)                                           \
    X(2, 5) X(3, 5) X(4, 5) X(5, 5) X(6, 5) X(2, 6) X(3, 6) X(4, 6)
#define SIG_COMBINE_ENTRY(d, N) {d, N, &launch<d, N>},
const Entry kEntries[] = {SIG_COMBINE_SHAPES(SIG_COMBINE_ENTRY){0, 0, nullptr}};

}  // namespace combine

bool combine_tree_compiled(int d, int depth)
{
    for (const combine::Entry *e = combine::kEntries; e->launch; ++e)
        if (e->d == d && e->depth == depth) return true;
    return false;
}

hipError_t launch_combine_tree(const float *a, const float *b, float *out, int64_t B, int d, int depth, hipStream_t st)
{
    for (const combine::Entry *e = combine::kEntries; e->launch; ++e)
        if (e->d == d && e->depth == depth) return e->launch(a, b, out, B, st);
    return hipErrorInvalidValue;
}

}  // namespace sig
