// Gradient of the FINAL signature with respect to the path, swept on Lie brackets (compiled per (d, depth N)).
//
// The layer is trained between other layers (paper Section 4.2, Eq. 11); this is the derivative of the paper's
// Eqs. 2-5 with respect to the points of the path, in a form that needs neither the prefix signatures nor their
// adjoint.  With S = S_{k} (x) T_k (everything up to step k, and everything after it) and G = d(loss)/d(S), let
//     F_k(x) = < G, S_k (x) x (x) T_k >
// be the loss as a function of an element inserted after step k.  Moving from step k to k - 1 conjugates x,
//     F_{k-1}(x) = F_k(exp(-v) x exp(v)),   v = dX_k,
// and the derivative of the loss with respect to v_k is F_k applied to  sum_i (-1)^i / (i+1)! ad_v^i e_a.  Both only
// ever evaluate F_k on Lie elements, so all that has to be carried are the values on nested brackets
//     f_n[w] = F(x_w),   x_w = [e_{w1}, [e_{w2}, ... [e_{w(n-1)}, e_{wn}]]],
// and because [e_a, x_w] = x_{aw} the step is a contraction over LEADING letters:
//     f_n'[w] = sum_i (-1)^i / i!  sum_{|u| = i} v^u f_{n+i}[u w].
// The top level never changes, x_w changes sign with its last two letters (only pairs a < b are kept), and level 1
// feeds nothing back: with C_i[ab] = sum_u v^u f_{2+i}[u ab] the gradient at a point needs two numbers per pair,
//     q_k[ab] = sum_i (-1)^i / (i+2)! C_i[ab],      y_k[ab] = -sum_i (-1)^i (i+1) / (i+2)! C_i[ab],
//     d(loss)/dX_j[b] = sum_a v_{j+1}[a] y_{j+1}[ab] - sum_a v_j[a] q_j[ab]
// with f_1 of the whole path at the two ends: F_K(e_b) for j = K in place of the first sum, -F_0(e_b) for j = 0 in
// place of the second.  No running sum over time and no difference of large numbers is left.
//
// Work per step and path for (5,4): 10 pairs x (25 + 2 x 5) multiply-adds, against 25 lanes x some 200 instructions
// for undoing the step on the whole signature and transposing it on its adjoint (sig_backward.hip).  Measured, sweep on the
// signature against this one: (5,4), 100 points, 128 paths 24.7 -> 9.9 us, 65,536 paths 697 -> 189 to 230 (by the card and what
// ran before; reading and writing what it must takes 92 at the rate of a copy); (4,4), 500 points, 65,536 paths 3,226 -> 407;
// (10,4), 100 points, 8,192 paths 2,990 -> 490; (12,3), 100 points, 128 paths, against the general sweep 678 -> 13.9.
// Rounding, over 522 settings of 29 shapes against 64 bits: 1.5e-7 (depth 2) to 1.6e-6 (depth 6) of the gradient's norm at
// most, 0.02 to 1.01 times the sweep on signatures' and 0.15 in the mean.
//
// Lanes.  A lane owns the words that end in its suffix of P letters: pre (P - 2 letters) and a pair a < b, so
// LQ = d^{P-2} d (d-1) / 2 lanes per path, each with the levels P .. N of its words in registers
// (1 + d + ... + d^{N-P} floats) and, being linear, a private PARTIAL value of the levels 2 .. P-1 below.
//
// Time.  R_k, the signature of the path walked backwards from its end to step k, moves f from the end of the path to
// step k in one go: f_n(k)[w] = sum_u R_k[u] f_{n+|u|}(K)[u w], with R to level N - 2 only.  A path's steps are cut into
// C chunks side by side in a workgroup (and W workgroups): each chunk folds its R, a scan joins them, and every
// chunk then walks its own steps.  A batch that fills the chip by itself packs several paths into a wavefront
// instead and walks them uncut.
#ifndef SIG_BRACKET_H_
#define SIG_BRACKET_H_

#include "sig_onchip.h"

namespace sig {
namespace bracket {

using onchip::cpow;
using onchip::geom;
using onchip::static_for;
using onchip::vec4f_u;

struct Args {
    const float *path;      // [B][L][d]
    const float *sig;       // [B][D], levels 1 .. N-1 are read
    const float *grad_out;  // [B][D]
    float *grad_path;       // [B][L][d]
    int64_t B, L;
    // cut in time (sig_bracket_chunked_kernel)
    int32_t chunks;         // C: chunks of a workgroup
    int32_t segs;           // W: workgroups of a path
    int32_t steps;          // T: steps of a chunk; W * C * T >= L - 1
    int32_t fold_slots;     // slots of QF lanes that fold what lies behind the workgroup (>= C; levels 3 and up of R only)
    int32_t groups;         // paths per workgroup (sig_bracket_packed_kernel, sig_bracket_depth2_kernel)
};

constexpr float inv_factorial(int n)
{
    double f = 1.0;
    for (int i = 2; i <= n; ++i) f *= i;
    return (float)(1.0 / f);
}
// (i + 1) / (i + 2)!
constexpr float y_factor(int i)
{
    double f = 1.0;
    for (int j = 2; j <= i + 2; ++j) f *= j;
    return (float)((i + 1) / f);
}

template <int d_, int N_, int P_>
struct Geo {
    static_assert(P_ >= 2 && P_ <= N_ && d_ >= 2, "a lane's suffix holds the antisymmetric pair");
    static constexpr int d = d_, N = N_, P = P_;
    static constexpr int R = N - P;                   // letters in front of a lane's suffix, at most
    static constexpr int PAIRS = d * (d - 1) / 2;
    static constexpr int PRE = cpow(d, P - 2);
    static constexpr int LQ = PRE * PAIRS;            // lanes per path
    static constexpr int SZ = geom(d, R + 1);         // floats of a lane's words (level P + r at sub_off(r))
    static constexpr int SZS = SZ | 1;                // ... as a row in LDS: an odd stride spreads the lanes over the banks
    static constexpr int sub_off(int r) { return geom(d, r); }
    static constexpr int MP = P > 2 ? P - 2 : 1;      // partial values of the levels 2 .. P-1
    static constexpr int tm_off(int m) { return PAIRS * (geom(d, m - 2)); }   // level m's values, m = 2 .. P-1
    static constexpr int TM = PAIRS * geom(d, P - 2);
    static constexpr int FST = LQ * SZS + TM;         // floats of a path's bracket values in LDS
    static constexpr int row_off(int n) { return geom(d, n) - 1; }
    static constexpr int LOW = geom(d, N) - 1;        // levels 1 .. N-1 of a row
    static constexpr int D = geom(d, N + 1) - 1;
    // reversed signatures: levels 1 .. N-2
    static constexpr int FN = N - 2;
    static constexpr int DR = FN >= 1 ? geom(d, FN + 1) - 1 : 0;
    static constexpr int PF = FN >= 2 && LQ >= d ? 1 : 0;
    static constexpr int QF = cpow(d, PF);            // lanes that fold them
    // the walk's tile, per slot (a path, or a chunk of one): TT + 1 rows of increments and of parked q and y
    static constexpr int VS = d | 1;
    static constexpr int RS = (2 * LQ) | 1;
    static constexpr int row_floats = VS + RS;
    // packed kernel: paths per wavefront, paths whose rows are staged together, steps per tile
    static constexpr int PG = LQ <= kWave ? kWave / LQ : 1;
    static constexpr int staged(int want) { return want < 1 ? 1 : (want > PG ? PG : want); }
    static constexpr int IP = staged(1100 / D);
    static constexpr int TT = PG >= 32 ? 4 : PG >= 12 ? 6 : PG >= 4 ? kWave / PG : 16;
    // chunked kernel: threads, and steps of every chunk per tile
    static constexpr int CT = D >= 256 ? 256 : 128;
    static constexpr int CTT = LQ >= 24 ? 16 : 8;
};

// Wavefronts per SIMD the kernels are built for: what a lane's words and some fifty more registers allow.  Without the bound
// the compiler spends registers on the sums over the rows, before the words exist, and halves the residency.
// The words of (5,4) to (7,4) fit four wavefronts, which takes a spare register off (5,4) (134 otherwise; 65,536 paths of 100
// points 186 -> 177 us on one card); at depth 5 and 6 it would spill ((4,5) 113 -> 126 us).
constexpr int min_waves(int depth, int state) { return state > 100 ? 2 : state > 57 ? 3 : depth == 4 && state > 24 ? 4 : 1; }

// Summands that `threads` threads split one of cnt sums per path into
constexpr int sum_parts(int threads, int paths, int cnt)
{
    const int p = threads / (paths * cnt);
    return p < 1 ? 1 : (p > 12 ? 12 : p);
}

// a < b of a pair's number (pairs in lexicographic order), as a * d + b
template <int d>
__device__ __forceinline__ void fill_pair_table(int *table, int tid, int nthr)
{
    for (int i = tid; i < d * d; i += nthr) {
        const int a = i / d, b = i - a * d;
        if (a < b) table[a * d - a * (a + 1) / 2 + (b - a - 1)] = i;
    }
}

// The words of [c, block] for a block of len letters that is a signed word itself: c to its left, or with a minus sign to
// its right.  Calls f(sign, word) for all 2^{n-1} words of the nested bracket of n letters let[0 .. n-1].
template <int d, int n, int len, int sign, class Fn>
__device__ __forceinline__ void bracket_words(const int (&let)[n], int idx, Fn &&f)
{
    if constexpr (len == n) f(std::integral_constant<int, sign>{}, idx);
    else {
        const int c = let[n - 1 - len];
        bracket_words<d, n, len + 1, sign>(let, c * cpow(d, len) + idx, f);
        bracket_words<d, n, len + 1, -sign>(let, idx * d + c, f);
    }
}

template <int M, int CNT>
struct Chain {   // contractions c_{r,i} of a level, i = 1 .. M
    float v[M > 0 ? M : 1][M > 0 ? CNT : 1];
};

// A lane's step, from f(k) to f(k-1); nv = -dX_k, du[i] = nv[letter i of the suffix].  down<r>: level P + r, of which c holds
// the values contracted i = 1 .. R - r times.  q and yy (= -y, with the signs of nv) as in the file comment.
template <class G>
struct Step {
    template <int m, int CNT>
    static __device__ __forceinline__ void low(float (&fm)[G::MP], const float (&du)[G::MP], const float (&C)[CNT], float &q, float &yy)
    {
        if constexpr (m == 2) {
            q = C[0] * inv_factorial(2);
            yy = C[0] * y_factor(0);
            static_for<1, CNT>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                q = fmaf(C[i], inv_factorial(i + 2), q);
                yy = fmaf(C[i], y_factor(i), yy);
            });
        } else {
            float E[CNT + 1];
            E[0] = fm[m - 3];
            float sum = E[0];
            static_for<0, CNT>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                E[i + 1] = du[G::P - m] * C[i];
                sum = fmaf(E[i + 1], inv_factorial(i + 1), sum);
            });
            fm[m - 3] = sum;
            low<m - 1, CNT + 1>(fm, du, E, q, yy);
        }
    }

    template <int r, int M>
    static __device__ __forceinline__ void down(float (&f)[G::SZ], float (&fm)[G::MP], const float (&nv)[G::d],
                                                const float (&du)[G::MP], const Chain<M, cpow(G::d, r)> &c, float &q, float &yy)
    {
        if constexpr (r == 0) {
            float C[M + 1];
            C[0] = f[0];
            float sum = f[0];
            static_for<1, M + 1>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
                C[i] = c.v[i - 1][0];
                sum = fmaf(C[i], inv_factorial(i), sum);
            });
            f[0] = sum;
            low<G::P, M + 1>(fm, du, C, q, yy);
        } else {
            constexpr int cnt = cpow(G::d, r - 1);
            Chain<M + 1, cnt> e;
#pragma unroll
            for (int w = 0; w < cnt; ++w) {
                float s = nv[0] * f[G::sub_off(r) + w];
#pragma unroll
                for (int a = 1; a < G::d; ++a) s = fmaf(nv[a], f[G::sub_off(r) + a * cnt + w], s);
                e.v[0][w] = s;
            }
            static_for<1, M + 1>([&](auto ic) __attribute__((always_inline)) {
                constexpr int i = decltype(ic)::value;
#pragma unroll
                for (int w = 0; w < cnt; ++w) {
                    float s = nv[0] * c.v[i - 1][w];
#pragma unroll
                    for (int a = 1; a < G::d; ++a) s = fmaf(nv[a], c.v[i - 1][a * cnt + w], s);
                    e.v[i][w] = s;
                }
#pragma unroll
                for (int w = 0; w < cnt * G::d; ++w)
                    f[G::sub_off(r) + w] = fmaf(c.v[i - 1][w], inv_factorial(i), f[G::sub_off(r) + w]);
            });
            down<r - 1, M + 1>(f, fm, nv, du, e, q, yy);
        }
    }

    static __device__ __forceinline__ void run(float (&f)[G::SZ], float (&fm)[G::MP], const float (&nv)[G::d],
                                               const float (&du)[G::MP], float &q, float &yy)
    {
        Chain<0, cpow(G::d, G::R)> none;
        down<G::R, 0>(f, fm, nv, du, none, q, yy);
    }
};

// f from the end of the path to an earlier step, given the row of R (levels 1 .. N-2, LDS) between the two
template <class G>
__device__ __forceinline__ void move_to(float (&f)[G::SZ], float (&fm)[G::MP], const float *row, int pre)
{
    constexpr int d = G::d, P = G::P;
    // partial values of the levels below the suffix, ascending: the levels above are still those of the end
    static_for<2, P>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        float sum = fm[m - 2];
        static_for<m + 1, P>([&](auto lc) __attribute__((always_inline)) {
            constexpr int l = decltype(lc)::value;
            sum = fmaf(row[G::row_off(l - m) + (pre / cpow(d, m - 2)) % cpow(d, l - m)], fm[l - 2], sum);
        });
        const float *tail = row + pre / cpow(d, m - 2);
        static_for<0, G::R + 1>([&](auto rc) __attribute__((always_inline)) {
            constexpr int r = decltype(rc)::value;
#pragma unroll
            for (int u = 0; u < cpow(d, r); ++u)
                sum = fmaf(tail[G::row_off(r + P - m) + u * cpow(d, P - m)], f[G::sub_off(r) + u], sum);
        });
        fm[m - 2] = sum;
    });
    static_for<0, G::R>([&](auto rc) __attribute__((always_inline)) {
        constexpr int r = decltype(rc)::value;
        constexpr int cnt = cpow(d, r);
        static_for<1, G::R - r + 1>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
#pragma unroll
            for (int u = 0; u < cpow(d, i); ++u) {
                const float Ru = row[G::row_off(i) + u];
#pragma unroll
                for (int w = 0; w < cnt; ++w)
                    f[G::sub_off(r) + w] = fmaf(Ru, f[G::sub_off(r + i) + u * cnt + w], f[G::sub_off(r) + w]);
            }
        });
    });
}

// LDS of the stage that turns the rows of `paths` paths into bracket values: rows of G and levels 1 .. N-1 of S; then levels
// 1 .. N-1 of F, and the summands of F and of f_1
template <class G>
constexpr int summand_floats(int threads, int paths)
{
    int total = 2 * paths * G::d * sum_parts(threads, 2 * paths, G::d);
    for (int lev = 2; lev < G::N; ++lev) {
        const int cnt = cpow(G::d, lev), parts = sum_parts(threads, paths, cnt);
        if (parts > 1) total += paths * cnt * parts;
    }
    return total;
}
template <class G>
constexpr int rows_floats(int paths) { return (paths * (G::D + G::LOW) + 3) / 4 * 4; }
template <class G>
constexpr int work_floats(int threads, int paths) { return paths * G::LOW + summand_floats<G>(threads, paths); }

// sum over j of S[u_j] G[u_j * stride], u_j = part + j * PARTS < CNT
template <int CNT, int PARTS, int UNROLL>
__device__ __forceinline__ float strided_sum(const float *S, const float *G, int stride, int part, float sum)
{
    constexpr int full = CNT / PARTS;
#pragma unroll UNROLL
    for (int j = 0; j < full; ++j) sum = fmaf(S[part + j * PARTS], G[(part + j * PARTS) * stride], sum);
    if constexpr (CNT % PARTS != 0) {
        if (part + full * PARTS < CNT) sum = fmaf(S[part + full * PARTS], G[(part + full * PARTS) * stride], sum);
    }
    return sum;
}

// The rows that the bracket values of NP adjacent paths need, on their way to LDS ([path][D] of G, then [path][LOW] of S):
// fetch() leaves the loads in flight, put() writes what they brought.
template <class G, int NT, int NP>
struct Rows {
    static constexpr int VECS = (NP * G::D / 4 + NT - 1) / NT;
    static constexpr int LOWS = (NP * G::LOW + NT - 1) / NT;
    vec4f_u g[VECS > 0 ? VECS : 1];
    float tail;
    float s[LOWS];

    __device__ __forceinline__ void fetch(const Args &A, int64_t b0, int n, int tid)
    {
        const float *src = A.grad_out + b0 * G::D;
        const int total = n * G::D, vecs = total / 4;
#pragma unroll
        for (int j = 0; j < VECS; ++j) {
            const int i = tid + j * NT;
            g[j] = *reinterpret_cast<const vec4f_u *>(src + 4 * (i < vecs ? i : 0));
        }
        tail = tid < total - 4 * vecs ? src[4 * vecs + tid] : 0.0f;
        src = A.sig + b0 * G::D;
#pragma unroll
        for (int j = 0; j < LOWS; ++j) {
            const int i = tid + j * NT, p = i / G::LOW;
            s[j] = src[p < n ? p * G::D + (i - p * G::LOW) : 0];
        }
    }
    __device__ __forceinline__ void put(float *rows, int n, int tid) const
    {
        const int total = n * G::D, vecs = total / 4;
#pragma unroll
        for (int j = 0; j < VECS; ++j) {
            const int i = tid + j * NT;
            if (i < vecs) *reinterpret_cast<vec4f_u *>(rows + 4 * i) = g[j];
        }
        if (tid < total - 4 * vecs) rows[4 * vecs + tid] = tail;
        float *Ss = rows + NP * G::D;
#pragma unroll
        for (int j = 0; j < LOWS; ++j) {
            const int i = tid + j * NT;
            if (i < n * G::LOW) Ss[i] = s[j];
        }
    }
};

// the same without a stop in registers (rows too long for them)
template <class G, int NT, int NP>
__device__ __forceinline__ void stage_rows(const Args &A, int64_t b0, int n, float *rows, int tid)
{
    const float *g = A.grad_out + b0 * G::D;
    const int total = n * G::D, vecs = total / 4;
#pragma unroll 4
    for (int i = tid; i < vecs; i += NT) *reinterpret_cast<vec4f_u *>(rows + 4 * i) = *reinterpret_cast<const vec4f_u *>(g + 4 * i);
    for (int i = vecs * 4 + tid; i < total; i += NT) rows[i] = g[i];
    const float *s = A.sig + b0 * G::D;
    float *Ss = rows + NP * G::D;
#pragma unroll 4
    for (int i = tid; i < n * G::LOW; i += NT) {
        const int p = i / G::LOW;
        Ss[i] = s[p * G::D + (i - p * G::LOW)];
    }
}

// From the rows of n <= NP paths in LDS (the barrier after their staging is the caller's): f_1 at both ends
// ([path][2 d]: F_K(e_b), then F_0(e_b)) and the bracket values of the levels 2 .. N ([path][FST]).  `work` holds F and the
// summands.  All NT threads of the workgroup take part; ends with a barrier.
template <class G, int NT, int NP>
__device__ __forceinline__ void bracket_values(int n, const float *rows, float *work, float *f1, float *fst, const int *pairs, int tid)
{
    constexpr int d = G::d, N = G::N, P = G::P, D = G::D, LOW = G::LOW;
    const float *Gs = rows, *Ss = Gs + NP * D;
    float *Fs = work, *sums = Fs + NP * LOW;
    // f_1 = G_1 + sum over words u of the levels 1 .. N-1 of S[u] G[u b] (end of the path) or S[u] G[b u] (start), and
    // F_n[w] = G_n[w] + sum over u of S[u] G[u w], levels 2 .. N-1 (level N is G's own).  The short levels are sums over
    // many words: they are cut into summands as far as there are threads.
    constexpr int UNROLL = 8;
    constexpr int P1 = sum_parts(NT, 2 * NP, d);
    for (int it = tid; it < n * 2 * d * P1; it += NT) {
        const int o = it % (2 * d);
        const int part = (it / (2 * d)) % P1;
        const int p = it / (2 * d * P1);
        const int b = o % d;
        float sum = 0.0f;
        static_for<1, N>([&](auto ic) __attribute__((always_inline)) {
            constexpr int i = decltype(ic)::value;
            constexpr int cnt = cpow(d, i);
            sum = strided_sum<cnt, P1, UNROLL>(Ss + p * LOW + G::row_off(i), Gs + p * D + G::row_off(i + 1) + (o < d ? b : b * cnt), o < d ? d : 1, part, sum);
        });
        sums[it] = sum;
    }
    {
        float *part_sums = sums + 2 * NP * d * P1;
        static_for<2, N>([&](auto nc) __attribute__((always_inline)) {
            constexpr int lev = decltype(nc)::value;
            constexpr int cnt = cpow(d, lev);
            constexpr int parts = sum_parts(NT, NP, cnt);
            for (int it = tid; it < n * cnt * parts; it += NT) {
                const int w = it % cnt;
                const int part = (it / cnt) % parts;
                const int p = it / (cnt * parts);
                float sum = parts == 1 ? Gs[p * D + G::row_off(lev) + w] : 0.0f;
                static_for<1, N - lev + 1>([&](auto ic) __attribute__((always_inline)) {
                    constexpr int i = decltype(ic)::value;
                    sum = strided_sum<cpow(d, i), parts, UNROLL>(Ss + p * LOW + G::row_off(i), Gs + p * D + G::row_off(lev + i) + w, cnt, part, sum);
                });
                if constexpr (parts == 1) Fs[p * LOW + G::row_off(lev) + w] = sum;
                else part_sums[it] = sum;
            }
            if constexpr (parts > 1) part_sums += NP * cnt * parts;
        });
    }
    __syncthreads();
    for (int it = tid; it < n * 2 * d; it += NT) {
        const int p = it / (2 * d), o = it - p * (2 * d);
        float sum = Gs[p * D + o % d];
#pragma unroll
        for (int j = 0; j < P1; ++j) sum += sums[(p * P1 + j) * 2 * d + o];
        f1[it] = sum;
    }
    {
        const float *part_sums = sums + 2 * NP * d * P1;
        static_for<2, N>([&](auto nc) __attribute__((always_inline)) {
            constexpr int lev = decltype(nc)::value;
            constexpr int cnt = cpow(d, lev);
            constexpr int parts = sum_parts(NT, NP, cnt);
            if constexpr (parts > 1) {
                for (int it = tid; it < n * cnt; it += NT) {
                    const int p = it / cnt, w = it - p * cnt;
                    float sum = Gs[p * D + G::row_off(lev) + w];
#pragma unroll
                    for (int j = 0; j < parts; ++j) sum += part_sums[(p * parts + j) * cnt + w];
                    Fs[p * LOW + G::row_off(lev) + w] = sum;
                }
                part_sums += NP * cnt * parts;
            }
        });
    }
    __syncthreads();
    // Brackets; the pair is the fastest index, so that neighbouring threads read neighbouring words.  From level 4 on a thread
    // takes the d values that differ in the outermost letter: the words of the inner block are worked out once for all.
    static_for<2, N + 1>([&](auto nc) __attribute__((always_inline)) {
        constexpr int lev = decltype(nc)::value;
        constexpr int outer = lev >= 4 ? d : 1;
        constexpr int inner = lev >= 4 ? lev - 1 : lev;     // letters of the block whose words are listed
        constexpr int cnt = cpow(d, inner - 2) * G::PAIRS;
        for (int it = tid; it < n * cnt; it += NT) {
            const int p = it / cnt, w = it - p * cnt;
            const int head = w / G::PAIRS;                  // the letters in front of the pair
            const int pair = w - head * G::PAIRS;
            const int ab = pairs[pair];
            int let[inner];
            let[inner - 1] = ab % d;
            let[inner - 2] = ab / d;
            int rest = head;
#pragma unroll
            for (int i = inner - 3; i >= 0; --i) { let[i] = rest % d; rest /= d; }
            const float *F = lev == N ? Gs + p * D + G::row_off(N) : Fs + p * LOW + G::row_off(lev);
            float val[outer];
#pragma unroll
            for (int c = 0; c < outer; ++c) val[c] = 0.0f;
            bracket_words<d, inner, 1, 1>(let, let[inner - 1], [&](auto sc, int idx) __attribute__((always_inline)) {
                constexpr int sign = decltype(sc)::value;
                if constexpr (outer == 1) val[0] += sign > 0 ? F[idx] : -F[idx];
                else {
                    const float *left = F + idx, *right = F + idx * d;
#pragma unroll
                    for (int c = 0; c < outer; ++c) {
                        const float x = left[c * cpow(d, inner)] - right[c];
                        val[c] += sign > 0 ? x : -x;
                    }
                }
            });
            float *dst = fst + p * G::FST;
#pragma unroll
            for (int c = 0; c < outer; ++c) {
                const int h = outer == 1 ? head : c * cpow(d, inner - 2) + head;
                if constexpr (lev < P) dst[G::LQ * G::SZS + G::tm_off(lev) + h * G::PAIRS + pair] = val[c];
                else {
                    const int u = h / G::PRE, pre = h - u * G::PRE;
                    dst[(pre * G::PAIRS + pair) * G::SZS + G::sub_off(lev - P) + u] = val[c];
                }
            }
        }
    });
    __syncthreads();
}

// a lane's registers from a path's bracket values
template <class G>
__device__ __forceinline__ void load_lane(float (&f)[G::SZ], float (&fm)[G::MP], const float *fst, int lane, int pre, int pair)
{
#pragma unroll
    for (int i = 0; i < G::SZ; ++i) f[i] = fst[lane * G::SZS + i];
    fm[0] = 0.0f;
    static_for<2, G::P>([&](auto mc) __attribute__((always_inline)) {
        constexpr int m = decltype(mc)::value;
        constexpr int words = cpow(G::d, m - 2);
        // the lane whose leading letters are zero starts with the level's value, the others with nothing
        fm[m - 2] = pre < words ? fst[G::LQ * G::SZS + G::tm_off(m) + pre * G::PAIRS + pair] : 0.0f;
    });
}

// The gradient at point k from a step's parked rows: `row` is step k's (increment, q, y), `above` step k+1's.
template <class G>
__device__ __forceinline__ void emit_point(float *dst, const float *vrow, const float *prow, const float *vabove, const float *pabove,
                                           const float *f1, bool last, bool first)
{
    constexpr int d = G::d;
    float acc[d], v[d];
    auto pairs_of = [&](const float *p) __attribute__((always_inline)) {
        static_for<0, d>([&](auto ac) __attribute__((always_inline)) {
            constexpr int a = decltype(ac)::value;
            static_for<a + 1, d>([&](auto bc) __attribute__((always_inline)) {
                constexpr int b = decltype(bc)::value;
                constexpr int pair = a * d - a * (a + 1) / 2 + (b - a - 1);
                float x = 0.0f;
#pragma unroll
                for (int pre = 0; pre < G::PRE; ++pre) x += p[pre * G::PAIRS + pair];
                acc[b] = fmaf(v[a], x, acc[b]);
                acc[a] = fmaf(-v[b], x, acc[a]);
            });
        });
    };
#pragma unroll
    for (int b = 0; b < d; ++b) acc[b] = 0.0f;
    if (last) {
#pragma unroll
        for (int b = 0; b < d; ++b) acc[b] = f1[b];
    } else {
#pragma unroll
        for (int a = 0; a < d; ++a) v[a] = vabove[a];
        pairs_of(pabove + G::LQ);
    }
#pragma unroll
    for (int a = 0; a < d; ++a) v[a] = vrow[a];
    pairs_of(prow);
    onchip::store_run<0, d, d>(dst, acc);
    if (first) {   // step 1 also settles point 0
#pragma unroll
        for (int b = 0; b < d; ++b) acc[b] = -f1[d + b];
        pairs_of(prow + G::LQ);
        onchip::store_run<0, d, d>(dst - d, acc);
    }
}

extern __shared__ __align__(16) float sig_bracket_smem[];

// ------------------------------------------------------------------------------------------
// Several whole paths per wavefront (one wavefront per workgroup, so no barrier costs anything), each walked uncut.
// Per step and wavefront some 50 vector instructions for the walk, 20 for the outputs and 8 for the loads, after some 700 per
// path for the bracket values.  Bound by waiting, mostly for LDS: (5,4), 100 points, 65,536 paths issue 81,000 vector
// instructions per SIMD in 372,000 cycles (4.6 cycles each, against 2.2 where the pipe is full), the LDS is busy 78 % of
// the time (28 % of that bank conflicts), and 537 MB move where 507 must (184 to 211 us under the counters).  Registers decide
// the residency (128 there: four wavefronts per SIMD; two to seven over the shapes); keeping the paths' bracket values in
// registers as they are formed, instead of all paths' in LDS, and having the next path's rows in flight took a quarter
// off (246 -> 188 us on one card).  Places of the tile in 32 bits, loaded without a condition, and the fourth wavefront took 6 to 8 % more:
// 190 to 199 us and 179 to 186 in turn on each of two cards (82 of them the bracket values; calls behind an idle card take 200 to 215 on
// both sides, so that single calls show less); (2,6) with 700 points 365 -> 280.
template <class G>
constexpr int packed_lds_floats()
{
    const int init = rows_floats<G>(G::IP) + work_floats<G>(kWave, G::IP) + G::IP * G::FST;
    const int walk = G::PG * (G::TT + 1) * G::row_floats;
    return (G::PAIRS + G::PG * 2 * G::d + 3) / 4 * 4 + (init > walk ? init : walk);
}

template <int d, int N, int P>
__global__ __launch_bounds__(kWave) __attribute__((amdgpu_waves_per_eu(min_waves(N, Geo<d, N, P>::SZ))))
void sig_bracket_packed_kernel(Args A)
{
    using G = Geo<d, N, P>;
    constexpr int PG = G::PG, LQ = G::LQ, TT = G::TT, IP = G::IP;
    const int tid = threadIdx.x;
    const int K = (int)(A.L - 1);
    const int64_t b0 = (int64_t)blockIdx.x * A.groups;
    const int npaths = A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups;   // groups <= PG
    const int slot_raw = tid / LQ;
    const bool active = slot_raw < npaths;
    const int slot = active ? slot_raw : 0;
    const int lane = active ? tid - slot_raw * LQ : 0;
    const int pre = lane / G::PAIRS, pair = lane - pre * G::PAIRS;

    int *pairs = reinterpret_cast<int *>(sig_bracket_smem);
    float *f1 = sig_bracket_smem + G::PAIRS;            // [PG][2 d]
    float *area = sig_bracket_smem + (G::PAIRS + PG * 2 * d + 3) / 4 * 4;
    fill_pair_table<d>(pairs, tid, kWave);

    // The bracket values, IP paths at a time, with the rows of the next ones in flight; the lanes of a path take theirs at
    // once, which keeps the workgroup's LDS (and so the number of resident wavefronts) independent of PG.
    float f[G::SZ], fm[G::MP];
#pragma unroll
    for (int i = 0; i < G::SZ; ++i) f[i] = 0.0f;
#pragma unroll
    for (int i = 0; i < G::MP; ++i) fm[i] = 0.0f;
    {
        constexpr bool PREFETCH = Rows<G, kWave, IP>::VECS <= 6;
        float *work = area + rows_floats<G>(IP), *fst = work + work_floats<G>(kWave, IP);
        Rows<G, kWave, PREFETCH ? IP : 1> next;
        if constexpr (PREFETCH) next.fetch(A, b0, npaths < IP ? npaths : IP, tid);
        for (int p0 = 0; p0 < npaths; p0 += IP) {
            const int n = npaths - p0 < IP ? npaths - p0 : IP;
            if constexpr (PREFETCH) {
                next.put(area, n, tid);
                const int left = npaths - p0 - IP;
                if (left > 0) next.fetch(A, b0 + p0 + IP, left < IP ? left : IP, tid);
            } else {
                stage_rows<G, kWave, IP>(A, b0 + p0, n, area, tid);
            }
            __syncthreads();
            bracket_values<G, kWave, IP>(n, area, work, f1 + p0 * 2 * d, fst, pairs, tid);
            if (active && slot >= p0 && slot < p0 + IP) load_lane<G>(f, fm, fst + (slot - p0) * G::FST, lane, pre, pair);
            __syncthreads();
        }
    }

    // A tile is the TT increments below the last one; a thread brings the same places of every tile, and has the next
    // tile's points in flight while the current one is walked.
    constexpr int NV = (PG * TT * d + kWave - 1) / kWave;
    const int path_floats = (int)A.L * d;               // PG paths stay below 2^31 floats (checked on the host)
    const float *block = A.path + b0 * path_floats;
    float *grads = A.grad_path + b0 * path_floats;
    int from_block[NV], where[NV];                      // its place in the tile of its path, in the block, and its row in LDS (-1: none)
    float lo[NV], hi[NV];
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = tid + j * kWave;
        const int p = i / (TT * d), x = i - p * (TT * d);
        const int kk = x / d, a = x - kk * d;
        from_block[j] = p < npaths ? p * path_floats + x : 0;
        where[j] = p < PG ? (p * (TT + 1) + TT - kk) * G::VS + a : -1;
    }
    // (steps below the first one, and slots without a path, bring floats that nothing reads: the places are only kept inside the block)
    auto fetch = [&](int t0) __attribute__((always_inline)) {
        const int from = (K - t0 - TT) * d;             // of the tile in its path; below 0 in the last tile
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int at = from_block[j] + from;
            const float *src = block + (unsigned)(at > 0 ? at : 0);
            lo[j] = src[0];
            hi[j] = src[d];
        }
    };
    fetch(0);
    int let[G::MP];
    let[0] = 0;
    {
        int rest = pre;
#pragma unroll
        for (int i = P - 3; i >= 0; --i) { let[i] = rest % d; rest /= d; }
    }

    // row 0 of a slot is the step above the tile's first, rows 1 .. TT the tile
    float *vrows = area, *prows = area + PG * (TT + 1) * G::VS;
    const float *myv = vrows + slot * (TT + 1) * G::VS;
    float *myp = prows + slot * (TT + 1) * G::RS;
    float q = 0.0f, yy = 0.0f;
    for (int t0 = 0; t0 < K; t0 += TT) {
        const int steps = K - t0 < TT ? K - t0 : TT;
        if (t0 > 0) {
            if (active) myp[LQ + lane] = yy;
            for (int i = tid; i < PG * d; i += kWave) {
                float *v = vrows + (i / d) * (TT + 1) * G::VS + i % d;
                v[0] = v[TT * G::VS];
            }
            __syncthreads();
        }
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (where[j] >= 0) vrows[where[j]] = lo[j] - hi[j];
        if (t0 + TT < K) fetch(t0 + TT);
        __syncthreads();
        for (int t = 1; t <= steps; ++t) {
            float nv[d], du[G::MP];
#pragma unroll
            for (int a = 0; a < d; ++a) nv[a] = myv[t * G::VS + a];
            du[0] = 0.0f;
#pragma unroll
            for (int i = 0; i < P - 2; ++i) du[i] = myv[t * G::VS + let[i]];
            Step<G>::run(f, fm, nv, du, q, yy);
            if (active) {
                myp[t * G::RS + lane] = q;
                myp[t * G::RS + LQ + lane] = yy;
            }
        }
        __syncthreads();
        for (int it = tid; it < PG * TT; it += kWave) {
            const int p = it / TT, t = it - p * TT + 1;
            if (p >= npaths || t > steps) continue;
            const int k = K - t0 - t + 1;
            const float *v = vrows + (p * (TT + 1) + t) * G::VS, *w = prows + (p * (TT + 1) + t) * G::RS;
            emit_point<G>(grads + p * path_floats + k * d, v, w, v - G::VS, w - G::RS, f1 + p * 2 * d, k == K, k == 1);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------
// One path (or, with segs > 1, one stretch of C * T steps of it) per workgroup, C chunks of T steps side by side.  Bound by
// latency: a dozen phases of 0.3 to 1.5 us with a barrier between them (load, chunk folds, scan, sums, brackets, walk,
// outputs), and on large batches by how many workgroups the rows of D floats in LDS leave resident.
constexpr int kFoldTile = 16;    // steps of every chunk per tile of the fold of the reversed signatures

// LDS: pair table, f_1, R rows; then the rows of G and S with, behind them, first the fold's buffers and later F, summands and
// bracket values; the walk's tile takes the place of all of these
// What lies behind the workgroup's stretch is folded by more slots than its chunks, as many as the threads and the LDS hold: a
// chunk of the walk takes LQ lanes, a slot of this fold QF of them ((6,5): 2 chunks of 90 lanes, 13 slots of 6).
template <class G>
constexpr int64_t behind_floats(int slots) { return 2 * (int64_t)(slots + 1) * G::DR + (int64_t)slots * kFoldTile * G::d; }
template <class G>
constexpr int chunked_rows_at(int C) { return (G::PAIRS + 2 * G::d + (C + 1) * G::DR + 3) / 4 * 4; }
template <class G>
int64_t chunked_lds_floats(int C, int fold_slots = 0)
{
    const int64_t init = work_floats<G>(G::CT, 1) + G::FST;
    int64_t fold = G::FN >= 2 ? (int64_t)(C + 1) * G::DR + (int64_t)C * kFoldTile * G::d : 0;
    if (fold_slots > C && behind_floats<G>(fold_slots) > fold) fold = behind_floats<G>(fold_slots);
    const int64_t rows = rows_floats<G>(1) + (init > fold ? init : fold);
    const int64_t walk = (int64_t)C * (G::CTT + 1) * G::row_floats;
    return chunked_rows_at<G>(C) + (rows > walk ? rows : walk);
}

template <int d, int N, int P>
__global__ __launch_bounds__((Geo<d, N, P>::CT)) __attribute__((amdgpu_waves_per_eu(min_waves(N, Geo<d, N, P>::SZ))))
void sig_bracket_chunked_kernel(Args A)
{
    using G = Geo<d, N, P>;
    constexpr int LQ = G::LQ, TT = G::CTT, DR = G::DR;
    constexpr int nthr = G::CT;
    const int tid = threadIdx.x;
    const int64_t K = A.L - 1;
    const int C = A.chunks, W = A.segs, T = A.steps;
    const int64_t b = blockIdx.x / W;
    const int64_t k_start = (int64_t)(blockIdx.x - b * W) * C * T;   // the workgroup settles the points k_start + 1 .. k_end
    const int64_t k_end = k_start + (int64_t)C * T;                  // (beyond K: zero increments)
    const int slot = tid / LQ;                                       // slot 0 is the last chunk in time
    const int lane = tid - slot * LQ;
    const bool active = slot < C;
    const int pre = lane / G::PAIRS, pair = lane - pre * G::PAIRS;
    // a chunk walks T + 1 steps: the one above its own provides y for its last point
    const float *X = A.path + b * A.L * d;

    int *pairs = reinterpret_cast<int *>(sig_bracket_smem);
    float *f1 = sig_bracket_smem + G::PAIRS;
    float *moved = f1 + 2 * d;          // [C + 1][DR]: R between the end of the path and slot s's first step
    float *area = sig_bracket_smem + chunked_rows_at<G>(C);
    float *work = area + rows_floats<G>(1);
    fill_pair_table<d>(pairs, tid, nthr);
    stage_rows<G, nthr, 1>(A, b, 1, area, tid);

    // A tile of the walk is TT steps of every chunk, downwards from the one above its own.  The next one is on its way while the
    // current one is walked, the first from here on, unless the lane's words need the registers.
    constexpr bool AHEAD = G::SZ <= 57;
    constexpr int NV = (nthr / LQ * TT * d + nthr - 1) / nthr;
    int where[NV];
    float lo[NV], hi[NV];
    auto fetch = [&](int t0) __attribute__((always_inline)) {
#pragma unroll
        for (int j = 0; j < NV; ++j) {
            const int i = tid + j * nthr;
            const int s = i / (TT * d), x = i - s * (TT * d);
            const int64_t at = (k_end - t0 - (TT - 1) - (int64_t)s * T) * d + x;   // the step's lower point, in floats
            lo[j] = hi[j] = 0.0f;
            if (s < C && at >= 0 && at < K * d) {
                lo[j] = X[at];
                hi[j] = X[at + d];
            }
        }
    };
#pragma unroll
    for (int j = 0; j < NV; ++j) {
        const int i = tid + j * nthr;
        const int s = i / (TT * d), x = i - s * (TT * d);
        const int kk = x / d, a = x - kk * d;
        where[j] = (s * (TT + 1) + TT - kk) * G::VS + a;
    }
    if constexpr (AHEAD) fetch(0);

    // steps t0 .. t0 + steps - 1 below top0 - s * stride of every slot s into its part of a tile of the folds, negated; steps
    // outside (kmin, K] count as zero
    auto stage_steps = [&](float *tile, int slots, int64_t top0, int64_t stride, int t0, int steps, int64_t kmin) __attribute__((always_inline)) {
        for (int i = tid; i < slots * kFoldTile * d; i += nthr) {
            const int s = i / (kFoldTile * d), x = i - s * (kFoldTile * d);
            const int t = x / d, a = x - t * d;
            if (t >= steps) continue;
            const int64_t k = top0 - s * stride - t0 - t;
            float v = 0.0f;
            if (k > kmin && k <= K) v = X[(k - 1) * d + a] - X[k * d + a];
            tile[(s * kFoldTile + t) * d + a] = v;
        }
    };
    (void)stage_steps;

    if constexpr (G::FN == 1) {
        // level 1 only: the way from the end of the path back to the step
        for (int i = tid; i < C * d; i += nthr) {
            const int s = i / d, a = i - s * d;
            const int64_t top = k_end - (int64_t)s * T + 1;
            moved[i] = top < K ? X[top * d + a] - X[K * d + a] : 0.0f;
        }
    } else if constexpr (G::FN == 2) {
        // level 1 is the way back again, and given that, a chunk's share of level 2 is a plain sum over its steps: the chunks'
        // shares add up, no products are needed
        constexpr int AL = (d + LQ - 1) / LQ;         // first letters of a lane (one, but for d = 2)
        float *tile = work;                           // [C][kFoldTile][d]
        float *shares = tile + C * kFoldTile * d;     // [C][d][d]
        auto fold = [&](int64_t top0, int64_t stride, int count, int64_t kmin) __attribute__((always_inline)) {
            float r1[AL], r2[AL][d];
            const int64_t top = top0 - slot * stride;
#pragma unroll
            for (int j = 0; j < AL; ++j) {
                const int a = lane + j * LQ;
                r1[j] = active && a < d && top < K && top >= 0 ? X[top * d + a] - X[K * d + a] : 0.0f;
#pragma unroll
                for (int b2 = 0; b2 < d; ++b2) r2[j][b2] = 0.0f;
            }
            for (int t0 = 0; t0 < count; t0 += kFoldTile) {
                const int steps = count - t0 < kFoldTile ? count - t0 : kFoldTile;
                __syncthreads();
                stage_steps(tile, C, top0, stride, t0, steps, kmin);
                __syncthreads();
                if (active && lane < d) {
                    const float *row = tile + slot * kFoldTile * d;
                    for (int t = 0; t < steps; ++t, row += d) {
#pragma unroll
                        for (int j = 0; j < AL; ++j) {
                            const float va = row[lane + j * LQ];   // (the lanes of d = 2 hold all letters: no index is beyond d)
                            const float h = fmaf(0.5f, va, r1[j]);
#pragma unroll
                            for (int b2 = 0; b2 < d; ++b2) r2[j][b2] = fmaf(h, row[b2], r2[j][b2]);
                            r1[j] += va;
                        }
                    }
                }
            }
#pragma unroll
            for (int j = 0; j < AL; ++j) {
                const int a = lane + j * LQ;
                if (active && a < d) {
#pragma unroll
                    for (int b2 = 0; b2 < d; ++b2) shares[(slot * d + a) * d + b2] = r2[j][b2];
                }
            }
            __syncthreads();
        };
        float *base2 = moved + C * DR + d;            // level 2 of what lies behind the workgroup
        const int64_t behind = K - k_end - 1;
        if (behind > 0) {
            const int count = (int)((behind + C - 1) / C);
            fold(K, count, count, k_end + 1);
            for (int e = tid; e < d * d; e += nthr) {
                float sum = 0.0f;
                for (int s = 0; s < C; ++s) sum += shares[s * d * d + e];
                base2[e] = sum;
            }
        } else {
            for (int e = tid; e < d * d; e += nthr) base2[e] = 0.0f;
        }
        fold(k_end + 1, T, T, 0);
        for (int i = tid; i < C * d * d; i += nthr) {
            const int s = i / (d * d), e = i - s * (d * d);
            float sum = base2[e];
            for (int s2 = 0; s2 < s; ++s2) sum += shares[s2 * d * d + e];
            moved[s * DR + d + e] = sum;
        }
        for (int i = tid; i < C * d; i += nthr) {
            const int s = i / d, a = i - s * d;
            const int64_t top = k_end - (int64_t)s * T + 1;
            moved[s * DR + a] = top < K ? X[top * d + a] - X[K * d + a] : 0.0f;
        }
        __syncthreads();
    } else if constexpr (G::FN > 2) {
        using Fold = onchip::Lane<d, G::FN, G::PF>;
        // `slots` slots of lanes, of which this thread is lane `u` of slot `at` if it folds at all
        struct Place {
            int slots, at;
            unsigned u;
            bool folds;
        };
        float *tile = work;                           // [C][kFoldTile][d]
        float *buf = tile + C * kFoldTile * d;        // [C + 1][DR]
        const Place mine = {C, slot, active && lane < G::QF ? (unsigned)lane : 0u, active && lane < G::QF};
        // folds `count` steps downwards from top0 - slot * stride, those in (kmin, K], and joins the slots' results in order
        auto fold = [&](Fold &ln, const Place &p, float *rows, int64_t top0, int64_t stride, int count, int64_t kmin) __attribute__((always_inline)) {
            int letter[1] = {(int)p.u};
            for (int t0 = 0; t0 < count; t0 += kFoldTile) {
                const int steps = count - t0 < kFoldTile ? count - t0 : kFoldTile;
                __syncthreads();
                stage_steps(rows, p.slots, top0, stride, t0, steps, kmin);
                __syncthreads();
                if (p.folds) {
                    const float *row = rows + p.at * kFoldTile * d;
                    for (int t = 0; t < steps; ++t, row += d) {
                        onchip::Inc<d, G::PF> inc;
                        onchip::load_inc<d, G::PF>(inc, row, letter);
                        onchip::fused_step<d, G::FN, G::PF>(ln, inc);
                    }
                }
            }
        };
        // inclusive products over the slots 0 .. limit-1 in log2 rounds (rows alternate between two buffers, slot s at
        // row s + 1); returns the buffer that holds them
        auto scan = [&](Fold &ln, const Place &p, float *cur, float *nxt, int limit) __attribute__((always_inline)) {
            if (p.folds) onchip::store_state<d, G::FN, G::PF>(cur + (p.at + 1) * DR, p.u, ln);
            __syncthreads();
            for (int st = 1; st < limit; st <<= 1) {
                if (p.folds) {
                    if (p.at < st) onchip::store_state<d, G::FN, G::PF>(nxt + (p.at + 1) * DR, p.u, ln);
                    if (p.at + st < limit) {
                        onchip::reg_product<d, G::FN, G::PF>(ln, cur + (p.at + 1 + st) * DR, p.u);
                        onchip::store_state<d, G::FN, G::PF>(nxt + (p.at + 1 + st) * DR, p.u, ln);
                    }
                }
                __syncthreads();
                if (p.folds && p.at < limit) onchip::load_state<d, G::FN, G::PF>(nxt + (p.at + 1) * DR, p.u, ln);
                float *t = cur; cur = nxt; nxt = t;
            }
            return cur;
        };
        Fold ln;
        onchip::identity_state<d, G::FN, G::PF>(ln);
        const int64_t behind = K - k_end - 1;         // steps between the workgroup's first one and the end of the path
        if (behind > 0) {
            const int CF = A.fold_slots;              // C, or more where the two buffers fit beside each other
            const int at = tid / G::QF;
            const Place wide = {CF, at, (unsigned)(tid - at * G::QF), at < CF};
            const Place place = CF > C ? wide : mine;
            const int count = (int)((behind + CF - 1) / CF);
            float *cur = tile + CF * kFoldTile * d, *nxt = CF > C ? cur + (CF + 1) * DR : moved;
            fold(ln, place, tile, K, count, count, k_end + 1);
            const float *all = scan(ln, place, cur, nxt, CF) + CF * DR;
            __syncthreads();
            // every slot's lanes take what they need of it before the buffers are used again
            onchip::identity_state<d, G::FN, G::PF>(ln);
            if (mine.folds && slot == 0) onchip::load_state<d, G::FN, G::PF>(all, mine.u, ln);
            __syncthreads();
        }
        int rounds = 0;
        for (int st = 1; st < C - 1; st <<= 1) ++rounds;
        // row 0: what lies behind the workgroup (zeros: nothing); the other rows end up in `moved` too
        float *first = rounds & 1 ? buf : moved, *second = rounds & 1 ? moved : buf;
        if (mine.folds && slot == 0) {
            if (behind > 0) onchip::store_state<d, G::FN, G::PF>(moved, mine.u, ln);
        }
        if (behind <= 0)
            for (int i = tid; i < DR; i += nthr) moved[i] = 0.0f;
        fold(ln, mine, tile, k_end + 1, T, T, 0);
        scan(ln, mine, first, second, C - 1);
        __syncthreads();
    }

    if constexpr (G::FN < 2) __syncthreads();
    float *fst = work + work_floats<G>(nthr, 1);
    bracket_values<G, nthr, 1>(1, area, work, f1, fst, pairs, tid);
    float f[G::SZ], fm[G::MP];
    load_lane<G>(f, fm, fst, active ? lane : 0, active ? pre : 0, active ? pair : 0);
    if constexpr (G::FN >= 1) {
        if (active) move_to<G>(f, fm, moved + slot * DR, pre);
    }
    int let[G::MP];
    let[0] = 0;
    {
        int rest = active ? pre : 0;
#pragma unroll
        for (int i = P - 3; i >= 0; --i) { let[i] = rest % d; rest /= d; }
    }
    __syncthreads();

    float *vrows = area, *prows = area + C * (TT + 1) * G::VS;
    const int sl = active ? slot : 0;
    const float *myv = vrows + sl * (TT + 1) * G::VS;
    float *myp = prows + sl * (TT + 1) * G::RS;
    float q = 0.0f, yy = 0.0f;
    for (int t0 = 0; t0 <= T; t0 += TT) {
        const int steps = T + 1 - t0 < TT ? T + 1 - t0 : TT;
        if (t0 > 0) {   // row 0: the step above the tile
            if (active) myp[LQ + lane] = yy;
            for (int i = tid; i < C * d; i += nthr) {
                float *v = vrows + (i / d) * (TT + 1) * G::VS + i % d;
                v[0] = v[TT * G::VS];
            }
            __syncthreads();
        }
        if constexpr (!AHEAD) fetch(t0);
#pragma unroll
        for (int j = 0; j < NV; ++j)
            if (tid + j * nthr < C * TT * d) vrows[where[j]] = lo[j] - hi[j];
        if constexpr (AHEAD) {
            if (t0 + TT <= T) fetch(t0 + TT);
        }
        __syncthreads();
        if (active) {
            for (int t = 1; t <= steps; ++t) {
                float nv[d], du[G::MP];
#pragma unroll
                for (int a = 0; a < d; ++a) nv[a] = myv[t * G::VS + a];
                du[0] = 0.0f;
#pragma unroll
                for (int i = 0; i < P - 2; ++i) du[i] = myv[t * G::VS + let[i]];
                Step<G>::run(f, fm, nv, du, q, yy);
                myp[t * G::RS + lane] = q;
                myp[t * G::RS + LQ + lane] = yy;
            }
        }
        __syncthreads();
        for (int it = tid; it < C * TT; it += nthr) {
            const int s = it / TT, t = it - s * TT + 1;
            const int64_t k = k_end - (int64_t)s * T + 2 - t0 - t;
            if (t > steps || t0 + t == 1 || k < 1 || k > K) continue;
            const float *v = vrows + (s * (TT + 1) + t) * G::VS, *w = prows + (s * (TT + 1) + t) * G::RS;
            emit_point<G>(A.grad_path + (b * A.L + k) * d, v, w, v - G::VS, w - G::RS, f1, k == K, k == 1);
        }
        __syncthreads();
    }
}

// ------------------------------------------------------------------------------------------
// Depth 2: the bracket values f[ab] = G[ab] - G[ba] do not change along the path, so that
//     d(loss)/dX_j[b] = sum_a (X_{j-1} - X_{j+1})[a] f[ab] / 2
// with the point itself in place of its missing neighbour and -F_0(e_b) or F_K(e_b) added at the ends: a thread per point,
// the d x d matrix of its path in LDS.  Bound by reading and writing the path.
constexpr int kDepth2Threads = 256;
template <int d>
constexpr int depth2_row() { return (d + 3) / 4 * 4; }
template <int d>
constexpr int depth2_floats(int paths) { return paths * (d * depth2_row<d>() + 2 * d); }

// a workgroup takes `groups` whole paths, or (segs > 1) one stretch of kDepth2Threads points of one path
template <int d>
__global__ __launch_bounds__(kDepth2Threads) void sig_bracket_depth2_kernel(Args A)
{
    constexpr int D = d + d * d, ROW = depth2_row<d>(), M = d * ROW;
    const int tid = threadIdx.x;
    const int W = A.segs;
    const int64_t b0 = W > 1 ? blockIdx.x / W : (int64_t)blockIdx.x * A.groups;
    const int64_t j0 = W > 1 ? (blockIdx.x - b0 * W) * A.steps : 0;
    const int64_t L = A.L;
    const int paths = W > 1 ? 1 : (A.B - b0 < A.groups ? (int)(A.B - b0) : A.groups);
    const int points = W > 1 && L - j0 > A.steps ? A.steps : (int)(L - j0);
    float *mat = sig_bracket_smem, *ends = mat + paths * M;
    const float *g = A.grad_out + b0 * D, *s = A.sig + b0 * D;
    for (int i = tid; i < paths * d * d; i += kDepth2Threads) {
        const int p = i / (d * d), w = i - p * (d * d);
        const int a = w / d, b = w - a * d;
        const float *G2 = g + (int64_t)p * D + d;
        mat[p * M + a * ROW + b] = 0.5f * (G2[w] - G2[b * d + a]);
    }
    for (int i = tid; i < paths * 2 * d; i += kDepth2Threads) {
        const int p = i / (2 * d), o = i - p * (2 * d);
        const int b = o % d;
        const float *Gp = g + (int64_t)p * D, *Sp = s + (int64_t)p * D;
        float sum = Gp[b];
#pragma unroll
        for (int a = 0; a < d; ++a) sum = fmaf(Sp[a], Gp[d + (o < d ? a * d + b : b * d + a)], sum);
        ends[i] = o < d ? sum : -sum;
    }
    __syncthreads();
    for (int i = tid; i < paths * points; i += kDepth2Threads) {
        const int p = paths == 1 ? 0 : i / points;
        const int64_t j = j0 + (i - p * points);
        const float *X = A.path + ((b0 + p) * A.L + j) * d;
        const float *before = j > 0 ? X - d : X, *after = j < L - 1 ? X + d : X;
        float v[d], acc[d];
#pragma unroll
        for (int a = 0; a < d; ++a) v[a] = before[a] - after[a];
#pragma unroll
        for (int b = 0; b < d; ++b) acc[b] = 0.0f;
        if (j == 0 || j == L - 1) {
            const float *e = ends + p * 2 * d + (j == 0 ? d : 0);
#pragma unroll
            for (int b = 0; b < d; ++b) acc[b] = e[b];
        }
        const float *m = mat + p * M;
#pragma unroll
        for (int a = 0; a < d; ++a)
#pragma unroll
            for (int b = 0; b < d; ++b) acc[b] = fmaf(v[a], m[a * ROW + b], acc[b]);
        onchip::store_run<0, d, d>(A.grad_path + ((b0 + p) * A.L + j) * d, acc);
    }
}

}  // namespace bracket
}  // namespace sig

#endif  // SIG_BRACKET_H_
