// Host-side sweep of libsig's planning and validation logic, built with AddressSanitizer and
// UndefinedBehaviorSanitizer by tests/test_host_sanitized.py (no GPU: nothing is launched, every entry point used here is
// host only or takes a NULL context).  Any out-of-bounds access, signed overflow or other undefined arithmetic in the
// planner, the plan checks or the gradient's segment rule ends the run; the invariants below are checked on top.
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <initializer_list>

#include "sig.h"

namespace sig {   // csrc/sig_internal.h
bool bracket_depth2_geometry(int d, int64_t B, int64_t L, int cus, int64_t *grid, int64_t *segs, int64_t *steps, int64_t *groups,
                             int64_t *lds_bytes);
bool stream_gradient_geometry(int d, int64_t B, int64_t L, int cus, bool scratch, int64_t *scratch_floats, int64_t *grid, int64_t *segs,
                              int64_t *groups, int64_t *chunks, int64_t *steps, int64_t *rows);
int64_t stream_gradient3_scratch_floats(int d, int64_t B, int64_t L, int cus);
struct SplitRowsCut {
    int64_t lds_bytes, workgroups, scratch_floats;
    int threads;
    int64_t segs, rows;
    int64_t slices, lanes;
    int64_t chunks, groups;
};
bool split_rows_geometry(int d, int depth, int64_t B, int64_t L, int segs, int cus, bool registers, SplitRowsCut *cut);
}

static uint64_t state = 0x9E3779B97F4A7C15ull;
static uint64_t rnd()
{
    state ^= state << 13;
    state ^= state >> 7;
    state ^= state << 17;
    return state;
}
static int64_t pick(const int64_t *v, int n) { return v[rnd() % (uint64_t)n]; }

static long checked = 0, planned = 0, failures = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { ++failures; std::printf("FAILED %s: ", #cond); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)

static void one_shape(int64_t B, int64_t L, int d, int depth, int stream)
{
    ++checked;
    sig_plan_t pl;
    const int rc = sig_plan(nullptr, B, L, d, depth, stream, &pl);
    EXPECT(rc == SIG_OK || rc == SIG_ERR_INVALID || rc == SIG_ERR_TOO_LARGE, "sig_plan(%lld,%lld,%d,%d,%d) = %d", (long long)B, (long long)L, d, depth, stream, rc);
    const int segs = sig_backward_segments(nullptr, B, L, d, depth, stream);
    EXPECT(segs >= -6 && segs <= 32, "sig_backward_segments = %d", segs);
    if (rc == SIG_ERR_INVALID) EXPECT(segs == -SIG_ERR_INVALID, "arguments invalid for the forward call but not for the gradient: %d", segs);
    if (rc != SIG_OK) return;
    ++planned;
    EXPECT(pl.variant >= SIG_VARIANT_HBM_STREAMING && pl.variant <= SIG_VARIANT_LEVEL_SCAN, "variant %d", pl.variant);
    const int v = sig_plan_validate(B, L, d, depth, stream, &pl);
    EXPECT(v == SIG_OK, "the planner's own plan is refused (%d): B=%lld L=%lld d=%d depth=%d stream=%d variant=%d p=%d chunks=%d segments=%d threads=%d",
           v, (long long)B, (long long)L, d, depth, stream, pl.variant, pl.prefix_depth, pl.chunks, pl.segments, pl.threads);
    int64_t lds = 0, wgs = 0, scratch = 0;
    const int f = sig_plan_footprint(B, L, d, depth, stream, &pl, &lds, &wgs, &scratch);
    EXPECT(f == SIG_OK, "footprint %d", f);
    if (f == SIG_OK) {
        EXPECT(lds <= 64 * 1024, "LDS %lld bytes: B=%lld L=%lld d=%d depth=%d stream=%d", (long long)lds, (long long)B, (long long)L, d, depth, stream);
        EXPECT(wgs <= INT32_MAX && (wgs >= 1 || wgs == -1 || B == 0), "workgroups %lld", (long long)wgs);
        EXPECT(scratch >= 0 && scratch <= (int64_t)8 << 30, "scratch %lld: B=%lld L=%lld d=%d depth=%d stream=%d segments=%d", (long long)scratch, (long long)B, (long long)L, d, depth, stream, pl.segments);
        if (pl.variant == SIG_VARIANT_ON_CHIP) EXPECT(wgs * pl.threads < (int64_t)1 << 32, "%lld workgroups of %d threads: B=%lld L=%lld d=%d depth=%d stream=%d", (long long)wgs, pl.threads, (long long)B, (long long)L, d, depth, stream);
    }
    if (pl.variant == SIG_VARIANT_ON_CHIP) {
        EXPECT(pl.threads >= 64 && pl.threads <= 512 && pl.threads % 64 == 0, "threads %d", pl.threads);
        EXPECT(pl.chunks >= 1 && pl.segments >= 1 && (int64_t)pl.chunks * pl.segments <= L - 1, "chunks %d segments %d for %lld increments", pl.chunks, pl.segments, (long long)(L - 1));
        EXPECT(sig_on_chip_available(d, depth, pl.prefix_depth) == 1, "no kernel for (%d,%d,%d)", d, depth, pl.prefix_depth);
        EXPECT(!stream || pl.segments == 1, "stream mode cut across workgroups");
    }
}

int main()
{
    // ---- sizes and tables
    for (int d = -1; d <= 40; ++d)
        for (int depth = -1; depth <= 70; ++depth) {
            const int64_t D = sig_size(d, depth);
            EXPECT(D >= -1, "sig_size");
            (void)sig_on_chip_available(d, depth, depth > 0 ? depth - 1 : 0);
            (void)sig_backward_available(d, depth);
        }
    for (int s = -3; s <= 12; ++s) EXPECT(sig_strerror(s) != nullptr, "sig_strerror(%d)", s);

    // ---- the planner on seeded shapes: the compiled grid (channels 2-10, depths 1-7), odd shapes beyond it, extremes
    const int64_t Bs[] = {0, 1, 2, 3, 7, 16, 64, 128, 300, 1000, 4096, 65536, 1 << 20, 5000000, (int64_t)1 << 31, (int64_t)1 << 40};
    const int64_t Ls[] = {1, 2, 3, 9, 16, 50, 100, 128, 129, 256, 257, 500, 1000, 2000, 4001, 50000, 1 << 20, (int64_t)1 << 33};
    for (int it = 0; it < 6000; ++it) {
        const int64_t B = pick(Bs, sizeof Bs / sizeof *Bs), L = pick(Ls, sizeof Ls / sizeof *Ls);
        const int d = (int)(rnd() % 11), depth = (int)(rnd() % 8), stream = (int)(rnd() % 2);
        one_shape(B, L, d, depth, stream);
    }
    for (int it = 0; it < 2000; ++it) {
        const int64_t B = (int64_t)(rnd() % 3000), L = (int64_t)(rnd() % 5000);
        const int d = (int)(rnd() % 300), depth = (int)(rnd() % 12), stream = (int)(rnd() % 3) - (int)(rnd() % 2);
        one_shape(B, L, d, depth, stream);
    }
    for (int it = 0; it < 4000; ++it) {   // more than ten channels: large batches and long paths
        const int d = 11 + (int)(rnd() % 10), depth = d <= 12 && (rnd() & 1) ? 3 : 2;
        one_shape((int64_t)1 << (rnd() % 25), 2 + (int64_t)(rnd() % ((uint64_t)1 << (1 + rnd() % 14))), d, depth, (int)(rnd() % 2));
    }
    const int ds[] = {1, 2, 10, 255, 256, 257, 8192, 8193, 100000};
    const int depths[] = {1, 2, 8, 9, 29, 30, 31, 64};
    for (int d : ds)
        for (int depth : depths)
            for (int64_t B : {(int64_t)1, (int64_t)100, (int64_t)1 << 45})
                for (int64_t L : {(int64_t)2, (int64_t)1000, (int64_t)1 << 50})
                    for (int stream = 0; stream < 2; ++stream) one_shape(B, L, d, depth, stream);

    // ---- the launch of the depth-2 gradient: every point has its workgroup, and a launch holds fewer than 2^32 threads,
    // for every batch that a GPU of 288 GB could hold (path and its gradient, the rows and theirs)
    for (int it = 0; it < 20000; ++it) {
        const int d = 2 + (int)(rnd() % 19);
        const int64_t L = it & 1 ? pick(Ls, sizeof Ls / sizeof *Ls) : 2 + (int64_t)(rnd() % 3000);
        if (L < 2) continue;
        int64_t B = it & 2 ? (int64_t)1 << (rnd() % 33) : 1 + (int64_t)(rnd() % ((uint64_t)1 << (1 + rnd() % 33)));
        const int64_t most = ((int64_t)288 << 30) / (8 * (L * d + d + d * d));
        if (B > most) B = most;
        if (B < 1) continue;
        int64_t grid = 0, segs = 0, steps = 0, groups = 0, lds = 0;
        const bool ok = sig::bracket_depth2_geometry(d, B, L, 256, &grid, &segs, &steps, &groups, &lds);
        EXPECT(ok && grid >= 1 && grid * 256 < (int64_t)1 << 32 && lds <= 64 * 1024, "depth 2, d=%d B=%lld L=%lld: %d grid %lld lds %lld", d, (long long)B, (long long)L, ok, (long long)grid, (long long)lds);
        if (segs > 1) EXPECT(grid == B * segs && groups == 1 && segs * steps >= L && (segs - 1) * steps < L, "stretches: d=%d B=%lld L=%lld %lld x %lld", d, (long long)B, (long long)L, (long long)segs, (long long)steps);
        else EXPECT(grid * groups >= B && (grid - 1) * groups < B, "paths: d=%d B=%lld L=%lld grid %lld x %lld", d, (long long)B, (long long)L, (long long)grid, (long long)groups);
        ++checked;
    }

    // ---- the launches of the every-prefix gradient at depth 2: every row of every path has its slot, in one workgroup only
    for (int it = 0; it < 20000; ++it) {
        const int d = 2 + (int)(rnd() % 19);
        const int64_t L = it & 1 ? pick(Ls, sizeof Ls / sizeof *Ls) : 2 + (int64_t)(rnd() % 3000), K = L - 1, D = d + d * d;
        if (L < 2) continue;
        const int64_t B = it & 2 ? (int64_t)1 << (rnd() % 33) : 1 + (int64_t)(rnd() % ((uint64_t)1 << (1 + rnd() % 20)));
        const bool scratch = (it & 4) != 0;
        int64_t floats = 0, grid = 0, segs = 0, groups = 0, chunks = 0, steps = 0, rows = 0;
        const int answer = sig_backward_segments(nullptr, B, L, d, 2, 1);
        if (!sig::stream_gradient_geometry(d, B, L, 256, scratch, &floats, &grid, &segs, &groups, &chunks, &steps, &rows)) {
            // (a path to each workgroup at least, or whole paths side by side, and offsets of 32 bits)
            EXPECT(L > INT32_MAX / 2 || K > INT32_MAX / D / (scratch && B <= 8 ? 32 : 1) - 16 || B >= (int64_t)1 << 26 || (B >= (int64_t)1 << 24 && L > INT32_MAX / D / (64 / d)), "no launch: d=%d B=%lld L=%lld", d, (long long)B, (long long)L);
            continue;
        }
        EXPECT(!scratch || answer == segs || answer < 0, "sig_backward_segments = %d for %lld: d=%d B=%lld L=%lld", answer, (long long)segs, d, (long long)B, (long long)L);
        const bool uncut = segs == 1 && chunks == 1 && groups == 64 / d;
        EXPECT(grid >= 1 && grid * (uncut ? 64 : 256) < (int64_t)1 << 32, "threads: d=%d B=%lld L=%lld", d, (long long)B, (long long)L);
        EXPECT(groups * (segs > 1 ? rows : K) <= INT32_MAX / D, "offsets: d=%d B=%lld L=%lld", d, (long long)B, (long long)L);
        EXPECT(floats == (segs > 1 ? B * segs * D : 0) && (scratch || segs == 1) && segs <= 32, "scratch: d=%d B=%lld L=%lld", d, (long long)B, (long long)L);
        if (segs > 1) EXPECT(grid == B * segs && groups == 1 && rows % (chunks * steps) == 0 && segs * rows >= K && (segs - 1) * rows < K, "d=%d B=%lld L=%lld: %lld x %lld rows", d, (long long)B, (long long)L, (long long)segs, (long long)rows);
        else EXPECT(grid * groups >= B && (grid - 1) * groups < B && (groups == 1 || chunks * steps >= K), "d=%d B=%lld L=%lld: %lld paths", d, (long long)B, (long long)L, (long long)groups);
        if (d == 11 || d == 12) {
            const int64_t need = sig::stream_gradient3_scratch_floats(d, B, L, 256);
            EXPECT(need >= B * K * d * (d + 2) || (need == -1 && (L * D * d * 2 > INT32_MAX || B > (int64_t)1 << 24)), "depth 3: d=%d B=%lld L=%lld scratch %lld", d, (long long)B, (long long)L, (long long)need);
        }
        EXPECT(groups * chunks <= 4 * (64 / d), "slots: d=%d B=%lld L=%lld", d, (long long)B, (long long)L);
        ++checked;
    }

    // ---- ... and of calls whose whole paths take one workgroup more than the chip holds, or too few of them
    const int64_t bands[][3] = {{8, 2631, 255}, {10, 1970, 318}, {7, 2970, 311}, {7, 3072, 380}, {9, 2498, 243}, {6, 3588, 338}};
    for (const auto &b : bands) {
        int64_t floats = 0, grid = 0, segs = 0, groups = 0, chunks = 0, steps = 0, rows = 0;
        EXPECT(sig::stream_gradient_geometry((int)b[0], b[1], b[2], 256, true, &floats, &grid, &segs, &groups, &chunks, &steps, &rows) && chunks > 1,
               "d=%lld B=%lld L=%lld stays uncut", (long long)b[0], (long long)b[1], (long long)b[2]);
    }

    // ---- rows split across workgroups, and depth-2 rows: every word of every row of every path has its lane, in one workgroup only
    const int split_shapes[][2] = {{10, 3}, {8, 4}, {9, 4}, {10, 4}, {5, 5}, {6, 5}, {4, 6}};
    for (int it = 0; it < 40000; ++it) {
        const bool two = it % 3 != 0;
        const int *shape = split_shapes[rnd() % 7];
        const int d = two ? 2 + (int)(rnd() % 19) : shape[0], depth = two ? 2 : shape[1];
        const int64_t L = it & 1 ? pick(Ls, sizeof Ls / sizeof *Ls) : 2 + (int64_t)(rnd() % 3000), K = L - 1;
        const int64_t B = it & 2 ? (int64_t)1 << (rnd() % 33) : 1 + (int64_t)(rnd() % ((uint64_t)1 << (1 + rnd() % 20)));
        const int segs = 1 + (int)(rnd() % 32), cus = it & 4 ? 256 : 64 << (rnd() % 3);
        int64_t words = 1, row = 0, power = 1;
        for (int n = 1; n < depth; ++n) words *= d;
        for (int n = 1; n <= depth; ++n) row += power *= d;
        sig::SplitRowsCut c{};
        if (!sig::split_rows_geometry(d, depth, B, L, segs, cus, (it & 8) != 0, &c)) {
            EXPECT(L < 2 || segs > K || L > INT32_MAX / (two ? 32 * row : 2) || B >= ((int64_t)1 << (two ? 24 : 21)) / segs, "no cut: d=%d depth=%d B=%lld L=%lld segs=%d", d, depth, (long long)B, (long long)L, segs);
            continue;
        }
        EXPECT(c.lds_bytes <= 64 * 1024 && c.workgroups >= 1 && c.workgroups * c.threads < (int64_t)1 << 32, "d=%d depth=%d B=%lld L=%lld segs=%d: %lld x %d threads", d, depth, (long long)B, (long long)L, segs, (long long)c.workgroups, c.threads);
        EXPECT(c.segs >= 1 && c.segs <= segs && c.segs * c.rows >= K && (c.segs - 1) * c.rows < K, "rows: d=%d depth=%d B=%lld L=%lld segs=%d: %lld x %lld", d, depth, (long long)B, (long long)L, segs, (long long)c.segs, (long long)c.rows);
        if (two) {
            EXPECT(c.groups * c.chunks <= c.lanes && c.lanes <= c.threads / 64 * (64 / d) && c.scratch_floats == 0, "slots: d=%d B=%lld L=%lld segs=%d", d, (long long)B, (long long)L, segs);
            EXPECT(c.segs > 1 ? c.groups == 1 && c.workgroups == B * c.segs : c.workgroups * c.groups >= B && (c.workgroups - 1) * c.groups < B, "paths: d=%d B=%lld L=%lld segs=%d", d, (long long)B, (long long)L, segs);
            EXPECT(c.groups * L <= INT32_MAX / row, "offsets: d=%d B=%lld L=%lld segs=%d", d, (long long)B, (long long)L, segs);
        } else {
            EXPECT(c.workgroups == B * c.segs * c.slices && c.scratch_floats == B * (c.segs - 1) * row && c.rows % 8 == 0, "d=%d depth=%d B=%lld L=%lld segs=%d", d, depth, (long long)B, (long long)L, segs);
            EXPECT(c.slices * c.lanes >= words && (c.slices - 1) * c.lanes < words && c.lanes <= c.threads && c.lanes > c.threads - 64, "words: d=%d depth=%d B=%lld L=%lld segs=%d: %lld x %lld", d, depth, (long long)B, (long long)L, segs, (long long)c.slices, (long long)c.lanes);
        }
        ++checked;
    }

    // ---- arbitrary plans through the checks: they may be refused, they must not misbehave
    for (int it = 0; it < 20000; ++it) {
        sig_plan_t pl;
        int32_t *f = reinterpret_cast<int32_t *>(&pl);
        for (unsigned i = 0; i < sizeof pl / sizeof(int32_t); ++i) {
            const uint64_t r = rnd();
            f[i] = (r & 7) == 0 ? (int32_t)(r >> 32) : (int32_t)((r >> 8) % 40) - 2;
        }
        pl.variant = (int32_t)(rnd() % 5);
        if (rnd() & 1) pl.threads = 64 * (int32_t)(1 + rnd() % 8);
        const int64_t B = pick(Bs, 12), L = pick(Ls, 14);
        const int d = 1 + (int)(rnd() % 10), depth = 1 + (int)(rnd() % 6), stream = (int)(rnd() % 2);
        const int v = sig_plan_validate(B, L, d, depth, stream, &pl);
        int64_t lds = 0, wgs = 0, scratch = 0;
        const int fp = sig_plan_footprint(B, L, d, depth, stream, &pl, &lds, &wgs, &scratch);
        EXPECT((v == SIG_OK) == (fp == SIG_OK), "validate %d but footprint %d", v, fp);
        if (fp == SIG_OK) EXPECT(lds <= 64 * 1024 && wgs <= INT32_MAX && scratch >= 0, "forced plan: lds %lld workgroups %lld scratch %lld", (long long)lds, (long long)wgs, (long long)scratch);
        ++checked;
    }
    EXPECT(sig_plan(nullptr, 1, 2, 2, 2, 0, nullptr) == SIG_ERR_INVALID, "NULL plan");
    EXPECT(sig_plan_validate(1, 2, 2, 2, 0, nullptr) == SIG_ERR_INVALID, "NULL plan");
    EXPECT(sig_plan_footprint(1, 2, 2, 2, 0, nullptr, nullptr, nullptr, nullptr) == SIG_ERR_INVALID, "NULL plan");

    std::printf("host sweep: %ld cases, %ld planned, %ld failures\n", checked, planned, failures);
    if (failures == 0) std::printf("host sweep ok\n");
    return failures == 0 ? 0 : 1;
}
