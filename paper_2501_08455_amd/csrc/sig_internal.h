// Internal declarations shared by the host API and the kernel translation units of libsig.
// Nothing here is part of the C ABI (that is include/sig.h).
#ifndef SIG_INTERNAL_H
#define SIG_INTERNAL_H

#include <hip/hip_runtime.h>
#include <stdint.h>

#include "sig.h"

namespace sig {

constexpr int kMaxDepth = 30;        // d^depth must also fit in int32
constexpr int kWave = 64;
constexpr int kMaxLdsBytes = 64 * 1024;  // per-workgroup LDS this library asks for at most
constexpr int kCuLdsBytes = 160 * 1024;  // LDS of one compute unit, shared by its resident workgroups
constexpr int kTileLdsBytes = 19968;     // LDS the increment tile(s) of one workgroup may take (8 workgroups share 160 KB)
constexpr int kFoldTileSteps = 32;       // increments a wavefront of the fold kernel stages at a time
constexpr int kLoaderStage = 8;          // floats of the next tile one thread holds in registers when tiles are pipelined

// Offsets of the levels inside an output row (Eq. 10: level 0 dropped): level n starts at
// d + ... + d^{n-1} and holds d^n floats.
struct RowShape {
    int d;
    int depth;
    int64_t D;                      // row length
    int64_t pow[kMaxDepth + 2];     // pow[n] = d^n
    int64_t off[kMaxDepth + 2];     // off[n] = start of level n (n >= 1), off[depth + 1] = D
};

// returns false if d^depth or D overflow the supported range
bool make_row_shape(int d, int depth, RowShape *rs);

// ---------------------------------------------------------------- HBM-streaming family (any d, depth)
// One workgroup per (path, sub-tree of prefix depth p); the state is the output row itself.
hipError_t launch_hbm_streaming(const float *path, float *out, int64_t B, int64_t L, const RowShape &rs,
                                int p, int stream_flag, int threads, hipStream_t st);

// out[b] = a[b] (x) b[b] on rows of D floats (Eq. 4 with implied level 0 = 1); strides in floats.
hipError_t launch_combine_rows(const float *a, int64_t a_stride, const float *b, int64_t b_stride,
                               float *out, int64_t out_stride, int64_t B, const RowShape &rs,
                               hipStream_t st);

// The same for rows that follow each other without a gap, compiled (d, depth) only (sig_combine.hip).
bool combine_tree_compiled(int d, int depth);
hipError_t launch_combine_tree(const float *a, const float *b, float *out, int64_t B, int d, int depth, hipStream_t st);

// ---------------------------------------------------------------- level-scan family (d <= 256, depth <= 8)
// The level-by-level formulation of the paper's Section 3.2: one launch per level, each a cumulative sum over time
// of per-step terms built from the lower levels of every prefix, which live in `scratch` (level_scan_scratch_floats
// floats in both modes, one dense [B][L-1][d^m] tensor per level m < depth).
bool level_scan_available(int d, int depth);
int64_t level_scan_scratch_floats(int64_t B, int64_t L, const RowShape &rs, int stream_flag);
// false if the rows of one path cannot be addressed with 32-bit offsets
bool level_scan_fits(int64_t L, const RowShape &rs, int stream_flag);
// time chunks of one (path, parent word) at `level`; forced > 0 overrides the choice (clamped to the path)
int level_scan_chunks(int64_t B, int64_t L, const RowShape &rs, int level, int forced, int cus);
hipError_t launch_level_scan(const float *path, float *out, float *scratch, int64_t B, int64_t L, const RowShape &rs,
                             int stream_flag, int forced_chunks, int cus, hipStream_t st);

// ---------------------------------------------------------------- gradient with respect to the path (compiled (d, depth) only)
bool backward_available(int d, int depth);
// false if even one path per workgroup does not fit the LDS of the uncut sweep (the increments of a whole path are
// staged at once); such paths are walked in tiles by launch_backward (sequential in time, needs scratch)
bool backward_fits(int d, int depth, int64_t L);
// whether a tile of the tiled sweep fits LDS (true for every compiled shape; checked before launching)
bool backward_tiles_fit(int d, int depth);
// device scratch the launch needs (shapes whose lanes per path span several workgroups keep per-slice sums), in floats
int64_t backward_scratch_floats(int d, int depth, int64_t B, int64_t L);
hipError_t launch_backward(const float *path, const float *sig, const float *grad_out, float *grad_path, float *scratch,
                           int64_t B, int64_t L, int d, int depth, int stream_flag, int cus, hipStream_t st);

// d(loss)/dX from per-slice sums of d(loss)/d(increment), part = [B][slices][L-1][d]
hipError_t launch_backward_finish(const float *part, float *grad_path, int64_t B, int64_t L, int d, int slices,
                                  hipStream_t st);

// ---------------------------------------------------------------- gradient cut in time across workgroups
// Time segments the sweep should be cut into (<= 1: do not cut); uncut_fits = backward_fits(d, depth, L)
int backward_segments(int d, int depth, int64_t B, int64_t L, int cus, bool uncut_fits, int stream_flag);
int64_t backward_segmented_scratch_floats(int d, int depth, int64_t B, int64_t L, int segs);
hipError_t launch_backward_segmented(const float *path, const float *sig, const float *grad_out, float *grad_path,
                                     float *scratch, int64_t B, int64_t L, int d, int depth, int stream_flag, int segs,
                                     int cus, hipStream_t st);

// ---------------------------------------------------------------- gradient of the final signature on Lie brackets
// (sig_bracket.h; any length).  Compiled shapes:
constexpr bool bracket_compiled(int d, int depth)
{
    return d >= 2 && (depth == 2 ? d <= 20 : depth == 3 ? d <= 16 : depth == 4 ? d <= 10 : depth == 5 ? d <= 6 : depth == 6 && d <= 4);
}
// The sweep on brackets pays for the bracket values of a path once (2^{depth-1} words each) and then next to nothing per
// step; the sweep on signatures (sig_backward.hip) has no such start, and stays for paths of fewer points than this.  From
// depth 4 on some 12 + D / 150, twice the second term at depth 6, and D 2^{depth-1} / 2500 where the rows are too long for the
// packed kernel at depth 5 and 6.  Measured on batches that fill the chip, points per path where the two meet: (4,4) 14, (5,4)
// 15, (6,4) 16, (7,4) 33, (8,4) 12, (10,4) 9, (3,5) 17, (4,5) 16, (5,5) 25, (6,5) 45, (3,6) 32, (4,6) 80.  The other terms:
// where the batch moves that point (a grid of all compiled shapes x 2 ... 70 points x 1 ... 100,000 paths).  Some hundred to
// ten thousand paths leave a wavefront of the packed kernel few of them, and its start is not shared ((2,3), 10 points,
// 1,600 paths 4.3 us on signatures and 6.8 on brackets; (3,5), 14 points, 8,000 paths 13.5 and 18.0); tens of thousands of
// short paths are bound by reading their rows, which the packed kernel stages a few at a time ((7,3), 8 points, 100,000
// paths 50 and 87 us); up to some hundred of 8 to 10 channels pay for the chunked kernel's phases ((8,3), 8 points 4.5 and 6.0).
constexpr int64_t bracket_min_points(int d, int depth, int64_t B)
{
    const bool some = B >= 512, many = B >= 4096, full = B >= 16384, flood = B >= 65536;
    const bool lone = B >= 1024 && B < 2048;   // a wavefront of the packed kernel for every path
    if (d > 10) return 2;
    if (depth == 2) return B < 64 ? 2 : flood ? (d > 8 ? 8 : d) : many && (!full || d > 8) ? d - 2 : full ? d - 1 : d;
    if (depth == 3) {
        if (d == 2) return full ? 7 : lone ? 21 : some ? 17 : 13;
        if (d <= 4) return many ? (flood && d == 4 ? 9 : 8) : some ? 12 : 8;
        if (d <= 7) return d == 5 ? (flood ? 9 : some ? 8 : 5) : flood ? 17 : full ? 13 : some ? 8 : 5;
        if (d == 8) return many ? 8 : 12;
        return B < 1024 ? 10 : 6;
    }
    if (depth == 4 && d > 7) return d > 8 && B < 128 ? 3 * d - 14 : 12;
    if (depth == 4 && d == 2) return full ? 12 : lone ? 25 : some ? 17 : 13;
    if (depth == 4 && d == 4 && many) return 17;
    if (depth == 5 && d == 3 && B >= 1024) return many && !full ? 20 : 17;
    int64_t D = 0, p = 1;
    for (int n = 1; n <= depth; ++n) D += p *= d;
    if (D > 3000) return (D << (depth - 1)) / 2500 + (B < 1024 ? 0 : depth == 6 ? 9 : 1);
    return 12 + (depth >= 6 ? 2 : 1) * D / 150;
}
constexpr bool bracket_wanted(int d, int depth, int64_t B, int64_t L) { return bracket_compiled(d, depth) && L >= bracket_min_points(d, depth, B); }
// workgroups a path's steps are cut across (1: not cut)
int bracket_segments(int d, int depth, int64_t B, int64_t L, int cus);
bool bracket_depth2_geometry(int d, int64_t B, int64_t L, int cus, int64_t *grid, int64_t *segs, int64_t *steps, int64_t *groups,
                             int64_t *lds_bytes);
hipError_t launch_bracket(const float *path, const float *sig, const float *grad_out, float *grad_path, int64_t B, int64_t L,
                          int d, int depth, int segs, int cus, hipStream_t st);

// ---------------------------------------------------------------- gradient of the every-prefix signature at depth 2 and 3 (sig_stream_gradient.hip)
// Floats of scratch the launch would like (0: none); < 0 if there is no such launch (more than 20 channels, 2^30 points).  Without
// scratch (null) a path stays in one workgroup (hipErrorNotSupported: its rows take 2^31 floats).
int64_t stream_gradient_scratch_floats(int d, int64_t B, int64_t L, int cus);
bool stream_gradient_geometry(int d, int64_t B, int64_t L, int cus, bool scratch, int64_t *scratch_floats, int64_t *grid, int64_t *segs,
                              int64_t *groups, int64_t *chunks, int64_t *steps, int64_t *rows);
hipError_t launch_stream_gradient(const float *path, const float *grad_out, float *grad_path, float *scratch, int64_t B, int64_t L,
                                  int d, int cus, hipStream_t st);
// Workgroups a path, of either depth's launch with scratch (0: there is none)
int stream_gradient_segments(int d, int depth, int64_t B, int64_t L, int cus);
// Depth 3, eleven and twelve channels: floats of scratch the launches need (< 0: there are none), and the launches.  sig: [B][L-1][D]
int64_t stream_gradient3_scratch_floats(int d, int64_t B, int64_t L, int cus);
hipError_t launch_stream_gradient3(const float *path, const float *sig, const float *grad_out, float *grad_path, float *scratch, int64_t B,
                                   int64_t L, int d, int cus, hipStream_t st);

// ---------------------------------------------------------------- gradient, any (d <= 256, depth): one workgroup per path
bool backward_general_available(int d);
int64_t backward_general_scratch_floats(int64_t B, int64_t L, const RowShape &rs);
hipError_t launch_backward_general(const float *path, const float *sig, const float *grad_out, float *grad_path,
                                   float *scratch, int64_t B, int64_t L, const RowShape &rs, int stream_flag,
                                   hipStream_t st);

// ---------------------------------------------------------------- on-chip family (compiled (d, depth, p) only)
struct OnChipArgs {
    const float *path;   // [B][L][d]
    float *out;          // final: [B][D]; stream: [B][K][D]
    float *partial;      // [B][segments][D] scratch when segments > 1, else unused
    int64_t B;
    int64_t L;
    int32_t chunks;      // C: time chunks per (path, segment) folded side by side in one workgroup
    int32_t segments;    // W: workgroups per path along time
    int32_t chunk_steps; // T: increments per chunk; segments * chunks * T >= L - 1
    int32_t tile_steps;  // TT: increments per LDS tile
    int32_t threads;     // workgroup size
    int32_t groups;      // (path, segment) pairs per workgroup (1 when a chunk's lanes span several workgroups)
    int32_t row_shift;   // log2 of the padded length of one chunk's stretch of a tile (tile_steps * d floats)
    int32_t resident_workgroups;  // workgroups the device keeps resident at once (persistent kernels); 0: no limit
    int32_t stagger_ticks;  // start delay (100 MHz ticks) per residency slot of the first wave of workgroups; 0: none
    int32_t num_cus;        // compute units of the device
    int32_t cooperative;  // chunks == 1 only: 1 = workgroup-wide tiles with barriers instead of independent wavefronts
    int32_t pipe;         // several tiles per chunk: 1 = the next tile's loads stay in flight in registers while the current
                          // one is consumed (hides the load latency inside one workgroup), 0 = load, barrier, consume
                          // (fewer registers; the other resident workgroups hide the latency)
    int32_t flat_tile;    // 1: the workgroup's paths are whole and adjacent in memory and fit one tile: the tile is a
                          // straight copy of that range (rows of L * d floats), differenced on the way
    int32_t stream_flag;
    int32_t shared_chain; // 1: final mode, one chunk, lanes of a path spanning several workgroups, prefix depth >= 2: the
                          // prefix part of the Horner chains comes from a table in LDS that a few lanes of the workgroup
                          // fill once (the whole (path, segment) is one tile: tile_steps = chunk_steps)
};

// The fold that shares the prefix part of the Horner chains (sig_shared_chain_kernel) takes the `steps` increments of a
// (path, segment) as one tile.  LDS floats of a workgroup: the increments [steps][d], the table [steps][nq][depth - p + 1]
// with nq the prefixes of length p - 1 the words of one workgroup can have, the chunk totals of the table's running sums
// (one float per thread and level at most), and the totals of the words at the segment's end.
constexpr int64_t shared_chain_round4(int64_t x) { return (x + 3) / 4 * 4; }
constexpr int64_t shared_chain_prefixes(int d, int threads) { return (threads - 1) / d + 2; }
constexpr int64_t shared_chain_lds_floats(int d, int depth, int p, int threads, int64_t steps)
{
    const int64_t nq = shared_chain_prefixes(d, threads);
    return shared_chain_round4(steps * d) + shared_chain_round4(steps * nq * (depth - p + 1)) + (p - 1) * shared_chain_round4(threads) +
           shared_chain_round4((p - 1) * nq);
}
// whether a segment of `steps` increments fits: 52 KB of LDS (three workgroups per compute unit), a table builder per
// prefix among the threads, and at most 16 steps per builder (prefixes take a power of two of thread slots, the chunks of
// steps the rest)
constexpr bool shared_chain_fits(int d, int depth, int p, int threads, int64_t steps)
{
    const int64_t nq = shared_chain_prefixes(d, threads);
    int64_t slots = 1;
    while (slots < nq) slots *= 2;
    return steps >= 1 && slots <= threads && (threads / slots) * 16 >= steps &&
           shared_chain_lds_floats(d, depth, p, threads, steps) * (int64_t)sizeof(float) <= 52 * 1024;
}

struct OnChipKernelInfo {
    int d, depth, p;
    int lanes_per_chunk;                       // Q = d^p
    int state_floats;                          // registers of state per lane
    int row_floats;                            // LDS floats per staged increment (= d)
    hipError_t (*launch)(const OnChipArgs &, hipStream_t);
    // LDS bytes the launch needs for these arguments (for validation before launching)
    int64_t (*lds_bytes)(const OnChipArgs &);
    // out[b] = product over the `segments` partial rows of path b (second launch when segments > 1)
    hipError_t (*join)(const float *partial, float *out, int64_t B, int segments, hipStream_t);
    bool final_only;                           // no stream mode is compiled
    bool matrix_fold;                          // final-mode folds on matrix instructions (quad_fold in sig_onchip.h)
};

// Work items of an on-chip launch with Q = d^p lanes per (path, chunk): one per slice of a path's lanes when they exceed
// a workgroup, else one per `groups` (path, segment) pairs.  <= 0: invalid arguments.
inline int64_t on_chip_work_items(int Q, const OnChipArgs &A)
{
    const int64_t ngroups = A.B * A.segments;
    if (Q > A.threads) {
        if (A.chunks != 1 || A.groups != 1) return -1;
        return ngroups * ((Q + A.threads - 1) / A.threads);
    }
    if (A.groups < 1) return -1;
    return (ngroups + A.groups - 1) / A.groups;
}
// Workgroups launched: one per work item, except that the kernels with independent wavefronts launch no more workgroups
// than stay resident and let each walk the same number of items.
inline int64_t on_chip_workgroups(int Q, const OnChipArgs &A)
{
    int64_t grid = on_chip_work_items(Q, A);
    if (A.chunks == 1 && !A.cooperative && grid > 0) {
        int64_t resident = A.resident_workgroups > 0 ? A.resident_workgroups : grid;
        if (resident > grid) resident = grid;
        const int64_t rounds = (grid + resident - 1) / resident;
        grid = (grid + rounds - 1) / rounds;
    }
    return grid;
}

// ---------------------------------------------------------------- stream mode, rows written straight from registers (sig_stream_rows.h)
// workgroups a path is cut across, 0 if the call stays with the other kernels (held_p: prefix depth of the register kernel that it
// would take, -1 for one launch per level)
int stream_rows_wanted(int d, int depth, int64_t B, int64_t L, int cus, int held_p);
// ... that a launch would cut them across whether or not it is wanted, 0 if there is none
int stream_rows_segments(int d, int depth, int64_t B, int64_t L, int cus);
// the launch with `segs` workgroups a path; false if there is none
bool stream_rows_geometry(int d, int depth, int64_t B, int64_t L, int segs, int cus, int64_t *lds_bytes, int64_t *workgroups, int *threads);
hipError_t launch_stream_rows(const float *path, float *out, int64_t B, int64_t L, int d, int depth, int segs, int cus, hipStream_t st);

// ---------------------------------------------------------------- what the planners of the kernels below and of the every-prefix gradient share
// Workgroups of so much LDS that a unit holds at once (it hands LDS out in 128 pieces of 1,280 bytes)
inline int held_by_lds(size_t bytes)
{
    const int fit = (int)(128 / ((bytes + 1279) / 1280));
    return fit < 1 ? 1 : fit;
}
// Time of `grid` equal workgroups, in units of one that has its unit to itself; `held`: how many a unit holds at once; `beside`: what each
// other one on the unit adds.  They start and end together, so that a round that is not full takes as long as if every unit had
// one more.
inline double rounds_of(int64_t grid, int cus, int held, double beside)
{
    const int64_t each = (grid + cus - 1) / cus, full = each / held, rest = each - full * held;
    return (double)full * (1.0 + beside * (held - 1)) + (rest > 0 ? 1.0 + beside * (double)(rest - 1) : 0.0);
}

// ---------------------------------------------------------------- stream mode, rows split across workgroups (sig_split_rows.h)
// stretches a path is cut into, 0 if the call stays with the other kernels
int split_rows_wanted(int d, int depth, int64_t B, int64_t L, int cus, int held_chunks, bool held_rows);
// The launch with `segs` stretches a path; false if there is none.  registers: the plan without it takes a register kernel (depth 2).
struct SplitRowsCut {
    int64_t lds_bytes, workgroups, scratch_floats;
    int threads;                  // of a workgroup
    int64_t segs, rows;           // stretches of a path in different workgroups, and their rows
    int64_t slices, lanes;        // workgroups of a stretch, and their words (depth 2: 1, and the slots of a workgroup)
    int64_t chunks, groups;       // depth 2: stretches side by side in a workgroup, of so many paths (1)
};
bool split_rows_geometry(int d, int depth, int64_t B, int64_t L, int segs, int cus, bool registers, SplitRowsCut *cut);
// scratch: those floats, or null (what lies before a stretch is folded again).  sticky: a point that is not a number spoils level 1 of the
// rows behind it, not of its own row only.
hipError_t launch_split_rows(const float *path, float *out, float *scratch, int64_t B, int64_t L, int d, int depth, int segs, bool sticky,
                             bool registers, int cus, hipStream_t st);

// ---------------------------------------------------------------- ... and at depth 2, where they need no scratch (sig_depth2_rows.hip)
// chunks: of the register kernel that the call would take, 0 if it would take another.  Workgroups a path, 0 if it stays with those.
// registers: that it would take one (its plan without split_rows), which decides between the cuts.
int depth2_rows_wanted(int d, int64_t B, int64_t L, int cus, int chunks);
bool depth2_rows_geometry(int d, int64_t B, int64_t L, int segs, int cus, bool registers, SplitRowsCut *cut);
hipError_t launch_depth2_rows(const float *path, float *out, int64_t B, int64_t L, int d, int segs, bool sticky, bool registers, int cus, hipStream_t st);

// table of compiled on-chip kernels; terminated by an entry with launch == nullptr
// The compiled kernels live in several translation units (so that they build in parallel); sub-table i ends
// with an entry whose launch pointer is null, and on_chip_subtable(i) is null past the last sub-table.  Entries
// of one (d, depth) are adjacent and ordered by increasing prefix depth.
const OnChipKernelInfo *on_chip_subtable(int i);
const OnChipKernelInfo *on_chip_table_base();      // sub-tables 0 .. 5, one translation unit each
const OnChipKernelInfo *on_chip_table_depth2();
const OnChipKernelInfo *on_chip_table_depth3();
const OnChipKernelInfo *on_chip_table_depth4();
const OnChipKernelInfo *on_chip_table_depth56();
const OnChipKernelInfo *on_chip_table_odd();
const OnChipKernelInfo *on_chip_table_wide();
const OnChipKernelInfo *find_on_chip(int d, int depth, int p);

}  // namespace sig
#endif
