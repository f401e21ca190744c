// Workspace plan of the SnapKV score (shared by its kernels and the C ABI).
#pragma once

#include <stddef.h>

namespace kve {

constexpr size_t kAlign = 256;
inline size_t align_up(size_t x) { return (x + kAlign - 1) / kAlign * kAlign; }

// ---------------------------------------------------------------------------
// SnapKV score: rows of one segment are the G*W window queries (head-major),
// taken in row groups (a segment and a row group form a vseg) of 128 rows, or
// of 256 for bf16 when the window has more than 128 rows: a wave then holds
// two sets of 32 rows, so that K is read once per pass for up to 256 rows.  Each
// vseg's keys are split into ranges of whole 64-key chunks, one workgroup each;
// pass 1 writes the statistics of each (vseg, range, row), a {reference, sum}
// pair or one log-sum-exp; a combine step, or pass 2 itself, reduces them to one
// log-sum-exp per row; pass 2 writes the column sums of each row group (a
// plane), and the pool step adds the planes and max-pools the prefix.
// ---------------------------------------------------------------------------
constexpr int kSnapRowsPerGroup = 128;
constexpr int kSnapMaxRows = 1024;
constexpr int kSnapChunkKeys = 64;
constexpr int kSnapTargetGroups = 4096;  // most workgroups per pass that the range size aims at
constexpr int kSnapMaxRangeChunks = 128;  // at most 8192 keys per range
constexpr int kSnapCus = 256;             // compute units the ranges are balanced over

// Fused role epilogue: per (segment, bucket), the number of candidate
// positions by the top kRoleHistBits bits of their order-preserving score key
// (the top-k's first radix digit), counted by the pool step.  The pool counts
// each tile of kRoleHistTile positions in a window of kRoleHistWindow bins from
// the tile's lowest bin, as 16-bit counts (a tile has fewer than 2^16
// positions); a tile record is a header of four words {lowest bin (all ones:
// no candidate), window overflowed (0/1), 0, 0} and R x kRoleHistWindow / 2
// words of count pairs.  The top-k adds the records of a segment's tiles, or
// counts the segment itself when a tile's bins did not fit its window.
constexpr int kRoleHistBits = 11;
constexpr int kRoleHistBins = 1 << kRoleHistBits;
constexpr int kRoleHistMaxR = 8;
constexpr int kRoleHistTile = 4096;
constexpr int kRoleHistWindow = 512;
constexpr int kRoleHistHeader = 4;

inline size_t role_hist_tile_words(int R) { return (size_t)kRoleHistHeader + (size_t)R * kRoleHistWindow / 2; }
inline int role_hist_tiles(int N) { return (N + kRoleHistTile - 1) / kRoleHistTile; }

// Bytes of the static device scratch array the allocation-free SnapKV entry
// point uses as its workspace (one copy per GPU, held until the process ends).
constexpr size_t kSnapScratchBytes = (size_t)64 << 20;

// Chunks per range.  A workgroup's start (its queries' fragments, the first
// chunk's latency) costs about four chunks of its time, and a pass ends when
// the fullest compute unit does: of the range sizes that give at most k
// workgroups per unit, k = 1 .. 16, the one with the least
//   rounds (chunks per range + 4),   rounds = ceil(workgroups / units)
// is taken.  Where rounds are few, less hides their latencies, and their chunks count more
// often: a single one 1.25 times (float32, whose chunks are split between
// barriers, and 64-element rows of 16 bits, whose chunks are half as long, 1.4:
// one float32 layer of 32768 keys takes 98 us at 16 chunks, one per unit, and 90
// at eight), two and three of such rows 1.11 and 1.07 times (8 layers x 8
// segments of 65536 keys: 243 us at k = 2, 236 at 3, 218 at 4).  With 16-bit
// rows in one set four workgroups share a unit: groups of four rounds follow
// each other, and a last group that is not full takes nearly a range's time
// more than its share (128 segments of 81344 keys, d = 128: 1009 us at five
// rounds, 928 at six, 918 at eight; 256 of 40000: 963 at five and 883 at eight;
// two sets and float32 show no such steps).  `least` is the range size that gives
// kSnapTargetGroups workgroups: shorter ranges never pay, and from
// kSnapMaxRangeChunks on it stands, the chip being full either way.
// Measured as a score call with `least` and with the rule (32 heads over 8,
// d = 128, bf16): 1 layer, N = 8192, W = 32: 24.8 -> 23.5 us; N = 32768: 60.7
// -> 43.6; N = 131072, W = 64: 240 -> 158; 4 layers, N = 20011: 104 -> 88;
// 8 layers x 2, N = 20011: 285 -> 252 us.
inline long long snap_range_chunks(long long chunks, long long vsegs, long long least, bool one_set16,
                                   bool split, int d) {
    const bool short_chunks = one_set16 && d == 64;
    const double few[4] = {1.0, split || short_chunks ? 1.4 : 1.25, short_chunks ? 1.11 : 1.0,
                           short_chunks ? 1.07 : 1.0};
    if (least >= kSnapMaxRangeChunks) return least;
    long long best = least;
    double cost = -1.0;
    for (int k = 1; k <= 16; ++k) {
        long long nr = (long long)kSnapCus * k / vsegs;
        if (nr < 1) continue;
        if (nr > chunks) nr = chunks;
        const long long per = (chunks + nr - 1) / nr;
        if (per < least) break;
        if (per > kSnapMaxRangeChunks) continue;
        const long long rounds = (vsegs * ((chunks + per - 1) / per) + kSnapCus - 1) / kSnapCus;
        const double factor = rounds < 4 ? few[rounds] : 1.0;
        const double tail = one_set16 && rounds > 4 && rounds % 4 != 0 ? 0.8 * (double)per : 0.0;
        const double c = (double)rounds * (factor * (double)per + 4.0) + tail;
        if (cost < 0.0 || c < cost) {
            cost = c;
            best = per;
        }
    }
    return best;
}

struct SnapPlan {
    int segs, rows, sets, rpg, rgroups, n_vsegs, range_keys, nranges, planes;
    int pair;  // a range's statistics are {reference, sum} pairs, not one log-sum-exp
    size_t off_stats, off_lse, off_raw, total;
};

// elem: bytes per element of the inputs (2 for bf16, 4 for fp32)
inline SnapPlan snap_plan(int L, int B, int Hq, int Hkv, int N, int W, int d, int elem) {
    SnapPlan p{};
    p.segs = L * B * Hkv;
    p.rows = (Hq / Hkv) * W;
    p.sets = (elem == 2 && p.rows > kSnapRowsPerGroup) ? 2 : 1;  // 32-row sets per wave
    p.rpg = p.sets * kSnapRowsPerGroup;                           // rows per row group
    p.rgroups = (p.rows + p.rpg - 1) / p.rpg;
    p.n_vsegs = p.segs * p.rgroups;
    p.planes = p.rgroups;
    // whole chunks per range: at least what gives kSnapTargetGroups workgroups
    // per pass and as many keys as the group has query rows (a workgroup loads
    // its rows' queries once, so its keys should outweigh them)
    const long long chunks = (N + kSnapChunkKeys - 1) / kSnapChunkKeys;
    long long per = (chunks * p.n_vsegs + kSnapTargetGroups - 1) / kSnapTargetGroups;
    const int group_rows = p.rows < p.rpg ? p.rows : p.rpg;
    const long long min_per = (group_rows + kSnapChunkKeys - 1) / kSnapChunkKeys;
    if (per < min_per) per = min_per;
    if (per > kSnapMaxRangeChunks) per = kSnapMaxRangeChunks;
    if (per > chunks) per = chunks;
    // the workspace holds the statistics of the smallest ranges: its size does
    // not depend on how the rule below balances them
    const size_t stats_ranges = (size_t)((chunks + per - 1) / per);
    per = snap_range_chunks(chunks, p.n_vsegs, per, elem == 2 && p.sets == 1, elem == 4, d);
    p.range_keys = (int)(per * kSnapChunkKeys);
    p.nranges = (int)((chunks + per - 1) / per);
    // longer ranges leave room for two floats each: the pair keeps the rounding
    // of a log-sum-exp (2^-20 at a magnitude of 8 to 16) out of the ranges'
    // merge, where over fewer ranges it averages out less
    p.pair = 2 * (size_t)p.nranges <= stats_ranges;
    size_t off = 0;
    p.off_stats = off;
    off = align_up(off + (size_t)p.n_vsegs * stats_ranges * p.rpg * sizeof(float));
    p.off_lse = off;
    off = align_up(off + (size_t)p.n_vsegs * p.rpg * sizeof(float));
    p.off_raw = off;
    off = align_up(off + (size_t)p.planes * p.segs * N * sizeof(float));
    p.total = off;
    return p;
}

}  // namespace kve
