// Which kernels a top-k selection takes, by size.  Plain C++.
#pragma once

#include <stddef.h>

#include <algorithm>

#include "kve_snap_plan.h"

namespace kve {

// topk_regs: whole segments in registers, 16 keys per thread of 1024 at most (at
// 32 the keys spill; 1024 segments of 16384 keys take 62 us either way).
constexpr int kRegsMax = 16384;
// Many segments of more than kRegsShort keys and few buckets: topk_kernel's
// workgroups of four waves use the chip better than topk_regs' of sixteen, of
// which two share a compute unit and end together (2048 segments of 12000 keys,
// four buckets: 84 us and 112, 16384 keys 103 and 120; with eight buckets, whose
// histograms leave two workgroups per unit either way, 140 and 126; 768 segments
// of 12000, where topk_kernel does not fill the chip, 51 and 46).
constexpr int kRegsShort = 8192;
constexpr size_t kRegsSegs = 1024;
constexpr int kRegsFewBuckets = 4;

inline bool topk_in_regs(size_t segs, int N, int R) {
    return N <= kRegsShort || (N <= kRegsMax && !(segs >= kRegsSegs && R <= kRegsFewBuckets));
}

// Segments split into slices, one workgroup each (topk_count, topk_stage), up to
// kSplitSegs segments, where each still has four slices: 64 x 65536 keys take
// 48 us split and 60 whole, 64 x 131072 73 and 94.  In three or two slices the
// two further kernels take back what they give (one bucket, split and whole: 72
// x 20000 keys 30 and 27 us, x 131072 80 and 90; 96 x 65536 52 and 55, x 131072
// 104 and 91; 128 x 65536 54 and 55; 160, two queueing rounds, 71 and 56; 255
// 80 and 71).
constexpr size_t kSplitSegs = 64;
constexpr int kMaxSlices = 64;
// Workgroups of all segments up to one per compute unit, slices of at least
// kSliceLeast positions (a quarter of a workgroup's step; its record needs
// kSliceRecord R + kSliceMinPad), but short enough for 16-bit counts and
// offsets.  More slices queue for the chip, each with its histogram to clear and
// to add up: with as many as the records allow, 64 x 65536 keys took 143 us with
// one bucket (30 slices), 80 with two, 58 with four; now 44, 46 and 48.
constexpr int kSplitGroups = 256;
constexpr int kSliceLeast = 4096;
constexpr int kSliceMost = 65504;
constexpr int kSliceRecord = 1 << kRoleHistBits;
constexpr int kSliceMinPad = 128;

// Slices per segment; 0 where segments are not split.
inline int topk_slices(size_t segs, int N, int R) {
    if (segs > kSplitSegs || N > kMaxSlices * kSliceMost) return 0;
    int s = std::min(N / std::max(kSliceRecord * R + kSliceMinPad, kSliceLeast), kMaxSlices);
    s = std::min(s, std::max(2, kSplitGroups / (int)segs));
    s = std::max(s, (N + kSliceMost - 1) / kSliceMost);
    return s > 1 ? s : 0;
}

}  // namespace kve
