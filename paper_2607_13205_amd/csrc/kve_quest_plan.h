// Plan of the Quest page step.  Plain C++.
#pragma once

#include <stddef.h>

#include "kve_snap_plan.h"

namespace kve {

// One-shot Quest analogue: a first step writes each head's mean window query
// (the workspace, [segs, G, d] float32); the page step cuts the prefix of a
// segment into pages and gives each workgroup a range of whole wave steps of
// pages: up to kQuestMaxSteps, fewer where that left under kQuestMinGroups
// workgroups.  A workgroup's start (the mean queries, the first pages' latency)
// is spread over its steps, and more steps than four only lengthen the tail:
// 1 layer of 131072 keys (8 KV heads, d = 128, bf16) takes 82 us at one step
// per workgroup, 55 at two, 50 at four and at eight; 4 x 2 x 24571 keys 79 at
// two, 71 at four, 73 at eight; 32 x 4 x 32768 keys 1394 at four, 1457 at 16.
// 1 layer of 8192 keys: 12.8 us at one or two, 15.4 at four (64 workgroups).
// Pages of fewer than 16 keys take as many keys per workgroup, up to 32 steps (4
// layers of 32768 keys, pages of one: 308 us at 63 steps, 264 at 32).
// Where a start weighs less, half the steps in more workgroups: with fewer than
// four heads per group (64 segments of 28834 keys, one head: 86 us at two steps,
// 90 at four), and with float32, whose step is half as many keys of the same
// bytes, up to pages of 32 (9 segments of 105344 keys: 80 us at two steps, 86 at
// four; pages of one, 256 segments of 5345, one head: 324 at 16, 362 at 64; pages
// of 64, 64 segments of 32768: 187 at two, 175 at four).  A step of 16-bit pages
// of 64 keys and more is 256 KB or more, and 2880 of them are enough workgroups
// (141 us at one step each, 154 at two).
constexpr int kQuestMinGroups = 1024;
constexpr int kQuestMaxSteps = 4;
constexpr int kQuestMostSteps = 32;  // of short pages
constexpr int kQuestMaxGroup = 8;  // query heads per KV head
constexpr int kQuestMaxPage = 1024;

struct QuestPlan {
    int segs, G, n_pages, range_pages, nranges;
    size_t total;
};

inline QuestPlan quest_plan(int L, int B, int Hq, int Hkv, int N, int W, int d, int elem, int page) {
    QuestPlan p{};
    p.segs = L * B * Hkv;
    p.G = Hq / Hkv;
    const int P = N - W;
    p.n_pages = (P + page - 1) / page;
    const int step = 4 * (64 / (d * elem / 16));  // pages per workgroup step: 4 waves
    const long long steps = (p.n_pages + step - 1) / step;
    const bool light = p.G < 4, f32 = elem == 4 && page < 32;
    const int half = light || f32 ? 2 : 1;
    const int groups = light || (elem == 2 && page >= 64) ? 2 * kQuestMinGroups : kQuestMinGroups * (f32 ? 3 : 2) / 2;
    long long per = (steps * p.segs + (f32 && !light ? groups / 2 : 0)) / groups;
    int most = page < 16 ? kQuestMaxSteps * 16 / page / (light ? 2 : 1) : kQuestMaxSteps / half;
    if (most > kQuestMostSteps / (light ? 2 : 1)) most = kQuestMostSteps / (light ? 2 : 1);
    if (per > most) per = most;
    if (per < 1) per = 1;
    p.range_pages = (int)(per * step);
    p.nranges = p.n_pages > 0 ? (int)((p.n_pages + p.range_pages - 1) / p.range_pages) : 1;
    p.total = align_up((size_t)p.segs * p.G * d * sizeof(float));
    return p;
}

}  // namespace kve
