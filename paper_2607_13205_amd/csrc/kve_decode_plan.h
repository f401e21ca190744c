// Plan of the decode over a compacted cache: how a segment's rows are cut into
// splits.  Plain C++.
#pragma once

#include <stddef.h>

#include "kve_snap_plan.h"

namespace kve {

// The k_cap rows of a segment are cut into splits of whole kDecodeQuantum-row
// quanta, one workgroup each; each writes per head the partial output o[d] and
// its (reference, denominator) pair, merged by a last step.  The workspace is
// sized for kDecodeSizeGroups workgroups.
constexpr int kDecodeQuantum = 128;
constexpr int kDecodeUnits = 256;  // compute units
constexpr int kDecodeSizeGroups = 1024;
constexpr int kDecodeMaxGroup = 8;  // query heads per KV head
constexpr int kDecodeLongest = 16;  // quanta per split from which more workgroups than one per unit pay
constexpr int kDecodeShort = 4;       // quanta of 128-element rows per split for which only latency counts,
constexpr int kDecodeShortWhole = 7;  // and of a segment in one split

struct DecodePlan {
    int segs, G, nsplit, split_keys;
    size_t off_o, off_ml, total;
};

// Quanta per split for about `ns` splits of a segment, and the splits of that size.
inline long long decode_sized(long long ns, long long quanta, long long* splits) {
    if (ns > quanta) ns = quanta;
    if (ns < 1) ns = 1;
    const long long per = (quanta + ns - 1) / ns;
    *splits = (quanta + per - 1) / per;
    return per;
}

// Quanta per split and splits per segment: about k workgroups per compute unit,
// the fewest k = 1 .. 4 that leaves no split longer than kDecodeLongest quanta
// and the last round of one workgroup per unit not emptier than 0.85 of all
// rounds allows.  On equal counts one per unit is best, since more splits only
// add starts and partials to merge (bf16, d = 128: 8 segments of 20000 rows take
// 19.6 us at k = 1 and 24 at 4, 32 of 1639 11.3 and 13.1, 128 of 1639 23 and 25;
// float32, 32 of 6000 36 and 40).  The counts of a batch differ, though, and are
// not known here: long splits leave the units that have none idle (one sample of
// four with 32768 rows, the others 655, 8 heads each: 47 us at k = 1, 35 at 2;
// one of sixteen: 162 us at k = 1, 66 at 4).  Equal counts lose 1 to 5% by it
// (256 segments of 6000 rows: 134 us at k = 1, 139 at 3).  Uneven rounds: 136
// segments of 1639 rows take 30.7 us at k = 1 and 25.9 at 4, 264 48.6 and 42.2
// at 3 (where no k fills the rounds, 3 is taken).
// Short splits are their latency however the rounds fill, and a merge is one
// more kernel: up to kDecodeShort quanta, or kDecodeShortWhole of a segment that
// is one split, k = 1 stands (bf16: 288 segments of 400 rows 16.4 us at k = 1
// and 20.9 at 3, 384 of 820 27.6 and 32.0); rows of 64 elements: twice that, and
// one split of up to twice kDecodeLongest (bf16, seven heads: 512 segments of
// 3277 rows 78 us whole and 86 in two, 384 of 820 20.0 and 25.7).  Longer ones of
// 64 elements lose more than those of 128 where counts are equal (bf16: 256 of
// 8192 88 us at k = 1, 101 at 4) and gain as much where they are not (every
// fourth long 55 and 41, one of 32 71 and 39).
inline long long decode_splits(long long segs, long long quanta, int d, long long* splits) {
    const int shorter = d == 64 ? 2 : 1;  // as many bytes in twice the rows
    long long per = 0;
    for (int k = 1; k <= 4; ++k) {
        per = decode_sized((k * kDecodeUnits + segs - 1) / segs, quanta, splits);
        const long long rounds = (segs * *splits + kDecodeUnits - 1) / kDecodeUnits;
        const bool brief = k == 1 && per <= shorter * (*splits == 1 ? kDecodeShortWhole : kDecodeShort);
        const bool even = brief || rounds == 1 || 20 * segs * *splits >= 17 * kDecodeUnits * rounds;
        if (per <= (*splits == 1 ? shorter : 1) * kDecodeLongest && even) return per;
    }
    for (int k = 3; k <= 4; ++k) {
        per = decode_sized((k * kDecodeUnits + segs - 1) / segs, quanta, splits);
        if (per <= kDecodeLongest && *splits > 1) break;
    }
    return per;
}

inline DecodePlan decode_plan(int L, int B, int Hq, int Hkv, int k_cap, int d) {
    DecodePlan p{};
    p.segs = L * B * Hkv;
    p.G = Hq / Hkv;
    const long long quanta = ((long long)k_cap + kDecodeQuantum - 1) / kDecodeQuantum;
    long long splits;
    decode_sized((kDecodeSizeGroups + p.segs - 1) / p.segs, quanta, &splits);
    const size_t parts = (size_t)p.segs * splits * p.G;
    p.split_keys = (int)(decode_splits(p.segs, quanta, d, &splits) * kDecodeQuantum);
    p.nsplit = (int)splits;
    p.off_o = 0;
    p.off_ml = align_up(parts * d * sizeof(float));
    p.total = p.off_ml + align_up(parts * 2 * sizeof(float));
    return p;
}

}  // namespace kve
