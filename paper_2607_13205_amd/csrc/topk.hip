// Per-role top-k selection (Algorithm 1, per-bucket top-k) with the window
// always kept, and the coalesced K/V compaction of the kept rows (§6: the
// dense cache of a compacting implementation).
//
// Scores are mapped to order-preserving 32-bit keys (-0 -> +0, NaN lowest), and
// each bucket's quota-th largest key is found digit by digit (11, 11 and 10
// bits) from LDS histograms.  Three forms, by size (launch_topk):
//   topk_regs    a segment (layer, sample, KV head) of up to 16384 keys (8192
//                when there are many segments and few buckets): one
//                workgroup with the whole segment in registers.
//   topk_count, topk_stage, topk_finish
//                up to 64 longer segments, each split over several workgroups.
//   topk_kernel  many longer ones, or scores with fused histograms: one
//                workgroup per segment, of 4 waves, or of 16 when there are too
//                few segments to fill the chip with 4-wave ones; two sweeps over
//                the segment's scores and labels:
//   1. Histogram sweep: the top 11 bits of every labelled candidate's key (sign,
//      exponent and two mantissa bits), one LDS histogram per bucket.  Per
//      bucket this gives the population, which decides whether the bucket is
//      kept whole, skipped or selected, and the top digit of the quota-th
//      largest key: the threshold's bin.
//   2. Staging sweep: each wave walks a contiguous share of the positions in
//      order and sets aside, in order, every position that is surely kept (the
//      window, whole buckets, keys above the threshold's bin) and every key
//      inside the bin (with its bucket and the low 21 bits of its key), in its
//      own part of the segment's workspace row (a position is staged at most
//      once, so a wave's part never overflows).
//   Two more digit passes over the staged keys of the bins fix each bucket's
//   threshold key and how many keys equal to it stay; each wave then walks its
//   staged entries twice: it counts what it keeps (keys equal to a threshold
//   are kept lowest position first, so the earlier waves' counts come first),
//   then writes the kept positions in ascending order.
// A lane takes up to 16 consecutive positions at a time, in 16-byte score loads
// and 4-byte label words at whatever alignment the rows have (a row of odd
// length used to be read position by position: 1024 segments of 40007 keys
// took 262 us, now 99).  Bucket state is looked up per key in small LDS tables
// rather than picked from registers with a chain of selects.
#include <stdint.h>

#include <algorithm>

#include "kve_device.h"
#include "kve_internal.h"
#include "kve_topk_plan.h"

namespace kve {
namespace {

constexpr int kThreads = 256;        // top-k workgroup when segments fill the chip (and compaction)
constexpr int kWideThreads = 1024;   // top-k workgroup when there are few segments
constexpr int kWideBelow = 512;      // segments below which the wide workgroup is used
constexpr int kDigitBits = kRoleHistBits;  // the first digit is the fused score epilogue's histogram bin
constexpr int kDigits = 1 << kDigitBits;
constexpr int kLowBits = 32 - kDigitBits;  // key bits below the top digit
constexpr uint32_t kLowMask = (1u << kLowBits) - 1u;
constexpr int kSpan = 16;                  // consecutive positions per lane and step
constexpr int kWaveStep = kWave * kSpan;   // positions per wave step
constexpr int kBatch = 8;                  // staged entries per lane loaded before use
constexpr uint32_t kNoKey = 0xffffffffu;   // above every key (+inf maps to 0xff800000)
constexpr uint32_t kKept = 0xffffffffu;    // tag of a staged position that is surely kept

enum : int { kModeNone = 0, kModeSelect = 1, kModeAll = 2 };

// inclusive prefix sum over the lanes of a wave, on the vector unit's lane shifts
__device__ __forceinline__ int wave_scan(int v) {
    v += __builtin_amdgcn_update_dpp(0, v, 0x111, 0xf, 0xf, true);   // row_shr:1
    v += __builtin_amdgcn_update_dpp(0, v, 0x112, 0xf, 0xf, true);   // row_shr:2
    v += __builtin_amdgcn_update_dpp(0, v, 0x114, 0xf, 0xf, true);   // row_shr:4
    v += __builtin_amdgcn_update_dpp(0, v, 0x118, 0xf, 0xf, true);   // row_shr:8
    v += __builtin_amdgcn_update_dpp(0, v, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1 and 3
    v += __builtin_amdgcn_update_dpp(0, v, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2 and 3
    return v;
}

// What is known of a bucket's threshold.  While mode is kModeSelect: the top
// 32 - lo bits `pref` of the quota-th largest key, and how many of the keys
// that share them are kept.  At the end keys >= keep_from are kept, and of the
// keys equal to `tie` the first `need` by position (tie = kNoKey: none).
// match: pref while digits are missing, else kNoKey.
struct Bucket {
    int mode, lo, need;
    uint32_t pref, keep_from, tie, match;
};

// One wave: the next digit of a bucket from its histogram (bins from the top; 32
// bins per lane and two lane scans, no workgroup barrier inside),
// which is cleared for the next pass.  first: the first digit, whose
// population decides with the quota q whether the bucket is kept whole,
// skipped or selected.
__device__ __forceinline__ void find_digit(Bucket& b, uint32_t* hist, bool first, int q) {
    const int lane = threadIdx.x & 63;
    const int mode = b.mode, lo0 = b.lo;
    uint4* h4 = reinterpret_cast<uint4*>(hist);
    if (mode == kModeSelect && lo0 > 0) {  // uniform
        const int p0 = (kDigits - 32 * (lane + 1)) / 4;  // this lane's 32 bins as eight 16-byte pieces
        int sum = 0;
#pragma unroll
        for (int i = 0; i < 8; ++i) {  // each lane starts at another piece: fewer bank conflicts
            const uint4 x = h4[p0 + ((i + lane) & 7)];
            sum += (int)(x.x + x.y + x.z + x.w);
        }
        const int incl = wave_scan(sum);
        const int total = __builtin_amdgcn_readlane(incl, kWave - 1);
        int want = b.need;
        bool done = false;
        if (first) {
            want = max(q, 0);
            if (want == 0 || want >= total) {
                done = true;
                if (lane == 0) {
                    b.mode = want == 0 ? kModeNone : kModeAll;
                    b.keep_from = want == 0 ? kNoKey : 0u;
                    b.tie = kNoKey;
                }
            }
        }
        if (!done) {  // uniform
            const int L = __builtin_ctzll(__ballot(incl >= want));
            const int above = __builtin_amdgcn_readlane(incl - sum, L);
            const int bin = kDigits - 32 * L - 1 - (lane & 31);
            const int h = lane < 32 ? (int)hist[bin] : 0;
            const int in2 = wave_scan(h);
            const int L2 = __builtin_ctzll(__ballot(above + in2 >= want));
            if (lane == L2) {
                const int w = min(kDigitBits, lo0);
                const int lo = lo0 - w, need = want - (above + in2 - h);
                const uint32_t pref = (lo0 < 32 ? b.pref << w : 0u) | (uint32_t)bin;
                const bool whole = need == h;  // every key that shares the digits stays
                b.pref = pref;
                b.need = need;
                b.lo = whole ? 0 : lo;
                b.keep_from = whole ? pref << lo : (lo == 0 ? pref + 1u : kNoKey);
                b.tie = !whole && lo == 0 ? pref : kNoKey;
                b.match = !whole && lo > 0 ? pref : kNoKey;
            }
        }
    }
#pragma unroll
    for (int i = 0; i < kDigits / 4 / kWave; ++i) h4[i * kWave + lane] = make_uint4(0u, 0u, 0u, 0u);
}

// Scores and labels of SPAN consecutive positions from t0, inside a row of N
// (SPAN a multiple of 4): 16-byte score loads at any 4-byte address, label
// words at any address (both allowed by the hardware for global memory).
// Spans that reach past the row end: one load per position, clamped.
typedef uint32_t u32x4_a4 __attribute__((ext_vector_type(4), aligned(4)));
typedef uint32_t u32_a1 __attribute__((aligned(1)));
template <int SPAN>
__device__ __forceinline__ void load_span_any(const float* sc, const int8_t* ro, int t0, int N, float (&s)[SPAN],
                                              uint32_t (&lab)[SPAN / 4]) {
    if (t0 + SPAN <= N) {
#pragma unroll
        for (int j = 0; j < SPAN / 4; ++j) {
            const u32x4_a4 v = *reinterpret_cast<const u32x4_a4*>(sc + t0 + 4 * j);
#pragma unroll
            for (int i = 0; i < 4; ++i) s[4 * j + i] = __uint_as_float(v[i]);
            lab[j] = *reinterpret_cast<const u32_a1*>(ro + t0 + 4 * j);
        }
    } else {
#pragma unroll
        for (int j = 0; j < SPAN / 4; ++j) {
            uint32_t w = 0u;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                const int t = min(t0 + 4 * j + i, N - 1);
                s[4 * j + i] = sc[t];
                w |= (uint32_t)(uint8_t)ro[t] << (8 * i);
            }
            lab[j] = w;
        }
    }
}

// Counts of a thread's keys: runs of equal (bucket, bin), the max-pool's
// plateaus, go in with one LDS atomic.  bin_of(e): the histogram word of key
// e, kNoKey for none; taken eight keys at a time before any atomic, whose
// order the compiler keeps against the tables bin_of reads.
template <int SPAN, typename F>
__device__ __forceinline__ void count_runs(uint32_t* hist, F&& bin_of) {
    constexpr int G = SPAN < 8 ? SPAN : 8;
    static_assert(SPAN % G == 0, "whole groups");
    uint32_t cur = kNoKey, cnt = 0u;
#pragma unroll
    for (int g = 0; g < SPAN; g += G) {
        uint32_t w[G];
#pragma unroll
        for (int e = 0; e < G; ++e) w[e] = bin_of(g + e);
#pragma unroll
        for (int e = 0; e < G; ++e) {
            if (w[e] != cur) {
                if (cur != kNoKey) atomicAdd(&hist[cur], cnt);
                cur = w[e];
                cnt = 0u;
            }
            ++cnt;
        }
    }
    if (cur != kNoKey) atomicAdd(&hist[cur], cnt);
}

// Exclusive prefix sum over the lanes of a wave of v in [0, 31] (lane order),
// and the wave's total: one ballot per bit.
__device__ __forceinline__ int wave_exclusive_scan(int v, int& total) {
    int excl = 0;
    total = 0;
#pragma unroll
    for (int bit = 0; bit < 5; ++bit) {
        const uint64_t m = __ballot((v >> bit) & 1);
        excl += (int)__builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u))
                << bit;
        total += __popcll(m) << bit;
    }
    return excl;
}

// The second or third digit (pass 1 or 2: w bits below bit lo) of a staged
// undecided key, whose tag is its bucket and its low bits.  Every such key
// shares its bucket's first digit, so the second digits are counted without a
// look at the tables, which would put its latency between the atomics (1024 x
// 32768 keys 84.4 -> 83.2 us, 1024 x 40007 101.5 -> 99.2; topk_finish, whose
// entries are in registers, gained nothing).
template <int R>
__device__ __forceinline__ void count_digit(uint32_t* hist, const Bucket* bk, uint32_t tag, int pass, int lo, int w) {
    const uint32_t r = tag >> kLowBits, low = tag & kLowMask;
    if (pass == 1) {
        atomicAdd(&hist[r * kDigits + (low >> (lo - w))], 1u);
    } else {
        const uint32_t m = bk[r].match;
        if (m != kNoKey && (low >> lo) == (m & ((1u << kDigitBits) - 1u)))
            atomicAdd(&hist[r * kDigits + (low & ((1u << w) - 1u))], 1u);
    }
}

// bucket of the label of position t0 + e; R for labels outside [0, R)
template <int R>
__device__ __forceinline__ uint32_t bucket_of(const uint32_t (&lab)[4], int e) {
    return min((lab[e >> 2] >> (8 * (e & 3))) & 0xffu, (uint32_t)R);
}

template <int R, int NT>
__global__ __launch_bounds__(NT) void topk_kernel(const float* __restrict__ score, const int8_t* __restrict__ roles,
                                                  const int32_t* __restrict__ quota,
                                                  const uint32_t* __restrict__ hist_in, int B, int Hkv, int N,
                                                  int W, int k_cap, int32_t* __restrict__ idx_out,
                                                  int32_t* __restrict__ count_out, uint2* __restrict__ stage) {
    constexpr int NW = NT / kWave;
    constexpr int kGroupStep = NT * kSpan;  // positions per workgroup step
    __shared__ __align__(16) uint32_t hist[R * kDigits];
    __shared__ Bucket bk[R];
    // staging: {lowest surely kept key, top digit of the threshold's bin} per
    // bucket; entry R (labels outside [0, R)) is never kept and never staged
    __shared__ uint2 cls[R + 1];
    __shared__ int over;            // a fused-histogram tile of this segment overflowed its window
    __shared__ int wave_eq[NW][R];  // staged keys equal to a threshold, per wave
    __shared__ int wave_keep[NW];   // kept positions per wave
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x;
    const int b = (seg / Hkv) % B;
    const float* sc = score + (size_t)seg * N;
    const int8_t* ro = roles + (size_t)b * N;
    const int P = N - W;

    if (tid < R) bk[tid] = Bucket{kModeSelect, 32, 0, 0u, kNoKey, kNoKey, kNoKey};  // decided after the first histogram
    for (int e = tid; e < R * kDigits / 4; e += NT) reinterpret_cast<uint4*>(hist)[e] = make_uint4(0u, 0u, 0u, 0u);
    // 1. the first digit's counts: added up from the fused score epilogue's tile
    //    records when every tile fitted its window, otherwise counted in a sweep
    bool sweep = true;
    if (hist_in != nullptr) {
        const int tiles = (N + kRoleHistTile - 1) / kRoleHistTile;
        constexpr int kTw = kRoleHistHeader + R * kRoleHistWindow / 2;  // words per tile record
        const uint32_t* rec = hist_in + (size_t)seg * tiles * kTw;
        if (tid == 0) over = 0;
        __syncthreads();
        for (int t = tid; t < tiles; t += NT)
            if (rec[(size_t)t * kTw + 1] != 0u) over = 1;
        __syncthreads();  // also orders the zero fill before the adds
        sweep = over != 0;  // uniform
        if (!sweep) {
            constexpr int kQ = R * kRoleHistWindow / 8;  // 16-byte words of count pairs per record
            for (int e = tid; e < tiles * kQ; e += NT) {
                const int t = e / kQ, q = e - t * kQ;
                const uint32_t* r0 = rec + (size_t)t * kTw;
                const uint32_t lo = r0[0];
                const u32x4 c = reinterpret_cast<const u32x4*>(r0 + kRoleHistHeader)[q];
                const int r = (4 * q) / (kRoleHistWindow / 2);
                const uint32_t bin0 = lo + 2u * (uint32_t)(4 * q - r * (kRoleHistWindow / 2));
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    const uint32_t w = c[i], b = bin0 + 2u * i;
                    if ((w & 0xffffu) != 0u && b < (uint32_t)kDigits) atomicAdd(&hist[r * kDigits + b], w & 0xffffu);
                    if ((w >> 16) != 0u && b + 1u < (uint32_t)kDigits) atomicAdd(&hist[r * kDigits + b + 1], w >> 16);
                }
            }
        }
    }
    __syncthreads();
    if (sweep) {
        // the top digit of every labelled candidate's key; each step's span is in
        // flight while the previous one is counted
        float s[kSpan] = {}, sn[kSpan] = {};
        uint32_t lab[4] = {}, labn[4] = {};
        int t0 = kSpan * tid;
        if (t0 < P) load_span_any<kSpan>(sc, ro, t0, N, s, lab);
        for (int base = 0; base < P; base += kGroupStep) {
            const int tn = t0 + kGroupStep;
            if (tn < P) load_span_any<kSpan>(sc, ro, tn, N, sn, labn);
            if (t0 < P) {
                const int nv = min(kSpan, P - t0);
                count_runs<kSpan>(hist, [&](int e) {
                    const uint32_t r = bucket_of<R>(lab, e);
                    return e < nv && r < (uint32_t)R ? r * kDigits + (score_key(s[e]) >> kLowBits) : kNoKey;
                });
            }
#pragma unroll
            for (int e = 0; e < kSpan; ++e) s[e] = sn[e];
#pragma unroll
            for (int j = 0; j < 4; ++j) lab[j] = labn[j];
            t0 = tn;
        }
    }
    __syncthreads();
    for (int r = wave; r < R; r += NW) find_digit(bk[r], hist + r * kDigits, true, quota[(size_t)b * R + r]);
    __syncthreads();
    if (tid <= R) {
        uint2 c = make_uint2(kNoKey, kNoKey);
        if (tid < R) {
            c.x = bk[tid].keep_from;
            // top digits are at most +inf's 0x7fc, so the shift does not overflow
            if (bk[tid].match != kNoKey) c = make_uint2((bk[tid].pref + 1u) << kLowBits, bk[tid].pref);
        }
        cls[tid] = c;
    }
    __syncthreads();

    // 2. staging sweep over this wave's run [w0, w1), in order
    const int run = (N + NW * kWaveStep - 1) / (NW * kWaveStep) * kWaveStep;
    const int w0 = min(N, wave * run), w1 = min(N, w0 + run);
    uint2* st = stage + (size_t)seg * N + w0;  // room for w1 - w0 entries
    int n_st = 0;
    {
        // each step's span is in flight while the previous one is staged; lanes
        // past the run load nothing and stage nothing
        float s[kSpan] = {}, sn[kSpan] = {};
        uint32_t lab[4] = {}, labn[4] = {};
        int t0 = w0 + kSpan * lane;
        if (t0 < w1) load_span_any<kSpan>(sc, ro, t0, N, s, lab);
        for (int s0 = w0; s0 < w1; s0 += kWaveStep) {
            const int tn = t0 + kWaveStep;
            if (tn < w1) load_span_any<kSpan>(sc, ro, tn, N, sn, labn);
            const int nv = max(0, min(kSpan, w1 - t0));
            uint32_t smask = 0u, tag[kSpan];
#pragma unroll
            for (int e = 0; e < kSpan; ++e) {
                const int t = t0 + e;
                const uint32_t key = score_key(s[e]);
                const uint32_t r = t < P ? bucket_of<R>(lab, e) : (uint32_t)R;
                const uint2 c = cls[r];
                const bool keep = t >= P || key >= c.x;
                const bool cand = (key >> kLowBits) == c.y;
                tag[e] = keep ? kKept : ((r << kLowBits) | (key & kLowMask));
                smask |= (e < nv && (keep || cand)) ? (1u << e) : 0u;
            }
            int tot;
            uint2* dst = st + n_st + wave_exclusive_scan(__popc(smask), tot);
#pragma unroll
            for (int e = 0; e < kSpan; ++e)
                if ((smask >> e) & 1u) *dst++ = make_uint2((uint32_t)(t0 + e), tag[e]);
            n_st += tot;
#pragma unroll
            for (int e = 0; e < kSpan; ++e) s[e] = sn[e];
#pragma unroll
            for (int j = 0; j < 4; ++j) lab[j] = labn[j];
            t0 = tn;
        }
    }
    __syncthreads();

    // the staged entries of this wave, kBatch per lane loaded before any is used;
    // visit(position, tag) for every entry in order, (0, kKept) with valid =
    // false past the end (every lane takes part in every step)
    auto sweep_staged = [&](auto&& visit) {
        for (int i0 = 0; i0 < n_st; i0 += kWave * kBatch) {
            uint2 ent[kBatch];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) ent[j] = st[min(i0 + j * kWave + lane, n_st - 1)];
#pragma unroll
            for (int j = 0; j < kBatch; ++j) visit(ent[j].x, ent[j].y, i0 + j * kWave + lane < n_st);
        }
    };
    // full key of a staged key of a threshold bin
    auto bin_key = [&](uint32_t tg, uint32_t& r) {
        r = tg >> kLowBits;
        return (cls[r].y << kLowBits) | (tg & kLowMask);
    };

    // 3. the remaining digits (11 and 10 bits) over the staged keys of the bins
    for (int pass = 1; pass < 3; ++pass) {
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= bk[r].match != kNoKey;
        if (!any) break;  // uniform: every thread reads the same LDS values
        const int lo = 32 - kDigitBits * pass;  // the same for every selecting bucket
        const int w = min(kDigitBits, lo);
        sweep_staged([&](uint32_t, uint32_t tg, bool valid) {
            if (valid && tg != kKept) count_digit<R>(hist, bk, tg, pass, lo, w);
        });
        __syncthreads();
        for (int r = wave; r < R; r += NW) find_digit(bk[r], hist + r * kDigits, false, 0);
        __syncthreads();
    }

    // 4. ordered output.  Class of a staged entry: 1 kept, 2 + r equal to bucket
    //    r's threshold (of which some stay), 0 dropped.
    int need[R];
#pragma unroll
    for (int r = 0; r < R; ++r) need[r] = bk[r].need;
    auto classify = [&](uint32_t tg, bool valid) {
        if (!valid) return 0;
        if (tg == kKept) return 1;
        uint32_t r;
        const uint32_t key = bin_key(tg, r);
        return key >= bk[r].keep_from ? 1 : (key == bk[r].tie ? 2 + (int)r : 0);
    };
    const uint64_t lt = (1ull << lane) - 1ull;
    int keep = 0, eq[R];
#pragma unroll
    for (int r = 0; r < R; ++r) eq[r] = 0;
    sweep_staged([&](uint32_t, uint32_t tg, bool valid) {
        const int c = classify(tg, valid);
        keep += c == 1;
#pragma unroll
        for (int r = 0; r < R; ++r) eq[r] += c == 2 + r;
    });
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        keep += __shfl_xor(keep, off);
#pragma unroll
        for (int r = 0; r < R; ++r) eq[r] += __shfl_xor(eq[r], off);
    }
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) wave_eq[wave][r] = eq[r];
    }
    __syncthreads();
    // equal keys are kept lowest position first: the earlier waves' come first
    int eq_seen[R];
#pragma unroll
    for (int r = 0; r < R; ++r) {
        eq_seen[r] = 0;
        for (int w = 0; w < wave; ++w) eq_seen[r] += wave_eq[w][r];
        keep += max(0, min(eq[r], need[r] - eq_seen[r]));
    }
    if (lane == 0) wave_keep[wave] = keep;
    __syncthreads();
    int pos = 0, total = 0;
    for (int w = 0; w < NW; ++w) {
        if (w < wave) pos += wave_keep[w];
        total += wave_keep[w];
    }
    sweep_staged([&](uint32_t t, uint32_t tg, bool valid) {
        const int c = classify(tg, valid);
        bool k = c == 1;
        if (__ballot(c >= 2) != 0ull) {  // rare: keys equal to a threshold in this step
#pragma unroll
            for (int r = 0; r < R; ++r) {
                const uint64_t m = __ballot(c == 2 + r);
                if (c == 2 + r) k = eq_seen[r] + (int)__popcll(m & lt) < need[r];
                eq_seen[r] += (int)__popcll(m);
            }
        }
        const uint64_t km = __ballot(k);
        const int at = pos + __popcll(km & lt);
        if (k && at < k_cap) idx_out[(size_t)seg * k_cap + at] = (int32_t)t;
        pos += __popcll(km);
    });
    if (tid == 0 && count_out != nullptr) count_out[seg] = total;
}

// ---------------------------------------------------------------------------
// Whole segments in registers, and segments split over workgroups
//
// A short or lonely segment's time is a chain of latencies, not bytes: with one
// topk_kernel workgroup each, 8 segments of 8192 keys took 27 us (0.3 MB of
// scores) and 8 of 100003 keys 175 us, eight workgroups on 256 compute units.
//   topk_regs    one workgroup per segment, each thread's SPAN consecutive keys
//                in registers through all digit passes and the output; nothing
//                is staged in memory.  1 x 512 keys: 23.3 -> 9.4 us, 8 x 8192:
//                26.7 -> 11.1 us, 8 x 16384: 31.4 -> 15.4 us.
//   topk_count, topk_stage, topk_finish
//                a segment in S slices: one workgroup per slice counts the first
//                digit, then (with the slices' counts added up, the same in
//                every workgroup) stages the slice's kept and undecided keys in
//                order; one workgroup per segment finds the other digits over
//                the staged keys and writes the output.  8 x 100003: 175 -> 40
//                us, 8 x 131072: 90 -> 44 us, 64 x 40001: 86 -> 35 us (four
//                buckets).
// ---------------------------------------------------------------------------

// exclusive prefix sum of one value per thread over a workgroup of NW waves;
// tmp: two rows of NW ints, used in turn (`turn`), so that one barrier suffices
template <int NW>
__device__ __forceinline__ int block_scan(int v, int& total, int (*tmp)[NW], int& turn) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int incl = wave_scan(v);
    int* t = tmp[turn & 1];
    ++turn;
    if (lane == kWave - 1) t[wave] = incl;
    __syncthreads();
    int before = 0;
    total = 0;
#pragma unroll
    for (int w = 0; w < NW; ++w) {
        const int x = t[w];
        before += w < wave ? x : 0;
        total += x;
    }
    return before + incl - v;
}

template <int R, int NT, int SPAN>
__global__ __launch_bounds__(NT) void topk_regs(const float* __restrict__ score, const int8_t* __restrict__ roles,
                                                const int32_t* __restrict__ quota, int B, int Hkv, int N, int W,
                                                int k_cap, int32_t* __restrict__ idx_out,
                                                int32_t* __restrict__ count_out) {
    constexpr int NW = NT / kWave;
    __shared__ __align__(16) uint32_t hist[R * kDigits];
    __shared__ Bucket bk[R + 1];  // entry R: no bucket, never kept
    __shared__ int tmp[2][NW];
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x;
    const int b = (seg / Hkv) % B;
    const int P = N - W;
    const int t0 = tid * SPAN;

    float s[SPAN];
    uint32_t lab[SPAN / 4];
    if (t0 < N) load_span_any<SPAN>(score + (size_t)seg * N, roles + (size_t)b * N, t0, N, s, lab);
    int q[(R + NW - 1) / NW];  // quotas of the buckets this wave searches
#pragma unroll
    for (int i = 0; i < (R + NW - 1) / NW; ++i) {
        const int r = wave + i * NW;
        q[i] = r < R ? quota[(size_t)b * R + r] : 0;
    }
    for (int e = tid; e < R * kDigits / 4; e += NT) reinterpret_cast<uint4*>(hist)[e] = make_uint4(0u, 0u, 0u, 0u);
    if (tid <= R) bk[tid] = Bucket{tid < R ? kModeSelect : kModeNone, 32, 0, 0u, kNoKey, kNoKey, kNoKey};
    uint32_t key[SPAN];
    uint32_t bkt[SPAN / 4];  // bucket of each key, a byte each; R: not a candidate
#pragma unroll
    for (int j = 0; j < SPAN / 4; ++j) {
        bkt[j] = 0u;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            key[4 * j + i] = score_key(s[4 * j + i]);
            const uint32_t r = t0 + 4 * j + i < P ? min((lab[j] >> (8 * i)) & 0xffu, (uint32_t)R) : (uint32_t)R;
            bkt[j] |= r << (8 * i);
        }
    }
    auto bucket = [&](int e) { return (bkt[e >> 2] >> (8 * (e & 3))) & 0xffu; };
    __syncthreads();
    count_runs<SPAN>(hist, [&](int e) {
        const uint32_t r = bucket(e);
        return r < (uint32_t)R ? r * kDigits + (key[e] >> kLowBits) : kNoKey;
    });
    for (int pass = 0; pass < 3; ++pass) {
        __syncthreads();
#pragma unroll
        for (int i = 0; i < (R + NW - 1) / NW; ++i) {
            const int r = wave + i * NW;
            if (r < R) find_digit(bk[r], hist + r * kDigits, pass == 0, q[i]);
        }
        __syncthreads();
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= bk[r].match != kNoKey;
        if (!any) break;  // uniform
        // bits below the digits known, and of the next digit (pass 0: 21 and 11, pass 1: 10 and 10)
        const int lo = pass == 0 ? kLowBits : kLowBits - kDigitBits;
        const int w = min(kDigitBits, lo);
        count_runs<SPAN>(hist, [&](int e) {
            const uint32_t r = bucket(e);
            return (key[e] >> lo) == bk[r].match ? r * kDigits + ((key[e] >> (lo - w)) & ((1u << w) - 1u)) : kNoKey;
        });
    }
    uint32_t keep = 0u;
#pragma unroll
    for (int e = 0; e < SPAN; ++e) {
        const int t = t0 + e;
        if (t < N && (t >= P || key[e] >= bk[bucket(e)].keep_from)) keep |= 1u << e;
    }
    int turn = 0, total;
    // equal keys of which only some stay: lowest position first
    for (int r = 0; r < R; ++r) {
        const uint32_t tie = bk[r].tie;
        if (tie == kNoKey) continue;  // uniform
        uint32_t eq = 0u;
#pragma unroll
        for (int e = 0; e < SPAN; ++e)
            if (bucket(e) == (uint32_t)r && key[e] == tie) eq |= 1u << e;
        int left = bk[r].need - block_scan<NW>(__popc(eq), total, tmp, turn);
        for (; eq != 0u && left > 0; --left, eq &= eq - 1u) keep |= eq & (0u - eq);
    }
    int at = block_scan<NW>(__popc(keep), total, tmp, turn);
    int32_t* dst = idx_out + (size_t)seg * k_cap;
    for (; keep != 0u && at < k_cap; ++at, keep &= keep - 1u) dst[at] = t0 + __builtin_ctz(keep);
    if (tid == 0 && count_out != nullptr) count_out[seg] = total;
}

// Segments split into S slices.  Workspace of a slice of `len` positions, 8
// bytes each: tags [len] uint32, offsets [len] uint16, then from the next
// multiple of 16 bytes the record: first-digit counts [R][kDigits] uint16 and
// kSliceWords words of state.  len >= kDigits R + kSliceMinPad.
constexpr int kSplitThreads = 1024;
constexpr int kSplitSpan = 16;
constexpr int kSplitStep = kSplitThreads * kSplitSpan;
// staged keys per lane of topk_finish held in registers; with one bucket 32 of
// them spill (69 registers; 64 x 40001 keys 35.7 us, 31.5 with 16)
template <int R>
constexpr int kHoldOf = R == 1 ? 16 : 32;
constexpr int kSliceWords = 4 + 3 * kRoleHistMaxR;  // lowest bin, bins' end, staged keys, -, buckets of the segment
static_assert(2 * kSliceMinPad >= 16 + 4 * kSliceWords + 32, "a record fits the slice's spare bytes");

// first position of slice s of S (a multiple of 16; N for s = S); N < 2^22 + 2^16, S <= kMaxSlices
__device__ __forceinline__ int slice_begin(int s, int S, int N) {
    return s == S ? N : (int)((unsigned)(N / 16) * (unsigned)s / (unsigned)S) * 16;
}
struct Slice {
    int begin, len;
    uint32_t* tags;
    uint16_t* offs;
    uint32_t* counts;  // pairs of 16-bit counts
    uint32_t* state;
};
template <int R>
__device__ __forceinline__ Slice slice_of(char* ws, int seg, int s, int S, int N) {
    Slice x;
    x.begin = slice_begin(s, S, N);
    x.len = slice_begin(s + 1, S, N) - x.begin;
    char* base = ws + ((size_t)seg * N + x.begin) * 8;
    x.tags = reinterpret_cast<uint32_t*>(base);
    x.offs = reinterpret_cast<uint16_t*>(base + (size_t)x.len * 4);
    char* rec = base + (size_t)x.len * 6;
    rec += (0 - reinterpret_cast<uintptr_t>(rec)) & 15u;
    x.counts = reinterpret_cast<uint32_t*>(rec);
    x.state = x.counts + R * kDigits / 2;
    return x;
}

template <int R>
__global__ __launch_bounds__(kSplitThreads) void topk_count(const float* __restrict__ score,
                                                            const int8_t* __restrict__ roles, int B, int Hkv, int N,
                                                            int W, int S, char* __restrict__ ws) {
    __shared__ __align__(16) uint32_t hist[R * kDigits];
    __shared__ uint32_t range[2];
    const int tid = threadIdx.x;
    const int seg = blockIdx.x / S;
    const Slice sl = slice_of<R>(ws, seg, blockIdx.x - seg * S, S, N);
    const int b = (seg / Hkv) % B;
    const int P = N - W, end = sl.begin + sl.len;
    for (int e = tid; e < R * kDigits / 4; e += kSplitThreads)
        reinterpret_cast<uint4*>(hist)[e] = make_uint4(0u, 0u, 0u, 0u);
    if (tid == 0) {
        range[0] = kDigits;
        range[1] = 0u;
    }
    __syncthreads();
    uint32_t lo = kDigits, hi = 0u;
    for (int base = sl.begin; base < end; base += kSplitStep) {
        const int t0 = base + tid * kSplitSpan;
        if (t0 < end) {
            float s[kSplitSpan];
            uint32_t lab[kSplitSpan / 4];
            load_span_any<kSplitSpan>(score + (size_t)seg * N, roles + (size_t)b * N, t0, N, s, lab);
            const int nv = min(end, P) - t0;
            count_runs<kSplitSpan>(hist, [&](int e) {
                const uint32_t r = bucket_of<R>(lab, e);
                if (e >= nv || r >= (uint32_t)R) return kNoKey;
                const uint32_t bin = score_key(s[e]) >> kLowBits;
                lo = min(lo, bin);
                hi = max(hi, bin + 1u);
                return r * kDigits + bin;
            });
        }
    }
#pragma unroll
    for (int off = 1; off < kWave; off <<= 1) {
        lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
        hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
    }
    if ((tid & 63) == 0) {
        atomicMin(&range[0], lo);
        atomicMax(&range[1], hi);
    }
    __syncthreads();
    // counts of the occupied bins as pairs (a slice has fewer than 2^16 positions)
    const int p0 = (int)range[0] / 2, np = max(0, ((int)range[1] + 1) / 2 - p0);
    for (int e = tid; e < R * np; e += kSplitThreads) {
        const int w = (e / np) * (kDigits / 2) + p0 + e % np;
        sl.counts[w] = hist[2 * w] | (hist[2 * w + 1] << 16);
    }
    if (tid < 2) sl.state[tid] = range[tid];
}

template <int R>
__global__ __launch_bounds__(kSplitThreads) void topk_stage(const float* __restrict__ score,
                                                            const int8_t* __restrict__ roles,
                                                            const int32_t* __restrict__ quota, int B, int Hkv, int N,
                                                            int W, int S, char* __restrict__ ws) {
    constexpr int NW = kSplitThreads / kWave;
    __shared__ __align__(16) uint32_t hist[R * kDigits];
    __shared__ Bucket bk[R];
    __shared__ uint2 cls[R + 1];  // {lowest surely kept key, top digit of the undecided ones}
    __shared__ uint32_t range[2];
    __shared__ int tmp[2][NW];
    __shared__ uint4 rec[kMaxSlices];  // per slice: its counts as words from the workspace start of the segment, its bins
    const int tid = threadIdx.x;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x / S, me = blockIdx.x - seg * S;
    const Slice sl = slice_of<R>(ws, seg, me, S, N);
    const int b = (seg / Hkv) % B;
    const int P = N - W, end = sl.begin + sl.len;
    const float* sc = score + (size_t)seg * N;
    const int8_t* ro = roles + (size_t)b * N;
    // the first step's keys are in flight while the counts are added up
    float s[kSplitSpan];
    uint32_t lab[kSplitSpan / 4];
    if (sl.begin + tid * kSplitSpan < end) load_span_any<kSplitSpan>(sc, ro, sl.begin + tid * kSplitSpan, N, s, lab);

    const uint32_t* seg_ws = reinterpret_cast<const uint32_t*>(ws + (size_t)seg * N * 8);
    if (tid < kMaxSlices) {  // one wave: the bins occupied in any slice
        uint32_t lo = kDigits, hi = 0u;
        if (tid < S) {
            const Slice o = slice_of<R>(ws, seg, tid, S, N);
            lo = o.state[0];
            hi = o.state[1];
            rec[tid] = make_uint4((uint32_t)(o.counts - seg_ws), lo, hi, 0u);
        }
#pragma unroll
        for (int off = 1; off < kWave; off <<= 1) {
            lo = min(lo, (uint32_t)__shfl_xor((int)lo, off));
            hi = max(hi, (uint32_t)__shfl_xor((int)hi, off));
        }
        if (tid == 0) {
            range[0] = lo;
            range[1] = hi;
        }
    }
    for (int e = tid; e < R * kDigits / 4; e += kSplitThreads)
        reinterpret_cast<uint4*>(hist)[e] = make_uint4(0u, 0u, 0u, 0u);
    if (tid < R) bk[tid] = Bucket{kModeSelect, 32, 0, 0u, kNoKey, kNoKey, kNoKey};
    __syncthreads();
    const int p0 = (int)range[0] / 2, np = max(0, ((int)range[1] + 1) / 2 - p0);
    for (int e = tid; e < R * np; e += kSplitThreads) {
        const int p = p0 + e % np, w = (e / np) * (kDigits / 2) + p;
        uint32_t c0 = 0u, c1 = 0u;
#pragma unroll 8
        for (int o = 0; o < S; ++o) {
            const uint4 x = rec[o];
            // pairs of a slice outside its own bins were not written
            const uint32_t v = 2 * p + 1 >= (int)x.y && 2 * p < (int)x.z ? seg_ws[x.x + w] : 0u;
            c0 += v & 0xffffu;
            c1 += v >> 16;
        }
        hist[2 * w] = c0;
        hist[2 * w + 1] = c1;
    }
    __syncthreads();
    if (wave < R) find_digit(bk[wave], hist + wave * kDigits, true, quota[(size_t)b * R + wave]);
    __syncthreads();
    if (tid <= R) {
        uint2 c = make_uint2(kNoKey, kNoKey);
        if (tid < R) {
            const Bucket& x = bk[tid];
            c.x = x.keep_from;
            // top digits are at most +inf's 0x7fc, so the shift does not overflow
            if (x.mode == kModeSelect && x.lo > 0) c = make_uint2((x.pref + 1u) << kLowBits, x.pref);
            if (me == 0) {  // for topk_finish
                sl.state[4 + 3 * tid] = (uint32_t)(x.mode == kModeSelect && x.lo > 0);
                sl.state[5 + 3 * tid] = x.pref;
                sl.state[6 + 3 * tid] = (uint32_t)x.need;
            }
        }
        cls[tid] = c;
    }
    __syncthreads();
    int turn = 0, staged = 0;
    for (int base = sl.begin; base < end; base += kSplitStep) {
        const int t0 = base + tid * kSplitSpan;
        if (base > sl.begin && t0 < end) load_span_any<kSplitSpan>(sc, ro, t0, N, s, lab);
        uint32_t smask = 0u, tag[kSplitSpan];
#pragma unroll
        for (int e = 0; e < kSplitSpan; ++e) {
            const int t = t0 + e;
            const uint32_t key = score_key(s[e]);
            const uint32_t r = t < P ? bucket_of<R>(lab, e) : (uint32_t)R;
            const uint2 c = cls[r];
            const bool kept = t >= P || key >= c.x;
            tag[e] = kept ? kKept : ((r << kLowBits) | (key & kLowMask));
            smask |= (t < end && (kept || (key >> kLowBits) == c.y)) ? (1u << e) : 0u;
        }
        int total;
        int at = staged + block_scan<NW>(__popc(smask), total, tmp, turn);
#pragma unroll
        for (int e = 0; e < kSplitSpan; ++e)
            if ((smask >> e) & 1u) {
                sl.tags[at] = tag[e];
                sl.offs[at] = (uint16_t)(t0 + e - sl.begin);
                ++at;
            }
        staged += total;
    }
    if (tid == 0) sl.state[2] = (uint32_t)staged;
}

template <int R>
__global__ __launch_bounds__(kSplitThreads) void topk_finish(int N, int S, int k_cap, const char* __restrict__ ws,
                                                             int32_t* __restrict__ idx_out,
                                                             int32_t* __restrict__ count_out) {
    constexpr int NW = kSplitThreads / kWave, kHold = kHoldOf<R>;
    __shared__ __align__(16) uint32_t hist[R * kDigits];
    __shared__ Bucket bk[R + 1];
    __shared__ uint32_t top[R];          // first digit of the undecided keys
    __shared__ int first[kMaxSlices + 1];  // staged keys before each slice
    __shared__ int begin[kMaxSlices + 1];  // first position of each slice
    __shared__ int wave_eq[NW][R], wave_keep[NW];
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int seg = blockIdx.x;
    char* w8 = const_cast<char*>(ws);
    if (tid < kMaxSlices) {  // one wave
        const int n = tid < S ? (int)slice_of<R>(w8, seg, tid, S, N).state[2] : 0;
        first[tid + 1] = wave_scan(n);
        begin[tid] = slice_begin(min(tid, S), S, N);
        if (tid == 0) {
            first[0] = 0;
            begin[kMaxSlices] = N;
        }
    }
    if (tid <= R) {
        Bucket x{kModeNone, 0, 0, 0u, kNoKey, kNoKey, kNoKey};
        if (tid < R) {
            const uint32_t* st = slice_of<R>(w8, seg, 0, S, N).state + 4 + 3 * tid;
            if (st[0] != 0u) x = Bucket{kModeSelect, kLowBits, (int)st[2], st[1], kNoKey, kNoKey, st[1]};
            top[tid] = st[1];
        }
        bk[tid] = x;
    }
    for (int e = tid; e < R * kDigits / 4; e += kSplitThreads)
        reinterpret_cast<uint4*>(hist)[e] = make_uint4(0u, 0u, 0u, 0u);
    __syncthreads();
    const char* seg_ws = ws + (size_t)seg * N * 8;  // below 2^32 bytes long
    // each wave takes a contiguous share of the staged keys, kHold per lane at a
    // time (entry j of lane l: base + 64 j + l), all loads in flight together; a
    // share of at most 64 kHold keys is loaded once and stays in registers
    const int T = first[S];
    const int i0 = (int)((long long)T * wave / NW), i1 = (int)((long long)T * (wave + 1) / NW);
    const bool once = i1 - i0 <= kWave * kHold;
    // the slice of staged key i, for growing i: first staged key and end, first position, length
    struct Cursor {
        int s, f, nx, p, len;
    };
    auto seek = [&](Cursor& c, int i) __attribute__((always_inline)) {
        while (c.nx <= i) {  // ends: i < T = first[S]
            ++c.s;
            c.f = c.nx;
            c.nx = first[c.s + 1];
            c.p = begin[c.s];
            c.len = begin[c.s + 1] - c.p;
        }
    };
    auto open = [&](int i) __attribute__((always_inline)) {
        int s = 0;
        for (int step = kMaxSlices / 2; step > 0; step >>= 1)
            if (s + step < S && first[s + step] <= i) s += step;
        return Cursor{s, first[s], first[s + 1], begin[s], begin[s + 1] - begin[s]};
    };
    uint32_t tg[kHold];
    auto load = [&](int base) __attribute__((always_inline)) {
        Cursor c = open(min(base + lane, i1 - 1));
#pragma unroll
        for (int j = 0; j < kHold; ++j) {
            const int i = min(base + j * kWave + lane, i1 - 1);
            seek(c, i);
            tg[j] = *reinterpret_cast<const uint32_t*>(seg_ws + 4u * (uint32_t)(2 * c.p + i - c.f));
        }
    };
    // visit(j, tag, valid) for every entry of the share in order
    auto sweep = [&](auto&& visit) __attribute__((always_inline)) {
        for (int base = i0; base < i1; base += kWave * kHold) {
            if (!once) load(base);
#pragma unroll
            for (int j = 0; j < kHold; ++j)
                if (base + j * kWave < i1)  // uniform
                    visit(base + j * kWave, tg[j], base + j * kWave + lane < i1);
        }
    };
    if (once && i0 < i1) load(i0);
    auto full_key = [&](uint32_t tg, uint32_t& r) {
        r = tg >> kLowBits;
        return (top[r] << kLowBits) | (tg & kLowMask);
    };
    for (int pass = 1; pass < 3; ++pass) {
        bool any = false;
#pragma unroll
        for (int r = 0; r < R; ++r) any |= bk[r].match != kNoKey;
        if (!any) break;  // uniform
        const int lo = 32 - kDigitBits * pass, w = min(kDigitBits, lo);
        sweep([&](int, uint32_t tg, bool valid) {
            if (valid && tg != kKept) {
                uint32_t r;
                const uint32_t key = full_key(tg, r);
                if ((key >> lo) == bk[r].match)
                    atomicAdd(&hist[r * kDigits + ((key >> (lo - w)) & ((1u << w) - 1u))], 1u);
            }
        });
        __syncthreads();
        if (wave < R) find_digit(bk[wave], hist + wave * kDigits, false, 0);
        __syncthreads();
    }
    // class of a staged key: 1 kept, 2 + r equal to the threshold of bucket r
    // (of which some stay), 0 dropped
    auto classify = [&](uint32_t tg, bool valid) {
        if (!valid) return 0;
        if (tg == kKept) return 1;
        uint32_t r;
        const uint32_t key = full_key(tg, r);
        return key >= bk[r].keep_from ? 1 : (key == bk[r].tie ? 2 + (int)r : 0);
    };
    int keep = 0, eq[R];
#pragma unroll
    for (int r = 0; r < R; ++r) eq[r] = 0;
    sweep([&](int, uint32_t tg, bool valid) {
        const int c = classify(tg, valid);
        keep += (int)__popcll(__ballot(c == 1));
        if (__ballot(c >= 2) != 0ull) {
#pragma unroll
            for (int r = 0; r < R; ++r) eq[r] += (int)__popcll(__ballot(c == 2 + r));
        }
    });
    if (lane == 0) {
#pragma unroll
        for (int r = 0; r < R; ++r) wave_eq[wave][r] = eq[r];
    }
    __syncthreads();
    int eq_left[R];  // keys equal to the threshold that may still be kept, from this wave's first on
#pragma unroll
    for (int r = 0; r < R; ++r) {
        eq_left[r] = bk[r].need;
        for (int v = 0; v < wave; ++v) eq_left[r] -= wave_eq[v][r];
        keep += max(0, min(eq[r], eq_left[r]));
    }
    if (lane == 0) wave_keep[wave] = keep;
    __syncthreads();
    int pos = 0, total = 0;
#pragma unroll
    for (int v = 0; v < NW; ++v) {
        pos += v < wave ? wave_keep[v] : 0;
        total += wave_keep[v];
    }
    const uint64_t lt = (1ull << lane) - 1ull;
    Cursor cur{};
    if (i0 < i1) cur = open(min(i0 + lane, i1 - 1));
    // positions loaded together, for kept and dropped entries alike (one at a
    // time 8 segments of 10^6 keys take 237 us, by eights 211)
    constexpr int kGroup = 8;
    static_assert(kHold % kGroup == 0, "whole groups");
    for (int base = i0; base < i1; base += kWave * kHold) {
        if (!once) load(base);
#pragma unroll
        for (int g = 0; g < kHold; g += kGroup) {
            if (base + g * kWave < i1) {  // uniform
                int32_t ps[kGroup];
#pragma unroll
                for (int j = 0; j < kGroup; ++j) {
                    const int i = min(base + (g + j) * kWave + lane, i1 - 1);
                    seek(cur, i);
                    ps[j] = cur.p + (int32_t)*reinterpret_cast<const uint16_t*>(
                                        seg_ws + 2u * (uint32_t)(4 * cur.p + 2 * cur.len + i - cur.f));
                }
#pragma unroll
                for (int j = 0; j < kGroup; ++j) {
                    const int c = classify(tg[g + j], base + (g + j) * kWave + lane < i1);
                    bool k = c == 1;
                    if (__ballot(c >= 2) != 0ull) {
#pragma unroll
                        for (int r = 0; r < R; ++r) {
                            const uint64_t m = __ballot(c == 2 + r);
                            if (c == 2 + r) k = (int)__popcll(m & lt) < eq_left[r];
                            eq_left[r] -= (int)__popcll(m);
                        }
                    }
                    const uint64_t km = __ballot(k);
                    const int at = pos + (int)__popcll(km & lt);
                    if (k && at < k_cap) idx_out[(size_t)seg * k_cap + at] = ps[j];
                    pos += (int)__popcll(km);
                }
            }
        }
    }
    if (tid == 0 && count_out != nullptr) count_out[seg] = total;
}

constexpr int kCompactRows = 64;

// One workgroup per (segment, 64 kept rows); a row is PARTS pieces of 16 bytes
// (8, 16 or 32), piece e of the block being part e % PARTS of row e / PARTS.
// Source rows are read through views (any row strides), the compacted rows
// are written dense.
// Every thread takes 64 PARTS / 256 pieces, in rounds of at most four: it
// issues the round's index loads, then its row loads, then its stores, so that
// a block waits for memory about twice per round instead of once per piece.
// Every row is read once and written once: non-temporal loads and stores.  8
// layers, 13108 of 65536 token-major rows each (862 MB): 169 us with cached
// accesses, 162 with non-temporal loads, 156 with non-temporal stores, 147
// with both (5.9 TB/s); 1024 segments, 1639 of 32768 rows: 333 and 301 us.
template <int PARTS>
__global__ __launch_bounds__(kThreads) void compact_kernel(RowView kv, RowView vv_, int B, int Hkv,
                                                           const int32_t* __restrict__ idx,
                                                           const int32_t* __restrict__ count, int N,
                                                           int k_cap, int nblk, char* __restrict__ k_out,
                                                           char* __restrict__ v_out) {
    constexpr int kRowBytes = PARTS * 16;
    constexpr int kItems = kCompactRows * PARTS / kThreads;
    constexpr int kRound = kItems < 4 ? kItems : 4;
    static_assert(kItems * kThreads == kCompactRows * PARTS && kItems % kRound == 0, "whole pieces per thread");
    const int blk = blockIdx.x % nblk;
    const int seg = blockIdx.x / nblk;
    const int cnt = min(count[seg], k_cap);
    const int m0 = blk * kCompactRows;
    if (m0 >= cnt) return;
    const int total = min(kCompactRows, cnt - m0) * PARTS;
    // segments are (layer, sample, KV head), KV head fastest
    const int lb = seg / Hkv;
    const long long so_k = (long long)(lb / B) * kv.s_layer + (long long)(lb % B) * kv.s_batch +
                           (long long)(seg % Hkv) * kv.s_head;
    const long long so_v = (long long)(lb / B) * vv_.s_layer + (long long)(lb % B) * vv_.s_batch +
                           (long long)(seg % Hkv) * vv_.s_head;
    const char* k = kv.base + so_k;
    const char* v = vv_.base != nullptr ? vv_.base + so_v : nullptr;
    const bool same_rows = vv_.s_token == kv.s_token;  // K and V rows equally spaced: one offset for both
    for (int i0 = 0; i0 < kItems; i0 += kRound) {
        if (i0 * kThreads >= total) break;  // uniform
        int t[kRound];
#pragma unroll
        for (int i = 0; i < kRound; ++i) {
            const int e = min((i0 + i) * kThreads + (int)threadIdx.x, total - 1);
            t[i] = idx[(size_t)seg * k_cap + m0 + e / PARTS];
        }
        u32x4 kr[kRound], vr[kRound];
#pragma unroll
        for (int i = 0; i < kRound; ++i) {
            const int e = min((i0 + i) * kThreads + (int)threadIdx.x, total - 1);
            const int tt = min(max(t[i], 0), N - 1);  // out-of-range indices are skipped below
            // token strides are below 2^25 bytes (checked by the caller): 32 x 32-bit products
            const unsigned piece = (unsigned)(e % PARTS) * 16u;
            const unsigned long long ko = (unsigned long long)(unsigned)tt * (unsigned)kv.s_token + piece;
            kr[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(k + ko));
            if (v != nullptr)
                vr[i] = __builtin_nontemporal_load(reinterpret_cast<const u32x4*>(
                    v + (same_rows ? ko : (unsigned long long)(unsigned)tt * (unsigned)vv_.s_token + piece)));
        }
#pragma unroll
        for (int i = 0; i < kRound; ++i) {
            const int e = (i0 + i) * kThreads + (int)threadIdx.x;
            if (e < total && t[i] >= 0 && t[i] < N) {
                const size_t dst = ((size_t)seg * k_cap + m0 + e / PARTS) * kRowBytes + (size_t)(e % PARTS) * 16;
                __builtin_nontemporal_store(kr[i], reinterpret_cast<u32x4*>(k_out + dst));
                if (v != nullptr) __builtin_nontemporal_store(vr[i], reinterpret_cast<u32x4*>(v_out + dst));
            }
        }
    }
}

#define KVE_TOPK_R(X) X(1) X(2) X(3) X(4) X(5) X(6) X(7) X(8)

template <int R>
hipError_t run_regs(const float* score, const int8_t* roles, const int32_t* quota, unsigned segs, int B, int Hkv,
                    int N, int W, int k_cap, int32_t* idx_out, int32_t* count_out, hipStream_t st) {
#define KVE_REGS_LAUNCH(NT, SPAN)                                                                              \
    hipLaunchKernelGGL((topk_regs<R, NT, SPAN>), dim3(segs), dim3(NT), 0, st, score, roles, quota, B, Hkv, N, W, \
                       k_cap, idx_out, count_out)
    if (N <= 1024)
        KVE_REGS_LAUNCH(256, 4);
    else if (N <= 4096)
        KVE_REGS_LAUNCH(1024, 4);
    else if (N <= 8192)
        KVE_REGS_LAUNCH(1024, 8);
    else
        KVE_REGS_LAUNCH(1024, 16);
#undef KVE_REGS_LAUNCH
    return hipGetLastError();
}

template <int R>
hipError_t run_split(const float* score, const int8_t* roles, const int32_t* quota, unsigned segs, int slices, int B,
                     int Hkv, int N, int W, int k_cap, int32_t* idx_out, int32_t* count_out, void* ws,
                     hipStream_t st) {
    char* w = static_cast<char*>(ws);
    hipLaunchKernelGGL(topk_count<R>, dim3(segs * slices), dim3(kSplitThreads), 0, st, score, roles, B, Hkv, N, W,
                       slices, w);
    hipLaunchKernelGGL(topk_stage<R>, dim3(segs * slices), dim3(kSplitThreads), 0, st, score, roles, quota, B, Hkv, N,
                       W, slices, w);
    hipLaunchKernelGGL(topk_finish<R>, dim3(segs), dim3(kSplitThreads), 0, st, N, slices, k_cap, w, idx_out,
                       count_out);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_topk(const float* score, const int8_t* roles, const int32_t* quota, const uint32_t* hist,
                       int L, int B, int Hkv, int N, int W, int R, int k_cap, int32_t* idx_out, int32_t* count_out,
                       void* ws, hipStream_t st) {
    const size_t segs = (size_t)L * B * Hkv;
    if (hist == nullptr && topk_in_regs(segs, N, R)) {
        switch (R) {
#define KVE_TOPK_CASE(RR) \
    case RR:              \
        return run_regs<RR>(score, roles, quota, (unsigned)segs, B, Hkv, N, W, k_cap, idx_out, count_out, st);
            KVE_TOPK_R(KVE_TOPK_CASE)
#undef KVE_TOPK_CASE
            default:
                return hipErrorInvalidValue;
        }
    }
    const int slices = hist == nullptr ? topk_slices(segs, N, R) : 0;
    if (slices > 1) {
        switch (R) {
#define KVE_TOPK_CASE(RR)                                                                                       \
    case RR:                                                                                                    \
        return run_split<RR>(score, roles, quota, (unsigned)segs, slices, B, Hkv, N, W, k_cap, idx_out, count_out, \
                             ws, st);
            KVE_TOPK_R(KVE_TOPK_CASE)
#undef KVE_TOPK_CASE
            default:
                return hipErrorInvalidValue;
        }
    }
    uint2* stage = static_cast<uint2*>(ws);
    // few segments: sixteen waves per segment instead of four
    const bool wide = segs < (size_t)kWideBelow;
    const dim3 grid((unsigned)segs);
    switch (R) {
#define KVE_TOPK_LAUNCH(RR, NT)                                                                             \
    hipLaunchKernelGGL((topk_kernel<RR, NT>), grid, dim3(NT), 0, st, score, roles, quota, hist, B, Hkv, N, W, \
                       k_cap, idx_out, count_out, stage)
#define KVE_TOPK_CASE(RR)                      \
    case RR:                                   \
        if (wide)                              \
            KVE_TOPK_LAUNCH(RR, kWideThreads); \
        else                                   \
            KVE_TOPK_LAUNCH(RR, kThreads);     \
        break;
        KVE_TOPK_R(KVE_TOPK_CASE)
#undef KVE_TOPK_CASE
#undef KVE_TOPK_LAUNCH
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

hipError_t launch_compact(const RowView& k, const RowView& v, int elem_bytes, const int32_t* idx,
                          const int32_t* count, int L, int B, int Hkv, int N, int d, int k_cap,
                          void* k_out, void* v_out, hipStream_t st) {
    const size_t segs = (size_t)L * B * Hkv;
    const int nblk = (k_cap + kCompactRows - 1) / kCompactRows;
    if (nblk == 0 || segs == 0) return hipSuccess;
    const dim3 grid((unsigned)(segs * nblk));
    char* ko = static_cast<char*>(k_out);
    char* vo = static_cast<char*>(v_out);
    switch (d * elem_bytes / 16) {  // 16-byte pieces per row
        case 8:
            hipLaunchKernelGGL(compact_kernel<8>, grid, dim3(kThreads), 0, st, k, v, B, Hkv, idx, count, N, k_cap,
                               nblk, ko, vo);
            break;
        case 16:
            hipLaunchKernelGGL(compact_kernel<16>, grid, dim3(kThreads), 0, st, k, v, B, Hkv, idx, count, N, k_cap,
                               nblk, ko, vo);
            break;
        case 32:
            hipLaunchKernelGGL(compact_kernel<32>, grid, dim3(kThreads), 0, st, k, v, B, Hkv, idx, count, N, k_cap,
                               nblk, ko, vo);
            break;
        default:
            return hipErrorInvalidValue;
    }
    return hipGetLastError();
}

}  // namespace kve
