// float32 rows as pairs of float16 rows, for contractions of float32 operands
// on the 16-bit matrix instructions.
//
// A row x is scaled by a power of two that takes its largest element into
// [2^14, 2^15) and split into hi = f16(x) and lo = f16(x - hi), both rounded to
// nearest: hi + lo holds x to 2^-23 of its value for elements down to 2^-16 of
// the row's largest, and to 2^-39 of the largest below that.  A product of two
// rows is hi hi + hi lo + lo hi, summed in float32; lo lo, up to 2^-22 of the
// product, is left out.  The scale of a row is undone by an exact
// multiplication of the sums.
//
// Why: v_mfma_f32_32x32x2_f32 does 64 multiply-adds per cycle and SIMD, the
// 16-bit form 1024 with the sums in float32 too, so three products take less
// than a fifth of the time.  Against sum |a| |b| of two rows a logit is off by
// up to 8 units of 2^-24 (two operands, the term left out) and the sums' 24
// roundings per 128 elements; with the float32 instruction by 64 roundings.
//
// The 2^-39 of a row's largest element are an absolute error, which the other
// row may meet with a large element: through them a logit is off by up to
//   sl2 2^-39 (max|a| sum|b| + max|b| sum|a|).
// Where this passes 2^-22 for a chunk's rows and the workgroup's register rows
// (below it, it is less of the softmax weights than float32's rounding), or a
// row is infinite or its scale is no normal number, the kernels leave the
// pairs: the chunks from the last check of the flag on go through the float32
// instruction, with the register rows loaded again as float32 into the
// registers that held the pairs (rest_f32).  Rows of N(0, 1) elements stay
// below the line by a factor of several hundred, rows with one channel 2^8
// times the others by about ten.
#pragma once

#include <type_traits>

#include "kve_stream.h"

namespace kve {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));
typedef float f32x4 __attribute__((ext_vector_type(4)));

struct SplitScale {
    float scale, unscale;
};
// Largest magnitude and sum of magnitudes of a row.
struct RowMag {
    float mx, sum;
};
constexpr float kSplitWide = 0x1p-17f;  // sl2 (max|a| sum|b| + ..) 2^-17 <= 1: below 2^-22 of a logit
// rows of smaller elements would have a subnormal unscale, rows for which sl2
// takes it below kSplitTinyScale a subnormal product of the two
constexpr float kSplitTiny = 0x1p-110f, kSplitTinyScale = 0x1p-120f;

// scale and unscale = 1 / scale of a row whose largest magnitude is mx, finite;
// a row of zeros, or of elements below 2^-113, is scaled by 2^127
__device__ __forceinline__ SplitScale split_scale(float mx) {
    const int e = (int)(__float_as_uint(mx) >> 23) & 0xff;
    const int s = min(127 + 14 - (e - 127), 254);  // biased exponent of the scale, >= 13
    SplitScale r;
    r.scale = __uint_as_float((uint32_t)s << 23);
    r.unscale = s == 254 ? 0x1p-127f : __uint_as_float((uint32_t)(254 - s) << 23);
    return r;
}
__device__ __forceinline__ void split8(const f32x8& x, float scale, f16x8& hi, f16x8& lo) {
    const f32x8 y = x * scale;
    hi = __builtin_convertvector(y, f16x8);
    f32x8 d;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = __builtin_fmaf((float)hi[e], -1.0f, y[e]);
    lo = __builtin_convertvector(d, f16x8);
}
__device__ __forceinline__ float abs_max8(const f32x8& x) {
    float m = fabsf(x[0]);
#pragma unroll
    for (int e = 1; e < 8; ++e) m = fmaxf(m, fabsf(x[e]));
    return m;
}

// maximum (sum) of a lane's value and that of lane l ^ 32, or l ^ 16
__device__ __forceinline__ float half_wave_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row16_max(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row16_sum(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// lane 31: the maximum over lanes 0 .. 31 of x >= 0
__device__ __forceinline__ float max_to_lane31(float x) {
    auto shifted = [](float v, auto ctrl, auto rows) {
        return __uint_as_float((uint32_t)__builtin_amdgcn_update_dpp(0, (int)__float_as_uint(v), decltype(ctrl)::value,
                                                                     decltype(rows)::value, 0xf, true));
    };
    using std::integral_constant;
    x = fmaxf(x, shifted(x, integral_constant<int, 0x111>{}, integral_constant<int, 0xf>{}));  // row_shr:1
    x = fmaxf(x, shifted(x, integral_constant<int, 0x112>{}, integral_constant<int, 0xf>{}));  // row_shr:2
    x = fmaxf(x, shifted(x, integral_constant<int, 0x114>{}, integral_constant<int, 0xf>{}));  // row_shr:4
    x = fmaxf(x, shifted(x, integral_constant<int, 0x118>{}, integral_constant<int, 0xf>{}));  // row_shr:8
    return fmaxf(x, shifted(x, integral_constant<int, 0x142>{}, integral_constant<int, 0xa>{}));  // row_bcast:15
}

// Chunks of 64 float32 rows of D elements: `raw` as the chunk loads leave them
// in LDS, split into the planes hi and lo, each laid out like a chunk of 64
// 16-bit rows.  The two planes take the room of a second raw chunk, which is
// what they are once a workgroup has left the pairs.
template <int D>
struct SplitChunk {
    static constexpr int KEYS = 64;
    using Raw = KChunk<float, D, KEYS>;
    using Half = KChunk<__bf16, D, KEYS>;
    static constexpr int NSTEP = Half::NSTEP;
    static constexpr int PLANE = Half::BYTES;
    struct Frags {
        f16x8 hi[NSTEP], lo[NSTEP];
    };
    static constexpr int NQ = D / 8;
    struct FragsF32 {
        f32x4 x[NQ];  // lane l: 16-byte pieces 2 j + l / 32 of its row
    };
    struct Lds {  // the small arrays first: a read's immediate offset ends at 65535
        __align__(16) float unscale[KEYS];
        __align__(16) RowMag mag[4];  // per wave: of its register rows
        int wide;                     // set: some row split so far needs float32
        __align__(16) char raw[Raw::BYTES];
        __align__(16) char planes[2 * PLANE];  // hi, lo
        __device__ __forceinline__ char* hi() { return planes; }
        __device__ __forceinline__ char* lo() { return planes + PLANE; }
    };
    static_assert(2 * PLANE == Raw::BYTES, "the planes hold a raw chunk");
    // Addresses differ from one per lane by an exclusive or of constants (the
    // swizzle is one); `opaque` keeps the compiler from holding every one of
    // them in a register across the chunk loop.
    __device__ __forceinline__ static int opaque(int x) {
        asm volatile("" : "+v"(x));
        return x;
    }

    // Fragments of one register row (element k of lane l as in Mma): lanes l
    // and l ^ 32 hold the two halves of the row.  Zero when !valid.  Returns
    // the row's unscale and its magnitudes.
    __device__ __forceinline__ static float load_row(Frags& f, RowMag& mag, const char* row, bool valid, int lane) {
        f32x8 x[NSTEP];
        mag = RowMag{0.0f, 0.0f};
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            const float* p = reinterpret_cast<const float*>(row) + st * 16 + (lane >> 5) * 8;
            x[st] = f32x8{};
            if (valid) {
                const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
                x[st] = f32x8{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            }
            mag.mx = fmaxf(mag.mx, abs_max8(x[st]));
#pragma unroll
            for (int e = 0; e < 8; ++e) mag.sum += fabsf(x[st][e]);
        }
        mag = RowMag{half_wave_max(mag.mx), half_wave_sum(mag.sum)};
        const SplitScale s = split_scale(mag.mx);
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            split8(x[st], s.scale, f.hi[st], f.lo[st]);
            pin(f.hi[st]);
            pin(f.lo[st]);
        }
        return s.unscale;
    }
    __device__ __forceinline__ static void load_row_f32(FragsF32& f, const char* row, bool valid, int lane) {
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            f.x[j] = valid ? *reinterpret_cast<const f32x4*>(row + (2 * j + (lane >> 5)) * 16) : f32x4{};
            pin(f.x[j]);
        }
    }

    // The largest magnitudes of a workgroup's register rows (mag[s]: of the
    // lane's row of set s, ls[s] its unscale times sl2), times sl2 and the
    // bound's factor.  A row whose scale is no normal number, or whose sum is
    // not finite, makes them infinite.  Every wave calls it, once, before the
    // first split; its barrier also publishes chunk 0.
    template <int RS>
    __device__ __forceinline__ static RowMag group_mag(Lds& sh, const RowMag (&mag)[RS], const float (&ls)[RS],
                                                       float sl2, int wave, int lane) {
        RowMag m{0.0f, 0.0f};
#pragma unroll
        for (int s = 0; s < RS; ++s) {
            const bool out = !(mag[s].sum < INFINITY) || (mag[s].mx > 0.0f && !(ls[s] >= kSplitTinyScale));
            m.mx = fmaxf(m.mx, out ? INFINITY : mag[s].mx);
            m.sum = fmaxf(m.sum, out ? INFINITY : mag[s].sum);
        }
        m.mx = max_to_lane31(m.mx);
        m.sum = max_to_lane31(m.sum);
        if (lane == 31) {
            *reinterpret_cast<float2*>(&sh.mag[wave]) = make_float2(m.mx, m.sum);
            sh.wide = 0;
        }
        wait_vmcnt<0>();
        lds_barrier();
        m = RowMag{0.0f, 0.0f};
#pragma unroll
        for (int w = 0; w < 4; ++w) {
            m.mx = fmaxf(m.mx, sh.mag[w].mx);
            m.sum = fmaxf(m.sum, sh.mag[w].sum);
        }
        const float k = sl2 * kSplitWide;
        m.mx = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(m.mx * k)));
        m.sum = __uint_as_float(__builtin_amdgcn_readfirstlane(__float_as_uint(m.sum * k)));
        return m;
    }
    // Chunks after which the flag is tested: a test after each costs 4% of the
    // H2O passes, a test before the products holds a second set of accumulators
    // in registers.  What was summed since the last test is dropped where the
    // flag is set.
    static constexpr int kCheck = 8;
    __device__ __forceinline__ static bool check(int s, int nch) { return s % kCheck == kCheck - 1 || s + 1 == nch; }
    // The same for every wave of the workgroup between the barrier that follows
    // a split and the one before the next.
    __device__ __forceinline__ static bool wide(const Lds& sh) {
        return __builtin_expect(__builtin_amdgcn_readfirstlane(sh.wide) != 0, 0);
    }

    // Split of one chunk by the four waves of a workgroup: wave w takes rows
    // 16 w .. 16 w + 15, lane l the quarter l / 16 of row 16 w + l % 16 (the
    // sixteen lanes of an LDS cycle are sixteen rows at the same piece, which
    // the layout puts on sixteen bank groups, in the reads and in the writes).
    // The rows' unscale goes to LDS with the planes, and whether one of them is
    // too wide for pairs beside register rows of magnitudes `reg`: first by the
    // row's largest magnitude alone (its sum is at most D times that), which
    // settles it for ordinary rows, then by its sum.
    __device__ __forceinline__ static void convert(Lds& sh, const RowMag& reg, int wave, int lane) {
        constexpr int NP = D / 32;  // 16-byte pieces of a plane row per lane
        const int r = 16 * wave + (lane & 15), j = lane >> 4;
        f32x8 x[NP];
        float mx = 0.0f;
        const int ro = opaque(chunk_swz<Raw::ROW>(r, 2 * NP * j));
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float4 a = *reinterpret_cast<const float4*>(sh.raw + (ro ^ (32 * i)));
            const float4 b = *reinterpret_cast<const float4*>(sh.raw + (ro ^ (32 * i + 16)));
            x[i] = f32x8{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            mx = fmaxf(mx, abs_max8(x[i]));
        }
        mx = half_wave_max(row16_max(mx));
        const SplitScale s = split_scale(mx);
        const float at_most = fmaf((float)D, reg.mx, reg.sum);  // uniform
        const bool tiny = __float_as_uint(mx) - 1u < __float_as_uint(kSplitTiny) - 1u;  // false for 0
        if (__builtin_amdgcn_ballot_w64(!(mx * at_most <= 1.0f) || tiny) != 0) {  // rare
            float sum = 0.0f;
#pragma unroll
            for (int i = 0; i < NP; ++i)
#pragma unroll
                for (int e = 0; e < 8; ++e) sum += fabsf(x[i][e]);
            sum = half_wave_sum(row16_sum(sum));
            if (!(fmaf(mx, reg.sum, sum * reg.mx) <= 1.0f) || tiny) sh.wide = 1;
        }
        const int po = opaque(chunk_swz<Half::ROW>(r, NP * j));
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            f16x8 h, l;
            split8(x[i], s.scale, h, l);
            const int o = po ^ (16 * i);
            *reinterpret_cast<f16x8*>(sh.hi() + o) = h;
            *reinterpret_cast<f16x8*>(sh.lo() + o) = l;
        }
        if (j == 0) sh.unscale[r] = s.unscale;
    }

    // Products of the chunk's 64 rows with RS sets of 32 register rows, still
    // scaled.  LDS_A: the chunk rows are the A operand (element i of acc[s][b]
    // belongs to chunk row 32 b + c_row(i, lane), the lane to register row
    // lane % 32 of set s), otherwise the register rows are.  The small terms
    // go in before the large one of each k-step.
    template <bool LDS_A, int RS>
    __device__ __forceinline__ static void mma(f32x16 (&acc)[RS][2], Lds& sh, const Frags (&reg)[RS], int lane) {
        const char *hi = sh.hi(), *lo = sh.lo();
        const int fo = opaque(chunk_swz<Half::ROW>(lane & 31, lane >> 5));  // k-step st: piece 2 st + lane / 32
        auto one = [](f16x8 f, f16x8 g, f32x16 c) {
            return LDS_A ? __builtin_amdgcn_mfma_f32_32x32x16_f16(f, g, c, 0, 0, 0)
                         : __builtin_amdgcn_mfma_f32_32x32x16_f16(g, f, c, 0, 0, 0);
        };
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            f16x8 fh[2], fl[2];
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                fh[b] = *reinterpret_cast<const f16x8*>(hi + (fo ^ (32 * st)) + b * 32 * Half::ROW);
                fl[b] = *reinterpret_cast<const f16x8*>(lo + (fo ^ (32 * st)) + b * 32 * Half::ROW);
            }
#pragma unroll
            for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    acc[rs][b] = one(fl[b], reg[rs].hi[st], st > 0 ? acc[rs][b] : f32x16{});
#pragma unroll
            for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[rs][b] = one(fh[b], reg[rs].lo[st], acc[rs][b]);
#pragma unroll
            for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                for (int b = 0; b < 2; ++b) acc[rs][b] = one(fh[b], reg[rs].hi[st], acc[rs][b]);
        }
        // the next k-step's fragments are read once the lo ones of this step are
        // used up: 24 registers of fragments at most
        __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            __builtin_amdgcn_sched_group_barrier(0x008, 2 * RS, 0);
            if (st + 1 < NSTEP) __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 4 * RS, 0);
        }
    }

    // The same products with float32 operands on the float32 matrix
    // instruction, the chunk as loaded in `slot`; unscaled.  Four products of 64
    // cycles per 16-byte read and register set, as fast as the instruction allows.
    template <bool LDS_A, int RS>
    __device__ __forceinline__ static void mma_f32(f32x16 (&acc)[RS][2], const char* slot, const FragsF32 (&reg)[RS],
                                                   int lane) {
        const int fo = opaque(chunk_swz<Raw::ROW>(lane & 31, lane >> 5));  // step j: piece 2 j + lane / 32
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            f32x4 f[2];
#pragma unroll
            for (int b = 0; b < 2; ++b)
                f[b] = *reinterpret_cast<const f32x4*>(slot + (fo ^ (32 * j)) + b * 32 * Raw::ROW);
#pragma unroll
            for (int e = 0; e < 4; ++e)
#pragma unroll
                for (int rs = 0; rs < RS; ++rs)
#pragma unroll
                    for (int b = 0; b < 2; ++b) {
                        const f32x16 c = j > 0 || e > 0 ? acc[rs][b] : f32x16{};
                        acc[rs][b] = LDS_A ? Mma<float>::mma(f[b][e], reg[rs].x[j][e], c)
                                           : Mma<float>::mma(reg[rs].x[j][e], f[b][e], c);
                    }
        }
        // one step's fragments ahead
        __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
#pragma unroll
        for (int j = 0; j < NQ; ++j) {
            if (j + 1 < NQ) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
            __builtin_amdgcn_sched_group_barrier(0x008, 8 * RS, 0);
        }
    }

    // The chunks from s on with float32 operands: the planes and the raw slot
    // take turns.  issue(c, slot) starts chunk c's loads, use(c, slot) takes its
    // products.
    template <typename Issue, typename Use>
    __device__ __forceinline__ static void rest_f32(Lds& sh, int s, int nch, const Issue& issue, const Use& use) {
        wait_vmcnt<0>();
        lds_barrier();  // nothing is on its way to the raw slot, every wave is done with the planes
        issue(s, sh.planes);
#pragma unroll 1
        for (int c = s; c < nch; ++c) {
            char* slot = ((c - s) & 1) ? sh.raw : sh.planes;
            char* other = ((c - s) & 1) ? sh.planes : sh.raw;
            wait_vmcnt<0>();
            lds_barrier();  // chunk c landed; every wave is done with the other slot
            if (c + 1 < nch) issue(c + 1, other);
            use(c, slot);
        }
    }
};

}  // namespace kve
