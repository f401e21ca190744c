// float32 rows as pairs of float16 rows, for contractions of float32 operands
// on the 16-bit matrix instructions.
//
// A row x is scaled by a power of two that takes its largest element into
// [2^14, 2^15) and split into hi = f16(x) and lo = f16(x - hi), both rounded to
// nearest: hi + lo holds x to 2^-24 of its value, the rounding of float32
// itself, for elements down to 2^-17 of the row's largest, and to 2^-39 of the
// largest below that.  A product of two rows is hi hi + hi lo + lo hi, summed
// in float32; lo lo, below 2^-24 of the product, is left out.  The scale of a
// row is undone by an exact multiplication of the sums.
//
// Why: v_mfma_f32_32x32x2_f32 does 64 multiply-adds per cycle and SIMD, the
// 16-bit form 1024 with the sums in float32 too, so three products take less
// than a fifth of the time.  The sums see 24 roundings per 128 elements in
// place of 64: the logits are not further off their 64-bit values than those
// of the float32 instruction.
//
// A row with an infinite element has unscale = +inf: its infinite elements
// become +-1 and the others 0, so a product is +-inf by the sign of the other
// operand (NaN where that is 0), as in float32.  NaN elements stay NaN.
#pragma once

#include "kve_stream.h"

namespace kve {

typedef _Float16 f16x8 __attribute__((ext_vector_type(8)));
typedef float f32x8 __attribute__((ext_vector_type(8)));

struct SplitScale {
    float scale, unscale;
};
// scale and unscale = 1 / scale of a row whose largest magnitude is mx; a row
// of zeros, or of elements below 2^-113, is scaled by 2^127
__device__ __forceinline__ SplitScale split_scale(float mx) {
    const int e = (int)(__float_as_uint(mx) >> 23) & 0xff;
    const int s = min(127 + 14 - (e - 127), 254);  // biased exponent of the scale, >= 13
    SplitScale r;
    r.scale = __uint_as_float((uint32_t)s << 23);
    r.unscale = e == 255 ? INFINITY : (s == 254 ? 0x1p-127f : __uint_as_float((uint32_t)(254 - s) << 23));
    return r;
}
// elements of a row with an infinite one (see above)
__device__ __forceinline__ float split_inf(float x) {
    const uint32_t b = __float_as_uint(x);
    if ((b & 0x7fffffffu) > 0x7f800000u) return x;
    return __uint_as_float((b & 0x80000000u) | ((b & 0x7fffffffu) == 0x7f800000u ? 0x3f800000u : 0u));
}
__device__ __forceinline__ void split8(const f32x8& x, float scale, f16x8& hi, f16x8& lo) {
    const f32x8 y = x * scale;
    hi = __builtin_convertvector(y, f16x8);
    f32x8 d;
#pragma unroll
    for (int e = 0; e < 8; ++e) d[e] = __builtin_fmaf((float)hi[e], -1.0f, y[e]);
    lo = __builtin_convertvector(d, f16x8);
}
__device__ __forceinline__ float abs_max8(float m, const f32x8& x) {
#pragma unroll
    for (int e = 0; e < 8; ++e) m = fmaxf(m, fabsf(x[e]));
    return m;
}

// maximum of a lane's value and that of lane l ^ 32, or l ^ 16
__device__ __forceinline__ float half_wave_max(float x) {
    const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}
__device__ __forceinline__ float row16_max(float x) {
    const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

// Chunks of 64 float32 rows of D elements: `raw` as the chunk loads leave them
// in LDS, split into the planes hi and lo, each laid out like a chunk of 64
// 16-bit rows.
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
    // Addresses differ from one per lane by an exclusive or of constants (the
    // swizzle is one); `opaque` keeps the compiler from holding every one of
    // them in a register across the chunk loop.
    __device__ __forceinline__ static int opaque(int x) {
        asm volatile("" : "+v"(x));
        return x;
    }

    // Fragments of one register row (element k of lane l as in Mma): lanes l
    // and l ^ 32 hold the two halves of the row.  Zero when !valid.  Returns
    // the row's unscale.
    __device__ __forceinline__ static float load_row(Frags& f, const char* row, bool valid, int lane) {
        f32x8 x[NSTEP];
        float mx = 0.0f;
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            const float* p = reinterpret_cast<const float*>(row) + st * 16 + (lane >> 5) * 8;
            x[st] = f32x8{};
            if (valid) {
                const float4 a = *reinterpret_cast<const float4*>(p), b = *reinterpret_cast<const float4*>(p + 4);
                x[st] = f32x8{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            }
            mx = abs_max8(mx, x[st]);
        }
        mx = half_wave_max(mx);
        const SplitScale s = split_scale(mx);
#pragma unroll
        for (int st = 0; st < NSTEP; ++st) {
            if (s.unscale == INFINITY) {
#pragma unroll
                for (int e = 0; e < 8; ++e) x[st][e] = split_inf(x[st][e]);
            }
            split8(x[st], s.unscale == INFINITY ? 1.0f : s.scale, f.hi[st], f.lo[st]);
            pin(f.hi[st]);
            pin(f.lo[st]);
        }
        return s.unscale;
    }

    // Split of one chunk by the four waves of a workgroup: wave w takes rows
    // 16 w .. 16 w + 15, lane l the quarter l / 16 of row 16 w + l % 16 (the
    // sixteen lanes of an LDS cycle are sixteen rows at the same piece, which
    // the layout puts on sixteen bank groups, in the reads and in the writes).
    // unscale[row] goes to LDS with the planes.
    __device__ __forceinline__ static void convert(const char* raw, char* hi, char* lo, float* unscale, int wave,
                                                   int lane) {
        constexpr int NP = D / 32;  // 16-byte pieces of a plane row per lane
        const int r = 16 * wave + (lane & 15), j = lane >> 4;
        f32x8 x[NP];
        float mx = 0.0f;
        const int ro = opaque(chunk_swz<Raw::ROW>(r, 2 * NP * j));
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            const float4 a = *reinterpret_cast<const float4*>(raw + (ro ^ (32 * i)));
            const float4 b = *reinterpret_cast<const float4*>(raw + (ro ^ (32 * i + 16)));
            x[i] = f32x8{a.x, a.y, a.z, a.w, b.x, b.y, b.z, b.w};
            mx = abs_max8(mx, x[i]);
        }
        mx = half_wave_max(row16_max(mx));
        const SplitScale s = split_scale(mx);
        if (__builtin_amdgcn_ballot_w64(s.unscale == INFINITY) != 0) {  // rare
            if (s.unscale == INFINITY) {
#pragma unroll
                for (int i = 0; i < NP; ++i)
#pragma unroll
                    for (int e = 0; e < 8; ++e) x[i][e] = split_inf(x[i][e]);
            }
        }
        const float sc = s.unscale == INFINITY ? 1.0f : s.scale;
        const int po = opaque(chunk_swz<Half::ROW>(r, NP * j));
#pragma unroll
        for (int i = 0; i < NP; ++i) {
            f16x8 h, l;
            split8(x[i], sc, h, l);
            const int o = po ^ (16 * i);
            *reinterpret_cast<f16x8*>(hi + o) = h;
            *reinterpret_cast<f16x8*>(lo + o) = l;
        }
        if (j == 0) unscale[r] = s.unscale;
    }

    // Products of the chunk's 64 rows with RS sets of 32 register rows, still
    // scaled.  LDS_A: the chunk rows are the A operand (element i of acc[s][b]
    // belongs to chunk row 32 b + c_row(i, lane), the lane to register row
    // lane % 32 of set s), otherwise the register rows are.  The small terms
    // go in before the large one of each k-step.
    template <bool LDS_A, int RS>
    __device__ __forceinline__ static void mma(f32x16 (&acc)[RS][2], const char* hi, const char* lo,
                                               const Frags (&reg)[RS], int lane) {
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
};

}  // namespace kve
