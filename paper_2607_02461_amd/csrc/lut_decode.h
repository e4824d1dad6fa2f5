// What the LUT-decode GEMM kernels share: the decode of packed codes to bf16, code loads, and the
// layer epilogue (rescaling, bias, GELU, output type) of finished sums.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "device.h"

namespace orbit {

namespace {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float floatx16 __attribute__((ext_vector_type(16)));
typedef float floatx4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x3 __attribute__((ext_vector_type(3)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// 32 packed codes of one row: 4*BITS bytes, in BITS words (4 words for 2- and 3-bit codes too)
template <int BITS>
using Codes = uint32_t[BITS == 6 ? 6 : 4];

struct ByteTables {
    uint32_t lo[2], hi[2];  // byte e of lo[e/4] (hi[e/4]) is the low (high) byte of table entry e
};

// `lut` holds the levels in label order (entry l is the level of sign-magnitude label l).  Tables
// of at most eight levels hold every label.  The 4-bit table holds labels 0..7 only, the positive
// levels by rank: the codebook is antisymmetric (L[15-c] = -L[c], Sec. 3's symmetric marginal),
// so label 8 + m is the negation of label m, and the decoder looks up the low three bits and
// moves bit 3 into the bf16 sign bit.  The host checks the antisymmetry bit for bit.
template <int BITS>
__device__ __forceinline__ ByteTables make_tables(const uint16_t* lut) {
    constexpr int n = BITS == 4 ? 8 : BITS == 6 ? 0 : 1 << BITS, first = 0;
    ByteTables t;
#pragma unroll
    for (int w = 0; w < 2; ++w) {
        uint32_t lo = 0, hi = 0;
#pragma unroll
        for (int b = 0; b < 4; ++b) {
            const int e = 4 * w + b;
            const uint32_t v = e < n ? lut[first + e] : 0u;
            lo |= (v & 0xFFu) << (8 * b);
            hi |= (v >> 8) << (8 * b);
        }
        t.lo[w] = lo;
        t.hi[w] = hi;
    }
    return t;
}

// Canonical slot order.  The eight codes of each aligned group k0..k7 are written to eight
// consecutive bf16 slots in the order k0 k2 k4 k6 k1 k3 k5 k7.  Both operands use the same order
// for every bit width, so every MFMA still contracts matching k; the order is the one the 4-bit
// decoder produces without any byte shuffling (even and odd nibbles of a code word).

// Four table indices (one per byte of sel, each below 8) -> bf16 low and high bytes.
__device__ __forceinline__ void lookup_bytes(uint32_t sel, const ByteTables& t, uint32_t& lo, uint32_t& hi) {
    lo = __builtin_amdgcn_perm(t.lo[1], t.lo[0], sel);
    hi = __builtin_amdgcn_perm(t.hi[1], t.hi[0], sel);
}

// low/high byte words of four values -> two bf16x2 words (values 0,1 and 2,3)
__device__ __forceinline__ void interleave(uint32_t lo, uint32_t hi, uint32_t& d0, uint32_t& d1) {
    d0 = __builtin_amdgcn_perm(hi, lo, 0x05010400u);  // [lo0 hi0 lo1 hi1]
    d1 = __builtin_amdgcn_perm(hi, lo, 0x07030602u);  // [lo2 hi2 lo3 hi3]
}

// Group g (codes 8g .. 8g+7) of 32 packed codes (4*BITS bytes, LSB-first) -> four bf16x2 words in
// canonical slot order, in eight pieces (0-3 the even codes, 4-7 the odd ones, with a few exceptions)
// that the kernels place between their MFMAs: with the decode in one lump behind four MFMAs the
// large kernel runs 5% slower.  The empty asm on the code word pins the decode at its use: otherwise
// the compiler starts it right after the codes' load, which then has to complete a whole K-step early.
template <int BITS>
struct Decode8 {
    uint32_t x, lo, hi, out[4];

    template <int P>
    __device__ __forceinline__ void piece(const Codes<BITS>& w, int g, const ByteTables& t) {
        if constexpr (BITS == 4) {
            // nibble j of x is the label of code k_j: bits 0-2 index the magnitude table, bit 3 (the
            // sign) becomes bit 7 of the high byte, where bf16 keeps its sign
            if constexpr (P == 0) {
                x = w[g];
                asm volatile("" : "+v"(x));
                lookup_bytes(x & 0x07070707u, t, lo, hi);          // k0 k2 k4 k6
            } else if constexpr (P == 1) {
                hi |= (x << 4) & 0x80808080u;
            } else if constexpr (P == 2) {
                interleave(lo, hi, out[0], out[1]);
            } else if constexpr (P == 3) {
                lookup_bytes((x >> 4) & 0x07070707u, t, lo, hi);   // k1 k3 k5 k7
            } else if constexpr (P == 4) {
                hi |= x & 0x80808080u;
            } else if constexpr (P == 5) {
                interleave(lo, hi, out[2], out[3]);
            }
        } else if constexpr (BITS == 3) {
            // 24 bits, code j at bits 3j.  Four fields 6 bits apart move 2, 4 and 6 bits up to the bytes
            // of a word in two steps (fields 2, 3 by four, then fields 1, 3 by two)
            if constexpr (P == 0) {
                const int bit = 24 * g;
                x = bit == 0 ? w[0] : bit == 24 ? __builtin_amdgcn_alignbit(w[1], w[0], 24)
                  : bit == 48 ? __builtin_amdgcn_alignbit(w[2], w[1], 16) : w[2] >> 8;
                asm volatile("" : "+v"(x));
                lo = spread6(x);
            } else if constexpr (P == 1) {
                lookup_bytes(lo, t, lo, hi);
            } else if constexpr (P == 2) {
                interleave(lo, hi, out[0], out[1]);
            } else if constexpr (P == 4) {
                lo = spread6(x >> 3);
            } else if constexpr (P == 5) {
                lookup_bytes(lo, t, lo, hi);
            } else if constexpr (P == 6) {
                interleave(lo, hi, out[2], out[3]);
            }
        } else {
            static_assert(BITS == 2, "bits");
            if constexpr (P == 0) {
                uint32_t xw = w[g >> 1];
                asm volatile("" : "+v"(xw));
                x = xw >> (16 * (g & 1));                        // 16 bits, code j at bits 2j
                const uint32_t e = x & 0x3333u;                  // nibble i holds k2i
                lo = __builtin_amdgcn_perm(e >> 4, e, 0x05010400u) & 0x03030303u;
            } else if constexpr (P == 1) {
                lookup_bytes(lo, t, lo, hi);
            } else if constexpr (P == 2) {
                interleave(lo, hi, out[0], out[1]);
            } else if constexpr (P == 4) {
                const uint32_t o = (x >> 2) & 0x3333u;           // nibble i holds k2i+1
                lo = __builtin_amdgcn_perm(o >> 4, o, 0x05010400u) & 0x03030303u;
            } else if constexpr (P == 5) {
                lookup_bytes(lo, t, lo, hi);
            } else if constexpr (P == 6) {
                interleave(lo, hi, out[2], out[3]);
            }
        }
    }

    static __device__ __forceinline__ uint32_t spread6(uint32_t v) {
        v = (v & 0x00000FFFu) | ((v << 4) & 0xFFFFF000u);        // fields at 0, 6, 16, 22
        return ((v & 0x00FF00FFu) | ((v << 2) & 0xFF00FF00u)) & 0x07070707u;
    }
};

// 6-bit groups: 64 levels are too many for byte permutes, so the bf16 levels sit in a 64-entry
// LDS table with a 4-byte stride; every entry has its own bank, so a wave's 64 lookups never
// conflict (equal codes broadcast).
template <>
struct Decode8<6> {
    uint32_t lo, hi, v[8], out[4];
    const uint32_t* tab;

    template <int P>
    __device__ __forceinline__ void piece(const Codes<6>& w, int g, const ByteTables&) {
        if constexpr (P == 0) {
            // group g covers bits 48g .. 48g+47 of the 192-bit stream (selects, not an indexed load
            // from the register array)
            lo = g == 0 ? w[0] : g == 1 ? w[1] : g == 2 ? w[3] : w[4];
            hi = g == 0 ? w[1] : g == 1 ? w[2] : g == 2 ? w[4] : w[5];
            asm volatile("" : "+v"(lo), "+v"(hi));
        }
        if constexpr (P < 4) {
            const uint64_t x = (((uint64_t)hi << 32) | lo) >> ((g & 1) * 16);
            v[2 * P] = tab[(uint32_t)(x >> (12 * P)) & 63u];
            v[2 * P + 1] = tab[(uint32_t)(x >> (12 * P + 6)) & 63u];
        } else if constexpr (P == 4) {
            out[0] = v[0] | (v[2] << 16);
        } else if constexpr (P == 5) {
            out[1] = v[4] | (v[6] << 16);
        } else if constexpr (P == 6) {
            out[2] = v[1] | (v[3] << 16);
        } else {
            out[3] = v[5] | (v[7] << 16);
        }
    }
};

template <int P>
using Piece = std::integral_constant<int, P>;

// Pieces 2Q and 2Q + 1; all eight
template <int Q, int BITS>
__device__ __forceinline__ void two_pieces(Decode8<BITS>& d, const Codes<BITS>& w, int g, const ByteTables& t) {
    d.template piece<2 * Q>(w, g, t);
    d.template piece<2 * Q + 1>(w, g, t);
}
template <int BITS>
__device__ __forceinline__ uint4 decode_all(Decode8<BITS>& d, const Codes<BITS>& w, int g, const ByteTables& t) {
    two_pieces<0>(d, w, g, t);
    two_pieces<1>(d, w, g, t);
    two_pieces<2>(d, w, g, t);
    two_pieces<3>(d, w, g, t);
    return make_uint4(d.out[0], d.out[1], d.out[2], d.out[3]);
}

template <int BITS>
__device__ __forceinline__ void load_codes32(const uint8_t* src, Codes<BITS>& w) {
    if constexpr (BITS == 4) {
        const uint4 v = *(const uint4*)src;
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else if constexpr (BITS == 6) {
        // 24 bytes at an 8-byte aligned offset
        const uint2 a = *(const uint2*)src, b = *(const uint2*)(src + 8), c = *(const uint2*)(src + 16);
        w[0] = a.x; w[1] = a.y; w[2] = b.x; w[3] = b.y; w[4] = c.x; w[5] = c.y;
    } else if constexpr (BITS == 2) {
        const uint2 v = *(const uint2*)src;
        w[0] = v.x; w[1] = v.y; w[2] = 0; w[3] = 0;
    } else {
        const uint32_t* s = (const uint32_t*)src;
        w[0] = s[0]; w[1] = s[1]; w[2] = s[2]; w[3] = 0;
    }
}

__device__ __forceinline__ float bf16_to_f32(uint16_t v) { return __uint_as_float((uint32_t)v << 16); }

__device__ __forceinline__ uint32_t f32_to_bf16_rne(float x) {
    const uint32_t u = __float_as_uint(x);
    if ((u & 0x7FFFFFFFu) > 0x7F800000u) return 0x7FC0u;  // NaN stays NaN
    return (u + 0x7FFFu + ((u >> 16) & 1u)) >> 16;
}

// GELU(v) = v * Phi(v), Phi the standard normal CDF, with Phi from the complementary error
// function: Phi(v) = 1 - q for v >= 0 and q for v < 0, q = erfc(|v|/sqrt(2)) / 2.  erfc is the
// Chebyshev-fitted form of Numerical Recipes in C (2nd ed., Sec. 6.2, erfcc): for x >= 0,
//     erfc(x) = t exp(-x^2 + P(t)),  t = 1 / (1 + x/2),  P a degree-9 polynomial,
// with fractional error below 1.2e-7 everywhere, so GELU keeps its relative accuracy in the
// negative tail too.  log2(e) is folded into the coefficients (the hardware exponential is base
// 2) and the factor 1/2 of q into the constant term.  One reciprocal, one exp2 and nine fused
// multiply-adds without branches: on a layer's outputs (|Y| up to a few units) the library erff
// takes several ranges whose branches diverge across a wave.
__device__ __forceinline__ float gelu_erfc(float v) {
    constexpr float L2E = 1.4426950408889634f;
    constexpr float c0 = -1.26551223f * L2E - 1.f, c1 = 1.00002368f * L2E, c2 = 0.37409196f * L2E,
                    c3 = 0.09678418f * L2E, c4 = -0.18628806f * L2E, c5 = 0.27886807f * L2E,
                    c6 = -1.13520398f * L2E, c7 = 1.48851587f * L2E, c8 = -0.82215223f * L2E,
                    c9 = 0.17087277f * L2E;
    const float t = __builtin_amdgcn_rcpf(fmaf(0.35355339059327373f, fabsf(v), 1.f));  // x = |v|/sqrt(2)
    float P = fmaf(t, c9, c8);
    P = fmaf(t, P, c7);
    P = fmaf(t, P, c6);
    P = fmaf(t, P, c5);
    P = fmaf(t, P, c4);
    P = fmaf(t, P, c3);
    P = fmaf(t, P, c2);
    P = fmaf(t, P, c1);
    P = fmaf(t, P, c0);
    const float q = t * __builtin_amdgcn_exp2f(fmaf(v * v, -0.5f * L2E, P));
    return v * (v >= 0.f ? 1.f - q : q);
}

// The rest of the layer after the rescaled contraction: bias, then GELU (x * Phi(x)).
__device__ __forceinline__ float epilogue_value(const GemmParams& p, float v, float bias) {
    v += bias;
    if (p.gelu) v = gelu_erfc(v);
    return v;
}

__device__ __forceinline__ void store_one(const GemmParams& p, int64_t row, int64_t col, float v) {
    if (p.out_bf16)
        ((uint16_t*)p.Y)[row * p.ldy + col] = (uint16_t)f32_to_bf16_rne(v);
    else
        ((float*)p.Y)[row * p.ldy + col] = v;
}

// bf16 r' and bias (zero without one) of columns c .. c+3, zero past the last column
__device__ __forceinline__ void load_columns(const GemmParams& p, int64_t c, uint2& rw, uint2& bias) {
    if (c + 3 < p.N && p.vec4) {
        rw = *(const uint2*)(p.wn + c);
        bias = p.bias ? *(const uint2*)(p.bias + c) : make_uint2(0u, 0u);
    } else {
        uint16_t v[4], w[4];
#pragma unroll
        for (int r = 0; r < 4; ++r) {
            v[r] = c + r < p.N ? p.wn[c + r] : (uint16_t)0;
            w[r] = p.bias && c + r < p.N ? p.bias[c + r] : (uint16_t)0;
        }
        rw = make_uint2(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16));
        bias = make_uint2(w[0] | ((uint32_t)w[1] << 16), w[2] | ((uint32_t)w[3] << 16));
    }
}

// finished outputs of columns c .. c+3 of a row, as one vector where the layout allows it
__device__ __forceinline__ void store_four(const GemmParams& p, int64_t row, int64_t c, const floatx4& v) {
    const bool full = c + 3 < p.N && p.vec4;
    if (full && p.out_bf16) {
        *(uint2*)((uint16_t*)p.Y + row * p.ldy + c) =
            make_uint2(f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16),
                       f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16));
    } else if (full) {
        *(float4*)((float*)p.Y + row * p.ldy + c) = make_float4(v[0], v[1], v[2], v[3]);
    } else {
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (c + r < p.N) store_one(p, row, c + r, v[r]);
    }
}

}  // namespace

}  // namespace orbit
