// LUT-decode GEMM on packed Lloyd-Max codes for gfx950 (bf16 MFMA, fp32 accumulate).
//
// Computes Y[n][i] = s_n * r'_i * sum_k L_a[xc[n][k]] * L_w[wc[i][k]]: the rotation cancels in
// the product (Sec. 4.3), so the two code sets are contracted directly in the rotated basis;
// the paper's limitations section names this codebook GEMM as the missing kernel.
//
// Operands: codes are dequantized to the bf16 images of the levels and multiplied in bf16, the
// arithmetic the paper runs its layers in (codes dequantized to BF16, matmul in BF16); on the
// matrix cores the products accumulate in fp32.
//
// Decode: codes are widened to bytes and looked up with v_perm_b32 against byte tables of the
// bf16 levels (low bytes and high bytes of the 2^b levels, 8 entries per register pair), which
// needs no memory access.  Each code of a block tile is decoded exactly once, into a bf16 tile
// in LDS that the matrix cores then read.  bf16 products are exact in fp32, so the result
// differs from an fp64 evaluation with the same bf16 levels only by fp32 accumulation.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.h"
#include "lut_decode.h"

namespace orbit {

namespace {

constexpr int BM = 128, BN = 128, BK = 64;
constexpr int LDS_STRIDE = BK + 8;  // halves per tile row (padding against bank conflicts)

// c += b a^T for 16 rows of b and of a, 32 deep.  Written out so that the accumulator stays in its
// registers: the compiler gives the intrinsic's result a fresh quad, and with 32 quads of
// accumulators in 256 registers it then spills (2 to 22 registers; at 6-bit codes the large kernel ran
// at 0.79 of the rate).  The compiler's hazard tracking does not look inside asm, so the wait states are
// ours: mfma_ready() stands between the accumulators' zeroing and their first MFMA, mfma_done() between
// their last one and any other use, and nothing else writes them; the fragments come from LDS loads
// (waited for by counter).  A test reads both distances off the built code.
__device__ __forceinline__ void mfma16(floatx4& c, const bf16x8& b, const bf16x8& a) {
    asm volatile("v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" : "+v"(c) : "v"(b), "v"(a));
}

// Two wait states between a VALU write of the accumulators and an MFMA that reads them.
__device__ __forceinline__ void mfma_ready(floatx4 (&c)[4]) {
    asm volatile("s_nop 1" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]));
}

// The wait states between the last MFMAs and the first other use of their results (eleven are needed).
__device__ __forceinline__ void mfma_done(floatx4 (&c)[4]) {
    asm volatile("s_nop 15" : "+v"(c[0]), "+v"(c[1]), "+v"(c[2]), "+v"(c[3]));
}

// The code rows of a block tile as a buffer resource, and the same load through it: the tile's base
// and the K-step's offset are scalar, so a load takes one address register per lane and no address
// arithmetic.  Offsets are 32-bit: the caller keeps a tile's rows below 4 GiB.
__device__ __forceinline__ __amdgpu_buffer_rsrc_t code_buffer(const uint8_t* base, uint32_t bytes) {
    return __builtin_amdgcn_make_buffer_rsrc((void*)base, 0, (int)bytes, 0x00027000);
}

template <int BITS>
__device__ __forceinline__ void load_codes32(__amdgpu_buffer_rsrc_t buf, uint32_t voff, uint32_t soff, Codes<BITS>& w) {
    if constexpr (BITS == 4) {
        const u32x4 v = __builtin_amdgcn_raw_buffer_load_b128(buf, voff, soff, 0);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = v.w;
    } else if constexpr (BITS == 6) {
        const u32x2 a = __builtin_amdgcn_raw_buffer_load_b64(buf, voff, soff, 0);
        const u32x2 b = __builtin_amdgcn_raw_buffer_load_b64(buf, voff + 8, soff, 0);
        const u32x2 c = __builtin_amdgcn_raw_buffer_load_b64(buf, voff + 16, soff, 0);
        w[0] = a.x; w[1] = a.y; w[2] = b.x; w[3] = b.y; w[4] = c.x; w[5] = c.y;
    } else if constexpr (BITS == 2) {
        const u32x2 v = __builtin_amdgcn_raw_buffer_load_b64(buf, voff, soff, 0);
        w[0] = v.x; w[1] = v.y; w[2] = 0; w[3] = 0;
    } else {
        const u32x3 v = __builtin_amdgcn_raw_buffer_load_b96(buf, voff, soff, 0);
        w[0] = v.x; w[1] = v.y; w[2] = v.z; w[3] = 0;
    }
}

// SPLIT: workgroup z of a K-split contracts K-steps z*steps .. (z+1)*steps - 1 (the last split
// fewer) and stores its raw sums to p.ws[z][M][N]; lut_gemm_reduce applies the epilogue.
//
// 128x128 block tiles, K-step 64, four waves of 64x64.  This kernel serves grids too small for the
// 256x256 kernel where wave tiles are not faster (often one workgroup per compute unit, so one wave per SIMD), where each
// workgroup's time is its chain of K-steps: it is pipelined like the large kernel.  The block
// tile's codes are decoded once per K-step into a double-buffered bf16 tile in LDS (74 KB); while
// the matrix cores work on step s, each wave decodes step s+1 into the other stage (groups 0-1,
// 2, 3 in slices 0, 1, 2), fragments are read one 16-wide slice ahead, one barrier per step sits
// before the last slice, and the codes of the next five steps are in flight.
constexpr int SMALL_TILE = BM * LDS_STRIDE;  // halves per operand tile

template <int BA, int BW, bool SPLIT>
__global__ __launch_bounds__(256) void lut_gemm_kernel(GemmParams p) {
    extern __shared__ __align__(16) __bf16 slds[];  // [stage][A, B][128][72], then the 6-bit table
    constexpr int STAGE = 2 * SMALL_TILE;
    uint32_t* const tab6 = (uint32_t*)(slds + 2 * STAGE);  // 6-bit activation levels (bf16 in the low half)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 1, wn = wave & 1;
    const int64_t m0 = (int64_t)blockIdx.y * BM, n0 = (int64_t)blockIdx.x * BN;
    const ByteTables ta = make_tables<BA>(p.lut_a);
    const ByteTables tw = make_tables<BW>(p.lut_w);
    Decode8<BA> da;
    Decode8<BW> db;
    if constexpr (BA == 6) {
        if (tid < 64) tab6[tid] = p.lut_a[tid];
        __syncthreads();
        da.tab = tab6;
    }

    // this thread decodes 32 codes of one A row and 32 codes of one B row per K-step
    const int lr = tid >> 1, lh = tid & 1;
    const int64_t arow = min(m0 + lr, p.M - 1), brow = min(n0 + lr, p.N - 1);
    const int64_t a_row_bytes = (int64_t)p.K * BA / 8, b_row_bytes = (int64_t)p.K * BW / 8;
    // the K-steps this workgroup contracts
    const int kb = SPLIT ? (int)blockIdx.z * p.split_steps : 0;
    const int nk = SPLIT ? min(p.split_steps, p.K / BK - kb) : p.K / BK;
    const uint8_t* asrc = p.xc + arow * a_row_bytes + lh * 4 * BA + (int64_t)kb * (BK * BA / 8);
    const uint8_t* bsrc = p.wc + brow * b_row_bytes + lh * 4 * BW + (int64_t)kb * (BK * BW / 8);

    floatx16 acc[2][2];
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = 0.f;

    const int64_t astep = BK * BA / 8, bstep = BK * BW / 8;
    __bf16* const a_dst0 = slds + lr * LDS_STRIDE + lh * 32;  // this thread's decode slots, stage 0
    const __bf16* const a_frag0 = slds + (wm * 64 + (lane & 31)) * LDS_STRIDE + (lane >> 5) * 8;
    const __bf16* const b_frag0 = slds + SMALL_TILE + (wn * 64 + (lane & 31)) * LDS_STRIDE + (lane >> 5) * 8;

    auto decode_group = [&](int stage, int g, const Codes<BA>& ca, const Codes<BW>& cb) {
        *(uint4*)(a_dst0 + stage + 8 * g) = decode_all(da, ca, g, ta);
        *(uint4*)(a_dst0 + stage + SMALL_TILE + 8 * g) = decode_all(db, cb, g, tw);
    };

    // a ring of RING code register sets: set u holds the codes of the steps congruent to u, so
    // each load has RING - 1 K-steps to land (a workgroup here is often alone on its compute unit,
    // with nothing else to cover the memory latency)
    constexpr int RING = 6;
    Codes<BA> ca[RING];
    Codes<BW> cb[RING];
    load_codes32<BA>(asrc, ca[0]);
    load_codes32<BW>(bsrc, cb[0]);
#pragma unroll
    for (int g = 0; g < 4; ++g) decode_group(0, g, ca[0], cb[0]);
#pragma unroll
    for (int u = 1; u < RING; ++u) {
        const int64_t su = min(u, nk - 1);
        load_codes32<BA>(asrc + su * astep, ca[u]);
        load_codes32<BW>(bsrc + su * bstep, cb[u]);
    }
    __syncthreads();

    // fragments of one 16-wide k slice of a stage
    bf16x8 a[2][2], b[2][2];
    auto read_frags = [&](int stage, int kk, bf16x8 (&af)[2], bf16x8 (&bf)[2]) {
#pragma unroll
        for (int i = 0; i < 2; ++i) af[i] = *(const bf16x8*)(a_frag0 + stage + i * 32 * LDS_STRIDE + kk * 16);
#pragma unroll
        for (int j = 0; j < 2; ++j) bf[j] = *(const bf16x8*)(b_frag0 + stage + j * 32 * LDS_STRIDE + kk * 16);
    };
    read_frags(0, 0, a[0], b[0]);

    // as the large kernel's K-step: decode step s+1 (codes ca, cb) in slices 0-2, barrier before
    // slice 3, whose MFMAs overlap the next step's first fragments; the codes of step s+RING load
    // into (na, nb), the set step s came from
    auto kstep = [&](int s, const Codes<BA>& ca, const Codes<BW>& cb, Codes<BA>& na, Codes<BW>& nb) {
        // the last steps re-load the final step's codes; they are never used
        const int64_t sl = min(s + RING, nk - 1);
        load_codes32<BA>(asrc + sl * astep, na);
        load_codes32<BW>(bsrc + sl * bstep, nb);
        __builtin_amdgcn_sched_barrier(0);

        const int cur = (s & 1) * STAGE, nxt = STAGE - cur;
#pragma unroll
        for (int kk = 0; kk < BK / 16; ++kk) {
            const int f = kk & 1;
            if (kk == 3) __syncthreads();
            if (kk < 3) read_frags(cur, kk + 1, a[f ^ 1], b[f ^ 1]);
            else read_frags(nxt, 0, a[f ^ 1], b[f ^ 1]);
            if (kk == 0) {
                decode_group(nxt, 0, ca, cb);
                decode_group(nxt, 1, ca, cb);
            } else if (kk < 3) {
                decode_group(nxt, kk + 1, ca, cb);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[f][j], a[f][i], acc[i][j], 0, 0, 0);
            // next fragments first, then each MFMA followed by a share of the decode, the decoded
            // rows' LDS writes last
            __builtin_amdgcn_sched_group_barrier(0x100, 4, 0);
            if (kk == 0) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 15, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x200, 4, 0);
            } else if (kk < 3) {
#pragma unroll
                for (int m = 0; m < 4; ++m) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 8, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x200, 2, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    // step s + u decodes set (u + 1) % RING and refills set u; unrolled by RING so that every set
    // index is a constant (registers, none copied)
    int s = 0;
    for (; s + RING - 1 < nk; s += RING) {
#pragma unroll
        for (int u = 0; u < RING; ++u) kstep(s + u, ca[(u + 1) % RING], cb[(u + 1) % RING], ca[u], cb[u]);
    }
#pragma unroll
    for (int u = 0; u < RING - 1; ++u)
        if (s + u < nk) kstep(s + u, ca[(u + 1) % RING], cb[(u + 1) % RING], ca[u], cb[u]);

    // epilogue.  As in the large kernel, the MFMAs computed the transposed tile: element e of
    // accumulator (i, j) belongs to row i*32 + lane%32 and column j*32 + 8*(e/4) + 4*(lane/32) + e%4,
    // so each lane holds runs of four consecutive columns of one row and stores each run as one
    // vector.  Every load comes before the first store (as far as the compiler knows, Y may alias
    // xn, wn or the bias, and a wait placed among the stores would make each store wait for the
    // one before).
    const int64_t col0 = n0 + wn * 64 + 4 * (lane >> 5);
    // With a multiple of 4 columns (and, for Y, rows that allow 4-wide stores) the outputs go
    // through LDS, free after the main loop, so that each store covers 4 rows of contiguous bytes
    // (256 of fp32, 128 of bf16) instead of 32 rows of 16 or 8: each wave writes its 64 x 64
    // sub-tile into a region of its own (68 floats or 72 bf16 per row, padding that keeps the
    // accesses conflict-free) and reads it back by rows.
    constexpr int TS = 68, TSB = 72;
    float* const tl = (float*)slds + wave * (64 * TS);
    uint16_t* const tlb = (uint16_t*)tl;
    const int64_t colg = n0 + wn * 64 + 4 * (lane & 15);
    if constexpr (SPLIT) {
        float* const ws = p.ws + (int64_t)blockIdx.z * p.M * p.N;
        const bool vec = (p.N & 3) == 0;
        if (vec) {
            __syncthreads();   // every wave is done reading the stages
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < 2; ++j)
#pragma unroll
                    for (int q = 0; q < 4; ++q)
                        *(float4*)(tl + (i * 32 + (lane & 31)) * TS + j * 32 + 8 * q + 4 * (lane >> 5)) =
                            make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]);
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int r = 4 * t + (lane >> 4);
                const int64_t row = m0 + wm * 64 + r;
                const float4 v = *(const float4*)(tl + r * TS + 4 * (lane & 15));
                if (row < p.M && colg < p.N) *(float4*)(ws + row * p.N + colg) = v;
            }
            return;
        }
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int64_t row = m0 + wm * 64 + i * 32 + (lane & 31);
            if (row >= p.M) continue;
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int64_t c = col0 + j * 32 + 8 * q;
                    float* const dst = ws + row * p.N + c;
                    if (vec && c + 3 < p.N) {
                        *(float4*)dst = make_float4(acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2],
                                                    acc[i][j][4 * q + 3]);
                    } else {
#pragma unroll
                        for (int r = 0; r < 4; ++r)
                            if (c + r < p.N) dst[r] = acc[i][j][4 * q + r];
                    }
                }
        }
        return;
    }
    float xsv[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t row = m0 + wm * 64 + i * 32 + (lane & 31);
        xsv[i] = row < p.M ? p.xn[row] : 0.f;
    }
    uint2 rwv[2][4], bv[2][4];  // bf16 r' and bias of the lane's columns, four per (j, run)
#pragma unroll
    for (int j = 0; j < 2; ++j)
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int64_t c = col0 + j * 32 + 8 * q;
            if (c + 3 < p.N && p.vec4) {
                rwv[j][q] = *(const uint2*)(p.wn + c);
                bv[j][q] = p.bias ? *(const uint2*)(p.bias + c) : make_uint2(0u, 0u);
            } else {
                uint16_t v[4], w[4];
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    v[r] = c + r < p.N ? p.wn[c + r] : (uint16_t)0;
                    w[r] = p.bias && c + r < p.N ? p.bias[c + r] : (uint16_t)0;
                }
                rwv[j][q] = make_uint2(v[0] | ((uint32_t)v[1] << 16), v[2] | ((uint32_t)v[3] << 16));
                bv[j][q] = make_uint2(w[0] | ((uint32_t)w[1] << 16), w[2] | ((uint32_t)w[3] << 16));
            }
        }
    // every output value first, then the stores
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const uint2 rw = rwv[j][q], bb = bv[j][q];
                const float r4[4] = {__uint_as_float(rw.x << 16), __uint_as_float(rw.x & 0xFFFF0000u),
                                     __uint_as_float(rw.y << 16), __uint_as_float(rw.y & 0xFFFF0000u)};
                const float b4[4] = {__uint_as_float(bb.x << 16), __uint_as_float(bb.x & 0xFFFF0000u),
                                     __uint_as_float(bb.y << 16), __uint_as_float(bb.y & 0xFFFF0000u)};
#pragma unroll
                for (int r = 0; r < 4; ++r)
                    acc[i][j][4 * q + r] = epilogue_value(p, acc[i][j][4 * q + r] * xsv[i] * r4[r], b4[r]);
            }
    if (p.vec4 && (p.N & 3) == 0) {
        __syncthreads();   // every wave is done reading the stages
#pragma unroll
        for (int i = 0; i < 2; ++i)
#pragma unroll
            for (int j = 0; j < 2; ++j)
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const int lrow = i * 32 + (lane & 31), lcol = j * 32 + 8 * q + 4 * (lane >> 5);
                    const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
                    if (p.out_bf16)
                        *(uint2*)(tlb + lrow * TSB + lcol) =
                            make_uint2(f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16),
                                       f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16));
                    else
                        *(float4*)(tl + lrow * TS + lcol) = make_float4(v[0], v[1], v[2], v[3]);
                }
#pragma unroll
        for (int t = 0; t < 16; ++t) {
            const int r = 4 * t + (lane >> 4);
            const int64_t row = m0 + wm * 64 + r;
            if (p.out_bf16) {
                const uint2 v = *(const uint2*)(tlb + r * TSB + 4 * (lane & 15));
                if (row < p.M && colg < p.N) *(uint2*)((uint16_t*)p.Y + row * p.ldy + colg) = v;
            } else {
                const float4 v = *(const float4*)(tl + r * TS + 4 * (lane & 15));
                if (row < p.M && colg < p.N) *(float4*)((float*)p.Y + row * p.ldy + colg) = v;
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int64_t row = m0 + wm * 64 + i * 32 + (lane & 31);
        if (row >= p.M) continue;
#pragma unroll
        for (int j = 0; j < 2; ++j)
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int64_t c = col0 + j * 32 + 8 * q;
                const float v[4] = {acc[i][j][4 * q], acc[i][j][4 * q + 1], acc[i][j][4 * q + 2], acc[i][j][4 * q + 3]};
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
    }
}

// ------------------------------------------------------------------------------------------
// Large-problem kernel: 256x256 block tiles, K-step 64, eight waves of 128x64 each.  Every code
// of a block tile is decoded once per K-step into a double-buffered bf16 tile in LDS (128 KB),
// which halves the decodes per flop of the 128x128 kernel.  While the matrix cores work on step
// s, each wave decodes step s+1 into the other stage, and the codes of steps s+2 and s+3 are in
// flight.  Block tiles are visited so that the workgroups resident on one XCD (round-robin
// dispatch) share A and B panels in that XCD's L2.
//
// The kernel is bound by power: under its load the clock settles at 1.8-1.9 GHz of 2.4, so what
// counts is the energy of a step.  Hence v_mfma_f32_16x16x32_bf16 and not the 32x32x16 form: per
// product it moves a quarter of the accumulator bytes and twice the operand bytes, 0.5 against
// 0.62 bytes per multiply-add of register traffic, and a register-only loop on 4-bit Lloyd-Max
// levels runs at 2035 against 1800 TFLOP/s with it (2420 and 2460 on constant operands, where
// power does not bind).  Measured with it on 33272 x 5120 outputs, K = 13824, W4A4: 3.82 -> 3.50 ms
// (1233 -> 1346 TFLOP/s); 9216 x 9216, K = 3072, W2A4: 480 -> 432 us; 33272 x 13824, K = 5120, W4A6
// with GELU: 4.78 -> 4.56 ms.  Of that, the chunk swizzle below is 1.6% (padded rows of 144 bytes
// conflict two ways under the 16-row fragment reads) and walking the B fragments back and forth,
// so that neighbouring MFMAs share an operand, 1.3%.  The same loop without its decode runs 10%
// faster, without its LDS writes 7%.
constexpr int BM2 = 256, BN2 = 256, BK2 = 64;
constexpr uint32_t LDS2_TILE = BM2 * BK2 * 2;          // bytes per operand tile (rows of 128)
constexpr uint32_t LDS2_BYTES = 8 * 64 * 68 * 4;       // the epilogue's regions: more than two stages
static_assert(LDS2_BYTES >= 4 * LDS2_TILE, "the stages fit");
constexpr int64_t MAX_K2 = (int64_t)1 << 24;           // 256 rows of 6-bit codes stay below 4 GiB
constexpr int GROUP_M = 8;                            // block rows per L2 group

template <int BA, int BW>
__global__ __launch_bounds__(512, 2) void lut_gemm_big(GemmParams p, int ntm, int ntn, int per_xcd) {
    extern __shared__ __align__(16) unsigned char lds[];  // A, B: [stage][256][64] bf16, chunks swizzled
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int wm = wave >> 2, wn = wave & 3;

    // XCD-aware tile order: workgroup pid runs on XCD pid % 8; consecutive ids per XCD
    const int pid = blockIdx.x;
    const int nid = (pid & 7) * per_xcd + (pid >> 3);
    const int total = ntm * ntn;
    if (nid >= total) return;
    const int in_group = GROUP_M * ntn;
    const int first_m = (nid / in_group) * GROUP_M;
    const int gsize = min(ntm - first_m, GROUP_M);
    const int tm = first_m + (nid % in_group) % gsize;
    const int tn = (nid % in_group) / gsize;
    const int64_t m0 = (int64_t)tm * BM2, n0 = (int64_t)tn * BN2;

    const ByteTables ta = make_tables<BA>(p.lut_a);
    const ByteTables tw = make_tables<BW>(p.lut_w);
    Decode8<BA> da;
    Decode8<BW> db;
    if constexpr (BA == 6) {
        uint32_t* const tab6 = (uint32_t*)(lds + LDS2_BYTES);  // 6-bit levels, after the tiles
        if (tid < 64) tab6[tid] = p.lut_a[tid];
        __syncthreads();
        da.tab = tab6;
    }

    // this thread decodes 32 codes of one A row and 32 codes of one B row per K-step
    const int lr = tid >> 1, lh = tid & 1;
    const int64_t arow = min(m0 + lr, p.M - 1), brow = min(n0 + lr, p.N - 1);
    const uint32_t a_row = (uint32_t)p.K / 8 * BA, b_row = (uint32_t)p.K / 8 * BW;  // bytes (K <= MAX_K2)
    const __amdgpu_buffer_rsrc_t abuf = code_buffer(p.xc + m0 * a_row, (uint32_t)min((int64_t)BM2, p.M - m0) * a_row);
    const __amdgpu_buffer_rsrc_t bbuf = code_buffer(p.wc + n0 * b_row, (uint32_t)min((int64_t)BN2, p.N - n0) * b_row);
    const uint32_t aoff = (uint32_t)(arow - m0) * a_row + lh * 4 * BA;
    const uint32_t boff = (uint32_t)(brow - n0) * b_row + lh * 4 * BW;

    floatx4 acc[8][4];
#pragma unroll
    for (int i = 0; i < 8; ++i)
#pragma unroll
        for (int j = 0; j < 4; ++j)
#pragma unroll
            for (int e = 0; e < 4; ++e) acc[i][j][e] = 0.f;
#pragma unroll
    for (int i = 0; i < 8; ++i) mfma_ready(acc[i]);

    const int nk = p.K / BK2;
    const int astep = BK2 * BA / 8, bstep = BK2 * BW / 8;
    // A tile row is 128 bytes; its 16-byte chunk c sits at chunk c ^ (row & 7).  A fragment read (16
    // rows, four chunks of each) and a decode's write (32 rows, two chunks of each) are then free of
    // bank conflicts.  The two stages of an operand are neighbours (an immediate offset).
    uint32_t adst[4], bdst[4];
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        adst[g] = lr * 128 + (((lh * 4) ^ (lr & 7)) ^ g) * 16;
        bdst[g] = adst[g] + 2 * LDS2_TILE;
    }
    const uint32_t fswz = (uint32_t)((lane >> 4) ^ (lane & 7)) * 16;
    const uint32_t afrag = (wm * 128 + (lane & 15)) * 128 + fswz;
    const uint32_t bfrag = (wn * 64 + (lane & 15)) * 128 + fswz + 2 * LDS2_TILE;

    // four code register sets: set u holds the codes of the steps congruent to u
    Codes<BA> sa[4];
    Codes<BW> sb[4];
    load_codes32<BA>(abuf, aoff, 0, sa[0]);
    load_codes32<BW>(bbuf, boff, 0, sb[0]);
#pragma unroll
    for (int g = 0; g < 4; ++g) {
        *(uint4*)(lds + adst[g]) = decode_all(da, sa[0], g, ta);
        *(uint4*)(lds + bdst[g]) = decode_all(db, sb[0], g, tw);
    }
    {
        const int s1 = nk > 1 ? 1 : 0, s2 = nk > 2 ? 2 : nk - 1;
        load_codes32<BA>(abuf, aoff, s1 * astep, sa[1]);
        load_codes32<BA>(abuf, aoff, s2 * astep, sa[2]);
        load_codes32<BW>(bbuf, boff, s1 * bstep, sb[1]);
        load_codes32<BW>(bbuf, boff, s2 * bstep, sb[2]);
    }
    __syncthreads();

    // A K-step is sixteen groups of 4 MFMAs: group q contracts the 32-deep k slice q / 8 of A fragment
    // q % 8 with the slice's four B fragments.  A fragments are read three groups ahead.
    bf16x8 a[4], b[2][4];
    auto read_a = [&](uint32_t stage, int q) {
        a[q & 3] = *(const bf16x8*)(lds + (afrag ^ (64 * (q >> 3))) + stage + (q & 7) * 2048);
    };
    auto read_b = [&](uint32_t stage, int slice, int j) {
        b[slice][j] = *(const bf16x8*)(lds + (bfrag ^ (64 * slice)) + stage + j * 2048);
    };
    read_a(0, 0);
#pragma unroll
    for (int j = 0; j < 4; ++j) read_b(0, 0, j);
    read_a(0, 1);
    read_a(0, 2);

    // Groups 0-11 decode the codes of step s+1 into the other stage, a piece behind every MFMA; then
    // one barrier makes that stage complete and retires every read of this step's stage, so groups
    // 13-15 can already fetch the next step's first fragments while their MFMAs run.  Even steps load
    // the codes of steps s+3 and s+4 (64 bytes of each row in one go: 1.3-2% over one step at a time,
    // a quarter fewer requests to the L2), so each load has two K-steps to land.
    auto kstep = [&](auto u_tag, int s) {
        constexpr int U = decltype(u_tag)::value;
        const Codes<BA>& ca = sa[(U + 1) & 3];
        const Codes<BW>& cb = sb[(U + 1) & 3];
        if constexpr (U % 2 == 0) {
            // the last steps re-load the final step's codes; they are never used
            const int s3 = min(s + 3, nk - 1), s4 = min(s + 4, nk - 1);
            load_codes32<BA>(abuf, aoff, s3 * astep, sa[(U + 3) & 3]);
            load_codes32<BA>(abuf, aoff, s4 * astep, sa[U]);
            load_codes32<BW>(bbuf, boff, s3 * bstep, sb[(U + 3) & 3]);
            load_codes32<BW>(bbuf, boff, s4 * bstep, sb[U]);
        }
        __builtin_amdgcn_sched_barrier(0);

        constexpr uint32_t cur = (U & 1) * LDS2_TILE, nxt = LDS2_TILE - cur;
#pragma unroll
        for (int q = 0; q < 16; ++q) {
            const int slice = q >> 3, r = q & 7;
            if (q == 13) __syncthreads();
            // (on the final step the fragments come from a refilled stage nobody uses)
            if (q < 13) read_a(cur, q + 3);
            else read_a(nxt, q - 13);
            if (q >= 2 && q < 6) read_b(cur, 1, q - 2);
            else if (q == 13 || q == 14) {
                read_b(nxt, 0, 2 * (q - 13));
                read_b(nxt, 0, 2 * (q - 13) + 1);
            }
            // the next step's eight decodes (A and B of each code group): one in each of groups 0-3,
            // one in each two of groups 4-11
            const int item = q < 4 ? q : 4 + ((q - 4) >> 1), g = item >> 1;
            auto pieces = [&](auto qt) {
                constexpr int Q = decltype(qt)::value;
                if (q < 4) {
                    if (item & 1) two_pieces<Q>(db, cb, g, tw);
                    else two_pieces<Q>(da, ca, g, ta);
                } else if (q < 12) {
                    if (item & 1) {
                        if (q & 1) db.template piece<Q + 4>(cb, g, tw);
                        else db.template piece<Q>(cb, g, tw);
                    } else {
                        if (q & 1) da.template piece<Q + 4>(ca, g, ta);
                        else da.template piece<Q>(ca, g, ta);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            };
            // B fragments forth and back, so that neighbouring MFMAs share an operand
            const int j0 = (r & 1) ? 3 : 0, dj = (r & 1) ? -1 : 1;
            __builtin_amdgcn_sched_barrier(0);
            mfma16(acc[r][j0], b[slice][j0], a[q & 3]);
            pieces(Piece<0>{});
            mfma16(acc[r][j0 + dj], b[slice][j0 + dj], a[q & 3]);
            pieces(Piece<1>{});
            mfma16(acc[r][j0 + 2 * dj], b[slice][j0 + 2 * dj], a[q & 3]);
            pieces(Piece<2>{});
            mfma16(acc[r][j0 + 3 * dj], b[slice][j0 + 3 * dj], a[q & 3]);
            pieces(Piece<3>{});
            if (q < 4 || (q < 12 && (q & 1))) {
                if (item & 1) *(uint4*)(lds + bdst[g] + nxt) = make_uint4(db.out[0], db.out[1], db.out[2], db.out[3]);
                else *(uint4*)(lds + adst[g] + nxt) = make_uint4(da.out[0], da.out[1], da.out[2], da.out[3]);
            }
        }
    };

    // unrolled by four so that every register set and stage is a constant
    int s = 0;
    for (; s + 3 < nk; s += 4) {
        kstep(Piece<0>{}, s);
        kstep(Piece<1>{}, s + 1);
        kstep(Piece<2>{}, s + 2);
        kstep(Piece<3>{}, s + 3);
    }
    if (s < nk) kstep(Piece<0>{}, s);
    if (s + 1 < nk) kstep(Piece<1>{}, s + 1);
    if (s + 2 < nk) kstep(Piece<2>{}, s + 2);
#pragma unroll
    for (int i = 0; i < 8; ++i) mfma_done(acc[i]);

    // epilogue.  The MFMAs computed the transposed tile, so element e of accumulator (i, j)
    // belongs to row i*16 + lane%16 and column j*16 + 4*(lane/16) + e: each lane
    // holds runs of four consecutive columns of one row and stores them as one vector (16 bytes
    // of fp32 or 8 of bf16).
    const int64_t col0 = n0 + wn * 64 + 4 * (lane >> 4);
    uint2 rwv[4], bv[4];  // bf16 r' and bias (zero without one) of the lane's columns, four per j
#pragma unroll
    for (int j = 0; j < 4; ++j) load_columns(p, col0 + j * 16, rwv[j], bv[j]);
    const bool plain = !p.bias && !p.gelu && !p.out_bf16;
    // the lane's eight row norms before the first store (Y may alias xn as far as the compiler
    // knows, so a load after a store would wait for it)
    float xsv[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t row = m0 + wm * 128 + i * 16 + (lane & 15);
        xsv[i] = row < p.M ? p.xn[row] : 0.f;
    }
    // the four outputs of accumulator (i, j)
    auto outputs = [&](int i, int j) {
        floatx4 v;
        const float xs = xsv[i];
        v[0] = acc[i][j][0] * xs * __uint_as_float(rwv[j].x << 16);
        v[1] = acc[i][j][1] * xs * __uint_as_float(rwv[j].x & 0xFFFF0000u);
        v[2] = acc[i][j][2] * xs * __uint_as_float(rwv[j].y << 16);
        v[3] = acc[i][j][3] * xs * __uint_as_float(rwv[j].y & 0xFFFF0000u);
        if (!plain) {
            v[0] = epilogue_value(p, v[0], __uint_as_float(bv[j].x << 16));
            v[1] = epilogue_value(p, v[1], __uint_as_float(bv[j].x & 0xFFFF0000u));
            v[2] = epilogue_value(p, v[2], __uint_as_float(bv[j].y << 16));
            v[3] = epilogue_value(p, v[3], __uint_as_float(bv[j].y & 0xFFFF0000u));
        }
        return v;
    };
    // Rows that allow 4-wide stores (and a multiple of 4 columns): the finished outputs go through
    // LDS (free after the main loop) so that each store covers 4 rows of contiguous bytes (256 of
    // fp32, 128 of bf16) instead of 16 rows of 64 or 32 bytes.  Each wave owns a region of 64 rows
    // (68 floats or 72 bf16 per row, padding that keeps the accesses conflict-free) and turns its
    // 128 x 64 sub-tile around in two halves; a wave's LDS accesses run in order, so the halves
    // reuse the region without a barrier.
    if (p.vec4 && (p.N & 3) == 0) {
        __syncthreads();   // every wave is done reading the stages
        constexpr int TS = 68, TSB = 72;
        float* const tl = (float*)lds + wave * (64 * TS);
        uint16_t* const tlb = (uint16_t*)tl;
        const int64_t colg = n0 + wn * 64 + 4 * (lane & 15);
#pragma unroll
        for (int half = 0; half < 2; ++half) {
#pragma unroll
            for (int ii = 0; ii < 4; ++ii) {
                const int lrow = ii * 16 + (lane & 15);
#pragma unroll
                for (int j = 0; j < 4; ++j) {
                    const floatx4 v = outputs(4 * half + ii, j);
                    const int lcol = j * 16 + 4 * (lane >> 4);
                    if (p.out_bf16)
                        *(uint2*)(tlb + lrow * TSB + lcol) =
                            make_uint2(f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16),
                                       f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16));
                    else
                        *(floatx4*)(tl + lrow * TS + lcol) = v;
                }
            }
#pragma unroll
            for (int t = 0; t < 16; ++t) {
                const int r = 4 * t + (lane >> 4);
                const int64_t row = m0 + wm * 128 + 64 * half + r;
                if (p.out_bf16) {
                    const uint2 v = *(const uint2*)(tlb + r * TSB + 4 * (lane & 15));
                    if (row < p.M && colg < p.N) *(uint2*)((uint16_t*)p.Y + row * p.ldy + colg) = v;
                } else {
                    const float4 v = *(const float4*)(tl + r * TS + 4 * (lane & 15));
                    if (row < p.M && colg < p.N) *(float4*)((float*)p.Y + row * p.ldy + colg) = v;
                }
            }
        }
        return;
    }
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int64_t row = m0 + wm * 128 + i * 16 + (lane & 15);
        if (row >= p.M) continue;
#pragma unroll
        for (int j = 0; j < 4; ++j) store_four(p, row, col0 + j * 16, outputs(i, j));
    }
}

template <int BA, int BW>
hipError_t launch_big(const GemmParams& p, hipStream_t stream) {
    static std::atomic<uint64_t> attr{0};
    const size_t smem = (size_t)LDS2_BYTES + (BA == 6 ? 64 * sizeof(uint32_t) : 0);
    const hipError_t e = raise_lds_limit((const void*)lut_gemm_big<BA, BW>, (int)smem, attr);
    if (e != hipSuccess) return e;
    const int ntm = (int)((p.M + BM2 - 1) / BM2), ntn = (int)((p.N + BN2 - 1) / BN2);
    const int per_xcd = (ntm * ntn + 7) / 8;
    hipLaunchKernelGGL((lut_gemm_big<BA, BW>), dim3(per_xcd * 8), dim3(512), smem, stream, p, ntm, ntn, per_xcd);
    return hipGetLastError();
}

// The K-splits' sums in split order (deterministic), rescaled and through the layer epilogue:
// one thread per four consecutive outputs of a row.
__global__ __launch_bounds__(256) void lut_gemm_reduce(GemmParams p, int splits) {
    const int64_t nq = (p.N + 3) / 4;
    const int64_t t = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (t >= p.M * nq) return;
    const int64_t row = t / nq, c0 = (t - row * nq) * 4;
    const float xs = p.xn[row];
    if (p.vec4 && (p.N & 3) == 0) {
        // whole runs of four, 16-byte aligned in the workspace and in Y: vector loads and stores
        const int64_t plane = p.M * p.N;
        const float* src = p.ws + row * p.N + c0;
        float4 a = make_float4(0.f, 0.f, 0.f, 0.f);
        for (int z = 0; z < splits; ++z) {
            const float4 b = *(const float4*)(src + z * plane);
            a.x += b.x;
            a.y += b.y;
            a.z += b.z;
            a.w += b.w;
        }
        const uint2 rw = *(const uint2*)(p.wn + c0);
        const uint2 bb = p.bias ? *(const uint2*)(p.bias + c0) : make_uint2(0u, 0u);
        float v[4] = {a.x * xs * __uint_as_float(rw.x << 16), a.y * xs * __uint_as_float(rw.x & 0xFFFF0000u),
                      a.z * xs * __uint_as_float(rw.y << 16), a.w * xs * __uint_as_float(rw.y & 0xFFFF0000u)};
        v[0] = epilogue_value(p, v[0], __uint_as_float(bb.x << 16));
        v[1] = epilogue_value(p, v[1], __uint_as_float(bb.x & 0xFFFF0000u));
        v[2] = epilogue_value(p, v[2], __uint_as_float(bb.y << 16));
        v[3] = epilogue_value(p, v[3], __uint_as_float(bb.y & 0xFFFF0000u));
        if (p.out_bf16)
            *(uint2*)((uint16_t*)p.Y + row * p.ldy + c0) =
                make_uint2(f32_to_bf16_rne(v[0]) | (f32_to_bf16_rne(v[1]) << 16),
                           f32_to_bf16_rne(v[2]) | (f32_to_bf16_rne(v[3]) << 16));
        else
            *(float4*)((float*)p.Y + row * p.ldy + c0) = make_float4(v[0], v[1], v[2], v[3]);
        return;
    }
    const int nc = (int)min((int64_t)4, p.N - c0);
    float v[4] = {0.f, 0.f, 0.f, 0.f};
    for (int z = 0; z < splits; ++z) {
        const float* src = p.ws + (int64_t)z * p.M * p.N + row * p.N + c0;
#pragma unroll
        for (int r = 0; r < 4; ++r)
            if (r < nc) v[r] += src[r];
    }
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        if (r >= nc) continue;
        const int64_t col = c0 + r;
        const float out = epilogue_value(p, v[r] * xs * bf16_to_f32(p.wn[col]), p.bias ? bf16_to_f32(p.bias[col]) : 0.f);
        store_one(p, row, col, out);
    }
}

// The kernel for rows that do not fill the device with large tiles, by an estimate of each one's
// microseconds.  Fitted to 1600 layers timed on all three (M 1 .. 8000, N 96 .. 18432, K 256 .. 16384, every
// bit pair, 256 compute units): nine in ten estimates within 13%, and where rows are not stored in
// vectors (N no multiple of 4) four in five within 15%.  The row stride of Y does not enter, so that a
// layer's outputs are the same bits wherever they are written.  The choice costs 0.1% over the fastest
// kernel on average, 25% at worst; 6 of 2986 calls (each layer with a workspace and without) are over 3%
// slower than on 128 x 128 tiles, the worst 9%.  A tie stays on the 128 x 128 kernel.
enum class Kernel { kSmall, kWave, kLarge };

Kernel fastest_kernel(int64_t M, int64_t N, int64_t K, int ba, int bw, int splits, int split_steps, int cus) {
    auto tiles = [&](int64_t bm, int64_t bn) { return ((M + bm - 1) / bm) * ((N + bn - 1) / bn); };
    // decode cost relative to 4-bit codes, per operand: 1.3 at 3 bits, 1.85 at 6
    auto cost = [](int b) { return b == 3 ? 1.3 : b == 6 ? 1.85 : 1.0; };
    const double f = 0.5 * (cost(ba) + cost(bw)), steps = (double)(K / BK);
    const bool vectors = N % 4 == 0;
    // 128 x 128: k co-resident workgroups per compute unit take 0.58, 1.03, 1.64 and 2.13 us per K-step
    // for k = 1 .. 4, 0.48 us each beyond.  A split costs the reduction 0.23 us (its threads walk the
    // splits one by one) and its sums' round trip at 5.3 TB/s; element by element, 0.49 us and 1.7
    // TB/s (156 x 385 x 13824 W4A4 in 31 splits: 44.8 us, 18.0 on wave tiles).  Without a split, stores element by
    // element add 9 us for each further workgroup.
    const int64_t wgs = tiles(BM, BN) * splits, k = (wgs + cus - 1) / cus;
    const double step = k == 1 ? 0.58 : k == 2 ? 1.03 : k == 3 ? 1.64 : k == 4 ? 2.13 : 0.48 * (double)wgs / cus;
    // (beside another workgroup's MFMAs the dearer decodes hide better)
    const double fs = k > 1 ? 1.0 + 0.85 * (f - 1.0) : f;
    const double more = (double)(k - 1), sums = (double)splits * (double)M * (double)N * 8e-6;  // MB
    double best;
    if (splits > 1 && vectors) best = 6.4 + 0.45 * more + step * fs * split_steps + 0.23 * splits + 0.19 * sums;
    else if (splits > 1) best = 7.3 + 0.9 * step * fs * split_steps + 0.49 * splits + 0.6 * sums;
    else best = (vectors ? 6.4 + 0.45 * more : 9.5 + 9.0 * more) + step * fs * steps;
    Kernel kernel = Kernel::kSmall;
    // 256 x 256, one round: 1.27 us per K-step while up to 0.6 of the compute units have a tile, 1.52 us
    // when all do (the clock falls).  4429 x 3072 x 3072 W3A3: 85 us against 129 on 128 x 128 tiles;
    // 4608 x 3072 x 12288 W4A4 280 against 408, 2048 x 5120 x 5120 113 against 138 (135 on wave tiles).
    const int64_t large = tiles(BM2, BN2);
    if (large <= cus && K <= MAX_K2) {
        const double full = std::max(0.0, (double)large / cus - 0.6) / 0.4;
        const double t = (vectors ? 10.0 : 22.0) + steps * (1.27 + 0.25 * full) * (0.5 + 0.5 * f);
        if (t < best) {
            best = t;
            kernel = Kernel::kLarge;
        }
    }
    // wave tiles, whole chunks of 128 only: the busiest compute unit's tiles, 1.2 us for a 64 x 64 one and
    // 0.34 us for each of its chunks (4-bit codes decode a little faster than 2-bit ones there), others 0.3
    // in proportion to their decode.  (Without the cost of a tile, short contractions went here wrongly:
    // 1319 x 5120 x 640 W4A2 27.4 us, 20.2 on 128 x 128 tiles.)
    if (K % 128 == 0 && (M + 15) / 16 <= 65535) {
        const WaveTile w = lut_gemm_wave_tile(M, N, K, cus);
        const double per_cu = (double)((tiles(16 * w.mt, 16 * w.nt) + cus - 1) / cus) * (w.mt + w.nt) / 8.0;
        const bool whole = w.mt == 4 && w.nt == 4;
        const double fw = whole ? f - 0.025 * ((ba == 4) + (bw == 4)) : f;
        const double t = 3.3 + per_cu * ((whole ? 1.2 : 0.0) + (whole ? 0.34 : 0.3) * fw * (double)(K / 128));
        if (t < best) kernel = Kernel::kWave;
    }
    return kernel;
}

template <int BA, int BW>
hipError_t launch_small(const GemmParams& p, hipStream_t stream, int cus) {
    switch (fastest_kernel(p.M, p.N, p.K, BA, BW, p.ws ? p.splits : 1, p.split_steps, cus)) {
        case Kernel::kWave: return launch_lut_gemm_wave(p, BA, BW, cus, stream);
        case Kernel::kLarge: return launch_big<BA, BW>(p, stream);
        default: break;
    }
    dim3 grid((unsigned)((p.N + BN - 1) / BN), (unsigned)((p.M + BM - 1) / BM));
    const size_t smem = (size_t)2 * 2 * SMALL_TILE * sizeof(__bf16) + (BA == 6 ? 64 * sizeof(uint32_t) : 0);
    static std::atomic<uint64_t> attr_split{0}, attr_whole{0};
    if (p.ws && p.splits > 1) {
        const hipError_t ea = raise_lds_limit((const void*)lut_gemm_kernel<BA, BW, true>, (int)smem, attr_split);
        if (ea != hipSuccess) return ea;
        grid.z = (unsigned)p.splits;
        hipLaunchKernelGGL((lut_gemm_kernel<BA, BW, true>), grid, dim3(256), smem, stream, p);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
        const int64_t threads = p.M * ((p.N + 3) / 4);
        hipLaunchKernelGGL(lut_gemm_reduce, dim3((unsigned)((threads + 255) / 256)), dim3(256), 0, stream, p, p.splits);
        return hipGetLastError();
    }
    const hipError_t ew = raise_lds_limit((const void*)lut_gemm_kernel<BA, BW, false>, (int)smem, attr_whole);
    if (ew != hipSuccess) return ew;
    hipLaunchKernelGGL((lut_gemm_kernel<BA, BW, false>), grid, dim3(256), smem, stream, p);
    return hipGetLastError();
}

// Rows m0 .. M-1 of the layer as a layer of their own (operands and output shifted by m0 rows).
inline GemmParams rows_from(const GemmParams& p, int64_t m0, int ba) {
    GemmParams q = p;
    q.xc = p.xc + m0 * ((int64_t)p.K * ba / 8);
    q.xn = p.xn + m0;
    q.Y = (char*)p.Y + m0 * p.ldy * (p.out_bf16 ? 2 : 4);
    q.M = p.M - m0;
    return q;
}

template <int BA, int BW>
hipError_t launch_one(const GemmParams& p, hipStream_t stream, int cus) {
    const int64_t m_big = lut_gemm_big_rows(p.M, p.N, p.K, cus);
    if (m_big == 0) return launch_small<BA, BW>(p, stream, cus);
    if (m_big == p.M) return launch_big<BA, BW>(p, stream);
    GemmParams head = p;
    head.M = m_big;
    hipError_t e = launch_big<BA, BW>(head, stream);
    if (e != hipSuccess) return e;
    return launch_small<BA, BW>(rows_from(p, m_big, BA), stream, cus);
}

}  // namespace

int64_t lut_gemm_big_rows(int64_t M, int64_t N, int64_t K, int cus) {
    // the large kernel from one 256x256 tile per compute unit up (measured: at 432 tiles on 256
    // compute units it beats the 128x128 kernel by a quarter, despite its half-empty second round)
    const int64_t ntm = (M + BM2 - 1) / BM2, ntn = (N + BN2 - 1) / BN2, tiles = ntm * ntn;
    // (its 32-bit code offsets cover rows up to MAX_K2 inputs)
    if (tiles < (int64_t)cus || K > MAX_K2) return 0;
    // Wave quantization: the large kernel runs one tile per compute unit at a time, so a last round
    // that is only partly full costs as long as a full one (c4's down-projection: 2600 tiles, an
    // eleventh round of 40).  When that pays, the large kernel takes the tile rows that fill its
    // full rounds and another kernel the rest, priced here as 128x128 tiles (fastest_kernel may find a
    // faster one).  A round of those does a quarter of a large tile's work per workgroup but, with
    // one workgroup per compute unit, is latency-bound and takes 0.6-0.8 of a large round (c4's down-projection: 4.61 -> 4.53 ms; the up-projection,
    // whose last round is 42% full, is left alone).
    const int64_t rows_big = (tiles / cus) * cus / ntn;
    if (rows_big > 0 && rows_big < ntm) {
        const int64_t m0 = rows_big * BM2;
        const int64_t small_wgs = ((M - m0 + BM - 1) / BM) * ((N + BN - 1) / BN);
        const double whole = (double)((tiles + cus - 1) / cus);
        const double split = (double)((rows_big * ntn + cus - 1) / cus) + 0.6 * (double)((small_wgs + cus - 1) / cus);
        if (split + 0.1 < whole) return m0;
    }
    return M;
}

int lut_gemm_small_splits(int64_t M, int64_t N, int64_t K, int cus, int* split_steps) {
    const int nk = (int)(K / BK);
    *split_steps = nk;
    // The 128x128 workgroups are each one K-step chain that is latency-bound.  The count of splits
    // minimises an estimate of the busiest compute unit's time, in K-steps: k co-resident
    // workgroups of `steps` K-steps take w(k) * steps (measured on 256 compute units: 1, 1.66 and
    // 2.58 for k = 1, 2, 3, then about 0.86 k), plus the partial sums' round trip through the
    // workspace at about 7 MB per K-step's time.  At least 4 K-steps per split, at most 64 splits.
    const int64_t wgs = ((M + BM - 1) / BM) * ((N + BN - 1) / BN);
    auto busiest = [&](int splits, int steps) {
        const int64_t k = (wgs * splits + cus - 1) / cus;
        return (k == 1 ? 1.0 : k == 2 ? 1.66 : k == 3 ? 2.58 : 0.86 * (double)k) * steps;
    };
    int best_splits = 1, best_steps = nk;
    double best = busiest(1, nk);
    for (int s = 2; s <= std::min(64, nk / 4); ++s) {
        const int steps = (nk + s - 1) / s, splits = (nk + steps - 1) / steps;
        const double cost = busiest(splits, steps) + (double)splits * (double)M * (double)N * 8.0 / 7.0e6;
        if (cost < best) {
            best = cost;
            best_splits = splits;
            best_steps = steps;
        }
    }
    *split_steps = best_steps;
    return best_splits;
}

hipError_t launch_lut_gemm(const GemmParams& p, int ba, int bw, int cus, hipStream_t stream) {
    switch (ba * 8 + bw) {
        case 2 * 8 + 2: return launch_one<2, 2>(p, stream, cus);
        case 2 * 8 + 3: return launch_one<2, 3>(p, stream, cus);
        case 2 * 8 + 4: return launch_one<2, 4>(p, stream, cus);
        case 3 * 8 + 2: return launch_one<3, 2>(p, stream, cus);
        case 3 * 8 + 3: return launch_one<3, 3>(p, stream, cus);
        case 3 * 8 + 4: return launch_one<3, 4>(p, stream, cus);
        case 6 * 8 + 2: return launch_one<6, 2>(p, stream, cus);
        case 6 * 8 + 3: return launch_one<6, 3>(p, stream, cus);
        case 6 * 8 + 4: return launch_one<6, 4>(p, stream, cus);
        case 4 * 8 + 2: return launch_one<4, 2>(p, stream, cus);
        case 4 * 8 + 3: return launch_one<4, 3>(p, stream, cus);
        default: return launch_one<4, 4>(p, stream, cus);
    }
}

}  // namespace orbit
