// INT4 round-to-nearest weight-only layer of the AdaLN modulation projections, for gfx950.
//
// The experimental setup (Sec. 5) keeps the adaptive-layer-norm modulation projections at INT4
// weight round-to-nearest, and the supplementary material fixes group size 64 with BF16
// activations: those layers are not rotated, because their timestep-dependent scale-and-shift
// cannot be folded into neighbouring weights and their input is one conditioning token per step.
//
// Offline: each group of 64 consecutive inputs of a weight row gets the FP16 scale
// fp16(absmax / 7) (the FP32 quotient rounded to nearest even, saturating at the largest finite
// FP16) and codes clamp(RNE(w / scale), -8, 7), the quotient in FP32; codes are stored as q + 8
// in LSB-first nibbles.
//
// Online: Y = X (q * scale)^T (+ bias) for a handful of BF16 rows of X.  The layer streams its
// weights once, so it is bound by HBM and, a few microseconds long per projection, by how much
// of it is in flight.  A code nibble u becomes the BF16 value 128 + u by OR-ing it into
// the mantissa of 128 (0x4300 | u is exact: 128..143 are BF16 integers), two per register at
// bits 0 and 16, so one v_dot2_f32_bf16 takes two codes against two activations with exact
// products; per chunk the accumulator starts at -136 * sum(x), which removes the 128 + 8 offset.
// The activations of a chunk are paired to match: element j of each 8 with element j + 4.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.h"

namespace orbit {

namespace {

typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

constexpr int kRtnGroup = 64;

__device__ __forceinline__ float bf16_lo(uint32_t w) { return __uint_as_float(w << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t w) { return __uint_as_float(w & 0xFFFF0000u); }

__device__ __forceinline__ float dot2(uint32_t a, uint32_t b, float c) {
    return __builtin_amdgcn_fdot2_f32_bf16(__builtin_bit_cast(bf16x2, a), __builtin_bit_cast(bf16x2, b), c, false);
}

// One thread per group of 64 weights: 128 bytes in, 32 bytes of codes and one FP16 scale out.
__global__ __launch_bounds__(256) void adaln_int4_quantize_kernel(const uint16_t* __restrict__ W, int64_t N, int K,
                                                                  int64_t ldw, uint8_t* __restrict__ q,
                                                                  uint16_t* __restrict__ scales) {
    const int groups = K / kRtnGroup;
    const int64_t gid = (int64_t)blockIdx.x * blockDim.x + threadIdx.x;
    if (gid >= N * groups) return;
    const int64_t n = gid / groups;
    const int g = (int)(gid - n * groups);
    const uint4* src = (const uint4*)(W + n * ldw + (int64_t)g * kRtnGroup);
    uint32_t w[32];
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const uint4 v = src[i];
        w[4 * i] = v.x;
        w[4 * i + 1] = v.y;
        w[4 * i + 2] = v.z;
        w[4 * i + 3] = v.w;
    }
    float amax = 0.f;
#pragma unroll
    for (int j = 0; j < 32; ++j) amax = fmaxf(amax, fmaxf(fabsf(bf16_lo(w[j])), fabsf(bf16_hi(w[j]))));
    const _Float16 sh = (_Float16)fminf(amax / 7.0f, 65504.0f);  // IEEE fp32 quotient, then RNE to fp16
    const float s = (float)sh;
    uint32_t out[8];
#pragma unroll
    for (int t = 0; t < 8; ++t) {
        uint32_t word = 0;
#pragma unroll
        for (int e = 0; e < 8; ++e) {
            const uint32_t src_w = w[4 * t + (e >> 1)];
            const float v = (e & 1) ? bf16_hi(src_w) : bf16_lo(src_w);
            float r = s > 0.f ? rintf(v / s) : 0.f;  // IEEE quotient, round half to even
            r = fminf(fmaxf(r, -8.f), 7.f);
            word |= (uint32_t)((int)r + 8) << (4 * e);
        }
        out[t] = word;
    }
    uint4* dst = (uint4*)(q + n * (int64_t)(K / 2) + (int64_t)g * (kRtnGroup / 2));
    dst[0] = make_uint4(out[0], out[1], out[2], out[3]);
    dst[1] = make_uint4(out[4], out[5], out[6], out[7]);
    scales[n * groups + g] = __builtin_bit_cast(uint16_t, sh);
}

template <int CTRL>
__device__ __forceinline__ float dpp_add(float v) {
    return v + __int_as_float(__builtin_amdgcn_mov_dpp(__float_as_int(v), CTRL, 0xF, 0xF, true));
}

// A workgroup of 256 threads is 16 groups of 16 lanes, ROWS rows of Y each; a lane takes every sixteenth
// chunk (32 codes) of its rows and has the loads of up to six of them in flight, all of a row up to
// K = 3072.  One projection is 29 MB and a few microseconds, so what counts for one token is the chain of
// latencies in front of the last byte: the weights' loads are issued right behind the tokens' and before
// anything waits for those, the chunk sums come out of the staging registers (no second barrier), and one
// row per group spreads 18432 rows over 4.5 workgroups per compute unit.  Measured, device time of a call in
// a sequence, against two rows per group staged ahead of the loads: 1 x 3072 -> 18432 9.7 -> 8.1 us (3.7
// TB/s), 9216 rows 6.9 -> 5.5, 1 x 5120 -> 60001 33.4 -> 29.5, 1 x 3072 -> 1050624 320 -> 313 (5.5 TB/s).
//
// Several tokens are bound by the token vectors' LDS reads and the dot products instead: two rows per
// group read each vector once for both (16 x 3072 -> 18432 43.2 -> 37.6 us).  The launchers below have the
// choice and its figures.
constexpr int kRtnLanes = 16;
constexpr int rtn_block_rows(int rows) { return 16 * rows; }

// Persistent: a workgroup stages its tokens once, then walks row blocks blockIdx.x, +gridDim.x, ...
template <int MT, int ROWS>
__global__ __launch_bounds__(256) void adaln_int4_linear_kernel(RtnLinearParams p) {
    // The workgroup's MT tokens, paired per 8 as (x0,x4) (x1,x5) (x2,x6) (x3,x7): 16-byte vector t of
    // chunk c sits at t * nchunk + c, so that 16 lanes reading 16 chunks read 256 contiguous bytes
    // (chunk by chunk their vectors would be 64 bytes apart, four to a bank).  Then one fp32 sum per chunk.
    constexpr int kRtnBlockRows = rtn_block_rows(ROWS), kRtnBatch = 6 / ROWS;
    extern __shared__ __align__(16) uint4 xlds[];
    const int nchunk = p.K / 32, nvec = p.K / 8;
    float* const csum = (float*)(xlds + MT * nvec);
    const int m0 = blockIdx.y * MT;
    const uint32_t magic = 0x43004300u, one_one = 0x3F803F80u;

    auto token_load = [&](int i) {
        const int m = i / nvec, v = i - m * nvec;
        return *(const uint4*)(p.X + (int64_t)min(m0 + m, (int)p.M - 1) * p.ldx + (int64_t)v * 8);
    };
    // i runs over whole quads of lanes (nvec is a multiple of 8), one chunk each
    auto token_store = [&](int i, const uint4& v) {
        const int m = i / nvec, j = i - m * nvec;
        float sum = dot2(v.w, one_one, dot2(v.z, one_one, dot2(v.y, one_one, dot2(v.x, one_one, 0.f))));
        sum = dpp_add<0xB1>(sum);  // quad_perm [1,0,3,2]
        sum = dpp_add<0x4E>(sum);  // quad_perm [2,3,0,1]
        xlds[m * nvec + (j & 3) * nchunk + (j >> 2)] =
            make_uint4(__builtin_amdgcn_perm(v.z, v.x, 0x05040100u), __builtin_amdgcn_perm(v.z, v.x, 0x07060302u),
                       __builtin_amdgcn_perm(v.w, v.y, 0x05040100u), __builtin_amdgcn_perm(v.w, v.y, 0x07060302u));
        if ((j & 3) == 0) csum[m * nchunk + (j >> 2)] = sum;
    };

    const int lane = threadIdx.x & (kRtnLanes - 1), grp = threadIdx.x / kRtnLanes;
    const uint32_t qrow = p.K / 2, srow = p.K / kRtnGroup * 2;  // bytes
    const uint32_t qoff = grp * ROWS * qrow + lane * 16, soff = grp * ROWS * srow + (lane >> 1) * 2;
    const int64_t nblocks = (p.N + kRtnBlockRows - 1) / kRtnBlockRows;
    u32x4 cw[kRtnBatch][ROWS];
    uint16_t sc[kRtnBatch][ROWS];
    // A batch's loads, through its block's rows as a buffer: rows past the last one read zero, chunks
    // past a row's end the next row's (dropped below), and no address is formed per load.
    struct Batch {
        __amdgpu_buffer_rsrc_t q, s;
        int c0, slots;  // first chunk, slots of 16 chunks (uniform)
    };
    auto batch_at = [&](int64_t blk, int c0) {
        Batch t;
        const int64_t n0 = blk * kRtnBlockRows;
        const int rows = (int)min((int64_t)kRtnBlockRows, p.N - n0);
        t.q = __builtin_amdgcn_make_buffer_rsrc((void*)(p.q + n0 * qrow), 0, rows * (int)qrow, 0x00027000);
        t.s = __builtin_amdgcn_make_buffer_rsrc((void*)((const uint8_t*)p.scales + n0 * srow), 0, rows * (int)srow, 0x00027000);
        t.c0 = c0;
        t.slots = min(kRtnBatch, (nchunk - c0 + kRtnLanes - 1) / kRtnLanes);
        return t;
    };
    auto weight_load = [&](const Batch& t, int b) {
        if (b < t.slots) {
#pragma unroll
            for (int r = 0; r < ROWS; ++r) {
                cw[b][r] = __builtin_amdgcn_raw_buffer_load_b128(t.q, qoff + r * qrow + 256 * b, t.c0 * 16, 0);
                sc[b][r] = __builtin_amdgcn_raw_buffer_load_b16(t.s, soff + r * srow + 16 * b, t.c0, 0);
            }
        }
    };

    const int total = MT * nvec, i1 = threadIdx.x + 256;
    uint4 v0 = make_uint4(0u, 0u, 0u, 0u), v1 = v0;
    if ((int)threadIdx.x < total) v0 = token_load(threadIdx.x);
    if (i1 < total) v1 = token_load(i1);
    Batch cur = batch_at(blockIdx.x, 0);
#pragma unroll
    for (int b = 0; b < kRtnBatch; ++b) weight_load(cur, b);
    if ((int)threadIdx.x < total) token_store(threadIdx.x, v0);
    if (i1 < total) token_store(i1, v1);
    for (int i = threadIdx.x + 512; i < total; i += 256) token_store(i, token_load(i));
    __syncthreads();

    auto contract = [&](int b, int c0, float (&tot)[ROWS][MT]) {
        const int c = c0 + lane + kRtnLanes * b, cc = min(c, nchunk - 1);
        float acc[ROWS][MT];
#pragma unroll
        for (int m = 0; m < MT; ++m) {
            const float v = -136.f * csum[m * nchunk + cc];
#pragma unroll
            for (int r = 0; r < ROWS; ++r) acc[r][m] = v;
        }
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            uint32_t u[ROWS][4];  // (128 + u_j, 128 + u_{j+4}) of 8 codes, as BF16 pairs
#pragma unroll
            for (int r = 0; r < ROWS; ++r)
#pragma unroll
                for (int j = 0; j < 4; ++j) u[r][j] = ((cw[b][r][t] >> (4 * j)) & 0x000F000Fu) | magic;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                const uint4 x = xlds[m * nvec + t * nchunk + cc];
#pragma unroll
                for (int r = 0; r < ROWS; ++r) {
                    acc[r][m] = dot2(u[r][0], x.x, acc[r][m]);
                    acc[r][m] = dot2(u[r][1], x.y, acc[r][m]);
                    acc[r][m] = dot2(u[r][2], x.z, acc[r][m]);
                    acc[r][m] = dot2(u[r][3], x.w, acc[r][m]);
                }
            }
        }
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const float s = (float)__builtin_bit_cast(_Float16, sc[b][r]);
#pragma unroll
            for (int m = 0; m < MT; ++m) tot[r][m] = c < nchunk ? fmaf(s, acc[r][m], tot[r][m]) : tot[r][m];
        }
    };
    for (int64_t blk = blockIdx.x; blk < nblocks; blk += gridDim.x) {
        float tot[ROWS][MT];
#pragma unroll
        for (int r = 0; r < ROWS; ++r)
#pragma unroll
            for (int m = 0; m < MT; ++m) tot[r][m] = 0.f;
        for (int c0 = 0; c0 < nchunk; c0 += kRtnLanes * kRtnBatch) {
            if (c0 > 0 || blk != blockIdx.x) {
                cur = batch_at(blk, c0);
#pragma unroll
                for (int b = 0; b < kRtnBatch; ++b) weight_load(cur, b);
            }
#pragma unroll
            for (int b = 0; b < kRtnBatch; ++b) {
                if (c0 + kRtnLanes * b >= nchunk) break;  // uniform: no chunk of this slot exists
                contract(b, c0, tot);
                __builtin_amdgcn_sched_barrier(0);  // one chunk's token reads at a time (registers)
            }
        }

        // fixed-order sum over the 16 lanes of the group (one DPP row): pairs, quads, 8, 16
#pragma unroll
        for (int r = 0; r < ROWS; ++r) {
            const int64_t n = blk * kRtnBlockRows + grp * ROWS + r;
#pragma unroll
            for (int m = 0; m < MT; ++m) {
                float v = tot[r][m];
                v = dpp_add<0xB1>(v);   // quad_perm [1,0,3,2]
                v = dpp_add<0x4E>(v);   // quad_perm [2,3,0,1]
                v = dpp_add<0x141>(v);  // row_half_mirror
                v = dpp_add<0x140>(v);  // row_mirror
                if (lane == 0 && n < p.N && m0 + m < p.M) {
                    if (p.bias) v += __uint_as_float((uint32_t)p.bias[n] << 16);
                    p.Y[(int64_t)(m0 + m) * p.ldy + n] = v;
                }
            }
        }
    }
}

// LDS of a workgroup that stages mt tokens
size_t rtn_lds(int mt, int K) { return (size_t)mt * ((size_t)K / 8 * sizeof(uint4) + (size_t)K / 32 * sizeof(float)); }

int64_t rtn_blocks(int64_t N, int rows) { return (N + rtn_block_rows(rows) - 1) / rtn_block_rows(rows); }

template <int MT, int ROWS>
hipError_t raise_rtn_lds(int K) {
    static std::atomic<uint64_t> attr{0};
    return rtn_lds(MT, K) > 64 * 1024 ? raise_lds_limit((const void*)adaln_int4_linear_kernel<MT, ROWS>, 160 * 1024, attr)
                                      : hipSuccess;
}

// Workgroups walk the row blocks, the same number of blocks each as far as that goes: at most `per_cu` of
// them per compute unit.
struct RtnGrid {
    int64_t workgroups, rounds;
};
RtnGrid rtn_grid(int64_t N, int rows, int per_cu, int cus) {
    const int64_t blocks = rtn_blocks(N, rows), most = (int64_t)per_cu * cus, rounds = (blocks + most - 1) / most;
    return RtnGrid{(blocks + rounds - 1) / rounds, rounds};
}

template <int MT, int ROWS>
hipError_t launch_linear(const RtnLinearParams& p, int per_cu, int cus, hipStream_t stream) {
    const hipError_t e = raise_rtn_lds<MT, ROWS>(p.K);
    if (e != hipSuccess) return e;
    const dim3 grid((unsigned)rtn_grid(p.N, ROWS, per_cu, cus).workgroups, (unsigned)((p.M + MT - 1) / MT));
    hipLaunchKernelGGL((adaln_int4_linear_kernel<MT, ROWS>), grid, dim3(256), rtn_lds(MT, p.K), stream, p);
    return hipGetLastError();
}

// One token: six workgroups per compute unit, where their waves cover each other's latencies.  One row per
// group while that grid is resident at once (3072 -> 18432: 8.1 us, two rows 10.7), or where it splits the
// rows more evenly over the compute units (3072 -> 73728: 21.8 and 22.6); two rows otherwise (5120 ->
// 30720: 18.4 -> 17.8, 8192 -> 65536: 55.4 -> 50.9), and from four workgroups per compute unit on where a
// row's chunks fill at most half of the six loads (512 -> 18432: 4.2 -> 3.7).  Hundreds of thousands of
// rows (a step's projections in one call) want fewer, longer walks: three workgroups per compute unit
// (3072 -> 1050624: 313 us, 320 with six).  Where the token leaves LDS for four workgroups only, two rows
// never pay (16384 -> 30720: 52 us, 59) and longer grids are of four (16384 -> 65536: 119 -> 110).
hipError_t launch_one_token(const RtnLinearParams& p, int cus, hipStream_t stream) {
    const int64_t blocks = rtn_blocks(p.N, 1);
    if (5 * rtn_lds(1, p.K) > 160 * 1024) return launch_linear<1, 1>(p, blocks <= (int64_t)6 * cus ? 6 : 4, cus, stream);
    if (blocks > (int64_t)48 * cus) return launch_linear<1, 2>(p, 3, cus, stream);
    auto busiest = [&](int rows) {  // rows of the busiest compute unit
        const RtnGrid g = rtn_grid(p.N, rows, 6, cus);
        return (g.workgroups + cus - 1) / cus * g.rounds * rtn_block_rows(rows);
    };
    const bool resident = blocks <= (int64_t)(p.K <= 1024 ? 4 : 6) * cus;
    if (resident || (p.K > 1024 && busiest(1) < busiest(2))) return launch_linear<1, 1>(p, 6, cus, stream);
    return launch_linear<1, 2>(p, 6, cus, stream);
}

// Several tokens: two or four a pass over the weights, one row per group of lanes or two, by an estimate in
// microseconds fitted to 900 calls timed all four ways (2 to 100 tokens, N 512 .. 80000, K 512 .. 8192, 256
// compute units): `base`, and per 1024 inputs `load` for each round of resident workgroups and `work` for
// each block of 16 rows on the busiest compute unit.  The choice costs 1% over the fastest of the four on
// average.  Three forms are left out beforehand:
//   - two rows per group where the grid of one row is resident at once, as latencies decide there (4 x 3072 ->
//     12288: 10.1 us, two rows 11.1; 9 x 5120 -> 1993: 10.0 and 10.6);
//   - one row and two tokens where workgroups queue and a call has several passes, or LDS holds fewer than three
//     workgroups (10 x 5120 -> 3182: 16.8 us, two rows 10.8; 13 x 15296 -> 1264: 36.7 and 27.5).  Two tokens, a
//     single pass, go by which form spreads the rows more evenly (2 x 5120 -> 35225: 24.1 us, two rows
//     27.1; -> 37000: 28.9 and 27.4);
//   - four tokens where LDS holds one workgroup of them (16 x 16384 -> 18432: 335 us, two tokens 282).
struct RtnWay {
    int mt, rows, per_cu;     // per_cu: workgroups that a compute unit's registers hold
    double base, load, work;
    hipError_t (*launch)(const RtnLinearParams&, int, int, hipStream_t);
};
constexpr RtnWay kRtnWays[] = {{2, 1, 3, 2.85, 0.35, 0.343, launch_linear<2, 1>},
                               {2, 2, 3, 2.65, 0.40, 0.348, launch_linear<2, 2>},
                               {4, 1, 4, 3.00, 0.62, 0.527, launch_linear<4, 1>},
                               {4, 2, 3, 3.00, 0.62, 0.510, launch_linear<4, 2>}};

hipError_t launch_tokens(const RtnLinearParams& p, int cus, hipStream_t stream) {
    const RtnWay* fastest = nullptr;
    double best = 0.0;
    bool once = false;  // the grid of one row per group is resident at once (each pair's first entry sets it)
    for (const RtnWay& w : kRtnWays) {
        const RtnGrid g = rtn_grid(p.N, w.rows, w.per_cu, cus);
        const int64_t workgroups = g.workgroups * ((p.M + w.mt - 1) / w.mt);
        const int64_t fit = (int64_t)(160 * 1024 / rtn_lds(w.mt, p.K));
        const int64_t resident = std::min<int64_t>(w.per_cu, fit) * cus;
        if (w.rows == 1) once = g.rounds == 1 && workgroups <= resident;
        if (w.mt == 4 && (p.M == 2 || fit < 2)) continue;
        if (w.rows == 2 && once) continue;
        if (w.mt == 2 && w.rows == 1 && !once && (p.M > 2 || fit < 3)) continue;
        const double t = w.base + std::max(p.K, 32 * kRtnLanes) / 1024.0 * (double)g.rounds *
                                      (w.load * (double)((workgroups + resident - 1) / resident) +
                                       w.work * w.rows * (double)((workgroups + cus - 1) / cus));
        if (!fastest || t < best) {
            fastest = &w;
            best = t;
        }
    }
    return fastest->launch(p, fastest->per_cu, cus, stream);
}

}  // namespace

hipError_t launch_adaln_int4_quantize(const uint16_t* W, int64_t N, int K, int64_t ldw, uint8_t* q, uint16_t* scales,
                                      hipStream_t stream) {
    const int64_t total = N * (K / kRtnGroup);
    const int64_t blocks = (total + 255) / 256;
    hipLaunchKernelGGL(adaln_int4_quantize_kernel, dim3((unsigned)blocks), dim3(256), 0, stream, W, N, K, ldw, q,
                       scales);
    return hipGetLastError();
}

hipError_t launch_adaln_int4_linear(const RtnLinearParams& p, int cus, hipStream_t stream) {
    return p.M == 1 ? launch_one_token(p, cus, stream) : launch_tokens(p, cus, stream);
}

}  // namespace orbit
