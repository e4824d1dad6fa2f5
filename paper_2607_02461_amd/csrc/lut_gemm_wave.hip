// LUT-decode GEMM for grids too small for the block-tile kernels: one output tile of at most 64 x 64
// per workgroup, its contraction split over the workgroup's waves.
//
// Such a layer is a chain of latencies: on 128 x 128 tiles 256 x 3072 outputs are 48 workgroups, and
// splitting K over workgroups to fill the device costs a round trip of the partial sums through
// memory and a second launch.  Here every wave contracts its own chunks of K, decodes both operands
// straight into MFMA fragments (no LDS and no barrier in the loop, so waves never wait for each
// other) and the partial sums meet once, in LDS, in wave order (deterministic).  The price is that
// the decode is not shared: 14 (mt + nt) VALU operations of decode (4-bit codes) go with mt nt MFMAs, and
// the VALU bounds it (4 x 4 tiles: 700-800 TFLOP/s once the device is full, against 1340 for
// the large kernel).  Loads are 16-byte vectors of 32 codes (at 4 bits), one or two chunks ahead.
//
// Measured (W4A4, device time; before: the 128 x 128 kernel, split over K with a workspace | without):
//     1 x 3072 x 3072 (M x N x K)   12.0 | 33.3 -> 4.6 us     16 x 13824 x 5120   32.8 | 52.8 -> 11.1
//     256 x 3072 x 3072             22.8 | 34.4 -> 13.0       512 x 9216 x 3072   62.5 | 53.3 -> 47.8
//     1024 x 5120 x 5120            92.8 | 83.9 -> 73.4       1560 x 5120 x 5120   137 | 136 -> 111
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <algorithm>

#include "device.h"
#include "lut_decode.h"

namespace orbit {

namespace {

constexpr int KC = 128;    // inputs per chunk: 32 codes of a row per lane
constexpr int kWaves = 8;  // at most, of a workgroup

template <int BA, int BW, int MT, int NT, int DEPTH>
__global__ __launch_bounds__(64 * kWaves) void lut_gemm_wave(GemmParams p) {
    extern __shared__ __align__(16) unsigned char lds[];  // [wave][16 MT][16 NT + 4] fp32 sums; then the 6-bit table
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6), waves = (int)blockDim.x >> 6;
    const int64_t m0 = (int64_t)blockIdx.y * (16 * MT), n0 = (int64_t)blockIdx.x * (16 * NT);
    constexpr int TS = 16 * NT + 4;
    const ByteTables ta = make_tables<BA>(p.lut_a);
    const ByteTables tw = make_tables<BW>(p.lut_w);
    Decode8<BA> da;
    Decode8<BW> db;
    if constexpr (BA == 6) {
        uint32_t* const tab6 = (uint32_t*)((float*)lds + (size_t)waves * (16 * MT * TS));
        if (tid < 64) tab6[tid] = p.lut_a[tid];
        __syncthreads();
        da.tab = tab6;
    }

    // Lane l holds, of row l % 16 of every 16-row tile, the 32 codes l / 16 of a chunk: one vector
    // load.  MFMA m of the chunk contracts code groups 8m .. 8m+7 of the four lane groups, the same
    // inputs on both sides.
    const uint8_t* asrc[MT];
    const uint8_t* bsrc[NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
        asrc[i] = p.xc + min(m0 + 16 * i + (lane & 15), p.M - 1) * ((int64_t)p.K * BA / 8) + (lane >> 4) * 4 * BA;
#pragma unroll
    for (int j = 0; j < NT; ++j)
        bsrc[j] = p.wc + min(n0 + 16 * j + (lane & 15), p.N - 1) * ((int64_t)p.K * BW / 8) + (lane >> 4) * 4 * BW;

    floatx4 acc[MT][NT];
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = floatx4{0.f, 0.f, 0.f, 0.f};

    // this wave's chunks: wave, wave + waves, ...; DEPTH of them in flight
    const int nc = (p.K / KC - wave + waves - 1) / waves;
    Codes<BA> sa[DEPTH][MT];
    Codes<BW> sb[DEPTH][NT];
    auto load = [&](int c, Codes<BA> (&ca)[MT], Codes<BW> (&cb)[NT]) {
        const int64_t k = (int64_t)(wave + c * waves) * KC;
#pragma unroll
        for (int j = 0; j < NT; ++j) load_codes32<BW>(bsrc[j] + k * BW / 8, cb[j]);
#pragma unroll
        for (int i = 0; i < MT; ++i) load_codes32<BA>(asrc[i] + k * BA / 8, ca[i]);
    };
    auto contract = [&](const Codes<BA> (&ca)[MT], const Codes<BW> (&cb)[NT]) {
#pragma unroll
        for (int m = 0; m < 4; ++m) {
            bf16x8 a[MT], b[NT];
#pragma unroll
            for (int j = 0; j < NT; ++j) b[j] = __builtin_bit_cast(bf16x8, decode_all(db, cb[j], m, tw));
#pragma unroll
            for (int i = 0; i < MT; ++i) a[i] = __builtin_bit_cast(bf16x8, decode_all(da, ca[i], m, ta));
#pragma unroll
            for (int i = 0; i < MT; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    acc[i][j] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(b[j], a[i], acc[i][j], 0, 0, 0);
        }
    };
#pragma unroll
    for (int u = 0; u < DEPTH; ++u)
        if (u < nc) load(u, sa[u], sb[u]);
    for (int c = 0; c < nc; c += DEPTH) {
#pragma unroll
        for (int u = 0; u < DEPTH; ++u) {
            if (c + u >= nc) break;
            contract(sa[u], sb[u]);
            if (c + u + DEPTH < nc) load(c + u + DEPTH, sa[u], sb[u]);
        }
    }

    // element e of accumulator (i, j) belongs to row 16 i + lane % 16, column 16 j + 4 (lane / 16) + e
    float* const part = (float*)lds + (size_t)wave * (16 * MT * TS);
#pragma unroll
    for (int i = 0; i < MT; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
            *(floatx4*)(part + (16 * i + (lane & 15)) * TS + 16 * j + 4 * (lane >> 4)) = acc[i][j];
    __syncthreads();
    // the waves' sums in wave order, then the layer's epilogue
    for (int t = tid; t < 16 * MT * 4 * NT; t += blockDim.x) {
        const int r = t / (4 * NT), c4 = 4 * (t % (4 * NT));
        const int64_t row = m0 + r, c = n0 + c4;
        if (row >= p.M || c >= p.N) continue;
        uint2 rw, bias;
        load_columns(p, c, rw, bias);
        const float xs = p.xn[row];
        const float* src = (const float*)lds + r * TS + c4;
        floatx4 v = *(const floatx4*)src;
        for (int w = 1; w < waves; ++w) v += *(const floatx4*)(src + (size_t)w * (16 * MT * TS));
        v[0] = epilogue_value(p, v[0] * xs * __uint_as_float(rw.x << 16), __uint_as_float(bias.x << 16));
        v[1] = epilogue_value(p, v[1] * xs * __uint_as_float(rw.x & 0xFFFF0000u), __uint_as_float(bias.x & 0xFFFF0000u));
        v[2] = epilogue_value(p, v[2] * xs * __uint_as_float(rw.y << 16), __uint_as_float(bias.y << 16));
        v[3] = epilogue_value(p, v[3] * xs * __uint_as_float(rw.y & 0xFFFF0000u), __uint_as_float(bias.y & 0xFFFF0000u));
        store_four(p, row, c, v);
    }
}

template <int BA, int BW, int MT, int NT, int DEPTH>
hipError_t launch_tile(const GemmParams& p, int waves, hipStream_t stream) {
    static std::atomic<uint64_t> attr{0};
    const size_t smem = (size_t)waves * (16 * MT) * (16 * NT + 4) * sizeof(float) + (BA == 6 ? 64 * sizeof(uint32_t) : 0);
    if (smem > 64 * 1024) {
        const hipError_t e = raise_lds_limit((const void*)lut_gemm_wave<BA, BW, MT, NT, DEPTH>, 160 * 1024, attr);
        if (e != hipSuccess) return e;
    }
    const dim3 grid((unsigned)((p.N + 16 * NT - 1) / (16 * NT)), (unsigned)((p.M + 16 * MT - 1) / (16 * MT)));
    hipLaunchKernelGGL((lut_gemm_wave<BA, BW, MT, NT, DEPTH>), grid, dim3(64 * waves), smem, stream, p);
    return hipGetLastError();
}

template <int BA, int BW>
hipError_t launch_wave(const GemmParams& p, const WaveTile& t, hipStream_t stream) {
    if (t.mt == 1) {
        if (t.nt == 1) return launch_tile<BA, BW, 1, 1, 2>(p, t.waves, stream);
        return launch_tile<BA, BW, 1, 4, 2>(p, t.waves, stream);
    }
    if (t.mt == 2) {
        if (t.nt == 2) return launch_tile<BA, BW, 2, 2, 2>(p, t.waves, stream);
        // two chunks of 6-bit codes in flight, beside 3- or 4-bit ones, are over 128 registers: spills with two
        // workgroups on a compute unit, or only one there (128 x 3072 x 3072 W4A6: 16.7 us spilling, 13.2
        // alone, 12.5 with one chunk; 128 x 5120 x 1536: 16.2, 16.3, 11.3).  Beside 2-bit codes two fit (118
        // registers; 18 x 12288 x 12288 W2A6: 33.3 us, 35.7 with one).
        return launch_tile<BA, BW, 2, 4, (BA == 6 && BW > 2) ? 1 : 2>(p, t.waves, stream);
    }
    if (t.waves > 4) return launch_tile<BA, BW, 4, 4, 1>(p, t.waves, stream);
    return launch_tile<BA, BW, 4, 4, 2>(p, t.waves, stream);
}

}  // namespace

WaveTile lut_gemm_wave_tile(int64_t M, int64_t N, int64_t K, int cus) {
    auto tiles = [&](int mt, int nt) { return ((M + 16 * mt - 1) / (16 * mt)) * ((N + 16 * nt - 1) / (16 * nt)); };
    // The largest tile that still gives 0.7 workgroups per compute unit, with no more than half of its
    // rows empty; the smallest for its row count otherwise.  Decode per flop falls with the tile, but
    // idle compute units cost more: 128 x 3072 outputs take 9.4 us as 192 tiles of 32 x 64 and over
    // 10 as 96 of 64 x 64.  Eight waves share a tile: they are what hides the load latency when the
    // compute unit has no second tile; with more than one 64 x 64 tile per compute unit, four (K = 3072:
    // 256 x 3072, 192 tiles, 12.7 us with eight and 14.2 with four; 512 x 3072, 384 tiles, 23.1 and 21.5).
    WaveTile t{1, 1, kWaves};
    const int64_t want = (int64_t)cus * 7 / 10;
    if (M > 32 && tiles(4, 4) >= want) t = WaveTile{4, 4, tiles(4, 4) <= cus ? kWaves : kWaves / 2};
    else if (M > 16) t = WaveTile{2, tiles(2, 4) >= want ? 4 : 2, kWaves};
    else if (tiles(1, 4) >= want) t = WaveTile{1, 4, kWaves};
    t.waves = (int)std::min<int64_t>(t.waves, K / KC);
    return t;
}

hipError_t launch_lut_gemm_wave(const GemmParams& p, int ba, int bw, int cus, hipStream_t stream) {
    const WaveTile t = lut_gemm_wave_tile(p.M, p.N, p.K, cus);
    switch (ba * 8 + bw) {
        case 2 * 8 + 2: return launch_wave<2, 2>(p, t, stream);
        case 2 * 8 + 3: return launch_wave<2, 3>(p, t, stream);
        case 2 * 8 + 4: return launch_wave<2, 4>(p, t, stream);
        case 3 * 8 + 2: return launch_wave<3, 2>(p, t, stream);
        case 3 * 8 + 3: return launch_wave<3, 3>(p, t, stream);
        case 3 * 8 + 4: return launch_wave<3, 4>(p, t, stream);
        case 6 * 8 + 2: return launch_wave<6, 2>(p, t, stream);
        case 6 * 8 + 3: return launch_wave<6, 3>(p, t, stream);
        case 6 * 8 + 4: return launch_wave<6, 4>(p, t, stream);
        case 4 * 8 + 2: return launch_wave<4, 2>(p, t, stream);
        case 4 * 8 + 3: return launch_wave<4, 3>(p, t, stream);
        default: return launch_wave<4, 4>(p, t, stream);
    }
}

}  // namespace orbit
