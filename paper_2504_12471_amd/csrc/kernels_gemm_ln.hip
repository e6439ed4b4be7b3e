// LayerNorm and the product behind it in one launch, for calls of few rows:
//
//   y = LayerNorm(x) * gamma + beta          (kept, with the rows' mean and 1/std, for the backward call)
//   C = epilogue( y B^T )
//
// One image (197 tokens) through the base model, whose QKV and first feed-forward products take this form: 581 -> 521 us; one fp32 block of 260 tokens
// of width 192, forward and backward: 100.9 -> 98.7 us.
//
// What bounds it: latency.  As two launches the norm takes 3.2 us, nearly all of it the way to the first load and back,
// and the product then waits for its first slabs again.  Here a workgroup (32 x 64 or 96 of C) requests everything it will ever
// read as early as its registers allow: its 32 rows of x, gamma and beta, behind them the fragments of B, straight to the
// registers of the wavefront that multiplies with them.  It normalises its rows into LDS, where all of K fits, and
// multiplies.  Each workgroup of a row of tiles normalises the same rows again; the first of them writes y.  Four K
// groups (slabs kg, kg + 4, ..) of two or three wavefronts, a 32x32 part each; the groups' sums are added in group order, as in
// kernels_gemm_tile64.hip, whose products these are otherwise.
#include <stdio.h>

#include "d2ft_common.h"
#include "gemm_tile.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

namespace {

constexpr int kTM = 32, kGroups = 4, kNormThreads = 512;
constexpr int kSlabBytes = kTM * 128;            // 128 bytes of K per row
constexpr int kStagePad = 4;                     // floats between the rows of a group's sums
constexpr int kMaxRowBytes = 2048;

// byte offset of 16-byte piece `piece` of row `row` in a slab: eight rows, eight slots
__device__ __forceinline__ int piece_at(int row, int piece) { return row * 128 + ((piece ^ (row & 7)) << 4); }

__device__ __forceinline__ void unpack(u32x4 p, float (&o)[8]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        o[2 * i] = __uint_as_float(p[i] << 16);
        o[2 * i + 1] = __uint_as_float(p[i] & 0xffff0000u);
    }
}
__device__ __forceinline__ void unpack(u32x4 p, float (&o)[4]) {
#pragma unroll
    for (int i = 0; i < 4; ++i) o[i] = __uint_as_float(p[i]);
}
__device__ __forceinline__ u32x4 pack(const float (&v)[8]) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = pack_bf16x2(v[2 * i], v[2 * i + 1]);
    return r;
}
__device__ __forceinline__ u32x4 pack(const float (&v)[4]) {
    u32x4 r;
#pragma unroll
    for (int i = 0; i < 4; ++i) r[i] = __float_as_uint(v[i]);
    return r;
}
template <int LANES>
__device__ __forceinline__ float lanes_sum(float v) {
    static_assert(LANES == 16 || LANES == 32, "one row of lanes or two");
    v = row16_sum(v);
    return LANES == 16 ? v : v + __shfl_xor(v, 16, kWave);
}
template <typename T> __device__ __forceinline__ void mma(f32x16& acc, u32x4 a, u32x4 b);
template <> __device__ __forceinline__ void mma<bf16>(f32x16& acc, u32x4 a, u32x4 b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), acc, 0, 0, 0);
}
template <> __device__ __forceinline__ void mma<float>(f32x16& acc, u32x4 a, u32x4 b) {
    const f32x4 x = __builtin_bit_cast(f32x4, a), y = __builtin_bit_cast(f32x4, b);
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(x[j], y[j], acc, 0, 0, 0);
}

// NS: slabs per K group, i.e. rows of at most 512 NS bytes.  TN: columns of the tile; its first eight wavefronts normalise.
template <typename T, int NS, int TN>
__global__ __launch_bounds__(8 * TN, TN == 64 && !(NS == 4 && sizeof(T) == 2) ? 4 : TN / 32) void gemm_ln_kernel(GemmArgs g, LnArgs n) {
    // lanes that share a row, and a thread's rows (r, r + kRowStep).  16 lanes take the shorter reduction; with 32 gamma and
    // beta are fewer registers per thread, which long rows need.
    constexpr int kRowLanes = NS < 3 ? 16 : 32, kRowStep = kNormThreads / kRowLanes, kRows = kTM / kRowStep;
    constexpr int E = 16 / sizeof(T), NP = 512 * NS / (16 * kRowLanes);   // elements of a piece; pieces of a row per thread
    constexpr int kFirst = NS < 3 ? NS : 1;   // slabs of B requested ahead of the norm: with more, two workgroups of a CU run out of registers
    constexpr int kStride = TN + kStagePad;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / (TN / 32), wj = wave % (TN / 32) * 32;   // K group; columns of the tile
    const bool norms = wave < kNormThreads / 64;
    int tm, tn, split;
    const int tiles_m = (g.M + kTM - 1) / kTM, tiles_n = (g.N + TN - 1) / TN;
    tile_of_block(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn, split);
    const int m0 = tm * kTM, n0 = tn * TN;
    const int pieces = g.K / E, slabs = pieces >> 3;

    // of a row the pieces j, j + kRowLanes, ..
    const int r = threadIdx.x / kRowLanes, j = threadIdx.x % kRowLanes;
    const __amdgpu_buffer_rsrc_t rx = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, kBufBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rg = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(n.gamma), 0, kBufBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rt = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(n.beta), 0, kBufBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, kBufBytes, 0x00020000);
    u32x4 x[kRows][NP], ga[NP], be[NP], b[NS][4];
    if (norms) {
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            const int m = m0 + r + kRowStep * i;
            const uint32_t row_at = (uint32_t)m * (uint32_t)pieces * 16u;
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                const int p = j + kRowLanes * c;
                x[i][c] = __builtin_amdgcn_raw_buffer_load_b128(rx, m < g.M && p < pieces ? row_at + p * 16u : kOutside, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const int p = j + kRowLanes * c;
            ga[c] = __builtin_amdgcn_raw_buffer_load_b128(rg, p < pieces ? p * 16u : kOutside, 0, 0);
            be[c] = __builtin_amdgcn_raw_buffer_load_b128(rt, p < pieces ? p * 16u : kOutside, 0, 0);
        }
    }
    // a lane's column of B, 16 bytes of every 32: quarter q of a slab's K
    const int col = n0 + wj + (lane & 31);
    const uint32_t col_at = (uint32_t)(g.remap == REMAP_B_N ? g.tbl.start[(n0 + wj) >> 6] + (col & 63) : col) * (uint32_t)pieces * 16u + (uint32_t)(lane >> 5) * 16u;
    auto fetch = [&](int s) {
        const int slab = kg + kGroups * s;
        const bool in = col < g.N && slab < slabs;
#pragma unroll
        for (int q = 0; q < 4; ++q) b[s][q] = __builtin_amdgcn_raw_buffer_load_b128(rb, in ? col_at + slab * 128u + q * 32u : kOutside, 0, 0);
    };
#pragma unroll
    for (int s = 0; s < kFirst; ++s) fetch(s);

    // the rows' statistics, as ln_fwd_kernel takes them: the mean first, then the squares of the differences
    if (norms) {
        float mu[kRows], rs[kRows];
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            float sum = 0.f;
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                float v[E];
                unpack(x[i][c], v);
#pragma unroll
                for (int e = 0; e < E; ++e) sum += v[e];   // zeros past the row's end
            }
            mu[i] = lanes_sum<kRowLanes>(sum) / (float)g.K;
        }
#pragma unroll
        for (int i = 0; i < kRows; ++i) {
            float sq = 0.f;
#pragma unroll
            for (int c = 0; c < NP; ++c) {
                float v[E];
                unpack(x[i][c], v);
                if (j + kRowLanes * c < pieces) {
#pragma unroll
                    for (int e = 0; e < E; ++e) {
                        const float d = v[e] - mu[i];
                        sq += d * d;
                    }
                }
            }
            rs[i] = 1.0f / sqrtf(lanes_sum<kRowLanes>(sq) / (float)g.K + n.eps);
        }
#pragma unroll
        for (int c = 0; c < NP; ++c) {
            const int p = j + kRowLanes * c;
            if (p < pieces) {
                float gv[E], bv[E];
                unpack(ga[c], gv);
                unpack(be[c], bv);
#pragma unroll
                for (int i = 0; i < kRows; ++i) {
                    const int row = r + kRowStep * i;
                    float v[E];
                    unpack(x[i][c], v);
#pragma unroll
                    for (int e = 0; e < E; ++e) v[e] = (v[e] - mu[i]) * rs[i] * gv[e] + bv[e];
                    const u32x4 out = pack(v);
                    *reinterpret_cast<u32x4*>(smem + (p >> 3) * kSlabBytes + piece_at(row, p & 7)) = out;
                    if (tn == 0 && m0 + row < g.M) *reinterpret_cast<u32x4*>(static_cast<T*>(n.y) + (long)(m0 + row) * g.K + p * E) = out;
                }
            }
        }
        if (tn == 0 && j == 0) {
#pragma unroll
            for (int i = 0; i < kRows; ++i) {
                const int m = m0 + r + kRowStep * i;
                if (m < g.M) {
                    n.mean[m] = mu[i];
                    n.rstd[m] = rs[i];
                }
            }
        }
    }
#pragma unroll
    for (int s = kFirst; s < NS; ++s) fetch(s);
    // what the epilogue reads for this thread's 8 columns
    constexpr int kPieces = kTM * TN / 8, kRowPieces = TN / 8;
    const int er = threadIdx.x / kRowPieces, ec = threadIdx.x % kRowPieces * 8;
    const bool emits = threadIdx.x < kPieces && m0 + er < g.M && n0 + ec < g.N;
    EpilogueOperands<T> early;
    if (emits) early.request(g, m0 + er, n0 + ec);
    __syncthreads();

    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
#pragma unroll
    for (int s = 0; s < NS; ++s) {
        const int slab = kg + kGroups * s;
        if (slab < slabs) {
            const unsigned char* const a = smem + slab * kSlabBytes;
#pragma unroll
            for (int q = 0; q < 4; ++q)
                mma<T>(acc, *reinterpret_cast<const u32x4*>(a + piece_at(lane & 31, 2 * q + (lane >> 5))), b[s][q]);
        }
    }
    __syncthreads();   // the stage below reuses the rows' place
    float* const stage = reinterpret_cast<float*>(smem) + kg * kTM * kStride;
#pragma unroll
    for (int e = 0; e < 16; ++e) stage[(8 * (e >> 2) + 4 * (lane >> 5) + (e & 3)) * kStride + wj + (lane & 31)] = acc[e];
    __syncthreads();
    if (!emits) return;
    float o[8];
    const float* const mine = reinterpret_cast<const float*>(smem) + er * kStride + ec;
    load8(mine, o);
#pragma unroll
    for (int w = 1; w < kGroups; ++w) {
        float more[8];
        load8(mine + w * kTM * kStride, more);
#pragma unroll
        for (int i = 0; i < 8; ++i) o[i] += more[i];
    }
    emit<T>(g, m0 + er, n0 + ec, o, early);
}

struct KernelName {
    char s[48];
    KernelName(const char* type, int ns, int tn) { snprintf(s, sizeof(s), "gemm_ln_kernel<%s, %d, %d>", type, ns, tn); }
};

template <typename T, int NS, int TN>
hipError_t launch_form(const GemmArgs& g, const LnArgs& n, hipStream_t s) {
    static const KernelName name(sizeof(T) == 4 ? "float" : "__bf16", NS, TN);
    launch_label(name.s);
    const unsigned grid = (unsigned)((g.M + kTM - 1) / kTM) * (unsigned)((g.N + TN - 1) / TN);
    constexpr int stage = kGroups * kTM * (TN + kStagePad) * 4;
    const int rows = g.K * (int)sizeof(T) * kTM;   // at most 64 KB
    hipLaunchKernelGGL((gemm_ln_kernel<T, NS, TN>), dim3(grid), dim3(8 * TN), rows > stage ? rows : stage, s, g, n);
    return hipGetLastError();
}

template <typename T, int TN>
hipError_t launch(const GemmArgs& g, const LnArgs& n, hipStream_t s) {
    const int row_bytes = g.K * (int)sizeof(T);
    if (row_bytes <= 512) return launch_form<T, 1, TN>(g, n, s);
    if (row_bytes <= 1024) return launch_form<T, 2, TN>(g, n, s);
    if (row_bytes <= 1536) return launch_form<T, 3, TN>(g, n, s);
    return launch_form<T, 4, TN>(g, n, s);
}


}  // namespace

// g as for gemm_tile64_supported, its A the rows before the norm
static bool gemm_ln_supported(const GemmArgs& g, const LnArgs& n, int dtype) {
    const int es = dtype == D2FT_F32 ? 4 : 2;
    if (!gemm_tile64_supported(g, dtype) || g.a_cs != 1 || g.a_rs != g.K || g.b_rs != 1 || g.b_cs != g.K) return false;
    if (g.remap == REMAP_B_K || g.partial || g.colsum) return false;
    if (g.K * es % 128 != 0 || g.K * es > kMaxRowBytes) return false;
    return al16(n.gamma) && al16(n.beta) && al16(n.y);
}

// Columns of the tile, or 0 where the norm and the cheapest product are the faster as two launches.  Microseconds saved per
// pair in a pass of 12 blocks, 33 to 2561 rows, by workgroups: a gain while each has a CU of its own, with 64 columns
// (bf16, width 768: 108 1.3, 240 2.2, 252 2.1, 324 -1.1, 336 -0.7; 1024: 240 2.8, 320 -2.2; 384: 126 1.1, 234 1.6, 312 -0.4;
// fp32, 384: 234 1.8, 312 0.9), beyond that with 96 (bf16, 768: 216 0.7, 224 1.5, 288 -4.9; 384: 208 1.3, 304 -3.1; fp32, 384: 208 3.5,
// 304 -5.6).  bf16 rows of up to 512 bytes leave registers for three workgroups to a CU (width 192: 300 1.7, 600 1.5, 729 1.1, 972
// -0.3).  fp32: the matrix instruction is slow enough that two to a CU still gain (384: 456 1.8, 558 1.3, 900 -0.9; 512: 456
// 0.5, 608 -1.2), and that few workgroups of long rows lose against 32x32 tiles (512: 72 -1.1, 120 -1.6, 160 1.3; 384: 126
// -0.3, 162 1.6).  Tiles of 64 rows lose everywhere.
static int gemm_ln_columns(const GemmArgs& g, const LnArgs& n, int dtype) {
    if (!gemm_ln_supported(g, n, dtype)) return 0;
    const long rows = (g.M + kTM - 1) / kTM, units64 = rows * ((g.N + 63) / 64), units96 = rows * ((g.N + 95) / 96);
    const bool f32 = dtype == D2FT_F32;
    if (f32 && g.K > 320 && units64 < 144) return 0;
    if (units64 <= 256) return 64;
    if (units96 <= 256) return 96;
    return units64 <= (f32 ? 512 : g.K <= 256 ? 768 : 0) ? 64 : 0;
}
bool gemm_ln_faster(const GemmArgs& g, const LnArgs& n, int dtype) { return gemm_ln_columns(g, n, dtype) != 0; }

hipError_t launch_gemm_ln(const GemmArgs& g, const LnArgs& n, int dtype, hipStream_t s) {
    const int columns = gemm_ln_columns(g, n, dtype);
    if (columns == 0) return hipErrorNotSupported;
    if (dtype == D2FT_F32) return columns == 64 ? launch<float, 64>(g, n, s) : launch<float, 96>(g, n, s);
    return columns == 64 ? launch<bf16, 64>(g, n, s) : launch<bf16, 96>(g, n, s);
}

}  // namespace d2ft
