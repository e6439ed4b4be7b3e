// bf16 products of the forward pass with many rows and a short K: two workgroups to a CU, so that the epilogue of one runs
// under the multiplications of the other.
//
//   C[m][n] = epilogue( sum_k A[m][k] * B[n][k] ),  K a multiple of 64; epilogue: bias, GELU with its derivative
//
// The 256x256 tile (kernels_gemm_mfma.hip) has a CU to itself, and at K = 768 its epilogue takes as long as its
// multiplications: GELU with its derivative is 25 thousand cycles of vector instructions a tile, beside 25 thousand of
// matrix instructions.  Here a workgroup of four wavefronts owns a 128x256 tile, a wavefront 128x64 of it, and needs half
// of the CU's LDS and registers.  The price is 1.5 times the operand bytes from L2 per multiplication, which is why long
// K stays with the large tile, and so do products beside another stream's: they leave CUs to it, this kernel does not.
// 12608 x 3072 x 768 with GELU: 90 -> 78 us (bound by LDS, which takes 96 KB and gives 192 KB in the time of 2048 cycles
// of multiplications); 15760 x 1536 x 384: 43 -> 36; 12608 x 768 x 3072, not sent here: 57 and 75.
//
// LDS (80 KB): three slabs of A (128 rows x 64 k) and one of B (256 columns x 64 k).  A wavefront loads its own 64 columns
// of B and nobody else reads them; it takes all their fragments of a slab into registers at the slab's start, so the
// next slab of B is on its way into the same place while they are multiplied.  A is shared: slab s + 2 is requested in
// slab s, one barrier per slab.  Both are loaded straight into LDS (no registers hold them on the way), always whole
// 128-byte lines: rows of 64 bytes, which a slab of 32 k would have, load at half the rate (24 against 41 bytes per clock
// and CU).
#include <type_traits>

#include "gemm_large.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

namespace {

constexpr int BM = 128, BN = 256, BK = 64, kWaves = 4;
constexpr int kSlabA = BM * BK * 2, kSlabB = BN * BK * 2, kLds = 3 * kSlabA + kSlabB;
constexpr int kLoadA = kSlabA / kWaves / 1024, kLoadB = kSlabB / kWaves / 1024;   // a wavefront's loads of 1024 bytes per slab
constexpr int MT = 4, NT = 2;   // 32x32 parts of a wavefront's 128x64

__device__ __forceinline__ void wait_lds() { asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory"); }

// the 16-byte pieces of a slab's rows of 128 bytes change places, so that a fragment read (16 lanes want the same piece of
// 16 rows) touches all banks: piece p of row r sits at p ^ swizzle(r)
__device__ __forceinline__ int swizzle(int row) { return (row >> 1) & 7; }

// REMAP: B's row index n through g.tbl
template <int ACT, bool REMAP>
__global__ __launch_bounds__(64 * kWaves, 2) void gemm_pair_kernel(GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    lds_u8* const lds = (lds_u8*)smem_raw;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, c32 = lane & 31;
    const int tiles_m = (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN, total = tiles_m * tiles_n;
    const __amdgpu_buffer_rsrc_t ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.A), 0, kBufBytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(g.B), 0, kBufBytes, 0x00020000);
    const uint32_t lda = (uint32_t)g.a_rs * 2, ldb = (uint32_t)g.b_cs * 2;   // bytes
    const int ns = g.K / BK;

    // a lane's place in the fragments of rows 32*t + c32, for each 16 k of a slab
    uint32_t row_at[4];
#pragma unroll
    for (int q = 0; q < 4; ++q) row_at[q] = c32 * 128 + (((2 * q + h) ^ swizzle(c32)) << 4);
    lds_u8* const own_b = lds + 3 * kSlabA + wave * (kSlabB / kWaves);

    uint32_t off_a[kLoadA], off_b[kLoadB];   // byte offsets of the lane's pieces in slab 0
    int m0 = 0, n0 = 0;
    auto load_a = [&](int s) {
        lds_u8* const d = lds + s % 3 * kSlabA + wave * (kSlabA / kWaves);
#pragma unroll
        for (int c = 0; c < kLoadA; ++c) __builtin_amdgcn_raw_ptr_buffer_load_lds(ra, (lds_u32*)(d + c * 1024), 16, off_a[c], s * (BK * 2), 0, 0);
    };
    auto load_b = [&](int s) {
#pragma unroll
        for (int c = 0; c < kLoadB; ++c) __builtin_amdgcn_raw_ptr_buffer_load_lds(rb, (lds_u32*)(own_b + c * 1024), 16, off_b[c], s * (BK * 2), 0, 0);
    };
    // fixes a tile's coordinates and load addresses and requests its first slabs
    auto setup = [&](int pid) {
        int tm, tn;
        tile_at(xcd_range(pid, total), tiles_m, tiles_n, tm, tn);
        m0 = tm * BM;
        n0 = tn * BN;
#pragma unroll
        for (int c = 0; c < kLoadA; ++c) {
            const int r = (wave * kLoadA + c) * 8 + (lane >> 3), m = m0 + r;
            off_a[c] = m < g.M ? (uint32_t)m * lda + (((lane & 7) ^ swizzle(r)) << 4) : kOutside;
        }
        const int nw = n0 + wave * 64;   // the wavefront's 64 columns: one block of the remap table
        const int nb = REMAP ? (nw < g.N ? g.tbl.start[nw >> 6] : 0) : nw;
#pragma unroll
        for (int c = 0; c < kLoadB; ++c) {
            const int r = c * 8 + (lane >> 3);
            off_b[c] = nw + r < g.N ? (uint32_t)(nb + r) * ldb + (((lane & 7) ^ swizzle(r)) << 4) : kOutside;
        }
        load_a(0);
        load_b(0);
        if (ns > 1) load_a(1);
    };

    f32x16 acc[MT][NT];
    if ((int)blockIdx.x < total) {
        setup(blockIdx.x);
        wait_vm<0>();
    }
    for (int pid = blockIdx.x; pid < total; pid += gridDim.x) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[t][u][e] = 0.f;
        bf16x8 af[2][MT], bf[4][NT];
        auto read_a = [&](int slot, int q, bf16x8 (&a)[MT]) {
            const lds_u8* p = lds + slot * kSlabA + row_at[q];
#pragma unroll
            for (int t = 0; t < MT; ++t) a[t] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p + t * (32 * 128));
        };
        auto read_b = [&](int q, bf16x8 (&b)[NT]) {
#pragma unroll
            for (int u = 0; u < NT; ++u)
                b[u] = *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(own_b + row_at[q] + u * (32 * 128));
        };
        auto mfma_group = [&](const bf16x8 (&a)[MT], const bf16x8 (&b)[NT]) {
#pragma unroll
            for (int t = 0; t < MT; ++t)
#pragma unroll
                for (int u = 0; u < NT; ++u) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[t], b[u], acc[t][u], 0, 0, 0);
        };
        int slot = 0;
        // one slab: 4 groups of 16 k.  MORE1, MORE2: the tile has a slab s + 1, s + 2.
        auto slab = [&](int s, auto more1_tag, auto more2_tag) {
            constexpr bool MORE1 = decltype(more1_tag)::value, MORE2 = decltype(more2_tag)::value;
            // A(s) and B(s) have landed; requested behind them: A(s + 1).  Those of slabs 0 and 1 were waited for ahead of
            // the stores of the tile before.
            if (s > 0) {
                if constexpr (MORE1) wait_vm<kLoadA>();
                else wait_vm<0>();
            }
            __builtin_amdgcn_s_barrier();   // A(s) of all wavefronts; A's slab s - 1 has been read by all
            __builtin_amdgcn_sched_barrier(0);
            read_a(slot, 0, af[0]);
            read_b(0, bf[0]);
            read_a(slot, 1, af[1]);
            read_b(1, bf[1]);
            read_b(2, bf[2]);
            read_b(3, bf[3]);
            __builtin_amdgcn_sched_barrier(0);
            mfma_group(af[0], bf[0]);
            __builtin_amdgcn_sched_barrier(0);
            wait_lds();   // B(s) is in registers: its place is free
            read_a(slot, 2, af[0]);
            if constexpr (MORE1) load_b(s + 1);
            mfma_group(af[1], bf[1]);
            __builtin_amdgcn_sched_group_barrier(0x100, MT, 0);   // LDS reads
#pragma unroll
            for (int i = 0; i < MT * NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
                if constexpr (MORE1) __builtin_amdgcn_sched_group_barrier(0x010, kLoadB / (MT * NT), 0);   // load
            }
            __builtin_amdgcn_sched_barrier(0);
            read_a(slot, 3, af[1]);
            if constexpr (MORE2) load_a(s + 2);
            mfma_group(af[0], bf[2]);
            __builtin_amdgcn_sched_group_barrier(0x100, MT, 0);
#pragma unroll
            for (int i = 0; i < MT * NT; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                if (MORE2 && i < kLoadA) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            mfma_group(af[1], bf[3]);
            __builtin_amdgcn_sched_barrier(0);
            slot = slot == 2 ? 0 : slot + 1;
        };
        {
            constexpr std::true_type yes{};
            constexpr std::false_type no{};
            int s = 0;
            for (; s + 2 < ns; ++s) slab(s, yes, yes);
            if (s + 1 < ns) {
                slab(s, yes, no);
                ++s;
            }
            slab(s, no, no);
        }
        __syncthreads();   // A's slabs have been read by all: 0 and 1 take the next tile's, 2 the epilogue's stage
        const int em0 = m0, en0 = n0;
        if (pid + (int)gridDim.x < total) setup(pid + gridDim.x);

        // ---- epilogue: 16 rows at a time through 4 KB of LDS per wavefront (fp32), back 8 consecutive columns per lane.
        // Odd rows have the 16-byte halves of their 32-byte pieces exchanged, so that two rows read at once touch all banks.
        constexpr int CPR = 8, CPL = 4;   // 8-column chunks per row; chunks of a lane in 32 rows
        float* const stage = reinterpret_cast<float*>(smem_raw + 2 * kSlabA) + wave * (16 * 64);
        float* const to_even = stage + 4 * h * 64 + c32;
        float* const to_odd = stage + 4 * h * 64 + (c32 ^ 4);
        const float* const from_lo = stage + (lane / CPR) * 64 + (((lane % CPR) * 2) ^ (lane / CPR & 1)) * 4;
        const float* const from_hi = stage + (lane / CPR) * 64 + (((lane % CPR) * 2 + 1) ^ (lane / CPR & 1)) * 4;
        const int n = en0 + wave * 64 + (lane % CPR) * 8, mrow = em0 + lane / CPR;
        bf16* const C = static_cast<bf16*>(g.C);
        bf16* const Z = static_cast<bf16*>(g.Z);
        u32x4 braw = {0u, 0u, 0u, 0u};
        if (g.bias && n < g.N)
            braw = *reinterpret_cast<const u32x4*>(static_cast<const bf16*>(g.bias) + (g.bias_remap ? g.tbl(n) : n));
#pragma unroll
        for (int t = 0; t < MT; ++t) {
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                if (c % 2 == 0) {
                    __builtin_amdgcn_wave_barrier();
#pragma unroll
                    for (int u = 0; u < NT; ++u)
#pragma unroll
                        for (int e = 0; e < 8; ++e) ((e & 1) ? to_odd : to_even)[(8 * (e >> 2) + (e & 3)) * 64 + u * 32] = acc[t][u][c * 4 + e];
                    __builtin_amdgcn_wave_barrier();
                }
                const int m = mrow + t * 32 + c * (64 / CPR);
                const float4 lo = *reinterpret_cast<const float4*>(from_lo + (c & 1) * (8 * 64));
                const float4 hi = *reinterpret_cast<const float4*>(from_hi + (c & 1) * (8 * 64));
                float v[8] = {lo.x, lo.y, lo.z, lo.w, hi.x, hi.y, hi.z, hi.w};
#pragma unroll
                for (int i = 0; i < 4; ++i) {   // braw is zero without a bias
                    v[2 * i] += __uint_as_float(braw[i] << 16);
                    v[2 * i + 1] += __uint_as_float(braw[i] & 0xffff0000u);
                }
                // the next tile's slabs have to be there before the first store: a load cannot be told to have arrived
                // while stores ahead of it have not
                if (t == 0 && c == 0) {
                    __builtin_amdgcn_sched_barrier(0);
                    wait_vm<0>();
                    __builtin_amdgcn_sched_barrier(0);
                }
                if (m < g.M && n < g.N) {
                    if constexpr (ACT == ACT_GELU) {
                        float d[8];
                        gelu_pair8(v, d);
                        store8(Z + (long)m * g.ldz + n, d);
                    }
                    store8(C + (long)m * g.ldc + n, v);
                }
            }
        }
    }
}

template <int ACT, bool REMAP>
hipError_t launch_form(const GemmArgs& g, hipStream_t s) {
    auto kern = gemm_pair_kernel<ACT, REMAP>;
    static KernelLimits limits;
    int resident = 0;
    if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 64 * kWaves, kLds, &resident); e != hipSuccess) return e;
    resident = in_eights(resident);
    const long tiles = (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN);
    const dim3 grid((unsigned)(tiles < resident ? tiles : resident)), block(64 * kWaves);
    return launch_signalling(kern, grid, block, kLds, s, g);
}

}  // namespace

bool gemm_pair_supported(const GemmArgs& g) {
    return g.a_cs == 1 && g.b_rs == 1 && g.K % BK == 0 && !g.partial && !g.residual && !g.colsum && g.act != ACT_DGELU && g.remap != REMAP_B_K;
}

// Microseconds: launch + rounds * (start + slab * slabs of K + GELU), a round being two workgroups on each CU; one that fills
// part of the chip costs less by little.  Fitted to 85 products of 700 to 18900 rows, widths 192 to 1024: rms error 5 %.
float gemm_pair_us(const GemmArgs& g) {
    const long tiles = (long)((g.M + BM - 1) / BM) * ((g.N + BN - 1) / BN), rest = tiles % 512;
    const float rounds = (float)(tiles / 512) + (rest ? 0.27f + 0.73f * (float)rest / 512.0f : 0.0f);
    return 7.5f + rounds * (3.5f + 1.57f * (float)(g.K / BK) + (g.act == ACT_GELU ? 7.6f : 0.0f));
}

const char* gemm_pair_name(const GemmArgs& g) {
    static const char* const names[2][2] = {{"gemm_pair_kernel<0, false>", "gemm_pair_kernel<0, true>"}, {"gemm_pair_kernel<1, false>", "gemm_pair_kernel<1, true>"}};
    return names[g.act == ACT_GELU][g.remap == REMAP_B_N];
}

hipError_t launch_gemm_pair(const GemmArgs& g, hipStream_t s) {
    const bool remap = g.remap == REMAP_B_N;
    if (g.act == ACT_GELU) return remap ? launch_form<ACT_GELU, true>(g, s) : launch_form<ACT_GELU, false>(g, s);
    return remap ? launch_form<ACT_NONE, true>(g, s) : launch_form<ACT_NONE, false>(g, s);
}

}  // namespace d2ft
