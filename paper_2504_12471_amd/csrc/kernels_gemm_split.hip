// fp32 products on the bf16 matrix cores: every operand element is cut into three bf16 parts, x = hi + mid + lo, and six
// of the nine products of parts are summed in fp32,
//   a b = (hi lo + lo hi + mid mid + hi mid + mid hi) + hi hi,
// what is left out (mid lo, lo mid, lo lo) being below 2^-25 of the product.  The parts are exact, 8 + 8 + 8 significant
// bits, because they are parts of x * 2^24: no bit of it is below bf16's smallest normal value, whatever x (parts of x itself
// would lose bits below |x| = 2^-110).  The results are multiplied by 2^-48.  Against fp64, relative 2-norm error over normal inputs, K = 384 / 768 / 1536: this kernel 1.1e-7 / 1.5e-7 /
// 2.5e-7, the fp32 matrix instruction 3.5e-7 / 4.9e-7 / 7.2e-7: sixteen products enter the accumulator per rounding instead
// of two, and the small products have one of their own (in one accumulator with the others, with parts cut off instead
// of rounded: 3.8e-7 / 5.5e-7 / 1.1e-6).
//
// A part of an infinity or NaN is a NaN, an operand of 2^104 and more has no parts, and a scaled sum of 2^128 and more
// overflows: a wavefront that finds a value that is not finite among its results forms them again with the fp32
// instruction, so those come out as they always did.  That redo loads single elements: a pass over the small fp32 model (12
// blocks, width 384, 80 images of 197 tokens) takes 22 ms, with an infinity in the output gradient 42 to 51 ms, with a NaN
// in every image 82 ms.
//
//   C[m][n] = epilogue( sum_k A(m,k) * B(k,n) )
//
// A workgroup makes a 128 x 64 tile with four wavefronts of 64 x 32; a slab is 32 of k.  The next slab is in flight in
// registers while the present one is multiplied; its parts are cut on the way to LDS, once per element and workgroup (6.5
// vector instructions per element).  LDS holds one slab (36 KB), so that four workgroups share a CU and some cut and
// store while others multiply.  A 128 x 128 tile was measured equal (15760 x 1536 x 384: 120 us both) to slower.
//
// Bound: the matrix cores (24 products of 32 cycles per slab and wavefront, 768 cycles) with LDS beside them (72 KB of
// fragment reads and 36 KB of stores per slab and workgroup, some 860 cycles).  15760 x 384 x 1536 takes 115 us (166 us
// with the fp32 instruction): 970 TFLOP/s of bf16 products.
//
// LDS layouts, per part: row form [index][32 k], rows of 64 bytes, 16-byte pieces permuted by bits 2..3 of the row; column
// form [k][W indices], 32-byte chunks permuted by the low bits of k, read by the transposing read.  Both are free of bank
// conflicts in stores and reads.
#include <type_traits>

#include "gemm_tile.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

namespace {

constexpr int BK = 32;
constexpr int TM = 128, TN = 64;
constexpr float kUp = 16777216.f;            // 2^24
constexpr float kDown = 3.5527136788e-15f;   // 2^-48
static_assert(kDown * kUp * kUp == 1.f, "powers of two");

// eight floats -> the three parts of them times kUp, eight bf16 each
__device__ __forceinline__ void cut(const u32x4& x0, const u32x4& x1, u32x4 (&part)[3]) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        x[i] = __uint_as_float(x0[i]) * kUp;
        x[4 + i] = __uint_as_float(x1[i]) * kUp;
    }
#pragma unroll
    for (int p = 0; p < 3; ++p)
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint32_t two = pack_bf16x2(x[2 * i], x[2 * i + 1]);
            part[p][i] = two;
            if (p < 2) {
                x[2 * i] -= __uint_as_float(two << 16);
                x[2 * i + 1] -= __uint_as_float(two & 0xffff0000u);
            }
        }
}

template <bool COL, int W>
__device__ __forceinline__ int piece_offset(int row, int piece) {   // pieces of 8 elements
    if constexpr (!COL) return row * 64 + ((piece ^ ((row >> 2) & 3)) << 4);
    const int chunk = (piece >> 1) ^ (W == 128 ? (row & 3) << 1 : ((row >> 1) & 1) << 1);
    return row * 2 * W + chunk * 32 + (piece & 1) * 16;
}

// a thread's pieces of a slab of W indices
template <bool COL, int W>
struct Loader {
    static constexpr int kN = W / 64;
    static constexpr int kPerRow = COL ? W / 8 : 4;
    static constexpr int kPart = W * 64;   // bytes of one part
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t base[kN], sk;
    int k_in[kN];
    u32x4 raw[kN][2];
    template <typename F>
    __device__ __forceinline__ void init(const void* p, long s_i, long s_k, int i0, int I, F&& index_of) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kBufBytes, 0x00020000);
        sk = (uint32_t)s_k * 4u;
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            const int id = threadIdx.x + 256 * c, row = id / kPerRow, p8 = id % kPerRow * 8;
            const int i = i0 + (COL ? p8 : row);
            k_in[c] = COL ? row : p8;
            const uint32_t off = ((uint32_t)index_of(i < I ? i : 0) * (uint32_t)s_i + (uint32_t)k_in[c] * (uint32_t)s_k) * 4u;
            base[c] = i < I ? off : kOutside;
        }
    }
    // the slab at k0 (valid k < k_end) whose first k sits at k_at in memory
    __device__ __forceinline__ void fetch(int k0, int k_at, int k_end) {
        const uint32_t slab = slab_offset(k0, k_at, k_end, sk);
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            const uint32_t at = k_in[c] < k_end - k0 ? base[c] : kOutside;
            raw[c][0] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at, slab, 0);
            raw[c][1] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, at + 16u, slab, 0);
        }
    }
    __device__ __forceinline__ void cut_all(u32x4 (&part)[kN][3]) const {
#pragma unroll
        for (int c = 0; c < kN; ++c) cut(raw[c][0], raw[c][1], part[c]);
    }
    static __device__ __forceinline__ void store(const u32x4 (&part)[kN][3], unsigned char* slab) {
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            const int id = threadIdx.x + 256 * c, off = piece_offset<COL, W>(id / kPerRow, id % kPerRow);
#pragma unroll
            for (int p = 0; p < 3; ++p) *reinterpret_cast<u32x4*>(slab + p * kPart + off) = part[c][p];
        }
    }
};

// 32 indices from i0, k = 16 kk + 8h + {0..7} of one part
template <bool COL, int W>
__device__ __forceinline__ bf16x8 read_frag(const unsigned char* part, int i0, int kk, int lane) {
    if constexpr (!COL) {
        return *reinterpret_cast<const bf16x8*>(part + piece_offset<false, W>(i0 + (lane & 31), 2 * kk + (lane >> 5)));
    } else {
        const int j = lane & 15, r = 16 * kk + 8 * (lane >> 5) + (j >> 2);
        const unsigned char* p = part + piece_offset<true, W>(r, 2 * ((i0 >> 4) + ((lane >> 4) & 1))) + (j & 3) * 8;
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * 2 * W));   // rows 4 apart permute alike
        s16x8 v;
        v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3];
        v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
        return __builtin_bit_cast(bf16x8, v);
    }
}

constexpr int kLds = 3 * 64 * (TM + TN);   // one slab; the stage and a rider's workgroup need less
static_assert(kLds >= 4 * 32 * (TN / 2 + 4) * 4 && kLds >= kTailLds, "");

template <bool A_COL, bool B_COL, typename Args>
__global__ __launch_bounds__(256, 4) void gemm_split_kernel(Args g) {
    constexpr bool GROUPED = std::is_same<Args, Tile64Grouped>::value;
    static_assert(!GROUPED || (A_COL && B_COL), "weight gradients: both operands with k strided");
    constexpr int WTN = TN / 2, NT = WTN / 32;   // a wavefront's columns; its 32-wide parts along n (two along m)
    __shared__ __attribute__((aligned(16))) unsigned char smem[kLds];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wi = (wave >> 1) * 64, wj = (wave & 1) * WTN;

    int m0, n0, M, N, kb, ke, split, tile = 0, gi = 0;
    typedef Loader<A_COL, TM> LA;
    typedef Loader<B_COL, TN> LB;
    LA la;
    LB lb;
    auto same = [](int i) { return i; };
    if constexpr (GROUPED) {
        if ((int)blockIdx.x >= g.units) {
            tail_work<float>(g.tail, blockIdx.x - g.units, threadIdx.x, 256, smem);
            return;
        }
        const int total = g.units, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
        const int u = xcd * (total >> 3) + min(xcd, total & 7) + idx;
        split = u / g.total_tiles;
        tile = u - split * g.total_tiles;
        while (gi + 1 < g.n && tile >= g.grp[gi + 1].tile0) ++gi;
        const Tile64Group& G = g.grp[gi];
        const int lt = tile - G.tile0;
        M = G.M;
        N = G.N;
        m0 = (lt % G.tiles_m) * TM;
        n0 = (lt / G.tiles_m) * TN;
        kb = split * g.slabs_per_split * BK;
        ke = min(g.K, kb + g.slabs_per_split * BK);
        la.init(G.A, 1, G.lda, m0, M, same);
        lb.init(G.B, 1, G.ldb, n0, N, same);
    } else {
        const int tiles_m = (g.M + TM - 1) / TM, tiles_n = (g.N + TN - 1) / TN;
        int tm, tn;
        tile_of_block(blockIdx.x, tiles_m * tiles_n, tiles_m, tiles_n, tm, tn, split);
        M = g.M;
        N = g.N;
        m0 = tm * TM;
        n0 = tn * TN;
        kb = 0;
        ke = g.K;
        la.init(g.A, g.a_rs, g.a_cs, m0, M, same);
        if (g.remap == REMAP_B_N) lb.init(g.B, g.b_cs, g.b_rs, n0, N, [&](int i) { return g.tbl(i); });
        else lb.init(g.B, g.b_cs, g.b_rs, n0, N, same);
    }
    auto fetch = [&](int k0) {
        int k_at = k0;   // k of the slab as B is stored
        if constexpr (!GROUPED) {
            if (g.remap == REMAP_B_K && k0 < ke) k_at = g.tbl.start[k0 >> 6] + (k0 & 63);
        }
        la.fetch(k0, k0, ke);
        lb.fetch(k0, k_at, ke);
    };

    f32x16 acc[2][NT], low[2][NT];   // hi hi, and the other five
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[i][j][e] = low[i][j][e] = 0.f;
    unsigned char* const As = smem;
    unsigned char* const Bs = smem + 3 * LA::kPart;
    fetch(kb);
    for (int k0 = kb; k0 < ke; k0 += BK) {
        {
            u32x4 pa[LA::kN][3], pb[LB::kN][3];
            la.cut_all(pa);
            lb.cut_all(pb);
            __syncthreads();   // the slab before has been read
            LA::store(pa, As);
            LB::store(pb, Bs);
        }
        fetch(k0 + BK);        // past the end: zeros, unused
        __syncthreads();
#pragma unroll
        for (int kk = 0; kk < 2; ++kk) {
            bf16x8 fa[2][3], fb[NT][3];
#pragma unroll
            for (int p = 2; p >= 0; --p) {
#pragma unroll
                for (int i = 0; i < 2; ++i) fa[i][p] = read_frag<A_COL, TM>(As + p * LA::kPart, wi + 32 * i, kk, lane);
#pragma unroll
                for (int j = 0; j < NT; ++j) fb[j][p] = read_frag<B_COL, TN>(Bs + p * LB::kPart, wj + 32 * j, kk, lane);
            }
            constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};   // the small products first
#pragma unroll
            for (int q = 0; q < 6; ++q)
#pragma unroll
                for (int i = 0; i < 2; ++i)
#pragma unroll
                    for (int j = 0; j < NT; ++j) {
                        f32x16& to = q == 5 ? acc[i][j] : low[i][j];
                        to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(fa[i][kPa[q]], fb[j][kPb[q]], to, 0, 0, 0);
                    }
        }
    }
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j) acc[i][j] = (acc[i][j] + low[i][j]) * kDown;

    const int c = lane & 31, h = lane >> 5;
    // results that are not finite: again with the fp32 instruction, operands from memory
    bool odd = false;
#pragma unroll
    for (int i = 0; i < 2; ++i)
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) odd |= !(fabsf(acc[i][j][e]) < INFINITY);
    if (__any(odd)) {
        const float* pA;
        const float* pB;
        long a_i, a_k, b_i, b_k;
        if constexpr (GROUPED) {
            const Tile64Group& G = g.grp[gi];
            pA = static_cast<const float*>(G.A); pB = static_cast<const float*>(G.B);
            a_i = b_i = 1; a_k = G.lda; b_k = G.ldb;
        } else {
            pA = static_cast<const float*>(g.A); pB = static_cast<const float*>(g.B);
            a_i = g.a_rs; a_k = g.a_cs; b_i = g.b_cs; b_k = g.b_rs;
        }
#pragma unroll 1
        for (int t = 0; t < 2 * NT; ++t) {
            const int m = m0 + wi + t / NT * 32 + c, n = n0 + wj + t % NT * 32 + c;
            long bn = n < N ? n : 0;
            if constexpr (!GROUPED) {
                if (g.remap == REMAP_B_N) bn = g.tbl((int)bn);
            }
            f32x16 s;
#pragma unroll
            for (int e = 0; e < 16; ++e) s[e] = 0.f;
#pragma unroll 1
            for (int k = kb; k < ke; k += 2) {
                const int kh = k + h;
                long bk = kh;
                if constexpr (!GROUPED) {
                    if (g.remap == REMAP_B_K && kh < ke) bk = g.tbl(kh);
                }
                const float a = m < M && kh < ke ? pA[m * a_i + kh * a_k] : 0.f;
                const float b = n < N && kh < ke ? pB[bn * b_i + bk * b_k] : 0.f;
                s = __builtin_amdgcn_mfma_f32_32x32x2f32(a, b, s, 0, 0, 0);
            }
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int j = 0; j < NT; ++j)
                    if (t == i * NT + j) acc[i][j] = s;
        }
    }

    // ---- epilogue: 32 rows of the wavefront's results at a time through its own part of LDS ----
    __syncthreads();   // the operands have been read
    constexpr int kStride = WTN + 4, kPer = WTN / 8;
    float* const stage = reinterpret_cast<float*>(smem) + wave * 32 * kStride;
    float csum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) csum[i] = 0.f;
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int j = 0; j < NT; ++j)
#pragma unroll
            for (int e = 0; e < 16; ++e) stage[(8 * (e >> 2) + 4 * h + (e & 3)) * kStride + 32 * j + c] = acc[i][j][e];
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int u = 0; u < 32 * kPer / 64; ++u) {
            const int p = u * 64 + lane, r = p / kPer, cc = p % kPer * 8;
            const int rt = wi + 32 * i + r, ct = wj + cc;   // within the tile
            const int m = m0 + rt, n = n0 + ct;
            float v[8];
            load8(stage + r * kStride + cc, v);
            if constexpr (GROUPED) {
                if (g.splits > 1) store8(g.partial + ((long)split * g.total_tiles + tile) * (TM * TN) + rt * TN + ct, v);
                else if (m < M && n < N) emit_grouped<float>(g, gi, m, n, v);
            } else if (m < M && n < N) {
                emit<float>(g, m, n, v);
#pragma unroll
                for (int q = 0; q < 8; ++q) csum[q] += v[q];
            }
        }
    }
    if constexpr (!GROUPED) {
        if (!g.colsum) return;   // uniform over the grid
        // a band is the wavefront's 64 rows: lanes kPer apart share their columns
#pragma unroll
        for (int q = 0; q < 8; ++q) {
            float s = csum[q];
#pragma unroll
            for (int w = kPer; w < 64; w <<= 1) s += __shfl_xor(s, w, 64);
            csum[q] = s;
        }
        const int n = n0 + wj + lane * 8;
        if (lane < kPer && n < N && m0 + wi < M) store8(g.colsum + (long)(g.colsum_row0 + (m0 + wi) / 64) * N + n, csum);
    }
}

// the splits of a tile of a grouped launch in split order; blockIdx.x = tile, a thread owns 4 columns of every 16th row
__global__ __launch_bounds__(256) void reduce_split_kernel(Tile64Grouped g) {
    const int tile = blockIdx.x;
    int gi = 0;
    while (gi + 1 < g.n && tile >= g.grp[gi + 1].tile0) ++gi;
    const Tile64Group& G = g.grp[gi];
    const int lt = tile - G.tile0;
    const int r = blockIdx.y * 16 + (threadIdx.x >> 4), cc = (threadIdx.x & 15) * 4;
    const int m = (lt % G.tiles_m) * TM + r, n = (lt / G.tiles_m) * TN + cc;
    if (m >= G.M || n >= G.N) return;
    const float* src = g.partial + (long)tile * (TM * TN) + r * TN + cc;
    const long stride = (long)g.total_tiles * (TM * TN);
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 4 <= g.splits; k += 4) {
        f32x4 v[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) v[j] = *reinterpret_cast<const f32x4*>(src + (k + j) * stride);
#pragma unroll
        for (int j = 0; j < 4; ++j) s += v[j];
    }
    for (; k < g.splits; ++k) s += *reinterpret_cast<const f32x4*>(src + k * stride);
    int mo = m, no = n;
    if (G.remap == RED_REMAP_ROWS) mo = g.tbl[G.table][m >> 6] * 64 + (m & 63);
    if (G.remap == RED_REMAP_COLS) no = g.tbl[G.table][n >> 6] * 64 + (n & 63);
    f32x4* o = reinterpret_cast<f32x4*>(static_cast<float*>(G.out) + (long)mo * G.ldo + no);
    if (g.accumulate && G.remap != RED_REMAP_F32) s += *o;
    *o = s;
}

template <typename Kernel, typename Args>
hipError_t launch(const char* name, Kernel kern, unsigned grid, hipStream_t s, const Args& a) {
    launch_label(name);
    return launch_signalling(kern, dim3(grid), dim3(256), 0, s, a);
}

// launch + rounds of four workgroups per CU x (start + slab * slabs + epilogue), a partly filled round at no less than
// 0.37 of a full one: fitted on this part to 112 products of 260 to 15760 rows, rms error 6 %
float cost_us(long units, int slabs, float epilogue) {
    float rounds = (float)(units / 1024);
    if (const int rest = (int)(units % 1024)) rounds += 0.37f + 0.63f * (float)rest / 1024.0f;
    return 3.3f + rounds * (3.4f + 2.62f * (float)slabs + epilogue);
}

}  // namespace

float gemm_split_us(const GemmArgs& g) {
    if (g.a_cs != 1 || g.partial) return 1e30f;
    const long units = (long)((g.M + TM - 1) / TM) * ((g.N + TN - 1) / TN);
    return cost_us(units, (g.K + BK - 1) / BK, g.act == ACT_GELU ? 17.8f : (g.act == ACT_DGELU ? 2.2f : (g.residual ? 3.2f : 0.0f)));
}

hipError_t launch_gemm_split(const GemmArgs& g, hipStream_t s) {
    const unsigned grid = (unsigned)((g.M + TM - 1) / TM) * (unsigned)((g.N + TN - 1) / TN);
    if (g.b_rs == 1) return launch("gemm_split_kernel<false, false, d2ft::GemmArgs>", gemm_split_kernel<false, false, GemmArgs>, grid, s, g);
    return launch("gemm_split_kernel<false, true, d2ft::GemmArgs>", gemm_split_kernel<false, true, GemmArgs>, grid, s, g);
}

float gemm_split_grouped_plan(Tile64Grouped* a, size_t partial_floats) {
    int tiles = 0;
    for (int i = 0; i < a->n; ++i) {
        a->grp[i].tiles_m = (a->grp[i].M + TM - 1) / TM;
        a->grp[i].tile0 = tiles;
        tiles += a->grp[i].tiles_m * ((a->grp[i].N + TN - 1) / TN);
    }
    a->total_tiles = tiles;
    // splits of K: the cheapest, with a second launch that reads the partial tiles (about 3 TB/s there and back)
    const int slabs = (a->K + BK - 1) / BK;
    float best = 1e30f;
    for (int sp = 1; sp <= 32 && (sp == 1 || (slabs / sp >= 8 && (size_t)sp * tiles * (TM * TN) <= partial_floats)); ++sp) {
        const int per = (slabs + sp - 1) / sp;
        const float t = cost_us((long)tiles * sp, per, 0.0f) + (sp > 1 ? 4.0f + (float)tiles * sp * 0.022f : 0.0f);
        if (t < best) {
            best = t;
            a->slabs_per_split = per;
            a->splits = (slabs + per - 1) / per;
        }
    }
    a->units = tiles * a->splits;
    return best;
}

hipError_t launch_gemm_split_grouped(const Tile64Grouped& a, hipStream_t s) {
    hipError_t e = launch("gemm_split_kernel<true, true, d2ft::Tile64Grouped>", gemm_split_kernel<true, true, Tile64Grouped>, (unsigned)(a.units + a.tail.blocks), s, a);
    if (e != hipSuccess || a.splits == 1) return e;
    hipLaunchKernelGGL(reduce_split_kernel, dim3((unsigned)a.total_tiles, TM / 16), dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace d2ft
