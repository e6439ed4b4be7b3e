// GEMM on the matrix cores with small output tiles (64x64, 64x32, 32x32) and K split between the workgroup's wavefronts:
// the fp32 path (v_mfma_f32_32x32x2_f32) and the bf16 path (v_mfma_f32_32x32x16_bf16) for shapes whose larger
// tiles would leave most of the chip idle.
//
//   C[m][n] = epilogue( sum_k A(m,k) * B(k,n) )
//
// A workgroup has WK groups of wavefronts.  A group multiplies every WK-th K slab (128 bytes of k per row: 64
// bf16 or 32 fp32) of the same tile, a wavefront of it one 32x32 part; the groups' sums are added in group order
// through LDS before the epilogue, so a small problem gets WK times the wavefronts without a second launch and
// without partial sums in memory.
//
// What bounds it.  fp32: the matrix cores (256 FLOP per clock and CU); a 64x64 tile asks for 16 bytes of operands per
// clock and CU, which L2 delivers, so a larger tile would gain nothing and the small one deals evenly: four to five
// workgroups share a CU and cover each other's latencies.  bf16: a problem of a few hundred rows gives the 128x128 tile
// a few dozen workgroups with one slab in flight each, at the 30 to 45 bytes per clock that one CU loads; here the
// smallest tile that still fits the chip's CUs is taken (pick_form) and kAhead slabs per group are in flight in
// registers.
//
// The forward pass of 12 bf16 blocks on one image (197 tokens, width 768), whose products all ran on the 128x128 tile:
// 1038 -> 619 us; 5 images of width 384, forward and backward: 1899 -> 1668 us.
//
// Measured against the vector-ALU kernel it replaced for fp32: one block of 260 tokens of width 192, forward and
// backward, 721 -> 171 us (its 12 products 594 -> 104 us); the products of a 12-block stack of width 384 on 80 x 197
// tokens 63.5 -> 21.2 ms, i.e. 30 -> 90 TFLOP/s (the vendor library reaches 127-133 on the largest of them).
//
// Slabs are kept in LDS without padding, their 16-byte pieces permuted within a row so that both the stores and the
// fragment reads are free of bank conflicts (piece_offset).  Operands with K strided stay in their natural
// [k][index] layout: bf16 fragments come out of it by the transposing read, fp32 ones by plain 4-byte reads.
#include <stdio.h>

#include <atomic>
#include <type_traits>
#include <utility>

#include "d2ft_common.h"
#include "gemm_tile.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

namespace {

constexpr int kAhead = 3;                     // slabs in flight in registers
constexpr int kStagePad = 4;                  // floats between the rows of the epilogue's stage

// Byte offset of 16-byte piece `piece` of row `row` in the slab of an operand with W indices (64 or 32).  Row form: W
// rows of 128 bytes ([index][k]); column form: [k][W indices], i.e. 64 rows of 2W bytes for bf16, 32 rows of 4W for fp32.
template <typename T, bool COL, int W>
__device__ __forceinline__ int piece_offset(int row, int piece) {
    if constexpr (!COL) return row * 128 + ((piece ^ (row & 7)) << 4);               // eight rows, eight slots
    else if constexpr (sizeof(T) == 2 && W == 64) return row * 128 + ((((piece >> 1) ^ (row & 3)) << 5) | ((piece & 1) << 4));
    else if constexpr (sizeof(T) == 2) return row * 64 + (piece << 4);               // four rows fill the banks as they are
    else if constexpr (W == 64) return row * 256 + ((piece ^ (((row >> 2) & 1) << 3)) << 4);   // rows 4 apart: other half of the banks
    else return (row ^ ((row >> 2) & 1)) * 128 + (piece << 4);                       // likewise
}

// a thread's 16-byte pieces of a slab of W indices, loaded by GT threads: global offsets and LDS offsets
template <typename T, bool COL, int W, int GT>
struct Loader {
    static constexpr int kE = 16 / sizeof(T);          // elements per piece
    static constexpr int kBK = 128 / sizeof(T);        // k per slab
    static constexpr int kPerRow = COL ? W / kE : 8;   // pieces per slab row
    static constexpr int kN = W * 8 / GT;              // pieces per thread
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t base[kN], sk;
    int k_in[kN];     // k of the piece within the slab

    // index_of(i): the row (or column) of the operand that tile index i stands for
    template <typename F>
    __device__ __forceinline__ void init(const void* p, long s_i, long s_k, int i0, int I, int t, F&& index_of) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(p), 0, kBufBytes, 0x00020000);
        sk = (uint32_t)s_k * (uint32_t)sizeof(T);
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            const int id = t + GT * c;
            int i;
            if constexpr (!COL) {
                i = id >> 3;
                k_in[c] = (id & 7) * kE;
            } else {
                i = (id % kPerRow) * kE;
                k_in[c] = id / kPerRow;
            }
            i += i0;
            const uint32_t off = ((uint32_t)index_of(i < I ? i : 0) * (uint32_t)s_i + (uint32_t)k_in[c] * (uint32_t)s_k) * (uint32_t)sizeof(T);
            base[c] = i < I ? off : kOutside;
        }
    }
    // the slab at k0 (valid k < k_end) whose first k sits at k_at in memory
    __device__ __forceinline__ void load(u32x4 (&v)[kN], int k0, int k_at, int k_end) const {
        const uint32_t slab = slab_offset(k0, k_at, k_end, sk);
#pragma unroll
        for (int c = 0; c < kN; ++c)
            v[c] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, k_in[c] < k_end - k0 ? base[c] : kOutside, slab, 0);
    }
    static __device__ __forceinline__ void store(const u32x4 (&v)[kN], unsigned char* slab, int t) {
#pragma unroll
        for (int c = 0; c < kN; ++c) {
            const int id = t + GT * c;
            *reinterpret_cast<u32x4*>(slab + piece_offset<T, COL, W>(id / kPerRow, id % kPerRow)) = v[c];
        }
    }
};

// operand fragments of a slab: 32 indices from i0, quarter q of the slab's k.  bf16: the 16 k of one product; fp32:
// 8 k, lane half h holding k = 8q + 4h + {0..3}, i.e. four products of two k each.
template <typename T, bool COL, int W>
__device__ __forceinline__ auto read_frag(const unsigned char* slab, int i0, int q, int lane) {
    const int c = lane & 31, h = lane >> 5;
    if constexpr (sizeof(T) == 2) {
        if constexpr (!COL) {
            return *reinterpret_cast<const bf16x8*>(slab + piece_offset<T, false, W>(i0 + c, 2 * q + h));
        } else {
            // a group of 16 lanes turns a 4 (k) x 16 (index) block into 4 consecutive k per lane
            const int j = lane & 15, r = 16 * q + 8 * h + (j >> 2);
            const int pair = (i0 >> 4) + ((lane >> 4) & 1);
            const unsigned char* p = slab + piece_offset<T, true, W>(r, 2 * pair) + (j & 3) * 8;
            typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * 2 * W));
            s16x8 v;
            v[0] = lo[0]; v[1] = lo[1]; v[2] = lo[2]; v[3] = lo[3];
            v[4] = hi[0]; v[5] = hi[1]; v[6] = hi[2]; v[7] = hi[3];
            return __builtin_bit_cast(bf16x8, v);
        }
    } else {
        if constexpr (!COL) {
            return *reinterpret_cast<const f32x4*>(slab + piece_offset<T, false, W>(i0 + c, 2 * q + h));
        } else {
            const int i = i0 + c;
            const int r = 8 * q + 4 * h;   // bit 2 of rows r .. r + 3 is h
            const unsigned char* p = slab + (W == 64 ? r * 256 + (((i >> 2) ^ (h << 3)) << 4) + (i & 3) * 4 : r * 128 + i * 4);
            f32x4 v;
#pragma unroll
            for (int j = 0; j < 4; ++j)
                v[j] = *reinterpret_cast<const float*>(p + (W == 64 ? j * 256 : (h ? j ^ 1 : j) * 128));
            return v;
        }
    }
}
__device__ __forceinline__ void mma(f32x16& acc, bf16x8 a, bf16x8 b) {
    acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, acc, 0, 0, 0);
}
__device__ __forceinline__ void mma(f32x16& acc, f32x4 a, f32x4 b) {
#pragma unroll
    for (int j = 0; j < 4; ++j) acc = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], b[j], acc, 0, 0, 0);
}

template <int N, typename F, int I = 0>
__device__ __forceinline__ void unroll(F&& f) {
    if constexpr (I < N) {
        f(std::integral_constant<int, I>{});
        unroll<N, F, I + 1>(static_cast<F&&>(f));
    }
}

// wavefronts of a K group, and LDS bytes of it: two buffers of (A, B) slabs, later its stage
template <int TM, int TN> constexpr int group_waves() { return (TM / 32) * (TN / 32); }
template <int TM, int TN> constexpr int group_bytes() {
    return 2 * (TM + TN) * 128 > TM * (TN + kStagePad) * 4 ? 2 * (TM + TN) * 128 : TM * (TN + kStagePad) * 4;
}

template <typename T, int TM, int TN, bool A_COL, bool B_COL, int WK, typename Args>
__global__ __launch_bounds__((64 * group_waves<TM, TN>() * WK), TM == 64 && TN == 64 && WK == 1 ? 4 : 1) void gemm_tile64_kernel(Args g) {
    constexpr bool GROUPED = std::is_same<Args, Tile64Grouped>::value;
    static_assert(!GROUPED || (A_COL && B_COL && TM == 64 && TN == 64), "weight gradients: both operands with k strided");
    constexpr int BK = 128 / sizeof(T);
    constexpr int GW = group_waves<TM, TN>(), GT = 64 * GW, SA = TM * 128, SB = TN * 128;   // SA, SB: slab bytes
    constexpr int kStageStride = TN + kStagePad;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int lane = threadIdx.x & 63;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int kg = wave / GW, part = wave % GW;         // K group; 32x32 part of the tile
    const int t = threadIdx.x % GT;                     // thread within the K group
    const int wi = part / (TN / 32) * 32, wj = part % (TN / 32) * 32;

    int m0, n0, M, N, kb, ke, split, tile = 0, gi = 0;
    typedef Loader<T, A_COL, TM, GT> LA;
    typedef Loader<T, B_COL, TN, GT> LB;
    LA la;
    LB lb;
    auto same = [](int i) { return i; };
    if constexpr (GROUPED) {
        if ((int)blockIdx.x >= g.units) {
            tail_work<T>(g.tail, blockIdx.x - g.units, threadIdx.x, 256 * WK, smem);
            return;
        }
        // units: (split, tile), the tiles of one split next to each other
        const int total = g.units, xcd = blockIdx.x & 7, idx = blockIdx.x >> 3;
        const int u = xcd * (total >> 3) + min(xcd, total & 7) + idx;
        split = u / g.total_tiles;
        tile = u - split * g.total_tiles;
        while (gi + 1 < g.n && tile >= g.grp[gi + 1].tile0) ++gi;
        const Tile64Group& G = g.grp[gi];
        const int lt = tile - G.tile0;
        M = G.M;
        N = G.N;
        m0 = (lt % G.tiles_m) * 64;
        n0 = (lt / G.tiles_m) * 64;
        kb = split * g.slabs_per_split * BK;
        ke = min(g.K, kb + g.slabs_per_split * BK);
        la.init(G.A, 1, G.lda, m0, M, t, same);
        lb.init(G.B, 1, G.ldb, n0, N, t, same);
    } else {
        const int tiles_m = (g.M + TM - 1) / TM, tiles_n = (g.N + TN - 1) / TN;
        const int splits = g.partial ? g.splits : 1;
        int tm, tn;
        tile_of_block(blockIdx.x, tiles_m * tiles_n * splits, tiles_m, tiles_n, tm, tn, split);
        M = g.M;
        N = g.N;
        m0 = tm * TM;
        n0 = tn * TN;
        kb = 0;
        ke = g.K;
        if (splits > 1) {
            const int per = ((g.K + splits - 1) / splits + BK - 1) / BK * BK;
            kb = split * per;
            ke = min(g.K, kb + per);
        }
        la.init(g.A, g.a_rs, g.a_cs, m0, M, t, same);
        if (g.remap == REMAP_B_N) lb.init(g.B, g.b_cs, g.b_rs, n0, N, t, [&](int i) { return g.tbl(i); });
        else lb.init(g.B, g.b_cs, g.b_rs, n0, N, t, same);
    }

    // this group's slabs: kb + (kg + s * WK) * BK, s = 0 .. n_slabs - 1; a slab past the end loads zeros
    const int n_slabs = ke > kb ? ((ke - kb + BK - 1) / BK + WK - 1) / WK : 0;
    u32x4 ra[kAhead][LA::kN], rb[kAhead][LB::kN];
    auto fetch = [&](int s, u32x4 (&va)[LA::kN], u32x4 (&vb)[LB::kN]) {
        const int k0 = kb + (kg + s * WK) * BK;
        int k_at = k0;   // k of the slab as B is stored
        if constexpr (!GROUPED) {
            if (g.remap == REMAP_B_K && k0 < ke) k_at = g.tbl.start[k0 >> 6] + (k0 & 63);
        }
        la.load(va, k0, k0, ke);
        lb.load(vb, k0, k_at, ke);
    };
    unsigned char* const mine = smem + kg * group_bytes<TM, TN>();
    unroll<kAhead>([&](auto i) { fetch(i.value, ra[i.value], rb[i.value]); });
    // The thread's piece of the tile and what the epilogue reads for it, requested here, so that a launch of few workgroups
    // does not end with the latency of one more load.  The larger tiles have no registers for it.  bf16, in passes of eight
    // models: 248 workgroups of 32x32 5.30 -> 4.91 us, 186 of 64x32 5.61 -> 5.40, three rounds (768 of 64x32) 10.26 -> 10.07, none slower
    // by more than its runs differ.  fp32: only where each workgroup has a CU of its own; in later
    // rounds others cover that latency, and the slabs wait behind these loads (913 x 832 x 3328 with bias and residual, 754
    // workgroups, 48.4 us without and 51.8 with).
    constexpr bool kEarly = !GROUPED && TN == 32 && (TM == 32 || sizeof(T) == 2);
    const bool ahead = sizeof(T) == 2 || gridDim.x <= 256;
    constexpr int kThreads = GT * WK, kPieces = TM * TN / 8, kRowPieces = TN / 8;
    const int r0 = threadIdx.x / kRowPieces, c0 = threadIdx.x % kRowPieces * 8;
    EpilogueOperands<T> early;
    if constexpr (kEarly) {
        if (ahead && !g.partial && (kThreads <= kPieces || (int)threadIdx.x < kPieces) && m0 + r0 < M && n0 + c0 < N) early.request(g, m0 + r0, n0 + c0);
    }
    f32x16 acc;
#pragma unroll
    for (int e = 0; e < 16; ++e) acc[e] = 0.f;
    if (n_slabs > 0) {
        LA::store(ra[0], mine, t);
        LB::store(rb[0], mine + SA, t);
        fetch(kAhead, ra[0], rb[0]);
    }
    // slab s sits in LDS buffer s & 1, slabs s + 1 .. s + kAhead in registers (slab x in slot x % kAhead).  One
    // barrier per slab: behind it the stores of slab s are visible and buffer (s + 1) & 1 is free.  A group of one
    // wavefront shares its slabs with no other, and its LDS accesses complete in order: a fence at wavefront scope,
    // which costs no instruction, keeps the compiler from moving one lane's reads over another lane's stores.
    auto step = [&](int s, auto slot_tag) {
        constexpr int slot = decltype(slot_tag)::value;
        unsigned char* const cur = mine + (s & 1) * (SA + SB);
        unsigned char* const nxt = mine + ((s + 1) & 1) * (SA + SB);
        if constexpr (GW > 1) {
            __syncthreads();
        } else {
            __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
            __builtin_amdgcn_wave_barrier();
        }
        decltype(read_frag<T, A_COL, TM>(cur, 0, 0, 0)) fa[4];
        decltype(read_frag<T, B_COL, TN>(cur, 0, 0, 0)) fb[4];
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            fa[q] = read_frag<T, A_COL, TM>(cur, wi, q, lane);
            fb[q] = read_frag<T, B_COL, TN>(cur + SA, wj, q, lane);
        }
        if (s + 1 < n_slabs) {
            LA::store(ra[slot], nxt, t);
            LB::store(rb[slot], nxt + SA, t);
            fetch(s + 1 + kAhead, ra[slot], rb[slot]);
        }
#pragma unroll
        for (int q = 0; q < 4; ++q) mma(acc, fa[q], fb[q]);
    };
    for (int s = 0; s < n_slabs; s += kAhead)
        unroll<kAhead>([&](auto i) {
            if (s + i.value < n_slabs) step(s + i.value, std::integral_constant<int, (i.value + 1) % kAhead>{});
        });
    __syncthreads();   // the stage below reuses the operand buffers

    // ---- epilogue: the groups' sums meet in LDS, results leave as 8 consecutive columns per thread ----
    float* const stage = reinterpret_cast<float*>(mine);
    {
        const int c = lane & 31, h = lane >> 5;
#pragma unroll
        for (int e = 0; e < 16; ++e) stage[(wi + 8 * (e >> 2) + 4 * h + (e & 3)) * kStageStride + wj + c] = acc[e];
    }
    __syncthreads();
    float csum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) csum[i] = 0.f;
#pragma unroll 1   // short code: a launch fetches its instructions from memory
    for (int p0 = 0; p0 < kPieces; p0 += kThreads) {
        const int p = p0 + threadIdx.x;
        if (kThreads > kPieces && p >= kPieces) break;
        const int r = p / kRowPieces, cc = p % kRowPieces * 8;
        const int m = m0 + r, n = n0 + cc;
        float v[8];
        load8(reinterpret_cast<float*>(smem) + r * kStageStride + cc, v);
#pragma unroll
        for (int w = 1; w < WK; ++w) {
            float o[8];
            load8(reinterpret_cast<float*>(smem + w * group_bytes<TM, TN>()) + r * kStageStride + cc, o);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] += o[i];
        }
        if constexpr (GROUPED) {
            if (g.splits > 1) {
                store8(g.partial + ((long)split * g.total_tiles + tile) * 4096 + r * 64 + cc, v);
            } else if (m < M && n < N) {
                emit_grouped<T>(g, gi, m, n, v);
            }
        } else if (m < M && n < N) {
            if (g.partial) {
                store8(g.partial + (long)split * M * N + (long)m * N + n, v);
                continue;
            }
            if constexpr (kEarly) {
                static_assert(kThreads >= kPieces, "one piece per thread");
                if (!ahead) early.request(g, m, n);
                emit<T>(g, m, n, v, early);
            } else {
                emit<T>(g, m, n, v);
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) csum[i] += v[i];
        }
    }
    if constexpr (!GROUPED) {
        if (!g.colsum) return;   // uniform over the grid
        // column sums of the tile's rows: lanes kRowPieces apart share their columns, then the wavefronts in order
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float s = csum[i];
#pragma unroll
            for (int w = kRowPieces; w < 64; w <<= 1) s += __shfl_xor(s, w, 64);
            csum[i] = s;
        }
        __syncthreads();
        float* const red = reinterpret_cast<float*>(smem);
        constexpr int kWaves = (kThreads < kPieces ? kThreads : kPieces) / 64;   // wavefronts that hold results
        if (lane < kRowPieces && wave < kWaves) store8(red + wave * TN + lane * 8, csum);
        __syncthreads();
        if (threadIdx.x < TN && n0 + (int)threadIdx.x < N) {
            float s = 0.f;
#pragma unroll
            for (int w = 0; w < kWaves; ++w) s += red[w * TN + threadIdx.x];
            g.colsum[(long)(g.colsum_row0 + m0 / TM) * N + n0 + threadIdx.x] = s;
        }
    }
}

// sums of a grouped launch with more than one split: the splits of a tile are added in split order.  blockIdx.x =
// tile, a thread owns 4 consecutive columns of every 16th row.
template <typename T>
__global__ __launch_bounds__(256) void reduce_tile64_kernel(Tile64Grouped g) {
    const int tile = blockIdx.x;
    int gi = 0;
    while (gi + 1 < g.n && tile >= g.grp[gi + 1].tile0) ++gi;
    const Tile64Group& G = g.grp[gi];
    const int lt = tile - G.tile0;
    const int r0 = blockIdx.y * 16 + (threadIdx.x >> 4), c = (threadIdx.x & 15) * 4;
    const int m = (lt % G.tiles_m) * 64 + r0, n = (lt / G.tiles_m) * 64 + c;
    if (m >= G.M || n >= G.N) return;
    const float* src = g.partial + (long)tile * 4096 + r0 * 64 + c;
    const long stride = (long)g.total_tiles * 4096;
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
    if (G.remap == RED_REMAP_F32) {
        *reinterpret_cast<f32x4*>(static_cast<float*>(G.out) + (long)m * G.ldo + n) = s;
        return;
    }
    const int mo = G.remap == RED_REMAP_ROWS ? g.tbl[G.table][m >> 6] * 64 + (m & 63) : m;
    const int no = G.remap == RED_REMAP_COLS ? g.tbl[G.table][n >> 6] * 64 + (n & 63) : n;
    T* o = static_cast<T*>(G.out) + (long)mo * G.ldo + no;
#pragma unroll
    for (int i = 0; i < 4; ++i) {
        float v = s[i];
        if (g.accumulate) v += ld<T>(o + i);
        st<T>(o + i, v);
    }
}

struct KernelName {
    char s[96];
    KernelName(const char* type, int tm, int tn, bool a_col, bool b_col, int wk, bool grouped) {
        snprintf(s, sizeof(s), "gemm_tile64_kernel<%s, %d, %d, %s, %s, %d, d2ft::%s>", type, tm, tn, a_col ? "true" : "false",
                 b_col ? "true" : "false", wk, grouped ? "Tile64Grouped" : "GemmArgs");
    }
};

template <typename T, int TM, int TN, bool A_COL, bool B_COL, int WK, typename Args>
hipError_t launch_wk(unsigned grid, hipStream_t s, const Args& a) {
    static const KernelName name(sizeof(T) == 4 ? "float" : "__bf16", TM, TN, A_COL, B_COL, WK, std::is_same<Args, Tile64Grouped>::value);
    launch_label(name.s);
    auto kern = gemm_tile64_kernel<T, TM, TN, A_COL, B_COL, WK, Args>;
    constexpr int lds = WK * group_bytes<TM, TN>(), threads = 64 * group_waves<TM, TN>() * WK;
    if constexpr (lds > 64 * 1024) {
        static std::atomic<uint32_t> set_on{0};   // devices, one bit each: the attribute belongs to a device's copy of the kernel
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev >= 32 || !(set_on.load() >> dev & 1)) {
            e = hipFuncSetAttribute(reinterpret_cast<const void*>(kern), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
            if (e != hipSuccess) return e;
            if (dev < 32) set_on.fetch_or(1u << dev);
        }
    }
    return launch_signalling(kern, dim3(grid), dim3(threads), lds, s, a);
}

template <typename T, int TM, int TN, bool A_COL, bool B_COL, typename Args>
hipError_t launch_form(int wk, unsigned grid, hipStream_t s, const Args& a) {
    if constexpr (TM * TN == 64 * 64) {
        if (wk == 1) return launch_wk<T, TM, TN, A_COL, B_COL, 1>(grid, s, a);
    }
    if constexpr (TM * TN == 32 * 32 && sizeof(T) == 2) {
        if (wk == 8) return launch_wk<T, TM, TN, A_COL, B_COL, 8>(grid, s, a);
    }
    if (wk == 4) return launch_wk<T, TM, TN, A_COL, B_COL, 4>(grid, s, a);
    return launch_wk<T, TM, TN, A_COL, B_COL, 2>(grid, s, a);
}

// K groups per workgroup: as many as it takes to give every CU two workgroups' worth of wavefronts, as long as each
// group keeps two slabs to multiply
int pick_wk(long units, int slabs) {
    int wk = 1;
    while (wk < 4 && units * wk < 512 && slabs >= 4 * wk) wk *= 2;
    return wk;
}


}  // namespace

bool gemm_tile64_supported(const GemmArgs& g, int dtype) {
    const long es = dtype == D2FT_F32 ? 4 : 2;
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
    const bool a_row = (g.a_cs == 1), a_col = (g.a_rs == 1), b_row = (g.b_rs == 1), b_col = (g.b_cs == 1);
    if (!(a_row || a_col) || !(b_row || b_col) || (!a_row && b_row)) return false;
    if (a_row ? !(mult8(g.K) && mult8(g.a_rs)) : !(mult8(g.M) && mult8(g.a_cs))) return false;
    if (b_row ? !(mult8(g.K) && mult8(g.b_cs)) : !mult8(g.b_rs)) return false;
    if (!al16(g.A) || !al16(g.B) || !mult8(g.N)) return false;
    const long a_span = a_row ? (long)g.M * g.a_rs : (long)g.K * g.a_cs;
    long b_n = g.N, b_k = g.K;   // extents of B as stored (through the remap, if any)
    if (g.remap != REMAP_NONE) {
        const int nblk = ((g.remap == REMAP_B_N ? g.N : g.K) + 63) / 64;
        if (nblk > kMaxBlocks64) return false;
        long top = 0;
        for (int i = 0; i < nblk; ++i) {
            if (g.tbl.start[i] < 0) return false;
            if (g.tbl.start[i] + 64 > top) top = g.tbl.start[i] + 64;
        }
        (g.remap == REMAP_B_N ? b_n : b_k) = top;
    }
    const long b_span = b_row ? b_n * g.b_cs : b_k * g.b_rs;
    if (a_span * es >= (1L << 31) || b_span * es >= (1L << 31)) return false;   // 32-bit byte offsets
    if ((long)((g.M + 63) / 64) * ((g.N + 63) / 64) * (g.partial ? g.splits : 1) > 0x7fffffffL) return false;
    if (g.colsum && (g.partial || !al16(g.colsum))) return false;
    if (g.partial) return al16(g.partial);
    if (!g.C || !al16(g.C) || !mult8(g.ldc)) return false;
    if (g.bias && !al16(g.bias)) return false;
    if (g.residual && (!al16(g.residual) || !mult8(g.ldr))) return false;
    if (g.act != ACT_NONE && (!g.Z || !al16(g.Z) || !mult8(g.ldz))) return false;
    return true;
}

// Tile and K groups of a product without split-K partials: the cheapest of the kernel's forms in microseconds,
//   fixed + slabs * first + (rounds - 1) * (slabs * next + change) + rounds * gelu,   rounds = workgroups per CU, rounded up:
// a first round that waits for its loads, further ones beside it.  Fitted on this part, bf16 to 1766 shapes (M 17 .. 12608,
// N and K 64 .. 8192; rms error 5 to 8 %), fp32 to some 150 (M 64 .. 3152, N and K 64 .. 4096).  bf16: a CU's loads set the pace, so a slab costs in proportion to the tile's rows
// + columns and a small tile pays where large ones leave CUs idle: 197 x 768 x 3072, 64x64 tiles 16.2 us, 64x32 12.3,
// 32x32 8.9; 985 x 384 x 1536: 10.3, 8.6, 8.9; 985 x 2304 x 768: 13.6, 15.2, 17.2.  Eight K groups of a 32x32 tile have twice
// the slabs in flight and more sums to add: 197 x 768 x 3072 8.8 -> 8.4 us, x 4096 10.4 -> 9.4, x 2304 none.  fp32: the matrix cores, so a slab
// costs in proportion to the tile's area and what a small tile saves is the last, partly empty round: 197 x 2304 x 768:
// 19.5, 20.7, 12.8; 3152 x 384 x 1536: 61, 51, 46; 3152 x 1536 x 384: 47.9, 52.4, 56.6.
struct Tile64Form {
    int tm, tn, wk;
    float fixed, first, next, change, gelu;   // us
};
constexpr Tile64Form kFormsBf16[] = {{64, 64, 1, 3.71f, 0.370f, 0.183f, 0.77f, 0.77f}, {64, 64, 2, 3.91f, 0.262f, 0.208f, 1.24f, 0.77f},
                                     {64, 32, 2, 3.67f, 0.217f, 0.133f, 0.77f, 0.36f}, {64, 32, 4, 4.47f, 0.171f, 0.181f, 2.99f, 0.75f},
                                     {32, 32, 2, 3.49f, 0.168f, 0.082f, 0.55f, 0.19f}, {32, 32, 4, 3.94f, 0.111f, 0.084f, 1.22f, 0.33f},
                                     {32, 32, 8, 5.55f, 0.061f, 0.1f, 10.0f, 0.33f}};   // one to a CU
constexpr Tile64Form kFormsF32[] = {{64, 64, 1, 4.4f, 0.61f, 0.52f, 3.0f, 0.0f}, {64, 32, 2, 3.4f, 0.37f, 0.26f, 1.9f, 0.0f},
                                    {32, 32, 2, 3.2f, 0.30f, 0.145f, 1.1f, 0.0f}, {32, 32, 4, 3.9f, 0.18f, 0.145f, 1.4f, 0.0f}};
static Tile64Form pick_form(const GemmArgs& g, int dtype, float* us) {
    const bool f32 = dtype == D2FT_F32;
    const Tile64Form* f = f32 ? kFormsF32 : kFormsBf16;
    const int slabs = f32 ? (g.K + 31) / 32 : (g.K + 63) / 64;
    Tile64Form best = f[0];
    *us = 1e30f;
    for (int i = 0; i < (f32 ? 4 : 7); ++i) {
        if (g.colsum && f[i].tm != 64) continue;   // a band of column sums is 64 rows
        const long units = (long)((g.M + f[i].tm - 1) / f[i].tm) * ((g.N + f[i].tn - 1) / f[i].tn);
        const float rounds = (float)((units + 255) / 256);
        const float t = f[i].fixed + f[i].first * slabs + (rounds - 1.0f) * (f[i].next * slabs + f[i].change) + (g.act == ACT_GELU ? rounds * f[i].gelu : 0.0f);
        if (t < *us) {
            *us = t;
            best = f[i];
        }
    }
    return best;
}

template <typename T, int TM, int TN>
static hipError_t launch_tile(const GemmArgs& g, int wk, hipStream_t s) {
    const unsigned units = (unsigned)((g.M + TM - 1) / TM) * (unsigned)((g.N + TN - 1) / TN);
    return g.b_rs == 1 ? launch_form<T, TM, TN, false, false>(wk, units, s, g) : launch_form<T, TM, TN, false, true>(wk, units, s, g);
}

template <typename T>
static hipError_t launch_tile64(const GemmArgs& g, int dtype, hipStream_t s) {
    if constexpr (std::is_same<T, float>::value) {   // bf16: gemm_tile64_faster takes neither
        if (g.partial || g.a_cs != 1) {
            const long units = (long)((g.M + 63) / 64) * ((g.N + 63) / 64) * (g.partial ? g.splits : 1);
            const int slabs = (g.K / (g.partial ? g.splits : 1) + 31) / 32;
            const int wk = pick_wk(units, slabs);
            if (g.a_cs != 1) return launch_form<T, 64, 64, true, true>(wk, (unsigned)units, s, g);
            return g.b_rs == 1 ? launch_form<T, 64, 64, false, false>(wk, (unsigned)units, s, g) : launch_form<T, 64, 64, false, true>(wk, (unsigned)units, s, g);
        }
    }
    float us;
    const Tile64Form f = pick_form(g, dtype, &us);
    // fp32 by bf16 parts: 15760 x 1536 x 384 with the GELU epilogue 140 us (212 here), 3152 x 384 x 1536 59 and 48
    if (std::is_same<T, float>::value && gemm_split_us(g) < us) return launch_gemm_split(g, s);
    if (f.tm == 32) return launch_tile<T, 32, 32>(g, f.wk, s);
    if (f.tn == 32) return launch_tile<T, 64, 32>(g, f.wk, s);
    return launch_tile<T, 64, 64>(g, f.wk, s);
}

// bf16: against the 128x128 tile with a CU for each workgroup, by a fitted cost (1086 products, rms error 5 %).  In the middle
// of the range both are close (985 x 1536 x 384: 9.2 and 10.4 us); at the ends they are not (197 x 768 x 768: 5.0 and 9.5;
// 1576 x 768 x 3072: 37 and 25).  Where that tile has more workgroups than the chip CUs, it leaves none idle (8192 x 576 x 256,
// 320 workgroups: 9.7 us and 11.4 on 64x64 tiles; 3152 x 3072 x 768: 27 and 46).
bool gemm_tile64_faster(const GemmArgs& g) {
    if (g.partial || g.a_cs != 1 || gemm_mfma_tile_rows(g) != 128) return false;
    const long units = (long)((g.M + 127) / 128) * ((g.N + 127) / 128);
    if (units > 256) return false;
    float us;
    pick_form(g, D2FT_BF16, &us);
    const float slabs = (float)((g.K + 63) / 64), epilogue = g.act == ACT_GELU ? 2.6f : 0.0f;
    return us < 0.95f * (5.2f + 0.365f * slabs * (1.0f + 0.404f * (float)units / 256.0f) + epilogue);
}

hipError_t launch_gemm_tile64(const GemmArgs& g, int dtype, hipStream_t s) {
    if (!gemm_tile64_supported(g, dtype)) return hipErrorNotSupported;
    return dtype == D2FT_F32 ? launch_tile64<float>(g, dtype, s) : launch_tile64<bf16>(g, dtype, s);
}

// out_g = A_g^T B_g for the groups of g (grp, n_groups, K, partial), through r's remaps: one launch, and a reduction
// behind it if K is split.  partial_floats: size of g.partial.
hipError_t launch_gemm_tile64_grouped(const GemmArgs& g, const ReduceGroupedArgs& r, int dtype, int accumulate,
                                      size_t partial_floats, TailJobs* tail, hipStream_t s) {
    const long es = dtype == D2FT_F32 ? 4 : 2;
    if (g.n_groups < 1 || g.n_groups > kMaxGemmGroups || g.K <= 0) return hipErrorNotSupported;
    Tile64Grouped a;
    a.n = g.n_groups;
    a.K = g.K;
    a.accumulate = accumulate;
    a.partial = g.partial;
    long tiles = 0;
    for (int i = 0; i < g.n_groups; ++i) {
        const GemmGroup& G = g.grp[i];
        if (G.M <= 0 || G.N <= 0 || !al16(G.A) || !al16(G.B) || !mult8(G.M) || !mult8(G.N) || !mult8(G.lda) || !mult8(G.ldb)) return hipErrorNotSupported;
        if ((long)g.K * G.lda * es >= (1L << 31) || (long)g.K * G.ldb * es >= (1L << 31)) return hipErrorNotSupported;
        Tile64Group& o = a.grp[i];
        o.A = G.A; o.B = G.B; o.out = r.grp[i].out;
        o.lda = G.lda; o.ldb = G.ldb; o.ldo = r.grp[i].ldo;
        o.M = G.M; o.N = G.N;
        o.tiles_m = (G.M + 63) / 64;
        o.tile0 = (int)tiles;
        o.remap = r.grp[i].remap; o.table = r.grp[i].table;
        tiles += (long)o.tiles_m * ((G.N + 63) / 64);
        if (tiles > (1 << 20)) return hipErrorNotSupported;
    }
    for (int i = 0; i < 3; ++i)
        for (int j = 0; j < kMaxBlocks64; ++j) a.tbl[i][j] = (uint16_t)(r.tbl[i].start[j] >> 6);
    a.total_tiles = (int)tiles;
    // Splits of K: enough units for four workgroups per CU (bf16: one, its partial sums cost more than an idle slot),
    // while each keeps eight slabs and the partial tiles fit
    const int bk = 128 / (int)es, slabs = (g.K + bk - 1) / bk, enough = dtype == D2FT_F32 ? 1024 : 256;
    int splits = 1;
    while (splits < 64 && tiles * splits < enough && slabs / (splits + 1) >= 8 && (size_t)(splits + 1) * tiles * 4096 <= partial_floats) ++splits;
    a.slabs_per_split = (slabs + splits - 1) / splits;
    a.splits = (slabs + a.slabs_per_split - 1) / a.slabs_per_split;
    const long units = tiles * a.splits;
    const int wk = pick_wk(units, a.slabs_per_split);
    a.units = (int)units;
    a.tail.blocks = 0;
    if (tail) {
        tail_blocks(tail);
        a.tail = *tail;
    }
    if (dtype == D2FT_F32) {   // by bf16 parts, or here (one K group per workgroup at these sizes)
        Tile64Grouped b = a;
        const float us = gemm_split_grouped_plan(&b, partial_floats);
        const float here = 4.4f + 0.61f * a.slabs_per_split + (float)((units + 255) / 256 - 1) * (0.52f * a.slabs_per_split + 3.0f) + (a.splits > 1 ? 4.0f : 0.0f);
        if (us < here) return launch_gemm_split_grouped(b, s);
    }
    const unsigned grid_all = (unsigned)(units + a.tail.blocks);
    hipError_t e = dtype == D2FT_F32 ? launch_form<float, 64, 64, true, true>(wk, grid_all, s, a)
                                     : launch_form<bf16, 64, 64, true, true>(wk, grid_all, s, a);
    if (e != hipSuccess || a.splits == 1) return e;
    const dim3 grid((unsigned)tiles, 4);
    if (dtype == D2FT_F32) hipLaunchKernelGGL(reduce_tile64_kernel<float>, grid, dim3(256), 0, s, a);
    else hipLaunchKernelGGL(reduce_tile64_kernel<bf16>, grid, dim3(256), 0, s, a);
    return hipGetLastError();
}

}  // namespace d2ft
