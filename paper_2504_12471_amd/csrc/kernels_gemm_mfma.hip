// bf16 GEMM on the CDNA4 matrix cores (v_mfma_f32_32x32x16_bf16, fp32 accumulate).
//
//   C[m][n] = epilogue( sum_k A(m,k) * B(k,n) )
//
// A workgroup of WGM x WGN wavefronts owns a BM x BN tile of C at a time (256x256 and 192x256 with
// 2 x 4 wavefronts, one workgroup per CU; 128x128 with 2 x 2, two per CU); each wavefront owns
// (BM/WGM) x (BN/WGN) of it as a grid of 32x32 MFMA tiles.  K is consumed BK at a time: the slab
// after next is fetched from global memory into registers while the current one is multiplied
// out of LDS and the next one is written to the other LDS buffer (one barrier per slab).
// Workgroups are persistent: the grid is what the chip holds at once and each walks its tiles.
//
// Either operand may be stored with K contiguous ("row" form: A[m][k], B[n][k]) or with its
// other index contiguous ("col" form: A[k][m], B[k][n]).  The MFMA wants 8 consecutive k per
// lane.  Row-form slabs are stored in LDS as [index][k] and read with one 128-bit load per
// fragment; col-form slabs are stored as [k][index] and read with two transposing LDS loads
// (ds_read_b64_tr_b16), so no operand is ever transposed in global memory.
//
// B's n or k index may go through a 64-granular remap table: that is how the compacted
// live-head list selects rows / columns of the full weight tensors without copying them.
#include <cstdio>
#include <type_traits>

#include "gemm_large.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;

namespace {


// LDS row strides (in bf16 elements), chosen so that the fragment reads are bank-conflict free
template <int BK> constexpr int row_form_stride() { return BK + 8; }          // [index][k]: +16 bytes
template <int BI> constexpr int col_form_stride() { return BI + 32; }         // [k][index]: +64 bytes

// elements of one slab buffer; the last row of a col-form slab carries no padding, which is what lets
// two 128x128 workgroups with both operands in col form share a CU's 160 KB
template <int BI, int BK, bool COL> constexpr int slab_elems() {
    return COL ? (BK - 1) * col_form_stride<BI>() + BI : BI * row_form_stride<BK>();
}

// ---- global -> registers: one slab of an operand, 16-byte chunks, zero fill outside the matrix ----
// ROW form: element (i, k) at base + i*s_i + k          (k contiguous, s_k == 1)
// COL form: element (i, k) at base + k*s_k + i          (i contiguous, s_i == 1)
// Loads are raw buffer loads: a chunk outside the matrix gets an offset beyond the buffer's
// declared size, for which the hardware returns zeros without touching memory, so there is no
// branch and no select in the loop.  The part of the address that does not change from slab to
// slab (the index part) is computed once.
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;
// LDS is addressed through pointers that carry the LDS address space: their arithmetic is 32-bit and
// constant offsets fold into the instructions' offset fields (generic pointers cost a null check and a
// 64-bit select per use)
typedef __attribute__((address_space(3))) bf16 lds_bf16;
template <int BI, int BK, bool COL, int kThreads>
struct SlabLoader {
    static constexpr int kChunks = BI * BK / 8;
    static constexpr int kPerThread = kChunks / kThreads;
    static_assert(kChunks % kThreads == 0, "slab must divide over the workgroup");
    static_assert(BK == 64, "the k remap is resolved once per slab, which needs 64-aligned slabs");
    // COL form with the thread count a multiple of the chunks per k row: a thread's chunks all have the
    // same index part and k rows a fixed distance apart, so one offset register serves them all and the
    // distance goes into the load's scalar offset
    static constexpr bool kOneBase = COL && (kThreads % (BI / 8) == 0);
    static constexpr int kBases = kOneBase ? 1 : kPerThread;
    static constexpr int kRowStep = kThreads / (BI / 8);   // kOneBase: k rows between a thread's consecutive chunks
    u32x4 v[kPerThread];
    uint32_t base[kBases];   // byte offset of the chunk within slab 0, kOutside if its index is outside
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t sk_bytes;

    static __device__ __forceinline__ int k_local(int c) {
        const int id = threadIdx.x + c * kThreads;
        return COL ? id / (BI / 8) : (id % (BK / 8)) * 8;
    }

    template <bool REMAP_I>
    __device__ __forceinline__ void init(const bf16* p, long s_i, long s_k, int i0, int I, const Remap64& tbl) {
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(p), 0, kBufBytes, 0x00020000);
        sk_bytes = (uint32_t)s_k * 2u;
#pragma unroll
        for (int c = 0; c < kBases; ++c) {
            const int id = threadIdx.x + c * kThreads;
            const int i = i0 + (COL ? (id % (BI / 8)) * 8 : id / (BK / 8));
            const int is = REMAP_I ? tbl(min(i, I - 1)) : i;
            const uint32_t off = ((uint32_t)is * (uint32_t)s_i + (uint32_t)k_local(c) * (uint32_t)s_k) * 2u;
            base[c] = (i < I) ? off : kOutside;
        }
    }

    // slab starting at k0 (a multiple of 64 counted from 0), valid k < k_end; chunk c alone, or all chunks
    // TAIL: the slab may reach beyond k_end (K is not a multiple of 64), so every chunk checks its k
    template <bool REMAP_K, bool TAIL>
    __device__ __forceinline__ void load_one(int c, int k0, int k_end, const Remap64& tbl) {
        const uint32_t kstart = REMAP_K ? (uint32_t)tbl.start[k0 >> 6] : (uint32_t)k0;
        uint32_t koff = kstart * sk_bytes;   // uniform over the workgroup
        if constexpr (kOneBase) koff += (uint32_t)(c * kRowStep) * sk_bytes;
        if constexpr (kOneBase && TAIL) koff = min(koff, kBufBytes - 1u);   // rows past the end: see the bounds check above
        const uint32_t mine = base[kOneBase ? 0 : c];
        const uint32_t off = (!TAIL || k_local(c) < k_end - k0) ? mine : kOutside;
        v[c] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, off, koff, 0);
    }
    template <bool REMAP_K, bool TAIL>
    __device__ __forceinline__ void load(int k0, int k_end, const Remap64& tbl) {
#pragma unroll
        for (int c = 0; c < kPerThread; ++c) load_one<REMAP_K, TAIL>(c, k0, k_end, tbl);
    }

    __device__ __forceinline__ void store_one(int c, lds_bf16* lds) const {
        const int id = threadIdx.x + c * kThreads;
        int off;
        if (COL) {
            off = (id / (BI / 8)) * col_form_stride<BI>() + (id % (BI / 8)) * 8;
        } else {
            off = (id / (BK / 8)) * row_form_stride<BK>() + (id % (BK / 8)) * 8;
        }
        *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(lds + off) = v[c];
    }
    __device__ __forceinline__ void store(lds_bf16* lds) const {
#pragma unroll
        for (int c = 0; c < kPerThread; ++c) store_one(c, lds);
    }
};

// ---- LDS -> MFMA operand fragment: rows i_base + lane%32, k = kk + 8*(lane/32) .. +7 ----
// The address is split into a part that depends on the lane and the wavefront (computed once per
// kernel, one register) and a compile-time part (buffer, MFMA tile, k step) that goes into the
// instruction's offset field.
template <int BI, int BK, bool COL>
__device__ __forceinline__ int fragment_lane_offset(int i_wave, int lane) {
    if (!COL) return (i_wave + (lane & 31)) * row_form_stride<BK>() + 8 * (lane >> 5);
    // transposing read: a group of 16 lanes turns a 4 (k) x 16 (index) block into 4 consecutive k per lane;
    // lane j of the group supplies the address of row k = j/4, columns 4*(j%4) .. +3
    const int j = lane & 15;
    return (8 * (lane >> 5) + (j >> 2)) * col_form_stride<BI>() + i_wave + 16 * ((lane >> 4) & 1) + 4 * (j & 3);
}
template <int BI, int BK, bool COL>
__device__ __forceinline__ bf16x8 read_fragment(const lds_bf16* lane_base, int i_tile, int kk) {
    if (!COL) {
        const lds_bf16* p = lane_base + (i_tile * row_form_stride<BK>() + kk);
        return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p);
    } else {
        const lds_bf16* p = lane_base + (kk * col_form_stride<BI>() + i_tile);
        typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
        const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
        const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 4 * col_form_stride<BI>()));
        typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
        s16x8 r;
        r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
        r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
        return __builtin_bit_cast(bf16x8, r);
    }
}

// ---- issue order of one MFMA group ----
// A group is NM MFMAs with, between them, the NR LDS reads of the next group's fragments and NS LDS
// stores of the next slab, each store followed by the global load that refills its registers.  The
// reads ride on the first MFMAs of the group so that every fragment has at least two MFMAs of time to
// arrive before the next group starts; the stores follow (LDS reads cannot be moved across LDS
// stores: the compiler must assume the buffers alias).  Expressed as scheduling-group barriers.
template <int NM, int NR, int NS, int I = 0>
__device__ __forceinline__ void pace_group() {
    constexpr int RA0 = NS > 0 ? NM / 2 : NM - 2;
    constexpr int RA = RA0 > 0 ? RA0 : 1;   // MFMAs that carry the reads
    if constexpr (I < NM) {
        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
        if constexpr (I < RA) {
            constexpr int nr = (I + 1) * NR / RA - I * NR / RA;
            if constexpr (nr > 0) __builtin_amdgcn_sched_group_barrier(0x100, nr, 0);   // LDS read
        } else if constexpr (NS > 0) {
            constexpr int J = I - RA, NB = NM - RA;
            constexpr int nw = (J + 1) * NS / NB - J * NS / NB;
            if constexpr (nw > 0) {
                __builtin_amdgcn_sched_group_barrier(0x200, nw, 0);   // LDS store
                __builtin_amdgcn_sched_group_barrier(0x020, nw, 0);   // global load
            }
        }
        pace_group<NM, NR, NS, I + 1>();
    }
}

// bytes of the epilogue's fp32 stage: one 32-row band of every wavefront's tile, rows padded by 4 floats
template <int BN, int WGM, int WGN> constexpr size_t stage_bytes() {
    return (size_t)WGM * WGN * 32 * (BN / WGN + 4) * sizeof(float);
}

// epilogues with an instantiation of their own: C = (A B) * Z (the backward's dz) and C = A B + bias + R (the
// products that close a residual branch); both fetch their operand a band ahead
enum { EPI_ANY = 0, EPI_DGELU = 1, EPI_RESIDUAL = 2 };

template <int BM, int BN, int BK, int WGM, int WGN, bool A_COL, bool B_COL, int REMAP, bool KTAIL, bool SEGMENTS = false,
          int EPI = EPI_ANY>
__global__ __launch_bounds__(64 * WGM * WGN, 2) void gemm_mfma_kernel(GemmArgs g) {
    constexpr int kThreads = 64 * WGM * WGN;    // WGM x WGN wavefronts
    constexpr bool KSEG = REMAP == REMAP_B_KSEG;    // K walk over the positions of the tile's row segments
    constexpr bool REMAP_BK = REMAP == REMAP_B_K || KSEG;
    static_assert(!KSEG || (!KTAIL && !SEGMENTS && !A_COL), "the K-segment form: A row-major, K a multiple of 64");
    constexpr int WTM = BM / WGM, WTN = BN / WGN;   // wavefront tile
    constexpr int MT = WTM / 32, NT = WTN / 32; // MFMA tiles per wavefront
    constexpr int A_ELEMS = slab_elems<BM, BK, A_COL>();
    constexpr int B_ELEMS = slab_elems<BN, BK, B_COL>();
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    lds_bf16* const smem = (lds_bf16*)smem_raw;
    constexpr int STAGE_ELEMS = A_ELEMS + B_ELEMS;   // LDS buffer p: A slab at p * STAGE_ELEMS, B slab behind it

    const bf16* __restrict__ A = static_cast<const bf16*>(g.A);
    const bf16* __restrict__ B = static_cast<const bf16*>(g.B);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int wm = wave / WGN, wn = wave % WGN;
    // K-segment form: every segment has tile rows of its own (g.seg.live_tiles of them in all), so that no tile
    // has rows of two segments
    const int tiles_m = REMAP == REMAP_B_KSEG ? g.seg.live_tiles : (g.M + BM - 1) / BM, tiles_n = (g.N + BN - 1) / BN;
    const int total = SEGMENTS ? g.seg.live_tiles : tiles_m * tiles_n * (g.partial ? g.splits : 1);

    f32x16 acc[MT][NT];
    SlabLoader<BM, BK, A_COL, kThreads> la;
    SlabLoader<BN, BK, B_COL, kThreads> lb;

    // The kernel is persistent: workgroup b works on tiles b, b + gridDim.x, ... (the grid is a
    // multiple of 8, so all of them map to its own XCD's range).  setup_tile fixes a tile's
    // coordinates and K range and fetches its first slab into the loader registers; it is called for
    // the next tile ahead of the current tile's epilogue, and the epilogue's global stores drain while
    // the next tile is being multiplied.
    int m0 = 0, n0 = 0, split = 0, kb = 0, ke = 0, nslabs = 0;
    // K-segment form: the positions still to walk (the lowest set bit is the current one), the 64-wide block
    // within the current position, and k of the next slab to fetch
    uint64_t kseg_left = 0;
    int kseg_sub = 0, kseg_k = 0, mlim = 0;   // mlim: the end of the tile's segment
    auto kseg_advance = [&]() {
        if (++kseg_sub * BK >= g.seg.slice) {
            kseg_sub = 0;
            kseg_left &= kseg_left - 1;
            kseg_k = kseg_left ? __builtin_ctzll(kseg_left) * g.seg.slice : 0;
        } else {
            kseg_k += BK;
        }
    };
    auto setup_tile = [&](int pid) {
        int tile_m, tile_n;
        if (SEGMENTS && total == tiles_m * tiles_n) {   // every tile has work: the plain order
            tile_of_block(pid, total, tiles_m, tiles_n, tile_m, tile_n, split);
        } else if constexpr (SEGMENTS) {
            // the pid-th tile with work, counted row by row (ids with equal id mod 8 get a contiguous range)
            const int xcd = pid & 7, idx = pid >> 3;
            const int lid = xcd * (total >> 3) + min(xcd, total & 7) + idx;
            int hi = tiles_m;   // the last tile row with row_before <= lid (bisection: each probe is a scalar load)
            tile_m = 0;
            while (hi - tile_m > 1) {
                const int mid = (tile_m + hi) >> 1;
                if ((int)g.seg.row_before[mid] <= lid) tile_m = mid; else hi = mid;
            }
            uint32_t live = g.seg.row_live[tile_m];
            for (int j = lid - (int)g.seg.row_before[tile_m]; j > 0; --j) live &= live - 1;
            tile_n = __builtin_ctz(live);
            split = 0;
        } else {
            tile_of_block(pid, total, tiles_m, tiles_n, tile_m, tile_n, split);
        }
        m0 = tile_m * BM;
        n0 = tile_n * BN;
        kb = 0;
        ke = g.K;
        if (!SEGMENTS && g.partial) {
            int per = (g.K + g.splits - 1) / g.splits;
            per = (per + BK - 1) / BK * BK;
            kb = split * per;
            ke = min(g.K, kb + per);
        }
        if constexpr (KSEG) {
            // the tile row's segment (row_before[i]: the first tile row of segment i), its rows and its positions
            // (constant indices into the kernel arguments: the segment is picked by comparisons)
            int lo = 0;
#pragma unroll
            for (int i = 0; i < kMaxGemmSegments; ++i) {
                const int first = (int)g.seg.row_before[i], hi = g.seg.end[i];
                const bool mine = i < g.seg.n && tile_m >= first && (i + 1 >= g.seg.n || tile_m < (int)g.seg.row_before[i + 1]);
                if (mine) {
                    m0 = lo + (tile_m - first) * BM;
                    mlim = hi;
                    kseg_left = g.seg.pos[i];
                }
                lo = hi;
            }
        }
        // strides as (index stride, k stride)
        int a_rows = g.M;
        if constexpr (KSEG) a_rows = mlim;
        la.template init<false>(A, g.a_rs, g.a_cs, m0, a_rows, g.tbl);
        lb.template init<REMAP == REMAP_B_N>(B, g.b_cs, g.b_rs, n0, g.N, g.tbl);
        nslabs = (ke > kb) ? (ke - kb + BK - 1) / BK : 0;
        if constexpr (KSEG) {
            const uint64_t take = kseg_left;
            kseg_sub = 0;
            kseg_k = take ? __builtin_ctzll(take) * g.seg.slice : 0;
            nslabs = __builtin_popcountll(take) * (g.seg.slice / BK);
            if (nslabs > 0) {
                la.template load<false, false>(kseg_k, ke, g.tbl);
                lb.template load<true, false>(kseg_k, ke, g.tbl);
                kseg_advance();
            }
        } else if (nslabs > 0) {
            la.template load<false, KTAIL>(kb, ke, g.tbl);
            lb.template load<REMAP_BK, KTAIL>(kb, ke, g.tbl);
        }
    };

    // Software pipeline.  LDS buffer (s & 1) holds slab s; the registers of the slab loaders hold
    // slab s + 1, fetched one slab ahead; operand fragments are double-buffered too, so every LDS
    // read is issued one MFMA group (16 k) before it is used.  The single barrier of a slab sits
    // before its last MFMA group: by then all fragment reads of the slab are done (its buffer may be
    // refilled from the next slab on) and the stores of slab s + 1 have landed, so the first
    // fragments of slab s + 1 are fetched behind that last group.  The stores of slab s + 1 (and
    // behind each the load of slab s + 2 into the registers it frees) are spread over the first three
    // groups: all eight wavefronts store at the same time, and a whole slab in one group keeps the LDS
    // busy for longer than the group's MFMAs last.  A slab's LDS addresses are one add per base
    // register (buffer offset, chosen by the slab's parity) plus compile-time instruction offsets.
    bf16x8 af[2][MT], bfg[2][NT];
    const lds_bf16* const a_lane = smem + fragment_lane_offset<BM, BK, A_COL>(wm * WTM, lane);
    const lds_bf16* const b_lane = smem + A_ELEMS + fragment_lane_offset<BN, BK, B_COL>(wn * WTN, lane);
    auto read_frags = [&](int buf, int stage, int kk) {   // stage: LDS buffer 0 / 1, a constant at every call
        const lds_bf16* as = a_lane + stage * STAGE_ELEMS;
        const lds_bf16* bs = b_lane + stage * STAGE_ELEMS;
        // in the order the MFMAs of the group need them
        af[buf][0] = read_fragment<BM, BK, A_COL>(as, 0, kk);
#pragma unroll
        for (int u = 0; u < NT; ++u) bfg[buf][u] = read_fragment<BN, BK, B_COL>(bs, u * 32, kk);
#pragma unroll
        for (int t = 1; t < MT; ++t) af[buf][t] = read_fragment<BM, BK, A_COL>(as, t * 32, kk);
    };
    auto mfma_group = [&](int buf) {
#pragma unroll
        for (int t = 0; t < MT; ++t)
#pragma unroll
            for (int u = 0; u < NT; ++u)
                acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(af[buf][t], bfg[buf][u], acc[t][u], 0, 0, 0);
    };
    constexpr int NM = MT * NT;
    constexpr int NR = MT * (A_COL ? 2 : 1) + NT * (B_COL ? 2 : 1);   // LDS reads per group
    constexpr int KA = SlabLoader<BM, BK, A_COL, kThreads>::kPerThread;
    constexpr int NW = KA + SlabLoader<BN, BK, B_COL, kThreads>::kPerThread;   // stores = loads per slab
    static_assert(BK == 64, "the pipeline below is written for four MFMA groups per slab");

    int pid = blockIdx.x;
    bool have_work = true;
    if constexpr (SEGMENTS) have_work = pid < total;
    if (have_work) setup_tile(pid);
    while (have_work) {
#pragma unroll
    for (int t = 0; t < MT; ++t)
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e) acc[t][u][e] = 0.f;
    if (nslabs > 0) {
        la.store(smem);
        lb.store(smem + A_ELEMS);
        if (nslabs > 1) {
            int k1 = kb + BK;
            if constexpr (KSEG) k1 = kseg_k;
            la.template load<false, KTAIL>(k1, ke, g.tbl);
            lb.template load<REMAP_BK, KTAIL>(k1, ke, g.tbl);
            if constexpr (KSEG) kseg_advance();
        }
    }
    __syncthreads();
    if (nslabs > 0) read_frags(0, 0, 0);

    // one slab; STORE: slab s+1 is in the loader registers and goes to the other buffer,
    // LOAD: slab s+2 exists and is fetched into the loader registers
    auto slab = [&](int s, auto store_tag, auto load_tag) {
        constexpr bool STORE = decltype(store_tag)::value, LOAD = decltype(load_tag)::value;
        const int CUR = s & 1;
        lds_bf16* as_next = smem + (1 - CUR) * STAGE_ELEMS;
        lds_bf16* bs_next = as_next + A_ELEMS;
        int k_next = kb + (s + 2) * BK;
        if constexpr (KSEG) k_next = kseg_k;
        auto move_third = [&](auto third_tag) {   // a third of the slab's chunks: store, then reload
            constexpr int P = decltype(third_tag)::value;
#pragma unroll
            for (int c = P * NW / 3; c < (P + 1) * NW / 3; ++c) {
                if (c < KA) {
                    if (STORE) la.store_one(c, as_next);
                    if (LOAD) la.template load_one<false, KTAIL>(c, k_next, ke, g.tbl);
                } else {
                    if (STORE) lb.store_one(c - KA, bs_next);
                    if (LOAD) lb.template load_one<REMAP_BK, KTAIL>(c - KA, k_next, ke, g.tbl);
                }
            }
        };
        read_frags(1, CUR, 16);   // ahead of the stores: LDS reads are not moved across LDS stores
        move_third(std::integral_constant<int, 0>{});
        mfma_group(0);
        pace_group<NM, NR, STORE ? NW / 3 : 0>();
        __builtin_amdgcn_sched_barrier(0);   // groups are scheduled one by one
        read_frags(0, CUR, 32);
        move_third(std::integral_constant<int, 1>{});
        mfma_group(1);
        pace_group<NM, NR, STORE ? 2 * NW / 3 - NW / 3 : 0>();
        __builtin_amdgcn_sched_barrier(0);
        read_frags(1, CUR, 48);
        move_third(std::integral_constant<int, 2>{});
        if constexpr (KSEG && LOAD) kseg_advance();
        mfma_group(0);
        pace_group<NM, NR, STORE ? NW - 2 * NW / 3 : 0>();
        __builtin_amdgcn_sched_barrier(0);
        __syncthreads();
        if (STORE) read_frags(0, 1 - CUR, 0);
        mfma_group(1);
        pace_group<NM, STORE ? NR : 0, 0>();
        __builtin_amdgcn_sched_barrier(0);
    };
    {
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        int s = 0;
        for (; s + 2 < nslabs; ++s) slab(s, yes, yes);
        if (s + 1 < nslabs) {
            slab(s, yes, no);
            ++s;
        }
        if (s < nslabs) slab(s, no, no);
    }
    __syncthreads();   // the epilogue reuses the operand buffers
    const int em0 = m0, en0 = n0, esplit = split;
    int m_lim = g.M;   // rows of the tile below it are written
    if constexpr (KSEG) m_lim = mlim;
    // the next tile's first slab arrives under the epilogue
    pid += gridDim.x;
    have_work = pid < total;
    if (have_work) setup_tile(pid);

    // ---- epilogue ----
    // Accumulator element e of MFMA tile (t,u) is row 8*(e/4) + 4*(lane/32) + e%4, column lane%32.
    // Each wavefront passes one 32-row band of its tile through its own LDS area (fp32) and reads it
    // back 8 consecutive columns per lane, so bias / residual / activation operands are fetched and
    // results stored as 16-byte rows.
    constexpr int SST = WTN + 4;                 // stage row stride in floats
    constexpr int CPR = WTN / 8;                 // 8-column chunks per stage row
    constexpr int CPL = 32 * CPR / 64;           // chunks per lane
    float* stage = reinterpret_cast<float*>(smem_raw) + wave * (32 * SST);
    const int col_l = lane & 31, row_l = 4 * (lane >> 5);
    bf16* __restrict__ C = static_cast<bf16*>(g.C);
    const bf16* bias = static_cast<const bf16*>(g.bias);
    const bf16* R = SEGMENTS ? nullptr : static_cast<const bf16*>(g.residual);   // the segment form takes neither
    bf16* Z = static_cast<bf16*>(g.Z);
    float* P = (!SEGMENTS && g.partial) ? g.partial + (long)esplit * g.M * g.N : nullptr;
    // a lane reads back the same 8 columns in every chunk (64 is a multiple of the chunks per row),
    // so its bias values are fetched once per tile
    static_assert(64 % CPR == 0, "a lane keeps its columns over the chunks of a band");
    // row segments: bit t * CPL + c of rows_alive = the lane's row of chunk c in band t lies in a segment in which
    // the wavefront's 64 columns (all of one position) take part
    uint32_t rows_alive = 0;
    if constexpr (SEGMENTS) {
        static_assert(MT * CPL <= 32, "one bit per row a lane reads back");
        // the segments in which the position takes part, one bit each (two scalar loads, both issued at once)
        const int p = __builtin_amdgcn_readfirstlane((en0 + wn * WTN) / g.seg.slice);
        const uint32_t segs = g.seg.pos_segs[p & 63];
        const int first = __builtin_amdgcn_readfirstlane(em0 + wm * WTM);
        // the segment ends are fetched here, per tile: as loop invariants they would be held in registers the
        // main loop has no room for
        int at;
        asm volatile("s_mov_b32 %0, 0" : "=s"(at));
        int ends[kMaxGemmSegments - 1];
#pragma unroll
        for (int i = 0; i + 1 < kMaxGemmSegments; ++i) ends[i] = g.seg.end[at + i];
        int s0 = 0, s1 = 0;   // segments of the wavefront's first and last row
#pragma unroll
        for (int i = 0; i + 1 < kMaxGemmSegments; ++i) {
            s0 += (first >= ends[i]) ? 1 : 0;
            s1 += (first + WTM - 1 >= ends[i]) ? 1 : 0;
        }
        if (s0 == s1) {   // nearly always: no segment ends inside the wavefront's rows
            rows_alive = ((segs >> s0) & 1) ? 0xffffffffu : 0u;
        } else {
            const int mbase = first + lane / CPR;
#pragma unroll
            for (int j = 0; j < MT * CPL; ++j) {
                const int m = mbase + (j / CPL) * 32 + (j % CPL) * (64 / CPR);
                int si = 0;
#pragma unroll
                for (int i = 0; i + 1 < kMaxGemmSegments; ++i) si += (m >= ends[i]) ? 1 : 0;
                rows_alive |= ((segs >> si) & 1) << j;
            }
        }
    }
    u32x4 braw = {0u, 0u, 0u, 0u};
    {
        const int nb = en0 + wn * WTN + (lane % CPR) * 8;
        if (!P && bias && nb < g.N) braw = *reinterpret_cast<const u32x4*>(bias + (g.bias_remap ? g.tbl(nb) : nb));
    }
    // column sums of the tile's results (the bias gradient of the layer that produced the GEMM's input):
    // a lane adds up its 8 columns over all its rows, the lanes that share columns are combined at the
    // end of the tile, and the wavefront's WTM-row band becomes one row of g.colsum
    constexpr bool kColsum = !A_COL;   // weight-gradient forms (A with K strided) never ask for it
    float csum[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) csum[i] = 0.f;
    // EPI_DGELU: C = (A B) * Z with nothing else in the epilogue; EPI_RESIDUAL: C = A B + bias + R.  The operand
    // (Z or R) is fetched a band ahead - each chunk's registers are refilled for the next band as soon as the
    // chunk is stored - instead of one dependent load per chunk.
    if constexpr (EPI != EPI_ANY) {
        static_assert(!A_COL, "a plain product with A row-major");
        const int mrow = em0 + wm * WTM + lane / CPR;           // the lane's row of chunk 0 in band 0
        const int n = en0 + wn * WTN + (lane % CPR) * 8;        // its columns in every chunk
        const long ldop = EPI == EPI_DGELU ? g.ldz : g.ldr;
        const bf16* zp = (EPI == EPI_DGELU ? Z : static_cast<const bf16*>(g.residual)) + (long)mrow * ldop + n;
        bf16* cp = C + (long)mrow * g.ldc + n;
        const long zstep = (long)(64 / CPR) * ldop, cstep = (long)(64 / CPR) * g.ldc;   // rows between chunks
        u32x4 zq[CPL];
        auto fetch = [&](int t, int c) {   // zeros for a row outside the problem or outside its segment's slices
            const int m = mrow + t * 32 + c * (64 / CPR);
            const bool live = m < m_lim && n < g.N && (!SEGMENTS || ((rows_alive >> (t * CPL + c)) & 1));
            zq[c] = u32x4{0u, 0u, 0u, 0u};
            if (live) zq[c] = *reinterpret_cast<const u32x4*>(zp);
            zp += zstep;   // chunks are fetched in the order they are stored
        };
#pragma unroll
        for (int c = 0; c < CPL; ++c) fetch(0, c);
#pragma unroll
        for (int t = 0; t < MT; ++t) {
#pragma unroll
            for (int u = 0; u < NT; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e)
                    stage[(8 * (e >> 2) + row_l + (e & 3)) * SST + u * 32 + col_l] = acc[t][u][e];
            __builtin_amdgcn_wave_barrier();
#pragma unroll
            for (int c = 0; c < CPL; ++c) {
                const int r = lane / CPR + c * (64 / CPR), cc = (lane % CPR) * 8;
                const int m = mrow + t * 32 + c * (64 / CPR);
                float v[8];
                const float4 lo = *reinterpret_cast<const float4*>(stage + r * SST + cc);
                const float4 hi = *reinterpret_cast<const float4*>(stage + r * SST + cc + 4);
                v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
#pragma unroll
                for (int i = 0; i < 4; ++i) {
                    if constexpr (EPI == EPI_DGELU) {
                        v[2 * i] *= __uint_as_float(zq[c][i] << 16);
                        v[2 * i + 1] *= __uint_as_float(zq[c][i] & 0xffff0000u);
                    } else {   // braw is zero without a bias
                        v[2 * i] += __uint_as_float(braw[i] << 16);
                        v[2 * i + 1] += __uint_as_float(braw[i] & 0xffff0000u);
                        v[2 * i] += __uint_as_float(zq[c][i] << 16);
                        v[2 * i + 1] += __uint_as_float(zq[c][i] & 0xffff0000u);
                    }
                }
                if (t + 1 < MT) fetch(t + 1, c);
                if (m < m_lim && n < g.N) {
                    store8(cp, v);
                    if (g.colsum) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) csum[i] += v[i];
                    }
                }
                cp += cstep;
            }
            __builtin_amdgcn_wave_barrier();
        }
    } else
#pragma unroll
    for (int t = 0; t < MT; ++t) {
#pragma unroll
        for (int u = 0; u < NT; ++u)
#pragma unroll
            for (int e = 0; e < 16; ++e)
                stage[(8 * (e >> 2) + row_l + (e & 3)) * SST + u * 32 + col_l] = acc[t][u][e];
        __builtin_amdgcn_wave_barrier();
#pragma unroll 1
        for (int c = 0; c < CPL; ++c) {
            const int id = lane + 64 * c;
            const int r = id / CPR, cc = (id % CPR) * 8;
            const int m = em0 + wm * WTM + t * 32 + r;
            const int n = en0 + wn * WTN + cc;
            if (m < m_lim && n < g.N) {
                float v[8];
                const float4 lo = *reinterpret_cast<const float4*>(stage + r * SST + cc);
                const float4 hi = *reinterpret_cast<const float4*>(stage + r * SST + cc + 4);
                v[0] = lo.x; v[1] = lo.y; v[2] = lo.z; v[3] = lo.w; v[4] = hi.x; v[5] = hi.y; v[6] = hi.z; v[7] = hi.w;
                const bool alive = !SEGMENTS || ((rows_alive >> (t * CPL + c)) & 1);
                if (P) {
                    store8(P + (long)m * g.N + n, v);
                } else {
                    if (bias) {
#pragma unroll
                        for (int i = 0; i < 4; ++i) {
                            v[2 * i] += __uint_as_float(braw[i] << 16);
                            v[2 * i + 1] += __uint_as_float(braw[i] & 0xffff0000u);
                        }
                    }
                    if (g.act == ACT_GELU) {
                        // Z <- GELU'(z), C <- GELU(z), both of the fp32 pre-activation
                        float gp[8];
                        gelu_pair8(v, gp);
                        if (SEGMENTS && !alive) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) gp[i] = 0.f;
                        }
                        store8(Z + (long)m * g.ldz + n, gp);
                    } else if (g.act == ACT_DGELU) {
                        float gp[8];
                        load8(Z + (long)m * g.ldz + n, gp);
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] *= gp[i];
                    }
                    if (SEGMENTS && !alive) {
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] = 0.f;
                    }
                    if (R) {
                        float rr[8];
                        load8(R + (long)m * g.ldr + n, rr);
#pragma unroll
                        for (int i = 0; i < 8; ++i) v[i] += rr[i];
                    }
                    store8(C + (long)m * g.ldc + n, v);
                    if constexpr (kColsum) {
                        if (g.colsum) {
#pragma unroll
                            for (int i = 0; i < 8; ++i) csum[i] += v[i];
                        }
                    }
                }
            }
        }
        __builtin_amdgcn_wave_barrier();
    }
    if (kColsum && g.colsum) {   // uniform over the grid
        static_assert(CPR == 8, "lanes 8 apart share their columns");
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            float t = csum[i];
            t += __shfl_xor(t, 8, 64);
            t += __shfl_xor(t, 16, 64);
            t += __shfl_xor(t, 32, 64);
            csum[i] = t;
        }
        const int n = en0 + wn * WTN + lane * 8;
        if (lane < CPR && n < g.N)
            store8(g.colsum + (long)(g.colsum_row0 + (em0 / BM) * WGM + wm) * g.N + n, csum);
    }
    __syncthreads();   // the stage area is operand buffer space of the next tile
    }
    if constexpr (SEGMENTS) {
        // Tiles without work: zeros (results, saved derivative, column-sum bands), written in strips of 32 rows by
        // the workgroups that had one tile less to multiply while the others are still busy, or by all of them,
        // the last ones first, if those would be too few to keep the memory system busy.
        const int dead = (tiles_m * tiles_n - total) * (BM / 32);
        const int grid = gridDim.x, heavy = total % grid;   // workgroups 0 .. heavy-1 had the extra tile
        const bool all_fill = grid - heavy < 64;
        const int fillers = all_fill ? grid : grid - heavy;
        bf16* Cz = static_cast<bf16*>(g.C);
        bf16* Zz = static_cast<bf16*>(g.Z);
        const float zero8[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
        for (int du = all_fill ? grid - 1 - (int)blockIdx.x : (int)blockIdx.x - heavy; du >= 0 && du < dead; du += fillers) {
            const int d = du / (BM / 32), strip = du % (BM / 32);
            int tm = 0, hi = tiles_m;   // the last tile row with no more than d tiles without work before it
            while (hi - tm > 1) {
                const int mid = (tm + hi) >> 1;
                if (mid * tiles_n - (int)g.seg.row_before[mid] <= d) tm = mid; else hi = mid;
            }
            uint32_t bits = ~(uint32_t)g.seg.row_live[tm] & ((1u << tiles_n) - 1u);
            for (int j = d - (tm * tiles_n - (int)g.seg.row_before[tm]); j > 0; --j) bits &= bits - 1;
            const int tn = __builtin_ctz(bits);
            for (int i = threadIdx.x; i < 32 * (BN / 8); i += kThreads) {
                const int m = tm * BM + strip * 32 + i / (BN / 8), n = tn * BN + (i % (BN / 8)) * 8;
                if (m < g.M && n < g.N) {
                    store8(Cz + (long)m * g.ldc + n, zero8);
                    if (g.act == ACT_GELU) store8(Zz + (long)m * g.ldz + n, zero8);
                }
            }
            if (g.colsum && strip < WGM && threadIdx.x < BN / 8) {
                const int n = tn * BN + threadIdx.x * 8;
                if (n < g.N) store8(g.colsum + (long)(g.colsum_row0 + tm * WGM + strip) * g.N + n, zero8);
            }
        }
    }
}

template <int BM, int BN, int BK, int WGM, int WGN, bool A_COL, bool B_COL>
constexpr size_t lds_bytes() {
    constexpr size_t slabs = 2 * (slab_elems<BM, BK, A_COL>() + slab_elems<BN, BK, B_COL>()) * sizeof(bf16);
    constexpr size_t stage = stage_bytes<BN, WGM, WGN>();
    return slabs > stage ? slabs : stage;
}

template <int BM, int BN, int BK, int WGM, int WGN, bool A_COL, bool B_COL, int REMAP, bool KTAIL, int EPI = EPI_ANY>
hipError_t launch_cfg(const GemmArgs& g, hipStream_t s) {
    constexpr size_t lds = lds_bytes<BM, BN, BK, WGM, WGN, A_COL, B_COL>();
    auto kern = gemm_mfma_kernel<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP, KTAIL, false, EPI>;
    static KernelLimits limits;
    int resident = 0;
    if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 64 * WGM * WGN, lds, &resident); e != hipSuccess) return e;
    resident = in_eights(resident);
    const int splits = g.partial ? g.splits : 1;
    const long tiles = (long)((g.N + BN - 1) / BN) * (REMAP == REMAP_B_KSEG ? g.seg.live_tiles : (g.M + BM - 1) / BM) * splits;
    // persistent: no more workgroups than are resident together; each walks tiles b, b + grid, ...
    const dim3 grid((unsigned)(tiles < resident ? tiles : resident)), block(64 * WGM * WGN);
    return launch_signalling(kern, grid, block, lds, s, g);
}

// C = (A B) * Z and nothing else in the epilogue: the instantiations with the band-ahead fetch of Z
inline bool dgelu_only(const GemmArgs& g) {
    return g.act == ACT_DGELU && !g.partial && !g.bias && !g.residual && g.a_cs == 1 && g.b_rs != 1;
}

// C = A B + bias + R: likewise
inline bool residual_only(const GemmArgs& g) {
    return g.act == ACT_NONE && !g.partial && g.residual && g.a_cs == 1 && g.b_rs == 1;
}

// row-segment launch: the 256x256 tile, A row-major, K a multiple of 64
template <bool B_COL, int REMAP>
hipError_t launch_seg_cfg(const GemmArgs& g, hipStream_t s) {
    constexpr int BM = 256, BN = 256, BK = 64, WGM = 2, WGN = 4;
    constexpr size_t lds = lds_bytes<BM, BN, BK, WGM, WGN, false, B_COL>();
    auto kern = gemm_mfma_kernel<BM, BN, BK, WGM, WGN, false, B_COL, REMAP, false, true, B_COL ? EPI_DGELU : EPI_ANY>;
    static KernelLimits limits;
    int resident = 0;
    if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 64 * WGM * WGN, lds, &resident); e != hipSuccess) return e;
    resident = in_eights(resident);
    const long tiles = (long)((g.N + BN - 1) / BN) * ((g.M + BM - 1) / BM);
    const long grid = tiles < resident ? (tiles + 7) / 8 * 8 : resident;
    return launch_signalling(kern, dim3((unsigned)grid), dim3(64 * WGM * WGN), lds, s, g);
}

// K-segment launch: A row-major, B's k through the remap table; the epilogue is the residual form (FC2 forward) or
// the generic one (the backward's dv)
template <int BM, bool B_COL, int EPI>
hipError_t launch_kseg_cfg(const GemmArgs& g, hipStream_t s) {
    return launch_cfg<BM, 256, 64, 2, 4, false, B_COL, REMAP_B_KSEG, false, EPI>(g, s);
}

// K a multiple of 64 (every shape of the model): the slab loads carry no per-chunk k check
template <int BM, int BN, int BK, int WGM, int WGN, bool A_COL, bool B_COL, int REMAP, int EPI = EPI_ANY>
hipError_t launch_tail(const GemmArgs& g, hipStream_t s) {
    if (g.K % BK) return launch_cfg<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP, true, EPI>(g, s);
    return launch_cfg<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP, false, EPI>(g, s);
}

template <int BM, int BN, int BK, int WGM, int WGN, bool A_COL, bool B_COL>
hipError_t launch_remap(const GemmArgs& g, hipStream_t s) {
    if constexpr (!A_COL && B_COL) {   // the backward's dz has an epilogue of its own (the remapped-k form never occurs)
        if (dgelu_only(g)) {
            if (g.remap == REMAP_B_N) return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_B_N, EPI_DGELU>(g, s);
            if (g.remap == REMAP_NONE) return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_NONE, EPI_DGELU>(g, s);
        }
    }
    if constexpr (!A_COL && !B_COL) {   // the forward products that close a residual branch (never with remapped columns)
        if (residual_only(g)) {
            if (g.remap == REMAP_B_K) return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_B_K, EPI_RESIDUAL>(g, s);
            if (g.remap == REMAP_NONE) return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_NONE, EPI_RESIDUAL>(g, s);
        }
    }
    switch (g.remap) {
        case REMAP_B_N: return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_B_N>(g, s);
        case REMAP_B_K: return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_B_K>(g, s);
        default: return launch_tail<BM, BN, BK, WGM, WGN, A_COL, B_COL, REMAP_NONE>(g, s);
    }
}

template <int BM, int BN, int BK, int WGM, int WGN>
hipError_t launch_layout(const GemmArgs& g, hipStream_t s) {
    const bool a_col = (g.a_cs != 1), b_col = (g.b_rs != 1);
    if (!a_col && !b_col) return launch_remap<BM, BN, BK, WGM, WGN, false, false>(g, s);
    if (!a_col && b_col) return launch_remap<BM, BN, BK, WGM, WGN, false, true>(g, s);
    if (a_col && b_col) return launch_remap<BM, BN, BK, WGM, WGN, true, true>(g, s);
    return hipErrorNotSupported;
}


}  // namespace

bool gemm_mfma_supported(const GemmArgs& g) {
    if (g.M <= 0 || g.N <= 0 || g.K <= 0) return false;
    const bool a_row = (g.a_cs == 1), a_col = (g.a_rs == 1);
    const bool b_row = (g.b_rs == 1), b_col = (g.b_cs == 1);
    if (!(a_row || a_col) || !(b_row || b_col)) return false;
    if (!a_row && b_row) return false;   // A col-form with B row-form is never needed
    // 16-byte chunks: contiguous extents and leading strides must be multiples of 8 elements
    if (a_row ? !(mult8(g.K) && mult8(g.a_rs)) : !(mult8(g.M) && mult8(g.a_cs))) return false;
    if (b_row ? !(mult8(g.K) && mult8(g.b_cs)) : !(mult8(g.N) && mult8(g.b_rs))) return false;
    if (!al16(g.A) || !al16(g.B)) return false;
    if (!mult8(g.N)) return false;
    // operands are addressed with 32-bit byte offsets below 2 GiB
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
    if (a_span * 2 >= (1L << 31) || b_span * 2 >= (1L << 31)) return false;
    if (g.colsum && (g.partial || g.a_cs != 1 || !al16(g.colsum))) return false;
    if (g.partial) return al16(g.partial);
    if (!g.C || !al16(g.C) || !mult8(g.ldc)) return false;
    if (g.bias && !al16(g.bias)) return false;
    if (g.residual && (!al16(g.residual) || !mult8(g.ldr))) return false;
    if (g.act != ACT_NONE && (!g.Z || !al16(g.Z) || !mult8(g.ldz))) return false;
    return true;
}

// Microseconds of a product on one of the three tiles (0 = 128x128, two workgroups per CU; 1 = 256x256 and 3 = 192x256,
// one per CU):  launch + rounds * (start + slab * slabs of 64 of K + epilogue).  A round that fills only part of the
// chip costs `least` of a full one and more the fuller it is.  Fitted on this part to 482 products of 2048 to 18912 rows,
// widths 384 to 1024, with the model's four epilogues and both forms of B: rms error 3 % for the large tiles, 8 % for
// the small one; the tile it picks is 0.1 % slower than the best of the three on average (the rule before it, by rounds
// alone, 1.5 %: 12608 x 1536 x 384 with the GELU' product took 34.8 us on 256x256 tiles, 29.8 on 128x128).
static float product_us(const GemmArgs& g, int tile, int M) {
    struct Cost { int bm, bn, at_once; float launch, least, start, slab, gelu, dgelu, residual, b_col; };
    constexpr Cost kCost[3] = {{128, 128, 512, 4.85f, 0.22f, 3.07f, 0.965f, 4.37f, 0.60f, 0.54f, 0.022f},
                               {256, 256, 256, 2.34f, 0.665f, 9.11f, 1.32f, 8.87f, 1.91f, 0.70f, 0.012f},
                               {192, 256, 256, 2.55f, 0.625f, 6.92f, 1.088f, 6.97f, 1.05f, 0.14f, 0.015f}};
    const Cost& c = kCost[tile == 3 ? 2 : tile];
    const long units = (long)((M + c.bm - 1) / c.bm) * ((g.N + c.bn - 1) / c.bn) * (g.partial ? g.splits : 1);
    float rounds = (float)(units / c.at_once);
    if (const int rest = (int)(units % c.at_once)) rounds += c.least + (1.0f - c.least) * (float)rest / (float)c.at_once;
    if (tile == 0 && rounds < 0.42f) rounds = 0.42f;   // a few workgroups: their own latency
    const float slabs = (float)((g.K + 63) / 64);
    const float epilogue = g.act == ACT_GELU ? c.gelu : (g.act == ACT_DGELU ? c.dgelu : (g.residual ? c.residual : 0.0f));
    return c.launch + rounds * (c.start + slabs * (c.slab + (g.b_rs != 1 ? c.b_col : 0.0f)) + epilogue);
}

// Beside another stream's launches the small tile is not the better one where it would be alone: its workgroups cover
// all CUs and take 1.5 times the operand bytes, the large ones leave CUs to the other stream (width 1024, 6304 rows:
// 24 blocks 13.2 ms with dv on 128x128 tiles, 12.8 with 192x256).
static float small_us(const GemmArgs& g) {
    if (g.shared && g.M >= 256 && g.N >= 256 && (long)((g.M + 255) / 256) * ((g.N + 255) / 256) >= 96) return 1e30f;
    return product_us(g, 0, g.M);
}

static int pick_one(const GemmArgs& g) {
    if (g.tile_hint) return g.tile_hint == 2 ? 0 : g.tile_hint;
    if (g.N < 256 || g.M < 192) return 0;
    const float small = small_us(g), mid = product_us(g, 3, g.M);
    const float big = g.M >= 256 ? product_us(g, 1, g.M) : 1e30f;
    return small <= mid && small <= big ? 0 : (mid <= big ? 3 : 1);
}

// The rows of the whole rounds of 256x256 tiles if those, with the remaining rows on 128x128 tiles, are cheaper than any
// one tile for all rows; 0 otherwise.
static int split_rows(const GemmArgs& g, float* us) {
    const long tn = (g.N + 255) / 256, total = (long)((g.M + 255) / 256) * tn;
    if (g.partial || g.tile_hint || g.M < 512 || g.N < 256 || total <= 256) return 0;
    const int rows = (int)(total / 256 * 256 / tn * 256);
    if (rows <= 0 || rows >= g.M) return 0;
    // the second launch waits for the first one's last tile; and near a tie one launch: 9232 x 1920 x 768 takes 34.6 us on
    // 192x256 tiles and 36.2 in two launches, 4096 x 4992 x 2048 77.9 and 84.2
    const float two = (product_us(g, 1, rows) + product_us(g, 0, g.M - rows) + 2.5f) * 1.015f;
    *us = two;
    return two < small_us(g) && two < product_us(g, 1, g.M) && two < product_us(g, 3, g.M) ? rows : 0;
}

// Two workgroups to a CU (kernels_gemm_pair.hip) where that is cheaper than the large tiles in one launch or two.  Below 640
// of its tiles, a round and a quarter, the costs do not tell the two apart; of 26 products of more that it takes by this
// rule the slowest is at 1.04 of the other's time, their mean at 0.94 (12608 x 3072 x 768 with GELU 90 -> 78 us, 15760 x
// 1536 x 384 43 -> 36).  Of whole passes, with this rule and without: base model, 64 images (12608 rows) 7754 and 7897 us, 384
// pixels (9232) 7277 and 7295, large model (6304) 12615 and 12669, subnets gated 7987 and 7980.  Not beside another stream's
// launches: the backward's dz on this kernel (then with a form for it) took 12.6 us off by itself and nothing off a pass.
static bool pair_faster(const GemmArgs& g) {
    if (g.tile_hint || g.shared || !gemm_pair_supported(g) || (long)((g.M + 127) / 128) * ((g.N + 255) / 256) <= 640) return false;
    float us = 1e30f;
    if (!split_rows(g, &us)) {
        const int tile = pick_one(g);
        us = product_us(g, tile, g.M);
    }
    return gemm_pair_us(g) < 0.96f * us;
}

// the tile of launch_gemm_mfma: 0 = 128x128, 1 = 256x256, 3 = 192x256, 4 = 128x256 with two workgroups to a CU
static int pick_tile(const GemmArgs& g) { return pair_faster(g) ? 4 : pick_one(g); }

int gemm_mfma_split_rows(const GemmArgs& g) {
    float us;
    return pair_faster(g) ? 0 : split_rows(g, &us);
}

int gemm_mfma_tile_rows(const GemmArgs& g) {
    const int tile = pick_tile(g);
    return tile == 0 ? 128 : (tile == 3 ? 192 : 256);
}

const char* gemm_mfma_config_name(const GemmArgs& g) {
    // the instantiation's name as a profiler prints it, so timing records and kernel traces can be matched
    const bool a_col = (g.a_cs != 1), b_col = (g.b_rs != 1);
    const int tile = pick_tile(g);
    const bool tail = (g.K % 64) != 0;
    const int epi = (!a_col && b_col && dgelu_only(g) && g.remap != REMAP_B_K) ? EPI_DGELU
                    : (!a_col && !b_col && residual_only(g) && g.remap != REMAP_B_N) ? EPI_RESIDUAL : EPI_ANY;
    if (tile == 4) return gemm_pair_name(g);
    static char names[4][3][3][2][3][88];
    char* name = names[tile][a_col ? 2 : (b_col ? 1 : 0)][g.remap == REMAP_B_N ? 1 : (g.remap == REMAP_B_K ? 2 : 0)][tail][epi];
    if (!name[0]) {
        const int bm = tile == 0 ? 128 : (tile == 3 ? 192 : 256), bn = tile == 0 ? 128 : 256;
        snprintf(name, sizeof(names[0][0][0][0][0]), "gemm_mfma_kernel<%d, %d, 64, 2, %d, %s, %s, %d, %s, false, %d>", bm, bn,
                 tile == 0 ? 2 : 4, a_col ? "true" : "false", b_col ? "true" : "false",
                 g.remap == REMAP_B_N ? 1 : (g.remap == REMAP_B_K ? 2 : 0), tail ? "true" : "false", epi);
    }
    return name;
}

hipError_t gemm_mfma_seg_prepare(GemmArgs* g) {
    GemmRowSegments& S = g->seg;
    if (!gemm_mfma_supported(*g) || g->partial || g->a_cs != 1 || g->K % 64) return hipErrorNotSupported;
    if (g->residual) return hipErrorNotSupported;   // a row that takes no part is written as zero, not as the residual
    if (g->b_rs != 1 && !dgelu_only(*g)) return hipErrorNotSupported;   // B with k strided: instantiated for dz only
    const int tiles_m = (g->M + 255) / 256, tiles_n = (g->N + 255) / 256;
    if (S.n < 1 || S.n > kMaxGemmSegments || S.slice < 64 || S.slice % 64 || tiles_m > kMaxSegTileRows || tiles_n > 16 ||
        (g->N + S.slice - 1) / S.slice > 64 || S.end[S.n - 1] != g->M)
        return hipErrorNotSupported;
    for (int i = 0; i < S.n; ++i)
        if (S.end[i] <= (i ? S.end[i - 1] : 0)) return hipErrorNotSupported;
    for (int i = S.n; i < kMaxGemmSegments; ++i) {   // rows beyond M belong to no segment that takes part
        S.end[i] = 0x7fffffff;
        S.pos[i] = 0;
    }
    int before = 0;
    for (int t = 0; t < tiles_m; ++t) {
        const int r0 = t * 256, r1 = (t + 1) * 256 < g->M ? (t + 1) * 256 : g->M;
        uint64_t pos = 0;   // positions that take part in any segment the tile row overlaps
        for (int i = 0; i < S.n; ++i)
            if ((i ? S.end[i - 1] : 0) < r1 && S.end[i] > r0) pos |= S.pos[i];
        uint32_t live = 0;
        for (int j = 0; j < tiles_n; ++j) {
            const int p0 = j * 256 / S.slice, p1 = ((j + 1) * 256 < g->N ? (j + 1) * 256 : g->N) - 1;
            for (int p = p0; p <= p1 / S.slice; ++p)
                if ((pos >> p) & 1) live |= 1u << j;
        }
        S.row_live[t] = (uint16_t)live;
        S.row_before[t] = (uint16_t)before;
        before += __builtin_popcount(live);
    }
    for (int t = tiles_m; t <= kMaxSegTileRows; ++t) S.row_before[t] = (uint16_t)before;
    for (int t = tiles_m; t < kMaxSegTileRows; ++t) S.row_live[t] = 0;
    for (int p = 0; p < 64; ++p) {
        S.pos_segs[p] = 0;
        for (int i = 0; i < S.n; ++i) S.pos_segs[p] |= (uint8_t)(((S.pos[i] >> p) & 1) << i);
    }
    S.live_tiles = before;
    return g->remap == REMAP_B_N ? hipSuccess : hipErrorNotSupported;   // the gated feed-forward forms
}

hipError_t launch_gemm_mfma_kseg(const GemmArgs& g, hipStream_t s) {
    const GemmRowSegments& S = g.seg;
    if (!gemm_mfma_supported(g) || g.remap != REMAP_B_K || g.a_cs != 1 || g.partial || g.colsum || g.act != ACT_NONE) return hipErrorNotSupported;
    if (S.n < 1 || S.n > kMaxGemmSegments || S.slice < 64 || S.slice % 64 || g.K % S.slice || g.K / S.slice > 64) return hipErrorNotSupported;
    const uint64_t all = g.K / S.slice >= 64 ? ~0ull : ((1ull << (g.K / S.slice)) - 1ull);
    int lo = 0;
    for (int i = 0; i < S.n; ++i) {
        if (S.end[i] <= lo || (S.pos[i] & ~all)) return hipErrorNotSupported;
        lo = S.end[i];
    }
    if (lo != g.M) return hipErrorNotSupported;
    const bool b_col = (g.b_rs != 1);
    if (!b_col && !residual_only(g)) return hipErrorNotSupported;   // instantiated for FC2 forward ...
    if (b_col && (g.residual || g.bias)) return hipErrorNotSupported;   // ... and the backward's dv
    // every segment gets tile rows of its own; the 192-row tile when it fills more of one round of the chip than
    // the 256-row tile (as pick_tile has it)
    auto tile_rows = [&](int bm) {
        long t = 0;
        for (int i = 0; i < S.n; ++i) t += (S.end[i] - (i ? S.end[i - 1] : 0) + bm - 1) / bm;
        return t;
    };
    const long tn = (g.N + 255) / 256;
    const long big = tile_rows(256) * tn, mid = tile_rows(192) * tn;
    const bool t192 = big < 256 && mid <= 256 && mid > big;
    const int bm = t192 ? 192 : 256;
    GemmArgs k = g;
    int t = 0;
    for (int i = 0; i < kMaxGemmSegments; ++i) {
        k.seg.row_before[i] = (uint16_t)t;
        if (i < S.n) t += (S.end[i] - (i ? S.end[i - 1] : 0) + bm - 1) / bm;
    }
    if (t > 0xffff) return hipErrorNotSupported;
    k.seg.live_tiles = t;
    if (!b_col) return t192 ? launch_kseg_cfg<192, false, EPI_RESIDUAL>(k, s) : launch_kseg_cfg<256, false, EPI_RESIDUAL>(k, s);
    return t192 ? launch_kseg_cfg<192, true, EPI_ANY>(k, s) : launch_kseg_cfg<256, true, EPI_ANY>(k, s);
}

hipError_t launch_gemm_mfma_seg(const GemmArgs& g, hipStream_t s) {
    const bool b_col = (g.b_rs != 1);
    if (g.remap != REMAP_B_N || g.seg.n < 1) return hipErrorNotSupported;
    return b_col ? launch_seg_cfg<true, REMAP_B_N>(g, s) : launch_seg_cfg<false, REMAP_B_N>(g, s);
}

hipError_t launch_gemm_mfma(const GemmArgs& g, hipStream_t s) {
    if (!gemm_mfma_supported(g)) return hipErrorNotSupported;
    switch (pick_tile(g)) {
        case 4: return launch_gemm_pair(g, s);
        case 1: return launch_layout<256, 256, 64, 2, 4>(g, s);
        case 3: return launch_layout<192, 256, 64, 2, 4>(g, s);
        default: return launch_layout<128, 128, 64, 2, 2>(g, s);
    }
}

}  // namespace d2ft
