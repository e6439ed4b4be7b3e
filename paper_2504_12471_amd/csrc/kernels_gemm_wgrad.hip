// bf16 weight gradients of a backward call on the CDNA4 matrix cores, all in one launch:
//
//   out_g[m][n] = sum_k A_g[k][m] * B_g[k][n],   k over the tokens, the same for every gradient g
//
// A unit of work is one 256x256 tile of one gradient over one run of K; it leaves its raw fp32 sums in a slot of its own,
// and reduce_grouped_kernel adds a tile's slots up and writes the gradient.
//
// What bounds it: alone on its CU a unit needs 2048 cycles of matrix instructions per 64 k, and this kernel takes 2350; on the
// whole chip the clock sets the pace (8192^3: 1.29 PFLOP/s, 1.5 without the loads).  One wavefront per SIMD, each with
// 128x128 of the tile: a third fewer bytes from LDS than eight wavefronts of 128x64 read.  Operands are loaded straight
// into LDS, five slabs of 32 k deep (160 KB: the loads of slab s + 4 are under way while s is multiplied), so that
// nothing waits for operands that come from memory beside another stream's traffic.  Against eight wavefronts, two
// slabs of 64 k and loads through registers, operands in no cache, 12608 tokens: 768 x 3072 twice 120 -> 109 us, with
// the attention half's (768 x 768, 2304 x 768) 173 -> 161, 1024 x 768 twice 60 -> 56; 8192^3 900 -> 852.
#include <type_traits>

#include "gemm_large.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) uint32_t lds_u32;

namespace {

constexpr int BT = 256, BK = 32, kWaves = 4, kStages = 5;   // tile edge, K slab, slabs in LDS
constexpr int kRow = BT * 2, kSlab = BK * kRow, kLds = 2 * kStages * kSlab;   // bytes: a row of k, an operand's slab, all (A and B in turn)
constexpr int kLoads = kSlab / kWaves / 1024;                       // a wavefront's loads of 1024 bytes (two rows of k) per slab
constexpr int kGroupedMaxSplits = 8;
constexpr int WT = 4;                                               // 32x32 parts of a wavefront's 128x128, each way

// The 16-byte pieces of a row of k change places: piece p of row k sits at p ^ swizzle(k).  A transposing read touches 32
// columns (64 bytes) of the rows k .. k + 3 and k + 8 .. k + 11, whose starts are all the same bank.
__device__ __forceinline__ int swizzle(int k) { return ((k & 3) << 2) | ((k >> 3 & 1) << 1); }

// 8 consecutive k of one column per lane.  The pointer's __restrict tells the compiler that no load into LDS which is under
// way writes what is read here (that is what the barriers are for): without it every read waits for all of them.
__device__ __forceinline__ bf16x8 fragment(const lds_u8* __restrict p) {
    typedef s16x4 __attribute__((address_space(3))) * tr_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)p), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)(p + 4 * kRow));
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

template <bool KTAIL>
__global__ __launch_bounds__(64 * kWaves, 1) void gemm_wgrad_kernel(GemmArgs g) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    lds_u8* const lds = (lds_u8*)smem_raw;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int h = lane >> 5, wm = wave >> 1, wn = wave & 1;

    // a lane's place in the transposing reads of part t, rows 8 h + (lane & 15) / 4 of a group of 16 k
    const int j = lane & 15, kr = 8 * h + (j >> 2);
    uint32_t at_a[WT], at_b[WT];
#pragma unroll
    for (int t = 0; t < WT; ++t) {
        const int piece = 4 * t + 2 * (lane >> 4 & 1) + ((j & 3) >> 1);
        at_a[t] = kr * kRow + (((16 * wm + piece) ^ swizzle(kr)) << 4) + (j & 1) * 8;
        at_b[t] = kSlab + kr * kRow + (((16 * wn + piece) ^ swizzle(kr)) << 4) + (j & 1) * 8;
    }

    __amdgpu_buffer_rsrc_t ra, rb;
    uint32_t off_a[2], off_b[2];   // load c is rows 8 wave + 2 c + h of the slab
    uint32_t lda = 0, ldb = 0;     // bytes
    int kb = 0, ke = 0, ns = 0, slot = 0;
    auto load = [&](__amdgpu_buffer_rsrc_t r, const uint32_t (&off)[2], uint32_t ld, int at, int s, int c, bool check) {
        const int k = kb + s * BK + wave * (2 * kLoads) + 2 * c;
        uint32_t o = off[c & 1], so = (uint32_t)k * ld;
        if (KTAIL && check) {   // the lane's row may be past the end of K; a scalar offset beyond the buffer must not be asked for
            if (k + h >= ke) o = kOutside;
            if (k >= ke) so = 0;
        }
        __builtin_amdgcn_raw_ptr_buffer_load_lds(r, (lds_u32*)(lds + at + wave * (kSlab / kWaves) + c * 1024), 16, o, so, 0, 0);
    };
    // check: the slab may be K's last
    auto load_a = [&](int place, int s, int c, bool check) { load(ra, off_a, lda, place * (2 * kSlab), s, c, check); };
    auto load_b = [&](int place, int s, int c, bool check) { load(rb, off_b, ldb, place * (2 * kSlab) + kSlab, s, c, check); };

    int unit = (blockIdx.x & 7) * (gridDim.x >> 3) + (blockIdx.x >> 3);   // an XCD's workgroups: neighbouring tiles of one run of K
    const int units = g.total_tiles * g.splits;
    // fixes a unit's operands and requests its first slabs: A's of five, B's of four
    auto setup = [&]() {
        const int t = unit % g.total_tiles, sp = unit / g.total_tiles;
        int gi = 0;
        while (gi + 1 < g.n_groups && t >= g.grp[gi + 1].tile0) ++gi;
        const GemmGroup& G = g.grp[gi];
        const int lt = t - G.tile0, m0 = (lt % G.tiles_m) * BT, n0 = (lt / G.tiles_m) * BT;
        kb = sp * g.units_per_wg * BK;
        ke = min(g.K, kb + g.units_per_wg * BK);
        ns = ke > kb ? (ke - kb + BK - 1) / BK : 0;
        slot = unit;
        lda = (uint32_t)G.lda * 2;
        ldb = (uint32_t)G.ldb * 2;
        ra = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(G.A), 0, kBufBytes, 0x00020000);
        rb = __builtin_amdgcn_make_buffer_rsrc(const_cast<void*>(G.B), 0, kBufBytes, 0x00020000);
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            const int col = ((lane & 31) ^ swizzle(wave * 8 + i * 2 + h)) * 8;
            off_a[i] = m0 + col < G.M ? (uint32_t)h * lda + (uint32_t)G.column(m0 + col) * 2 : kOutside;
            off_b[i] = n0 + col < G.N ? (uint32_t)h * ldb + (uint32_t)(n0 + col) * 2 : kOutside;
        }
#pragma unroll
        for (int s = 0; s < kStages; ++s) {
            if (s < ns) {
#pragma unroll
                for (int c = 0; c < kLoads; ++c) load_a(s, s, c, true);
#pragma unroll
                for (int c = 0; c < kLoads; ++c)
                    if (s + 1 < kStages) load_b(s, s, c, true);   // the last one's under the first multiplications
            }
        }
        unit += gridDim.x;
    };

    f32x16 acc[WT][WT];
    bf16x8 af[2][WT], bf[2][WT];
    auto read = [&](int buf, int place, int q) {
        const lds_u8* p = lds + place * (2 * kSlab) + q * (16 * kRow);
        bf[buf][0] = fragment(p + at_b[0]);
#pragma unroll
        for (int t = 0; t < WT; ++t) af[buf][t] = fragment(p + at_a[t]);
#pragma unroll
        for (int u = 1; u < WT; ++u) bf[buf][u] = fragment(p + at_b[u]);
    };
    // the operands' roles are exchanged: a lane's four consecutive elements are columns of one row
    auto multiply = [&](int buf, int u0, int u1) {
#pragma unroll
        for (int u = u0; u < u1; ++u)
#pragma unroll
            for (int t = 0; t < WT; ++t) acc[t][u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bf[buf][u], af[buf][t], acc[t][u], 0, 0, 0);
    };
    // N multiplications with R LDS reads, two with each of the first, and L loads behind those (mixed with them the two hold
    // each other up: 205 -> 252 us for 12608 x 3072 x 768 on 72 CUs)
    auto pace = [&](auto n_tag, auto reads_tag, auto loads_tag) {
        constexpr int N = decltype(n_tag)::value, R = decltype(reads_tag)::value, L = decltype(loads_tag)::value;
        constexpr int B = R / 2, F = N - B;   // F multiplications behind the reads
#pragma unroll
        for (int i = 0; i < N; ++i) {
            __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);   // MFMA
            if (i < B) __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);   // LDS reads
            else if ((i - B + 1) * L / F > (i - B) * L / F) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);   // load
        }
        __builtin_amdgcn_sched_barrier(0);
    };

    bool work = unit < units, first = true;
    if (work) setup();
    while (work) {
#pragma unroll
        for (int t = 0; t < WT; ++t)
#pragma unroll
            for (int u = 0; u < WT; ++u)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[t][u][e] = 0.f;
        int place = 0;   // s % 5
        // R: slabs behind this one (5: five or more, 6: six or more)
        auto slab = [&](int s, auto left_tag) {
            constexpr int R = decltype(left_tag)::value;
            constexpr std::integral_constant<int, 16> n16{};
            constexpr std::integral_constant<int, 12> n12{};
            constexpr std::integral_constant<int, 4> n4{};
            constexpr std::integral_constant<int, 0> n0{};
            constexpr std::integral_constant<int, R >= 1 ? 16 : 0> r1{};
            constexpr std::integral_constant<int, R >= 4 ? 4 : 0> l0{};
            constexpr std::integral_constant<int, R >= 5 ? 4 : 0> l1{};
            const int place1 = place == 4 ? 0 : place + 1, before = place == 0 ? 4 : place - 1;
            read(1, place, 1);
            if constexpr (R >= 4) {
#pragma unroll
                for (int c = 0; c < 4; ++c) load_b(before, s + 4, c, R == 4);
            }
            multiply(0, 0, WT);
            pace(n16, n16, l0);
            multiply(1, 0, 1);
            pace(n4, n0, n0);
            if constexpr (R >= 1) {
                // slab s has been read and slab s + 1 has landed; requested behind that one: all up to s + 4
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                wait_vm<2 * kLoads * (R >= 4 ? 3 : R - 1)>();
                __builtin_amdgcn_s_barrier();
                __builtin_amdgcn_sched_barrier(0);
                read(0, place1, 0);
                if constexpr (R >= 5) {
#pragma unroll
                    for (int c = 0; c < 4; ++c) load_a(place, s + 5, c, R == 5);
                }
            }
            multiply(1, 1, WT);
            pace(n12, r1, l1);
            place = place1;
        };
        if (ns > 0) {
            if (first) {   // later units' slabs were waited for ahead of the stores of the unit before
                if (ns >= kStages) wait_vm<7 * kLoads>();
                else wait_vm<0>();
            }
            __builtin_amdgcn_s_barrier();
            __builtin_amdgcn_sched_barrier(0);
            read(0, 0, 0);
            __builtin_amdgcn_sched_barrier(0);
            int s = 0;
            for (; s + 6 < ns; ++s) slab(s, std::integral_constant<int, 6>{});
            if (s + 5 < ns) slab(s++, std::integral_constant<int, 5>{});
            if (s + 4 < ns) slab(s++, std::integral_constant<int, 4>{});
            if (s + 3 < ns) slab(s++, std::integral_constant<int, 3>{});
            if (s + 2 < ns) slab(s++, std::integral_constant<int, 2>{});
            if (s + 1 < ns) slab(s++, std::integral_constant<int, 1>{});
            slab(s, std::integral_constant<int, 0>{});
        }
        __syncthreads();   // the last slab has been read by all
        float4* const out = reinterpret_cast<float4*>(g.partial + (long)slot * (BT * BT)) + wave * (BT * BT / 4 / kWaves) + lane;
        work = unit < units;
        if (work) {
            setup();
            wait_vm<0>();   // a load cannot be told to have arrived once stores are behind it
        }
        first = false;
#pragma unroll
        for (int t = 0; t < WT; ++t)
#pragma unroll
            for (int u = 0; u < WT; ++u)
#pragma unroll
                for (int e = 0; e < 16; e += 4)
                    out[((t * WT + u) * 4 + e / 4) * 64] = make_float4(acc[t][u][e], acc[t][u][e + 1], acc[t][u][e + 2], acc[t][u][e + 3]);
    }
}

// Adds the splits of a tile in split order (all loads in flight at once), then the sum goes to the tile's place in its
// gradient, rows or columns through the remap, added to what is there if asked.  A slot holds the tile as the product's lanes
// had it, 1 KB a store (in rows of the tile it would be pieces of 32 bytes: 4 to 5 us a launch): lane l of part (t, u) of
// wavefront w has four columns 8 j + 4 (l / 32) of row l % 32, j = 0 .. 3.  A wavefront here takes two j of one part; lanes
// 32 apart exchange halves, so that each writes 8 columns of a row.  blockIdx.y = tile, blockIdx.x = 4 of its 128 half parts.
__global__ __launch_bounds__(256) void reduce_grouped_kernel(GemmArgs g, ReduceGroupedArgs ra, int accumulate) {
    const int tile = blockIdx.y;
    int gi = 0;
    while (gi + 1 < g.n_groups && tile >= g.grp[gi + 1].tile0) ++gi;
    const GemmGroup& G = g.grp[gi];
    const ReduceGroup& R = ra.grp[gi];
    const int lt = tile - G.tile0, lane = threadIdx.x & 63;
    const int half = blockIdx.x * 4 + __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int wave = half >> 5, t = half >> 3 & 3, u = half >> 1 & 3, jp = half & 1;
    const int m_part = (lt % G.tiles_m) * BT + (wave >> 1) * 128 + t * 32, n_part = (lt / G.tiles_m) * BT + (wave & 1) * 128 + u * 32;
    if (m_part >= G.M || n_part >= G.N) return;
    const float4* src = reinterpret_cast<const float4*>(g.partial) + (long)tile * (BT * BT / 4) + (half * 2) * 64 + lane;
    const long stride = (long)g.total_tiles * (BT * BT / 4);
    float4 x[kGroupedMaxSplits], y[kGroupedMaxSplits];
#pragma unroll
    for (int k = 0; k < kGroupedMaxSplits; ++k)
        if (k < g.splits) {
            x[k] = src[k * stride];
            y[k] = src[k * stride + 64];
        }
    float a[4] = {0.f, 0.f, 0.f, 0.f}, b[4] = {0.f, 0.f, 0.f, 0.f};
#pragma unroll
    for (int k = 0; k < kGroupedMaxSplits; ++k)
        if (k < g.splits) {
            a[0] += x[k].x; a[1] += x[k].y; a[2] += x[k].z; a[3] += x[k].w;
            b[0] += y[k].x; b[1] += y[k].y; b[2] += y[k].z; b[3] += y[k].w;
        }
    float v[8];
#pragma unroll
    for (int i = 0; i < 4; ++i) {   // the upper lanes' a <-> the lower lanes' b
        const auto sw = __builtin_amdgcn_permlane32_swap(__float_as_uint(a[i]), __float_as_uint(b[i]), false, false);
        v[i] = __uint_as_float(sw[0]);
        v[4 + i] = __uint_as_float(sw[1]);
    }
    const int m = m_part + (lane & 31), n = n_part + jp * 16 + 8 * (lane >> 5);
    if (m >= G.M || n >= G.N) return;
    if (R.remap == RED_REMAP_F32) {
        store8(static_cast<float*>(R.out) + (long)G.column(m) * R.ldo + n, v);
        return;
    }
    const int ro = (R.remap == RED_REMAP_ROWS) ? ra.tbl[R.table](m) : m;
    const int co = (R.remap == RED_REMAP_COLS) ? ra.tbl[R.table](n) : n;
    bf16* o = static_cast<bf16*>(R.out) + (long)ro * R.ldo + co;
    if (accumulate) {
        float old[8];
        load8(o, old);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += old[i];
    }
    store8(o, v);
}

template <bool KTAIL>
hipError_t launch_form(GemmArgs* g, hipStream_t s) {
    auto kern = gemm_wgrad_kernel<KTAIL>;
    static KernelLimits limits;
    int resident = 0;
    if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 64 * kWaves, kLds, &resident); e != hipSuccess) return e;
    resident = in_eights(resident);
    int tile = 0;
    for (int i = 0; i < g->n_groups; ++i) {
        GemmGroup& G = g->grp[i];
        G.tiles_m = (G.M + BT - 1) / BT;
        G.tile0 = tile;
        tile += G.tiles_m * ((G.N + BT - 1) / BT);
    }
    g->total_tiles = tile;
    g->slabs_per_tile = (g->K + BK - 1) / BK;
    // Run count: the cheapest of 1 .. 8.  Microseconds of launch and reduction, up to a constant: a slab of K costs the more the
    // fuller the chip is (its clock), a round of workgroups 14 (first slabs, the partial tile), a unit its part of the
    // reduction.  Fitted to 128 launches of 30 to 156 tiles and 6304 to 18912 rows: rms error 3.4 %, the fastest count in 14 of 16
    // shapes and one 6 % slower in the others.  12608 rows: 93 tiles, 2 runs 152.5 us, 5 runs 167.6 (which a rule by rounds of equal
    // cost had picked); 84 tiles, 3 runs 128, 2 runs 145; 33 tiles, 7 runs 63, 8 runs 91.
    const int S = g->slabs_per_tile;
    int best = 1;
    double best_cost = 1e30;
    for (int sp = 1; sp <= kGroupedMaxSplits && sp <= S; ++sp) {
        const long units = (long)tile * sp;
        if (sp > 1 && g->max_units > 0 && units > g->max_units) break;   // the caller wants CUs left over
        const long rounds = (units + resident - 1) / resident;
        const double cost = ((S + sp - 1) / sp) * (0.46 * rounds + 0.38 * units / resident) + 14.0 * rounds + 0.04 * units;
        if (cost < best_cost) { best_cost = cost; best = sp; }
    }
    g->splits = best;
    g->units_per_wg = (S + best - 1) / best;
    const long units = (long)tile * best;
    const dim3 grid((unsigned)(units < resident ? (units + 7) / 8 * 8 : resident)), block(64 * kWaves);
    return launch_signalling(kern, grid, block, kLds, s, *g);
}

// operands in 16-byte pieces and 32-bit offsets, gradients in pieces of 8 columns
bool grouped_ok(const GemmArgs& g, const ReduceGroupedArgs& r) {
    if (g.n_groups < 1 || g.n_groups > kMaxGemmGroups || g.K <= 0 || !g.partial || !al16(g.partial)) return false;
    for (int i = 0; i < g.n_groups; ++i) {
        const GemmGroup& G = g.grp[i];
        if (G.M <= 0 || G.N <= 0 || !G.A || !G.B || !al16(G.A) || !al16(G.B)) return false;
        if (!mult8(G.M) || !mult8(G.N) || !mult8(G.lda) || !mult8(G.ldb)) return false;
        if ((long)g.K * G.lda * 2 >= (1L << 31) || (long)g.K * G.ldb * 2 >= (1L << 31)) return false;
        if (!al16(r.grp[i].out) || !mult8(r.grp[i].ldo)) return false;
    }
    return true;
}

}  // namespace

size_t gemm_grouped_slots(const GemmArgs& g) {
    size_t tiles = 0;
    for (int i = 0; i < g.n_groups; ++i) tiles += (size_t)((g.grp[i].M + BT - 1) / BT) * ((g.grp[i].N + BT - 1) / BT);
    return tiles * kGroupedMaxSplits;   // one slot per (tile, split)
}

hipError_t launch_gemm_grouped(GemmArgs* g, const ReduceGroupedArgs& r, hipStream_t s) {
    if (!grouped_ok(*g, r)) return hipErrorNotSupported;
    return g->K % BK ? launch_form<true>(g, s) : launch_form<false>(g, s);
}

hipError_t launch_reduce_grouped(const GemmArgs& g, const ReduceGroupedArgs& r, int accumulate, hipStream_t s) {
    if (g.total_tiles <= 0) return hipSuccess;
    hipLaunchKernelGGL(reduce_grouped_kernel, dim3(32, g.total_tiles), dim3(256), 0, s, g, r, accumulate);
    return hipGetLastError();
}

}  // namespace d2ft
