// Fused softmax attention on the CDNA4 matrix cores for head dimension 64 and up to 256 tokens (forward) or 224 tokens (backward)
// (bf16 storage, fp32 accumulate).  One 256-thread workgroup owns one (image, head); K and V of
// that pair stay in LDS for the whole kernel.
//
// Everything is computed in the transposed orientation S^T = K Q^T so that, in the MFMA result
// layout, one lane owns ONE query column: the row-wise softmax reductions are then in-lane plus a
// single cross-lane exchange, and a lane's 8 consecutive accumulator elements are exactly the
// 8 k-slots the next MFMA wants, so probabilities go from the S^T accumulators into the P.V
// product without leaving registers.  Operands whose reduction index is not their contiguous
// index (V in the forward pass; Q, K, dO in the backward pass) are read from their natural
// [token][channel] layout with the transposing LDS load (ds_read_b64_tr_b16).
//
// MFMA 32x32x16 bf16 layouts used throughout (h = lane / 32, c = lane % 32):
//   operand:  row-or-column c, k-slots 8h .. 8h+7
//   result :  column c, element e <-> row 8*(e/4) + 4h + e%4
#include <type_traits>
#include <utility>

#include "d2ft_common.h"
#include "launch.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(__bf16)))) __bf16 bf16x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

namespace {

constexpr float kScale = 0.125f;                         // 1/sqrt(64)
constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.f;
    return z;
}

// row-form operand: 8 consecutive channels of row `row` starting at channel ch (16-byte LDS read)
__device__ __forceinline__ bf16x8 frag_rows(const bf16* lds, int stride, int row, int ch) {
    return *reinterpret_cast<const bf16x8*>(lds + row * stride + ch);
}

// transposed operand from a [token][channel] tile: the lane gets, for channel ch0 + c, the tokens
// t0 + 4h + {0..3} (slots 0..3) and t0 + 8 + 4h + {0..3} (slots 4..7): the slot order in which a lane
// holds 8 consecutive result elements of a transposed score tile.
__device__ __forceinline__ bf16x8 frag_tr(const bf16* lds, int stride, int t0, int ch0, int lane) {
    const int j = lane & 15;
    const bf16* p = lds + (t0 + 4 * (lane >> 5) + (j >> 2)) * stride + ch0 + 16 * ((lane >> 4) & 1) + 4 * (j & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p));
    const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(p + 8 * stride));
    s16x8 r;
    r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
    r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
    return __builtin_bit_cast(bf16x8, r);
}

// 8 consecutive result elements -> bf16 operand
__device__ __forceinline__ bf16x8 pack8(const f32x16& v, int first) {
    bf16x8 r;
#pragma unroll
    for (int i = 0; i < 8; ++i) r[i] = static_cast<__bf16>(v[first + i]);
    return r;
}

// copy rows [0, rows_valid) x 64 channels of a [token][ld] global tile to LDS rows of `stride`, zero rows above.
// All global loads of the tile are issued before the first LDS store, so their latencies overlap.
template <int TP, int NTHR = 256>   // NTHR threads take part, numbered by t (threadIdx.x, or the lane for one wavefront)
__device__ __forceinline__ void load_tile64(const bf16* __restrict__ g, long ld, int rows_valid, bf16* lds, int stride,
                                            int t = threadIdx.x) {
    constexpr int N = TP * 8 / NTHR;
    static_assert(TP * 8 % NTHR == 0, "the tile divides over the threads");
    u32x4 v[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = t + i * NTHR;
        const int r = c >> 3, ch = (c & 7) * 8;
        v[i] = u32x4{0u, 0u, 0u, 0u};
        if (r < rows_valid) v[i] = *reinterpret_cast<const u32x4*>(g + (long)r * ld + ch);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = t + i * NTHR;
        *reinterpret_cast<u32x4*>(lds + (c >> 3) * stride + (c & 7) * 8) = v[i];
    }
}
// the same for two tiles at once (K and V): twice the loads in flight
template <int TP, int NTHR = 256>   // NTHR threads take part, numbered by t (threadIdx.x, or the lane for one wavefront)
__device__ __forceinline__ void load_two_tiles64(const bf16* __restrict__ g0, const bf16* __restrict__ g1, long ld,
                                                 int rows_valid, bf16* lds0, int stride0, bf16* lds1, int stride1,
                                                 int t = threadIdx.x) {
    constexpr int N = (TP * 8 + NTHR - 1) / NTHR;
    u32x4 v0[N], v1[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = t + i * NTHR;
        const int r = c >> 3, ch = (c & 7) * 8;
        v0[i] = u32x4{0u, 0u, 0u, 0u};
        v1[i] = u32x4{0u, 0u, 0u, 0u};
        if (r < rows_valid) {   // rows_valid <= TP, so chunks past the tile are skipped as well
            v0[i] = *reinterpret_cast<const u32x4*>(g0 + (long)r * ld + ch);
            v1[i] = *reinterpret_cast<const u32x4*>(g1 + (long)r * ld + ch);
        }
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = t + i * NTHR;
        if (TP * 8 % NTHR == 0 || c < TP * 8) {
            *reinterpret_cast<u32x4*>(lds0 + (c >> 3) * stride0 + (c & 7) * 8) = v0[i];
            *reinterpret_cast<u32x4*>(lds1 + (c >> 3) * stride1 + (c & 7) * 8) = v1[i];
        }
    }
}

// the same by ONE wavefront with every load of both tiles in flight: raw buffer loads whose declared size
// ends with the last valid row (rows above read as zeros without touching memory), one offset register
// for all chunks (a lane's chunks are 8 rows apart: the distance goes into the scalar offset)
template <int TP>
__device__ __forceinline__ void load_two_tiles64_wave(const bf16* __restrict__ g0, const bf16* __restrict__ g1, long ld,
                                                      int rows_valid, bf16* lds0, int stride0, bf16* lds1, int stride1,
                                                      int lane) {
    constexpr int N = TP * 8 / 64;
    const uint32_t bytes = (uint32_t)(rows_valid - 1) * (uint32_t)ld * 2u + 128u;
    const __amdgpu_buffer_rsrc_t r0 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(g0), 0, bytes, 0x00020000);
    const __amdgpu_buffer_rsrc_t r1 = __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(g1), 0, bytes, 0x00020000);
    const uint32_t off = (uint32_t)(lane >> 3) * (uint32_t)ld * 2u + (uint32_t)(lane & 7) * 16u;
    const uint32_t step = 8u * (uint32_t)ld * 2u;
    u32x4 v0[N], v1[N];
#pragma unroll
    for (int i = 0; i < N; ++i) {
        v0[i] = __builtin_amdgcn_raw_buffer_load_b128(r0, off, step * i, 0);
        v1[i] = __builtin_amdgcn_raw_buffer_load_b128(r1, off, step * i, 0);
    }
#pragma unroll
    for (int i = 0; i < N; ++i) {
        const int c = lane + i * 64;
        *reinterpret_cast<u32x4*>(lds0 + (c >> 3) * stride0 + (c & 7) * 8) = v0[i];
        *reinterpret_cast<u32x4*>(lds1 + (c >> 3) * stride1 + (c & 7) * 8) = v1[i];
    }
}

constexpr int kKS = 72;   // K rows in LDS: 144 bytes (row-form reads)
constexpr int kVS = 96;   // V rows in LDS: 192 bytes (transposing reads)

// ---------------------------------------------------------------------------
// forward: O = softmax(Q K^T / 8) V per (image, live head); log-sum-exp saved for p_f heads
// ---------------------------------------------------------------------------
struct WholeBatch {};   // no mask: every (image, head) pair is live, the first n_full positions are p_f

// One query tile of one pair: S^T = K Q^T against all key tiles, softmax over the keys, O^T = V^T P^T.
// qf: the tile's Q fragments (this lane's query); after_s() runs once the S products are issued (qf is
// free from then on).  Leaves the unnormalised O^T in ot, the row maximum in m, the row sum in sum.
template <int KT, typename AfterS>
__device__ __forceinline__ void fwd_unit(const bf16* Ks, const bf16* Vs, bf16x8 (&qf)[4], int tokens, int lane,
                                         f32x16 (&ot)[2], float& m, float& sum, AfterS&& after_s) {
    const int c = lane & 31, h = lane >> 5;
    // S^T tiles: rows = keys of tile u, column = this lane's query.  K fragments of tile u+1 are
    // fetched from LDS while the MFMAs of tile u run (one read behind each MFMA).
    f32x16 s[KT];
    const f32x16 zero_acc = zero16();   // shared C operand of every tile's first MFMA
    bf16x8 kf[3][4];   // the fragments of a tile are requested two tiles (eight products) before their use
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) kf[0][kk] = frag_rows(Ks, kKS, c, kk * 16 + 8 * h);
    if (KT > 1) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) kf[1][kk] = frag_rows(Ks, kKS, 32 + c, kk * 16 + 8 * h);
    }
#pragma unroll
    for (int u = 0; u < KT; ++u) {
        if (u + 2 < KT) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) kf[(u + 2) % 3][kk] = frag_rows(Ks, kKS, (u + 2) * 32 + c, kk * 16 + 8 * h);
        }
        s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u % 3][0], qf[0], zero_acc, 0, 0, 0);
#pragma unroll
        for (int kk = 1; kk < 4; ++kk)
            s[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[u % 3][kk], qf[kk], s[u], 0, 0, 0);
        if (u + 2 < KT) {
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    after_s();
    // first V fragments are fetched under the softmax arithmetic
    bf16x8 vf[2][4];
#pragma unroll
    for (int gp = 0; gp < 2; ++gp)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) vf[0][gp * 2 + dt] = frag_tr(Vs, kVS, 16 * gp, dt * 32, lane);
    {   // only the last key tile reaches past the last token (KT = ceil(tokens / 32)): element e of a lane
        // is key 32 (KT - 1) + 8 (e / 4) + 4 h + e % 4
        const int lim = tokens - (KT - 1) * 32 - 4 * h;
#pragma unroll
        for (int e = 0; e < 16; ++e)
            if (8 * (e >> 2) + (e & 3) >= lim) s[KT - 1][e] = -INFINITY;
    }
    m = -INFINITY;
#pragma unroll
    for (int u = 0; u < KT; ++u) {
        // three-input maxima: half the instructions of a chain of two-input ones
        float t0 = fmaxf(fmaxf(s[u][0], s[u][1]), s[u][2]);
        float t1 = fmaxf(fmaxf(s[u][3], s[u][4]), s[u][5]);
        float t2 = fmaxf(fmaxf(s[u][6], s[u][7]), s[u][8]);
        float t3 = fmaxf(fmaxf(s[u][9], s[u][10]), s[u][11]);
        float t4 = fmaxf(fmaxf(s[u][12], s[u][13]), s[u][14]);
        t0 = fmaxf(fmaxf(t0, t1), t2);
        t3 = fmaxf(fmaxf(t3, t4), s[u][15]);
        m = fmaxf(fmaxf(m, t0), t3);
    }
    m = fmaxf(m, __shfl_xor(m, 32, 64));
    const float cexp = kScale * kLog2e;
    const float mc = m * cexp;
    sum = 0.f;
    auto exp_tile = [&](int u) {
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const float p = __builtin_amdgcn_exp2f(fmaf(s[u][e], cexp, -mc));
            s[u][e] = p;
            sum += p;
        }
    };
    exp_tile(0);
    // O^T = V^T P^T: rows = channels, column = this lane's query.  The products of key tile u run on the
    // matrix cores while the vector units take the exponentials of tile u + 1; V fragments one tile ahead.
    ot[0] = zero16();
    ot[1] = zero16();
#pragma unroll
    for (int u = 0; u < KT; ++u) {
        const bf16x8 pf0 = pack8(s[u], 0), pf1 = pack8(s[u], 8);
        if (u + 1 < KT) {
#pragma unroll
            for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
                    vf[(u + 1) & 1][gp * 2 + dt] = frag_tr(Vs, kVS, (u + 1) * 32 + 16 * gp, dt * 32, lane);
        }
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) ot[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u & 1][dt], pf0, ot[dt], 0, 0, 0);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) ot[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[u & 1][2 + dt], pf1, ot[dt], 0, 0, 0);
        if (u + 1 < KT) {
            exp_tile(u + 1);
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);    // one product
                __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);    // two fragment reads
                __builtin_amdgcn_sched_group_barrier(0x002, 12, 0);   // a quarter of the tile's exponentials
            }
        }
        __builtin_amdgcn_sched_barrier(0);
    }
    sum += __shfl_xor(sum, 32, 64);   // the two lanes of a query hold different keys
}

// A transposed 64 x 32 result (rows = channels in two 32-row halves, column = this lane's token) times mul
// goes to the token's row.  A lane holds 4 consecutive channels per group of 8 and its partner 32 lanes up
// (same token) the other 4: the two exchange halves (v_permlane32_swap), so each stores 16-byte pieces and a
// row goes out as 32 contiguous bytes per store instruction.  All lanes must call; ok says whether this
// lane's token exists.
__device__ __forceinline__ void store_t_rows(const f32x16 (&ot)[2], float mul, bf16* orow, int h, bool ok) {
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t a[2], b[2];   // groups 2p and 2p + 1: this lane's 4 channels of each, packed
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                a[r] = pack_bf16x2(ot[dt][8 * p + 2 * r] * mul, ot[dt][8 * p + 2 * r + 1] * mul);
                b[r] = pack_bf16x2(ot[dt][8 * p + 4 + 2 * r] * mul, ot[dt][8 * p + 4 + 2 * r + 1] * mul);
                // upper half of a <-> lower half of b
                const auto sw = __builtin_amdgcn_permlane32_swap(a[r], b[r], false, false);
                a[r] = sw[0];
                b[r] = sw[1];
            }
            // lower lanes now hold channels 8 (2p) .. + 7 (their own 4, then the partner's), upper lanes 8 (2p + 1) .. + 7
            if (ok) *reinterpret_cast<uint4*>(orow + dt * 32 + 8 * (2 * p + h)) = make_uint4(a[0], a[1], b[0], b[1]);
        }
}

// this lane's query row of a forward unit: O = O^T columns / sum, and the log-sum-exp if asked for
__device__ __forceinline__ void fwd_store(const f32x16 (&ot)[2], float m, float sum, bf16* orow, float* lse_q, int h, bool ok) {
    store_t_rows(ot, 1.0f / sum, orow, h, ok);
    if (ok && h == 0 && lse_q) *lse_q = m * kScale + __logf(sum);
}

// the Q fragments of query q (16 bytes per 16-channel step), zeros for a query past the last token
__device__ __forceinline__ void load_q_frags(const bf16* Qb, long ldq, int q, bool q_ok, int h, bf16x8 (&qf)[4]) {
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        u32x4 v = {0u, 0u, 0u, 0u};
        if (q_ok) v = *reinterpret_cast<const u32x4*>(Qb + (long)q * ldq + kk * 16 + 8 * h);
        qf[kk] = __builtin_bit_cast(bf16x8, v);
    }
}

// which pair a (image, slot) position works on.  Without a mask slot j is live head j and the first n_full
// of them are p_f.  With a mask the position first zero-fills its share of the image's skipped heads (all
// threads of the workgroup), then takes the slot-th live head of the image's micro-batch, if there is one.
template <typename Mask>
__device__ __forceinline__ bool fwd_pair(const Mask& mask, int b, int slot, int n_live, int n_full, int tokens, bf16* o, long ldo,
                                         int& j, bool& save_lse) {
    j = slot;
    save_lse = slot < n_full;
    if constexpr (std::is_same<Mask, MicroMask>::value) {
        const long row0 = (long)b * tokens;
        const int mb = mask.micro_of(b);
        const uint64_t live = mask.live[mb];
        const uint64_t skipped = ~live & (mask.n_live_pos >= 64 ? ~0ull : ((1ull << mask.n_live_pos) - 1ull));
        int r = 0;
        for (uint64_t mm = skipped; mm; mm &= mm - 1, ++r)   // heads skipped in this image's micro-batch: O = 0
            if (r % n_live == slot) {
                const int p = __builtin_ctzll(mm);
                const u32x4 z = {0u, 0u, 0u, 0u};
                for (int i = threadIdx.x; i < tokens * 8; i += blockDim.x)
                    *reinterpret_cast<u32x4*>(o + (row0 + (i >> 3)) * ldo + p * 64 + (i & 7) * 8) = z;
            }
        if (slot >= __builtin_popcountll(live)) return false;
        uint64_t mm = live;
        for (int t = 0; t < slot; ++t) mm &= mm - 1;
        j = __builtin_ctzll(mm);   // this slot's live head
        save_lse = (mask.full[mb] >> j) & 1;
    }
    return true;
}

// One or two (gridDim.y) workgroups per (image, slot), four wavefronts each, that share the query tiles (tokens above 224,
// where the kernel below would need a ninth wavefront).  The exponentials of a query tile are most of a wavefront's time, so
// with few pairs a second workgroup takes half the tiles, at the price of loading K and V too, and the Q of a wavefront's first
// tile is requested ahead of them.  256 tokens: 12 pairs 10.2 -> 7.4 us, 120 pairs 12.8 -> 9.8, 384 pairs (one workgroup each)
// 24.8 -> 24.3.  Up to 224 tokens the kernel below is as fast in a pass of many kernels.
template <int KT, typename Mask>   // KT: number of 32-token tiles
__global__ __launch_bounds__(256, 2) void attn_fwd_mfma_kernel(const bf16* __restrict__ qkv, long ldq,
                                                            bf16* __restrict__ o, long ldo, float* __restrict__ lse,
                                                            int tokens, int n_live, int n_full, long rows_total,
                                                            Mask mask) {
    constexpr int TP = KT * 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16* Ks = reinterpret_cast<bf16*>(smem_raw);
    bf16* Vs = Ks + TP * kKS;
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int b = blockIdx.x / n_live;   // with a mask n_live is the number of slots per image
    const long row0 = (long)b * tokens;
    int j;
    bool save_lse;
    if (!fwd_pair(mask, b, blockIdx.x % n_live, n_live, n_full, tokens, o, ldo, j, save_lse)) return;
    const bf16* Qb = qkv + row0 * ldq + j * 192;
    const int first = blockIdx.y * 4 + wave, step = gridDim.y * 4;
    bf16x8 qf[4];
    load_q_frags(Qb, ldq, first * 32 + c, first * 32 + c < tokens, h, qf);   // ahead of K and V, which it would wait behind
    load_two_tiles64<TP>(Qb + 64, Qb + 128, ldq, tokens, Ks, kKS, Vs, kVS);
    __syncthreads();
    for (int qt = first; qt < KT; qt += step) {
        const int q = qt * 32 + c;
        const bool q_ok = q < tokens;
        if (qt != first) load_q_frags(Qb, ldq, q, q_ok, h, qf);
        f32x16 ot[2];
        float m, sum;
        fwd_unit<KT>(Ks, Vs, qf, tokens, lane, ot, m, sum, [] {});
        fwd_store(ot, m, sum, o + (row0 + q) * ldo + j * 64, save_lse ? lse + (long)j * rows_total + row0 + q : nullptr, h, q_ok);
    }
}

// Persistent form for up to 224 tokens: a workgroup of KT + 1 wavefronts walks the positions
// blockIdx.x, blockIdx.x + gridDim.x, ... (the grid is what the chip holds at once).  Wavefront t < KT
// owns query tile t of every pair; the last wavefront is the loader: while the others work on pair i out
// of one LDS buffer it copies K and V of pair i + 1 into the other, all its loads in flight at once, so
// after the first pair no wavefront waits for K or V.  A compute wavefront fetches the Q fragments of its
// next pair as soon as the S products of the current one are issued.  One barrier per pair.
template <int KT, typename Mask>
__global__ __launch_bounds__(64 * (KT + 1), 2) void attn_fwd_pipe_kernel(const bf16* __restrict__ qkv, long ldq,
                                                                        bf16* __restrict__ o, long ldo,
                                                                        float* __restrict__ lse, int tokens, int n_live,
                                                                        int n_full, long rows_total, int n_pos,
                                                                        Mask mask) {
    constexpr int TP = KT * 32, NTHR = 64 * (KT + 1);
    constexpr int BUF = TP * (kKS + kVS);   // elements of one K + V buffer
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    bf16* const smem = reinterpret_cast<bf16*>(smem_raw);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;

    int pos = blockIdx.x;
    int j = 0;
    bool save_lse = false;
    bool active = fwd_pair(mask, pos / n_live, pos % n_live, n_live, n_full, tokens, o, ldo, j, save_lse);
    {
        const bf16* Qb = qkv + (long)(pos / n_live) * tokens * ldq + j * 192;
        if (active) load_two_tiles64<TP, NTHR>(Qb + 64, Qb + 128, ldq, tokens, smem, kKS, smem + TP * kKS, kVS);
    }
    if (wave == KT) {
        // ---- loader: K and V of the next position into the other buffer, every load in flight at once ----
        __syncthreads();
        for (int i = 0; pos < n_pos; ++i) {
            const int npos = pos + gridDim.x;
            if (npos < n_pos) {
                int nj;
                bool nsave;
                if (fwd_pair(mask, npos / n_live, npos % n_live, n_live, n_full, tokens, o, ldo, nj, nsave)) {
                    const bf16* nQb = qkv + (long)(npos / n_live) * tokens * ldq + nj * 192;
                    bf16* nK = smem + ((i + 1) & 1) * BUF;
                    load_two_tiles64_wave<TP>(nQb + 64, nQb + 128, ldq, tokens, nK, kKS, nK + TP * kKS, kVS, lane);
                }
            }
            __syncthreads();
            pos = npos;
        }
    } else {
        // ---- compute: query tile `wave` of every position ----
        const int q = wave * 32 + c;
        const bool q_ok = q < tokens;
        bf16x8 qf[4];
        if (active) load_q_frags(qkv + (long)(pos / n_live) * tokens * ldq + j * 192, ldq, q, q_ok, h, qf);
        __syncthreads();
        for (int i = 0; pos < n_pos; ++i) {
            const bf16* const Ks = smem + (i & 1) * BUF;
            const bf16* const Vs = Ks + TP * kKS;
            const int npos = pos + gridDim.x;   // the next position of this workgroup (uniform over it)
            int nj = 0;
            bool nsave = false, nactive = false;
            if (npos < n_pos) nactive = fwd_pair(mask, npos / n_live, npos % n_live, n_live, n_full, tokens, o, ldo, nj, nsave);
            const bf16* nQb = qkv + (long)(npos < n_pos ? npos / n_live : 0) * tokens * ldq + nj * 192;
            if (active) {
                const long row0 = (long)(pos / n_live) * tokens;
                f32x16 ot[2];
                float m, sum;
                fwd_unit<KT>(Ks, Vs, qf, tokens, lane, ot, m, sum, [&] {
                    if (nactive) load_q_frags(nQb, ldq, q, q_ok, h, qf);
                });
                fwd_store(ot, m, sum, o + (row0 + q) * ldo + j * 64, save_lse ? lse + (long)j * rows_total + row0 + q : nullptr, h, q_ok);
            } else if (nactive) {
                load_q_frags(nQb, ldq, q, q_ok, h, qf);
            }
            __syncthreads();
            pos = npos;
            j = nj;
            save_lse = nsave;
            active = nactive;
        }
    }
}

template <int KT, typename Mask>
hipError_t launch_fwd_kt(const bf16* qkv, long ldq, bf16* o, long ldo, float* lse, int batch, int tokens, int n_live,
                         int n_full, const Mask& mask, hipStream_t s) {
    if constexpr (KT <= 7) {
        constexpr size_t lds = 2 * (size_t)KT * 32 * (kKS + kVS) * sizeof(bf16);
        constexpr int threads = 64 * (KT + 1);
        auto kern = attn_fwd_pipe_kernel<KT, Mask>;
        static KernelLimits limits;
        int resident = 0;
        if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), threads, lds, &resident); e != hipSuccess) return e;
        const int n_pos = batch * n_live;
        // every workgroup gets the same number of positions, give or take one
        const int rounds = (n_pos + resident - 1) / resident;
        const int grid = (n_pos + rounds - 1) / rounds;
        hipLaunchKernelGGL(kern, dim3(grid), dim3(threads), lds, s, qkv, ldq, o, ldo, lse, tokens, n_live, n_full,
                           (long)batch * tokens, n_pos, mask);
        return hipGetLastError();
    } else {
        constexpr size_t lds = (size_t)KT * 32 * (kKS + kVS) * sizeof(bf16);
        auto kern = attn_fwd_mfma_kernel<KT, Mask>;
        static KernelLimits limits;
        int resident = 0;   // not persistent
        if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 256, lds, &resident); e != hipSuccess) return e;
        const int pairs = batch * n_live, parts = pairs <= 128 ? 2 : 1;   // two: while each finds a CU of its own
        if (parts == 2) launch_label("attn_fwd_mfma, two per pair");
        hipLaunchKernelGGL(kern, dim3(pairs, parts), dim3(256), lds, s, qkv, ldq, o, ldo, lse, tokens, n_live, n_full,
                           (long)batch * tokens, mask);
        return hipGetLastError();
    }
}

// ---------------------------------------------------------------------------
// backward for p_f heads: dQ, dK, dV from Q, K, V, O, dO and the saved log-sum-exp
//
// Per 32x32 tile pair (query tile i, key tile u), in the orientation S = Q K^T (a lane owns one KEY
// column, its 16 result elements are 16 queries):
//     S  = Q_i K_u^T              P  = exp(S/8 - lse_q)          (probabilities are rebuilt, never stored)
//     dP = dO_i V_u^T             dS = P * (dP - delta_q),       delta_q = sum_d dO[q][d] O[q][d]
//     dV_u^T += dO_i^T P          dK_u^T += Q_i^T dS             (P, dS feed the MFMA straight from registers)
//     dQ_i^T  = sum_u K_u^T dS_iu^T
// The workgroup has KT wavefronts and all of Q, dO and dS in LDS (bf16; 160 KB at KT = 7).  Wavefront w first owns key
// tile w: K_w, V_w, dK_w and dV_w stay in registers while it walks the query tiles, which takes no barrier, and
// leaves every dS_iw in LDS.  Behind one barrier it owns query tile w: K has taken Q's place, and dQ_w is MFMA chains over
// all key tiles in a fixed order, so no partial sums cross wavefronts.  The walk is software-pipelined: the S and
// dP products of query tile i + 1 are issued before the exponentials of tile i, so the matrix cores work under the
// vector arithmetic.
// The per-query constants ride in the products: a query has -8 lse_q and -delta_q as three bf16 terms each in an
// extra channel group that meets ones on the K / V side, so the MFMAs deliver S - 8 lse and dP - delta (as the sums'
// initial values they are four times the LDS reads: 1 % slower).
// If bsum is given the kernel also writes the column sums of the pair's dQ, dK, dV rows (the
// gradient of the QKV bias: one row of 192 partial sums per image).
// What bounds it: two wavefronts of a SIMD, whose matrix and vector instructions do not overlap (a step of the walk is 1050
// cycles for each, 576 of them of products), then memory: 215 KB a pair, 19 us for 448 pairs.  With a wavefront
// apart for dQ and a barrier a query tile, 448 pairs of 197 tokens took 43.0 us in a block's passes; now 36 (0.7 of it for the
// sums of db_k and db_v as they are), 2048 pairs 165 -> 130, 1024 pairs of 64 tokens 24.4 -> 14.8.
// ---------------------------------------------------------------------------
typedef __attribute__((address_space(3))) unsigned char lds_u8;
typedef __attribute__((address_space(3))) float lds_f32;
typedef __attribute__((address_space(3))) bf16x4 lds_bf16x4;
// Rows of Q, dO and K are 128 bytes, whose eight 16-byte pieces change places: piece p of row r sits at p ^ row_swizzle(r).
// Both kinds of read are then free of bank conflicts: 16-byte pieces p of 16 rows (a row-form fragment), and 64 bytes of the
// four rows 4n .. 4n + 3 (half of a transposing one).
__device__ __forceinline__ int row_swizzle(int r) { return (r >> 1 & 1) << 2 | (r >> 2 & 1) << 1 | (r >> 3 & 1); }
// dS tiles are [32 keys][32 queries] in rows of 64 bytes with their four pieces exchanged likewise
__device__ __forceinline__ int ds_swizzle(int key) { return key >> 2 & 3; }

__device__ __forceinline__ bf16x8 read_piece(const lds_u8* p) { return *reinterpret_cast<const __attribute__((address_space(3))) bf16x8*>(p); }
__device__ __forceinline__ bf16x8 read_tr(const lds_u8* lo_at, const lds_u8* hi_at) {
    typedef s16x4 __attribute__((address_space(3))) * tr_ptr;
    const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)lo_at), hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((tr_ptr)hi_at);
    return __builtin_bit_cast(bf16x8, __builtin_shufflevector(lo, hi, 0, 1, 2, 3, 4, 5, 6, 7));
}

// Sums over the 32 columns of a transposed result t[2] (rows = channels, a column per lane of each half): lane l of a half gets
// channel 32 * (l / 16) + 8 * (l % 16 / 4) + 4 h + l % 4.  Each step adds lane to lane and halves the values that a lane keeps.
__device__ __forceinline__ float column_sum(const f32x16 (&t)[2], int lane) {
    float v[16];
#pragma unroll
    for (int e = 0; e < 16; ++e) {   // rows of 16 lanes: even ones keep t[0], odd ones t[1]
        const auto sw = __builtin_amdgcn_permlane16_swap(__float_as_uint(t[0][e]), __float_as_uint(t[1][e]), false, false);
        v[e] = __uint_as_float(sw[0]) + __uint_as_float(sw[1]);
    }
    auto halve = [&](auto n_tag, auto ctrl_tag, bool upper) {   // the lane across has `upper` the other way
        constexpr int N = decltype(n_tag)::value, CTRL = decltype(ctrl_tag)::value;
#pragma unroll
        for (int e = 0; e < N; ++e) {
            const float keep = upper ? v[e + N] : v[e], give = upper ? v[e] : v[e + N];
            v[e] = keep + dpp<CTRL>(give);
        }
    };
    constexpr int kDppRor8 = 0x128;
    halve(std::integral_constant<int, 8>{}, std::integral_constant<int, kDppRor8>{}, (lane & 8) != 0);
    halve(std::integral_constant<int, 4>{}, std::integral_constant<int, kDppHalfMirror>{}, (lane & 4) != 0);
    halve(std::integral_constant<int, 2>{}, std::integral_constant<int, kDppXor2>{}, (lane & 2) != 0);
    halve(std::integral_constant<int, 1>{}, std::integral_constant<int, kDppXor1>{}, (lane & 1) != 0);
    return v[0];
}

// f(integral_constant<int, 0>), f(integral_constant<int, 1>), ...: a loop whose index is a compile-time constant
template <typename F, int... I>
__device__ __forceinline__ void static_for_impl(F&& f, std::integer_sequence<int, I...>) {
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

// Pair n of those that are p_f (FULL) or of the others: its image and its position in the union layout.  n is below their number.
// A persistent workgroup takes every so many-th pair, so only those with work are numbered: dealt by image and slot, slots being
// the busiest micro-batch's p_f heads, 64 images of 9, 7, 7, 7 and 6 p_f heads made three rounds of the chip of 462 pairs.
template <bool FULL>
__host__ __device__ __forceinline__ uint64_t pairs_of(const MicroMask& mask, int micro) {
    return FULL ? mask.full[micro] : ~mask.full[micro] & (mask.n_full_pos >= 64 ? ~0ull : (1ull << mask.n_full_pos) - 1);
}
template <bool FULL>
__device__ __forceinline__ void nth_pair(const MicroMask& mask, int n, int& image, int& position) {
    int micro = 0, first = 0, count;   // of the micro-batch: its first image and its pairs per image
    for (;; ++micro) {
        count = __builtin_popcountll(pairs_of<FULL>(mask, micro));
        const int all = (mask.img_end[micro] - first) * count;
        if (n < all || micro + 1 >= mask.n) break;
        n -= all;
        first = mask.img_end[micro];
    }
    image = first + n / count;
    uint64_t m = pairs_of<FULL>(mask, micro);
    for (int k = n % count; k > 0; --k) m &= m - 1;
    position = __builtin_ctzll(m);
}
template <bool FULL>
int number_of_pairs(const MicroMask& mask) {
    int n = 0;
    for (int i = 0; i < mask.n; ++i) n += (mask.img_end[i] - (i ? mask.img_end[i - 1] : 0)) * __builtin_popcountll(pairs_of<FULL>(mask, i));
    return n;
}

template <int KT> struct BwdLds {   // byte offsets
    static constexpr int kTile = 32 * 128, kDsTile = 32 * 64;
    static constexpr int kQ = 0, kDo = KT * kTile;                 // Q, then K; dO
    static constexpr int kDs = 2 * KT * kTile;                     // [key tile][query tile]
    static constexpr int kLse = kDs + KT * KT * kDsTile;           // [query] three bf16 terms and 0 of -8 lse, ...
    static constexpr int kDelta = kLse + KT * 32 * 8;              // ... of -delta
    static constexpr int kSumV = kLse, kSumK = kDelta, kSumQ = kDo;   // later [tile][64] column sums of dV, dK and dQ
    static constexpr int kSk = kDelta + KT * 32 * 8;               // [key tile][3][32] sum over the queries of dS
    static constexpr int kBytes = kSk + KT * 192;
};

template <int KT, typename Mask>
__global__ __launch_bounds__(64 * KT, 2) void attn_bwd_mfma_kernel(const bf16* __restrict__ qkv, long ldq,
                                                                const bf16* __restrict__ o, long ldo,
                                                                const float* __restrict__ lse,
                                                                const bf16* __restrict__ d_o, long ld_do,
                                                                bf16* __restrict__ dqkv, long ld_dqkv,
                                                                float* __restrict__ bsum, long ld_bsum,
                                                                int tokens, int n_full, int pairs, int zeros, long rows_total,
                                                                Mask mask) {
    using At = BwdLds<KT>;
    constexpr bool kMasked = std::is_same<Mask, MicroMask>::value;
    constexpr int TP = KT * 32, NTHR = 64 * KT, NCH = 4;   // 16-byte pieces of a [TP][64] operand per thread
    static_assert(TP * 8 == NCH * NTHR, "an operand divides over the threads");
    extern __shared__ __attribute__((aligned(16))) unsigned char smem_raw[];
    lds_u8* const lds = (lds_u8*)smem_raw;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const u32x4 zero4 = {0u, 0u, 0u, 0u};
    // The workgroup takes pairs blockIdx.x, + gridDim.x, ...  Of the next pair it has the operands in registers, requested ahead
    // of the current one's dQ: all workgroups' first loads together take a third of a pair's time (36 MB at once).
    int pair = blockIdx.x;
    bf16* dQb = nullptr;
    float* bout = nullptr;
    u32x4 lq[NCH], lo[NCH], ldo_[NCH];   // pieces threadIdx.x + k * NTHR of Q, O, dO: eight lanes a row
    bf16x8 kfr[4], vfr[4];               // rows key of K and V: 8 channels at kk * 16 + 8 h
    float lse_q = 0.f;
    // What depends on the thread is formed anew for each pair: carried from one to the next it would take the registers that the
    // walk needs (26 of them spilled, and a reload waits for all stores under way).
    auto own_thread = [&]() {
        int t = threadIdx.x;
        asm volatile("" : "+v"(t));
        return t;
    };
    auto request = [&]() {   // every load of pair's operands
        int b, j;
        if constexpr (kMasked) {
            nth_pair<true>(mask, pair, b, j);
        } else {
            b = pair / n_full;
            j = pair % n_full;
        }
        const long row0 = (long)b * tokens;
        // Raw buffer loads whose declared size ends with the last token's row: rows above read as zeros.  Places of queries past
        // the last repeat its Q and log-sum-exp under a dO of zero: with a Q of zero a key that is infinite has a score of NaN there.
        auto rows_of = [&](const bf16* p, long ld) {
            return __builtin_amdgcn_make_buffer_rsrc(const_cast<bf16*>(p), 0, (uint32_t)(tokens - 1) * (uint32_t)ld * 2u + 128u, 0x00020000);
        };
        const bf16* Qb = qkv + row0 * ldq + j * 192;
        const __amdgpu_buffer_rsrc_t rq = rows_of(Qb, ldq), rk = rows_of(Qb + 64, ldq), rv = rows_of(Qb + 128, ldq);
        const __amdgpu_buffer_rsrc_t ro = rows_of(o + row0 * ldo + j * 64, ldo), rd = rows_of(d_o + row0 * ld_do + j * 64, ld_do);
        const int tid = own_thread();
        const uint32_t row = tid >> 3, ch = (tid & 7) * 16, krow = wave * 32 + (tid & 31), kch = (tid >> 5 & 1) * 16;
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            const uint32_t q = row + k * (NTHR / 8);
            ldo_[k] = __builtin_amdgcn_raw_buffer_load_b128(rd, q * (uint32_t)ld_do * 2u + ch, 0, 0);
            lo[k] = __builtin_amdgcn_raw_buffer_load_b128(ro, q * (uint32_t)ldo * 2u + ch, 0, 0);
            const bool past = (k + 1) * (NTHR / 8) > TP - 31;   // whether some of these rows may be: tokens is TP - 31 or more
            lq[k] = __builtin_amdgcn_raw_buffer_load_b128(rq, (past ? min(q, (uint32_t)tokens - 1u) : q) * (uint32_t)ldq * 2u + ch, 0, 0);
        }
        lse_q = lse[(long)j * rows_total + row0 + min(tid, tokens - 1)];   // tokens <= TP <= NTHR
        const uint32_t at_kv = krow * (uint32_t)ldq * 2u + kch;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            kfr[kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rk, at_kv + kk * 32, 0, 0));
            vfr[kk] = __builtin_bit_cast(bf16x8, __builtin_amdgcn_raw_buffer_load_b128(rv, at_kv + kk * 32, 0, 0));
        }
        dQb = dqkv + row0 * ld_dqkv + j * 192;
        bout = bsum ? bsum + (long)b * ld_bsum + j * 192 : nullptr;
    };
    // Pairs that are not p_f in their image's micro-batch: dQ = dK = dV = 0.  The workgroups take them in turn from the last one on,
    // whose list of pairs may be the shorter one, and write one block with each pair and the rest at the end.
    int zero = (int)(gridDim.x - 1 - blockIdx.x);
    auto zero_next = [&]() {
        if constexpr (kMasked) {
            if (zero >= zeros) return;
            int b, j;
            nth_pair<false>(mask, zero, b, j);
            zero += gridDim.x;
            bf16* const zb = dqkv + (long)b * tokens * ld_dqkv + j * 192;
            const int t = own_thread();
            for (int i = t; i < tokens * 24; i += NTHR) *reinterpret_cast<u32x4*>(zb + (long)(i / 24) * ld_dqkv + (i % 24) * 8) = zero4;
            if (bsum)
                for (int i = t; i < 192; i += NTHR) bsum[(long)b * ld_bsum + j * 192 + i] = 0.f;
        }
    };
    auto store_terms = [&](int at, float a) {
        const __bf16 t0 = static_cast<__bf16>(a);
        const float r1 = a - static_cast<float>(t0);
        const __bf16 t1 = static_cast<__bf16>(r1);
        const __bf16 t2 = static_cast<__bf16>(r1 - static_cast<float>(t1));
        *reinterpret_cast<lds_bf16x4*>(lds + at) = bf16x4{t0, t1, t2, static_cast<__bf16>(0.f)};
    };

    const float cexp = kScale * kLog2e;
    auto next = [&]() -> bool {   // to the workgroup's next pair
        // (what the registers held is not kept where there is none: they are free during the walk)
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            lq[k] = lo[k] = ldo_[k] = zero4;
            kfr[k] = vfr[k] = bf16x8{};
        }
        if (pair >= pairs) return false;
        request();
        return true;
    };
    bool more = next();
    while (more) {
        // a lane's places in a tile's rows of 128 bytes: formed anew behind the walk as well
        int tid, lane, c, h, key;               // key: the lane's key in the walk, its query behind it
        uint32_t at_row[4], at_tr[2][2];   // [kk]; [channel half][lower, upper rows]
        auto tr_row = [&]() { return 4 * h + ((lane & 15) >> 2); };                                   // of a transposing read,
        auto tr_piece = [&]() { return 2 * (lane >> 4 & 1) + ((lane & 3) >> 1); };                    // its 16-byte piece,
        auto tr_half = [&]() { return (lane & 1) * 8; };                                              // and half of that
        auto locate = [&]() {
            tid = own_thread();
            lane = tid & 63;
            c = lane & 31;
            h = lane >> 5;
            key = wave * 32 + c;
#pragma unroll
            for (int i = 0; i < 4; ++i) at_row[i] = c * 128 + (((2 * i + h) ^ row_swizzle(c)) << 4);
#pragma unroll
            for (int i = 0; i < 2; ++i)
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) {
                    const int r = tr_row() + 8 * i;
                    at_tr[dt][i] = r * 128 + (((4 * dt + tr_piece()) ^ row_swizzle(r)) << 4) + tr_half();
                }
        };
        locate();
        const float key_off = key < tokens ? 0.f : -INFINITY;   // keys beyond the last token: P = 0
        const short one_h = h == 0 ? (short)0x3F80 : (short)0;   // bf16 1.0 against the three terms of a query's constant
        const s16x8 ones_s = {one_h, one_h, one_h, 0, 0, 0, 0, 0};
        const bf16x8 ones = __builtin_bit_cast(bf16x8, ones_s);
        uint32_t at_ds[4];   // of the lane's eight bytes eg in the dS of its key
#pragma unroll
        for (int i = 0; i < 4; ++i) at_ds[i] = At::kDs + wave * (KT * At::kDsTile) + c * 64 + ((i ^ ds_swizzle(c)) << 4) + h * 8;
        auto rows = [&](int region, int tile, int kk) { return read_piece(lds + at_row[kk] + (region + tile * At::kTile)); };
        auto terms = [&](int region, int tile) {   // the upper lanes' terms meet zeros
            const bf16x4 v = *reinterpret_cast<const lds_bf16x4*>(lds + region + c * 8 + tile * 256);
            return __builtin_shufflevector(v, bf16x4{}, 0, 1, 2, 3, 4, 5, 6, 7);
        };
        auto columns = [&](int region, int tile, int gp, int dt) {   // tokens 16 gp + .. of a tile, channels dt * 32 + c
            const int at = region + tile * At::kTile + gp * (16 * 128);
            return read_tr(lds + at_tr[dt][0] + at, lds + at_tr[dt][1] + at);
        };
#pragma unroll
        for (int k = 0; k < NCH; ++k) {
            const int id = tid + k * NTHR, q = id >> 3;
            const int at = q * 128 + (((id & 7) ^ row_swizzle(q)) << 4);
            *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(lds + At::kQ + at) = lq[k];
            *reinterpret_cast<__attribute__((address_space(3))) u32x4*>(lds + At::kDo + at) = ldo_[k];
            // delta_q = sum_d dO[q][d] O[q][d]: eight lanes per query
            float dl = 0.f;
#pragma unroll
            for (int i = 0; i < 4; ++i) {
                dl = fmaf(__uint_as_float(ldo_[k][i] << 16), __uint_as_float(lo[k][i] << 16), dl);
                dl = fmaf(__uint_as_float(ldo_[k][i] & 0xffff0000u), __uint_as_float(lo[k][i] & 0xffff0000u), dl);
            }
            dl += __shfl_xor(dl, 1, 64);
            dl += __shfl_xor(dl, 2, 64);
            dl += __shfl_xor(dl, 4, 64);
            if ((id & 7) == 0) store_terms(At::kDelta + q * 8, -dl);
        }
        if (tid < TP) store_terms(At::kLse + tid * 8, -8.f * lse_q);

        __syncthreads();
        float sk = 0.f;   // sum over the queries of dS[.][key]
        {
            f32x16 dKt[2], dVt[2];   // dK^T and dV^T of the key tile: rows = channels, column = key
#pragma unroll
            for (int dt = 0; dt < 2; ++dt) {
                dKt[dt] = zero16();
                dVt[dt] = zero16();
            }
            f32x16 sc[2];   // S - 8 lse of query tile t: [t & 1]
            sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(terms(At::kLse, 0), ones, zero16(), 0, 0, 0);
#pragma unroll
            for (int kk = 0; kk < 4; ++kk) sc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(rows(At::kQ, 0, kk), kfr[kk], sc[0], 0, 0, 0);
            bf16x8 dof[5], qnf[5];   // rows of dO of the step's tile, of Q of the next one
            auto request_rows = [&](int i) {
                dof[4] = terms(At::kDelta, i);
#pragma unroll
                for (int kk = 0; kk < 4; ++kk) dof[kk] = rows(At::kDo, i, kk);
                if (i + 1 < KT) {
                    qnf[4] = terms(At::kLse, i + 1);
#pragma unroll
                    for (int kk = 0; kk < 4; ++kk) qnf[kk] = rows(At::kQ, i + 1, kk);
                }
            };
            request_rows(0);
            __builtin_amdgcn_sched_barrier(0);
            static_for<KT>([&](auto step_index) {
                constexpr int i = decltype(step_index)::value;
                constexpr bool NEXT = i + 1 < KT;
                // Issue order of a step: dP of this tile and S of the next one on the matrix cores, with the transposing
                // reads and, on the vector ALUs, the exponentials of this tile's S (computed one step ago) between
                // them; the next step's rows; dV with dS and its hand-over between the MFMAs; dK.
                bf16x8 dot[2][2], qt[2][2];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) dot[gp][dt] = columns(At::kDo, i, gp, dt);
#pragma unroll
                for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) qt[gp][dt] = columns(At::kQ, i, gp, dt);
                f32x16 dp = zero16(), sn = zero16();   // dP - delta, and S - 8 lse of the next tile
                f32x16& s = sc[i & 1];
#pragma unroll
                for (int kk = 0; kk < 5; ++kk) {
                    dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dof[kk], kk < 4 ? vfr[kk & 3] : ones, dp, 0, 0, 0);
                    if (NEXT) sn = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qnf[kk], kk < 4 ? kfr[kk & 3] : ones, sn, 0, 0, 0);
                }
#pragma unroll
                for (int e = 0; e < 16; ++e) s[e] = __builtin_amdgcn_exp2f(fmaf(s[e], cexp, key_off));   // P
                bf16x8 pf[2];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) pf[gp] = pack8(s, 8 * gp);
                {
                    constexpr int NM = NEXT ? 10 : 5;   // MFMAs of this phase; 40 vector ALU instructions
#pragma unroll
                    for (int k = 0; k < NM; ++k) {
                        __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                        if (k < 8) __builtin_amdgcn_sched_group_barrier(0x100, NEXT ? 2 : 4, 0);
                        __builtin_amdgcn_sched_group_barrier(0x002, (40 + NM - 1) / NM, 0);
                    }
                }
                if (NEXT) sc[(i + 1) & 1] = sn;
                __builtin_amdgcn_sched_barrier(0);
                if (NEXT) request_rows(i + 1);   // they arrive under the rest of the step
                __builtin_amdgcn_sched_barrier(0);
                f32x16 ds;
                bf16x8 dsf[2];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt)
                        dVt[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(dot[gp][dt], pf[gp], dVt[dt], 0, 0, 0);
#pragma unroll
                for (int e = 0; e < 16; ++e) ds[e] = s[e] * dp[e];
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) dsf[gp] = pack8(ds, 8 * gp);
                // elements 4 eg .. + 3 are queries 8 eg + 4 h .. of the tile: 8-byte pieces of the key's row
#pragma unroll
                for (int eg = 0; eg < 4; ++eg) {
                    const bf16x4 v = eg & 1 ? __builtin_shufflevector(dsf[eg >> 1], dsf[eg >> 1], 4, 5, 6, 7)
                                            : __builtin_shufflevector(dsf[eg >> 1], dsf[eg >> 1], 0, 1, 2, 3);
                    *reinterpret_cast<__attribute__((address_space(3))) bf16x4*>(lds + at_ds[eg] + i * At::kDsTile) = v;
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {   // 4 MFMAs; 16 products, 8 conversions, 4 stores
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x002, 6, 0);
                    __builtin_amdgcn_sched_group_barrier(0x200, 1, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt)
                        dKt[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qt[gp][dt], dsf[gp], dKt[dt], 0, 0, 0);
                if (bsum) {   // uniform over the grid; under the products above
                    float t = 0.f;
#pragma unroll
                    for (int e = 0; e < 16; ++e) t += ds[e];
                    sk += t;
                }
                __builtin_amdgcn_sched_barrier(0);
            });
            locate();
            // dK^T and dV^T: straight from the accumulators, 16-byte pieces after a half-wave exchange.  dK's column sums are not
            // formed: sum_k dK[k][.] = (1/8) sum_q (sum_k dS[q][k]) Q[q][.] and sum_k dS[q][k] = sum_k P dP - delta_q = 0 (softmax
            // does not see a shift of all keys), so the key bias gradient is written as the zero it is, but for channels in which a
            // dK is not finite: those show it.
            store_t_rows(dKt, kScale, dQb + (long)key * ld_dqkv + 64, h, key < tokens);
            store_t_rows(dVt, 1.f, dQb + (long)key * ld_dqkv + 128, h, key < tokens);
            // the column sums of the wavefront's dV and dK, fp32; this lane's channel
            const int sum_channel = (lane >> 4 & 1) * 32 + (lane >> 2 & 3) * 8 + h * 4 + (lane & 3);
            float sum_v = 0.f, sum_k = 0.f;
            if (bsum) {
                if (key >= tokens) dKt[0] = dKt[1] = dVt[0] = dVt[1] = zero16();   // zeros, or NaN
                sum_v = column_sum(dVt, lane);
                float odd = 0.f;   // stays 0, or becomes NaN
#pragma unroll
                for (int e = 0; e < 16; ++e) odd = fmaf(dKt[0][e], 0.f, fmaf(dKt[1][e], 0.f, odd));
                if (__any(odd != 0.f)) {
                    sum_k = column_sum(dKt, lane);
                    if (fabsf(sum_k) < INFINITY) sum_k = 0.f;
                }
            }
            __syncthreads();   // dS is complete; Q and dO are free
#pragma unroll
            for (int kk = 0; kk < 4; ++kk)   // K in Q's place
                *reinterpret_cast<__attribute__((address_space(3))) bf16x8*>(lds + at_row[kk] + (At::kQ + wave * At::kTile)) = kfr[kk];
            if (bsum) {
                sk += __shfl_xor(sk, 32, 64);
                if (h == 0) {   // rows of 32 keys: three bf16 terms
                    float rest = sk;
#pragma unroll
                    for (int i = 0; i < 3; ++i) {
                        const __bf16 term = static_cast<__bf16>(rest);
                        rest = fabsf(static_cast<float>(term)) < INFINITY ? rest - static_cast<float>(term) : 0.f;   // infinity is one term
                        *reinterpret_cast<__attribute__((address_space(3))) __bf16*>(lds + At::kSk + wave * 192 + i * 64 + c * 2) = term;
                    }
                }
            }
            if (bsum) {
                *reinterpret_cast<lds_f32*>(lds + At::kSumK + (wave * 64 + sum_channel) * 4) = sum_k;
                *reinterpret_cast<lds_f32*>(lds + At::kSumV + (wave * 64 + sum_channel) * 4) = sum_v;
            }
        }
        __syncthreads();   // K is in LDS
        bf16* const dq_now = dQb;
        float* const bout_now = bout;
        zero_next();
        pair += gridDim.x;
        more = next();
        {
            // dQ^T of query tile `wave`: rows = channels, column = query c; four MFMA chains (channel half x 16-key half),
            // added pairwise at the end
            f32x16 acc[2][2] = {{zero16(), zero16()}, {zero16(), zero16()}};
            uint32_t at_dst[2];   // [lower, upper keys] of a transposing read of dS
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const int r = tr_row() + 8 * i;
                at_dst[i] = At::kDs + wave * At::kDsTile + r * 64 + ((tr_piece() ^ ds_swizzle(r)) << 4) + tr_half();
            }
            bf16x8 dsf[2][2], ktf[2][2][2];   // a key tile's fragments are requested ahead of the products of the one before
            auto request_tile = [&](int v) {
                const int at = v * (KT * At::kDsTile);
#pragma unroll
                for (int gp = 0; gp < 2; ++gp) {
                    dsf[v & 1][gp] = read_tr(lds + at_dst[0] + at + gp * (16 * 64), lds + at_dst[1] + at + gp * (16 * 64));   // column = query, slots = keys
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt) ktf[v & 1][gp][dt] = columns(At::kQ, v, gp, dt);
                }
            };
            request_tile(0);
            static_for<KT>([&](auto v_index) {
                constexpr int v = decltype(v_index)::value;
                if constexpr (v + 1 < KT) request_tile(v + 1);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int gp = 0; gp < 2; ++gp)
#pragma unroll
                    for (int dt = 0; dt < 2; ++dt)
                        acc[gp][dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(ktf[v & 1][gp][dt], dsf[v & 1][gp], acc[gp][dt], 0, 0, 0);
                __builtin_amdgcn_sched_barrier(0);
            });
#pragma unroll
            for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                for (int e = 0; e < 16; ++e) acc[0][dt][e] += acc[1][dt][e];
            store_t_rows(acc[0], kScale, dq_now + (long)key * ld_dqkv, h, key < tokens);
        }
        if (bsum) {
            // The column sums of dQ = (1/8) dS K follow from the query sums of dS: sum_q dQ[q][d] = (1/8) sum_k sk[k] K[k][d].  Each
            // wavefront takes its 32 keys, sk as three rows of bf16 terms.
            f32x16 sum[2] = {zero16(), zero16()};
#pragma unroll
            for (int gp = 0; gp < 2; ++gp) {
                const lds_u8* const at = lds + At::kSk + wave * 192 + min(c, 2) * 64 + (16 * gp + 4 * h) * 2;   // further rows' results go unread
                const bf16x4 lower = *reinterpret_cast<const lds_bf16x4*>(at), upper = *reinterpret_cast<const lds_bf16x4*>(at + 16);
                const bf16x8 sf = __builtin_shufflevector(lower, upper, 0, 1, 2, 3, 4, 5, 6, 7);
#pragma unroll
                for (int dt = 0; dt < 2; ++dt) sum[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(sf, columns(At::kQ, wave, gp, dt), sum[dt], 0, 0, 0);
            }
            if (h == 0) {
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)   // rows 0 to 2
                    *reinterpret_cast<lds_f32*>(lds + At::kSumQ + (wave * 64 + dt * 32 + c) * 4) = (sum[dt][0] + sum[dt][1] + sum[dt][2]) * kScale;
            }
            __syncthreads();
            for (int i = tid; i < 192; i += NTHR) {   // tiles added in index order
                float t = 0.f;
                const lds_u8* const at = lds + (i < 64 ? At::kSumQ : i < 128 ? At::kSumK : At::kSumV);
#pragma unroll
                for (int v = 0; v < KT; ++v) t += reinterpret_cast<const lds_f32*>(at)[v * 64 + (i & 63)];
                bout_now[i] = t;
            }
        }
        __syncthreads();   // all of it has been read: the next pair takes its place
    }
    if constexpr (kMasked)
        while (zero < zeros) zero_next();
}

template <int KT, typename Mask>
hipError_t launch_bwd_kt(const bf16* qkv, long ldq, const bf16* o, long ldo, const float* lse, const bf16* d_o, long ld_do,
                         bf16* dqkv, long ld_dqkv, float* bsum, long ld_bsum, int batch, int tokens, int n_full,
                         const Mask& mask, hipStream_t s) {
    constexpr size_t lds = BwdLds<KT>::kBytes;
    static_assert(lds <= 160 * 1024, "the pair's tiles must fit a compute unit's LDS");
    auto kern = attn_bwd_mfma_kernel<KT, Mask>;
    static KernelLimits limits;
    int resident = 0;
    if (const hipError_t e = limits.get(reinterpret_cast<const void*>(kern), 64 * KT, lds, &resident); e != hipSuccess) return e;
    int pairs = batch * n_full, zeros = 0;
    if constexpr (std::is_same<Mask, MicroMask>::value) {
        pairs = number_of_pairs<true>(mask);
        zeros = number_of_pairs<false>(mask);
    }
    const dim3 grid(pairs + zeros < resident ? pairs + zeros : resident), block(64 * KT);
    return launch_signalling(kern, grid, block, lds, s, qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, ld_bsum, tokens, n_full, pairs,
                             zeros, (long)batch * tokens, mask);
}

}  // namespace

bool attn_mfma_supported(int tokens, long ldq, long ldo) {
    return tokens >= 1 && tokens <= 256 && (ldq % 8) == 0 && (ldo % 8) == 0;
}
// The backward keeps Q, dO and dS of a pair in LDS, which holds them for at most seven tiles of 32 tokens.
bool attn_bwd_mfma_supported(int tokens, long ldq, long ldo) {
    return attn_mfma_supported(tokens, ldq, ldo) && tokens <= 224;
}

template <typename Mask>
static hipError_t attn_fwd_dispatch(const void* qkv, long ldq, void* o, long ldo, float* lse, int batch, int tokens,
                                    int n_live, int n_full, const Mask& mask, hipStream_t s) {
    if (n_live <= 0) return hipSuccess;
    const bf16* q = static_cast<const bf16*>(qkv);
    bf16* op = static_cast<bf16*>(o);
#define D2FT_FWD_CASE(KT) \
    case KT: return launch_fwd_kt<KT, Mask>(q, ldq, op, ldo, lse, batch, tokens, n_live, n_full, mask, s);
    switch ((tokens + 31) / 32) {
        D2FT_FWD_CASE(1) D2FT_FWD_CASE(2) D2FT_FWD_CASE(3) D2FT_FWD_CASE(4)
        D2FT_FWD_CASE(5) D2FT_FWD_CASE(6) D2FT_FWD_CASE(7) D2FT_FWD_CASE(8)
        default: return hipErrorNotSupported;
    }
#undef D2FT_FWD_CASE
}

hipError_t launch_attn_fwd_mfma(const void* qkv, long ldq, void* o, long ldo, float* lse, int batch, int tokens,
                                int n_live, int n_full, hipStream_t s) {
    return attn_fwd_dispatch(qkv, ldq, o, ldo, lse, batch, tokens, n_live, n_full, WholeBatch{}, s);
}

static int busiest(const uint64_t* sel, int n) {   // most pairs that take part in one micro-batch
    int slots = 0;
    for (int i = 0; i < n; ++i) {
        const int c = __builtin_popcountll(sel[i]);
        slots = c > slots ? c : slots;
    }
    return slots;
}

hipError_t launch_attn_fwd_mfma_masked(const void* qkv, long ldq, void* o, long ldo, float* lse, int batch, int tokens,
                                       int n_live, const MicroMask& mask, hipStream_t s) {
    if (n_live != mask.n_live_pos) return hipErrorInvalidValue;
    const int slots = busiest(mask.live, mask.n);
    return attn_fwd_dispatch(qkv, ldq, o, ldo, lse, batch, tokens, slots > 0 ? slots : 1, 0, mask, s);
}

}  // namespace d2ft

namespace d2ft {

template <typename Mask>
static hipError_t attn_bwd_dispatch(const void* qkv, long ldq, const void* o, long ldo, const float* lse, const void* d_o,
                                    long ld_do, void* dqkv, long ld_dqkv, float* bsum, long ld_bsum, int batch, int tokens,
                                    int n_full, const Mask& mask, hipStream_t s) {
    if (n_full <= 0) return hipSuccess;
    const bf16* q = static_cast<const bf16*>(qkv);
    const bf16* op = static_cast<const bf16*>(o);
    const bf16* dop = static_cast<const bf16*>(d_o);
    bf16* dq = static_cast<bf16*>(dqkv);
#define D2FT_BWD_CASE(KT) \
    case KT: return launch_bwd_kt<KT, Mask>(q, ldq, op, ldo, lse, dop, ld_do, dq, ld_dqkv, bsum, ld_bsum, batch, tokens, n_full, mask, s);
    switch ((tokens + 31) / 32) {
        D2FT_BWD_CASE(1) D2FT_BWD_CASE(2) D2FT_BWD_CASE(3) D2FT_BWD_CASE(4)
        D2FT_BWD_CASE(5) D2FT_BWD_CASE(6) D2FT_BWD_CASE(7)
        default: return hipErrorNotSupported;
    }
#undef D2FT_BWD_CASE
}

hipError_t launch_attn_bwd_mfma(const void* qkv, long ldq, const void* o, long ldo, const float* lse, const void* d_o,
                                long ld_do, void* dqkv, long ld_dqkv, float* bsum, long ld_bsum, int batch, int tokens,
                                int n_full, hipStream_t s) {
    return attn_bwd_dispatch(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, ld_bsum, batch, tokens, n_full,
                             WholeBatch{}, s);
}

hipError_t launch_attn_bwd_mfma_masked(const void* qkv, long ldq, const void* o, long ldo, const float* lse,
                                       const void* d_o, long ld_do, void* dqkv, long ld_dqkv, float* bsum, long ld_bsum,
                                       int batch, int tokens, int n_full, const MicroMask& mask, hipStream_t s) {
    if (n_full != mask.n_full_pos) return hipErrorInvalidValue;
    return attn_bwd_dispatch(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, ld_bsum, batch, tokens, n_full, mask, s);
}

}  // namespace d2ft
