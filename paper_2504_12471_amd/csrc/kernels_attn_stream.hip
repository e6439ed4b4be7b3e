// Softmax attention on the matrix cores for head dimension 64 with the keys (forward, dQ) or the queries (dK, dV)
// streamed through LDS: any number of tokens, bf16 and fp32 storage, fp32 accumulate.  It serves fp32 at every token
// count, bf16 above the tokens that kernels_attn_mfma.hip keeps on chip whole (256 forward, 224 backward), and below them,
// from 129 tokens on, the backward of few pairs (attn_bwd_stream_faster).
//
// A wavefront owns 32 queries (or keys): their rows sit in registers as the B operand of every product and their
// results as accumulators, so nothing but the streamed tiles goes through LDS and no partial sum crosses a
// wavefront.  Four wavefronts of a workgroup share the streamed tiles, which are double-buffered with the next
// stage's loads in flight under the current one's products (one barrier per stage).
//   forward  S^T = K Q^T (a lane owns one query), running maximum and sum per lane, O^T += V^T P^T
//   dQ       S^T and dP^T = V dO^T from the same tiles, dS^T = P^T (dP^T - delta), dQ^T += K^T dS^T
//   dK, dV   S = Q K^T and dP = dO V^T (a lane owns one key), dV^T += dO^T P, dK^T += Q^T dS
// Probabilities are rebuilt from the saved log-sum-exp.  P and dS enter the second products with all their bits: as three
// bf16 parts each (cut8), for bf16 storage three products instead of one.  fp32 operands are cut likewise, on their way to LDS or
// registers, and six of the nine products of parts are formed (kernels_gemm_split.hip): 1152 cycles of the matrix cores where
// the fp32 instruction takes 3072 for the same k.  Up to 224 tokens the bf16
// backward rounds them to bf16, as kernels_attn_mfma.hip does, which runs the other calls of those lengths (TR_PARTS).
// Relative 2-norm error against fp64 of O / dQ / dV, N(0, 1) operands, 577 tokens: bf16 1.66e-3 / 1.68e-3 / 1.66e-3, the
// same as the vector-ALU kernels (with P and dS rounded to bf16 2.18e-3 / 2.39e-3 / 2.38e-3); fp32 4.0e-7 / 5.4e-7 /
// 5.3e-7 (by the fp32 instruction 4.8e-7 / 6.1e-7 / 5.8e-7, the vector-ALU kernels 5.3e-7 / 6.5e-7 / 6.3e-7); with scores of
// 16 times the spread 5.6e-7 / 1.8e-6 / 1.2e-6 (8.7e-7 / 2.4e-6 / 1.4e-6 and 1.5e-6 / 3.8e-6 / 1.8e-6).
//
// dQ and dK/dV workgroups are independent (both form delta_q = sum_d dO[q][d] O[q][d] for the rows they touch) and
// share one launch, so that the second kind fills the last round of the first.  S and dP are formed twice, 7 products of 64 x 32 x 32 per tile pair instead of 5: keeping
// dQ partial sums instead would mean fp32 atomics, whose order is not fixed, or a pass over them.
//
// Bound: fp32 by the matrix cores (a 32 x 32 tile pair is 48 products of 32 cycles forward, 168 backward) and by what runs
// between them: a part of an infinity is a NaN, an operand of 2^104 and more has no parts, and sums end at 2^80, as products
// carry 2^48.  So a workgroup with a result that is not finite, with a Q or K above 2^36 or with a query whose log-sum-exp is beyond
// 1024 forms its rows again with the fp32 instruction.  (These tests cost 1 %: 197 tokens, 260 pairs, forward 38.7 -> 38.8
// us, backward 136.0 -> 136.6; a test of the log-sum-exp where it is fetched, not where it is stored, 5 %.  Where every pair
// falls back, 400 pairs take 107 and 396 us instead of 48 and 176.)  The backward holds two row operands in parts (96
// registers): one wavefront per SIMD.  bf16 by the
// matrix cores and the vector ALUs alike (forward 16 products of 32 cycles per tile pair, beside 16 exponentials, twice as
// many subtractions and multiplications, maxima, sums and the cutting into parts, 5.5 operations for each of 16 elements).
//
// Measured against the vector-ALU kernels it replaced (one wavefront per row, every row of K and V from cache for
// every query), per launch: bf16, 16 images of 577 tokens, 160 live / 112 p_f pairs: forward 1440 -> 53 us, backward
// 4004 -> 94 us (30 and 65 with P and dS in one part); fp32, 16 images of 197 tokens, 80 / 64 pairs: forward 172 -> 21 -> 17 us,
// backward 486 -> 39 -> 30 us (by the fp32 instruction, by parts); 400 / 320 pairs 68 -> 46 and 159 -> 131; 4 images of 65
// tokens, 8 / 4 pairs 10.3 -> 8.9 and 18.2 -> 14.9.
//
// Result layout of both products: column c = lane % 32, element e <-> row 8*(e/4) + 4h + e%4, h = lane / 32.
#include <atomic>
#include <type_traits>

#include "d2ft_common.h"
#include "launch.h"

namespace d2ft {

typedef __attribute__((__vector_size__(8 * sizeof(__bf16)))) __bf16 bf16x8;
typedef __attribute__((__vector_size__(16 * sizeof(float)))) float f32x16;
typedef __attribute__((__vector_size__(4 * sizeof(float)))) float f32x4;
typedef __attribute__((__vector_size__(4 * sizeof(short)))) short s16x4;
typedef __attribute__((__vector_size__(8 * sizeof(short)))) short s16x8;
typedef __attribute__((__vector_size__(4 * sizeof(uint32_t)))) uint32_t u32x4;

namespace {

// How fp32 storage is multiplied: Parts, as three bf16 parts of each element on the bf16 matrix cores, or float, by the fp32
// instruction, which a workgroup falls back on when a result of the parts is not finite.  bf16 is its own.
struct Parts {};
template <typename Op> struct Storage { typedef Op type; };      // in memory
template <> struct Storage<Parts> { typedef float type; };
template <typename Op> struct InTile { typedef Op type; };       // in LDS
template <> struct InTile<Parts> { typedef bf16 type; };

// The parts are those of x * 2^24, exact whatever x (kernels_gemm_split.hip); products are 2^48 of theirs.
constexpr float kUp = 16777216.f;            // 2^24
constexpr float kDown = 3.5527136788e-15f;   // 2^-48
static_assert(kDown * kUp * kUp == 1.f, "powers of two");
template <typename Op> constexpr float unscale() { return 1.f; }
template <> constexpr float unscale<Parts>() { return kDown; }
// pairs of parts that are multiplied, the small products first (what is left out is below 2^-25 of the product)
constexpr int kPa[6] = {2, 0, 1, 1, 0, 0}, kPb[6] = {0, 2, 1, 0, 1, 0};
// Largest log-sum-exp of a query by parts.  A probability is rebuilt by subtracting it from a score, whose bits must be those that
// went into it: scores of 800 by parts and by the fp32 instruction leave probabilities up to 1.8e-4 apart, scores of 2^20 nothing.
// Beyond it every workgroup that meets the query uses the instruction, in the forward and the backward call.
constexpr float kMostLse = 1024.f;
__device__ __forceinline__ bool beyond_parts(float lse) { return !(fabsf(lse) <= kMostLse); }
// Largest Q and K by parts: 64 products of 2^72 are below 2^80, where a sum of 2^48 times the size ends.  A score of minus infinity in
// place of a finite one would show in no result: its probability is zero.
constexpr float kMostScoreOperand = 68719476736.f;   // 2^36
template <int N>
__device__ __forceinline__ void largest(float& most, const float (&x)[N]) {
#pragma unroll
    for (int i = 0; i < N; ++i) most = fmaxf(most, fabsf(x[i]));
}

constexpr float kScale = 0.125f;   // 1/sqrt(64)
constexpr float kLog2e = 1.4426950408889634f;
constexpr int kRows = 32;          // rows of a tile, queries or keys of a wavefront
constexpr int kWaves = 4;

__device__ __forceinline__ f32x16 zero16() {
    f32x16 z;
#pragma unroll
    for (int e = 0; e < 16; ++e) z[e] = 0.f;
    return z;
}

// A streamed tile in LDS: 32 rows of 64 channels, read both row-wise (128-bit) and with the row index as k.
//   bf16: row r of a group of eight sits at position (0, 2, 4, 6, 1, 3, 5, 7)[r % 8], rows 176 bytes apart, which keeps
//         the row-wise and the transposing reads free of bank conflicts; fp32: rows 272 bytes apart.
template <typename T> struct Tile;
template <> struct Tile<bf16> {
    static constexpr int kStride = 88, kPieces = 8, kStage = 2;   // kStage: tiles per stage
    static __device__ __forceinline__ int at(int r) { return ((r & ~7) | ((r & 3) << 1) | ((r >> 2) & 1)) * kStride; }
};
template <> struct Tile<float> {
    static constexpr int kStride = 68, kPieces = 16, kStage = 1;
    static __device__ __forceinline__ int at(int r) { return r * kStride; }
};
template <> struct Tile<Parts> {   // each part like a bf16 tile, one after the other
    static constexpr int kStride = 88, kPieces = 16, kStage = 1;
    static __device__ __forceinline__ int at(int r) { return Tile<bf16>::at(r); }
};
constexpr int kPartElems = kRows * Tile<Parts>::kStride;
template <typename T> constexpr int tile_elems() { return kRows * Tile<T>::kStride; }
template <> constexpr int tile_elems<Parts>() { return 3 * kPartElems; }

// N floats times kUp as three bf16 parts each
template <int N>
__device__ __forceinline__ void cut_up(const float (&in)[N], uint32_t (&part)[3][N / 2]) {
    float x[N];
#pragma unroll
    for (int i = 0; i < N; ++i) x[i] = in[i] * kUp;
#pragma unroll
    for (int k = 0; k < 3; ++k)
#pragma unroll
        for (int i = 0; i < N / 2; ++i) {
            asm("v_cvt_pk_bf16_f32 %0, %1, %2" : "=v"(part[k][i]) : "v"(x[2 * i]), "v"(x[2 * i + 1]));   // written as conversions, half of them are made twice
            if (k < 2) {
                x[2 * i] -= __uint_as_float(part[k][i] << 16);
                x[2 * i + 1] -= __uint_as_float(part[k][i] & 0xffff0000u);
            }
        }
}

// 32 rows x 64 channels as the B operand of row-wise products: this lane's row in registers
template <typename T> struct RowOp;
template <> struct RowOp<bf16> {
    bf16x8 f[4];   // channels 16 kk + 8h .. + 7
    __device__ __forceinline__ void load(const bf16* row, bool ok, int h) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            u32x4 v = {0u, 0u, 0u, 0u};
            if (ok) v = *reinterpret_cast<const u32x4*>(row + kk * 16 + 8 * h);
            f[kk] = __builtin_bit_cast(bf16x8, v);
        }
    }
    // sum over this lane's channels of its own row times another
    static __device__ __forceinline__ float dot(const RowOp& a, const RowOp& b) {
        float s = 0.f;
#pragma unroll
        for (int kk = 0; kk < 4; ++kk)
#pragma unroll
            for (int i = 0; i < 8; ++i) s = fmaf(static_cast<float>(a.f[kk][i]), static_cast<float>(b.f[kk][i]), s);
        return s;
    }
};
template <> struct RowOp<float> {
    f32x4 f[8];    // channels 8 i + 4h .. + 3
    __device__ __forceinline__ void load(const float* row, bool ok, int h) {
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            f[i] = f32x4{0.f, 0.f, 0.f, 0.f};
            if (ok) f[i] = *reinterpret_cast<const f32x4*>(row + 8 * i + 4 * h);
        }
    }
    static __device__ __forceinline__ float dot(const RowOp& a, const RowOp& b) {   // short chains: few roundings
        float s[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            s[i] = a.f[i][0] * b.f[i][0];
#pragma unroll
            for (int j = 1; j < 4; ++j) s[i] = fmaf(a.f[i][j], b.f[i][j], s[i]);
        }
        return ((s[0] + s[1]) + (s[2] + s[3])) + ((s[4] + s[5]) + (s[6] + s[7]));
    }
};

template <> struct RowOp<Parts> {
    bf16x8 f[3][4];   // [part]: channels 16 kk + 8h .. + 7
    float most = 0.f;   // largest magnitude in this lane
    __device__ __forceinline__ void load(const float* row, bool ok, int h) {
#pragma unroll
        for (int kk = 0; kk < 4; ++kk) {
            float x[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
            if (ok) load8(row + kk * 16 + 8 * h, x);
            largest(most, x);
            uint32_t part[3][4];
            cut_up(x, part);
#pragma unroll
            for (int k = 0; k < 3; ++k) f[k][kk] = __builtin_bit_cast(bf16x8, u32x4{part[k][0], part[k][1], part[k][2], part[k][3]});
        }
        asm volatile("" : "+v"(most));   // formed here: at its use, behind the loops, it would keep the row in registers
    }
};

// acc[row of the tile][this wavefront's row] += tile . op^T; CHAINS: of sums along the channels, for fp32.  Two halve the
// roundings of the scores, which an exponential follows; for both products of the backward they would not fit the registers.
// SWAP: the tile holds the queries.  Products of parts are then added in the order in which the transposed product adds
// them, so that a score has the same bits wherever it is formed.
template <int CHAINS, bool SWAP = false>
__device__ __forceinline__ void mma_rows(f32x16& acc, const bf16* tile, const RowOp<bf16>& op, int lane) {
    const bf16* p = tile + Tile<bf16>::at(lane & 31) + 8 * (lane >> 5);
#pragma unroll
    for (int kk = 0; kk < 4; ++kk)
        acc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(*reinterpret_cast<const bf16x8*>(p + kk * 16), op.f[kk], acc, 0, 0, 0);
}
template <int CHAINS, bool SWAP = false>
__device__ __forceinline__ void mma_rows(f32x16& acc, const float* tile, const RowOp<float>& op, int lane) {
    const float* p = tile + Tile<float>::at(lane & 31) + 4 * (lane >> 5);
    f32x16 other = zero16();
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const f32x4 a = *reinterpret_cast<const f32x4*>(p + 8 * i);
        f32x16& to = CHAINS == 2 && (i & 1) ? other : acc;
#pragma unroll
        for (int j = 0; j < 4; ++j) to = __builtin_amdgcn_mfma_f32_32x32x2f32(a[j], op.f[i][j], to, 0, 0, 0);
    }
    if constexpr (CHAINS == 2) acc += other;
}

template <int CHAINS, bool SWAP = false>   // acc: zero
__device__ __forceinline__ void mma_rows(f32x16& acc, const bf16* tile, const RowOp<Parts>& op, int lane) {
    const bf16* p = tile + Tile<Parts>::at(lane & 31) + 8 * (lane >> 5);
    f32x16 low = zero16();   // the small products have an accumulator of their own
#pragma unroll
    for (int kk = 0; kk < 4; ++kk) {
        bf16x8 a[3];
#pragma unroll
        for (int k = 0; k < 3; ++k) a[k] = *reinterpret_cast<const bf16x8*>(p + k * kPartElems + kk * 16);
#pragma unroll
        for (int q = 0; q < 6; ++q) {
            f32x16& to = q == 5 ? acc : low;
            to = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[SWAP ? kPb[q] : kPa[q]], op.f[SWAP ? kPa[q] : kPb[q]][kk], to, 0, 0, 0);
        }
    }
    acc = (acc + low) * kDown;
}

// elements first .. first + 7 of p as PARTS bf16 parts, the largest first; the sum of three has every bit of p down to 2^-133
template <int PARTS>
__device__ __forceinline__ void cut8(const f32x16& p, int first, bf16x8 (&part)[PARTS]) {
    float x[8];
#pragma unroll
    for (int i = 0; i < 8; ++i) x[i] = p[first + i];
#pragma unroll
    for (int k = 0; k < PARTS; ++k) {
        u32x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            v[i] = pack_bf16x2(x[2 * i], x[2 * i + 1]);
            x[2 * i] -= __uint_as_float(v[i] << 16);
            x[2 * i + 1] -= __uint_as_float(v[i] & 0xffff0000u);
        }
        part[k] = __builtin_bit_cast(bf16x8, v);
    }
}

// out[channel][this wavefront's row] += tile^T . p, p a result of mma_rows (rows of the tile x the wavefront's rows)
template <typename Op, int PARTS>
__device__ __forceinline__ std::enable_if_t<std::is_same<Op, Parts>::value> mma_tr(f32x16 (&out)[2], const bf16* tile, const f32x16& p, int lane) {
    const int j = lane & 15;
    const bf16* base = tile + (2 * (j >> 2) + (lane >> 5)) * Tile<Parts>::kStride + 16 * ((lane >> 4) & 1) + 4 * (j & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
#pragma unroll
    for (int gp = 0; gp < 2; ++gp) {
        float x[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) x[i] = p[8 * gp + i];
        uint32_t part[3][4];
        cut_up(x, part);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            bf16x8 a[3];
#pragma unroll
            for (int k = 0; k < 3; ++k) {
                const bf16* q = base + k * kPartElems + 16 * gp * Tile<Parts>::kStride + 32 * dt;
                const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(q));
                const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(q + 8 * Tile<Parts>::kStride));
                s16x8 r;
                r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
                r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
                a[k] = __builtin_bit_cast(bf16x8, r);
            }
#pragma unroll
            for (int q = 0; q < 6; ++q) {
                const bf16x8 b = __builtin_bit_cast(bf16x8, u32x4{part[kPb[q]][0], part[kPb[q]][1], part[kPb[q]][2], part[kPb[q]][3]});
                out[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(a[kPa[q]], b, out[dt], 0, 0, 0);
            }
        }
    }
}
template <typename Op, int PARTS>
__device__ __forceinline__ std::enable_if_t<std::is_same<Op, bf16>::value> mma_tr(f32x16 (&out)[2], const bf16* tile, const f32x16& p, int lane) {
    const int j = lane & 15;
    // rows t0 + 4h + {0..3} and t0 + 8 + 4h + {0..3} of the tile: the order in which a lane holds 8 result elements
    const bf16* base = tile + (2 * (j >> 2) + (lane >> 5)) * Tile<bf16>::kStride + 16 * ((lane >> 4) & 1) + 4 * (j & 3);
    typedef s16x4 __attribute__((address_space(3))) * lds_ptr_t;
#pragma unroll
    for (int gp = 0; gp < 2; ++gp) {
        bf16x8 pf[PARTS];
        cut8(p, 8 * gp, pf);
#pragma unroll
        for (int dt = 0; dt < 2; ++dt) {
            const bf16* q = base + 16 * gp * Tile<bf16>::kStride + 32 * dt;
            const s16x4 lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(q));
            const s16x4 hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_ptr_t)(q + 8 * Tile<bf16>::kStride));
            s16x8 r;
            r[0] = lo[0]; r[1] = lo[1]; r[2] = lo[2]; r[3] = lo[3];
            r[4] = hi[0]; r[5] = hi[1]; r[6] = hi[2]; r[7] = hi[3];
#pragma unroll
            for (int k = PARTS - 1; k >= 0; --k)   // the small parts first
                out[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, r), pf[k], out[dt], 0, 0, 0);
        }
    }
}
template <typename Op, int>
__device__ __forceinline__ std::enable_if_t<std::is_same<Op, float>::value> mma_tr(f32x16 (&out)[2], const float* tile, const f32x16& p, int lane) {
    const float* base = tile + Tile<float>::at(4 * (lane >> 5)) + (lane & 31);
#pragma unroll
    for (int e = 0; e < 16; ++e)
#pragma unroll
        for (int dt = 0; dt < 2; ++dt)
            out[dt] = __builtin_amdgcn_mfma_f32_32x32x2f32(base[(8 * (e >> 2) + (e & 3)) * Tile<float>::kStride + 32 * dt], p[e], out[dt], 0, 0, 0);
}

// transposed result [64 channels][this lane's row] times mul -> the row in memory
__device__ __forceinline__ void store_row(const f32x16 (&t)[2], float mul, bf16* row, int h, bool ok) {
    // the two lanes of a row exchange halves, so that each stores 16-byte pieces
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int p = 0; p < 2; ++p) {
            uint32_t a[2], b[2];
#pragma unroll
            for (int r = 0; r < 2; ++r) {
                a[r] = pack_bf16x2(t[dt][8 * p + 2 * r] * mul, t[dt][8 * p + 2 * r + 1] * mul);
                b[r] = pack_bf16x2(t[dt][8 * p + 4 + 2 * r] * mul, t[dt][8 * p + 4 + 2 * r + 1] * mul);
                const auto sw = __builtin_amdgcn_permlane32_swap(a[r], b[r], false, false);
                a[r] = sw[0];
                b[r] = sw[1];
            }
            if (ok) *reinterpret_cast<uint4*>(row + dt * 32 + 8 * (2 * p + h)) = make_uint4(a[0], a[1], b[0], b[1]);
        }
}
__device__ __forceinline__ void store_row(const f32x16 (&t)[2], float mul, float* row, int h, bool ok) {
    if (!ok) return;
#pragma unroll
    for (int dt = 0; dt < 2; ++dt)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const f32x4 v = {t[dt][4 * g] * mul, t[dt][4 * g + 1] * mul, t[dt][4 * g + 2] * mul, t[dt][4 * g + 3] * mul};
            *reinterpret_cast<f32x4*>(row + dt * 32 + 8 * g + 4 * h) = v;
        }
}

// One operand of a stage: kStage tiles of 32 rows, this thread's 16-byte pieces on their way from memory to LDS.  The
// buffer's declared size ends with the last valid row, rows beyond it read as zeros; REPEAT: as the last valid row, so
// that a probability of zero times them is not finite only where that row's own product is not.
template <typename Op, bool REPEAT = false>
struct Stream {
    typedef typename Storage<Op>::type T;
    static constexpr int kPer = Tile<Op>::kStage * kRows * Tile<Op>::kPieces / (64 * kWaves);   // pieces per thread
    static constexpr int kStep = 64 * kWaves / Tile<Op>::kPieces;                              // rows between them
    __amdgpu_buffer_rsrc_t rsrc;
    uint32_t off, ld_bytes, last;
    u32x4 v[kPer];
    float most = 0.f;   // Parts: largest magnitude that this thread has stored
    __device__ __forceinline__ void init(const T* p, long ld, int tokens) {
        ld_bytes = (uint32_t)ld * (uint32_t)sizeof(T);
        rsrc = __builtin_amdgcn_make_buffer_rsrc(const_cast<T*>(p), 0, (uint32_t)(tokens - 1) * ld_bytes + 64u * (uint32_t)sizeof(T), 0x00020000);
        off = (uint32_t)(threadIdx.x / Tile<Op>::kPieces) * ld_bytes + (uint32_t)(threadIdx.x % Tile<Op>::kPieces) * 16u;
        last = (uint32_t)(tokens - 1) * ld_bytes + (uint32_t)(threadIdx.x % Tile<Op>::kPieces) * 16u;
    }
    __device__ __forceinline__ void fetch(int row0) {
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const uint32_t at = off + (uint32_t)(row0 + k * kStep) * ld_bytes;
            v[k] = __builtin_amdgcn_raw_buffer_load_b128(rsrc, REPEAT ? min(at, last) : at, 0, 0);
        }
    }
    __device__ __forceinline__ void store(typename InTile<Op>::type* lds) {   // lds: kStage tiles, one after the other
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int r = threadIdx.x / Tile<Op>::kPieces + k * kStep;
            if constexpr (std::is_same<Op, Parts>::value) {
                const float x[4] = {__uint_as_float(v[k][0]), __uint_as_float(v[k][1]), __uint_as_float(v[k][2]), __uint_as_float(v[k][3])};
                largest(most, x);   // dead code where nothing asks for it
                uint32_t part[3][2];
                cut_up(x, part);
                bf16* const to = lds + Tile<Op>::at(r) + (threadIdx.x % Tile<Op>::kPieces) * 4;
#pragma unroll
                for (int w = 0; w < 3; ++w) *reinterpret_cast<uint2*>(to + w * kPartElems) = make_uint2(part[w][0], part[w][1]);
            } else *reinterpret_cast<u32x4*>(lds + (r / kRows) * tile_elems<Op>() + Tile<Op>::at(r % kRows) + (threadIdx.x % Tile<Op>::kPieces) * (16 / (int)sizeof(T))) = v[k];
        }
    }
};

// Column sums of a workgroup's rows: t holds a row per lane (transposed result), ok = the row exists.  All wavefronts call
// it; lds: the operand buffers, red: a row of 64 per wavefront.  Through LDS and in a short loop: shuffles between the
// lanes take a third of the time once the instructions are cached, but in a pass of different kernels they are not, and
// fetching the unrolled exchange cost 11 us a launch.
__device__ __forceinline__ void store_colsum(const f32x16 (&t)[2], float mul, bool ok, float* lds, float (*red)[64], float* out) {
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6, c = lane & 31, h = lane >> 5;
    constexpr int kStride = 68;
    float* const mine = lds + wave * kRows * kStride;
    __syncthreads();   // the last stage has been read
#pragma unroll
    for (int i = 0; i < 8; ++i) {
        const int dt = i >> 2, g = 4 * (i & 3);
        const f32x4 v = {t[dt][g] * mul, t[dt][g + 1] * mul, t[dt][g + 2] * mul, t[dt][g + 3] * mul};
        *reinterpret_cast<f32x4*>(mine + c * kStride + 32 * dt + 2 * g + 4 * h) = ok ? v : f32x4{0.f, 0.f, 0.f, 0.f};
    }
    __syncthreads();
    float s = 0.f;
#pragma unroll 4
    for (int r = 0; r < kRows; ++r) s += mine[r * kStride + lane];
    red[wave][lane] = s;
    __syncthreads();
    if (wave == 0) out[lane] = red[0][lane] + red[1][lane] + red[2][lane] + red[3][lane];
}

// workgroup ids of one XCD (equal mod 8) become a contiguous range: the blocks of a pair share its rows through L2
__device__ __forceinline__ int xcd_order(int pid, int total) {
    const int xcd = pid & 7;
    return xcd * (total >> 3) + min(xcd, total & 7) + (pid >> 3);
}

// ---------------------------------------------------------------------------
// forward: workgroup = 128 queries of one (image, live head)
// ---------------------------------------------------------------------------
template <typename Op> constexpr int lds_bytes() { return 4 * Tile<Op>::kStage * tile_elems<Op>() * (int)sizeof(typename InTile<Op>::type); }

// true, for Parts: not in their range, and nothing has been written
template <typename Op, typename T>
__device__ __forceinline__ bool fwd_body(const T* __restrict__ qkv, long ldq, T* __restrict__ o, long ldo, float* __restrict__ lse,
                                         int tokens, int n_live, int n_full, long rows_total, int blocks, unsigned char* smem) {
    typedef typename InTile<Op>::type E;
    constexpr int ST = Tile<Op>::kStage;
    E (&lds)[2][2][ST * tile_elems<Op>()] = *reinterpret_cast<E (*)[2][2][ST * tile_elems<Op>()]>(smem);   // [buffer][K, V]
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int id = xcd_order(blockIdx.x, gridDim.x);
    const int pair = id / blocks, b = pair / n_live, j = pair % n_live;
    const long row0 = (long)b * tokens;
    const T* Qb = qkv + row0 * ldq + j * 192;
    const int q0 = (id % blocks) * (kRows * kWaves) + wave * kRows, q = q0 + c;

    Stream<Op> sk, sv;
    sk.init(Qb + 64, ldq, tokens);
    sv.init(Qb + 128, ldq, tokens);
    sk.fetch(0);
    sv.fetch(0);
    RowOp<Op> qf;
    qf.load(Qb + (long)q * ldq, q < tokens, h);
    f32x16 ot[2] = {zero16(), zero16()};
    // of the raw scores; sum over this lane's keys only.  The maximum starts at a finite value: a query whose scores so far
    // are all minus infinity keeps a defined difference from it, and probabilities of zero.
    float m = -3.402823466e38f, sum = 0.f;
    const float cexp = kScale * kLog2e;
    const int stages = (tokens + ST * kRows - 1) / (ST * kRows);
    sk.store(lds[0][0]);
    sv.store(lds[0][1]);
    for (int s = 0; s < stages; ++s) {
        if (s + 1 < stages) {
            sk.fetch((s + 1) * ST * kRows);
            sv.fetch((s + 1) * ST * kRows);
        }
        __syncthreads();
        const E* Ks = lds[s & 1][0];
        const E* Vs = lds[s & 1][1];
        if (q0 < tokens) {   // uniform over the wavefront
            f32x16 p[ST];
#pragma unroll
            for (int u = 0; u < ST; ++u) {
                p[u] = zero16();
                mma_rows<2>(p[u], Ks + u * tile_elems<Op>(), qf, lane);
            }
            if (s + 1 == stages) {   // keys past the last token
#pragma unroll
                for (int u = 0; u < ST; ++u) {
                    const int lim = tokens - (s * ST + u) * kRows - 4 * h;
#pragma unroll
                    for (int e = 0; e < 16; ++e)
                        if (8 * (e >> 2) + (e & 3) >= lim) p[u][e] = -INFINITY;
                }
            }
            float mt = m;
#pragma unroll
            for (int u = 0; u < ST; ++u)
#pragma unroll
                for (int e = 0; e < 16; e += 2) mt = fmaxf(fmaxf(mt, p[u][e]), p[u][e + 1]);
            mt = fmaxf(mt, __shfl_xor(mt, 32, 64));
            if (__any(mt > m)) {   // a new maximum somewhere: rescale (by exactly 1 where there is none)
                const float alpha = __builtin_amdgcn_exp2f((m - mt) * cexp);
                m = mt;
                sum *= alpha;
#pragma unroll
                for (int dt = 0; dt < 2; ++dt)
#pragma unroll
                    for (int e = 0; e < 16; ++e) ot[dt][e] *= alpha;
            }
            // the difference first: folded into one multiply-add, the rounding of m * cexp would reach every probability
#pragma unroll
            for (int u = 0; u < ST; ++u) {
#pragma unroll
                for (int e = 0; e < 16; ++e) p[u][e] = __builtin_amdgcn_exp2f((p[u][e] - m) * cexp);
                f32x16 t = p[u];
#pragma unroll
                for (int w = 8; w > 0; w >>= 1)
#pragma unroll
                    for (int e = 0; e < w; ++e) t[e] += t[e + w];
                sum += t[0];
                mma_tr<Op, 3>(ot, Vs + u * tile_elems<Op>(), p[u], lane);
            }
        }
        if (s + 1 < stages) {   // the other buffer was last read before the barrier above
            sk.store(lds[(s + 1) & 1][0]);
            sv.store(lds[(s + 1) & 1][1]);
        }
    }
    sum += __shfl_xor(sum, 32, 64);   // the two lanes of a query hold different keys
    const float l = m * kScale + __logf(sum);
    if constexpr (std::is_same<Op, Parts>::value) {
        float odd = 0.f;   // stays 0, or becomes NaN
#pragma unroll
        for (int e = 0; e < 16; ++e) odd = fmaf(ot[0][e], 0.f, fmaf(ot[1][e], 0.f, odd));
        if (__syncthreads_or(sk.most > kMostScoreOperand || (q < tokens && (odd != 0.f || qf.most > kMostScoreOperand || beyond_parts(l))))) return true;
    }
    if (q0 >= tokens) return false;
    store_row(ot, unscale<Op>() / sum, o + (row0 + q) * ldo + j * 64, h, q < tokens);
    if (q < tokens && h == 0 && j < n_full) lse[(long)j * rows_total + row0 + q] = l;
    return false;
}

// Op: how the operands are multiplied.  fp32 by parts falls back on the fp32 instruction, which is also a kernel of its own for
// the calls that fp32_by_instruction names.
template <typename T, typename Op = T>
__global__ __launch_bounds__(64 * kWaves, (std::is_same<Op, Parts>::value ? 2 : 3)) void attn_fwd_stream_kernel(const T* __restrict__ qkv, long ldq,
                                                                         T* __restrict__ o, long ldo, float* __restrict__ lse,
                                                                         int tokens, int n_live, int n_full, long rows_total,
                                                                         int blocks) {
    if constexpr (std::is_same<Op, Parts>::value) {
        static_assert(lds_bytes<Parts>() >= lds_bytes<float>(), "");
        extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
        if (!fwd_body<Parts>(qkv, ldq, o, ldo, lse, tokens, n_live, n_full, rows_total, blocks, dyn)) return;
        __syncthreads();   // the last stage has been read
        fwd_body<float>(qkv, ldq, o, ldo, lse, tokens, n_live, n_full, rows_total, blocks, dyn);
    } else {
        __shared__ __attribute__((aligned(16))) unsigned char smem[lds_bytes<T>()];
        fwd_body<T>(qkv, ldq, o, ldo, lse, tokens, n_live, n_full, rows_total, blocks, smem);
    }
}


// ---------------------------------------------------------------------------
// backward for p_f heads: the first half of the workgroups 128 keys of one (image, head) each, the rest 128 queries
// ---------------------------------------------------------------------------
struct BwdShared {
    float consts[2][2][2 * kRows];   // [buffer]: lse (see prob) and delta of a stage's queries
    float red[kWaves][64];
};

// true, for Parts: not in their range, and nothing has been written
template <typename Op, int TR_PARTS, typename T>
__device__ __forceinline__ bool bwd_body(const T* __restrict__ qkv, long ldq, const T* __restrict__ o, long ldo,
                                         const float* __restrict__ lse, const T* __restrict__ d_o, long ld_do,
                                         T* __restrict__ dqkv, long ld_dqkv, float* __restrict__ bsum, int tokens, int n_full,
                                         long rows_total, int blocks, unsigned char* smem, BwdShared& sh) {
    typedef typename InTile<Op>::type E;
    constexpr int ST = Tile<Op>::kStage;
    E (&lds)[2][2][ST * tile_elems<Op>()] = *reinterpret_cast<E (*)[2][2][ST * tile_elems<Op>()]>(smem);
    auto& consts = sh.consts;
    auto& red = sh.red;
    static_assert(lds_bytes<Op>() >= kWaves * kRows * 68 * 4 && kWaves == 4, "store_colsum");
    constexpr bool kParts = std::is_same<Op, Parts>::value;
    constexpr float kBack = unscale<Op>();
    auto odd_of = [](const f32x16 (&t)[2]) {   // 0, or NaN
        float odd = 0.f;
#pragma unroll
        for (int e = 0; e < 16; ++e) odd = fmaf(t[0][e], 0.f, fmaf(t[1][e], 0.f, odd));
        return odd;
    };
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c = lane & 31, h = lane >> 5;
    const int half = gridDim.x >> 1;
    const bool keys = (int)blockIdx.x < half;
    const int id = xcd_order(keys ? blockIdx.x : blockIdx.x - half, half);
    const int pair = id / blocks, b = pair / n_full, j = pair % n_full;
    const long row0 = (long)b * tokens;
    const T* Qb = qkv + row0 * ldq + j * 192;
    const T* dOb = d_o + row0 * ld_do + j * 64;
    const T* Ob = o + row0 * ldo + j * 64;
    const float* lse_b = lse + (long)j * rows_total + row0;
    T* dQb = dqkv + row0 * ld_dqkv + j * 192;
    const int i0 = (id % blocks) * (kRows * kWaves) + wave * kRows, i = i0 + c;   // this wavefront's rows, this lane's row
    const bool ok = i < tokens;
    const int stages = (tokens + ST * kRows - 1) / (ST * kRows);
    // probability of raw score s under the log-sum-exp l of its query.  In one multiply-add, with l in units of log2(e),
    // where P is rounded to bf16; else the difference first, so that the roundings of the two products do not reach P.
    constexpr bool kExact = sizeof(T) == 4 || TR_PARTS == 3;
    constexpr float kLse = kExact ? 1.f : kLog2e;
    auto prob = [](float s, float l) {
        if constexpr (kExact) return __builtin_amdgcn_exp2f(fmaf(s, kScale, -l) * kLog2e);
        else return __builtin_amdgcn_exp2f(fmaf(s, kScale * kLog2e, -l));
    };

    if (keys) {
        RowOp<Op> kf, vf;
        kf.load(Qb + (long)i * ldq + 64, ok, h);
        vf.load(Qb + (long)i * ldq + 128, ok, h);
        f32x16 dk[2] = {zero16(), zero16()}, dv[2] = {zero16(), zero16()};
        Stream<Op, true> sq, sd, so;
        sq.init(Qb, ldq, tokens);
        sd.init(dOb, ld_do, tokens);
        so.init(Ob, ldo, tokens);
        float l = 0.f;
        bool beyond = false;   // of the queries whose log-sum-exp this thread fetches
        auto fetch = [&](int s) {
            sq.fetch(s * ST * kRows);
            sd.fetch(s * ST * kRows);
            so.fetch(s * ST * kRows);
            if (threadIdx.x < ST * kRows) {
                const int q = s * ST * kRows + threadIdx.x;
                l = q < tokens ? lse_b[q] * kLse : INFINITY;   // a query past the last token: P = 0
            }
        };
        auto store = [&](int s) {
            const int buf = s & 1;
            sq.store(lds[buf][0]);
            sd.store(lds[buf][1]);
            if (threadIdx.x < ST * kRows) consts[buf][0][threadIdx.x] = l;
            if (kParts && threadIdx.x < ST * kRows && s * ST * kRows + (int)threadIdx.x < tokens) beyond |= beyond_parts(l);
            // delta of the rows this thread holds a piece of: the lanes of a row are neighbours
#pragma unroll
            for (int k = 0; k < Stream<Op>::kPer; ++k) {
                float dl = 0.f;
                if constexpr (sizeof(T) == 2) {
#pragma unroll
                    for (int x = 0; x < 4; ++x) {
                        dl = fmaf(__uint_as_float(sd.v[k][x] << 16), __uint_as_float(so.v[k][x] << 16), dl);
                        dl = fmaf(__uint_as_float(sd.v[k][x] & 0xffff0000u), __uint_as_float(so.v[k][x] & 0xffff0000u), dl);
                    }
                } else {
#pragma unroll
                    for (int x = 0; x < 4; ++x) dl = fmaf(__uint_as_float(sd.v[k][x]), __uint_as_float(so.v[k][x]), dl);
                }
#pragma unroll
                for (int w = 1; w < Tile<Op>::kPieces; w <<= 1) dl += __shfl_xor(dl, w, 64);
                if (threadIdx.x % Tile<Op>::kPieces == 0) consts[buf][1][threadIdx.x / Tile<Op>::kPieces + k * Stream<Op>::kStep] = dl;
            }
        };
        fetch(0);
        store(0);
        for (int s = 0; s < stages; ++s) {
            if (s + 1 < stages) fetch(s + 1);
            __syncthreads();
            if (i0 < tokens) {
#pragma unroll
                for (int u = 0; u < ST; ++u) {
                    const E* Qs = lds[s & 1][0] + u * tile_elems<Op>();
                    const E* dOs = lds[s & 1][1] + u * tile_elems<Op>();
                    f32x16 p = zero16(), dp = zero16();   // element e: query 8*(e/4) + 4h + e%4 of the tile
                    mma_rows<2, true>(p, Qs, kf, lane);
                    mma_rows<1, true>(dp, dOs, vf, lane);
#pragma unroll
                    for (int g = 0; g < 4; ++g) {
                        const f32x4 lq = *reinterpret_cast<const f32x4*>(&consts[s & 1][0][u * kRows + 8 * g + 4 * h]);
                        const f32x4 dq = *reinterpret_cast<const f32x4*>(&consts[s & 1][1][u * kRows + 8 * g + 4 * h]);
#pragma unroll
                        for (int x = 0; x < 4; ++x) {
                            p[4 * g + x] = prob(p[4 * g + x], lq[x]);
                            dp[4 * g + x] = p[4 * g + x] * (dp[4 * g + x] - dq[x]);
                        }
                    }
                    mma_tr<Op, TR_PARTS>(dv, dOs, p, lane);
                    mma_tr<Op, TR_PARTS>(dk, Qs, dp, lane);
                }
            }
            if (s + 1 < stages) store(s + 1);
        }
        const float odd = odd_of(dk);
        if constexpr (kParts) {
            if (__syncthreads_or(beyond || sq.most > kMostScoreOperand || (ok && (odd != 0.f || odd_of(dv) != 0.f || kf.most > kMostScoreOperand)))) return true;
        }
        if (i0 < tokens) {
            store_row(dk, kScale * kBack, dQb + (long)i * ld_dqkv + 64, h, ok);
            store_row(dv, kBack, dQb + (long)i * ld_dqkv + 128, h, ok);
        }
        if (bsum) {
            float* const row = bsum + ((long)b * blocks + id % blocks) * n_full * 192 + j * 192;
            // softmax does not see a common shift of the keys: the columns of dK sum to zero, unless some are not finite
            if (!kParts && __syncthreads_or(ok && odd != 0.f)) store_colsum(dk, kScale, ok, reinterpret_cast<float*>(lds), red, row + 64);
            else if (threadIdx.x < 64) row[64 + threadIdx.x] = 0.f;
            store_colsum(dv, kBack, ok, reinterpret_cast<float*>(lds), red, row + 128);
        }
    } else {
        float delta;
        {
            RowOp<T> of, df;
            of.load(Ob + (long)i * ldo, ok, h);
            df.load(dOb + (long)i * ld_do, ok, h);
            delta = RowOp<T>::dot(df, of);
            delta += __shfl_xor(delta, 32, 64);
        }
        RowOp<Op> qf, df;
        qf.load(Qb + (long)i * ldq, ok, h);
        df.load(dOb + (long)i * ld_do, ok, h);
        const float lq = ok ? lse_b[i] * kLse : 0.f;
        f32x16 dq[2] = {zero16(), zero16()};
        Stream<Op> sk, sv;
        sk.init(Qb + 64, ldq, tokens);
        sv.init(Qb + 128, ldq, tokens);
        sk.fetch(0);
        sv.fetch(0);
        sk.store(lds[0][0]);
        sv.store(lds[0][1]);
        for (int s = 0; s < stages; ++s) {
            if (s + 1 < stages) {
                sk.fetch((s + 1) * ST * kRows);
                sv.fetch((s + 1) * ST * kRows);
            }
            __syncthreads();
            if (i0 < tokens) {
#pragma unroll
                for (int u = 0; u < ST; ++u) {
                    const E* Ks = lds[s & 1][0] + u * tile_elems<Op>();
                    const E* Vs = lds[s & 1][1] + u * tile_elems<Op>();
                    f32x16 p = zero16(), dp = zero16();   // element e: key 8*(e/4) + 4h + e%4 of the tile
                    mma_rows<2>(p, Ks, qf, lane);
                    mma_rows<1>(dp, Vs, df, lane);
                    if (s + 1 == stages) {   // keys past the last token: P = 0
                        const int lim = tokens - (s * ST + u) * kRows - 4 * h;
#pragma unroll
                        for (int e = 0; e < 16; ++e)
                            if (8 * (e >> 2) + (e & 3) >= lim) p[e] = -INFINITY;
                    }
#pragma unroll
                    for (int e = 0; e < 16; ++e) dp[e] = prob(p[e], lq) * (dp[e] - delta);
                    mma_tr<Op, TR_PARTS>(dq, Ks, dp, lane);
                }
            }
            if (s + 1 < stages) {
                sk.store(lds[(s + 1) & 1][0]);
                sv.store(lds[(s + 1) & 1][1]);
            }
        }
        if constexpr (kParts) {
            if (__syncthreads_or(sk.most > kMostScoreOperand || (ok && (odd_of(dq) != 0.f || qf.most > kMostScoreOperand || beyond_parts(lq))))) return true;
        }
        if (i0 < tokens) store_row(dq, kScale * kBack, dQb + (long)i * ld_dqkv, h, ok);
        if (bsum) store_colsum(dq, kScale * kBack, ok, reinterpret_cast<float*>(lds), red, bsum + ((long)b * blocks + id % blocks) * n_full * 192 + j * 192);
    }
    return false;
}

template <typename T, int TR_PARTS, typename Op = T>
__global__ __launch_bounds__(64 * kWaves, (std::is_same<Op, Parts>::value ? 1 : 2)) void attn_bwd_stream_kernel(const T* __restrict__ qkv, long ldq,
                                                                         const T* __restrict__ o, long ldo,
                                                                         const float* __restrict__ lse,
                                                                         const T* __restrict__ d_o, long ld_do,
                                                                         T* __restrict__ dqkv, long ld_dqkv,
                                                                         float* __restrict__ bsum, int tokens,
                                                                         int n_full, long rows_total, int blocks) {
    __shared__ __attribute__((aligned(16))) BwdShared sh;
    if constexpr (std::is_same<Op, Parts>::value) {
        extern __shared__ __attribute__((aligned(16))) unsigned char dyn[];
        if (!bwd_body<Parts, 1>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, tokens, n_full, rows_total, blocks, dyn, sh)) return;
        __syncthreads();   // the last stage has been read
        bwd_body<float, 1>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, tokens, n_full, rows_total, blocks, dyn, sh);
    } else {
        __shared__ __attribute__((aligned(16))) unsigned char smem[lds_bytes<T>()];
        bwd_body<T, TR_PARTS>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, tokens, n_full, rows_total, blocks, smem, sh);
    }
}


// The fp32 kernels' dynamic LDS is above the default limit: raised once per device.
hipError_t allow_lds(const void* kern, std::atomic<uint32_t>& set_on) {   // set_on: devices, one bit each
    int dev = 0;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess || (dev < 32 && (set_on.load() >> dev & 1))) return e;
    e = hipFuncSetAttribute(kern, hipFuncAttributeMaxDynamicSharedMemorySize, lds_bytes<Parts>());
    if (e == hipSuccess && dev < 32) set_on.fetch_or(1u << dev);
    return e;
}

}  // namespace

int attn_stream_blocks(int tokens) { return (tokens + kRows * kWaves - 1) / (kRows * kWaves); }

bool attn_stream_supported(int dtype, int tokens, long ldq, long ldo) {
    const long es = dtype == D2FT_F32 ? 4 : 2;
    return tokens >= 1 && mult8(ldq) && mult8(ldo) && (long)(tokens + 63) * (ldq > ldo ? ldq : ldo) * es < (1L << 31);   // 32-bit offsets
}

// bf16 backward of up to 224 tokens, against the kernel of kernels_attn_mfma.hip with one workgroup per pair, whose time for
// one pair is that of a round of the chip.  This one has two workgroups per pair and block of 128 tokens, so that two blocks of few
// pairs use the chip better.  This kernel first, us, at 32, 64, 96, 128 and 136 pairs:
//   129 tokens 12.0 and 11.9, 12.6 and 13.8, 14.3 and 14.0, 15.2 and 15.0, 21.2 and 15.1
//   160        12.6 and 12.6, 12.8 and 13.5, 14.8 and 14.9, 15.2 and 15.2, 21.0 and 15.3
//   192        12.7 and 13.6, 13.4 and 14.9, 15.6 and 15.7, 15.6 and 16.0, 21.4 and 15.7
//   224        13.4 and 15.2, 14.9 and 16.7, 17.4 and 17.2, 18.6 and 17.2, 25.9 and 17.4
// and at 4 pairs 10.4 and 11.1 to 13.0 and 13.6.  Of one block (up to 128 tokens) it is never the faster one by more than 0.3 us: 33
// tokens, 12 pairs 6.2 and 6.4, 520 pairs 16.9 and 12.1; 64 tokens, 12 pairs 6.4 and 6.3, 520 pairs 19.4 and 13.2; 128 tokens,
// 12 pairs 9.1 and 8.4, 136 pairs 12.7 and 11.6, 520 pairs 31.0 and 21.1.
bool attn_bwd_stream_faster(int tokens, int pairs) { return tokens > 128 && pairs <= 96; }

// fp32 attention by the fp32 instruction instead of three bf16 parts of each operand, the same in the forward and the backward call
// (kMostLse says why), so by the pairs of the backward.  The cutting is a fixed cost that 32 keys do not repay, and the backward by
// parts needs the registers of two wavefronts, so that beyond 128 pairs it takes a round of workgroups more; the forward gains at
// all sizes above.  Forward + backward, instruction against parts, us:
//   17 tokens: 52 pairs 15.6 and 16.8, 520 pairs 29 and 51; 32 tokens: 128 pairs 17.4 and 17.5, 144 pairs 18 and 24
//   33: 128 pairs 24.4 and 22.9, 144 pairs 30 and 32, 1040 pairs 107 and 128; 64: 128 pairs 25.2 and 23.7, 640 pairs 81 and 86
//   65: 144 pairs 40.8 and 40.1, 640 pairs 112 and 104, 780 pairs 136 and 136, 1040 pairs 166 and 172
//   96: 640 pairs 119 and 113, 780 pairs 146 and 147, 1040 pairs 178 and 188
//   97: 780 pairs 183 and 172, 1040 pairs 228 and 222, 2080 pairs 421 and 438; 128: 1040 pairs 244 and 242, 2080 pairs 447 and 470
//   197: 1040 pairs 675 and 621, 2080 pairs 1295 and 1205
static bool fp32_by_instruction(int tokens, int pairs) {
    return tokens <= (pairs > 1536 ? 128 : pairs > 768 ? 96 : pairs > 128 ? 64 : 32);
}
// The same of a forward call that no backward call follows, for want of p_f heads.  By parts it wins beyond 32 tokens except where
// its 512 workgroups a round need a round more than the 768 by the instruction, and few tokens make little of it: 33 tokens, 260
// pairs 12.4 us by the instruction and 10.8 by parts, 520 pairs 14.3 and 16.3, 640 pairs 14.8 and 16.8, 780 pairs 19.5 and 19.1; 64
// tokens, 520 pairs 16.4 and 18.4, 640 pairs 17.5 and 19.1; 65 tokens, 520 pairs 25.7 and 22.3.
static bool fp32_forward_by_instruction(int tokens, int pairs) { return tokens <= 32 || (tokens <= 64 && pairs > 512 && pairs <= 768); }

hipError_t launch_attn_fwd_stream(int dtype, const void* qkv, long ldq, void* o, long ldo, float* lse, int batch, int tokens,
                                  int n_live, int n_full, hipStream_t s) {
    if (n_live <= 0) return hipSuccess;
    const int blocks = attn_stream_blocks(tokens);
    const dim3 grid((unsigned)((long)batch * n_live * blocks)), block(64 * kWaves);
    const long rows = (long)batch * tokens;
    if (dtype == D2FT_F32 && (n_full ? fp32_by_instruction(tokens, batch * n_full) : fp32_forward_by_instruction(tokens, batch * n_live))) {
        launch_label("attn_fwd_stream_kernel<float>");
        hipLaunchKernelGGL((attn_fwd_stream_kernel<float>), grid, block, 0, s, (const float*)qkv, ldq, (float*)o, ldo, lse, tokens,
                           n_live, n_full, rows, blocks);
    } else if (dtype == D2FT_F32) {
        static std::atomic<uint32_t> set_on{0};
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(attn_fwd_stream_kernel<float, Parts>), set_on);
        if (e != hipSuccess) return e;
        launch_label("attn_fwd_stream_kernel<float, Parts>");
        hipLaunchKernelGGL((attn_fwd_stream_kernel<float, Parts>), grid, block, lds_bytes<Parts>(), s, (const float*)qkv, ldq, (float*)o, ldo, lse, tokens,
                           n_live, n_full, rows, blocks);
    } else
        hipLaunchKernelGGL((attn_fwd_stream_kernel<bf16>), grid, block, 0, s, (const bf16*)qkv, ldq, (bf16*)o, ldo, lse, tokens,
                           n_live, n_full, rows, blocks);
    return hipGetLastError();
}

template <typename T, int TR_PARTS, typename Op = T>
static hipError_t launch_bwd(const void* qkv, long ldq, const void* o, long ldo, const float* lse, const void* d_o, long ld_do,
                             void* dqkv, long ld_dqkv, float* bsum, int batch, int tokens, int n_full, hipStream_t s) {
    const int blocks = attn_stream_blocks(tokens);
    const dim3 grid((unsigned)(2L * batch * n_full * blocks)), block(64 * kWaves);
    auto kern = attn_bwd_stream_kernel<T, TR_PARTS, Op>;
    const T *q = (const T*)qkv, *op = (const T*)o, *dop = (const T*)d_o;
    T* dq = (T*)dqkv;
    const long rows = (long)batch * tokens;
    int lds = 0;
    if constexpr (std::is_same<Op, Parts>::value) {
        static std::atomic<uint32_t> set_on{0};
        const hipError_t e = allow_lds(reinterpret_cast<const void*>(kern), set_on);
        if (e != hipSuccess) return e;
        lds = lds_bytes<Parts>();
    }
    return launch_signalling(kern, grid, block, lds, s, q, ldq, op, ldo, lse, dop, ld_do, dq, ld_dqkv, bsum, tokens, n_full, rows, blocks);
}

hipError_t launch_attn_bwd_stream(int dtype, const void* qkv, long ldq, const void* o, long ldo, const float* lse,
                                  const void* d_o, long ld_do, void* dqkv, long ld_dqkv, float* bsum, int batch, int tokens,
                                  int n_full, hipStream_t s) {
    if (n_full <= 0) return hipSuccess;
    if (dtype == D2FT_F32) {
        const bool instruction = fp32_by_instruction(tokens, batch * n_full);
        launch_label(instruction ? "attn_bwd_stream_kernel<float, 1>" : "attn_bwd_stream_kernel<float, 1, Parts>");
        if (instruction)
            return launch_bwd<float, 1>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, batch, tokens, n_full, s);
        return launch_bwd<float, 1, Parts>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, batch, tokens, n_full, s);
    }
    if (tokens <= 224) return launch_bwd<bf16, 1>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, batch, tokens, n_full, s);
    return launch_bwd<bf16, 3>(qkv, ldq, o, ldo, lse, d_o, ld_do, dqkv, ld_dqkv, bsum, batch, tokens, n_full, s);
}

}  // namespace d2ft
