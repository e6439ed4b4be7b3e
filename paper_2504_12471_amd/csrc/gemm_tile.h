// What the small-tile products (kernels_gemm_tile64.hip) and the split fp32 products (kernels_gemm_split.hip) share: the
// arguments of a grouped weight-gradient launch, the order in which workgroups take tiles, and what happens to results.
#pragma once

#include "gemm_map.h"
#include "launch.h"
#include "tail_jobs.h"

namespace d2ft {

// One weight gradient of a grouped launch: out[m'][n'] (=|+=) sum_k A[k][m] * B[k][n], (m', n') through the remap
struct Tile64Group {
    const void* A;
    const void* B;
    void* out;
    long lda, ldb, ldo;
    int M, N;
    int tiles_m, tile0;
    int remap, table;        // RED_REMAP_*
};
struct Tile64Grouped {
    Tile64Group grp[kMaxGemmGroups];
    float* partial;          // splits > 1: raw sums, slot (split * total_tiles + tile), 64 x 64 floats each
    int n, K, splits, slabs_per_split, total_tiles, units, accumulate;   // units: workgroups that multiply, then tail's
    TailJobs tail;
    uint16_t tbl[3][kMaxBlocks64];   // the remap tables in units of 64
};

// scalar offset of the loads of the slab at k0 (valid k < k_end), whose first k sits at k_at in memory.  The next slabs'
// loads run past the end of K; there it is 0 and the lanes' own offsets are kOutside.  An offset beyond the buffer's size
// must not be asked for: the bounds check compares the lane's offset with the size less the scalar one.
__host__ __device__ __forceinline__ uint32_t slab_offset(int k0, int k_at, int k_end, uint32_t sk_bytes) {
    return k0 < k_end ? (uint32_t)k_at * sk_bytes : 0u;
}

// What the epilogue reads for columns n .. n + 7 of row m, as it lies in memory: the bias, and Z or the residual
template <typename T>
struct EpilogueOperands {
    static constexpr int kN = 8 * sizeof(T) / 16;
    uint4 bias[kN], other[kN];
    static __device__ __forceinline__ void load(uint4 (&v)[kN], const void* p, long at) {
#pragma unroll
        for (int i = 0; i < kN; ++i) v[i] = reinterpret_cast<const uint4*>(static_cast<const T*>(p) + at)[i];
    }
    static __device__ __forceinline__ void values(const uint4 (&v)[kN], float (&o)[8]) {
        load8(reinterpret_cast<const T*>(v), o);
    }
    __device__ __forceinline__ void request(const GemmArgs& g, int m, int n) {
        if (g.bias) load(bias, g.bias, g.bias_remap ? g.tbl(n) : n);
        if (g.act == ACT_DGELU) load(other, g.Z, (long)m * g.ldz + n);
        else if (g.residual) load(other, g.residual, (long)m * g.ldr + n);
    }
};

// results of row m, columns n .. n + 7, through the epilogue; v returns what was stored
template <typename T>
__device__ __forceinline__ void emit(const GemmArgs& g, int m, int n, float (&v)[8], const EpilogueOperands<T>& with) {
    if (g.bias) {
        float b[8];
        with.values(with.bias, b);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += b[i];
    }
    if (g.act == ACT_GELU) {
        // Z <- GELU'(z), C <- GELU(z), both of the fp32 pre-activation
        float d[8];
#pragma unroll
        for (int i = 0; i < 8; ++i) {
            const float z = v[i], cdf = 0.5f * (1.0f + erff(z * 0.70710678118654752440f));   // one erff for both: it is long
            d[i] = fmaf(z, 0.39894228040143267794f * __expf(-0.5f * z * z), cdf);
            v[i] = z * cdf;
        }
        store8(static_cast<T*>(g.Z) + (long)m * g.ldz + n, d);
    } else if (g.act == ACT_DGELU) {
        float d[8];
        with.values(with.other, d);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] *= d[i];
    }
    if (g.residual) {
        float x[8];
        if (g.act == ACT_DGELU) load8(static_cast<const T*>(g.residual) + (long)m * g.ldr + n, x);
        else with.values(with.other, x);
#pragma unroll
        for (int i = 0; i < 8; ++i) v[i] += x[i];
    }
    store8(static_cast<T*>(g.C) + (long)m * g.ldc + n, v);
}
template <typename T>
__device__ __forceinline__ void emit(const GemmArgs& g, int m, int n, float (&v)[8]) {
    EpilogueOperands<T> with;
    with.request(g, m, n);
    emit<T>(g, m, n, v, with);
}

// the same of weight gradient gi of a grouped launch
template <typename T>
__device__ __forceinline__ void emit_grouped(const Tile64Grouped& g, int gi, int m, int n, float (&v)[8]) {
    const Tile64Group& G = g.grp[gi];
    if (G.remap == RED_REMAP_F32) {
        store8(static_cast<float*>(G.out) + (long)m * G.ldo + n, v);
    } else {
        const int mo = G.remap == RED_REMAP_ROWS ? g.tbl[G.table][m >> 6] * 64 + (m & 63) : m;
        const int no = G.remap == RED_REMAP_COLS ? g.tbl[G.table][n >> 6] * 64 + (n & 63) : n;
        T* o = static_cast<T*>(G.out) + (long)mo * G.ldo + no;
        if (g.accumulate) {
            float old[8];
            load8(o, old);
#pragma unroll
            for (int i = 0; i < 8; ++i) v[i] += old[i];
        }
        store8(o, v);
    }
}

// fp32 products by bf16 parts (kernels_gemm_split.hip), for what gemm_tile64_supported takes: microseconds, 1e30 if the
// form is not one of it
float gemm_split_us(const GemmArgs& g);
hipError_t launch_gemm_split(const GemmArgs& g, hipStream_t s);
// fills the tiles, splits and units of a for its groups; microseconds with the reduction
float gemm_split_grouped_plan(Tile64Grouped* a, size_t partial_floats);
hipError_t launch_gemm_split_grouped(const Tile64Grouped& a, hipStream_t s);

}  // namespace d2ft
