// Bi-level knapsack selection on the GPU: DPSearching (Alg. 2) for the p_f stage and the p_o
// stage of every knapsack, then the merge of KnapsackScheduling (Alg. 1).
//
// Items are processed one after another (the recurrence is sequential in i); the capacities w = 0..C of
// one item are spread over the threads.  Only two rows of the value table are kept, in fp64; what the
// backtracking phase needs - whether T[i][w] differs from T[i-1][w] - is recorded per cell.  Each cell is
// one fp64 add and one compare, in the order the algorithm writes them, so the table equals a sequential
// CPU evaluation bit for bit.
//
// What bounds it is the latency of two serial chains, n items forward and n items back.  Where the tables of a
// knapsack fit the LDS of a CU (the change flags then as one bit per cell), one workgroup runs both stages and
// the merge in it; otherwise one workgroup runs one stage with its tables in the workspace, where a step of either
// chain is a round trip to L2.  144 items, capacities 259 and 1, from a host call: 133 us for the two launches of the second
// form, 43 us for the first (52 with a barrier for every item); back to back with warm caches 99 and 41 us.
#include "d2ft_common.h"

namespace d2ft {


// LDS of a knapsack: per stage two rows of `padded` doubles, n scores, n * padded bits of change flags, n selections
static size_t lds_bytes(int n, long padded) {
    return 2 * (size_t)(2 * padded * 8 + (size_t)n * 8 + (size_t)n * (padded / 64) * 8 + ((size_t)n + 7) / 8 * 8);
}

constexpr int kItems = 4;   // items per barrier of the fill

// one workgroup per knapsack; the first S = blockDim.x / 2 threads run the p_f stage, the others the p_o stage
__global__ __launch_bounds__(1024) void knapsack_lds_kernel(KnapsackArgs a, uint8_t* __restrict__ ops, int padded) {
    extern __shared__ __attribute__((aligned(16))) unsigned char smem[];
    const int k = blockIdx.x, n = a.n_items, S = blockDim.x >> 1;
    const int stage = (int)threadIdx.x >= S ? 1 : 0, t = threadIdx.x - stage * S;
    const int c = stage == 0 ? a.cost_fwd[k] + a.cost_bwd[k] : a.cost_fwd[k];   // W_b or W_f of Alg. 1
    const int C = stage == 0 ? a.cap_full[k] : a.cap_fwd[k];
    const int words = padded / 64;
    double* prev = reinterpret_cast<double*>(smem) + (long)stage * 2 * padded;
    double* cur = prev + padded;
    double* score = reinterpret_cast<double*>(smem) + 4 * (long)padded + (long)stage * n;
    uint64_t* bits = reinterpret_cast<uint64_t*>(smem) + 4 * (long)padded + 2 * (long)n + (long)stage * n * words;
    uint8_t* sel_all = reinterpret_cast<uint8_t*>(reinterpret_cast<uint64_t*>(smem) + 4 * (long)padded + 2 * (long)n + 2 * (long)n * words);
    uint8_t* sel = sel_all + stage * ((n + 7) / 8 * 8);

    for (int w = t; w < padded; w += S) prev[w] = 0.0;
    for (int i = t; i < n; i += S) {
        score[i] = (stage == 0 ? a.score_full : a.score_fwd)[(long)k * n + i];
        sel[i] = 0;
    }
    __syncthreads();

    // phase 1: fill.  Both stages walk the same n items, each over its own capacities.  All items of a stage cost c, so
    // T[i + kItems][w] follows from T[i][w - j c], j = 0 .. kItems: a thread forms the cells of kItems items that its
    // own needs, from kItems + 1 reads that are in flight together, and there is one barrier for all of them.
    const int top = (C + 64) & ~63;   // capacities in whole wavefronts: a ballot collects the flags of 64
    for (int i = 0; i < n; i += kItems) {
        for (int w = t; w < top; w += S) {
            double x[kItems + 1];   // cells at w - j c
#pragma unroll
            for (int j = 0; j <= kItems; ++j) x[j] = w / c >= j ? prev[w - j * c] : 0.0;
#pragma unroll
            for (int u = 0; u < kItems; ++u) {
                if (i + u >= n) break;   // uniform
                const double s = score[i + u], keep = x[0];
#pragma unroll
                for (int j = 0; j < kItems - u; ++j) {
                    const double take = __dadd_rn(x[j + 1], s);
                    x[j] = w / c > j && take > x[j] ? take : x[j];
                }
                const uint64_t changed = __ballot(x[0] != keep);
                if ((t & 63) == 0) bits[(long)(i + u) * words + (w >> 6)] = changed;
            }
            cur[w] = x[0];
        }
        __syncthreads();
        double* x = prev;
        prev = cur;
        cur = x;
    }

    // phase 2: backtracking
    if (t == 0) {
        int i = n, w = C;
        while (i > 0 && w > 0) {
            if ((bits[(long)(i - 1) * words + (w >> 6)] >> (w & 63)) & 1) {
                sel[i - 1] = 1;
                w -= c;
            }
            i -= 1;
        }
    }
    __syncthreads();

    // merge of Alg. 1: both or only p_f -> 1, only p_o -> 2, neither -> 3
    for (int i = threadIdx.x; i < n; i += blockDim.x)
        ops[(long)k * n + i] = sel_all[i] ? D2FT_OP_FULL : (sel_all[(n + 7) / 8 * 8 + i] ? D2FT_OP_FWD : D2FT_OP_SKIP);
}

__global__ __launch_bounds__(256) void knapsack_dp_kernel(KnapsackArgs a) {
    const int prob = blockIdx.x;           // knapsack * 2 + stage
    const int k = prob >> 1, stage = prob & 1;
    const int n = a.n_items;
    const int c = stage == 0 ? a.cost_fwd[k] + a.cost_bwd[k] : a.cost_fwd[k];   // W_b or W_f of Alg. 1
    const int C = stage == 0 ? a.cap_full[k] : a.cap_fwd[k];
    const double* score = (stage == 0 ? a.score_full : a.score_fwd) + (long)k * n;
    double* prev = a.rows + (long)prob * 2 * a.stride;
    double* cur = prev + a.stride;
    uint8_t* changed = a.changed + (long)prob * n * a.stride;
    uint8_t* sel = a.selected + (long)prob * n;

    for (int w = threadIdx.x; w <= C; w += blockDim.x) prev[w] = 0.0;
    for (int i = threadIdx.x; i < n; i += blockDim.x) sel[i] = 0;
    __syncthreads();

    // phase 1: fill
    for (int i = 1; i <= n; ++i) {
        const double s = score[i - 1];
        uint8_t* ch = changed + (long)(i - 1) * a.stride;
        for (int w = threadIdx.x; w <= C; w += blockDim.x) {
            const double keep = prev[w];
            double v = keep;
            if (w >= c) {
                const double take = __dadd_rn(prev[w - c], s);
                v = take > keep ? take : keep;
            }
            cur[w] = v;
            ch[w] = (v != keep) ? 1 : 0;
        }
        __syncthreads();
        double* t = prev;
        prev = cur;
        cur = t;
    }

    // phase 2: backtracking
    if (threadIdx.x == 0) {
        int i = n, w = C;
        while (i > 0 && w > 0) {
            if (changed[(long)(i - 1) * a.stride + w]) {
                sel[i - 1] = 1;
                w -= c;
            }
            i -= 1;
        }
    }
}

// merge of Alg. 1: both or only p_f -> 1, only p_o -> 2, neither -> 3
__global__ void knapsack_merge_kernel(const uint8_t* __restrict__ selected, uint8_t* __restrict__ ops, int n_knapsacks,
                                      int n_items) {
    const long idx = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (idx >= (long)n_knapsacks * n_items) return;
    const int k = (int)(idx / n_items), i = (int)(idx % n_items);
    const uint8_t pf = selected[((long)k * 2 + 0) * n_items + i];
    const uint8_t po = selected[((long)k * 2 + 1) * n_items + i];
    ops[idx] = pf ? D2FT_OP_FULL : (po ? D2FT_OP_FWD : D2FT_OP_SKIP);
}

constexpr size_t kLds = 160 * 1024;
bool knapsack_on_chip(int n_items, long cmax) {
    const long padded = (cmax + 64) / 64 * 64;
    return padded <= (long)kLds / 32 && n_items <= (int)kLds / 16 && lds_bytes(n_items, padded) <= kLds;
}

// cmax: the largest capacity.  The LDS form, wherever the tables fit, also with many knapsacks, of which only as many run at
// once as there are CUs with room for their tables: 12 items, 1 / 4096 knapsacks 5.4 / 11.0 us against 8.9 / 36.9 us for the
// other form; 144 items, 1 / 256 / 4096 knapsacks 41 / 45 / 389 us against 99 / 120 / 947; 384 items (one table per CU),
// 256 / 1024 knapsacks 156 / 601 us against 480 / 1255.
hipError_t launch_knapsack(const KnapsackArgs& a, long cmax, uint8_t* ops_dev, hipStream_t s) {
    if (knapsack_on_chip(a.n_items, cmax)) {
        const long padded = (cmax + 64) / 64 * 64;
        const hipError_t e = hipFuncSetAttribute(reinterpret_cast<const void*>(knapsack_lds_kernel), hipFuncAttributeMaxDynamicSharedMemorySize, (int)kLds);
        if (e != hipSuccess) return e;
        const int per_stage = padded < 512 ? (int)padded : 512;
        hipLaunchKernelGGL(knapsack_lds_kernel, dim3(a.n_knapsacks), dim3(2 * per_stage), lds_bytes(a.n_items, padded), s, a, ops_dev, (int)padded);
        return hipGetLastError();
    }
    hipLaunchKernelGGL(knapsack_dp_kernel, dim3(a.n_knapsacks * 2), dim3(256), 0, s, a);
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return e;
    const long total = (long)a.n_knapsacks * a.n_items;
    hipLaunchKernelGGL(knapsack_merge_kernel, dim3((unsigned)((total + 255) / 256)), dim3(256), 0, s, a.selected,
                       ops_dev, a.n_knapsacks, a.n_items);
    return hipGetLastError();
}

}  // namespace d2ft
