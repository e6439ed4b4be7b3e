// Device side of TailJobs (d2ft_common.h): one workgroup of the column reductions or of the zero fills, shared by the
// launch of its own (kernels_rowwise.hip) and the grouped weight-gradient launch it rides on (kernels_gemm_tile64.hip).
#pragma once

#include "d2ft_common.h"

namespace d2ft {

constexpr int kZeroBlocks = 16;                        // workgroups per head of the zero fills
constexpr int kTailLds = 32 * 8 * 4 * sizeof(float);   // bytes of LDS a workgroup needs

// rows x cols elements (cols a multiple of 8) with the given row stride, 16 or 32 bytes per thread
template <typename T>
__device__ __forceinline__ void zero_rect(void* base, long first, int rows, long cols, long stride, int tid, int nth) {
    if (!base) return;
    const uint32_t per = (uint32_t)(cols >> 3), n = (uint32_t)rows * per;
    const float z[8] = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
    for (uint32_t i = tid; i < n; i += nth) {
        const uint32_t r = rows == 1 ? 0 : i / per;
        store8(static_cast<T*>(base) + first + r * stride + (long)(i - r * per) * 8, z);
    }
}

// workgroup `blk` of t.blocks, threads tid < nth (at least 256); lds: kTailLds bytes
template <typename T>
__device__ __forceinline__ void tail_work(const TailJobs& t, int blk, int tid, int nth, void* lds) {
    if (blk >= t.red_blocks) {
        const int z = blk - t.red_blocks;
        const long h = t.zero.h[z / kZeroBlocks], H = t.H, D = t.D, r = t.r, S = t.slice;
        const int id = (z % kZeroBlocks) * nth + tid, n = kZeroBlocks * nth;
        for (int p = 0; p < 3; ++p) {
            zero_rect<T>(t.w_qkv, (p * H + h) * 64 * D, 1, 64 * D, 0, id, n);
            zero_rect<T>(t.b_qkv, (p * H + h) * 64, 1, 64, 0, id, n);
        }
        zero_rect<T>(t.w_o, h * 64, t.D, 64, H * 64, id, n);
        if (r > 0) {
            zero_rect<T>(t.la_q, h * r * D, 1, r * D, 0, id, n);
            zero_rect<T>(t.la_v, h * r * D, 1, r * D, 0, id, n);
            zero_rect<T>(t.lb_q, h * 64 * r, 1, 64 * r, 0, id, n);
            zero_rect<T>(t.lb_v, h * 64 * r, 1, 64 * r, 0, id, n);
        }
        if (S > 0) {
            zero_rect<T>(t.w1, h * S * D, 1, S * D, 0, id, n);
            zero_rect<T>(t.b1, h * S, 1, S, 0, id, n);
            zero_rect<T>(t.w2, h * S, t.D, S, t.Dm, id, n);
        }
        return;
    }
    // A workgroup owns 32 columns (8 threads x 4 columns) and spreads the chunks over 32 row lanes: lane l adds chunks
    // l, l + 32, ... in index order (eight loads in flight at a time), then the lanes' sums are added in four chains, which
    // round less than one of 32 (fp32, 65 chunks: relative error 8.1e-8 instead of 1.1e-7).
    int j = 0, b0 = 0;
    for (; j + 1 < t.red.n; ++j) {
        const int nb = (t.red.job[j].cols + 31) / 32;
        if (blk < b0 + nb) break;
        b0 += nb;
    }
    const ColReduceJob job = t.red.job[j];
    float4 (*red)[8] = static_cast<float4 (*)[8]>(lds);
    const int cg = tid & 7, rl = tid >> 3;
    const int c = (blk - b0) * 32 + cg * 4;
    float4 s = make_float4(0.f, 0.f, 0.f, 0.f);
    if (rl < 32) {
        if (c < job.cols) {
            const float* src = job.partial + c;
            int k = rl;
            for (; k + 7 * 32 < job.chunks; k += 8 * 32) {
                float4 v[8];
#pragma unroll
                for (int i = 0; i < 8; ++i) v[i] = *reinterpret_cast<const float4*>(src + (long)(k + 32 * i) * job.cols);
#pragma unroll
                for (int i = 0; i < 8; ++i) { s.x += v[i].x; s.y += v[i].y; s.z += v[i].z; s.w += v[i].w; }
            }
            for (; k < job.chunks; k += 32) {
                const float4 v = *reinterpret_cast<const float4*>(src + (long)k * job.cols);
                s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
            }
        }
        red[rl][cg] = s;
    }
    __syncthreads();
    if (rl != 0 || c >= job.cols) return;
    float4 a[3] = {red[1][cg], red[2][cg], red[3][cg]};
#pragma unroll 2
    for (int l = 4; l < 32; l += 4) {
        const float4 v = red[l][cg];
        s.x += v.x; s.y += v.y; s.z += v.z; s.w += v.w;
#pragma unroll
        for (int i = 0; i < 3; ++i) {
            const float4 w = red[l + 1 + i][cg];
            a[i].x += w.x; a[i].y += w.y; a[i].z += w.z; a[i].w += w.w;
        }
    }
    s.x = (s.x + a[0].x) + (a[1].x + a[2].x);
    s.y = (s.y + a[0].y) + (a[1].y + a[2].y);
    s.z = (s.z + a[0].z) + (a[1].z + a[2].z);
    s.w = (s.w + a[0].w) + (a[1].w + a[2].w);
    T* o = static_cast<T*>(job.out) + (job.remap_cols ? t.tbl[job.remap_cols - 1][c >> 6] * 64 + (c & 63) : c);
    if (t.accumulate) {
        s.x += ld<T>(o); s.y += ld<T>(o + 1); s.z += ld<T>(o + 2); s.w += ld<T>(o + 3);
    }
    st<T>(o, s.x); st<T>(o + 1, s.y); st<T>(o + 2, s.z); st<T>(o + 3, s.w);
}

}  // namespace d2ft
