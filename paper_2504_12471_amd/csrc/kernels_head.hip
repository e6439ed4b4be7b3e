// The two subnets outside the transformer blocks (Sec. IV-A, "Full fine-tuning partition settings"):
// the patch embedding at the start and the pooling + classification layer at the end.  The patch
// projection and its weight gradient run on the GEMM kernels; what is here is the bandwidth-bound
// data movement around them and the small per-image arithmetic of the classifier.
#include <type_traits>

#include "d2ft_common.h"

namespace d2ft {

namespace {

// ---------------------------------------------------------------------------
// images [B][C][H][W] -> patches [B * ny * nx][C * P * P], k = (c * P + i) * P + j; 8 pixels of one
// image row per thread (P is a multiple of 8)
// ---------------------------------------------------------------------------
template <typename T>
__global__ __launch_bounds__(256) void im2col_kernel(const T* __restrict__ img, T* __restrict__ patches, int B, int C,
                                                     int H, int W, int P) {
    const int nx = W / P, ny = H / P, K = C * P * P, k8 = K / 8;
    const long total = (long)B * ny * nx * k8;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int kc = (int)(i % k8);
        const long row = i / k8;                    // b * ny * nx + py * nx + px
        const int px = (int)(row % nx), py = (int)((row / nx) % ny), b = (int)(row / ((long)nx * ny));
        const int k = kc * 8, c = k / (P * P), ii = (k / P) % P, j = k % P;
        float v[8];
        load8(img + (((long)b * C + c) * H + py * P + ii) * W + px * P + j, v);
        store8(patches + row * K + k, v);
    }
}

// tokens[b][0] = cls + pos[0]; tokens[b][1 + p] = proj[b * Np + p] + pos[1 + p]
template <typename T>
__global__ __launch_bounds__(256) void assemble_tokens_kernel(const T* __restrict__ proj, const T* __restrict__ cls,
                                                              const T* __restrict__ pos, T* __restrict__ tokens, int B,
                                                              int Np, int D) {
    const int d8 = D / 8, Tn = Np + 1;
    const long total = (long)B * Tn * d8;
    for (long i = (long)blockIdx.x * 256 + threadIdx.x; i < total; i += (long)gridDim.x * 256) {
        const int dc = (int)(i % d8) * 8;
        const long row = i / d8;
        const int t = (int)(row % Tn), b = (int)(row / Tn);
        float a[8], p[8];
        if (t == 0) load8(cls + dc, a); else load8(proj + ((long)b * Np + t - 1) * D + dc, a);
        load8(pos + (long)t * D + dc, p);
#pragma unroll
        for (int j = 0; j < 8; ++j) a[j] += p[j];
        store8(tokens + row * D + dc, a);
    }
}

// backward of the assembly: dproj[b * Np + p] = dtokens[b][1 + p]; dpos[t] = sum_b dtokens[b][t]; dcls = dpos[0].
// A workgroup owns 256 / LANES pieces of 8 channels and has LANES lanes of images: lane l takes images l, l + LANES, ..., four in
// flight, and the lanes' sums are added in lane order.
template <typename T, int LANES>
__global__ __launch_bounds__(256) void embed_bwd_gather_kernel(const T* __restrict__ dtokens, T* __restrict__ dproj,
                                                               T* g_pos, T* g_cls, int B, int Np, int D, int accumulate) {
    constexpr int kPieces = 256 / LANES;
    __shared__ __attribute__((aligned(16))) float part[LANES][kPieces][8];   // one lane: not used
    const int d8 = D / 8, Tn = Np + 1;
    const int lane = threadIdx.x / kPieces, at = threadIdx.x % kPieces, i = blockIdx.x * kPieces + at;
    const bool on = i < Tn * d8;
    const int dc = (i % d8) * 8, t = i / d8;
    float s[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) s[j] = 0.f;
    if (on) {
        for (int b0 = lane; b0 < B; b0 += 4 * LANES) {
            float v[4][8];
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = b0 + q * LANES;
                if (b < B) load8(dtokens + ((long)b * Tn + t) * D + dc, v[q]);
            }
#pragma unroll
            for (int q = 0; q < 4; ++q) {
                const int b = b0 + q * LANES;
                if (b < B) {
                    if (t > 0) store8(dproj + ((long)b * Np + t - 1) * D + dc, v[q]);
#pragma unroll
                    for (int j = 0; j < 8; ++j) s[j] += v[q][j];
                }
            }
        }
    }
    if constexpr (LANES > 1) {
        store8(part[lane][at], s);
        __syncthreads();
        if (lane != 0) return;
#pragma unroll
        for (int l = 1; l < LANES; ++l) {
            float v[8];
            load8(part[l][at], v);
#pragma unroll
            for (int j = 0; j < 8; ++j) s[j] += v[j];
        }
    }
    if (!on) return;
    auto emit = [&](T* out) {
        float o[8];
#pragma unroll
        for (int j = 0; j < 8; ++j) o[j] = s[j];
        if (accumulate) {
            float old[8];
            load8(out, old);
#pragma unroll
            for (int j = 0; j < 8; ++j) o[j] += old[j];
        }
        store8(out, o);
    };
    if (g_pos) emit(g_pos + (long)t * D + dc);
    if (g_cls && t == 0) emit(g_cls + dc);
}

// ---------------------------------------------------------------------------
// classifier: LayerNorm of the class token, logits, softmax cross-entropy, and their gradients.  All arithmetic fp32.
//   xhat, h, dh: [B][D] fp32; logits, dl: [B][n] fp32; loss_b: [B]
// A few megabytes of work whose time is the latency of its loads, so each kernel has enough of them in flight: classes go
// to wavefronts by the eight, images of a parameter's gradient by the eight.  One workgroup per image (or class) that took
// its classes (or images) one after the other: 80 images, 384 channels, 100 classes 62 + 32 + 45 us; now 7.8 + 9.1 + 7.5.
// Pointers are only as aligned as their elements.
// ---------------------------------------------------------------------------
constexpr int kClasses = 8;            // of a wavefront, together in registers
constexpr int kHeadThreads = 1024, kHeadWaves = kHeadThreads / 64;   // of classifier_bwd_kernel
constexpr int kHeadCols = 512;         // channels it works on at a time, 8 per lane
constexpr int kZeroBytes = 32 * 1024;  // of dtokens that one of its workgroups clears

// grid (B, ceil(n / 32)): a wavefront normalises the class token by itself and forms the logits of 8 classes
template <typename T>
__global__ __launch_bounds__(256) void classifier_logits_kernel(const T* __restrict__ tokens, const T* __restrict__ ln_g,
                                                                const T* __restrict__ ln_b, const T* __restrict__ w_c,
                                                                const T* __restrict__ b_c, int Tn, int D, int n, float eps,
                                                                float* __restrict__ xhat, float* __restrict__ h,
                                                                float* __restrict__ rstd_out, float* __restrict__ logits) {
    const int b = blockIdx.x, lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int c0 = (blockIdx.y * 4 + wave) * kClasses;
    if (c0 >= n) return;
    const T* x = tokens + (long)b * Tn * D;
    float s = 0.f;
#pragma unroll 4
    for (int d = lane; d < D; d += 64) s += ld<T>(x + d);
    const float mean = wave_sum(s) / D;
    float q = 0.f;
#pragma unroll 4
    for (int d = lane; d < D; d += 64) {
        const float c = ld<T>(x + d) - mean;
        q += c * c;
    }
    const float rstd = rsqrtf(wave_sum(q) / D + eps);
    const T* w[kClasses];
#pragma unroll
    for (int i = 0; i < kClasses; ++i) w[i] = w_c + (long)min(c0 + i, n - 1) * D;
    float acc[kClasses];
#pragma unroll
    for (int i = 0; i < kClasses; ++i) acc[i] = 0.f;
#pragma unroll 2
    for (int d = lane; d < D; d += 64) {
        const float xh = (ld<T>(x + d) - mean) * rstd, hv = xh * ld<T>(ln_g + d) + ld<T>(ln_b + d);
#pragma unroll
        for (int i = 0; i < kClasses; ++i) acc[i] = fmaf(hv, ld<T>(w[i] + d), acc[i]);
        if (c0 == 0) {
            xhat[(long)b * D + d] = xh;
            h[(long)b * D + d] = hv;
        }
    }
    if (c0 == 0 && lane == 0) rstd_out[b] = rstd;
    float mine = 0.f;   // lane i: class c0 + i
#pragma unroll
    for (int i = 0; i < kClasses; ++i) {
        const float v = wave_sum(acc[i]);
        if (lane == i) mine = v;
    }
    if (lane < kClasses && c0 + lane < n) logits[(long)b * n + c0 + lane] = mine + ld<T>(b_c + c0 + lane);
}

template <typename F>
__device__ __forceinline__ float head_block(float v, float* red, F&& combine) {   // v: the wavefront's
    __syncthreads();
    if ((threadIdx.x & 63) == 0) red[threadIdx.x >> 6] = v;
    __syncthreads();
    v = red[0];
#pragma unroll
    for (int w = 1; w < kHeadWaves; ++w) v = combine(v, red[w]);
    return v;
}

// Softmax cross-entropy and its gradient with respect to the logits, dh = dl W_c, LayerNorm backward of the class-token row
// (blockIdx.y == 0); zeros in the image's other rows of dtokens (the other blockIdx.y, kZeroBytes each)
template <typename T>
__global__ __launch_bounds__(kHeadThreads) void classifier_bwd_kernel(const float* __restrict__ logits, const T* __restrict__ w_c,
                                                                      const T* __restrict__ ln_g,
                                                                      const int32_t* __restrict__ labels,
                                                                      const float* __restrict__ xhat,
                                                                      const float* __restrict__ rstd, int B, int Tn, int D, int n,
                                                                      float* dl, float* __restrict__ loss_b, float* dh,
                                                                      T* __restrict__ dtokens) {
    const int b = blockIdx.x, tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    T* out = dtokens + (long)b * Tn * D;
    if (blockIdx.y > 0) {
        constexpr int kItems = kZeroBytes / (int)sizeof(T);
        const long first = D + (long)(blockIdx.y - 1) * kItems, all = (long)Tn * D;   // rows of 16 bytes: D is a multiple of 8
        const long end = first + kItems < all ? first + kItems : all;
        if (((uintptr_t)dtokens & 15) == 0) {
            constexpr int kE = 16 / sizeof(T);
            for (long i = first + (long)tid * kE; i < end; i += (long)kHeadThreads * kE) *reinterpret_cast<uint4*>(out + i) = make_uint4(0, 0, 0, 0);
        } else {
            for (long i = first + tid; i < end; i += kHeadThreads) out[i] = static_cast<T>(0.0f);
        }
        return;
    }
    __shared__ float red[kHeadWaves];
    __shared__ float part[kHeadWaves][kHeadCols];
    auto add = [](float u, float v) { return u + v; };
    const float* z = logits + (long)b * n;
    float m = -INFINITY;
    for (int c = tid; c < n; c += kHeadThreads) m = fmaxf(m, z[c]);
    m = head_block(wave_max(m), red, [](float u, float v) { return fmaxf(u, v); });
    float e = 0.f;
    for (int c = tid; c < n; c += kHeadThreads) e += __expf(z[c] - m);
    const float lse = m + __logf(head_block(wave_sum(e), red, add));
    const int label = labels[b];
    dl += (long)b * n;
    for (int c = tid; c < n; c += kHeadThreads) dl[c] = (__expf(z[c] - lse) - (c == label ? 1.f : 0.f)) / B;
    if (tid == 0) loss_b[b] = lse - z[label];
    __syncthreads();
    // dh: wavefront w adds classes w, w + 16, ..., then the wavefronts' sums in order
    float m1 = 0.f, m2 = 0.f;
    for (int d0 = 0; d0 < D; d0 += kHeadCols) {
        float acc[kHeadCols / 64];
#pragma unroll
        for (int j = 0; j < kHeadCols / 64; ++j) acc[j] = 0.f;
#pragma unroll 4
        for (int c = wave; c < n; c += kHeadWaves) {
            const float v = dl[c];
            const T* w = w_c + (long)c * D + d0 + lane;
#pragma unroll
            for (int j = 0; j < kHeadCols / 64; ++j) acc[j] = fmaf(v, ld<T>(w + (d0 + lane + 64 * j < D ? 64 * j : -lane)), acc[j]);
        }
#pragma unroll
        for (int j = 0; j < kHeadCols / 64; ++j) part[wave][lane + 64 * j] = acc[j];
        __syncthreads();
        const int d = d0 + tid;
        if (tid < kHeadCols && d < D) {
            float v = part[0][tid];
#pragma unroll
            for (int w = 1; w < kHeadWaves; ++w) v += part[w][tid];
            dh[(long)b * D + d] = v;
            const float dg = v * ld<T>(ln_g + d);
            m1 += dg;
            m2 += dg * xhat[(long)b * D + d];
        }
        __syncthreads();
    }
    m1 = head_block(wave_sum(m1), red, add) / D;
    m2 = head_block(wave_sum(m2), red, add) / D;
    const float rs = rstd[b];
    for (int d = tid; d < D; d += kHeadCols) {   // the thread that wrote dh[d]
        if (tid >= kHeadCols) break;
        const float dg = dh[(long)b * D + d] * ld<T>(ln_g + d);
        st<T>(out + d, rs * (dg - m1 - xhat[(long)b * D + d] * m2));
    }
}

// parameter gradients and the mean loss: images added in index order, 256 of them staged at a time.  Grid (n + 1, ceil(D / 256)):
//   blockIdx.x < n: row c of dW_c and db_c[c]; the last workgroups: dln_g, dln_b and the loss
template <typename T>
__global__ __launch_bounds__(256) void classifier_param_grad_kernel(const float* __restrict__ dl, const float* __restrict__ h,
                                                                    const float* __restrict__ dh,
                                                                    const float* __restrict__ xhat,
                                                                    const float* __restrict__ loss_b, int B, int D, int n,
                                                                    T* g_w_c, T* g_b_c, T* g_ln_g, T* g_ln_b,
                                                                    float* __restrict__ loss, int accumulate) {
    __shared__ float staged[256];
    auto emit = [&](T* p, float v) {
        if (accumulate) v += ld<T>(p);
        st<T>(p, v);
    };
    const int c = blockIdx.x, d = blockIdx.y * 256 + threadIdx.x;
    const bool row = c < n, on = d < D, first = blockIdx.y == 0 && threadIdx.x == 0;
    const long dd = on ? d : 0;
    float a = 0.f, s = 0.f, t = 0.f;   // row: dW_c, -, db_c; last: dln_g, dln_b, loss
    for (int b0 = 0; b0 < B; b0 += 256) {
        const int nb = min(B - b0, 256);
        __syncthreads();
        if ((int)threadIdx.x < nb) staged[threadIdx.x] = row ? dl[(long)(b0 + threadIdx.x) * n + c] : loss_b[b0 + threadIdx.x];
        __syncthreads();
        if (row) {
            const float* hp = h + (long)b0 * D + dd;
#pragma unroll 8
            for (int b = 0; b < nb; ++b) a = fmaf(staged[b], hp[(long)b * D], a);
        } else {
            const float *dp = dh + (long)b0 * D + dd, *xp = xhat + (long)b0 * D + dd;
#pragma unroll 8
            for (int b = 0; b < nb; ++b) {
                const float v = dp[(long)b * D];
                a = fmaf(v, xp[(long)b * D], a);
                s += v;
            }
        }
        if (first)
            for (int b = 0; b < nb; ++b) t += staged[b];
    }
    if (row) {
        if (g_w_c && on) emit(g_w_c + (long)c * D + d, a);
        if (g_b_c && first) emit(g_b_c + c, t);
        return;
    }
    if (g_ln_g && on) emit(g_ln_g + d, a);
    if (g_ln_b && on) emit(g_ln_b + d, s);
    if (first) *loss = t / B;
}

#define D2FT_HEAD_DISPATCH(dtype, ...) \
    if ((dtype) == D2FT_F32) {         \
        typedef float T;               \
        __VA_ARGS__                    \
    } else {                           \
        typedef bf16 T;                \
        __VA_ARGS__                    \
    }

inline unsigned grid_for(long items) {
    long g = (items + 255) / 256;
    return (unsigned)(g < 1 ? 1 : (g > 8192 ? 8192 : g));
}

}  // namespace

hipError_t launch_im2col(int dtype, const void* img, void* patches, int B, int C, int H, int W, int P, hipStream_t s) {
    const long items = (long)B * (H / P) * (W / P) * (C * P * P / 8);
    D2FT_HEAD_DISPATCH(dtype, hipLaunchKernelGGL(im2col_kernel<T>, dim3(grid_for(items)), dim3(256), 0, s, (const T*)img,
                                                 (T*)patches, B, C, H, W, P);)
    return hipGetLastError();
}

hipError_t launch_assemble_tokens(int dtype, const void* proj, const void* cls, const void* pos, void* tokens, int B, int Np,
                                  int D, hipStream_t s) {
    const long items = (long)B * (Np + 1) * (D / 8);
    D2FT_HEAD_DISPATCH(dtype, hipLaunchKernelGGL(assemble_tokens_kernel<T>, dim3(grid_for(items)), dim3(256), 0, s,
                                                 (const T*)proj, (const T*)cls, (const T*)pos, (T*)tokens, B, Np, D);)
    return hipGetLastError();
}

hipError_t launch_embed_bwd_gather(int dtype, const void* dtokens, void* dproj, void* g_pos, void* g_cls, int B, int Np, int D,
                                   int accumulate, hipStream_t s) {
    const int items = (Np + 1) * (D / 8);
    auto launch = [&](auto lanes) {
        constexpr int kLanes = decltype(lanes)::value, kPieces = 256 / kLanes;
        D2FT_HEAD_DISPATCH(dtype, hipLaunchKernelGGL((embed_bwd_gather_kernel<T, kLanes>), dim3((items + kPieces - 1) / kPieces), dim3(256), 0,
                                                     s, (const T*)dtokens, (T*)dproj, (T*)g_pos, (T*)g_cls, B, Np, D, accumulate);)
    };
    // Lanes shorten the chain of loads of a piece, which is the time of many images (80 images of 197 x 384, 37 workgroups with one
    // lane, 26.3 -> 7.9 us), and cost workgroups where there is no chain.  bf16, one, two and eight lanes: 577 x 768, 4 images
    // 3.4, 3.2 and 3.9 us, 8 images 4.7, 4.1 and 5.0, 32 images 13.2, 10.9 and 10.0; 577 x 1024, 8 images 5.0, 5.0 and 5.8, 16 images
    // 8.4, 5.9 and 6.8; 4097 x 1024, 1 image 5.7, 6.1 and 12.1, 4 images 12.3, 12.9 and 16.0, 8 images 21.9, 22.6 and 21.9; below
    // 50000 pieces: 197 x 768, 4 images 2.9, 2.8 and 3.1, 8 images 3.8, 3.3 and 3.4, 96 images 30.9, 18.2 and 10.5.
    if (B <= 4) launch(std::integral_constant<int, 1>{});
    else if (B <= 16 && items >= 50000) launch(std::integral_constant<int, 2>{});
    else launch(std::integral_constant<int, 8>{});
    return hipGetLastError();
}

hipError_t launch_classifier(int dtype, const void* tokens, const void* ln_g, const void* ln_b, const void* w_c, const void* b_c,
                             const int32_t* labels, int B, int Tn, int D, int n, float eps, float* xhat, float* h, float* rstd,
                             float* logits, float* dl, float* loss_b, float* dh, void* dtokens, void* g_w_c, void* g_b_c,
                             void* g_ln_g, void* g_ln_b, float* loss, int accumulate, hipStream_t s) {
    const int es = dtype == D2FT_F32 ? 4 : 2;
    const unsigned zeros = (unsigned)(((long)(Tn - 1) * D * es + kZeroBytes - 1) / kZeroBytes);
    D2FT_HEAD_DISPATCH(dtype,
        hipLaunchKernelGGL(classifier_logits_kernel<T>, dim3(B, (n + 4 * kClasses - 1) / (4 * kClasses)), dim3(256), 0, s,
                           (const T*)tokens, (const T*)ln_g, (const T*)ln_b, (const T*)w_c, (const T*)b_c, Tn, D, n, eps, xhat, h,
                           rstd, logits);
        hipLaunchKernelGGL(classifier_bwd_kernel<T>, dim3(B, 1 + zeros), dim3(kHeadThreads), 0, s, logits, (const T*)w_c,
                           (const T*)ln_g, labels, xhat, rstd, B, Tn, D, n, dl, loss_b, dh, (T*)dtokens);
        hipLaunchKernelGGL(classifier_param_grad_kernel<T>, dim3(n + 1, (D + 255) / 256), dim3(256), 0, s, dl, h, dh, xhat, loss_b,
                           B, D, n, (T*)g_w_c, (T*)g_b_c, (T*)g_ln_g, (T*)g_ln_b, loss, accumulate);)
    return hipGetLastError();
}

}  // namespace d2ft
