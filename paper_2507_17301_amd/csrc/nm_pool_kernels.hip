// The pooling layers between the convolutions of a ResNet: 3x3/2 max pooling
// after the first layer and global average pooling before the classifier.
// Both are plain HBM-bound passes over NHWC tensors: one thread handles 4
// consecutive channels (8 or 16 bytes) of one output position, so that a
// wavefront reads and writes contiguous runs.
#include "nm_conv_kernel.h"

namespace nm {
namespace {

inline int grid_for_items(size_t items)
{
    size_t g = (items + 255) / 256;
    if (g > 256 * 16) g = 256 * 16;
    return g < 1 ? 1 : (int)g;
}

template <typename T>
__global__ __launch_bounds__(256) void maxpool_kernel(const T* __restrict__ x, T* __restrict__ y, int B,
                                                      int H, int W, int C, int k, int stride, int pad,
                                                      int Ho, int Wo)
{
    const int C4 = (C + 3) / 4;
    const size_t total = (size_t)B * Ho * Wo * C4;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const int c4 = (int)(i % C4);
        size_t r = i / C4;
        const int wo = (int)(r % Wo); r /= Wo;
        const int ho = (int)(r % Ho);
        const int b = (int)(r / Ho);
        const int c0 = c4 * 4;
        const bool vec = (C % 4 == 0);
        f4 m = {-INFINITY, -INFINITY, -INFINITY, -INFINITY};
        for (int kh = 0; kh < k; ++kh) {
            const int hi = ho * stride - pad + kh;
            if ((unsigned)hi >= (unsigned)H) continue;
            for (int kw = 0; kw < k; ++kw) {
                const int wi = wo * stride - pad + kw;
                if ((unsigned)wi >= (unsigned)W) continue;
                const T* px = x + ((size_t)(b * H + hi) * W + wi) * C + c0;
                if (vec) {
                    const f4 v = load4(px);
                    m.x = fmaxf(m.x, v.x); m.y = fmaxf(m.y, v.y);
                    m.z = fmaxf(m.z, v.z); m.w = fmaxf(m.w, v.w);
                } else {
                    for (int e = 0; e < 4 && c0 + e < C; ++e) m[e] = fmaxf(m[e], load1(px + e));
                }
            }
        }
        T* py = y + ((size_t)(b * Ho + ho) * Wo + wo) * C + c0;
        if (vec) {
            store4(py, m);
        } else {
            for (int e = 0; e < 4 && c0 + e < C; ++e) store1(py + e, m[e]);
        }
    }
}

// Max pooling where pixels are whole 16-byte granules: one thread per output granule, KT x KT loads in
// flight (KT = 0: any window, one row of it at a time), no division but one of 32 bits by the granules
// of a pixel.  Bound by memory; with 8-byte loads and four 64-bit divisions per output the 3x3/2 pass of
// ResNet-50 (batch 64, 112x112x64, 128 MB in bf16) took 44 us in bf16 and takes 29.
template <typename T, int KT>
__global__ __launch_bounds__(256) void maxpool_vec_kernel(const T* __restrict__ x, T* __restrict__ y, int H, int W, int C,
                                                          int k_, int stride, int pad, int Ho, int Wo, int rows,
                                                          int blocks_per_row, int per_xcd)
{
    constexpr int V = 16 / (int)sizeof(T);
    const int k = KT ? KT : k_;
    // neighbouring output rows share input rows: each XCD gets a contiguous range of them
    const int bid = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    const int row = bid / blocks_per_row;                 // b * Ho + ho
    if (row >= rows) return;
    const unsigned CV = (unsigned)C / V;
    const unsigned i = (unsigned)(bid - row * blocks_per_row) * 256u + threadIdx.x;
    const unsigned wo = i / CV, cv = i - wo * CV;
    if (wo >= (unsigned)Wo) return;
    const int b = row / Ho, h0 = (row - b * Ho) * stride - pad, w0 = (int)wo * stride - pad;
    const T* const img = x + (size_t)b * H * W * C + cv * V;
    float m[V];
#pragma unroll
    for (int e = 0; e < V; ++e) m[e] = -INFINITY;
    auto take = [&](const u4v v, bool in) {
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            if constexpr (V == 4) {
                m[g] = fmaxf(m[g], in ? __uint_as_float(v[g]) : -INFINITY);
            } else {
                m[2 * g] = fmaxf(m[2 * g], in ? __uint_as_float(v[g] << 16) : -INFINITY);
                m[2 * g + 1] = fmaxf(m[2 * g + 1], in ? __uint_as_float(v[g] & 0xffff0000u) : -INFINITY);
            }
        }
    };
    // (a tap outside the image loads a clamped pixel and is not taken)
    auto at = [&](int kh, int kw, bool* in) {
        const int hi = h0 + kh, wi = w0 + kw;
        *in = ((unsigned)hi < (unsigned)H) & ((unsigned)wi < (unsigned)W);
        return *reinterpret_cast<const u4v*>(img + ((size_t)(*in ? hi : 0) * W + (*in ? wi : 0)) * C);
    };
    if constexpr (KT > 0) {
        u4v v[KT * KT];
        bool in[KT * KT];
#pragma unroll
        for (int t = 0; t < KT * KT; ++t) v[t] = at(t / KT, t % KT, &in[t]);
#pragma unroll
        for (int t = 0; t < KT * KT; ++t) take(v[t], in[t]);
    } else {
        for (int kh = 0; kh < k; ++kh)
            for (int kw = 0; kw < k; ++kw) {
                bool in;
                const u4v v = at(kh, kw, &in);
                take(v, in);
            }
    }
    T* const py = y + ((size_t)row * Wo + wo) * C + cv * V;
    u4v o;
#pragma unroll
    for (int g = 0; g < 4; ++g) o[g] = V == 4 ? __float_as_uint(m[g]) : pack_bf16(m[g * V / 4], m[g * V / 4 + V / 4 - 1]);
    store_out16<false>(py, o);
}

// one workgroup per (image, 64-channel slab): 4 wavefronts split the positions,
// lanes run along the channels; fp32 partial sums meet in LDS
template <typename T>
__global__ __launch_bounds__(256) void avgpool_kernel(const T* __restrict__ x, T* __restrict__ y, int HW, int C)
{
    __shared__ float part[4][64];
    const int b = blockIdx.y;
    const int c = blockIdx.x * 64 + (threadIdx.x & 63);
    const int wv = threadIdx.x >> 6;
    float s = 0.f;
    if (c < C)
        for (int i = wv; i < HW; i += 4) s += load1(x + ((size_t)b * HW + i) * C + c);
    part[wv][threadIdx.x & 63] = s;
    __syncthreads();
    if (wv == 0 && c < C) {
        const float t = ((part[0][threadIdx.x] + part[1][threadIdx.x]) + part[2][threadIdx.x]) + part[3][threadIdx.x];
        store1(y + (size_t)b * C + c, t / (float)HW);
    }
}

// im2col written out: one thread per (pixel, run of V channels of one tap), V elements = 16 bytes
// when the channel count allows, else one element
template <typename T, int V>
__global__ __launch_bounds__(256) void im2col_kernel(const T* __restrict__ x, T* __restrict__ a, int B, int H,
                                                     int W, int C, int Kh, int Kw, int sh, int sw, int ph, int pw,
                                                     int dh, int dw, int Ho, int Wo)
{
    const int CV = C / V;
    const size_t total = (size_t)B * Ho * Wo * Kh * Kw * CV;
    for (size_t i = (size_t)blockIdx.x * blockDim.x + threadIdx.x; i < total;
         i += (size_t)gridDim.x * blockDim.x) {
        const int cv = (int)(i % CV);
        size_t r = i / CV;
        const int kw_ = (int)(r % Kw); r /= Kw;
        const int kh_ = (int)(r % Kh); r /= Kh;
        const int wo = (int)(r % Wo); r /= Wo;
        const int ho = (int)(r % Ho);
        const int b = (int)(r / Ho);
        const int hi = ho * sh - ph + kh_ * dh, wi = wo * sw - pw + kw_ * dw;
        const bool in = ((unsigned)hi < (unsigned)H) & ((unsigned)wi < (unsigned)W);
        T* dst = a + i * V;     // (pixel, tap, channel run) is exactly the order of a[p][k]
        if constexpr (V == 1) {
            T z; if constexpr (sizeof(T) == 4) z = 0; else z.v = 0;
            dst[0] = in ? x[((size_t)(b * H + hi) * W + wi) * C + cv] : z;
        } else {
            u4v v = {0u, 0u, 0u, 0u};
            if (in) v = *reinterpret_cast<const u4v*>(x + ((size_t)(b * H + hi) * W + wi) * C + cv * V);
            *reinterpret_cast<u4v*>(dst) = v;
        }
    }
}

// The traffic of a layer and nothing else: read nx 16-byte units, write ny, both spread over
// every thread of the grid in grid-stride order (whole 1 KB runs per wavefront), four loads in
// flight per thread before the first use.  What is read only steers a store that never happens.
__global__ __launch_bounds__(256) void stream_floor_kernel(const u4v* __restrict__ x, size_t nx,
                                                           u4v* __restrict__ y, size_t ny)
{
    const size_t step = (size_t)gridDim.x * blockDim.x;
    const size_t i0 = (size_t)blockIdx.x * blockDim.x + threadIdx.x;
    unsigned acc = 0;
    size_t i = i0;
    for (; i + 3 * step < nx; i += 4 * step) {
        const u4v a = x[i], b = x[i + step], c = x[i + 2 * step], d = x[i + 3 * step];
        acc += (a.x ^ b.y) + (c.z ^ d.w);
    }
    for (; i < nx; i += step) acc += x[i].x;
    const u4v v = {1u, 2u, 3u, 4u};
    for (size_t j = i0; j < ny; j += step) y[j] = v;
    if (acc == 0x9e3779b9u && ny > 0 && i0 == 0) y[0].x = acc;   // keeps the loads alive
}

// Where the partial sums of a K split meet: one thread per 4 consecutive channels of one
// pixel (or per element when Cout is not a multiple of 4) adds the splits in ascending order,
// then bias, residual, activation, one rounding.
// S splits are all requested before the first is added.
template <typename TOUT, int S>
__global__ __launch_bounds__(256) void splitk_reduce_kernel(const ConvParams p)
{
    const unsigned total = (unsigned)p.P * (unsigned)p.Cout;   // below 2^31
    TOUT* __restrict__ y = reinterpret_cast<TOUT*>(p.y);
    const float* __restrict__ part = p.partial;
    if (p.Cout % 4 == 0) {
        for (unsigned i = (blockIdx.x * blockDim.x + threadIdx.x) * 4; i < total; i += gridDim.x * blockDim.x * 4) {
            f4 v[S];
#pragma unroll
            for (int s = 0; s < S; ++s) v[s] = *reinterpret_cast<const f4*>(part + (size_t)s * total + i);
            f4 t = v[0];
#pragma unroll
            for (int s = 1; s < S; ++s) t = t + v[s];
            if (p.bias) t = t + *reinterpret_cast<const f4*>(p.bias + i % (unsigned)p.Cout);
            emit4(p, y, i, t);
        }
    } else {
        for (unsigned i = blockIdx.x * blockDim.x + threadIdx.x; i < total; i += gridDim.x * blockDim.x) {
            float v = part[i];
            for (int s = 1; s < S; ++s) v += part[(size_t)s * total + i];
            if (p.bias) v += p.bias[i % (unsigned)p.Cout];
            emit1(p, y, i, v);
        }
    }
}

}  // namespace

int run_splitk_reduce(const ConvParams& p, nm_dtype_t ydt, hipStream_t s)
{
    const size_t total = (size_t)p.P * p.Cout;
    const size_t items = p.Cout % 4 == 0 ? total / 4 : total;
    const int grid = grid_for_items(items);
#define NM_REDUCE(T, S) hipLaunchKernelGGL((splitk_reduce_kernel<T, S>), dim3(grid), dim3(256), 0, s, p)
#define NM_REDUCE_ANY(T)              \
    switch (p.ksplit) {               \
    case 2: NM_REDUCE(T, 2); break;   \
    case 4: NM_REDUCE(T, 4); break;   \
    case 8: NM_REDUCE(T, 8); break;   \
    case 16: NM_REDUCE(T, 16); break; \
    default: set_error("internal: no reduction of %d splits", p.ksplit); return NM_ERR_UNSUPPORTED; \
    }
    if (ydt == NM_F32) {
        NM_REDUCE_ANY(float)
    } else {
        NM_REDUCE_ANY(bf16_t)
    }
#undef NM_REDUCE_ANY
#undef NM_REDUCE
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

int run_stream_floor(const void* x, size_t x_bytes, void* y, size_t y_bytes, hipStream_t s)
{
    const size_t nx = x_bytes / 16, ny = y_bytes / 16;
    const size_t most = nx > ny ? nx : ny;
    // enough workgroups to fill every CU several times over, never more threads than units
    int grid = (int)((most + 255) / 256);
    if (grid > 256 * 8) grid = 256 * 8;
    if (grid < 1) grid = 1;
    hipLaunchKernelGGL(stream_floor_kernel, dim3(grid), dim3(256), 0, s, reinterpret_cast<const u4v*>(x), nx,
                       reinterpret_cast<u4v*>(y), ny);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

int run_im2col(const void* x, nm_dtype_t dt, int B, int H, int W, int C, int Kh, int Kw, int sh, int sw,
               int ph, int pw, int dh, int dw, int Ho, int Wo, void* a, hipStream_t s)
{
    const int V = dt == NM_F32 ? 4 : 8;
    const bool vec = (C % V == 0);
    const size_t total = (size_t)B * Ho * Wo * Kh * Kw * (vec ? C / V : C);
    const unsigned grid = (unsigned)std::min<size_t>((total + 255) / 256, 1u << 20);
#define NM_IM2COL(T, VV)                                                                                    \
    hipLaunchKernelGGL((im2col_kernel<T, VV>), dim3(grid), dim3(256), 0, s, (const T*)x, (T*)a, B, H, W, C, Kh, \
                       Kw, sh, sw, ph, pw, dh, dw, Ho, Wo)
    if (dt == NM_F32) { if (vec) NM_IM2COL(float, 4); else NM_IM2COL(float, 1); }
    else { if (vec) NM_IM2COL(bf16_t, 8); else NM_IM2COL(bf16_t, 1); }
#undef NM_IM2COL
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

template <typename T, int KT>
int launch_maxpool_vec(const void* x, int B, int H, int W, int C, int k, int stride, int pad, int Ho, int Wo, void* y, hipStream_t s)
{
    const int bpr = (int)(((size_t)Wo * (C * sizeof(T) / 16) + 255) / 256), rows = B * Ho;
    const int per_xcd = (int)(((size_t)rows * bpr + 7) / 8);
    hipLaunchKernelGGL((maxpool_vec_kernel<T, KT>), dim3(per_xcd * 8), dim3(256), 0, s, (const T*)x, (T*)y, H, W, C, k,
                       stride, pad, Ho, Wo, rows, bpr, per_xcd);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

int run_maxpool(const void* x, nm_dtype_t dt, int B, int H, int W, int C, int k, int stride, int pad,
                int Ho, int Wo, void* y, hipStream_t s)
{
    // whole 16-byte granules per pixel, and block numbers that fit an int
    const size_t es = dt == NM_F32 ? 4 : 2;
    if ((size_t)C * es % 16 == 0 && (size_t)B * Ho * (((size_t)Wo * C * es / 16 + 255) / 256) < (1u << 30)) {
        if (dt == NM_F32)
            return k == 3 ? launch_maxpool_vec<float, 3>(x, B, H, W, C, k, stride, pad, Ho, Wo, y, s)
                          : launch_maxpool_vec<float, 0>(x, B, H, W, C, k, stride, pad, Ho, Wo, y, s);
        return k == 3 ? launch_maxpool_vec<bf16_t, 3>(x, B, H, W, C, k, stride, pad, Ho, Wo, y, s)
                      : launch_maxpool_vec<bf16_t, 0>(x, B, H, W, C, k, stride, pad, Ho, Wo, y, s);
    }
    const size_t total = (size_t)B * Ho * Wo * ((C + 3) / 4);
    const unsigned grid = (unsigned)std::min<size_t>((total + 255) / 256, 1u << 20);
    if (dt == NM_F32)
        hipLaunchKernelGGL(maxpool_kernel<float>, dim3(grid), dim3(256), 0, s, (const float*)x, (float*)y, B, H,
                           W, C, k, stride, pad, Ho, Wo);
    else
        hipLaunchKernelGGL(maxpool_kernel<bf16_t>, dim3(grid), dim3(256), 0, s, (const bf16_t*)x, (bf16_t*)y, B,
                           H, W, C, k, stride, pad, Ho, Wo);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

int run_avgpool(const void* x, nm_dtype_t dt, int B, int HW, int C, void* y, hipStream_t s)
{
    const dim3 grid((C + 63) / 64, B);
    if (dt == NM_F32)
        hipLaunchKernelGGL(avgpool_kernel<float>, grid, dim3(256), 0, s, (const float*)x, (float*)y, HW, C);
    else
        hipLaunchKernelGGL(avgpool_kernel<bf16_t>, grid, dim3(256), 0, s, (const bf16_t*)x, (bf16_t*)y, HW, C);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
