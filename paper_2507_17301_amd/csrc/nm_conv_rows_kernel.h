// Convolution for layers with very few input channels (the 7x7 first layer of the ResNets: Cin = 3) out of
// staged input rows.
//
// A kernel row of such a layer is one contiguous run of Kw * Cin values per pixel, and the runs of
// neighbouring pixels overlap: 7 x 21 values a pixel, of which a pixel brings 2 x 7 new ones (stride 2).
// A workgroup therefore stages the input rows under R output rows as they are -- every value once, the
// image's zero padding included -- and reads the matrix operands straight out of them: K is laid out as
// Kh runs of GR 16-byte granules (the run starts `par` elements early so that it is 4-byte aligned, the
// weights are zero in every padding slot), so an operand is 16 bytes of one row at
//   (output row * sh + kh * dh) * row pitch + output column * sw * Cin * 2 + granule * 16.
// The weights of a wavefront's channels stay in its registers for the whole workgroup, and the finished
// blocks of 16 pixels leave through a wavefront-private LDS piece in whole 128-byte rows: after the rows
// are staged there is no barrier.
//
// PL = 1: bf16 tensors.  PL = 3: fp32 tensors cut into three bf16 planes while they are staged (once per
// value), six products per operand; see the three-plane kernel for the arithmetic and for the outputs
// that are computed again.  The five products of lower planes have accumulators of their own: a layer
// of few columns spreads them over several half-empty instructions, and added to the sum one by one they
// would round it more often than the fp32 instruction does (3x3x3: x1.06 of its distance from float64, so
// x0.45; 7x7x3 x0.84 and x0.33).
//
// Bound: memory (bf16, batch 64, 224x224x3 -> 112x112x64: 122 MB) and, in fp32, the matrix cores (K = 147
// padded to 192, six products: 54 us).  36 and 114 us; the kernel before this one staged every pixel's 24 granules separately, 48 KB
// into LDS and ~360 vector instructions a thread for 8 KB
// of output (80 us), the element-wise fp32 one took 190.
#pragma once

#include <type_traits>

#include "nm_conv_split_kernel.h"

namespace nm {

template <int PL, int NJ, int KS>
__global__ __launch_bounds__(256, PL == 1 && KS < 4 ? 3 : 2) void nm_conv_rows_kernel(const ConvParams p)
{
    typedef typename std::conditional<PL == 1, bf16_t, float>::type T;
    constexpr int ES = (int)sizeof(T);
    constexpr int WC = 4 / NJ, WP = NJ;          // wavefronts along the channels (64 a workgroup) and along the pixels
    constexpr int NS = KS * 2;                   // matrix instructions of 32 K positions
    extern __shared__ __attribute__((aligned(16))) char lds8[];   // [PL][rows][pitch], then four output pieces

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    const int n = lane & 15;
    const int logical = ((int)blockIdx.x & 7) * p.wg_per_xcd + ((int)blockIdx.x >> 3);
    if (logical >= p.n_wg) return;
    const int cblock = logical % p.n_cblocks;
    const int rt = logical / p.n_cblocks;
    const int per_img = (p.Ho + p.rows_r - 1) / p.rows_r;
    const int b = rt / per_img, ho0 = (rt - b * per_img) * p.rows_r;
    const int npx = (p.Ho - ho0 < p.rows_r ? p.Ho - ho0 : p.rows_r) * p.Wo;   // output pixels of this workgroup, one run of y
    const int wpx = wave % WP, wcx = wave / WP;
    const int rb0 = (cblock * WC + wcx) * NJ;

    char* const piece = lds8 + p.rows_lds + wave * kRowsPiece;
    constexpr int ROWB = NJ * 16 * ES, PITCH = ROWB + 16;       // a piece's row

    // weights of this wavefront's row blocks: [row block][instruction][plane][lane] x 16 bytes
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wfrag, p.wfrag_bytes);
    u4v a[NJ][NS][PL];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int rb = rb0 + jj < p.n_rowblocks ? rb0 + jj : p.n_rowblocks - 1;
#pragma unroll
        for (int m = 0; m < NS; ++m)
#pragma unroll
            for (int pl = 0; pl < PL; ++pl)
                a[jj][m][pl] = __builtin_amdgcn_raw_buffer_load_b128(wr, (unsigned)lane * 16u + (unsigned)((m * PL + pl) * 1024),
                                                                     (unsigned)rb * (NS * PL * 1024), 0);
    }

    // ---- input rows ho0 * sh - ph ... into LDS, zero outside the image -------------------------------
    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, p.x_bytes);
    const int G = p.rows_pitch / 16;             // granules per row of a plane
    const int h0 = ho0 * p.sh - p.ph;
    const int row_el = p.W * p.Cin;
    const int plane = p.rows_n * p.rows_pitch;
    const bool vec = (row_el * ES) % 16 == 0;    // rows of x start on 16 bytes
    auto row_base = [&](int r, bool* in) {       // element of x where staged row r starts
        const int hi = h0 + r;
        *in = (r < p.rows_n) & ((unsigned)hi < (unsigned)p.H);
        return (unsigned)(b * p.H + hi) * (unsigned)row_el;
    };
    if constexpr (PL == 1) {
        // straight into LDS: lane L of a wave-wide load fills granule (or word) L of a window
        const int total = p.rows_n * G;
        if (vec) {
            for (int w = wave * 64; w < total; w += 256) {
                const int r = (int)fdiv((unsigned)(w + lane), p.rowg_mul, p.rowg_shift);
                bool in;
                const unsigned rb = row_base(r, &in);
                const int off = (w + lane - r * G) * 16 - p.rows_data;
                const bool ok = in & ((unsigned)off < (unsigned)(row_el * 2));
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr_t)(lds8 + w * 16), 16, ok ? rb * 2u + (unsigned)off : kOOB, 0, 0, 0);
            }
        } else {
            for (int w = wave * 64; w < total * 4; w += 256) {
                const int r = (int)fdiv((unsigned)(w + lane) >> 2, p.rowg_mul, p.rowg_shift);
                bool in;
                const unsigned rb = row_base(r, &in);
                const int off = (w + lane - r * G * 4) * 4 - p.rows_data;
                const bool ok = in & ((unsigned)off < (unsigned)(row_el * 2));
                __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr_t)(lds8 + w * 4), 4, ok ? rb * 2u + (unsigned)off : kOOB, 0, 0, 0);
            }
        }
        NM_WAIT_VMCNT(0);
    } else {
        const int total = p.rows_n * G * 2;      // quads of four values: 8 bytes of a plane
        unsigned lost = 0u;                      // (see the three-plane kernel)
        for (int i0 = tid; i0 < total; i0 += 4 * 256) {
            f4 v[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                const int i = i0 + u * 256;
                const int r = (int)fdiv((unsigned)i >> 1, p.rowg_mul, p.rowg_shift);
                bool in;
                const unsigned rb = row_base(r, &in);
                const int e = (i - r * G * 2) * 4 - p.rows_data / 2;
                if (vec) {
                    v[u] = buf_load4(xr, (in && (unsigned)e < (unsigned)row_el) ? (rb + (unsigned)e) * 4u : kOOB, 0, (const float*)nullptr);
                } else {
#pragma unroll
                    for (int k = 0; k < 4; ++k)
                        v[u][k] = buf_load1(xr, (in && (unsigned)(e + k) < (unsigned)row_el) ? (rb + (unsigned)(e + k)) * 4u : kOOB,
                                            (const float*)nullptr);
                }
            }
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i0 + u * 256 >= total) continue;
                u2v pl[3];
                f4 rest[2];
                split_planes(v[u], pl, rest);
                split_lost(rest, lost);
#pragma unroll
                for (int k = 0; k < 3; ++k) *reinterpret_cast<u2v*>(lds8 + k * plane + (i0 + u * 256) * 8) = pl[k];
            }
        }
        const bool any = __builtin_amdgcn_ballot_w64((lost & 0xffffu) != 0u) != 0ull;
        if (lane == 0) *reinterpret_cast<int*>(piece + ROWB) = any;   // (the padding of a piece's first row)
    }

    // bias of this lane's rows, and where instruction m of a pixel finds this lane's granule
    f4 bb[NJ];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int co = (rb0 + jj) * 16 + q * 4;
        bb[jj] = f4{0.f, 0.f, 0.f, 0.f};
        if (p.bias && co < p.Cout) bb[jj] = *reinterpret_cast<const f4*>(p.bias + co);
    }
    int off[NS];
#pragma unroll
    for (int m = 0; m < NS; ++m) {
        const int g = 8 * (m / 2) + 2 * q + (m & 1);
        const int kh = (int)fdiv((unsigned)g, p.gr_mul, p.gr_shift), gi = g - kh * p.run_gr;
        off[m] = p.rows_front + (kh < p.Kh ? kh * p.dh * p.rows_pitch + gi * 16 : 0);   // (padding: any staged granule, weight 0; see `blocks` below)
    }
    __syncthreads();

    constexpr int GPR = ROWB / 16, RPP = 64 / GPR, NP = 16 / RPP;
    const int pix0 = (b * p.Ho + ho0) * p.Wo;
    const int r0 = lane / GPR, cg = lane % GPR;
    const int co_out = rb0 * 16 + cg * (16 / ES);
    // fp32: the planes of a staged value leave bits out
    int any = 0;
    if constexpr (PL == 3) {
#pragma unroll
        for (int w = 0; w < 4; ++w) any |= *reinterpret_cast<const int*>(lds8 + p.rows_lds + w * kRowsPiece + ROWB);
        any = __builtin_amdgcn_readfirstlane(any);
    }
    float most = 0.f;                            // bf16: the largest sum so far, a NaN once there was one
    T* __restrict__ y = reinterpret_cast<T*>(p.y);
    const T* __restrict__ res = reinterpret_cast<const T*>(p.res);
    // (real_only: elements that are no tap of a run are taken for zero)
    auto blocks = [&](auto real_only) {
        for (int blk = wpx * 16; blk < npx; blk += WP * 16) {
            const int i = blk + n < npx ? blk + n : npx - 1;
            const int orow = (int)fdiv((unsigned)i, p.wo_mul, p.wo_shift), wo = i - orow * p.Wo;
            const char* const src = lds8 + orow * p.sh * p.rows_pitch + wo * p.sw * p.Cin * 2;
            f4 acc[NJ], low[NJ];                 // low: the products of lower planes, so that they do not meet the sum one by one
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                acc[jj] = bb[jj];
                low[jj] = f4{0.f, 0.f, 0.f, 0.f};
            }
#pragma unroll
            for (int m = 0; m < NS; ++m) {
                u4v x[PL];
#pragma unroll
                for (int pl = 0; pl < PL; ++pl) {
                    const unsigned* const w = reinterpret_cast<const unsigned*>(src + off[m] + pl * plane);   // 4-byte aligned
                    x[pl] = u4v{w[0], w[1], w[2], w[3]};
                }
                if constexpr (real_only) {
                    int g = 8 * (m / 2) + 2 * q + (m & 1);
                    asm volatile("" : "+v"(g));      // (the masks are worked out here, not kept in registers)
                    const int kh = (int)fdiv((unsigned)g, p.gr_mul, p.gr_shift), e0 = (g - kh * p.run_gr) * 8 - p.run_d;
                    const int len = kh < p.Kh ? p.Kw * p.Cin : 0;
#pragma unroll
                    for (int u = 0; u < 4; ++u)
                        x[0][u] &= ((unsigned)(e0 + 2 * u) < (unsigned)len ? 0x0000ffffu : 0u) |
                                   ((unsigned)(e0 + 2 * u + 1) < (unsigned)len ? 0xffff0000u : 0u);
                }
                constexpr int NK = PL == 1 ? 1 : 6, K0 = 6 - NK;
                constexpr int XP[6] = {2, 1, 0, 1, 0, 0}, WPL[6] = {0, 1, 2, 0, 1, 0};   // smallest products first
#pragma unroll
                for (int k = K0; k < 6; ++k)
#pragma unroll
                    for (int jj = 0; jj < NJ; ++jj) {
                        f4& to = k < 5 ? low[jj] : acc[jj];
                        to = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8x, a[jj][m][WPL[k] % PL]),
                                                                     __builtin_bit_cast(bf8x, x[XP[k] % PL]), to, 0, 0, 0);
                    }
            }
            if constexpr (PL == 3) {
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) acc[jj] = acc[jj] + low[jj];
            }
            if constexpr (PL == 1 && !real_only) {
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
                    for (int r = 0; r < 4; r += 2)
                        most = __builtin_elementwise_maximum(__builtin_elementwise_maximum(fabsf(acc[jj][r]), fabsf(acc[jj][r + 1])), most);
                asm volatile("" : "+v"(most));   // (here: put off to the end of the block it would keep the sums alive beside their rounded form)
            }
            if constexpr (PL == 1) {
                // residual (accumulator layout: the first layer of a network has none), activation, the one rounding
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) {
                    const int co = (rb0 + jj) * 16 + q * 4;
                    if (res && blk + n < npx && co < p.Cout)
                        acc[jj] = acc[jj] + load4(res + ((unsigned)(pix0 + blk + n) * (unsigned)p.Cout + (unsigned)co));
                    if (p.relu) acc[jj] = relu4(acc[jj]);
                    store4(reinterpret_cast<bf16_t*>(piece + n * PITCH + jj * 32 + q * 8), acc[jj]);
                }
            } else {
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj) *reinterpret_cast<f4*>(piece + n * PITCH + jj * 64 + q * 16) = acc[jj];
            }
            __builtin_amdgcn_wave_barrier();
            const unsigned out0 = (unsigned)(pix0 + blk + r0) * (unsigned)p.Cout + (unsigned)co_out;
            u4v v[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) v[k] = *reinterpret_cast<const u4v*>(piece + (r0 + k * RPP) * PITCH + cg * 16);
            unsigned lo = ~0u, hi = 0u;              // (three planes) of the words without their sign; a zero counts as large in lo
#pragma unroll
            for (int k = 0; k < NP; ++k) {
                if constexpr (PL == 3) {
                    const bool live = blk + r0 + k * RPP < npx && co_out < p.Cout;
                    f4 f = __builtin_bit_cast(f4, v[k]);
#pragma unroll
                    for (int r = 0; r < 4; ++r) {
                        const unsigned w = v[k][r] << 1;
                        lo = w - 1u < lo ? w - 1u : lo;
                        hi = w > hi ? w : hi;
                    }
                    if (res) f = f + load4(res + (live ? out0 + (unsigned)(k * RPP) * (unsigned)p.Cout : 0u));
                    if (p.relu) f = relu4(f);
                    v[k] = __builtin_bit_cast(u4v, f);
                }
            }
            // Which way is asked once a block.  Asked for every row, a first layer in bf16 at batch 64 took 38.9 us where plain stores
            // without a question took 36.7; so, 37.9 and 38.0 (another card).
            auto rows = [&](auto put) {
#pragma unroll
                for (int k = 0; k < NP; ++k)
                    if (blk + r0 + k * RPP < npx && co_out < p.Cout) put(y + (out0 + (unsigned)(k * RPP) * (unsigned)p.Cout), v[k]);
            };
            if (p.stream) rows([](T* to, u4v x) { store_out16<true>(to, x); });
            else if (PL == 1 && p.keep) rows([](T* to, u4v x) { store_out16_kept(to, x); });
            else rows([](T* to, u4v x) { store_out16<false>(to, x); });
            if constexpr (PL == 3) {
                if (__builtin_expect(lo < kSplitTiny || hi >= kSplitInf || any, 0)) {
                    kernarg_t kp = (kernarg_t)__builtin_amdgcn_kernarg_segment_ptr();
                    __builtin_amdgcn_s_waitcnt(0);   // the stores above come first
                    const unsigned below = any ? kp->redo_below : kSplitTiny;
#pragma unroll 1
                    for (int row = r0; row < 16; row += RPP)
                        if (blk + row < npx && co_out < p.Cout)
                            split_again(kp, *reinterpret_cast<const u4v*>(piece + row * PITCH + cg * 16), pix0 + blk + row, co_out, below,
                                        any != 0, 0, p.K, p.bias, res, p.relu != 0, y);
                }
            }
            __builtin_amdgcn_wave_barrier();
        }
    };
    blocks(std::false_type());
    if constexpr (PL == 1) {
        // An infinity or NaN in a padding slot (the lead-in and the rest of a run, K positions beyond the last kernel
        // row) times its weight 0 is a NaN that the output is not due: once more without those slots.
        // (224x224x3 -> 64, batch 64: x1.045 of the time without the look; one multiply-add or class test a sum x1.06, the
        // staged granules looked at instead x1.05, a branch per block x1.6.)
        if (__builtin_expect(__builtin_amdgcn_ballot_w64(!(most < INFINITY)) != 0ull, 0)) {
            __builtin_amdgcn_s_waitcnt(0);       // the stores above come first
            blocks(std::true_type());
        }
    }
}

template <int PL, int NJ, int KS>
int launch_rows_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_rows_kernel<PL, NJ, KS>;
    const size_t lds = (size_t)p.rows_lds + 4 * kRowsPiece;
    if (lds > 160 * 1024 || p.Cout % (PL == 1 ? 8 : 4) != 0) {
        set_error("internal: the staged rows need %zu bytes of LDS and whole 16-byte pixels", lds);
        return NM_ERR_UNSUPPORTED;
    }
    {
        static unsigned long long done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(kern), 160 * 1024, &done);
        if (rc != NM_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3(p.wg_per_xcd * 8), dim3(256), lds, s, p);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
