// fp32 convolution on the bf16 matrix cores, at fp32 accuracy.
//
// The fp32 matrix instruction (16x16x4, 32 clocks) contracts four kept columns; the bf16 ones are 16 times
// faster per multiply.  An fp32 number is the exact sum of three bf16 numbers (8 + 8 + 8 significant bits),
// v = v1 + v2 + v3, and a product x1 w1 + (x1 w2 + x2 w1) + (x1 w3 + x2 w2 + x3 w1) + terms of at most 2^-24
// of it with either sign (the weights are cut by rounding): six bf16 products, added up in fp32.  With the
// sparse instruction (see the gather-free bf16 kernel: the two kept columns of an aligned group of four)
// 64 channels at 2:4 cost 6 x 16 clocks against 8 x 32.  The accumulator is rounded once per 32 kept columns
// and product instead of once per four columns, so the result is nearer to float64 than the fp32
// instruction's (2-norm, He-normal weights: 2304 kept columns 7.2e-7 against 8.3e-7, 288 2.3e-7 against
// 2.9e-7, 18 4e-8 against 8e-8).
//
//   SPARSE = true   at most two kept columns in every aligned group of four channels
//   SPARSE = false  the dense instruction on zero-filled weights (N = M, 4:8, groups over all channels)
//
// Eight wavefronts.  Four producers fetch the im2col strip (16-byte fp32 loads, two chunks ahead in
// registers), cut it into its three bf16 planes and write those to LDS; the cutting is vector work that
// runs beside the matrix instructions of the four contracting wavefronts, and is done once per value and
// workgroup.  The contracting wavefronts take their weights, cut into planes by nm_prune and laid out in
// lane order, straight from memory into registers one chunk ahead, and read each strip operand once for
// six instructions, so LDS reads (the bound of the plain bf16 form) cost half as much per instruction.
// Two LDS stages, one barrier per chunk of 64 channels of one tap.
//
// Row blocks are 16 consecutive output channels whatever the column tile T: in the sparse instruction
// every row has its own index operand, so rows of different column tiles (T < 16) share a block.
//
// What the planes cannot carry: an infinite x1 makes inf * 0 = NaN in the products with an empty w2 or w3, and
// bits below 2^-133, bf16's smallest subnormal (which the matrix cores do count, as fp32 instructions do).
//   weights: nm_prune makes no tables for a layer whose kept weights the planes do not hold exactly.
//   activations (under 2^-110): the producers say so, each product is then off by at most 2^-132 |w|, and outputs
//     below redo_below = K' max|w| 2^-105, where that may be more than 2^-27 of them, are computed again, zeros
//     among them.
// An output that comes out infinite, NaN or (not zero and) below 2^-100, where lower planes' products meet the
// end of fp32's subnormals, is computed again as well, one fp32 multiply-add per kept column (split_redo).
//
// Bound: on the 3x3 layers the matrix cores (14x14 256 -> 256, batch 64: 78 -> 56 us; with staging and weight
// loads switched off 40 us, of which 8 are the launch and the rest 196 of 256 CUs at 36 x 96 instructions);
// on the 1x1 layers the stores of the output (28x28 128 -> 512: 50 -> 46 us).
#pragma once

#include "nm_conv_sp16_kernel.h"

namespace nm {

constexpr unsigned kSplitInf = 0xff000000u;              // infinity, as a word shifted left by one
constexpr unsigned kSplitTiny = (127u - 100u) << 24;     // 2^-100, likewise
// wavefronts per SIMD to leave registers for: two workgroups per CU where accumulators and the two
// weight sets fit 128 registers, one otherwise
constexpr int split_waves(int NBLK, int WP, int NJ, bool sparse)
{
    const int regs = 4 * NBLK * NJ + 2 * NJ * (sparse ? 13 : 24) + 24;
    return regs <= 110 && 16 * NBLK * WP <= 104 ? 4 : 2;   // (two stages of more pixels leave LDS for one workgroup)
}

// Four fp32 values as three planes of four bf16 values (8 bytes each), cut at bits 16 and 8: the first
// plane is the upper half of the word, the second the next 8 significant bits, the third the last 8
// (both exact differences, rest[0] and rest[1]: what the planes leave out, bits below 2^-133, are lower halves of
// theirs that are not zero).  22 full-rate instructions; the converting instruction instead of the
// byte permutes: 14x14 3x3 256 -> 256, 128-pixel tiles, 66.8 us against 63.0.
__device__ inline void split_planes(const f4 v, u2v (&out)[3], f4 (&rest)[2])
{
    auto pair = [](float a, float b) { return __builtin_amdgcn_perm(__float_as_uint(b), __float_as_uint(a), 0x07060302u); };
    auto top = [](float a, unsigned mask) { return __uint_as_float(__float_as_uint(a) & mask); };
    const f4 t = f4{top(v.x, 0xffffff00u), top(v.y, 0xffffff00u), top(v.z, 0xffffff00u), top(v.w, 0xffffff00u)};
    const f4 b = t - f4{top(v.x, 0xffff0000u), top(v.y, 0xffff0000u), top(v.z, 0xffff0000u), top(v.w, 0xffff0000u)};
    const f4 c = v - t;
    out[0] = u2v{pair(v.x, v.y), pair(v.z, v.w)};
    out[1] = u2v{pair(b.x, b.y), pair(b.z, b.w)};
    out[2] = u2v{pair(c.x, c.y), pair(c.z, c.w)};
    rest[0] = b;
    rest[1] = c;
}

__device__ inline void split_lost(const f4 (&rest)[2], unsigned& lost)
{
#pragma unroll
    for (int r = 0; r < 4; ++r) lost |= __float_as_uint(rest[0][r]) | __float_as_uint(rest[1][r]);
}

// The kernel's arguments where they lie: what only the end of a tile needs is read there, not held in scalar
// registers through the chunks.
typedef const __attribute__((address_space(4))) ConvParams* kernarg_t;

// Output (pixel pp, channel co) over the kept columns with flat index in [k_lo, k_hi), one fp32
// multiply-add each.  A NaN stays one, so the loop ends there.
__device__ inline float split_redo(kernarg_t kp, int pp, int co, int k_lo, int k_hi, float acc)
{
    const int HoWo = kp->Ho * kp->Wo;
    const int b = pp / HoWo, rem = pp - b * HoWo, ho = rem / kp->Wo, wo = rem - ho * kp->Wo;
    const int j = co / kp->ctile, t = co - j * kp->ctile;
    const float* x = reinterpret_cast<const float*>(kp->x);
    for (int kk = 0; kk < kp->kprime; ++kk) {
        const size_t at = (size_t)j * kp->kprime + kk;
        const int k = kp->idx[at];
        if (k < k_lo || k >= k_hi) continue;
        const int tap = k / kp->Cin, ci = k - tap * kp->Cin, kh = tap / kp->Kw, kw = tap - kh * kp->Kw;
        const int hi = ho * kp->sh - kp->ph + kh * kp->dh, wi = wo * kp->sw - kp->pw + kw * kp->dw;
        if ((unsigned)hi >= (unsigned)kp->H || (unsigned)wi >= (unsigned)kp->W) continue;
        acc = fmaf(kp->vals[at * kp->ctile + t], x[((size_t)((size_t)b * kp->H + hi) * kp->W + wi) * kp->Cin + ci], acc);
        if (acc != acc) break;
    }
    return acc;
}

// The same for the channels co .. co + 3 of one column tile: the kept columns in pairs, whose loads are
// under way together, the tap worked out anew only where it changes.
__device__ inline f4 split_redo4(kernarg_t kp, int pp, int co, int k_lo, int k_hi, f4 acc)
{
    const int HoWo = kp->Ho * kp->Wo, Cin = kp->Cin, kprime = kp->kprime, T = kp->ctile;
    const int b = pp / HoWo, rem = pp - b * HoWo, ho = rem / kp->Wo, wo = rem - ho * kp->Wo;
    const int j = co / T, t = co - j * T, b_H = b * kp->H;
    const int h0 = ho * kp->sh - kp->ph, w0 = wo * kp->sw - kp->pw;
    const float* x = reinterpret_cast<const float*>(kp->x);
    const int* const idx = kp->idx + (size_t)j * kprime;
    const float* const vals = kp->vals + (size_t)j * kprime * T + t;
    int kk = 0;
    for (int n = kprime; n > 0;) {               // the first kept column from k_lo on
        const int half = n >> 1;
        if (idx[kk + half] < k_lo) { kk += half + 1; n -= half + 1; } else n = half;
    }
    int tap_end = -1;
    bool in = false;
    unsigned base = 0;                           // element of x (of fewer than 2^31) that column k of the tap is: base + k
    for (; kk < kprime; kk += 2) {
        int k[2];
        f4 w[2];
        float v[2];
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            const int at = kk + u < kprime ? kk + u : kprime - 1;
            k[u] = idx[at];
            w[u] = *reinterpret_cast<const f4*>(vals + (size_t)at * T);
        }
#pragma unroll
        for (int u = 0; u < 2; ++u) {
            if (k[u] >= tap_end) {
                kernarg_t kq = kp;               // (read here, not held through the loop)
                asm volatile("" : "+s"(kq));
                const int tap = k[u] / Cin, kh = tap / kq->Kw, kw = tap - kh * kq->Kw;
                const int hi = h0 + kh * kq->dh, wi = w0 + kw * kq->dw;
                in = ((unsigned)hi < (unsigned)kq->H) & ((unsigned)wi < (unsigned)kq->W);
                base = (unsigned)(((b_H + hi) * kq->W + wi - tap) * Cin);
                tap_end = (tap + 1) * Cin;
            }
            const bool live = in & (kk + u < kprime) & (k[u] < k_hi);
            v[u] = x[live ? base + (unsigned)k[u] : 0u];
            v[u] = live ? v[u] : 0.f;
        }
#pragma unroll
        for (int u = 0; u < 2; ++u)
#pragma unroll
            for (int r = 0; r < 4; ++r) acc[r] = fmaf(w[u][r], v[u], acc[r]);
        if (k[1] >= k_hi || ((acc[0] != acc[0]) & (acc[1] != acc[1]) & (acc[2] != acc[2]) & (acc[3] != acc[3]))) break;
    }
    return acc;
}

// Computes those of the outputs (pixel pp, channels co .. co + 3) again whose sums `sum` say so, and stores them.
__device__ inline void split_again(kernarg_t kp, const u4v sum, int pp, int co, unsigned below, bool inexact, int k_lo, int k_hi,
                                   const float* bias, const float* res, bool relu, float* y)
{
    asm volatile("" : "+s"(kp));
    unsigned again = 0u;                         // a bit per channel
    const int Cout = kp->Cout;
#pragma unroll
    for (int r = 0; r < 4; ++r) {
        const unsigned w = sum[r] << 1;
        again |= ((inexact ? w : w - 1u) < below || w >= kSplitInf) && co + r < Cout ? 1u << r : 0u;
    }
    if (!again) return;
    unsigned off = (unsigned)pp * (unsigned)Cout + (unsigned)co;
    const bool quad = kp->ctile % 4 == 0 && Cout % 4 == 0;
    f4 o = f4{0.f, 0.f, 0.f, 0.f};
    if (quad) o = split_redo4(kp, pp, co, k_lo, k_hi, bias ? *reinterpret_cast<const f4*>(bias + co) : o);
#pragma unroll 1
    for (; again; again >>= 1, ++off, ++co, o = f4{o.y, o.z, o.w, 0.f}) {
        if (!(again & 1u)) continue;
        float v = quad ? o.x : split_redo(kp, pp, co, k_lo, k_hi, bias ? bias[co] : 0.f);
        if (res) v += res[off];
        y[off] = relu ? relu1(v) : v;
    }
}

// LDS accesses of a stage are ordered by hand around a bare barrier: this wavefront's LDS writes have
// landed and its LDS reads have returned; global loads in flight stay in flight.
__device__ inline void split_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

// The finished blocks of a wavefront (pixels from pix0, row blocks from rb0): bias (where rows do not come in whole quads,
// `fast`, and it is not in the accumulators), residual, activation, store, and what has to be computed again; span(lo, hi)
// says which kept columns the sums run over.  `piece` is the wavefront's own LDS, split_out_rows(NBLK) rows.
template <int NBLK, int NJ, typename Span>
__device__ inline __attribute__((always_inline)) void split_finish(kernarg_t kp, const f4 (&acc)[NJ][NBLK], char* piece, int lane, int pix0, int rb0,
                                                                   int inexact, bool fast, float* __restrict__ y,
                                                                   const float* __restrict__ res, bool relu, Span&& span)
{
    const int q = lane >> 4, n = lane & 15;
    // Through LDS, so that every store covers whole rows of this wavefront's channels (64 NJ bytes a pixel)
    // instead of 64-byte pieces.  The piece is the wavefront's own: no barrier, and the producers are
    // already staging the next tile.
    constexpr int PITCH = split_out_pitch(NJ);
    constexpr int PB = split_out_rows(NBLK) / 16;   // blocks per piece
    constexpr int GPR = NJ * 4;                     // 16-byte granules per row
    constexpr int RPP = 64 / GPR;                   // rows per pass of the wavefront
    const int r0 = lane / GPR, cg = lane % GPR;
    const int co = rb0 * 16 + cg * 4;
    const char* const src = piece + r0 * PITCH + cg * 16;
    const int P = kp->P, Cout = kp->Cout;
    constexpr int NP = PB * 16 / RPP;               // passes per piece
#pragma unroll
    for (int b0 = 0; b0 < NBLK; b0 += PB) {
#pragma unroll
        for (int b = b0; b < b0 + PB && b < NBLK; ++b)
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj)
                *reinterpret_cast<f4*>(piece + ((b - b0) * 16 + n) * PITCH + jj * 64 + q * 16) = acc[jj][b];
        __builtin_amdgcn_wave_barrier();
        const int rows = (NBLK - b0 < PB ? NBLK - b0 : PB) * 16;
        const int pp0 = pix0 + b0 * 16 + r0;
        unsigned lo = ~0u, hi = 0u;          // of the words without their sign; a zero counts as large in lo
        auto look = [&](const f4 v) {
#pragma unroll
            for (int r = 0; r < 4; ++r) {
                const unsigned w = __float_as_uint(v[r]) << 1;
                lo = w - 1u < lo ? w - 1u : lo;
                hi = w > hi ? w : hi;
            }
        };
        if (fast) {
            f4 v[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) v[k] = *reinterpret_cast<const f4*>(src + k * (RPP * PITCH));
#pragma unroll
            for (int k = 0; k < NP; ++k) look(v[k]);   // (values of rows that do not exist are sorted out below)
            if (res) {   // all of the piece's at once: the memory counter makes a load wait for the stores before it
                f4 rv[NP];
#pragma unroll
                for (int k = 0; k < NP; ++k) {
                    const bool live = k * RPP + r0 < rows && pp0 + k * RPP < P && co < Cout;
                    rv[k] = load4(res + (live ? (unsigned)(pp0 + k * RPP) * (unsigned)Cout + (unsigned)co : 0u));
                }
#pragma unroll
                for (int k = 0; k < NP; ++k) v[k] = v[k] + rv[k];
            }
            if (relu) {
#pragma unroll
                for (int k = 0; k < NP; ++k) v[k] = relu4(v[k]);
            }
            auto store = [&](auto stream) {
#pragma unroll
                for (int k = 0; k < NP; ++k)
                    if (k * RPP + r0 < rows && pp0 + k * RPP < P && co < Cout)
                        store_out16<decltype(stream)::value>(y + ((unsigned)(pp0 + k * RPP) * (unsigned)Cout + (unsigned)co),
                                                             __builtin_bit_cast(u4v, v[k]));
            };
            if (kp->stream) store(std::true_type());
            else store(std::false_type());
        } else {
#pragma unroll 1
            for (int row = 0; row < rows; row += RPP) {
                const f4 v = *reinterpret_cast<const f4*>(src + row * PITCH);
                if (pp0 + row >= P) continue;
                look(v);
#pragma unroll
                for (int r = 0; r < 4; ++r) {
                    if (co + r >= Cout) continue;
                    const unsigned off = (unsigned)(pp0 + row) * (unsigned)Cout + (unsigned)(co + r);
                    float o = v[r] + (kp->bias && kp->ksplit <= 1 ? kp->bias[co + r] : 0.f);
                    if (res) o += res[off];
                    if (relu) o = relu1(o);
                    y[off] = o;
                }
            }
        }
        if (__builtin_expect(lo < kSplitTiny || hi >= kSplitInf || inexact, 0)) {
            __builtin_amdgcn_s_waitcnt(0);   // the stores above come first
            const unsigned below = inexact ? kp->redo_below : kSplitTiny;
            int k_lo, k_hi;
            span(k_lo, k_hi);
#pragma unroll 1
            for (int row = 0; row < rows; row += RPP)
                if (pp0 + row < P && co < Cout)
                    split_again(kp, *reinterpret_cast<const u4v*>(src + row * PITCH), pp0 + row, co, below, inexact != 0, k_lo, k_hi,
                                kp->ksplit <= 1 ? kp->bias : nullptr, res, relu, y);
        }
        __builtin_amdgcn_wave_barrier();
    }
}

template <int NBLK, int WP, int NJ, bool SPARSE>
__global__ __launch_bounds__(512, split_waves(NBLK, WP, NJ, SPARSE)) void nm_conv_split_kernel(const ConvParams p)
{
    constexpr int BPW = 16 * NBLK;
    constexpr int BP = BPW * WP;
    constexpr int WC = 4 / WP;
    constexpr int AH = SPARSE ? 1 : 2;           // 16-byte weight operands per plane and row block
    constexpr int RB = kSplitCK * 2;             // bytes per pixel row of a plane
    constexpr int PLANE = BP * RB;
    constexpr int STAGE = split_stage_bytes(BP);
    constexpr int RING = split_waves(NBLK, WP, NJ, SPARSE) == 2 ? 2 : 1;   // strip operands held per wavefront
    static_assert(RING == 1 || NBLK % 2 == 0, "a chunk ends on the ring slot it began with");

    extern __shared__ __attribute__((aligned(16))) char lds8[];   // [2][3][BP][64] bf16, then the output pieces

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_id = __builtin_amdgcn_readfirstlane(tid >> 6);   // 0..3 contract, 4..7 produce

    // Each XCD has a contiguous range of output tiles (those that share pixels are neighbours and meet in
    // its L2); its workgroups take them in turn, wg_per_xcd apart.
    const int bid = blockIdx.x;
    const int per_xcd = (p.n_wg + 7) / 8;
    const int t_end = ((bid & 7) + 1) * per_xcd < p.n_wg ? ((bid & 7) + 1) * per_xcd : p.n_wg;
    const int t_first = (bid & 7) * per_xcd + (bid >> 3);
    if (t_first >= t_end) return;
    const int n_out_tiles = p.n_ptiles * p.n_cblocks;
    // (with a K split a workgroup has one tile, so the chunk range is the same for all its tiles)
    const int ks = p.ksplit > 1 ? t_first / n_out_tiles : 0;
    const int c_begin = ks * p.cps;
    const int c_end = c_begin + p.cps < p.nchunks ? c_begin + p.cps : p.nchunks;
    const int nc = c_end - c_begin;
    const int total = nc * ((t_end - t_first + p.wg_per_xcd - 1) / p.wg_per_xcd);   // chunks of all tiles, one stream

    if (wave_id >= 4) {
        // ---- producers: item = (pixel, 4-channel quad); a thread keeps its quad and NIT pixels ----------
        constexpr int NIT = BP / 16;
        const int t = tid - 256;
        const int quad = t & 15, pl0 = t >> 4;
        const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, p.x_bytes);
        int hi0[NIT], wi0[NIT];
        unsigned base[NIT], voff[NIT];
        const int HoWo = p.Ho * p.Wo;
        const int tap0 = c_begin / p.ncpt;
        int f_tile = t_first, f_c = c_begin, f_kh = 0, f_kw = 0, f_ci0 = 0, f_left = total;
        auto retap = [&]() {
            const int dhh = f_kh * p.dh, dww = f_kw * p.dw;
            const unsigned tapoff = (unsigned)((dhh * p.W + dww) * p.Cin) * 4u;
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int hi = hi0[it] + dhh, wi = wi0[it] + dww;
                const bool inb = ((unsigned)hi < (unsigned)p.H) & ((unsigned)wi < (unsigned)p.W);
                voff[it] = inb ? base[it] + tapoff : kOOB;
            }
        };
        auto open_tile = [&]() {   // pixels of tile f_tile, first chunk
            const int ptile = (f_tile - ks * n_out_tiles) / p.n_cblocks;
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                const int pp = ptile * BP + pl0 + it * 16;
                const int b = (int)fdiv((unsigned)pp, p.howo_mul, p.howo_shift);
                const int rem = pp - b * HoWo;
                const int ho = (int)fdiv((unsigned)rem, p.wo_mul, p.wo_shift);
                const int wo = rem - ho * p.Wo;
                const int h0 = ho * p.sh - p.ph, w0 = wo * p.sw - p.pw;
                hi0[it] = pp < p.P ? h0 : -(1 << 28);   // a dead pixel has every tap outside the image
                wi0[it] = w0;
                base[it] = (unsigned)(((b * p.H + h0) * p.W + w0) * p.Cin + quad * 4) * 4u;
            }
            f_c = c_begin;
            f_ci0 = (c_begin - tap0 * p.ncpt) * kSplitCK;
            f_kh = tap0 / p.Kw;
            f_kw = tap0 - f_kh * p.Kw;
            retap();
        };
        f4 sa[NIT], sb[NIT];
        auto fetch = [&](f4 (&st)[NIT]) {   // the next chunk of the stream into registers; past the last one nothing is read
            const unsigned dead = (f_left <= 0 || f_ci0 + quad * 4 >= p.Cin) ? kOOB : 0u;
#pragma unroll
            for (int it = 0; it < NIT; ++it)
                st[it] = buf_load4(xr, (voff[it] + (unsigned)(f_ci0 * 4)) | dead, 0, (const float*)nullptr);
            --f_left;
            ++f_c;
            f_ci0 += kSplitCK;
            if (f_c == c_end) {
                f_tile += p.wg_per_xcd;
                if (f_left > 0) open_tile();
            } else if (f_ci0 >= p.Cin) {   // uniform, once per tap
                f_ci0 = 0;
                f_kw = f_kw + 1 == p.Kw ? 0 : f_kw + 1;
                f_kh += f_kw == 0 ? 1 : 0;
                retap();
            }
        };
        // Whether planes left bits out so far: a word per producer in the padding of an output piece's first row, written
        // with the last chunk of a tile, so that the others find it when they finish that tile.
        unsigned lost = 0u;
        int s_left = nc;
        int* const lossy = reinterpret_cast<int*>(lds8 + 2 * STAGE + (wave_id - 4) * (split_out_rows(NBLK) * split_out_pitch(NJ)) + NJ * 64);
        char* const wdst = lds8 + pl0 * RB + (((quad >> 1) ^ sp16_swz(pl0, RB)) * 16) + (quad & 1) * 8;
        f4 rest[NIT][2];
        auto stash = [&](const f4 (&st)[NIT], int stage) {
#pragma unroll
            for (int it = 0; it < NIT; ++it) {
                u2v pl[3];
                split_planes(st[it], pl, rest[it]);
#pragma unroll
                for (int k = 0; k < 3; ++k)
                    *reinterpret_cast<u2v*>(wdst + stage * STAGE + k * PLANE + it * (16 * RB)) = pl[k];
            }
        };
        // (behind the writes and the next loads, which it would hold up.  14x14 3x3 256 -> 256, batch 32: 30.7 us without
        // the look, 31.6 with it in front of them, 31.2 here; ResNet-50 in fp32, batch 64, 2803 and 2838.)
        auto note = [&]() {
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int it = 0; it < NIT; ++it) split_lost(rest[it], lost);
            if (--s_left == 0) {
                *lossy = __builtin_amdgcn_ballot_w64((lost & 0xffffu) != 0u) != 0ull;
                s_left = nc;
            }
        };
        open_tile();
        fetch(sa);
        fetch(sb);
        stash(sa, 0);
        fetch(sa);
        note();
        int g = 0;
        // barrier g: chunk g is staged; then chunk g + 1 goes to the stage the others left at that barrier
        for (; g + 1 < total; g += 2) {
            split_barrier();
            stash(sb, 1);
            fetch(sb);
            note();
            split_barrier();
            if (g + 2 < total) {
                stash(sa, 0);
                fetch(sa);
                note();
            }
        }
        if (g < total) split_barrier();
        return;
    }

    // ---- contracting wavefronts ---------------------------------------------------------------------
    const int wave = wave_id;
    const int q = lane >> 4;
    const int n = lane & 15;
    const int wpx = wave % WP, wcx = wave / WP;
    const int wpix = wpx * BPW;
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wfrag, p.wfrag_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.rows, p.rows_bytes);
    constexpr unsigned WCH = 3 * AH * 1024;      // weight bytes per (row block, chunk)
    const bool fast = p.Cout % 4 == 0;           // output rows come in whole quads
    int tile = t_first, p0 = 0, rb0 = 0;
    auto first_rb = [&](int t) { return ((t - ks * n_out_tiles) % p.n_cblocks * WC + wcx) * NJ; };
    struct Ops {
        u4v a[NJ][3][AH];
        unsigned idx[NJ];
    };
    // operands of row block rb (beyond the last one: of the last one, computed and not stored) in chunk c
    auto load_op = [&](Ops& o, int jj, int rb, int c) {
        const unsigned at = (unsigned)(rb + jj < p.n_rowblocks ? rb + jj : p.n_rowblocks - 1) * (unsigned)p.nchunks + (unsigned)c;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int h = 0; h < AH; ++h)
                o.a[jj][pl][h] = __builtin_amdgcn_raw_buffer_load_b128(
                    wr, (unsigned)lane * 16u + (unsigned)(pl * AH + h) * 1024u, at * WCH, 0);
        if constexpr (SPARSE) o.idx[jj] = __builtin_amdgcn_raw_buffer_load_b32(rr, (unsigned)lane * 4u, at * 256u, 0);
    };
    f4 acc[NJ][NBLK];
    // the accumulators of the current tile start from the bias where rows come in whole quads
    auto open_tile = [&]() {
        p0 = (tile - ks * n_out_tiles) / p.n_cblocks * BP;
        rb0 = first_rb(tile);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            f4 bb = f4{0.f, 0.f, 0.f, 0.f};
            const int co = (rb0 + jj) * 16 + q * 4;
            if (fast && p.bias && p.ksplit <= 1 && co < p.Cout) bb = *reinterpret_cast<const f4*>(p.bias + co);
#pragma unroll
            for (int b = 0; b < NBLK; ++b) acc[jj][b] = bb;
        }
    };
    Ops oa, ob;
    open_tile();
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) load_op(oa, jj, rb0, c_begin);

    unsigned roff[2];
#pragma unroll
    for (int h = 0; h < 2; ++h) roff[h] = (unsigned)((wpix + n) * RB + (((q * 2 + h) ^ sp16_swz(n, RB)) * 16));

    // One workgroup per CU (RING = 2): the next block's operands are requested one block ahead, and across
    // chunks too -- the barrier that says the next chunk is staged stands before the last block, when every
    // read of this stage has returned, and the last block's instructions cover the first reads behind it.
    // Two workgroups per CU (RING = 1): the other one covers the wait; the barrier opens the chunk.
    u4v ring[RING][3][2];
    auto read_plane = [&](int stage, int b, int pl, u4v (&d)[3][2]) {
#pragma unroll
        for (int h = 0; h < 2; ++h)
            d[pl][h] = *reinterpret_cast<const u4v*>(lds8 + stage * STAGE + roff[h] + pl * PLANE + b * (16 * RB));
    };
    auto read_b = [&](int stage, int b, u4v (&d)[3][2]) {
#pragma unroll
        for (int pl = 2; pl >= 0; --pl) read_plane(stage, b, pl, d);
    };
    // one chunk out of stage st (`more`: the stream goes on in the other one); the operands of the next one (row
    // blocks from rbn, chunk cn) are loaded on the way, spread over the blocks: a burst leaves the matrix cores idle
    auto chunk = [&](const Ops& o, Ops& next, int st, bool more, int rbn, int cn) {
        if constexpr (RING == 1) split_barrier();
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            const int slot = RING == 2 ? b & 1 : 0;
            if constexpr (RING == 1) read_b(st, b, ring[0]);
            else if (b + 1 == NBLK && more) split_barrier();
            __builtin_amdgcn_sched_barrier(0);
            const u4v(&x)[3][2] = ring[slot];
            // smallest products first; the row blocks take turns, so that no instruction waits for the one before it
            constexpr int XP[6] = {2, 1, 0, 1, 0, 0}, WPL[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
            for (int k = 0; k < 6; ++k) {
                if constexpr (SPARSE) {
                    const bf16x bv = __builtin_shufflevector(__builtin_bit_cast(bf8x, x[XP[k]][0]),
                                                             __builtin_bit_cast(bf8x, x[XP[k]][1]), 0, 1, 2, 3, 4, 5,
                                                             6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
#pragma unroll
                    for (int jj = 0; jj < NJ; ++jj)
                        acc[jj][b] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(
                            __builtin_bit_cast(bf8x, o.a[jj][WPL[k]][0]), bv, acc[jj][b], (int)o.idx[jj], 0, 0);
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
#pragma unroll
                        for (int jj = 0; jj < NJ; ++jj)
                            acc[jj][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                                __builtin_bit_cast(bf8x, o.a[jj][WPL[k]][AH == 2 ? h : 0]),
                                __builtin_bit_cast(bf8x, x[XP[k]][h]), acc[jj][b], 0, 0, 0);
                }
                // behind the products: the next block's planes in the order they are needed (past the last chunk
                // a stage nobody fills is read and not used), then the row blocks whose turn to be loaded it is
                if constexpr (RING == 2)
                    if (k < 3) read_plane(b + 1 < NBLK ? st : st ^ 1, b + 1 < NBLK ? b + 1 : 0, 2 - k, ring[(slot + 1) % RING]);
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
                    if (jj * NBLK / NJ == b && jj - (b * NJ + NBLK - 1) / NBLK == (k + 3) % 6) load_op(next, jj, rbn, cn);
                if constexpr (RING == 2) __builtin_amdgcn_sched_barrier(0);
            }
            __builtin_amdgcn_sched_barrier(0);
        }
    };

    char* const piece = lds8 + 2 * STAGE + wave * (split_out_rows(NBLK) * split_out_pitch(NJ));
    // The finished tile: bias (where it is not in the accumulators yet), residual, activation, store.
    auto close_tile = [&]() {
        kernarg_t kp = (kernarg_t)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(kp));
        int lane = tid & 63;                     // (opaque: the addresses below are worked out here, not kept through the chunks)
        asm volatile("" : "+v"(lane));
        // K split: partial sums [split][pixel][channel]; bias, residual and activation come where they are added up
        float* __restrict__ y = kp->ksplit > 1 ? kp->partial + (size_t)ks * (size_t)kp->P * (size_t)kp->Cout : reinterpret_cast<float*>(kp->y);
        const float* __restrict__ res = kp->ksplit > 1 ? nullptr : reinterpret_cast<const float*>(kp->res);
        const bool relu = kp->ksplit <= 1 && kp->relu;
        int inexact = 0;                         // the planes of some activation so far left bits out
#pragma unroll
        for (int w = 0; w < 4; ++w)
            inexact |= *reinterpret_cast<const int*>(lds8 + 2 * STAGE + w * (split_out_rows(NBLK) * split_out_pitch(NJ)) + NJ * 64);
        split_finish<NBLK, NJ>(kp, acc, piece, lane, p0 + wpix, rb0, inexact, fast, y, res, relu, [&](int& k_lo, int& k_hi) {
            k_lo = (c_begin / kp->ncpt) * kp->Cin + (c_begin % kp->ncpt) * kSplitCK;
            k_hi = c_end < kp->nchunks ? (c_end / kp->ncpt) * kp->Cin + (c_end % kp->ncpt) * kSplitCK : kp->K;
        });
    };

    if constexpr (RING == 2) {
        split_barrier();
        read_b(0, 0, ring[0]);
    }
    int c = 0;   // chunk of the current tile
    auto step = [&](const Ops& o, Ops& next, int g, const int stage) {
        const bool last = c + 1 == nc, more = g + 1 < total;
        const int tn = last && more ? tile + p.wg_per_xcd : tile;
        chunk(o, next, stage, more, last ? first_rb(tn) : rb0, last ? c_begin : c_begin + c + 1);
        ++c;
        if (last) {
            close_tile();
            if (more) {
                tile = tn;
                open_tile();
                c = 0;
            }
        }
    };
    for (int g = 0;;) {
        step(oa, ob, g, 0);
        if (++g == total) break;
        step(ob, oa, g, 1);
        if (++g == total) break;
    }
}

template <int NBLK, int WP, int NJ, bool SPARSE>
int launch_split_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_split_kernel<NBLK, WP, NJ, SPARSE>;
    constexpr size_t lds = split_lds_bytes(NBLK, WP, NJ);
    static_assert(lds <= 160 * 1024, "two stages and the output pieces must fit the CU");
    {
        static unsigned long long done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, &done);
        if (rc != NM_OK) return rc;
    }
    // As many workgroups as the 256 CUs hold at once; they walk the output tiles, the producers fetching the
    // next tile while this one is finished and stored.  A K split is for few tiles: one each.
    constexpr int resident = 256 * (split_waves(NBLK, WP, NJ, SPARSE) > 2 && 2 * lds <= 160 * 1024 ? 2 : 1);
    ConvParams q = p;
    if (p.ksplit <= 1 && p.n_wg > resident) q.wg_per_xcd = resident / 8;
    hipLaunchKernelGGL(kern, dim3(q.wg_per_xcd * 8), dim3(512), lds, s, q);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
