// fp32 convolution of small layers: the K axis dealt out over the wavefronts of one workgroup.
//
// A layer of a few thousand outputs (one image, or the last stages of a few) is a launch, one trip to memory
// and a chain of chunks: nm_conv_kernel walks its K axis chunk by chunk with a barrier each, 9 to 72 of them
// in a row on a chip that is mostly idle, or splits it over workgroups and pays a second launch for the sum.
// Here a workgroup owns 16 PB pixels x 16 NJ channels and each of its up to 16 wavefronts contracts chunks of
// its own: it asks for the strip, the weights and the row table of its first two chunks at once, turns the
// strip through a wavefront-private piece of LDS (no barrier), and the wavefronts meet once, at the end, to
// add up their sums in LDS.  What bounds it is one round trip to memory (4.2 us with launch, sums and stores, of
// which an empty launch is 1.75) and the bytes that a CU's share brings into registers (16 pixels x K and 16 rows
// x K', 64 bytes a clock), then the fp32 instruction.  One image, 2:4, cold tensors, the best form before (K split
// and its second launch, where there is one) and this kernel, us: 28x28 3x3 128 -> 128 8.9 and 6.8, 28x28 s2
// 128 -> 256 8.2 and 5.7, 14x14 3x3 256 8.9 and 7.2, 7x7 3x3 512 9.6 and 8.9, 14x14 1x1 1024 -> 256 7.6 and 5.4,
// 512 -> 1000 dense 6.4 and 5.5, 56x56 3x3 64 8.1 and 7.6; untuned, where no K split is taken: 11.7, 11.7, 18.5,
// 32.5, 10.5, 8.3, 8.1.  The network of 21 such layers: 266 and 219.
//
// Operands as in nm_conv_kernel (16x16x4 fp32 instruction, the weights of its table); the row table is a
// second one of one byte a slot, the kept column's place in a pixel's row behind four zeros: an empty slot (0)
// reads a zero there and never another value of the strip.
#pragma once

#include "nm_conv_kernel.h"

namespace nm {

template <int PB, int NJ, int CK, int SPC, int NW>
__global__ __launch_bounds__(64 * NW) void nm_conv_wave_kernel(const ConvParams p)
{
    constexpr int ROW = wave_row_bytes(CK);   // a pixel's channels and four zeros; the rows of 16 pixels start in different banks
    constexpr int STRIP = 16 * PB * ROW;
    constexpr int GPR = CK / 4;               // 16-byte granules of a pixel
    constexpr int PPL = 64 / GPR;             // pixels per wave-wide load
    constexpr int NIT = 16 * PB / PPL;
    extern __shared__ char ldsc[];

    const int tid = threadIdx.x, lane = tid & 63, q = lane >> 4, n = lane & 15;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // A contiguous range of tiles per XCD; neighbours share what is larger, the weights of a row-block group or the
    // pixels.  (Divisions are multiply-shifts with factors from the host, here and below, and no branch before the
    // first loads: with the compiler's divisions and the arguments loaded block by block a workgroup took 1.3 us to
    // its first load.)
    const unsigned bid = blockIdx.x, xcd = bid & 7u, per = (unsigned)p.n_wg >> 3, more = (unsigned)p.n_wg & 7u;
    const unsigned logical = xcd * per + (xcd < more ? xcd : more) + (bid >> 3);
    const int n_fast = p.px_fast ? p.n_ptiles : p.n_cblocks;
    const int slow = (int)fdiv(logical, p.fast_mul, p.fast_shift), fast = (int)logical - slow * n_fast;
    const int ptile = p.px_fast ? fast : slow, cblock = p.px_fast ? slow : fast;
    const int p0 = ptile * 16 * PB, rb0 = cblock * NJ;

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, p.x_bytes);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wfrag, p.wfrag_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.rows, p.rows_bytes);

    // chunks [c_begin, c_end) of this wavefront, at least one
    const int c_begin = wave * p.cps;
    const int c_end = c_begin + p.cps < p.nchunks ? c_begin + p.cps : p.nchunks;

    const int g = lane % GPR, pl0 = lane / GPR;
    char* const strip = ldsc + wave * STRIP;
    // the zeros before each pixel's row
    if (lane < 16 * PB) *reinterpret_cast<f4*>(strip + lane * ROW) = f4{0.f, 0.f, 0.f, 0.f};

    f4 acc[PB][NJ];
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) acc[b][jj] = f4{0.f, 0.f, 0.f, 0.f};

    int hi0[NIT], wi0[NIT];
    unsigned base[NIT], voff[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int pp = p0 + pl0 + it * PPL;
        const int b = (int)fdiv((unsigned)pp, p.howo_mul, p.howo_shift);
        const int rem = pp - b * (p.Ho * p.Wo);
        const int ho = (int)fdiv((unsigned)rem, p.wo_mul, p.wo_shift);
        const int wo = rem - ho * p.Wo;
        const int h0 = ho * p.sh - p.ph, w0 = wo * p.sw - p.pw;
        hi0[it] = pp < p.P ? h0 : -(1 << 28);   // a pixel that does not exist has every tap outside the image
        wi0[it] = w0;
        base[it] = (unsigned)(((b * p.H + h0) * p.W + w0) * p.Cin + g * 4) * 4u;   // (wraps at borders, used with valid taps only)
    }
    int kh, kw, ci0;   // the chunk that the next fetch brings in
    {
        const int tap = (int)fdiv((unsigned)c_begin, p.ncpt_mul, p.ncpt_shift);
        ci0 = (c_begin - tap * p.ncpt) * CK;
        kh = (int)fdiv((unsigned)tap, p.kw_mul, p.kw_shift);
        kw = tap - kh * p.Kw;
    }
    auto retap = [&]() {
        const int dhh = kh * p.dh, dww = kw * p.dw;
        const unsigned tapoff = (unsigned)((dhh * p.W + dww) * p.Cin) * 4u;
#pragma unroll
        for (int it = 0; it < NIT; ++it) {
            const int hi = hi0[it] + dhh, wi = wi0[it] + dww;
            const bool inb = ((unsigned)hi < (unsigned)p.H) & ((unsigned)wi < (unsigned)p.W);
            voff[it] = inb ? base[it] + tapoff : kOOB;
        }
    };
    retap();

    unsigned woff[NJ], roff[NJ];   // this lane's weights and columns of the chunk that the next fetch brings in
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int rb = rb0 + jj < p.n_rowblocks ? rb0 + jj : p.n_rowblocks - 1;   // (one beyond the last is not stored)
        woff[jj] = ((unsigned)(rb * p.nchunks + c_begin) * 64 + (unsigned)lane) * (SPC * 4);
        roff[jj] = ((fdiv((unsigned)rb, p.rbpt_mul, p.rbpt_shift) * p.nchunks + (unsigned)c_begin) * 4 + (unsigned)q) * SPC;
    }
    struct Regs {
        f4 x[NIT];
        unsigned w[NJ][SPC], col[NJ][(SPC + 3) / 4];
    };
    // The loads of chunk c; beyond the wavefront's last they are out of range, which costs no memory and keeps the
    // loop free of a branch that the waits of both its sides would meet behind.
    auto fetch = [&](Regs& r, int c) {
        const bool live = c < c_end;
#pragma unroll
        for (int it = 0; it < NIT; ++it)   // (channels beyond the tap's last are not asked for)
            r.x[it] = buf_load4(xr, (live & (ci0 + g * 4 < p.Cin)) ? voff[it] + (unsigned)(ci0 * 4) : kOOB, 0, (const float*)nullptr);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            load_words<SPC>(r.w[jj], wr, live ? woff[jj] : kOOB, 0);
            const unsigned at = live ? roff[jj] : kOOB;
            if constexpr (SPC == 2) r.col[jj][0] = __builtin_amdgcn_raw_buffer_load_b16(rr, at, 0, 0);
            else load_words<SPC / 4>(r.col[jj], rr, at, 0);
            woff[jj] += 64 * SPC * 4;
            roff[jj] += 4 * SPC;
        }
        ci0 += CK;
        if (ci0 >= p.Cin) {
            ci0 = 0;
            if (++kw == p.Kw) { kw = 0; ++kh; }
            retap();
        }
    };
    auto contract = [&](const Regs& r) {
        __builtin_amdgcn_wave_barrier();
#pragma unroll
        for (int it = 0; it < NIT; ++it)
            *reinterpret_cast<f4*>(strip + (pl0 + it * PPL) * ROW + 16 + g * 16) = r.x[it];
        // the wavefront reads what its own lanes wrote: LDS operations of one wavefront run in order
        __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront");
        __builtin_amdgcn_wave_barrier();
        float v[SPC][NJ][PB];
#pragma unroll
        for (int s = 0; s < SPC; ++s)
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                const unsigned at = (unsigned)(n * ROW) + ((r.col[jj][s / 4] >> (8 * (s % 4)) & 0xffu) << 2);
#pragma unroll
                for (int b = 0; b < PB; ++b) v[s][jj][b] = *reinterpret_cast<const float*>(strip + at + b * 16 * ROW);
            }
        __builtin_amdgcn_sched_barrier(0);   // (all reads on their way before the first is waited for)
#pragma unroll
        for (int s = 0; s < SPC; ++s)
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
                for (int b = 0; b < PB; ++b)
                    acc[b][jj] = __builtin_amdgcn_mfma_f32_16x16x4f32(__uint_as_float(r.w[jj][s]), v[s][jj][b], acc[b][jj], 0, 0, 0);
    };
    Regs r0, r1;
    int c = c_begin;
    fetch(r0, c);
    fetch(r1, ++c);

    // Outputs are dealt out one by one, channels fastest; the first two of a thread have their bias and residual
    // asked for now, so that the end of the kernel waits for no memory.
    const int nthreads = p.waves * 64;
    auto output = [&](int e, int* co, unsigned* off) {   // whether output e of the tile exists, its channel and place
        const int ch = e % (16 * NJ), pp = p0 + e / (16 * NJ);
        const int rb = rb0 + (ch >> 4), j = (int)fdiv((unsigned)rb, p.rbpt_mul, p.rbpt_shift), rit = (rb - j * p.rbpt) * 16 + (ch & 15);
        *co = j * p.tile + rit;
        *off = (unsigned)pp * (unsigned)p.Cout + (unsigned)*co;
        return e < PB * NJ * 256 && pp < p.P && rb < p.n_rowblocks && rit < p.tile && *co < p.Cout;
    };
    const float* const res = reinterpret_cast<const float*>(p.res);
    float add_b[2] = {0.f, 0.f}, add_r[2] = {0.f, 0.f};
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int co;
        unsigned off;
        if (output(tid + i * nthreads, &co, &off)) {
            if (p.bias) add_b[i] = p.bias[co];
            if (res) add_r[i] = res[off];
        }
    }

    // The loads of the next chunk are in flight while one is contracted.  (One exit: with a break after each chunk
    // the compiler kept the second set of weights of the eight-step form in registers that it used for something else.)
    for (int left = c_end - c_begin; left > 0; left -= 2) {
        contract(r0);
        fetch(r0, ++c);
        if (left > 1) contract(r1);
        fetch(r1, ++c);
    }

    // the wavefronts' sums meet in LDS; lane quarters 80 floats apart, so that 16 channels x 4 pixels read different banks
    constexpr int PIECE = kWavePiece / 4, WAVE = PB * NJ * PIECE;
    float* const red = reinterpret_cast<float*>(ldsc);
    __syncthreads();
#pragma unroll
    for (int b = 0; b < PB; ++b)
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
            *reinterpret_cast<f4*>(red + wave * WAVE + (b * NJ + jj) * PIECE + q * 80 + n * 4) = acc[b][jj];
    __syncthreads();
    const int nw = p.waves;
    float* const y = reinterpret_cast<float*>(p.y);
    auto sum_and_store = [&](int e, int co, unsigned off, float bias, float r) {
        const int ch = e % (16 * NJ), px = e / (16 * NJ);
        const float* const src = red + ((px >> 4) * NJ + (ch >> 4)) * PIECE + (ch >> 2 & 3) * 80 + (px & 15) * 4 + (ch & 3);
        float sum = 0.f;
#pragma unroll 8
        for (int w = 0; w < nw; ++w) sum += src[w * WAVE];
        const float v = (sum + bias) + r;
        y[off] = p.relu ? relu1(v) : v;
    };
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        int co;
        unsigned off;
        if (output(tid + i * nthreads, &co, &off)) sum_and_store(tid + i * nthreads, co, off, add_b[i], add_r[i]);
    }
    for (int e = tid + 2 * nthreads; e < PB * NJ * 256; e += nthreads) {
        int co;
        unsigned off;
        if (output(e, &co, &off)) sum_and_store(e, co, off, p.bias ? p.bias[co] : 0.f, res ? res[off] : 0.f);
    }
}

template <int PB, int NJ, int CK, int SPC, int NW>
int launch_wave_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_wave_kernel<PB, NJ, CK, SPC, NW>;
    {
        static unsigned long long done = 0;
        const int rc = allow_lds(reinterpret_cast<const void*>(kern), (size_t)wave_lds_bytes(PB, NJ, CK, NW), &done);
        if (rc != NM_OK) return rc;
    }
    hipLaunchKernelGGL(kern, dim3(p.n_wg), dim3(64 * p.waves), wave_lds_bytes(PB, NJ, CK, p.waves), s, p);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
