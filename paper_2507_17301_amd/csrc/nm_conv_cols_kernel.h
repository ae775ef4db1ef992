// bf16 1x1 convolution with few input channels and many output channels: a workgroup keeps its pixels' whole input and walks
// the output channels, 256 at a time.
//
// Contraction and operand tables are those of nm_conv_sp16_kernel (sparse matrix instruction, 64-channel k-steps).  Such a
// layer is memory traffic, output and residual above all, and a workgroup per output tile loads, contracts, loads the residual
// and stores one after the other, a round trip to memory each.  Here the four wavefronts load up to 256 channels of 16 NBLK pixels
// into LDS once, and from then on each runs by itself, without a barrier, over row blocks of its own.  While it contracts
// for 64 output channels, the weights and the bias of its next 64 are requested into the registers that it has just read for
// the last time, and the residual into those that it has just emptied into LDS: all of it before its stores, since the
// memory counter counts in order, and a load behind a store is a load that waits for the store.
//
// What bounds it: memory, and the start and end of a launch.  14x14 256 -> 1024 with a residual, out of cache, against the fastest
// of the others and the one that untuned calls took: batch 64 16.2 us, 17.8 and 23.7; batch 256 (231 MB) 60.4, 63.0 and 74 to
// 78.  28x28 128 -> 512 at batch 256 (463 MB) 89.6, 90.2 and 95.3; up to 256 output channels there is nothing to walk, x1.2 to
// x1.5.  Beginning the walk of neighbouring tiles at different groups: 61.4 for 60.4, 94 for 90.  Without requests past the last group
// of a walk (another card, before and after): 14x14 at batch 64, 128 and 256 15.7 and 15.5, 34.5 and 33.7, 60.5 and 59.1, 28x28 at 256
// 88.4 and 86.7.
#pragma once

#include "nm_conv_sp16_kernel.h"

namespace nm {

template <int NBLK, int NCH>
__global__ __launch_bounds__(256, 2) void nm_conv_cols_kernel(const ConvParams p)
{
    constexpr int BP = 16 * NBLK;
    constexpr int NJ = 4;                        // row blocks of a wavefront: whole 128-byte lines of output
    constexpr int NIT = BP / 32;                 // wave-wide loads per wavefront and 64 channels
    constexpr int NP = BP / 8;                   // passes of 8 rows over the output piece
    static_assert(BP % 32 == 0, "four wavefronts share the loads of a chunk evenly");

    extern __shared__ __attribute__((aligned(16))) char lds8[];   // [chunk][pixel][64 channels], then a piece per wavefront

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    const int n = lane & 15;

    const int bid = blockIdx.x;
    const int logical = (bid & 7) * p.wg_per_xcd + (bid >> 3);
    if (logical >= p.n_wg) return;
    const int parts = (p.n_cblocks + p.cps - 1) / p.cps;       // workgroups that share a pixel tile
    const int p0 = logical / parts * BP;
    const int first = logical % parts * p.cps;
    const int end = first + p.cps < p.n_cblocks ? first + p.cps : p.n_cblocks;

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, p.x_bytes);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wfrag, p.wfrag_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.rows, p.rows_bytes);

    // ---- the input: load i of a chunk brings granules 64 i .. 64 i + 63, swizzled as in nm_conv_sp16_kernel --------------
    unsigned xoff[NIT];
#pragma unroll
    for (int it = 0; it < NIT; ++it) {
        const int G = (wave + 4 * it) * 64 + lane;
        const int pl = G / 8, oct = (G % 8) ^ sp16_swz(pl, 128);
        const int pp = p0 + pl;
        const int b = (int)fdiv((unsigned)pp, p.howo_mul, p.howo_shift);
        const int rem = pp - b * (p.Ho * p.Wo);
        const int ho = (int)fdiv((unsigned)rem, p.wo_mul, p.wo_shift);
        const int wo = rem - ho * p.Wo;
        xoff[it] = pp < p.P ? (unsigned)(((b * p.H + ho * p.sh) * p.W + wo * p.sw) * p.Cin + oct * 8) * 2u : kOOB;
    }
    auto fetch = [&](char* dst, unsigned off, int c) { __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr_t)dst, 16, off, c * 128, 0, 0); };
#pragma unroll
    for (int c = 0; c < NCH; ++c)
#pragma unroll
        for (int it = 0; it < NIT; ++it) fetch(lds8 + c * (BP * 128) + (wave + 4 * it) * 1024, xoff[it], c);

    // ---- operands of row blocks rb .. rb + 3 (beyond the last one: of the last one, computed and not stored) -------------
    // [row block][chunk][lane] x 16 bytes; index words [column tile][chunk][lane group]: lane n takes those of row block n % 4,
    // which are handed round in the quad
    struct Ops {
        u4v a[NJ];
        unsigned idx;
    };
    Ops ops[NCH];
    f4 bb[NJ];
    u4v rv[NP];
    auto index_words = [&](int rb) {             // offset of those of this lane, chunk 0
        int at = rb + (n & 3);
        if (at >= p.n_rowblocks) at = p.n_rowblocks - 1;
        return fdiv((unsigned)at, p.rbpt_mul, p.rbpt_shift) * (NCH * 16u) + (unsigned)q * 4u;
    };
    auto load_ops = [&](Ops& o, int rb, unsigned mine, unsigned words, int c) {
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            const int at = rb + jj < p.n_rowblocks ? rb + jj : p.n_rowblocks - 1;
            o.a[jj] = __builtin_amdgcn_raw_buffer_load_b128(wr, mine, (unsigned)(at * NCH + c) * 1024u, 0);
        }
        o.idx = __builtin_amdgcn_raw_buffer_load_b32(rr, words, (unsigned)c * 16u, 0);
    };
    auto load_bias = [&](int rb) {
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) {
            const int co = (rb + jj) * 16 + q * 4;   // (T is a multiple of 16 here: row blocks are 16 consecutive channels)
            bb[jj] = f4{0.f, 0.f, 0.f, 0.f};
            if (p.bias && co < p.Cout) bb[jj] = *reinterpret_cast<const f4*>(p.bias + co);
        }
    };
    // a wavefront's piece of the output and the residual: 128 bytes a pixel, eight lanes a row
    const int r0 = lane >> 3, cg = lane & 7;
    const bf16_t* const res = reinterpret_cast<const bf16_t*>(p.res);
    bf16_t* const y = reinterpret_cast<bf16_t*>(p.y);
    auto load_res = [&](int rb) {
        const int co = rb * 16 + cg * 8;
#pragma unroll
        for (int k = 0; k < NP; ++k) {
            // (a row or column that does not exist reads the first elements of the tensor; its sum is not stored)
            const bool live = p0 + k * 8 + r0 < p.P && co < p.Cout;
            rv[k] = *reinterpret_cast<const u4v*>(res + (live ? (unsigned)(p0 + k * 8 + r0) * (unsigned)p.Cout + (unsigned)co : 0u));
        }
    };
    auto row_block = [&](int it) { return (it * 4 + wave) * NJ; };
    int rb0 = row_block(first);
#pragma unroll
    for (int c = 0; c < NCH; ++c) load_ops(ops[c], rb0, (unsigned)lane * 16u, index_words(rb0), c);
    load_bias(rb0);
    if (res) load_res(rb0);

    unsigned roff[2];                            // this lane's operand of block 0
#pragma unroll
    for (int h = 0; h < 2; ++h) roff[h] = (unsigned)(n * 128 + (((q * 2 + h) ^ sp16_swz(n, 128)) * 16));
    constexpr int PITCH = 128 + 16;
    char* const piece = lds8 + NCH * (BP * 128) + wave * (BP * PITCH);

    NM_WAIT_VMCNT(0);
    __syncthreads();                             // the input is there
    for (int it = first; it < end; ++it) {
        // Past the last group nothing is requested: weights and index words out of range (which costs no memory traffic and keeps the
        // loop in one piece), the residual not at all.  (Its addresses set to one place of the tensor instead: 60.5 -> 67, every
        // workgroup asking for the same line.)
        const bool more = it + 1 < end;
        const int rbn = row_block(more ? it + 1 : it);
        const unsigned mine = more ? (unsigned)lane * 16u : kOOB, words = more ? index_words(rbn) : kOOB;
        f4 acc[NJ][NBLK];
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int b = 0; b < NBLK; ++b) acc[jj][b] = bb[jj];
#pragma unroll
        for (int c = 0; c < NCH; ++c) {
            int idx[NJ];                         // quad_perm: lane jj of each four to all of them
            idx[0] = __builtin_amdgcn_update_dpp(0, (int)ops[c].idx, 0x00, 0xf, 0xf, true);
            idx[1] = __builtin_amdgcn_update_dpp(0, (int)ops[c].idx, 0x55, 0xf, 0xf, true);
            idx[2] = __builtin_amdgcn_update_dpp(0, (int)ops[c].idx, 0xaa, 0xf, 0xf, true);
            idx[3] = __builtin_amdgcn_update_dpp(0, (int)ops[c].idx, 0xff, 0xf, 0xf, true);
#pragma unroll
            for (int b = 0; b < NBLK; ++b) {
                u4v x[2];
#pragma unroll
                for (int h = 0; h < 2; ++h) x[h] = *reinterpret_cast<const u4v*>(lds8 + c * (BP * 128) + b * 2048 + roff[h]);
                const bf16x bv = __builtin_shufflevector(__builtin_bit_cast(bf8x, x[0]), __builtin_bit_cast(bf8x, x[1]), 0, 1, 2, 3, 4, 5, 6,
                                                         7, 8, 9, 10, 11, 12, 13, 14, 15);
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
                    acc[jj][b] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf8x, ops[c].a[jj]), bv, acc[jj][b], idx[jj], 0, 0);
            }
            __builtin_amdgcn_sched_barrier(0);
            load_ops(ops[c], rbn, mine, words, c);
        }
        load_bias(rbn);
        // the output: residual, activation and the one rounding in the wavefront's own piece of LDS, then whole lines
        if (res) {
#pragma unroll
            for (int k = 0; k < NP; ++k) *reinterpret_cast<u4v*>(piece + (k * 8 + r0) * PITCH + cg * 16) = rv[k];
            __builtin_amdgcn_wave_barrier();
            if (more) load_res(rbn);
        }
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int b = 0; b < NBLK; ++b) tile_put4_lds<bf16_t>(p, piece + (b * 16 + n) * PITCH + (jj * 16 + q * 4) * 2, acc[jj][b]);
        __builtin_amdgcn_wave_barrier();
        const int co = rb0 * 16 + cg * 8;
        auto rows = [&](auto stream) {
            u4v v[NP];
#pragma unroll
            for (int k = 0; k < NP; ++k) v[k] = *reinterpret_cast<const u4v*>(piece + (k * 8 + r0) * PITCH + cg * 16);
#pragma unroll
            for (int k = 0; k < NP; ++k)
                if (p0 + k * 8 + r0 < p.P && co < p.Cout)
                    store_out16<decltype(stream)::value>(y + ((unsigned)(p0 + k * 8 + r0) * (unsigned)p.Cout + (unsigned)co), v[k]);
        };
        if (p.stream) rows(std::true_type());
        else rows(std::false_type());
        __builtin_amdgcn_wave_barrier();
        rb0 = rbn;
    }
}

template <int NBLK, int NCH>
int launch_cols_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_cols_kernel<NBLK, NCH>;
    constexpr size_t lds = cols_lds_bytes(NBLK, NCH);
    static_assert(2 * lds <= 160 * 1024, "two workgroups a CU");
    static unsigned long long done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(kern), lds, &done);
    if (rc != NM_OK) return rc;
    if (p.Cin != 64 * NCH || p.Kh != 1 || p.Kw != 1 || p.ph != 0 || p.pw != 0 || p.tile % 16 != 0 || p.Cout % 8 != 0 || p.cps < 1) {
        set_error("internal: a layer that the channel-walking kernel does not do");
        return NM_ERR_UNSUPPORTED;
    }
    hipLaunchKernelGGL(kern, dim3(p.wg_per_xcd * 8), dim3(256), lds, s, p);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
