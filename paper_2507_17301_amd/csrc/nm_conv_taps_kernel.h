// bf16 k x k convolution that stages the input of a pixel tile once for all its taps.
//
// Contraction and operand tables are those of nm_conv_sp16_kernel (sparse matrix instruction on dense
// activations, or the dense one on zero-filled weights; 64-channel k-steps, weights and index words straight into
// registers).  That kernel stages every tap's strip anew, with a barrier per tap after which its wavefronts start
// reading from nothing.  Where the output is as large as the input (stride 1, 2 pad = dilation (k - 1)) a stage can
// hold 64 channels of the tile's pixels and of what its taps reach around them, and serve all taps: the image lies in LDS
// with zeros for `pw` pixels after every row and `ph` zero rows after every image (the padding on either side of
// them), so tap (kh, kw) is the same distance, kh dh rows and kw dw pixels, from every output pixel.  The strip
// reads of a contracting wavefront then run on from tap to tap, and so do its weights, two chunks ahead.
//
// A pixel is nine granules, eight of channels and one of padding, and the zeros after a row are a multiple of 128 bytes:
// the strip reads of eight consecutive output pixels then fall on eight different granules modulo 128 bytes, also where
// a row ends between them.
//
// The sums run over all taps of 64 channels, then the next 64, where that kernel's run over all channels of a tap: beyond 64
// input channels the last bits differ, by as much as between that kernel and the gather kernel (1 output in 10^4 is not the
// bf16 number nearest to the exact one either way; logits of ResNet-50 x1.0005 +- 0.0015 as far from float64, of ResNet-101
// x0.9998 +- 0.0019).
//
// What bounds it: a contracting wavefront has a SIMD to itself (but for one, which shares its with the wavefront that fetches),
// so the chunks run at the rate of its instruction issue.  On
// 28x28 128 -> 128 at batch 64 (196 or 224 workgroups, one round) of 16.0 us 2.7 are the launch, 3.5 the first stage and
// the output tile, 2.7 its stores and 4.4 the matrix instructions; without the loads of the weights it takes 15.0, without
// the strip reads 15.3.  Steps on the way: requests dealt out behind single matrix instructions and not behind four 17.3 ->
// 16.2, the offsets of a stage's loads worked out once and kept in LDS 21.9 -> 17.4.  Against the strip-per-tap form, cold
// tensors, batch 64: 28x28 128 -> 128 18.9 -> 16.5 us, 56x56 64 -> 64 27.5 -> 24.6; batch 256, T = 32: 14x14 256 -> 256 2:8
// 47.3 -> 41.6, 56x56 64 -> 64 1:4 84.9 -> 78.7, 7x7 512 -> 512 4:8 (dense instruction) 56.2 -> 53.7; larger layers more, 32x8
// 576 -> 256 at batch 112 60.6 -> 38.7.  Few pixels (14x14 256 at batch 64: 196 tiles of 128 x 128, whose weights are as many
// bytes as the strip) stay with the other.
//
// Four wavefronts contract; a fifth fills the other stage meanwhile.  (One is enough for a stage every nine taps.  Of the
// smallest form, 64 x 128 on 104 registers, two workgroups fit a CU; the others take 172 to 230 and have it to themselves.)
// Or eight contract, two a SIMD, so that one issues while the other's matrix instruction runs, on twice the channels (or half
// of each wavefront's), and each requests an eighth of the next stage as it leaves the last one, which costs it a register
// per request and no wavefront that registers would have to be left for.  One tile of 224 x 256 replaces two of 224 x 128 and
// stages its input once.  Batch 256, T = 32, out of cache: 14x14 256 -> 256 2:8 38.2 -> 31.8 us (224 workgroups in one round for
// 448 in two), 7x7 512 -> 512 4:8 (dense, 224 x 128) 50.9 -> 48.2.  Of 34.5 us (another card) 31.4 are left without the loads of
// the weights, 32.5 without the strip reads, 29.1 without either: 13.4 of matrix instructions and what one round cannot hide,
// the launch, the first stage and the output.  A longer ring of strip reads (4 to 6 blocks) gains nothing.
#pragma once

#include "nm_conv_sp16_kernel.h"

namespace nm {

// four contracting wavefronts and the one that fetches, or eight that do both
constexpr int taps_threads(int NW) { return NW == 4 ? 320 : 512; }

// keeps what is computed from (into) these scalars behind (before) this place
template <typename... T> __device__ inline __attribute__((always_inline)) void taps_pin(T&... v)
{
    ((v = (T)__builtin_amdgcn_readfirstlane((int)v)), ...);
}

// n steps, step i as step(i % U) with a constant argument
template <int N> struct TapsInt {
    __device__ constexpr operator int() const { return N; }
};
template <int U, int I = 0, typename F> __device__ inline __attribute__((always_inline)) bool taps_round(int& left, F& step)
{
    if constexpr (I < U) {
        step(TapsInt<I>{});
        if (--left == 0) return true;
        return taps_round<U, I + 1>(left, step);
    }
    return false;
}
template <int U, typename F> __device__ inline __attribute__((always_inline)) void taps_run(int n, F& step)
{
    while (!taps_round<U>(n, step)) {}
}

template <int NBLK, int WP, int NJ, bool SPARSE, int NW>
__global__ __launch_bounds__(taps_threads(NW), NW == 4 && NBLK * NJ <= 16 ? 3 : 2) void nm_conv_taps_kernel(const ConvParams p)
{
    static_assert((NW == 4 || NW == 8) && NW % WP == 0, "contracting wavefronts");
    constexpr bool WIDE = NW == 8;
    constexpr int BPW = 16 * NBLK;
    constexpr int BP = BPW * WP;
    constexpr int WC = NW / WP;
    constexpr int AH = SPARSE ? 1 : 2;           // 16-byte A operands per k-step and row block
    constexpr int WGC = WC * NJ * 16;            // output channels of the workgroup

    extern __shared__ __attribute__((aligned(16))) char lds8[];   // [stages][granules], the loads' offsets

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);   // (of five: 4 is the producer)
    const int q = lane >> 4;
    const int n = lane & 15;

    const int bid = blockIdx.x;
    const int logical = (bid & 7) * p.wg_per_xcd + (bid >> 3);
    if (logical >= p.n_wg) return;
    const int cblock = logical % p.n_cblocks;
    const int ptile = logical / p.n_cblocks;
    const int p0 = ptile * BP;
    const int Lg = taps_line(p.W, p.pw);         // granules of an image row and the zeros after it
    const int Hp = p.H + p.ph;                   // rows of an image and the zeros after it

    const __amdgpu_buffer_rsrc_t xr = make_rsrc(p.x, p.x_bytes);
    const __amdgpu_buffer_rsrc_t wr = make_rsrc(p.wfrag, p.wfrag_bytes);
    const __amdgpu_buffer_rsrc_t rr = make_rsrc(p.rows, p.rows_bytes);

    // place of an output pixel among the padded rows, in granules
    auto place = [&](unsigned pp) {
        const unsigned img = fdiv(pp, p.howo_mul, p.howo_shift);
        const unsigned rem = pp - img * (unsigned)(p.H * p.W);
        const unsigned ho = fdiv(rem, p.wo_mul, p.wo_shift);
        return (int)((img * Hp + ho) * Lg + (rem - ho * p.W) * 9);
    };
    const int at0 = place((unsigned)p0);

    // ---- staging: wave-wide loads of 64 consecutive granules ----
    const int nload = taps_loads(p.rows_n);
    // (one padded image is added so that what lies before the first image is not negative)
    const unsigned t0 = (unsigned)(at0 - (p.ph * Lg + p.pw * 9) + Hp * Lg + lane);
    auto offset = [&](int i) {                   // byte offset of this lane's granule of load i, channels 0 .. 63
        const TapsSource s = taps_source(t0 + (unsigned)(i * 64), Lg, p.padw_mul, p.padw_shift, p.padh_mul, p.padh_shift, p.B, p.H, p.W, p.ph);
        return s.pixel >= 0 ? (taps_mul((unsigned)s.pixel, (unsigned)p.Cin) + s.oct * 8) * 2 : kOOB;
    };
    auto fetch = [&](int i, unsigned off, int cc) {
        char* dst = lds8 + (cc & 1) * p.rows_lds + i * 1024;
        __builtin_amdgcn_raw_ptr_buffer_load_lds(xr, (lds_ptr_t)dst, 16, off, cc * 128, 0, 0);
    };
    // Eight wavefronts: each issues every eighth load of every stage, whose offsets it keeps.
    unsigned woff[WIDE ? kTapsWideLoads : 1];
    auto fetch_own = [&](int cc) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < (WIDE ? kTapsWideLoads : 1); ++k)
            if (wave + 8 * k < nload) fetch(wave + 8 * k, woff[k], cc);
    };
    if constexpr (WIDE) {
#pragma unroll
        for (int k0 = 0; k0 < kTapsWideLoads; k0 += 4) {
            if (wave + 8 * k0 >= nload) break;
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k) woff[k] = offset(min(wave + 8 * k, nload - 1));
#pragma unroll
            for (int k = k0; k < k0 + 4; ++k)
                if (wave + 8 * k < nload) fetch(wave + 8 * k, woff[k], 0);
        }
    } else {
        // The first stage is fetched by all five wavefronts, four loads at a time so that their address arithmetic overlaps
        // (past the last load it is repeated); the offsets are left in LDS for the stages that follow, which the producer fetches
        unsigned* const offs = reinterpret_cast<unsigned*>(lds8 + (p.ncpt > 1 ? 2 : 1) * p.rows_lds) + lane;
        for (int i0 = wave; i0 < nload; i0 += 20) {
            unsigned off[4];
#pragma unroll
            for (int k = 0; k < 4; ++k) off[k] = offset(min(i0 + 5 * k, nload - 1));
#pragma unroll
            for (int k = 0; k < 4; ++k) {
                const int i = min(i0 + 5 * k, nload - 1);
                fetch(i, off[k], 0);
                if (p.ncpt > 1) offs[i * 64] = off[k];
            }
        }

        if (wave == 4) {
            for (int cc = 0; cc < p.ncpt; ++cc) {
                asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // stage cc is there
                if (cc > 0) asm volatile("s_barrier" ::: "memory");                        // stage cc - 1 has been read
                if (cc + 1 == p.ncpt) break;
                for (int i0 = 0; i0 < nload; i0 += 8) {
                    unsigned off[8];
#pragma unroll
                    for (int k = 0; k < 8; ++k) off[k] = offs[min(i0 + k, nload - 1) * 64];
#pragma unroll
                    for (int k = 0; k < 8; ++k) fetch(min(i0 + k, nload - 1), off[k], cc + 1);
                }
            }
            // the barriers of the epilogue
            __syncthreads();
            if (p.res) __syncthreads();
            __syncthreads();
            return;
        }
    }

    const int wpx = wave % WP, wcx = wave / WP;
    const int rb0 = (cblock * WC + wcx) * NJ;
    const int wpix = wpx * BPW;

    // ---- operand streams: [row block][chunk][AH][lane] x 16 bytes, index words [column tile][chunk][lane group];
    // chunk c of the tables is tap c / ncpt, channels 64 (c % ncpt) and up, here the taps of a stage come first ----
    // The index words of up to four row blocks come in one load, lane n taking those of row block n % 4, and are handed
    // round inside the quad.
    const unsigned wvoff = (unsigned)lane * 16;
    unsigned wsoff[NJ];
    static_assert(NJ == 1 || NJ == 2 || NJ == 4, "a quad of lanes holds the index words");
    unsigned ivoff;
    {
        int rb = rb0 + (n & 3);
        if (rb >= p.n_rowblocks) rb = p.n_rowblocks - 1;
        ivoff = (unsigned)(rb / p.rbpt) * p.nchunks * 16u + (unsigned)q * 4;
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        int rb = rb0 + jj;
        if (rb >= p.n_rowblocks) rb = p.n_rowblocks - 1;
        wsoff[jj] = (unsigned)rb * p.nchunks * (AH * 1024u);
    }
    constexpr int NSET = SPARSE ? 3 : 2;         // (a chunk takes the dense instruction twice as long)
    struct Ops {
        u4v a[NJ][AH];
        unsigned idx;
    };
    Ops ops[NSET];
    auto load_ops = [&](Ops& o, int jj, int c) {
#pragma unroll
        for (int h = 0; h < AH; ++h)
            o.a[jj][h] = __builtin_amdgcn_raw_buffer_load_b128(wr, wvoff + h * 1024, wsoff[jj] + (unsigned)c * (AH * 1024u), 0);
        if constexpr (SPARSE)
            if (jj == 0) o.idx = __builtin_amdgcn_raw_buffer_load_b32(rr, ivoff, (unsigned)c * 16u, 0);
    };
    // chunk number of the operands to load next; past the end it stays on the last
    const int ntaps = p.Kh * p.Kw;
    int f_tap = 0, f_cc = 0, f_chunk = 0;
    auto advance = [&]() {
        ++f_tap;
        f_chunk += p.ncpt;
        if (__builtin_expect(f_tap == ntaps, 0)) {
            const bool end = f_cc + 1 == p.ncpt;
            f_chunk = end ? f_chunk - p.ncpt : f_cc + 1;
            f_tap = end ? ntaps - 1 : 0;
            f_cc = end ? f_cc : f_cc + 1;
        }
    };
#pragma unroll
    for (int s = 0; s + 1 < NSET; ++s) {
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) load_ops(ops[s], jj, f_chunk);
        advance();
    }

    // the accumulators start from the bias
    f4 acc[NJ][NBLK];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int co = (rb0 + jj) * 16 + q * 4;  // (T is a multiple of 16 here: row blocks are 16 consecutive channels)
        f4 b4 = f4{0.f, 0.f, 0.f, 0.f};
        if (p.bias && co < p.Cout) b4 = *reinterpret_cast<const f4*>(p.bias + co);
#pragma unroll
        for (int b = 0; b < NBLK; ++b) acc[jj][b] = b4;
    }

    // LDS address of this lane's operand of each pixel block at tap (0, 0)
    const unsigned lds0 = (unsigned)(uintptr_t)(__attribute__((address_space(3))) char*)lds8;
    unsigned base[NBLK];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int pp = p0 + wpix + b * 16 + n;   // (a pixel past the end reads as the last one, and is not stored)
        base[b] = lds0 + (unsigned)((place((unsigned)(pp < p.P ? pp : p.P - 1)) - at0) * 16 + q * 32);
    }

    // The strip reads run RD - 1 pixel blocks ahead, through the taps and from one stage into the next; inline assembly
    // with hand-placed waits, as in nm_conv_sp16_kernel.
    constexpr int RD = NBLK % 4 == 0 ? 4 : 3;
    u4v ring[RD][2];
    auto read_lo = [&](unsigned addr, u4v (&dst)[2]) {
        asm volatile("ds_read_b128 %0, %1" : "=v"(dst[0]) : "v"(addr) : "memory");
    };
    auto read_hi = [&](unsigned addr, u4v (&dst)[2]) {
        asm volatile("ds_read_b128 %0, %1 offset:16" : "=v"(dst[1]) : "v"(addr) : "memory");
    };
    // Distances from `base` of the chunk being contracted and of the next (at the very end: of the first tap again), and
    // whether that one begins a stage
    const unsigned kw_step = (unsigned)(p.dw * 144), kh_step = (unsigned)(p.dh * Lg * 16) - (unsigned)p.Kw * kw_step;
    unsigned here = 0, there = 0;
    int g_kw = 0, g_tap = 0, g_cc = 0;
    int cross = 0;
    auto follow = [&]() {                        // moves `there` on
        there += kw_step;
        const bool wrap = ++g_kw == p.Kw;
        there += wrap ? kh_step : 0u;
        g_kw = wrap ? 0 : g_kw;
        cross = 0;
        if (__builtin_expect(++g_tap == ntaps, 0)) {
            cross = g_cc + 1 < p.ncpt ? 1 : 0;
            g_cc += cross;
            g_tap = 0;
            there = (g_cc & 1) * (unsigned)p.rows_lds;
        }
    };
    follow();
    int idx[NJ];
    auto spread = [&](unsigned v) {              // quad_perm: lane jj of each four to all of them
        if constexpr (SPARSE) {
            idx[0] = __builtin_amdgcn_update_dpp(0, (int)v, 0x00, 0xf, 0xf, true);
            if constexpr (NJ > 1) idx[1] = __builtin_amdgcn_update_dpp(0, (int)v, 0x55, 0xf, 0xf, true);
            if constexpr (NJ > 2) idx[2] = __builtin_amdgcn_update_dpp(0, (int)v, 0xaa, 0xf, 0xf, true);
            if constexpr (NJ > 2) idx[NJ - 1] = __builtin_amdgcn_update_dpp(0, (int)v, 0xff, 0xf, 0xf, true);
        }
    };
    // One chunk.  A wavefront has its SIMD to itself, and what it issues between two matrix instructions is free only up to
    // the 12 clocks that the first leaves: requests, addresses and counters are dealt out one by one, the counters of the
    // next chunk in the middle of this one.
    auto step = [&](auto U) {
        constexpr int u = U;
        const Ops& now = ops[u % NSET];
        Ops& nxt = ops[(u + NSET - 1) % NSET];
        const int stage = cross;
        const unsigned next = there;
        const int fc = f_chunk;
        // the next stage is there (of these eight: all but the last chunk's loads of weights are older than that)
        if (__builtin_expect(stage, 0)) {
            if constexpr (WIDE) NM_WAIT_VMCNT(NJ * AH + (SPARSE ? 1 : 0));
            asm volatile("s_barrier" ::: "memory");
        }
#pragma unroll
        for (int b = 0; b < NBLK; ++b) {
            constexpr int first = (u * NBLK) % RD;
            const int nb = b + RD - 1;
            const unsigned addr = base[nb % NBLK] + (nb < NBLK ? here : next);
            u4v(&bo)[2] = ring[(first + b) % RD];
            asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(bo[0]), "+v"(bo[1]) : "n"(2 * (RD - 2)));
#pragma unroll
            for (int jj = 0; jj < NJ; ++jj) {
                if constexpr (SPARSE) {
                    const bf16x bv = __builtin_shufflevector(__builtin_bit_cast(bf8x, bo[0]), __builtin_bit_cast(bf8x, bo[1]),
                                                             0, 1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
                    acc[jj][b] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(__builtin_bit_cast(bf8x, now.a[jj][0]), bv, acc[jj][b],
                                                                           idx[jj], 0, 0);
                } else {
#pragma unroll
                    for (int h = 0; h < 2; ++h)
                        acc[jj][b] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(__builtin_bit_cast(bf8x, now.a[jj][h]),
                                                                             __builtin_bit_cast(bf8x, bo[h]), acc[jj][b], 0, 0, 0);
                }
                __builtin_amdgcn_sched_barrier(0);
                if (jj == 0) read_lo(addr, ring[(first + nb) % RD]);
                if (jj == (NJ > 1 ? 1 : 0)) read_hi(addr, ring[(first + nb) % RD]);
                if (jj == (NJ > 2 ? 2 : NJ - 1)) {
#pragma unroll
                    for (int j2 = 0; j2 < NJ; ++j2)
                        if (j2 * NBLK / NJ == b) load_ops(nxt, j2, fc);
                }
                if (jj == NJ - 1) {
                    if (b == (NBLK > 3 ? NBLK - 3 : 0)) {
                        taps_pin(f_chunk, f_tap, f_cc);   // (keeps the arithmetic here)
                        advance();
                        taps_pin(f_chunk, f_tap, f_cc);
                    }
                    if (b == (NBLK > 2 ? NBLK - 2 : 0)) {
                        taps_pin(there, g_kw, g_tap, g_cc);
                        follow();
                        taps_pin(there, g_kw, g_tap, g_cc, cross);
                    }
                }
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        if (__builtin_expect(stage, 0)) {
            asm volatile("s_barrier" ::: "memory");   // the last stage has been read
            if constexpr (WIDE) {
                if (g_cc + 1 < p.ncpt) fetch_own(g_cc + 1);
                __builtin_amdgcn_sched_barrier(0);
            }
        }
        here = next;
        spread(ops[(u + 1) % NSET].idx);
    };
    asm volatile("s_waitcnt vmcnt(0) lgkmcnt(0)\n\ts_barrier" ::: "memory");   // the first stage and the offsets are there
    if constexpr (WIDE) {
        if (p.ncpt > 1) fetch_own(1);
        __builtin_amdgcn_sched_barrier(0);
    }
#pragma unroll
    for (int b = 0; b < RD - 1; ++b) {
        read_lo(base[b], ring[b]);
        read_hi(base[b], ring[b]);
    }
    spread(ops[0].idx);
    taps_run<NSET * (NBLK % RD == 0 ? 1 : NSET == RD ? 1 : RD)>(p.nchunks, step);
#pragma unroll
    for (int i = 0; i < RD; ++i) asm volatile("s_waitcnt lgkmcnt(0)" : "+v"(ring[i][0]), "+v"(ring[i][1]) : : "memory");   // reads ahead of the end

    // ---- epilogue: whole 128-byte lines through an LDS tile, once every wavefront is past its last strip read ------
    constexpr int PITCH = tile_pitch<bf16_t>(WGC);
    ResTile<bf16_t, BP, WGC, 64 * NW> rt;
    if (p.res) rt.load(p, tid, p0, cblock * WGC);
    __syncthreads();
    if (p.res) {
        rt.put(lds8, tid);
        __syncthreads();
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
            tile_put4_lds<bf16_t>(p, lds8 + (wpix + b * 16 + n) * PITCH + ((wcx * NJ + jj) * 16 + q * 4) * 2, acc[jj][b]);
    __syncthreads();
    tile_flush<bf16_t, BP, WGC, 64 * NW>(p, lds8, p0, cblock * WGC);
}

template <int NBLK, int WP, int NJ, bool SPARSE, int NW>
int launch_taps_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_taps_kernel<NBLK, WP, NJ, SPARSE, NW>;
    constexpr size_t most = 160 * 1024;
    static unsigned long long done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(kern), most, &done);
    if (rc != NM_OK) return rc;
    const size_t lds = taps_lds_bytes(NBLK, WP, NJ, p.rows_n, p.ncpt, NW);
    if (lds > most || p.tile % 16 != 0 || p.Cout % 8 != 0 || p.Cin % 64 != 0 || p.sh != 1 || p.sw != 1 || p.Ho != p.H ||
        p.Wo != p.W || (NW == 8 && taps_loads(p.rows_n) > 8 * kTapsWideLoads)) {
        set_error("internal: a layer that the tap-staged kernel does not do");
        return NM_ERR_UNSUPPORTED;
    }
    hipLaunchKernelGGL(kern, dim3(p.wg_per_xcd * 8), dim3(taps_threads(NW)), lds, s, p);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
