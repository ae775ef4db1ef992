// fp32 k x k convolution as three bf16 planes, a pixel tile's input staged and cut once for all its taps.
//
// Arithmetic, operand tables and care for what planes cannot carry are those of nm_conv_split_kernel, the layout of a stage
// that of nm_conv_taps_kernel, three times, a plane after the other.  The strip-per-tap form loads, cuts and writes every
// value to LDS once per tap, and its four contracting wavefronts have a SIMD each; here all eight wavefronts contract, two a
// SIMD, and each cuts an eighth of a stage every `ntaps` chunks, from registers that it filled a stage earlier.
//
// The wavefronts are KG groups, which share the staged input and take the chunks (tap, 64 channels) in turn, so that a
// wavefront's own tile is 64 pixels x 16 NJ channels whatever the workgroup's: smaller ones read more from LDS and from the
// cache of the weights than these deliver beside six matrix instructions a block (64 x 64: half of 1536 clocks either).
// The groups' sums are added in the order of the groups, each of them by the group that finishes the block, and chunks that do
// not make a whole round are done by all groups, each on its blocks (nine taps of 64 channels in four groups: 2.25 rounds for 3),
// and added last.
//
// Barriers: all wavefronts have done m chunks each at the same time, whatever group, so both kinds stand at a place m of
// their own.  "Stage w - 2 has been read" at ceil(ntaps (w - 1) / KG), behind which its place may be written for stage w;
// "stage w is there" at floor(ntaps w / KG), just before the first group needs it.  Half of the wavefronts (one of each SIMD)
// cut a chunk earlier than the others where there is room, so that one contracts while the other cuts.
//
// What bounds it: the matrix cores at the clock they hold.  14x14 256 -> 256 at batch 64, out of cache: 49.5 -> 42.0 us where six
// bf16 products take 36.6 at the rate of a large bf16 matrix product on the same card; batch 32 31.8 -> 25.7; 7x7 512 -> 512 52.0
// -> 46.4 (and no K split over workgroups, which it was); 28x28 128 -> 128, half of all channels kept (dense), batch 16 23.4 ->
// 22.5.  Strip operands of the next block requested a block ahead (24 more registers) gain nothing: 48.7 for 48.9 on a slower
// card.  128 pixels x 64 and x 128 channels were first on no layer: with 64 input channels (56x56: 77 for 74 us) a tile is one
// stage, which nothing runs beside.
#pragma once

#include "nm_conv_split_kernel.h"

namespace nm {

template <int NBLK, int WP, int NJ, int KG, bool SPARSE>
__global__ __launch_bounds__(512, 2) void nm_conv_split_taps_kernel(const ConvParams p)
{
    static_assert(NBLK % KG == 0 && 8 % (WP * KG) == 0, "every group finishes whole blocks");
    constexpr int BPW = 16 * NBLK;
    constexpr int BP = BPW * WP;
    constexpr int GW = 8 / KG;                   // wavefronts of a group
    constexpr int WC = GW / WP;
    constexpr int NO = NBLK / KG;                // blocks that a wavefront finishes
    constexpr int AH = SPARSE ? 1 : 2;           // 16-byte weight operands per plane and row block

    extern __shared__ __attribute__((aligned(16))) char lds8[];   // a word per wavefront, the stages [stage][plane][granule]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int q = lane >> 4;
    const int n = lane & 15;
    const int grp = wave / GW, cell = wave % GW;
    const int wpx = cell % WP, wcx = cell / WP;

    const int bid = blockIdx.x;
    const int logical = (bid & 7) * p.wg_per_xcd + (bid >> 3);
    if (logical >= p.n_wg) return;
    const int cblock = logical % p.n_cblocks;
    const int p0 = logical / p.n_cblocks * BP;
    const int rb0 = (cblock * WC + wcx) * NJ;
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

    // ---- staging: granule tid + 512 k of a stage, eight channels of a pixel (or zeros) -----------------------------
    const int plane = p.rows_lds;                // bytes
    const int ngran = plane / 16;                // (a multiple of 64: a wavefront has all of its lanes' granules or none)
    const unsigned t0 = (unsigned)(at0 - (p.ph * Lg + p.pw * 9) + Hp * Lg);   // (one padded image is added: not negative)
    auto offset = [&](int t) __attribute__((always_inline)) {
        const TapsSource s = taps_source(t0 + (unsigned)t, Lg, p.padw_mul, p.padw_shift, p.padh_mul, p.padh_shift, p.B, p.H, p.W, p.ph);
        return s.pixel >= 0 ? (taps_mul((unsigned)s.pixel, (unsigned)p.Cin) + s.oct * 8) * 4 : kOOB;
    };
    unsigned soff[kSplitTapsItems];
    f4 sv[kSplitTapsItems][2];
    unsigned lost = 0u;                          // bits that planes left out so far
    auto fetch = [&](int cc) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kSplitTapsItems; ++k)
#pragma unroll
            for (int h = 0; h < 2; ++h) sv[k][h] = buf_load4(xr, soff[k] + h * 16, (unsigned)cc * 256u, (const float*)nullptr);
    };
    auto stash = [&](int cc, int k0) __attribute__((always_inline)) {
        char* const dst = lds8 + kSplitTapsFlags + (cc & 1) * 3 * plane + tid * 16;
#pragma unroll
        for (int k = 0; k < kSplitTapsItems; ++k) {
            if (tid + (k0 + k) * 512 >= ngran) continue;
            u2v pl[2][3];
            f4 rest[2];
#pragma unroll
            for (int h = 0; h < 2; ++h) {
                split_planes(sv[k][h], pl[h], rest);
                split_lost(rest, lost);
            }
#pragma unroll
            for (int s = 0; s < 3; ++s)
                *reinterpret_cast<u4v*>(dst + s * plane + (k0 + k) * 8192) = u4v{pl[0][s].x, pl[0][s].y, pl[1][s].x, pl[1][s].y};
        }
    };

    // ---- operands: as in nm_conv_split_kernel, chunk c of the tables is tap c / ncpt, channels 64 (c % ncpt) and up -------
    constexpr unsigned WCH = 3 * AH * 1024;      // weight bytes per (row block, chunk)
    const bool fast = p.Cout % 4 == 0;           // output rows come in whole quads
    struct Ops {
        u4v a[NJ][3][AH];
        unsigned idx[NJ];
    };
    auto load_op = [&](Ops& o, int jj, int c) {
        const unsigned at = (unsigned)(rb0 + jj < p.n_rowblocks ? rb0 + jj : p.n_rowblocks - 1) * (unsigned)p.nchunks + (unsigned)c;
#pragma unroll
        for (int pl = 0; pl < 3; ++pl)
#pragma unroll
            for (int h = 0; h < AH; ++h)
                o.a[jj][pl][h] = __builtin_amdgcn_raw_buffer_load_b128(
                    wr, (unsigned)lane * 16u + (unsigned)(pl * AH + h) * 1024u, at * WCH, 0);
        if constexpr (SPARSE) o.idx[jj] = __builtin_amdgcn_raw_buffer_load_b32(rr, (unsigned)lane * 4u, at * 256u, 0);
    };

    // ---- the first stage, up to 512 kSplitTapsItems granules at a time (layers of one stage may have more) -----------------
    auto place_items = [&](int k0) __attribute__((always_inline)) {
#pragma unroll
        for (int k = 0; k < kSplitTapsItems; ++k) {
            const int t = tid + (k0 + k) * 512;
            soff[k] = t < ngran ? offset(t) : kOOB;
        }
    };
    place_items(0);
    fetch(0);
    const int ntaps = p.Kh * p.Kw, total = p.nchunks;
    int tap = grp, cc = 0;                       // of this group's chunk (KG <= ntaps)
    Ops oa, ob;
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) load_op(oa, jj, tap * p.ncpt);

    f4 acc[NJ][NBLK];                            // of group 0 from the bias, where rows come in whole quads
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj) {
        const int co = (rb0 + jj) * 16 + q * 4;
        f4 bb = f4{0.f, 0.f, 0.f, 0.f};
        if (grp == 0 && fast && p.bias && co < p.Cout) bb = *reinterpret_cast<const f4*>(p.bias + co);
#pragma unroll
        for (int b = 0; b < NBLK; ++b) acc[jj][b] = bb;
    }
    // this lane's operand of each pixel block at tap (0, 0) (a pixel past the end reads as the last one, and is not stored)
    unsigned base[NBLK];
#pragma unroll
    for (int b = 0; b < NBLK; ++b) {
        const int pp = p0 + wpx * BPW + b * 16 + n;
        base[b] = (unsigned)(kSplitTapsFlags + (place((unsigned)(pp < p.P ? pp : p.P - 1)) - at0) * 16 + q * 32);
    }

    __builtin_amdgcn_sched_barrier(0);           // (all of this is under way before the first stage is waited for)
    stash(0, 0);
    for (int k0 = kSplitTapsItems; k0 * 512 < ngran; k0 += kSplitTapsItems) {
        place_items(k0);
        fetch(0);
        stash(0, k0);
    }
    if (p.ncpt > 1) fetch(1);

    // products of pixel block b, smallest first; the row blocks take turns, so that no instruction waits for the one before it
    // (added to sum[row block][sb])
    auto products = [&](const Ops& o, unsigned off, int b, auto& sum, int sb, auto&& behind) __attribute__((always_inline)) {
        u4v x[3][2];
#pragma unroll
        for (int pl = 2; pl >= 0; --pl)
#pragma unroll
            for (int h = 0; h < 2; ++h)
                x[pl][h] = *reinterpret_cast<const u4v*>(lds8 + (base[b] + off + (unsigned)(pl * plane)) + h * 16);
        __builtin_amdgcn_sched_barrier(0);
        constexpr int XP[6] = {2, 1, 0, 1, 0, 0}, WPL[6] = {0, 1, 2, 0, 1, 0};
#pragma unroll
        for (int k = 0; k < 6; ++k) {
            if constexpr (SPARSE) {
                const bf16x bv = __builtin_shufflevector(__builtin_bit_cast(bf8x, x[XP[k]][0]),
                                                         __builtin_bit_cast(bf8x, x[XP[k]][1]), 0, 1, 2, 3, 4, 5,
                                                         6, 7, 8, 9, 10, 11, 12, 13, 14, 15);
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
                    sum[jj][sb] = __builtin_amdgcn_smfmac_f32_16x16x64_bf16(
                        __builtin_bit_cast(bf8x, o.a[jj][WPL[k]][0]), bv, sum[jj][sb], (int)o.idx[jj], 0, 0);
            } else {
#pragma unroll
                for (int h = 0; h < 2; ++h)
#pragma unroll
                    for (int jj = 0; jj < NJ; ++jj)
                        sum[jj][sb] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(
                            __builtin_bit_cast(bf8x, o.a[jj][WPL[k]][AH == 2 ? h : 0]),
                            __builtin_bit_cast(bf8x, x[XP[k]][h]), sum[jj][sb], 0, 0, 0);
            }
            behind(k);
        }
        __builtin_amdgcn_sched_barrier(0);
    };
    // The chunks are dealt out in `full` rounds; those that are left over, fewer than groups, all groups do, each on the
    // blocks that it finishes, in a sum of its own: added to the group's, whose turn a chunk is would depend on the block, and
    // the same image would come out in other bits at another place of the batch.  Chunk i of the sum is tap i % ntaps of stage
    // i / ntaps.
    const int full = total / KG;
    auto advance = [&](int m) {                  // from this wavefront's chunk m to the next one
        const int step = m + 1 < full ? KG : m + 1 == full ? KG - grp : 1;
        tap += step;
        if (tap >= ntaps) {
            tap -= ntaps;
            ++cc;
        }
    };
    auto place_of = [&]() {
        const int kh = (int)fdiv((unsigned)tap, p.kw_mul, p.kw_shift), kw = tap - kh * p.Kw;
        return (unsigned)((cc & 1) * 3 * plane + kh * p.dh * Lg * 16 + kw * p.dw * 144);
    };
    // one chunk; the operands of the next one are loaded on the way (past the last one those of the same)
    auto chunk = [&](const Ops& o, Ops& next, int m) __attribute__((always_inline)) {
        const unsigned off = place_of();
        const int c = tap * p.ncpt + cc;
        advance(m);
        const int cn = cc < p.ncpt ? tap * p.ncpt + cc : c;
#pragma unroll
        for (int b = 0; b < NBLK; ++b)
            products(o, off, b, acc, b, [&](int k) __attribute__((always_inline)) {
#pragma unroll
                for (int jj = 0; jj < NJ; ++jj)
                    if (jj * NBLK / NJ == b && jj - (b * NJ + NBLK - 1) / NBLK == (k + 3) % 6) load_op(next, jj, cn);
            });
    };
    f4 rest[NJ][NO];                             // of the chunks left over
    auto left_over = [&](int m) __attribute__((always_inline)) {
        const unsigned off = place_of();
#pragma unroll
        for (int to = 0; to < KG; ++to)
            if (to == grp) {
#pragma unroll
                for (int b = 0; b < NO; ++b) products(oa, off, to * NO + b, rest, b, [](int) {});
            }
        advance(m);
        if (cc == p.ncpt) return;
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj) load_op(oa, jj, tap * p.ncpt + cc);
    };

    // Stage w is the next to be written: behind place m_free, by this wavefront at m_write, there for all from place m_there on.
    int w = 1, m_free = 0, m_write = 0, m_there = 0;
    bool free = true, written = false;
    const int early = wave >> 2;                 // (wavefronts 0 .. 3 and 4 .. 7 are those of the four SIMDs)
    auto plan = [&]() {
        m_free = w > 1 ? (ntaps * (w - 1) + KG - 1) / KG : 0;
        m_there = ntaps * w / KG;
        m_write = m_there - early > m_free ? m_there - early : m_free;
        free = w < 2;
        written = false;
    };
    plan();
    auto stages = [&](int m) __attribute__((always_inline)) {
        bool here = false;                       // this place's last barrier has everyone behind chunk m - 1
        while (w < p.ncpt) {
            if (!free && m >= m_free) {
                if (!here) split_barrier();
                free = true;
            }
            if (free && !written && m >= m_write) {
                stash(w, 0);
                if (w + 1 < p.ncpt) fetch(w + 1);
                written = true;
            }
            if (!written || m < m_there) break;
            split_barrier();
            here = true;
            ++w;
            plan();
        }
    };
    split_barrier();                             // the first stage is there
    for (int m = 0;;) {
        stages(m);
        chunk(oa, ob, m);
        if (++m == full) {
            oa = ob;
            break;
        }
        stages(m);
        chunk(ob, oa, m);
        if (++m == full) break;
    }
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
        for (int b = 0; b < NO; ++b) rest[jj][b] = f4{0.f, 0.f, 0.f, 0.f};
    const bool more = total % KG != 0;
    for (int m = full; m < full + total % KG; ++m) left_over(m);

    // ---- the groups' sums, and the output ------------------------------------------------------------------------------
    reinterpret_cast<int*>(lds8)[wave] = __builtin_amdgcn_ballot_w64((lost & 0xffffu) != 0u) != 0ull;
    split_barrier();                             // every wavefront is past its last read
    char* const sums = lds8 + kSplitTapsFlags;
    auto slot = [&](int to, int from) { return sums + ((cell * KG + to) * (KG - 1) + (from < to ? from : from - 1)) * (NO * NJ * 1024) + lane * 16; };
    f4 fin[NJ][NO];
#pragma unroll
    for (int to = 0; to < KG; ++to) {
        char* const dst = slot(to, grp);
#pragma unroll
        for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
            for (int b = 0; b < NO; ++b) {
                if (to == grp) fin[jj][b] = acc[jj][to * NO + b];
                else *reinterpret_cast<f4*>(dst + (b * NJ + jj) * 1024) = acc[jj][to * NO + b];
            }
    }
    split_barrier();
    int inexact = 0;                             // the planes of some activation left bits out
#pragma unroll
    for (int v = 0; v < 8; ++v) inexact |= reinterpret_cast<const int*>(lds8)[v];
#pragma unroll
    for (int jj = 0; jj < NJ; ++jj)
#pragma unroll
        for (int b = 0; b < NO; ++b) {
            const f4 own = fin[jj][b];
            f4 s = f4{0.f, 0.f, 0.f, 0.f};
#pragma unroll
            for (int from = 0; from < KG; ++from) {
                f4 v = own;
                if (from != grp) v = *reinterpret_cast<const f4*>(slot(grp, from) + (b * NJ + jj) * 1024);
                s = from == 0 ? v : s + v;
            }
            fin[jj][b] = more ? s + rest[jj][b] : s;
        }
    kernarg_t kp = (kernarg_t)__builtin_amdgcn_kernarg_segment_ptr();
    asm volatile("" : "+s"(kp));
    char* const piece = sums + split_taps_sums(NBLK, NJ, KG) + wave * (split_out_rows(NO) * split_out_pitch(NJ));
    split_finish<NO, NJ>(kp, fin, piece, lane, p0 + wpx * BPW + grp * (16 * NO), rb0, inexact, fast, reinterpret_cast<float*>(kp->y),
                         reinterpret_cast<const float*>(kp->res), kp->relu != 0, [&](int& k_lo, int& k_hi) {
                             k_lo = 0;
                             k_hi = kp->K;
                         });
}

template <int NBLK, int WP, int NJ, int KG, bool SPARSE>
int launch_split_taps_t(const ConvParams& p, hipStream_t s)
{
    auto kern = nm_conv_split_taps_kernel<NBLK, WP, NJ, KG, SPARSE>;
    constexpr size_t most = 160 * 1024;
    static unsigned long long done = 0;
    const int rc = allow_lds(reinterpret_cast<const void*>(kern), most, &done);
    if (rc != NM_OK) return rc;
    const size_t lds = split_taps_lds_bytes(NBLK, NJ, KG, p.rows_n, p.ncpt);
    if (lds > most || p.Cin % 64 != 0 || p.sh != 1 || p.sw != 1 || p.Ho != p.H || p.Wo != p.W || p.Kh * p.Kw < KG ||
        (p.ncpt > 1 && taps_loads(p.rows_n) > 8 * kSplitTapsItems)) {
        set_error("internal: a layer that the tap-staged kernel does not do");
        return NM_ERR_UNSUPPORTED;
    }
    hipLaunchKernelGGL(kern, dim3(p.wg_per_xcd * 8), dim3(512), lds, s, p);
    NM_HIP_CHECK(hipGetLastError());
    return NM_OK;
}

}  // namespace nm
