// Address- and undefined-behaviour-sanitizer run of the library's host layer
// (csrc/nm_api.hip: argument checks, geometry, operand-table planning, variant
// choice, the tuner's loop, the tuning cache and its file format) with no GPU.
// Built by tests/test_sanitizers.py from nm_api.hip compiled host-only with
// -fsanitize=address,undefined and this file, which stands in for everything
// below the host layer:
//   * the HIP runtime calls nm_api.hip makes ("device" memory is host memory),
//   * the kernel launchers (variant table, prune / table-build / fill kernels).
// The stand-ins check what the host layer hands them: launch_conv verifies the
// geometry in ConvParams against its own arithmetic and that every pointer
// it would pass to a kernel is one the fake allocator handed out, large enough.
#include <math.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <map>
#include <string>
#include <vector>

#include "nm_internal.h"

#define CHECK(c)                                                            \
    do {                                                                    \
        if (!(c)) {                                                         \
            fprintf(stderr, "check failed at line %d: %s (last error: %s)\n", __LINE__, #c, nm_last_error()); \
            exit(1);                                                        \
        }                                                                   \
    } while (0)

// ------------------------------------------------------------------ fake HIP
static std::map<char*, size_t> g_allocs;
static bool g_fail_malloc = false, g_no_device = false;
static int g_launches = 0;
static int g_walk = 0;   // groups of output channels that a workgroup of the last such launch walks
static int g_stream = -1, g_keep = -1;   // whether the last launch was to store past the caches, to leave the output to the L2

static bool inside(const void* p, size_t need)
{
    const char* c = (const char*)p;
    for (const auto& kv : g_allocs)
        if (c >= kv.first && c + need <= kv.first + kv.second) return true;
    return false;
}

extern "C" {
hipError_t hipGetDevice(int* d) { *d = 0; return g_no_device ? hipErrorNoDevice : hipSuccess; }
hipError_t hipGetDeviceProperties(hipDeviceProp_t* p, int)
{
    memset(p, 0, sizeof(*p));
    snprintf(p->name, sizeof(p->name), "Fake GPU for host tests");
    snprintf(p->gcnArchName, sizeof(p->gcnArchName), "gfx950:sramecc+:xnack-");
    p->multiProcessorCount = 256;
    return hipSuccess;
}
const char* hipGetErrorString(hipError_t) { return "fake HIP error"; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n)
{
    if (g_fail_malloc) { *p = nullptr; return hipErrorOutOfMemory; }
    char* c = (char*)malloc(n ? n : 1);
    g_allocs[c] = n;
    *p = c;
    return hipSuccess;
}
hipError_t hipFree(void* p)
{
    if (!p) return hipSuccess;
    auto it = g_allocs.find((char*)p);
    if (it == g_allocs.end()) { fprintf(stderr, "hipFree of a pointer that was never allocated\n"); exit(1); }
    g_allocs.erase(it);
    free(p);
    return hipSuccess;
}
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { memset(d, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
static bool g_capturing = false;
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st)
{
    *st = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipEventCreate(hipEvent_t* e) { *e = (hipEvent_t)malloc(1); return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t e) { free(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
// "time" = launches since the last query, so that variants differ deterministically
static int g_timer_variant = 0;
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t)
{
    *ms = 0.01f * (float)(1 + (g_timer_variant * 7919) % 101);
    return hipSuccess;
}
}

// ------------------------------------------------------- fake kernel layer
namespace nm {

static const VariantDesc kFake[] = {
    // name, BP, NBLK, WP, NJ, CK, SPC, vec, kind, share, ksplit, areg, spec, waves
    {"F_NB4_WP1_NJ1_CK32_SPC2", 64, 4, 1, 1, 32, 2, 1, 0, 1, 1, 0},
    {"F_NB4_WP1_NJ1_CK32_SPC4", 64, 4, 1, 1, 32, 4, 1, 0, 1, 1, 0},
    {"F_NB4_WP1_NJ1_CK32_SPC8", 64, 4, 1, 1, 32, 8, 1, 0, 1, 1, 0},
    {"F_NB8_WP1_NJ2_CK64_SPC4", 128, 8, 1, 2, 64, 4, 1, 0, 1, 1, 0},
    {"F_NB8_WP1_NJ2_CK64_SPC8", 128, 8, 1, 2, 64, 8, 1, 0, 1, 1, 0},
    {"F_NB8_WP1_NJ2_CK64_SPC2", 128, 8, 1, 2, 64, 2, 1, 0, 1, 1, 0},
    {"F_SCALAR_CK32_SPC8", 256, 4, 4, 4, 32, 8, 0, 0, 1, 1, 0},
    {"F_VAR_NB4_CK32_SPC8", 64, 4, 1, 1, 32, 8, 1, 5, 1, 1, 0},
    {"F_B16_NB4_CK64_SPC1", 64, 4, 1, 1, 64, 1, 1, 1, 1, 1, 0},
    {"F_B16_NB4_CK64_SPC2", 64, 4, 1, 1, 64, 2, 1, 1, 1, 1, 0},
    {"F_SP1_NB4_NJ2_CK64", 64, 4, 1, 2, 64, 1, 1, 2, 1, 1, 0},
    {"F_SP0_NB4_NJ2_CK128", 64, 4, 1, 2, 128, 2, 1, 3, 1, 1, 0},
    {"F_SP0_NB4_NJ2_CK64", 64, 4, 1, 2, 64, 1, 1, 3, 1, 1, 0},
    {"F_SPR1_NB4_NJ2_CK64", 64, 4, 1, 2, 64, 1, 1, 2, 1, 1, 1},
    {"F_RUN_NB4_KS3", 64, 4, 1, 1, 192, 3, 1, 4, 1, 1, 0},
    {"F_RUN_NB4_KS1", 64, 4, 1, 1, 64, 1, 1, 4, 1, 1, 0},
    {"F_F8_NB4_WP1_NJ4", 64, 4, 1, 4, 64, 1, 1, 6, 1, 1, 0},
    {"F_F8S_NB4_WP1_NJ2_CK64", 64, 4, 1, 2, 64, 1, 1, 7, 1, 1, 0},
    {"F_F8R_NB4_WP1_NJ2_CK128", 64, 4, 1, 2, 128, 2, 1, 7, 1, 1, 1},
    // K-split forms of the fp32 kernel
    {"F_NB4_WP1_NJ1_CK32_SPC4_S2", 64, 4, 1, 1, 32, 4, 1, 0, 1, 2, 0},
    {"F_NB4_WP1_NJ1_CK32_SPC4_S4", 64, 4, 1, 1, 32, 4, 1, 0, 1, 4, 0},
    {"F_NB4_WP1_NJ1_CK32_SPC2_S16", 64, 4, 1, 1, 32, 2, 1, 0, 1, 16, 0},
    {"F_SCALAR_CK32_SPC8_S2", 256, 4, 4, 4, 32, 8, 0, 0, 1, 2, 0},
    // fp32 as three bf16 planes, and few input channels out of staged rows (NBLK output rows a workgroup)
    {"F_X3S_NB4_WP1_NJ2", 64, 4, 1, 2, 64, 1, 1, 8, 1, 1, 0, 1},
    {"F_X3D_NB2_WP1_NJ1", 32, 2, 1, 1, 64, 1, 1, 9, 1, 1, 0, 1},
    {"F_X3S_NB4_WP1_NJ2_S2", 64, 4, 1, 2, 64, 1, 1, 8, 1, 2, 0, 1},
    {"F_RUN_ROWS1_NJ4_KS3", 16, 1, 4, 4, 192, 3, 1, 10, 1, 1, 0},
    {"F_RUN_ROWS8_NJ4_KS3", 16, 8, 4, 4, 192, 3, 1, 10, 1, 1, 0},
    {"F_RUN_ROWS4_NJ4_KS1", 16, 4, 4, 4, 64, 1, 1, 10, 1, 1, 0},
    {"F_ROWF_R2_NJ2_KS3", 16, 2, 2, 2, 192, 3, 1, 11, 1, 1, 0},
    {"F_ROWF_R4_NJ1_KS1", 16, 4, 1, 1, 64, 1, 1, 11, 1, 1, 0},
    // small fp32 layers, the K axis over wavefronts, and bf16 k x k layers staged once for all taps
    {"F_KW_PB1_NJ1_CK32_SPC2", 16, 1, 4, 1, 32, 2, 1, 12, 1, 1, 0, 0, 16},
    {"F_KW_PB1_NJ2_CK32_SPC4", 16, 1, 4, 2, 32, 4, 1, 12, 1, 1, 0, 0, 16},
    {"F_KW_PB2_NJ2_CK32_SPC8", 32, 2, 4, 2, 32, 8, 1, 12, 1, 1, 0, 0, 12},
    {"F_SPR1_TAPS_NB4_WP1_NJ2", 64, 4, 1, 2, 64, 1, 1, 13, 1, 1, 1, 1},
    {"F_SPR1_TAPS_NB7_WP2_NJ4", 224, 7, 2, 4, 64, 1, 1, 13, 1, 1, 1, 1},
    {"F_SPR0_TAPS_NB5_WP2_NJ4", 160, 5, 2, 4, 64, 1, 1, 14, 1, 1, 1, 1},
    // the same with eight contracting wavefronts; fp32 as three planes staged once for all taps; 1x1, output channels over resident pixels
    {"F_SPR1_TAP8_NB7_WP2_NJ4", 224, 7, 2, 4, 64, 1, 1, 13, 1, 1, 1, 1, 8},
    {"F_SPR0_TAP8_NB7_WP2_NJ2", 224, 7, 2, 2, 64, 1, 1, 14, 1, 1, 1, 1, 8},
    {"F_X3S_TAP_NB4_WP1_NJ4_KG2", 64, 4, 1, 4, 64, 1, 1, 15, 1, 1, 1, 0, 2},
    {"F_X3S_TAP_NB4_WP1_NJ4_KG4", 64, 4, 1, 4, 64, 1, 1, 15, 1, 1, 1, 0, 4},
    {"F_X3D_TAP_NB4_WP1_NJ2_KG4", 64, 4, 1, 2, 64, 1, 1, 16, 1, 1, 1, 0, 4},
    {"F_SPR1_COLS_NB4_C1", 64, 4, 1, 4, 64, 1, 1, 17, 1, 1, 1, 0, 1},
    {"F_SPR1_COLS_NB2_C1", 32, 2, 1, 4, 64, 1, 1, 17, 1, 1, 1, 0, 1},
    {"F_SPR1_COLS_NB4_C4", 64, 4, 1, 4, 64, 1, 1, 17, 1, 1, 1, 0, 4},
    {"F_SPR1_COLS_NB2_C4", 32, 2, 1, 4, 64, 1, 1, 17, 1, 1, 1, 0, 4},
};
int variant_count() { return (int)(sizeof(kFake) / sizeof(kFake[0])); }
const VariantDesc& variant_desc(int v) { return kFake[v]; }

int launch_conv(int v, nm_dtype_t xdt, nm_dtype_t ydt, const ConvParams& p, hipStream_t)
{
    CHECK(v >= 0 && v < variant_count());
    const VariantDesc& d = kFake[v];
    g_timer_variant = v;
    ++g_launches;
    g_stream = p.stream;
    g_keep = p.keep;
    CHECK(p.keep == 0 || (d.kind == 10 && p.stream == 0));
    const size_t es = xdt == NM_F32 ? 4 : (xdt == NM_BF16 ? 2 : 1), yes = ydt == NM_F32 ? 4 : 2;
    CHECK(xdt == ydt || (xdt == NM_F8E4M3 && ydt == NM_BF16));
    const bool f8 = d.kind == 6 || d.kind == 7;
    CHECK(f8 == (xdt == NM_F8E4M3));
    CHECK(p.oscale > 0.f && (f8 || p.oscale == 1.f));
    if (f8) {   // whole chunks per tap, and the table holds every 64-channel k-step of every row block
        CHECK(p.Cin % d.CK == 0 && p.nchunks == p.Kh * p.Kw * (p.Cin / d.CK));
        CHECK(p.wfrag_bytes == (size_t)p.n_rowblocks * (p.K / 64) * 1024);
    }
    // the geometry the kernels rely on
    const long eh = (long)p.H + 2L * p.ph - (long)p.dh * (p.Kh - 1) - 1, ew = (long)p.W + 2L * p.pw - (long)p.dw * (p.Kw - 1) - 1;
    CHECK(eh >= 0 && ew >= 0 && p.Ho == eh / p.sh + 1 && p.Wo == ew / p.sw + 1);
    CHECK(p.P == p.B * p.Ho * p.Wo && p.K == p.Kh * p.Kw * p.Cin);
    const bool rows = d.kind == 10 || d.kind == 11;
    CHECK(p.n_ptiles == (rows ? p.B * ((p.Ho + d.NBLK - 1) / d.NBLK) : (p.P + d.BP - 1) / d.BP));
    const bool walks = d.kind == 17, staged = d.kind >= 13 && d.kind <= 16, planes = d.kind == 15 || d.kind == 16;
    CHECK(p.n_wg == (walks ? p.n_ptiles * ((p.n_cblocks + p.cps - 1) / p.cps) : p.n_ptiles * p.n_cblocks * p.ksplit));
    if ((d.kind >= 8 && d.kind <= 11) || planes) CHECK(p.tile == 16 && p.rbpt == 1 && p.n_rowblocks == (p.Cout + 15) / 16);
    if (rows) {
        // every operand of every output pixel of a workgroup lies in the staged rows, and these in the CU's LDS
        const long last = (long)p.rows_front + ((long)(d.NBLK - 1) * p.sh + (long)(p.Kh - 1) * p.dh) * p.rows_pitch +
                          2L * (p.Wo - 1) * p.sw * p.Cin + 16L * p.run_gr;
        const long plane = (long)p.rows_n * p.rows_pitch;
        CHECK(p.rows_r == d.NBLK && p.rows_pitch % 16 == 0 && p.rows_data % 16 == 0 && p.rows_front >= 0 && last <= plane);
        // column 0 of the image is where the run of output column 0 finds it, and a whole row fits
        CHECK((long)p.rows_data - p.rows_front == 2 * ((long)p.pw * p.Cin + p.run_d));
        CHECK((long)p.rows_data + 2L * p.W * p.Cin <= p.rows_pitch);
        CHECK(plane * (d.kind == 10 ? 1 : 3) <= p.rows_lds && p.rows_lds % 1024 == 0 && p.rows_lds + 4 * 16 * 144 <= 160 * 1024);
        CHECK(p.dw == 1 && (p.sw * (long)p.Cin) % 2 == 0 && (p.W * p.Cin) % 2 == 0);
    }
    auto exact = [](unsigned div, unsigned mul, unsigned shift, unsigned most) {
        for (unsigned x : {0u, 1u, div - 1, div, div + 1, most / 2, most / div * div, most})
            if ((unsigned)(((unsigned long long)(2ull * x) * mul) >> 32) >> shift != x / div) return false;
        return true;
    };
    if (d.kind == 12) {
        // every wavefront owns chunks, together they cover the K axis; a place in a byte; what is divided by is the divisor
        CHECK(p.waves >= 1 && p.waves <= d.waves && p.cps >= 1 && (p.waves - 1) * p.cps < p.nchunks && p.waves * p.cps >= p.nchunks);
        CHECK(d.CK + 4 <= 256 && p.rows_bytes == (size_t)((p.Cout + p.tile - 1) / p.tile) * p.nchunks * 4 * d.SPC);
        CHECK(wave_lds_bytes(d.NBLK, d.NJ, d.CK, p.waves) <= 160 * 1024);
        CHECK(exact((unsigned)(p.px_fast ? p.n_ptiles : p.n_cblocks), p.fast_mul, p.fast_shift, (unsigned)p.n_wg));
        CHECK(exact((unsigned)p.ncpt, p.ncpt_mul, p.ncpt_shift, (unsigned)p.nchunks) && exact((unsigned)p.Kw, p.kw_mul, p.kw_shift, (unsigned)(p.Kh * p.Kw)));
        CHECK(exact((unsigned)p.rbpt, p.rbpt_mul, p.rbpt_shift, (unsigned)p.n_rowblocks + 16));
    }
    if (staged) {
        // an output as large as the input, whole granules and row blocks of 16 channels, the stages and what follows in the CU's LDS
        CHECK(p.sh == 1 && p.sw == 1 && p.Ho == p.H && p.Wo == p.W && p.Cin % 64 == 0 && p.tile % 16 == 0 && (planes || p.Cout % 8 == 0));
        CHECK(p.rows_n == taps_granules(d.BP, p.H, p.W, p.ph, p.pw) && p.rows_lds == taps_loads(p.rows_n) * 1024 && p.rows_lds >= p.rows_n * 16);
        const int waves = d.waves == 8 ? 8 : 4;
        CHECK((planes ? split_taps_lds_bytes(d.NBLK, d.NJ, d.waves, p.rows_n, p.ncpt)
                      : taps_lds_bytes(d.NBLK, d.WP, d.NJ, p.rows_n, p.ncpt, waves)) <= 160 * 1024 && p.ncpt == p.Cin / 64);
        const long line = taps_line(p.W, p.pw), lines = (long)(p.B + 2) * (p.H + p.ph);
        CHECK(lines < 1 << 24 && lines * line < 1l << 31 && p.P < 1 << 24);
        CHECK(exact((unsigned)line, p.padw_mul, p.padw_shift, (unsigned)(lines * line)) && exact((unsigned)(p.H + p.ph), p.padh_mul, p.padh_shift, (unsigned)lines));
        // what the registers of a wavefront or thread hold of a stage; a group of wavefronts for every tap at least
        CHECK(planes ? p.ncpt == 1 || taps_loads(p.rows_n) <= 8 * kSplitTapsItems : d.waves != 8 || taps_loads(p.rows_n) <= 8 * kTapsWideLoads);
        CHECK(!planes || (p.Kh * p.Kw >= d.waves && exact((unsigned)p.Kw, p.kw_mul, p.kw_shift, (unsigned)(p.Kh * p.Kw))));
    }
    if (walks) {
        // 1x1 without padding, the channels of the form, whole granules; every group of 256 output channels is walked by one workgroup
        CHECK(p.Kh == 1 && p.Kw == 1 && p.ph == 0 && p.pw == 0 && p.Cin == 64 * d.waves && p.nchunks == d.waves && p.Cout % 8 == 0 && p.tile % 16 == 0);
        g_walk = p.cps;
        CHECK(p.cps >= 1 && p.cps <= p.n_cblocks && cols_lds_bytes(d.NBLK, d.waves) <= 80 * 1024);
        CHECK(exact((unsigned)p.rbpt, p.rbpt_mul, p.rbpt_shift, (unsigned)p.n_rowblocks));
    }
    CHECK(p.ksplit == (d.ksplit > 1 ? d.ksplit : 1));
    if (p.ksplit > 1) {   // every split owns chunks, together they cover the K axis, and the partial sums have a home
        CHECK(p.cps >= 1 && (p.ksplit - 1) * p.cps < p.nchunks && p.ksplit * p.cps >= p.nchunks);
        CHECK(inside(p.partial, (size_t)p.ksplit * p.P * p.Cout * 4));
    }
    const int wc = (planes ? 8 / d.waves : staged && d.waves == 8 ? 8 : 4) / d.WP;   // wavefronts along the output channels
    CHECK(p.n_cblocks * wc * d.NJ >= p.n_rowblocks && (p.n_cblocks - 1) * wc * d.NJ < p.n_rowblocks);
    CHECK(p.wg_per_xcd * 8 >= p.n_wg);
    CHECK((size_t)p.x_elems * es == p.x_bytes && p.x_bytes < 0x80000000u);
    // multiply-shift division is exact on every value the kernels feed it
    const unsigned howo = (unsigned)(p.Ho * p.Wo);
    for (unsigned x : {0u, 1u, howo - 1, howo, howo + 1, (unsigned)p.P - 1, (unsigned)p.P + 1023u, 0x7ffffffeu}) {
        const unsigned q = (unsigned)(((unsigned long long)(2ull * x) * p.howo_mul) >> 32) >> p.howo_shift;
        CHECK(q == x / howo);
        const unsigned q2 = (unsigned)(((unsigned long long)(2ull * x) * p.wo_mul) >> 32) >> p.wo_shift;
        CHECK(q2 == x / (unsigned)p.Wo);
    }
    // every pointer is an allocation of the right size
    CHECK(inside(p.x, p.x_bytes) && inside(p.y, (size_t)p.P * p.Cout * yes));
    CHECK(!p.bias || inside(p.bias, (size_t)p.Cout * 4));
    CHECK(!p.res || inside(p.res, (size_t)p.P * p.Cout * yes));
    CHECK(inside(p.wfrag, p.wfrag_bytes));
    CHECK(p.rows_bytes == 0 || inside(p.rows, p.rows_bytes));
    if (!d.vec) CHECK(p.ktab && inside(p.ktab, (size_t)p.nchunks * d.CK * 4));
    return NM_OK;
}

// "prune": keep the first n columns of every group (ascending, valid), except that column
// tile 0 of handles with m >= 32 keeps the LAST n, so that kept sets crowd into some chunks;
// behind the indices, whether a weight is not finite
int run_prune(const float* w, nm_packed* wp, hipStream_t)
{
    CHECK(inside(wp->d_idx, ((size_t)wp->n_tiles * wp->kprime + 1) * 4) && inside(w, (size_t)wp->cout * wp->K * 4));
    for (size_t i = 0; i < (size_t)wp->cout * wp->K; ++i)
        if (!isfinite(w[i])) wp->d_idx[(size_t)wp->n_tiles * wp->kprime] = 1;
    CHECK(inside(wp->d_vals, (size_t)wp->n_tiles * wp->kprime * wp->tile * 4));
    for (int j = 0; j < wp->n_tiles; ++j)
        for (int g = 0; g < wp->G; ++g)
            for (int i = 0; i < wp->n; ++i)
                wp->d_idx[((size_t)j * wp->G + g) * wp->n + i] =
                    g * wp->m + ((j == 0 && wp->m >= 32) ? wp->m - wp->n + i : i);
    return NM_OK;
}
int run_build_prepack(nm_packed* wp, Prepack& pp, hipStream_t)
{
    CHECK(inside(pp.d_wfrag, pp.wfrag_bytes));
    CHECK(pp.rows_bytes == 0 || inside(pp.d_rows, pp.rows_bytes));
    CHECK(pp.cols_bytes == 0 || (inside(pp.d_cols, pp.cols_bytes) && pp.cols_bytes * 4 == pp.rows_bytes));
    memset(pp.d_wfrag, 0, pp.wfrag_bytes);   // touches every byte the kernel would fill
    (void)wp;
    return NM_OK;
}
int run_quantize_e4m3(nm_packed* wp, hipStream_t)
{
    CHECK(wp->scale > 0.f && inside(wp->d_vals, (size_t)wp->n_tiles * wp->kprime * wp->tile * 4));
    int e = 0;
    CHECK(frexpf(wp->scale, &e) == 0.5f);   // a power of two
    return NM_OK;
}
int run_build_mask(const nm_packed* wp, uint8_t* d_mask, hipStream_t)
{
    CHECK(inside(d_mask, (size_t)wp->cout * wp->K));
    memset(d_mask, 0, (size_t)wp->cout * wp->K);
    return NM_OK;
}
int run_fill_random(void* d, size_t n, nm_dtype_t dt, uint32_t, hipStream_t)
{
    CHECK(inside(d, n * (dt == NM_F32 ? 4 : (dt == NM_BF16 ? 2 : 1))));
    return NM_OK;
}
int run_maxpool(const void*, nm_dtype_t, int, int, int, int, int, int, int, int, int, void*, hipStream_t) { return NM_OK; }
int run_avgpool(const void*, nm_dtype_t, int, int, int, void*, hipStream_t) { return NM_OK; }
int run_im2col(const void*, nm_dtype_t, int, int, int, int, int, int, int, int, int, int, int, int, int, int, void*,
               hipStream_t) { return NM_OK; }
static char* fake = nullptr;
int static_scratch(int, float** out)
{
    if (!fake) {   // this "device's" copy of the static scratch array; never freed
        fake = (char*)malloc(kStaticScratchBytes);
        g_allocs[fake] = kStaticScratchBytes;
    }
    *out = (float*)fake;
    return NM_OK;
}
int run_splitk_reduce(const ConvParams& p, nm_dtype_t, hipStream_t)
{
    CHECK(p.ksplit > 1 && inside(p.partial, (size_t)p.ksplit * p.P * p.Cout * 4));
    return NM_OK;
}
int run_stream_floor(const void* x, size_t xb, void* y, size_t yb, hipStream_t)
{
    CHECK(inside(x, xb) && inside(y, yb));
    return NM_OK;
}
}  // namespace nm

// ------------------------------------------------------------------- driver
static void* dev_alloc(size_t n)
{
    void* p = nullptr;
    CHECK(hipMalloc(&p, n) == hipSuccess);
    return p;
}

static int g_taps_ran = 0, g_wide_ran = 0, g_planes_ran = 0, g_cols_ran = 0;

static void conv_case(int b, int h, int w, int cin, int cout, int kh, int kw, int n, int m, int tile, nm_dtype_t dt,
                      int sh, int sw, int ph, int pw, int dh, int dw)
{
    std::vector<float> wt((size_t)cout * kh * kw * cin, 0.5f);
    nm_packed_t* wp = nullptr;
    CHECK(nm_prune(wt.data(), cout, kh, kw, cin, n, m, tile, dt, &wp) == NM_OK && wp);
    int nt, g, nn, kp;
    CHECK(nm_packed_dims(wp, &nt, &g, &nn, &kp) == NM_OK && nt == (cout + tile - 1) / tile && kp == g * n);
    std::vector<int32_t> idx((size_t)nt * kp);
    std::vector<float> vals((size_t)nt * kp * tile);
    std::vector<uint8_t> mask((size_t)cout * kh * kw * cin);
    CHECK(nm_packed_indices(wp, idx.data()) == NM_OK);
    CHECK(nm_packed_values(wp, vals.data()) == NM_OK);
    CHECK(nm_packed_mask(wp, mask.data()) == NM_OK);
    const nm_dtype_t ydt = dt == NM_F8E4M3 ? NM_BF16 : dt;
    const size_t es = dt == NM_F32 ? 4 : (dt == NM_BF16 ? 2 : 1), yes = ydt == NM_F32 ? 4 : 2;
    const long eh = (long)h + 2L * ph - (long)dh * (kh - 1) - 1, ew = (long)w + 2L * pw - (long)dw * (kw - 1) - 1;
    const int ho = (int)(eh / sh) + 1, wo = (int)(ew / sw) + 1;
    void* x = dev_alloc((size_t)b * h * w * cin * es);
    void* y = dev_alloc((size_t)b * ho * wo * cout * yes);
    void* r = dev_alloc((size_t)b * ho * wo * cout * yes);
    float* bias = (float*)dev_alloc((size_t)cout * 4);
    const int before = g_launches;
    CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_OK);
    CHECK(g_launches == before + 1 && nm_last_variant() >= 0);
    CHECK(nm_conv2d_res(x, dt, b, h, w, cin, wp, nullptr, r, sh, sw, ph, pw, dh, dw, 0, y, ydt, nullptr) == NM_OK);
    CHECK(nm_conv2d_res(x, dt, b, h, w, cin, wp, nullptr, y, sh, sw, ph, pw, dh, dw, 0, y, ydt, nullptr) == NM_ERR_ARG);
    // the block of arguments: the same call, and the same refusals
    nm_conv_args_t args = {x, wp, bias, r, y, nullptr, dt, b, h, w, cin, sh, sw, ph, pw, dh, dw, 1, ydt, 0};
    for (int only = 0; only < 2; ++only) {
        args.static_only = only;
        CHECK(nm_conv2d_args(&args) == NM_OK);
        auto refused = [&](int code, auto change) {
            nm_conv_args_t a = args;
            change(a);
            return nm_conv2d_args(&a) == code;
        };
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.x_dev = nullptr; }));
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.wp = nullptr; }));
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.y_dev = nullptr; }));
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.residual_dev = a.y_dev; }));
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.cin += 1; }));
        CHECK(refused(NM_ERR_ARG, [](nm_conv_args_t& a) { a.stride_w = 0; }));
        CHECK(refused(NM_ERR_UNSUPPORTED, [](nm_conv_args_t& a) { a.y_dtype = a.y_dtype == NM_F32 ? NM_BF16 : NM_F32; }));
        CHECK(refused(NM_ERR_SHAPE, [](nm_conv_args_t& a) { a.b = 1 << 20; a.h = a.w = 4096; }));
    }
    CHECK(nm_conv2d_args(nullptr) == NM_ERR_ARG);
    int v = -1;
    float ms = 0.f;
    CHECK(nm_autotune(dt, b, h, w, cin, wp, 1, sh, sw, ph, pw, dh, dw, 1, ydt, nullptr, &v, &ms) == NM_OK);
    auto named = [](int u, const char* part) { return strstr(nm_variant_name(u), part) != nullptr; };
    auto taps = [&](int u) { return named(u, "_TAP") || named(u, "_COLS_"); };   // (depend on more than the handle)
    CHECK(v >= 0 && ms > 0.f && nm_variant_legal(v, wp, dt, ydt) == (taps(v) ? 0 : 1));
    CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_OK);
    CHECK(nm_last_variant() == v);
    // every legal variant forced in turn, an illegal one refused
    for (int u = 0; u < nm_variant_count(); ++u) {
        CHECK(nm_force_variant(u) == NM_OK);
        const int legal = nm_variant_legal(u, wp, dt, ydt);
        const int rc = nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr);
        CHECK(legal || taps(u) ? (rc == NM_OK || rc == NM_ERR_UNSUPPORTED) : rc == NM_ERR_UNSUPPORTED);
        if (rc != NM_OK) continue;
        g_taps_ran += named(u, "_TAPS_");
        g_wide_ran += named(u, "_TAP8_");
        g_planes_ran += named(u, "_TAP_");
        g_cols_ran += named(u, "_COLS_");
    }
    CHECK(nm_force_variant(-1) == NM_OK);
    // K-split variants: through the growable workspace, through the static scratch, and under capture
    for (int u = 0; u < nm_variant_count(); ++u) {
        const char* nme = nm_variant_name(u);
        if (!strstr(nme, "_S") || nm_variant_legal(u, wp, dt, ydt) != 1) continue;
        CHECK(nm_force_variant(u) == NM_OK);
        CHECK(nm_conv2d_static(x, dt, b, h, w, cin, wp, bias, r, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_OK);
        CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_OK);
        g_capturing = true;   // large enough already: no allocation, so capture is fine
        CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_OK);
        g_capturing = false;
    }
    CHECK(nm_force_variant(-1) == NM_OK);
    // argument and shape errors
    CHECK(nm_conv2d(x, dt, b, h, w, cin + 1, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_ERR_ARG);
    CHECK(nm_conv2d((char*)x + 2, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_ERR_ARG);
    CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, 0, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_ERR_ARG);
    CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, h + 2 * ph + 1, dw, 1, y, ydt, nullptr) ==
          (kh > 1 ? NM_ERR_SHAPE : NM_OK));
    CHECK(nm_conv2d(x, dt, b, h, w, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt == NM_F32 ? NM_BF16 : NM_F32, nullptr) ==
          NM_ERR_UNSUPPORTED);
    CHECK(nm_conv2d(x, dt, 1 << 20, 4096, 4096, cin, wp, bias, sh, sw, ph, pw, dh, dw, 1, y, ydt, nullptr) == NM_ERR_SHAPE);
    CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && hipFree(r) == hipSuccess && hipFree(bias) == hipSuccess);
    CHECK(nm_packed_free(wp) == NM_OK);
}

// one layer of few input channels, each row-staged form forced: runs of both alignments, a padding far wider than any row,
// a stride that leaves one column of a huge padded image
static void rows_case(int b, int h, int w, int cin, int kh, int kw, nm_dtype_t dt, int sh, int sw, int ph, int pw, bool any)
{
    const int cout = 24;
    std::vector<float> wt((size_t)cout * kh * kw * cin, 0.5f);
    nm_packed_t* wp = nullptr;
    CHECK(nm_prune(wt.data(), cout, kh, kw, cin, 1, 1, 16, dt, &wp) == NM_OK);
    const size_t es = dt == NM_F32 ? 4 : 2;
    const int ho = (int)(((long)h + 2L * ph - kh) / sh) + 1, wo = (int)(((long)w + 2L * pw - kw) / sw) + 1;
    void* x = dev_alloc((size_t)b * h * w * cin * es);
    void* y = dev_alloc((size_t)b * ho * wo * cout * es);
    int ran = 0;
    for (int u = -1; u < nm_variant_count(); ++u) {
        if (u >= 0 && (!strstr(nm_variant_name(u), "ROW") || nm_variant_legal(u, wp, dt, dt) != 1)) continue;
        CHECK(nm_force_variant(u) == NM_OK);
        const int rc = nm_conv2d(x, dt, b, h, w, cin, wp, nullptr, sh, sw, ph, pw, 1, 1, 0, y, dt, nullptr);
        CHECK(rc == NM_OK || (u >= 0 && rc == NM_ERR_UNSUPPORTED));
        ran += u >= 0 && rc == NM_OK;
    }
    CHECK((ran > 0) == any);
    CHECK(nm_force_variant(-1) == NM_OK);
    CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
}

// a K split whose partial sums outgrow the static scratch, and one that would have to allocate under capture
static void split_limits()
{
    const int cout = 64, cin = 64;
    std::vector<float> wt((size_t)cout * 9 * cin, 0.5f);
    nm_packed_t* wp = nullptr;
    CHECK(nm_prune(wt.data(), cout, 3, 3, cin, 2, 4, 16, NM_F32, &wp) == NM_OK);
    int forced = -1;
    for (int u = 0; u < nm_variant_count(); ++u)
        if (strstr(nm_variant_name(u), "_S4") && nm_variant_legal(u, wp, NM_F32, NM_F32) == 1) forced = u;
    CHECK(forced >= 0 && nm_force_variant(forced) == NM_OK);
    const int b = 8, h = 96, w = 96;   // 4 splits x 73728 pixels x 64 channels x 4 bytes = 75 MB
    void* x = dev_alloc((size_t)b * h * w * cin * 4);
    void* y = dev_alloc((size_t)b * h * w * cout * 4);
    CHECK(nm_conv2d_static(x, NM_F32, b, h, w, cin, wp, nullptr, nullptr, 1, 1, 1, 1, 1, 1, 0, y, NM_F32, nullptr) == NM_ERR_SHAPE);
    CHECK(strstr(nm_last_error(), "static buffer"));
    g_capturing = true;
    CHECK(nm_conv2d(x, NM_F32, b, h, w, cin, wp, nullptr, 1, 1, 1, 1, 1, 1, 0, y, NM_F32, nullptr) == NM_ERR_ALLOC);
    g_capturing = false;
    CHECK(nm_conv2d(x, NM_F32, b, h, w, cin, wp, nullptr, 1, 1, 1, 1, 1, 1, 0, y, NM_F32, nullptr) == NM_OK);
    CHECK(nm_force_variant(-1) == NM_OK);
    CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
}

// Which outputs are stored past the caches, on either side of the line: by their size, the same for every form that may run a layer
// but those of staged rows, which run first layers; and which of these are left to the L2
static void store_limits()
{
    auto all = [](nm_dtype_t dt, int b, int hw, int cin, int cout, int k, int stride, int pad, const char* form, int want, int keep = 0) {
        std::vector<float> wt((size_t)cout * k * k * cin, 0.5f);
        nm_packed_t* wp = nullptr;
        CHECK(nm_prune(wt.data(), cout, k, k, cin, 1, cin % 4 ? 1 : 4, 16, dt, &wp) == NM_OK);
        const size_t es = dt == NM_F32 ? 4 : 2;
        const int ho = (hw + 2 * pad - k) / stride + 1;
        void* x = dev_alloc((size_t)b * hw * hw * cin * es);
        void* y = dev_alloc((size_t)b * ho * ho * cout * es);
        int ran = 0;
        for (int u = 0; u < nm_variant_count(); ++u) {
            if (!strstr(nm_variant_name(u), form)) continue;
            CHECK(nm_force_variant(u) == NM_OK);
            const int rc = nm_conv2d(x, dt, b, hw, hw, cin, wp, nullptr, stride, stride, pad, pad, 1, 1, 0, y, dt, nullptr);
            CHECK(rc == NM_OK || rc == NM_ERR_UNSUPPORTED);
            if (rc != NM_OK) continue;
            CHECK(g_stream == want && g_keep == keep);
            ++ran;
        }
        CHECK(ran > 0 && nm_force_variant(-1) == NM_OK);
        CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
    };
    for (const char* form : {"F_RUN_NB4", "F_RUN_ROWS"}) {   // 1.6 MB an image
        const int rows = strstr(form, "ROWS") != nullptr;
        all(NM_BF16, 44, 224, 3, 64, 7, 2, 3, form, 0, 0);
        all(NM_BF16, 45, 224, 3, 64, 7, 2, 3, form, 0, rows);
        all(NM_BF16, 64, 224, 3, 64, 7, 2, 3, form, 0, rows);
        all(NM_BF16, 93, 224, 3, 64, 7, 2, 3, form, 0, rows);
        all(NM_BF16, 94, 224, 3, 64, 7, 2, 3, form, !rows, rows);
        all(NM_BF16, 159, 224, 3, 64, 7, 2, 3, form, !rows, rows);
        all(NM_BF16, 160, 224, 3, 64, 7, 2, 3, form, 1, 0);
    }
    for (const char* form : {"F_SP", "F_B16"}) {
        all(NM_BF16, 93, 56, 64, 256, 1, 1, 0, form, 0);
        all(NM_BF16, 94, 56, 64, 256, 1, 1, 0, form, 1);
    }
    all(NM_F32, 46, 56, 64, 256, 1, 1, 0, "F_", 0);          // 3.2 MB an image
    all(NM_F32, 47, 56, 64, 256, 1, 1, 0, "F_X3S_NB4_WP1_NJ2", 1);
    all(NM_F32, 79, 224, 3, 64, 7, 2, 3, "F_ROWF", 0);
    all(NM_F32, 80, 224, 3, 64, 7, 2, 3, "F_ROWF", 1);
}

// The tap-staged forms on either side of what bounds them: rows of 3000 pixels, padded rows below 2^24, padded granules below
// 2^31 (padding far wider than the image), 32 taps
static void taps_limits()
{
    std::vector<float> wt((size_t)8 * 35 * 64, 0.5f);
    int form = -1;
    for (int u = 0; u < nm_variant_count(); ++u)
        if (strstr(nm_variant_name(u), "SPR1_TAPS_NB4")) form = u;
    auto run = [&](int b, int h, int w, int kh, int kw, int dh, int dw, int ph, int pw) {
        nm_packed_t* wp = nullptr;
        CHECK(nm_prune(wt.data(), 8, kh, kw, 64, 2, 4, 16, NM_BF16, &wp) == NM_OK);
        void* x = dev_alloc((size_t)b * h * w * 64 * 2);
        void* y = dev_alloc((size_t)b * h * w * 8 * 2);
        CHECK(nm_force_variant(form) == NM_OK);
        const int rc = nm_conv2d(x, NM_BF16, b, h, w, 64, wp, nullptr, 1, 1, ph, pw, dh, dw, 0, y, NM_BF16, nullptr);
        CHECK(nm_force_variant(-1) == NM_OK && (rc == NM_OK || rc == NM_ERR_UNSUPPORTED));
        CHECK(nm_conv2d(x, NM_BF16, b, h, w, 64, wp, nullptr, 1, 1, ph, pw, dh, dw, 0, y, NM_BF16, nullptr) == NM_OK);
        CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
        return rc == NM_OK;
    };
    CHECK(run(1, 2, 3000, 1, 3, 1, 1, 0, 1) && !run(1, 2, 3001, 1, 3, 1, 1, 0, 1));
    CHECK(run(8388605, 1, 1, 3, 3, 1, 1, 1, 1) && !run(8388606, 1, 1, 3, 3, 1, 1, 1, 1));
    CHECK(run(3976819, 1, 4, 1, 3, 1, 56, 0, 56) && !run(3976820, 1, 4, 1, 3, 1, 56, 0, 56));
    CHECK(run(1, 1, 64, 1, 3, 1, 300, 0, 300) && !run(1, 1, 64, 1, 3, 1, 1001, 0, 1001) && !run(1, 1, 64, 3, 1, 0x20000000, 1, 0x20000000, 0));
    CHECK(run(1, 9, 9, 31, 1, 1, 1, 15, 0) && !run(1, 9, 9, 5, 7, 1, 1, 2, 3) && !run(1, 9, 9, 1, 1, 1, 1, 0, 0));
    // ... and as the untuned default of a layer with enough workgroups
    wt.resize((size_t)128 * 9 * 128, 0.5f);
    nm_packed_t* wp = nullptr;
    CHECK(nm_prune(wt.data(), 128, 3, 3, 128, 2, 4, 16, NM_BF16, &wp) == NM_OK);
    void* x = dev_alloc((size_t)64 * 28 * 28 * 128 * 2);
    void* y = dev_alloc((size_t)64 * 28 * 28 * 128 * 2);
    CHECK(nm_conv2d(x, NM_BF16, 64, 28, 28, 128, wp, nullptr, 1, 1, 1, 1, 1, 1, 0, y, NM_BF16, nullptr) == NM_OK);
    CHECK(strstr(nm_variant_name(nm_last_variant()), "_TAPS_"));
    CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
}

// Layers whose output channels a workgroup walks whole or in part, forced and as the untuned default
static void cols_walks()
{
    struct Case { int b, cin, cout, walk2, walk4; };   // groups of 256 channels walked with tiles of 32 and 64 pixels
    for (const Case& c : {Case{70, 64, 2056, 9, 5}, Case{40, 64, 1000, 2, 1}, Case{64, 256, 1024, 4, 2}, Case{256, 256, 1024, 4, 4}}) {
        std::vector<float> wt((size_t)c.cout * c.cin, 0.5f);
        nm_packed_t* wp = nullptr;
        CHECK(nm_prune(wt.data(), c.cout, 1, 1, c.cin, 2, 4, 16, NM_BF16, &wp) == NM_OK);
        void* x = dev_alloc((size_t)c.b * 14 * 14 * c.cin * 2);
        void* y = dev_alloc((size_t)c.b * 14 * 14 * c.cout * 2);
        auto run = [&]() { return nm_conv2d(x, NM_BF16, c.b, 14, 14, c.cin, wp, nullptr, 1, 1, 0, 0, 1, 1, 0, y, NM_BF16, nullptr); };
        for (int u = 0; u < nm_variant_count(); ++u) {
            if (!strstr(nm_variant_name(u), "_COLS_")) continue;
            const int walk = strstr(nm_variant_name(u), "NB2") ? c.walk2 : c.walk4;
            const bool fits = strstr(nm_variant_name(u), c.cin == 64 ? "_C1" : "_C4") != nullptr;
            CHECK(nm_force_variant(u) == NM_OK && run() == (fits ? NM_OK : NM_ERR_UNSUPPORTED) && (!fits || g_walk == walk));
        }
        CHECK(nm_force_variant(-1) == NM_OK && run() == NM_OK);
        if (c.cin == 256) CHECK(strstr(nm_variant_name(nm_last_variant()), "_COLS_"));
        CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(wp) == NM_OK);
    }
}

// The default remembered for a shape, met by a handle that agrees in everything that the key holds but has no table for it
// (the key holds a hash of the tables); and more shapes than the table holds.
static void remembered_defaults()
{
    const int cout = 16, cin = 8;
    std::vector<float> wt((size_t)cout * cin, 0.5f);
    nm_packed_t *a = nullptr, *b = nullptr;
    CHECK(nm_prune(wt.data(), cout, 1, 1, cin, 2, 4, 16, NM_F32, &a) == NM_OK);
    CHECK(nm_prune(wt.data(), cout, 1, 1, cin, 2, 4, 16, NM_F32, &b) == NM_OK && a->sig == b->sig);
    void* x = dev_alloc((size_t)6000 * cin * 4);
    void* y = dev_alloc((size_t)6000 * cout * 4);
    auto call = [&](nm_packed_t* wp, int h) {
        return nm_conv2d(x, NM_F32, 1, h, 1, cin, wp, nullptr, 1, 1, 0, 0, 1, 1, 0, y, NM_F32, nullptr);
    };
    CHECK(call(a, 5) == NM_OK);
    const int first = nm_last_variant();
    const nm::VariantDesc& d = nm::variant_desc(first);
    for (size_t i = 0; i < b->prepacks.size(); ++i)
        if (b->prepacks[i].kind == d.kind && b->prepacks[i].geom.CK == d.CK && b->prepacks[i].SPC == d.SPC)
            b->prepacks.erase(b->prepacks.begin() + (long)i--);
    CHECK(!b->prepacks.empty() && nm_variant_legal(first, b, NM_F32, NM_F32) == 0);
    CHECK(call(b, 5) == NM_OK && nm_last_variant() != first);
    CHECK(call(a, 5) == NM_OK && nm_variant_legal(nm_last_variant(), a, NM_F32, NM_F32) == 1);
    for (int h = 1; h <= 6000; ++h) CHECK(call(a, h) == NM_OK);
    CHECK(call(a, 5) == NM_OK && nm_last_variant() == first);
    CHECK(hipFree(x) == hipSuccess && hipFree(y) == hipSuccess && nm_packed_free(a) == NM_OK && nm_packed_free(b) == NM_OK);
}

// Weights that are not finite are refused as such, few or many, and whatever else would have gone wrong
static void not_finite()
{
    for (int cout : {16, 600}) {   // 4096 weights and 153600: looked at by the host, and by the selection kernel
        std::vector<float> wt((size_t)cout * 256, 0.5f);
        nm_packed_t* wp = nullptr;
        auto prune = [&]() { return nm_prune(wt.data(), cout, 1, 1, 256, 2, 4, 16, NM_F32, &wp); };
        const size_t before = g_allocs.size();
        for (float bad : {NAN, -INFINITY}) {
            wt[1001] = wt[3000] = bad;
            for (int how = 0; how < 3; ++how) {
                g_fail_malloc = how == 1;
                g_no_device = how == 2;
                CHECK(prune() == NM_ERR_ARG && !wp && strstr(nm_last_error(), "weight 1001 is not finite"));
                g_fail_malloc = g_no_device = false;
            }
        }
        wt[1001] = wt[3000] = 1;
        g_fail_malloc = true;
        CHECK(prune() == NM_ERR_ALLOC && !wp);
        g_fail_malloc = false;
        g_no_device = true;
        CHECK(prune() == NM_ERR_HIP && !wp && g_allocs.size() == before);
        g_no_device = false;
        CHECK(prune() == NM_OK && nm_packed_free(wp) == NM_OK && g_allocs.size() == before);
    }
}

int main(int argc, char** argv)
{
    const std::string tmp = argc > 1 ? argv[1] : "/tmp";
    CHECK(nm_variant_count() > 0 && nm_variant_name(-1) == nullptr && nm_variant_name(nm_variant_count()) == nullptr);
    CHECK(nm_last_variant() == -1);

    // ---- nm_prune argument checks
    nm_packed_t* wp = nullptr;
    float w4[16] = {1, 2, 3, 4, 5, 6, 7, 8, 9, 10, 11, 12, 13, 14, 15, 16};
    CHECK(nm_prune(nullptr, 1, 1, 1, 16, 2, 4, 16, NM_F32, &wp) == NM_ERR_ARG);
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 16, NM_F32, nullptr) == NM_ERR_ARG);
    CHECK(nm_prune(w4, 0, 1, 1, 16, 2, 4, 16, NM_F32, &wp) == NM_ERR_ARG && !wp);
    CHECK(nm_prune(w4, 1, 1, 1, 16, 5, 4, 16, NM_F32, &wp) == NM_ERR_ARG);
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 5, 16, NM_F32, &wp) == NM_ERR_ARG);     // K % m
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 0, NM_F32, &wp) == NM_ERR_ARG);
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 16, (nm_dtype_t)7, &wp) == NM_ERR_ARG);
    w4[7] = INFINITY;
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 16, NM_F32, &wp) == NM_ERR_ARG && strstr(nm_last_error(), "finite"));
    w4[7] = NAN;
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 16, NM_F32, &wp) == NM_ERR_ARG);
    w4[7] = 8;
    g_fail_malloc = true;      // an allocation failure half way frees everything it had
    CHECK(nm_prune(w4, 1, 1, 1, 16, 2, 4, 16, NM_F32, &wp) == NM_ERR_ALLOC && !wp && g_allocs.empty());
    g_fail_malloc = false;
    CHECK(nm_packed_dims(nullptr, nullptr, nullptr, nullptr, nullptr) == NM_ERR_ARG);
    CHECK(nm_packed_indices(nullptr, nullptr) == NM_ERR_ARG && nm_packed_values(nullptr, nullptr) == NM_ERR_ARG);
    CHECK(nm_packed_mask(nullptr, nullptr) == NM_ERR_ARG && nm_packed_free(nullptr) == NM_OK);
    CHECK(nm_force_variant(-2) == NM_ERR_ARG && nm_force_variant(nm_variant_count()) == NM_ERR_ARG);
    CHECK(nm_conv2d(nullptr, NM_F32, 1, 1, 1, 1, nullptr, nullptr, 1, 1, 0, 0, 1, 1, 0, nullptr, NM_F32, nullptr) == NM_ERR_ARG);
    CHECK(nm_autotune(NM_F32, 1, 1, 1, 1, nullptr, 0, 1, 1, 0, 0, 1, 1, 0, NM_F32, nullptr, nullptr, nullptr) == NM_ERR_ARG);

    {
        void* a = dev_alloc(100);
        void* b = dev_alloc(64);
        CHECK(nm_stream_floor(a, 100, b, 64, nullptr) == NM_OK);
        CHECK(nm_stream_floor(nullptr, 100, b, 64, nullptr) == NM_ERR_ARG);
        CHECK(nm_stream_floor((char*)a + 4, 96, b, 64, nullptr) == NM_ERR_ARG);
        CHECK(hipFree(a) == hipSuccess && hipFree(b) == hipSuccess);
    }

    // ---- planning, launching, tuning over a grid of layers (ragged tiles, strides, dilation,
    // few input channels, groups wider than a chunk, T = 8 / 32, both tensor types)
    CHECK(nm_cache_clear() == NM_OK);
    conv_case(2, 9, 7, 16, 20, 3, 3, 2, 4, 16, NM_F32, 1, 1, 1, 1, 1, 1);
    conv_case(1, 12, 12, 3, 24, 7, 7, 1, 1, 16, NM_F32, 2, 2, 3, 3, 1, 1);     // element-wise staging
    conv_case(1, 12, 12, 3, 24, 7, 7, 1, 1, 16, NM_BF16, 2, 2, 3, 3, 1, 1);    // kernel-row runs
    conv_case(3, 8, 8, 64, 40, 1, 1, 2, 4, 8, NM_BF16, 2, 2, 0, 0, 1, 1);
    conv_case(1, 6, 10, 64, 64, 3, 3, 32, 64, 32, NM_F32, 1, 2, 2, 1, 2, 1);   // one group per tap
    conv_case(1, 5, 5, 128, 16, 1, 1, 4, 8, 16, NM_BF16, 1, 1, 0, 0, 1, 1);    // dense instruction only
    conv_case(1, 1, 1, 8, 5, 1, 1, 1, 2, 5, NM_F32, 1, 1, 0, 0, 1, 1);
    conv_case(2, 7, 6, 128, 40, 3, 3, 2, 4, 16, NM_F8E4M3, 2, 1, 1, 1, 1, 1);    // fp8 in, bf16 out
    CHECK(g_taps_ran == 0);
    conv_case(3, 9, 7, 128, 40, 3, 3, 2, 4, 16, NM_BF16, 1, 1, 1, 1, 1, 1);    // a tile's input staged once for all taps
    conv_case(1, 12, 5, 64, 24, 1, 3, 4, 8, 32, NM_BF16, 1, 1, 0, 2, 3, 2);    // ... dense instruction only
    CHECK(g_taps_ran == 3 + 1 && g_wide_ran == 2 + 1 && g_planes_ran == 0);
    conv_case(3, 9, 7, 128, 37, 3, 3, 2, 4, 5, NM_F32, 1, 1, 1, 1, 1, 1);      // ... as three planes
    conv_case(1, 56, 40, 64, 24, 1, 3, 1, 1, 16, NM_F32, 1, 1, 0, 1, 1, 1);    // ... dense, fewer taps than groups
    conv_case(1, 56, 60, 64, 24, 2, 2, 1, 1, 16, NM_F32, 1, 1, 1, 1, 2, 2);    // ... as many, one stage that threads take in two passes
    CHECK(g_planes_ran == 2 + 0 + 1);
    g_cols_ran = 0;
    conv_case(3, 28, 27, 64, 776, 1, 1, 2, 8, 48, NM_BF16, 2, 1, 0, 0, 1, 1);  // output channels walked over resident pixels
    conv_case(2, 7, 7, 256, 1024, 1, 1, 1, 4, 16, NM_BF16, 1, 1, 0, 0, 1, 1);
    CHECK(g_cols_ran == 2 + 2);
    cols_walks();
    taps_limits();
    {   // E4M3 weights that the fp8 kernel cannot take, and fp8 tensors on weights of another type
        std::vector<float> wt(16 * 48, 0.25f);
        nm_packed_t* h8 = nullptr;
        CHECK(nm_prune(wt.data(), 16, 1, 1, 48, 2, 4, 16, NM_F8E4M3, &h8) == NM_ERR_UNSUPPORTED && !h8);
        CHECK(nm_prune(wt.data(), 12, 1, 1, 64, 2, 4, 16, NM_F8E4M3, &h8) == NM_ERR_UNSUPPORTED && !h8);
        std::vector<float> w64(16 * 64, 0.25f);
        CHECK(nm_prune(w64.data(), 16, 1, 1, 64, 2, 4, 16, NM_F32, &h8) == NM_OK);
        void* xb = dev_alloc(64), *yb = dev_alloc(64);
        CHECK(nm_conv2d(xb, NM_F8E4M3, 1, 1, 1, 64, h8, nullptr, 1, 1, 0, 0, 1, 1, 0, yb, NM_BF16, nullptr) == NM_ERR_UNSUPPORTED);
        float sc = 0.f;
        CHECK(nm_packed_scale(h8, &sc) == NM_OK && sc == 1.f && nm_packed_scale(nullptr, &sc) == NM_ERR_ARG);
        CHECK(hipFree(xb) == hipSuccess && hipFree(yb) == hipSuccess && nm_packed_free(h8) == NM_OK);
    }
    split_limits();
    store_limits();
    remembered_defaults();
    not_finite();
    for (nm_dtype_t dt : {NM_F32, NM_BF16}) {
        rows_case(2, 17, 20, 3, 7, 7, dt, 2, 2, 3, 3, true);
        rows_case(1, 9, 10, 2, 3, 3, dt, 1, 1, 1, 1, true);
        rows_case(1, 9, 10, 2, 3, 3, dt, 3, 1, 0, 0, true);
        rows_case(1, 9, 10, 2, 3, 3, dt, 1, 1, 1, 20000, false);                          // the padding alone fills the LDS
        rows_case(1, 9, 10, 2, 3, 3, dt, 1, 0x3fffffff, 1, 0x20000000, false);            // two columns, 2^30 apart
        rows_case(1, 9, 10, 2, 3, 3, dt, 1, 0x40000000, 1, 0x3ffffffa, false);
    }
    // nothing leaked on the "device": what is left is the K-split workspace and the static scratch
    CHECK(g_allocs.size() <= 2);
    const int n_entries = nm_cache_size();
    CHECK(n_entries == 15);

    // ---- cache file round trip and hostile files
    const std::string path = tmp + "/nm_cache_san.txt";
    CHECK(nm_cache_save(path.c_str()) == NM_OK);
    CHECK(nm_cache_clear() == NM_OK && nm_cache_size() == 0);
    CHECK(nm_cache_load(path.c_str()) == NM_OK && nm_cache_size() == n_entries);
    CHECK(nm_cache_load((tmp + "/does_not_exist.txt").c_str()) == NM_ERR_IO);
    CHECK(nm_cache_save((tmp + "/no_such_dir/x.txt").c_str()) == NM_ERR_IO);
    CHECK(nm_cache_save(nullptr) == NM_ERR_ARG && nm_cache_load(nullptr) == NM_ERR_ARG);
    const char* hostile[] = {
        "", "nmconv-cache", "nmconv-cache 1 5\n", "garbage garbage\n1 2 3\n",
        "nmconv-cache 2 14 24 dev\n1 2 3\n",                                  // truncated entry
        "nmconv-cache 2 14 24 dev\n0 0 1 1 1 1 1 1 1 1 1 0 0 1 1 1 1 1 0 0 0 0 0 0 NO_SUCH_VARIANT 0.5\n",
        "nmconv-cache 2 14 24 dev\n0 0 1 1 1 1 1 1 1 1 1 0 0 1 1 1 1 1 0 0 0 0 0 0 "
        "AAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAAA 1.0\n",
        "nmconv-cache 2 14 24 "
        "DDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDDD\n",
        "nmconv-cache 2 14 24 dev\n99999999999999999999 1 2\n",
    };
    for (const char* text : hostile) {
        const std::string hp = tmp + "/nm_cache_hostile.txt";
        FILE* f = fopen(hp.c_str(), "w");
        CHECK(f);
        fputs(text, f);
        fclose(f);
        const int before = nm_cache_size();
        const int rc = nm_cache_load(hp.c_str());
        CHECK(rc == NM_OK || rc == NM_ERR_IO);
        CHECK(nm_cache_size() == before);          // nothing it holds names a real variant of a real shape
    }
    CHECK(nm_cache_clear() == NM_OK);
    CHECK(nm_workspace_free() == NM_OK);
    g_allocs.erase(nm::fake);
    free(nm::fake);
    CHECK(g_allocs.empty());
    puts("host-layer sanitizer run: ok");
    return 0;
}
