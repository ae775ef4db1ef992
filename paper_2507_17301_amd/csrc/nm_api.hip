// C ABI of libnmconv: argument checking, the packed-weights handle, variant
// choice, the tuning cache and the profiler-driven tuner.  All arithmetic of
// the method runs in the kernels; this file only plans and launches.
#include <math.h>
#include <stdarg.h>
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>

#include "nm_internal.h"

namespace nm {

static thread_local char g_err[512] = "";
static thread_local int g_last_variant = -1;

void set_error(const char* fmt, ...)
{
    va_list ap;
    va_start(ap, fmt);
    vsnprintf(g_err, sizeof(g_err), fmt, ap);
    va_end(ap);
}

int allow_lds(const void* fn, size_t bytes, unsigned long long* done)
{
    if (bytes <= 64 * 1024) return NM_OK;
    int dev = 0;
    NM_HIP_CHECK(hipGetDevice(&dev));
    const unsigned long long bit = 1ull << (dev & 63);
    static std::mutex mu;
    std::lock_guard<std::mutex> lk(mu);
    if (*done & bit) return NM_OK;
    const hipError_t e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (e != hipSuccess) {
        set_error("hipFuncSetAttribute(LDS %zu) failed: %s", bytes, hipGetErrorString(e));
        return NM_ERR_HIP;
    }
    *done |= bit;
    return NM_OK;
}

namespace {

inline size_t elem_size(nm_dtype_t dt) { return dt == NM_F32 ? 4 : (dt == NM_BF16 ? 2 : 1); }
// the pairs the kernels exist for: fp32 -> fp32, bf16 -> bf16, E4M3 -> bf16
inline bool dtype_pair_ok(nm_dtype_t xdt, nm_dtype_t ydt)
{
    return (xdt == NM_F32 && ydt == NM_F32) || (xdt == NM_BF16 && ydt == NM_BF16) ||
           (xdt == NM_F8E4M3 && ydt == NM_BF16);
}

constexpr int kMaxLdsBytes = 160 * 1024;
constexpr int kNumCU = 256;

constexpr int kKeyInts = 24;
struct ShapeKey {
    int v[kKeyInts];
    bool operator<(const ShapeKey& o) const { return memcmp(v, o.v, sizeof(v)) < 0; }
};
struct CacheVal {
    int variant;
    float ms;
};

std::mutex g_mu;
std::map<ShapeKey, CacheVal> g_cache;
int g_forced = -1;

// 31-bit FNV-1a
unsigned fnv(unsigned h, const void* data, size_t n)
{
    const unsigned char* b = (const unsigned char*)data;
    for (size_t i = 0; i < n; ++i) h = (h ^ b[i]) * 16777619u;
    return h;
}

// Identity of a device for the tuning cache: a timing taken on one kind of GPU says
// nothing about another.  Architecture string and CU count, hashed; kept per ordinal.
struct DeviceId {
    int hash = 0;
    char name[128] = "";
};
const DeviceId* device_id(int dev)
{
    static std::mutex mu;
    static std::map<int, DeviceId> ids;
    std::lock_guard<std::mutex> lk(mu);
    auto it = ids.find(dev);
    if (it != ids.end()) return &it->second;
    hipDeviceProp_t prop;
    if (hipGetDeviceProperties(&prop, dev) != hipSuccess) return nullptr;
    DeviceId id;
    // (the marketing name is left out: it comes from a system file that may be missing, and then
    //  differs from one process to the next)
    snprintf(id.name, sizeof(id.name), "%s|%dCU", prop.gcnArchName, prop.multiProcessorCount);
    for (char* c = id.name; *c; ++c)
        if (*c == ' ' || *c == '\n') *c = '_';   // one token in the cache file
    id.hash = (int)(fnv(2166136261u, id.name, strlen(id.name)) & 0x7fffffffu);
    return &ids.emplace(dev, id).first->second;
}

// kinds 8 (sparse instruction) and 9 (dense): fp32 tensors as three bf16 planes
inline bool is_split_kind(int kind) { return kind == 8 || kind == 9; }
// kinds 10 (bf16) and 11 (fp32): few input channels out of staged rows
inline bool is_rows_kind(int kind) { return kind == 10 || kind == 11; }
// kinds 13 (sparse instruction) and 14 (dense): bf16, a tile's input staged once for all taps
inline bool is_taps_kind(int kind) { return kind == 13 || kind == 14; }
// kinds 15 and 16: the three planes of 8 and 9, a tile's input staged once for all taps
inline bool is_split_taps_kind(int kind) { return kind == 15 || kind == 16; }
// wavefronts of a workgroup along the output channels
inline int channel_waves(const VariantDesc& d)
{
    if (is_split_taps_kind(d.kind)) return 8 / d.waves / d.WP;
    return (is_taps_kind(d.kind) && d.waves == 8 ? 8 : 4) / d.WP;
}
// kinds whose row blocks are 16 consecutive output channels, whatever the column tile
inline bool flat_rowblocks(int kind) { return is_split_kind(kind) || is_rows_kind(kind) || is_split_taps_kind(kind); }

// Which variants may run a layer depends on its weights, not only on its shape: the
// k-steps per chunk its kept sets need (groups wider than a chunk spread unevenly) and
// which operand tables were built.  Two layers of one shape that differ there must not
// share a cache entry.
int prepack_signature(const nm_packed* wp, bool no_planes)
{
    unsigned h = no_planes ? 2166136262u : 2166136261u;
    for (const Prepack& pp : wp->prepacks) {
        const int t[5] = {pp.kind, pp.geom.CK, pp.geom.vec, pp.SPC, pp.par};
        if (!flat_rowblocks(pp.kind)) h = fnv(h, t, sizeof(t));   // (implied by the rest of the key)
    }
    return (int)(h & 0x7fffffffu);
}

ShapeKey make_key(nm_dtype_t xdt, nm_dtype_t ydt, int b, int h, int w, const nm_packed* wp,
                  int sh, int sw, int ph, int pw, int dh, int dw, int has_bias, int relu)
{
    ShapeKey k;
    const int vals[kKeyInts] = {(int)xdt, (int)ydt, b, h, w, wp->cin, wp->cout, wp->kh, wp->kw,
                                sh, sw, ph, pw, dh, dw, wp->n, wp->m, wp->tile, (int)wp->value_dtype,
                                has_bias ? 1 : 0, relu ? 1 : 0, wp->device_hash, wp->sig, 0};
    memcpy(k.v, vals, sizeof(vals));
    return k;
}

constexpr size_t kRowsPieces = 4 * kRowsPiece;   // kinds 10, 11: the output pieces of four wavefronts

// LDS footprint of variant d on the layer wp (the ring of the gather-free bf16
// kernel is only as deep as the layer's K loop is long).
size_t lds_bytes(const VariantDesc& d, const nm_packed* wp)
{
    // the epilogue's output tile [BP][channels of the workgroup] plus 16 bytes per pixel
    const size_t otile = (size_t)d.BP * ((size_t)(4 / d.WP) * d.NJ * 16 * (d.kind == 0 || d.kind == 5 ? 4 : 2) + 16);
    if (is_split_kind(d.kind)) return (size_t)split_lds_bytes(d.NBLK, d.WP, d.NJ);
    if (is_taps_kind(d.kind)) return taps_lds_bytes(d.NBLK, d.WP, d.NJ, 9 * d.BP, 1, channel_waves(d) * d.WP);   // and what depends on the image
    if (is_split_taps_kind(d.kind)) return split_taps_lds_bytes(d.NBLK, d.NJ, d.waves, 9 * d.BP, 1);
    if (d.kind == 17) return (size_t)cols_lds_bytes(d.NBLK, d.waves);
    if (d.kind == 12) return (size_t)wave_lds_bytes(d.NBLK, d.NJ, d.CK, d.waves);
    if (is_rows_kind(d.kind)) return kRowsPieces;   // and the staged rows, which depend on the image (rows_layout)
    if (d.kind == 6)   // only the wavefront-private output tiles [16 NBLK][16 NJ] bf16 with 16 bytes of padding per row
        return (size_t)4 * 16 * d.NBLK * (d.NJ * 32 + 16);
    if (d.kind == 7) {   // up to three stages of the strip [BP][CK] bytes plus each wave's operands (1 KB per k-step and row block)
        const int nchunks = wp->kh * wp->kw * ((wp->cin + d.CK - 1) / d.CK);
        const size_t ops = d.areg ? 0 : (size_t)4 * d.NJ * (d.CK / 64) * 1024;
        return std::max(otile, (size_t)std::min(3, nchunks) * ((size_t)d.BP * d.CK + ops));
    }
    if (d.kind == 4)   // the strip [BP][64 SPC] bf16 plus the dense weights of the workgroup's row blocks
        return std::max(otile, (size_t)d.BP * d.SPC * 128 + (size_t)(4 / d.WP) * d.NJ * d.SPC * 2048);
    if (d.kind >= 2 && d.kind <= 4) {   // up to three stages of the strip [BP][CK] bf16 plus each wave's operands
        const int nchunks = wp->kh * wp->kw * ((wp->cin + d.CK - 1) / d.CK);
        const size_t ops = d.areg ? 0 : (size_t)4 * d.NJ * (d.CK / 64) * (d.kind == 2 ? 1024 + 256 : 2048);
        return std::max(otile, (size_t)std::min(3, nchunks) * ((size_t)d.BP * d.CK * 2 + ops));
    }
    if (d.kind == 1) {
        const int opr = d.CK / 8, pstep = 256 / opr, nit = (d.BP * opr + 255) / 256;
        const int rows = nit * pstep > d.BP ? nit * pstep : d.BP;
        return std::max(otile, (size_t)2 * rows * (d.CK * 2 + 4));
    }
    return std::max(otile, (size_t)2 * d.CK * strip_stride(d.BP, d.CK, d.vec != 0) * sizeof(float));
}

// The part of the convolution arguments that decides whether the kernels for few input
// channels apply and which of their two operand tables they need.
struct RunArgs {
    int w, sw, pw, dw, sh, dh, ph, h, b;
};

// Elements of lead-in, 0 or 1, that put a kernel-row run on 4 bytes.
int run_par(int pw, int cin) { return (int)((long)pw * cin % 2); }

// Layout of the staged rows of kinds 10 and 11 (bytes of one plane; the data starts on 16 bytes, the run of
// column 0 at `front`, 2 * lead bytes before it).  Worked out in 64 bits, since any padding and stride may be
// asked for: a layout that fits the LDS fits an int.
struct RowsLayout {
    int n, pitch, front, data;
    size_t lds;   // all planes, whole 1 KB windows; (size_t)-1 and nothing else where they do not fit
};
RowsLayout rows_layout(const VariantDesc& d, const nm_packed* wp, const RunArgs& ra)
{
    const int par = run_par(ra.pw, wp->cin);
    const long lead = (long)ra.pw * wp->cin + par, gr = (par + wp->kw * wp->cin + 7) / 8;
    const long wo = (ra.w + 2L * ra.pw - wp->kw) / ra.sw + 1;
    const long n = (d.NBLK - 1L) * ra.sh + (wp->kh - 1L) * ra.dh + 1;
    const long data = (2 * lead + 15) / 16 * 16, front = data - 2 * lead;
    const long end = std::max(data + 2L * ra.w * wp->cin, front + 2 * (wo - 1) * ra.sw * wp->cin + gr * 16);
    const long pitch = (end + 15) / 16 * 16;
    RowsLayout r = {0, 0, 0, 0, (size_t)-1};
    if (n > kMaxLdsBytes || pitch > kMaxLdsBytes) return r;
    r.n = (int)n; r.pitch = (int)pitch; r.front = (int)front; r.data = (int)data;
    r.lds = (size_t)((n * pitch * (d.kind == 10 ? 1 : 3) + 1023) / 1024 * 1024);
    return r;
}

// k-steps the kernel-row-run kernel needs for this layer when runs start `par` elements early
int run_ksteps(const nm_packed* wp, int par)
{
    const int gr = (par + wp->kw * wp->cin + 7) / 8;
    return (wp->kh * gr + 7) / 8;
}

// kind 12 reads the tables of kind 0, kind 17 those of 2, kinds 13 and 14 those of 2 and 3, kinds 15 and 16 those of 8 and 9
inline int table_kind(int kind) { return kind == 12 ? 0 : kind == 17 ? 2 : is_taps_kind(kind) ? kind - 11 : is_split_taps_kind(kind) ? kind - 7 : kind; }

const Prepack* find_prepack(const nm_packed* wp, const VariantDesc& d, int par = -1)
{
    for (const Prepack& pp : wp->prepacks)
        if (pp.kind == table_kind(d.kind) && (d.kind != 12 || pp.d_cols) && pp.geom.CK == d.CK && pp.geom.vec == d.vec && pp.SPC == d.SPC &&
            (d.vec || pp.d_ktab) && ((d.kind != 4 && !is_rows_kind(d.kind)) || par < 0 || pp.par == par))
            return &pp;
    return nullptr;
}

// kinds 6 (register-streaming) and 7 (LDS-staged) are the fp8 kernels; they share one operand table layout
inline bool is_f8_kind(int kind) { return kind == 6 || kind == 7; }

// With `ra` the answer is for that convolution; without, "for some convolution" (the tap-staged kinds: no, since nearly all
// that decides about them is in the call).
bool variant_legal(int v, const nm_packed* wp, nm_dtype_t xdt, const RunArgs* ra = nullptr)
{
    if (v < 0 || v >= variant_count()) return false;
    const VariantDesc& d = variant_desc(v);
    if (lds_bytes(d, wp) > (size_t)kMaxLdsBytes) return false;
    if ((d.kind == 5 || d.kind == 11 || d.kind == 12 || is_split_kind(d.kind) || is_split_taps_kind(d.kind)) && xdt != NM_F32) return false;   // instantiated for fp32 tensors only
    // fp8: E4M3 tensors with an E4M3 handle run the fp8 kernels and nothing else does
    if (is_f8_kind(d.kind) != (xdt == NM_F8E4M3) || is_f8_kind(d.kind) != (wp->value_dtype == NM_F8E4M3)) return false;
    if ((d.kind >= 1 && d.kind <= 4) || d.kind == 10 || d.kind == 17 || is_taps_kind(d.kind)) {
        // bf16 matrix cores: bf16 tensors, weights already rounded to bf16, and a
        // shared operand only for column tiles made of exactly two row blocks
        if (xdt != NM_BF16 || wp->value_dtype != NM_BF16) return false;
        if (d.share != 1 && d.share != wp->rbpt) return false;
    }
    if (is_rows_kind(d.kind) && wp->cout % (d.kind == 10 ? 8 : 4) != 0) return false;   // whole 16-byte output granules
    if (d.kind == 17) {   // 1x1 without padding, this many input channels; whole row blocks and 16-byte output granules
        if (!ra || ra->ph != 0 || ra->pw != 0 || wp->kh != 1 || wp->kw != 1 || wp->cin != 64 * d.waves) return false;
        if (wp->tile % 16 != 0 || wp->cout % 8 != 0) return false;
    }
    if (is_taps_kind(d.kind) || is_split_taps_kind(d.kind)) {
        // an output as large as the input, so that a tap is one shift of the whole tile; whole 16-byte output granules
        if (!ra || ra->sh != 1 || ra->sw != 1 || wp->kh * wp->kw < 2 || wp->kh * wp->kw > 32) return false;
        if (2L * ra->ph != (long)ra->dh * (wp->kh - 1) || 2L * ra->pw != (long)ra->dw * (wp->kw - 1)) return false;
        if (is_taps_kind(d.kind) && (wp->tile % 16 != 0 || wp->cout % 8 != 0)) return false;
        if (is_split_taps_kind(d.kind) && (wp->cin % 64 != 0 || wp->kh * wp->kw < d.waves)) return false;
        // (small enough for what follows, and for the kernel's products of 24 bits and quotients of 31)
        if (ra->ph > 1000 || ra->pw > 1000 || ra->w > 3000) return false;
        const double lines = (ra->b + 2.0) * ((double)ra->h + ra->ph);
        if (lines >= 16777216.0 || lines * taps_line(ra->w, ra->pw) >= 2147483648.0) return false;
        const long granules = taps_granules(d.BP, ra->h, ra->w, ra->ph, ra->pw);
        if (is_split_taps_kind(d.kind)) {
            if (split_taps_lds_bytes(d.NBLK, d.NJ, d.waves, granules, wp->cin / 64) > (size_t)kMaxLdsBytes) return false;
            if (wp->cin > 64 && taps_loads(granules) > 8 * kSplitTapsItems) return false;
        } else if (taps_lds_bytes(d.NBLK, d.WP, d.NJ, granules, wp->cin / 64, channel_waves(d) * d.WP) > (size_t)kMaxLdsBytes) return false;
        if (is_taps_kind(d.kind) && d.waves == 8 && taps_loads(granules) > 8 * kTapsWideLoads) return false;
    }
    if (d.ksplit > 1) {
        // every split must own at least one chunk of the K axis
        const Prepack* pp = find_prepack(wp, d);
        if (!pp) return false;
        const int cps = (pp->geom.nchunks + d.ksplit - 1) / d.ksplit;
        if ((d.ksplit - 1) * cps >= pp->geom.nchunks) return false;
    }
    if ((d.kind == 4 || is_rows_kind(d.kind)) && ra) {
        // a kernel row must be one contiguous, 4-byte aligned run of every pixel
        if (ra->dw != 1 || ((long)ra->sw * wp->cin) % 2 != 0 || ((long)ra->w * wp->cin) % 2 != 0) return false;
        if (is_rows_kind(d.kind) && rows_layout(d, wp, *ra).lds > (size_t)kMaxLdsBytes - kRowsPieces) return false;
        return find_prepack(wp, d, run_par(ra->pw, wp->cin)) != nullptr;
    }
    return find_prepack(wp, d) != nullptr;
}

// Three planes take the place of the fp32 instruction only where that loses nothing: they leave out three of the nine
// partial products (about one fp32 rounding of each product), and their fewer roundings of the sum make up for it from
// some number of kept columns on.  Distance from float64 over the fp32 instruction's, 1x1 and small kernels, worst of
// uniform and signed activations, with bias and without: 1 column x1.95, 2 x1.5, 3 x1.3, 4 x1.2, 5 x1.02, 6 x1.01,
// 7 x0.94, 9 x0.91, 18 x0.8 and falling.  Of a K split each part counts.  (A forced variant runs all the same.)
constexpr int kPlanesMinKept = 7;
bool keeps_precision(int v, const nm_packed* wp)
{
    const VariantDesc& d = variant_desc(v);
    if (!is_split_kind(d.kind) && !is_split_taps_kind(d.kind) && d.kind != 11) return true;
    long kept = wp->kprime;
    if (is_split_taps_kind(d.kind)) return kept / d.waves >= kPlanesMinKept;
    if (d.ksplit > 1) {
        const int nchunks = wp->kh * wp->kw * ((wp->cin + d.CK - 1) / d.CK);
        kept = kept * ((nchunks + d.ksplit - 1) / d.ksplit) / nchunks;
    }
    return kept >= kPlanesMinKept;
}

// Largest number of kept columns any (tile, chunk) pair holds.  Kept positions ascend inside a
// tile, so a chunk's columns are one run: the chunk is worked out once per run, not per column.
int max_kept_per_chunk(const nm_packed* wp, const ChunkGeom& g)
{
    // Whole groups to a chunk (and to a tap, where chunks do not cross taps): what a group keeps, times the groups of the longest.
    // (Counted, the two chunk lengths of a 512x3x3x512 layer took 0.10 ms of 0.63.)
    const int most = std::min(g.CK, g.vec ? wp->cin : wp->K);
    if (g.CK % wp->m == 0 && (!g.vec || wp->cin % wp->m == 0)) return most / wp->m * wp->n;
    int best = 0;
    for (int j = 0; j < wp->n_tiles; ++j) {
        const int32_t* idx = wp->h_idx.data() + (size_t)j * wp->kprime;
        int cnt = 0, end = 0;   // columns of the current chunk, first k beyond it
        for (int kk = 0; kk < wp->kprime; ++kk) {
            const int k = idx[kk];
            if (k >= end) {
                if (g.vec) {
                    const int tap = k / wp->cin, ci = k - tap * wp->cin;
                    end = tap * wp->cin + std::min(wp->cin, (ci / g.CK + 1) * g.CK);
                } else {
                    end = (k / g.CK + 1) * g.CK;
                }
                cnt = 0;
            }
            best = std::max(best, ++cnt);
        }
    }
    return best;
}

// What nm_prune works out once per chunk geometry, however many variants share it.
struct GeomNeeds {
    const nm_packed* wp;
    struct Kept { int CK, vec, most; };
    struct Pick { int kind, CK, vec, spc; };
    std::vector<Kept> kept;
    std::vector<Pick> picks;

    int max_kept(const ChunkGeom& g)
    {
        for (const Kept& k : kept)
            if (k.CK == g.CK && k.vec == g.vec) return k.most;
        kept.push_back({g.CK, g.vec, max_kept_per_chunk(wp, g)});
        return kept.back().most;
    }
    // smallest instantiated number of k-steps per chunk that holds the layer's kept columns (0: none)
    int steps(const VariantDesc& d, const ChunkGeom& g)
    {
        for (const Pick& p : picks)
            if (p.kind == d.kind && p.CK == d.CK && p.vec == d.vec) return p.spc;
        const int per_step = d.kind == 1 ? 32 : 4;   // kept columns per k-step
        const int need = (max_kept(g) + per_step - 1) / per_step;
        int pick = 0;
        for (int u = 0; u < variant_count(); ++u) {
            const VariantDesc& e = variant_desc(u);
            if (e.kind == d.kind && e.CK == d.CK && e.vec == d.vec && e.SPC >= need && (pick == 0 || e.SPC < pick))
                pick = e.SPC;
        }
        picks.push_back({d.kind, d.CK, d.vec, pick});
        return pick;
    }
};

// Index of the first NaN or infinity, n if there is none.  The pass that decides has no exit, so that it runs on
// vector registers.
size_t first_not_finite(const float* w, size_t n)
{
    const uint32_t top = 0x7f800000u;
    uint32_t bad = 0;
    for (size_t i = 0; i < n; ++i) {
        uint32_t u;
        memcpy(&u, w + i, sizeof(u));
        bad |= (u & top) == top ? 1u : 0u;
    }
    if (!bad) return n;
    size_t i = 0;
    while (i < n && isfinite(w[i])) ++i;
    return i;
}

// Outputs below this (as a word shifted left by one) are computed again by the three-plane kernels where they meet
// activations under 2^-110: what the planes of those lose, 2^-132 |w| a product, is then more than 2^-27 of the output.
unsigned redo_below(float max_w, int kprime)
{
    const float t = (float)std::min(std::max(ldexp((double)max_w * kprime, -105), ldexp(1.0, -100)), 3e38);
    uint32_t u;
    memcpy(&u, &t, sizeof(u));
    return u << 1;
}

struct Geometry {
    int Ho, Wo, P;
};

int conv_geometry(int b, int h, int w, const nm_packed* wp, int sh, int sw, int ph, int pw, int dh,
                  int dw, size_t es, Geometry* g)
{
    if (b < 1 || h < 1 || w < 1 || sh < 1 || sw < 1 || ph < 0 || pw < 0 || dh < 1 || dw < 1) {
        set_error("bad convolution arguments (sizes, stride, dilation must be >= 1, padding >= 0)");
        return NM_ERR_ARG;
    }
    const long eh = (long)h + 2L * ph - (long)dh * (wp->kh - 1) - 1;
    const long ew = (long)w + 2L * pw - (long)dw * (wp->kw - 1) - 1;
    if (eh < 0 || ew < 0) {
        set_error("output would be empty: input %dx%d, kernel %dx%d, pad %d,%d, dilation %d,%d", h, w,
                  wp->kh, wp->kw, ph, pw, dh, dw);
        return NM_ERR_SHAPE;
    }
    g->Ho = (int)(eh / sh) + 1;
    g->Wo = (int)(ew / sw) + 1;
    const long long P = (long long)b * g->Ho * g->Wo;
    const long long xin = (long long)b * h * w * wp->cin;
    const long long yout = P * wp->cout;
    if (P > 0x7fffffffLL - 1024 || xin > 0x7fffffffLL || yout > 0x7fffffffLL) {
        set_error("tensor too large: more than 2^31 - 1 elements");
        return NM_ERR_SHAPE;
    }
    if (xin * (long long)es >= 0x80000000LL) {
        set_error("input tensor too large: the kernels address x through a 2 GiB buffer window");
        return NM_ERR_SHAPE;
    }
    g->P = (int)P;
    return NM_OK;
}

// x / d for x < 2^31 as umulhi(2 x, mul) >> shift: shift = ceil(log2 d) and
// mul = floor(2^(31 + shift) / d) + 1, which fits 32 bits and is exact on that range.
void magic_div(unsigned d, unsigned* mul, unsigned* shift)
{
    unsigned s = 0;
    while ((1ull << s) < d) ++s;
    *mul = (unsigned)(((1ull << (31 + s)) / d) + 1);
    *shift = s;
}

// Whether an output of so many bytes is stored past the caches: where the 256 MB last-level cache would not hold it (and the
// rest of a layer's tensors) until the next layer reads it.  Whole networks, called again and again, no output past the caches,
// those over 256 MB, those over 150: ResNet-101 in bf16 at batch 256 5742, 5672 and 5632 us, ResNet-50 in bf16 at batch 96 1561,
// 1563 and 1532, in fp32 at batch 64 2785, 2782 and 2770; called once after other memory has been filled, the same order
// (5767, 5710, 5670) or no difference.  By themselves such layers gain nothing, and lose where the cache is full of what others
// wrote: bf16 56x56 64 -> 256 with a residual, through and past, repeated 74 and 71 us (167 MB), 88 and 85 (206), once after a fill
// 105 and 114, 122 and 140.
// First layers (kinds 10 and 11) are read by the pool at once, and not as a residual later: past only where the cache does not hold
// the output.  In bf16, left to the L2 (keep_output) and past: the layer and its pool, 77, 103, 128, 180, 206 and 257 MB, on three
// tensors in turn 40 and 50, 56 and 64, 78 and 76, 103 and 108, 116 and 113, 143 and 137, on one 38 and 44, 51 and 59, 58 and 69, 92 and
// 95, 97 and 103, 138 and 129; ResNet-18, 77, 103, 134, 154, 206 and 257 MB, 354 and 358, 417 and 426, 462 and 478, 550 and 557, 678
// and 681, 775 and 769, once after a fill 371 and 382, 435 and 449, 486 and 512, 563 and 596, 703 and 719, 803 and 799; ResNet-50, 103,
// 134, 154, 206 and 257 MB, 1123 and 1132, 1334 and 1328, 1536 and 1541, 1911 and 1916, 2264 and 2253.  (The first layer alone, whose
// output nobody reads, is faster past them where it does not find its output in the cache: 128 MB on three tensors in turn 43 and 39,
// on one 35 and 37.)  fp32, through and past, with the pool on three tensors 206, 254 and 308 MB 154 and 156, 197 and 194, 242 and 236.
bool stream_output(int kind, double bytes) { return bytes > (is_rows_kind(kind) ? 256e6 : 150e6); }

// Whether kind 10 leaves its output to the L2's own write-back: stores that pass the L2 one by one slow a first layer in bf16 down from
// about 72 MB on (likely where it writes faster than the memory behind takes them).  The layer on three tensors in turn,
// through and kept, 13, 38, 51, 64, 77, 82, 103, 128, 149 and 180 MB: 8.1 and 9.0, 13.3 and 15.0, 17.2 and 18.3, 21.2 and 22.2, 27.2
// and 24.4, 32.4 and 29.8, 39.4 and 37.1, 44.8 and 43.0, 55.1 and 52.7, 65.2 and 62.4 us; with the pool, 38 to 180 MB, 22.5 and 24.3,
// 28.7 and 29.2, 37.7 and 35.9, 41.8 and 40.3, 50.9 and 48.2, 57.1 and 55.8, 79.6 and 77.7, 94.2 and 93.3, 105.5 and 103.2; ResNet-18, 51,
// 77, 103, 154 and 206 MB 281 and 282, 356 and 354, 421 and 417, 555 and 550, 683 and 678.  (fp32, whose arithmetic takes longer, is
// faster through the L2 up to 51 MB and the same beyond.)
bool keep_output(int kind, double bytes) { return kind == 10 && bytes > 72e6 && !stream_output(kind, bytes); }

// Groups of 256 output channels that a workgroup of kind 17 walks: all of them where the pixel tiles alone are three quarters of the
// CUs' places (two a CU) or more, else an equal part of them, of as many parts as that takes, rounded up to whole groups (so that there
// may be fewer workgroups: 130 tiles and four groups are three parts, walks of two groups, 260 of 384).  14x14 256 -> 1024 with a residual, 1, 2 and 4 groups: batch 256 (784 pixel tiles) 67.7, 60.4 and 61.0
// us, batch 64 19.2, 16.2 and 19.0.
int cols_walk(int n_ptiles, int n_cblocks)
{
    const int parts = (3 * kNumCU / 2 + n_ptiles - 1) / n_ptiles;
    return parts >= n_cblocks ? 1 : (n_cblocks + parts - 1) / parts;
}

void fill_params(ConvParams& p, const VariantDesc& d, const Prepack& pp, const nm_packed* wp,
                 const void* x, void* y, const float* bias, int b, int h, int w, const Geometry& g,
                 int sh, int sw, int ph, int pw, int dh, int dw, int relu, size_t es)
{
    p.x = x; p.y = y; p.bias = bias; p.res = nullptr;
    p.wfrag = pp.d_wfrag; p.rows = pp.d_rows; p.ktab = pp.d_ktab;
    p.wfrag_bytes = (unsigned)pp.wfrag_bytes; p.rows_bytes = (unsigned)pp.rows_bytes;
    p.B = b; p.H = h; p.W = w; p.Cin = wp->cin; p.Cout = wp->cout; p.Kh = wp->kh; p.Kw = wp->kw;
    p.Ho = g.Ho; p.Wo = g.Wo;
    p.sh = sh; p.sw = sw; p.ph = ph; p.pw = pw; p.dh = dh; p.dw = dw;
    p.relu = relu ? 1 : 0;
    const double ybytes = (double)g.P * wp->cout * (es == 4 ? 4 : 2);   // (fp8 layers write bf16)
    p.stream = stream_output(d.kind, ybytes) ? 1 : 0;
    p.keep = keep_output(d.kind, ybytes) ? 1 : 0;
    p.P = g.P; p.K = wp->K;
    p.nchunks = pp.geom.nchunks; p.ncpt = pp.geom.ncpt;
    p.tile = wp->tile; p.rbpt = wp->rbpt; p.n_rowblocks = wp->n_rowblocks;
    if (flat_rowblocks(d.kind)) {
        p.tile = 16; p.rbpt = 1; p.n_rowblocks = (wp->cout + 15) / 16;
    }
    p.idx = wp->d_idx; p.vals = wp->d_vals; p.kprime = wp->kprime; p.ctile = wp->tile;
    p.redo_below = wp->redo_below;
    const int rb_per_wg = channel_waves(d) * d.NJ;
    p.n_ptiles = (g.P + d.BP - 1) / d.BP;
    p.n_cblocks = (p.n_rowblocks + rb_per_wg - 1) / rb_per_wg;
    p.oscale = 1.0f / wp->scale;
    p.ksplit = d.ksplit > 1 ? d.ksplit : 1;
    p.cps = (pp.geom.nchunks + p.ksplit - 1) / p.ksplit;
    p.px_fast = 0;
    if (d.kind == 12) {
        p.rows = reinterpret_cast<const uint32_t*>(pp.d_cols);
        p.rows_bytes = (unsigned)pp.cols_bytes;
        p.cps = (pp.geom.nchunks + d.waves - 1) / d.waves;   // chunks of a wavefront
        p.waves = (pp.geom.nchunks + p.cps - 1) / p.cps;       // those that have a chunk
        p.px_fast = pp.wfrag_bytes > (size_t)b * h * w * wp->cin * es ? 1 : 0;
        magic_div((unsigned)(p.px_fast ? p.n_ptiles : p.n_cblocks), &p.fast_mul, &p.fast_shift);
        magic_div((unsigned)pp.geom.ncpt, &p.ncpt_mul, &p.ncpt_shift);
        magic_div((unsigned)wp->kw, &p.kw_mul, &p.kw_shift);
        magic_div((unsigned)wp->rbpt, &p.rbpt_mul, &p.rbpt_shift);
    }
    if (is_taps_kind(d.kind) || is_split_taps_kind(d.kind)) {
        magic_div((unsigned)wp->kw, &p.kw_mul, &p.kw_shift);
        p.rows_n = (int)taps_granules(d.BP, h, w, ph, pw);
        p.rows_lds = taps_loads(p.rows_n) * 1024;
        magic_div((unsigned)taps_line(w, pw), &p.padw_mul, &p.padw_shift);
        magic_div((unsigned)(h + ph), &p.padh_mul, &p.padh_shift);
    }
    p.partial = nullptr;   // the caller points it at a workspace of split_bytes()
    if (is_rows_kind(d.kind)) {
        const RowsLayout r = rows_layout(d, wp, RunArgs{w, sw, pw, dw, sh, dh, ph, h, b});
        p.rows_r = d.NBLK; p.rows_n = r.n; p.rows_pitch = r.pitch; p.rows_front = r.front; p.rows_data = r.data;
        p.rows_lds = (int)r.lds;
        magic_div((unsigned)(r.pitch / 16), &p.rowg_mul, &p.rowg_shift);
        p.n_ptiles = b * ((g.Ho + d.NBLK - 1) / d.NBLK);
    }
    p.n_wg = p.n_ptiles * p.n_cblocks * p.ksplit;
    if (d.kind == 17) {
        magic_div((unsigned)wp->rbpt, &p.rbpt_mul, &p.rbpt_shift);
        p.cps = cols_walk(p.n_ptiles, p.n_cblocks);
        p.n_wg = p.n_ptiles * ((p.n_cblocks + p.cps - 1) / p.cps);
    }
    p.wg_per_xcd = (p.n_wg + 7) / 8;
    magic_div((unsigned)(g.Ho * g.Wo), &p.howo_mul, &p.howo_shift);
    magic_div((unsigned)g.Wo, &p.wo_mul, &p.wo_shift);
    p.x_elems = (unsigned)((size_t)b * h * w * wp->cin);
    p.x_bytes = (unsigned)((size_t)b * h * w * wp->cin * es);
    p.run_d = pp.par;
    p.run_gr = (pp.par + wp->kw * wp->cin + 7) / 8;
    magic_div((unsigned)p.run_gr, &p.gr_mul, &p.gr_shift);
    magic_div((unsigned)wp->cin, &p.cin_mul, &p.cin_shift);
}

// The variants without a K split, in table order: what an untuned call chooses from.  Of these only the kinds
// that the handle has operand tables for are looked at: the choice is made at the first untuned call of a shape (and where a
// full table has forgotten it), and a look at all 1500 variants took 20 us of it.
const std::vector<int>& base_variants()
{
    static const std::vector<int> t = [] {
        std::vector<int> r;
        for (int v = 0; v < variant_count(); ++v)
            if (variant_desc(v).ksplit <= 1) r.push_back(v);
        return r;
    }();
    return t;
}
// Those of one kind (a look at all of them is 1.5 us).
const std::vector<int>& variants_of(int kind)
{
    static const std::vector<std::vector<int>> t = [] {
        std::vector<std::vector<int>> r(32);
        for (int v : base_variants()) r[(size_t)variant_desc(v).kind].push_back(v);
        return r;
    }();
    return t[(size_t)kind];
}
unsigned kinds_of(const nm_packed* wp)
{
    unsigned m = 0;
    for (const Prepack& pp : wp->prepacks) m |= 1u << pp.kind;
    return m;
}

// The tap-staged form of a layer on three planes that runs without tuning, -1 where the strip-per-tap one does it: the cheaper of two and four groups by rounds of
// workgroups (one a CU) x (14 000 clocks of start and output + 1.2 x the matrix instructions), in one round where that fills
// half of the CUs and two thirds of the channels exist; in more with three quarters of them, a last round that is not mostly
// empty, and a sum long enough to pay for a staging that nothing else runs beside.  Of 136 random 3x3 layers that the
// rule below does on three planes 32 on the sparse instruction take x0.78 to x1.01 of their time, x0.88 on average, and 59 on
// the dense one x0.66 to x0.99, x0.87; with several rounds of 9 to 27 chunks it would be x1.02 to x1.27.
int split_taps_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra, bool sparse)
{
    int pick = -1;
    double best = 0;
    const int chunks = wp->K / 64;
    for (int v : variants_of(sparse ? 15 : 16)) {
        const VariantDesc& d = variant_desc(v);
        if (!keeps_precision(v, wp) || !variant_legal(v, wp, xdt, ra)) continue;
        const int channels = channel_waves(d) * d.NJ * 16;
        const long n_cb = (wp->cout + channels - 1) / channels, n_wg = (long)((P + d.BP - 1) / d.BP) * n_cb;
        const long rounds = (n_wg + kNumCU - 1) / kNumCU;
        if (rounds == 1 && (2 * n_wg < kNumCU || 3L * wp->cout < 2L * n_cb * channels)) continue;
        if (rounds > 1 && (chunks < (sparse ? 36 : 27) || 4L * wp->cout < 3L * n_cb * channels || 5L * rounds * kNumCU > 7L * n_wg)) continue;
        const double cost = rounds * (14000.0 + 1.2 * 12 * 16 * d.NBLK * d.NJ * (sparse ? 1 : 2) * chunks / d.waves);
        if (pick < 0 || cost < best) {
            pick = v;
            best = cost;
        }
    }
    return pick;
}

// The three-plane form of an fp32 layer that runs without tuning, -1 where the fp32 instruction does it.
//
// Clocks of the matrix cores per 64 channels and 16 x 16 outputs: 16 x 32 times the kept fraction on the fp32
// instruction (more where T leaves rows of its 16 empty), 6 x 16 on the sparse bf16 one, 12 x 16 on the dense one;
// what surrounds them costs the three-plane kernel as much again.  Measured over 210 random layers (1:4, 2:4, 1:8,
// 2:8, 4:8 and half of all channels, T 8 to 32, 100 to 180 000 pixels), fp32 instruction against three planes:
//   sparse, 256 clocks and more (2:4; 1:4 at T = 8): x1.04 to x1.7 faster on every layer;
//           128 clocks (1:4, 2:8): x0.66 to x1.13, 64 clocks (1:8): x0.78 to x1.0
//   dense, 256 clocks (4:8, half of all channels): x1.04 to x1.5 from 300 000 outputs and 128 channels on, x0.9 below
//   fewer than 48 channels (a chunk of 64 mostly empty): x0.6 to x0.9
// and the ends of the first range at ResNet-50's sizes: 64 output channels and at most 9 chunks are x0.9 to x0.97.
// Tiles: 64 pixels x 128 channels where they give every CU one, else 32 pixels, else 32 x 64; 64 channels
// where the layer has no more, or where (dense form) 128 would leave more than an eighth of them empty.
int split_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra)
{
    if (wp->cin < 48) return -1;
    const double fp32_clocks = 512.0 * wp->n / wp->m * (16.0 * wp->rbpt / wp->tile);
    const int cout = wp->cout;
    const bool sparse = wp->n <= 2 && wp->m % 4 == 0;
    if (fp32_clocks < 256.0) return -1;
    if (sparse && cout <= 64 && wp->kh * wp->kw * ((wp->cin + 63) / 64) <= 9 && P > 16 * kNumCU) return -1;
    if (!sparse && fp32_clocks < 512.0 && (cout < 128 || (long)P * cout < 300000)) return -1;
    const int taps = split_taps_default(wp, P, xdt, ra, sparse);
    if (taps >= 0) return taps;
    const int c64 = (cout + 63) / 64, c128 = (cout + 127) / 128;
    const bool wide = cout > 64 && (sparse || 16 * c128 <= 9 * c64);
    const long t64 = (long)((P + 63) / 64) * (wide ? c128 : c64), t32 = (long)((P + 31) / 32) * c128;
    const int nblk = t64 >= kNumCU ? 4 : 2, nj = wide && (nblk == 4 || t32 >= 100) ? 2 : 1;
    for (int v : base_variants()) {
        const VariantDesc& d = variant_desc(v);
        if (is_split_kind(d.kind) && d.NBLK == nblk && d.WP == 1 && d.NJ == nj && variant_legal(v, wp, xdt, ra))
            return v;
    }
    return -1;
}

// The row-staged form of a layer with few input channels that runs without tuning: as many output rows a
// workgroup as leave every CU two workgroups, at most 8 in bf16 and 4 in fp32 (the planes' LDS).  Measured on the
// 224x224x3 -> 64 7x7 layer, 1, 2, 4, 8 rows: bf16 batch 64 58, 47, 39, 36 us (a strip of runs per pixel: 80), batch 1
// 5.6, 6.7, 8.6, 12.7 (5.6); fp32 batch 64 146, 121, 112, 155 (element-wise: 190), batch 1 10.2, 13.2, 20.6, 35 (9.7).
int rows_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs& ra)
{
    const int wo = (int)((ra.w + 2L * ra.pw - (long)ra.dw * (wp->kw - 1) - 1) / ra.sw) + 1;
    int pick = -1;
    for (int v : base_variants()) {
        const VariantDesc& d = variant_desc(v);
        if (!is_rows_kind(d.kind) || !keeps_precision(v, wp) || !variant_legal(v, wp, xdt, &ra)) continue;
        const long n_wg = (long)(P / wo + d.NBLK - 1) / d.NBLK * ((wp->cout + 63) / 64);
        if (d.NBLK > (d.kind == 10 ? 8 : 4) || (d.NBLK > 1 && n_wg < 2L * kNumCU)) continue;
        // (within one form the table lists the heights in ascending order, and the wider form last)
        pick = v;
    }
    return pick;
}

// The tap-staged form of a bf16 layer that runs without tuning, -1 where the others do it: the cheapest by rounds of
// workgroups (one a CU) x (12 000 clocks of start and output + 1.2 x the matrix instructions of its chunks; 11 000 and 1.14
// with eight contracting wavefronts), where that
// gives at least 176 CUs a workgroup of 224 pixels or more (224 CUs one of 160), more than half of its channels exist and
// the launch is not a round and less than 0.4 of a second one.  Of 600 random 3x3 layers, sparse instruction, tensors out of
// cache, the 393 within that take x0.58 to x1.00 of the time that the rule below gives them, x0.82 on average; where just
// half of the channels exist (128 of 256) it would be x1.26 to x1.35, at 1.16 rounds x1.11.  Eight wavefronts: of 220 such
// layers the 82 that go from a form of four to one of eight take x0.73 to x1.07 of its time, x0.85 on average.
// The dense instruction (layers that the sparse one does not do): the forms of eight wavefronts alone, from 150 workgroups on
// and with two thirds of their channels in existence.  67 of 100 random layers are within that and take x0.72 to x1.05 of the
// time that the rule below gives them, x0.83 on average; at 128 to 150 workgroups it would be up to x1.32.  (Four wavefronts:
// x0.93 at best, x1.2 on most.)
int taps_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra)
{
    int pick = -1;
    double best = 0;
    const bool sparse = kinds_of(wp) >> 2 & 1u;
    for (int v : variants_of(sparse ? 13 : 14)) {
        const VariantDesc& d = variant_desc(v);
        const int channels = channel_waves(d) * d.NJ * 16;
        const bool wide = d.waves == 8;
        if (d.NBLK < 5 || (!sparse && !wide) || !variant_legal(v, wp, xdt, ra)) continue;
        const long n_cb = (wp->cout + channels - 1) / channels, n_wg = (long)((P + d.BP - 1) / d.BP) * n_cb;
        if (2L * wp->cout <= n_cb * channels || (channels > 64 && wp->cout <= 64)) continue;
        if (!sparse && 3L * wp->cout < 2L * n_cb * channels) continue;
        if (n_wg < (!sparse ? 150 : d.NBLK < 7 ? 224 : 176) || (n_wg > kNumCU && 5L * n_wg < 7L * kNumCU)) continue;
        const double rounds = (double)((n_wg + kNumCU - 1) / kNumCU);
        const double clocks = (sparse ? 16.0 : 32.0) * d.NBLK * d.NJ * (wp->K / 64);   // of a wavefront's matrix instructions
        const double cost = rounds * (wide ? 11000.0 + 1.14 * 2 * clocks : 12000.0 + 1.2 * clocks);
        if (pick < 0 || cost < best) {
            pick = v;
            best = cost;
        }
    }
    return pick;
}

// The channel-walking form of a bf16 1x1 layer that runs without tuning, -1 where the others do it: from 4096 pixels on and with
// more than one group of 256 output channels, half of the last of which may be empty in launches that the CUs hold at once (448
// tiles of 64 pixels), a quarter beyond, where fewer than 192 input channels stay with the others too; 64 pixels a tile from 400
// such tiles on.  Of 330 random 1x1 layers of up to 256 input channels the 68 within take x0.57 to x1.03 of the time that the
// rule below gives them, x0.84 on average; beyond, one group x1.2 to x1.5, 128 input channels and 2000 tiles x1.1 to x1.2.
int cols_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra)
{
    const long n_cb = (wp->cout + 255) / 256, tiles = (P + 63) / 64;
    if (P < 4096 || n_cb < 2 || 2L * wp->cout < n_cb * 256) return -1;
    if (tiles > 448 && (wp->cin < 192 || 4L * wp->cout < 3 * n_cb * 256)) return -1;
    for (int v : variants_of(17)) {
        const VariantDesc& d = variant_desc(v);
        if (d.NBLK == (tiles >= 400 ? 4 : 2) && variant_legal(v, wp, xdt, ra)) return v;
    }
    return -1;
}

// 16 x 16 blocks of outputs: what the small-layer fp32 kernel (kind 12) deals out.
long wave_blocks(const nm_packed* wp, int P) { return (long)((P + 15) / 16) * wp->n_rowblocks; }

// The small-layer fp32 kernel for a layer that runs without tuning, -1 where the others do it.  What it saves is the chain
// of chunks and the second launch, so that it wants the more chunks of 32 channels the more blocks a CU gets.  Over 440
// random layers up to four blocks a CU (1 to 288 chunks, 1:8 to dense), tensors out of cache, time over that of what the
// rules below pick: up to one block a CU 1 to 3 chunks x0.62 to x1.40, from 4 on x0.20 to x0.93; up to two 4 to 7 chunks
// x0.82 to x1.09, from 8 on x0.30 to x0.93; up to three 9 to 35 chunks x0.80 to x1.32, from 40 on x0.50 to x0.93; up to
// four 36 to 63 chunks x0.72 to x1.08, from 64 on x0.60 to x0.87.  Layers that keep all of a chunk take a row block a
// workgroup: from two blocks a CU on x0.89 to x1.30 at any length.
// One row block a workgroup up to 256 blocks, and where all of a chunk is kept (the weights are then more than the
// pixels); else two, which share the pixels.  (x1.06 of the fastest of its forms on average.)
int wave_default(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra)
{
    long blocks = wave_blocks(wp, P);
    if (blocks > kNumCU) blocks = (long)((P + 15) / 16) * (wp->n_rowblocks + wp->n_rowblocks % 2);   // (dealt out in pairs)
    const int chunks = wp->K / 32;
    if (blocks > 4L * kNumCU || chunks < (blocks <= kNumCU ? 4 : blocks <= 2L * kNumCU ? 8 : blocks <= 3L * kNumCU ? 40 : 64)) return -1;
    for (int v : base_variants()) {
        const VariantDesc& d = variant_desc(v);
        if (d.SPC == 8 && blocks > 2L * kNumCU) continue;
        if (d.kind != 12 || d.NBLK != 1 || d.NJ != (blocks <= kNumCU || d.SPC == 8 ? 1 : 2)) continue;
        if (variant_legal(v, wp, xdt, ra)) return v;
    }
    return -1;
}

// Clocks of one launch of an fp32-instruction (kinds 0, 5) or gather (kind 1) variant, up to a constant: the
// contraction, staging and barrier of a chunk in one wavefront, shared by the wavefronts of a SIMD, times the
// chunks; the start and the output of a workgroup; the rounds of workgroups that the CUs hold.  The factors were
// fitted to every variant's time on 407 random layers (4 to 500 odd and even channels, 1:4 to 4:8 and half of all
// channels, T 8 to 32, 100 to 300 000 pixels): the variant it picks takes x1.04 (fp32) and x1.05 (bf16) of the time
// of the fastest without a K split on average, x1.36 at worst.  "Rounds x tile area", which knows neither the
// number nor the depth of the chunks, was x1.23 and x1.42 (x2.3 and x4.0 at worst: 256-channel chunks on eight
// channels, say).
double model_clocks(const VariantDesc& d, const nm_packed* wp, int P)
{
    const int rb_per_wg = (4 / d.WP) * d.NJ;
    const double n_wg = (double)((P + d.BP - 1) / d.BP) * ((wp->n_rowblocks + rb_per_wg - 1) / rb_per_wg);
    const int nchunks = d.vec ? wp->kh * wp->kw * ((wp->cin + d.CK - 1) / d.CK) : (wp->K + d.CK - 1) / d.CK;
    const double kept = (double)std::min(d.CK, d.vec ? wp->cin : wp->K) * wp->n / wp->m;   // columns of a chunk
    const bool gather = d.kind == 1;
    const double items = (double)d.BP * d.CK / (gather ? 2048 : 1024);                    // staged 16 bytes a thread
    // registers: accumulators, two sets of operands, staged values and their addresses; the forms beyond 200 spill
    const double regs = 40.0 + 4.0 * d.NBLK * d.NJ + 8.0 * items + 4.0 * d.NJ * d.SPC * (d.kind == 0 ? 1.0 : gather ? 3.0 : 2.4);
    if (regs > 200.0) return 1e18 + regs;
    const double steps = d.kind == 5 ? kept / 4 : d.SPC;
    const double mfma = gather ? d.NBLK * d.SPC * (d.NJ * 16.0 + 29.0 * d.NJ / d.share)    // and the 2-byte reads
                               : d.NBLK * d.NJ * 32.0 * (d.kind == 5 ? steps + 0.3 : steps);
    const double reads = gather ? 0.0 : 6.9 * (d.NBLK / 4.0 + 2.1) * d.NJ * steps;
    const double chunk = mfma + reads + items * (gather ? 45.0 : 36.6) + 16.0 + (d.kind == 5 ? 10.0 * d.NJ : 0.0);
    const double ends = 453.0 * d.NBLK * d.NJ + 18.0 * items;   // the workgroup's output and its first staging
    const int occ = std::max(1, std::min({(int)(kMaxLdsBytes / lds_bytes(d, wp)), (int)(512.0 / regs), 8}));
    const double per_cu = n_wg / kNumCU;
    if (per_cu <= occ) {
        const double w = ceil(per_cu);
        return nchunks * std::max(431.0, w * chunk) + (w + 1.13) * ends;
    }
    const double rounds = per_cu / occ;
    return (0.32 * ceil(rounds) + 0.68 * rounds) * (5020.0 + nchunks * std::max(431.0, occ * chunk) + occ * ends) + 1.13 * ends;
}

// Deterministic default when the shape has not been tuned: rows_default, wave_default, split_default, taps_default, cols_default, else the cheapest
// by model_clocks.
//
// For the gather-free bf16 and the staged fp8 kernels there is a rule read off tuned ResNet stacks: a tile of 128
// pixels x 128 channels (64 pixels where that leaves under half the CUs a workgroup, 64 channels
// where the layer has no more), all four wavefronts along the channels; producer wavefronts and
// register-held weights unless the launch is many rounds of workgroups on a 1x1 layer; 128-channel
// chunks on deep, small layers, 64 otherwise.  Variants are ranked by their distance from that.
int heuristic_variant(const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs* ra)
{
    const unsigned kinds = kinds_of(wp);
    if (ra && (kinds & (1u << 10 | 1u << 11))) {
        const int v = rows_default(wp, P, xdt, *ra);
        if (v >= 0) return v;
    }
    if (xdt == NM_F32 && (kinds & 1u)) {
        const int v = wave_default(wp, P, xdt, ra);
        if (v >= 0) return v;
    }
    if (xdt == NM_F32 && (kinds & (1u << 8 | 1u << 9))) {
        const int v = split_default(wp, P, xdt, ra);
        if (v >= 0) return v;
    }
    if (ra && (kinds & (1u << 2 | 1u << 3))) {
        const int v = taps_default(wp, P, xdt, ra);
        if (v >= 0) return v;
    }
    if (ra && (kinds & (1u << 2))) {
        const int v = cols_default(wp, P, xdt, ra);
        if (v >= 0) return v;
    }
    if (kinds & (1u << 2 | 1u << 3 | 1u << 7)) {
        const long wg128 = (long)((P + 127) / 128) * ((wp->n_rowblocks + 7) / 8);
        const int bp_t = wg128 >= kNumCU / 2 ? 128 : 64;
        const int wgc_t = wp->n_rowblocks >= 8 ? 128 : 64;
        const long n_wg_t = (long)((P + bp_t - 1) / bp_t) * ((wp->n_rowblocks * 16 + wgc_t - 1) / wgc_t);
        const bool plain_t = wp->kh * wp->kw == 1 && n_wg_t >= 4L * kNumCU;
        const int ck_t = (wp->cin >= 256 && n_wg_t <= 2L * kNumCU) ? 128 : 64;
        auto lg = [](double a, double b) { return fabs(log2(a / b)); };
        int pick = -1;
        double pick_score = 0;
        for (int v : base_variants()) {
            const VariantDesc& d = variant_desc(v);
            if ((d.kind != 2 && d.kind != 3 && d.kind != 7) || !(kinds >> d.kind & 1u)) continue;
            if (!variant_legal(v, wp, xdt, ra)) continue;
            const int wgc = (4 / d.WP) * d.NJ * 16;
            double score = 4.0 * lg(d.BP, bp_t) + 4.0 * lg(wgc, wgc_t) + 1.0 * lg(d.CK, ck_t) + (d.WP != 1 ? 1.5 : 0.0);
            score += d.kind == 3 ? 6.0 : 0.0;                       // the sparse instruction where its operand exists
            score += plain_t ? (d.spec ? 2.0 : 0.0) : (d.areg ? 0.0 : d.spec ? 1.0 : 3.0);
            if (pick < 0 || score < pick_score - 1e-9) {
                pick = v;
                pick_score = score;
            }
        }
        if (pick >= 0) return pick;
    }
    // (a K split needs a workspace: only where the tuner has shown that it pays)
    int best = -1;
    double best_cost = 0;
    // the kernel-row-run and the register-streaming fp8 forms where they apply: rounds of workgroups x work of one
    if (kinds & (1u << 4 | 1u << 6))
        for (int v : base_variants()) {
            const VariantDesc& d = variant_desc(v);
            if ((d.kind != 4 && d.kind != 6) || !variant_legal(v, wp, xdt, ra)) continue;
            // (7 blocks, and 4 wavefronts along the pixels: rounds x work takes them where they are the slower ones, 45.5 us
            // for 42.1 with 224x224x3 -> 68 7x7 at batch 16, 33.5 for 27.5 with 112x112x2 -> 100 5x5)
            if (d.kind == 4 && (d.NBLK == 7 || d.WP == 4)) continue;
            const int rb_per_wg = (4 / d.WP) * d.NJ;
            const long n_wg = (long)((P + d.BP - 1) / d.BP) * ((wp->n_rowblocks + rb_per_wg - 1) / rb_per_wg);
            const int occ = std::max(1, (int)std::min<size_t>(2, kMaxLdsBytes / lds_bytes(d, wp)));
            const long rounds = (n_wg + (long)kNumCU * occ - 1) / ((long)kNumCU * occ);
            const double cost = (double)rounds * occ * d.BP * (rb_per_wg + 2.0);
            if (best < 0 || cost < best_cost * 0.999) {
                best = v;
                best_cost = cost;
            }
        }
    if (best >= 0) return best;
    for (int v : base_variants()) {
        const VariantDesc& d = variant_desc(v);
        if ((d.kind != 0 && d.kind != 1 && d.kind != 5) || !(kinds >> d.kind & 1u)) continue;
        if (!variant_legal(v, wp, xdt, ra)) continue;
        const double cost = model_clocks(d, wp, P);
        if (best < 0 || cost < best_cost * 0.999) {
            best = v;
            best_cost = cost;
        }
    }
    return best;
}

// The default of a shape, worked out once: it depends on nothing that the tuning key does not hold, and looking
// through the variants took 3 to 13 us of a call.  The key holds the handle's tables as a hash of 31 bits, so that the
// handle at hand is asked all the same, as for a tuned entry.  Bounded; a full table starts anew.
constexpr size_t kMaxDefaults = 4096;
std::map<ShapeKey, int> g_defaults;   // guarded by g_mu

int default_variant(const ShapeKey& key, const nm_packed* wp, int P, nm_dtype_t xdt, const RunArgs& ra)
{
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_defaults.find(key);
        if (it != g_defaults.end() && variant_legal(it->second, wp, xdt, &ra) && keeps_precision(it->second, wp)) return it->second;
    }
    const int v = heuristic_variant(wp, P, xdt, &ra);
    try {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_defaults.size() >= kMaxDefaults) g_defaults.clear();
        g_defaults[key] = v;
    } catch (const std::bad_alloc&) {   // (it is then worked out again)
    }
    return v;
}

// ---- workspace for the partial sums of K-split variants -----------------------------------
// One grow-only device buffer per device, shared by every call on that device (calls that
// overlap on different streams and both run a K-split variant would race on it: such variants
// are chosen only by the tuner or the test hook, and a serving loop that overlaps convolutions
// should not tune with them).  Growing it allocates, which a stream under capture cannot do.
size_t split_bytes(const VariantDesc& d, const Geometry& g, const nm_packed* wp)
{
    return d.ksplit > 1 ? (size_t)d.ksplit * (size_t)g.P * (size_t)wp->cout * sizeof(float) : 0;
}

struct Workspace {
    float* ptr = nullptr;
    size_t bytes = 0;
};
std::mutex g_ws_mu;
std::map<int, Workspace> g_ws;

// rc NM_OK and *out = a buffer of at least `bytes`, or an error; with may_alloc false the
// buffer must already be large enough
int get_workspace(int dev, size_t bytes, bool may_alloc, float** out)
{
    std::lock_guard<std::mutex> lk(g_ws_mu);
    Workspace& w = g_ws[dev];
    if (w.bytes < bytes) {
        if (!may_alloc) {
            set_error("the K-split workspace holds %zu bytes, this call needs %zu and may not allocate", w.bytes, bytes);
            return NM_ERR_ALLOC;
        }
        (void)hipFree(w.ptr);   // waits for the kernels still using it
        w.ptr = nullptr;
        w.bytes = 0;
        const size_t want = (bytes + ((size_t)1 << 20) - 1) & ~(((size_t)1 << 20) - 1);
        const hipError_t e = hipMalloc(reinterpret_cast<void**>(&w.ptr), want);
        if (e != hipSuccess) {
            w.ptr = nullptr;
            set_error("hipMalloc(%zu) for the K-split workspace failed: %s", want, hipGetErrorString(e));
            return NM_ERR_ALLOC;
        }
        w.bytes = want;
    }
    *out = w.ptr;
    return NM_OK;
}

int check_conv_args(const void* x, nm_dtype_t xdt, int cin, const nm_packed* wp, void* y,
                    nm_dtype_t ydt)
{
    if (!wp || !x || !y) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    if (cin != wp->cin) {
        set_error("cin %d does not match the packed weights (%d)", cin, wp->cin);
        return NM_ERR_ARG;
    }
    if ((xdt != NM_F32 && xdt != NM_BF16 && xdt != NM_F8E4M3) || (ydt != NM_F32 && ydt != NM_BF16 && ydt != NM_F8E4M3)) {
        set_error("unknown dtype");
        return NM_ERR_ARG;
    }
    if (!dtype_pair_ok(xdt, ydt)) {
        set_error("unsupported dtype pair: fp32 -> fp32, bf16 -> bf16 or E4M3 -> bf16");
        return NM_ERR_UNSUPPORTED;
    }
    if ((xdt == NM_F8E4M3) != (wp->value_dtype == NM_F8E4M3)) {
        set_error("E4M3 activations need weights packed as E4M3 (and the other way round)");
        return NM_ERR_UNSUPPORTED;
    }
    if (((uintptr_t)x % 16) || ((uintptr_t)y % 16)) {
        set_error("x and y must be 16-byte aligned");
        return NM_ERR_ARG;
    }
    int dev = -1;
    NM_HIP_CHECK(hipGetDevice(&dev));
    if (dev != wp->device) {
        set_error("packed weights live on device %d, current device is %d", wp->device, dev);
        return NM_ERR_ARG;
    }
    return NM_OK;
}

void free_packed(nm_packed* wp)
{
    if (!wp) return;
    (void)hipFree(wp->d_idx);
    (void)hipFree(wp->d_vals);
    (void)hipFree(wp->d_tables);
    delete wp;
}

}  // namespace
}  // namespace nm

using namespace nm;

extern "C" {

const char* nm_last_error(void) { return g_err; }

int nm_variant_count(void) { return variant_count(); }

const char* nm_variant_name(int variant)
{
    if (variant < 0 || variant >= variant_count()) return nullptr;
    return variant_desc(variant).name;
}

int nm_prune(const float* w, int cout, int kh, int kw, int cin, int n, int m, int tile,
             nm_dtype_t value_dtype, nm_packed_t** out)
{
    if (!w || !out) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    *out = nullptr;
    if (cout < 1 || kh < 1 || kw < 1 || cin < 1 || n < 1 || m < 1 || tile < 1 || n > m) {
        set_error("bad sizes: cout %d kh %d kw %d cin %d n %d m %d tile %d", cout, kh, kw, cin, n, m, tile);
        return NM_ERR_ARG;
    }
    if (value_dtype != NM_F32 && value_dtype != NM_BF16 && value_dtype != NM_F8E4M3) {
        set_error("unknown value dtype");
        return NM_ERR_ARG;
    }
    if (value_dtype == NM_F8E4M3 && (cin % 64 != 0 || tile % 16 != 0 || cout % 8 != 0)) {
        set_error("E4M3 weights need cin %% 64 == 0, tile %% 16 == 0 and cout %% 8 == 0 (cin %d, tile %d, cout %d)",
                  cin, tile, cout);
        return NM_ERR_UNSUPPORTED;
    }
    const long long K = (long long)kh * kw * cin;
    if (K % m != 0) {
        set_error("K = %lld is not a multiple of m = %d", K, m);
        return NM_ERR_ARG;
    }
    if (m > 16384) {
        set_error("m = %d exceeds the supported group size 16384", m);
        return NM_ERR_ARG;
    }
    if (K * cout > 0x7fffffffLL) {
        set_error("weight tensor too large");
        return NM_ERR_ARG;
    }
    const size_t nw = (size_t)cout * K;
    auto refuse_not_finite = [&]() {
        const size_t bad = first_not_finite(w, nw);
        if (bad < nw) set_error("weight %zu is not finite", bad);
        return bad < nw;
    };
    // up to 128K weights here, before any device work (at most 7 us, what clearing the flag costs); more by the selection
    // kernel, or here where the call fails before that has spoken: such weights are refused as what they are all the same
    const bool flagged = nw > 131072;
    bool unseen = flagged;
    if (!flagged && refuse_not_finite()) return NM_ERR_ARG;
    nm_packed* wp = new (std::nothrow) nm_packed();
    if (!wp) {
        set_error("out of host memory");
        return NM_ERR_ALLOC;
    }
    wp->cout = cout; wp->kh = kh; wp->kw = kw; wp->cin = cin; wp->K = (int)K;
    wp->n = n; wp->m = m; wp->tile = tile;
    wp->G = (int)(K / m); wp->kprime = wp->G * n; wp->n_tiles = (cout + tile - 1) / tile;
    wp->rbpt = (tile + 15) / 16; wp->n_rowblocks = wp->n_tiles * wp->rbpt;
    wp->value_dtype = value_dtype;

    float* d_w = nullptr;
    int rc = NM_OK;
    hipStream_t s = nullptr;
    auto fail = [&](int code) {
        if (unseen && refuse_not_finite()) code = NM_ERR_ARG;
        (void)hipFree(d_w);
        free_packed(wp);
        return code;
    };
#define NM_TRY_HIP(expr, code)                                                             \
    do {                                                                                   \
        hipError_t e__ = (expr);                                                           \
        if (e__ != hipSuccess) {                                                           \
            set_error("%s failed: %s", #expr, hipGetErrorString(e__));                     \
            return fail(code);                                                             \
        }                                                                                  \
    } while (0)

    NM_TRY_HIP(hipGetDevice(&wp->device), NM_ERR_HIP);
    NM_TRY_HIP(hipMalloc(&d_w, nw * sizeof(float)), NM_ERR_ALLOC);
    const size_t n_idx = (size_t)wp->n_tiles * wp->kprime;
    NM_TRY_HIP(hipMalloc(&wp->d_idx, (n_idx + 1) * sizeof(int32_t)), NM_ERR_ALLOC);   // and whether a weight is not finite
    NM_TRY_HIP(hipMalloc(&wp->d_vals, (size_t)wp->n_tiles * wp->kprime * tile * sizeof(float)), NM_ERR_ALLOC);
    NM_TRY_HIP(hipMemcpyAsync(d_w, w, nw * sizeof(float), hipMemcpyHostToDevice, s), NM_ERR_HIP);
    if (flagged) NM_TRY_HIP(hipMemsetAsync(wp->d_idx + n_idx, 0, sizeof(int32_t), s), NM_ERR_HIP);
    rc = run_prune(d_w, wp, s);
    if (rc != NM_OK) return fail(rc);
    wp->h_idx.resize(n_idx + (flagged ? 1 : 0));
    NM_TRY_HIP(hipMemcpyAsync(wp->h_idx.data(), wp->d_idx, wp->h_idx.size() * sizeof(int32_t),
                              hipMemcpyDeviceToHost, s), NM_ERR_HIP);
    NM_TRY_HIP(hipStreamSynchronize(s), NM_ERR_HIP);
    if (flagged) {
        if (wp->h_idx.back()) {
            set_error("a weight is not finite");   // (if the caller has changed it by now)
            return fail(NM_ERR_ARG);
        }
        wp->h_idx.pop_back();
        unseen = false;
    }

    if (value_dtype == NM_F8E4M3) {
        // one power-of-two scale per layer: the largest 2^e that keeps every kept weight within
        // the format (|w| 2^e <= 448); the kept values become the E4M3 numbers they are stored as
        float most = 0.f;
        for (int j = 0; j < wp->n_tiles; ++j) {   // row by row: the kept positions of a tile ascend
            const int32_t* idx = wp->h_idx.data() + (size_t)j * wp->kprime;
            const int r1 = std::min(cout, (j + 1) * tile);
            for (int r = j * tile; r < r1; ++r)
                for (int kk = 0; kk < wp->kprime; ++kk) most = std::max(most, fabsf(w[(size_t)r * K + idx[kk]]));
        }
        float scale = 1.f;
        if (most > 0.f) {
            int e = 0;
            (void)frexpf(448.0f / most, &e);       // 448 / most = f 2^e with 0.5 <= f < 1
            scale = ldexpf(1.0f, e - 1);
            while (most * scale > 448.0f) scale *= 0.5f;   // the quotient above is rounded
        }
        wp->scale = scale;
        rc = run_quantize_e4m3(wp, s);
        if (rc != NM_OK) return fail(rc);
    }

    // Operand tables for every chunk geometry a kernel variant may ask for: planned first, then
    // allocated as one block and built with one wait at the end.  (One allocation, one error flag and
    // one synchronisation per table, and above all the kept columns of each chunk counted again for
    // every variant, made this function take 159 ms for a 512x3x3x512 layer whose kernels run for
    // 0.1 ms; planned once it takes 0.75 ms.)
    GeomNeeds needs{wp, {}, {}};
    const bool vec_ok = cin % 4 == 0;
    const size_t kWindow = 0x80000000ull;   // the kernels read a table through a 2 GiB buffer window
    for (int v : base_variants()) {
        const VariantDesc& d = variant_desc(v);
        if (table_kind(d.kind) != d.kind) continue;   // (reads another kind's)
        if (is_f8_kind(d.kind) != (value_dtype == NM_F8E4M3)) continue;   // E4M3 handles feed the fp8 kernels only
        Prepack pp;
        pp.kind = d.kind;
        pp.SPC = d.SPC;
        if (is_f8_kind(d.kind)) {
            // one table layout for both kernels (64-channel k-steps in K order); an entry per
            // chunk size, because the chunk geometry travels with the table
            if (cin % d.CK != 0 || find_prepack(wp, d)) continue;
            pp.geom = make_chunk_geom(cin, wp->K, d.CK, 1);
            pp.wfrag_bytes = (size_t)wp->n_rowblocks * (wp->K / 64) * 64 * 16;
            if (pp.wfrag_bytes < kWindow) wp->prepacks.push_back(pp);
            continue;
        }
        if (is_split_kind(d.kind)) {
            // 16-byte loads; the sparse instruction where no aligned group of four keeps more than two columns
            if (value_dtype != NM_F32 || !vec_ok || (d.kind == 8) != (n <= 2 && m % 4 == 0) || find_prepack(wp, d)) continue;
            pp.geom = make_chunk_geom(cin, wp->K, 64, 1);
            const size_t blocks = (size_t)((cout + 15) / 16) * pp.geom.nchunks;
            pp.rows_bytes = d.kind == 8 ? blocks * 256 : 0;
            pp.wfrag_bytes = blocks * 3 * (d.kind == 8 ? 1 : 2) * 1024;
            if (pp.wfrag_bytes < kWindow) wp->prepacks.push_back(pp);
            continue;
        }
        if (is_rows_kind(d.kind)) {
            // the same runs out of staged rows: one table per alignment and number of k-steps
            if (d.kind == 10 ? value_dtype != NM_BF16 || cin % 8 == 0 : value_dtype != NM_F32 || cin % 4 == 0) continue;
            for (int par = 0; par < 2; ++par) {
                if (run_ksteps(wp, par) != d.SPC || find_prepack(wp, d, par)) continue;
                pp.geom.vec = 1; pp.geom.CK = d.CK; pp.geom.ncpt = 1; pp.geom.nchunks = 1;
                pp.par = par;
                pp.wfrag_bytes = (size_t)((cout + 15) / 16) * d.SPC * 2 * (d.kind == 10 ? 1 : 3) * 1024;
                if (pp.wfrag_bytes < kWindow) wp->prepacks.push_back(pp);
            }
            continue;
        }
        if (d.kind == 4) {
            // kernel-row runs: only where channel runs are too short for the other bf16 kernels
            if (value_dtype != NM_BF16 || cin % 8 == 0) continue;
            for (int par = 0; par < 2; ++par) {
                if (run_ksteps(wp, par) != d.SPC || find_prepack(wp, d, par)) continue;
                pp.geom.vec = 1; pp.geom.CK = d.CK; pp.geom.ncpt = 1; pp.geom.nchunks = 1;
                pp.par = par;
                pp.wfrag_bytes = (size_t)wp->n_rowblocks * pp.SPC * 2 * 64 * 8 * sizeof(uint16_t);
                wp->prepacks.push_back(pp);
            }
            continue;
        }
        if (d.kind == 5) {
            if (!vec_ok || value_dtype != NM_F32) continue;
        } else if (d.kind >= 2) {
            // gather-free bf16 kernel: whole 64-channel k-steps of one tap per chunk; the
            // sparse operand holds at most 2 kept columns per aligned group of 4
            if (value_dtype != NM_BF16 || cin % d.CK != 0) continue;
            if (d.kind == 2 && !(n <= 2 && m % 4 == 0)) continue;
        } else if (d.kind == 1) {
            if (value_dtype != NM_BF16 || cin % 8 != 0) continue;
        } else if ((d.vec != 0) != vec_ok) {
            continue;
        }
        const ChunkGeom g = make_chunk_geom(cin, wp->K, d.CK, d.vec);
        if (d.kind < 2) {
            const int pick = needs.steps(d, g);
            if (pick == 0 || pick != d.SPC) continue;
        } else if (d.kind == 5) {
            // worth its table only where the kept columns are spread unevenly over the
            // chunks: otherwise the fixed-step form does the same work
            if ((long)needs.max_kept(g) * g.nchunks * 10 <= (long)wp->kprime * 11) continue;
        }
        bool have = false;   // (find_prepack would not count an element-wise table whose decode table is not there yet)
        for (const Prepack& q : wp->prepacks)
            have = have || (q.kind == d.kind && q.geom.CK == d.CK && q.geom.vec == d.vec && q.SPC == d.SPC);
        if (have) continue;
        pp.geom = g;
        if (d.kind >= 2 && d.kind <= 4) {
            pp.rows_bytes = (size_t)wp->n_tiles * g.nchunks * 4 * pp.SPC * sizeof(uint32_t);
            pp.wfrag_bytes = (size_t)wp->n_rowblocks * g.nchunks * pp.SPC * (d.kind == 2 ? 1 : 2) * 64 * 8 *
                             sizeof(uint16_t);
        } else if (d.kind == 1) {
            pp.rows_bytes = (size_t)wp->n_tiles * g.nchunks * pp.SPC * 4 * 8 * sizeof(uint32_t);
            pp.wfrag_bytes = (size_t)wp->n_rowblocks * g.nchunks * pp.SPC * 64 * 8 * sizeof(uint16_t);
        } else {
            pp.rows_bytes = (size_t)wp->n_tiles * g.nchunks * 4 * pp.SPC * sizeof(uint32_t);
            pp.wfrag_bytes = (size_t)wp->n_rowblocks * g.nchunks * 64 * pp.SPC * sizeof(float);
            if (d.kind == 0 && g.vec && g.CK == 32 && value_dtype == NM_F32) pp.cols_bytes = pp.rows_bytes / 4;
        }
        if (pp.wfrag_bytes >= kWindow || pp.rows_bytes >= kWindow) continue;
        // element-wise staging decodes k through a table of 8-, 8- and 16-bit fields
        if (!g.vec && kh <= 255 && kw <= 255 && cin <= 65535) pp.ktab_bytes = (size_t)g.nchunks * g.CK * sizeof(uint32_t);
        wp->prepacks.push_back(pp);
    }
    bool no_planes = false;
    {
        auto up = [](size_t b) { return (b + 255) & ~(size_t)255; };
        size_t total = 256;   // the builders' flags
        for (const Prepack& pp : wp->prepacks) total += up(pp.rows_bytes) + up(pp.wfrag_bytes) + up(pp.ktab_bytes) + up(pp.cols_bytes);
        NM_TRY_HIP(hipMalloc(reinterpret_cast<void**>(&wp->d_tables), total), NM_ERR_ALLOC);
        NM_TRY_HIP(hipMemsetAsync(wp->d_tables, 0, total, s), NM_ERR_HIP);
        char* at = wp->d_tables + 256;
        auto take = [&](size_t b) {
            char* r = at;
            at += up(b);
            return r;
        };
        std::vector<uint32_t> kt;   // one layer has at most one element-wise geometry; kept until the copy is done
        for (Prepack& pp : wp->prepacks) {
            if (pp.rows_bytes) pp.d_rows = reinterpret_cast<uint32_t*>(take(pp.rows_bytes));
            pp.d_wfrag = reinterpret_cast<float*>(take(pp.wfrag_bytes));
            if (pp.cols_bytes) pp.d_cols = reinterpret_cast<uint8_t*>(take(pp.cols_bytes));
            rc = run_build_prepack(wp, pp, s);
            if (rc != NM_OK) return fail(rc);
            if (pp.ktab_bytes) {
                // decode table of the flat k axis (layout only: which tap and channel row k is)
                pp.d_ktab = reinterpret_cast<uint32_t*>(take(pp.ktab_bytes));
                kt.assign((size_t)pp.geom.nchunks * pp.geom.CK, 0xffffffffu);
                for (int k = 0; k < wp->K; ++k) {
                    const int tap = k / cin, ci = k - tap * cin;
                    kt[k] = (uint32_t)(tap / kw) | ((uint32_t)(tap % kw) << 8) | ((uint32_t)ci << 16);
                }
                NM_TRY_HIP(hipMemcpy(pp.d_ktab, kt.data(), kt.size() * sizeof(uint32_t), hipMemcpyHostToDevice),
                           NM_ERR_HIP);
            }
        }
        int h_err[3] = {0, 0, 0};
        NM_TRY_HIP(hipMemcpyAsync(h_err, wp->d_tables, sizeof(h_err), hipMemcpyDeviceToHost, s), NM_ERR_HIP);
        NM_TRY_HIP(hipStreamSynchronize(s), NM_ERR_HIP);
        if (h_err[0]) {
            set_error("internal: a K chunk holds more kept columns than the operand table allows");
            return fail(NM_ERR_UNSUPPORTED);
        }
        if (h_err[1]) {   // a weight that three bf16 planes do not hold exactly: the fp32 instruction runs this layer
            no_planes = true;
            auto planes = [](const Prepack& pp) { return is_split_kind(pp.kind) || pp.kind == 11; };
            wp->prepacks.erase(std::remove_if(wp->prepacks.begin(), wp->prepacks.end(), planes), wp->prepacks.end());
        }
        float max_w;
        memcpy(&max_w, &h_err[2], sizeof(max_w));
        wp->redo_below = redo_below(max_w, wp->kprime);
    }
#undef NM_TRY_HIP
    (void)hipFree(d_w);
    if (wp->prepacks.empty()) {
        set_error("no kernel variant can run this layer (cin %d, n:m %d:%d, tile %d)", cin, n, m, tile);
        free_packed(wp);
        return NM_ERR_UNSUPPORTED;
    }
    wp->sig = prepack_signature(wp, no_planes);
    const DeviceId* const id = device_id(wp->device);
    wp->device_hash = id ? id->hash : 0;
    *out = wp;
    return NM_OK;
}

int nm_packed_free(nm_packed_t* wp)
{
    free_packed(wp);
    return NM_OK;
}

int nm_packed_dims(const nm_packed_t* wp, int* n_tiles, int* groups, int* n, int* kprime)
{
    if (!wp) {
        set_error("null handle");
        return NM_ERR_ARG;
    }
    if (n_tiles) *n_tiles = wp->n_tiles;
    if (groups) *groups = wp->G;
    if (n) *n = wp->n;
    if (kprime) *kprime = wp->kprime;
    return NM_OK;
}

int nm_packed_indices(const nm_packed_t* wp, int32_t* idx_host)
{
    if (!wp || !idx_host) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    std::copy(wp->h_idx.begin(), wp->h_idx.end(), idx_host);
    return NM_OK;
}

int nm_packed_values(const nm_packed_t* wp, float* vals_host)
{
    if (!wp || !vals_host) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    NM_HIP_CHECK(hipMemcpy(vals_host, wp->d_vals,
                           (size_t)wp->n_tiles * wp->kprime * wp->tile * sizeof(float),
                           hipMemcpyDeviceToHost));
    return NM_OK;
}

int nm_packed_mask(const nm_packed_t* wp, uint8_t* mask_host)
{
    if (!wp || !mask_host) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    uint8_t* d_mask = nullptr;
    const size_t bytes = (size_t)wp->cout * wp->K;
    hipError_t e = hipMalloc(&d_mask, bytes);
    if (e != hipSuccess) {
        set_error("hipMalloc(%zu) failed: %s", bytes, hipGetErrorString(e));
        return NM_ERR_ALLOC;
    }
    int rc = run_build_mask(wp, d_mask, nullptr);
    if (rc == NM_OK) {
        e = hipMemcpy(mask_host, d_mask, bytes, hipMemcpyDeviceToHost);
        if (e != hipSuccess) {
            set_error("hipMemcpy failed: %s", hipGetErrorString(e));
            rc = NM_ERR_HIP;
        }
    }
    (void)hipFree(d_mask);
    return rc;
}

int nm_packed_scale(const nm_packed_t* wp, float* scale)
{
    if (!wp || !scale) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    *scale = wp->scale;
    return NM_OK;
}

int nm_force_variant(int v)
{
    if (v < -1 || v >= variant_count()) {
        set_error("variant %d out of range", v);
        return NM_ERR_ARG;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    g_forced = v;
    return NM_OK;
}

int nm_last_variant(void) { return g_last_variant; }

int nm_variant_legal(int variant, const nm_packed_t* wp, nm_dtype_t xdt, nm_dtype_t ydt)
{
    if (!wp || variant < 0 || variant >= variant_count()) {
        set_error("bad arguments");
        return NM_ERR_ARG;
    }
    if (!dtype_pair_ok(xdt, ydt)) return 0;
    return variant_legal(variant, wp, xdt) ? 1 : 0;
}

static int conv2d_impl(const void* x, nm_dtype_t xdt, int b, int h, int w, int cin, const nm_packed_t* wp,
                       const float* bias, const void* res, int sh, int sw, int ph, int pw, int dh, int dw,
                       int relu, void* y, nm_dtype_t ydt, void* stream, bool static_only = false)
{
    int rc = check_conv_args(x, xdt, cin, wp, y, ydt);
    if (rc != NM_OK) return rc;
    if (res && ((uintptr_t)res % 16)) {
        set_error("residual must be 16-byte aligned");
        return NM_ERR_ARG;
    }
    Geometry g;
    rc = conv_geometry(b, h, w, wp, sh, sw, ph, pw, dh, dw, elem_size(xdt), &g);
    if (rc != NM_OK) return rc;
    if (res) {
        const size_t ybytes = (size_t)g.P * wp->cout * elem_size(ydt);
        const uintptr_t r0 = (uintptr_t)res, y0 = (uintptr_t)y;
        if (r0 < y0 + ybytes && y0 < r0 + ybytes) {
            set_error("residual must not overlap y");
            return NM_ERR_ARG;
        }
    }

    int v = -1;
    bool forced = false;
    const ShapeKey key = make_key(xdt, ydt, b, h, w, wp, sh, sw, ph, pw, dh, dw, bias != nullptr, relu);
    {
        std::lock_guard<std::mutex> lk(g_mu);
        if (g_forced >= 0) {
            v = g_forced;
            forced = true;
        } else {
            auto it = g_cache.find(key);
            if (it != g_cache.end()) v = it->second.variant;
        }
    }
    const RunArgs ra = {w, sw, pw, dw, sh, dh, ph, h, b};
    if (v >= 0 && (!variant_legal(v, wp, xdt, &ra) || (!forced && !keeps_precision(v, wp)))) {
        if (forced) {
            set_error("variant %d (%s) cannot run this layer", v, nm_variant_name(v));
            return NM_ERR_UNSUPPORTED;
        }
        v = -1;   // stale cache entry: fall back to the default
    }
    if (v < 0) v = default_variant(key, wp, g.P, xdt, ra);
    if (v < 0) {
        set_error("no kernel variant can run this layer");
        return NM_ERR_UNSUPPORTED;
    }
    const VariantDesc& d = variant_desc(v);
    ConvParams p;
    fill_params(p, d, *find_prepack(wp, d, run_par(pw, wp->cin)), wp, x, y, bias, b, h, w, g, sh, sw, ph, pw,
                dh, dw, relu, elem_size(xdt));
    p.res = res;
    if (d.ksplit > 1) {
        const size_t need = split_bytes(d, g, wp);
        if (static_only) {
            if (need > kStaticScratchBytes) {
                set_error("variant %s needs %zu bytes of scratch for its partial sums; the static buffer holds %u",
                          d.name, need, (unsigned)kStaticScratchBytes);
                return NM_ERR_SHAPE;
            }
            rc = static_scratch(wp->device, &p.partial);
        } else {
            // growing the workspace allocates, which a stream under capture must not do
            hipStreamCaptureStatus cs = hipStreamCaptureStatusNone;
            (void)hipStreamIsCapturing((hipStream_t)stream, &cs);
            rc = get_workspace(wp->device, need, cs == hipStreamCaptureStatusNone, &p.partial);
        }
        if (rc != NM_OK) return rc;
    }
    rc = launch_conv(v, xdt, ydt, p, (hipStream_t)stream);
    if (rc == NM_OK && d.ksplit > 1) rc = run_splitk_reduce(p, ydt, (hipStream_t)stream);
    if (rc == NM_OK) g_last_variant = v;
    return rc;
}

int nm_conv2d(const void* x, nm_dtype_t xdt, int b, int h, int w, int cin, const nm_packed_t* wp,
              const float* bias, int sh, int sw, int ph, int pw, int dh, int dw, int relu, void* y,
              nm_dtype_t ydt, void* stream)
{
    return conv2d_impl(x, xdt, b, h, w, cin, wp, bias, nullptr, sh, sw, ph, pw, dh, dw, relu, y, ydt, stream);
}

int nm_conv2d_res(const void* x, nm_dtype_t xdt, int b, int h, int w, int cin, const nm_packed_t* wp,
                  const float* bias, const void* res, int sh, int sw, int ph, int pw, int dh, int dw,
                  int relu, void* y, nm_dtype_t ydt, void* stream)
{
    return conv2d_impl(x, xdt, b, h, w, cin, wp, bias, res, sh, sw, ph, pw, dh, dw, relu, y, ydt, stream);
}

int nm_conv2d_static(const void* x, nm_dtype_t xdt, int b, int h, int w, int cin, const nm_packed_t* wp,
                     const float* bias, const void* res, int sh, int sw, int ph, int pw, int dh, int dw,
                     int relu, void* y, nm_dtype_t ydt, void* stream)
{
    return conv2d_impl(x, xdt, b, h, w, cin, wp, bias, res, sh, sw, ph, pw, dh, dw, relu, y, ydt, stream, true);
}

int nm_conv2d_args(const nm_conv_args_t* a)
{
    if (!a) {
        set_error("null pointer argument");
        return NM_ERR_ARG;
    }
    return conv2d_impl(a->x_dev, (nm_dtype_t)a->x_dtype, (int)a->b, (int)a->h, (int)a->w, (int)a->cin, a->wp, a->bias_dev,
                       a->residual_dev, (int)a->stride_h, (int)a->stride_w, (int)a->pad_h, (int)a->pad_w, (int)a->dil_h,
                       (int)a->dil_w, (int)a->relu, a->y_dev, (nm_dtype_t)a->y_dtype, a->hip_stream, a->static_only != 0);
}

int nm_maxpool2d(const void* x, nm_dtype_t dt, int b, int h, int w, int c, int k, int stride, int pad,
                 void* y, void* stream)
{
    if (!x || !y || b < 1 || h < 1 || w < 1 || c < 1 || k < 1 || stride < 1 || pad < 0 || pad >= k ||
        (dt != NM_F32 && dt != NM_BF16)) {
        set_error("bad max-pooling arguments");
        return NM_ERR_ARG;
    }
    if (h + 2 * pad < k || w + 2 * pad < k) {
        set_error("output would be empty: input %dx%d, window %d, pad %d", h, w, k, pad);
        return NM_ERR_SHAPE;
    }
    const int ho = (h + 2 * pad - k) / stride + 1, wo = (w + 2 * pad - k) / stride + 1;
    if (((uintptr_t)x % 16) || ((uintptr_t)y % 16)) {
        set_error("x and y must be 16-byte aligned");
        return NM_ERR_ARG;
    }
    return run_maxpool(x, dt, b, h, w, c, k, stride, pad, ho, wo, y, (hipStream_t)stream);
}

int nm_im2col(const void* x, nm_dtype_t dt, int b, int h, int w, int cin, int kh, int kw, int sh, int sw,
              int ph, int pw, int dh, int dw, void* a_out, void* stream)
{
    if (!x || !a_out || b < 1 || h < 1 || w < 1 || cin < 1 || kh < 1 || kw < 1 || sh < 1 || sw < 1 || ph < 0 ||
        pw < 0 || dh < 1 || dw < 1 || (dt != NM_F32 && dt != NM_BF16)) {
        set_error("bad im2col arguments");
        return NM_ERR_ARG;
    }
    if (((uintptr_t)x % 16) || ((uintptr_t)a_out % 16)) {
        set_error("x and a must be 16-byte aligned");
        return NM_ERR_ARG;
    }
    const long eh = (long)h + 2L * ph - (long)dh * (kh - 1) - 1, ew = (long)w + 2L * pw - (long)dw * (kw - 1) - 1;
    if (eh < 0 || ew < 0) {
        set_error("output would be empty");
        return NM_ERR_SHAPE;
    }
    const int ho = (int)(eh / sh) + 1, wo = (int)(ew / sw) + 1;
    if ((long long)b * ho * wo * kh * kw * cin > 0x7fffffffLL * 4) {
        set_error("im2col matrix too large");
        return NM_ERR_SHAPE;
    }
    return run_im2col(x, dt, b, h, w, cin, kh, kw, sh, sw, ph, pw, dh, dw, ho, wo, a_out, (hipStream_t)stream);
}

int nm_stream_floor(const void* x, size_t x_bytes, void* y, size_t y_bytes, void* stream)
{
    if (!x || !y || ((uintptr_t)x % 16) || ((uintptr_t)y % 16)) {
        set_error("x and y must be non-null and 16-byte aligned");
        return NM_ERR_ARG;
    }
    return run_stream_floor(x, x_bytes, y, y_bytes, (hipStream_t)stream);
}

int nm_avgpool_global(const void* x, nm_dtype_t dt, int b, int h, int w, int c, void* y, void* stream)
{
    if (!x || !y || b < 1 || h < 1 || w < 1 || c < 1 || (dt != NM_F32 && dt != NM_BF16)) {
        set_error("bad average-pooling arguments");
        return NM_ERR_ARG;
    }
    if (b > 65535) {
        set_error("batch %d exceeds 65535", b);
        return NM_ERR_ARG;
    }
    return run_avgpool(x, dt, b, h * w, c, y, (hipStream_t)stream);
}

int nm_autotune(nm_dtype_t xdt, int b, int h, int w, int cin, const nm_packed_t* wp, int has_bias,
                int sh, int sw, int ph, int pw, int dh, int dw, int relu, nm_dtype_t ydt,
                void* stream, int* chosen, float* best_ms)
{
    if (!wp) {
        set_error("null handle");
        return NM_ERR_ARG;
    }
    if (cin != wp->cin) {
        set_error("cin %d does not match the packed weights (%d)", cin, wp->cin);
        return NM_ERR_ARG;
    }
    if (!dtype_pair_ok(xdt, ydt) || (xdt == NM_F8E4M3) != (wp->value_dtype == NM_F8E4M3)) {
        set_error("unsupported dtype pair: fp32 -> fp32, bf16 -> bf16 or E4M3 -> bf16 (E4M3 with E4M3 weights)");
        return NM_ERR_UNSUPPORTED;
    }
    Geometry g;
    int rc = conv_geometry(b, h, w, wp, sh, sw, ph, pw, dh, dw, elem_size(xdt), &g);
    if (rc != NM_OK) return rc;
    const ShapeKey key = make_key(xdt, ydt, b, h, w, wp, sh, sw, ph, pw, dh, dw, has_bias, relu);
    const RunArgs ra = {w, sw, pw, dw, sh, dh, ph, h, b};
    {
        std::lock_guard<std::mutex> lk(g_mu);
        auto it = g_cache.find(key);
        if (it != g_cache.end() && variant_legal(it->second.variant, wp, xdt, &ra) && keeps_precision(it->second.variant, wp)) {
            if (chosen) *chosen = it->second.variant;
            if (best_ms) *best_ms = it->second.ms;
            return NM_OK;
        }
    }
    hipStream_t s = (hipStream_t)stream;
    const size_t es = elem_size(xdt), yes = elem_size(ydt);
    const size_t xn = (size_t)b * h * w * cin, yn = (size_t)g.P * wp->cout;
    // Cold-cache protocol: in a network every layer finds the 256 MB last-level
    // cache full of other layers' data, so the candidates are timed on a ring
    // of input/output sets (about 768 MB in total) and no launch reuses the
    // set of a recent one.
    const size_t xbytes = (xn * es + 255) & ~(size_t)255, ybytes = (yn * yes + 255) & ~(size_t)255;
    const size_t pool = (size_t)768 << 20;
    int nbuf = (int)std::min<size_t>(64, std::max<size_t>(1, pool / (xbytes + ybytes)));
    char* dpool = nullptr;
    float* dbias = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    auto cleanup = [&]() {
        (void)hipFree(dpool); (void)hipFree(dbias);
        if (e0) (void)hipEventDestroy(e0);
        if (e1) (void)hipEventDestroy(e1);
    };
#define NM_TRY(expr, code)                                                       \
    do {                                                                         \
        hipError_t e__ = (expr);                                                 \
        if (e__ != hipSuccess) {                                                 \
            set_error("%s failed: %s", #expr, hipGetErrorString(e__));           \
            cleanup();                                                           \
            return code;                                                         \
        }                                                                        \
    } while (0)
    NM_TRY(hipMalloc(&dpool, (xbytes + ybytes) * nbuf), NM_ERR_ALLOC);
    if (has_bias) {
        NM_TRY(hipMalloc(&dbias, wp->cout * sizeof(float)), NM_ERR_ALLOC);
        rc = run_fill_random(dbias, wp->cout, NM_F32, 7u, s);
        if (rc != NM_OK) { cleanup(); return rc; }
    }
    for (int i = 0; i < nbuf; ++i) {
        rc = run_fill_random(dpool + (xbytes + ybytes) * i, xn, xdt, 1u + i, s);
        if (rc != NM_OK) { cleanup(); return rc; }
    }
    NM_TRY(hipEventCreate(&e0), NM_ERR_HIP);
    NM_TRY(hipEventCreate(&e1), NM_ERR_HIP);

    int best_v = -1;
    float best = 0.f;
    int turn = 0;
    int rc_t = NM_OK;
    // one timed group of `reps` launches of variant v on fresh tensor sets: ms per launch, < 0 on error
    auto time_group = [&](int v, int reps) -> float {
        const VariantDesc& d = variant_desc(v);
        const Prepack* pp = find_prepack(wp, d, run_par(pw, wp->cin));
        ConvParams p;
        float* partial = nullptr;
        if (d.ksplit > 1) {   // sized here, once: nm_conv2d then finds the workspace large enough
            rc_t = get_workspace(wp->device, split_bytes(d, g, wp), true, &partial);
            if (rc_t != NM_OK) return -1.f;
        }
        if (hipEventRecord(e0, s) != hipSuccess) { rc_t = NM_ERR_HIP; return -1.f; }
        for (int i = 0; i < reps; ++i) {
            char* set = dpool + (xbytes + ybytes) * (turn++ % nbuf);
            fill_params(p, d, *pp, wp, set, set + xbytes, dbias, b, h, w, g, sh, sw, ph, pw, dh, dw, relu, es);
            p.partial = partial;
            rc_t = launch_conv(v, xdt, ydt, p, s);
            if (rc_t == NM_OK && d.ksplit > 1) rc_t = run_splitk_reduce(p, ydt, s);
            if (rc_t != NM_OK) return -1.f;
        }
        float ms = 0.f;
        if (hipEventRecord(e1, s) != hipSuccess || hipEventSynchronize(e1) != hipSuccess ||
            hipEventElapsedTime(&ms, e0, e1) != hipSuccess) {
            set_error("timing a tuning candidate failed");
            rc_t = NM_ERR_HIP;
            return -1.f;
        }
        return ms / reps;
    };
    // First pass: every legal variant, one warm-up launch (code object, attributes) and the
    // median of three groups.  Second pass: the five fastest (up to ten if that close) again, interleaved so that clock
    // and cache drift hit them alike, median of seven groups -- single passes were seen to
    // pick variants a few percent off the best from run to run.
    std::vector<std::pair<float, int>> first;
    for (int v = 0; v < variant_count(); ++v) {
        if (!variant_legal(v, wp, xdt, &ra) || !keeps_precision(v, wp)) continue;
        {   // a K split is worth its second kernel only where the output tiles are one short, ragged round (at most two per CU)
            const VariantDesc& d = variant_desc(v);
            const int nrb = flat_rowblocks(d.kind) ? (wp->cout + 15) / 16 : wp->n_rowblocks;
            const long tiles = (long)((g.P + d.BP - 1) / d.BP) * ((nrb + (4 / d.WP) * d.NJ - 1) / ((4 / d.WP) * d.NJ));
            if (d.kind == 12 && wave_blocks(wp, g.P) > 16 * kNumCU) continue;   // (first on no layer from 3000 blocks on)
            if (d.ksplit > 1 && (tiles > 2 * kNumCU || tiles * d.ksplit > 8 * kNumCU)) continue;
        }
        if (time_group(v, 1) < 0.f) { cleanup(); return rc_t; }
        float t[3];
        for (int r = 0; r < 3; ++r)
            if ((t[r] = time_group(v, 3)) < 0.f) { cleanup(); return rc_t; }
        std::sort(t, t + 3);
        first.push_back(std::make_pair(t[1], v));
    }
    std::sort(first.begin(), first.end());
    if (getenv("NM_TUNE_VERBOSE")) {   // the whole field, fastest first: what the choice was made from
        fprintf(stderr, "nm_autotune %dx%dx%d -> %d, %dx%d, b %d, %d:%d T%d: %zu candidates\n", h, w, cin, wp->cout,
                wp->kh, wp->kw, b, wp->n, wp->m, wp->tile, first.size());
        for (const auto& c : first) fprintf(stderr, "  %9.2f us  %s\n", c.first * 1e3f, variant_desc(c.second).name);
    }
    // finalists: the five fastest, and whatever else came within 5 % of the fastest (at most ten)
    int finalists = (int)std::min<size_t>(5, first.size());
    while (finalists < (int)std::min<size_t>(10, first.size()) && first[finalists].first <= first[0].first * 1.05f)
        ++finalists;
    std::vector<std::vector<float>> again(finalists);
    for (int r = 0; r < 7 && finalists > 1; ++r)
        for (int c = 0; c < finalists; ++c) {
            const float t = time_group(first[c].second, 4);
            if (t < 0.f) { cleanup(); return rc_t; }
            again[c].push_back(t);
        }
    for (int c = 0; c < finalists; ++c) {
        float t = first[c].first;
        if (!again[c].empty()) {
            std::sort(again[c].begin(), again[c].end());
            t = again[c][again[c].size() / 2];
        }
        if (best_v < 0 || t < best) {
            best_v = first[c].second;
            best = t;
        }
    }
#undef NM_TRY
    cleanup();
    if (best_v < 0) {
        set_error("no kernel variant can run this layer");
        return NM_ERR_UNSUPPORTED;
    }
    {
        std::lock_guard<std::mutex> lk(g_mu);
        g_cache[key] = CacheVal{best_v, best};
    }
    if (chosen) *chosen = best_v;
    if (best_ms) *best_ms = best;
    return NM_OK;
}

int nm_autotune_tile(const float* w, int cout, int kh, int kw, int cin, int n, int m,
                     const int* tiles, int n_candidates, nm_dtype_t value_dtype,
                     nm_dtype_t xdt, int b, int h, int wd, int has_bias,
                     int sh, int sw, int ph, int pw, int dh, int dw, int relu, nm_dtype_t ydt,
                     void* stream, nm_packed_t** out, int* best_tile, float* ms_per_candidate)
{
    if (!out || !tiles || n_candidates < 1) {
        set_error("null output or empty candidate list");
        return NM_ERR_ARG;
    }
    *out = nullptr;
    nm_packed_t* best = nullptr;
    float best_ms = 0.f;
    for (int i = 0; i < n_candidates; ++i) {
        nm_packed_t* wp = nullptr;
        int rc = nm_prune(w, cout, kh, kw, cin, n, m, tiles[i], value_dtype, &wp);
        float ms = 0.f;
        if (rc == NM_OK)
            rc = nm_autotune(xdt, b, h, wd, cin, wp, has_bias, sh, sw, ph, pw, dh, dw, relu, ydt, stream,
                             nullptr, &ms);
        if (rc != NM_OK) {   // the message of the failing call stands
            free_packed(wp);
            free_packed(best);
            return rc;
        }
        if (ms_per_candidate) ms_per_candidate[i] = ms;
        if (!best || ms < best_ms) {
            free_packed(best);
            best = wp;
            best_ms = ms;
            if (best_tile) *best_tile = tiles[i];
        } else {
            free_packed(wp);
        }
    }
    *out = best;
    return NM_OK;
}

int nm_workspace_free(void)
{
    std::lock_guard<std::mutex> lk(g_ws_mu);
    for (auto& kv : g_ws) {
        (void)hipFree(kv.second.ptr);   // waits for the kernels still using it
        kv.second = Workspace();
    }
    return NM_OK;
}

int nm_cache_clear(void)
{
    std::lock_guard<std::mutex> lk(g_mu);
    g_cache.clear();
    return NM_OK;
}

int nm_cache_size(void)
{
    std::lock_guard<std::mutex> lk(g_mu);
    return (int)g_cache.size();
}

// File format: first line "nmconv-cache 2 <variant count> <key integers per line>
// <device of the writer>", then one line per entry: the key integers (shape,
// dtypes, N:M, tile, bias / activation flags, device identity, operand-table
// signature), the variant's name, its time in ms.  Variants are stored by name so
// that a cache written by a build with a different variant table cannot select
// the wrong kernel; entries tuned on another kind of device stay in the file but
// never match a key made on this one.
int nm_cache_save(const char* path)
{
    if (!path) {
        set_error("null path");
        return NM_ERR_ARG;
    }
    FILE* f = fopen(path, "w");
    if (!f) {
        set_error("cannot open %s for writing", path);
        return NM_ERR_IO;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    int dev = 0;
    const DeviceId* id = hipGetDevice(&dev) == hipSuccess ? device_id(dev) : nullptr;
    fprintf(f, "nmconv-cache 2 %d %d %s\n", variant_count(), kKeyInts, id ? id->name : "unknown");
    for (const auto& kv : g_cache) {
        for (int i = 0; i < kKeyInts; ++i) fprintf(f, "%d ", kv.first.v[i]);
        fprintf(f, "%s %.6f\n", variant_desc(kv.second.variant).name, kv.second.ms);
    }
    const bool ok = fclose(f) == 0;
    if (!ok) {
        set_error("write to %s failed", path);
        return NM_ERR_IO;
    }
    return NM_OK;
}

int nm_cache_load(const char* path)
{
    if (!path) {
        set_error("null path");
        return NM_ERR_ARG;
    }
    FILE* f = fopen(path, "r");
    if (!f) {
        set_error("cannot open %s", path);
        return NM_ERR_IO;
    }
    int ver = 0, cnt = 0, nkey = 0;
    char devname[128];
    if (fscanf(f, "nmconv-cache %d %d %d %127s", &ver, &cnt, &nkey, devname) != 4 || ver != 2 ||
        nkey != kKeyInts) {
        fclose(f);
        set_error("%s is not an nmconv cache file of this format", path);
        return NM_ERR_IO;
    }
    std::lock_guard<std::mutex> lk(g_mu);
    while (true) {
        ShapeKey k;
        bool ok = true;
        for (int i = 0; i < kKeyInts && ok; ++i) ok = fscanf(f, "%d", &k.v[i]) == 1;
        char name[128];
        float ms = 0.f;
        if (!ok || fscanf(f, "%127s %f", name, &ms) != 2) break;
        for (int v = 0; v < variant_count(); ++v)
            if (strcmp(name, variant_desc(v).name) == 0) {
                g_cache[k] = CacheVal{v, ms};
                break;
            }
    }
    fclose(f);
    return NM_OK;
}

}  // extern "C"
