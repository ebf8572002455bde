// Host side of libcomet: context / workspace, argument checks, launch geometry
// and the extern "C" entry points declared in include/comet.h.
#include <hip/hip_runtime.h>

#include <cmath>
#include <cstdio>
#include <cstring>
#include <mutex>
#include <numeric>
#include <new>
#include <vector>

#include "../../include/comet.h"
#include "comet_bands.h"
#include "comet_kernels.h"

using namespace comet;

namespace {

thread_local char g_hip_msg[256] = "no HIP error recorded";

int hip_fail(hipError_t e, const char *what) {
    snprintf(g_hip_msg, sizeof(g_hip_msg), "%s: %s", what, hipGetErrorString(e));
    return COMET_ERR_HIP;
}
#define HIP_TRY(expr)                                                   \
    do {                                                                \
        hipError_t e_ = (expr);                                         \
        if (e_ != hipSuccess) return hip_fail(e_, #expr);               \
    } while (0)

constexpr uint64_t kMaxElems = (1ull << 31) - 1ull;
constexpr uint32_t kMaxW = 8192;
constexpr uint32_t kMaxBins = 65536;

inline uint64_t align_up(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

bool valid_eb(float eb) { return std::isfinite(eb) && eb >= 0x1p-100f && eb <= 0x1p100f; }
bool valid_nbins(uint32_t nb) { return nb >= 4u && nb <= kMaxBins && (nb & 1u) == 0u; }
bool valid_chunk(uint32_t s) { return s == 64u || s == 128u || s == 256u; }

bool shape_elems(comet_shape s, uint64_t *n) {
    if (!s.n || !s.c || !s.h || !s.w) return false;
    const uint64_t a = (uint64_t)s.n * s.c, b = (uint64_t)s.h * s.w;
    if (a > kMaxElems || b > kMaxElems) return false;
    const uint64_t t = a * b;
    if (t > kMaxElems) return false;
    *n = t;
    return true;
}

uint32_t ilog2(uint32_t v) { uint32_t l = 0; while ((1u << l) < v) ++l; return l; }

}  // namespace

// Persistent device words followed by the per-call control block.
struct DevState {
    uint32_t latched;      // first-come device errors since the last synchronising call
    uint32_t pad[3];
    Control ctl;
};

struct comet_ctx {
    int device = 0;
    int num_cu = 0;
    uint64_t max_elems = 0;
    uint32_t max_nbins = 0;
    uint32_t chunk_syms = COMET_DEFAULT_CHUNK_SYMS;
    uint32_t zero_chunks = 0;                       // containers of version 2: chunks of nothing but centre codes take no words
    // device memory
    DevState *state = nullptr;       // latched + Control, then histogram + descriptors (zero region)
    uint8_t *zero_region = nullptr;  // == (uint8_t*)&state->ctl
    uint64_t zero_cap = 0;
    uint16_t *codes = nullptr;
    uint32_t *rec_stage = nullptr;   // row-walking quantise kernel: staging area of every run's outlier records
    uint32_t *run_count = nullptr;   //   and per run: record count, non-zero inputs, verbatim records
    uint64_t max_runs = 0;
    uint64_t stage_bytes = 0;        // size of rec_stage, which also holds the band sums of a decompression
    uint32_t *hist_parts = nullptr;  // partial histograms of the row-walking quantise kernel, kPartsBytes
    bool parts_clean = false;        //   they are zero: the last call that used them has launched all of its kernels
    uint64_t *enc = nullptr;
    BookScratch book{};
    DecodeTables tables{};
    void *tables_blob = nullptr;
    // pinned host
    DevState *host_state = nullptr;
    Header *host_hdr = nullptr;
    CallResult *host_result = nullptr;              // written by the kernel that seals a container's header
    double *stats = nullptr;      // kStatsPartialMax partial sums and, behind them, the mean
    // optional per-kernel timing
    struct Timed { uint32_t id; hipEvent_t a, b; };
    bool profiling = false;
    std::vector<Timed> pool;      // pre-created event pairs
    size_t used = 0;
};

namespace {

constexpr uint64_t kPartsBytes = 4ull * kQuantHistPartsWords + 256u;

struct ZeroLayout {          // sub-allocation of the zero region for one call
    uint64_t off_hist, off_desc_e, bytes;
};

// Does the row-walking quantise kernel count its codes (what it can of them, for an alphabet larger than its window)?
// (Planes wider than kQuantRowsMaxW: all of them.)
bool quantize_counts(uint64_t n, uint32_t w, uint32_t nbins) { return nbins <= kHistWindowMax || n >= kQuantCountMin || w > kQuantRowsMaxW; }

// partial histograms of the row-walking quantise kernel for an alphabet of nbins
uint32_t hist_copies(uint32_t nbins) {
    if (nbins <= kBookPartsMax) return kQuantHistCopiesBook;
    const uint32_t c = kQuantHistPartsWords / nbins;
    return c < 1u ? 1u : (c > kQuantHistCopiesMax ? kQuantHistCopiesMax : c);
}

// nbins_hist: entries of the histogram itself (0 if the caller brings its own)
ZeroLayout zero_layout(uint32_t nbins_hist, uint64_t tiles_e) {
    ZeroLayout z;
    uint64_t o = align_up(sizeof(Control), 256);
    z.off_desc_e = o; o += align_up(8 * tiles_e, 256);
    z.off_hist = o; o += align_up(4ull * nbins_hist, 256);
    z.bytes = o;
    return z;
}

int status_to_error(uint32_t st) {
    if (st & ST_INTERNAL) return COMET_ERR_INTERNAL;
    if (st & ST_CODEBOOK) return COMET_ERR_CODEBOOK;
    if (st & ST_FORMAT) return COMET_ERR_FORMAT;
    if (st & ST_CAPACITY) return COMET_ERR_CAPACITY;
    return COMET_OK;
}

// Clears memory: a plain kernel rather than a memset node for callers that capture the call in a graph.  n16: 16-byte words.
// Only for partial histograms that a call may have left dirty: a compression's first kernel clears the control block, and its
// last one leaves the partial histograms zero for the next call (a launch of its own in front of the first one cost
// every call 3 us).
__global__ __launch_bounds__(256) void k_clear(uint4 *p, uint32_t n16) {
    const uint32_t i = blockIdx.x * 256u + threadIdx.x;
    if (i < n16) p[i] = make_uint4(0u, 0u, 0u, 0u);
}

__global__ void k_latch(DevState *s) {           // fold this call's status into the persistent word
    if (s->ctl.status) atomicOr(&s->latched, s->ctl.status);
}

// Brackets a kernel launch with two events when profiling is on.
struct TimedScope {
    comet_ctx *c; hipStream_t st; comet_ctx::Timed *t = nullptr;
    TimedScope(comet_ctx *ctx, hipStream_t s, uint32_t id) : c(ctx), st(s) {
        if (c && c->profiling && c->used < c->pool.size()) {
            t = &c->pool[c->used++];
            t->id = id;
            (void)hipEventRecord(t->a, st);
        }
    }
    ~TimedScope() { if (t) (void)hipEventRecord(t->b, st); }
};

struct ReconGeometry { uint32_t planes_per_unit, tile_rows, n_units, pitch, use_carry; size_t lds; };

bool recon_geometry(comet_shape s, ReconGeometry *g) {
    const uint64_t planes = (uint64_t)s.n * s.c;
    const uint64_t P = (uint64_t)s.h * s.w;
    g->pitch = s.w | 1u;
    if (P <= kDecTileElems) {
        uint64_t G = kDecTileElems / P;
        if (G > planes) G = planes;
        g->planes_per_unit = (uint32_t)G;
        g->tile_rows = (uint32_t)(G * s.h);
        g->n_units = (uint32_t)((planes + G - 1) / G);
        g->use_carry = 0;
    } else {
        uint32_t R = kDecTileElems / s.w;
        if (R < 1) R = 1;
        if (R > s.h) R = s.h;
        g->planes_per_unit = 1;
        g->tile_rows = R;
        g->n_units = (uint32_t)planes;
        g->use_carry = 1;
    }
    g->lds = (size_t)g->tile_rows * g->pitch * 4u + (g->use_carry ? (size_t)s.w * 4u : 0u);
    return g->lds <= 96u * 1024u;
}

int fused_opt_in();          // k_decode_scan: opt in to its dynamic LDS size (defined with the decompression)
// segments of the encode kernel: (chunks per segment, number of segments)
void encode_geometry(const comet_ctx *ctx, uint64_t n_chunks, uint32_t nbins, uint32_t *seg_chunks, uint32_t *n_seg);
// Work split of the quantise kernel: `grid` workgroups of four wavefronts, each wavefront on rows_per_wave consecutive rows.
// vec: columns per lane of the row-walking kernel (2 if W is even and the input is 8-byte aligned).
// chunk_align: if not 0, every run is a whole number of chunks of that many symbols (single-pass compression).
struct QuantGeom { uint32_t grid, run_elems, wg_elems, rows_per_wave, rows_per_wg, rows_per_step, vec, words64; };
// nbins: the alphabet (its histogram window decides how many workgroups a compute unit holds at once).
QuantGeom quantize_geometry(const comet_ctx *ctx, comet_shape s, uint64_t n, const void *x, uint32_t nbins, uint32_t elem_bytes = 4, uint32_t chunk_align = 0);

// Single-pass compression with a given code book: what the quantise kernel needs to encode its own codes.
struct SinglePass {
    const uint64_t *enc;       // encode table of the given lengths (k_codebook has run)
    uint32_t chunk_syms, zero_pair;
    uint32_t *chunk_off;       // chunk table of the container
    uint32_t *run_words;       // one entry per run
    uint32_t *work_words;      // kWordsRun or kWordsWide for every 64 symbols
    uint64_t stage_bytes;      // what is left of the staging area for records
};

// recs: receives what the kernels behind this one need to place the outlier records
// reset_ctl: the kernel clears the call's control block (no reuse)
// reuse_len: code book reuse (device u8[nbins], row-walking kernel only, with sp); else null
// in_type: element type of x (0 fp32, COMET_F16, COMET_BF16; the 16-bit types: row-walking kernel only, no reuse)
int launch_quantize(comet_ctx *ctx, const void *x, comet_shape s, uint64_t n, float eb, uint32_t nbins,
                    hipStream_t st, uint16_t *codes, uint32_t *hist_parts, uint32_t *rec, uint64_t rec_cap,
                    RecordArgs *recs, bool reset_ctl, const uint8_t *reuse_len = nullptr, int in_type = 0, const SinglePass *sp = nullptr) {
    if (in_type != 0 && (reuse_len || s.w > kQuantRowsMaxW)) return COMET_ERR_INVALID;
    if ((reuse_len != nullptr) != (sp != nullptr) || (reuse_len && s.w > kQuantRowsMaxW)) return COMET_ERR_INVALID;
    QuantArgs a{};
    a.x = x; a.n = n;
    a.divW = make_fastdiv(s.w); a.divH = make_fastdiv(s.h);
    a.eb = eb; a.ebx2 = 2.0f * eb; a.r = (float)(1.0 / (double)a.ebx2);
    a.radius = (int32_t)(nbins / 2u); a.nbins = nbins;
    a.win_n = nbins < kHistWindowMax ? nbins : kHistWindowMax;
    a.win_lo = (nbins - a.win_n) / 2u;
    a.codes = codes; a.ctl = &ctx->state->ctl;
    const QuantGeom g = quantize_geometry(ctx, s, n, x, nbins, in_type ? 2u : 4u, sp ? sp->chunk_syms : 0u);
    const uint32_t grid = g.grid;
    {
        a.rows_total = (uint32_t)((uint64_t)s.n * s.c * s.h);
        a.rows_per_wave = g.rows_per_wave; a.rows_per_wg = g.rows_per_wg;
        a.rows_per_step = g.rows_per_step;
        if ((uint64_t)grid * (kQuantBlock / kWave) > ctx->max_runs) return COMET_ERR_INTERNAL;
        a.stage = ctx->rec_stage;
        {
            const uint64_t room = (sp ? sp->stage_bytes : ctx->stage_bytes) / 8u / ((uint64_t)grid * kQuantWaves), most = 2ull * g.run_elems;    // (two records per element at most)
            a.rec_run = (uint32_t)(room < most ? room : most);
        }
        a.run_count = ctx->run_count;
        a.hist_parts = hist_parts;
        a.hist_copies = hist_copies(nbins);
        a.hist_shift = a.win_n <= 2048u ? 2u : 0u;            // four copies while they fit 32 KB
        const bool full = a.win_n == nbins;
        const bool counts = quantize_counts(n, s.w, nbins);
        const size_t lds = counts ? (((size_t)a.win_n << a.hist_shift) + kQuantBlock) * 4u + (full ? 0u : (size_t)(kQuantBlock / kWave) * kQuantOowList * 2u) : 0u;
        a.run_from = ctx->run_count + 3u * ctx->max_runs;
        a.reset_ctl = reset_ctl ? 1u : 0u;
        RecordArgs &ra = *recs;
        ra.x = x; ra.in_type = (uint32_t)in_type; ra.divW = a.divW; ra.divH = a.divH; ra.r = a.r; ra.ebx2 = a.ebx2; ra.eb = eb;
        ra.radius = a.radius; ra.nbins = nbins; ra.reuse_len = reuse_len; ra.n = n; ra.run_elems = a.run_elems = g.run_elems; ra.wg_elems = g.wg_elems;
        ra.n_wg = grid; ra.stage = ctx->rec_stage; ra.rec_run = a.rec_run; ra.run_count = ctx->run_count; ra.rec = rec; ra.rec_cap = rec_cap; ra.ctl = a.ctl;
        ra.ring = record_ring(s.w);
        // (an alphabet larger than the window: what the sweep does not count is counted from memory, behind it)
        auto count_codes = [&]() {
            if (full || reuse_len || s.w > kQuantRowsMaxW) return;
            CodeHistArgs h{};
            h.codes = codes; h.n = n; h.nbins = nbins; h.radius = nbins / 2u;
            h.win_n = nbins < kCodeHistWindow ? nbins : kCodeHistWindow;
            h.win_lo = (nbins - h.win_n) / 2u;
            h.run_from = a.run_from;
            h.divRun = make_fastdiv(g.run_elems);
            h.parts = hist_parts; h.copies = a.hist_copies;
            // one workgroup per compute unit, with at least 8192 codes (clearing and adding up its bins costs as much as those);
            // runs have kQuantRunMin codes or more and are at most 4 * kQuantRunsPerSimd per compute unit, so a slice sees fewer than kCodeHistRuns
            static_assert(8192u / kQuantRunMin + 3u <= kCodeHistRuns && 4u * kQuantRunsPerSimd + 3u <= kCodeHistRuns, "runs of a slice");
            uint64_t wg = (n + 8191u) / 8192u;
            if (wg > (uint64_t)ctx->num_cu) wg = (uint64_t)ctx->num_cu;
            const size_t lds_h = ((size_t)h.win_n + 4u * kCodeHistHot + kCodeHistBlock) * 4u;
            TimedScope ts(ctx, st, COMET_KERNEL_QUANTIZE);
            if (counts) hipLaunchKernelGGL(k_code_hist<true>, dim3((uint32_t)wg), dim3(kCodeHistBlock), lds_h, st, h);
            else hipLaunchKernelGGL(k_code_hist<false>, dim3((uint32_t)wg), dim3(kCodeHistBlock), lds_h, st, h);
        };
#define COMET_LAUNCH_QR_IN(VEC, NSEG, MULTI, IN)                                                                       \
        do {                                                                                                           \
            {                                                                                                          \
                TimedScope ts(ctx, st, COMET_KERNEL_QUANTIZE);                                                         \
                if (full) hipLaunchKernelGGL((k_quantize_rows<VEC, NSEG, MULTI, kHistFull, false, IN>), dim3(grid), dim3(kQuantBlock), lds, st, a);        \
                else if (counts) hipLaunchKernelGGL((k_quantize_rows<VEC, NSEG, MULTI, kHistPart, false, IN>), dim3(grid), dim3(kQuantBlock), lds, st, a); \
                else hipLaunchKernelGGL((k_quantize_rows<VEC, NSEG, MULTI, kHistNone, false, IN>), dim3(grid), dim3(kQuantBlock), lds, st, a);             \
            }                                                                                                          \
            count_codes();                                                                                             \
        } while (0)
#define COMET_LAUNCH_QR(VEC, NSEG, MULTI)                                                                              \
        do {                                                                                                           \
            if (in_type == COMET_F16) { COMET_LAUNCH_QR_IN(VEC, NSEG, MULTI, 1); break; }                              \
            if (in_type == COMET_BF16) { COMET_LAUNCH_QR_IN(VEC, NSEG, MULTI, 2); break; }                             \
            if (!reuse_len) { COMET_LAUNCH_QR_IN(VEC, NSEG, MULTI, 0); break; }                                        \
            {                                                                                                          \
                TimedScope ts(ctx, st, COMET_KERNEL_QUANTIZE);                                                         \
                if (a.enc_n == nbins) hipLaunchKernelGGL((k_quantize_rows<VEC, NSEG, MULTI, kHistFull, true>), dim3(grid), dim3(kQuantBlock), lds_single, st, a); \
                else hipLaunchKernelGGL((k_quantize_rows<VEC, NSEG, MULTI, kHistNone, true>), dim3(grid), dim3(kQuantBlock), lds_single, st, a);                 \
            }                                                                                                          \
        } while (0)
        a.reuse_len = reuse_len;
        const size_t lds_reuse = ((size_t)nbins + 7u) & ~(size_t)7u;    // the given length table, one byte per bin
        size_t lds_single = 0;
        if (sp) {
            // the kernel encodes its own codes: part of the encode table, a ring of codes and an assembly buffer per wavefront
            a.enc = sp->enc;
            a.enc_n = nbins < kEncTableMax ? nbins : kEncTableMax;
            a.enc_lo = (nbins - a.enc_n) / 2u;
            a.chunk_syms = sp->chunk_syms; a.zero_pair = sp->zero_pair;
            a.chunk_off = sp->chunk_off; a.run_words = sp->run_words; a.work_words = sp->work_words; a.words64 = g.words64;
            lds_single = (a.enc_n == nbins ? 0u : lds_reuse) + ((size_t)a.enc_n + 1u) * 8u +
                         (size_t)(kQuantBlock / kWave) * ((kEncRingSyms + 4u) * 2u + kEncRunBufWords * 4u);
        }
        const uint32_t lanes_per_row = s.w / g.vec;
        if (s.w > kQuantRowsMaxW) {
            TimedScope ts(ctx, st, COMET_KERNEL_QUANTIZE);
            const dim3 gr(grid), bl(kQuantBlock);
            if (g.vec == 2u && full) hipLaunchKernelGGL((k_quantize_rows<2, 0, false, kHistFull, false, 0>), gr, bl, lds, st, a);
            else if (g.vec == 2u) hipLaunchKernelGGL((k_quantize_rows<2, 0, false, kHistPart, false, 0>), gr, bl, lds, st, a);
            else if (full) hipLaunchKernelGGL((k_quantize_rows<1, 0, false, kHistFull, false, 0>), gr, bl, lds, st, a);
            else hipLaunchKernelGGL((k_quantize_rows<1, 0, false, kHistPart, false, 0>), gr, bl, lds, st, a);
        } else if (g.vec == 2u) {
            if (lanes_per_row <= 32u) COMET_LAUNCH_QR(2, 1, true);
            else if (lanes_per_row <= 64u) COMET_LAUNCH_QR(2, 1, false);
            else if (lanes_per_row <= 128u) COMET_LAUNCH_QR(2, 2, false);
            else COMET_LAUNCH_QR(2, 4, false);
        } else {
            if (lanes_per_row <= 32u) COMET_LAUNCH_QR(1, 1, true);
            else if (lanes_per_row <= 64u) COMET_LAUNCH_QR(1, 1, false);
            else if (lanes_per_row <= 128u) COMET_LAUNCH_QR(1, 2, false);
            else if (lanes_per_row <= 256u) COMET_LAUNCH_QR(1, 4, false);
            else COMET_LAUNCH_QR(1, 8, false);
        }
#undef COMET_LAUNCH_QR
#undef COMET_LAUNCH_QR_IN
    }
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

// Partial histograms that are zero, whatever the last call has left there, for a call that adds to them: dirty from here until all of
// its kernels have been launched.
int clean_parts(comet_ctx *ctx, hipStream_t st) {
    if (!ctx->parts_clean) {
        hipLaunchKernelGGL(k_clear, dim3((uint32_t)(kPartsBytes / 16u + 255u) / 256u), dim3(256), 0, st, reinterpret_cast<uint4 *>(ctx->hist_parts), (uint32_t)(kPartsBytes / 16u));
        HIP_TRY(hipGetLastError());
    }
    ctx->parts_clean = false;
    return COMET_OK;
}

// The outlier records of a quantisation that no code book follows; hist: receives the sum of the partial histograms, or null.
int launch_gather(comet_ctx *ctx, const RecordArgs &recs, hipStream_t st, uint32_t *hist, const uint32_t *parts) {
    TimedScope ts(ctx, st, COMET_KERNEL_GATHER);
    static_assert((uint32_t)(kGatherBlock / kWave) == kQuantWaves, "its grid is the quantise kernel's");
    hipLaunchKernelGGL(k_gather_records, dim3(recs.n_wg), dim3(kGatherBlock), kQuantWaves * record_lds(recs.ring), st, recs, hist, parts, hist_copies(recs.nbins));
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

// The code book kernel, behind the sort kernels that an alphabet too large for LDS needs.  b.ctl->n_active
// must be zero on entry (the call's control block has just been cleared).
int launch_codebook(comet_ctx *ctx, BookArgs &b, hipStream_t st) {
    TimedScope ts(ctx, st, COMET_KERNEL_CODEBOOK);
    // (up to kBookBySymbolMax bins the occurring symbols mostly fit LDS, and the launches would cost more than
    // the kernel's own sort does when they do not)
    if (!b.given_len && b.nbins > kBookBySymbolMax) {
        uint32_t tiles = 1;
        while (tiles * (uint32_t)kBookBlock < b.nbins) tiles <<= 1;
        const uint32_t total = tiles * (uint32_t)kBookBlock;          // <= kMaxBins: what the scratch arrays hold
        uint64_t *src = b.scratch.keys, *dst = b.scratch.iw;
        hipLaunchKernelGGL(k_book_sort_tiles, dim3(tiles), dim3(kBookBlock), 0, st, b);
        for (uint32_t run = (uint32_t)kBookBlock; run < total;) {
            const uint32_t left = total / run, ways = left >= 4u ? 4u : left;
            const dim3 grid(total / (uint32_t)kBookMergeBlock), block(kBookMergeBlock);
            if (ways == 4u) hipLaunchKernelGGL(k_book_merge<4u>, grid, block, 0, st, src, dst, run, b.ctl);
            else hipLaunchKernelGGL(k_book_merge<2u>, grid, block, 0, st, src, dst, run, b.ctl);
            uint64_t *t = src; src = dst; dst = t;
            run *= ways;
        }
        b.scratch.keys = src; b.scratch.iw = dst;
        b.presorted = 1u;
    }
    const uint32_t runs = b.recs.n_wg * kQuantWaves;
    b.lds_leaves = b.presorted ? kBookLdsLeaves : 0u;
    constexpr uint32_t waves = (uint32_t)(kBookBlock / kWave);
    static_assert(waves * (kDeriveBuf * 8u + 1024u * 4u) <= kBookLdsBytesLarge, "the widest ring");
    uint32_t lds = b.presorted ? kBookLdsBytesLarge : kBookLdsBytes;
    if (runs && lds < waves * record_lds(b.recs.ring)) lds = waves * record_lds(b.recs.ring);
    // one workgroup with records per compute unit at most: a compute unit holds no second one, and the wavefronts that are left with a
    // second run have their SIMD to themselves (a quarter of 411 M elements escaped: 1798 us with 320 workgroups, 1716 with 244)
    const uint32_t cus = ctx->num_cu > 1 ? (uint32_t)ctx->num_cu - 1u : 1u;
    uint32_t rec_wgs = (runs + waves - 1u) / waves;
    if (rec_wgs > cus) rec_wgs = cus;
    b.rec_wg_runs = rec_wgs ? (runs + rec_wgs - 1u) / rec_wgs : 0u;
    if (rec_wgs) rec_wgs = (runs + b.rec_wg_runs - 1u) / b.rec_wg_runs;
    hipLaunchKernelGGL(k_codebook, dim3(1u + rec_wgs), dim3(kBookBlock), lds, st, b);
    if (b.presorted) {                                       // (they leave an alphabet whose occurring symbols fit LDS alone)
        hipLaunchKernelGGL(k_book_depths, dim3((b.nbins + kBookDepthBlock - 1u) / kBookDepthBlock), dim3(kBookDepthBlock), 0, st, b);
        hipLaunchKernelGGL(k_book_codes, dim3((b.nbins + kBookBlock - 1u) / kBookBlock), dim3(kBookBlock), 0, st, b);
    }
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int launch_encode(comet_ctx *ctx, const uint16_t *codes, uint64_t n, uint32_t nbins, uint32_t chunk_syms,
                  hipStream_t st, uint32_t *chunk_off, uint8_t *container, uint64_t capacity,
                  uint32_t *payload, uint64_t payload_cap, uint64_t *payload_words_out, uint64_t *desc,
                  CallResult *host = nullptr, uint32_t *clear = nullptr, uint64_t clear_bytes = 0) {
    EncodeArgs a{};
    a.len8 = container ? container + kHeaderBytes : nullptr;      // the length section k_codebook has written
    a.codes = codes; a.n = n; a.chunk_syms = chunk_syms;
    a.zero_pair = ctx->zero_chunks ? ((nbins / 2u) << 16) | (nbins / 2u) : 0u;
    a.n_chunks = (uint32_t)((n + chunk_syms - 1) / chunk_syms);
    a.enc = ctx->enc; a.nbins = nbins;
    a.tbl_n = nbins < kEncTableMax ? nbins : kEncTableMax;
    a.tbl_lo = (nbins - a.tbl_n) / 2u;
    uint32_t seg, grid;
    encode_geometry(ctx, a.n_chunks, nbins, &seg, &grid);
    a.seg_chunks = seg;
    // table and a zero entry (or, for a large alphabet, the lengths of enc_len_window() symbols: whichever is larger), word counts
    const size_t lenw = a.len8 ? enc_len_window(nbins) + 8u : 0u;
    const size_t tbl_bytes = ((size_t)a.tbl_n + 1u) * 8u;
    a.tbl_room = (uint32_t)((a.tbl_n < nbins && lenw > tbl_bytes ? lenw : tbl_bytes) + 7u) & ~7u;
    const size_t lds_count = (size_t)a.tbl_room + (size_t)seg * 4u;
    static_assert(kBookBySymbolMax >= kEncPackWindow, "the window lies inside the alphabet");
    const bool pack_wide = nbins > kBookBySymbolMax && seg >= kEncPackMinChunks;
    const size_t lds_pack = (pack_wide ? (size_t)kEncPackWindow * 4u : ((size_t)a.tbl_n + 1u) * 8u) + (size_t)((pack_wide ? kEncBlockWide : kEncBlock) / kWave) * kEncBufWords * 4u;
    a.chunk_off = chunk_off; a.container = container; a.capacity = capacity;
    a.payload = payload; a.payload_cap_words = payload_cap; a.payload_words_out = payload_words_out;
    a.desc = desc; a.ctl = &ctx->state->ctl;
    a.latched = container ? &ctx->state->latched : nullptr;
    a.host = host;
    a.clear = reinterpret_cast<uint4 *>(clear); a.clear_n16 = (uint32_t)((clear_bytes + 15u) / 16u);
    const bool full = (a.tbl_n == nbins);
    const bool wide = a.len8 && enc_wide(nbins);             // (a stage call brings no lengths)
#define COMET_LAUNCH_ENC(S)                                                                                            \
    do {                                                                                                               \
        {                                                                                                              \
            TimedScope ts(ctx, st, COMET_KERNEL_ENCODE_COUNT);                                                         \
            if (full) hipLaunchKernelGGL((k_encode_count<S, true, kEncBlock>), dim3(grid), dim3(kEncBlock), lds_count, st, a);    \
            else if (wide) hipLaunchKernelGGL((k_encode_count<S, false, kEncBlockWide>), dim3(grid), dim3(kEncBlockWide), lds_count, st, a); \
            else hipLaunchKernelGGL((k_encode_count<S, false, kEncBlock>), dim3(grid), dim3(kEncBlock), lds_count, st, a);        \
        }                                                                                                              \
        TimedScope ts(ctx, st, COMET_KERNEL_ENCODE);                                                                   \
        if (full) hipLaunchKernelGGL((k_encode_pack<S, true, kEncBlock>), dim3(grid), dim3(kEncBlock), lds_pack, st, a); \
        else if (pack_wide) hipLaunchKernelGGL((k_encode_pack<S, false, kEncBlockWide>), dim3(grid), dim3(kEncBlockWide), lds_pack, st, a); \
        else hipLaunchKernelGGL((k_encode_pack<S, false, kEncBlock>), dim3(grid), dim3(kEncBlock), lds_pack, st, a);   \
    } while (0)
    if (chunk_syms == 64u) COMET_LAUNCH_ENC(64);
    else if (chunk_syms == 128u) COMET_LAUNCH_ENC(128);
    else COMET_LAUNCH_ENC(256);
#undef COMET_LAUNCH_ENC
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

void encode_geometry(const comet_ctx *ctx, uint64_t n_chunks, uint32_t nbins, uint32_t *seg_chunks, uint32_t *n_seg) {
    // one segment of consecutive chunks per workgroup: about as many segments as workgroups fit the chip
    const uint64_t want = (uint64_t)ctx->num_cu * 6u;
    uint64_t seg = (n_chunks + want - 1) / want;
    seg = (seg + 3u) & ~(uint64_t)3u;
    if (seg < 4u) seg = 4u;
    const uint64_t most = enc_wide(nbins) ? kEncSegChunksWide : kEncSegChunksMax;
    if (seg > most) seg = most;
    *seg_chunks = (uint32_t)seg;
    *n_seg = (uint32_t)((n_chunks + seg - 1) / seg);
}

QuantGeom quantize_geometry(const comet_ctx *ctx, comet_shape s, uint64_t n, const void *x, uint32_t nbins, uint32_t elem_bytes, uint32_t chunk_align) {
    QuantGeom g{};
    g.vec = 1;
    {
        const uint64_t rows_total = (uint64_t)s.n * s.c * s.h;
        // two columns per lane: every row then starts at an even element, so pairs are aligned to their size
        if ((s.w & 1u) == 0u && ((uintptr_t)x & (2u * elem_bytes - 1u)) == 0u) g.vec = 2;
        const uint32_t lanes_per_row = s.w / g.vec;
        const uint32_t K = lanes_per_row <= 32u ? (uint32_t)kWave / lanes_per_row : 1u;
        g.rows_per_step = K;
        // runs of whole steps; single-pass compression: and of whole chunks (chunk sizes are powers of two)
        uint32_t unit = K;
        if (chunk_align) {
            uint32_t rows_per_chunk = chunk_align;               // rows after which a chunk boundary is a row boundary
            for (uint32_t w = s.w; (w & 1u) == 0u && rows_per_chunk > 1u; w >>= 1) rows_per_chunk >>= 1;
            unit = K / std::gcd(K, rows_per_chunk) * rows_per_chunk;
        }
        // a few wavefronts per SIMD, but runs of at least kReuseRunElems elements (every run re-reads one row), or fewer, down to
        // kQuantRunMin, while that leaves SIMDs without a run (one image, 64 x 28 x 28: 26 wavefronts -> 102, the call 36.5 us -> 33.2)
        // All runs should be resident at once: a run that has to wait for a place makes the launch take two rounds.
        // A workgroup is one wavefront per SIMD; how many a compute unit holds follows from the LDS they need (the
        // histogram window of a large alphabet leaves room for three; the encoder's ring and tables of the single-pass
        // compression for four).
        uint32_t runs_per_simd = chunk_align ? kQuantRunsPerSimdSingle : kQuantRunsPerSimd;
        if (!chunk_align) {
            const uint32_t win_n = nbins < kHistWindowMax ? nbins : kHistWindowMax;
            const size_t window = (((size_t)win_n << (win_n <= 2048u ? 2u : 0u)) + kQuantBlock) * 4u +
                                  (win_n < nbins ? (size_t)(kQuantBlock / kWave) * kQuantOowList * 2u : 0u);
            const size_t lds = (quantize_counts(n, s.w, nbins) ? window : 0u) + kQuantStaticLds;
            const uint32_t fit = (uint32_t)(kLdsPerCu / lds);
            if (fit < runs_per_simd) runs_per_simd = fit ? fit : 1u;
        }
        const uint64_t want = (uint64_t)ctx->num_cu * 4u * runs_per_simd;
        const uint64_t share = n / ((uint64_t)ctx->num_cu * 4u);
        const uint64_t least = chunk_align || share >= kReuseRunElems ? kReuseRunElems : (share < kQuantRunMin ? kQuantRunMin : share);
        if (s.w > kQuantRowsMaxW) {
            // wide planes: whole rows, or less than half a row, in multiples of a batch of steps
            uint64_t per = (n + want - 1) / want;
            if (per < least) per = least;
            per = 2u * per < s.w ? (per + 255u) / 256u * 256u : (per + s.w - 1u) / s.w * s.w;
            const uint64_t waves = (n + per - 1) / per;
            g.run_elems = (uint32_t)per; g.wg_elems = kQuantWaves * g.run_elems;
            g.grid = (uint32_t)((waves + kQuantWaves - 1u) / kQuantWaves);
            return g;
        }
        uint64_t per = (rows_total + want - 1) / want;
        const uint64_t min_rows = (least + s.w - 1u) / s.w;
        if (per < min_rows) per = min_rows;
        per = (per + unit - 1) / unit * unit;
        if (per > rows_total) per = (rows_total + unit - 1) / unit * unit;
        // a run must stay below 2^28 elements (buffer offsets): cannot be exceeded, rows_total * w < 2^31 and
        // the run count is in the thousands unless the tensor itself is small
        const uint64_t waves = (rows_total + per - 1) / per;
        const bool quarters = chunk_align && share < kReuseRunElems && per >= 2u * unit;     // a workgroup takes one run (kReuseRunElems)
        const uint64_t sub = quarters ? (per / unit + kQuantWaves - 1u) / kQuantWaves * unit : per, per_wg = quarters ? per : kQuantWaves * per;
        g.words64 = quarters ? kWordsWide : kWordsRun;
        g.rows_per_wave = (uint32_t)sub; g.rows_per_wg = (uint32_t)per_wg;
        g.run_elems = (uint32_t)(sub * s.w); g.wg_elems = (uint32_t)(per_wg * s.w);
        g.grid = (uint32_t)(quarters ? waves : (waves + kQuantWaves - 1u) / kQuantWaves);
        return g;
    }
}

}  // namespace

extern "C" {

int comet_create(comet_ctx **out, uint64_t max_elems, uint32_t max_nbins) {
    if (!out || max_elems == 0 || max_elems > kMaxElems || !valid_nbins(max_nbins)) return COMET_ERR_INVALID;
    comet_ctx *c = new (std::nothrow) comet_ctx();
    if (!c) return COMET_ERR_NOMEM;
    c->max_elems = max_elems;
    c->max_nbins = max_nbins;
    int rc = COMET_OK;
    auto fail = [&](int code) { comet_destroy(c); return code; };
    hipError_t e;
    if ((e = hipGetDevice(&c->device)) != hipSuccess) return fail(hip_fail(e, "hipGetDevice"));
    hipDeviceProp_t prop;
    if ((e = hipGetDeviceProperties(&prop, c->device)) != hipSuccess) return fail(hip_fail(e, "hipGetDeviceProperties"));
    c->num_cu = prop.multiProcessorCount > 0 ? prop.multiProcessorCount : 256;

    // scan descriptors: one per segment of the quantise / encode kernels (worst case over chunk sizes)
    const uint64_t tiles_e = (uint64_t)c->num_cu * 8u + max_elems / 64u / kEncSegChunksWide + 16u;
    const ZeroLayout z = zero_layout(kMaxBins, tiles_e);
    c->zero_cap = z.bytes;
    const uint64_t parts_at = align_up(offsetof(DevState, ctl) + z.bytes, 256);
    const uint64_t state_bytes = parts_at + kPartsBytes;     // the partial histograms behind it: 2 MB
    if ((e = hipMalloc((void **)&c->state, state_bytes)) != hipSuccess) return fail(COMET_ERR_NOMEM);
    if ((e = hipMemset(c->state, 0, state_bytes)) != hipSuccess) return fail(hip_fail(e, "hipMemset"));
    c->zero_region = reinterpret_cast<uint8_t *>(&c->state->ctl);
    c->hist_parts = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(c->state) + parts_at);
    c->parts_clean = true;                                   // (just cleared)
    if ((e = hipMalloc((void **)&c->codes, align_up(2 * max_elems + 64, 256))) != hipSuccess) return fail(COMET_ERR_NOMEM);
    if ((e = hipMalloc((void **)&c->enc, 8ull * kMaxBins)) != hipSuccess) return fail(COMET_ERR_NOMEM);
    if ((e = hipMalloc((void **)&c->stats, 8ull * (kStatsPartialMax + 1u))) != hipSuccess) return fail(COMET_ERR_NOMEM);
    c->max_runs = (uint64_t)c->num_cu * 4u * kQuantRunsPerSimd + 8u;
    c->stage_bytes = c->max_runs * kQuantRecRun * 8ull;
    if (c->stage_bytes < band_bytes_max(max_elems)) c->stage_bytes = band_bytes_max(max_elems);
    if ((e = hipMalloc((void **)&c->rec_stage, c->stage_bytes)) != hipSuccess) return fail(COMET_ERR_NOMEM);
    // (a fourth array of one entry per run: the words of every run of the single-pass compression)
    if ((e = hipMalloc((void **)&c->run_count, 4ull * c->max_runs * 4ull)) != hipSuccess) return fail(COMET_ERR_NOMEM);
    {
        // one blob: book scratch + decode tables
        uint64_t o = 0;
        const uint64_t o_keys = o; o += 8ull * kMaxBins;
        const uint64_t o_iw = o; o += 8ull * kMaxBins;
        const uint64_t o_lp = o; o += 4ull * kMaxBins;
        const uint64_t o_ip = o; o += 4ull * kMaxBins;
        const uint64_t o_limit = o; o += 8ull * 72;
        const uint64_t o_first = o; o += 8ull * 72;
        const uint64_t o_findex = o; o += 4ull * 72;
        const uint64_t o_lut = o; o += 4ull * kLutSize;
        const uint64_t o_lut16 = o; o += 2ull * kLut16Size;
        const uint64_t o_sub16 = o; o += 2ull * kSubEntries;
        const uint64_t o_meta = o; o += 64;
        const uint64_t o_sorted = o; o += 2ull * kMaxBins;
        const uint64_t o_resid = o; o += 2ull * kMaxBins;
        const uint64_t o_tcnt = o; o += 4ull * (kMaxBins / kBookBlock) * kBookLens;
        uint8_t *blob = nullptr;
        if ((e = hipMalloc((void **)&blob, align_up(o, 256))) != hipSuccess) return fail(COMET_ERR_NOMEM);
        c->tables_blob = blob;
        c->book.keys = (uint64_t *)(blob + o_keys); c->book.iw = (uint64_t *)(blob + o_iw);
        c->book.leaf_parent = (uint32_t *)(blob + o_lp); c->book.int_parent = (uint32_t *)(blob + o_ip);
        c->tables.limit = (uint64_t *)(blob + o_limit); c->tables.first_code = (uint64_t *)(blob + o_first);
        c->tables.first_index = (uint32_t *)(blob + o_findex); c->tables.lut = (uint32_t *)(blob + o_lut);
        c->tables.meta = (uint32_t *)(blob + o_meta); c->tables.sorted = (uint16_t *)(blob + o_sorted);
        c->tables.resid = (uint16_t *)(blob + o_resid);
        c->book.tile_cnt = (uint32_t *)(blob + o_tcnt);
        c->tables.lut16 = (uint16_t *)(blob + o_lut16);
        c->tables.sub16 = (uint16_t *)(blob + o_sub16);
    }
    if ((e = hipHostMalloc((void **)&c->host_state, sizeof(DevState) + sizeof(Header) + sizeof(CallResult), hipHostMallocDefault)) != hipSuccess)
        return fail(COMET_ERR_NOMEM);
    c->host_hdr = reinterpret_cast<Header *>(reinterpret_cast<uint8_t *>(c->host_state) + sizeof(DevState));
    c->host_result = reinterpret_cast<CallResult *>(c->host_hdr + 1);

    // kernels that need more than 64 KB of dynamic LDS must opt in
    if ((e = hipFuncSetAttribute((const void *)k_reconstruct<0>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024)) != hipSuccess)
        return fail(hip_fail(e, "hipFuncSetAttribute(k_reconstruct<0>)"));
    if ((e = hipFuncSetAttribute((const void *)k_reconstruct<1>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024)) != hipSuccess)
        return fail(hip_fail(e, "hipFuncSetAttribute(k_reconstruct<1>)"));
    if (fused_opt_in() != COMET_OK) return fail(COMET_ERR_HIP);
    for (const void *fn : {(const void *)k_encode_count<64, false, kEncBlockWide>, (const void *)k_encode_count<128, false, kEncBlockWide>,
                           (const void *)k_encode_count<256, false, kEncBlockWide>})
        if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024)) != hipSuccess)
            return fail(hip_fail(e, "hipFuncSetAttribute(k_encode_count)"));
    if ((e = hipFuncSetAttribute((const void *)k_codebook, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kBookLdsBytesLarge)) != hipSuccess)
        return fail(hip_fail(e, "hipFuncSetAttribute(k_codebook)"));
    for (const void *fn : {(const void *)k_code_hist<true>, (const void *)k_code_hist<false>})
        if ((e = hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)((kCodeHistWindow + 4u * kCodeHistHot + kCodeHistBlock) * 4u))) != hipSuccess)
            return fail(hip_fail(e, "hipFuncSetAttribute(k_code_hist)"));
    (void)rc;
    *out = c;
    return COMET_OK;
}

void comet_destroy(comet_ctx *c) {
    if (!c) return;
    if (c->state) (void)hipFree(c->state);
    if (c->codes) (void)hipFree(c->codes);
    if (c->stats) (void)hipFree(c->stats);
    if (c->rec_stage) (void)hipFree(c->rec_stage);
    if (c->run_count) (void)hipFree(c->run_count);
    if (c->enc) (void)hipFree(c->enc);
    if (c->tables_blob) (void)hipFree(c->tables_blob);
    if (c->host_state) (void)hipHostFree(c->host_state);
    for (auto &t : c->pool) { (void)hipEventDestroy(t.a); (void)hipEventDestroy(t.b); }
    delete c;
}

int comet_set_zero_chunks(comet_ctx *ctx, int enable) {
    if (!ctx) return COMET_ERR_INVALID;
    ctx->zero_chunks = enable ? 1u : 0u;
    return COMET_OK;
}

int comet_set_chunk_syms(comet_ctx *ctx, uint32_t chunk_syms) {
    if (!ctx || !valid_chunk(chunk_syms)) return COMET_ERR_INVALID;
    ctx->chunk_syms = chunk_syms;
    return COMET_OK;
}

uint64_t comet_compress_bound(comet_shape s, uint32_t nbins, uint32_t chunk_syms) {
    uint64_t n;
    if (!shape_elems(s, &n) || !valid_nbins(nbins) || chunk_syms == 0) return 0;
    const uint64_t n_chunks = (n + chunk_syms - 1) / chunk_syms;
    uint64_t sz = kHeaderBytes;
    sz = align16(sz + nbins);
    sz = align16(sz + 4 * n_chunks);
    sz = align16(sz + 16 * n);                          // every element both escaped and verbatim
    sz += 4 * ((17 * n + 31) / 32 + n_chunks);         // an optimal code averages < log2(nbins) + 1 <= 17 bits
    return sz;
}

namespace {
int compress_impl(comet_ctx *ctx, const void *dev_in, int in_type, comet_shape s, float eb, uint32_t nbins, const uint8_t *dev_len,
                  void *stream, void *dev_out, uint64_t capacity, uint64_t *bytes_out);
}

int comet_compress(comet_ctx *ctx, const float *dev_in, comet_shape s, float eb, uint32_t nbins,
                   void *stream, void *dev_out, uint64_t capacity, uint64_t *bytes_out) {
    return compress_impl(ctx, dev_in, 0, s, eb, nbins, nullptr, stream, dev_out, capacity, bytes_out);
}

int comet_compress_16(comet_ctx *ctx, const void *dev_in, int dtype, comet_shape s, float eb, uint32_t nbins,
                      void *stream, void *dev_out, uint64_t capacity, uint64_t *bytes_out) {
    if ((dtype != COMET_F16 && dtype != COMET_BF16) || s.w > kQuantRowsMaxW) return COMET_ERR_INVALID;
    return compress_impl(ctx, dev_in, dtype, s, eb, nbins, nullptr, stream, dev_out, capacity, bytes_out);
}

int comet_compress_with_codebook(comet_ctx *ctx, const float *dev_in, comet_shape s, float eb, uint32_t nbins,
                                 const uint8_t *dev_len, void *stream, void *dev_out, uint64_t capacity,
                                 uint64_t *bytes_out) {
    if (!dev_len || nbins > kQuantReuseMaxBins || s.w > kQuantRowsMaxW) return COMET_ERR_INVALID;
    return compress_impl(ctx, dev_in, 0, s, eb, nbins, dev_len, stream, dev_out, capacity, bytes_out);
}

namespace {
int compress_impl(comet_ctx *ctx, const void *dev_in, int in_type, comet_shape s, float eb, uint32_t nbins, const uint8_t *dev_len,
                  void *stream, void *dev_out, uint64_t capacity, uint64_t *bytes_out) {
    uint64_t n;
    if (!ctx || !dev_in || !dev_out || !shape_elems(s, &n) || !valid_eb(eb) || !valid_nbins(nbins) ||
        s.w > kMaxW || ((uintptr_t)dev_out & 15u) || ((uintptr_t)dev_in & 15u)) return COMET_ERR_INVALID;
    if (n > ctx->max_elems || nbins > ctx->max_nbins) return COMET_ERR_NOMEM;
    hipStream_t st = (hipStream_t)stream;
    const uint32_t S = ctx->chunk_syms;
    const uint64_t n_chunks = (n + S - 1) / S;
    uint32_t e_seg, e_grid;
    encode_geometry(ctx, n_chunks, nbins, &e_seg, &e_grid);
    const QuantGeom qg = quantize_geometry(ctx, s, n, dev_in, nbins, in_type ? 2u : 4u, dev_len ? S : 0u);
    const uint64_t tiles_e = e_grid;

    Header proto{};
    proto.magic = kMagic; proto.version = ctx->zero_chunks ? 2u : 1u; proto.N = s.n; proto.C = s.c; proto.H = s.h; proto.W = s.w;
    proto.nbins = nbins; proto.chunk_syms = S; proto.n_chunks = (uint32_t)n_chunks;
    const float ebx2 = 2.0f * eb;
    const float r = (float)(1.0 / (double)ebx2);
    memcpy(&proto.eb_bits, &eb, 4); memcpy(&proto.ebx2_bits, &ebx2, 4); memcpy(&proto.r_bits, &r, 4);
    proto.off_len = kHeaderBytes;
    proto.off_chunk = align16(proto.off_len + nbins);
    proto.off_outlier = align16(proto.off_chunk + 4 * n_chunks);
    if (proto.off_outlier > capacity) return COMET_ERR_CAPACITY;

    const ZeroLayout z = zero_layout(nbins, tiles_e);
    if (z.bytes > ctx->zero_cap) return COMET_ERR_NOMEM;
    const bool parts = !dev_len;                             // this call adds to the partial histograms
    uint32_t *hist = reinterpret_cast<uint32_t *>(ctx->zero_region + z.off_hist);
    uint64_t *desc_e = reinterpret_cast<uint64_t *>(ctx->zero_region + z.off_desc_e);
    uint8_t *out = static_cast<uint8_t *>(dev_out);

    BookArgs b{};
    b.hist = hist; b.given_len = dev_len; b.nbins = nbins; b.len_out = out + proto.off_len; b.code_out = nullptr; b.enc = ctx->enc;
    b.narrow = n < 0x7fffffffull ? 1u : 0u;
    b.scratch = ctx->book; b.ctl = &ctx->state->ctl; b.hdr = reinterpret_cast<Header *>(out); b.proto = proto; b.capacity = capacity;
    uint32_t *rec = reinterpret_cast<uint32_t *>(out + proto.off_outlier);
    const uint64_t rec_cap = (capacity - proto.off_outlier) / 8u;
    uint32_t *chunk_off = reinterpret_cast<uint32_t *>(out + proto.off_chunk);
    int rc;
    RecordArgs recs{};
    if (dev_len) {
        // Single pass over the input: the code book first (header, length section, encode table), then the quantise
        // kernel encodes its own codes into the work area, then the words of every run move to their place.
        b.reset_ctl = 1u;
        if ((rc = launch_codebook(ctx, b, st))) return rc;
        SinglePass sp{};
        sp.enc = ctx->enc; sp.chunk_syms = S;
        sp.zero_pair = ctx->zero_chunks ? ((nbins / 2u) << 16) | (nbins / 2u) : 0u;
        sp.chunk_off = chunk_off;
        sp.run_words = ctx->run_count + 3u * ctx->max_runs;
        sp.work_words = reinterpret_cast<uint32_t *>(ctx->codes);
        sp.stage_bytes = ctx->stage_bytes;
        if (qg.words64 != kWordsRun) {                       // (tensors so small that the end of the staging area has room for any code words)
            static_assert(4u * kQuantRunsPerSimd * kQuantRecRun * 8u >= 4u * kReuseRunElems * kWordsWide / 64u * 4u + 4u * 4u * 256u * 8u, "and for 256 records per run");
            sp.stage_bytes = (sp.stage_bytes - (n + 63u) / 64u * kWordsWide * 4u) & ~255ull;
            sp.work_words = reinterpret_cast<uint32_t *>(reinterpret_cast<uint8_t *>(ctx->rec_stage) + sp.stage_bytes);
        }
        if ((rc = launch_quantize(ctx, dev_in, s, n, eb, nbins, st, nullptr, nullptr, rec, rec_cap, &recs, false, dev_len, 0, &sp))) return rc;
        PlaceArgs p{};
        p.run_words = sp.run_words;
        p.rows_per_wave = qg.rows_per_wave; p.rows_per_wg = qg.rows_per_wg; p.words64 = qg.words64; p.rows_total = (uint32_t)((uint64_t)s.n * s.c * s.h); p.W = s.w;
        p.recs = recs;
        p.n_runs = qg.words64 == kWordsRun ? (p.rows_total + qg.rows_per_wave - 1u) / qg.rows_per_wave : qg.grid * kQuantWaves;
        p.chunk_syms = S; p.work_words = sp.work_words; p.container = out; p.capacity = capacity;
        p.ctl = &ctx->state->ctl; p.latched = &ctx->state->latched; p.host = bytes_out ? ctx->host_result : nullptr;
        constexpr uint32_t per_wg = (uint32_t)(kPlaceBlock / kWave);
        TimedScope ts(ctx, st, COMET_KERNEL_ENCODE);
        hipLaunchKernelGGL(k_place_payload, dim3((p.n_runs + per_wg - 1u) / per_wg), dim3(kPlaceBlock), per_wg * record_lds(recs.ring), st, p);
        HIP_TRY(hipGetLastError());
    } else {
        if (parts && (rc = clean_parts(ctx, st))) return rc;
        if ((rc = launch_quantize(ctx, dev_in, s, n, eb, nbins, st, ctx->codes, ctx->hist_parts, rec, rec_cap, &recs, true, nullptr, in_type))) return rc;
        if (parts && nbins > kBookPartsMax && nbins <= kBookBySymbolMax) {
            if ((rc = launch_gather(ctx, recs, st, hist, ctx->hist_parts))) return rc;
        } else {
            b.recs = recs;
            if (parts) { b.hist_parts = ctx->hist_parts; b.hist_copies = hist_copies(nbins); b.hist_sum = hist; }
        }
        if ((rc = launch_codebook(ctx, b, st))) return rc;
        if ((rc = launch_encode(ctx, ctx->codes, n, nbins, S, st, chunk_off, out, capacity, nullptr, 0, nullptr, desc_e,
                                bytes_out ? ctx->host_result : nullptr, parts ? ctx->hist_parts : nullptr,
                                parts ? 4ull * nbins * hist_copies(nbins) : 0ull))) return rc;
        if (parts) ctx->parts_clean = true;
    }
    if (bytes_out) {
        HIP_TRY(hipStreamSynchronize(st));
        // this call's own bits, and whatever earlier asynchronous calls on this context have latched
        const uint32_t own = ctx->host_result->own, stt = ctx->host_result->latched;
        if (!own) *bytes_out = ctx->host_result->total_bytes;
        if (stt) {
            HIP_TRY(hipMemsetAsync(&ctx->state->latched, 0, 4, st));
            HIP_TRY(hipStreamSynchronize(st));
            return status_to_error(stt);
        }
    }
    return COMET_OK;
}
}  // namespace

namespace {
// What a decompression needs beyond its input and its output: the control block, the decode tables and the
// residual work buffer, in a context's workspace or in the library's static scratch array.
struct DecompWs {
    DevState *state;
    DecodeTables tables;
    int16_t *resid;            // one int16 per element, max_elems of them
    uint64_t max_elems;
    uint8_t *band;             // sums of the reconstruction in bands
    uint64_t band_bytes;
    int num_cu;
    uint32_t chunk_syms;       // chunk size the launch geometry is estimated with
    comet_ctx *prof;           // per-kernel timing, or null
    int32_t *dev_status;       // if set, the tables kernel stores 0 or COMET_ERR_FORMAT there
};
int decompress_impl(const DecompWs &ws, const void *dev_in, uint64_t bytes, comet_shape s, void *stream, void *dev_out, int out_type);
DecompWs ctx_ws(comet_ctx *ctx) {
    DecompWs ws{};
    ws.state = ctx->state; ws.tables = ctx->tables; ws.resid = reinterpret_cast<int16_t *>(ctx->codes);
    ws.band = reinterpret_cast<uint8_t *>(ctx->rec_stage); ws.band_bytes = ctx->stage_bytes;
    ws.max_elems = ctx->max_elems; ws.num_cu = ctx->num_cu; ws.chunk_syms = ctx->chunk_syms; ws.prof = ctx; ws.dev_status = nullptr;
    return ws;
}
}

int comet_decompress(comet_ctx *ctx, const void *dev_in, uint64_t bytes, comet_shape s, void *stream, float *dev_out) {
    if (!ctx) return COMET_ERR_INVALID;
    return decompress_impl(ctx_ws(ctx), dev_in, bytes, s, stream, dev_out, 0);
}

int comet_decompress_16(comet_ctx *ctx, const void *dev_in, uint64_t bytes, comet_shape s, int dtype, void *stream, void *dev_out) {
    if (!ctx || (dtype != COMET_F16 && dtype != COMET_BF16)) return COMET_ERR_INVALID;
    return decompress_impl(ctx_ws(ctx), dev_in, bytes, s, stream, dev_out, dtype);
}

namespace {
constexpr size_t kFuLdsBytes = (size_t)kFuWaves * kFuRegionWords * 4u;

// instantiation of k_decode_scan for (64-lane segments per row, lane mapping, output type, columns per lane)
const void *fused_kernel(int nseg, int mode, int out, int vec) {
#define COMET_FU(NS, MO, OU, VE) if (nseg == NS && mode == MO && out == OU && vec == VE) return (const void *)k_decode_scan<NS, MO, OU, VE>;
#define COMET_FU_OUT(OU)                                                                     \
    COMET_FU(1, 0, OU, 1) COMET_FU(1, 1, OU, 1) COMET_FU(1, 2, OU, 1) COMET_FU(2, 2, OU, 1) \
    COMET_FU(4, 2, OU, 1) COMET_FU(8, 2, OU, 1) COMET_FU(1, 0, OU, 2) COMET_FU(1, 1, OU, 2) \
    COMET_FU(1, 2, OU, 2) COMET_FU(2, 2, OU, 2) COMET_FU(4, 2, OU, 2)
    COMET_FU_OUT(0) COMET_FU_OUT(1) COMET_FU_OUT(2)
#undef COMET_FU_OUT
#undef COMET_FU
    return nullptr;
}

// every instantiation needs more than 64 KB of dynamic LDS: opt in once per device
int fused_opt_in() {
    static const int nsegs[] = {1, 2, 4, 8};
    for (int out = 0; out < 3; ++out)
        for (int vec = 1; vec <= 2; ++vec)
            for (int mode = 0; mode < 3; ++mode)
                for (int ns : nsegs) {
                    const void *fn = fused_kernel(ns, mode, out, vec);
                    if (fn) HIP_TRY(hipFuncSetAttribute(fn, hipFuncAttributeMaxDynamicSharedMemorySize, (int)kFuLdsBytes));
                }
    return COMET_OK;
}

// Work split of k_decode_scan: units of G whole planes, one wavefront per unit at a time.  A unit costs as
// many strips (decode phases of 64 symbols per lane) as its elements take at about 4032 per strip, and the
// launch takes as long as its busiest wavefront: G minimises (units per wavefront) * (strips per unit).
struct FusedGeom { uint32_t G, n_units, grid; };
FusedGeom fused_geometry(int num_cu, comet_shape s) {
    const uint64_t planes = (uint64_t)s.n * s.c, P = (uint64_t)s.h * s.w;
    const uint64_t waves = (uint64_t)num_cu * kFuWaves;
    auto strips_of = [&](uint64_t G) {                       // a unit that starts on a chunk boundary
        uint64_t a = 0, cnt = 0;
        const uint64_t end = G * P;
        while (a < end) {
            uint64_t lim = ((a >> 6) + 64u) * 64u / s.w * s.w;
            a = lim < end ? lim : end;
            ++cnt;
        }
        return cnt;
    };
    uint64_t g_max = 2u * ((planes + waves - 1) / waves) + 2u * (4096u / P) + 2u;
    if (g_max > planes) g_max = planes;
    uint64_t best_g = 1, best_cost = ~0ull;
    for (uint64_t G = 1; G <= g_max; ++G) {
        const uint64_t units = (planes + G - 1) / G;
        const uint64_t cost = ((units + waves - 1) / waves) * strips_of(G);
        if (cost < best_cost) { best_cost = cost; best_g = G; }
    }
    FusedGeom f;
    f.G = (uint32_t)best_g;
    f.n_units = (uint32_t)((planes + best_g - 1) / best_g);
    f.grid = (uint32_t)(f.n_units < (uint64_t)num_cu ? f.n_units : (uint64_t)num_cu);
    return f;
}

// Huffman decode of a whole container into int16 residuals.
void launch_decode_chunks(const DecompWs &ws, const DsArgs &d, hipStream_t st) {
    // groups of 64 chunks, one per wavefront at a time; the same number of groups for every
    // wavefront of a grid that is resident at once (estimated with the context's chunk size)
    const uint64_t groups = (d.n + (uint64_t)ws.chunk_syms * kWave - 1) / ((uint64_t)ws.chunk_syms * kWave);
    const uint64_t resident = (uint64_t)ws.num_cu * 4u * kDsWaves;
    const uint64_t per_wave = (groups + resident - 1) / resident;
    const uint64_t waves = (groups + per_wave - 1) / per_wave;
    const uint32_t grid = (uint32_t)((waves + kDsWaves - 1) / kDsWaves);
    TimedScope ts(ws.prof, st, COMET_KERNEL_DECODE);
    hipLaunchKernelGGL(k_decode_chunks, dim3(grid), dim3(kDsBlock), (size_t)kDsWaves * kDsStageWords * 4u, st, d);
}

int decompress_impl(const DecompWs &ws, const void *dev_in, uint64_t bytes, comet_shape s, void *stream, void *dev_out, int out_type) {
    uint64_t n;
    if (!dev_in || !dev_out || !shape_elems(s, &n) || s.w > kMaxW || ((uintptr_t)dev_in & 15u)) return COMET_ERR_INVALID;
    if (bytes < kHeaderBytes) return COMET_ERR_FORMAT;
    if (n > ws.max_elems) return COMET_ERR_NOMEM;        // the work buffer holds one residual per element of the context's size
    hipStream_t st = (hipStream_t)stream;
    ReconGeometry g;
    if (!recon_geometry(s, &g)) return COMET_ERR_INVALID;
    const uint8_t *in = static_cast<const uint8_t *>(dev_in);
    // scan kernel: two adjacent columns per lane if every pair is aligned in the output; a row then takes
    // lpr lanes, and ppi planes lie side by side in a wavefront
    const uint32_t out_elem = out_type ? 2u : 4u;
    const uint32_t vec = ((s.w & 1u) == 0u && ((uintptr_t)dev_out & (2u * out_elem - 1u)) == 0u) ? 2u : 1u;
    const uint32_t lpr = s.w / vec;
    const uint32_t ppi = lpr <= 16u ? 4u * (16u / lpr) : (lpr <= 32u ? 2u : 1u);
    // (buffer offsets: a strip of whole rows, or the planes side by side in a wavefront, stays below 2^28 elements)
    const bool fast_path = s.w <= kDsMaxW && (uint64_t)ppi * s.h * s.w < (1ull << 28);
    const uint64_t planes = (uint64_t)s.n * s.c;
    const BandGeom bg = band_geometry(planes, s.h, s.w, vec);
    const bool bands = s.w >= kBandMinW && bg.bytes <= ws.band_bytes && bg.n_units < (1ull << 31) &&
                       (!fast_path || band_pays(ws.num_cu, planes, s.h, s.w, bg, ws.chunk_syms == 64u));
    if (out_type != 0 && !fast_path) return COMET_ERR_INVALID;       // 16-bit outputs: planes of at most kDsMaxW columns
    // Chunks of 64 symbols (what the caller's context compresses with tells what to expect) go through the
    // single fused kernel; it leaves a container with another chunk size alone, and the kernels launched
    // behind it, which take any chunk size, leave one with 64 alone.
    const bool fused = fast_path && !bands && ws.chunk_syms == 64u;
    {
        TablesArgs t{};
        t.len = in + kHeaderBytes; t.nbins = 0; t.t = ws.tables; t.ctl = &ws.state->ctl;
        t.hdr = reinterpret_cast<const Header *>(in);
        t.expect.N = s.n; t.expect.C = s.c; t.expect.H = s.h; t.expect.W = s.w; t.bytes = bytes;
        t.compact_only = (fast_path || bands) ? 1u : 0u;
        t.general_unless_chunk64 = (fused && out_type == 0) ? 1u : 0u;   // the kernel behind k_decode_scan reads the general table
        // the only kernel of a decompression that raises status bits: it clears the call's control block itself
        // and latches what it raises, so the call needs neither a fill before nor a kernel after
        t.reset_ctl = 1u; t.latched = &ws.state->latched; t.status_out = ws.dev_status;
        {
            TimedScope ts(ws.prof, st, COMET_KERNEL_TABLES);
            hipLaunchKernelGGL(k_decode_tables, dim3(1), dim3(kBookBlock), 0, st, t);
        }
        HIP_TRY(hipGetLastError());
    }
    if (fused) {
        FuArgs f{};
        f.container = in; f.t = ws.tables; f.n = n; f.planes = s.n * s.c; f.H = s.h; f.W = s.w;
        f.divW = make_fastdiv(s.w); f.divH = make_fastdiv(s.h); f.divL = make_fastdiv(lpr);
        f.divSpr = make_fastdiv(lpr <= 16u ? 16u / lpr : 1u);
        f.divK = make_fastdiv(lpr <= 16u ? 4u * (16u / lpr) : (lpr <= 32u ? 2u : 1u));
        f.out = dev_out; f.ctl = &ws.state->ctl;
        const int mode = lpr <= 16u ? 0 : (lpr <= 32u ? 1 : 2);
        const int nseg = lpr <= 64u ? 1 : (lpr <= 128u ? 2 : (lpr <= 256u ? 4 : 8));
        // planes of at most 128 lanes per row: one segment of planes per workgroup, its strips dealt to all its
        // wavefronts; wider planes: units of whole planes per wavefront
        const bool coop = nseg <= 2;
        FusedGeom fg = fused_geometry(ws.num_cu, s);
        if (coop) {
            fg.grid = (uint32_t)(planes < (uint64_t)ws.num_cu ? planes : (uint64_t)ws.num_cu);
        }
        f.G = fg.G; f.n_units = fg.n_units;
        const void *fn = fused_kernel(nseg, mode, out_type, (int)vec);
        if (!fn) return COMET_ERR_INTERNAL;
        void *kargs[] = {&f};
        TimedScope ts(ws.prof, st, COMET_KERNEL_FUSED);
        HIP_TRY(hipLaunchKernel(fn, dim3(fg.grid), dim3(kFuBlock), kargs, kFuLdsBytes, st));
    }
    if (fused && out_type == 0) {
        // any other chunk size: the general kernel, on a small grid (it is rarely needed)
        ReconArgs a{};
        a.container = in; a.t = ws.tables; a.n = n; a.planes = s.n * s.c; a.H = s.h; a.W = s.w; a.divW = make_fastdiv(s.w);
        a.planes_per_unit = g.planes_per_unit; a.tile_rows = g.tile_rows; a.n_units = g.n_units; a.pitch = g.pitch; a.use_carry = g.use_carry;
        a.out = static_cast<float *>(dev_out); a.ctl = &ws.state->ctl; a.skip_chunk64 = 1u;
        uint32_t grid = g.n_units;
        const uint32_t cap = (uint32_t)ws.num_cu * 4u;
        if (grid > cap) grid = cap;
        hipLaunchKernelGGL(k_reconstruct<0>, dim3(grid), dim3(kDecBlock), g.lds, st, a);
    } else if (bands) {
        DsArgs d{};
        d.container = in; d.t = ws.tables; d.n = n; d.planes = s.n * s.c; d.H = s.h; d.W = s.w;
        d.resid = ws.resid; d.out = dev_out; d.ctl = &ws.state->ctl;
        launch_decode_chunks(ws, d, st);
        HIP_TRY(hipGetLastError());
        BandArgs a{};
        a.container = in; a.planes = s.n * s.c; a.H = s.h; a.W = s.w; a.R = bg.R;
        a.divSegs = make_fastdiv(bg.segs); a.divBands = make_fastdiv(bg.bands); a.n_units = (uint32_t)bg.n_units;
        a.resid = ws.resid;
        a.col_sums = reinterpret_cast<int32_t *>(ws.band); a.row_sums = reinterpret_cast<int32_t *>(ws.band + bg.off_row);
        a.unit_sums = reinterpret_cast<int32_t *>(ws.band + bg.off_unit);
        a.out = dev_out; a.ctl = &ws.state->ctl;
        const dim3 rec_grid((uint32_t)ws.num_cu), grid((uint32_t)((bg.n_units + kBandBlock / kWave - 1u) / (kBandBlock / kWave))), block(kBandBlock);
        TimedScope ts(ws.prof, st, COMET_KERNEL_RECONSTRUCT);
        hipLaunchKernelGGL(k_band_patch, rec_grid, block, 0, st, a);
        if (bg.bands > 1u || bg.segs > 1u) {
            if (vec == 2u) hipLaunchKernelGGL(k_band_sums<2>, grid, block, 0, st, a);
            else hipLaunchKernelGGL(k_band_sums<1>, grid, block, 0, st, a);
        }
#define COMET_LAUNCH_BAND(OUT)                                                              \
        do {                                                                                \
            if (vec == 2u) hipLaunchKernelGGL((k_band_store<2, OUT>), grid, block, 0, st, a); \
            else hipLaunchKernelGGL((k_band_store<1, OUT>), grid, block, 0, st, a);         \
            hipLaunchKernelGGL(k_band_verbatim<OUT>, rec_grid, block, 0, st, a);            \
        } while (0)
        if (out_type == COMET_F16) COMET_LAUNCH_BAND(1);
        else if (out_type == COMET_BF16) COMET_LAUNCH_BAND(2);
        else COMET_LAUNCH_BAND(0);
#undef COMET_LAUNCH_BAND
    } else if (fast_path) {
        // Huffman decode into int16 residuals (the code buffer of the context doubles as
        // the work buffer), then scans and stores
        DsArgs d{};
        d.skip_chunk64 = fused ? 1u : 0u;
        d.container = in; d.t = ws.tables; d.n = n; d.planes = s.n * s.c; d.H = s.h; d.W = s.w; d.divW = make_fastdiv(s.w); d.divL = make_fastdiv(lpr);
        d.resid = ws.resid; d.out = dev_out; d.ctl = &ws.state->ctl;
        launch_decode_chunks(ws, d, st);
        HIP_TRY(hipGetLastError());
        // small planes: a unit of work is a group of whole planes, `passes` times the planes that sit side by
        // side in a wavefront: about kScanStripElems elements, fewer if that leaves the chip short of wavefronts
        const uint64_t P = (uint64_t)s.h * s.w;
        uint64_t G = 1;
        if (lpr <= 32u) {
            uint64_t passes = kScanStripElems / (ppi * P);
            const uint64_t spread = (uint64_t)d.planes / ((uint64_t)ppi * ws.num_cu * 32u);
            if (passes > spread) passes = spread;
            G = ppi * (passes ? passes : 1u);
        }
        d.group_planes = (uint32_t)G;
        const uint64_t units = ((uint64_t)d.planes + G - 1) / G;
        uint64_t grid = (units + kDsWaves - 1) / kDsWaves;
        const uint64_t cap = (uint64_t)ws.num_cu * 8u;
        if (grid > cap) grid = cap;
        const size_t lds = (size_t)kDsWaves * kScanListWords * 4u;
        TimedScope ts(ws.prof, st, COMET_KERNEL_RECONSTRUCT);
        const dim3 g3((uint32_t)grid), b3(kDsBlock);
#define COMET_LAUNCH_SCAN(OUT)                                                                           \
        do {                                                                                             \
            if (vec == 2u) {                                                                             \
                if (lpr <= 16u) hipLaunchKernelGGL((k_scan_store<1, 0, OUT, 2>), g3, b3, lds, st, d);    \
                else if (lpr <= 32u) hipLaunchKernelGGL((k_scan_store<1, 1, OUT, 2>), g3, b3, lds, st, d); \
                else if (lpr <= 64u) hipLaunchKernelGGL((k_scan_store<1, 2, OUT, 2>), g3, b3, lds, st, d); \
                else if (lpr <= 128u) hipLaunchKernelGGL((k_scan_store<2, 2, OUT, 2>), g3, b3, lds, st, d); \
                else hipLaunchKernelGGL((k_scan_store<4, 2, OUT, 2>), g3, b3, lds, st, d);               \
            } else {                                                                                     \
                if (lpr <= 16u) hipLaunchKernelGGL((k_scan_store<1, 0, OUT, 1>), g3, b3, lds, st, d);    \
                else if (lpr <= 32u) hipLaunchKernelGGL((k_scan_store<1, 1, OUT, 1>), g3, b3, lds, st, d); \
                else if (lpr <= 64u) hipLaunchKernelGGL((k_scan_store<1, 2, OUT, 1>), g3, b3, lds, st, d); \
                else if (lpr <= 128u) hipLaunchKernelGGL((k_scan_store<2, 2, OUT, 1>), g3, b3, lds, st, d); \
                else if (lpr <= 256u) hipLaunchKernelGGL((k_scan_store<4, 2, OUT, 1>), g3, b3, lds, st, d); \
                else hipLaunchKernelGGL((k_scan_store<8, 2, OUT, 1>), g3, b3, lds, st, d);               \
            }                                                                                            \
        } while (0)
        if (out_type == COMET_F16) COMET_LAUNCH_SCAN(1);
        else if (out_type == COMET_BF16) COMET_LAUNCH_SCAN(2);
        else COMET_LAUNCH_SCAN(0);
#undef COMET_LAUNCH_SCAN
    } else {
        ReconArgs a{};
        a.container = in; a.t = ws.tables; a.n = n; a.planes = s.n * s.c; a.H = s.h; a.W = s.w; a.divW = make_fastdiv(s.w);
        a.planes_per_unit = g.planes_per_unit; a.tile_rows = g.tile_rows; a.n_units = g.n_units; a.pitch = g.pitch; a.use_carry = g.use_carry;
        a.out = static_cast<float *>(dev_out); a.ctl = &ws.state->ctl;
        uint32_t grid = g.n_units;
        const uint32_t cap = (uint32_t)ws.num_cu * 32u;
        if (grid > cap) grid = cap;
        TimedScope ts(ws.prof, st, COMET_KERNEL_RECONSTRUCT);
        hipLaunchKernelGGL(k_reconstruct<0>, dim3(grid), dim3(kDecBlock), g.lds, st, a);
    }
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}
}  // namespace

// ---------------------------------------------------------------------------
// decompression without a context, for callers that cannot allocate
// ---------------------------------------------------------------------------
namespace {
constexpr uint64_t kStaticMaxElems = COMET_STATIC_MAX_ELEMS;
// layout of the static scratch array: control block | decode tables | residual work buffer
constexpr size_t kSsState = 0;
constexpr size_t kSsLimit = 512;
constexpr size_t kSsFirst = kSsLimit + 8 * 72;
constexpr size_t kSsFindex = kSsFirst + 8 * 72;
constexpr size_t kSsMeta = kSsFindex + 4 * 72 + 32;          // 16-byte aligned
constexpr size_t kSsLut = kSsMeta + 64;
constexpr size_t kSsLut16 = kSsLut + 4 * kLutSize;
constexpr size_t kSsSub16 = kSsLut16 + 2 * kLut16Size;
constexpr size_t kSsSorted = kSsSub16 + 2 * kSubEntries;
constexpr size_t kSsSymResid = kSsSorted + 2 * (size_t)kMaxBins;
constexpr size_t kSsResid = (kSsSymResid + 2 * (size_t)kMaxBins + 255) / 256 * 256;
constexpr size_t kSsBand = (kSsResid + 2 * (size_t)kStaticMaxElems + 256 + 255) / 256 * 256;
constexpr size_t kSsBytes = kSsBand + (size_t)band_bytes_max(kStaticMaxElems);
static_assert(sizeof(DevState) <= kSsLimit && kSsMeta % 16 == 0 && kSsLut % 16 == 0, "scratch layout");
constexpr int kStaticMaxDevices = 64;
struct StaticDev { void *ptr; int num_cu; };
StaticDev g_static_dev[kStaticMaxDevices];       // filled once per device, under the lock
bool g_static_ready[kStaticMaxDevices];
std::mutex g_static_lock;
}  // namespace

// Device memory of comet_decompress_static: every GPU the library runs on holds its own copy until
// the process ends.  In host code this name is a stand-in, not a device address; the address comes
// from hipGetSymbolAddress (static_scratch below).
static __device__ __align__(256) unsigned char scratch[kSsBytes];

namespace {
// The current device's copy of `scratch` (looked up once per device, with that device current).
int static_scratch(StaticDev *out) {
    int dev = 0;
    HIP_TRY(hipGetDevice(&dev));
    if (dev < 0 || dev >= kStaticMaxDevices) return COMET_ERR_INVALID;
    std::lock_guard<std::mutex> guard(g_static_lock);
    if (!g_static_ready[dev]) {
        void *ptr = nullptr;
        HIP_TRY(hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)));
        if (!ptr) return COMET_ERR_HIP;
        int cus = 0;
        HIP_TRY(hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev));
        // the general kernel (other chunk sizes behind k_decode_scan) may need more than 64 KB of dynamic LDS
        HIP_TRY(hipFuncSetAttribute((const void *)k_reconstruct<0>, hipFuncAttributeMaxDynamicSharedMemorySize, 96 * 1024));
        {
            const int rc = fused_opt_in();
            if (rc) return rc;
        }
        g_static_dev[dev].ptr = ptr;
        g_static_dev[dev].num_cu = cus > 0 ? cus : 256;
        g_static_ready[dev] = true;
    }
    *out = g_static_dev[dev];
    return COMET_OK;
}
}  // namespace

int comet_decompress_static(const void *dev_in, uint64_t bytes, comet_shape s, void *stream, float *dev_out, int32_t *dev_status) {
    uint64_t n;
    if (!shape_elems(s, &n)) return COMET_ERR_INVALID;
    if (n > kStaticMaxElems) return COMET_ERR_NOMEM;         // the static work buffer holds COMET_STATIC_MAX_ELEMS residuals
    StaticDev sd{};
    const int rc = static_scratch(&sd);
    if (rc) return rc;
    uint8_t *base = static_cast<uint8_t *>(sd.ptr);
    DecompWs ws{};
    ws.state = reinterpret_cast<DevState *>(base + kSsState);
    ws.tables.limit = reinterpret_cast<uint64_t *>(base + kSsLimit);
    ws.tables.first_code = reinterpret_cast<uint64_t *>(base + kSsFirst);
    ws.tables.first_index = reinterpret_cast<uint32_t *>(base + kSsFindex);
    ws.tables.meta = reinterpret_cast<uint32_t *>(base + kSsMeta);
    ws.tables.lut = reinterpret_cast<uint32_t *>(base + kSsLut);
    ws.tables.lut16 = reinterpret_cast<uint16_t *>(base + kSsLut16);
    ws.tables.sub16 = reinterpret_cast<uint16_t *>(base + kSsSub16);
    ws.tables.sorted = reinterpret_cast<uint16_t *>(base + kSsSorted);
    ws.tables.resid = reinterpret_cast<uint16_t *>(base + kSsSymResid);
    ws.resid = reinterpret_cast<int16_t *>(base + kSsResid);
    ws.band = base + kSsBand; ws.band_bytes = kSsBytes - kSsBand;
    ws.max_elems = kStaticMaxElems; ws.num_cu = sd.num_cu; ws.chunk_syms = COMET_DEFAULT_CHUNK_SYMS;
    ws.prof = nullptr; ws.dev_status = dev_status;
    // Nothing in the array has to start at zero: the tables kernel clears the control block and stores
    // the status, every table entry and residual that is read has been written by this call.
    return decompress_impl(ws, dev_in, bytes, s, stream, dev_out, 0);
}

int comet_sync(comet_ctx *ctx, void *stream) {
    if (!ctx) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipMemcpyAsync(ctx->host_state, ctx->state, sizeof(DevState), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    const uint32_t latched = ctx->host_state->latched;
    if (latched) {
        HIP_TRY(hipMemsetAsync(&ctx->state->latched, 0, 4, st));
        HIP_TRY(hipStreamSynchronize(st));
    }
    return status_to_error(latched);
}

int comet_peek(comet_ctx *ctx, const void *dev_in, uint64_t bytes, void *stream, comet_info *info) {
    if (!ctx || !dev_in || !info) return COMET_ERR_INVALID;
    if (bytes < kHeaderBytes) return COMET_ERR_FORMAT;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipMemcpyAsync(ctx->host_hdr, dev_in, sizeof(Header), hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    const Header &h = *ctx->host_hdr;
    comet_shape s{h.N, h.C, h.H, h.W};
    uint64_t n;
    if (h.magic != kMagic || (h.version != 1 && h.version != 2) || h.status != 0 || !shape_elems(s, &n) || !valid_nbins(h.nbins) ||
        h.chunk_syms == 0 || h.total_bytes > bytes || h.total_bytes != h.off_payload + 4 * h.payload_words) return COMET_ERR_FORMAT;
    info->shape = s; info->nbins = h.nbins; info->chunk_syms = h.chunk_syms; info->n_chunks = h.n_chunks;
    info->n_active = h.n_active; info->max_len = h.max_len; info->n_outlier_records = h.n_rec; info->n_value_records = h.n_vrec;
    memcpy(&info->eb, &h.eb_bits, 4);
    info->nnz = h.nnz; info->payload_words = h.payload_words; info->total_bytes = h.total_bytes;
    return COMET_OK;
}

void comet_adapt_defaults(comet_adapt_cfg *cfg) {
    if (!cfg) return;
    cfg->a = 0.32; cfg->sigma_frac = 0.01; cfg->eb_min = 0x1p-100f; cfg->eb_max = 0x1p100f;
}

int comet_adapt_eb(const comet_layer_stats *s, const comet_adapt_cfg *cfg_in, float *eb_out) {
    if (!s || !eb_out) return COMET_ERR_INVALID;
    comet_adapt_cfg cfg;
    if (cfg_in) cfg = *cfg_in; else comet_adapt_defaults(&cfg);
    if (!std::isfinite(s->momentum_abs_mean) || !std::isfinite(s->loss_grad_mean) || !std::isfinite(s->nonzero_ratio) ||
        !std::isfinite(cfg.a) || !std::isfinite(cfg.sigma_frac)) return COMET_ERR_INVALID;
    if (s->momentum_abs_mean < 0.0 || s->loss_grad_mean < 0.0 || s->nonzero_ratio < 0.0 || s->nonzero_ratio > 1.0 ||
        s->batch == 0 || !(cfg.a > 0.0) || !(cfg.sigma_frac > 0.0) || !(cfg.eb_min > 0.0f) || !(cfg.eb_max >= cfg.eb_min)) return COMET_ERR_INVALID;
    if (s->loss_grad_mean == 0.0 || s->nonzero_ratio == 0.0) { *eb_out = cfg.eb_max; return COMET_OK; }
    const double sigma = cfg.sigma_frac * s->momentum_abs_mean;                                 // Sec. 3.2
    const double eb = sigma / (cfg.a * s->loss_grad_mean * std::sqrt((double)s->batch * s->nonzero_ratio));   // Sec. 3.3
    float e = (float)eb;
    if (!(e >= cfg.eb_min)) e = cfg.eb_min;
    if (e > cfg.eb_max) e = cfg.eb_max;
    *eb_out = e;
    return COMET_OK;
}

// ---------------------------------------------------------------------------
// controller glue (Sec. 3.1)
// ---------------------------------------------------------------------------

int comet_abs_mean(comet_ctx *ctx, const float *dev_in, uint64_t n, void *stream, double *mean_out) {
    if (!ctx || !dev_in || !mean_out || n == 0) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    // a slice of at least 16384 values per workgroup, a few workgroups per CU at most
    uint64_t grid = (n + 16383u) / 16384u;
    const uint64_t cap = (uint64_t)ctx->num_cu * 8u < kStatsPartialMax ? (uint64_t)ctx->num_cu * 8u : kStatsPartialMax;
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL(k_abs_sum, dim3((uint32_t)grid), dim3(kStatsBlock), 0, st, dev_in, n, ctx->stats);
    hipLaunchKernelGGL(k_abs_mean_final, dim3(1), dim3(kWave), 0, st, ctx->stats, (uint32_t)grid, n, ctx->stats + kStatsPartialMax);
    HIP_TRY(hipGetLastError());
    HIP_TRY(hipMemcpyAsync(mean_out, ctx->stats + kStatsPartialMax, 8, hipMemcpyDeviceToHost, st));
    HIP_TRY(hipStreamSynchronize(st));
    return COMET_OK;
}

int comet_controller_init(comet_controller *c, uint32_t w_default) {
    if (!c) return COMET_ERR_INVALID;
    c->w_default = w_default ? w_default : 1000u;
    c->w = c->w_default;
    c->since = 0;
    return COMET_OK;
}

int comet_controller_tick(comet_controller *c, int *collect) {
    if (!c || !collect || c->w == 0) return COMET_ERR_INVALID;
    *collect = 0;
    if (++c->since >= c->w) { c->since = 0; *collect = 1; }
    return COMET_OK;
}

int comet_controller_update(comet_controller *c, const float *eb_old, const float *eb_new, uint32_t n_layers) {
    if (!c || !eb_old || !eb_new || n_layers == 0 || c->w == 0) return COMET_ERR_INVALID;
    bool moved = false;                                   // some layer's bound changed by more than 2x, up or down
    for (uint32_t l = 0; l < n_layers; ++l) {
        const double a = (double)eb_old[l], b = (double)eb_new[l];
        if (!(a > 0.0) || !(b > 0.0) || !std::isfinite(a) || !std::isfinite(b)) return COMET_ERR_INVALID;
        if (a > 2.0 * b || b > 2.0 * a) moved = true;
    }
    if (moved) c->w = c->w > 1u ? c->w / 2u : 1u;
    else c->w = c->w_default;
    return COMET_OK;
}

// ---------------------------------------------------------------------------
// stage-level entry points
// ---------------------------------------------------------------------------

int comet_stage_quantize(comet_ctx *ctx, const float *dev_in, comet_shape s, float eb, uint32_t nbins, void *stream,
                         uint16_t *dev_codes, uint32_t *dev_hist, uint32_t *dev_records, uint64_t rec_capacity,
                         uint64_t *dev_counts) {
    uint64_t n;
    if (!ctx || !dev_in || !dev_codes || !dev_hist || !dev_counts || (rec_capacity && !dev_records) ||
        !shape_elems(s, &n) || !valid_eb(eb) || !valid_nbins(nbins) || s.w > kMaxW || ((uintptr_t)dev_in & 15u) ||
        ((uintptr_t)dev_codes & 7u) || ((uintptr_t)dev_records & 7u)) return COMET_ERR_INVALID;
    if (n > ctx->max_elems) return COMET_ERR_NOMEM;
    hipStream_t st = (hipStream_t)stream;
    const ZeroLayout z = zero_layout(0, 1);
    if (z.bytes > ctx->zero_cap) return COMET_ERR_NOMEM;
    HIP_TRY(hipMemsetAsync(ctx->zero_region, 0, z.bytes, st));
    HIP_TRY(hipMemsetAsync(dev_hist, 0, 4ull * nbins, st));
    RecordArgs recs{};
    int rc;
    if ((rc = clean_parts(ctx, st))) return rc;
    rc = launch_quantize(ctx, dev_in, s, n, eb, nbins, st, dev_codes, ctx->hist_parts, dev_records, rec_capacity, &recs, false);
    if (rc) return rc;
    if ((rc = launch_gather(ctx, recs, st, dev_hist, ctx->hist_parts))) return rc;
    if ((rc = clean_parts(ctx, st))) return rc;              // (at once, not in the next call: that one may have been captured in a graph already)
    ctx->parts_clean = true;
    HIP_TRY(hipMemcpyAsync(dev_counts, &ctx->state->ctl.n_rec, 24, hipMemcpyDeviceToDevice, st));
    hipLaunchKernelGGL(k_latch, dim3(1), dim3(1), 0, st, ctx->state);
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int comet_stage_codebook(comet_ctx *ctx, const uint32_t *dev_hist, uint32_t nbins, void *stream, uint8_t *dev_len, uint64_t *dev_code) {
    if (!ctx || !dev_hist || !dev_len || nbins == 0 || nbins > kMaxBins) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipMemsetAsync(ctx->zero_region, 0, sizeof(Control), st));
    BookArgs b{};
    b.hist = dev_hist; b.nbins = nbins; b.len_out = dev_len; b.code_out = dev_code; b.enc = ctx->enc;
    b.scratch = ctx->book; b.ctl = &ctx->state->ctl; b.hdr = nullptr; b.capacity = 0;
    const int rc = launch_codebook(ctx, b, st);
    if (rc) return rc;
    hipLaunchKernelGGL(k_latch, dim3(1), dim3(1), 0, st, ctx->state);
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int comet_stage_encode(comet_ctx *ctx, const uint16_t *dev_codes, uint64_t n, uint32_t nbins, uint32_t chunk_syms, void *stream,
                       uint32_t *dev_chunk_off, uint32_t *dev_payload, uint64_t payload_capacity_words, uint64_t *dev_payload_words) {
    if (!ctx || !dev_codes || !dev_chunk_off || !dev_payload_words || (payload_capacity_words && !dev_payload) ||
        n == 0 || n > kMaxElems || nbins == 0 || nbins > kMaxBins || !valid_chunk(chunk_syms) || ((uintptr_t)dev_codes & 15u)) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    const uint64_t n_chunks = (n + chunk_syms - 1) / chunk_syms;
    uint32_t e_seg, e_grid;
    encode_geometry(ctx, n_chunks, nbins, &e_seg, &e_grid);
    const uint64_t tiles_e = e_grid;
    const ZeroLayout z = zero_layout(0, tiles_e);
    if (z.bytes > ctx->zero_cap) return COMET_ERR_NOMEM;
    HIP_TRY(hipMemsetAsync(ctx->zero_region, 0, z.bytes, st));
    uint64_t *desc_e = reinterpret_cast<uint64_t *>(ctx->zero_region + z.off_desc_e);
    int rc = launch_encode(ctx, dev_codes, n, nbins, chunk_syms, st, dev_chunk_off, nullptr, 0, dev_payload, payload_capacity_words,
                           dev_payload_words, desc_e);
    if (rc) return rc;
    hipLaunchKernelGGL(k_latch, dim3(1), dim3(1), 0, st, ctx->state);
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int comet_stage_decode(comet_ctx *ctx, const uint8_t *dev_len, uint32_t nbins, const uint32_t *dev_chunk_off, const uint32_t *dev_payload,
                       uint64_t payload_words, uint64_t n, uint32_t chunk_syms, void *stream, uint16_t *dev_codes_out) {
    if (!ctx || !dev_len || !dev_chunk_off || !dev_codes_out || (payload_words && !dev_payload) || n == 0 || n > kMaxElems ||
        nbins == 0 || nbins > kMaxBins || chunk_syms == 0) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    HIP_TRY(hipMemsetAsync(ctx->zero_region, 0, sizeof(Control), st));
    TablesArgs t{};
    t.len = dev_len; t.nbins = nbins; t.t = ctx->tables; t.ctl = &ctx->state->ctl; t.hdr = nullptr;
    hipLaunchKernelGGL(k_decode_tables, dim3(1), dim3(kBookBlock), 0, st, t);
    HIP_TRY(hipGetLastError());
    ReconArgs a{};
    a.chunk_off = dev_chunk_off; a.payload = dev_payload; a.payload_words = payload_words; a.chunk_syms = chunk_syms;
    a.n_chunks = (uint32_t)((n + chunk_syms - 1) / chunk_syms); a.t = ctx->tables; a.n = n; a.codes_out = dev_codes_out; a.ctl = &ctx->state->ctl;
    a.zero_chunks = ctx->zero_chunks;
    uint32_t grid = (a.n_chunks + kDecBlock - 1) / kDecBlock;
    const uint32_t cap = (uint32_t)ctx->num_cu * 32u;
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL(k_decode_only, dim3(grid), dim3(kDecBlock), 0, st, a);
    HIP_TRY(hipGetLastError());
    hipLaunchKernelGGL(k_latch, dim3(1), dim3(1), 0, st, ctx->state);
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int comet_stage_reconstruct(comet_ctx *ctx, const uint16_t *dev_codes, const uint32_t *dev_records, uint64_t n_records, comet_shape s,
                            uint32_t nbins, float eb, void *stream, float *dev_out) {
    uint64_t n;
    if (!ctx || !dev_codes || !dev_out || (n_records && !dev_records) || !shape_elems(s, &n) || !valid_nbins(nbins) || !valid_eb(eb) ||
        s.w > kMaxW) return COMET_ERR_INVALID;
    hipStream_t st = (hipStream_t)stream;
    ReconGeometry g;
    if (!recon_geometry(s, &g)) return COMET_ERR_INVALID;
    ReconArgs a{};
    a.codes_in = dev_codes; a.rec = dev_records; a.n_rec = n_records; a.n = n; a.planes = s.n * s.c; a.H = s.h; a.W = s.w;
    a.divW = make_fastdiv(s.w); a.radius = (int32_t)(nbins / 2u); a.eb = eb; a.ebx2 = 2.0f * eb;
    a.planes_per_unit = g.planes_per_unit; a.tile_rows = g.tile_rows; a.n_units = g.n_units; a.pitch = g.pitch; a.use_carry = g.use_carry;
    a.out = dev_out; a.ctl = &ctx->state->ctl; a.chunk_syms = 1;
    uint32_t grid = g.n_units;
    const uint32_t cap = (uint32_t)ctx->num_cu * 32u;
    if (grid > cap) grid = cap;
    hipLaunchKernelGGL(k_reconstruct<1>, dim3(grid), dim3(kDecBlock), g.lds, st, a);
    HIP_TRY(hipGetLastError());
    return COMET_OK;
}

int comet_profile_enable(comet_ctx *ctx, int enable) {
    if (!ctx) return COMET_ERR_INVALID;
    if (enable && ctx->pool.empty()) {
        ctx->pool.reserve(16384);
        for (int i = 0; i < 16384; ++i) {
            comet_ctx::Timed t{};
            HIP_TRY(hipEventCreate(&t.a));
            HIP_TRY(hipEventCreate(&t.b));
            ctx->pool.push_back(t);
        }
    }
    ctx->profiling = enable != 0;
    return COMET_OK;
}

int comet_profile_reset(comet_ctx *ctx) {
    if (!ctx) return COMET_ERR_INVALID;
    ctx->used = 0;
    return COMET_OK;
}

int comet_profile_read(comet_ctx *ctx, uint32_t kernel_id, uint32_t *launches, double *total_ms) {
    if (!ctx || !launches || !total_ms || kernel_id >= COMET_KERNEL_COUNT) return COMET_ERR_INVALID;
    uint32_t cnt = 0;
    double sum = 0.0;
    for (size_t i = 0; i < ctx->used; ++i) {
        const comet_ctx::Timed &t = ctx->pool[i];
        if (t.id != kernel_id) continue;
        HIP_TRY(hipEventSynchronize(t.b));
        float ms = 0.0f;
        HIP_TRY(hipEventElapsedTime(&ms, t.a, t.b));
        sum += ms;
        ++cnt;
    }
    *launches = cnt;
    *total_ms = sum;
    return COMET_OK;
}

const char *comet_strerror(int code) {
    switch (code) {
        case COMET_OK: return "ok";
        case COMET_ERR_INVALID: return "invalid argument";
        case COMET_ERR_CAPACITY: return "container does not fit the output buffer";
        case COMET_ERR_FORMAT: return "malformed container or shape mismatch";
        case COMET_ERR_HIP: return g_hip_msg;
        case COMET_ERR_NOMEM: return "out of memory, or request larger than the context was created for";
        case COMET_ERR_INTERNAL: return "device-side consistency check failed";
        case COMET_ERR_CODEBOOK: return "the given code lengths are no complete prefix code, or lack a code word for an escape the tensor needs";
        default: return "unknown error code";
    }
}

}  // extern "C"
