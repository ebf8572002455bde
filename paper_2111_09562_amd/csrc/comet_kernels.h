// Kernel argument blocks and launch constants shared by the host API and the
// kernel translation units.
#pragma once
#include "comet_bands.h"
#include "comet_dev.h"

namespace comet {

// ---- quantise (prequantise + Lorenzo + codes + histogram + records) ----------
constexpr int kQuantBlock = 256;
constexpr uint32_t kQuantWaves = (uint32_t)(kQuantBlock / kWave);   // runs per workgroup of the row-walking kernel
constexpr uint32_t kHistWindowMax = 8192;  // LDS-private histogram bins per workgroup

struct QuantArgs {
    const void *x;             // fp32; the row-walking kernels also take IEEE half or bfloat16 (template parameter IN)
    uint64_t n;
    FastDiv divW, divH;        // plane width / height
    float r, ebx2, eb;
    int32_t radius;
    uint32_t nbins;
    uint32_t win_lo, win_n;    // histogram bins [win_lo, win_lo + win_n) are counted in LDS
    uint32_t rows_total;       // planes * H rows of W elements
    uint32_t rows_per_wave;    //   consecutive rows per wavefront (a multiple of rows_per_step)
    uint32_t rows_per_wg;      //   rows per workgroup: kQuantWaves * rows_per_wave, or fewer (kReuseRunElems)
    uint32_t run_elems;        //   elements per run: rows_per_wave * W, or, for planes wider than kQuantRowsMaxW, what their runs hold
    uint32_t rows_per_step;    //   rows a wavefront covers per step (64 / lanes per row if a row takes at most 32 lanes, else 1)
    uint32_t hist_shift;       //   log2 of the copies of the LDS histogram window (lane & (copies - 1) picks one)
    uint32_t *stage;           //   staging area: rec_run (key, payload) pairs per run
    uint32_t rec_run;
    uint32_t *run_count;       //   records per run; then per workgroup: records, non-zero inputs, verbatim records
    const uint8_t *reuse_len;  //   code book reuse (REUSE kernels): u8[nbins] code lengths; a code of length 0 becomes an escape; no histogram
    uint32_t *hist_parts;      //   hist_copies partial histograms of nbins entries, zero: workgroup b adds to copy b % hist_copies
    uint32_t hist_copies;      //   (the code book kernels add them up)
    uint32_t reset_ctl;        //   1: this kernel is the first of its call and clears *ctl itself
    // single-pass compression (REUSE kernels): the codes are encoded by the wavefront that makes them
    const uint64_t *enc;       //   encode table of the given lengths: (code << 6) | length per symbol
    uint32_t enc_lo, enc_n;    //   table entries [enc_lo, enc_lo + enc_n) are cached in LDS
    uint32_t chunk_syms;       //   64, 128 or 256; a run is a whole number of chunks
    uint32_t zero_pair;        //   container version 2: (centre << 16) | centre, else 0
    uint32_t *chunk_off;       //   chunk table of the container: offsets relative to the run (k_place_payload makes them absolute)
    uint32_t *run_words;       //   words of every run
    uint32_t *run_from;        // kHistPart: element of every run from which on k_code_hist counts its codes
    uint32_t *work_words;      //   work area: the words of the run that starts at element e at word e / 64 * words64
    uint32_t words64;          //   kWordsRun or kWordsWide
    uint16_t *codes;
    Control *ctl;
};

constexpr uint32_t kQuantRowsMaxW = 512;  // widest plane whose rows a wavefront holds in registers; wider ones are walked in segments (NSEG == 0)

// What the kernels behind the row-walking quantise kernel need to bring its outlier records into element order.
struct RecordArgs {
    const void *x;             // the input (for runs with more records than their staging area holds)
    uint32_t in_type;          // 0 fp32, 1 IEEE half, 2 bfloat16
    FastDiv divW, divH;
    float r, ebx2, eb;
    int32_t radius;
    uint32_t nbins;
    const uint8_t *reuse_len;  // code book reuse: the given lengths, or null
    uint64_t n;
    uint32_t run_elems, wg_elems;  // elements per run and per workgroup of the quantise kernel
    uint32_t n_wg;             // workgroups of the quantise kernel (kQuantWaves runs each); 0: there are no records to place
    const uint32_t *stage;     // rec_run (key, payload) pairs per run
    uint32_t rec_run;
    const uint32_t *run_count; // as in QuantArgs
    uint32_t *rec;             // (key, payload) pairs of the container, in element order
    uint64_t rec_cap;          // room for so many
    uint32_t ring;             // record_ring(W)
    Control *ctl;
};
// Records that leave a run's staging area out are derived from the input once more (comet_records.h), with a buffer of kDeriveBuf records and
// a ring of differences per wavefront: a power of two that holds a row and a step of 256 elements, or none.
constexpr uint32_t kDeriveBuf = 256;
inline uint32_t record_ring(uint32_t w) { return w < 4u || w > kQuantRowsMaxW ? 0u : (w <= 256u ? 512u : 1024u); }
__host__ __device__ inline uint32_t record_lds(uint32_t ring) { return kDeriveBuf * 8u + ring * 4u; }    // bytes per wavefront
constexpr int kGatherBlock = 256;
// hist: if not null, the sum of the `copies` partial histograms of nbins entries in `parts` goes there
__global__ void k_gather_records(RecordArgs a, uint32_t *hist, const uint32_t *parts, uint32_t copies);
constexpr uint32_t kEncRingSyms = 1024;    // single-pass compression: codes a wavefront keeps in LDS between quantisation and encoding (a batch of at most 512, and less than 256 not yet encoded)
constexpr uint32_t kEncRunBufWords = 476;  //   its assembly buffer: the words of one step of 256 symbols (at most 456 of code words of 57 bits, two more touched) and slack
// Compression with a given code book: what the words of a run of kReuseRunElems elements or more may take, 16 bits per symbol of
// the whole run (more expands the data and is refused).  While such runs leave SIMDs without work (fewer elements than kReuseRunElems
// per SIMD), a workgroup of four wavefronts takes one of them instead of four: its runs are a quarter as long, the words
// of each may be of any length (kWordsWide), and the limit holds for the four of them together, so the length of a
// run decides nothing about what is refused.
// A call with a wavefront per run of 2048 elements / with four: 64 x 28 x 28 31.4 / 24.6 us, 4 x 64 x 56 x 56 32.2 / 27.1,
// 10 x 64 x 56 x 56 (2.0 M elements) 34.0 / 31.8; beyond the line 12 x 64 x 56 x 56 34.6 / 38.6.
constexpr uint32_t kReuseRunElems = 2048;
constexpr uint32_t kWordsRun = 32, kWordsWide = 114;     // work words per 64 symbols: 16 bits per symbol, the longest code words (57 bits)
// Outlier records staged per run (one run of rows per wavefront): kQuantRecRun of them while there are as many runs as there can
// be, 31 MB of a context, more in fewer runs.  What a run has beyond that is derived from the input once more (comet_records.h).
// 64 x 256 x 56 x 56, where a run's share is 7.6 % of its elements, 8 / 21 / 41 % records: 166 / 226 / 261 us; with room for 25 % of the elements
// (103 MB) 162 / 205 / 326 (a slower derivation then).  411 M elements, a share of 1 %, 4 / 8 / 21 / 41 %: 1448 / 1566 / 1716 / 1866 us; with 822 MB
// 1206 / 1310 / 1684 / 2516.  A container with 21 % records is hardly smaller than the tensor (8 bytes per record alone).
constexpr uint32_t kQuantRecRun = 768;
constexpr uint32_t kQuantRecLds2 = 256;   // records a wavefront buffers in LDS before it writes them to the staging area in bulk
constexpr uint32_t kQuantRunsPerSimd = 5; // runs the launch aims at, per SIMD
constexpr uint32_t kQuantRunMin = 512;    // elements of the shortest run (whole rows, so a little more), while SIMDs have none
// Alphabets larger than the histogram window: a wavefront counts its run's codes while those outside the window, which it
// lists in LDS (kQuantOowList of them) and adds to a partial histogram in bulk, are at most kQuantOowFree plus one in
// kQuantOowShare; beyond, k_code_hist counts them from memory (why the line lies there: see that kernel) ...
constexpr uint32_t kQuantOowList = 512, kQuantOowFree = 32, kQuantOowShare = 32;
// ... and only for tensors of at least so many elements.  Smaller ones leave all codes to k_code_hist: beginning to count costs
// 10 to 30 us where a run then stops (LDS for three workgroups per compute unit instead of five, bins to add up), which
// fine bounds do.  Measured, all codes in k_code_hist / counted here, us: 12.8 M elements at 1e-4, 65536 bins 349 / 377, at 1e-2, 16384 bins
// 114 / 109; 51.4 M 507 / 521, 222 / 201; 67.4 M 552 / 557, 266 / 228; 205 M 1237 / 1231, 684 / 569.
constexpr uint64_t kQuantCountMin = 1ull << 26;
constexpr uint32_t kQuantStaticLds = 8448; // static LDS of k_quantize_rows (the record buffers of its four wavefronts and a few words), rounded up
constexpr uint32_t kLdsPerCu = 160u * 1024u;
constexpr uint32_t kQuantRunsPerSimdSingle = 4;   //   ... of the single-pass compression (all of them resident at once)
// Partial histograms the workgroups spread their flushes over: the occupied bins are a few cache lines, and a thousand
// workgroups adding to one copy of them queue up for 10 to 20 us.  Up to kBookPartsMax bins the one workgroup of the code book
// kernel adds them up itself: 8 copies (32 of them: 64 x 64 x 112 x 112, 1024 bins 153.0 us instead of 151.5).  Above, many
// workgroups do, of k_gather_records or k_book_sort_tiles (the code book kernel's one: 64 x 256 x 56 x 56, 8192 bins 161.3 us -> 164.7):
// up to 32 copies and 2 MB (eight of the largest alphabet).
constexpr uint32_t kQuantHistCopiesMax = 32, kQuantHistCopiesBook = 8;
constexpr uint32_t kBookPartsMax = 2048;   // (no alphabet of the code book kernel's that has more symbols than fit its LDS)
constexpr uint32_t kQuantHistPartsWords = 8u * 65536u;
// VEC adjacent columns per lane (2 needs an even W and 8-byte aligned input), NSEG segments of 64 lanes per row,
// MULTI: several rows per step; HIST: which codes are counted here: all (every bin is in the LDS window), those of a run as
// long as few of them lie outside the window, or none (k_code_hist counts the others)
// REUSE: code book reuse: escapes follow the given length table, no histogram (kHistFull then says that the whole encode table is in LDS, kHistNone that part of it is)
// IN: element type of x (0 fp32, 1 IEEE half, 2 bfloat16; 16-bit inputs are widened exactly as they are loaded;
// VEC = 2 then needs 4-byte aligned input)
constexpr int kHistNone = 0, kHistFull = 1, kHistPart = 2;
template <int VEC, int NSEG, bool MULTI, int HIST, bool REUSE = false, int IN = 0> __global__ void k_quantize_rows(QuantArgs a);
constexpr uint32_t kQuantReuseMaxBins = 8192;   // largest alphabet whose length table the REUSE kernels keep in LDS

// ---- histogram of the codes of a large alphabet ----------------------------------
constexpr int kCodeHistBlock = 1024;
constexpr uint32_t kCodeHistWindow = 32768;   // bins counted in LDS at most (128 KB: one workgroup per compute unit)
constexpr uint32_t kCodeHistHot = 1024;       // innermost bins with four counters each
constexpr uint32_t kCodeHistRuns = 64;        // runs of the quantise kernel that reach into a workgroup's slice, at most
struct CodeHistArgs {
    const uint16_t *codes;     // 8-byte aligned (its 16-byte loads need four)
    uint64_t n;
    uint32_t nbins, radius;
    uint32_t win_lo, win_n;    // bins counted in LDS
    const uint32_t *run_from;  // SHARED: per run, element of the run from which on its codes are counted here
    FastDiv divRun;            // SHARED: elements per run
    uint32_t *parts;           // `copies` partial histograms of nbins entries
    uint32_t copies;
};
template <bool SHARED> __global__ void k_code_hist(CodeHistArgs a);   // SHARED: the quantise kernel has counted part of them (kHistPart); else all codes

// ---- statistics ---------------------------------------------------------------
constexpr int kStatsBlock = 256;
constexpr uint32_t kStatsPartialMax = 4096;     // workgroups of k_abs_sum at most (one partial sum each)
__global__ void k_abs_sum(const float *x, uint64_t n, double *partial);
__global__ void k_abs_mean_final(const double *partial, uint32_t n_partial, uint64_t n, double *mean_out);

// ---- codebook -----------------------------------------------------------------
constexpr int kBookBlock = 1024;
constexpr uint32_t kBookLdsSyms = 2048;    // alphabets up to this size are built entirely in LDS
constexpr uint32_t kBookBySymbolMax = 8192; // nbins up to which the code lengths also fit LDS by symbol (one byte each)

struct BookScratch {                        // global scratch for large alphabets (>= 65536 entries each)
    uint64_t *keys;        // sort keys
    uint64_t *iw;          // internal-node weights
    uint32_t *leaf_parent;
    uint32_t *int_parent;
    uint32_t *tile_cnt;    // [tile of kBookBlock symbols][kBookLens]: symbols per length (alphabets above kBookBySymbolMax)
};
constexpr uint32_t kBookLens = 65u;        // lengths 0 .. 64 (64 stands for every length the container cannot hold)

struct BookArgs {
    const uint32_t *hist;
    const uint32_t *hist_parts;  // up to kBookPartsMax bins: kQuantHistCopiesBook partial histograms instead of hist; above kBookBySymbolMax,
    uint32_t hist_copies;        // k_book_sort_tiles adds hist_copies of them up into hist_sum (which hist then points to)
    uint32_t *hist_sum;
    RecordArgs recs;           // outlier records to place beside the code book, by the workgroups behind the first one (n_wg == 0: none)
    uint32_t rec_wg_runs;      // so many runs each (a wavefront per run, then the next)
    uint32_t reset_ctl;        // 1: this kernel is the first of its call and clears *ctl itself
    const uint8_t *given_len;  // code book reuse: take these lengths instead of building them from hist (which is then unused)
    uint32_t nbins;
    uint8_t *len_out;          // u8[nbins]
    uint64_t *code_out;        // u64[nbins] or null (stage output)
    uint64_t *enc;             // u64[nbins]: (code << 6) | len, 0 for unused symbols
    BookScratch scratch;
    uint32_t presorted;        // scratch.keys holds the leaves in (frequency, symbol) order (k_book_sort_tiles, k_book_merge) if more than kBookLdsSyms symbols occur
    uint32_t lds_leaves;       // leaves whose weights fit the LDS of the launch (presorted)
    uint32_t narrow;           // all frequencies together are below 2^31 - 1 (a container's header only; a stage call looks for itself)
    Control *ctl;
    // container finalisation (null header = stage call)
    Header *hdr;
    Header proto;              // host-filled fields
    uint64_t capacity;
};
// Dynamic LDS of k_codebook: BookLds; alphabets of more than kBookBySymbolMax bins: what a compute unit has but for a kilobyte, for the weights
// of up to kBookLdsLeaves leaves and one word.  The workgroups that place records ask for as much (one launch), so each waits for
// a compute unit to itself; beside other streams that costs less than the tree in LDS saves: four layers at batch 16 on four
// streams, 65536 bins, 1e-3 567 us -> 486, 1e-4 854 -> 600 (64 KB for all, tree in global memory, records in a kernel of their own).
constexpr uint32_t kBookLdsBytes = 70016u, kBookLdsBytesLarge = kLdsPerCu - 1024u, kBookLdsLeaves = kBookLdsBytesLarge / 4u - 4u;
__global__ void k_codebook(BookArgs a);
constexpr int kBookMergeBlock = 256;
constexpr int kBookDepthBlock = 256;
__global__ void k_book_sort_tiles(BookArgs a);
__global__ void k_book_depths(BookArgs a);
__global__ void k_book_codes(BookArgs a);
template <uint32_t WAYS> __global__ void k_book_merge(const uint64_t *src, uint64_t *dst, uint32_t run, const Control *ctl);   // WAYS: 2 or 4

// ---- encode -------------------------------------------------------------------
constexpr int kEncBlock = 256;             // four wavefronts, each encodes 256 symbols per step cooperatively
constexpr uint32_t kEncTableMax = 2048;    // table entries cached in LDS
constexpr uint32_t kPackBits = 27u;        // longest code word of an entry of 32 bits
// Code lengths (one byte each) the count kernel caches in LDS instead of part of the encode table, if every symbol that
// occurs lies among them: 16384 around the centre (the room of the table's cached part).  Above 32768 bins: all of
// them (64 KB), with twice the wavefronts per workgroup, so that a compute unit holds sixteen of them (two workgroups; a
// window of 32768 lengths, three workgroups of half the size: twelve); a field whose codes reached beyond such a window
// was looked up in global memory instead, 98 us for 64 x 256 x 56 x 56 at a bound of 1e-4, now 38.  Between 16384 and 32768
// bins it is still 16384 of them: all would cost a field whose symbols lie among those 2 % (32768 bins, 128 x 64 x 224 x 224
// smoothed at 3.2e-4 the whole compression 1561 -> 1595 us: fewer workgroups per compute unit) and spare one that
// reaches beyond them the look-ups in global memory (Laplace at 1e-3 2076 -> 1683).
constexpr int kEncBlockWide = 512;
// Entries of 32 bits the pack kernel caches in LDS for alphabets beyond kBookBySymbolMax bins, with eight wavefronts per workgroup (the
// room per wavefront of four wavefronts' 2048 entries of 64 bits): a look-up in global memory costs a cycle per lane.  Filling the
// table costs a workgroup some 10 us, hence for segments of kEncPackMinChunks chunks and more only.  Whole compressions, us, without / with:
//   elements        65536 bins, 1e-4   Laplace 1e-3   16384 bins, 3e-4   1e-3
//     3 M                194 / 204       169 / 179        139 / 149      126 / 136
//    13 M                240 / 243       206 / 215        173 / 180      159 / 165
//    26 M                293 / 293       249 / 256        216 / 222      199 / 204
//    51 M (the line)     400 / 387       342 / 344        303 / 304      282 / 285
//   103 M                621 / 573       482 / 468        436 / 420      406 / 394
//   206 M               1140 / 974       810 / 752        751 / 696      709 / 672
// The cost is one of symbols, the rule counts chunks: with chunks of 128 or 256 symbols the figures are these within 1 % (256 symbols, 103 M
// elements, 1e-4: 608 / 560), the line lies at 101 and 201 M elements.  Where nearly all symbols lie among 2048 entries the table
// is only longer (64 x 256 x 56 x 56, 4096 bins with 4096 such entries 154 -> 164).
constexpr uint32_t kEncPackWindow = 8192, kEncPackMinChunks = 512;
static_assert((kEncTableMax + 1u) * 8u <= kEncPackWindow * 4u, "either kind of entries");
__host__ __device__ inline bool enc_wide(uint32_t nbins) { return nbins > 32768u; }
__host__ __device__ inline uint32_t enc_len_window(uint32_t nbins) { return nbins <= 16384u || enc_wide(nbins) ? nbins : 16384u; }
constexpr uint32_t kEncSegChunksMax = 4096;   // chunks per workgroup segment (their word counts live in LDS)
// ... for enc_wide() alphabets: the lengths, the counts of the largest segment and the scan's words have to fit LDS twice.  With
// 4096 chunks they were 80 bytes too many, and one workgroup per compute unit took 362 us for 128 x 64 x 224 x 224; two
// take 240.  (Other alphabets keep the larger segments: 16384 bins 1152 us at that size instead of 1216.)
constexpr uint32_t kEncSegChunksWide = 4064;
static_assert(2u * (65536u + 8u + 4u * kEncSegChunksWide + 4u * (kEncBlockWide / kWave)) <= kLdsPerCu, "two workgroups of the wide count kernel per compute unit");

// What a call that waits for its container's size is told.  The kernel that seals the header stores it straight into
// the context's pinned host memory, and the end of the stream's work makes it visible: a copy of the control block behind
// that kernel cost 1.8 us of a call (one image, 64 x 28 x 28: 62.0 -> 60.2).
struct CallResult {
    uint64_t total_bytes;
    uint32_t own;              // ST_* bits of this call
    uint32_t latched;          // those and what earlier asynchronous calls on the context have latched
};
__device__ inline void tell_host(CallResult *host, uint64_t total, uint32_t own, uint32_t *latched) {
    const uint32_t before = own || host ? atomicOr(latched, own) : 0u;
    if (host) { host->total_bytes = total; host->own = own; host->latched = before | own; }
}

struct EncodeArgs {
    const uint16_t *codes;
    uint64_t n;
    uint32_t chunk_syms;       // 64, 128 or 256
    uint32_t n_chunks;
    uint32_t seg_chunks;       // chunks per segment (one segment per workgroup)
    const uint64_t *enc;
    const uint8_t *len8;       // device u8[nbins]: the code lengths alone (the container's length section), or null
    uint32_t nbins;
    uint32_t tbl_lo, tbl_n;    // table entries [tbl_lo, tbl_lo + tbl_n) are cached in LDS
    uint32_t tbl_room;         // count kernel: bytes of LDS in front of the word counts (the table, or the lengths of a large alphabet)
    uint32_t *chunk_off;
    uint8_t *container;        // product path: payload position comes from ctl->off_payload
    uint64_t capacity;
    uint32_t *payload;         // stage path: explicit payload buffer
    uint64_t payload_cap_words;
    uint64_t *payload_words_out;   // stage path
    uint64_t *desc;            // words of every segment (written by the count kernel, read by the pack kernel)
    Control *ctl;
    uint32_t *latched;         // product path: the context's persistent status word (the pack kernel seals the header); else null
    CallResult *host;          // product path: pinned host memory for a caller that waits, or null
    uint32_t zero_pair;        // container version 2: (centre << 16) | centre, a chunk of nothing but centre codes takes no words; else 0
    uint4 *clear;              // pack kernel: clear_n16 16-byte words that the next call on the context finds zero (the partial histograms,
    uint32_t clear_n16;        // which have been read by now)
};
// single-pass compression: the words of every run from the work area to the payload
struct PlaceArgs {
    const uint32_t *run_words;     // words of every run
    uint32_t n_runs;               // runs up to the last that holds rows, or a workgroup's more
    uint32_t rows_per_wave, rows_per_wg, rows_total, W;
    uint32_t chunk_syms;
    const uint32_t *work_words;    // the run that starts at element e has its words from word e / 64 * words64 on
    uint32_t words64;
    uint8_t *container;
    uint64_t capacity;
    RecordArgs recs;               // the outlier records, which each wavefront places for its own run as well
    Control *ctl;
    uint32_t *latched;             // the context's persistent status word
    CallResult *host;              // pinned host memory for a caller that waits, or null
};
constexpr int kPlaceBlock = 256;
__global__ void k_place_payload(PlaceArgs a);

constexpr uint32_t kEncUnroll = 4;         // steps of 256 symbols a wavefront handles per iteration
constexpr uint32_t kEncStepWordsMax = 468; // 256 code words of up to 58 bits, in 32-bit words, plus slack
constexpr uint32_t kEncBufWords = 640;     // assembly buffer of a wavefront (ordinary code books fill a fraction of it)
// S: symbols per chunk (64, 128, 256); FULLTBL: the whole encode table is in LDS
template <int S, bool FULLTBL, int NT> __global__ void k_encode_count(EncodeArgs a);   // NT threads (kEncBlock, or kEncBlockWide)
template <int S, bool FULLTBL, int NT> __global__ void k_encode_pack(EncodeArgs a);

// ---- decode tables ------------------------------------------------------------
constexpr int kLutBits = 11;
constexpr uint32_t kLutSize = 1u << kLutBits;
// Alphabets of at most kLut16MaxBins bins (residuals fit 12 signed bits) also get a compact table on
// the next 12 bits: same 8 KB of LDS, half as many codes too long for it.
constexpr int kLut16Bits = 12;
constexpr uint32_t kLut16Size = 1u << kLut16Bits;
constexpr uint32_t kLut16MaxBins = 4096;
constexpr int32_t kLut16Escape = -2048;    // residual value that stands for the escape symbol in the compact table
constexpr int kLenBits = 13;
constexpr uint32_t kLenMixed = 0x80u;
constexpr uint32_t kLenFast = 32u;         // longest code of a length table entry without the mark
static_assert((1u << kLenBits) == 2u * kLut16Size && 4u * kLutSize == 2u * kLut16Size, "the tables the chunk decoders load are of one size");
constexpr uint32_t kSubEntries = 2048;     // second level of the compact table: entries of all sub-tables together

struct DecodeTables {          // all in the workspace (global memory)
    uint32_t *lut;             // kLutSize entries: (residual << 8) | length with residual = symbol - radius
                               // (-32768 for the escape symbol 0); length 0 = code longer than kLutBits, the
                               // residual field then holds the shortest length a code with this prefix can have
    uint64_t *limit;           // [65]: left-aligned exclusive upper bound of the codes of each length
    uint64_t *first_code;      // [65]
    uint32_t *first_index;     // [65]: position of the first symbol of each length in `sorted`
    uint16_t *lut16;           // (if the alphabet is too large for the compact table: the length table instead, of the same size, so that
                               // the chunk decoders always load from here; meta[4] tells which it is.  One byte per prefix of kLenBits
                               // bits: the length of the codes under it if they are all as long, at most 32 bits; else kLenMixed plus
                               // the shortest length)
                               // kLut16Size entries: (residual << 4) | length, residual in 12 signed bits (kLut16Escape for
                               // the escape symbol); length 0 = longer code: the upper 12 bits are (offset / 2) << 2 | width
                               // code of the prefix's sub-table in sub16 (width 1, 2, 4, 6 bits), all zero if it has none
    uint16_t *sub16;           // (too large an alphabet: the first kSubEntries entries of `resid`)
                               // kSubEntries entries: (residual << 4) | (length - kLut16Bits), 0 = longer still
    uint16_t *sorted;          // symbols in canonical (length, symbol) order
    uint16_t *resid;           // (too large an alphabet) their residuals, int16, -32768 for the escape symbol; 65536 entries
    uint32_t *meta;            // [0] max_len, [1] n_active, [2] min_len, [3] radius, [4] 1 if lut16 is valid
};

struct TablesArgs {
    const uint8_t *len;        // u8[nbins]
    uint32_t nbins;
    DecodeTables t;
    uint32_t compact_only;     // 1: the caller decodes with the chunk decoders, which never read the general table
    uint32_t general_unless_chunk64;   // 1: ... except for a container whose chunks are not 64 symbols (its kernel reads the general table)
    Control *ctl;
    uint32_t reset_ctl;        // 1: this kernel is the first of its call and clears *ctl itself (no separate fill before it)
    uint32_t *latched;         // if set, a status bit raised here also goes into this persistent word (no separate kernel after the call)
    int32_t *status_out;       // if set: receives 0, or -3 (the library's code for a malformed container) if the header or the table is refused
    // container validation (null = stage call)
    const Header *hdr;
    Header expect;             // shape the caller passed
    uint64_t bytes;
};
__global__ void k_decode_tables(TablesArgs a);

// ---- decode + reconstruct -----------------------------------------------------
constexpr int kDecBlock = 64;
constexpr uint32_t kDecTileElems = 8192;   // elements per strip held in LDS

struct ReconArgs {
    // source: a container (product) or explicit arrays (stage calls)
    const uint8_t *container;
    const uint16_t *codes_in;      // stage reconstruct: codes come from memory
    const uint32_t *chunk_off;
    const uint32_t *payload;
    uint64_t payload_words;
    const uint32_t *rec;
    uint64_t n_rec;
    uint32_t chunk_syms, log2_chunk, n_chunks;
    DecodeTables t;
    uint64_t n;
    uint32_t planes, H, W;
    FastDiv divW;
    int32_t radius;
    float eb, ebx2;
    // strip geometry
    uint32_t planes_per_unit;      // >= 1 when a unit is a group of whole planes
    uint32_t rows_per_strip;       // rows of one strip when a plane is cut into strips
    uint32_t n_units;
    uint32_t pitch;                // LDS row pitch (odd)
    uint32_t tile_rows;            // rows held in LDS
    uint32_t use_carry;            // 1 if planes are cut into strips (column carry in LDS)
    float *out;
    uint32_t skip_chunk64;         // 1: do nothing for a container with chunks of 64 symbols (k_decode_scan has handled it)
    uint16_t *codes_out;           // stage decode: write codes instead of reconstructing
    uint32_t zero_chunks;          // stage decode: a chunk without words is the centre code throughout (a container says so in its version)
    Control *ctl;
};
template <int MODE> __global__ void k_reconstruct(ReconArgs a);   // 0 container, 1 codes from memory
__global__ void k_decode_only(ReconArgs a);

// ---- decode + reconstruct, fast path (planes up to 512 columns): two kernels ------
constexpr int kDsWaves = 4;                           // wavefronts per workgroup, each working on its own
constexpr int kDsBlock = kDsWaves * kWave;
constexpr uint32_t kDsStageWords = 1536u;             // decode: Huffman words of 64 chunks per wavefront (LDS)
constexpr uint32_t kDsStageBatch = 8u;                // decode: loads in flight per lane while those words are fetched
constexpr uint32_t kDsMaxW = 512u;
constexpr uint32_t kDsTailEntries = 1024u;            // decode, compact table: residuals of long codes kept in LDS
constexpr uint32_t kScanListWords = 1024u;            // scan: escape list of a strip per wavefront (pairs) (LDS)
constexpr uint32_t kScanStripElems = 4096u;           // scan: elements per strip (unit of the escape list)

struct DsArgs {
    const uint8_t *container;
    DecodeTables t;
    uint64_t n;
    uint32_t planes, H, W;
    uint32_t group_planes;     // scan kernel, planes of at most 32 columns: whole planes per unit of work (a multiple of the planes side by side in a wavefront)
    FastDiv divW;
    FastDiv divL;              // scan kernel: lanes per row (W / columns per lane)
    uint32_t skip_chunk64;     // 1: do nothing for a container with chunks of 64 symbols (k_decode_scan has handled it)
    int16_t *resid;            // work buffer: one int16 residual per element (-32768 = escaped)
    void *out;                 // fp32, or IEEE half / bfloat16 (template parameter OUT of the scan kernel)
    Control *ctl;
};
__global__ void k_decode_chunks(DsArgs a);
// NSEG = ceil(lanes per row / 64) rounded up to 1, 2, 4, 8; OUT: element type of the output (0 fp32, 1 IEEE half, 2 bfloat16:
// the fp32 result rounded to nearest even)
// VEC: adjacent columns per lane (2: even W, output aligned to two elements); the lane mapping follows W / VEC
template <int NSEG, int MODE, int OUT = 0, int VEC = 1> __global__ void k_scan_store(DsArgs a);

// ---- reconstruct from the residuals of k_decode_chunks, planes cut into bands of rows and segments of columns -------
constexpr int kBandBlock = 256;                       // four wavefronts, each on a unit of its own
static_assert(kBandLanes == (uint32_t)kWave && kBandRowsMax <= kBandLanes, "lanes of a unit");

struct BandArgs {
    const uint8_t *container;
    uint32_t planes, H, W;
    uint32_t R;                // rows per band (the last band of a plane may have fewer)
    FastDiv divSegs;           // segments of 64 lanes per row (one or two columns per lane)
    FastDiv divBands;          // bands per plane
    uint32_t n_units;          // planes * bands * segments; segments of a band are neighbours, bands of a plane as well
    int16_t *resid;            // work buffer: one int16 residual per element
    int32_t *col_sums;         // [plane][band, but the last][W]
    int32_t *row_sums;         // [plane, band][segment, but the last][R]
    int32_t *unit_sums;        // [n_units]: of those that are neither in the last band nor in the last segment
    void *out;
    Control *ctl;
};
__global__ void k_band_patch(BandArgs a);
template <int VEC> __global__ void k_band_sums(BandArgs a);
template <int VEC, int OUT> __global__ void k_band_store(BandArgs a);
template <int OUT> __global__ void k_band_verbatim(BandArgs a);

// ---- decode + reconstruct in one kernel (planes up to 512 columns, chunks of 64 symbols) ----------
constexpr int kFuWaves = 16;                          // wavefronts per workgroup, each working on its own; one workgroup per CU
static_assert((uint32_t)kFuWaves == kBandFuWaves, "the rule for bands counts with them");
constexpr int kFuBlock = kFuWaves * kWave;
constexpr uint32_t kFuStripWords = 64u * 32u;         // a strip's residuals, element after element (64 chunks of 64 int16); before that, the words of its chunks
constexpr uint32_t kFuEscEntries = 32u;               // values of a strip's escaped residuals kept in LDS
constexpr uint32_t kFuRegionWords = kFuStripWords + kFuEscEntries;
constexpr uint32_t kFuPrefetch = 20u;                 // words per lane (of a strip's chunks) loaded while the strip before is scanned
constexpr uint32_t kFuCarryW = 128u;                  // widest plane whose strips are dealt to all wavefronts of a workgroup (column sums handed on through LDS), one column per lane; twice that with two

struct FuArgs {
    const uint8_t *container;
    DecodeTables t;
    uint64_t n;
    uint32_t planes, H, W;
    uint32_t G;                // whole planes per unit of work (one wavefront walks a unit)
    uint32_t n_units;
    FastDiv divW, divH;
    FastDiv divL;              // lanes per row (W / columns per lane)
    FastDiv divSpr;            // rows of at most 16 lanes: rows side by side in 16 lanes
    FastDiv divK;              // rows per step
    void *out;                 // fp32, or IEEE half / bfloat16 (template parameter OUT)
    Control *ctl;
};
// NSEG, MODE, OUT, VEC as for k_scan_store; MODE 0 / 1 walk several consecutive rows per step
template <int NSEG, int MODE, int OUT = 0, int VEC = 1> __global__ void k_decode_scan(FuArgs a);

}  // namespace comet
