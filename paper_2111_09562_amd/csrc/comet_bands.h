// Geometry of the reconstruction in bands (k_band_*) and the rule that chooses it.  Plain C++: host code, and a CPU test
// that compiles it by itself.
#pragma once
#include <cstdint>

namespace comet {

constexpr uint32_t kBandLanes = 64;                         // lanes of a wavefront
constexpr uint32_t kBandRowsMin = 8u, kBandRowsMax = 64u;   // rows of a unit (the upper limit: one lane per row)
constexpr uint32_t kBandFuWaves = 16;                       // wavefronts of a workgroup of k_decode_scan

inline uint64_t band_align(uint64_t v, uint64_t a) { return (v + a - 1) / a * a; }

// Reconstruction in bands (k_band_*): columns per lane, rows per band, segments per row, bands per plane, units, and
// the offsets of the three arrays of sums inside their workspace of `bytes` bytes.
struct BandGeom { uint32_t vec, R, segs, bands; uint64_t n_units, off_row, off_unit, bytes; };
// About 2^19 * 64 elements or more: bands of 64 rows; smaller tensors: fewer rows, so that there are enough units to
// fill the chip (a unit has 128 columns at most; 2^19 / 128 = 4096 units, four per SIMD).
inline BandGeom band_geometry(uint64_t planes, uint32_t H, uint32_t W, uint32_t vec) {
    const uint64_t n = planes * H * W;
    BandGeom g{};
    g.vec = vec;
    const uint32_t seg_w = kBandLanes * vec;
    g.segs = (W + seg_w - 1u) / seg_w;
    uint64_t R = n >> 19;
    if (R < kBandRowsMin) R = kBandRowsMin;
    if (R > kBandRowsMax) R = kBandRowsMax;
    g.bands = (uint32_t)((H + R - 1u) / R);
    g.R = (H + g.bands - 1u) / g.bands;
    g.bands = (H + g.R - 1u) / g.R;
    // sums that some unit reads: of columns for every band of a plane but its last, of rows for every segment but the
    // last, of whole units if there are both
    g.n_units = planes * g.bands * g.segs;
    g.off_row = band_align(4ull * planes * (g.bands - 1u) * W, 256);
    g.off_unit = g.off_row + band_align(4ull * planes * g.bands * (g.segs - 1u) * g.R, 256);
    g.bytes = g.off_unit + (g.bands > 1u && g.segs > 1u ? band_align(4ull * g.n_units, 256) : 0u);
    return g;
}
constexpr uint32_t kBandMinW = 128;     // narrower planes leave lanes of a unit idle (and a workgroup of k_decode_scan shares a plane)
// What the sums of any tensor of up to n elements take, planes of at least kBandMinW columns.  With R0 the rows per band that
// band_geometry starts from (8 below 4.7 million elements, about n / 2^19 up to 2^25, then 64): less than a column sum per R0
// elements (2^21 of them at most below 2^25 elements); less than a row sum per 64, times ten ninths (a plane of nine rows has
// bands of five); a unit sum per 43 (129 columns in three segments) times (R0 + 1) / 2.
constexpr uint64_t band_bytes_max(uint64_t n) {
    const uint64_t col = n / 2u < (5ull << 19) ? n / 2u : (n / 16u > (5ull << 19) ? n / 16u : (5ull << 19));
    const uint64_t unit = n / 48u < (1ull << 17) ? n / 48u : (n / 348u > (1ull << 17) ? n / 348u : (1ull << 17));
    return col + n / 14u + unit + 1024u;
}

// Planes of at most 512 columns: is the reconstruction in bands quicker than the kernels with a plane per wavefront or
// workgroup?  Those take as long as their longest serial chain (or as the elements take, for many planes); the bands
// have no chain, and move more bytes.  Estimates in us from measurements (old kernel / bands):
//   k_decode_scan, a plane per wavefront (10 us a strip of 4032 elements, 20 with one column per lane):
//     4 planes of 512 x 512 672 / 48, 64 721 / 91, 1024 848 / 991; 256 planes of 257 x 257 361 / 99, 1024 452 / 340, 4096 757 / 1260
//   k_decode_scan, a plane's strips dealt to the sixteen wavefronts of a workgroup (20 us a round):
//     8 planes of 3000 x 256 265 / 84, 32 of 256 x 256 45 / 51, 512 of them 75 / 127
//   k_scan_store (a plane per wavefront, 0.25 us a row and 0.06 more per 64 lanes of it; 1.3 us per million elements,
//   2 if a row takes more than 128 lanes), chunks of 128 symbols:
//     16 planes of 224 x 224 107 / 52, 4096 of them 664 / 767, 1024 of 512 x 512 1086 / 955, 4096 of 257 x 257 973 / 1227
//   and on top of the bands' linear cost, what k_band_store reads of the column sums above it, (bands per plane)^2 / 2 rows of
//   them per plane, at 20 TB/s (15 where a plane's do not fit the caches):
//     60 planes of 262143 x 128 11.4 ms / 19.2, 30 of them 11.3 / 9.7, 15 of 1048575 x 128 45 / 59, 7 of 2097151 x 128 91 / 133, 3 of them 90 / 57
inline bool band_pays(int num_cu, uint64_t planes, uint32_t H, uint32_t W, const BandGeom &g, bool chunk64) {
    const uint64_t P = (uint64_t)H * W;
    const uint32_t vec = g.vec, lpr = W / vec;
    const double mega = (double)planes * (double)P * 1e-6;
    const double col = 4.0 * (double)g.bands * (double)W;    // bytes of a plane's column sums
    const double above = g.bands > 1u ? (double)planes * (double)g.bands * 0.5 * col / (col <= 10e6 ? 20e6 : 15e6) : 0.0;
    if (!chunk64) {                                          // (the decoding itself is the same kernel on both sides)
        const double row = 0.25 + 0.06 * (double)((lpr + 63u) / 64u);
        const uint64_t waves = (uint64_t)num_cu * 32u;
        const double chain = row * (double)H * (double)((planes + waves - 1u) / waves);
        const double flow = (lpr <= 128u ? 1.3 : 2.0) * mega;
        return 30.0 + (vec == 2u ? 1.7 : 2.6) * mega + above < (chain > flow ? chain : flow);
    }
    const double bands = 45.0 + (vec == 2u ? 3.6 : 4.5) * mega + above;
    const uint64_t strip = 4032u / W * W, strips = (P + strip - 1u) / strip;
    if (lpr <= 128u) {
        const uint64_t seg_planes = (planes + (uint64_t)num_cu - 1u) / (uint64_t)num_cu;
        return bands < 20.0 * (double)((seg_planes * strips + (uint64_t)kBandFuWaves - 1u) / (uint64_t)kBandFuWaves);
    }
    const uint64_t waves = (uint64_t)num_cu * kBandFuWaves;
    return bands < (vec == 2u ? 10.0 : 20.0) * (double)(strips * ((planes + waves - 1u) / waves));
}

}  // namespace comet
