// Lorenzo reconstruction for tensors whose planes are too few or too wide to keep the chip busy with a plane per
// wavefront or workgroup (COMET Sec. 3.4 / Sec. 4.1 run backwards): every plane is cut into units of at most 64 rows
// by 64 lanes of columns, and all units of the tensor are scanned side by side.
//
// The value at (r, w) is the sum of the residuals at or above row r and at or left of column w.  Behind
// k_decode_chunks, which leaves the residuals as int16 in the work buffer:
//   k_band_patch   escaped residuals from the outlier records into the work buffer (those beyond int16 keep the
//                  marker and are looked up where they are met);
//   k_band_sums    per unit: the sum of every column, of every row, and of the whole unit;
//   k_band_store   per unit: what lies above its columns (column sums of the bands above, then a prefix over the
//                  columns), left of its rows (row sums of the units to the left, then a prefix over the rows) and
//                  above and left of it (unit sums), then the scan of its own rows, dequantised and stored;
//   k_band_verbatim  values stored verbatim overwrite what lies on the lattice.
// No unit waits for another one: ten bytes per element move instead of four (the residuals are written once and read
// twice), but a plane is no longer a serial chain.  Bound by the memory behind the residual stores for large tensors,
// by the five launches for small ones.  32 planes of 480 x 854 (13.1 M elements), the whole decompression: 5210 us with
// a plane per wavefront (k_reconstruct, strips of 8192 elements one after the other), 85 us in these; 3.6 us per
// further million elements.  The sums above a unit are added up by the unit, so what is read of them grows with the square
// of the bands per plane: nothing to speak of for images, but a plane of 2097151 x 128 takes 19 ms, 18 of them for that (see
// band_pays).
#include "comet_kernels.h"
#include "comet_scan.h"

namespace comet {

namespace {

struct BandUnit {
    uint32_t pb, s;                     // (plane, band), segment of columns
    uint32_t plane, band, rows;
    uint32_t e0;                        // first element
    uint32_t lanes;                     // lanes that hold columns
};

template <int VEC>
__device__ inline BandUnit band_unit(const BandArgs &a, uint32_t u) {
    BandUnit b;
    b.pb = fdiv(u, a.divSegs);
    b.s = u - b.pb * a.divSegs.d;
    b.plane = fdiv(b.pb, a.divBands);
    b.band = b.pb - b.plane * a.divBands.d;
    const uint32_t r0 = b.band * a.R;
    b.rows = (a.H - r0 < a.R) ? a.H - r0 : a.R;
    const uint32_t w0 = b.s * (uint32_t)kWave * VEC;
    b.e0 = (b.plane * a.H + r0) * a.W + w0;
    const uint32_t left = (a.W - w0) / VEC;
    b.lanes = left < (uint32_t)kWave ? left : (uint32_t)kWave;
    return b;
}

constexpr uint32_t kBandOob = 0x80000000u;  // byte offset beyond every unit

// The rows of a unit, eight loads in flight while eight rows are worked on: f(row, residuals of my columns).
template <int VEC, typename F>
__device__ inline void band_rows(const BandArgs &a, const BandUnit &b, uint32_t lane, F f) {
    constexpr uint32_t U = 8;
    const uint32_t bytes = ((b.rows - 1u) * a.W + b.lanes * VEC) * 2u;
    const __amdgpu_buffer_rsrc_t r_in = make_rsrc(a.resid + b.e0, bytes);
    const uint32_t voff = lane < b.lanes ? lane * (VEC * 2u) : kBandOob;
    uint32_t cur[U], nxt[U];
    auto fetch = [&](uint32_t r0, uint32_t (&raw)[U]) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            const uint32_t r = r0 + u < b.rows ? r0 + u : b.rows - 1u;       // (uniform; past the end the last row again, unused)
            if (VEC == 2) raw[u] = __builtin_amdgcn_raw_buffer_load_b32(r_in, (int)voff, (int)(r * a.W * 2u), 0);
            else raw[u] = (uint32_t)__builtin_amdgcn_raw_buffer_load_b16(r_in, (int)voff, (int)(r * a.W * 2u), 0);
        }
    };
    auto work = [&](uint32_t r0, const uint32_t (&raw)[U]) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
            if (r0 + u >= b.rows) break;                                      // uniform
            int32_t d[VEC];
            d[0] = (int32_t)(int16_t)(raw[u] & 0xffffu);
            if (VEC == 2) d[VEC - 1] = (int32_t)raw[u] >> 16;
            bool esc = false;
#pragma unroll
            for (int v = 0; v < VEC; ++v) esc = esc || d[v] == kEscape;
            if (__builtin_expect(wave_ballot(esc) != 0ull, 0)) {              // an escaped residual beyond int16: from the records
#pragma unroll
                for (int v = 0; v < VEC; ++v)
                    if (d[v] == kEscape) {
                        const uint32_t key = 2u * (b.e0 + (r0 + u) * a.W + lane * VEC + (uint32_t)v);
                        const Header *hdr = reinterpret_cast<const Header *>(a.container);
                        const uint32_t *rec = reinterpret_cast<const uint32_t *>(a.container + hdr->off_outlier);
                        const uint32_t n_rec = hdr->n_rec;
                        uint32_t lo = 0, hi = n_rec;
                        while (lo < hi) { const uint32_t mid = lo + ((hi - lo) >> 1); if (rec[2 * (size_t)mid] < key) lo = mid + 1; else hi = mid; }
                        d[v] = (lo < n_rec && rec[2 * (size_t)lo] == key) ? (int32_t)rec[2 * (size_t)lo + 1] : 0;
                    }
            }
            f(r0 + u, d);
        }
    };
    fetch(0, cur);
    for (uint32_t r0 = 0; r0 < b.rows; r0 += 2u * U) {
        fetch(r0 + U, nxt);
        work(r0, cur);
        fetch(r0 + 2u * U, cur);
        work(r0 + U, nxt);
    }
}

}  // namespace

// Escaped residuals that fit int16 become residuals like any other.
__global__ __launch_bounds__(kBandBlock) void k_band_patch(BandArgs a) {
    if (a.ctl->status & ST_FORMAT) return;
    const Header *hdr = reinterpret_cast<const Header *>(a.container);
    const uint2 *rec = reinterpret_cast<const uint2 *>(a.container + hdr->off_outlier);
    const uint32_t n_rec = hdr->n_rec, n = a.planes * a.H * a.W;
    for (uint64_t i = (uint64_t)blockIdx.x * kBandBlock + threadIdx.x; i < n_rec; i += (uint64_t)gridDim.x * kBandBlock) {
        const uint2 r = rec[i];
        const int32_t v = (int32_t)r.y;
        if (!(r.x & 1u) && (r.x >> 1) < n) a.resid[r.x >> 1] = (int16_t)((v > kEscape && v < 32768) ? v : kEscape);
    }
}

template <int VEC>
__global__ __launch_bounds__(kBandBlock) void k_band_sums(BandArgs a) {
    if (a.ctl->status & ST_FORMAT) return;
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t u = blockIdx.x * (uint32_t)(kBandBlock / kWave) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (u >= a.n_units) return;
    const BandUnit b = band_unit<VEC>(a, u);
    int32_t col[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) col[v] = 0;
    int32_t row = 0, unit = 0;                                   // lane r: the sum of row r; the sum of the rows so far (uniform)
    band_rows<VEC>(a, b, lane, [&](uint32_t r, const int32_t (&d)[VEC]) {
        int32_t mine = 0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) {
            col[v] = (int32_t)((uint32_t)col[v] + (uint32_t)d[v]);
            mine = (int32_t)((uint32_t)mine + (uint32_t)d[v]);
        }
        const int32_t total = __builtin_amdgcn_readlane(run_scan<2>(mine, lane, (uint32_t)kWave), 63);
        row = lane == r ? total : row;
        unit = (int32_t)((uint32_t)unit + (uint32_t)total);
    });
    if (b.s + 1u < a.divSegs.d && lane < b.rows) a.row_sums[((size_t)b.pb * (a.divSegs.d - 1u) + b.s) * a.R + lane] = row;
    if (b.band + 1u < a.divBands.d) {
        int32_t *dst = a.col_sums + (size_t)(b.pb - b.plane) * a.W + b.s * (uint32_t)kWave * VEC + lane * VEC;
        if (lane < b.lanes) {
            if (VEC == 2) *reinterpret_cast<int2 *>(dst) = make_int2(col[0], col[VEC - 1]);
            else *dst = col[0];
        }
        if (b.s + 1u < a.divSegs.d && lane == 0) a.unit_sums[u] = unit;
    }
}

template <int VEC, int OUT>
__global__ __launch_bounds__(kBandBlock) void k_band_store(BandArgs a) {
    constexpr uint32_t OS = OUT ? 2u : 4u;
    if (a.ctl->status & ST_FORMAT) return;
    const uint32_t lane = (uint32_t)lane_id();
    const uint32_t u = blockIdx.x * (uint32_t)(kBandBlock / kWave) + (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
    if (u >= a.n_units) return;
    const BandUnit b = band_unit<VEC>(a, u);
    const float ebx2 = __uint_as_float(reinterpret_cast<const Header *>(a.container)->ebx2_bits);
    const uint32_t segs = a.divSegs.d;

    // above my columns
    uint32_t q[VEC];
#pragma unroll
    for (int v = 0; v < VEC; ++v) q[v] = 0;
    if (lane < b.lanes) {
        const int32_t *src = a.col_sums + (size_t)b.plane * (a.divBands.d - 1u) * a.W + b.s * (uint32_t)kWave * VEC + lane * VEC;
#pragma unroll 8
        for (uint32_t k = 0; k < b.band; ++k, src += a.W) {
            if (VEC == 2) { const int2 t = *reinterpret_cast<const int2 *>(src); q[0] += (uint32_t)t.x; q[VEC - 1] += (uint32_t)t.y; }
            else q[0] += (uint32_t)*src;
        }
    }
    // left of my rows (lane r: row r), and above and left of me
    uint32_t left = 0, corner = 0;
    if (lane < b.rows) {
        const int32_t *src = a.row_sums + (size_t)b.pb * (segs - 1u) * a.R + lane;
#pragma unroll 8
        for (uint32_t k = 0; k < b.s; ++k, src += a.R) left += (uint32_t)*src;
    }
    for (uint32_t i = lane; i < b.band * b.s; i += (uint32_t)kWave) {
        const uint32_t k = i / b.s;
        corner += (uint32_t)a.unit_sums[(size_t)(b.pb - b.band + k) * segs + (i - k * b.s)];
    }
    const uint32_t base = wave_incl_scan<uint32_t>(left) + wave_sum<uint32_t>(corner);
    {
        uint32_t mine = 0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) mine += q[v];
        const uint32_t incl = (uint32_t)run_scan<2>((int32_t)mine, lane, (uint32_t)kWave);
        if (VEC == 2) q[0] = incl - q[VEC - 1];
        q[VEC - 1] = incl;
    }
    const __amdgpu_buffer_rsrc_t r_out = make_rsrc(reinterpret_cast<char *>(a.out) + (size_t)b.e0 * OS, ((b.rows - 1u) * a.W + b.lanes * VEC) * OS);
    const uint32_t voff = lane < b.lanes ? lane * (VEC * OS) : kBandOob;
    band_rows<VEC>(a, b, lane, [&](uint32_t r, const int32_t (&d)[VEC]) {
        uint32_t mine = 0;
#pragma unroll
        for (int v = 0; v < VEC; ++v) mine += (uint32_t)d[v];
        const uint32_t incl = (uint32_t)run_scan<2>((int32_t)mine, lane, (uint32_t)kWave);
        const uint32_t over = (uint32_t)__builtin_amdgcn_readlane((int)base, (int)r);
        if (VEC == 2) q[0] += incl - (uint32_t)d[VEC - 1];
        q[VEC - 1] += incl;
        float val[VEC];
#pragma unroll
        for (int v = 0; v < VEC; ++v) val[v] = (float)(int32_t)(q[v] + over) * ebx2;
        const int soff = (int)(r * a.W * OS);
        if (OUT == 0 && VEC == 2) {
            u32x2_t two;
            two.x = __float_as_uint(val[0]); two.y = __float_as_uint(val[VEC - 1]);
            __builtin_amdgcn_raw_buffer_store_b64(two, r_out, (int)voff, soff, 0);
        } else if (OUT == 0) {
            __builtin_amdgcn_raw_buffer_store_b32(__float_as_uint(val[0]), r_out, (int)voff, soff, 0);
        } else if (VEC == 2) {
            __builtin_amdgcn_raw_buffer_store_b32(narrow16<OUT>(val[0]) | (narrow16<OUT>(val[VEC - 1]) << 16), r_out, (int)voff, soff, 0);
        } else {
            __builtin_amdgcn_raw_buffer_store_b16((unsigned short)narrow16<OUT>(val[0]), r_out, (int)voff, soff, 0);
        }
    });
}

template <int OUT>
__global__ __launch_bounds__(kBandBlock) void k_band_verbatim(BandArgs a) {
    if (a.ctl->status & ST_FORMAT) return;
    const Header *hdr = reinterpret_cast<const Header *>(a.container);
    const uint2 *rec = reinterpret_cast<const uint2 *>(a.container + hdr->off_outlier);
    const uint32_t n_rec = hdr->n_rec, n = a.planes * a.H * a.W;
    const float eb = __uint_as_float(hdr->eb_bits);
    for (uint64_t i = (uint64_t)blockIdx.x * kBandBlock + threadIdx.x; i < n_rec; i += (uint64_t)gridDim.x * kBandBlock) {
        const uint2 r = rec[i];
        if ((r.x & 1u) && (r.x >> 1) < n) {
            float v = __uint_as_float(r.y);
            if (fabsf(v) <= eb) v = 0.0f;
            if (OUT == 0) static_cast<float *>(a.out)[r.x >> 1] = v;
            else static_cast<unsigned short *>(a.out)[r.x >> 1] = (unsigned short)narrow16<OUT>(v);
        }
    }
}

template __global__ void k_band_sums<1>(BandArgs);
template __global__ void k_band_sums<2>(BandArgs);
#define COMET_INST_BAND(OUT)                                \
    template __global__ void k_band_store<1, OUT>(BandArgs); \
    template __global__ void k_band_store<2, OUT>(BandArgs); \
    template __global__ void k_band_verbatim<OUT>(BandArgs);
COMET_INST_BAND(0)
COMET_INST_BAND(1)
COMET_INST_BAND(2)
#undef COMET_INST_BAND

}  // namespace comet
