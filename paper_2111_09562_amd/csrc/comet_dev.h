// Shared device-side definitions of libcomet: container header, per-call control
// block, wavefront/block scans.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

namespace comet {

constexpr uint32_t kMagic = 0x31544D43u;   // bytes 'C','M','T','1'
constexpr uint32_t kHeaderBytes = 128u;
constexpr int kWave = 64;                   // CDNA wavefront width

// device-side status bits, latched in Control::status
enum : uint32_t { ST_CAPACITY = 1u, ST_FORMAT = 2u, ST_INTERNAL = 4u, ST_CODEBOOK = 8u };

// Container header.  Field order is the on-disk order (little-endian).
struct Header {
    uint32_t magic, version, status, N, C, H, W, nbins;
    uint32_t chunk_syms, n_chunks, eb_bits, ebx2_bits, r_bits, n_active, max_len, n_rec;
    uint64_t nnz, payload_words, total_bytes, off_len, off_chunk, off_outlier, off_payload;
    uint32_t n_vrec, zero;
};
static_assert(sizeof(Header) == kHeaderBytes, "header layout");

// Per-call control block in the workspace; zeroed by the first kernel of every call.
struct Control {
    uint32_t status;        // ST_* bits of this call
    uint32_t pad;
    uint64_t n_rec;         // all outlier records
    uint64_t n_vrec;        // verbatim (type 1) records
    uint64_t nnz;           // non-zero inputs
    uint64_t payload_words;
    uint64_t off_payload;   // byte offset of the payload section (known once the records are counted)
    uint64_t total_bytes;
    uint32_t n_active;
    uint32_t max_len;
    uint32_t enc_in_window;  // k_codebook: every symbol with a code word, but for the escape symbol, lies in the part of the encode table the encoders cache in LDS
    uint32_t len_in_window;  // k_codebook: ... in the (wider) part whose lengths the count kernel caches
    uint32_t outside;        // k_book_sort_tiles: bit 0: a symbol outside the first part occurs, bit 1: outside the second, bit 2: outside the third
    uint32_t pack_in_window; // ... in the part whose entries the pack kernel caches, and no code word is too long for those
};

// Orders the LDS accesses of the lanes of one wavefront (writes before, reads after).  Only the
// LDS counter is waited for: a fence over all address spaces would also wait for every global
// load and store in flight, which turns a streaming loop into one memory round trip per step.
__device__ inline void wave_lds_fence() {
    __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup", "local");
    __builtin_amdgcn_wave_barrier();
}

// A barrier of the workgroup that orders accesses to LDS only: __syncthreads also waits until every global store in flight has
// arrived, which costs a loop that stores results it never reads a round trip per turn.
__device__ inline void lds_barrier() {
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// Lanes of the wavefront for which `p` holds.  (The HIP __ballot takes an int: its bool -> int -> compare
// round trip costs two extra vector instructions per call.)
__device__ inline uint64_t wave_ballot(bool p) { return __builtin_amdgcn_ballot_w64(p); }

__host__ __device__ inline uint64_t align16(uint64_t v) { return (v + 15u) & ~(uint64_t)15u; }

// ---------------------------------------------------------------------------
// exact unsigned division of 32-bit values by a runtime constant:
// floor(x / d) = mulhi64(x, ceil(2^64 / d)) for every x < 2^32, d >= 2
// (error term x * (d*M - 2^64) < 2^32 * d <= 2^64).  d == 1 is the identity.
// ---------------------------------------------------------------------------
struct FastDiv {
    uint64_t magic;
    uint32_t d;
};
inline FastDiv make_fastdiv(uint32_t d) {
    FastDiv f;
    f.d = d;
    f.magic = (d <= 1u) ? 0ull : (~0ull / d + 1ull);
    return f;
}
__device__ inline uint32_t fdiv(uint32_t x, const FastDiv &f) {
    return (f.d <= 1u) ? x : (uint32_t)__umul64hi((uint64_t)x, f.magic);
}

// ---------------------------------------------------------------------------
// wavefront / block scans
// ---------------------------------------------------------------------------
__device__ inline int lane_id() { return (int)__lane_id(); }

template <typename T>
__device__ inline T wave_incl_scan(T v) {
    const int lane = lane_id();
#pragma unroll
    for (int d = 1; d < kWave; d <<= 1) {
        T t = __shfl_up(v, d, kWave);
        if (lane >= d) v += t;
    }
    return v;
}

template <typename T>
__device__ inline T wave_sum(T v) {
#pragma unroll
    for (int d = kWave / 2; d > 0; d >>= 1) v += __shfl_xor(v, d, kWave);
    return v;
}

// Exclusive scan over the block; `total` receives the block sum.  s_part must
// hold one T per wavefront.  Contains two barriers.
template <typename T, int NWAVES>
__device__ inline T block_excl_scan(T v, T *s_part, T &total) {
    const int lane = lane_id();
    const int wave = threadIdx.x / kWave;
    T incl = wave_incl_scan(v);
    if (lane == kWave - 1) s_part[wave] = incl;
    __syncthreads();
    T off = 0, tot = 0;
#pragma unroll
    for (int w = 0; w < NWAVES; ++w) {
        T t = s_part[w];
        if (w < wave) off += t;
        tot += t;
    }
    __syncthreads();
    total = tot;
    return off + incl - v;
}

}  // namespace comet
