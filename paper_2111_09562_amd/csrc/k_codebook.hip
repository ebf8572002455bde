// Codebook kernels (COMET Sec. 4.1, "customized Huffman coding"):
//   k_codebook       histogram -> Huffman code lengths -> canonical codes -> encode
//                    table; also lays out the container (header, section offsets).  Its
//                    workgroups behind the first one place the outlier records meanwhile.
//   k_decode_tables  length table -> canonical decode tables; validates a header.
// One workgroup each for the tables: the work is a few thousand symbols at most and sits on
// the critical path between the two streaming kernels, so it is latency- not
// bandwidth-bound.  Alphabets up to kBookLdsSyms live entirely in LDS.  Larger ones:
//   k_book_sort_tiles, k_book_merge  the leaves in (frequency, symbol) order, by as many
//                    workgroups as the alphabet has tiles of 1024 symbols (a merge sort:
//                    tiles sorted in registers, then runs merged by ranking, four per launch);
//                    k_codebook then builds the tree on the leaves' weights in LDS, or, where
//                    those do not fit, in global memory while many items wait and in LDS at the end.
//
// Length rule (must give exactly one answer): leaves ordered by (frequency,
// symbol); two queues; at every step the two smallest heads are merged, the leaf
// first when a leaf and an internal node weigh the same; internal nodes are
// consumed in creation order.
#include <type_traits>

#include "comet_kernels.h"
#include "comet_records.h"

namespace comet {

namespace {

// Ascending bitonic sort of n2 (power of two) 64-bit keys by the whole workgroup.
__device__ void bitonic_sort(uint64_t *keys, uint32_t n2) {
    for (uint32_t k = 2; k <= n2; k <<= 1) {
        for (uint32_t j = k >> 1; j > 0; j >>= 1) {
            for (uint32_t i = threadIdx.x; i < n2; i += blockDim.x) {
                const uint32_t p = i ^ j;
                if (p > i) {
                    const uint64_t x = keys[i], y = keys[p];
                    const bool asc = (i & k) == 0;
                    if ((x > y) == asc) { keys[i] = y; keys[p] = x; }
                }
            }
            __syncthreads();
        }
    }
}

// Value of lane (mine ^ J) of the wavefront, by data-parallel primitives (no LDS access): quad permutes, row
// rotation, and for 16 and 32 the row and half swaps, whose two results are the values of both partners.
template <int J> __device__ inline uint32_t lane_xor(uint32_t v) {
    if (J == 1) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0xB1, 0xf, 0xf, true);      // quad_perm:[1,0,3,2]
    if (J == 2) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x4E, 0xf, 0xf, true);      // quad_perm:[2,3,0,1]
    if (J == 4) {                                                                                   // ^3, then ^7
        const int t = __builtin_amdgcn_update_dpp(0, (int)v, 0x1B, 0xf, 0xf, true);                 // quad_perm:[3,2,1,0]
        return (uint32_t)__builtin_amdgcn_update_dpp(0, t, 0x141, 0xf, 0xf, true);                  // row_half_mirror
    }
    if (J == 8) return (uint32_t)__builtin_amdgcn_update_dpp(0, (int)v, 0x128, 0xf, 0xf, true);     // row_ror:8
    if (J == 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(v, v, false, false);
        return (lane_id() & 16) ? r[0] : r[1];
    }
    const auto r = __builtin_amdgcn_permlane32_swap(v, v, false, false);
    return (lane_id() & 32) ? r[0] : r[1];
}
template <int J> __device__ inline uint64_t lane_xor(uint64_t v) {
    return ((uint64_t)lane_xor<J>((uint32_t)(v >> 32)) << 32) | lane_xor<J>((uint32_t)v);
}
// One comparison of a sorting network with the partner J lanes away.
template <int J> __device__ inline uint64_t compare_exchange(uint64_t v, bool keep_min) {
    const uint64_t o = lane_xor<J>(v);
    return (v < o) == keep_min ? v : o;
}
// (32 bits: minimum, maximum and a selection by a mask that does not change, nothing through the scalar unit)
template <int J> __device__ inline uint32_t compare_exchange(uint32_t v, bool keep_min) {
    const uint32_t o = lane_xor<J>(v);
    const uint32_t lo = v < o ? v : o, hi = v < o ? o : v;
    return keep_min ? lo : hi;
}
// The lanes' values (a bitonic sequence) in ascending order, or descending.
template <typename T> __device__ inline T wave_merge(T v, uint32_t lane, bool ascending) {
    v = compare_exchange<32>(v, ((lane & 32u) == 0u) == ascending);
    v = compare_exchange<16>(v, ((lane & 16u) == 0u) == ascending);
    v = compare_exchange<8>(v, ((lane & 8u) == 0u) == ascending);
    v = compare_exchange<4>(v, ((lane & 4u) == 0u) == ascending);
    v = compare_exchange<2>(v, ((lane & 2u) == 0u) == ascending);
    v = compare_exchange<1>(v, ((lane & 1u) == 0u) == ascending);
    return v;
}

// Ascending bitonic sort by the whole workgroup of kBookBlock threads: thread i holds the keys i and, NK == 2,
// i + kBookBlock of the first n2 (a power of two, at least a wavefront).  Partners closer than a wavefront exchange by
// data-parallel primitives, the others through LDS (s_x: 2 * NK * kBookBlock keys, two buffers in turn, so that an
// exchange needs one barrier).  512 keys: 2.6 us; with shuffles through the LDS unit and two barriers 7.2.
template <int NK>
__device__ inline void block_sort(uint64_t (&key)[NK], uint64_t *s_x, uint32_t n2) {
    const uint32_t tid = threadIdx.x, lane = tid & (uint32_t)(kWave - 1);
    const bool mine = (tid & ~(uint32_t)(kWave - 1)) < n2;           // my wavefront holds keys (NK == 2: both or none)
    if (mine) {
#pragma unroll
        for (int v = 0; v < NK; ++v) {
            uint64_t k = key[v];
            const uint32_t i = lane;
            k = compare_exchange<1>(k, ((i & 2u) == 0u) == ((i & 1u) == 0u));
            k = compare_exchange<2>(k, ((i & 4u) == 0u) == ((i & 2u) == 0u));
            k = compare_exchange<1>(k, ((i & 4u) == 0u) == ((i & 1u) == 0u));
            k = compare_exchange<4>(k, ((i & 8u) == 0u) == ((i & 4u) == 0u));
            k = compare_exchange<2>(k, ((i & 8u) == 0u) == ((i & 2u) == 0u));
            k = compare_exchange<1>(k, ((i & 8u) == 0u) == ((i & 1u) == 0u));
            k = compare_exchange<8>(k, ((i & 16u) == 0u) == ((i & 8u) == 0u));
            k = compare_exchange<4>(k, ((i & 16u) == 0u) == ((i & 4u) == 0u));
            k = compare_exchange<2>(k, ((i & 16u) == 0u) == ((i & 2u) == 0u));
            k = compare_exchange<1>(k, ((i & 16u) == 0u) == ((i & 1u) == 0u));
            k = compare_exchange<16>(k, ((i & 32u) == 0u) == ((i & 16u) == 0u));
            k = compare_exchange<8>(k, ((i & 32u) == 0u) == ((i & 8u) == 0u));
            k = compare_exchange<4>(k, ((i & 32u) == 0u) == ((i & 4u) == 0u));
            k = compare_exchange<2>(k, ((i & 32u) == 0u) == ((i & 2u) == 0u));
            k = compare_exchange<1>(k, ((i & 32u) == 0u) == ((i & 1u) == 0u));
            key[v] = wave_merge(k, lane, n2 == (uint32_t)kWave || (tid & (uint32_t)kWave) == 0u);
        }
    }
    uint32_t flip = 0;
    for (uint32_t k = 2u * kWave; k <= n2; k <<= 1) {
        for (uint32_t j = k >> 1; j >= (uint32_t)kWave; j >>= 1) {
            if (NK == 2 && j == (uint32_t)kBookBlock) {              // (k == 2 * kBookBlock: ascending throughout)
                const uint64_t x = key[0], y = key[NK - 1];
                key[0] = x < y ? x : y;
                key[NK - 1] = x < y ? y : x;
                continue;
            }
            uint64_t *buf = s_x + flip * (uint32_t)(NK * kBookBlock);
            flip ^= 1u;
            if (mine) {
#pragma unroll
                for (int v = 0; v < NK; ++v) buf[v * kBookBlock + tid] = key[v];
            }
            __syncthreads();
            if (mine) {
#pragma unroll
                for (int v = 0; v < NK; ++v) {
                    const uint32_t i = v * (uint32_t)kBookBlock + tid;
                    const uint64_t o = buf[i ^ j];
                    const bool keep_min = ((i & k) == 0u) == ((i & j) == 0u);
                    key[v] = (key[v] < o) == keep_min ? key[v] : o;
                }
            }
        }
        if (mine) {
#pragma unroll
            for (int v = 0; v < NK; ++v) key[v] = wave_merge(key[v], lane, ((v * (uint32_t)kBookBlock + tid) & k) == 0u);
        }
    }
}

// arr[begin, end) is non-decreasing in (arr[i] >> shift); number of entries <= t
// (or < t when strict).  Gallops from the front: the answer is usually small.
__device__ inline uint32_t count_below(const uint64_t *arr, uint32_t begin, uint32_t end, uint64_t t, int shift, bool strict) {
    const uint32_t n = end - begin;
    uint32_t pos = 0, step = 1;
    auto ok = [&](uint32_t idx) { const uint64_t w = arr[begin + idx] >> shift; return strict ? (w < t) : (w <= t); };
    while (pos + step <= n && ok(pos + step - 1)) { pos += step; step <<= 1; }
    uint32_t lo = pos, hi = (pos + step - 1 < n) ? pos + step - 1 : n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (ok(mid)) lo = mid + 1; else hi = mid;
    }
    return lo;
}

__device__ inline uint32_t next_pow2(uint32_t v) {
    uint32_t p = 1;
    while (p < v) p <<= 1;
    return p;
}

// Value of lane `src` (wavefront-uniform).
__device__ inline uint32_t lane_value(uint32_t v, uint32_t src) { return (uint32_t)__builtin_amdgcn_readlane((int)v, (int)src); }
__device__ inline uint64_t lane_value(uint64_t v, uint32_t src) {
    const uint32_t lo = lane_value((uint32_t)v, src), hi = lane_value((uint32_t)(v >> 32), src);
    return ((uint64_t)hi << 32) | lo;
}

// Canonical first codes per length from the per-length symbol counts (cnt[1 .. 64]; 64 stands for
// every length the container cannot hold); returns false if the lengths are not a complete prefix
// code (or a single 1-bit code).  By one whole wavefront: every lane of it must call, the results
// are wavefront-uniform.  The first code of length L is (first code of L-1 + count of L-1) * 2,
// i.e. the sum over k < L of cnt[k] * 2^(L-k): lane L holds the count of length L and the first
// codes are an exclusive scan of the counts in units of 2^-57.  A table is a valid code exactly
// if no length above 57 is used, the Kraft sum does not exceed one, and it equals one unless the
// code has a single symbol (of length 1).
__device__ inline bool canonical_first_codes_wave(const uint32_t *cnt, uint32_t n_active, uint64_t *first_code,
                                                  uint32_t *first_index, uint32_t *max_len_out, uint32_t *min_len_out) {
    const uint32_t L = (uint32_t)lane_id();                  // lane 0 stands for no length; length 64 is looked at apart
    const uint32_t c = L ? cnt[L] : 0u;
    const uint32_t c64 = cnt[64];
    const uint64_t used = wave_ballot(c != 0u);
    // a count above 2^L alone breaks the Kraft inequality (and would overflow the sum below)
    const bool too_many = L && L < 17u && c > (1u << L);
    const bool too_long = (L > 57u && c != 0u);
    const bool broken = wave_ballot(too_many || too_long) != 0ull || c64 != 0u;
    const uint64_t term = (L && L <= 57u && !too_many) ? (uint64_t)c << (57u - L) : 0ull;
    const uint64_t incl = wave_incl_scan<uint64_t>(term);
    const uint32_t idx_incl = wave_incl_scan<uint32_t>(c);
    const uint64_t excl = incl - term;
    if (L) {
        first_code[L] = (L <= 57u) ? excl >> (57u - L) : excl << (L - 57u);
        first_index[L] = idx_incl - c;
    }
    const uint64_t kraft = lane_value(incl, 63);       // in units of 2^-57
    const uint32_t total = (uint32_t)__builtin_amdgcn_readlane((int)idx_incl, 63);
    if (L == 0u) { first_code[64] = lane_value(excl, 63) << 7; first_index[64] = total; }   // (length 64 is never valid)
    const uint32_t max_len = c64 ? 64u : (used ? 63u - (uint32_t)__builtin_clzll(used) : 0u);
    const uint32_t min_len = used ? (uint32_t)__builtin_ctzll(used) : (c64 ? 64u : 0u);
    bool ok = !broken && total + c64 == n_active && max_len != 0u && max_len <= 57u && kraft <= (1ull << 57);
    if (ok && n_active > 1u && kraft != (1ull << 57)) ok = false;
    if (ok && n_active == 1u && max_len != 1u) ok = false;
    *max_len_out = max_len;
    *min_len_out = min_len;
    return ok;
}

}  // namespace


// The merge rounds.
//
// State: leaves [li, m) and internal nodes [ii, ni) not yet merged.  With t the sum
// of the two smallest heads, every new node weighs at least t, so every waiting item
// of weight <= t is merged before any node created now: those items, taken in merged
// order (leaf before node on equal weight) and paired consecutively, are exactly the
// next steps of the sequential two-queue construction.  An odd item out waits for the
// next round.  iw[0, m) must be zero on entry.
//
// Entries of arr[begin, end) with (arr[i] >> shift) <= t, by one whole wavefront probing 64 consecutive ones per step
// (the entries are sorted, so the lanes that pass form a prefix).
__device__ inline uint32_t count_below_wave(const uint64_t *arr, uint32_t begin, uint32_t end, uint64_t t, int shift) {
    uint32_t cnt = 0;
    const uint32_t lane = (uint32_t)lane_id();
    while (true) {
        const uint32_t idx = begin + cnt + lane;
        const bool ok = idx < end && (arr[idx] >> shift) <= t;
        const uint64_t mask = __ballot(ok);
        const uint32_t c = (~mask == 0ull) ? 64u : (uint32_t)(__ffsll((unsigned long long)~mask) - 1);
        cnt += c;
        if (c < 64u) break;
    }
    return cnt;
}

// The same count by a whole workgroup of kBookBlock threads (every thread must call; arrays in global memory):
// every thread probes one entry per step, kBookBlock entries evenly spread over what is left of the range, so
// two steps (two memory round trips) settle a range of a million entries, where the galloping search of one
// thread takes two dependent loads per bit of the answer.
__device__ inline uint32_t count_below_block(const uint64_t *arr, uint32_t begin, uint32_t end, uint64_t t, int shift) {
    uint32_t lo = begin, hi = end;                   // the first entry above t lies in [lo, hi]
    while (true) {
        const uint32_t n = hi - lo;
        if (n == 0u) return lo - begin;
        const uint32_t stride = (n + (uint32_t)kBookBlock - 1u) / (uint32_t)kBookBlock;
        const uint32_t p = lo + (threadIdx.x + 1u) * stride - 1u;         // my probe: the last entry of my piece
        const bool ok = p < hi && (arr[p] >> shift) <= t;                 // (the probes that pass are the first ones)
        const uint32_t c = (uint32_t)__syncthreads_count(ok ? 1 : 0);
        const uint32_t new_lo = lo + c * stride;
        if (stride == 1u) return new_lo - begin;
        const uint32_t next_probe = new_lo + stride - 1u;                 // the first probe that failed, or beyond the range
        hi = next_probe < hi ? next_probe : hi;
        lo = new_lo;
    }
}

// One round, control part: how many leaves (nl) and internal nodes (nn) are merged now.  Uniform
// over the callers.  BLOCK: the counts are taken by the whole workgroup (every thread of it calls), else
// by a whole wavefront probing 64 entries per step.
template <bool BLOCK>
__device__ inline void round_control(const uint64_t *keys, const uint64_t *iw, uint32_t m, uint32_t li, uint32_t ii, uint32_t ni,
                                     uint32_t *nl_out, uint32_t *nn_out) {
    const uint64_t inf = ~0ull;
    const uint64_t a0 = li < m ? keys[li] >> 16 : inf, a1 = li + 1 < m ? keys[li + 1] >> 16 : inf;
    const uint64_t b0 = ii < ni ? iw[ii] : inf, b1 = ii + 1 < ni ? iw[ii + 1] : inf;
    uint64_t s0, s1;
    if (a0 <= b0) { s0 = a0; s1 = (a1 <= b0) ? a1 : b0; }
    else { s0 = b0; s1 = (a0 <= b1) ? a0 : b1; }
    const uint64_t t = s0 + s1;
    uint32_t nl = BLOCK ? count_below_block(keys, li, m, t, 16) : count_below_wave(keys, li, m, t, 16);
    uint32_t nn = BLOCK ? count_below_block(iw, ii, ni, t, 0) : count_below_wave(iw, ii, ni, t, 0);
    if ((nl + nn) & 1u) {
        const uint64_t la = nl ? keys[li + nl - 1] >> 16 : 0, lb = nn ? iw[ii + nn - 1] : 0;
        if (nn && (!nl || la <= lb)) --nn; else --nl;
    }
    *nl_out = nl; *nn_out = nn;
}

// One round, the items: lane `lane` of `nlanes` takes every nlanes-th of the nl + nn items.
// ITEMS: items a lane works on side by side (arrays in global memory: every item is a chain of dependent loads).
template <uint32_t ITEMS = 1>
__device__ inline void round_items(const uint64_t *keys, uint64_t *iw, uint32_t *leaf_parent, uint32_t *int_parent,
                                   uint32_t li, uint32_t ii, uint32_t ni, uint32_t nl, uint32_t nn, uint32_t lane, uint32_t nlanes) {
    if (ITEMS > 1) {
        for (uint32_t idx0 = lane; idx0 < nl + nn; idx0 += ITEMS * nlanes) {
            uint64_t w[ITEMS];
            bool on[ITEMS], leaf[ITEMS];
            // the item's weight, then its rank among the items of the other kind (both loops: ITEMS loads in flight)
#pragma unroll
            for (uint32_t k = 0; k < ITEMS; ++k) {
                const uint32_t idx = idx0 + k * nlanes;
                on[k] = idx < nl + nn;
                leaf[k] = idx < nl;
                w[k] = !on[k] ? 0ull : (leaf[k] ? keys[li + idx] >> 16 : iw[ii + (idx - nl)]);
            }
            uint32_t rank[ITEMS];
#pragma unroll
            for (uint32_t k = 0; k < ITEMS; ++k) {
                const uint32_t idx = idx0 + k * nlanes;
                rank[k] = 0;
                if (on[k]) rank[k] = leaf[k] ? idx + count_below(iw, ii, ii + nn, w[k], 0, true)
                                             : (idx - nl) + count_below(keys, li, li + nl, w[k], 16, false);
            }
#pragma unroll
            for (uint32_t k = 0; k < ITEMS; ++k) {
                const uint32_t idx = idx0 + k * nlanes;
                if (on[k]) {
                    if (leaf[k]) leaf_parent[li + idx] = ni + (rank[k] >> 1);
                    else int_parent[ii + (idx - nl)] = ni + (rank[k] >> 1);
                    atomicAdd(reinterpret_cast<unsigned long long *>(&iw[ni + (rank[k] >> 1)]), (unsigned long long)w[k]);
                }
            }
        }
        return;
    }
    for (uint32_t idx = lane; idx < nl + nn; idx += nlanes) {
        uint64_t w;
        uint32_t rank;
        if (idx < nl) {
            w = keys[li + idx] >> 16;
            rank = idx + count_below(iw, ii, ii + nn, w, 0, true);
            leaf_parent[li + idx] = ni + (rank >> 1);
        } else {
            const uint32_t b = idx - nl;
            w = iw[ii + b];
            rank = b + count_below(keys, li, li + nl, w, 16, false);
            int_parent[ii + b] = ni + (rank >> 1);
        }
        atomicAdd(reinterpret_cast<unsigned long long *>(&iw[ni + (rank >> 1)]), (unsigned long long)w);
    }
}

// Rounds by the whole workgroup while more than `stop` items wait; the state is handed back.
__device__ inline void huffman_rounds(const uint64_t *keys, uint64_t *iw, uint32_t *leaf_parent, uint32_t *int_parent,
                                      uint32_t m, uint32_t stop, uint32_t &li, uint32_t &ii, uint32_t &ni) {
    li = 0; ii = 0; ni = 0;
    while ((m - li) + (ni - ii) > stop) {
        uint32_t nl, nn;
        round_control<true>(keys, iw, m, li, ii, ni, &nl, &nn);
        round_items<4u>(keys, iw, leaf_parent, int_parent, li, ii, ni, nl, nn, threadIdx.x, (uint32_t)kBookBlock);
        __syncthreads();
        li += nl; ii += nn; ni += (nl + nn) >> 1;
    }
}

// The same rounds for arrays in LDS, by the whole workgroup.  The first wavefront runs the rounds of
// at most 64 items alone and in registers: lane l holds the l-th waiting leaf and the l-th waiting
// node, the counts of a round are two ballots (the queues are sorted, so the items merged now are
// a prefix of each), and the merged order of the items comes from a short counting loop or from
// one bitonic merge across the lanes instead of a binary search in LDS per item.  A round with more items is shared by all
// wavefronts through the general routines (every wavefront works out the round's counts for
// itself).  state: three words of LDS.  n_wait: nodes that wait already, iw[0, n_wait) (a
// construction that was begun elsewhere); iw beyond them must be zero on entry.
__device__ inline void huffman_rounds_lds(const uint64_t *keys, uint64_t *iw, uint32_t *leaf_parent, uint32_t *int_parent,
                                          uint32_t m, uint32_t tid, uint32_t nthreads, uint32_t *state, uint32_t n_wait = 0) {
    uint32_t li = 0, ii = 0, ni = n_wait;
    const uint32_t lane = tid & (uint32_t)(kWave - 1);
    const uint64_t inf = ~0ull;
    while (true) {
        if (tid < (uint32_t)kWave) {
            while ((m - li) + (ni - ii) > 1u) {
                const uint64_t A = li + lane < m ? keys[li + lane] >> 16 : inf;      // waiting leaves
                const uint64_t B = ii + lane < ni ? iw[ii + lane] : inf;             // waiting nodes
                const uint64_t a0 = lane_value(A, 0), a1 = lane_value(A, 1), b0 = lane_value(B, 0), b1 = lane_value(B, 1);
                uint64_t s0, s1;
                if (a0 <= b0) { s0 = a0; s1 = (a1 <= b0) ? a1 : b0; }
                else { s0 = b0; s1 = (a0 <= b1) ? a0 : b1; }
                const uint64_t t = s0 + s1;
                uint32_t nl = (uint32_t)__popcll(wave_ballot(A != inf && A <= t));
                uint32_t nn = (uint32_t)__popcll(wave_ballot(B != inf && B <= t));
                if (nl == (uint32_t)kWave || nn == (uint32_t)kWave) break;   // there may be more beyond the window: everybody's round
                if ((nl + nn) & 1u) {
                    const uint64_t la = nl ? lane_value(A, nl - 1u) : 0, lb = nn ? lane_value(B, nn - 1u) : 0;
                    if (nn && (!nl || la <= lb)) --nn; else --nl;
                }
                if (nl + nn > (uint32_t)kWave) break;        // more items than lanes: everybody's round
                if ((nl < nn ? nl : nn) <= 8u) {
                    // A short queue: an item's rank in the other queue is counted in a loop over the shorter
                    // one (one broadcast and one comparison per step): my leaf counts the merged nodes lighter
                    // than it, my node the merged leaves not heavier than it.
                    uint32_t before_leaf = 0, before_node = 0;
                    if (nn <= nl) {
                        for (uint32_t k = 0; k < nn; ++k) {
                            const uint64_t bk = lane_value(B, k);
                            before_leaf += (bk < A) ? 1u : 0u;
                            const uint32_t c = (uint32_t)__popcll(wave_ballot(lane < nl && A <= bk));
                            before_node = (lane == k) ? c : before_node;
                        }
                    } else {
                        for (uint32_t k = 0; k < nl; ++k) {
                            const uint64_t ak = lane_value(A, k);
                            before_node += (ak <= B) ? 1u : 0u;
                            const uint32_t c = (uint32_t)__popcll(wave_ballot(lane < nn && B < ak));
                            before_leaf = (lane == k) ? c : before_leaf;
                        }
                    }
                    if (lane < nl) {
                        const uint32_t parent = ni + ((lane + before_leaf) >> 1);
                        leaf_parent[li + lane] = parent;
                        atomicAdd(reinterpret_cast<unsigned long long *>(&iw[parent]), (unsigned long long)A);
                    }
                    if (lane < nn) {
                        const uint32_t parent = ni + ((lane + before_node) >> 1);
                        int_parent[ii + lane] = parent;
                        atomicAdd(reinterpret_cast<unsigned long long *>(&iw[parent]), (unsigned long long)B);
                    }
                } else {
                    // Merged order of the round's items: the leaves ascending from lane 0, the nodes descending
                    // from lane 63 and infinity between them are a bitonic sequence, which six compare-exchange
                    // steps sort.  Key = (weight, node after leaf, position in its queue): the order of the
                    // sequential construction, and no two keys are equal (weights stay below 2^57: at most
                    // 65536 counts of 32 bits).
                    const uint64_t Brev = __shfl(B, (int)(kWave - 1u - lane), kWave);
                    uint64_t key = inf;
                    if (lane < nl) key = (A << 7) | lane;
                    else if ((uint32_t)kWave - 1u - lane < nn) key = (Brev << 7) | 64u | ((uint32_t)kWave - 1u - lane);
#pragma unroll
                    for (uint32_t j = kWave / 2; j > 0; j >>= 1) {
                        const uint64_t other = __shfl_xor(key, (int)j, kWave);
                        const uint64_t lo = key < other ? key : other, hi = key < other ? other : key;
                        key = (lane & j) ? hi : lo;
                    }
                    // lane r now holds the item of rank r: items 2j and 2j+1 become node ni + j
                    const uint64_t w = key >> 7;
                    const uint64_t w_next = __shfl_xor(w, 1, kWave);
                    if (lane < nl + nn) {
                        const uint32_t parent = ni + (lane >> 1);
                        const uint32_t pos = (uint32_t)key & 63u;
                        if (key & 64u) int_parent[ii + pos] = parent;
                        else leaf_parent[li + pos] = parent;
                        if ((lane & 1u) == 0u) iw[parent] = w + w_next;
                    }
                }
                __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "workgroup");
                __builtin_amdgcn_wave_barrier();
                li += nl; ii += nn; ni += (nl + nn) >> 1;
            }
            if (lane == 0) { state[0] = li; state[1] = ii; state[2] = ni; }
        }
        __syncthreads();
        li = state[0]; ii = state[1]; ni = state[2];
        if ((m - li) + (ni - ii) <= 1u) break;
        uint32_t nl, nn;
        round_control<false>(keys, iw, m, li, ii, ni, &nl, &nn);
        round_items(keys, iw, leaf_parent, int_parent, li, ii, ni, nl, nn, tid, nthreads);
        __syncthreads();
        li += nl; ii += nn; ni += (nl + nn) >> 1;
    }
}

// The merge rounds of an alphabet that fits LDS, by one wavefront.  A round looks at the 64 lightest waiting items: lane
// l holds the l-th waiting leaf and the (63 - l)-th waiting node, and the smaller of the two values is one of the 64
// lightest (a bitonic sequence), which six compare-exchange steps put into merged order.  A key is (weight, node after
// leaf): of equal keys the one earlier in its queue comes first whatever the network does with them, because only its
// kind is read off the key and its place in its queue is the number of items of that kind in front of it.  With t the
// sum of the two lightest, the items of weight <= t, or the first 64 of them, are the next steps of the sequential
// construction (a node created now weighs t at least); an odd one out waits.
// W: 32-bit keys as long as all weights together stay below 2^31 - 1, else 64-bit ones.
// leafw: the leaves' keys in order, 64 keys of all ones behind the last; nodew: all ones on entry.  About 0.2 us a round
// (0.8 with the merged order from a loop over the shorter queue and the weights added up atomically).
// parent: of leaf i at i, of node i at kBookLdsSyms + i, of nobody at 2 * kBookLdsSyms + 0 .. 63; every lane writes in every
// round, those that merge nothing to a place of their own (switching the execution mask costs more).
template <typename W>
__device__ inline void huffman_rounds_wave(const W *leafw, W *nodew, uint16_t *parent, uint32_t m, uint32_t lane) {
    uint32_t li = 0, ii = 0, ni = 0;
    const uint32_t nobody = 2u * kBookLdsSyms + lane;
    while (ni + 1u < m) {
        const W a = leafw[li + lane], b = nodew[ii + (uint32_t)kWave - 1u - lane];
        const W key = wave_merge<W>(a < b ? a : b, lane, true);
        const W two = (lane_value(key, 0) | (W)1u) + (lane_value(key, 1) & ~(W)1u);        // (key of a node that weighs both)
        const uint32_t cnt = (uint32_t)__popcll(wave_ballot(key <= two)) & ~1u;
        const bool taken = lane < cnt, node = (key & (W)1u) != 0u;
        const uint64_t nodes = wave_ballot(node) & (cnt < (uint32_t)kWave ? (1ull << cnt) - 1ull : ~0ull);
        const uint32_t before = __builtin_amdgcn_mbcnt_hi((uint32_t)(nodes >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)nodes, 0u));
        const uint32_t nn = (uint32_t)__popcll(nodes), up = ni + (lane >> 1);
        const W other = lane_xor<1>(key);
        // (lanes that make no node write all ones where nodes to come are all ones already)
        nodew[(taken && (lane & 1u) == 0u) ? up : kBookLdsSyms] = (taken && (lane & 1u) == 0u) ? (key | (W)1u) + (other & ~(W)1u) : ~(W)0;
        parent[taken ? (node ? kBookLdsSyms + ii + before : li + lane - before) : nobody] = (uint16_t)up;
        __builtin_amdgcn_wave_barrier();                     // (a wavefront's LDS accesses happen in order: nothing to wait for)
        li += cnt - nn; ii += nn; ni += cnt >> 1;
    }
}

// LDS of k_codebook: one piece, used in turn for what follows.
constexpr uint32_t kBookPad = kBookLdsSyms + (uint32_t)kWave;
struct BookLds {
    // by construction: sort exchange (two buffers of 2 * kBookBlock keys), then the leaves' and the nodes' keys
    union {
        uint64_t exchange[4 * kBookBlock];
        struct { uint64_t leafw[kBookPad], nodew[kBookPad]; } q;
        struct { uint16_t sym[kBookBySymbolMax]; uint8_t depth[kBookBySymbolMax]; } given;      // code book reuse: up to kBookBySymbolMax symbols
        struct { uint64_t keys[kBookLdsSyms], iw[kBookLdsSyms]; } large;                        // construction in global memory, its last rounds
    } u;
    union {
        struct { uint16_t parent[2 * kBookLdsSyms + kWave], order[kBookLdsSyms]; } t;
        struct { uint32_t lp[kBookLdsSyms], ip[kBookLdsSyms]; } large;
        uint32_t wc[(kBookBlock / kWave) * 64 + 65];         // canonical order: symbols per (wavefront, length), and per length so far
    } v;
    uint16_t sym[kBookLdsSyms];       // the symbols that occur, ascending
    uint8_t depth[kBookLdsSyms];      // their code lengths
    uint32_t cnt[65];                 // symbols per length
    uint64_t first[65];
    uint32_t findex[65];
    uint32_t part[kBookBlock / kWave];
    uint32_t word[4];
    uint64_t total[3];                // records, non-zero inputs, verbatim records of the tensor
};
static_assert(sizeof(BookLds) <= kBookLdsBytes, "dynamic LDS");

// Canonical codes of the symbols sym[0, m) (ascending) from their lengths: the code of a symbol is the first code of its
// length plus the number of smaller symbols of the same length (per wavefront the lanes of one length are found with a
// ballot per length that occurs, then a prefix over the wavefronts in front).  sym == nullptr: every symbol of the
// alphabet (m of them), length 0 if it does not occur.
__device__ inline void book_codes(const BookArgs &a, const uint16_t *syms, const uint8_t *depths, uint32_t m, const uint64_t *first, uint32_t *s_wc) {
    const uint32_t tid = threadIdx.x, lane = tid & (uint32_t)(kWave - 1), wave = tid / (uint32_t)kWave;
    constexpr uint32_t kWaves = kBookBlock / kWave;
    uint32_t *s_run = s_wc + kWaves * 64u;                   // symbols per length in front of the current 1024 symbols
    for (uint32_t i = tid; i < 65u; i += kBookBlock) s_run[i] = 0;
    for (uint32_t base = 0; base < m; base += kBookBlock) {
        for (uint32_t i = tid; i < kWaves * 64u; i += kBookBlock) s_wc[i] = 0;
        __syncthreads();
        const uint32_t at = base + tid;
        const uint32_t L = (at < m) ? depths[at] : 0u;
        uint32_t in_wave = 0;
        uint64_t todo = wave_ballot(L != 0u);
        while (todo) {                                       // one step per length that occurs in the wavefront
            const uint32_t Lc = (uint32_t)__builtin_amdgcn_readlane((int)L, __builtin_ctzll(todo));
            const uint64_t same = wave_ballot(L == Lc);
            if (L == Lc) in_wave = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
            if (lane == 0) s_wc[wave * 64u + (Lc & 63u)] = (uint32_t)__popcll(same);
            todo &= ~same;
        }
        __syncthreads();
        if (L) {
            uint32_t before = s_run[L & 63u];
            for (uint32_t w = 0; w < wave; ++w) before += s_wc[w * 64u + (L & 63u)];
            const uint64_t code = first[L] + before + in_wave;
            const uint32_t sym = syms ? syms[at] : at;
            a.len_out[sym] = (uint8_t)L;
            a.enc[sym] = (code << 6) | (uint64_t)(L & 63u);
            if (a.code_out) a.code_out[sym] = code;
        }
        if (base + kBookBlock >= m) break;
        __syncthreads();
        if (tid < 64u) {
            uint32_t add = 0;
            for (uint32_t w = 0; w < kWaves; ++w) add += s_wc[w * 64u + tid];
            s_run[tid] += add;
        }
        __syncthreads();                                     // the counts are cleared for the next 1024 symbols
    }
}

// First codes per length from the counts s.cnt; a table that is no complete prefix code raises a status bit.
__device__ inline void book_first_codes(const BookArgs &a, BookLds &s, uint32_t m, bool given) {
    if (threadIdx.x < (uint32_t)kWave) {
        uint32_t mx = 0, mn;
        const bool ok = (m == 0 && !given) || (m != 0 && canonical_first_codes_wave(s.cnt, m, s.first, s.findex, &mx, &mn));
        if (threadIdx.x == 0) {
            s.word[2] = mx;
            if (!ok) atomicOr(&a.ctl->status, given ? (uint32_t)ST_CODEBOOK : (uint32_t)ST_INTERNAL);   // a given table must be a complete code
        }
    }
    __syncthreads();
}

// The tensor's record counts, a wavefront each (the second to the fourth, while the first one builds the tree).
__device__ inline void book_totals(const RecordArgs &recs, BookLds &s) {
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / (uint32_t)kWave)), lane = (uint32_t)lane_id();
    if (recs.n_wg && wave >= 1u && wave <= 3u) {
        const uint64_t total = record_total(recs, wave - 1u, lane);
        if (lane == 0) s.total[wave - 1u] = total;
    }
}

// The code lengths (s.depth, s.cnt) of m <= kBookLdsSyms symbols: thread i holds the i-th and, n_keys == 2, the
// (i + kBookBlock)-th (frequency, place in s.sym) key in order; all ones behind the last.
template <typename W>
__device__ inline void book_tree(BookLds &s, const RecordArgs &recs, uint32_t m, const uint64_t (&key)[2], uint32_t n_keys) {
    const uint32_t tid = threadIdx.x;
    // ---- leaves in order, waiting; no nodes yet ----
    W *leafw = reinterpret_cast<W *>(s.u.q.leafw), *nodew = reinterpret_cast<W *>(s.u.q.nodew);
    __syncthreads();                                         // the exchange buffers of the sort are free
#pragma unroll
    for (uint32_t v = 0; v < 2; ++v) {
        const uint32_t i = tid + v * kBookBlock;
        const bool on = i < m;
        if (on) s.v.t.order[i] = (uint16_t)(key[v] & 0xffffu);
        if (v < n_keys && i < m + (uint32_t)kWave) leafw[i] = on ? (W)((key[v] >> 16) << 1) : ~(W)0;
    }
    for (uint32_t i = n_keys * kBookBlock + tid; i < m + (uint32_t)kWave; i += kBookBlock) leafw[i] = ~(W)0;
    for (uint32_t i = tid; i < m + (uint32_t)kWave; i += kBookBlock) nodew[i] = ~(W)0;
    __syncthreads();
    if (tid < (uint32_t)kWave) huffman_rounds_wave<W>(leafw, nodew, s.v.t.parent, m, tid);
    else book_totals(recs, s);
    __syncthreads();
    // ---- depth of every leaf: walk to the root (node m - 2) ----
    for (uint32_t i = tid; i < m; i += kBookBlock) {
        uint32_t depth = 1;
        if (m >= 2) {
            const uint16_t *node_parent = s.v.t.parent + kBookLdsSyms;
            for (uint32_t p = s.v.t.parent[i]; p != m - 2u && depth < 64u; p = node_parent[p]) ++depth;
        }
        s.depth[s.v.t.order[i]] = (uint8_t)depth;
        atomicAdd(&s.cnt[depth], 1u);
    }
    __syncthreads();
}

// The rounds of a tree in global memory while more than `stop` items wait, by the whole workgroup, with the round's items in
// LDS: the next kBookWin leaves and nodes come in with one memory round trip, the threads count those of weight <= t in
// registers, ranks are searched in LDS, and the new nodes' weights are sums of neighbours in merged order, stored in a
// row.  32-bit weights: all of them together stay below 2^31.  A round that takes a whole window (thousands of leaves of one
// weight, as the first rounds of a heavy-tailed alphabet have) goes through the general routines.  About 4.5 us a round
// instead of 8 (searches for the counts and the ranks in global memory, atomic additions).
constexpr uint32_t kBookWin = 2u * (uint32_t)kBookBlock;
__device__ inline void huffman_rounds_window(const uint64_t *keys, uint64_t *iw, uint32_t *leaf_parent, uint32_t *int_parent,
                                             uint32_t m, uint32_t *s_x, uint32_t *s_part, uint32_t stop,
                                             uint32_t &li, uint32_t &ii, uint32_t &ni) {
    const uint32_t tid = threadIdx.x, lane = tid & (uint32_t)(kWave - 1), wave = tid / (uint32_t)kWave;
    uint32_t *leaf = s_x, *node = s_x + kBookWin, *merged = s_x + 2u * kBookWin;
    auto below = [](const uint32_t *arr, uint32_t n, uint32_t w, uint32_t or_equal) -> uint32_t {     // entries < w + or_equal
        uint32_t lo = 0, hi = n;
        const uint32_t lim = w + or_equal;
        while (lo < hi) {
            const uint32_t mid = (lo + hi) >> 1;
            if (arr[mid] < lim) lo = mid + 1u; else hi = mid;
        }
        return lo;
    };
    li = 0; ii = 0; ni = 0;
    while ((m - li) + (ni - ii) > stop) {
        uint32_t a[2], b[2];
#pragma unroll
        for (uint32_t v = 0; v < 2; ++v) {
            const uint32_t i = tid + v * (uint32_t)kBookBlock;
            a[v] = li + i < m ? (uint32_t)(keys[li + i] >> 16) : ~0u;
            b[v] = ii + i < ni ? (uint32_t)iw[ii + i] : ~0u;
        }
#pragma unroll
        for (uint32_t v = 0; v < 2; ++v) {
            leaf[tid + v * (uint32_t)kBookBlock] = a[v];
            node[tid + v * (uint32_t)kBookBlock] = b[v];
        }
        __syncthreads();
        const uint32_t a0 = leaf[0], a1 = leaf[1], b0 = node[0], b1 = node[1];
        const uint32_t t = a0 <= b0 ? a0 + (a1 <= b0 ? a1 : b0) : b0 + (a0 <= b1 ? a0 : b1);      // the two lightest (they exist)
        const uint32_t ca = (uint32_t)__popcll(wave_ballot(a[0] <= t)) + (uint32_t)__popcll(wave_ballot(a[1] <= t));
        const uint32_t cb = (uint32_t)__popcll(wave_ballot(b[0] <= t)) + (uint32_t)__popcll(wave_ballot(b[1] <= t));
        if (lane == 0) s_part[wave] = ca | (cb << 16);
        __syncthreads();
        uint32_t both = 0;
#pragma unroll
        for (uint32_t w = 0; w < (uint32_t)(kBookBlock / kWave); ++w) both += s_part[w];
        uint32_t nl = both & 0xffffu, nn = both >> 16;
        if (nl == kBookWin || nn == kBookWin) {              // (uniform) perhaps more than the window shows
            round_control<true>(keys, iw, m, li, ii, ni, &nl, &nn);
            round_items<4u>(keys, iw, leaf_parent, int_parent, li, ii, ni, nl, nn, tid, (uint32_t)kBookBlock);
        } else {
            if ((nl + nn) & 1u) {
                const uint32_t la = nl ? leaf[nl - 1u] : 0u, lb = nn ? node[nn - 1u] : 0u;
                if (nn && (!nl || la <= lb)) --nn; else --nl;
            }
#pragma unroll
            for (uint32_t v = 0; v < 2; ++v) {
                const uint32_t i = tid + v * (uint32_t)kBookBlock;
                if (i < nl) {
                    const uint32_t rank = i + below(node, nn, a[v], 0u);
                    merged[rank] = a[v];
                    leaf_parent[li + i] = ni + (rank >> 1);
                }
                if (i < nn) {
                    const uint32_t rank = i + below(leaf, nl, b[v], 1u);
                    merged[rank] = b[v];
                    int_parent[ii + i] = ni + (rank >> 1);
                }
            }
            __syncthreads();
            for (uint32_t k = tid; k < (nl + nn) >> 1; k += (uint32_t)kBookBlock) iw[ni + k] = (uint64_t)merged[2u * k] + merged[2u * k + 1u];
        }
        __syncthreads();
        li += nl; ii += nn; ni += (nl + nn) >> 1;
    }
}

// Entries of w[lo, hi), sorted ascending, that are <= t; by every wavefront for itself, 64 probes at a time.
__device__ inline uint32_t count_le_wave(const uint32_t *w, uint32_t lo, uint32_t hi, uint32_t t, uint32_t lane) {
    const uint32_t begin = lo;
    while (lo < hi) {
        const uint32_t stride = (hi - lo + (uint32_t)kWave - 1u) / (uint32_t)kWave;
        const uint32_t p = lo + (lane + 1u) * stride - 1u;                // (the probes that pass are the first ones)
        const uint32_t c = (uint32_t)__popcll(wave_ballot(p < hi && w[p] <= t));
        lo += c * stride;
        if (stride == 1u) break;
        hi = lo + stride - 1u < hi ? lo + stride - 1u : hi;
    }
    return lo - begin;
}

// All rounds of a tree with the weights of m <= kBookLdsLeaves presorted leaves in LDS, by the whole workgroup: w[i] is the weight of
// leaf i until it is merged, and w[k] that of node k from then on.  (Two items make a node, so node k is made after leaf k has been
// merged: the nodes never need a place that a waiting leaf has.)  A round takes the items of weight <= t, or the first kRoundItems of
// them in merged order: thread by thread the new nodes find their two items by a search along the diagonal of both queues (the
// merge-path method of Odeh, Green, Mwassi, Shmueli and Birk, 2012), and
// their weights are stored once everybody has read.  Weights of all leaves together: below 2^31.
// Bound by the latency of the searches in LDS, about 1.5 us a round; 26 000 symbols take 26 rounds.  With the queues in global
// memory (huffman_rounds_window) a round took 5 to 15 us: the queues' next items and the new nodes went through L2.
constexpr uint32_t kRoundNodes = 4;                          // new nodes per thread and round
constexpr uint32_t kRoundItems = 2u * kRoundNodes * (uint32_t)kBookBlock;
__device__ inline void huffman_rounds_weights(const uint64_t *keys, uint32_t *w, uint32_t *leaf_parent, uint32_t *int_parent, uint32_t m) {
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id();
    for (uint32_t i0 = tid; i0 < m; i0 += 8u * (uint32_t)kBookBlock) {
        uint64_t k[8];
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j) k[j] = i0 + j * (uint32_t)kBookBlock < m ? keys[i0 + j * (uint32_t)kBookBlock] : 0ull;
#pragma unroll
        for (uint32_t j = 0; j < 8u; ++j)
            if (i0 + j * (uint32_t)kBookBlock < m) w[i0 + j * (uint32_t)kBookBlock] = (uint32_t)(k[j] >> 16);
    }
    lds_barrier();
    uint32_t li = 0, ii = 0, ni = 0;                         // leaves and nodes merged so far, nodes made so far
    while ((m - li) + (ni - ii) > 1u) {
        const uint32_t a0 = li < m ? w[li] : ~0u, a1 = li + 1u < m ? w[li + 1u] : ~0u;
        const uint32_t b0 = ii < ni ? w[ii] : ~0u, b1 = ii + 1u < ni ? w[ii + 1u] : ~0u;
        const uint32_t t = (uint32_t)__builtin_amdgcn_readfirstlane((int)(a0 <= b0 ? a0 + (a1 <= b0 ? a1 : b0) : b0 + (a0 <= b1 ? a0 : b1)));      // the two lightest (they exist)
        uint32_t nl = count_le_wave(w, li, m - li < kRoundItems ? m : li + kRoundItems, t, lane);
        uint32_t nn = count_le_wave(w, ii, ni - ii < kRoundItems ? ni : ii + kRoundItems, t, lane);
        uint32_t items = nl + nn;
        items = items < kRoundItems ? items & ~1u : kRoundItems;          // (an odd one out waits)
        const uint32_t nodes = items / 2u;
        // leaves among the first `diag` items in merged order (a leaf before a node of the same weight)
        uint32_t lo[kRoundNodes], hi[kRoundNodes], sum[kRoundNodes], longest = nl < nn ? nl : nn;
#pragma unroll
        for (uint32_t v = 0; v < kRoundNodes; ++v) {
            const uint32_t diag = 2u * (v * (uint32_t)kBookBlock + tid);
            lo[v] = diag > nn ? diag - nn : 0u;
            hi[v] = diag < nl ? diag : nl;
            if (diag >= items) hi[v] = lo[v];
        }
        for (; longest; longest >>= 1) {
#pragma unroll
            for (uint32_t v = 0; v < kRoundNodes; ++v) {
                if (v * (uint32_t)kBookBlock >= nodes) break;             // (uniform)
                const uint32_t diag = 2u * (v * (uint32_t)kBookBlock + tid);
                const uint32_t mid = (lo[v] + hi[v]) >> 1;
                const bool on = lo[v] < hi[v];
                const bool leaf = on && w[li + mid] <= w[ii + diag - 1u - mid];
                lo[v] = leaf ? mid + 1u : lo[v];
                hi[v] = on && !leaf ? mid : hi[v];
            }
        }
#pragma unroll
        for (uint32_t v = 0; v < kRoundNodes; ++v) {
            sum[v] = 0;
            const uint32_t k = v * (uint32_t)kBookBlock + tid;
            if (k < nodes) {
                uint32_t i = lo[v], j = 2u * k - lo[v];
#pragma unroll
                for (uint32_t two = 0; two < 2u; ++two) {
                    const uint32_t x = i < nl ? w[li + i] : ~0u, y = j < nn ? w[ii + j] : ~0u;
                    const bool leaf = i < nl && (j >= nn || x <= y);
                    if (leaf) leaf_parent[li + i] = ni + k; else int_parent[ii + j] = ni + k;
                    sum[v] += leaf ? x : y;
                    i += leaf ? 1u : 0u;
                    j += leaf ? 0u : 1u;
                }
                if (k + 1u == nodes) { w[m] = i; }           // (leaves merged in this round, for everybody)
            }
        }
        lds_barrier();
        const uint32_t took = (uint32_t)__builtin_amdgcn_readfirstlane((int)w[m]);
#pragma unroll
        for (uint32_t v = 0; v < kRoundNodes; ++v) {
            const uint32_t k = v * (uint32_t)kBookBlock + tid;
            if (k < nodes) w[ni + k] = sum[v];
        }
        lds_barrier();
        li += took; ii += items - took; ni += nodes;
    }
    __syncthreads();
}

// More symbols than fit LDS, built from the histogram in global memory; keys[0, m): the leaves in order if presorted.
__device__ inline void book_large(const BookArgs &a, BookLds &s, uint32_t m) {
    const uint32_t tid = threadIdx.x;
    const uint32_t nbins = a.nbins;
    uint64_t *keys = a.scratch.keys, *iw = a.scratch.iw;
    uint32_t *leaf_parent = a.scratch.leaf_parent, *int_parent = a.scratch.int_parent;
    book_totals(a.recs, s);
    // ---- 1. the symbols that occur as sort keys (frequency << 16 | symbol), unless the sort kernels have done that ----
    if (!a.presorted) {
        __syncthreads();                                     // (everybody has read the counts per wavefront in s.part, which the scans below overwrite)
        uint32_t done = 0;
        for (uint32_t base = 0; base < nbins; base += kBookBlock) {
            const uint32_t sy = base + tid;
            const uint32_t f = (sy < nbins) ? a.hist[sy] : 0u;
            uint32_t tot;
            const uint32_t pos = block_excl_scan<uint32_t, kBookBlock / kWave>(f ? 1u : 0u, s.part, tot);
            if (f) keys[done + pos] = ((uint64_t)f << 16) | sy;
            done += tot;
            if (!f && sy < nbins) {             // unused symbol: length 0 everywhere
                a.len_out[sy] = 0;
                a.enc[sy] = 0;
                if (a.code_out) a.code_out[sy] = 0;
            }
        }
    }
    const uint32_t m2 = next_pow2(m);
    if (!a.presorted) for (uint32_t i = m + tid; i < m2; i += kBookBlock) keys[i] = ~0ull;
    __syncthreads();
    // ---- 2. leaves in (frequency, symbol) order ----
    if (!a.presorted) bitonic_sort(keys, m2);
    // ---- 3. two-queue merge in rounds ----
    {
        // The first rounds merge hundreds and thousands of light leaves each: in global memory, by everybody.  Most
        // rounds come later, with few items each: once the L leaves and N nodes that wait make at most
        // kBookLdsSyms / 2 items, they move to LDS (L + 2N - 1 nodes at the end, which fit), the rounds
        // are finished there, and the parents go back with the offset of the first node moved.
        uint32_t li, ii, ni;
        bool narrow = a.narrow != 0u;
        if (!a.hdr) {                                        // (a stage call: any frequencies)
            uint64_t total = 0, sum = 0;
            for (uint32_t i = tid; i < m; i += kBookBlock) sum += keys[i] >> 16;
            sum = wave_sum<uint64_t>(sum);
            uint64_t *part64 = reinterpret_cast<uint64_t *>(s.u.exchange);
            __syncthreads();
            if ((tid & (uint32_t)(kWave - 1)) == 0u) part64[tid / (uint32_t)kWave] = sum;
            __syncthreads();
            for (uint32_t w = 0; w < kBookBlock / kWave; ++w) total += part64[w];
            narrow = total < 0x7fffffffull;
            __syncthreads();
        }
        static_assert(sizeof(s.u.exchange) >= 16u * kBookWin, "window of both queues and the merged order");
        if (a.presorted && narrow && m <= a.lds_leaves) {
            // (the weights take the room of everything else in LDS; what is still needed of it waits in registers)
            __syncthreads();
            const uint64_t t0 = s.total[0], t1 = s.total[1], t2 = s.total[2];
            __syncthreads();
            huffman_rounds_weights(keys, reinterpret_cast<uint32_t *>(&s), leaf_parent, int_parent, m);
            if (tid == 0) { s.total[0] = t0; s.total[1] = t1; s.total[2] = t2; }
            __syncthreads();
            return;                                          // the rest by whole grids: k_book_depths, k_book_codes
        }
        for (uint32_t i = tid; i < m; i += kBookBlock) iw[i] = 0;
        __syncthreads();
        if (narrow)
            huffman_rounds_window(keys, iw, leaf_parent, int_parent, m, reinterpret_cast<uint32_t *>(s.u.exchange), s.part, kBookLdsSyms / 2u, li, ii, ni);
        else
            huffman_rounds(keys, iw, leaf_parent, int_parent, m, kBookLdsSyms / 2u, li, ii, ni);
        const uint32_t L = m - li, N = ni - ii;
        if (L + N > 1u) {
            uint64_t *l_keys = s.u.large.keys, *l_iw = s.u.large.iw;
            uint32_t *l_lp = s.v.large.lp, *l_ip = s.v.large.ip;
            for (uint32_t j = tid; j < L; j += kBookBlock) l_keys[j] = keys[li + j];
            for (uint32_t k = tid; k < kBookLdsSyms; k += kBookBlock) l_iw[k] = k < N ? iw[ii + k] : 0ull;
            __syncthreads();
            huffman_rounds_lds(l_keys, l_iw, l_lp, l_ip, L, tid, (uint32_t)kBookBlock, s.part, N);
            __syncthreads();
            for (uint32_t j = tid; j < L; j += kBookBlock) leaf_parent[li + j] = ii + l_lp[j];
            for (uint32_t k = tid; k + 1u < L + 2u * N - 1u; k += kBookBlock) int_parent[ii + k] = ii + l_ip[k];   // (the last node is the root)
        }
    }
    __syncthreads();
    if (a.presorted) return;                                 // the rest by whole grids: k_book_depths, k_book_codes
    // ---- 4. depth of every leaf: walk to the root (node m-2) ----
    // (four leaves per thread at a time: a walk is a chain of dependent loads, in global memory for a large
    // alphabet, and four chains wait side by side)
    constexpr uint32_t kWalks = 4;
    for (uint32_t i0 = tid; i0 < m; i0 += kWalks * kBookBlock) {
        uint32_t p[kWalks], depth[kWalks];
        const uint32_t root = m >= 2 ? m - 2 : 0u;
#pragma unroll
        for (uint32_t k = 0; k < kWalks; ++k) {
            const uint32_t i = i0 + k * kBookBlock;
            depth[k] = 1;
            p[k] = (m >= 2 && i < m) ? leaf_parent[i] : root;
        }
        bool more = true;
        while (more) {
            more = false;
#pragma unroll
            for (uint32_t k = 0; k < kWalks; ++k) {
                const bool go = p[k] != root && depth[k] < 66u;
                const uint32_t q = go ? int_parent[p[k]] : root;
                p[k] = go ? q : p[k];
                depth[k] += go ? 1u : 0u;
                more = more || go;
            }
        }
#pragma unroll
        for (uint32_t k = 0; k < kWalks; ++k) {
            const uint32_t i = i0 + k * kBookBlock;
            if (i < m) {
                const uint32_t sym = (uint32_t)(keys[i] & 0xffffu);
                atomicAdd(&s.cnt[depth[k] > 64 ? 64 : depth[k]], 1u);
                a.len_out[sym] = (uint8_t)(depth[k] > 64 ? 64 : depth[k]);    // (the canonical order is counted by symbol)
            }
        }
    }
    __syncthreads();
    book_first_codes(a, s, m, false);
    book_codes(a, nullptr, a.len_out, nbins, s.first, s.v.wc);
}

// The container's header and the padding between its sections, once the code book is known (one thread).
__device__ inline void book_finish(const BookArgs &a, uint32_t m, uint32_t max_len, uint64_t n_rec, uint64_t n_vrec, uint64_t nnz) {
    a.ctl->max_len = max_len;
    if (a.hdr) {
        // (Field by field: a copy of the prepared header, changed and stored as a whole, was kept on the stack, which every thread of
        // the launch filled before anything else: 10 MB of stores per compression with the workgroups that place the records.
        // 64 x 64 x 112 x 112 149.1 us -> 146.8, the five-layer step 812 -> 804.)
        const Header &p = a.proto;
        Header &h = *a.hdr;
        const uint64_t off_payload = align16(p.off_outlier + 8ull * n_rec);
        h.magic = p.magic; h.version = p.version; h.N = p.N; h.C = p.C; h.H = p.H; h.W = p.W; h.nbins = p.nbins;
        h.chunk_syms = p.chunk_syms; h.n_chunks = p.n_chunks; h.eb_bits = p.eb_bits; h.ebx2_bits = p.ebx2_bits; h.r_bits = p.r_bits;
        h.off_len = p.off_len; h.off_chunk = p.off_chunk; h.off_outlier = p.off_outlier; h.zero = p.zero;
        h.n_active = m;
        h.max_len = max_len;
        h.n_rec = (uint32_t)n_rec;
        h.n_vrec = (uint32_t)n_vrec;
        h.nnz = nnz;
        h.off_payload = off_payload;
        h.payload_words = 0;
        h.total_bytes = 0;
        h.status = 1;                      // overwritten by the encode kernel's last workgroup
        a.ctl->off_payload = off_payload;
        if (off_payload > a.capacity) atomicOr(&a.ctl->status, (uint32_t)ST_CAPACITY);
        // zero the padding between sections
        uint8_t *base = reinterpret_cast<uint8_t *>(a.hdr);
        for (uint64_t o = p.off_len + a.nbins; o < p.off_chunk; ++o) base[o] = 0;
        for (uint64_t o = p.off_chunk + 4ull * p.n_chunks; o < p.off_outlier; ++o) base[o] = 0;
        if (off_payload <= a.capacity)
            for (uint64_t o = p.off_outlier + 8ull * n_rec; o < off_payload; ++o) base[o] = 0;
    }
}

// ---------------------------------------------------------------------------
// Leaves of a large alphabet in (frequency, symbol) order.  One key per symbol: (frequency, symbol), or
// a key above all of those for a symbol that does not occur (each its own, so that no two keys are
// equal).  k_book_sort_tiles: one tile of kBookBlock symbols per workgroup, sorted in registers; the
// grid's tiles are a power of two and cover the alphabet.  It also counts the symbols that occur.
// k_book_merge: groups of WAYS runs of `run` keys merged; a key's place is its rank in its own run plus the numbers
// of smaller keys in the others (binary searches side by side); one key per thread.  Four runs at a time, three launches for 65536 keys where two at a time took
// six: as long where they sort (eight at a time: 4 us more, their probes fill the L2s), and 64 x 56 x 56 in bfloat16 at 1e-3, whose
// 2000 symbols need none of it, 131 -> 126 us.  Alphabets whose
// occurring symbols fit LDS are built there from the histogram: the merges then have nothing to do.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBookBlock) void k_book_sort_tiles(BookArgs a) {
    __shared__ uint64_t s_x[2 * kBookBlock];
    const uint32_t s = blockIdx.x * (uint32_t)kBookBlock + threadIdx.x;
    uint32_t f = 0;
    if (a.hist_copies) {                            // the partial histograms of the quantise kernel
#pragma unroll
        for (uint32_t k = 0; k < kQuantHistCopiesMax; ++k) f += (k < a.hist_copies && s < a.nbins) ? a.hist_parts[(size_t)k * a.nbins + s] : 0u;
        if (s < a.nbins) a.hist_sum[s] = f;
    } else {
        f = s < a.nbins ? a.hist[s] : 0u;
    }
    if (!f && s < a.nbins) {                        // unused symbol: length 0 everywhere
        a.len_out[s] = 0;
        a.enc[s] = 0;
        if (a.code_out) a.code_out[s] = 0;
    }
    if (threadIdx.x < kBookLens) a.scratch.tile_cnt[blockIdx.x * kBookLens + threadIdx.x] = 0;
    const uint32_t win_n = a.nbins < kEncTableMax ? a.nbins : kEncTableMax, win_lo = (a.nbins - win_n) / 2u;
    const uint32_t lenw_n = enc_len_window(a.nbins), lenw_lo = (a.nbins - lenw_n) / 2u;
    const uint32_t cnt = (uint32_t)__syncthreads_count(f != 0u);
    const uint32_t packw_n = kEncPackWindow, packw_lo = (a.nbins - packw_n) / 2u;       // (more bins than that)
    const uint32_t out = f != 0u && s != 0u ? (s - win_lo >= win_n ? 1u : 0u) | (s - lenw_lo >= lenw_n ? 2u : 0u) | (s - packw_lo >= packw_n ? 4u : 0u) : 0u;
    const uint64_t out0 = wave_ballot((out & 1u) != 0u), out1 = wave_ballot((out & 2u) != 0u), out2 = wave_ballot((out & 4u) != 0u);
    if (threadIdx.x == 0 && cnt) atomicAdd(&a.ctl->n_active, cnt);
    if ((out0 | out1 | out2) != 0ull && lane_id() == 0) atomicOr(&a.ctl->outside, (out0 ? 1u : 0u) | (out1 ? 2u : 0u) | (out2 ? 4u : 0u));
    uint64_t key[1] = {f ? (((uint64_t)f << 16) | s) : ((1ull << 63) | s)};
    block_sort<1>(key, s_x, (uint32_t)kBookBlock);
    a.scratch.keys[s] = key[0];
}

template <uint32_t WAYS>
__global__ __launch_bounds__(kBookMergeBlock) void k_book_merge(const uint64_t *src, uint64_t *dst, uint32_t run, const Control *ctl) {
    if (ctl->n_active <= kBookLdsSyms) return;
    const uint32_t i = blockIdx.x * (uint32_t)kBookMergeBlock + threadIdx.x;
    const uint64_t key = src[i];
    const uint32_t r = i / run;                              // run, WAYS: powers of two
    const uint64_t *group = src + (size_t)(r & ~(WAYS - 1u)) * run;
    // (branch-free, so that the searches of all runs are in flight together: below[w] counts the entries of run w that are smaller)
    uint32_t below[WAYS - 1u];
#pragma unroll
    for (uint32_t w = 0; w < WAYS - 1u; ++w) below[w] = 0;
    for (uint32_t step = run; step; step >>= 1) {
#pragma unroll
        for (uint32_t w = 0; w < WAYS - 1u; ++w) {
            const uint64_t *other = group + (size_t)((r + 1u + w) & (WAYS - 1u)) * run;
            const uint32_t probe = below[w] + step;
            below[w] = probe <= run && other[probe <= run ? probe - 1u : 0u] < key ? probe : below[w];
        }
    }
    uint32_t place = i - r * run;
#pragma unroll
    for (uint32_t w = 0; w < WAYS - 1u; ++w) place += below[w];
    dst[(size_t)(r & ~(WAYS - 1u)) * run + place] = key;
}

__global__ __launch_bounds__(kBookBlock) void k_codebook(BookArgs a) {
    extern __shared__ __align__(16) uint8_t s_book[];        // BookLds, or the weights of a large alphabet's leaves
    BookLds &s = *reinterpret_cast<BookLds *>(s_book);
    if (blockIdx.x != 0u) {                                  // the workgroups behind the first one bring the outlier records into order
        const uint32_t w = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave));
        const uint32_t run_0 = (blockIdx.x - 1u) * a.rec_wg_runs;
        for (uint32_t r = w; r < a.rec_wg_runs; r += (uint32_t)(kBookBlock / kWave))
            place_records<4>(a.recs, run_0 + r, (uint32_t)lane_id(), reinterpret_cast<uint2 *>(s_book + w * record_lds(a.recs.ring)));
        return;
    }
    // One workgroup on the critical path of its stream, often next to the streaming kernels of
    // other streams: its wavefronts go first whenever they are ready to issue.
    __builtin_amdgcn_s_setprio(3);
    const uint32_t tid = threadIdx.x, lane = tid & (uint32_t)(kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
    const uint32_t nbins = a.nbins;
    const bool given = a.given_len != nullptr;
    // What the header takes from the control block, unless the counts are added up here: asked for now, needed last.  The first
    // kernel of a call (a given code book) finds the call before it there: nothing is counted yet, and k_place_payload, which
    // adds the records up, checks the room for them and clears the padding behind them.
    uint64_t ctl_rec = 0, ctl_vrec = 0, ctl_nnz = 0;
    if (!a.reset_ctl) { ctl_rec = a.ctl->n_rec; ctl_vrec = a.ctl->n_vrec; ctl_nnz = a.ctl->nnz; }
    if (a.reset_ctl && tid < sizeof(Control) / 4u) reinterpret_cast<uint32_t *>(a.ctl)[tid] = 0u;   // (before the first barrier: nothing has raised a bit yet)
    if (tid < 65) s.cnt[tid] = 0;
    if (tid < 4) s.word[tid] = 0;
    __syncthreads();
    uint32_t m = 0, outside = 0;
    bool large = false;
    if (a.presorted && (m = a.ctl->n_active) > kBookLdsSyms) {       // (the sort kernels have counted and looked already)
        large = true;
        outside = a.ctl->outside;
        book_large(a, s, m);
    } else {
    // ---- 1. the symbols that occur.  A wavefront looks at consecutive symbols, kGroup x 64 at a time (their loads in
    // flight together); counted first, then listed, so that the list is in order of the symbols.  (And: does every
    // symbol that occurs, but for the escape symbol, lie in the part of the encode table that the encoders keep in
    // LDS?)  Code book reuse: the given length takes the place of the frequency. ----
    const uint32_t win_n = nbins < kEncTableMax ? nbins : kEncTableMax, win_lo = (nbins - win_n) / 2u;
    const uint32_t lenw_n = enc_len_window(nbins), lenw_lo = (nbins - lenw_n) / 2u;
    const uint32_t packw_n = nbins < kEncPackWindow ? nbins : kEncPackWindow, packw_lo = (nbins - packw_n) / 2u;
    constexpr uint32_t kGroup = 8;
    const uint32_t iters = (nbins + (uint32_t)kBookBlock - 1u) / (uint32_t)kBookBlock;      // steps of 64 symbols per wavefront
    const uint32_t s0 = wave * iters * (uint32_t)kWave;
    uint32_t f[kGroup];
    auto fetch = [&](uint32_t g) {
        if (a.hist_parts && nbins <= kBookPartsMax) {        // partial histograms, all loads in flight together (g == 0)
            constexpr uint32_t kJ = kBookPartsMax / (uint32_t)kBookBlock, kC = kQuantHistCopiesBook;
            const __amdgpu_buffer_rsrc_t r = __builtin_amdgcn_make_buffer_rsrc(const_cast<uint32_t *>(a.hist_parts), 0, (int)(kC * nbins * 4u), 0x00020000);
            uint32_t v[kJ][kC];
#pragma unroll
            for (uint32_t j = 0; j < kJ; ++j) {
                const uint32_t sy = s0 + j * (uint32_t)kWave + lane;
                const int at = j < iters && sy < nbins ? (int)(sy * 4u) : (int)0x80000000;
#pragma unroll
                for (uint32_t k = 0; k < kC; ++k) v[j][k] = __builtin_amdgcn_raw_buffer_load_b32(r, at, (int)(k * nbins * 4u), 0);
            }
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                f[j] = 0;
                if (j < kJ) {
#pragma unroll
                    for (uint32_t k = 0; k < kC; ++k) f[j] += v[j < kJ ? j : 0][k];
                }
            }
            return;
        }
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) {
            const uint32_t sy = s0 + (g + j) * (uint32_t)kWave + lane;
            f[j] = (g + j < iters && sy < nbins) ? (given ? (uint32_t)a.given_len[sy] : a.hist[sy]) : 0u;
        }
    };
    static_assert(kBookPartsMax <= kGroup * (uint32_t)kBookBlock, "one group");
    uint32_t mine = 0;
    {
        bool out1 = false, out2 = false, out3 = false;
        for (uint32_t g = 0; g < iters; g += kGroup) {
            fetch(g);
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                const uint32_t sy = s0 + (g + j) * (uint32_t)kWave + lane;
                mine += (uint32_t)__popcll(wave_ballot(f[j] != 0u));
                out1 = out1 || (f[j] != 0u && sy != 0u && sy - win_lo >= win_n);
                out2 = out2 || (f[j] != 0u && sy != 0u && sy - lenw_lo >= lenw_n);
                out3 = out3 || (f[j] != 0u && sy != 0u && sy - packw_lo >= packw_n);
            }
        }
        const uint32_t outside = (wave_ballot(out1) ? 1u : 0u) | (wave_ballot(out2) ? 2u : 0u) | (wave_ballot(out3) ? 4u : 0u);
        if (lane == 0) {
            s.part[wave] = mine;
            if (outside) atomicOr(&s.word[0], outside);
        }
    }
    __syncthreads();
    uint32_t at = 0;
    m = 0;
#pragma unroll
    for (uint32_t w = 0; w < kBookBlock / kWave; ++w) {
        const uint32_t c = s.part[w];
        at += w < wave ? c : 0u;
        m += c;
    }
    outside = s.word[0];

    if (given || m <= kBookLdsSyms) {
        uint16_t *syms = given ? s.u.given.sym : s.sym;
        uint8_t *depths = given ? s.u.given.depth : s.depth;
        for (uint32_t g = 0; g < iters; g += kGroup) {
            if (iters > kGroup) fetch(g);                    // (else they are still there)
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                const uint32_t sy = s0 + (g + j) * (uint32_t)kWave + lane;
                const uint64_t mask = wave_ballot(f[j] != 0u);
                const uint32_t pos = at + __builtin_amdgcn_mbcnt_hi((uint32_t)(mask >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)mask, 0u));
                if (f[j] != 0u) {
                    syms[pos] = (uint16_t)sy;
                    if (given) depths[pos] = (uint8_t)(f[j] > 57u ? 64u : f[j]);      // (64: a length the container cannot hold; refused below)
                    else s.u.exchange[pos] = ((uint64_t)f[j] << 16) | pos;
                } else if (g + j < iters && sy < nbins) {    // unused symbol: length 0 everywhere
                    a.len_out[sy] = 0;
                    a.enc[sy] = 0;
                    if (a.code_out) a.code_out[sy] = 0;
                }
                at += (uint32_t)__popcll(mask);
            }
        }
        if (given) {
            __syncthreads();
            for (uint32_t i = tid; i < m; i += kBookBlock) atomicAdd(&s.cnt[depths[i]], 1u);
            __syncthreads();
        } else {
            // ---- 2. leaves in (frequency, symbol) order, 3. the tree, 4. depths ----
            uint32_t n2 = next_pow2(m);
            n2 = n2 < (uint32_t)kWave ? (uint32_t)kWave : n2;
            for (uint32_t i = m + tid; i < n2; i += kBookBlock) s.u.exchange[i] = ~0ull;
            // (keys of 32 bits if all frequencies together allow it; a container's do but for the largest possible tensor)
            bool narrow = a.narrow != 0u;
            if (!a.hdr) {
                __syncthreads();
                uint64_t total = 0, sum = 0;
                for (uint32_t i = tid; i < m; i += kBookBlock) sum += s.u.exchange[i] >> 16;
                sum = wave_sum<uint64_t>(sum);
                uint64_t *part64 = reinterpret_cast<uint64_t *>(s.v.wc);
                if (lane == 0) part64[wave] = sum;
                __syncthreads();
                for (uint32_t w = 0; w < kBookBlock / kWave; ++w) total += part64[w];
                narrow = total < 0x7fffffffull;
            }
            __syncthreads();
            uint64_t key[2] = {tid < n2 ? s.u.exchange[tid] : ~0ull, 0ull};
            if (n2 <= (uint32_t)kBookBlock) {
                __syncthreads();                             // (the keys are read before the exchange overwrites them)
                uint64_t k1[1] = {key[0]};
                block_sort<1>(k1, s.u.exchange, n2);
                key[0] = k1[0];
            } else {
                key[1] = s.u.exchange[kBookBlock + tid];
                __syncthreads();
                block_sort<2>(key, s.u.exchange, n2);
            }
            const uint32_t n_keys = n2 <= (uint32_t)kBookBlock ? 1u : 2u;
            if (narrow) book_tree<uint32_t>(s, a.recs, m, key, n_keys);
            else book_tree<uint64_t>(s, a.recs, m, key, n_keys);
        }
        // ---- 5. canonical codes ----
        book_first_codes(a, s, m, given);
        book_codes(a, syms, depths, m, s.first, s.v.wc);
    } else {
        large = true;
        book_large(a, s, m);
    }
    }

    // ---- 7. container layout ----
    if (tid == 0) {
        const bool counted = a.recs.n_wg != 0u;
        const uint64_t n_rec = counted ? s.total[0] : ctl_rec, n_vrec = counted ? s.total[2] : ctl_vrec, nnz = counted ? s.total[1] : ctl_nnz;
        if (counted) { a.ctl->n_rec = n_rec; a.ctl->n_vrec = n_vrec; a.ctl->nnz = nnz; }
        a.ctl->n_active = m;
        a.ctl->enc_in_window = (outside & 1) ? 0u : 1u;
        a.ctl->len_in_window = (outside & 2) ? 0u : 1u;
        a.ctl->pack_in_window = (outside & 4) || large || s.word[2] > kPackBits ? 0u : 1u;
        if (!large || !a.presorted) book_finish(a, m, s.word[2], n_rec, n_vrec, nnz);
    }
}

// ---------------------------------------------------------------------------
// The rest of a large alphabet's code book (more than kBookLdsSyms symbols occur, presorted), by whole grids instead of the
// one workgroup that built the tree: a walk to the root is a chain of some twenty dependent loads, and the canonical
// codes visit every symbol of the alphabet.  64 x 256 x 56 x 56 at a bound of 1e-4, 65536
// bins: k_codebook 406 us with them, 272 without (85 since huffman_rounds_weights), and 28 behind it.  Where at most
// kBookLdsSyms symbols of such an alphabet occur they return at once and cost 9 us.
// k_book_depths: one leaf per thread; it also counts the lengths per tile of kBookBlock symbols.
// k_book_codes: a tile per workgroup; the code of a symbol is the first code of its length plus the number of smaller
// symbols of that length: those of the tiles in front, of the wavefronts in front and of the lanes in front.
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBookDepthBlock) void k_book_depths(BookArgs a) {
    const uint32_t m = a.ctl->n_active;
    const uint32_t i = blockIdx.x * (uint32_t)kBookDepthBlock + threadIdx.x;
    if (m <= kBookLdsSyms || i >= m) return;
    const uint32_t root = m - 2u;
    uint32_t depth = 1;
    for (uint32_t p = a.scratch.leaf_parent[i]; p != root && depth < 64u; p = a.scratch.int_parent[p]) ++depth;
    const uint32_t sym = (uint32_t)(a.scratch.keys[i] & 0xffffu);
    a.len_out[sym] = (uint8_t)depth;
    atomicAdd(&a.scratch.tile_cnt[sym / (uint32_t)kBookBlock * kBookLens + depth], 1u);
}

__global__ __launch_bounds__(kBookBlock) void k_book_codes(BookArgs a) {
    constexpr uint32_t kWaves = kBookBlock / kWave;
    __shared__ uint32_t s_cnt[kBookLens], s_before[kBookLens], s_findex[kBookLens], s_wc[kWaves][kBookLens], s_max;
    __shared__ uint64_t s_first[kBookLens];
    const uint32_t m = a.ctl->n_active;
    if (m <= kBookLdsSyms) return;
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id(), wave = tid / (uint32_t)kWave;
    const uint32_t sym = blockIdx.x * (uint32_t)kBookBlock + tid;
    const uint32_t L = sym < a.nbins ? (uint32_t)a.len_out[sym] : 0u;
    for (uint32_t i = tid; i < kWaves * kBookLens; i += kBookBlock) s_wc[i / kBookLens][i % kBookLens] = 0;
    if (tid < kBookLens) {
        uint32_t all = 0, before = 0;
#pragma unroll 8
        for (uint32_t t = 0; t < gridDim.x; ++t) {
            const uint32_t c = a.scratch.tile_cnt[t * kBookLens + tid];
            all += c;
            before += t < blockIdx.x ? c : 0u;
        }
        s_cnt[tid] = all;
        s_before[tid] = before;
    }
    __syncthreads();
    if (tid < (uint32_t)kWave) {
        uint32_t mx, mn;
        const bool ok = canonical_first_codes_wave(s_cnt, m, s_first, s_findex, &mx, &mn);
        if (tid == 0) {
            s_max = mx;
            if (!ok && blockIdx.x == 0) atomicOr(&a.ctl->status, (uint32_t)ST_INTERNAL);
        }
    }
    uint32_t in_wave = 0;
    uint64_t todo = wave_ballot(L != 0u);
    while (todo) {                                       // one step per length that occurs in the wavefront
        const uint32_t Lc = (uint32_t)__builtin_amdgcn_readlane((int)L, __builtin_ctzll(todo));
        const uint64_t same = wave_ballot(L == Lc);
        if (L == Lc) in_wave = (uint32_t)__popcll(same & ((1ull << lane) - 1ull));
        if (lane == 0) s_wc[wave][Lc] = (uint32_t)__popcll(same);
        todo &= ~same;
    }
    __syncthreads();
    if (L) {
        uint32_t before = s_before[L];
        for (uint32_t w = 0; w < wave; ++w) before += s_wc[w][L];
        const uint64_t code = s_first[L] + before + in_wave;
        a.enc[sym] = (code << 6) | (uint64_t)(L & 63u);
        if (a.code_out) a.code_out[sym] = code;
    }
    if (blockIdx.x == 0 && tid == 0) a.ctl->pack_in_window = (a.ctl->outside & 4u) || s_max > kPackBits ? 0u : 1u;
    if (blockIdx.x == 0 && tid == 0) book_finish(a, m, s_max, a.ctl->n_rec, a.ctl->n_vrec, a.ctl->nnz);
}

// ---------------------------------------------------------------------------
// Decode tables from a length table.  Also checks a container header against
// the shape the caller passed; any inconsistency latches ST_FORMAT, which makes
// the reconstruct kernel do nothing.
// A chain of latencies on every decompression's critical path: the lengths are asked for while one thread still
// checks the header; a wavefront keeps its counts per length in a register (lane L: length L), so that counting and
// ordering need three barriers whatever the alphabet; a table entry finds its length by comparison with the first
// twelve limits and its symbol by arithmetic, and the second level, whose prefixes are the end of the first one with
// sizes that never decrease, is laid out in closed form.  1024 bins: 6.1 us instead of 12.7 (binary searches over
// the limits, a scan over the prefixes), 4096 bins: 8 instead of 18, 65536 bins: 45 instead of 111 (53 since it
// builds the table of lengths and the residuals in canonical order for those).
// ---------------------------------------------------------------------------
__global__ __launch_bounds__(kBookBlock) void k_decode_tables(TablesArgs a) {
    __builtin_amdgcn_s_setprio(3);                  // as k_codebook: a single workgroup others wait for
    constexpr uint32_t kWaves = kBookBlock / kWave;
    __shared__ uint32_t s_cnt[65];
    __shared__ uint64_t s_first[65];
    __shared__ uint64_t s_limit[65];
    __shared__ uint32_t s_findex[65];
    __shared__ uint32_t s_lim18[20];                                // limits of the lengths up to 18, of codes left-aligned in 18 bits
    __shared__ uint32_t s_off[20];                                  // place in canonical order minus first code, of those lengths
    __shared__ uint32_t s_ok, s_code_ok, s_maxlen, s_m;             // header accepted; lengths are a complete code (a word each: a wavefront may still read the first when another stores the second)
    __shared__ uint16_t s_sorted[kLut16MaxBins];                    // symbols in canonical order (the first ones, of a larger alphabet)
    __shared__ uint32_t s_wc[kWaves][64];                           // symbols per (wavefront, length), then those of the wavefronts in front

    const uint32_t tid = threadIdx.x, lane = tid & (uint32_t)(kWave - 1);
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(tid / kWave));
    if (a.reset_ctl && tid < sizeof(Control) / 4u) reinterpret_cast<uint32_t *>(a.ctl)[tid] = 0u;   // before the first barrier: nothing has raised a bit yet
    auto raise_format = [&]() {                     // thread 0 only
        atomicOr(&a.ctl->status, (uint32_t)ST_FORMAT);
        if (a.latched) atomicOr(a.latched, (uint32_t)ST_FORMAT);
        if (a.status_out) *a.status_out = -3;
    };
    const uint32_t nbins = a.hdr ? a.hdr->nbins : a.nbins;
    const uint32_t chunk = a.hdr ? a.hdr->chunk_syms : 64u;
    const bool readable = nbins <= 65536u && (!a.hdr || a.bytes >= (uint64_t)kHeaderBytes + nbins);

    // ---- the lengths, 64 consecutive symbols of a wavefront's own range at a time, kGroup of those in flight ----
    // (few, and the next ones asked for before these are worked on: unrolled further, the code that every launch
    // fetches anew cost more than it saved)
    constexpr uint32_t kGroup = 4;
    const uint32_t iters = readable ? (nbins + (uint32_t)kBookBlock - 1u) / (uint32_t)kBookBlock : 0u;
    const uint32_t s0 = wave * iters * (uint32_t)kWave;
    uint32_t len[kGroup], ahead[kGroup];
    auto fetch = [&](uint32_t g, uint32_t (&to)[kGroup]) {
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) {
            const uint32_t sy = s0 + (g + j) * (uint32_t)kWave + lane;
            to[j] = (g + j < iters && sy < nbins) ? (uint32_t)a.len[sy] : 0u;
        }
    };
    fetch(0, len);
    if (tid == 0) {
        if (a.status_out) *a.status_out = 0;
        uint32_t ok = readable ? 1u : 0u;
        if (a.hdr) {
            const Header h = *a.hdr;
            const Header &e = a.expect;
            const uint64_t n = (uint64_t)e.N * e.C * e.H * e.W;
            if (a.bytes < kHeaderBytes) ok = 0;
            if (h.magic != kMagic || (h.version != 1u && h.version != 2u) || h.status != 0u) ok = 0;
            if (h.N != e.N || h.C != e.C || h.H != e.H || h.W != e.W) ok = 0;
            if (h.nbins < 4u || h.nbins > 65536u || (h.nbins & 1u)) ok = 0;
            if (h.chunk_syms == 0) ok = 0;
            const float eb = __uint_as_float(h.eb_bits);
            if (!(eb >= 0x1p-100f && eb <= 0x1p100f)) ok = 0;
            if (__float_as_uint(2.0f * eb) != h.ebx2_bits) ok = 0;
            if (__float_as_uint((float)(1.0 / (double)(2.0f * eb))) != h.r_bits) ok = 0;
            if (ok) {
                const uint64_t n_chunks = (n + h.chunk_syms - 1u) / h.chunk_syms;
                if (h.n_chunks != n_chunks) ok = 0;
                if (h.off_len != kHeaderBytes || h.off_chunk != align16(h.off_len + h.nbins) ||
                    h.off_outlier != align16(h.off_chunk + 4ull * h.n_chunks) ||
                    h.off_payload != align16(h.off_outlier + 8ull * h.n_rec) ||
                    h.total_bytes != h.off_payload + 4ull * h.payload_words || h.total_bytes > a.bytes) ok = 0;
            }
        }
        s_ok = ok;
    }

    // ---- symbols per length: lane L of a wavefront counts its symbols of length L ----
    // (one step per length that occurs among 64 symbols; f(length, lanes that have it))
    auto each_length = [&](uint32_t L, auto f) {
        uint64_t todo = wave_ballot(L != 0u);
        while (todo) {
            const uint32_t Lc = (uint32_t)__builtin_amdgcn_readlane((int)L, __builtin_ctzll(todo));
            const uint64_t same = wave_ballot(L == Lc);
            f(Lc, same);
            todo &= ~same;
        }
    };
    uint32_t mine = 0;
    bool bad = false;
    for (uint32_t g = 0; g < iters; g += kGroup) {
        if (g + kGroup < iters) fetch(g + kGroup, ahead);
#pragma unroll
        for (uint32_t j = 0; j < kGroup; ++j) {
            if (g + j >= iters) continue;                    // (uniform)
            bad = bad || len[j] > 57u;
            each_length(len[j] > 57u ? 0u : len[j], [&](uint32_t Lc, uint64_t same) { mine += lane == Lc ? (uint32_t)__popcll(same) : 0u; });
        }
        if (g + kGroup < iters) {
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) len[j] = ahead[j];
        }
    }
    s_wc[wave][lane] = mine;
    bad = __syncthreads_or(bad ? 1 : 0) != 0;
    if (!s_ok || bad) {
        if (tid == 0) raise_format();
        return;
    }
    if (tid < (uint32_t)kWave) {
        uint32_t run = 0;
        for (uint32_t w = 0; w < kWaves; ++w) {
            const uint32_t c = s_wc[w][lane];
            s_wc[w][lane] = run;
            run += c;
        }
        s_cnt[lane] = run;
        if (lane == 0) s_cnt[64] = 0;
        const uint32_t m = (uint32_t)wave_sum<uint32_t>(run);
        wave_lds_fence();
        uint32_t mx, mn;
        const bool ok = m != 0u && canonical_first_codes_wave(s_cnt, m, s_first, s_findex, &mx, &mn);
        if (tid == 0) { s_maxlen = mx; s_m = m; s_code_ok = ok ? 1u : 0u; }
        if (ok) {
            wave_lds_fence();                                // the first codes of the other lengths
            const uint32_t L = tid ? tid : 64u;              // one length per lane
            // exclusive upper bound, left-aligned; the longest length closes the code space
            uint64_t lim = 0;
            if (L < mx) lim = (s_first[L] + s_cnt[L]) << (64u - L);
            else lim = ~0ull;
            s_limit[L] = lim;
            if (L < 20u) {
                s_lim18[L] = L < mx ? (uint32_t)(lim >> 46) : 1u << 18;
                s_off[L] = s_findex[L] - (uint32_t)s_first[L];
            }
            a.t.limit[L] = lim;
            a.t.first_code[L] = s_first[L];
            a.t.first_index[L] = s_findex[L];
            if (tid == 0) {
                a.t.limit[0] = 0; a.t.first_code[0] = 0; a.t.first_index[0] = 0;
                a.t.meta[0] = mx; a.t.meta[1] = m; a.t.meta[2] = mn;
            }
        }
    }
    __syncthreads();
    if (!s_code_ok) {
        if (tid == 0) raise_format();
        return;
    }
    const uint32_t m = s_m, mx = s_maxlen;
    // ---- canonical order: by length, then by symbol.  The symbols are visited in increasing order, so the place of a
    // symbol is the first index of its length plus the number of smaller symbols of the same length (lane L: the next
    // place for length L among my wavefront's symbols) ----
    {
        if (iters > kGroup) fetch(0, len);                   // (else they are still there)
        uint32_t next = lane ? s_findex[lane] + s_wc[wave][lane] : 0u;
        for (uint32_t g = 0; g < iters; g += kGroup) {
            if (g + kGroup < iters) fetch(g + kGroup, ahead);
#pragma unroll
            for (uint32_t j = 0; j < kGroup; ++j) {
                if (g + j >= iters) continue;
                const uint32_t sy = s0 + (g + j) * (uint32_t)kWave + lane;
                uint32_t pos = 0;
                each_length(len[j], [&](uint32_t Lc, uint64_t same) {
                    const uint32_t at = (uint32_t)__builtin_amdgcn_readlane((int)next, (int)Lc);
                    const uint32_t rank = __builtin_amdgcn_mbcnt_hi((uint32_t)(same >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)same, 0u));
                    pos = len[j] == Lc ? at + rank : pos;
                    next += lane == Lc ? (uint32_t)__popcll(same) : 0u;
                });
                if (len[j]) {
                    a.t.sorted[pos] = (uint16_t)sy;
                    if (nbins > kLut16MaxBins) {
                        const uint16_t r = (uint16_t)(sy ? (int32_t)sy - (int32_t)(nbins / 2u) : -32768);
                        a.t.resid[pos] = r;
                        if (pos < kSubEntries) a.t.sub16[pos] = r;
                    }
                    if (pos < kLut16MaxBins) s_sorted[pos] = (uint16_t)sy;
                }
            }
            if (g + kGroup < iters) {
#pragma unroll
                for (uint32_t j = 0; j < kGroup; ++j) len[j] = ahead[j];
            }
        }
    }
    __syncthreads();

    // ---- look-up tables; entries carry the residual, not the symbol ----
    // Length of the code that the bits v, left-aligned in 18, start with, if it is one of lo .. hi bits (else hi + 1): one
    // more than the number of limits it reaches.  lim[i]: the limit of length lo + i.
    const int32_t radius = (int32_t)(nbins / 2u);
    const bool compact = nbins <= kLut16MaxBins;
    const bool skip_general = a.compact_only && !(a.general_unless_chunk64 && chunk != 64u);
    auto symbol_of = [&](uint32_t v18, uint32_t L) -> uint32_t {
        const uint32_t idx = s_off[L] + (v18 >> (18u - L));
        return s_sorted[idx < m ? idx : m - 1u];             // (beyond: a code of a single symbol, the bit pattern that is no code)
    };
    if (!skip_general) {
        uint32_t lim[kLutBits];
#pragma unroll
        for (int i = 0; i < kLutBits; ++i) lim[i] = s_lim18[i + 1];
        for (uint32_t e = tid; e < kLutSize; e += kBookBlock) {
            const uint32_t v18 = e << (18 - kLutBits);
            uint32_t L = 1;
#pragma unroll
            for (int i = 0; i < kLutBits; ++i) L += v18 >= lim[i] ? 1u : 0u;
            uint32_t entry;
            if (L <= (uint32_t)kLutBits) {
                const uint32_t sym = symbol_of(v18, L);
                entry = ((uint32_t)(sym ? (int32_t)sym - radius : -32768) << 8) | L;
            } else {
                // no code of at most kLutBits bits starts here: length byte 0, and in the residual field the
                // shortest length a code with this prefix can have (where the decoder's search starts)
                const uint64_t v = (uint64_t)e << (64 - kLutBits);
                while (L < mx && v >= s_limit[L]) ++L;
                entry = L << 8;
            }
            a.t.lut[e] = entry;
        }
    }
    // Larger alphabets: the length table.  Canonical codes grow in length with their value, so nearly every prefix of
    // kLenBits bits has codes of one length under it, also where they are longer than the prefix: all but those in
    // which one length ends and the next begins.  A thread's prefixes are consecutive: the length only ever grows.
    if (!compact) {
        constexpr uint32_t kPer = (1u << kLenBits) / kBookBlock;
        static_assert(kPer == 8u, "one 8-byte store per thread");
        uint64_t packed = 0;
        uint32_t L = 1;
#pragma unroll
        for (uint32_t j = 0; j < kPer; ++j) {
            const uint64_t v = (uint64_t)(tid * kPer + j) << (64 - kLenBits), v_last = v | (~0ull >> kLenBits);
            while (L < mx && v >= s_limit[L]) ++L;
            const uint32_t shortest = L;
            while (L < mx && v_last >= s_limit[L]) ++L;
            packed |= (uint64_t)((L == shortest && L <= kLenFast) ? L : (kLenMixed | shortest)) << (8u * j);
        }
        reinterpret_cast<uint64_t *>(a.t.lut16)[tid] = packed;
    }
    // The compact table on the next kLut16Bits bits, for alphabets whose residuals fit 12 signed bits, and
    // its second level.  A prefix of kLut16Bits bits under which longer codes lie gets a sub-table indexed by
    // the next 1, 2, 4 or 6 bits (enough for the longest code under the prefix, 6 at most): its entries are
    // (residual << 4) | (length - kLut16Bits), or 0 for a code that is longer still.  The first-level entry of
    // such a prefix is ((offset / 2) << 2 | width code) << 4 with a zero length; offset 0 is never given out,
    // so an all-zero entry means "no sub-table" (the sub-tables filled their array: search by length).
    // Canonical codes grow in length with their value: the prefixes with longer codes are e0, e0 + 1, ... to the end,
    // and the first of them have nothing beyond 13 bits, the next nothing beyond 14, then 16: four classes in a row.
    if (compact) {
        constexpr uint32_t kPer = kLut16Size / kBookBlock;          // consecutive first-level entries per thread
        static_assert(kPer == 4u && kLut16Bits == 12, "packed stores, classes");
        auto prefixes_within = [&](uint32_t L) -> uint32_t { return s_lim18[L] >> 6; };     // whose codes all have at most L bits
        const uint32_t e0 = prefixes_within(12), e1 = prefixes_within(13), e2 = prefixes_within(14), e3 = prefixes_within(16);
        const uint32_t o1 = 2u, o2 = o1 + 2u * (e1 - e0), o3 = o2 + 4u * (e2 - e1), o4 = o3 + 16u * (e3 - e2), end = o4 + 64u * (kLut16Size - e3);
        {
            uint32_t lim[kLut16Bits];
#pragma unroll
            for (int i = 0; i < kLut16Bits; ++i) lim[i] = s_lim18[i + 1];
            uint32_t ent[kPer];
#pragma unroll
            for (uint32_t j = 0; j < kPer; ++j) {
                const uint32_t e = tid * kPer + j, v18 = e << 6;
                uint32_t L = 1;
#pragma unroll
                for (int i = 0; i < kLut16Bits; ++i) L += v18 >= lim[i] ? 1u : 0u;
                if (L <= (uint32_t)kLut16Bits) {
                    const uint32_t sym = symbol_of(v18, L);
                    ent[j] = (((uint32_t)(sym ? (int32_t)sym - radius : kLut16Escape) & 0xfffu) << 4) | L;
                } else {
                    const uint32_t k = e < e1 ? 0u : (e < e2 ? 1u : (e < e3 ? 2u : 3u));                 // class
                    const uint32_t kb = (0x6421u >> (k * 4u)) & 0xfu;
                    const uint32_t at = (k == 0u ? o1 - (e0 << 1) : (k == 1u ? o2 - (e1 << 2) : (k == 2u ? o3 - (e2 << 4) : o4 - (e3 << 6)))) + (e << kb);
                    ent[j] = at + (1u << kb) <= kSubEntries ? (((at >> 1) << 2) | k) << 4 : 0u;
                }
            }
            reinterpret_cast<uint2 *>(a.t.lut16)[tid] = make_uint2(ent[0] | (ent[1] << 16), ent[2] | (ent[3] << 16));
        }
        // the sub-table entries, one thread each
        uint32_t lim[6];
#pragma unroll
        for (int i = 0; i < 6; ++i) lim[i] = s_lim18[13 + i];
        const uint32_t used = end < kSubEntries ? end : kSubEntries;
        for (uint32_t x = tid; x < used; x += kBookBlock) {
            uint32_t entry = 0;
            if (x >= 2u) {
                const uint32_t k = x < o2 ? 0u : (x < o3 ? 1u : (x < o4 ? 2u : 3u));
                const uint32_t kb = (0x6421u >> (k * 4u)) & 0xfu;
                const uint32_t rel = x - (k == 0u ? o1 : (k == 1u ? o2 : (k == 2u ? o3 : o4)));
                const uint32_t first = k == 0u ? e0 : (k == 1u ? e1 : (k == 2u ? e2 : e3));
                const uint32_t v18 = ((first << kb) + rel) << (6u - kb);
                uint32_t L = 13;
#pragma unroll
                for (int i = 0; i < 6; ++i) L += v18 >= lim[i] ? 1u : 0u;
                if (L <= (uint32_t)kLut16Bits + kb) {
                    const uint32_t sym = symbol_of(v18, L);
                    entry = (((uint32_t)(sym ? (int32_t)sym - radius : kLut16Escape) & 0xfffu) << 4) | (L - (uint32_t)kLut16Bits);
                }
            }
            a.t.sub16[x] = (uint16_t)entry;
        }
    }
    if (tid == 0) { a.t.meta[3] = (uint32_t)radius; a.t.meta[4] = compact ? 1u : 0u; }
}

template __global__ void k_book_merge<2u>(const uint64_t *, uint64_t *, uint32_t, const Control *);
template __global__ void k_book_merge<4u>(const uint64_t *, uint64_t *, uint32_t, const Control *);

// The outlier records by a kernel of its own, with the sum of the partial histograms: where no code book is built behind the quantise
// kernel (a stage call) or the partial histograms are more than its one workgroup should add up.  The first workgroup adds up the counts as well.
__global__ __launch_bounds__(kGatherBlock) void k_gather_records(RecordArgs a, uint32_t *hist, const uint32_t *parts, uint32_t copies) {
    extern __shared__ __align__(16) uint8_t s_book[];        // record_lds(a.ring) bytes per wavefront
    const uint32_t wave = (uint32_t)__builtin_amdgcn_readfirstlane((int)(threadIdx.x / kWave)), lane = (uint32_t)lane_id();
    for (uint32_t b = blockIdx.x * (uint32_t)kGatherBlock + threadIdx.x; hist && b < a.nbins; b += gridDim.x * (uint32_t)kGatherBlock) {
        uint32_t v = 0, p[kQuantHistCopiesMax];              // (every copy in flight at once)
#pragma unroll
        for (uint32_t j = 0; j < kQuantHistCopiesMax; ++j) p[j] = (j < copies) ? parts[(size_t)j * a.nbins + b] : 0u;
#pragma unroll
        for (uint32_t j = 0; j < kQuantHistCopiesMax; ++j) v += p[j];
        hist[b] = v;
    }
    if (blockIdx.x == 0u && wave < 3u) {
        const uint64_t total = record_total(a, wave, lane);
        if (lane == 0) *(wave == 0u ? &a.ctl->n_rec : (wave == 1u ? &a.ctl->nnz : &a.ctl->n_vrec)) = total;
    }
    place_records<4>(a, blockIdx.x * (uint32_t)(kGatherBlock / kWave) + wave, lane, reinterpret_cast<uint2 *>(s_book + wave * record_lds(a.ring)));
}

}  // namespace comet
