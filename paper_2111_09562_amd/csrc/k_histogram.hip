// Histogram of the quantisation codes of an alphabet too large for the LDS window of the quantise kernel: of those that
// kernel does not count itself.
//
// Below kQuantCountMin elements that is all of them.  Above, a run of the quantise kernel counts its codes inside the
// window of 8192 bins nearly for free, and lists those outside while they are few; from the point at which they are more
// than one in 32 (kQuantOowShare) it leaves them to this kernel (run_from).  A listed code costs about 30 ps (an addition to
// global memory), a code read here 0.8 to 1.3 ps, counted or not: about 32 of these.  A slice without such a run ends at once.
// 128 x 64 x 224 x 224 at 1e-3, 65536 bins, one code in two thousand outside: 508 us in a sweep that does not count and 315 here;
// 546 and 4.5 as it is.
//
// The codes come back from memory (2 bytes each, mostly out of the last-level cache) and are counted with the whole LDS
// of a compute unit: one workgroup of sixteen wavefronts per compute unit, 32-bit counters for kCodeHistWindow bins around the
// centre, four copies of the kCodeHistHot innermost ones (lanes that meet in one bin mostly use different copies).  The
// centre bin and the escape symbol are counted in registers; what lies outside the window, far out in the tails, goes to
// the partial histogram in global memory.  At the end a workgroup adds its bins to one of the partial histograms,
// neighbouring lanes neighbouring bins.  Where the number of those is a multiple of eight (65536 bins: 8, 16384: 32; 40000: 13),
// the workgroups that share a copy run on one XCD, as consecutive ones go round the XCDs, and its lines stay in that XCD's L2.
// (In the quantise kernel itself, with everything outside its window listed and added to global memory, a
// tensor of 64 x 256 x 56 x 56 at a bound of 1e-4 and 65536 bins took 356 us, nearly all of it in those additions; now
// 59 us and 65 us here.)
#include "comet_kernels.h"

namespace comet {

template <bool SHARED>
__global__ __launch_bounds__(kCodeHistBlock) void k_code_hist(CodeHistArgs a) {
    extern __shared__ uint32_t s_dyn_ch[];          // a.win_n bins; kCodeHistHot x 4 (the innermost bins); a word per thread for what is not counted here
    __shared__ uint32_t s_from[SHARED ? kCodeHistRuns : 1u];   // run_from of the runs that reach into my slice
    uint32_t *s_win = s_dyn_ch;
    uint32_t *s_hot = s_dyn_ch + a.win_n;
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id();
    // A slice of consecutive groups of eight codes per workgroup, two groups per thread in flight; the first workgroup also
    // has the fewer than eight codes behind the last group.
    const uint64_t groups = a.n / 8u;
    const uint64_t per = (groups + gridDim.x - 1u) / gridDim.x;
    const uint64_t g0 = (uint64_t)blockIdx.x * per;
    const uint64_t g1 = g0 + per < groups ? g0 + per : groups;
    const uint64_t i_tail = groups * 8u + tid;
    const bool tail = blockIdx.x == 0u && i_tail < a.n;          // I have one of those
    const uint32_t run_n = SHARED ? a.divRun.d : 1u, r0 = SHARED ? fdiv((uint32_t)(g0 * 8u), a.divRun) : 0u;
    uint32_t r1 = 0;
    bool all = true, tail_on = tail;                             // (all: of my slice's codes, counted here)
    if (SHARED) {
        bool any = false, part_of = false;
        if (g0 < g1) {
            r1 = fdiv((uint32_t)(g1 * 8u - 1u), a.divRun);
            if (tid <= r1 - r0) {
                const uint32_t from = a.run_from[r0 + tid];
                const uint64_t b = (uint64_t)(r0 + tid) * run_n;
                any = from < (a.n - b < run_n ? (uint32_t)(a.n - b) : run_n);
                part_of = from != 0u;
                s_from[tid] = from;
            }
        }
        if (tail) {
            const uint32_t r = fdiv((uint32_t)i_tail, a.divRun);
            tail_on = (uint32_t)i_tail - r * run_n >= a.run_from[r];
        }
        if (!__syncthreads_or(any || tail_on ? 1 : 0)) return;   // (uniform) the quantise kernel has counted everything
        all = !__syncthreads_or(part_of ? 1 : 0);
    }
    const uint32_t hot_at = a.win_n, dummy = a.win_n + 4u * kCodeHistHot + tid;
    const uint32_t hot_lo = a.radius - kCodeHistHot / 2u;
    for (uint32_t i = tid; i < a.win_n + 4u * kCodeHistHot; i += kCodeHistBlock) s_dyn_ch[i] = 0;
    __syncthreads();

    uint32_t *part = a.parts + (size_t)(blockIdx.x % a.copies) * a.nbins;
    uint32_t centre = 0, escapes = 0;
    auto count = [&](uint32_t code, bool on) {
        centre += (on && code == a.radius) ? 1u : 0u;
        escapes += (on && code == 0u) ? 1u : 0u;
        const bool mine = on && code != a.radius && code != 0u;
        const uint32_t hot = code - hot_lo, bin = code - a.win_lo;
        const bool in = bin < a.win_n;
        uint32_t at = hot < kCodeHistHot ? hot_at + 4u * hot + (lane & 3u) : bin;
        at = (mine && in) ? at : dummy;
        atomicAdd(&s_dyn_ch[at], 1u);
        if (wave_ballot(mine && !in) != 0ull) {      // (uniform)
            if (mine && !in) atomicAdd(&part[code], 1u);
        }
    };
    // not all: which of the eight codes from element e on are counted here (bit j: element e + j); a run has more than eight elements
    auto wanted = [&](uint32_t e) -> uint32_t {
        const uint32_t r = fdiv(e, a.divRun) - r0, at = e - (r + r0) * run_n;
        const uint32_t from = s_from[r];
        if (at + 8u <= run_n && (at >= from || at + 8u <= from)) return at >= from ? 0xffu : 0u;
        uint32_t m = 0;
        for (uint32_t j = 0; j < 8u; ++j)
            if (at + j >= run_n ? at + j - run_n >= s_from[r + 1u] : at + j >= from) m |= 1u << j;     // (the group lies in my slice: so does the next run)
        return m;
    };
    const uint4 *src = reinterpret_cast<const uint4 *>(a.codes);
    // (the loops are the same for every lane: the ballots in them want them all; the masks of the one cost it a tenth of its time)
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    if (!SHARED || all) {
        auto eight = [&](uint4 v, bool on) {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (int j = 0; j < 4; ++j) { count(w[j] & 0xffffu, on); count(w[j] >> 16, on); }
        };
        uint4 a0 = g0 + tid < g1 ? src[g0 + tid] : zero, a1 = g0 + tid + kCodeHistBlock < g1 ? src[g0 + tid + kCodeHistBlock] : zero;
        for (uint64_t g = g0; g < g1; g += 2u * kCodeHistBlock) {
            const uint4 v0 = a0, v1 = a1;
            const uint64_t i0 = g + tid, i1 = i0 + kCodeHistBlock, n0 = i0 + 2u * kCodeHistBlock, n1 = i1 + 2u * kCodeHistBlock;
            if (n0 < g1) a0 = src[n0];
            if (n1 < g1) a1 = src[n1];
            eight(v0, i0 < g1);
            eight(v1, i1 < g1);
        }
    } else {
        auto load = [&](uint64_t i, uint4 &v, uint32_t &m) {
            v = i < g1 ? src[i] : zero;
            m = i < g1 ? wanted((uint32_t)(i * 8u)) : 0u;
        };
        auto eight = [&](uint4 v, uint32_t m) {
            const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
            for (uint32_t j = 0; j < 4u; ++j) { count(w[j] & 0xffffu, (m >> (2u * j) & 1u) != 0u); count(w[j] >> 16, (m >> (2u * j + 1u) & 1u) != 0u); }
        };
        uint4 a0, a1;
        uint32_t m0, m1;
        load(g0 + tid, a0, m0);
        load(g0 + tid + kCodeHistBlock, a1, m1);
        for (uint64_t g = g0; g < g1; g += 2u * kCodeHistBlock) {
            const uint4 v0 = a0, v1 = a1;
            const uint32_t w0 = m0, w1 = m1;
            load(g + tid + 2u * kCodeHistBlock, a0, m0);
            load(g + tid + 3u * kCodeHistBlock, a1, m1);
            eight(v0, w0);
            eight(v1, w1);
        }
    }
    if (blockIdx.x == 0u && tid < (uint32_t)kWave) count(tail ? a.codes[i_tail] : 0u, tail_on);
    __syncthreads();
    for (uint32_t i = tid; i < a.win_n; i += kCodeHistBlock) {
        const uint32_t hot = a.win_lo + i - hot_lo;
        uint32_t v = s_win[i];
        if (hot < kCodeHistHot) v += s_hot[4u * hot] + s_hot[4u * hot + 1u] + s_hot[4u * hot + 2u] + s_hot[4u * hot + 3u];
        if (v) atomicAdd(&part[a.win_lo + i], v);
    }
    centre = wave_sum<uint32_t>(centre);
    escapes = wave_sum<uint32_t>(escapes);
    if (lane == 0) {
        if (centre) atomicAdd(&part[a.radius], centre);
        if (escapes) atomicAdd(&part[0], escapes);
    }
}

template __global__ void k_code_hist<true>(CodeHistArgs);
template __global__ void k_code_hist<false>(CodeHistArgs);

}  // namespace comet
