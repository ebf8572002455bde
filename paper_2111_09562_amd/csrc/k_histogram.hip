// Histogram of the quantisation codes of an alphabet too large for the LDS window of the quantise kernel.
//
// The codes come back from memory (2 bytes each, mostly out of the last-level cache) and are counted with the whole LDS
// of a compute unit: one workgroup of sixteen wavefronts per compute unit, 32-bit counters for kCodeHistWindow bins around the
// centre, four copies of the kCodeHistHot innermost ones (lanes that meet in one bin mostly use different copies).  The
// centre bin and the escape symbol are counted in registers; what lies outside the window, far out in the tails, goes to
// the partial histogram in global memory.  At the end a workgroup adds its bins to one of the partial histograms,
// neighbouring lanes neighbouring bins; workgroups of one XCD (consecutive ones go round the XCDs) share a copy, so
// that its lines stay in that XCD's L2.
// (In the quantise kernel itself, with a window of 8192 bins and everything else listed and added to global memory, a
// tensor of 64 x 256 x 56 x 56 at a bound of 1e-4 and 65536 bins took 356 us, nearly all of it in those additions; now
// 59 us and 65 us here.)
#include "comet_kernels.h"

namespace comet {

__global__ __launch_bounds__(kCodeHistBlock) void k_code_hist(CodeHistArgs a) {
    extern __shared__ uint32_t s_dyn_ch[];          // a.win_n bins; kCodeHistHot x 4 (the innermost bins); a word per thread for what is not counted here
    uint32_t *s_win = s_dyn_ch;
    uint32_t *s_hot = s_dyn_ch + a.win_n;
    const uint32_t tid = threadIdx.x, lane = (uint32_t)lane_id();
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
    // A slice of consecutive groups of eight codes per workgroup, two groups per thread in flight.
    const uint64_t groups = a.n / 8u;
    const uint64_t per = (groups + gridDim.x - 1u) / gridDim.x;
    const uint64_t g0 = (uint64_t)blockIdx.x * per;
    const uint64_t g1 = g0 + per < groups ? g0 + per : groups;
    const uint4 *src = reinterpret_cast<const uint4 *>(a.codes);
    auto eight = [&](uint4 v, bool on) {
        const uint32_t w[4] = {v.x, v.y, v.z, v.w};
#pragma unroll
        for (int j = 0; j < 4; ++j) { count(w[j] & 0xffffu, on); count(w[j] >> 16, on); }
    };
    // (the loop is the same for every lane: the ballots in it want them all)
    const uint4 zero = make_uint4(0u, 0u, 0u, 0u);
    uint4 a0 = g0 + tid < g1 ? src[g0 + tid] : zero, a1 = g0 + tid + kCodeHistBlock < g1 ? src[g0 + tid + kCodeHistBlock] : zero;
    for (uint64_t g = g0; g < g1; g += 2u * kCodeHistBlock) {
        const uint4 v0 = a0, v1 = a1;
        const uint64_t i0 = g + tid, i1 = i0 + kCodeHistBlock, n0 = i0 + 2u * kCodeHistBlock, n1 = i1 + 2u * kCodeHistBlock;
        if (n0 < g1) a0 = src[n0];
        if (n1 < g1) a1 = src[n1];
        eight(v0, i0 < g1);
        eight(v1, i1 < g1);
    }
    if (blockIdx.x == 0 && tid < (uint32_t)kWave) {                  // fewer than eight codes are left
        const uint64_t i = groups * 8u + tid;
        count(i < a.n ? a.codes[i] : 0u, i < a.n);
    }
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

}  // namespace comet
