// Outlier records in element order (COMET Sec. 2.2: every element within the bound).  The quantise kernel has left the
// records of every run of rows, in order, in the run's staging area, and the number of them per run and per workgroup;
// a wavefront adds up what is in front of its run and copies the run's records to their place in the container.  It runs
// beside the code book (further workgroups of k_codebook): a kernel of its own between the two cost every compression 5 to 6 us.
#pragma once
#include "comet_kernels.h"

namespace comet {

namespace {

constexpr uint32_t kDeriveBuf = 256;

// Sum of counts[0, n) by one wavefront (uniform), eight loads in flight per lane.
__device__ inline uint64_t wave_total(const uint32_t *counts, uint32_t n, uint32_t lane) {
    uint64_t sum = 0;
    for (uint32_t i0 = 0; i0 < n; i0 += 8u * kWave) {
        uint32_t v[8];
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) {
            const uint32_t i = i0 + j * kWave + lane;
            v[j] = (i < n) ? counts[i] : 0u;
        }
#pragma unroll
        for (uint32_t j = 0; j < 8; ++j) sum += v[j];
    }
    return wave_sum<uint64_t>(sum);
}

// Totals over the whole tensor: kind 0 records, 1 non-zero inputs, 2 verbatim records.
__device__ inline uint64_t record_total(const RecordArgs &a, uint32_t kind, uint32_t lane) {
    return wave_total(a.run_count + a.n_wg * kQuantWaves + kind * a.n_wg, a.n_wg, lane);
}

// The records of a run that has more of them than its staging area holds, derived again from the input, 256 consecutive
// elements at a time, four per lane (in element order: lanes, a lane's elements, escape before verbatim), straight into their
// place dst[0 .. room).  Bound by instruction issue: two loads and two quantisations per element (what is to the left is the
// lane's own or the lane's to the left).  Two steps alternate, the loads of one in flight while the other is worked on; the
// records leave through a buffer in LDS (s_buf: kDeriveBuf of them per wavefront), in bulk: stored one by one where they
// belong, a quarter of 51 M elements took 160 us whatever the rest of the loop did.
// IN: element type (0 fp32, 1 IEEE half, 2 bfloat16).
template <int IN>
__device__ inline void derive_records(const RecordArgs &a, uint32_t run, uint32_t lane, uint32_t count, uint2 *dst, uint64_t room, uint2 *s_buf) {
    constexpr uint32_t V = 4, kStep = V * kWave;             // elements per lane and step
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    const uint32_t W = a.divW.d, H = a.divH.d;
    const uint64_t wg_lo = (uint64_t)(run / kQuantWaves) * a.wg_elems, wg_hi = wg_lo + a.wg_elems < a.n ? wg_lo + a.wg_elems : a.n;
    const uint64_t run_lo = wg_lo + run % kQuantWaves * a.run_elems;
    const uint32_t e_lo = (uint32_t)run_lo, e_hi = (uint32_t)(run_lo + a.run_elems < wg_hi ? run_lo + a.run_elems : wg_hi);       // (a run with records begins inside the tensor)
    const float eb_lo = a.eb * (1.0f - 0x1p-20f);            // (an fp32 error above needs the exact comparison)
    const uint32_t fits = room < count ? (uint32_t)room : count;
    auto elem = [&](uint32_t i) -> float {
        if (IN == 0) return static_cast<const float *>(a.x)[i];
        const uint32_t v = static_cast<const unsigned short *>(a.x)[i];
        return IN == 1 ? (float)__builtin_bit_cast(_Float16, (unsigned short)v) : __uint_as_float(v << 16);
    };
    auto left_of = [&](int32_t v) { return __builtin_amdgcn_update_dpp(0, v, 0x138, 0xf, 0xf, true); };   // wave_shr:1
    // column and row (inside its plane) of my first element; a step on they are dcol and drow_h further
    uint32_t w, h;
    {
        const uint32_t e = e_lo + lane * V, row = fdiv(e, a.divW);
        w = e - row * W;
        h = row - fdiv(row, a.divH) * H;
    }
    const uint32_t drow = fdiv(kStep, a.divW), dcol = kStep - drow * W, drow_h = drow - fdiv(drow, a.divH) * H;
    uint32_t cur = 0, buffered = 0;                          // records in their place, in the buffer (uniform)
    auto flush = [&]() {
        wave_lds_fence();
        for (uint32_t i = lane; i < buffered; i += kWave)
            if (cur + i < fits) dst[cur + i] = s_buf[i];
        wave_lds_fence();
        cur += buffered;
        buffered = 0;
    };
    int32_t carry = 0, carry_u = 0;                          // minus what lane 63 held last, one step back: the left neighbours of lane 0
    if (e_lo - fdiv(e_lo, a.divW) * W != 0u) {               // (a run that begins inside a row; the lane's masks drop what is not there)
        auto quant = [&](float v) -> int32_t { const float t = v * a.r; return (fabsf(t) < 16777216.0f) ? (int32_t)rintf(t) : 0; };
        carry = -quant(elem(e_lo - 1u));
        carry_u = e_lo > W ? -quant(elem(e_lo - 1u - W)) : 0;
    }
    auto fetch = [&](uint32_t e0, float (&x)[V], float (&up)[V]) {
        const uint32_t e = e0 + lane * V;
        if (IN == 0 && e0 >= W && e0 + kStep <= e_hi) {      // (uniform; everything is inside the tensor)
            const f32x4 vx = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.x) + e);
            const f32x4 vu = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.x) + (e - W));
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) { x[j] = vx[j]; up[j] = vu[j]; }
        } else {
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                const uint32_t at = e + j < e_hi ? e + j : e_hi - 1u;
                x[j] = elem(at);
                up[j] = elem(at >= W ? at - W : 0u);
            }
        }
    };
    auto work = [&](uint32_t e0, const float (&x)[V], const float (&up)[V]) {
        const uint32_t e = e0 + lane * V;
        int32_t q[V], qu[V];
        float qf[V];
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            const float t = x[j] * a.r, tu = up[j] * a.r;
            qf[j] = (fabsf(t) < 16777216.0f) ? rintf(t) : 0.0f;
            q[j] = (int32_t)qf[j];
            qu[j] = (fabsf(tu) < 16777216.0f) ? (int32_t)rintf(tu) : 0;
        }
        // (minus the left neighbours: shifted values are combined with additions only)
        int32_t nql = left_of(-q[V - 1]), nqul = left_of(-qu[V - 1]);
        nql = lane == 0u ? carry : nql;
        nqul = lane == 0u ? carry_u : nqul;
        carry = __builtin_amdgcn_readlane(-q[V - 1], 63); carry_u = __builtin_amdgcn_readlane(-qu[V - 1], 63);
        uint32_t d[V], wj = w, hj = h;
        bool esc[V];
        uint64_t em[V], any_v = 0ull;
        bool susp[V];
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            const uint32_t rd = (uint32_t)q[j] + (wj ? (uint32_t)nql : 0u), above = (uint32_t)qu[j] + (wj ? (uint32_t)nqul : 0u);
            nql = -q[j]; nqul = -qu[j];
            d[j] = rd - (hj ? above : 0u);
            ++wj;
            hj += wj == W ? 1u : 0u;
            wj = wj == W ? 0u : wj;
            hj = hj == H ? 0u : hj;
            const bool on = e + j < e_hi;
            const uint32_t c = d[j] + (uint32_t)a.radius;
            esc[j] = !((c - 1u) < a.nbins - 1u);
            if (a.reuse_len) esc[j] = esc[j] || a.reuse_len[esc[j] ? 0u : c] == 0;      // no code word in the given table
            esc[j] = esc[j] && on;
            em[j] = wave_ballot(esc[j]);
            susp[j] = !(fabsf(x[j] - qf[j] * a.ebx2) <= eb_lo) && on;
            any_v |= wave_ballot(susp[j]);
        }
        w += dcol; h += drow_h;
        h += w >= W ? 1u : 0u;
        w -= w >= W ? W : 0u;
        h -= h >= H ? H : 0u;
        uint32_t before = 0, add = 0;                        // records of the lanes below me, of the step
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            before += __builtin_amdgcn_mbcnt_hi((uint32_t)(em[j] >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)em[j], 0u));
            add += (uint32_t)__popcll(em[j]);
        }
        bool verb[V];
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) verb[j] = false;
        if (any_v != 0ull) {                                 // some element may miss the bound: the exact comparison
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                verb[j] = susp[j] && (!(fabsf(x[j] * a.r) < 16777216.0f) || !(fabs((double)x[j] - (double)((float)q[j] * a.ebx2)) <= (double)a.eb));
                const uint64_t vm = wave_ballot(verb[j]);
                before += __builtin_amdgcn_mbcnt_hi((uint32_t)(vm >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)vm, 0u));
                add += (uint32_t)__popcll(vm);
            }
        }
        if (add == 0u) return;                               // (uniform)
        if (buffered + add > kDeriveBuf) flush();
        const bool direct = add > kDeriveBuf;                // (uniform: more than the buffer holds, nearly every element has records)
        uint32_t pos = direct ? cur + before : buffered + before;
        auto put = [&](uint32_t key, uint32_t val) {
            if (!direct) s_buf[pos] = make_uint2(key, val);
            else if (pos < fits) dst[pos] = make_uint2(key, val);
            ++pos;
        };
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            if (esc[j]) put(2u * (e + j), d[j]);
            if (verb[j]) put(2u * (e + j) + 1u, __float_as_uint(x[j]));
        }
        if (direct) cur += add; else buffered += add;
    };
    float xa[V], ua[V], xb[V], ub[V];
    fetch(e_lo, xa, ua);
    for (uint32_t e0 = e_lo; e0 < e_hi; e0 += 2u * kStep) {
        fetch(e0 + kStep, xb, ub);
        work(e0, xa, ua);
        fetch(e0 + 2u * kStep, xa, ua);
        work(e0 + kStep, xb, ub);
    }
    flush();
    if (fits < count && lane == 0) atomicOr(&a.ctl->status, (uint32_t)ST_CAPACITY);
}

// The records of one run, by one wavefront (s_buf: kDeriveBuf records of LDS).
__device__ inline void place_records(const RecordArgs &a, uint32_t run, uint32_t lane, uint2 *s_buf) {
    const uint32_t n_runs = a.n_wg * kQuantWaves;
    if (run >= n_runs) return;
    const uint32_t mine = a.run_count[run];
    if (!mine) return;
    const uint32_t wg = run / kQuantWaves;
    uint64_t base = wave_total(a.run_count + n_runs, wg, lane);             // the workgroups in front ...
    for (uint32_t r = wg * kQuantWaves; r < run; ++r) base += a.run_count[r];   // ... and the runs in front in mine
    uint2 *dst = reinterpret_cast<uint2 *>(a.rec) + base;
    const uint64_t room = (base < a.rec_cap) ? a.rec_cap - base : 0ull;
    if (mine <= a.rec_run) {
        const uint2 *src = reinterpret_cast<const uint2 *>(a.stage) + (size_t)run * a.rec_run;
        for (uint32_t i = lane; i < mine; i += kWave)
            if (i < room) dst[i] = src[i];
        if (mine > room && lane == 0) atomicOr(&a.ctl->status, (uint32_t)ST_CAPACITY);
    } else {
        if (a.in_type == 0u) derive_records<0>(a, run, lane, mine, dst, room, s_buf);
        else if (a.in_type == 1u) derive_records<1>(a, run, lane, mine, dst, room, s_buf);
        else derive_records<2>(a, run, lane, mine, dst, room, s_buf);
    }
}

}  // namespace

}  // namespace comet
