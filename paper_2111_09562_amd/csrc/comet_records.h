// Outlier records in element order (COMET Sec. 2.2: every element within the bound).  The quantise kernel has left the
// records of every run of rows, in order, in the run's staging area, and the number of them per run and per workgroup;
// a wavefront adds up what is in front of its run and copies the run's records to their place in the container.  It runs
// beside the code book (further workgroups of k_codebook): a kernel of its own between the two cost every compression 5 to 6 us.
#pragma once
#include "comet_kernels.h"

namespace comet {

namespace {

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

// The records of a run that has more of them than its staging area holds, from the first one behind those (whose last key is
// last_key), derived again from the input, 256 consecutive elements at a time, four per lane (in element order: lanes, a lane's
// elements, escape before verbatim), straight into their place dst[held .. min(room, count)).
// Bound by instruction issue (four wavefronts per SIMD in the code book kernel), so few of them: one load and one
// quantisation per element (RING: what the row below needs stays in LDS, the last a.ring >= W + 256 differences between an
// element and the one to its left; planes without room for that load and quantise the row above once more), lane masks in
// scalar registers instead of a truth value per lane, no test for the ends of the range in the steps between.  The loads of
// a batch of steps are in flight while the batch before is worked on; the records leave through a buffer in LDS (s_buf:
// kDeriveBuf of them per wavefront, the ring behind it), in bulk: stored one by one where they belong, a quarter of 51 M elements took
// 160 us whatever the rest of the loop did.  64 x 256 x 56 x 56 with 21 % records 268 us -> 226 (row above loaded again, two
// steps in flight, truth values), 411 M elements 2201 -> 1716.
// IN: element type (0 fp32, 1 IEEE half, 2 bfloat16, -1 any).  U: steps per batch of loads: four, or two in k_place_payload, which
// then needs 60 registers instead of 78: eight wavefronts per SIMD instead of six, also where nothing is derived (five layers
// on five streams with their code books given 1460 -> 1486 GB/s; 21 % records 254 us -> 257).
template <int IN, bool RING, uint32_t U>
__device__ __forceinline__ void derive_records(const RecordArgs &a, uint32_t run, uint32_t lane, uint32_t held, uint32_t last_key, uint32_t count,
                                      uint2 *dst, uint64_t room, uint2 *s_buf) {
    constexpr uint32_t V = 4, kStep = V * kWave;             // elements per lane and step
    constexpr uint32_t kBatch = U * kStep;
    typedef float f32x4 __attribute__((ext_vector_type(4), aligned(4)));
    typedef unsigned short u16x4 __attribute__((ext_vector_type(4), aligned(2)));
    typedef int32_t i32x4 __attribute__((ext_vector_type(4)));
    const uint32_t W = a.divW.d, H = a.divH.d;
    const uint64_t wg_lo = (uint64_t)(run / kQuantWaves) * a.wg_elems, wg_hi = wg_lo + a.wg_elems < a.n ? wg_lo + a.wg_elems : a.n;
    const uint64_t run_lo = wg_lo + run % kQuantWaves * a.run_elems;
    const uint32_t e_hi = (uint32_t)(run_lo + a.run_elems < wg_hi ? run_lo + a.run_elems : wg_hi);       // (a run with records begins inside the tensor)
    // the first elements whose escape, whose verbatim value is not staged; the step they are in, and with the ring the row above it
    const uint32_t esc_lo = (last_key >> 1) + 1u, verb_lo = (last_key + 1u) >> 1;
    uint32_t e_lo = (uint32_t)run_lo + ((last_key >> 1) - (uint32_t)run_lo) / kStep * kStep;
    if (RING) {
        const uint32_t back = (W + kStep - 1u) / kStep * kStep;
        e_lo = e_lo > back ? e_lo - back : 0u;
    }
    const float eb_lo = a.eb * (1.0f - 0x1p-20f);            // (an fp32 error above needs the exact comparison)
    const uint32_t fits = room < count ? (uint32_t)room : count;
    int32_t *ring = reinterpret_cast<int32_t *>(s_buf + kDeriveBuf);
    const uint32_t ring_mask = a.ring * 4u - 1u;             // (of byte offsets)
    auto widen = [&](uint32_t v) -> float {
        return IN == 1 || (IN < 0 && a.in_type == 1u) ? (float)__builtin_bit_cast(_Float16, (unsigned short)v) : __uint_as_float(v << 16);
    };
    auto elem = [&](uint32_t i) -> float {
        if (IN == 0 || (IN < 0 && a.in_type == 0u)) return static_cast<const float *>(a.x)[i];
        return widen(static_cast<const unsigned short *>(a.x)[i]);
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
    uint32_t cur = held, buffered = 0;                       // records in their place, in the buffer (uniform)
    auto flush = [&]() {
        wave_lds_fence();
        for (uint32_t i = lane; i < buffered; i += kWave)
            if (cur + i < fits) dst[cur + i] = s_buf[i];
        wave_lds_fence();
        cur += buffered;
        buffered = 0;
    };
    int32_t carry = 0, carry_u = 0;                          // minus what lane 63 held last, one step back: the left neighbours of lane 0
    if (e_lo - fdiv(e_lo, a.divW) * W != 0u) {               // (it begins inside a row; the lane's masks drop what is not there)
        auto quant = [&](float v) -> int32_t { const float t = v * a.r; return (fabsf(t) < 16777216.0f) ? (int32_t)rintf(t) : 0; };
        carry = -quant(elem(e_lo - 1u));
        if (!RING) carry_u = e_lo > W ? -quant(elem(e_lo - 1u - W)) : 0;
    }
    auto fetch = [&](uint32_t e0, float (&x)[V], float (&up)[RING ? 1 : V]) __attribute__((always_inline)) {
        const uint32_t e = e0 + lane * V;
        if (e0 >= e_hi) {                                    // (uniform; not looked at)
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) { x[j] = 0.0f; if (!RING) up[RING ? 0 : j] = 0.0f; }
        } else if (e0 + kStep <= e_hi && (RING || (e0 >= W && a.in_type == 0u))) {      // (uniform; everything is inside the tensor)
            if (IN <= 0) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.x) + e);
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) x[j] = v[j];
            } else {
                const u16x4 v = *reinterpret_cast<const u16x4 *>(static_cast<const unsigned short *>(a.x) + e);
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) x[j] = widen(v[j]);
            }
            if (!RING) {
                const f32x4 v = *reinterpret_cast<const f32x4 *>(static_cast<const float *>(a.x) + (e - W));
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) up[RING ? 0 : j] = v[j];
            }
        } else {
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                const uint32_t at = e + j < e_hi ? e + j : e_hi - 1u;
                x[j] = elem(at);
                if (!RING) up[RING ? 0 : j] = elem(at >= W ? at - W : 0u);
            }
        }
    };
    auto ring_fence = [] { __builtin_amdgcn_fence(__ATOMIC_ACQ_REL, "wavefront", "local"); };     // (a wavefront's LDS accesses arrive in order: for the compiler)
    const bool whole4 = (W & 3u) == 0u;                      // (uniform) a lane's elements lie in one row: e_lo is a multiple of four as well
    auto work = [&](uint32_t e0, const float (&x)[V], const float (&up)[RING ? 1 : V]) __attribute__((always_inline)) {
        const uint32_t e = e0 + lane * V;
        const bool produces = e0 + kStep > verb_lo;          // (uniform) or the row above is only taken in
        int32_t q[V];
        float qf[V];
        uint32_t d[V];
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            const float t = x[j] * a.r;
            qf[j] = (fabsf(t) < 16777216.0f) ? rintf(t) : 0.0f;
            q[j] = (int32_t)qf[j];
        }
        // (minus the left neighbours: shifted values are combined with additions only)
        int32_t nql = left_of(-q[V - 1]);
        nql = lane == 0u ? carry : nql;
        carry = __builtin_amdgcn_readlane(-q[V - 1], 63);
        if constexpr (RING) {
            uint8_t *at = reinterpret_cast<uint8_t *>(ring);
            const uint32_t i = (e - e_lo) * 4u;
            if (whole4) {
                const i32x4 rd = {q[0] + (w ? nql : 0), q[1] - q[0], q[2] - q[1], q[3] - q[2]};
                *reinterpret_cast<i32x4 *>(at + (i & ring_mask)) = rd;
                ring_fence();
                const i32x4 up_rd = *reinterpret_cast<const i32x4 *>(at + ((i - 4u * W) & ring_mask));
                const uint32_t above = h ? ~0u : 0u;         // is there a row above
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) d[j] = (uint32_t)rd[j] - ((uint32_t)up_rd[j] & above);
            } else {
                // at least five columns: one row at most begins among my elements, at the p-th
                const uint32_t p = w ? W - w : 0u;
                const uint32_t h_p = w ? (h + 1u == H ? 0u : h + 1u) : h;
                i32x4 rd;
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) {
                    rd[j] = q[j] + (j == p ? 0 : nql);
                    nql = -q[j];
                }
                *reinterpret_cast<i32x4 *>(at + (i & ring_mask)) = rd;
                ring_fence();
#pragma unroll
                for (uint32_t j = 0; j < V; ++j) {
                    const uint32_t up_rd = *reinterpret_cast<const uint32_t *>(at + ((i + 4u * j - 4u * W) & ring_mask));
                    d[j] = (uint32_t)rd[j] - ((j < p ? h : h_p) ? up_rd : 0u);
                }
            }
            ring_fence();
        } else {
            int32_t qu[V];
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                const float tu = up[RING ? 0 : j] * a.r;
                qu[j] = (fabsf(tu) < 16777216.0f) ? (int32_t)rintf(tu) : 0;
            }
            int32_t nqul = left_of(-qu[V - 1]);
            nqul = lane == 0u ? carry_u : nqul;
            carry_u = __builtin_amdgcn_readlane(-qu[V - 1], 63);
            uint32_t wj = w, hj = h;
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                const uint32_t rd = (uint32_t)q[j] + (wj ? (uint32_t)nql : 0u), above = (uint32_t)qu[j] + (wj ? (uint32_t)nqul : 0u);
                nql = -q[j]; nqul = -qu[j];
                d[j] = rd - (hj ? above : 0u);
                ++wj;
                hj += wj == W ? 1u : 0u;
                wj = wj == W ? 0u : wj;
                hj = hj == H ? 0u : hj;
            }
        }
        w += dcol; h += drow_h;
        h += w >= W ? 1u : 0u;
        w -= w >= W ? W : 0u;
        h -= h >= H ? H : 0u;
        if (!produces) return;
        // (masks of lanes, not a truth value per lane: what is decided behind a uniform branch stays scalar)
        uint64_t em[V], vm[V], any_v = 0ull;
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) {
            em[j] = wave_ballot(d[j] + ((uint32_t)a.radius - 1u) >= a.nbins - 1u);
            vm[j] = wave_ballot(!(fabsf(x[j] - qf[j] * a.ebx2) <= eb_lo));
        }
        if (a.reuse_len) {                                   // no code word in the given table
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                const uint32_t c = d[j] + (uint32_t)a.radius;
                em[j] |= wave_ballot(a.reuse_len[c < a.nbins ? c : 0u] == 0);
            }
        }
        if (e0 < esc_lo || e0 + kStep > e_hi) {              // (uniform) the first or the last step of the range
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                em[j] &= wave_ballot(e + j - esc_lo < e_hi - esc_lo);
                vm[j] &= wave_ballot(e + j - verb_lo < e_hi - verb_lo);
            }
        }
        uint32_t before = 0, add = 0;                        // records of the lanes below me, of the step
        auto count = [&](uint64_t m) {
            before += __builtin_amdgcn_mbcnt_hi((uint32_t)(m >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u));
            add += (uint32_t)__popcll(m);
        };
#pragma unroll
        for (uint32_t j = 0; j < V; ++j) { count(em[j]); any_v |= vm[j]; }
        if (any_v != 0ull) {                                 // some element may miss the bound: the exact comparison
            any_v = 0ull;
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                vm[j] &= wave_ballot(!(fabsf(x[j] * a.r) < 16777216.0f) || !(fabs((double)x[j] - (double)((float)q[j] * a.ebx2)) <= (double)a.eb));
                any_v |= vm[j];
                count(vm[j]);
            }
        }
        if (add == 0u) return;                               // (uniform)
        if (buffered + add > kDeriveBuf) flush();
        // (add > kDeriveBuf: more than the buffer holds, nearly every element has records; they go to their place one by one)
        const bool direct = add > kDeriveBuf;
        uint32_t pos = direct ? cur + before : buffered + before;
        if (!direct && any_v == 0ull) {
#pragma unroll
            for (uint32_t j = 0; j < V; ++j)
                if (__builtin_amdgcn_inverse_ballot_w64(em[j])) s_buf[pos++] = make_uint2(2u * (e + j), d[j]);
        } else {
            auto put = [&](uint32_t key, uint32_t val) {
                if (!direct) s_buf[pos] = make_uint2(key, val);
                else if (pos < fits) dst[pos] = make_uint2(key, val);
                ++pos;
            };
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                if (__builtin_amdgcn_inverse_ballot_w64(em[j])) put(2u * (e + j), d[j]);
                if (__builtin_amdgcn_inverse_ballot_w64(vm[j])) put(2u * (e + j) + 1u, __float_as_uint(x[j]));
            }
        }
        if (direct) cur += add; else buffered += add;
    };
    float x[U][V], up[U][RING ? 1 : V], xn[U][V], upn[U][RING ? 1 : V];
#pragma unroll
    for (uint32_t u = 0; u < U; ++u) fetch(e_lo + u * kStep, xn[u], upn[u]);
    for (uint32_t e0 = e_lo; e0 < e_hi; e0 += kBatch) {
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) {
#pragma unroll
            for (uint32_t j = 0; j < V; ++j) {
                x[u][j] = xn[u][j];
                if (!RING) up[u][RING ? 0 : j] = upn[u][RING ? 0 : j];
            }
        }
#pragma unroll
        for (uint32_t u = 0; u < U; ++u) fetch(e0 + kBatch + u * kStep, xn[u], upn[u]);
#pragma unroll
        for (uint32_t u = 0; u < U; ++u)
            if (e0 + u * kStep < e_hi) work(e0 + u * kStep, x[u], up[u]);    // (uniform)
    }
    flush();
}

// The records of one run, by one wavefront (s_buf: record_lds(a.ring) bytes of LDS).
template <uint32_t U>
__device__ __forceinline__ void place_records(const RecordArgs &a, uint32_t run, uint32_t lane, uint2 *s_buf) {
    const uint32_t n_runs = a.n_wg * kQuantWaves;
    if (run >= n_runs) return;
    const uint32_t mine = a.run_count[run];
    if (!mine) return;
    const uint32_t wg = run / kQuantWaves;
    uint64_t base = wave_total(a.run_count + n_runs, wg, lane);             // the workgroups in front ...
    for (uint32_t r = wg * kQuantWaves; r < run; ++r) base += a.run_count[r];   // ... and the runs in front in mine
    uint2 *dst = reinterpret_cast<uint2 *>(a.rec) + base;
    const uint64_t room = (base < a.rec_cap) ? a.rec_cap - base : 0ull;
    const uint32_t held = mine < a.rec_run ? mine : a.rec_run;
    const uint2 *src = reinterpret_cast<const uint2 *>(a.stage) + (size_t)run * a.rec_run;
    for (uint32_t i = lane; i < held; i += kWave)
        if (i < room) dst[i] = src[i];
    if (mine > held && room > held) {                        // (uniform)
        const uint32_t last_key = (uint32_t)__builtin_amdgcn_readfirstlane((int)src[held - 1u].x);
        if (a.ring == 0u) derive_records<-1, false, (U + 1u) / 2u>(a, run, lane, held, last_key, mine, dst, room, s_buf);
        else if (a.in_type == 0u) derive_records<0, true, U>(a, run, lane, held, last_key, mine, dst, room, s_buf);
        else if (a.in_type == 1u) derive_records<1, true, U>(a, run, lane, held, last_key, mine, dst, room, s_buf);
        else derive_records<2, true, U>(a, run, lane, held, last_key, mine, dst, room, s_buf);
    }
    if (mine > room && lane == 0) atomicOr(&a.ctl->status, (uint32_t)ST_CAPACITY);
}

}  // namespace

}  // namespace comet
