// The decode-time append of one or a few tokens by one thread per (batch, KV head, channel): the recurrence's step, the stored row
// and its page's bounds.
#pragma once

#include "common.h"

namespace rs {

// what a step appends, and to where (storage type and channels: the shape's)
struct StepToken {
    const void *k, *v;
    const float *g;
    float *state_k, *state_v;
    void *k_cache, *v_cache;
    long Tcap;
};

// Element e = (batch * KV heads + head) * D + channel.  pos_state: the replayable step's words (the write position is the token
// count they hold; the step is refused, and nothing written, past T_max or with fewer pages than K_min_pages), or nullptr.
// Nothing but trips to memory: a token's loads, its page's bounds among them, all go out before the first value is needed,
// and the stored key enters the bounds from its register instead of by way of the cache row just
// written (one trip instead of three: 3.8 -> 2.8 us for 8 x 32 heads of 128 channels, and a
// decode step at 4096 tokens 22.1 -> 21.5 us).
template <typename ST>
__device__ __forceinline__ void append_element(uint32_t e, const ST *__restrict__ k, const ST *__restrict__ v, const float *__restrict__ g,
                                               float *__restrict__ state_k, float *__restrict__ state_v, ST *__restrict__ k_cache,
                                               ST *__restrict__ v_cache, ST *__restrict__ meta, int P, int D, long T_new, long t0,
                                               long Tcap, const uint32_t *__restrict__ pos_state, long T_max, int K_min_pages)
{
    const uint32_t bh = e / (uint32_t)D, c = e % (uint32_t)D;
    float sk = state_k[e], sv = state_v[e];
    const long in0 = (long)bh * T_new * D + c;
    float gg = g[in0];
    ST kx = k[in0], vx = v[in0];
    if (pos_state) {  // replayable step: the write position is the workspace's token count
        t0 = *reinterpret_cast<const long *>(pos_state + kCtrlStateT);
        // a step the attention kernel of the same call will refuse (past T_max, or fewer pages than
        // it must select) appends nothing either: the refused step leaves carries, caches and page
        // bounds as they were, and the attention kernel reports it
        if (t0 + T_new > T_max || (t0 + T_new + P - 1) / P < (long)K_min_pages) return;
    }
    const uint32_t shift = meta ? (uint32_t)__builtin_ctz((unsigned)P) : 0u;  // P is a power of two
    ST lo_b, hi_b;  // the bounds so far of the page of the row at hand, as stored
    if (meta && (t0 & (P - 1)) != 0) {
        const ST *mn = meta + (((long)bh * (Tcap >> shift) + (t0 >> shift)) * 2) * D + c;
        lo_b = mn[0];
        hi_b = mn[D];
    }
    for (long t = 0; t < T_new; ++t) {
        const float om = 1.f - gg;
        sk = fmaf(gg, sk, om * to_f32(kx));
        sv = fmaf(gg, sv, om * to_f32(vx));
        if (t + 1 < T_new) {
            const long off = in0 + (t + 1) * D;
            gg = g[off];
            kx = k[off];
            vx = v[off];
        }
        const long row = t0 + t, o = ((long)bh * Tcap + row) * D + c;
        ST ks, vs;
        from_f32(ks, sk);
        from_f32(vs, sv);
        k_cache[o] = ks;
        v_cache[o] = vs;
        if (meta) {
            // Quest page min/max of the stored key: a page's first row starts it, later rows fold in
            const float x = to_f32(ks);
            float lo = x, hi = x;
            if ((row & (P - 1)) != 0) {
                lo = fminf(to_f32(lo_b), x);
                hi = fmaxf(to_f32(hi_b), x);
            }
            from_f32(lo_b, lo);
            from_f32(hi_b, hi);
            ST *mn = meta + (((long)bh * (Tcap >> shift) + (row >> shift)) * 2) * D + c;
            mn[0] = lo_b;
            mn[D] = hi_b;
        }
    }
    state_k[e] = sk;
    state_v[e] = sv;
}

}  // namespace rs
