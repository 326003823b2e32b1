// Attention of one token's query heads over 16-row tiles of a cache, by the waves of a workgroup: the loop that the decode
// kernels share.
#pragma once

#include "common.h"

namespace rs {

// What a lane keeps: G running (m, l, o) over the rows of its row group, o over its 8 channels.
template <int G>
struct AttendState {
    float m[G], l[G], o[G][8];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int g = 0; g < G; ++g) {
            m[g] = -INFINITY;
            l[g] = 0.f;
#pragma unroll
            for (int c = 0; c < 8; ++c) o[g][c] = 0.f;
        }
    }
};

// The rows of a wave's step on their way: TPI tiles of 16 rows of K and V.
template <typename ST, int D, int TPI>
struct AttendStep {
    static constexpr int RPW = 64 / (D / 8), TR = 16, RPL = TR / RPW;
    typename Row8<ST>::raw_t k[TPI][RPL], v[TPI][RPL];
    int rows[TPI];  // valid rows of the tile, 0 .. 16 (0: none)

    // Tiles t .. t + TPI - 1 as far as they lie below te.  row_of(t): the tile's first row, or T_valid for none; called once
    // per tile, in order, by the whole wave (t, te: the same in all lanes).  The loads go through descriptors that end
    // with the last valid row of their tile, unconditionally: rows that do not exist come as zeros and count for nothing.
    // (Tiles of a last page may begin past T_valid, and a listed page may lie anywhere past it: a count below 0, which the
    // descriptor would take for 4 GB, or one cut to 32 bits would bring rows that are there, 0 times NaN among them.)
    template <bool STREAM, typename RowOf>
    __device__ __forceinline__ void load(const ST *kb, const ST *vb, long T_valid, long t, long te, RowOf row_of)
    {
        constexpr int AUX = STREAM ? 2 : 0, ROW = D * (int)sizeof(ST);
        const uint32_t at = (uint32_t)((threadIdx.x & 63) * 8 * (int)sizeof(ST));  // rows follow each other: the lane's place in RPW rows
        LdsSource kd[TPI], vd[TPI];
#pragma unroll
        for (int u = 0; u < TPI; ++u) {
            const long row0 = (t + u < te) ? row_of(t + u) : T_valid;
            const long left = T_valid - row0;
            rows[u] = left >= TR ? TR : left > 0 ? (int)left : 0;
            const long from = left > 0 ? row0 : 0;
            kd[u] = lds_source_sized(kb + from * D, rows[u] * ROW);
            vd[u] = lds_source_sized(vb + from * D, rows[u] * ROW);
        }
#pragma unroll
        for (int u = 0; u < TPI; ++u)
#pragma unroll
            for (int i = 0; i < RPL; ++i) k[u][i] = load_row8<ST, AUX>(kd[u], at + i * RPW * ROW);
#pragma unroll
        for (int u = 0; u < TPI; ++u)
#pragma unroll
            for (int i = 0; i < RPL; ++i) v[u][i] = load_row8<ST, AUX>(vd[u], at + i * RPW * ROW);
        // (they go out here: the compiler would put them off until the rows before them are done with)
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("" ::: "memory");
    }
};

// the rows of a step into a lane's state; the softmax moves its reference point once per step and head
template <typename ST, int D, int G, int TPI>
__device__ __forceinline__ void attend_one(const AttendStep<ST, D, TPI> &x, float scale, const RowDot<ST> (&qd)[G], AttendState<G> &st)
{
    constexpr int LPR = D / 8, RPW = 64 / LPR, RPL = 16 / RPW;
    const int rg = (threadIdx.x & 63) / LPR;
    float s[G][TPI][RPL];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float mt = st.m[g];
#pragma unroll
        for (int u = 0; u < TPI; ++u)
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                const float d = group_sum<LPR>(qd[g].dot(x.k[u][i])) * scale;
                s[g][u][i] = (i * RPW + rg < x.rows[u]) ? d : -INFINITY;
                mt = fmaxf(mt, s[g][u][i]);
            }
        const float ms = (mt == -INFINITY) ? 0.f : mt;  // nothing to attend yet: every weight below is 0
        const float corr = __expf(st.m[g] - ms);
        st.m[g] = mt;
        st.l[g] *= corr;
#pragma unroll
        for (int c = 0; c < 8; ++c) st.o[g][c] *= corr;
#pragma unroll
        for (int u = 0; u < TPI; ++u)
#pragma unroll
            for (int i = 0; i < RPL; ++i) {
                s[g][u][i] = __expf(s[g][u][i] - ms);
                st.l[g] += s[g][u][i];
            }
    }
#pragma unroll
    for (int u = 0; u < TPI; ++u)
#pragma unroll
        for (int i = 0; i < RPL; ++i) {
            float y[8];
            Row8<ST>::unpack(x.v[u][i], y);
#pragma unroll
            for (int g = 0; g < G; ++g)
#pragma unroll
                for (int c = 0; c < 8; ++c) st.o[g][c] = fmaf(s[g][u][i], y[c], st.o[g][c]);
        }
}

// Tiles t0, t0 + 1, ... + TPI - 1, whose rows are on their way in xa, then `stride` on, as far as they lie below te.  A wave
// has the next step's rows on their way while it works on the current ones: a tile of bfloat16 rows of 128 channels is 8 KB and
// 32 registers a step.
// (kb, vb: not through restricted pointers, which would let the compiler move the loads.)  in_last_step(): called before the
// arithmetic of the wave's last step.
struct NoLastStep {
    __device__ __forceinline__ void operator()() const {}
};
template <typename ST, int D, int G, int TPI, bool STREAM, typename RowOf, typename Last = NoLastStep>
__device__ __forceinline__ void attend_tiles(const ST *kb, const ST *vb, long T_valid, long t0, long te, long stride, float scale,
                                             const RowDot<ST> (&qd)[G], AttendState<G> &st, AttendStep<ST, D, TPI> &xa, RowOf row_of,
                                             Last in_last_step = Last())
{
    using Step = AttendStep<ST, D, TPI>;
    auto attend = [&](const Step &x) __attribute__((always_inline)) { attend_one<ST, D, G, TPI>(x, scale, qd, st); };
    if (t0 >= te) return;
    Step xb;
    for (long t = t0;;) {
        xb.template load<STREAM>(kb, vb, T_valid, t + stride, te, row_of);
        if (t + stride >= te) in_last_step();
        attend(xa);
        t += stride;
        if (t >= te) break;
        xa.template load<STREAM>(kb, vb, T_valid, t + stride, te, row_of);
        if (t + stride >= te) in_last_step();
        attend(xb);
        t += stride;
        if (t >= te) break;
    }
}
template <typename ST, int D, int G, int TPI, bool STREAM, typename RowOf, typename Last = NoLastStep>
__device__ __forceinline__ void attend_tiles(const ST *kb, const ST *vb, long T_valid, long t0, long te, long stride, float scale,
                                             const RowDot<ST> (&qd)[G], AttendState<G> &st, RowOf row_of, Last in_last_step = Last())
{
    AttendStep<ST, D, TPI> xa;
    xa.template load<STREAM>(kb, vb, T_valid, t0, te, row_of);
    attend_tiles<ST, D, G, TPI, STREAM>(kb, vb, T_valid, t0, te, stride, scale, qd, st, xa, row_of, in_last_step);
}

// The same a step at a time, for kernels whose other waves on the SIMD (four in all) fill the wait.
template <typename ST, int D, int G, int TPI, bool STREAM, typename RowOf, typename Last = NoLastStep>
__device__ __forceinline__ void attend_tiles_in_turn(const ST *kb, const ST *vb, long T_valid, long t0, long te, long stride, float scale,
                                                     const RowDot<ST> (&qd)[G], AttendState<G> &st, RowOf row_of, Last in_last_step = Last())
{
    for (long t = t0; t < te; t += stride) {
        AttendStep<ST, D, TPI> x;
        x.template load<STREAM>(kb, vb, T_valid, t, te, row_of);
        if (t + stride >= te) in_last_step();
        attend_one<ST, D, G, TPI>(x, scale, qd, st);
    }
}

// A wave's entries of a page list, one per lane, fetched 64 at a time: entry n is that of the n-th tile the wave takes.
// fetch(n): the word of that tile's page (>= 0), or -1 for none.
struct WavePages {
    int page = -1;
    int n = 0;
    template <typename Fetch>
    __device__ __forceinline__ int next(Fetch fetch)
    {
        if ((n & 63) == 0) {
            page = fetch(n + (int)(threadIdx.x & 63));
            asm volatile("" : "+v"(page));  // (waited for here, and not by every step)
        }
        return __builtin_amdgcn_readlane(page, n++ & 63);
    }
};

}  // namespace rs
