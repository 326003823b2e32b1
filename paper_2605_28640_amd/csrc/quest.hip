// Quest at decode (App. A.1, Quest paragraph; Sec. 2.2, Eq. 3-4): page min/max
// representatives, page scores + top-K selection, and softmax attention over the
// selected pages (or over everything: the dense path).
//
// Lane mapping used throughout: a row of D channels is covered by LPR = D/8 lanes with
// 8 channels (one 16-byte bf16 load) each, so a wave touches RPW = 64/LPR rows per load
// instruction and every global access is a run of full 128/256-byte rows.
#include <cstdlib>
#include "append.h"
#include "attend.h"
#include "common.h"
#include "knobs.h"
#include "select.h"

namespace rs {

// ------------------------------------------------------------------------------------
// page metadata: one wave per page
// ------------------------------------------------------------------------------------
template <typename ST, int D>
__global__ __launch_bounds__(256) void quest_page_meta_kernel(const ST *__restrict__ k_cache,
                                                              ST *__restrict__ meta, long Tcap, int P,
                                                              int p_begin, int n_pages, long t_end,
                                                              int segs_per_wave)
{
    // A wave owns a run of whole pages and walks it in segments of 16 rows (every page size is
    // a multiple of 16), four segments' loads in flight at a time; a page's bounds are folded
    // across the row groups and written when its last segment has been taken in.
    constexpr int LPR = D / 8;
    constexpr int RPW = 64 / LPR;
    constexpr int U = 16 / RPW;  // row loads of a lane per segment
    constexpr int J = 4;         // segments in flight
    using R = Row8<ST>;
    const int lane = threadIdx.x & 63;
    const int wave = threadIdx.x >> 6;
    const int rg = lane / LPR;
    const int c0 = (lane % LPR) * 8;
    const long bh = blockIdx.y;
    const long Np_cap = Tcap / P;
    const int spp = P / 16;  // segments per page
    const long seg_end = (long)n_pages * spp;
    const long seg0 = ((long)blockIdx.x * 4 + wave) * segs_per_wave;
    if (seg0 >= seg_end) return;
    const long seg1 = (seg0 + segs_per_wave < seg_end) ? seg0 + segs_per_wave : seg_end;
    const long t_base = (long)p_begin * P;
    const ST *kb = k_cache + bh * Tcap * D + c0;

    float lo[8], hi[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        lo[c] = INFINITY;
        hi[c] = -INFINITY;
    }
    for (long sg = seg0; sg < seg1; sg += J) {
        typename R::raw_t x[J][U];
#pragma unroll
        for (int j = 0; j < J; ++j)
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long t = t_base + (sg + j) * 16 + u * RPW + rg;
                x[j][u] = (sg + j < seg1 && t < t_end) ? R::load_raw(kb + t * D) : R::zero_raw();
            }
#pragma unroll
        for (int j = 0; j < J; ++j) {
            if (sg + j >= seg1) break;
#pragma unroll
            for (int u = 0; u < U; ++u) {
                const long t = t_base + (sg + j) * 16 + u * RPW + rg;
                if (t < t_end) {
                    float v[8];
                    R::unpack(x[j][u], v);
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        lo[c] = fminf(lo[c], v[c]);
                        hi[c] = fmaxf(hi[c], v[c]);
                    }
                }
            }
            if ((sg + j + 1) % spp == 0) {  // the page is complete
#pragma unroll
                for (int m = LPR; m < 64; m <<= 1) {
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        lo[c] = fminf(lo[c], shfl_xor_f(lo[c], m));
                        hi[c] = fmaxf(hi[c], shfl_xor_f(hi[c], m));
                    }
                }
                const long p = p_begin + (sg + j) / spp;
                ST *mrow = meta + ((bh * Np_cap + p) * 2) * D + c0;
                if (rg == 0) R::store(mrow, lo);
                if (rg == 1) R::store(mrow + D, hi);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    lo[c] = INFINITY;
                    hi[c] = -INFINITY;
                }
            }
        }
    }
}

void page_meta_dispatch(int dtype, int D, const void *k_cache, void *meta, int BH, long Tcap, int P,
                        int p_begin, int n_pages, long t_end, hipStream_t stream)
{
    // whole pages per wave, four segments (16 KiB of bf16 rows at D = 128, every load in flight at
    // once) when the page size allows: measured on 2.4 GB of keys with 16-token pages, 1 / 2 / 4 /
    // 8 / 16 segments per wave give 4.0 / 5.1 / 5.4 / 5.3 / 5.0 TB/s
    const int spp = P / 16;
    const long segs = (long)n_pages * spp;
    int spw = 4;
    if (knobs().meta_spw != kKnobUnset && knobs().meta_spw > 0) spw = knobs().meta_spw;
    while (spw > 1 && (segs * BH) / spw < 8192) spw >>= 1;
    if (spw < spp) spw = spp;
    spw = (spw / spp) * spp;
    const long waves = (segs + spw - 1) / spw;
    const dim3 grid((unsigned)((waves + 3) / 4), (unsigned)BH);
    if (dtype == RS_BF16) {
        if (D == 128) quest_page_meta_kernel<bf16, 128><<<grid, 256, 0, stream>>>((const bf16 *)k_cache, (bf16 *)meta, Tcap, P, p_begin, n_pages, t_end, spw);
        else quest_page_meta_kernel<bf16, 64><<<grid, 256, 0, stream>>>((const bf16 *)k_cache, (bf16 *)meta, Tcap, P, p_begin, n_pages, t_end, spw);
    } else {
        if (D == 128) quest_page_meta_kernel<float, 128><<<grid, 256, 0, stream>>>((const float *)k_cache, (float *)meta, Tcap, P, p_begin, n_pages, t_end, spw);
        else quest_page_meta_kernel<float, 64><<<grid, 256, 0, stream>>>((const float *)k_cache, (float *)meta, Tcap, P, p_begin, n_pages, t_end, spw);
    }
}

constexpr int kSelThreads = 512;

// ------------------------------------------------------------------------------------
// page scores; the last workgroup of a unit to arrive runs the selection.  GQ = 1: a unit
// is a (batch, query head).  GQ = Hq / Hkv > 1 (group-shared selection, an option for
// grouped-query attention that is not in the paper): a unit is a (batch, KV head), the
// page score is the sum of the bounds of its GQ query heads and the list is theirs in common.
// ------------------------------------------------------------------------------------
template <typename ST, int D, int GQ>
__global__ __launch_bounds__(kSelThreads) void quest_score_select_kernel(
    const ST *__restrict__ q, const ST *__restrict__ meta, uint64_t *scores, float *scores_out, int32_t *idx_out,
    int Hq, int Hkv, long Np_cap, int Np, int K, int n_first, int n_local, int splits, uint32_t *unit_ctr,
    uint32_t *err, uint32_t tag, int spin_limit, const uint32_t *state, long T_max, int P)
{
    // state (the replayable decode step): the sequence length and the tag are not arguments but words of
    // the workspace (tokens in the cache + 1: the step's append has run); score rows keep the stride of T_max
    long np_stride = Np;
    if (state) {
        const long T_valid = *reinterpret_cast<const long *>(state + kCtrlStateT) + 1;
        tag = state[kCtrlStateTag];
        if (tag == 0u) tag = 0x5bd1e995u;
        Np = (int)((T_valid + P - 1) / P);
        np_stride = (T_max + P - 1) / P;
        if (T_valid > T_max || K > Np) {  // outside what the buffers were sized for: report, do nothing
            if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) atomicExch(err, 1u);
            return;
        }
    }
    constexpr int LPR = D / 8;
    constexpr int RPW = 64 / LPR;
    constexpr int UNR = 4;  // pages per lane in flight
    using R = Row8<ST>;
    __shared__ SelectShared<kSelThreads> sh;
    __shared__ int s_last;
    extern __shared__ uint32_t s_keys[];  // Np keys

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int rg = lane / LPR;
    const int c0 = (lane % LPR) * 8;
    const int unit = blockIdx.y;  // b * Hq + h (GQ = 1) or b * Hkv + kvh
    const int u0 = unit * GQ;     // first (batch, query head) of the unit
    const int b = u0 / Hq, h = u0 % Hq;
    const int kvh = h / (Hq / Hkv);
    const ST *mbase = meta + ((long)(b * Hkv + kvh) * Np_cap) * 2 * D;
    uint64_t *srow = scores + (long)unit * np_stride;

    float qv[GQ][8];
#pragma unroll
    for (int g = 0; g < GQ; ++g) R::load(q + (long)(u0 + g) * D + c0, qv[g]);
    BoundDot<ST> bound[GQ];
#pragma unroll
    for (int g = 0; g < GQ; ++g) bound[g].set(qv[g]);

    // this workgroup's pages: a contiguous slice, walked UNR * RPW pages per wave step.
    // The LPR lanes of a row group share their page numbers, so the group-local
    // shuffles only ever read active lanes.
    const int per = (Np + splits - 1) / splits;
    const int pb = blockIdx.x * per;
    const int pe = (pb + per < Np) ? pb + per : Np;
    constexpr int PPI = UNR * RPW * (kSelThreads / 64);  // pages per workgroup iteration
    for (int base = pb + wave * (UNR * RPW) + rg; base < pe; base += PPI) {
        typename R::raw_t mn[UNR], mx[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int p = base + u * RPW;
            if (p < pe) {
                mn[u] = R::load_raw(mbase + ((long)p * 2) * D + c0);
                mx[u] = R::load_raw(mbase + ((long)p * 2 + 1) * D + c0);
            } else {
                mn[u] = R::zero_raw();
                mx[u] = R::zero_raw();
            }
        }
        // lane u of a row group keeps page u's sum; the wave's UNR * RPW scores (adjacent words) then
        // leave with one store instruction
        float mine = 0.f;
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            float s = 0.f;
#pragma unroll
            for (int g = 0; g < GQ; ++g) s = bound[g].add(s, mn[u], mx[u]);
            s = group_sum<LPR>(s);
            if ((lane % LPR) == u) mine = s;
        }
        {
            const int p = base + (lane % LPR) * RPW;
            if ((lane % LPR) < UNR && p < pe) publish_f32(&srow[p], mine, tag);
        }
    }

    if (tid == 0) {
        const uint32_t prev = atomicAdd(&unit_ctr[unit], 1u);
        s_last = (prev == (uint32_t)splits - 1u);
        if (s_last) atomicExch(&unit_ctr[unit], 0u);  // every split has arrived: reset for the next call
    }
    __syncthreads();
    if (!s_last) return;

    gather_page_keys<kSelThreads>(srow, Np, n_first, n_local, tag, spin_limit, err,
                                  scores_out ? scores_out + (long)unit * Np : nullptr, s_keys);
    int32_t *dst = idx_out + (long)unit * K;
    select_topk_lds<kSelThreads>(s_keys, Np, K, sh, [dst](int pos, int p) { dst[pos] = p; });
}

// GQ: query heads per unit: 1, or Hq / Hkv (2, 4 or 8) for group-shared selection
int score_select_dispatch(int dtype, int D, int GQ, const void *q, const void *meta, uint64_t *scores,
                          float *scores_out, int32_t *idx_out, int B, int Hq, int Hkv, long Np_cap, int Np, int K,
                          int n_first, int n_local, int splits, uint32_t *unit_ctr, uint32_t *err, uint32_t tag,
                          int spin_limit, const uint32_t *state, long T_max, int P, hipStream_t stream)
{
    const dim3 grid((unsigned)splits, (unsigned)(B * Hq / GQ));
    if (Np > 15360) return RS_UNSUPPORTED;  // keys must fit 60 KiB of LDS
    if (GQ != 1 && GQ != 2 && GQ != 4 && GQ != 8) return RS_UNSUPPORTED;
    const size_t lds = (size_t)Np * 4;
#define RS_LAUNCH(ST, DD, GG)                                                                                      \
    quest_score_select_kernel<ST, DD, GG><<<grid, kSelThreads, lds, stream>>>(                                    \
        (const ST *)q, (const ST *)meta, scores, scores_out, idx_out, Hq, Hkv, Np_cap, Np, K, n_first, n_local, \
        splits, unit_ctr, err, tag, spin_limit, state, T_max, P)
#define RS_LAUNCH_G(ST, DD)                     \
    do {                                        \
        if (GQ == 8) RS_LAUNCH(ST, DD, 8);      \
        else if (GQ == 4) RS_LAUNCH(ST, DD, 4); \
        else if (GQ == 2) RS_LAUNCH(ST, DD, 2); \
        else RS_LAUNCH(ST, DD, 1);              \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) RS_LAUNCH_G(bf16, 128);
        else RS_LAUNCH_G(bf16, 64);
    } else {
        if (D == 128) RS_LAUNCH_G(float, 128);
        else RS_LAUNCH_G(float, 64);
    }
#undef RS_LAUNCH_G
#undef RS_LAUNCH
    return RS_OK;
}

// ------------------------------------------------------------------------------------
// The same scores as order-preserving keys (pages that are always kept: the top key) for an attention kernel that selects
// for itself: no hand-over inside the launch, and the chip does not idle while one workgroup of a unit selects.
// STEP (the replayable decode step, with n_local > 0): the rows of the grid past the query heads append the step's token instead
// of a launch of their own.  They write the last page's bounds while its scores are formed from them, whatever they hold then: that
// page is kept anyway and its score goes unused.  32 over 8 heads x 32768, 256 pages 22.2 -> 19.7 us a step.
// ------------------------------------------------------------------------------------
template <typename ST, int D, bool STEP>
__global__ __launch_bounds__(kSelThreads) void quest_score_keys_kernel(const ST *__restrict__ q, ST *meta, uint32_t *keys,
                                                                       int Hq, int Hkv, long Np_cap, int Np, int K, int n_first,
                                                                       int n_local, int splits, uint32_t *err,
                                                                       const uint32_t *state, long T_max, int P, long key_stride,
                                                                       StepToken token, int units)
{
    if constexpr (STEP) {
        if ((int)blockIdx.y >= units) {
            const uint32_t e = ((blockIdx.y - units) * gridDim.x + blockIdx.x) * kSelThreads + threadIdx.x;
            if (e < (uint32_t)(units / Hq * Hkv * D))
                append_element(e, (const ST *)token.k, (const ST *)token.v, token.g, token.state_k, token.state_v, (ST *)token.k_cache,
                               (ST *)token.v_cache, meta, P, D, 1, 0, token.Tcap, state, T_max, K);
            return;
        }
    }
    if (state) {  // the replayable decode step: tokens in the cache + 1 (the step's append has run)
        const long T_valid = *reinterpret_cast<const long *>(state + kCtrlStateT) + 1;
        Np = (int)((T_valid + P - 1) / P);
        if (T_valid > T_max || K > Np) {  // outside what the buffers were sized for: report, do nothing
            if (blockIdx.x == 0 && blockIdx.y == 0 && threadIdx.x == 0) atomicExch(err, 1u);
            return;
        }
    }
    constexpr int LPR = D / 8, RPW = 64 / LPR, ROW = D * (int)sizeof(ST);
    constexpr int UNR = 4, PPW = UNR * RPW;  // pages of a lane and of a wave per step
    using R = Row8<ST>;
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int rg = lane / LPR, cl = lane % LPR;
    const int unit = blockIdx.y, b = unit / Hq, kvh = (unit % Hq) / (Hq / Hkv);
    const ST *mbase = meta + ((long)(b * Hkv + kvh) * Np_cap) * 2 * D;
    uint32_t *krow = keys + unit * key_stride;
    float qv[8];
    R::load(q + (long)unit * D + cl * 8, qv);
    BoundDot<ST> bound;
    bound.set(qv);
    const int per = (Np + splits - 1) / splits;
    const int pb = blockIdx.x * per;
    const int pe = (pb + per < Np) ? pb + per : Np;
    for (int base = pb + wave * PPW; base < pe; base += PPW * (kSelThreads / 64)) {
        const int n = (pe - base < PPW) ? pe - base : PPW;
        const LdsSource md = lds_source_sized(mbase + (long)base * 2 * D, n * 2 * ROW);
        const uint32_t at = (uint32_t)(rg * 2 * ROW + cl * 8 * (int)sizeof(ST));
        typename R::raw_t mn[UNR], mx[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            mn[u] = load_row8<ST, 0>(md, at + u * RPW * 2 * ROW);
            mx[u] = load_row8<ST, 0>(md, at + (u * RPW * 2 + 1) * ROW);
        }
        float mine = 0.f;  // lane u of a row group keeps page u's sum, and the wave's keys leave with one store
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const float x = group_sum<LPR>(bound.add(0.f, mn[u], mx[u]));
            if (cl == u) mine = x;
        }
        const int p = base + rg + cl * RPW;
        if (cl < UNR && p < pe) krow[p] = (p < n_first || p >= Np - n_local) ? 0xffffffffu : float_to_key(mine);
    }
}

void score_keys_dispatch(int dtype, int D, const void *q, void *meta, uint32_t *keys, int B, int Hq, int Hkv, long Np_cap,
                         int Np, int K, int n_first, int n_local, int splits, uint32_t *err, const uint32_t *state, long T_max,
                         int P, long key_stride, const StepToken *token, hipStream_t stream)
{
    const int units = B * Hq;
    const long n_append = token ? ((long)B * Hkv * D + kSelThreads - 1) / kSelThreads : 0;  // workgroups
    const dim3 grid((unsigned)splits, (unsigned)(units + (n_append + splits - 1) / splits));
    const StepToken tk = token ? *token : StepToken{};
#define RS_LAUNCH_S(ST, DD, SS)                                                                                                 \
    quest_score_keys_kernel<ST, DD, SS><<<grid, kSelThreads, 0, stream>>>((const ST *)q, (ST *)meta, keys, Hq, Hkv, Np_cap, Np, \
                                                                          K, n_first, n_local, splits, err, state, T_max, P, key_stride, tk, units)
#define RS_LAUNCH(ST, DD)                                \
    do {                                                 \
        if (token) RS_LAUNCH_S(ST, DD, true);            \
        else RS_LAUNCH_S(ST, DD, false);                 \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) RS_LAUNCH(bf16, 128);
        else RS_LAUNCH(bf16, 64);
    } else {
        if (D == 128) RS_LAUNCH(float, 128);
        else RS_LAUNCH(float, 64);
    }
#undef RS_LAUNCH_S
#undef RS_LAUNCH
}

// ------------------------------------------------------------------------------------
// decode attention over a list of 16-row tiles (selected pages, or all rows), split over
// workgroups; partial (m, l, o) per split; the last split to arrive merges them.
// ------------------------------------------------------------------------------------
// SELECT: the list is not given; every split selects it from the unit's page keys (keys, key_stride of them per unit) and
// keeps its own part in LDS, the first split writes it to idx_out.  Dynamic LDS then: key_stride keys, and the part.
template <typename ST, int D, int kAttThreads, bool STREAM, bool SELECT>
__global__ __launch_bounds__(kAttThreads) void decode_attend_kernel(
    const ST *__restrict__ q, const ST *k_cache, const ST *v_cache, const int32_t *idx,
    ST *__restrict__ out, float *__restrict__ lse_out, uint64_t *partial, int Hq, int Hkv, long Tcap, int P,
    long T_valid, int K, float scale, int splits, uint32_t *unit_ctr, uint32_t *err, uint32_t tag, int spin_limit,
    int idx_per_kv, uint32_t *state, long T_max, const uint32_t *keys, long key_stride, int32_t *idx_out)
{
    // state (the replayable decode step, listed pages): length and tag come from the workspace's words; the
    // last workgroup out of the grid advances them (every workgroup has read them by then)
    if (state) {
        T_valid = *reinterpret_cast<const long *>(state + kCtrlStateT) + 1;
        tag = state[kCtrlStateTag];
        if (tag == 0u) tag = 0x5bd1e995u;
        if (T_valid > T_max || (long)K > (T_valid + P - 1) / P) return;  // refused: the selection kernel has reported it
    }
    auto workgroup_done = [&]() {
        if (state && threadIdx.x == 0) {
            uint32_t *done = state + kCtrlDone;
            if (atomicAdd(done, 1u) == gridDim.x * gridDim.y - 1u) {
                atomicExch(done, 0u);
                *reinterpret_cast<long *>(state + kCtrlStateT) = T_valid;
                const uint32_t nt = tag + 0x85EBCA6Bu;
                state[kCtrlStateTag] = nt ? nt : 0x5bd1e995u;
            }
        }
    };
    constexpr int LPR = D / 8;
    constexpr int TR = 16;   // rows per tile
    // One tile to a wave's step, and the next one's rows on their way where a tile's K and V are 32 registers (64 with float32
    // rows of 128 channels): at most 128 registers in all, so that two workgroups share a CU and a grid that is not a
    // multiple of the CUs has no second turn.  Two tiles, or 64-register steps ahead (157-165 registers, one workgroup to a CU):
    // append + decode of 7 x 8 heads x 7055, 55 of 441 pages 22.9 -> 32.0 us, 5 x 8 x 20000, 156 of 1250 31.3 -> 40.0, 3 x 4 x 7473 dense
    // 21.1 -> 23.4, float32 7 x 16 x 8252 35.7 -> 42.1; where the grid is 256 workgroups anyway 32 over 8 heads x 16416 19.8 -> 21.5.
    constexpr int TPI = 1;
    constexpr bool AHEAD = D * (int)sizeof(ST) < 512;
    constexpr int kAttWaves = kAttThreads / 64;
    using R = Row8<ST>;
    __shared__ float s_m[kAttWaves], s_l[kAttWaves];
    __shared__ float s_o[kAttWaves][D];
    __shared__ int s_last;

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane / LPR;
    const int c0 = (lane % LPR) * 8;
    const int unit = blockIdx.y;
    const int b = unit / Hq, h = unit % Hq;
    const int kvh = h / (Hq / Hkv);
    const ST *kb = k_cache + (long)(b * Hkv + kvh) * Tcap * D;
    const ST *vb = v_cache + (long)(b * Hkv + kvh) * Tcap * D;
    // a page list belongs to the query head, or (group-shared selection) to its KV head
    const int32_t *idx_row = idx ? idx + (long)(idx_per_kv ? b * Hkv + kvh : unit) * K : nullptr;

    RowDot<ST> qd[1];
    {
        float qv[8];
        R::load(q + (long)unit * D + c0, qv);
        qd[0].set(qv);
    }

    const int page_shift = (SELECT || idx) ? __builtin_ctz((unsigned)(P / TR)) : 0;  // tiles of a page: a power of two
    const long n_tiles = (SELECT || idx) ? (long)K << page_shift : (T_valid + TR - 1) / TR;
    const long per = (n_tiles + splits - 1) / splits;
    const long tb = (long)blockIdx.x * per;
    const long te = (tb + per < n_tiles) ? tb + per : n_tiles;

    AttendState<1> st;
    st.clear();
    const long t_first = tb + wave * TPI, stride = kAttWaves * TPI;
    auto attend = [&](auto row_of) __attribute__((always_inline)) {
        if constexpr (AHEAD) attend_tiles<ST, D, 1, TPI, STREAM>(kb, vb, T_valid, t_first, te, stride, scale, qd, st, row_of);
        else attend_tiles_in_turn<ST, D, 1, TPI, STREAM>(kb, vb, T_valid, t_first, te, stride, scale, qd, st, row_of);
    };
    if constexpr (SELECT) {
        __shared__ SelectShared<kAttThreads> sh;
        extern __shared__ __attribute__((aligned(16))) uint32_t s_dyn[];
        uint32_t *s_keys = s_dyn;
        int *s_sel = reinterpret_cast<int *>(s_dyn + key_stride);
        const int Np = (int)((T_valid + P - 1) / P);
        const uint4 *src = reinterpret_cast<const uint4 *>(keys + unit * key_stride);
        for (int i = tid; i < (Np + 3) / 4; i += kAttThreads) {
            uint4 x = src[i];
            if (4 * i + 1 >= Np) x.y = 0u;  // (zeros up to a multiple of four)
            if (4 * i + 2 >= Np) x.z = 0u;
            if (4 * i + 3 >= Np) x.w = 0u;
            reinterpret_cast<uint4 *>(s_keys)[i] = x;
        }
        __syncthreads();
        const int first = (int)(tb >> page_shift), past = tb < te ? (int)((te - 1) >> page_shift) + 1 : first;  // this split's part
        int32_t *whole = (blockIdx.x == 0 && idx_out) ? idx_out + (long)unit * K : nullptr;
        auto emit = [=](int pos, int p) {
            if (pos >= first && pos < past) s_sel[pos - first] = p;
            if (whole) whole[pos] = p;
        };
        if (Np <= kAttThreads / 2) select_topk_few<kAttThreads>(s_keys, Np, K, sh.wave_tot, emit);
        else select_topk_lds<kAttThreads>(s_keys, Np, K, sh, emit);
        __syncthreads();
        attend([&](long t) __attribute__((always_inline)) -> long {
            const int page = __builtin_amdgcn_readfirstlane(s_sel[(int)(t >> page_shift) - first]);
            return (long)page * P + (t & ((1 << page_shift) - 1)) * TR;
        });
    } else if (idx) {
        WavePages pages;
        attend([&](long t) __attribute__((always_inline)) -> long {
            const int page = pages.next([&](int n) __attribute__((always_inline)) -> int {
                const long tt = t_first + (long)(n / TPI) * stride + n % TPI;
                return tt < te ? idx_row[tt >> page_shift] : -1;
            });
            return page >= 0 ? (long)page * P + (t & ((1 << page_shift) - 1)) * TR : T_valid;
        });
    } else {
        attend([&](long t) __attribute__((always_inline)) -> long { return t * TR; });
    }
    float m = st.m[0], l = st.l[0];
    float (&o)[8] = st.o[0];

    // merge the row groups of the wave
#pragma unroll
    for (int mask = LPR; mask < 64; mask <<= 1) {
        const float m2 = shfl_xor_f(m, mask);
        const float l2 = shfl_xor_f(l, mask);
        const float mn = fmaxf(m, m2);
        const float a1 = (m == -INFINITY) ? 0.f : __expf(m - mn);
        const float a2 = (m2 == -INFINITY) ? 0.f : __expf(m2 - mn);
        l = l * a1 + l2 * a2;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float o2 = shfl_xor_f(o[c], mask);
            o[c] = o[c] * a1 + o2 * a2;
        }
        m = mn;
    }
    if (rg == 0) {
        if ((lane % LPR) == 0) {
            s_m[wave] = m;
            s_l[wave] = l;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) s_o[wave][c0 + c] = o[c];
    }
    __syncthreads();

    // merge the waves; thread c owns channel c
    uint64_t *part = partial + ((long)unit * splits + blockIdx.x) * (D + 2);
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < kAttWaves; ++w) M = fmaxf(M, s_m[w]);
        float L = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < kAttWaves; ++w) {
            const float a = (s_m[w] == -INFINITY) ? 0.f : __expf(s_m[w] - M);
            L += s_l[w] * a;
            O += s_o[w][tid] * a;
        }
        if (splits == 1) {
            const float inv = (L > 0.f) ? 1.f / L : 0.f;
            from_f32(out[(long)unit * D + tid], O * inv);
            if (tid == 0 && lse_out) lse_out[unit] = (L > 0.f) ? M + __logf(L) : -INFINITY;
        } else {
            publish_f32(&part[2 + tid], O, tag);
            if (tid == 0) {
                publish_f32(&part[0], M, tag);
                publish_f32(&part[1], L, tag);
            }
        }
    }
    if (splits == 1) {
        workgroup_done();
        return;
    }

    if (tid == 0) {
        const uint32_t prev = atomicAdd(&unit_ctr[unit], 1u);
        s_last = (prev == (uint32_t)splits - 1u);
        if (s_last) atomicExch(&unit_ctr[unit], 0u);
    }
    __syncthreads();
    if (!s_last) {
        workgroup_done();
        return;
    }
    if (tid < D) {
        float M = -INFINITY, L = 0.f, O = 0.f;
        merge_partials(partial + (long)unit * splits * (D + 2), splits, D + 2, tid, tag, spin_limit, err, M, L, O);
        const float inv = (L > 0.f) ? 1.f / L : 0.f;
        from_f32(out[(long)unit * D + tid], O * inv);
        if (tid == 0 && lse_out) lse_out[unit] = (L > 0.f) ? M + __logf(L) : -INFINITY;
    }
    workgroup_done();
}

// ------------------------------------------------------------------------------------
// The same for the G query heads of a KV head at once, where they attend the same rows (all of
// them, or a page list of the KV head): a row is fetched once instead of G times, and its values
// are unpacked once.  A lane keeps G running (m, l, o).  A wave takes TPI tiles per step and has
// the next step's on their way while it works on the current ones; the softmax moves its reference
// point once per step and head.
// Bound by memory from about a hundred megabytes on (8 x 32 over 8 heads x 8000 rows: 268 MB in 57 us with the append against
// 153 us with a workgroup per head), by the merge below that.
// ------------------------------------------------------------------------------------
constexpr int kSharedThreads = 512;
constexpr int kSharedMaxSplits = 64;

template <typename ST, int D, int G>
__global__ __launch_bounds__(kSharedThreads) void decode_attend_shared_kernel(
    const ST *__restrict__ q, const ST *k_cache, const ST *v_cache, const int32_t *idx,
    ST *__restrict__ out, float *__restrict__ lse_out, uint64_t *partial, long Tcap, int P, long T_valid, int K,
    float scale, int splits, uint32_t *unit_ctr, uint32_t *err, uint32_t tag, int spin_limit)
{
    constexpr int LPR = D / 8;
    constexpr int RPW = 64 / LPR;  // rows per load instruction
    constexpr int TR = 16;         // rows per tile
    constexpr int TPI = (sizeof(ST) == 2 && G < 8) ? 2 : 1;  // tiles per step of a wave
    constexpr int NW = kSharedThreads / 64;
    using R = Row8<ST>;
    // partials of a workgroup that meet in LDS: one per row group of a wave (fewer trips than shuffles
    // between the row groups first), or one per wave where that many would not fit
    constexpr int PPW = G * RPW <= 16 ? RPW : 1, NP = NW * PPW;
    __shared__ float s_m[NP][G], s_l[NP][G];
    __shared__ __attribute__((aligned(16))) float s_o[NP][G][D];
    __shared__ int s_last;

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane / LPR, c0 = (lane % LPR) * 8;
    const int unit = blockIdx.y;  // b * Hkv + kvh; its query heads are rows unit * G .. of q, out and the partials
    const ST *kb = k_cache + (long)unit * Tcap * D;
    const ST *vb = v_cache + (long)unit * Tcap * D;
    const int32_t *idx_row = idx ? idx + (long)unit * K : nullptr;

    const int page_shift = idx ? __builtin_ctz((unsigned)(P / TR)) : 0;  // tiles of a page: a power of two
    const long n_tiles = idx ? (long)K << page_shift : (T_valid + TR - 1) / TR;
    const long per = (n_tiles + splits - 1) / splits;
    const long tb = (long)blockIdx.x * per;
    const long te = (tb + per < n_tiles) ? tb + per : n_tiles;

    RowDot<ST> qd[G];
#pragma unroll
    for (int g = 0; g < G; ++g) {
        float qv[8];
        R::load(q + ((long)unit * G + g) * D + c0, qv);
        qd[g].set(qv);
    }
    AttendState<G> st;
    st.clear();
    // (each row is read by this workgroup only: streaming loads)
    const long t_first = tb + wave * TPI, stride = NW * TPI;
    if (idx) {
        WavePages pages;
        attend_tiles<ST, D, G, TPI, true>(kb, vb, T_valid, t_first, te, stride, scale, qd, st, [&](long t) __attribute__((always_inline)) -> long {
            const int page = pages.next([&](int n) __attribute__((always_inline)) -> int {
                const long tt = t_first + (long)(n / TPI) * stride + n % TPI;
                return tt < te ? idx_row[tt >> page_shift] : -1;
            });
            return page >= 0 ? (long)page * P + (t & ((1 << page_shift) - 1)) * TR : T_valid;
        });
    } else {
        attend_tiles<ST, D, G, TPI, true>(kb, vb, T_valid, t_first, te, stride, scale, qd, st, [&](long t) __attribute__((always_inline)) -> long { return t * TR; });
    }
    float (&m)[G] = st.m, (&l)[G] = st.l, (&o)[G][8] = st.o;

#pragma unroll
    for (int g = 0; g < G; ++g) {
        if constexpr (PPW == 1) {  // merge the row groups of the wave
#pragma unroll
            for (int mask = LPR; mask < 64; mask <<= 1) {
                const float m2 = shfl_xor_f(m[g], mask);
                const float l2 = shfl_xor_f(l[g], mask);
                const float mn = fmaxf(m[g], m2);
                const float a1 = (m[g] == -INFINITY) ? 0.f : __expf(m[g] - mn);
                const float a2 = (m2 == -INFINITY) ? 0.f : __expf(m2 - mn);
                l[g] = l[g] * a1 + l2 * a2;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    const float o2 = shfl_xor_f(o[g][c], mask);
                    o[g][c] = o[g][c] * a1 + o2 * a2;
                }
                m[g] = mn;
            }
        }
        if (rg < PPW) {
            const int p = wave * PPW + rg;
            if (lane % LPR == 0) {
                s_m[p][g] = m[g];
                s_l[p][g] = l[g];
            }
            float4 *dst = reinterpret_cast<float4 *>(&s_o[p][g][c0]);
            dst[0] = make_float4(o[g][0], o[g][1], o[g][2], o[g][3]);
            dst[1] = make_float4(o[g][4], o[g][5], o[g][6], o[g][7]);
        }
    }
    __syncthreads();

    // merge them; thread (g, c) owns channel c of head g
    for (int e = tid; e < G * D; e += kSharedThreads) {
        const int g = e / D, c = e % D;
        const long head = (long)unit * G + g;
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NP; ++w) M = fmaxf(M, s_m[w][g]);
        float L = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < NP; ++w) {
            const float a = (s_m[w][g] == -INFINITY) ? 0.f : __expf(s_m[w][g] - M);
            L += s_l[w][g] * a;
            O += s_o[w][g][c] * a;
        }
        if (splits == 1) {
            const float inv = (L > 0.f) ? 1.f / L : 0.f;
            from_f32(out[head * D + c], O * inv);
            if (c == 0 && lse_out) lse_out[head] = (L > 0.f) ? M + __logf(L) : -INFINITY;
        } else {
            uint64_t *part = partial + (head * splits + blockIdx.x) * (D + 2);
            publish_f32(&part[2 + c], O, tag);
            if (c == 0) {
                publish_f32(&part[0], M, tag);
                publish_f32(&part[1], L, tag);
            }
        }
    }
    if (splits == 1) return;

    // The last split of the unit to arrive merges them all: every word it reads has been sent by a workgroup that ran, so
    // nothing here depends on the order in which workgroups start.  The words go by plain 16-byte loads, two channels a
    // lane (8-byte agent-scope loads take them at a third of that rate); one whose tag is not this call's, because it is
    // still on its way or a cache holds it from before, is polled at agent scope.  Four heads x 32 splits take about 3 us,
    // eight x 64 about 10 (a fence that empties the caches first costs 10 us by itself).
    if (tid == 0) {
        const uint32_t prev = atomicAdd(&unit_ctr[unit], 1u);
        s_last = (prev == (uint32_t)splits - 1u);
        if (s_last) atomicExch(&unit_ctr[unit], 0u);
    }
    __syncthreads();
    if (!s_last) return;
    constexpr int LR = D / 2, ROWS = kSharedThreads / LR;  // lanes per partial, partials at a time
    constexpr int PARTS = ROWS / G, U = 8;                 // of which each head has PARTS; partials a lane has on their way
    static_assert(PARTS >= 1 && PARTS <= NP, "the parts meet in the arrays above");
    typedef uint64_t u64x2 __attribute__((ext_vector_type(2)));
    const int g = (tid / LR) % G, part = tid / LR / G, c = (tid % LR) * 2;
    const uint64_t *ph = partial + ((long)unit * G + g) * splits * (D + 2);
    float M = -INFINITY, L = 0.f, O0 = 0.f, O1 = 0.f;
    for (int s0 = part; s0 < splits; s0 += U * PARTS) {
        u64x2 ml[U], oo[U];
#pragma unroll
        for (int u = 0; u < U; ++u) {
            const int sp = (s0 + u * PARTS < splits) ? s0 + u * PARTS : s0;
            ml[u] = *reinterpret_cast<const u64x2 *>(ph + (long)sp * (D + 2));
            oo[u] = *reinterpret_cast<const u64x2 *>(ph + (long)sp * (D + 2) + 2 + c);
        }
#pragma unroll
        for (int u = 0; u < U; ++u) {
            if (s0 + u * PARTS >= splits) break;
            const uint64_t *p = ph + (long)(s0 + u * PARTS) * (D + 2);
            auto value = [&](uint64_t w, int at) __attribute__((always_inline)) -> float {
                return (uint32_t)(w >> 32) == tag ? __uint_as_float((uint32_t)w) : acquire_f32(p + at, tag, spin_limit, err);
            };
            const float ms = value(ml[u].x, 0), ls = value(ml[u].y, 1), o0 = value(oo[u].x, 2 + c), o1 = value(oo[u].y, 3 + c);
            const float mn = fmaxf(M, ms);
            const float a1 = (M == -INFINITY) ? 0.f : __expf(M - mn);
            const float a2 = (ms == -INFINITY) ? 0.f : __expf(ms - mn);
            L = L * a1 + ls * a2;
            O0 = O0 * a1 + o0 * a2;
            O1 = O1 * a1 + o1 * a2;
            M = mn;
        }
    }
    if (c == 0) {
        s_m[part][g] = M;
        s_l[part][g] = L;
    }
    *reinterpret_cast<float2 *>(&s_o[part][g][c]) = make_float2(O0, O1);
    __syncthreads();
    for (int e = tid; e < G * D; e += kSharedThreads) {
        const int ge = e / D, ce = e % D;
        const long head = (long)unit * G + ge;
        M = -INFINITY;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) M = fmaxf(M, s_m[i][ge]);
        L = O0 = 0.f;
#pragma unroll
        for (int i = 0; i < PARTS; ++i) {
            const float a = (s_m[i][ge] == -INFINITY) ? 0.f : __expf(s_m[i][ge] - M);
            L += s_l[i][ge] * a;
            O0 += s_o[i][ge][ce] * a;
        }
        const float inv = (L > 0.f) ? 1.f / L : 0.f;
        from_f32(out[head * D + ce], O0 * inv);
        if (ce == 0 && lse_out) lse_out[head] = (L > 0.f) ? M + __logf(L) : -INFINITY;
    }
}

// ------------------------------------------------------------------------------------
// Short contexts (the paper's 4096 tokens): select-then-attend of one (batch, query head)
// inside one 512-thread workgroup -- page scores into LDS keys, the top-K selection, then
// attention over the picked pages with the waves splitting the tiles -- so nothing is handed
// between workgroups and the step is one launch.  Same score arithmetic, forced pages and tie
// rule as quest_score_select_kernel; the attention loop is decode_attend_kernel's.  Bound by its chain of phases, one workgroup
// to a CU at a batch of eight: hence the pages that are kept anyway are fetched first of all, up to 256 pages are
// selected by counting ranks instead of radix passes, and the next tile's rows are on their way behind the current one's.
// With the append, 4096 tokens, 8 pages of 64, before / after, us: 8 x 32 heads 21.5 / 17.7, 16 x 32 35.2 / 30.3, 32 14.5 / 12.8;
// 16 x 32 over 8 heads x 1000, 8 of 16 17.5 / 13.5; 4 x 32 over 8 heads x 8000, 31 of 32 23.8 / 20.9.
// Dynamic LDS: Np keys, then K picked pages.
// ------------------------------------------------------------------------------------
constexpr int kUnitThreads = 512;

// STATE (the replayable decode step): the sequence length is not an argument but the workspace's
// token count + 1 (the step's append has run); Np_lds = the page count the LDS was sized for;
// the last workgroup out advances the count and the tag word.
template <typename ST, int D, bool STATE>
__global__ __launch_bounds__(kUnitThreads) void quest_unit_decode_kernel(
    const ST *__restrict__ q, const ST *__restrict__ meta, const ST *k_cache,
    const ST *v_cache, ST *__restrict__ out, float *__restrict__ lse_out, int32_t *__restrict__ idx_out,
    int Hq, int Hkv, long Tcap, int P, long T_valid, int Np, int K, int n_first, int n_local, float scale,
    int Np_lds, uint32_t *state, long T_max)
{
    if constexpr (STATE) {
        T_valid = *reinterpret_cast<const long *>(state + kCtrlStateT) + 1;
        Np = (int)((T_valid + P - 1) / P);
        if (T_valid > T_max || K > Np) {  // outside what the buffers were sized for: report, do nothing
            if (blockIdx.x == 0 && threadIdx.x == 0) atomicExch(state + kCtrlAsyncErr, 1u);
            return;
        }
    }
    constexpr int LPR = D / 8;
    constexpr int RPW = 64 / LPR;
    constexpr int UNR = 4;
    constexpr int NW = kUnitThreads / 64;
    constexpr bool STREAM = false;
    constexpr int TR = 16;
    constexpr int TPI = 1;  // tiles of a wave's step (two: one workgroup a CU instead of two, and slower there too)
    using R = Row8<ST>;
    __shared__ SelectShared<kUnitThreads> sh;
    __shared__ float s_m[NW], s_l[NW];
    __shared__ float s_o[NW][D];
    extern __shared__ __attribute__((aligned(16))) uint32_t s_dyn[];
    uint32_t *s_keys = s_dyn;
    int *s_sel = reinterpret_cast<int *>(s_dyn + (Np_lds + 3) / 4 * 4);

    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int rg = lane / LPR;
    const int c0 = (lane % LPR) * 8;
    const int unit = blockIdx.x;
    const int b = unit / Hq, h = unit % Hq;
    const int kvh = h / (Hq / Hkv);
    const long Np_cap = Tcap / P;
    const ST *mbase = meta + ((long)(b * Hkv + kvh) * Np_cap) * 2 * D;
    const ST *kb = k_cache + (long)(b * Hkv + kvh) * Tcap * D;
    const ST *vb = v_cache + (long)(b * Hkv + kvh) * Tcap * D;

    float qv[8];
    R::load(q + (long)unit * D + c0, qv);
    BoundDot<ST> bound;
    bound.set(qv);

    // Pages that are kept whatever their scores, the local ones and then the first ones, come first in the attention below
    // (a rotation of the ascending list by the local ones), so that a wave whose first tiles lie in them has those rows
    // on their way from here on.
    const int page_shift = __builtin_ctz((unsigned)(P / TR));  // tiles of a page: a power of two
    const bool known = n_first >= 0 && n_local >= 0 && n_first + n_local <= K && n_first + n_local <= Np;
    const int rotate = known ? n_local : 0;
    const long known_tiles = known ? (long)(n_first + n_local) << page_shift : 0, n_tiles = (long)K << page_shift;
    AttendStep<ST, D, TPI> xa;
    auto known_row = [&](long t) __attribute__((always_inline)) -> long {
        const int i = (int)(t >> page_shift);
        return (long)(i < n_local ? Np - n_local + i : i - n_local) * P + (t & ((1 << page_shift) - 1)) * TR;
    };
    xa.template load<STREAM>(kb, vb, T_valid, wave * TPI, known_tiles, known_row);

    // page scores (Eq. 3 with the min/max bound) -> order-preserving keys (zeros up to a multiple of four)
    if (tid < ((-Np) & 3)) s_keys[Np + tid] = 0u;
    constexpr int PPI = UNR * RPW * NW;
    for (int base = wave * (UNR * RPW); base < Np; base += PPI) {
        const int n = (Np - base < UNR * RPW) ? Np - base : UNR * RPW;
        const LdsSource md = lds_source_sized(mbase + (long)base * 2 * D, n * 2 * D * (int)sizeof(ST));
        const uint32_t at = (uint32_t)((rg * 2 * D + c0) * (int)sizeof(ST));
        typename R::raw_t mn[UNR], mx[UNR];
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            mn[u] = load_row8<ST, 0>(md, at + u * RPW * 2 * D * (int)sizeof(ST));
            mx[u] = load_row8<ST, 0>(md, at + (u * RPW * 2 + 1) * D * (int)sizeof(ST));
        }
#pragma unroll
        for (int u = 0; u < UNR; ++u) {
            const int p = base + rg + u * RPW;
            const float s = group_sum<LPR>(bound.add(0.f, mn[u], mx[u]));
            if (p < Np && (lane % LPR) == 0) s_keys[p] = (p < n_first || p >= Np - n_local) ? 0xffffffffu : float_to_key(s);
        }
    }
    __syncthreads();
    int32_t *dst = idx_out ? idx_out + (long)unit * K : nullptr;
    auto emit = [s_sel, dst](int pos, int p) {
        s_sel[pos] = p;
        if (dst) dst[pos] = p;
    };
    // One histogram instead of the radix passes, us a step: 256 heads of 64 channels x 520 pages 20.0 -> 17.8, x 978 27.3 -> 24.6, of 128
    // channels x 520 28.4 -> 25.9, x 978 44.8 -> 42.3.  With more heads than CUs the gain is less and for some shapes a loss, on no
    // side of any line: 480 heads of 64 channels x 520 24.7 -> 22.4, x 978 37.8 -> 38.4, 512 over 128 KV heads x 800 33.3 -> 35.2, 768 x 800
    // 51.7 -> 49.8, of 128 channels 288 x 597 34.7 -> 36.0, 320 x 260 21.4 -> 18.6, x 520 31.4 -> 32.5, x 800 51.0 -> 49.6; over 40 drawn
    // shapes of 272 to 1024 heads 0.973 to 1.094 times the speed, 1.022 in the mean.
    if (Np <= kUnitThreads / 2) select_topk_few<kUnitThreads>(s_keys, Np, K, sh.wave_tot, emit);
    else select_topk_lds<kUnitThreads>(s_keys, Np, K, sh, emit);
    __syncthreads();

    // attention over the picked pages (Eq. 4): 16-row tiles, the waves take them in turn
    RowDot<ST> qd[1];
    qd[0].set(qv);
    AttendState<1> st;
    st.clear();
    auto row_of = [&](long t) __attribute__((always_inline)) -> long {
        const int i = (int)(t >> page_shift);
        const int page = __builtin_amdgcn_readfirstlane(s_sel[i < rotate ? K - rotate + i : i - rotate]);
        return (long)page * P + (t & ((1 << page_shift) - 1)) * TR;
    };
    // (a page whose score is a NaN may tie with the pages that are kept: the list decides)
    bool loaded = true;
#pragma unroll
    for (int u = 0; u < TPI; ++u) {
        const long t = wave * TPI + u;
        if (t < n_tiles && (t >= known_tiles || row_of(t) != known_row(t))) loaded = false;
    }
    if (!loaded) xa.template load<STREAM>(kb, vb, T_valid, wave * TPI, n_tiles, row_of);
    attend_tiles<ST, D, 1, TPI, STREAM>(kb, vb, T_valid, wave * TPI, n_tiles, NW * TPI, scale, qd, st, xa, row_of);
    float m = st.m[0], l = st.l[0];
    float (&o)[8] = st.o[0];
    // merge the row groups of the wave, then the waves
#pragma unroll
    for (int mask = LPR; mask < 64; mask <<= 1) {
        const float m2 = shfl_xor_f(m, mask);
        const float l2 = shfl_xor_f(l, mask);
        const float mn = fmaxf(m, m2);
        const float a1 = (m == -INFINITY) ? 0.f : __expf(m - mn);
        const float a2 = (m2 == -INFINITY) ? 0.f : __expf(m2 - mn);
        l = l * a1 + l2 * a2;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float o2 = shfl_xor_f(o[c], mask);
            o[c] = o[c] * a1 + o2 * a2;
        }
        m = mn;
    }
    if (rg == 0) {
        if ((lane % LPR) == 0) {
            s_m[wave] = m;
            s_l[wave] = l;
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) s_o[wave][c0 + c] = o[c];
    }
    __syncthreads();
    if (tid < D) {
        float M = -INFINITY;
#pragma unroll
        for (int w = 0; w < NW; ++w) M = fmaxf(M, s_m[w]);
        float L = 0.f, O = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float a = (s_m[w] == -INFINITY) ? 0.f : __expf(s_m[w] - M);
            L += s_l[w] * a;
            O += s_o[w][tid] * a;
        }
        const float inv = (L > 0.f) ? 1.f / L : 0.f;
        from_f32(out[(long)unit * D + tid], O * inv);
        if (tid == 0 && lse_out) lse_out[unit] = (L > 0.f) ? M + __logf(L) : -INFINITY;
    }
    if constexpr (STATE) {
        if (tid == 0 && atomicAdd(state + kCtrlDone, 1u) == gridDim.x - 1u) {  // every workgroup has read the state
            atomicExch(state + kCtrlDone, 0u);
            *reinterpret_cast<long *>(state + kCtrlStateT) = T_valid;
            const uint32_t nt = state[kCtrlStateTag] + 0x85EBCA6Bu;
            state[kCtrlStateTag] = nt ? nt : 0x5bd1e995u;
        }
    }
}

// state != NULL: the replayable step (T_valid = the largest length, Np = its page count)
void unit_decode_dispatch(int dtype, int D, const void *q, const void *meta, const void *k_cache, const void *v_cache,
                          void *out, float *lse_out, int32_t *idx_out, int B, int Hq, int Hkv, long Tcap, int P,
                          long T_valid, int Np, int K, int n_first, int n_local, float scale, uint32_t *state,
                          hipStream_t stream)
{
    const size_t lds = (size_t)((Np + 3) / 4 * 4 + K) * 4;
#define RS_LAUNCH1(ST, DD, SS)                                                                                   \
    quest_unit_decode_kernel<ST, DD, SS><<<(unsigned)(B * Hq), kUnitThreads, lds, stream>>>(                     \
        (const ST *)q, (const ST *)meta, (const ST *)k_cache, (const ST *)v_cache, (ST *)out, lse_out, idx_out, \
        Hq, Hkv, Tcap, P, T_valid, Np, K, n_first, n_local, scale, Np, state, T_valid)
#define RS_LAUNCH(ST, DD)                    \
    do {                                     \
        if (state) RS_LAUNCH1(ST, DD, true); \
        else RS_LAUNCH1(ST, DD, false);      \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) RS_LAUNCH(bf16, 128);
        else RS_LAUNCH(bf16, 64);
    } else {
        if (D == 128) RS_LAUNCH(float, 128);
        else RS_LAUNCH(float, 64);
    }
#undef RS_LAUNCH
#undef RS_LAUNCH1
}

// the G = Hq / Hkv query heads of a KV head over the same rows: all rows, or a page list per KV head
bool decode_attend_shared_fits(int dtype, int D, int G, int splits)
{
    if (dtype == RS_F32 && D == 128 && G == 8) return false;  // (its registers would not hold them)
    return (G == 2 || G == 4 || G == 8) && splits <= kSharedMaxSplits;
}

void decode_attend_shared_dispatch(int dtype, int D, const void *q, const void *k_cache, const void *v_cache,
                                   const int32_t *idx, void *out, float *lse_out, uint64_t *partial, int B, int Hq, int Hkv,
                                   long Tcap, int P, long T_valid, int K, float scale, int splits, uint32_t *unit_ctr,
                                   uint32_t *err, uint32_t tag, int spin_limit, hipStream_t stream)
{
    const dim3 grid((unsigned)splits, (unsigned)(B * Hkv));
    const int G = Hq / Hkv;
#define RS_LAUNCH(ST, DD, GG)                                                                                \
    decode_attend_shared_kernel<ST, DD, GG><<<grid, kSharedThreads, 0, stream>>>(                            \
        (const ST *)q, (const ST *)k_cache, (const ST *)v_cache, idx, (ST *)out, lse_out, partial, Tcap,     \
        P, T_valid, K, scale, splits, unit_ctr, err, tag, spin_limit)
#define RS_LAUNCH_G(ST, DD)                     \
    do {                                        \
        if (G == 2) RS_LAUNCH(ST, DD, 2);       \
        else if (G == 4) RS_LAUNCH(ST, DD, 4);  \
        else RS_LAUNCH(ST, DD, 8);              \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) RS_LAUNCH_G(bf16, 128);
        else RS_LAUNCH_G(bf16, 64);
    } else {
        if (D == 64) RS_LAUNCH_G(float, 64);
        else if (G == 2) RS_LAUNCH(float, 128, 2);
        else RS_LAUNCH(float, 128, 4);
    }
#undef RS_LAUNCH_G
#undef RS_LAUNCH
}

// LDS of a split that selects for itself: the keys, and its part of the list (a part may begin and end inside a page)
size_t attend_select_lds(long key_stride, int K, int P, int splits)
{
    const long tiles = (long)K * (P / 16), per = (tiles + splits - 1) / splits;
    return (size_t)(key_stride + per / (P / 16) + 2) * 4;
}

// keys != NULL: the kernel selects for itself (idx is not read; idx_out may be NULL)
void decode_attend_dispatch(int dtype, int D, const void *q, const void *k_cache, const void *v_cache,
                            const int32_t *idx, void *out, float *lse_out, uint64_t *partial, int B, int Hq,
                            int Hkv, long Tcap, int P, long T_valid, int K, float scale, int splits,
                            uint32_t *unit_ctr, uint32_t *err, uint32_t tag, int spin_limit, int idx_per_kv,
                            uint32_t *state, long T_max, const uint32_t *keys, long key_stride, int32_t *idx_out,
                            hipStream_t stream)
{
    const dim3 grid((unsigned)splits, (unsigned)(B * Hq));
    constexpr int kAttThreads = 512;  // about one such workgroup per CU (see the split rule of the caller)
    const size_t lds = keys ? attend_select_lds(key_stride, K, P, splits) : 0;
#define RS_LAUNCH1(ST, DD, SS, LL)                                                                          \
    decode_attend_kernel<ST, DD, kAttThreads, SS, LL><<<grid, kAttThreads, lds, stream>>>(                  \
        (const ST *)q, (const ST *)k_cache, (const ST *)v_cache, idx, (ST *)out, lse_out, partial, Hq, Hkv, \
        Tcap, P, T_valid, K, scale, splits, unit_ctr, err, tag, spin_limit, idx_per_kv, state, T_max, keys, key_stride, idx_out)
    // no other query head reads these rows: streaming loads
#define RS_LAUNCH(ST, DD)                                       \
    do {                                                        \
        if (keys && Hq == Hkv) RS_LAUNCH1(ST, DD, true, true);  \
        else if (keys) RS_LAUNCH1(ST, DD, false, true);         \
        else if (Hq == Hkv) RS_LAUNCH1(ST, DD, true, false);    \
        else RS_LAUNCH1(ST, DD, false, false);                  \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) RS_LAUNCH(bf16, 128);
        else RS_LAUNCH(bf16, 64);
    } else {
        if (D == 128) RS_LAUNCH(float, 128);
        else RS_LAUNCH(float, 64);
    }
#undef RS_LAUNCH
#undef RS_LAUNCH1
}

}  // namespace rs
