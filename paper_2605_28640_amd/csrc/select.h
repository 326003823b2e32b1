// Fence-free cross-workgroup hand-off (tagged words) and the register-resident top-K
// selection shared by the decode kernels.
#pragma once

#include "common.h"

#include <type_traits>

namespace rs {

// ------------------------------------------------------------------------------------
// Cross-workgroup hand-off without cache flushes.  Values that another workgroup must
// read within the same launch (page scores, split partials) are published as 64-bit
// words {tag : value} with agent-scope write-through stores; the reader polls each word
// with agent-scope loads until it carries the call's tag.  A word is its own validity
// flag, so no fence (and no L2 write-back / invalidate) is needed.  An arrival counter
// only elects the reader.  Waits are bounded; expiry is recorded in the workspace.
// ------------------------------------------------------------------------------------
__device__ __forceinline__ void publish_f32(uint64_t *p, float v, uint32_t tag)
{
    store_u64_agent(p, ((uint64_t)tag << 32) | __float_as_uint(v));
}

__device__ __forceinline__ float acquire_f32(const uint64_t *p, uint32_t tag, int spin_limit, uint32_t *err)
{
    uint64_t w = load_u64_agent(p);
    int spins = 0;
    while ((uint32_t)(w >> 32) != tag) {
        if (++spins > spin_limit) {
            atomicExch(err, 1u);
            break;
        }
        __builtin_amdgcn_s_sleep(1);
        w = load_u64_agent(p);
    }
    return __uint_as_float((uint32_t)w);
}

// ------------------------------------------------------------------------------------
// top-K of up to 64*NT keys held in LDS by an NT-thread workgroup; thread t handles
// candidates t, t+NT, t+2NT, ...  Radix select (4 passes of 8 bits) finds the K-th
// largest key; every key above it is taken, and of the keys equal to it the lowest
// indices; the result is written in ascending index order.
// ------------------------------------------------------------------------------------
template <int NT>
struct SelectShared {
    __attribute__((aligned(16))) uint32_t hist[4][256];  // one histogram per radix pass, zeroed once
    int wave_tot[NT / 64];
    __attribute__((aligned(16))) int ex_cnt[NT];  // (row, wave) table: greater-than count | equal count << 16
};

// wave64 inclusive prefix sum over ascending lanes, with DPP row shifts and row broadcasts
__device__ __forceinline__ int wave_incl_scan_dpp(int x)
{
    x += __builtin_amdgcn_update_dpp(0, x, 0x111, 0xf, 0xf, false);  // row_shr:1
    x += __builtin_amdgcn_update_dpp(0, x, 0x112, 0xf, 0xf, false);  // row_shr:2
    x += __builtin_amdgcn_update_dpp(0, x, 0x114, 0xf, 0xf, false);  // row_shr:4
    x += __builtin_amdgcn_update_dpp(0, x, 0x118, 0xf, 0xf, false);  // row_shr:8
    x += __builtin_amdgcn_update_dpp(0, x, 0x142, 0xa, 0xf, false);  // row_bcast:15 into rows 1, 3
    x += __builtin_amdgcn_update_dpp(0, x, 0x143, 0xc, 0xf, false);  // row_bcast:31 into rows 2, 3
    return x;
}

__device__ __forceinline__ int lanes_below(uint64_t ballot)
{
    return __builtin_amdgcn_mbcnt_hi((uint32_t)(ballot >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)ballot, 0u));
}

struct NoMark {
    __device__ __forceinline__ void operator()(int) const {}
};

// wave64 minimum, in lane 63: the same lane pattern
template <int CTRL, int ROWS>
__device__ __forceinline__ uint32_t min_step_dpp(uint32_t x)
{
    const uint32_t y = (uint32_t)__builtin_amdgcn_update_dpp((int)x, (int)x, CTRL, ROWS, 0xf, false);
    return y < x ? y : x;
}
__device__ __forceinline__ uint32_t wave_min_dpp(uint32_t x)
{
    x = min_step_dpp<0x111, 0xf>(x);
    x = min_step_dpp<0x112, 0xf>(x);
    x = min_step_dpp<0x114, 0xf>(x);
    x = min_step_dpp<0x118, 0xf>(x);
    x = min_step_dpp<0x142, 0xa>(x);
    return min_step_dpp<0x143, 0xc>(x);
}

// The same selection by one histogram, where the keys' numbers spread over their range: 1023 bins of equal width between the
// smallest and the largest number (the last bin: keys of 0xffffffff, the pages that are kept anyway), or, kByKey, between the
// smallest and the largest key, whose steps grow with the number (positive numbers of which a few hold nearly all of the range,
// as SnapKV's votes are), and the K-th largest is ranked among the few keys of its bin.  The keys stay in registers; four barriers, where the radix passes take nine, read the keys
// anew each time and spend their first pass on a handful of distinct top bytes.  Bound by the vector instructions of two waves
// a SIMD: 2049 keys by 512 threads 8.2 -> 3.2 us.  False, with nothing emitted, where it does not apply: infinities, NaN or an
// extreme range among the numbers (not kByKey), or more than 64 keys in the bin (kByKey: in the last of its subdivisions).  Requires Np <= spread_rows(NT) * NT.
// (16-wave workgroups: 15 rows, as many as the LDS of their callers holds)
constexpr int spread_rows(int NT) { return NT == 1024 ? 15 : 10; }
template <int R0, int R, typename Body>
__device__ __forceinline__ void rows_from(int rows, Body body)
{
    if constexpr (R0 < R) {
        if (R0 < rows) {
            body(std::integral_constant<int, R0>{});
            rows_from<R0 + 1, R>(rows, body);
        }
    }
}
enum SelectSpread { kNoSpread, kByNumber, kByKey };
template <int NT, SelectSpread HOW, typename Emit>
__device__ __forceinline__ bool select_topk_spread(const uint32_t *keys, int Np, int K, SelectShared<NT> &sh, Emit emit)
{
    constexpr int W = NT / 64, kBins = 4 * 256, R = spread_rows(NT);
    static_assert(W == 8 || W == 16, "the layout of the ranges and counts below");
    constexpr int E = W / 4;  // entries of the table of counts a lane sums (R * W of them at most)
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const int rows = (Np + NT - 1) / NT;
    uint32_t *bins = &sh.hist[0][0];
    uint32_t *range = reinterpret_cast<uint32_t *>(sh.ex_cnt);  // W minima, W complements of maxima; later the table of counts
    uint32_t *near_k = range + 256, *near_p = near_k + 64, *n_near = near_k + 128;  // the keys of the bin, their indices, how many
#pragma unroll
    for (int i = 0; i < kBins / NT; ++i) bins[i * NT + tid] = 0u;
    if (tid == 0) *n_near = 0u;
    // body(integral_constant<r>) for the rows that hold candidates (uniform)
    auto each_row = [&](auto body) __attribute__((always_inline)) { rows_from<0, R>(rows, body); };
    uint32_t kq[R];
    uint32_t lo = 0xffffffffu, nhi = 0xffffffffu;  // the smallest key, and the complement of the largest below 0xffffffff
    each_row([&](auto row) __attribute__((always_inline)) {
        constexpr int r = decltype(row)::value;
        const int p = r * NT + tid;
        kq[r] = keys[p < Np ? p : Np - 1];
        lo = kq[r] < lo ? kq[r] : lo;
        const uint32_t nk = kq[r] == 0xffffffffu ? 0xffffffffu : ~kq[r];
        nhi = nk < nhi ? nk : nhi;
    });
    lo = wave_min_dpp(lo);
    nhi = wave_min_dpp(nhi);
    if (lane == 63) {
        range[wave] = lo;
        range[W + wave] = nhi;
    }
    __syncthreads();
    {
        uint32_t x = range[lane & (2 * W - 1)];  // lanes W - 1 and 2 W - 1 come to hold the minima over W lanes
        x = min_step_dpp<0x111, 0xf>(x);
        x = min_step_dpp<0x112, 0xf>(x);
        x = min_step_dpp<0x114, 0xf>(x);
        if constexpr (W == 16) x = min_step_dpp<0x118, 0xf>(x);
        lo = (uint32_t)__builtin_amdgcn_readlane((int)x, W - 1);
        nhi = (uint32_t)__builtin_amdgcn_readlane((int)x, 2 * W - 1);
    }
    auto number = [](uint32_t k) __attribute__((always_inline)) {
        return __uint_as_float(k ^ (~(uint32_t)((int32_t)k >> 31) | 0x80000000u));
    };
    // finite numbers only: between the keys of the largest negative and positive ones
    const float f_lo = number(lo), width = number(~nhi) - f_lo;
    if (HOW == kByNumber && (lo < 0x00800000u || nhi < ~0xff7fffffu || !(width > 1e-30f && width < 1e38f))) {
        __syncthreads();
        return false;
    }
    const float per = (float)(kBins - 1) / width;
    const uint32_t reach = (~nhi > lo) ? ~nhi - lo : 0u;
    int shift = reach >= (uint32_t)kBins ? 22 - __builtin_clz(reach) : 0;  // reach >> shift < kBins
    // ascending with the number: difference and product are rounded monotonically
    int bn[R];
    each_row([&](auto row) __attribute__((always_inline)) {
        constexpr int r = decltype(row)::value;
        const int x = HOW == kByKey ? (int)((kq[r] - lo) >> shift) : (int)((number(kq[r]) - f_lo) * per);
        bn[r] = kq[r] == 0xffffffffu ? kBins - 1 : x < kBins - 1 ? x : kBins - 2;
        if (r * NT + tid < Np) atomicAdd(&bins[bn[r]], 1u);
        else bn[r] = -1;
    });
    __syncthreads();
    int bin, rank, n, want = K;  // rank: of the wanted key in its bin, from 0; n: keys in the bin
    for (;;) {
        // lane l owns bins 16 (63 - l) .. + 15: a prefix sum over ascending lanes counts its bins and every higher one; then the
        // same among the 16 bins of the lane that the wanted key falls to
        const uint4 *mine = reinterpret_cast<const uint4 *>(bins + 16 * (63 - lane));
        int own = 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            const uint4 x = mine[i];
            own += (int)(x.x + x.y) + (int)(x.z + x.w);
        }
        const int incl = wave_incl_scan_dpp(own);
        const uint64_t who = __ballot(incl - own < want && want <= incl);  // exactly one lane
        const int src = (int)__builtin_ctzll(who ? who : 1ull);
        const int above = __builtin_amdgcn_readlane(incl - own, src);
        const int b = 16 * (63 - src) + 15 - (lane & 15);
        const int x = (int)bins[b];
        int in = x;  // over the 16 lanes of a row
        in += __builtin_amdgcn_update_dpp(0, in, 0x111, 0xf, 0xf, false);
        in += __builtin_amdgcn_update_dpp(0, in, 0x112, 0xf, 0xf, false);
        in += __builtin_amdgcn_update_dpp(0, in, 0x114, 0xf, 0xf, false);
        in += __builtin_amdgcn_update_dpp(0, in, 0x118, 0xf, 0xf, false);
        const uint64_t hit = __ballot(above + in - x < want && want <= above + in) & 0xffffull;
        const int at = (int)__builtin_ctzll(hit ? hit : 1ull);
        bin = __builtin_amdgcn_readlane(b, at);
        n = __builtin_amdgcn_readlane(x, at);
        rank = want - 1 - above - __builtin_amdgcn_readlane(in - x, at);
        if (n <= 64) break;
        __syncthreads();
        if (HOW != kByKey || shift == 0 || bin == kBins - 1) return false;
        // a crowded bin: its keys over bins of their own, 1024 to the bin (more land in the last where its width is not that of one)
        lo += (uint32_t)bin << shift;
        shift = shift > 10 ? shift - 10 : 0;
        want = rank + 1;
#pragma unroll
        for (int i = 0; i < kBins / NT; ++i) bins[i * NT + tid] = 0u;
        __syncthreads();
        each_row([&](auto row) __attribute__((always_inline)) {
            constexpr int r = decltype(row)::value;
            const bool in_bin = bn[r] == bin;
            const uint32_t y = (kq[r] - lo) >> shift;
            bn[r] = in_bin ? (y < (uint32_t)(kBins - 1) ? (int)y : kBins - 2) : -1;
            if (in_bin) atomicAdd(&bins[bn[r]], 1u);
        });
        __syncthreads();
    }
    each_row([&](auto row) __attribute__((always_inline)) {
        constexpr int r = decltype(row)::value;
        if (bn[r] == bin) {
            const uint32_t at = atomicAdd(n_near, 1u);
            near_k[at] = kq[r];
            near_p[at] = (uint32_t)(r * NT + tid);
        }
    });
    __syncthreads();
    // the wanted key: larger keys come before it, and equal ones of lower index
    uint32_t kth;
    int pth;
    {
        const uint32_t mk = near_k[lane], mp = near_p[lane];  // (lanes from n on: anything)
        int before = 0;
        for (int j = 0; j < n; ++j) {
            const uint32_t kj = (uint32_t)__builtin_amdgcn_readlane((int)mk, j), pj = (uint32_t)__builtin_amdgcn_readlane((int)mp, j);
            before += (kj > mk || (kj == mk && pj < mp)) ? 1 : 0;
        }
        const uint64_t hit = __ballot(lane < n && before == rank);
        const int src = (int)__builtin_ctzll(hit ? hit : 1ull);
        kth = (uint32_t)__builtin_amdgcn_readlane((int)mk, src);
        pth = __builtin_amdgcn_readlane((int)mp, src);
    }
    // ascending output: order (row, wave, lane); every wave sums the table of counts for itself
    uint64_t who[R];
    each_row([&](auto row) __attribute__((always_inline)) {
        constexpr int r = decltype(row)::value;
        who[r] = __ballot(r * NT + tid < Np && (kq[r] > kth || (kq[r] == kth && r * NT + tid <= pth)));
        if (lane == 0) sh.ex_cnt[r * W + wave] = __popcll(who[r]);
    });
    __syncthreads();
    int ahead = 0;  // before the entry of this lane's E that has the place of this wave's
    {
        int c[E], sum = 0;
#pragma unroll
        for (int i = 0; i < E; ++i) {
            c[i] = (E * lane + i < rows * W) ? sh.ex_cnt[E * lane + i] : 0;
            ahead += i < wave % E ? c[i] : 0;
            sum += c[i];
        }
        ahead += wave_incl_scan_dpp(sum) - sum;
    }
    each_row([&](auto row) __attribute__((always_inline)) {
        constexpr int r = decltype(row)::value;
        const int base = __builtin_amdgcn_readlane(ahead, __builtin_amdgcn_readfirstlane((r * W + wave) / E));
        if ((who[r] >> lane) & 1ull) emit(base + lanes_below(who[r]), r * NT + tid);
    });
    return true;
}

// emit(pos, p): called once per chosen candidate p with its rank pos in ascending order.
// keys: Np keys in LDS.  Requires Np <= 64 * NT.
// SPREAD: try the one histogram first.
template <int NT, SelectSpread SPREAD = kByNumber, typename Emit, typename Mark = NoMark>
__device__ void select_topk_lds(const uint32_t *keys, int Np, int K, SelectShared<NT> &sh, Emit emit,
                                Mark mark = Mark())
{
    constexpr int kSelWaves = NT / 64;
    const int tid = threadIdx.x;
    const int lane = tid & 63, wave = tid >> 6;
    const int rows = (Np + NT - 1) / NT;
    if constexpr (SPREAD != kNoSpread) {
        if (Np <= spread_rows(NT) * NT && select_topk_spread<NT, SPREAD>(keys, Np, K, sh, emit)) return;
    }
    for (int i = tid; i < 4 * 256; i += NT) (&sh.hist[0][0])[i] = 0u;
    __syncthreads();
    // every wave tracks the digits found so far and the rank still wanted (same in all waves)
    uint32_t prefix = 0u;
    int remaining = K;
#pragma nounroll
    for (int pass = 3; pass >= 0; --pass) {
        uint32_t *hist = sh.hist[pass];
        const int shift = pass * 8;
        const uint32_t himask = (pass == 3) ? 0u : (0xffffffffu << (shift + 8));
        for (int r0 = 0; r0 < rows; r0 += 4) {
            // fetch a batch of keys before touching the histogram (LDS atomics in between would
            // keep each key load waiting for the previous one)
            uint32_t kq[4];
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int p = (r0 + j) * NT + tid;
                kq[j] = (p < Np) ? keys[p] : 0u;
            }
#pragma unroll
            for (int j = 0; j < 4; ++j) {
                const int p = (r0 + j) * NT + tid;
                const bool in = p < Np && (kq[j] & himask) == prefix;
                const uint32_t bin = (kq[j] >> shift) & 255u;
                if (pass == 3) {
                    // the top bytes of scores are nearly all alike: one atomic per distinct
                    // value in the wave instead of one per key on the same address
                    uint64_t todo = __ballot(in);
                    while (todo) {
                        const int leader = (int)__builtin_ctzll(todo);
                        const uint32_t lb = (uint32_t)__builtin_amdgcn_readlane((int)bin, leader);
                        const uint64_t same = __ballot(in && bin == lb);
                        if (lane == leader) atomicAdd(&hist[lb], (uint32_t)__popcll(same));
                        todo &= ~same;
                    }
                } else if (in) {
                    atomicAdd(&hist[bin], 1u);
                }
            }
        }
        __syncthreads();
        // lane l owns bins 4(63-l) .. 4(63-l)+3, so a prefix sum over ascending lanes counts
        // the keys in this lane's bins and every higher bin
        const int b0 = 4 * (63 - lane);
        const uint32_t h0 = hist[b0], h1 = hist[b0 + 1], h2 = hist[b0 + 2], h3 = hist[b0 + 3];
        const int own = (int)(h0 + h1 + h2 + h3);
        const int incl = wave_incl_scan_dpp(own);
        const int above = incl - own;
        int bin = 0, rem_new = 0;
        const bool found = above < remaining && remaining <= incl;  // the wanted rank falls in this lane's bins
        if (found) {
            int acc = above;
            bin = b0;
            const uint32_t hh[4] = {h0, h1, h2, h3};
            for (int bb = 3; bb >= 0; --bb) {
                if (acc + (int)hh[bb] >= remaining) {
                    bin = b0 + bb;
                    break;
                }
                acc += (int)hh[bb];
            }
            rem_new = remaining - acc;
        }
        const uint64_t who = __ballot(found);  // exactly one lane
        const int src = (int)__builtin_ctzll(who ? who : 1ull);
        bin = __builtin_amdgcn_readlane(bin, src);
        remaining = __builtin_amdgcn_readlane(rem_new, src);
        prefix |= (uint32_t)bin << shift;
        mark(8 + (3 - pass));
    }
    const uint32_t kth = prefix;   // the K-th largest key
    const int take_eq = remaining;  // how many keys equal to it are taken (lowest indices)

    // Ascending output.  Candidate index = row * NT + wave * 64 + lane, so the order is
    // (row, wave, lane): count per (row, wave) with ballots, scan the table of counts
    // over the workgroup, and rank inside the wave with the ballot bits below the lane.
    for (int r0 = 0; r0 < rows; r0 += 4) {
        uint32_t kq[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = (r0 + j) * NT + tid;
            kq[j] = (p < Np) ? keys[p] : 0u;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = (r0 + j) * NT + tid;
            const uint64_t bg = __ballot(p < Np && kq[j] > kth);
            const uint64_t be = __ballot(p < Np && kq[j] == kth);
            if (lane == 0 && r0 + j < rows) sh.ex_cnt[(r0 + j) * kSelWaves + wave] = __popcll(bg) | (__popcll(be) << 16);
        }
    }
    __syncthreads();
    {
        const int mine = (tid < rows * kSelWaves) ? sh.ex_cnt[tid] : 0;  // entry (i, w) belongs to thread i * waves + w
        const int incl = wave_incl_scan_dpp(mine);
        if (lane == 63) sh.wave_tot[wave] = incl;
        __syncthreads();
        int before = 0;
#pragma unroll
        for (int w = 0; w < kSelWaves; ++w)
            if (w < wave) before += sh.wave_tot[w];
        if (tid < rows * kSelWaves) sh.ex_cnt[tid] = before + incl - mine;
        __syncthreads();
    }
    mark(12);
    for (int r0 = 0; r0 < rows; r0 += 4) {
        uint32_t kq[4];
        int pk[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = (r0 + j) * NT + tid;
            kq[j] = (p < Np) ? keys[p] : 0u;
            pk[j] = (r0 + j < rows) ? sh.ex_cnt[(r0 + j) * kSelWaves + wave] : 0;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int p = (r0 + j) * NT + tid;
            const bool is_gt = p < Np && kq[j] > kth, is_eq = p < Np && kq[j] == kth;
            const int gt_lane = lanes_below(__ballot(is_gt)), eq_lane = lanes_below(__ballot(is_eq));
            const int gt_before = pk[j] & 0xffff, eq_before = pk[j] >> 16;
            const int quota = take_eq - eq_before;  // equal keys this wave-row may still take
            if (is_gt || (is_eq && eq_lane < quota)) {
                const int eq_taken_before = (eq_before < take_eq ? eq_before : take_eq) +
                                            (quota > 0 ? (eq_lane < quota ? eq_lane : quota) : 0);
                emit(gt_before + gt_lane + eq_taken_before, p);
            }
        }
    }
}

// The same for few candidates, Np <= NT / 2: a candidate's rank is counted outright, NT / Np threads (to a power of two)
// sharing the comparisons, where the radix passes spend their time at barriers.  keys: zeros up to the next multiple of 4;
// counts: NT / 64 words.
template <int NT, typename Emit>
__device__ __forceinline__ void select_topk_few(uint32_t *keys, int Np, int K, int *counts, Emit emit)
{
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    int lg = 31 - __builtin_clz((unsigned)NT) - (Np > 1 ? 32 - __builtin_clz((unsigned)(Np - 1)) : 0);
    if (lg > 6) lg = 6;  // 2^lg threads per candidate, lanes of one wave
    const int p = tid >> lg, part = tid & ((1 << lg) - 1);
    const uint32_t own = (p < Np) ? keys[p] : 1u;
    const int groups = (Np + 3) / 4, own_group = p / 4;  // of four keys; the threads of a candidate take them in turn
    int before = 0;
    if (__any(own == 0u)) {  // (the key of one NaN)
        for (int j = part; j < Np; j += 1 << lg) before += (keys[j] > own || (keys[j] == own && j < p)) ? 1 : 0;
    } else {
        // ahead of the candidate: above it, or equal and of an earlier group (its own group's equals follow)
        for (int gq = part; gq < groups; gq += 1 << lg) {
            const uint4 kq = *reinterpret_cast<const uint4 *>(keys + 4 * gq);
            const uint32_t above = (gq < own_group) ? own - 1u : own;
            before += (int)(kq.x > above) + (int)(kq.y > above) + (int)(kq.z > above) + (int)(kq.w > above);
        }
        if (part == 0 && p < Np) {
#pragma unroll
            for (int c = 0; c < 3; ++c) before += (c < (p & 3) && keys[4 * own_group + c] == own) ? 1 : 0;
        }
    }
    for (int d = 1; d < (1 << lg); d <<= 1) before += __shfl_xor(before, d, 64);
    const bool mine = p < Np && before < K && part == 0;
    const uint64_t who = __ballot(mine);
    if (lane == 0) counts[wave] = __popcll(who);
    __syncthreads();
    int pos = lanes_below(who);
#pragma unroll
    for (int w = 0; w < NT / 64; ++w)
        if (w < wave) pos += counts[w];
    if (mine) emit(pos, p);
}

// Read the Np tagged scores of a unit into keys in LDS, a few loads in flight at a time;
// always-kept pages get the top key.  Ends with a workgroup barrier.
template <int NT>
__device__ __forceinline__ void gather_page_keys(const uint64_t *srow, int Np, int n_first, int n_local,
                                                 uint32_t tag, int spin_limit, uint32_t *err, float *scores_out,
                                                 uint32_t *keys)
{
    // ten loads in flight per thread: 4096 + a few pages of 16 tokens (a 64K context that has grown
    // by some steps) still come in with one round trip
    constexpr int BATCH = 10;
    const int tid = threadIdx.x;
    for (int p0 = tid; p0 < Np; p0 += BATCH * NT) {
        uint64_t wd[BATCH];
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int p = p0 + j * NT;
            wd[j] = (p < Np) ? load_u64_agent(&srow[p]) : 0ull;
        }
#pragma unroll
        for (int j = 0; j < BATCH; ++j) {
            const int p = p0 + j * NT;
            if (p < Np) {
                float sc = __uint_as_float((uint32_t)wd[j]);
                if ((uint32_t)(wd[j] >> 32) != tag) sc = acquire_f32(&srow[p], tag, spin_limit, err);
                if (scores_out) scores_out[p] = sc;
                keys[p] = (p < n_first || p >= Np - n_local) ? 0xffffffffu : float_to_key(sc);
            }
        }
    }
    __syncthreads();
}

// Fold published partials (m, l, o[channel]) of one unit into (M, L, O) for channel `ch`
// (start from M = -inf, L = O = 0, or from the caller's own partial): of the S partials
// those numbered first, first + step, ... (so that several thread groups can share the
// work); words are fetched four splits at a time, stragglers polled.  partial layout per
// split: word 0 = m, word 1 = l, word 2 + c = o[c].
__device__ __forceinline__ void merge_partials(const uint64_t *pu, int S, int stride, int ch, uint32_t tag,
                                               int spin_limit, uint32_t *err, float &M, float &L, float &O,
                                               int first = 0, int step = 1)
{
    for (int s0 = first; s0 < S; s0 += 4 * step) {
        uint64_t wm[4], wl[4], wo[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const uint64_t *p = pu + (long)(s0 + j * step) * stride;
            const bool in = s0 + j * step < S;
            wm[j] = in ? load_u64_agent(p) : 0ull;
            wl[j] = in ? load_u64_agent(p + 1) : 0ull;
            wo[j] = in ? load_u64_agent(p + 2 + ch) : 0ull;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            if (s0 + j * step < S) {
                const uint64_t *p = pu + (long)(s0 + j * step) * stride;
                float ms = __uint_as_float((uint32_t)wm[j]), ls = __uint_as_float((uint32_t)wl[j]),
                      os = __uint_as_float((uint32_t)wo[j]);
                if ((uint32_t)(wm[j] >> 32) != tag) ms = acquire_f32(p, tag, spin_limit, err);
                if ((uint32_t)(wl[j] >> 32) != tag) ls = acquire_f32(p + 1, tag, spin_limit, err);
                if ((uint32_t)(wo[j] >> 32) != tag) os = acquire_f32(p + 2 + ch, tag, spin_limit, err);
                const float mn = fmaxf(M, ms);
                const float a1 = (M == -INFINITY) ? 0.f : __expf(M - mn);
                const float a2 = (ms == -INFINITY) ? 0.f : __expf(ms - mn);
                L = L * a1 + ls * a2;
                O = O * a1 + os * a2;
                M = mn;
            }
        }
    }
}

}  // namespace rs
