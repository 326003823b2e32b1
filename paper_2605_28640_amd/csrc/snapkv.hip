// SnapKV cache compression (App. A.1, SnapKV paragraph; Sec. 2.2, Eq. 3 over single tokens):
// the W observation queries at the end of the prompt attend causally; each prefix position
// collects its attention probability summed over the window and over the query heads of its
// KV head's group; the votes are max-pooled; per KV head the K_keep best positions are kept
// (ascending), followed by the window rows.
//
// The [G*W x T] score matrix of a KV head is a dense contraction, done on the matrix cores
// (v_mfma_f32_32x32x16_bf16) in two sweeps over the keys: sweep 1 forms S^T = K Q^T so that
// a lane owns one query row and gets its softmax statistics cheaply; sweep 2 forms S = Q K^T
// so that a lane owns one key column and its vote is an in-lane sum over the query rows.
#include "common.h"
#include "knobs.h"
#include "select.h"

#include <type_traits>

namespace rs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kSnapKeysPerWg = 2048;  // keys per workgroup, at most (fewer when that leaves the chip idle)
constexpr int kSnapKT = 128;          // a workgroup's share of the keys is a multiple of this
constexpr int kSnapTile = 32;         // keys of a wave's tile
// Up to this many chunks the second sweep's workgroups fold the first one's statistics for themselves, 8 KB at most for 128
// rows, and the launch between the sweeps falls away: 8 x 32 heads x 4096 (2 chunks) 134.8 -> 130.2 us, 4 x 8 x 2000 (8 chunks)
// 31.9 -> 30.1.  Every workgroup reads the statistics of all chunks of its head, so that the reads grow with the square of the
// chunks: without the line 2 heads x 128K (256 chunks of 256 rows) took 79 us for 67, one head 120 for 66.
constexpr int kSnapFoldChunks = 8;
constexpr int kSnapStep = 64;         // keys of a step of the first sweep

// Both sweeps bring the keys by direct global -> LDS loads (unpadded rows, 16-byte chunks permuted by chunk_swizzle; rows
// past the end of the keys read as zeros: finite, masked or never stored) that are counted, never drained, while keys are left.
// The second streams them by waves of their own: a wave takes every fourth 32-key tile of the workgroup's keys against
// all query rows of the row tile (up to 128, as fragments in registers) through two private slots of LDS.  A tile's
// fragments are read into registers at once, the slot is free again and the loads of the tile after next go out before the
// first matrix instruction, so that a wave has one to two tiles on their way all the time and waits for nobody but them.
// Bound by memory: 268 MB of keys in 43 us with 64 rows, 48 with 128 (8 heads x 128K, 8 x 32 heads x 4096), where reads alone
// take 38-43; all four waves on one tile of 128 keys, waiting together for the next, took 55-57.
template <int D>
struct SnapStage {
    static constexpr int CR = D / 8;               // 16-byte chunks per row
    static constexpr int RW = 64 / CR;             // rows one wave-wide load covers
    static constexpr int NP = kSnapTile / RW;      // loads per tile
    static constexpr int NO = 16 / RW;             // after this many loads the permutation of the rows' chunks repeats
    uint32_t off[NO];                              // the lane's byte in its row of load i, i modulo NO
    __device__ __forceinline__ SnapStage()
    {
        const int lane = threadIdx.x & 63, srow = lane / CR;
#pragma unroll
        for (int i = 0; i < NO; ++i) off[i] = (uint32_t)(srow * D + ((lane % CR) ^ chunk_swizzle<D>(i * RW + srow)) * 8) * 2u;
    }
    // rows row0 .. row0 + N - 1 of x into a slot, as far as they lie below `rows`
    template <int AUX = 0, int N = kSnapTile>
    __device__ __forceinline__ void tile(const bf16 *x, long row0, long rows, uint16_t *slot) const
    {
        const int n = (int)((rows - row0 < N) ? rows - row0 : N);
        const LdsSource src = lds_source_sized(x + row0 * D, (n > 0 ? n : 0) * D * 2);
#pragma unroll
        for (int i = 0; i < N / RW; ++i) load16_to_lds_at<AUX>(src, off[i % NO], (uint32_t)(i * RW * D * 2), slot + i * RW * D);
    }
};

// A tile's fragments out of a slot: all but the wave's last VM loads have landed, and when this returns the reads have left
// the slot, so that it can be loaded into again.  (One block with its own waits: the compiler would have these
// reads wait for the loads into the other slots too.)
template <int D, int VM>
__device__ __forceinline__ void snap_read_tile(const uint16_t *slots, uint32_t koff, bf16x8 (&kf)[D / 16])
{
    uint32_t at = (uint32_t)(size_t)(__attribute__((address_space(3))) const uint16_t *)slots + 2u * koff;
    asm volatile("" : "+v"(at));  // (the other places are worked out here and not held in registers)
    if constexpr (D == 128) {
        asm volatile("s_waitcnt vmcnt(%16)\n\t"
                     "ds_read_b128 %0, %8\n\tds_read_b128 %1, %9\n\tds_read_b128 %2, %10\n\tds_read_b128 %3, %11\n\t"
                     "ds_read_b128 %4, %12\n\tds_read_b128 %5, %13\n\tds_read_b128 %6, %14\n\tds_read_b128 %7, %15\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3]), "=&v"(kf[4]), "=&v"(kf[5]), "=&v"(kf[6]), "=&v"(kf[7])
                     : "v"(at), "v"(at ^ 32u), "v"(at ^ 64u), "v"(at ^ 96u), "v"(at ^ 128u), "v"(at ^ 160u), "v"(at ^ 192u),
                       "v"(at ^ 224u), "n"(VM)
                     : "memory");
    } else {
        asm volatile("s_waitcnt vmcnt(%8)\n\t"
                     "ds_read_b128 %0, %4\n\tds_read_b128 %1, %5\n\tds_read_b128 %2, %6\n\tds_read_b128 %3, %7\n\t"
                     "s_waitcnt lgkmcnt(0)"
                     : "=&v"(kf[0]), "=&v"(kf[1]), "=&v"(kf[2]), "=&v"(kf[3])
                     : "v"(at), "v"(at ^ 32u), "v"(at ^ 64u), "v"(at ^ 96u), "n"(VM)
                     : "memory");
    }
}

// The wave's tiles in turn: fragments to registers, the next loads, then use(kf, first key of the tile).
// The workgroup's keys are kc0 .. kc1 - 1 of kb; koff: the place of the first operand in the slots' arrays, the wave's
// slot included (operand c: chunk 2 c + h of row lq, permuted: 16 c away by exclusive or).
template <int D, int AUX, typename Use>
__device__ __forceinline__ void snap_stream_keys(const bf16 *kb, long kc0, long kc1, const SnapStage<D> &st, uint16_t *slots0,
                                                 uint16_t *slots1, uint32_t koff, Use use)
{
    constexpr int NC = D / 16;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int tiles = (int)((kc1 - kc0 + kSnapTile - 1) / kSnapTile);
    const int n = (tiles - wave + 3) / 4;  // tiles of this wave (<= 0: none)
    const long k0 = kc0 + (long)wave * kSnapTile;
    auto step = [&](uint16_t *slots, int it) __attribute__((always_inline)) {
        bf16x8 kf[NC];
        snap_read_tile<D, SnapStage<D>::NP>(slots, koff, kf);
        st.template tile<AUX>(kb, k0 + (long)(it + 2) * 4 * kSnapTile, kc1, slots + wave * kSnapTile * D);
        use(kf, k0 + (long)it * 4 * kSnapTile);
    };
    for (int it = 0; it < n; it += 2) {
        step(slots0, it);
        if (it + 1 >= n) break;
        step(slots1, it + 1);
    }
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing is on its way into the slots any more
}

// the row tile's queries (the R rows of a KV head follow each other) by way of the slots as 128 rows: whole rows per load,
// where fragments fetched directly touch 64 cache lines each; ends with the slots free
template <int D, int NRG>
__device__ __forceinline__ void snap_query_fragments(const bf16 *q, int rows, const SnapStage<D> &st, uint16_t *slots,
                                                     bf16x8 (&qf)[NRG][D / 16])
{
    const int lane = threadIdx.x & 63, lq = lane & 31, h = lane >> 5, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    if (wave < NRG) st.tile(q, wave * kSnapTile, rows, slots + wave * kSnapTile * D);
    __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0)
    __syncthreads();
#pragma unroll
    for (int rg = 0; rg < NRG; ++rg)
#pragma unroll
        for (int c = 0; c < D / 16; ++c) qf[rg][c] = *reinterpret_cast<const bf16x8 *>(slots + (rg * kSnapTile + lq) * D + (((2 * c + h) ^ chunk_swizzle<D>(lq)) * 8));
#pragma unroll
    for (int rg = 0; rg < NRG; ++rg)
#pragma unroll
        for (int c = 0; c < D / 16; ++c) asm volatile("" : "+v"(qf[rg][c]));
    __builtin_amdgcn_s_waitcnt(0xC07F);  // lgkmcnt(0)
    __syncthreads();
}

// sweep 1: partial softmax statistics (max, sum) per (query row, key chunk).  S^T = K Q^T: a
// lane owns one query row (a column of S^T), so its max and sum are in-lane reductions plus
// one cross-half shuffle.  Wave w holds rows 32 w .. 32 w + 31 of the 128-row tile and goes over all keys of the chunk,
// 64 at a time and in order: which positions are kept can hang on the last place of these sums (votes that tie to seven
// digits are not rare among thousands), so their order does not follow the shape of the launch.
// The keys of a step lie in one of four slots, loaded by all four waves three steps ahead.
// Bound by memory with up to 64 rows (268 MB of keys in 50 us), partly by the weights' arithmetic with 128 (51-60 us, by
// machine); two slots of 128 keys, loaded during a step and waited for at its end, took 60-68.  (Tiles of the waves' own, as in
// the second sweep, take 44-51 us, and give the sums another order.)
template <int D, bool STREAM>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void snapkv_stats_kernel(
    const bf16 *__restrict__ q_win, const bf16 *__restrict__ k_cache, float *__restrict__ stats, int Hq, int Hkv, long T,
    long Tcap, int W, int n_chunks, float scale, int keys_per_wg)
{
    constexpr int NC = D / 16, AUX = STREAM ? 2 : 0;
    using Stage = SnapStage<D>;
    constexpr int SLOT = kSnapStep * D, OWN = kSnapStep / 4;  // a slot's elements, a wave's rows of a step
    constexpr int LPS = OWN / Stage::RW;                      // a wave's loads of a step
    __shared__ __attribute__((aligned(1024))) uint16_t sK[4 * SLOT];

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, h = lane >> 5;
    const int chunk = blockIdx.x;
    const int bk = blockIdx.y;  // b * Hkv + kvh
    const int G = Hq / Hkv;
    const int R = G * W;  // query rows of this KV head
    const long L = T - W;
    const bf16 *kb = k_cache + (long)bk * Tcap * D;
    const long kc0 = (long)chunk * keys_per_wg;
    const long kc1 = (kc0 + keys_per_wg < T) ? kc0 + keys_per_wg : T;
    const int n_steps = (int)((kc1 - kc0 + kSnapStep - 1) / kSnapStep);
    const int n_row_tiles = (R + 127) / 128;
    const Stage st;
    const uint32_t koff = (uint32_t)(lq * D + ((h ^ chunk_swizzle<D>(lq)) * 8));  // K operand: row lq of a sub-tile, chunk h (chunk 2 c + h: 16 c away by exclusive or)
    const float cs = scale * 1.4426950408889634f;  // base-2 domain
    // a step's loads always go out (past the end of the keys: as zeros), so that the waits can count them
    auto load_step = [&](int it) __attribute__((always_inline)) {
        st.template tile<AUX, OWN>(kb, kc0 + (long)it * kSnapStep + wave * OWN, kc1, sK + (it & 3) * SLOT + wave * OWN * D);
    };

    for (int rt = 0; rt < n_row_tiles; ++rt) {
        const int r = rt * 128 + wave * 32 + lq;
        const bool wave_ok = rt * 128 + wave * 32 < R, r_ok = r < R;
        const long pos = L + (r_ok ? r % W : 0);  // absolute position of the query: keys <= pos are visible
        // the row tile's queries (the R rows of a KV head follow each other) by way of the last two slots: whole rows per
        // load, where fragments fetched directly touch 64 cache lines each
        uint16_t *sq = sK + 2 * SLOT + wave * 32 * D;
        st.tile(q_win + ((long)bk * R + rt * 128) * D, wave * 32, R - rt * 128, sq);
        load_step(0);
        load_step(1);
        bf16x8 qf[NC];
        snap_read_tile<D, 2 * LPS>(sq, koff, qf);
        asm volatile("s_barrier" ::: "memory");  // every wave has its queries: the last two slots are free for keys
        load_step(2);
        float m = -INFINITY, l = 0.f;
        for (int it = 0; it < n_steps; ++it) {
            // this wave's loads of the step have landed; behind the barrier everybody's have, and nobody reads the step before
            asm volatile("s_waitcnt vmcnt(%0)\n\ts_barrier" ::"n"(2 * LPS) : "memory");
            load_step(it + 3);
            if (!wave_ok) continue;
            const uint16_t *slot = sK + (it & 3) * SLOT;
            f32x16 sacc[2];
#pragma unroll
            for (int u = 0; u < 2; ++u) {
                bf16x8 kf[NC];
                snap_read_tile<D, 63>(slot + u * 32 * D, koff, kf);
#pragma unroll
                for (int v = 0; v < 16; ++v) sacc[u][v] = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c) sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[c], qf[c], sacc[u], 0, 0, 0);  // [key][row]
            }
            const long k0 = kc0 + (long)it * kSnapStep;
            if (k0 + kSnapStep > kc1 || k0 + kSnapStep - 1 > L) {  // (uniform)
                // keys of this step a lane may see, as offsets from k0: 0 .. hi
                const long hi_l = ((pos < kc1 - 1) ? pos : kc1 - 1) - k0;
                const int hi = (int)((hi_l > kSnapStep) ? kSnapStep : ((hi_l < -1) ? -1 : hi_l)) - 4 * h;
#pragma unroll
                for (int u = 0; u < 2; ++u)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int e = 32 * u + 8 * (v / 4) + (v % 4);  // + 4 h: folded into hi
                        if (e > hi) sacc[u][v] = -INFINITY;
                    }
            }
            float mx = -INFINITY;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[u][v]);
            mx = half_pair_max(mx) * cs;
            const float m_new = fmaxf(m, mx);
            const float m_safe = (m_new == -INFINITY) ? 0.f : m_new;
            float psum = 0.f;
#pragma unroll
            for (int u = 0; u < 2; ++u)
#pragma unroll
                for (int v = 0; v < 16; ++v) psum += __builtin_amdgcn_exp2f(fmaf(sacc[u][v], cs, -m_safe));
            psum = half_pair_sum(psum);
            l = l * ((m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - m_safe)) + psum;
            m = m_new;
        }
        __builtin_amdgcn_s_waitcnt(0x0F70);  // vmcnt(0): nothing is on its way into the slots any more
        asm volatile("s_barrier" ::: "memory");  // ... nor read out of them
        if (r_ok && h == 0) {  // (max, sum) back in the natural-log domain
            float *sp = stats + (((long)bk * n_chunks + chunk) * R + r) * 2;
            sp[0] = m * 0.6931471805599453f;
            sp[1] = l;
        }
    }
}

// sweep 2: the votes.  S = Q K^T: a lane owns one key column of the wave's tile against all query rows of the
// row tile, so a key's vote is an in-lane sum plus one cross-half shuffle and is written straight out.  Only
// prefix keys (< L) are stored, and every window query sees all of them: no mask is needed.
template <int D, int NRG, bool STREAM, bool FOLD>
__global__ __launch_bounds__(256) __attribute__((amdgpu_waves_per_eu(2, 2))) void snapkv_votes_kernel(
    const bf16 *__restrict__ q_win, const bf16 *__restrict__ k_cache, const float *__restrict__ lse,
    const float *__restrict__ stats, int n_chunks, float *__restrict__ votes, int Hq, int Hkv, long T, long Tcap, int W, float scale, int keys_per_wg,
    uint32_t *__restrict__ sel_hist, long n_hist)
{
    // the selection's bins start at zero
    for (long z = ((long)blockIdx.y * gridDim.x + blockIdx.x) * 256 + threadIdx.x; z < n_hist; z += (long)gridDim.x * gridDim.y * 256)
        sel_hist[z] = 0u;
    constexpr int NC = D / 16, ROWS = 32 * NRG, AUX = STREAM ? 2 : 0;
    using Stage = SnapStage<D>;
    __shared__ __attribute__((aligned(1024))) uint16_t sK0[4 * kSnapTile * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sK1[4 * kSnapTile * D];
    __shared__ __attribute__((aligned(16))) float s_lse2[ROWS];  // row log-sum-exp, base-2 domain

    const int tid = threadIdx.x, lane = tid & 63, wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int lq = lane & 31, h = lane >> 5;
    const int chunk = blockIdx.x;
    const int bk = blockIdx.y;  // b * Hkv + kvh
    const int G = Hq / Hkv;
    const int R = G * W;
    const long L = T - W;
    const bf16 *kb = k_cache + (long)bk * Tcap * D;
    const long kc0 = (long)chunk * keys_per_wg;
    const long kc1 = (kc0 + keys_per_wg < L) ? kc0 + keys_per_wg : L;  // prefix keys only
    const int n_row_tiles = (R + ROWS - 1) / ROWS;
    const Stage st;
    const uint32_t koff = (uint32_t)((wave * kSnapTile + lq) * D + ((h ^ chunk_swizzle<D>(lq)) * 8));
    const float cs = scale * 1.4426950408889634f;
    uint16_t *slot0 = sK0 + wave * kSnapTile * D, *slot1 = sK1 + wave * kSnapTile * D;

    for (int rt = 0; rt < n_row_tiles; ++rt) {
        st.template tile<AUX>(kb, kc0 + wave * kSnapTile, kc1, slot0);
        // the rows' log-sum-exp: from lse, or (FOLD) from the statistics of the first sweep's few chunks
        const int rr = rt * ROWS + tid;
        float2 part[kSnapFoldChunks];
        if (FOLD && tid < ROWS) {
            const float2 *sp = reinterpret_cast<const float2 *>(stats) + (long)bk * n_chunks * R + (rr < R ? rr : 0);
#pragma unroll
            for (int c = 0; c < kSnapFoldChunks; ++c) part[c] = (c < n_chunks) ? sp[(long)c * R] : make_float2(-INFINITY, 0.f);
        }
        bf16x8 qf[NRG][NC];
        snap_query_fragments<D, NRG>(q_win + ((long)bk * R + rt * ROWS) * D, R - rt * ROWS, st, sK1, qf);
        // (base-2 domain; +inf for padding rows: their votes vanish.  The previous row tile's readers are two barriers back.)
        if (tid < ROWS) {
            float x = INFINITY;
            if (!FOLD && rr < R) x = lse[(long)bk * R + rr] * 1.4426950408889634f;
            if (FOLD && rr < R) {
                float M = -INFINITY;
#pragma unroll
                for (int c = 0; c < kSnapFoldChunks; ++c) M = fmaxf(M, part[c].x);
                // (the launch's order of sums, whose lanes beyond the chunks add zeros: the same bits)
#pragma unroll
                for (int c = 0; c < kSnapFoldChunks; ++c) part[c].y = (part[c].x == -INFINITY) ? 0.f : part[c].y * __expf(part[c].x - M);
#pragma unroll
                for (int d = kSnapFoldChunks / 2; d >= 1; d /= 2)
#pragma unroll
                    for (int c = 0; c < d; ++c) part[c].y += part[c + d].y;
                x = (M + __logf(part[0].y)) * 1.4426950408889634f;
            }
            s_lse2[tid] = x;
        }
        __syncthreads();
        st.template tile<AUX>(kb, kc0 + (wave + 4) * kSnapTile, kc1, slot1);
        snap_stream_keys<D, AUX>(kb, kc0, kc1, st, sK0, sK1, koff, [&](const bf16x8 (&kf)[NC], long k0) __attribute__((always_inline)) {
            float vsum = 0.f;
            constexpr int PR = NRG < 2 ? 1 : 2;  // row groups at a time
#pragma unroll
            for (int rp = 0; rp < NRG; rp += PR) {
                f32x16 sacc[PR];
#pragma unroll
                for (int u = 0; u < PR; ++u)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sacc[u][v] = 0.f;
#pragma unroll
                for (int c = 0; c < NC; ++c)
#pragma unroll
                    for (int u = 0; u < PR; ++u)
                        sacc[u] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(qf[rp + u][c], kf[c], sacc[u], 0, 0, 0);  // [row][key]
                // accumulator value v: row 8 (v / 4) + 4 h + v % 4 of the group
#pragma unroll
                for (int u = 0; u < PR; ++u)
#pragma unroll
                    for (int qd = 0; qd < 4; ++qd) {
                        const float4 ls = *reinterpret_cast<const float4 *>(&s_lse2[(rp + u) * 32 + 8 * qd + 4 * h]);
                        vsum += __builtin_amdgcn_exp2f(fmaf(sacc[u][4 * qd], cs, -ls.x));
                        vsum += __builtin_amdgcn_exp2f(fmaf(sacc[u][4 * qd + 1], cs, -ls.y));
                        vsum += __builtin_amdgcn_exp2f(fmaf(sacc[u][4 * qd + 2], cs, -ls.z));
                        vsum += __builtin_amdgcn_exp2f(fmaf(sacc[u][4 * qd + 3], cs, -ls.w));
                    }
            }
            vsum = half_pair_sum(vsum);
            const long key = k0 + lq;
            if (h == 0 && key < kc1) {
                float *dst = votes + (long)bk * L + key;
                *dst = (rt == 0) ? vsum : *dst + vsum;
            }
        });
    }
}

// log-sum-exp of each row over its key chunks: one wave per row, lanes over chunks
__global__ __launch_bounds__(256) void snapkv_lse_kernel(const float *__restrict__ stats, float *__restrict__ lse, int R,
                                                         int n_chunks, long rows_total)
{
    const long i = (long)blockIdx.x * 4 + (threadIdx.x >> 6);
    const int lane = threadIdx.x & 63;
    if (i >= rows_total) return;
    const long bk = i / R;
    const int r = (int)(i % R);
    float M = -INFINITY;
    for (int c = lane; c < n_chunks; c += 64) M = fmaxf(M, stats[((bk * n_chunks + c) * R + r) * 2]);
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) M = fmaxf(M, shfl_xor_f(M, m));
    float Ls = 0.f;
    for (int c = lane; c < n_chunks; c += 64) {
        const float mc = stats[((bk * n_chunks + c) * R + r) * 2];
        if (mc != -INFINITY) Ls += stats[((bk * n_chunks + c) * R + r) * 2 + 1] * __expf(mc - M);
    }
    // fixed butterfly order: the same bits on every run
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) Ls += shfl_xor_f(Ls, m);
    if (lane == 0) lse[i] = M + __logf(Ls);
}

// ------------------------------------------------------------------------------------
// top-K_keep of L pooled votes per (batch, KV head): radix select over the order-preserving
// keys, 8 bits per pass, spread over workgroups of 4096 positions each (one workgroup per
// head would leave most of the chip idle at 128K positions).  Pass p histograms the keys that
// match the bits fixed so far into 256 global bins (the first pass also does the max-pooling); the
// next launch starts by locating the bin that holds the K-th largest key (every workgroup repeats that
// small search instead of passing it on).  After four passes the K-th key is known exactly.  The last
// pass leaves each slice's own bins and its number of keys above the 24 bits fixed before, so that the
// emit launch knows how many kept positions precede its slice and writes them in ascending order
// (equal keys: lowest positions first).  Bound by the launches, not by their work: pooling inside
// the first pass, the slices' bins instead of a launch that counts and 1024 threads a slice took the
// selection of 8 heads x 128K from 38 to 30 us (a first pass of 256 threads: 41).
// ------------------------------------------------------------------------------------
constexpr int kSelThreads = 1024;
constexpr int kSelPerThread = 4;
constexpr int kSelSlice = kSelThreads * kSelPerThread;
constexpr int kSelBins = 260;  // words a slice leaves: 256 bins, the count above them, padding to 16 bytes

// K-th largest key so far: the bits fixed by the first npass passes and the rank still wanted
// inside that prefix.  Called by the 64 lanes of one wave; every lane returns the result.
__device__ __forceinline__ void sel_resolve(const uint32_t *__restrict__ hist_bk, int npass, int K_keep,
                                            uint32_t &prefix, int &remaining)
{
    const int lane = threadIdx.x & 63;
    prefix = 0u;
    remaining = K_keep;
    for (int pp = 0; pp < npass; ++pp) {
        const uint32_t *hp = hist_bk + pp * 256;
        const uint4 hv = *reinterpret_cast<const uint4 *>(hp + lane * 4);
        const uint32_t hh[4] = {hv.x, hv.y, hv.z, hv.w};
        const int own = (int)(hh[0] + hh[1] + hh[2] + hh[3]);
        int suf = own;
#pragma unroll
        for (int d = 1; d < 64; d <<= 1) {
            const int o = __shfl_down(suf, d, 64);
            if (lane + d < 64) suf += o;
        }
        const int above = suf - own;
        const bool mine = above < remaining && remaining <= suf;
        int acc = above, bin = lane * 4;
        for (int bb = 3; bb >= 0; --bb) {
            if (acc + (int)hh[bb] >= remaining) {
                bin = lane * 4 + bb;
                break;
            }
            acc += (int)hh[bb];
        }
        const uint64_t who = __ballot(mine);  // exactly one lane while remaining <= candidates
        const int src = who ? (int)__builtin_ctzll(who) : 0;
        bin = __shfl(bin, src, 64);
        acc = __shfl(acc, src, 64);
        prefix |= (uint32_t)bin << (24 - 8 * pp);
        remaining -= acc;
    }
}

// this thread's keys of the slice: position slice_base + 256 wave + 64 j + lane (a wave
// walks its 256 positions in order); positions past L are flagged invalid
__device__ __forceinline__ void sel_load_keys(const float *__restrict__ src, long L, long slice_base, uint32_t *key,
                                              uint32_t &valid)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    float x[kSelPerThread];
    valid = 0u;
#pragma unroll
    for (int j = 0; j < kSelPerThread; ++j) {
        const long p = slice_base + wave * (64 * kSelPerThread) + j * 64 + lane;
        x[j] = (p < L) ? src[p] : 0.f;
        if (p < L) valid |= 1u << j;
    }
#pragma unroll
    for (int j = 0; j < kSelPerThread; ++j) key[j] = float_to_key(x[j]);
}

// FIRST: the first pass, which pools the raw votes (a slice and `half` positions on either side in LDS),
// stores the pooled ones and takes their keys; LAST: the last one, which leaves slice_bins [slice][257]
template <bool FIRST, bool LAST>
__global__ __launch_bounds__(kSelThreads) void snapkv_sel_hist_kernel(const float *__restrict__ votes, float *__restrict__ pooled,
                                                                      uint32_t *__restrict__ hist, long L, int K_keep,
                                                                      int pass, int half, uint32_t *__restrict__ slice_bins)
{
    constexpr int kHalo = 31;  // pool windows of up to 63
    __shared__ uint32_t lh[256];
    __shared__ uint32_t s_prefix;
    __shared__ float s_v[FIRST ? kSelSlice + 2 * kHalo : 1];
    __shared__ uint32_t s_above;
    const int tid = threadIdx.x;
    const long bk = blockIdx.y, base = (long)blockIdx.x * kSelSlice;
    uint32_t key[kSelPerThread], valid;
    if (tid < 256) lh[tid] = 0u;
    if (LAST && tid == 0) s_above = 0u;
    if constexpr (FIRST) {
        const float *row = votes + bk * L;
        for (int i = tid; i < kSelSlice + 2 * half; i += kSelThreads) {
            const long p = base - half + i;
            if (p >= 0 && p < L) s_v[i] = row[p];
        }
        __syncthreads();
        const int lane = tid & 63, wave = tid >> 6;
        valid = 0u;
#pragma unroll
        for (int j = 0; j < kSelPerThread; ++j) {
            const int off = wave * (64 * kSelPerThread) + j * 64 + lane;
            const long p = base + off;
            float m = 0.f;
            if (p < L) {
                valid |= 1u << j;
                const int lo = (p - half < 0) ? (int)(half - p) : 0;                       // window clipped at the ends,
                const int hi = (p + half > L - 1) ? (int)(L - 1 - p) + half : 2 * half;  // as places from p - half
                m = s_v[off + lo];
                if (lo == 0 && hi == 2 * half) {
#pragma unroll 4
                    for (int i = 1; i <= 2 * half; ++i) m = fmaxf(m, s_v[off + i]);
                } else {
                    for (int i = lo + 1; i <= hi; ++i) m = fmaxf(m, s_v[off + i]);
                }
                pooled[bk * L + p] = m;
            }
            key[j] = float_to_key(m);
        }
    } else {
        sel_load_keys(pooled + bk * L, L, base, key, valid);
        if (tid < 64) {
            uint32_t prefix;
            int remaining;
            sel_resolve(hist + bk * 1024, pass, K_keep, prefix, remaining);
            if (tid == 0) s_prefix = prefix;
        }
        __syncthreads();
    }
    const uint32_t prefix = FIRST ? 0u : s_prefix;
    const int shift = 24 - 8 * pass;
    const uint32_t himask = (pass == 0) ? 0u : (0xffffffffu << (shift + 8));
    int above = 0;
#pragma unroll
    for (int j = 0; j < kSelPerThread; ++j) {
        const bool ok = (valid >> j) & 1u;
        if (ok && (key[j] & himask) == prefix) atomicAdd(&lh[(key[j] >> shift) & 255u], 1u);
        if (LAST) above += (ok && (key[j] & himask) > prefix) ? 1 : 0;
    }
    if constexpr (LAST) {
#pragma unroll
        for (int d = 32; d >= 1; d >>= 1) above += __shfl_xor(above, d, 64);
        if ((tid & 63) == 0) atomicAdd(&s_above, (uint32_t)above);
    }
    __syncthreads();
    if (tid < 256 && lh[tid]) atomicAdd(&hist[(bk * 4 + pass) * 256 + tid], lh[tid]);
    if (LAST && tid < 256 && gridDim.x > 1) {  // (a single slice has none before it)
        uint32_t *mine = slice_bins + (bk * gridDim.x + blockIdx.x) * kSelBins;
        mine[tid] = lh[tid];
        if (tid == 0) mine[256] = s_above;
    }
}

__global__ __launch_bounds__(kSelThreads) void snapkv_sel_emit_kernel(const float *__restrict__ pooled,
                                                                      const uint32_t *__restrict__ hist,
                                                                      const uint32_t *__restrict__ slice_bins,
                                                                      int32_t *__restrict__ idx_out, long L, int K_keep)
{
    constexpr int NW = kSelThreads / 64;
    __shared__ int s_gt[NW], s_eq[NW], s_gt0[NW], s_eq0[NW];
    const int tid = threadIdx.x, lane = tid & 63, wave = tid >> 6;
    const long bk = blockIdx.y;
    const long slice_base = (long)blockIdx.x * kSelSlice;
    int32_t *dst = idx_out + bk * K_keep;
    uint32_t key[kSelPerThread], valid;
    sel_load_keys(pooled + bk * L, L, slice_base, key, valid);
    uint32_t kth;
    int take_eq;
    sel_resolve(hist + bk * 1024, 4, K_keep, kth, take_eq);
    // keys above / equal in the slices before this one: the waves take the slices in turn
    int gt_before = 0, eq_before = 0;
    for (int sl = wave; sl < (int)blockIdx.x; sl += NW) {
        const uint32_t *bins = slice_bins + (bk * gridDim.x + sl) * kSelBins;
        const uint4 b4 = *reinterpret_cast<const uint4 *>(bins + lane * 4);
        const uint32_t bb[4] = {b4.x, b4.y, b4.z, b4.w};
        const int b0 = lane * 4, kb = (int)(kth & 255u);
        gt_before += (lane == 0) ? (int)bins[256] : 0;
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            gt_before += (b0 + i > kb) ? (int)bb[i] : 0;
            eq_before += (b0 + i == kb) ? (int)bb[i] : 0;
        }
    }
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        gt_before += __shfl_xor(gt_before, d, 64);
        eq_before += __shfl_xor(eq_before, d, 64);
    }
    // and in the waves before this one
    int n_gt = 0, n_eq = 0;
#pragma unroll
    for (int j = 0; j < kSelPerThread; ++j) {
        const bool ok = (valid >> j) & 1u;
        n_gt += __popcll(__ballot(ok && key[j] > kth));
        n_eq += __popcll(__ballot(ok && key[j] == kth));
    }
    if (lane == 0) {
        s_gt[wave] = n_gt;
        s_eq[wave] = n_eq;
        s_gt0[wave] = gt_before;
        s_eq0[wave] = eq_before;
    }
    __syncthreads();
    gt_before = eq_before = 0;
#pragma unroll
    for (int w2 = 0; w2 < NW; ++w2) {
        gt_before += s_gt0[w2] + (w2 < wave ? s_gt[w2] : 0);
        eq_before += s_eq0[w2] + (w2 < wave ? s_eq[w2] : 0);
    }
#pragma unroll
    for (int j = 0; j < kSelPerThread; ++j) {
        const long p = slice_base + wave * (64 * kSelPerThread) + j * 64 + lane;
        const bool ok = (valid >> j) & 1u;
        const bool is_gt = ok && key[j] > kth, is_eq = ok && key[j] == kth;
        const uint64_t bg = __ballot(is_gt), be = __ballot(is_eq);
        const int gt_lane = __builtin_amdgcn_mbcnt_hi((uint32_t)(bg >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)bg, 0u));
        const int eq_lane = __builtin_amdgcn_mbcnt_hi((uint32_t)(be >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)be, 0u));
        const int eq_rank = eq_before + eq_lane;  // rank among all positions equal to the K-th vote
        if (is_gt || (is_eq && eq_rank < take_eq)) {
            const int eq_taken = (eq_rank < take_eq) ? eq_rank : take_eq;  // equal positions before this one that are kept
            dst[gt_before + gt_lane + (is_eq ? eq_rank : eq_taken)] = (int32_t)p;
        }
        gt_before += __popcll(bg);
        eq_before += __popcll(be);
    }
}

// copy the kept rows, then the window rows: one 16-byte chunk per thread.  STREAM: the rows are not in the memory-side
// cache (the sweeps streamed), ordinary loads would only evict others for them: 8 x 32 heads x 4096 to 512 33 -> 26 us
template <typename ST, bool STREAM>
__global__ void snapkv_gather_kernel(const ST *__restrict__ k_cache, const ST *__restrict__ v_cache,
                                     const int32_t *__restrict__ idx, ST *__restrict__ kc_out, ST *__restrict__ vc_out,
                                     long T, long Tcap, long Tcap_out, int W, int K_keep, int D, long total)
{
    const int cpr = D * (int)sizeof(ST) / 16;  // chunks per row
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i >= total) return;
    const long rows = K_keep + W;
    const long bk = i / (rows * cpr);
    const long rem = i % (rows * cpr);
    const long r = rem / cpr;
    const int c = (int)(rem % cpr);
    const long srow = (r < K_keep) ? idx[bk * K_keep + r] : (T - W) + (r - K_keep);
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    const u32x4 *ks = reinterpret_cast<const u32x4 *>(k_cache + (bk * Tcap + srow) * D) + c;
    const u32x4 *vs = reinterpret_cast<const u32x4 *>(v_cache + (bk * Tcap + srow) * D) + c;
    const u32x4 kx = STREAM ? __builtin_nontemporal_load(ks) : *ks, vx = STREAM ? __builtin_nontemporal_load(vs) : *vs;
    reinterpret_cast<u32x4 *>(kc_out + (bk * Tcap_out + r) * D)[c] = kx;
    reinterpret_cast<u32x4 *>(vc_out + (bk * Tcap_out + r) * D)[c] = vx;
}

// Short prefixes (at most kSnapOneWgKeys positions per head): pooling, the top-K_keep selection
// and the ascending output in one launch, one 1024-thread workgroup per (batch, KV head) with
// the order-preserving keys of the pooled votes in LDS (the selection the decode kernels use:
// keys above the K-th, then equal ones by lowest position).  At these sizes the five launches
// of the spread-out selection above cost more than the work in them.  The whole compression, one workgroup
// a head / spread out, us: 8 heads x 4096 26 / 40, x 8000 33 / 42, x 12000 40 / 45, x 15360 48 / 48; 8 x 32 heads
// x 4096 127 / 141, x 15360 465 / 502.  (The line is where the keys still fit beside the selection's own LDS.)
constexpr int kSnapOneWgKeys = 15360;  // 60 KiB of keys
constexpr int kSnapOneWgThreads = 1024;

// Up to 256 heads have a CU each, and the selection's chain of barriers is what the launch takes: one histogram (kByKey).  With more
// heads their workgroups cover each other's waits, and what counts is the work: the radix passes (kNoSpread), and up to 3072
// positions the window straight from the caches.  This launch with the radix passes and such windows only / with one histogram
// only / by this rule, us, pooling over 7: 256 heads x 2068 10.6 / 10.5 / 10.4, x 4064 14.5 / 11.7 / 12.0, x 10968 30.6 / 22.0 / 22.1;
// 288 x 2068 14.0 / 15.9 / 13.6, x 4064 19.5 / 19.6 / 17.2, x 8168 31.5 / 29.9 / 28.1; 512 x 668 12.4 / 12.8 / 11.6, x 2068 14.8 /
// 17.5 / 14.4, x 4064 19.7 / 22.1 / 19.2, x 8168 32.3 / 33.3 / 29.8; 1024 x 2068 26.4 / 33.1 / 25.5, x 4064 37.0 / 40.2 / 34.1.  From
// 10240 positions on one histogram is the faster one again, 384 x 14968 50.5 / 46.4.  (That its registers leave room for seven waves
// a SIMD and so for one workgroup a CU is not the reason: with 84 scalar registers, eight waves, 512 x 4064 is 23.1.)
template <SelectSpread HOW>
__global__ __launch_bounds__(kSnapOneWgThreads) void snapkv_pool_select_kernel(const float *__restrict__ votes,
                                                                               float *__restrict__ pooled_out,
                                                                               int32_t *__restrict__ idx_out, int L,
                                                                               int kernel, int K_keep)
{
    __shared__ SelectShared<kSnapOneWgThreads> sh;
    extern __shared__ uint32_t s_keys[];  // L keys; the raw votes at first
    const long bk = blockIdx.x;
    const float *row = votes + bk * L;
    const int half = kernel / 2, tid = threadIdx.x;
    if (HOW == kNoSpread && L <= 3 * kSnapOneWgThreads) {
        for (int p = tid; p < L; p += kSnapOneWgThreads) {
            const int lo = (p - half < 0) ? 0 : p - half;
            const int hi = (p + half > L - 1) ? L - 1 : p + half;
            float m = row[lo];
            for (int j = lo + 1; j <= hi; ++j) m = fmaxf(m, row[j]);
            if (pooled_out) pooled_out[bk * L + p] = m;
            s_keys[p] = float_to_key(m);
        }
    } else {
        // The votes come in by one trip and are pooled from LDS, a place of the window for all of a thread's positions at a time
        // (a window of dependent trips to the caches per position: 8 x 32 heads x 4096 13.1 us for the launch, now 12.0).
        constexpr int R = kSnapOneWgKeys / kSnapOneWgThreads;
        float m[R];
        auto each_row = [&](auto body) __attribute__((always_inline)) {
            rows_from<0, R>((L + kSnapOneWgThreads - 1) / kSnapOneWgThreads, body);
        };
        auto place = [&](int r) __attribute__((always_inline)) {  // positions past the end repeat the last one
            const int p = r * kSnapOneWgThreads + tid;
            return p < L ? p : L - 1;
        };
        each_row([&](auto r) __attribute__((always_inline)) { m[r] = row[place(r)]; });
        each_row([&](auto r) __attribute__((always_inline)) { s_keys[place(r)] = __float_as_uint(m[r]); });
        __syncthreads();
        each_row([&](auto r) __attribute__((always_inline)) {
            const int lo = place(r) - half;
            m[r] = __uint_as_float(s_keys[lo < 0 ? 0 : lo]);
        });
        for (int d = 1 - half; d <= half; ++d)
            each_row([&](auto r) __attribute__((always_inline)) {
                const int at = place(r) + d;
                m[r] = fmaxf(m[r], __uint_as_float(s_keys[at < 0 ? 0 : at < L ? at : L - 1]));
            });
        __syncthreads();
        each_row([&](auto r) __attribute__((always_inline)) {
            const int p = place(r);
            if (pooled_out) pooled_out[bk * L + p] = m[r];
            s_keys[p] = float_to_key(m[r]);
        });
    }
    __syncthreads();
    if (K_keep <= 0) return;
    int32_t *dst = idx_out + bk * K_keep;
    select_topk_lds<kSnapOneWgThreads, HOW>(s_keys, L, K_keep, sh, [dst](int pos, int p) { dst[pos] = p; });
}

static size_t al256s(size_t x) { return (x + 255) & ~(size_t)255; }

struct SnapLayout {
    int n_chunks, R, keys_per_wg;
    size_t off_stats, off_lse, off_votes, off_pooled, off_hist, total;
    int n_slices;
};

static SnapLayout snap_layout(const rs_shape *s, long T, int W)
{
    SnapLayout L;
    const long BK = (long)s->B * s->Hkv;
    L.R = (s->Hq / s->Hkv) * W;
    // keys per workgroup of the two sweeps: 2048, or fewer (a multiple of the 128-key step, at
    // least 256) when that many would leave fewer than about 512 workgroups
    long kpw = (T * BK / 512 + kSnapKT - 1) / kSnapKT * kSnapKT;
    kpw = kpw < 256 ? 256 : kpw > kSnapKeysPerWg ? kSnapKeysPerWg : kpw;
    L.keys_per_wg = (int)kpw;
    L.n_chunks = (int)((T + kpw - 1) / kpw);
    size_t o = RS_WS_CTRL_BYTES;
    L.off_stats = o;
    o += al256s((size_t)BK * L.n_chunks * L.R * 2 * 4);
    L.off_lse = o;
    o += al256s((size_t)BK * L.R * 4);
    L.off_votes = o;
    o += al256s((size_t)BK * (T - W) * 4);
    L.off_pooled = o;
    o += al256s((size_t)BK * (T - W) * 4);
    L.n_slices = (int)((T - W + kSelSlice - 1) / kSelSlice);
    L.off_hist = o;
    o += al256s((size_t)BK * 4 * 256 * 4);
    L.total = o;
    return L;
}

size_t snapkv_ws_bytes(const rs_shape *s, long T, int W) { return (T > W) ? snap_layout(s, T, W).total : RS_WS_CTRL_BYTES; }

int snapkv_dispatch(const rs_shape *s, const void *q_win, const void *k_cache, const void *v_cache, long T, int W,
                    int K_keep, int pool_kernel, float scale, void *kc_out, void *vc_out, long Tcap_out,
                    int32_t *idx_out, float *votes_out, const float *lse_in, char *ws, hipStream_t stream)
{
    if (s->dtype != RS_BF16) return RS_UNSUPPORTED;  // the matrix-core path takes bf16 operands
    const SnapLayout Ly = snap_layout(s, T, W);
    const long BK = (long)s->B * s->Hkv;
    const long L = T - W;
    float *stats = (float *)(ws + Ly.off_stats), *lse = (float *)(ws + Ly.off_lse);
    float *votes = (float *)(ws + Ly.off_votes);
    float *pooled = votes_out ? votes_out : (float *)(ws + Ly.off_pooled);
    const dim3 grid((unsigned)Ly.n_chunks, (unsigned)BK);
    const bf16 *qw = (const bf16 *)q_win, *kc = (const bf16 *)k_cache;
    // groups of 32 query rows a wave holds at a time
#define RS_SNAP_ROWS1(LAUNCH, DD, SS)           \
    do {                                        \
        if (Ly.R <= 32) LAUNCH(DD, 1, SS);      \
        else if (Ly.R <= 64) LAUNCH(DD, 2, SS); \
        else LAUNCH(DD, 4, SS);                 \
    } while (0)
#define RS_SNAP_ROWS(LAUNCH, DD)                    \
    do {                                            \
        if (streaming) RS_SNAP_ROWS1(LAUNCH, DD, true); \
        else RS_SNAP_ROWS1(LAUNCH, DD, false);      \
    } while (0)
    // From about 80 MB of keys on streaming loads: ordinary ones have the memory-side cache make room for every line (cold
    // keys 64 us a sweep against 47 at 268 MB), and what the first sweep leaves there saves the second one and the gather
    // less than that.  The whole compression (with a first sweep by the waves' own tiles), ordinary / streaming, us: 8 heads x 128K 168 / 156, x 97492 141 / 133, x 41000
    // (84 MB) 90.3 / 89.1, 8 x 32 heads x 4096 154 / 134, x 2000 92 / 81, 4 x 8 x 13070 101 / 93; the other way 8 heads x 32768
    // (67 MB) to 1/8 62.6 / 63.3, to 1/16 58.3 / 60.7.
    const bool streaming = BK * T * s->D * 2 >= 80l << 20;
    const bool fold = !lse_in && Ly.n_chunks <= kSnapFoldChunks;
    // the rows' log-sum-exp over all visible keys: handed in by the caller (the prefill attention of
    // the window rows has it), or from a first sweep over the keys
    // ([B, Hq, W] is [B * Hkv][G * W])
    if (!lse_in) {
#define RS_STATS(DD, SS) \
    snapkv_stats_kernel<DD, SS><<<grid, 256, 0, stream>>>(qw, kc, stats, s->Hq, s->Hkv, T, s->Tcap, W, Ly.n_chunks, scale, Ly.keys_per_wg)
        if (s->D == 128 && streaming) RS_STATS(128, true);
        else if (s->D == 128) RS_STATS(128, false);
        else if (streaming) RS_STATS(64, true);
        else RS_STATS(64, false);
#undef RS_STATS
        const long rows_total = BK * Ly.R;
        if (!fold) snapkv_lse_kernel<<<(unsigned)((rows_total + 3) / 4), 256, 0, stream>>>(stats, lse, Ly.R, Ly.n_chunks, rows_total);
    }
    // votes exist for prefix keys only: chunks that start past the prefix are not needed
    const dim3 grid2((unsigned)((L + Ly.keys_per_wg - 1) / Ly.keys_per_wg), (unsigned)BK);
    const bool one_wg = L <= kSnapOneWgKeys && knobs().snap_one_wg != 0;  // (knob 0: the spread-out selection at any length)
    uint32_t *sel_hist = (uint32_t *)(ws + Ly.off_hist);
    const long n_hist = one_wg ? 0 : BK * 1024;
#define RS_VOTES1(DD, GG, SS, FF) \
    snapkv_votes_kernel<DD, GG, SS, FF><<<grid2, 256, 0, stream>>>(qw, kc, lse_in ? lse_in : lse, stats, Ly.n_chunks, votes, s->Hq, s->Hkv, T, s->Tcap, W, scale, Ly.keys_per_wg, sel_hist, n_hist)
#define RS_VOTES(DD, GG, SS)                    \
    do {                                        \
        if (fold) RS_VOTES1(DD, GG, SS, true);  \
        else RS_VOTES1(DD, GG, SS, false);      \
    } while (0)
    if (s->D == 128) RS_SNAP_ROWS(RS_VOTES, 128);
    else RS_SNAP_ROWS(RS_VOTES, 64);
#undef RS_VOTES
#undef RS_VOTES1
#undef RS_SNAP_ROWS
#undef RS_SNAP_ROWS1
    if (one_wg) {
        const bool spread = BK <= 256 || L > 10 * kSnapOneWgThreads;
        auto kern = spread ? snapkv_pool_select_kernel<kByKey> : snapkv_pool_select_kernel<kNoSpread>;
        kern<<<(unsigned)BK, kSnapOneWgThreads, (size_t)L * 4, stream>>>(votes, votes_out, idx_out, (int)L, pool_kernel, K_keep);
    } else {
        const dim3 gs((unsigned)Ly.n_slices, (unsigned)BK);
        // the raw votes are not needed past the pooling: the slices' bins take their place (kSelBins words a slice
        // where there are several, and all but the last of them have kSelSlice votes)
        static_assert(2 * kSelBins <= kSelSlice, "two slices or more leave room for their bins");
        uint32_t *slice_bins = (uint32_t *)votes;
        snapkv_sel_hist_kernel<true, false><<<gs, kSelThreads, 0, stream>>>(votes, pooled, sel_hist, L, K_keep, 0, pool_kernel / 2, nullptr);
        if (K_keep > 0) {
            for (int pass = 1; pass < 3; ++pass)
                snapkv_sel_hist_kernel<false, false><<<gs, kSelThreads, 0, stream>>>(nullptr, pooled, sel_hist, L, K_keep, pass, 0, nullptr);
            snapkv_sel_hist_kernel<false, true><<<gs, kSelThreads, 0, stream>>>(nullptr, pooled, sel_hist, L, K_keep, 3, 0, slice_bins);
            snapkv_sel_emit_kernel<<<gs, kSelThreads, 0, stream>>>(pooled, sel_hist, slice_bins, idx_out, L, K_keep);
        }
    }
    const int cpr = s->D * 2 / 16;
    const long total = BK * (long)(K_keep + W) * cpr;
#define RS_GATHER(SS)                                                                                                  \
    snapkv_gather_kernel<bf16, SS><<<(unsigned)((total + 255) / 256), 256, 0, stream>>>(                               \
        (const bf16 *)k_cache, (const bf16 *)v_cache, idx_out, (bf16 *)kc_out, (bf16 *)vc_out, T, s->Tcap, Tcap_out, W, \
        K_keep, s->D, total)
    if (streaming) RS_GATHER(true);
    else RS_GATHER(false);
#undef RS_GATHER
    return hipGetLastError() == hipSuccess ? RS_OK : RS_LAUNCH_FAILED;
}

}  // namespace rs
