// Sparse evaluation at prefill (Sec. 2.2, Eq. 4; App. A.1, MoBA paragraph): every query token
// attends, with a float32 softmax, the tokens i <= t of the blocks its routing picked; the
// dense causal path is the same kernel with every block picked.
//
// Queries of one tile pick different KV blocks, but the matrix cores want dense tiles, so the
// work is regrouped by KV block: for each (batch, head, KV block j) the query rows that
// picked j (and do not live in j) are bucketed into a list; tiles of 128 listed rows attend
// block j as a dense [128 x block] problem and leave a partial (lse, o) per (row, slot); the
// rows' own blocks are dense causal tiles of the same kernel, launched afterwards: their
// epilogue folds in the row's partials and writes the output.  Executed flops stay at the algorithmic count (plus tile padding).
//
// Tile kernel, per wave: 32 query rows against 32-key steps with v_mfma_f32_32x32x16_bf16.
// Scores are formed transposed, S^T = K Q^T, so that a lane holds the keys of ONE query and
// the softmax row reductions are in-lane plus one cross-half swap; O^T = V^T P^T then
// takes P^T straight from the accumulator registers, and V^T through LDS transpose reads of
// the row-major V tile.  K/V tiles pass through a ring of three LDS slots filled by direct
// global -> LDS loads (no staging registers): the loads of the tile two steps ahead are issued one
// at a time between the current tile's matrix instructions, one barrier per step that waits for
// the next tile only.  Tiles are unpadded; an XOR permutation of the 16-byte chunks of each row
// keeps both operand reads conflict-free.
// What bounds it: the causal form holds the matrix units 73 % busy and is then limited by power (the
// clock falls to 1.54 GHz, from 1.69 at the 60 % of two waves per SIMD); the routed forms wait
// for memory and for the fixed parts of a tile (matrix units 46, 16 and 48 % busy in listed tiles, own-block
// tiles and by bit sets; 37, 15 and 39 % with two waves).  Hence 168 registers (steps of 32 keys, 48 KB of
// LDS) and three workgroups per CU instead of 64-key steps with two, every kind of tile as its own
// instantiation with nothing spilled in its loop, and causal tiles launched heaviest first over a
// group of heads per XCD (head by head, the last head's long tiles started late and the chip drained for a
// quarter of the launch).  Before / after, in a kernel trace: causal, 32 over 8 heads, 16001 tokens 2.00 / 1.82 ms
// (1.85 / 1.72 back to back); bit sets, 2 x 32 heads x 4001, blocks of 64, top-8 0.34 / 0.295 ms; regrouped, 32 heads
// x 32768, blocks of 512, top-3 1.20 / 1.12 ms (listed tiles 0.69, own-block tiles 0.43).
// The softmax runs in the base-2 domain (one FMA + one v_exp_f32 per score), moves its
// reference point (and rescales the accumulators) only when a row maximum has grown by more
// than 2^8 (in the causal form: when a lane's weights of a step add up to more than 2^8 each), and masks only on
// steps a boundary crosses.  Partials are kept as bfloat16 o
// (float32 log-sum-exp).  Output rows and partial records pass through LDS on their way out
// and in, so that global memory sees whole 2 D-byte rows.
#include <cstdlib>

#include "common.h"
#include "knobs.h"

#include <type_traits>

namespace rs {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef float f32x16 __attribute__((ext_vector_type(16)));

constexpr int kMT = 128;        // query rows per workgroup tile (4 waves x 32)
constexpr uint32_t kSlotShift = 27;
constexpr float kLazy = 8.f;    // slack (base-2 exponent) before the softmax reference point moves
constexpr float kLarge = 4096.f;  // 16 x 2^kLazy: above it one of a lane's 16 weights of a 32-key sub-tile has passed the slack

// ------------------------------------------------------------------------------------
// bucketing of (row, slot) pairs by picked block
// ------------------------------------------------------------------------------------
__global__ __launch_bounds__(256) void prefill_count_kernel(const int32_t *__restrict__ idx, uint32_t *cnt, long T,
                                                            int block, int Nb, int K)
{
    __shared__ uint32_t hist[256];
    const int tid = threadIdx.x;
    const long bh = blockIdx.y;
    hist[tid] = 0u;
    __syncthreads();
    const long t = (long)blockIdx.x * 256 + tid;
    if (t < T) {
        const int own = (int)(t / block);
        const int32_t *row = idx + (bh * T + t) * K;
        for (int k = 0; k < K; ++k) {
            const int j = row[k];
            if (j >= 0 && j < Nb && j != own) atomicAdd(&hist[j], 1u);
        }
    }
    __syncthreads();
    if (tid < Nb && hist[tid]) atomicAdd(&cnt[bh * Nb + tid], hist[tid]);
}

// per (batch, head): list offsets and tile offsets by block; resets the fill cursors
// tile descriptor of the listed-row launch: block, first list entry, rows
struct TileDesc {
    uint32_t j, lbase, lcount, pad;
};

__global__ __launch_bounds__(256) void prefill_scan_kernel(const uint32_t *cnt, uint32_t *off, uint32_t *tile_off,
                                                           uint32_t *cursor, TileDesc *desc, long desc_stride, int Nb)
{
    __shared__ uint32_t s_c[256], s_t[256];
    const int tid = threadIdx.x;
    const long bh = blockIdx.x;
    const uint32_t c = (tid < Nb) ? cnt[bh * Nb + tid] : 0u;
    s_c[tid] = c;
    s_t[tid] = (c + kMT - 1) / kMT;
    __syncthreads();
    if (tid == 0) {
        uint32_t a = 0, b = 0;
        for (int j = 0; j < Nb; ++j) {
            const uint32_t cj = s_c[j], tj = s_t[j];
            s_c[j] = a;
            s_t[j] = b;
            a += cj;
            b += tj;
        }
        off[bh * (Nb + 1) + Nb] = a;
        tile_off[bh * (Nb + 1) + Nb] = b;
    }
    __syncthreads();
    if (tid < Nb) {
        off[bh * (Nb + 1) + tid] = s_c[tid];
        tile_off[bh * (Nb + 1) + tid] = s_t[tid];
        cursor[bh * Nb + tid] = 0u;
        // one descriptor per tile of this block, so a tile workgroup needs a single dependent load
        const uint32_t nt = (c + kMT - 1) / kMT;
        for (uint32_t i = 0; i < nt; ++i) {
            TileDesc d;
            d.j = (uint32_t)tid;
            d.lbase = s_c[tid] + i * kMT;
            d.lcount = (c - i * kMT < (uint32_t)kMT) ? c - i * kMT : (uint32_t)kMT;
            d.pad = 0u;
            desc[bh * desc_stride + s_t[tid] + i] = d;
        }
    }
}

__global__ __launch_bounds__(256) void prefill_fill_kernel(const int32_t *__restrict__ idx, const uint32_t *off,
                                                           uint32_t *cursor, uint32_t *list, long T, int block, int Nb,
                                                           int K, long list_stride)
{
    __shared__ uint32_t hist[256], base[256];
    const int tid = threadIdx.x;
    const long bh = blockIdx.y;
    hist[tid] = 0u;
    __syncthreads();
    const long t = (long)blockIdx.x * 256 + tid;
    const int own = (int)(t / block);
    const int32_t *row = idx + (bh * T + (t < T ? t : 0)) * K;
    if (t < T) {
        for (int k = 0; k < K; ++k) {
            const int j = row[k];
            if (j >= 0 && j < Nb && j != own) atomicAdd(&hist[j], 1u);
        }
    }
    __syncthreads();
    if (tid < Nb) {
        base[tid] = hist[tid] ? atomicAdd(&cursor[bh * Nb + tid], hist[tid]) : 0u;
        hist[tid] = 0u;
    }
    __syncthreads();
    if (t < T) {
        for (int k = 0; k < K; ++k) {
            const int j = row[k];
            if (j >= 0 && j < Nb && j != own) {
                const uint32_t r = atomicAdd(&hist[j], 1u);
                list[bh * list_stride + off[bh * (Nb + 1) + j] + base[j] + r] = (uint32_t)t | ((uint32_t)k << kSlotShift);
            }
        }
    }
}

// ------------------------------------------------------------------------------------
// tile attention
// ------------------------------------------------------------------------------------
struct PrefillParams {
    const bf16 *q, *k_cache, *v_cache;
    const int32_t *idx;        // NULL: dense causal
    const uint32_t *tile_off, *list;
    const TileDesc *desc;
    long desc_stride;
    uint16_t *part_o;          // [units][T][K][D] bf16
    float *part_lse;           // [units][T][K]
    bf16 *out;
    float *lse_out;
    int Hq, Hkv, Nb, K, block, n_diag;
    int group;                 // causal tiles: units of an XCD whose tiles go out together
    int stream_records;        // partial records past the caches, both ways
    long T, Tcap, list_stride;
    float scale;
};

typedef short s16x4 __attribute__((ext_vector_type(4)));

// LDS transpose read (ds_read_b64_tr_b16): within a group of 16 lanes, lane L supplies the
// address of 4 consecutive 16-bit elements (row L of a 16 x 4 block); lane i receives column
// i % 4 of rows i / 4, i / 4 + 4, i / 4 + 8, i / 4 + 12.  With row L pointing at key (L / 4)
// of a key quad and at d offset 4 (L % 4), lane i ends up with V[key 0..3][d0 + i]: a 4-key x
// 16-channel block of row-major V, transposed into the MFMA operand layout.
__device__ __forceinline__ s16x4 lds_read_tr16(const uint16_t *p)
{
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((__attribute__((address_space(3))) s16x4 *)p);
}

// The four forms of the tile kernel.
//   kDense    causal tiles over all keys
//   kBitSets  the routed form for dense routings (small blocks, many picks per row): the dense
//             causal tiles, each lane carrying the bit set of its row's listed blocks (nothing is
//             attended that is not listed, the row's own block included); a step lies inside one
//             block (block % 64 == 0), a lane whose row did not list it adds nothing there, and a
//             wave none of whose rows listed it skips the step's arithmetic
//   kListed   tiles of listed rows against one block, leaving partials
//   kOwn      rows against their own blocks; folds the partials in and writes y
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));

// the bitwise or over the wave's lanes, as a scalar
__device__ __forceinline__ uint32_t wave_or(uint32_t x)
{
#pragma unroll
    for (int m = 32; m >= 1; m >>= 1) x |= (uint32_t)__shfl_xor((int)x, m);
    return (uint32_t)__builtin_amdgcn_readfirstlane((int)x);
}

enum PrefillForm { kDense, kBitSets, kListed, kOwn };

// SUB: 32-key sub-tiles per step.  One, with three workgroups per CU, where a launch fills the chip;
// two, with twice the independent matrix and vector instructions per wave, where a CU has a workgroup to itself.
// With two the kernel is declared for 512 threads (it is launched with 256): the compiler then keeps the accumulators
// in 256 vector registers, where it otherwise takes 512, half of them accumulation registers, and copies all of them
// every step (causal, 8 heads x 4000 tokens 60.6 -> 56.1 us, 2 x 8 x 535 14.6 -> 12.8).
template <int D, PrefillForm FORM, int SUB>
__global__ __launch_bounds__(SUB == 2 ? 512 : 256) __attribute__((amdgpu_waves_per_eu(SUB == 1 ? 3 : 2, SUB == 1 ? 3 : 2))) void prefill_attn_kernel(const PrefillParams a)
{
    constexpr int kKT = 32 * SUB;  // keys per step
    constexpr int NC = D / 16;     // 16-wide d chunks of the QK^T contraction
    constexpr int NDT = D / 32;    // 32-wide d tiles of O^T
    constexpr int CR = D / 8;      // 16-byte chunks per row
    constexpr int RW = 64 / CR;    // rows one wave-wide load covers
    constexpr int RPI = 4 * RW;    // rows one pass of the four waves covers
    constexpr int CPT = kKT / RPI; // passes per tile (loads per thread per tile, for K and for V)
    // Operands read this many matrix instructions ahead of their use, the order pinned; 0: in the compiler's order, which
    // under 168 registers reads most of them right before they are used, and every matrix instruction waits for an LDS trip.
    // Tiles of listed rows and own-block tiles wait longer than they multiply: 32 heads x 32768, blocks of 512, top-3
    // 1155 -> 1132 us with routing, 16 heads x 20000 380 -> 369, 2 x 32 over 8 heads x 16000, blocks of 256, top-4 1012 -> 1000.  (Three
    // ahead: 1154; six: 1156.)  Causal tiles are limited by power and have fewer registers left (2 x 32 heads x 4001 260 -> 270, by
    // bit sets 326 -> 325, 32 over 8 heads x 16001 1743 -> 1725), 64 channels have few operands (2 x 16 over 8 heads x 20000 392 -> 394).
    constexpr int kAhead = (D == 128 && (FORM == kListed || FORM == kOwn)) ? 4 : 0;
    // a ring of three K and three V tiles as separate objects, addressed with a compile-time index:
    // the compiler then knows that a step's operand reads and the direct loads into another slot
    // cannot overlap, and puts no wait between them
    __shared__ __attribute__((aligned(1024))) uint16_t sK0[kKT * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sK1[kKT * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sK2[kKT * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sV0[kKT * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sV1[kKT * D];
    __shared__ __attribute__((aligned(1024))) uint16_t sV2[kKT * D];

    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int lq = lane & 31, h = lane >> 5;
    // Workgroups are handed to the eight XCDs round-robin in launch order, and each XCD has an L2
    // of its own.  Launch slot L therefore runs on XCD L % 8; give that XCD a run of whole (batch,
    // head) units (query heads that share a KV head stay together).  Causal tiles go out heaviest
    // first over a.group units of the XCD at a time (the remainder first): the last ones to start are
    // the lightest, and the tiles of a unit that run together stream the same K and V rows through that
    // L2.  Tiles of listed rows and own-block tiles are about equally heavy and go out unit by unit.
    int unit, xtile;
    {
        const unsigned nu = gridDim.y, nt = gridDim.x;
        unsigned L = blockIdx.y * nt + blockIdx.x, base = 0, U = nu, group = (unsigned)a.group * 8;
        if (nu % 8 == 0) {
            U = nu / 8;
            base = (L & 7) * U;
            L >>= 3;
            group = (unsigned)a.group;
        }
        if (FORM == kDense || FORM == kBitSets) {
            if (group > U) group = U;
            unsigned n = U % group;  // units of the group at hand
            if (L >= n * nt) {
                L -= n * nt;
                base += n + L / (group * nt) * group;
                L %= group * nt;
                n = group;
            }
            unit = (int)(base + L % n);
            xtile = (int)(L / n);
        } else {
            unit = (int)(base + L / nt);
            xtile = (int)(L % nt);
        }
    }
    const int b = unit / a.Hq, hq = unit % a.Hq, kvh = hq / (a.Hq / a.Hkv);

    // ---- which tile is this ----
    long r0 = 0;       // first row of a contiguous tile
    long kv_begin;     // first key visited
    int n_keys;        // keys visited
    uint32_t lbase = 0, lcount = 0;
    if constexpr (FORM == kListed) {
        if ((uint32_t)xtile >= a.tile_off[(long)unit * (a.Nb + 1) + a.Nb]) return;
        const uint4 dd = *reinterpret_cast<const uint4 *>(a.desc + (long)unit * a.desc_stride + xtile);
        lbase = dd.y;
        lcount = dd.z;
        kv_begin = (long)dd.x * a.block;
        n_keys = (int)((kv_begin + a.block < a.T) ? a.block : a.T - kv_begin);
    } else {
        const int tile = (FORM == kOwn) ? xtile : a.n_diag - 1 - xtile;  // causal tiles: heavy ones first
        r0 = (long)tile * kMT;
        kv_begin = (FORM == kOwn) ? (r0 / a.block) * a.block : 0;
        n_keys = (int)(((r0 + kMT < a.T) ? r0 + kMT : a.T) - kv_begin);
    }
    const int n_steps = (n_keys + kKT - 1) / kKT;

    // ---- staging: global -> LDS, 2 CPT wave-wide loads per tile and wave ----
    // Pass i of a tile: this lane fetches 16 bytes of row RPI i + srow; the wave's rows land
    // contiguously.  The source is a buffer descriptor re-based to the tile's first row and sized
    // to its valid rows: rows past the last visited key read as zeros (finite; their scores are masked).
    const int srow = wave * RW + lane / CR;
    const uint32_t gk = (uint32_t)(srow * D + ((lane % CR) ^ chunk_swizzle<D>(srow)) * 8) * 2u;
    const uint32_t gv = (uint32_t)(srow * D + ((lane % CR) ^ chunk_swizzle<D>(srow & 7)) * 8) * 2u;
    const bf16 *kb = a.k_cache + ((long)(b * a.Hkv + kvh) * a.Tcap + kv_begin) * D;
    const bf16 *vb = a.v_cache + ((long)(b * a.Hkv + kvh) * a.Tcap + kv_begin) * D;
    auto stage = [&](const bf16 *base, uint32_t gsrc, uint16_t *tile, int i, int t) __attribute__((always_inline)) {
        const int rem = n_keys - t * kKT;  // valid rows from here on, >= 1
        const LdsSource src = lds_source_sized(base + (long)t * kKT * D, (rem < kKT ? rem : kKT) * D * 2);
        load16_to_lds_at(src, gsrc, (uint32_t)(i * RPI * D * 2), tile + (i * RPI + wave * RW) * D);
    };
#pragma unroll
    for (int i = 0; i < CPT; ++i) {  // the first tiles only need the block: issue them before the row list is chased
        stage(kb, gk, sK0, i, 0);
        stage(vb, gv, sV0, i, 0);
    }
    if (n_steps > 1) {
#pragma unroll
        for (int i = 0; i < CPT; ++i) {
            stage(kb, gk, sK1, i, 1);
            stage(vb, gv, sV1, i, 1);
        }
    }

    // ---- this lane's query (a column of S^T) ----
    const int rq = wave * 32 + lq;
    // whether the lane's row exists, the row, and (listed rows) its slot
    auto row_of_lane = [&](long &t, int &slot) __attribute__((always_inline)) {
        slot = 0;
        if constexpr (FORM == kListed) {
            const uint32_t e = ((uint32_t)rq < lcount) ? a.list[(long)unit * a.list_stride + lbase + rq] : 0xffffffffu;
            t = (e == 0xffffffffu) ? -1 : (long)(e & ((1u << kSlotShift) - 1u));
            slot = (int)(e >> kSlotShift);
        } else {
            t = (r0 + rq < a.T) ? r0 + rq : -1;
        }
    };
    // last key (from kv_begin) any lane of this wave may see: later steps are skipped by the wave
    // (a wave none of whose 32 rows exists skips every step; it still stages its share of the tiles)
    const bool wave_live = (FORM == kListed) ? ((uint32_t)(wave * 32) < lcount) : (r0 + wave * 32 < a.T);
    int wave_last = n_keys - 1;
    if constexpr (FORM != kListed) {
        const int e = (int)(r0 - kv_begin) + wave * 32 + 31;
        wave_last = (e < wave_last) ? e : wave_last;
    }
    if (!wave_live) wave_last = -1;

    // keys visible to this lane's query, as 32-bit offsets from kv_begin: vis_lo .. vis_hi (a row that
    // does not exist is treated as one; its results are dropped)
    int vis_lo = 0;  // kOwn: past every key where the row's own block is not listed
    auto vis_hi = [&]() __attribute__((always_inline)) -> int {
        if constexpr (FORM == kListed) return n_keys - 1;
        const int e = (int)(r0 - kv_begin) + wave * 32 + (lane & 31);
        return (e < n_keys - 1) ? e : n_keys - 1;
    };
    uint64_t selmask = ~0ull;  // kBitSets: the blocks this lane's row listed (its own block only if listed)
    uint32_t others = 0u;      // kOwn: the slots of the row's other blocks
    bf16x8 qf[NC];
    {
        long tq;
        int slot;
        row_of_lane(tq, slot);
        const bf16 *qrow = a.q + ((long)unit * a.T + (tq >= 0 ? tq : 0)) * D;
#pragma unroll
        for (int c = 0; c < NC; ++c) qf[c] = *reinterpret_cast<const bf16x8 *>(qrow + 16 * c + 8 * h);
        // the row's list, eight entries at a time so that their loads are on their way together
        if constexpr (FORM == kBitSets || FORM == kOwn) {
            selmask = 0ull;
            const int own = (FORM == kOwn && tq >= 0) ? (int)(tq / a.block) : -1;
            bool own_listed = false;
            const int32_t *row = a.idx + ((long)unit * a.T + (tq >= 0 ? tq : 0)) * a.K;
            for (int kk = 0; kk < a.K; kk += 8) {
                int j[8];
#pragma unroll
                for (int u = 0; u < 8; ++u) j[u] = row[(kk + u < a.K) ? kk + u : a.K - 1];
#pragma unroll
                for (int u = 0; u < 8; ++u) {
                    const bool in = tq >= 0 && kk + u < a.K && j[u] >= 0;
                    if constexpr (FORM == kBitSets) {
                        if (in && j[u] < 64) selmask |= 1ull << j[u];
                    } else {
                        own_listed = own_listed || j[u] == own;
                        if (in && j[u] != own) others |= 1u << (kk + u);
                    }
                }
            }
            if constexpr (FORM == kOwn) vis_lo = own_listed ? (int)((long)own * a.block - kv_begin) : INT32_MAX / 2;
        }
    }
    // kBitSets: the blocks any row of this wave listed, as a scalar: steps outside it are skipped by the wave
    uint64_t wave_mask = ~0ull;
    if constexpr (FORM == kBitSets) wave_mask = (uint64_t)wave_or((uint32_t)(selmask >> 32)) << 32 | wave_or((uint32_t)selmask);

    // ---- operand addresses inside a tile (elements), fixed per lane ----
    // K operand: row lq, chunk 2 c + h.  V operand through the transpose read: lane =
    // 32 h + 16 dg + L supplies 8 bytes of row 16 c + 4 h + (L >> 2) (+ 8 for the
    // second read) at d = 32 dt + 16 dg + 4 (L & 3).  The swizzle of K depends on the row modulo
    // 16 and that of V on the row modulo 8 (a transpose read touches eight consecutive rows), so c
    // and the second read enter as plain row offsets.
    const int L = lane & 15, dg = (lane >> 4) & 1;
    uint32_t koff[NC], voff[NDT];
    {
        const int sw = chunk_swizzle<D>(lq);
#pragma unroll
        for (int c = 0; c < NC; ++c) koff[c] = (uint32_t)(lq * D + (((2 * c + h) ^ sw) * 8));
        const int rowa = 4 * h + (L >> 2), sv = chunk_swizzle<D>(rowa);
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt) {
            const int cg = 4 * dt + 2 * dg + ((L & 3) >> 1);
            voff[dt] = (uint32_t)(rowa * D + ((cg ^ sv) * 8) + 4 * (L & 1));
        }
    }

    f32x16 oacc[NDT];
#pragma unroll
    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
        for (int v = 0; v < 16; ++v) oacc[dt][v] = 0.f;
    // running max (the reference point, -inf: none yet) and this lane's half of the running sum, in
    // the base-2 domain: p = 2^(s * scale * log2(e) - m)
    const float cs = a.scale * 1.4426950408889634f;
    float m = -INFINITY, l = 0.f;
    bool moving = true;  // kDense: the last step moved the reference of some row (uniform over the wave)

    const int steps_per_block = a.block / kKT;
    int cur_blk = 0, cur_rem = steps_per_block;  // kBitSets: kv_begin = 0
    // this wave's parts of the first tiles are in LDS
    __builtin_amdgcn_s_waitcnt(0x0F70);
    asm volatile("s_barrier" ::: "memory");

    // One step: keys kKT it .. kKT it + kKT - 1 from ring slot BUF; with NEXT, the tile two steps ahead is
    // staged into the slot the previous step has left, one load at a time between the matrix
    // instructions (a wave that issues its loads in one burst stalls until the CU's vector memory
    // path has taken them).
    auto step = [&](auto main_tag, auto skip_tag, auto mask_tag, auto buf_tag, int it) __attribute__((always_inline)) {
        // MAIN: a further tile two steps ahead is known to exist; otherwise that is looked up here
        constexpr bool MAIN = decltype(main_tag)::value, SKIP = decltype(skip_tag)::value, MASK = decltype(mask_tag)::value;
        constexpr bool NEXT = MAIN && !SKIP;  // stage between the matrix instructions
        constexpr int BUF = decltype(buf_tag)::value;
        const uint16_t *cK = BUF == 0 ? sK0 : BUF == 1 ? sK1 : sK2, *cV = BUF == 0 ? sV0 : BUF == 1 ? sV1 : sV2;
        uint16_t *nK = BUF == 0 ? sK2 : BUF == 1 ? sK0 : sK1, *nV = BUF == 0 ? sV2 : BUF == 1 ? sV0 : sV1;
        const int kr = it * kKT;

        bool sel = true;
        if constexpr (FORM == kBitSets) sel = (selmask >> cur_blk) & 1ull;
        const bool more = MAIN || it + 2 < n_steps;
        // a wave may skip a step past its rows, or of a block that none of its rows listed (whose values may be anything)
        const bool live = !SKIP || (kr <= wave_last && (FORM != kBitSets || ((wave_mask >> cur_blk) & 1ull)));
        if (!NEXT && more) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) stage(kb, gk, nK, i, it + 2);
        }
        if (live) {
            // S^T[key][query] = sum_d K[key][d] Q[query][d].  Matrix phases run at raised priority:
            // of the waves that share a SIMD, the one feeding the matrix pipe is issued first and the
            // others' softmax fills the gaps
            f32x16 sacc[SUB];
            auto scores = [&](auto load_tag) __attribute__((always_inline)) {
                constexpr bool LOAD = decltype(load_tag)::value;
                __builtin_amdgcn_s_setprio(1);
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                    for (int v = 0; v < 16; ++v) sacc[sub][v] = 0.f;
                if constexpr (kAhead > 0) {
                    bf16x8 kf[kAhead];
                    auto read = [&](int n) __attribute__((always_inline)) {
                        kf[n % kAhead] = *reinterpret_cast<const bf16x8 *>(&cK[koff[n]]);
                    };
#pragma unroll
                    for (int n = 0; n < kAhead; ++n) read(n);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int n = 0; n < NC; ++n) {
                        sacc[0] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf[n % kAhead], qf[n], sacc[0], 0, 0, 0);
                        if (n + kAhead < NC) read(n + kAhead);
                        if constexpr (LOAD) {
                            if (n % (NC / CPT) == 0) stage(kb, gk, nK, n / (NC / CPT), it + 2);
                        }
                        __builtin_amdgcn_sched_barrier(0);
                    }
                    __builtin_amdgcn_s_setprio(0);
                    return;
                }
                // kAhead = 0
#pragma unroll
                for (int c = 0; c < NC; ++c) {
                    if constexpr (LOAD) {
                        if (c % (NC / CPT) == 0) stage(kb, gk, nK, c / (NC / CPT), it + 2);
                    }
#pragma unroll
                    for (int sub = 0; sub < SUB; ++sub) {
                        const bf16x8 kf = *reinterpret_cast<const bf16x8 *>(&cK[32 * sub * D + koff[c]]);
                        sacc[sub] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(kf, qf[c], sacc[sub], 0, 0, 0);
                    }
                }
                // issue order: operand reads run three matrix instructions ahead of their use, the direct
                // loads go out one at a time in between
                __builtin_amdgcn_sched_group_barrier(0x100, 2 + SUB, 0);
#pragma unroll
                for (int g = 0; g < SUB * NC - 2 - SUB; ++g) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 1, 0);
                    if (LOAD && g % SUB == 0 && g / SUB < CPT) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 2 + SUB, 0);
                __builtin_amdgcn_s_setprio(0);
            };
            scores(std::integral_constant<bool, NEXT>{});
            // masks only where a boundary crosses this step (uniform over the wave)
            if (MASK && __any(kr < vis_lo || kr + kKT - 1 > vis_hi())) {
                // (in offsets from this lane's first key of the step; far values stay far)
                const int hi = vis_hi() - kr - 4 * h, lo = vis_lo - kr - 4 * h;
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                    for (int v = 0; v < 16; ++v) {
                        const int e = 32 * sub + 8 * (v / 4) + (v % 4);  // + 4 h: folded into lo, hi
                        if (e > hi || e < lo) sacc[sub][v] = -INFINITY;
                    }
            }
            // p = 2^(s * cs + bias) in place of the scores, and their sum over this lane's keys
            auto weights = [&](float bias) __attribute__((always_inline)) -> float {
                float sum = 0.f;
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub) {
                    f32x16 &p = sacc[sub];
#pragma unroll
                    for (int v = 0; v < 16; ++v) p[v] = __builtin_amdgcn_exp2f(fmaf(p[v], cs, bias));
                    float s4[4];
#pragma unroll
                    for (int v = 0; v < 4; ++v) s4[v] = (p[v] + p[v + 4]) + (p[v + 8] + p[v + 12]);
                    sum += (s4[0] + s4[1]) + (s4[2] + s4[3]);
                }
                return sum;
            };
            // the reference point of the exponentials follows the running maximum lazily: it moves
            // only when the maximum has grown by more than kLazy (p then stays below 2^kLazy, or below
            // kLarge * SUB where a step did without the maximum: harmless in float32 and bfloat16), so the accumulators are rarely rescaled
            // (-inf -> finite counts as a move; -inf -> -inf compares false)
            auto weights_by_maximum = [&]() __attribute__((always_inline)) -> float {
                float mx = sacc[0][0];
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub)
#pragma unroll
                    for (int v = 0; v < 16; ++v) mx = fmaxf(mx, sacc[sub][v]);
                mx = half_pair_max(mx) * cs;  // cs > 0: scaling commutes with max
                if (FORM == kBitSets && !sel) mx = -INFINITY;
                if (__any(mx - m > kLazy)) {
                    const float m_new = (mx - m > kLazy) ? mx : m;
                    const float alpha = (m == -INFINITY) ? 0.f : __builtin_amdgcn_exp2f(m - m_new);
                    l *= alpha;
#pragma unroll
                    for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                        for (int v = 0; v < 16; ++v) oacc[dt][v] *= alpha;
                    m = m_new;
                }
                // a row that did not list this step's block: every exponent is -inf, p = 0
                return weights((FORM == kBitSets && !sel) ? -INFINITY : (m == -INFINITY) ? 0.f : -m);
            };
            if constexpr (MAIN && FORM == kDense) {
                // The unmasked steps of a causal tile do without the maximum: the weights are formed with the
                // reference point as it is, and only where they have grown too large (or there is none yet:
                // its negative is +inf then, and they are infinite) the step is taken again by its maximum.
                // 15 of some 95 vector instructions fewer in a loop that power limits: 32 over 8 heads x 16001
                // tokens 1774 -> 1710 us.  (Tiles of listed rows have too few steps: 690 -> 715 us.)
                // Where one step moved the reference the next one goes by its maximum at once: keys whose scores grow by 2^13
                // every 32 tokens 2590 -> 2072 us at that size (1903 with the maximum formed in every step; growth by 2^2
                // 2016 -> 1995 and 1935; ordinary keys 1734 -> 1720 and 1845).
                float ps = 0.f;
                if (!moving) {
                    ps = weights((m == -INFINITY) ? INFINITY : -m);
                    moving = __any(!(ps <= kLarge * SUB));  // some weight is above 2^kLazy: the reference is sure to move
                    if (moving) scores(std::false_type{});
                }
                if (moving) {
                    const float m_old = m;
                    ps = weights_by_maximum();
                    moving = __any(m != m_old);
                }
                l += ps;
            } else {
                l += weights_by_maximum();
            }
            // P^T as the B operand: accumulator values 8c .. 8c+7 are this lane's keys
            // 16c + 4h + {0..3} and 16c + 8 + 4h + {0..3}; V^T is read in the same key order
            __builtin_amdgcn_s_setprio(1);
            if constexpr (kAhead > 0) {
                union {
                    s16x4 s[2];
                    bf16x8 f;
                } vf[kAhead];
                auto read = [&](int n) __attribute__((always_inline)) {
                    const uint16_t *vq = &cV[16 * (n / NDT) * D] + voff[n % NDT];
                    vf[n % kAhead].s[0] = lds_read_tr16(vq);
                    vf[n % kAhead].s[1] = lds_read_tr16(vq + 8 * D);
                };
#pragma unroll
                for (int n = 0; n < kAhead; ++n) read(n);
                bf16x8 pf;
#pragma unroll
                for (int n = 0; n < 2 * NDT; ++n) {
                    if (n % NDT == 0) {
#pragma unroll
                        for (int s8 = 0; s8 < 8; ++s8) pf[s8] = (__bf16)sacc[0][8 * (n / NDT) + s8];
                        if constexpr (NEXT) {
                            if (n / NDT < CPT) stage(vb, gv, nV, n / NDT, it + 2);
                        }
                    }
                    oacc[n % NDT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf[n % kAhead].f, pf, oacc[n % NDT], 0, 0, 0);
                    if (n + kAhead < 2 * NDT) read(n + kAhead);
                    __builtin_amdgcn_sched_barrier(0);
                }
            } else {
#pragma unroll
                for (int sub = 0; sub < SUB; ++sub) {
                    bf16x8 pf[2];
#pragma unroll
                    for (int c = 0; c < 2; ++c)
#pragma unroll
                        for (int s8 = 0; s8 < 8; ++s8) pf[c][s8] = (__bf16)sacc[sub][8 * c + s8];
#pragma unroll
                    for (int c = 0; c < 2; ++c) {
                        if constexpr (NEXT) {
                            if (2 * sub + c < CPT) stage(vb, gv, nV, 2 * sub + c, it + 2);
                        }
#pragma unroll
                        for (int dt = 0; dt < NDT; ++dt) {
                            const uint16_t *vq = &cV[(32 * sub + 16 * c) * D];
                            union {
                                s16x4 s[2];
                                bf16x8 f;
                            } vf;
                            vf.s[0] = lds_read_tr16(vq + voff[dt]);
                            vf.s[1] = lds_read_tr16(vq + voff[dt] + 8 * D);
                            oacc[dt] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(vf.f, pf[c], oacc[dt], 0, 0, 0);
                        }
                    }
                }
                __builtin_amdgcn_sched_group_barrier(0x100, 6, 0);
#pragma unroll
                for (int g = 0; g < SUB * 2 * NDT - 3; ++g) {
                    __builtin_amdgcn_sched_group_barrier(0x008, 1, 0);
                    __builtin_amdgcn_sched_group_barrier(0x100, 2, 0);
                    if (NEXT && g < CPT) __builtin_amdgcn_sched_group_barrier(0x010, 1, 0);
                }
                __builtin_amdgcn_sched_group_barrier(0x008, 3, 0);
            }
            __builtin_amdgcn_s_setprio(0);
        }
        if constexpr (FORM == kBitSets) {  // block of the next step (wave-uniform counters, no division)
            if (--cur_rem == 0) {
                cur_rem = steps_per_block;
                ++cur_blk;
            }
        }
        // (V at the other end of the step: a burst of both stalls the wave; 8 heads x 4000 by bit sets 90.2 -> 86.7 us)
        if (!NEXT && more) {
#pragma unroll
            for (int i = 0; i < CPT; ++i) stage(vb, gv, nV, i, it + 2);
        }
        // the next step's tile has landed (the one after it, staged above, may still be on its way),
        // and this wave has read what it needs of the current one
        if (more) __builtin_amdgcn_s_waitcnt(0x0070 | (2 * CPT));
        else __builtin_amdgcn_s_waitcnt(0x0070);
        asm volatile("s_barrier" ::: "memory");
    };
    {
        using B0 = std::integral_constant<int, 0>;
        using B1 = std::integral_constant<int, 1>;
        using B2 = std::integral_constant<int, 2>;
        using Main = std::integral_constant<bool, FORM == kBitSets || FORM == kOwn>;  // which loops may skip
        // keys past a row only occur in the last 4 / SUB steps of a tile (128 keys from the tile's own rows on;
        // kListed: past the block's end), keys before its own block only in kOwn
        using MainMask = std::integral_constant<bool, FORM == kOwn>;
        constexpr std::true_type yes{};
        constexpr std::false_type no{};
        int it = 0;
        if (FORM == kListed && !wave_live) {  // this wave only stages
            for (; it < n_steps; ++it) {
                const int slot2 = (it + 2) % 3;
                if (it + 2 < n_steps) {
                    uint16_t *nK = slot2 == 0 ? sK0 : slot2 == 1 ? sK1 : sK2, *nV = slot2 == 0 ? sV0 : slot2 == 1 ? sV1 : sV2;
#pragma unroll
                    for (int i = 0; i < CPT; ++i) {
                        stage(kb, gk, nK, i, it + 2);
                        stage(vb, gv, nV, i, it + 2);
                    }
                    __builtin_amdgcn_s_waitcnt(0x0070 | (2 * CPT));
                } else {
                    __builtin_amdgcn_s_waitcnt(0x0070);
                }
                asm volatile("s_barrier" ::: "memory");
            }
            return;
        }
        for (; it + 2 + 4 / SUB < n_steps; it += 3) {
            step(yes, Main{}, MainMask{}, B0{}, it);
            step(yes, Main{}, MainMask{}, B1{}, it + 1);
            step(yes, Main{}, MainMask{}, B2{}, it + 2);
        }
        for (;;) {  // at most six steps are left, the first of them in slot 0
            step(no, yes, yes, B0{}, it);
            if (++it == n_steps) break;
            step(no, yes, yes, B1{}, it);
            if (++it == n_steps) break;
            step(no, yes, yes, B2{}, it);
            if (++it == n_steps) break;
        }
    }
    l = half_pair_sum(l);

    // ---- epilogue ----
    // Rows leave (and partial records enter) through LDS, so that global memory sees whole rows:
    // a lane that wrote its own row's channels straight from the accumulator layout would touch
    // 64 cache lines per store instruction.  After the last step's barrier the tile buffers are
    // free; wave w takes one of them as 32 private rows of D bf16, chunks permuted as in the K/V
    // tiles.  Rows are in channel order: the lane of query row lq, half h holds channels
    // 32 dt + 8 g + 4 h + {0..3} in oacc[dt][4 g ..].
    if (!wave_live) return;  // no barrier below
    uint16_t *stg = (wave == 0) ? sK0 : (wave == 1) ? sK1 : (wave == 2) ? sV0 : sV1;
    const int sw_lq = chunk_swizzle<D>(lq);
    const int frow = lane / CR, fchunk = lane % CR;  // flush: RW rows of CR chunks per instruction
    auto put_rows = [&](float sc) __attribute__((always_inline)) {
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                uint2 w2;
                w2.x = pack_bf16x2(oacc[dt][4 * g] * sc, oacc[dt][4 * g + 1] * sc);
                w2.y = pack_bf16x2(oacc[dt][4 * g + 2] * sc, oacc[dt][4 * g + 3] * sc);
                *reinterpret_cast<uint2 *>(stg + lq * D + (((4 * dt + g) ^ sw_lq) * 8) + 4 * h) = w2;
            }
    };
    auto flush_rows = [&](auto dest_of_row) __attribute__((always_inline)) {
        int ln = lane;  // (opaque: the addresses below are worked out here and not held in registers until then)
        asm volatile("" : "+v"(ln));
#pragma unroll
        for (int i = 0; i < 32 / RW; ++i) {
            const int row = i * RW + ln / CR, c = ln % CR;
            bf16 *dst = dest_of_row(i, row);
            const uint4 v = *reinterpret_cast<const uint4 *>(stg + row * D + ((c ^ chunk_swizzle<D>(row)) * 8));
            if (dst && FORM == kListed && a.stream_records) __builtin_nontemporal_store(u32x4{v.x, v.y, v.z, v.w}, reinterpret_cast<u32x4 *>(dst + c * 8));
            else if (dst) *reinterpret_cast<uint4 *>(dst + c * 8) = v;
        }
    };
    long tq;
    int slot;
    row_of_lane(tq, slot);
    const float inv = (l > 0.f) ? 1.f / l : 0.f;
    const float lse = (l > 0.f) ? (m + __log2f(l)) * 0.6931471805599453f : -INFINITY;
    if constexpr (FORM == kListed) {
        // a partial record: the row's normalised output over one listed block as bf16 (channel
        // order), its log-sum-exp as float32 in an array of its own
        uint32_t ent[32 / RW];  // list entries of the rows this lane helps to flush
#pragma unroll
        for (int i = 0; i < 32 / RW; ++i) {
            const uint32_t rr = (uint32_t)(wave * 32 + i * RW + frow);
            ent[i] = (rr < lcount) ? a.list[(long)unit * a.list_stride + lbase + rr] : 0xffffffffu;
        }
        if (tq >= 0 && h == 0) a.part_lse[((long)unit * a.T + tq) * a.K + slot] = lse;
        put_rows(inv);
        flush_rows([&](int i, int) -> bf16 * {
            if (ent[i] == 0xffffffffu) return nullptr;
            const long t_r = (long)(ent[i] & ((1u << kSlotShift) - 1u));
            const int slot_r = (int)(ent[i] >> kSlotShift);
            return reinterpret_cast<bf16 *>(a.part_o) + (((long)unit * a.T + t_r) * a.K + slot_r) * D;
        });
        return;
    }
    const long wrow0 = r0 + wave * 32;  // contiguous tiles: the wave's first row
    float out_scale = inv;
    float out_lse = lse;
    if constexpr (FORM == kOwn) {
        // own-block tile: fold in the partials the listed-row tiles left for this row's other
        // blocks (they ran in the previous launch).  Two slots at a time: their records of the
        // wave's 32 rows come in by row-contiguous loads, pass through LDS one slot after the
        // other, and the lanes pick their channels there.
        const long rbase = ((long)unit * a.T + (tq >= 0 ? tq : wrow0)) * a.K;
        float M = lse;  // (-inf, and nothing accumulated, where the own block is not listed)
        float wsum = (M == -INFINITY) ? 0.f : 1.f;
#pragma unroll
        for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
            for (int v = 0; v < 16; ++v) oacc[dt][v] *= inv;
        const int rows_here = (int)((a.T - wrow0 < 32) ? a.T - wrow0 : 32);  // >= 1
        for (uint32_t todo = wave_or(others); todo != 0u;) {
            int slots[2];
            slots[0] = __builtin_ctz(todo);
            todo &= todo - 1u;
            const bool two = todo != 0u;
            slots[1] = two ? __builtin_ctz(todo) : slots[0];
            todo &= todo - 1u;  // (0 stays 0)
            u32x4 rec[2][32 / RW];
            float ls[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const bool valid = ((others >> slots[i]) & 1u) && (i == 0 || two);
                const float x = a.part_lse[rbase + slots[i]];
                ls[i] = valid ? x : -INFINITY;
                const uint16_t *src = a.part_o + (((long)unit * a.T + wrow0) * a.K + slots[i]) * D;
#pragma unroll
                for (int j = 0; j < 32 / RW; ++j) {
                    const int rr = j * RW + frow;
                    const int rc = (rr < rows_here) ? rr : rows_here - 1;
                    const u32x4 *p = reinterpret_cast<const u32x4 *>(src + (uint32_t)(rc * a.K * D + fchunk * 8));
                    rec[i][j] = a.stream_records ? __builtin_nontemporal_load(p) : *p;
                }
            }
            float Mn = M;
#pragma unroll
            for (int i = 0; i < 2; ++i) Mn = fmaxf(Mn, ls[i]);
            const float al = (M == -INFINITY || Mn == -INFINITY) ? 0.f : __expf(M - Mn);
            if (Mn != -INFINITY) {
                M = Mn;
                wsum *= al;
#pragma unroll
                for (int dt = 0; dt < NDT; ++dt)
#pragma unroll
                    for (int v = 0; v < 16; ++v) oacc[dt][v] *= al;
            }
#pragma unroll
            for (int i = 0; i < 2; ++i) {
#pragma unroll
                for (int j = 0; j < 32 / RW; ++j) {
                    const int rr = j * RW + frow;
                    *reinterpret_cast<u32x4 *>(stg + rr * D + ((fchunk ^ chunk_swizzle<D>(rr)) * 8)) = rec[i][j];
                }
                const float w = (ls[i] == -INFINITY) ? 0.f : __expf(ls[i] - M);
                wsum += w;
                if (ls[i] != -INFINITY) {  // a record that was never written may hold anything
#pragma unroll
                    for (int u = 0; u < 4 * NDT; ++u) {
                        const uint2 rc2 = *reinterpret_cast<const uint2 *>(stg + lq * D + ((u ^ sw_lq) * 8) + 4 * h);
                        const int dt = u >> 2, g = u & 3;
                        oacc[dt][4 * g] = fmaf(w, __uint_as_float(rc2.x << 16), oacc[dt][4 * g]);
                        oacc[dt][4 * g + 1] = fmaf(w, __uint_as_float(rc2.x & 0xffff0000u), oacc[dt][4 * g + 1]);
                        oacc[dt][4 * g + 2] = fmaf(w, __uint_as_float(rc2.y << 16), oacc[dt][4 * g + 2]);
                        oacc[dt][4 * g + 3] = fmaf(w, __uint_as_float(rc2.y & 0xffff0000u), oacc[dt][4 * g + 3]);
                    }
                }
            }
        }
        out_scale = (wsum > 0.f) ? 1.f / wsum : 0.f;
        out_lse = (wsum > 0.f) ? M + __logf(wsum) : -INFINITY;
    }
    if (tq >= 0 && h == 0 && a.lse_out) a.lse_out[(long)unit * a.T + tq] = out_lse;
    put_rows(out_scale);
    flush_rows([&](int, int row) -> bf16 * {
        return (wrow0 + row < a.T) ? a.out + ((long)unit * a.T + wrow0 + row) * D : nullptr;
    });
}

__global__ void prefill_zero_kernel(uint32_t *p, long n)
{
    const long i = (long)blockIdx.x * blockDim.x + threadIdx.x;
    if (i < n) p[i] = 0u;
}

// Causal tiles: steps of 64 keys while the launch leaves the chip idle, else of 32.  At 64 channels up to 512 tiles.  At
// 128 channels a 64-key workgroup has a CU's LDS to itself: up to 256 tiles, one a CU; above that the lightest tiles wait
// for a second turn, which pays as long as turn and fixed cost of a tile fit beside the heaviest tile: few such tiles, or long
// heads (up to a share of (n - 3) / 6 of 256 more tiles at n tiles a head, 512 at most).
// Steps of 64 / 32 keys, us in a kernel trace (in brackets the two-wave kernel of 64-key steps that this one replaced):
// 8 heads x 2000 33 / 49 (41), x 4000 64 / 92 (77), x 8000 158 / 194 (173), 32 over 8 x 500 13.9 / 17.3 (15.8), x 1000
// 23.2 / 30.1 (26.0), x 1300 28.6 / 37.2 (37.9), x 2000 49 / 57 (59), batch 2 x 600 19.3 / 21.7 (21.6), x 700 23.7 / 24.4 (22.6),
// 2 x 8 x 535 13.5 / 17.1 (14.5), by bit sets 8 heads x 4000 78 / 112 (80); the other way 32 over 8 heads batch 2 x 900
// 31.4 / 30.5 (31.0), batch 3 x 390 20.9 / 17.5 (18.2), x 640 25.7 / 24.8 (23.1), batch 4 x 390 23.1 / 18.5 (19.0), batch 8 x 200
// 19.0 / 14.6 (16.1), x 300 (768 tiles) 29 / 19 (25).  64 channels: batch 3 x 390 10.8 / 11.4 (13.0), 2000 30 / 34 (43), the
// other way batch 6 x 390 (768 tiles) 17.9 / 14.7 (21.2).
static bool prefill_small_launch(int D, long n, long tiles)
{
    if (D == 64) return tiles <= 512;
    return tiles <= 256 || (tiles <= 512 && 6 * (tiles - 256) <= (n - 3) * 256);
}
// 32-key workgroups of 128 channels come three to a CU.  From 513 to 768 tiles some CUs would hold three heavy ones and others
// two: with more LDS asked for than used only two fit, and the lightest tiles fill the second turn.  Two / three a CU, us in a
// kernel trace: 8 heads x 12000 317 / 335, 16 x 6000 172 / 177, 32 over 8 x 2200 63.5 / 64.4, by bit sets 3 x 16 heads x 1500
// 53.4 / 54.7, 32 x 2500 84 / 86 (the two-wave kernel of 64-key steps: 321, 172, 61.8, 51.3, 77); the other way where heads are
// short, batch 5 x 500 27 / 23, and from more tiles on, 32 x 4000 (1024) 142 / 134.
static unsigned prefill_spare_lds(int D, long n, long tiles)
{
    return D == 128 && n >= 9 && tiles > 512 && tiles <= 768 ? 24 * 1024 : 0;
}

// Units of an XCD whose causal tiles go out together.  The tiles of a group keep the XCD's 96 workgroups busy for about as
// long as its heaviest tile takes (group * n_diag^2 / 2 steps over 96, against n_diag).  Four instead of two or three where units
// fill XCDs: 32 heads x 16000 1771 -> 1758 us, 32 over 8 1743 -> 1719, of 64 channels 1007 -> 1000 (each side's runs within 7), 7 x 8 heads x
// 9549 1108 -> 1091; but not where that leaves one by itself: 5 x 8 heads x 9549 779 / 853, 9 x 8 1395 / 1502, 5 x 8 x 13000 1413 / 1590.
// More units than that only widen what the XCD's 4 MB of L2 see at a time: 8 x 32 heads x 4096 tokens by bit sets, 32 units at a time
// 1530 us, 6 at a time 1213, one after the other 1270.
// A remainder goes out first and does not fill the XCD.  Where every head has keys of its own, of 128 channels, the units are
// divided evenly instead if that is possible with more than half as many at a time.  With the remainder / divided evenly, us:
// 4 x 32 heads x 1983 (16 units an XCD: 4 + 12 / 8 + 8) 148 / 139, x 2300 192 / 179, x 2500 211 / 216, 6 x 32 x 1300 (6 + 18 / 12 + 12)
// 116 / 110, 8 x 32 x 1000 96 / 92, 2 x 32 x 4001 (2 + 6 / 4 + 4) 255 / 251, 3 x 32 x 6000 818 / 783, by bit sets with routing 2 x 32 x
// 4001 307 / 302, 8 x 32 x 4001 1208 / 1194.  The other way where heads share keys or have half the bytes, and L2 is not what counts:
// 6 x 32 over 8 heads x 1535 (8 + 16 / 12 + 12) 120 / 125, by bit sets 160 / 165, 4 x 32 over 8 x 2300 166 / 170, 64 channels 3 x 32 x
// 2300 77 / 83, 6 x 16 over 8 x 2500 90 / 95, 8 x 32 over 8 x 1000 48.7 / 51.5.
static int prefill_group(long units, int heads_per_kv, int D, int n_diag)
{
    int want = (192 + n_diag - 1) / n_diag;
    if (units % 8) return want;
    const long u = units / 8;
    if (want < 4) return u % 4 == 1 ? 3 : 4;
    if (heads_per_kv > 1 || D == 64) return want;
    for (int g = want; 2 * g > want; --g)
        if (u % g == 0) return g;
    return want;
}

template <int D, PrefillForm FORM>
static void prefill_causal_launch(const PrefillParams &p, dim3 grid, hipStream_t stream)
{
    const int sub = knob_or(knobs().prefill_sub, prefill_small_launch(D, grid.x, (long)grid.x * grid.y) ? 2 : 1);
    if (sub == 2) prefill_attn_kernel<D, FORM, 2><<<grid, 256, 0, stream>>>(p);
    else prefill_attn_kernel<D, FORM, 1><<<grid, 256, prefill_spare_lds(D, grid.x, (long)grid.x * grid.y), stream>>>(p);
}

static size_t al256(size_t x) { return (x + 255) & ~(size_t)255; }

struct PrefillLayout {
    size_t off_cnt, off_off, off_tile, off_cursor, off_list, off_desc, off_part_lse, off_part_o, total;
    long list_stride, desc_stride;
};

static PrefillLayout prefill_layout(const rs_shape *s, long T, int block, int K)
{
    PrefillLayout L;
    const long units = (long)s->B * s->Hq;
    const long Nb = (T + block - 1) / block;
    size_t o = RS_WS_CTRL_BYTES;
    L.off_cnt = o;
    o += al256((size_t)units * Nb * 4);
    L.off_off = o;
    o += al256((size_t)units * (Nb + 1) * 4);
    L.off_tile = o;
    o += al256((size_t)units * (Nb + 1) * 4);
    L.off_cursor = o;
    o += al256((size_t)units * Nb * 4);
    L.list_stride = T * (K > 0 ? K : 0);
    L.off_list = o;
    o += al256((size_t)units * L.list_stride * 4);
    L.desc_stride = (T * (K > 1 ? K - 1 : 0) + kMT - 1) / kMT + Nb;  // upper bound of listed-row tiles per (batch, head)
    L.off_desc = o;
    o += al256((size_t)units * L.desc_stride * sizeof(TileDesc));
    L.off_part_lse = o;
    o += al256((size_t)units * T * (K > 0 ? K : 0) * 4);
    L.off_part_o = o;
    o += al256((size_t)units * T * (K > 0 ? K : 0) * s->D * 2);
    L.total = o;
    return L;
}

size_t prefill_ws_bytes(const rs_shape *s, long T, int block, int K) { return prefill_layout(s, T, block, K).total; }

int prefill_dispatch(const rs_shape *s, const void *q, const void *k_cache, const void *v_cache, long T, int block,
                     float scale, const int32_t *idx, int K, void *out, float *lse_out, char *ws, hipStream_t stream)
{
    if (s->dtype != RS_BF16) return RS_UNSUPPORTED;  // the matrix-core path takes bf16 operands
    const long units = (long)s->B * s->Hq;
    const int Nb = (int)((T + block - 1) / block);
    if (T >= (1L << kSlotShift)) return RS_UNSUPPORTED;
    PrefillParams p;
    p.q = (const bf16 *)q;
    p.k_cache = (const bf16 *)k_cache;
    p.v_cache = (const bf16 *)v_cache;
    p.idx = idx;
    p.out = (bf16 *)out;
    p.lse_out = lse_out;
    p.Hq = s->Hq;
    p.Hkv = s->Hkv;
    p.Nb = Nb;
    p.K = K;
    p.block = block;
    p.n_diag = (int)((T + kMT - 1) / kMT);
    p.group = prefill_group(units, s->Hq / s->Hkv, s->D, p.n_diag);
    p.T = T;
    p.Tcap = s->Tcap;
    p.scale = scale;
    p.tile_off = p.list = nullptr;
    p.stream_records = 0;
    p.desc = nullptr;
    p.desc_stride = 0;
    p.part_o = nullptr;
    p.part_lse = nullptr;
    p.list_stride = 0;
    if (idx && Nb > 256) return RS_UNSUPPORTED;
    // Routings that are dense for their length (small blocks, many picks: the paper's 64- and
    // 128-token blocks with top-8 / top-16 at 4K) run as causal tiles with a bit set per row
    // instead of being regrouped by block.  Regrouped, a row costs (K - 1) listed tiles' worth of
    // steps plus a fixed cost per tile (row list, scattered queries, partial records: about 4.3
    // steps) and the fold (about 9); by bit sets it costs the causal steps of its tile, some
    // skipped.  Measured at 8 x 32 heads x 4096 tokens (regrouped / bit sets / plain causal, ms):
    // blocks of 64: top-16 3.14 / 1.20 / 1.30, top-8 1.75 / 1.16, top-4 0.98 / 1.08;
    // blocks of 128: top-8 1.72 / 1.19, top-4 0.98 / 1.15; 8192 tokens, 128, top-8: 0.92 / 1.03.
    const bool can_mask = idx && Nb <= 64 && block % 64 == 0;
    const double by_sets = 0.85 * (p.n_diag + 4.0), regrouped = (K - 1) * (4.3 + block / 64.0) + 9.0;
    const int masked = can_mask ? knob_or(knobs().prefill_masked, by_sets < regrouped ? 1 : 0) : 0;
    if (masked) {
        const dim3 grid((unsigned)p.n_diag, (unsigned)units);
        if (s->D == 128) prefill_causal_launch<128, kBitSets>(p, grid, stream);
        else prefill_causal_launch<64, kBitSets>(p, grid, stream);
        return hipGetLastError() == hipSuccess ? RS_OK : RS_LAUNCH_FAILED;
    }
    if (idx) {
        const PrefillLayout L = prefill_layout(s, T, block, K);
        uint32_t *cnt = (uint32_t *)(ws + L.off_cnt), *off = (uint32_t *)(ws + L.off_off);
        uint32_t *tile_off = (uint32_t *)(ws + L.off_tile), *cursor = (uint32_t *)(ws + L.off_cursor);
        uint32_t *list = (uint32_t *)(ws + L.off_list);
        const long ncnt = units * Nb;
        prefill_zero_kernel<<<(unsigned)((ncnt + 255) / 256), 256, 0, stream>>>(cnt, ncnt);
        const dim3 gr((unsigned)((T + 255) / 256), (unsigned)units);
        prefill_count_kernel<<<gr, 256, 0, stream>>>(idx, cnt, T, block, Nb, K);
        TileDesc *desc = (TileDesc *)(ws + L.off_desc);
        prefill_scan_kernel<<<(unsigned)units, 256, 0, stream>>>(cnt, off, tile_off, cursor, desc, L.desc_stride, Nb);
        prefill_fill_kernel<<<gr, 256, 0, stream>>>(idx, off, cursor, list, T, block, Nb, K, L.list_stride);
        p.tile_off = tile_off;
        p.list = list;
        p.desc = desc;
        p.desc_stride = L.desc_stride;
        p.part_o = (uint16_t *)(ws + L.off_part_o);
        p.part_lse = (float *)(ws + L.off_part_lse);
        p.list_stride = L.list_stride;
        // Records that the memory-side cache would lose before they are read anyway (written and read once, K - 1 a row) go
        // past it; smaller ones are found there.  Routing and attention, plain / streamed, us: 2 x 32 over 8 heads x 16000, blocks of
        // 256, top-4 (786 MB) 1053 / 1021, 16 heads x 20000 (246 MB) 415 / 398, 32 x 13000, 512, top-3 (213 MB) 479 / 473, 32 x
        // 32768 (537 MB) 1166 / 1160; the other way 8 x 16000, 256, top-4 (98 MB) 169 / 175.
        p.stream_records = units * T * (K - 1) * s->D * 2 >= 150l << 20;
    }
    if (idx) {
        // launch 1: tiles of listed rows leave partials; launch 2: own-block tiles fold them in
        const long gathered_tiles = p.desc_stride;  // upper bound per (batch, head)
        const dim3 g0((unsigned)gathered_tiles, (unsigned)units);
        if (K > 1) {
            if (s->D == 128) prefill_attn_kernel<128, kListed, 1><<<g0, 256, 0, stream>>>(p);
            else prefill_attn_kernel<64, kListed, 1><<<g0, 256, 0, stream>>>(p);
        }
    }
    const dim3 grid((unsigned)p.n_diag, (unsigned)units);
    if (idx) {
        if (s->D == 128) prefill_attn_kernel<128, kOwn, 1><<<grid, 256, 0, stream>>>(p);
        else prefill_attn_kernel<64, kOwn, 1><<<grid, 256, 0, stream>>>(p);
    } else {
        if (s->D == 128) prefill_causal_launch<128, kDense>(p, grid, stream);
        else prefill_causal_launch<64, kDense>(p, grid, stream);
    }
    return hipGetLastError() == hipSuccess ? RS_OK : RS_LAUNCH_FAILED;
}

}  // namespace rs
