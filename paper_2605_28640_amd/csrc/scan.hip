// Gated decay recurrence (Sec. 2.1, Eq. 1) as a single-pass chunked scan.
//
// s_t = g_t s_{t-1} + (1-g_t) x_t is a first-order linear recurrence: a run of tokens
// acts on the incoming state as s -> A s + B, and two runs compose as
// (A2, B2) o (A1, B1) = (A1 A2, A2 B1 + B2).  One workgroup owns one chunk of tokens of
// one (batch, KV head) for all D channels:
//   1. every lane loads NT consecutive tokens x 8 channels (16-byte loads) and keeps
//      them in registers; it folds them into its (A, Bk, Bv);
//   2. the row groups of a wave are scanned with wave shuffles, the waves of the
//      workgroup through LDS;
//   3. the chunk's incoming state comes from the previous chunk of the same head
//      through a value+tag record in global memory (chunks are numbered by a ticket
//      taken at start, so the predecessor is always already running); the chunk
//      publishes its outgoing state before doing anything else;
//   4. every lane replays its tokens from its incoming state out of registers and
//      stores the rounded states into the cache.
// Inputs are read once and outputs written once: 12 bytes per channel-token for a
// bf16 cache.
//
// The chunks of one unit form a serial chain (one hop is about 0.7 us), which bounds the
// time when there are few (batch, head) pairs.  The channels of Eq. 1 are independent, so
// the kernel can also take a unit to be a slab of DS < D channels of a (batch, head): more,
// shorter chains (a chunk then spans D / DS times as many tokens for the same bytes).  In that form
// the chunks may be laid out from a chunk boundary before the run, so that a run that starts anywhere
// leaves its pages' bounds too (8 heads x 3001 tokens from 5003: 19.6 -> 16.1 us, one launch for two).
#include <cstdlib>
#include <type_traits>

#include "append.h"
#include "common.h"
#include "knobs.h"

namespace rs {

// LEAD: the run starts inside a chunk; the chunks are laid out from the chunk boundary below t0, `lead` tokens before
// the run, where they pass the state on.  A form of its own, as its code takes 17 to 23 registers more: without it
// float32 slabs fit a CU twice (8 heads x 64K 313 -> 301 us), and the form without page bounds, which reads the same
// pieces, loses nothing to the tests against the run's start (bfloat16, 8 heads x 128K 403 -> 360 us).
// PAGE > 0 (a power of two from 16 tokens to the chunk length; the run starts on a chunk boundary, or LEAD): a wave's
// tokens (16 or 32 in bfloat16, 8 or 16 in float32, at 128 or 64 channels) are whole pages or an aligned part of one, so
// the page's channelwise min / max of the stored keys (App. A.1, Quest) leave with the states -- in-lane over the lane's four tokens, shuffles over the row
// groups of a page, and for pages longer than a wave's tokens a fold of the waves' bounds
// through LDS -- and the keys need no second pass.
// TURN: when a workgroup learns which chunk comes next, and sends its loads out.
enum ScanTurn {
    kOneAtATime,  // when the chunk in work is done: slabs, and whole rows in runs of one chunk
    kNextAtEnd,   // whole rows: the next chunk is known from the end of the one before, its loads go out under the replay
    kNextAhead,   // ... and drawn a chunk earlier still, so that nobody waits for the draw
};
template <typename ST, int D, int DS, int NT, int NW, int PAGE, bool LEAD, ScanTurn TURN>
__global__ __launch_bounds__(NW * 64) void rat_scan_chunk_kernel(
    const ST *__restrict__ k, const ST *__restrict__ v, const float *__restrict__ g,
    float *__restrict__ state_k, float *__restrict__ state_v, ST *__restrict__ k_cache,
    ST *__restrict__ v_cache, int BH, long T_new, long t0, long Tcap, int n_chunks,
    uint32_t *ctrl, uint64_t *rec, uint32_t tag, int spin_limit, ST *__restrict__ meta, int lead_arg)
{
    constexpr bool PIPE = TURN != kOneAtATime, AHEAD = TURN == kNextAhead;
    constexpr bool ROOM = TURN == kNextAtEnd && sizeof(ST) == 4;  // registers to spare beside the two sets
    constexpr bool EARLY = !PIPE || ROOM, FENCE = PIPE && !ROOM;
    static_assert(!PIPE || (DS == D && !LEAD), "");
    const int lead = LEAD ? lead_arg : 0;
    const int rec_chunks = LEAD ? n_chunks - 1 : n_chunks;  // records per unit (a lead may add a chunk, the last one leaves none)
    constexpr bool META = PAGE > 0;
    constexpr int TW = (64 / (DS / 8)) * NT;  // tokens of a wave
    static_assert(!META || (PAGE >= 16 && (NW * TW) % (PAGE > 0 ? PAGE : 1) == 0), "pages tile the chunk");
    constexpr bool PG_LDS = META && PAGE > TW;  // a page spans several waves
    __shared__ float s_pg[PG_LDS ? NW : 1][2][PG_LDS ? DS : 1];
    constexpr int LPR = DS / 8;      // lanes per row (of the slab)
    constexpr int RPW = 64 / LPR;    // row groups per wave
    constexpr int CHUNK = NW * RPW * NT;
    constexpr int NS = D / DS;       // slabs per (batch, head)
    using R = Row8<ST>;

    __shared__ int s_ticket;
    __shared__ int s_drawn;  // (a word of its own: s_ticket is still being read when the first chunk parks its drawn ticket)
    __shared__ float s_agg[NW][3][DS];
    __shared__ float s_carry[NW][2][DS];

    const int tid = threadIdx.x;
    const int wave = tid >> 6;
    const int lane = tid & 63;
    const int rg = lane / LPR;
    const int c0 = (lane % LPR) * 8;

    // Persistent workgroups: each keeps taking the next chunk (by ticket) until none is left.  The raw
    // inputs of a chunk live in registers from its loads to its replay; with whole rows (PIPE) there are two such register
    // sets, and the loads of the NEXT ticket go out right behind the current chunk's chain step, under its replay
    // and stores (one workgroup fills a CU).  The prefetched ticket is
    // larger than the one in work and tickets are handed out in increasing order, so the smallest
    // unfinished ticket is always some workgroup's chunk in work: the chain cannot deadlock.
    // Bound by memory: 4 x 32 heads x 64K (13.2 GB) take 2.73 ms, the same traffic without the arithmetic 2.48.  Waits that
    // count exactly are what the overlap hangs on: while the sets were copied into each other and loads and stores went
    // by branches, every chunk's replay waited for the next chunk's loads (us, then / now, 128 channels with bounds in
    // bfloat16: 4 x 32 heads x 64K 2763 / 2727, 32 x 64K 738 / 717; 4 x 32 x 8000 of 64 channels
    // 185 / 170; float32, 8 x 32 heads x 500 91 / 83).
    const int units = BH * NS;
    const int total = units * n_chunks;
    // (kept as 32-bit words: the sets are carried around the chunk loop, and this compiler's back end
    // fails on loop-carried 128-bit vector values)
    constexpr int KW = (int)(sizeof(typename R::raw_t) / 4);
    struct ChunkRegs {
        uint32_t kw[NT][KW], vw[NT][KW];
        float gw[NT][8];
    };
    auto next_ticket = [&]() __attribute__((always_inline)) -> int {
        __syncthreads();  // the previous use of s_ticket (and of the chunk's LDS) is over
        if (tid == 0) s_ticket = (int)atomicAdd(&ctrl[kCtrlTicket], 1u);
        __syncthreads();
        return s_ticket;
    };
    // Whole rows (PIPE) move by buffer instructions, their descriptors based at the chunk's first row and sized to its
    // rows: what lies past the run reads as zeros and is dropped on the way out, so that nothing branches between a
    // chunk's loads and the fold that waits for them, and the wait can count exactly.
    typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
    constexpr int kStream = 2;  // the instructions' bits for streaming access
    const uint32_t lane_el = (uint32_t)((wave * RPW + rg) * NT * D + c0);  // the lane's first channel in a whole-row chunk
    auto rows_of = [&](auto *p, long row0, int rows) __attribute__((always_inline)) {
        return lds_source_sized(p + row0 * D, rows * D * (int)sizeof(*p));
    };
    auto load_chunk = [&](int ticket, ChunkRegs &r) __attribute__((always_inline)) {
        const int j = ticket / units;
        const int unit = ticket % units;
        const int bh = unit / NS;
        const int ch0 = (unit % NS) * DS;
        const long in_row0 = (long)bh * T_new;
        if constexpr (PIPE) {
            const long first = (long)j * CHUNK;
            const int rows = (int)((T_new - first < CHUNK) ? T_new - first : CHUNK);
            const auto kd = rows_of(k, in_row0 + first, rows), vd = rows_of(v, in_row0 + first, rows);
            const auto gd = rows_of(g, in_row0 + first, rows);
            uint32_t el = lane_el;
            asm volatile("" : "+v"(el));  // (worked out here: the constants below then become the instructions' own offsets)
#pragma unroll
            for (int i = 0; i < NT; ++i) {
                auto fetch = [&](const LdsSource &d, uint32_t byte, auto *w) __attribute__((always_inline)) {
                    const u32x4 x = __builtin_amdgcn_raw_buffer_load_b128(d, byte, 0, kStream);
#pragma unroll
                    for (int c = 0; c < 4; ++c) w[c] = __builtin_bit_cast(std::remove_reference_t<decltype(w[0])>, (uint32_t)x[c]);
                };
#pragma unroll
                for (int c = 0; c < KW; c += 4) fetch(kd, el * (uint32_t)sizeof(ST) + i * D * (int)sizeof(ST) + 4 * c, r.kw[i] + c);
#pragma unroll
                for (int c = 0; c < KW; c += 4) fetch(vd, el * (uint32_t)sizeof(ST) + i * D * (int)sizeof(ST) + 4 * c, r.vw[i] + c);
#pragma unroll
                for (int c = 0; c < 8; c += 4) fetch(gd, el * 4u + i * D * 4 + 4 * c, r.gw[i] + c);
            }
            return;
        }
        const long tbase = (long)j * CHUNK + (long)(wave * RPW + rg) * NT - lead;
#pragma unroll
        for (int i = 0; i < NT; ++i) {
            const long t = tbase + i;
            typename R::raw_t kq = R::zero_raw(), vq = R::zero_raw();
            float4 ga = make_float4(1.f, 1.f, 1.f, 1.f), gb = ga;  // outside the run: the identity element (g = 1 keeps the state)
            if ((!LEAD || t >= 0) && t < T_new) {
                const long off = (in_row0 + t) * D + ch0 + c0;
                if constexpr (DS == D) {
                    kq = R::load_raw_nt(k + off);
                    vq = R::load_raw_nt(v + off);
                    typedef float f32x4 __attribute__((ext_vector_type(4)));
                    const f32x4 xa = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(g + off));
                    const f32x4 xb = __builtin_nontemporal_load(reinterpret_cast<const f32x4 *>(g + off + 4));
                    ga = make_float4(xa.x, xa.y, xa.z, xa.w);
                    gb = make_float4(xb.x, xb.y, xb.z, xb.w);
                } else {  // (a slab shares its cache lines with the other slabs of the row, which come by other workgroups: cached loads)
                    kq = R::load_raw(k + off);
                    vq = R::load_raw(v + off);
                    ga = *reinterpret_cast<const float4 *>(g + off);
                    gb = *reinterpret_cast<const float4 *>(g + off + 4);
                }
            }
            __builtin_memcpy(r.kw[i], &kq, sizeof(kq));
            __builtin_memcpy(r.vw[i], &vq, sizeof(vq));
            r.gw[i][0] = ga.x; r.gw[i][1] = ga.y; r.gw[i][2] = ga.z; r.gw[i][3] = ga.w;
            r.gw[i][4] = gb.x; r.gw[i][5] = gb.y; r.gw[i][6] = gb.z; r.gw[i][7] = gb.w;
        }
    };
    // nr: the register set of the next chunk, next: its ticket, unless it was drawn ahead; returns it (>= total: none)
    constexpr int kTicketThread = NW * 64 - 64;  // whole rows: who draws (a wave that does not handle the chain)
    int drawn = total;                           // ... and what it drew last
    auto draw = [&]() __attribute__((always_inline)) -> int {
        int at = kCtrlTicket;
        asm volatile("" : "+v"(at));  // (not known to be one address for all lanes: else the result is waited for at once)
        return (int)atomicAdd(&ctrl[at], 1u);
    };
    auto process_chunk = [&](int ticket, ChunkRegs &r, ChunkRegs &nr, int next) __attribute__((always_inline)) -> int {
    const int j = ticket / units;   // chunk index along T
    const int unit = ticket % units;  // consecutive tickets walk the units first
    const int bh = unit / NS;
    const int ch0 = (unit % NS) * DS;  // first channel of the slab
    const long tbase = (long)j * CHUNK + (long)(wave * RPW + rg) * NT - lead;
    typename R::raw_t kr[NT], vr[NT];
    float4 g0[NT], g1[NT];
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        __builtin_memcpy(&kr[i], r.kw[i], sizeof(kr[i]));
        __builtin_memcpy(&vr[i], r.vw[i], sizeof(vr[i]));
        g0[i] = make_float4(r.gw[i][0], r.gw[i][1], r.gw[i][2], r.gw[i][3]);
        g1[i] = make_float4(r.gw[i][4], r.gw[i][5], r.gw[i][6], r.gw[i][7]);
    }
    if constexpr (PIPE) {
        if (j == n_chunks - 1 && T_new % CHUNK != 0) {  // past the run: the identity element (g = 1 keeps the state; x is 0)
#pragma unroll
            for (int i = 0; i < NT; ++i)
                if (tbase + i >= T_new) g0[i] = g1[i] = make_float4(1.f, 1.f, 1.f, 1.f);
        }
    }

    // A first look at the previous chunk's outgoing state, issued behind the data loads so that its round trip
    // overlaps the fold; the wait below re-polls only if it was not there yet.  (Bfloat16 whole rows, and those drawn ahead, do
    // without: registers that may still be waiting for it hold up every wave's next use of them until the next chunk's
    // loads have landed.)
    uint64_t early0 = 0, early1 = 0;
    if constexpr (EARLY) {
        if (tid < DS && j > 0) {
            const uint64_t *p = rec + (((long)unit * rec_chunks + (j - 1)) * 2) * DS + tid;
            early0 = load_u64_agent(p);
            early1 = load_u64_agent(p + DS);
        }
    }

    // fold own tokens: state -> a * state + b
    float a[8], bk[8], bv[8];
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        a[c] = 1.f;
        bk[c] = 0.f;
        bv[c] = 0.f;
    }
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        float kx[8], vx[8];
        R::unpack(kr[i], kx);
        R::unpack(vr[i], vx);
        const float gg[8] = {g0[i].x, g0[i].y, g0[i].z, g0[i].w, g1[i].x, g1[i].y, g1[i].z, g1[i].w};
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float om = 1.f - gg[c];
            a[c] *= gg[c];
            bk[c] = fmaf(gg[c], bk[c], om * kx[c]);
            bv[c] = fmaf(gg[c], bv[c], om * vx[c]);
        }
        // (token by token: unpacked all at once they do not fit the registers)
        if constexpr (FENCE) {
#pragma unroll
            for (int c = 0; c < 8; ++c) asm volatile("" : "+v"(a[c]), "+v"(bk[c]), "+v"(bv[c]));
        }
    }

    if constexpr (RPW == 4) {
        // Four row groups = the four 16-lane rows of the wave.  Two register swaps (v_permlane16_swap,
        // v_permlane32_swap: no trip through the LDS crossbar) put both members of a pair of rows, then
        // both pairs, side by side in every lane; the wave's total and what precedes each row group
        // follow by composition (first X then Y: A = Ax Ay, B = Ay Bx + By).
        const bool odd = rg & 1, upper = rg >= 2;
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const auto sa = __builtin_amdgcn_permlane16_swap(__float_as_uint(a[c]), __float_as_uint(a[c]), false, false);
            const auto sk = __builtin_amdgcn_permlane16_swap(__float_as_uint(bk[c]), __float_as_uint(bk[c]), false, false);
            const auto sv = __builtin_amdgcn_permlane16_swap(__float_as_uint(bv[c]), __float_as_uint(bv[c]), false, false);
            const float ae = __uint_as_float(sa[0]), ao = __uint_as_float(sa[1]);  // even / odd row of the pair
            const float ke = __uint_as_float(sk[0]), ko = __uint_as_float(sk[1]);
            const float ve = __uint_as_float(sv[0]), vo = __uint_as_float(sv[1]);
            const float PA = ae * ao, PK = fmaf(ao, ke, ko), PV = fmaf(ao, ve, vo);  // the pair
            const auto ta = __builtin_amdgcn_permlane32_swap(__float_as_uint(PA), __float_as_uint(PA), false, false);
            const auto tk = __builtin_amdgcn_permlane32_swap(__float_as_uint(PK), __float_as_uint(PK), false, false);
            const auto tv = __builtin_amdgcn_permlane32_swap(__float_as_uint(PV), __float_as_uint(PV), false, false);
            const float A0 = __uint_as_float(ta[0]), A1 = __uint_as_float(ta[1]);  // lower / upper pair
            const float K0 = __uint_as_float(tk[0]), K1 = __uint_as_float(tk[1]);
            const float V0 = __uint_as_float(tv[0]), V1 = __uint_as_float(tv[1]);
            if (rg == RPW - 1) {  // the wave's total
                s_agg[wave][0][c0 + c] = A0 * A1;
                s_agg[wave][1][c0 + c] = fmaf(A1, K0, K1);
                s_agg[wave][2][c0 + c] = fmaf(A1, V0, V1);
            }
            // what precedes this row group inside its wave: inside its pair, then the lower pair before it
            float xa = odd ? ae : 1.f, xk = odd ? ke : 0.f, xv = odd ? ve : 0.f;
            if (upper) {
                xk = fmaf(xa, K0, xk);
                xv = fmaf(xa, V0, xv);
                xa *= A0;
            }
            a[c] = xa;
            bk[c] = xk;
            bv[c] = xv;
        }
    } else {
    // inclusive scan over the row groups of the wave
#pragma unroll
    for (int d = 1; d < RPW; d <<= 1) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const float pa = shfl_up_f(a[c], d * LPR);
            const float pk = shfl_up_f(bk[c], d * LPR);
            const float pv = shfl_up_f(bv[c], d * LPR);
            if (rg >= d) {
                bk[c] = fmaf(a[c], pk, bk[c]);
                bv[c] = fmaf(a[c], pv, bv[c]);
                a[c] *= pa;
            }
        }
    }
    if (rg == RPW - 1) {
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            s_agg[wave][0][c0 + c] = a[c];
            s_agg[wave][1][c0 + c] = bk[c];
            s_agg[wave][2][c0 + c] = bv[c];
        }
    }
    // exclusive within the wave: what precedes this lane's tokens inside its wave
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        const float pa = shfl_up_f(a[c], LPR);
        const float pk = shfl_up_f(bk[c], LPR);
        const float pv = shfl_up_f(bv[c], LPR);
        a[c] = (rg == 0) ? 1.f : pa;
        bk[c] = (rg == 0) ? 0.f : pk;
        bv[c] = (rg == 0) ? 0.f : pv;
    }
    }
    if constexpr (AHEAD) {
        if (tid == kTicketThread) s_drawn = drawn;  // read behind the barrier below; the chain step's barrier lies before the next write
    }
    __syncthreads();
    int nt = next;
    if constexpr (AHEAD) nt = __builtin_amdgcn_readfirstlane(s_drawn);

    if (tid < DS) {
        const int c = tid;
        float A = 1.f, Bk = 0.f, Bv = 0.f;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            const float aw = s_agg[w][0][c];
            Bk = fmaf(aw, Bk, s_agg[w][1][c]);
            Bv = fmaf(aw, Bv, s_agg[w][2][c]);
            A *= aw;
        }
        float Sk, Sv;
        if (j == 0) {
            Sk = state_k[bh * D + ch0 + c];
            Sv = state_v[bh * D + ch0 + c];
        } else {
            const uint64_t *p = rec + (((long)unit * rec_chunks + (j - 1)) * 2) * DS + c;
            uint64_t w0 = early0, w1 = early1;
            int spins = 0;
            if constexpr (!EARLY) {
                w0 = load_u64_agent(p);
                w1 = load_u64_agent(p + DS);
            }
            bool ok = ((uint32_t)(w0 >> 32) == tag) && ((uint32_t)(w1 >> 32) == tag);
            while (!ok) {
                if (++spins > spin_limit) break;
                __builtin_amdgcn_s_sleep(2);
                w0 = load_u64_agent(p);
                w1 = load_u64_agent(p + DS);
                ok = ((uint32_t)(w0 >> 32) == tag) && ((uint32_t)(w1 >> 32) == tag);
            }
            if (!ok) atomicExch(&ctrl[kCtrlAsyncErr], 1u);  // give up; outputs undefined
            Sk = __uint_as_float((uint32_t)w0);
            Sv = __uint_as_float((uint32_t)w1);
        }
        const float Ok = fmaf(A, Sk, Bk);
        const float Ov = fmaf(A, Sv, Bv);
        if (j == n_chunks - 1) {
            state_k[bh * D + ch0 + c] = Ok;
            state_v[bh * D + ch0 + c] = Ov;
        } else {
            uint64_t *p = rec + (((long)unit * rec_chunks + j) * 2) * DS + c;
            store_u64_agent(p, ((uint64_t)tag << 32) | __float_as_uint(Ok));
            store_u64_agent(p + DS, ((uint64_t)tag << 32) | __float_as_uint(Ov));
        }
        float ck = Sk, cv = Sv;
#pragma unroll
        for (int w = 0; w < NW; ++w) {
            s_carry[w][0][c] = ck;
            s_carry[w][1][c] = cv;
            const float aw = s_agg[w][0][c];
            ck = fmaf(aw, ck, s_agg[w][1][c]);
            cv = fmaf(aw, cv, s_agg[w][2][c]);
        }
    }
    // The next chunk's loads go out here, behind the chain step: a wave's loads return in order, so issued any earlier
    // they would hold up the chain waves' polls of the predecessor's record (the other waves come here at once).  Before them goes
    // the draw of the ticket after it (AHEAD), which is thus there when those loads are.
    if constexpr (PIPE) {
        if (nt < total) {
            if (AHEAD && tid == kTicketThread) drawn = draw();
            load_chunk(nt, nr);
        }
    }
    __syncthreads();

    // replay from the incoming state
    float sk[8], sv[8];
    // Whole rows with two sets: a token's inputs as new values to the compiler, which would otherwise keep what the fold made of
    // them (1 - g, unpacked keys) in registers until the replay; one token behind the states of the one before, as all
    // of them unpacked at once do not fit the registers beside the next chunk's.  (Slabs keep them: worked out again they cost
    // a short run 0.4 us, 2 x 8 heads x 600 in float32 17.7 / 18.7.  Float32 slabs sit at 120 to 128 registers, two workgroups to a
    // CU; two more and pages of 32 tokens lose the second: 8 heads x 64K 284 / 310, 128 x 6000 393 / 444.)
    auto fresh_inputs = [&](int i) __attribute__((always_inline)) {
        uint32_t w[2 * KW + 8];
        __builtin_memcpy(w, &kr[i], sizeof(kr[i]));
        __builtin_memcpy(w + KW, &vr[i], sizeof(vr[i]));
        __builtin_memcpy(w + 2 * KW, &g0[i], 16);
        __builtin_memcpy(w + 2 * KW + 4, &g1[i], 16);
        if constexpr (FENCE) {
#pragma unroll
            for (int c = 0; c < 8; ++c) asm volatile("" : "+v"(sk[c]), "+v"(sv[c]));
        }
#pragma unroll
        for (int c = 0; c < 2 * KW + 8; ++c) asm volatile("" : "+v"(w[c]));
        __builtin_memcpy(&kr[i], w, sizeof(kr[i]));
        __builtin_memcpy(&vr[i], w + KW, sizeof(vr[i]));
        __builtin_memcpy(&g0[i], w + 2 * KW, 16);
        __builtin_memcpy(&g1[i], w + 2 * KW + 4, 16);
    };
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        sk[c] = fmaf(a[c], s_carry[wave][0][c0 + c], bk[c]);
        sv[c] = fmaf(a[c], s_carry[wave][1][c0 + c], bv[c]);
    }
    const long out_row0 = (long)bh * Tcap + t0;
    float plo[8], phi[8];  // META: bounds of the stored (rounded) keys of this lane's tokens
#pragma unroll
    for (int c = 0; c < 8; ++c) {
        plo[c] = INFINITY;
        phi[c] = -INFINITY;
    }
    if constexpr (LEAD) {
        if (tbase < 0) {  // stored rows of the run's first page: only their bounds are wanted
            const int page0 = (int)(t0 & (PAGE - 1));
#pragma unroll 1
            for (int i = (int)(tbase < -page0 ? -page0 - tbase : 0); i < NT && tbase + i < 0; ++i) {
                float xs[8];
                R::load(k_cache + (out_row0 + tbase + i) * D + ch0 + c0, xs);
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    plo[c] = fminf(plo[c], xs[c]);
                    phi[c] = fmaxf(phi[c], xs[c]);
                }
            }
        }
    }
    const int rows_out = PIPE ? (int)((T_new - (long)j * CHUNK < CHUNK) ? T_new - (long)j * CHUNK : CHUNK) : 0;
    const auto kd_out = rows_of(k_cache, out_row0 + (long)j * CHUNK, rows_out), vd_out = rows_of(v_cache, out_row0 + (long)j * CHUNK, rows_out);
    uint32_t el_out = lane_el;
    if constexpr (PIPE) asm volatile("" : "+v"(el_out));
    auto store_row = [&](const LdsSource &d, int i, const float (&x)[8]) __attribute__((always_inline)) {  // whole rows
        const uint32_t byte = el_out * (uint32_t)sizeof(ST) + i * D * (int)sizeof(ST);
        if constexpr (sizeof(ST) == 2) {
            __builtin_amdgcn_raw_buffer_store_b128(u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                                                         pack_bf16x2(x[6], x[7])}, d, byte, 0, kStream);
        } else {
#pragma unroll
            for (int c = 0; c < 8; c += 4)
                __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(x[c]), __float_as_uint(x[c + 1]), __float_as_uint(x[c + 2]),
                                                             __float_as_uint(x[c + 3])}, d, byte + 4 * c, 0, kStream);
        }
    };
#pragma unroll
    for (int i = 0; i < NT; ++i) {
        const long t = tbase + i;
        // (whole rows past the run: their states go nowhere, and the bounds below leave them out)
        if (PIPE || ((!LEAD || t >= 0) && t < T_new)) {
            if constexpr (PIPE) fresh_inputs(i);
            float kx[8], vx[8];
            R::unpack(kr[i], kx);
            R::unpack(vr[i], vx);
            const float gg[8] = {g0[i].x, g0[i].y, g0[i].z, g0[i].w, g1[i].x, g1[i].y, g1[i].z, g1[i].w};
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                const float om = 1.f - gg[c];
                sk[c] = fmaf(gg[c], sk[c], om * kx[c]);
                sv[c] = fmaf(gg[c], sv[c], om * vx[c]);
            }
            if constexpr (PIPE) {
                store_row(kd_out, i, sk);
                store_row(vd_out, i, sv);
            } else {
                const long off = (out_row0 + t) * D + ch0 + c0;
                R::store_nt(k_cache + off, sk);
                R::store_nt(v_cache + off, sv);
            }
            if constexpr (META) {
                float xs[8];  // the values just stored
                if constexpr (sizeof(ST) == 2) {
                    const uint32_t w[4] = {pack_bf16x2(sk[0], sk[1]), pack_bf16x2(sk[2], sk[3]), pack_bf16x2(sk[4], sk[5]),
                                           pack_bf16x2(sk[6], sk[7])};
#pragma unroll
                    for (int c = 0; c < 4; ++c) {
                        xs[2 * c] = __uint_as_float(w[c] << 16);
                        xs[2 * c + 1] = __uint_as_float(w[c] & 0xffff0000u);
                    }
                } else {
#pragma unroll
                    for (int c = 0; c < 8; ++c) xs[c] = sk[c];
                }
                const bool in = !PIPE || t < T_new;
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    plo[c] = fminf(plo[c], in ? xs[c] : INFINITY);
                    phi[c] = fmaxf(phi[c], in ? xs[c] : -INFINITY);
                }
            }
        }
    }
    if constexpr (META) {
        if constexpr (!PG_LDS) {
            // PAGE / NT row groups make a page: fold them, then the first two lanes groups of a page write it
            constexpr int RGP = PAGE / NT;
#pragma unroll
            for (int msk = LPR; msk < LPR * RGP; msk <<= 1)
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    plo[c] = fminf(plo[c], shfl_xor_f(plo[c], msk));
                    phi[c] = fmaxf(phi[c], shfl_xor_f(phi[c], msk));
                }
            if constexpr (PIPE) {
                // (a lane without a row of bounds to write aims past the descriptor's end)
                const long page0 = (t0 + (long)j * CHUNK) / PAGE;
                const LdsSource md = lds_source_sized(meta + ((long)bh * (Tcap / PAGE) + page0) * 2 * D,
                                                      (rows_out + PAGE - 1) / PAGE * 2 * D * (int)sizeof(ST));
                const int row = (wave * TW / PAGE + rg / RGP) * 2 + rg % RGP;
                const uint32_t byte = (rg % RGP < 2) ? (uint32_t)(row * D + c0) * (uint32_t)sizeof(ST) : 0x40000000u;
                float x[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) x[c] = (rg % RGP == 0) ? plo[c] : phi[c];
                if constexpr (sizeof(ST) == 2) {
                    __builtin_amdgcn_raw_buffer_store_b128(u32x4{pack_bf16x2(x[0], x[1]), pack_bf16x2(x[2], x[3]), pack_bf16x2(x[4], x[5]),
                                                                 pack_bf16x2(x[6], x[7])}, md, byte, 0, 0);
                } else {
#pragma unroll
                    for (int c = 0; c < 8; c += 4)
                        __builtin_amdgcn_raw_buffer_store_b128(u32x4{__float_as_uint(x[c]), __float_as_uint(x[c + 1]), __float_as_uint(x[c + 2]),
                                                                     __float_as_uint(x[c + 3])}, md, byte + 4 * c, 0, 0);
                }
            } else {
                const long tp = (long)j * CHUNK + (long)wave * TW + (long)(rg / RGP) * PAGE - lead;  // the page's first token
                if (tp < T_new && (!LEAD || tp + PAGE > 0) && rg % RGP < 2) {
                    const long page = (t0 + tp) / PAGE;
                    ST *mrow = meta + (((long)bh * (Tcap / PAGE) + page) * 2) * D + ch0 + c0;
                    if (rg % RGP == 0) R::store(mrow, plo);
                    else R::store(mrow + D, phi);
                }
            }
        } else {
            // a page spans WPP waves: each folds all its row groups, their bounds meet in LDS, and
            // wave w < NW / WPP writes page w of the chunk
            constexpr int WPP = PAGE / TW;
#pragma unroll
            for (int msk = LPR; msk < 64; msk <<= 1)
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    plo[c] = fminf(plo[c], shfl_xor_f(plo[c], msk));
                    phi[c] = fmaxf(phi[c], shfl_xor_f(phi[c], msk));
                }
            if (rg == 0) {
#pragma unroll
                for (int c = 0; c < 8; ++c) {
                    s_pg[wave][0][c0 + c] = plo[c];
                    s_pg[wave][1][c0 + c] = phi[c];
                }
            }
            __syncthreads();
            const long tp = (long)j * CHUNK + (long)wave * PAGE - lead;  // first token of page `wave` of this chunk
            if (wave < NW / WPP && rg < 2 && tp < T_new && (!LEAD || tp + PAGE > 0)) {
                float x[8];
#pragma unroll
                for (int c = 0; c < 8; ++c) x[c] = s_pg[wave * WPP][rg][c0 + c];
#pragma unroll
                for (int w2 = 1; w2 < WPP; ++w2)
#pragma unroll
                    for (int c = 0; c < 8; ++c) {
                        const float y = s_pg[wave * WPP + w2][rg][c0 + c];
                        x[c] = rg == 0 ? fminf(x[c], y) : fmaxf(x[c], y);
                    }
                const long page = (t0 + tp) / PAGE;
                R::store(meta + (((long)bh * (Tcap / PAGE) + page) * 2 + rg) * D + ch0 + c0, x);
            }
        }
    }

    return nt;
    };  // process_chunk

    ChunkRegs A, B;
    int tA = (int)blockIdx.x;  // one chunk per unit: the grid is the units, no tickets
    if (n_chunks > 1) tA = next_ticket();
    if (tA < total) {
        if constexpr (PIPE) {
            // two register sets in turn, each under its own name: a set that changed its name at the end of a turn would be
            // copied, and the copies would wait for its loads
            if (AHEAD && tid == kTicketThread) drawn = draw();
            load_chunk(tA, A);
            int next = total;
            if constexpr (!AHEAD) next = next_ticket();
            for (;;) {
                const int tB = process_chunk(tA, A, B, next);
                if (tB >= total) break;
                if constexpr (!AHEAD) next = next_ticket();
                tA = process_chunk(tB, B, A, next);
                if (tA >= total) break;
                if constexpr (!AHEAD) next = next_ticket();
            }
        } else {
            load_chunk(tA, A);
            for (;;) {
                (void)process_chunk(tA, A, B, total);
                if (n_chunks == 1) break;
                tA = next_ticket();
                if (tA >= total) break;
                load_chunk(tA, A);
            }
        }
    }

    if (n_chunks > 1 && tid == 0) {
        if (atomicAdd(&ctrl[kCtrlDone], 1u) == gridDim.x - 1u) {  // last workgroup out resets the counters
            atomicExch(&ctrl[kCtrlTicket], 0u);
            atomicExch(&ctrl[kCtrlDone], 0u);
        }
    }
}

// few tokens (the decode-time append)
template <typename ST>
__global__ __launch_bounds__(256) void rat_step_kernel(
    const ST *__restrict__ k, const ST *__restrict__ v, const float *__restrict__ g,
    float *__restrict__ state_k, float *__restrict__ state_v, ST *__restrict__ k_cache,
    ST *__restrict__ v_cache, ST *__restrict__ meta, int P, int BH, int D, long T_new, long t0, long Tcap,
    const uint32_t *__restrict__ pos_state, long T_max, int K_min_pages)
{
    const uint32_t e = blockIdx.x * blockDim.x + threadIdx.x;
    if (e >= (uint32_t)(BH * D)) return;
    append_element(e, k, v, g, state_k, state_v, k_cache, v_cache, meta, P, D, T_new, t0, Tcap, pos_state, T_max, K_min_pages);
}

template <typename ST, int D, int DS, int PAGE, bool LEAD, ScanTurn TURN>
static void launch_scan_form(const void *k, const void *v, const float *g, float *state_k,
                       float *state_v, void *k_cache, void *v_cache, int BH, long T_new, long t0,
                       long Tcap, uint32_t *ctrl, uint64_t *rec, uint32_t tag, int spin_limit,
                       void *meta, int lead, hipStream_t stream)
{
    constexpr int NT = sizeof(ST) == 2 ? 4 : 2;
    constexpr int NW = 8;
    constexpr int CHUNK = NW * (64 / (DS / 8)) * NT;
    const int n_chunks = (int)((T_new + lead + CHUNK - 1) / CHUNK);
    long grid = (long)BH * (D / DS) * n_chunks;
    if (n_chunks > 1) {
        // resident workgroups of this kernel: both factors at once, as several host threads may be the first here
        struct Resident {
            long cus, all;
        };
        static const Resident resident = [] {
            int dev = 0, per_cu = 0, cus = 0;
            (void)hipGetDevice(&dev);
            if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&per_cu, rat_scan_chunk_kernel<ST, D, DS, NT, NW, PAGE, LEAD, TURN>, NW * 64, 0) != hipSuccess || per_cu < 1) per_cu = 1;
            if (hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess || cus < 1) cus = 256;
            return Resident{cus, (long)per_cu * cus};
        }();
        // With 16 chains or fewer one workgroup per CU: a second one only slows the chains' links down (float32, which
        // fits two; two / one per CU: 4 heads x 64K of 128 channels 243 / 199 us, 8 heads x 64K of 64 channels 226 / 197,
        // 2 heads 194 / 171; 32 chains, 8 heads of 128 channels: 300 / 314)
        long want = knob_or(knobs().scan_grid, (int)((long)BH * (D / DS) <= 16 ? resident.cus : resident.all));
        if (want > resident.all) want = resident.all;  // the knob only narrows: every workgroup stays resident
        if (want < 1) want = 1;
        if (grid > want) grid = want;
    }
    rat_scan_chunk_kernel<ST, D, DS, NT, NW, PAGE, LEAD, TURN><<<dim3((unsigned)grid), dim3(NW * 64), 0, stream>>>(
        (const ST *)k, (const ST *)v, g, state_k, state_v, (ST *)k_cache, (ST *)v_cache, BH, T_new,
        t0, Tcap, n_chunks, ctrl, rec, tag, spin_limit, (ST *)meta, lead);
}

template <typename ST, int D, int DS, int PAGE_ARG>
static void launch_scan(const void *k, const void *v, const float *g, float *state_k, float *state_v, void *k_cache,
                        void *v_cache, int BH, long T_new, long t0, long Tcap, uint32_t *ctrl, uint64_t *rec, uint32_t tag,
                        int spin_limit, void *meta, hipStream_t stream)
{
    constexpr int CHUNK = 8 * (64 / (DS / 8)) * (sizeof(ST) == 2 ? 4 : 2);
    constexpr int PAGE = (PAGE_ARG <= CHUNK) ? PAGE_ARG : 0;  // larger pages never get here with the bounds asked for
    if constexpr (PAGE > 0 && DS < D) {
        if (t0 % CHUNK != 0) {
            launch_scan_form<ST, D, DS, PAGE, true, kOneAtATime>(k, v, g, state_k, state_v, k_cache, v_cache, BH, T_new, t0, Tcap, ctrl, rec,
                                                    tag, spin_limit, meta, (int)(t0 % CHUNK), stream);
            return;
        }
    }
#define RS_TURN(TT)                                                                                                                   \
    launch_scan_form<ST, D, DS, PAGE, false, TT>(k, v, g, state_k, state_v, k_cache, v_cache, BH, T_new, t0, Tcap, ctrl, rec, tag, \
                                                 spin_limit, meta, 0, stream)
    if constexpr (DS < D) {
        RS_TURN(kOneAtATime);
    } else {
        // Runs of one chunk have nothing to send ahead, and waves without rows then skip loads, replay and stores (kernel alone, 96 heads
        // x 31 tokens 7.1 / 5.8 us).  A ticket drawn a chunk ahead saves a round trip to memory a chunk, and ties a chunk to a
        // workgroup that has two others to do first, which the chunk's successors wait for: it pays from eight chunks a CU on,
        // with 128 channels only for 48 chains and more.  Drawn ahead / at the end, us (with page bounds from t0 = 0, bfloat16 but for the last):
        // 4 x 32 heads x 64K 2293 / 2382, x 16000 571 / 577, x 2500 109 / 110, 2 x 32 x 64K 1196 / 1210, 64 channels 4 x 32 x 32000 593 / 624,
        // x 4000 93 / 94; the other way 4 x 32 x 700 42.9 / 38.9, x 1500 72.0 / 70.7, 8 x 32 x 400 46.1 / 43.8, 64 x 1000 from an odd start
        // 35.7 / 33.1, 44 x 1637 42.9 / 38.6, 24 x 32000 316 / 292, 32 x 64K 678 / 657, float32 24 x 20000 245 / 233.
        const long n_chunks = (T_new + CHUNK - 1) / CHUNK;
        if (n_chunks == 1) RS_TURN(kOneAtATime);
        else if ((D == 128 && BH < 48) || BH * n_chunks < 2048) RS_TURN(kNextAtEnd);
        else RS_TURN(kNextAhead);
    }
#undef RS_TURN
}

int scan_chunk_tokens(int dtype, int D)
{
    const int NT = dtype == RS_BF16 ? 4 : 2;
    return 8 * (64 / (D / 8)) * NT;
}

// host entry used by the C ABI (arguments already validated)
bool scan_uses_step_kernel(long T_new) { return T_new <= 8; }

// 32-channel slabs (shorter chains, more of them, four or two times the workgroups) or whole rows?
// Measured at 128 channels in bfloat16 from an aligned start with page bounds (rows / slabs, us):
// 8 heads x 400 12.9 / 9.7, x 2500 27.2 / 14.9, x 16000 110 / 62; 16 x 16000 127 / 114; 32 x 400
// 13.9 / 10.7, x 2500 41.6 / 39.4, x 6000 78.6 / 86.5; 64 x 400 16.5 / 13.5, x 2500 65 / 74; 128 x 400
// 31.3 / 24.3, x 1000 55 / 61; 256 x 400 46 / 49, x 40 9.9 / 25.8 (a slab's chunk is 512 tokens: short
// runs on many heads leave it empty).  The slabs read 64-byte pieces of the rows, which costs
// bandwidth once the chip is full; in float32 the pieces are whole 128-byte lines and the slabs stay
// ahead: 128 heads x 700 66 / 64, x 6000 461 / 429; 64 channels 43 / 33 and 256 / 225.
static bool scan_uses_slabs(int dtype, int D, int BH, long T_new)
{
    const int forced = knobs().scan_slab;
    if (forced != kKnobUnset) return forced != 0;
    if (BH <= 16) return true;
    const long chunk = (long)scan_chunk_tokens(dtype, D) * (D / 32), slabs = (long)BH * (D / 32);
    if (T_new < chunk / 4 || slabs > 512) return false;
    if (dtype == RS_F32) return true;
    return (long)BH * T_new * D <= (D == 128 && slabs <= 128 ? 10500000 : 6600000);
}

// whether the chunk kernel leaves the Quest page bounds of the rows it stores (else the caller
// recomputes the touched pages afterwards).  The slab form also does it for a run that starts inside
// a chunk (`lead` tokens of it lie before the run).  That may take one chunk more, which a short run on many heads does not
// pay back (32 heads x 150 tokens from an odd start: 15.4 us against 12.6 with the second pass; 32 x
// 2500 42.3 / 48.8, 8 x 2500 15.5 / 19.3); has_records: the workspace through which chunks hand their
// state on is there (a run of one chunk's length may have come without).
bool scan_writes_meta(int dtype, int D, int P, int BH, long T_new, long t0, bool has_records)
{
    if (scan_uses_step_kernel(T_new)) return true;  // the step kernel keeps the touched page current
    if (knobs().scan_meta == 0) return false;
    // tokens of a chunk: bfloat16 128 at D = 128, 256 at D = 64 (float32: half); 32-channel slabs: D / 32 times that
    const bool slabs = scan_uses_slabs(dtype, D, BH, T_new);
    const long chunk = (long)scan_chunk_tokens(dtype, D) * (slabs ? D / 32 : 1);
    if (P < 16 || P > chunk || (P & (P - 1)) != 0) return false;
    if (t0 % chunk == 0) return true;
    if (!slabs) return false;
    if (t0 % chunk + T_new <= chunk) return true;
    return has_records && ((long)BH * (D / 32) <= 64 || T_new > chunk * 3 / 2);
}

void scan_dispatch(int dtype, int D, const void *k, const void *v, const float *g, float *state_k,
                   float *state_v, void *k_cache, void *v_cache, void *meta, int P, int BH, long T_new, long t0,
                   long Tcap, uint32_t *ctrl, uint64_t *rec, uint32_t tag, int spin_limit,
                   hipStream_t stream)
{
    if (scan_uses_step_kernel(T_new)) {
        const long n = (long)BH * D;
        const unsigned blocks = (unsigned)((n + 255) / 256);
        if (dtype == RS_BF16)
            rat_step_kernel<bf16><<<blocks, 256, 0, stream>>>((const bf16 *)k, (const bf16 *)v, g, state_k, state_v,
                                                             (bf16 *)k_cache, (bf16 *)v_cache, (bf16 *)meta, P, BH, D, T_new, t0, Tcap, nullptr, 0, 0);
        else
            rat_step_kernel<float><<<blocks, 256, 0, stream>>>((const float *)k, (const float *)v, g, state_k, state_v,
                                                              (float *)k_cache, (float *)v_cache, (float *)meta, P, BH, D, T_new, t0, Tcap, nullptr, 0, 0);
        return;
    }
    const bool slab = scan_uses_slabs(dtype, D, BH, T_new);
#define RS_SCAN(ST, DD, DSS, MM) launch_scan<ST, DD, DSS, MM>(k, v, g, state_k, state_v, k_cache, v_cache, BH, T_new, t0, Tcap, ctrl, rec, tag, spin_limit, meta, stream)
    const bool in_scan = meta && scan_writes_meta(dtype, D, P, BH, T_new, t0, rec != nullptr);
    // page sizes up to 512 tokens have their own instantiation where they tile the form's chunk
#define RS_SCAN_P(ST, DD, DSS)                           \
    do {                                                 \
        if (!in_scan) RS_SCAN(ST, DD, DSS, 0);           \
        else if (P == 16) RS_SCAN(ST, DD, DSS, 16);      \
        else if (P == 32) RS_SCAN(ST, DD, DSS, 32);      \
        else if (P == 64) RS_SCAN(ST, DD, DSS, 64);      \
        else if (P == 128) RS_SCAN(ST, DD, DSS, 128);    \
        else if (P == 256) RS_SCAN(ST, DD, DSS, 256);    \
        else RS_SCAN(ST, DD, DSS, 512);                  \
    } while (0)
    if (dtype == RS_BF16) {
        if (D == 128) {
            if (slab) RS_SCAN_P(bf16, 128, 32);
            else RS_SCAN_P(bf16, 128, 128);
        } else {
            if (slab) RS_SCAN_P(bf16, 64, 32);
            else RS_SCAN_P(bf16, 64, 64);
        }
    } else {
        if (D == 128) {
            if (slab) RS_SCAN_P(float, 128, 32);
            else RS_SCAN_P(float, 128, 128);
        } else {
            if (slab) RS_SCAN_P(float, 64, 32);
            else RS_SCAN_P(float, 64, 64);
        }
    }
#undef RS_SCAN_P
#undef RS_SCAN
}

// the decode-time append of one token at the position the workspace's state words hold
void step_at_state_dispatch(int dtype, int D, const void *k, const void *v, const float *g, float *state_k,
                            float *state_v, void *k_cache, void *v_cache, void *meta, int P, int BH, long Tcap,
                            const uint32_t *pos_state, long T_max, int K, hipStream_t stream)
{
    const long n = (long)BH * D;
    const unsigned blocks = (unsigned)((n + 255) / 256);
    if (dtype == RS_BF16)
        rat_step_kernel<bf16><<<blocks, 256, 0, stream>>>((const bf16 *)k, (const bf16 *)v, g, state_k, state_v,
                                                         (bf16 *)k_cache, (bf16 *)v_cache, (bf16 *)meta, P, BH, D, 1, 0, Tcap, pos_state, T_max, K);
    else
        rat_step_kernel<float><<<blocks, 256, 0, stream>>>((const float *)k, (const float *)v, g, state_k, state_v,
                                                          (float *)k_cache, (float *)v_cache, (float *)meta, P, BH, D, 1, 0, Tcap, pos_state, T_max, K);
}

}  // namespace rs
