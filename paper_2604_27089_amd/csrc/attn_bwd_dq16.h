// dQ as in attn_bwd_dq.h, with 16x16x32 MFMAs: the program of long launches (bwd_long_launch()).
//
// Work, rings and deferral are those of attn_bwd_dq.h.  Here a wave's rows are blocks of 16 (RB of them): every operand
// fetched from LDS feeds 2*NQ MFMAs, one per row block, the vector-ALU work is spread a little behind every MFMA, and
// reads are issued sixteen MFMAs ahead.  The phases of a body:
//   S(u) + the loads of step u+6 | dP(u) + exponentials | dQ(u-1) + the rest of them, dS products
//
// What bounds it: the clock that the board's power leaves, then issue.  131072 rows, 4 heads, D = 128, everything included:
// with 32x32x16 a step takes 1780 cycles at 1.60 GHz, the matrix pipe busy 86 % of them, with 16x16x32 1910 at 1.86 GHz,
// busy 80 % (pipe time 1536): 18.3 -> 16.9 ms; 32768 rows 1.17 -> 1.09 ms, 16 x 4096 rows 333 -> 312 us; D = 64, 32768 rows,
// 1.85 -> 2.11 GHz, busy 63 -> 58 %, 678 -> 652 us.  Two MFMAs back to back with the other work behind each pair, instead of
// some behind every one, took 16 % more cycles; branches laid out so that the usual path takes no jump gave 1 %, the load
// cursor's update outside the S phase cost 3 %.
#pragma once
#include "attn_bwd_dq.h"

namespace sp {
namespace dq16 {

using namespace dq;

// The work of workgroup `wg` of n_ranks * Hq * B; smem holds Lds<D>::BYTES, 1 KB aligned.
template <int D, bool VARLEN, int NQ>
__device__ __forceinline__ void run(const DqParams& p, uint32_t wg, char* smem) {
    constexpr int RPW = kRowsPerWave<NQ>, BM = kRows<NQ>;
    constexpr int NS = D / 16;   // operand slots per phase: (16-key block, contraction step), resp. 16-wide blocks of the head dim
    constexpr int NK = D / 32;   // contraction steps over the head dim
    constexpr int RB = 2 * NQ;   // 16-row blocks of a wave
    constexpr int TILE_B = Lds<D>::TILE_B, KS = Lds<D>::KS, VS = Lds<D>::VS;
    constexpr int HALF_B = 16 * D * 2;  // 16 rows of a tile
    static_assert(KS + (NBUF - 1) * TILE_B + HALF_B < 65536, "immediate LDS offsets must fit 16 bits");

    const int tid = threadIdx.x, lane = tid & 63, lo = lane & 15, g4 = 4 * (lane >> 4);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // heads vary fastest (they share K/V tiles), then batch entries; query tiles from the last (longest) to the first
    const uint32_t n_heads = (uint32_t)p.Hq * (uint32_t)p.B;
    const int head_id = (int)(wg % n_heads), rank = (int)(wg / n_heads);
    const int h = head_id % p.Hq, b = head_id / p.Hq;
    int qt = p.n_qtiles - 1 - rank;
    if (VARLEN && p.order) {
        // longest 256-row tile first, its parts from the last; the value is clamped so that a bad entry cannot
        // become a wild address (a part past the last row has nothing to do)
        constexpr int SUB = kOrderTile / BM;
        const int v = __builtin_amdgcn_readfirstlane(p.order[rank / SUB]) * SUB + (SUB - 1 - rank % SUB);
        if (SUB > 1 && v >= p.n_qtiles) return;
        qt = v < 0 ? 0 : (v < p.n_qtiles ? v : p.n_qtiles - 1);
    }
    const int g = h / p.G;
    const int S = p.S, Skv = p.Skv;
    const __bf16* qb_ = p.q + ((size_t)b * S * p.Hq + h) * D;
    const __bf16* dob = p.dO + ((size_t)b * S * p.Hq + h) * D;

    const int i0 = qt * BM;
    const int wrow0 = i0 + RPW * wave;  // first row of this wave

    // resident B operands (Q^T, dO^T columns of this lane's rows) and accumulator seeds
    bf16x8 qreg[RB][NK], doreg[RB][NK];
    f32x4 seed_s[RB], seed_p[RB];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb) {
        const int row = wrow0 + 16 * rb + lo;
        const int rc = row < S ? row : S - 1;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            qreg[rb][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(qb_ + p.qmap.off(rc) + 32 * ks + 2 * g4));
            doreg[rb][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(dob + p.qmap.off(rc) + 32 * ks + 2 * g4));
        }
        const float ls = -p.lse[((size_t)b * p.Hq + h) * S + rc] / p.scale;
        const float dl = -p.delta[((size_t)b * p.Hq + h) * S + rc];
        seed_s[rb] = f32x4{ls, ls, ls, ls};
        seed_p[rb] = f32x4{dl, dl, dl, dl};
    }
    int wave_lo_max = 0, wg_lo_min = 0;
    int rlo_l[RB] = {};  // packed documents: the first key this lane's rows may see (their document's start)
    if (VARLEN) {
        wave_lo_max = __builtin_amdgcn_readfirstlane(p.row_lo[(wrow0 + RPW - 1 < S ? wrow0 + RPW - 1 : S - 1)]);
        wg_lo_min = __builtin_amdgcn_readfirstlane(p.row_lo[i0]);
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) {
            const int row = wrow0 + 16 * rb + lo;
            rlo_l[rb] = p.row_lo[row < S ? row : S - 1];
        }
    }

    f32x4 dqacc[RB][NS];
#pragma unroll
    for (int rb = 0; rb < RB; ++rb)
#pragma unroll
        for (int db = 0; db < NS; ++db) dqacc[rb][db] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS addresses of this lane's operand reads; everything that changes per step is an immediate
    const uint32_t sm = lds_addr(smem);
    uint32_t rk[NK], rv[NK];  // row-major operand (K, V rows): row lo (+16 per 16-key block), chunk 4*ks + g
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        rk[ks] = sm + tile16_off_b128<D>(lo, 4 * ks + (lane >> 4));
        rv[ks] = rk[ks] + VS;
    }
    uint32_t tb[NS];  // K^T operand: rows 4*g + (0..3) (+16), column 16*db + lo
#pragma unroll
    for (int db = 0; db < NS; ++db) tb[db] = sm + tile16_off_tr<D>(16 * db, lane);

    // the last key a row may see: i + off, at most the last key there is
    auto last_key = [&](int row) __attribute__((always_inline)) { return row + p.off < Skv - 1 ? row + p.off : Skv - 1; };
    const int jt_begin = VARLEN ? wg_lo_min / BN : 0;
    const int last_row = (i0 + BM - 1 < S ? i0 + BM - 1 : S - 1);
    const int jt_end = last_key(last_row) / BN + 1;  // exclusive
    const int total = jt_end - jt_begin;   // steps = key tiles, ascending

    // ---- global -> LDS loads of a step: K rows (PW), V rows (PW) per wave ----
    using Dma = TileDma<D, BN, kWaves>;
    constexpr int PW = Dma::PER_WAVE;
    constexpr int GROUP = 2 * PW;
    static_assert(GROUP < NS, "one load per slot of the S phase, and the cursor moves on in the slot behind them");
    const uint32_t stride_b = p.kvmap.row_stride * 2;
    // byte offset, from the tile's first row, of the 16 bytes this lane fetches in its K-th load; rows past
    // `lim` (tile-relative) re-read row `lim` (they are never used unmasked)
    auto lane_off = [&](int K, int lim) __attribute__((always_inline)) {
        const int row = Dma::RPI * (wave + kWaves * K) + lane / Dma::CH;
        const uint32_t chunk_b = (uint32_t)(((lane % Dma::CH) ^ swz16<D>(row)) * 16);
        return (uint32_t)(row < lim ? row : lim) * stride_b + chunk_b;
    };
    uint32_t voff[PW];  // offsets of the tile the load cursor is on
#pragma unroll
    for (int K = 0; K < PW; ++K) voff[K] = lane_off(K, BN - 1);
    const int jt_tail = (Skv % BN != 0) ? (Skv - 1) / BN : -1;  // the tile that runs past the last row, if any
    const int tiles_per_chunk_mask = (int)(p.kvmap.mask / BN);  // tiles per peer chunk - 1 (chunks are powers of two)

    // the step being loaded: scalar byte pointers to its tile in k and v
    struct LoadCursor { const char* k; const char* v; int jt, left; };
    LoadCursor dc;
    const size_t head0 = ((size_t)b * Skv * p.Hkv + g) * D * 2;
    const char* const k_head = reinterpret_cast<const char*>(p.k) + head0;
    const char* const v_head = reinterpret_cast<const char*>(p.v) + head0;
    const size_t tile_step_b = (size_t)BN * stride_b;
    // The tail tile is the last one the cursor can reach, and the cursor stays on it: its clamped lane offsets
    // replace the regular ones for good.
    auto enter_tile = [&]() __attribute__((always_inline)) {
        if (SP_RARE(VARLEN, dc.jt == jt_tail)) {  // rare
#pragma unroll
            for (int K = 0; K < PW; ++K) voff[K] = lane_off(K, Skv - 1 - dc.jt * BN);
        }
    };
    {
        dc.jt = jt_begin;
        const size_t off = p.kvmap.off(dc.jt * BN) * 2;
        dc.k = k_head + off;
        dc.v = v_head + off;
        dc.left = total - 1;
        enter_tile();
    }
    auto advance_load = [&]() __attribute__((always_inline)) {
        if (SP_LIKELY(dc.left > 0)) {  // past the last step the cursor stays (the padding steps re-read the last tile)
            --dc.left; dc.jt += 1;
            dc.k += tile_step_b; dc.v += tile_step_b;
            if (SP_RARE(VARLEN, (dc.jt & tiles_per_chunk_mask) == 0)) {  // rare: the first tile of the next peer's chunk
                const size_t off = p.kvmap.off(dc.jt * BN) * 2;
                dc.k = k_head + off; dc.v = v_head + off;
            }
            enter_tile();
        }
    };
    auto issue_load = [&](auto KC, int buf) __attribute__((always_inline)) {
        constexpr int K = decltype(KC)::value, KK = K % PW;
        const char* src = K < PW ? dc.k : dc.v;
        char* dst = smem + (K < PW ? KS : VS) + buf * TILE_B + (wave + kWaves * KK) * 1024;
        dma16(src + voff[KK], dst);
    };

    // ---- prologue: the first LEAD steps' tiles, and a finite stand-in for the deferred dQ of "step -1" ----
    int cur_jt = jt_begin;  // key tile of the step being computed
    int step_no = 0;        // its number (the step count is padded to a multiple of NBUF: steps >= total are not real)
    // steps whose S' needs masking: from the first whose keys reach past the last key the wave's first row
    // may see (and every padding step), and, for packed documents, those before the wave's last row's
    // document starts; from dead_from on the wave sees no key at all
    const int mask_from = (last_key(wrow0) / BN - jt_begin) < total ? (last_key(wrow0) / BN - jt_begin) : total;
    const int dead_from = (last_key(wrow0 + RPW - 1) / BN + 1 - jt_begin) < total ? (last_key(wrow0 + RPW - 1) / BN + 1 - jt_begin) : total;
    const int mask_until = VARLEN ? (wave_lo_max + BN - 1) / BN - jt_begin : 0;
    // ... there, the rows (their lanes) that see nothing of any step before start_step, in which the next row's document
    // starts.  Kept from step to step: four blocks' compares in each of them cost a wave with a boundary among its rows
    // more than the selects, and its workgroup waits for it (20000 rows in documents of 1024, 4 heads, D = 64, backward
    // 198 us with the compares, 176 without).
    uint64_t dead[RB] = {};
    int start_step = 0;
    {
        static_for<0, PW>([&](auto K) { issue_load(K, NBUF - 1); });  // K rows of step 0 again, as the stand-in
        static_for<0, LEAD>([&](auto T) {
            static_for<0, GROUP>([&](auto K) { issue_load(K, decltype(T)::value); });
            advance_load();
        });
    }

    f32x4 sacc[2][RB], pacc[2][RB];  // [16-key block][row block]
    u32x4 dsp[2][RB];  // bf16 B operands [parity of the step][row block]
#pragma unroll
    for (int par = 0; par < 2; ++par)
#pragma unroll
        for (int rb = 0; rb < RB; ++rb) dsp[par][rb] = u32x4{0, 0, 0, 0};

    // The operand slots of a body, x = 0 .. 3*NS-1 in the phases S | dP | dQ.  Reads of slot x are issued
    // kAhead slots early (behind the first MFMA of the issuing slot), possibly from the previous body (slots
    // x >= 3*NS name slots of the next body).  Waits happen once per pair of slots, at the even one.
    constexpr int P3 = 3 * NS;
    constexpr int kAhead = NQ == 2 ? 4 : 8;  // sixteen MFMAs
    auto nreads = [](int x) constexpr { return (x % P3) < 2 * NS ? 1 : 2; };
    // reads issued after those of slot s+1 by the time (even) slot s waits, which is before slot s issues
    // its own (none for the next body if `last`)
    auto young_reads = [=](int s, bool last) constexpr {
        int n = 0;
        for (int x = s + 2; x <= s - 1 + kAhead; ++x)
            if (!(last && x >= P3)) n += nreads(x);
        return n;
    };

    // in-flight operands (asynchronous reads: see the rule in attn_common.h)
    u32x4 ak[NS], av[NS];
    u32x2 t0[NS], t1[NS];

    // reads of slot s (0 .. 3*NS-1) of the body at ring position BUF
    auto issue_reads = [&](auto BUFC, auto SC, auto PART) __attribute__((always_inline)) {
        constexpr int BUF = decltype(BUFC)::value, PBUF = (BUF + NBUF - 1) % NBUF, s = decltype(SC)::value;
        if constexpr (decltype(PART)::value == 1) {  // the second transposing read
            if constexpr (s >= 2 * NS) t1[s - 2 * NS] = lds_async_tr16<KS + PBUF * TILE_B + HALF_B>(tb[s - 2 * NS]);
        } else if constexpr (s < NS) {
            ak[s] = lds_async_b128<KS + BUF * TILE_B + (s / NK) * HALF_B>(rk[s % NK]);
        } else if constexpr (s < 2 * NS) {
            av[s - NS] = lds_async_b128<BUF * TILE_B + ((s - NS) / NK) * HALF_B>(rv[s % NK]);
        } else {
            t0[s - 2 * NS] = lds_async_tr16<KS + PBUF * TILE_B>(tb[s - 2 * NS]);
        }
    };

    // dS of pair j of a step (of its elements as numbered below), into the operands of parity PAR
    auto ds_pair = [&](auto PARC, auto JC) __attribute__((always_inline)) {
        constexpr int i = 2 * decltype(JC)::value, kb = i / (4 * RB), rb = i / 4 % RB, r = i % 4;
        uint32_t w = pack_bf16(sacc[kb][rb][r] * pacc[kb][rb][r], sacc[kb][rb][r + 1] * pacc[kb][rb][r + 1]);
        asm volatile("" : "+v"(w));  // pins the arithmetic here: its consumers are far behind
        dsp[decltype(PARC)::value][rb][2 * kb + r / 2] = w;
    };

    // One body = step u at ring position BUF: (BUF-1)%8 holds step u-1 (its dQ is done here), (BUF+6)%8
    // receives step u+6.  FIRST: nothing was prefetched for this body (it follows the loop back-edge, which
    // asynchronous values must not cross); LAST: it prefetches nothing for the next body.  In the very
    // first body the deferred dQ multiplies the stand-in tile by zeros.
    auto body = [&](auto BUFC, auto FIRSTC, auto LASTC) __attribute__((always_inline)) {
        constexpr int BUF = decltype(BUFC)::value, DBUF = (BUF + LEAD) % NBUF, PAR = BUF % 2;
        constexpr bool FIRST = decltype(FIRSTC)::value, LAST = decltype(LASTC)::value;
        using NextBuf = std::integral_constant<int, (BUF + 1) % NBUF>;
        // Where the vector-ALU work goes: behind the MFMAs of the dP and dQ phases, numbered 0 .. 2*G-1.
        constexpr int G = NS * RB, N_EXP = 16 * NQ, N_PAIR = 8 * NQ;
        constexpr int kExp0 = 1, kExpL = G + G / 2, kPair0 = G + G / 2, kPairL = G / 2;
        auto exps_done = [](int x) constexpr { return x < kExp0 ? 0 : x - kExp0 + 1 >= kExpL ? N_EXP : (x - kExp0 + 1) * N_EXP / kExpL; };
        auto pairs_done = [](int x) constexpr { return x < kPair0 ? 0 : x - kPair0 + 1 >= kPairL ? N_PAIR : (x - kPair0 + 1) * N_PAIR / kPairL; };

        // The step's elements in the order in which the S phase finishes them: element i = key block i / (4*RB), then
        // row block, then register.  P stays in the S' registers; arguments are computed one place ahead, so that no
        // exponential waits for its own product.
        float arg[N_EXP];
        auto exp_args = [&](auto XC) __attribute__((always_inline)) {
            constexpr int x = decltype(XC)::value;
            static_for<exps_done(x - 1), exps_done(x)>([&](auto I) {
                constexpr int i = decltype(I)::value;
                arg[i] = sacc[i / (4 * RB)][i / 4 % RB][i % 4] * p.scale_log2;
            });
        };
        auto valu_at = [&](auto XC) __attribute__((always_inline)) {
            constexpr int x = decltype(XC)::value;
            static_for<exps_done(x - 1), exps_done(x)>([&](auto I) {
                constexpr int i = decltype(I)::value;
                sacc[i / (4 * RB)][i / 4 % RB][i % 4] = __builtin_amdgcn_exp2f(arg[i]);
            });
            if constexpr (x >= kExp0) exp_args(Int<x + 1>{});
            static_for<pairs_done(x - 1), pairs_done(x)>([&](auto J) { ds_pair(Int<PAR>{}, J); });
        };

        // Everybody is done with the previous body: nobody reads ring position (BUF+6)%8 = (BUF-2)%8 any
        // more.  This wave's loads of step u+1 have landed (those of the four steps after it may be in
        // flight); after the barrier so have everybody's.
        vmem_wait<(LEAD - 2) * GROUP>();
        __builtin_amdgcn_s_barrier();

        if constexpr (FIRST) static_for<0, kAhead>([&](auto XC) {
            issue_reads(BUFC, XC, Int<0>{});
            issue_reads(BUFC, XC, Int<1>{});
        });
        static_for<0, P3>([&](auto SC) {
            constexpr int s = decltype(SC)::value;
            constexpr bool even = s % 2 == 0;
            constexpr int W = even ? young_reads(s, LAST) : -1;  // reads allowed to stay in flight at the pair's wait
            __builtin_amdgcn_sched_barrier(0);
            // the reads this slot issues go out behind its first MFMA and (the second transposing one) its second
            auto issue_slot = [&](auto PART) __attribute__((always_inline)) {
                constexpr int x = s + kAhead;
                if constexpr (x < P3) issue_reads(BUFC, Int<x>{}, PART);
                else if constexpr (!LAST) issue_reads(NextBuf{}, Int<x - P3>{}, PART);
                __builtin_amdgcn_sched_barrier(0);
            };
            // The slot's MFMAs, one per row block, each followed by its share of the other work: a lone wave that issues
            // two MFMAs in a row stands still while the first one runs.
            static_for<0, RB>([&](auto N) {
                constexpr int n = decltype(N)::value, w = n == 0 ? W : -1;
                if constexpr (s < NS) {
                    // ---- S(u); the loads of step u+6 ----
                    constexpr int kb = s / NK, ks = s % NK;
                    if constexpr (ks == 0) mfma16_vc_ab<w>(sacc[kb][n], ak[s], qreg[n][ks], seed_s[n]);
                    else mfma16_v_ab<w>(sacc[kb][n], ak[s], qreg[n][ks]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (n < 2) issue_slot(N);
                    if constexpr (n == 1 && s == GROUP) advance_load();
                    if constexpr (n == 1 && s < GROUP) issue_load(SC, DBUF);
                } else if constexpr (s < 2 * NS) {
                    // ---- dP(u), two thirds of the exponentials ----
                    constexpr int kk = s - NS, kb = kk / NK, ks = kk % NK;
                    if constexpr (ks == 0) mfma16_vc_ab<w>(pacc[kb][n], av[kk], doreg[n][ks], seed_p[n]);
                    else mfma16_v_ab<w>(pacc[kb][n], av[kk], doreg[n][ks]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (n < 2) issue_slot(N);
                    if constexpr (kk == 0 && n == 1) {  // two MFMAs have issued since the last write of S'
                        // Causal / document mask: hidden positions get S' = -inf, i.e. P = 0.  Register r of key block kb
                        // is key j0 + 4*g + 16*kb + r, so "hidden" is one compare of a compile-time number with a per-lane
                        // limit and one select.  A step none of whose keys the wave
                        // sees (past its diagonal while the rest of the workgroup is still on theirs, and padding)
                        // is overwritten outright: a wave is in that state for up to six of the eight steps of a
                        // tile's diagonal, and every wave of the workgroup waits for it at each step's barrier
                        // (diagonal block of 256 rows: 14.3 us with bounds compared index by index on all eight
                        // steps, against 6.0 us for eight unmasked steps).
                        // With packed documents, a row whose document starts after the step's keys sees none of
                        // them: all its S' take one select on a per-lane flag (a select, not arithmetic: S' of
                        // such a pair may be anything, a NaN included); lower limits are compared element by element
                        // only on the step in which some row's document starts.
                        if (SP_RARE(VARLEN, step_no >= mask_from)) {
                            if (step_no >= dead_from) {
                                asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb)
#pragma unroll
                                    for (int r = 0; r < 8; ++r) sacc[r / 4][rb][r % 4] = -__builtin_inff();
                            } else {
                                asm volatile("" ::: "memory");  // keeps this a branch (not selects executed on every step)
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb) {
                                    const int row = wrow0 + 16 * rb + (int)(__lane_id() & 15);
                                    const int rhi = row + p.off < p.Skv - 1 ? row + p.off : p.Skv - 1;  // last key it may see
                                    const int lim = rhi - cur_jt * BN - 4 * (int)(__lane_id() >> 4);
#pragma unroll
                                    for (int r = 0; r < 8; ++r) sacc[r / 4][rb][r % 4] = 16 * (r / 4) + r % 4 <= lim ? sacc[r / 4][rb][r % 4] : -__builtin_inff();
                                }
                            }
                        }
                        if (VARLEN && step_no < mask_until) {  // some row's document starts at or after this step's keys
                            if (step_no >= start_step) {
                                const int j0 = cur_jt * BN;
                                bool starts = false;
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb) starts = starts || (rlo_l[rb] > j0 && rlo_l[rb] < j0 + BN);
                                if (__builtin_amdgcn_ballot_w64(starts) != 0) {
                                    asm volatile("" ::: "memory");  // keeps this a branch
                                    start_step = step_no + 1;
#pragma unroll
                                    for (int rb = 0; rb < RB; ++rb) dead[rb] = 0;
#pragma unroll
                                    for (int rb = 0; rb < RB; ++rb) {
                                        const int lim = rlo_l[rb] - j0 - 4 * (int)(__lane_id() >> 4);
#pragma unroll
                                        for (int r = 0; r < 8; ++r) sacc[r / 4][rb][r % 4] = 16 * (r / 4) + r % 4 >= lim ? sacc[r / 4][rb][r % 4] : -__builtin_inff();
                                    }
                                } else {
                                    // rows ascend, and so do their documents' starts: the next one is that of the first hidden row
                                    start_step = total;
#pragma unroll
                                    for (int rb = RB - 1; rb >= 0; --rb) {
                                        dead[rb] = __builtin_amdgcn_ballot_w64(rlo_l[rb] >= j0 + BN);
                                        if (dead[rb] != 0) start_step = __builtin_amdgcn_readlane(rlo_l[rb], __builtin_ctzll(dead[rb])) / BN - jt_begin;
                                    }
                                }
                            }
                            uint64_t any = 0;
#pragma unroll
                            for (int rb = 0; rb < RB; ++rb) any |= dead[rb];
                            if (any != 0) {
                                asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                                for (int rb = 0; rb < RB; ++rb) hide_lanes(sacc[0][rb], sacc[1][rb], dead[rb]);
                            }
                        }
                    }
                    if constexpr (kk * RB + n == kExp0) exp_args(Int<kExp0>{});
                    valu_at(Int<kk * RB + n>{});
                } else {
                    // ---- dQ(u-1); the last third of the exponentials, then the dS products of step u ----
                    // (row blocks forth in even slots, back in odd ones: each MFMA keeps an operand of the one before it)
                    constexpr int t = s - 2 * NS, rb = even ? n : RB - 1 - n;
                    const u32x4 kt = {t0[t][0], t0[t][1], t1[t][0], t1[t][1]};
                    mfma16_a<w>(dqacc[rb][t], kt, dsp[1 - PAR][rb]);
                    __builtin_amdgcn_sched_barrier(0);
                    if constexpr (n < 2) issue_slot(N);
                    valu_at(Int<G + t * RB + n>{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        __builtin_amdgcn_sched_barrier(0);
        ++step_no;
        if (step_no < total) cur_jt += 1;
    };

    // Eight steps per iteration, one per ring position; the step count is rounded up to a multiple of
    // eight with steps whose P is all zero (they re-read the last tile).
    for (int u = 0; u < total; u += NBUF) {
        body(std::integral_constant<int, 0>{}, std::true_type{}, std::false_type{});
        body(std::integral_constant<int, 1>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 2>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 3>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 4>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 5>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 6>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 7>{}, std::false_type{}, std::true_type{});
    }

    // ---- the deferred dQ of the last step (ring position 7, dS of parity 1) ----
    {
        static_for<0, NS>([&](auto TC) {
            constexpr int t = decltype(TC)::value;
            u32x2 h0 = lds_async_tr16<KS + (NBUF - 1) * TILE_B>(tb[t]);
            u32x2 h1 = lds_async_tr16<KS + (NBUF - 1) * TILE_B + HALF_B>(tb[t]);
            lds_wait<0>(h0, h1);
            const u32x4 kt = {h0[0], h0[1], h1[0], h1[1]};
#pragma unroll
            for (int rb = 0; rb < RB; ++rb) dqacc[rb][t] = mfma16(as_bf16x8(kt), as_bf16x8(dsp[1][rb]), dqacc[rb][t]);
        });
    }
    wait_vmem();  // no direct-to-LDS load may outlive the workgroup's LDS allocation, nor land in what is written next
    __syncthreads();

    // ---- write dQ (scaled), through LDS ----
    __bf16* const out = p.dq + ((size_t)b * S * p.Hq + h) * D;
#pragma unroll
    for (int qb = 0; qb < NQ; ++qb) {
        const int row0 = wrow0 + 32 * qb;
        if (row0 < S) store_rows16<D>(dqacc[2 * qb], dqacc[2 * qb + 1], p.scale, smem + wave * (32 * D * 2), S - row0, [&](int row) __attribute__((always_inline)) { return out + p.qmap.off(row0 + row); });
    }
}

}  // namespace dq16
}  // namespace sp
