// dK and dV as in attn_bwd_dkdv.h, with 16x16x32 MFMAs: the program of long launches (bwd_long_launch()).
//
// Work, ring, order of the rows and phases are those of attn_bwd_dkdv.h.  Here a wave's 64 keys are four 16-key blocks:
// their K stays in registers as MFMA B operand, their V sits in LDS for the whole kernel (D = 64: in registers too), and
// their dK, dV live in accumulation registers that only MFMAs touch.  A streamed operand fetched from LDS feeds four
// MFMAs (one per key block), the vector-ALU work is spread a little behind every MFMA, and reads are issued three or four
// slots ahead.
//
// What bounds it: the clock that the board's power leaves, and the instructions a lone wave issues beside its MFMAs.  131072
// rows, 4 heads, D = 128, everything included: with 32x32x16 a step takes 2590 cycles at 1.69 GHz, the matrix pipe busy 79 %
// of them, with 16x16x32 2890 at 1.95 GHz, busy 71 % (pipe time 2048): 12 % more cycles at a clock 15 % higher, 25.2 -> 24.3
// ms; 32768 rows 1.63 -> 1.54 ms, 16 x 4096 rows 441 -> 419 us.  D = 64 (V in registers included), 32768 rows: 1.96 -> 2.20
// GHz, busy 57 -> 54 %, 956 -> 887 us; at 2.2 of 2.4 GHz it is the instructions that are left.
// Left out one at a time in the 32x32x16 kernel: vector ALU -16 % of the time, LDS reads -10 %, tile loads -5 %, V reads
// alone -3 %; moving them about inside a slot changed nothing.
#pragma once
#include "attn_bwd_dkdv.h"

namespace sp {
namespace dkdv16 {

using namespace dkdv;

template <int D>
struct Lds {
    static constexpr int TILE_B = BMQ * D * 2;
    static constexpr bool kVRegs = D == 64;  // V operands resident in registers (at D = 128 there is no room for them)
    static constexpr int QS = 0, DOS = NBUF * TILE_B, VS = 2 * NBUF * TILE_B, VW_B = kVRegs ? 0 : KPW * D * 2;
    static constexpr int AUX = VS + kWaves * VW_B, AUX_SLOT = 1024, AUX_W = NBUF * AUX_SLOT;
    static constexpr int BYTES = AUX + kWaves * AUX_W;
};

// The work of workgroup `wg` of n_chunks * Hkv * B; smem holds Lds<D>::BYTES, 1 KB aligned.
template <int D, bool VARLEN, bool SPLIT>
__device__ __forceinline__ void run(const DkdvParams& p, uint32_t wg, char* smem) {
    constexpr int NS = D / 16;   // operand slots per phase: (16-row block, contraction step), resp. 16-wide blocks of the head dim
    constexpr int NK = D / 32;   // contraction steps over the head dim
    constexpr int KB = KPW / 16; // 16-key blocks of a wave
    constexpr int HALF_B = 16 * D * 2;  // 16 rows of a tile
    using L = Lds<D>;
    constexpr int TILE_B = L::TILE_B, QS = L::QS, DOS = L::DOS, VS = L::VS, VW_B = L::VW_B;
    constexpr int AUX = L::AUX, AUX_SLOT = L::AUX_SLOT, AUX_W = L::AUX_W;
    static_assert(DOS + (NBUF - 1) * TILE_B + HALF_B < 65536, "immediate LDS offsets must fit 16 bits");

    const int tid = threadIdx.x, lane = tid & 63, lo = lane & 15, g4 = 4 * (lane >> 4);
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // Earliest key tiles (most rows to visit) first, the chunks of a tile behind each other; KV heads and batch entries vary
    // fastest, so that everybody's longest key tiles are dispatched before anybody's short ones (one after the other, the
    // last one's longest tile started when the stage was two thirds done: 16 x 4096 rows 710 -> 510 us; 32768 rows of 8
    // heads, full attention, D = 64, whole backward 3944 -> 3246 us).
    const uint32_t n_heads = (uint32_t)p.Hkv * (uint32_t)p.B;
    const int chunk_id = (int)(wg / n_heads), head_id = (int)(wg % n_heads);
    int jt = chunk_id, split = 0;
    int tile_chunks = 1, first_chunk = 0;  // chunks of this tile, and of the tiles before it
    bool equal = false;
    if constexpr (SPLIT) {
        equal = p.chunks.len > 0;
        if (equal) {
            int count, upto;
            scan_chunks(p.n_ktiles, p.S, p.off, p.G, p.chunks.len, count, upto);
            jt = __builtin_popcountll(__builtin_amdgcn_ballot_w64(upto <= chunk_id));
            jt = jt < p.n_ktiles ? jt : p.n_ktiles - 1;
            tile_chunks = __builtin_amdgcn_readlane(count, jt);
            first_chunk = __builtin_amdgcn_readlane(upto, jt) - tile_chunks;
            split = chunk_id - first_chunk;
        } else {
            tile_chunks = p.chunks.nsplit;
            jt = chunk_id / tile_chunks;
            split = chunk_id % tile_chunks;
        }
    }
    if (VARLEN && p.order && !equal) {  // longest tile first; clamped so that a bad entry cannot become a wild address
        const int v = __builtin_amdgcn_readfirstlane(p.order[jt]);
        jt = v < 0 ? 0 : (v < p.n_ktiles ? v : p.n_ktiles - 1);
    }
    if (SPLIT && !equal) first_chunk = jt * tile_chunks;
    const int g = head_id % p.Hkv, b = head_id / p.Hkv;
    const int S = p.S, Skv = p.Skv;
    const __bf16* kb = p.k + ((size_t)b * Skv * p.Hkv + g) * D;
    const __bf16* vb = p.v + ((size_t)b * Skv * p.Hkv + g) * D;

    const int j0 = jt * BNK;
    const int wkey0 = j0 + KPW * wave;  // first key of this wave

    // resident B operands: K^T (and V^T) columns of this lane's keys
    bf16x8 kreg[KB][NK], vreg[L::kVRegs ? KB : 1][NK];
#pragma unroll
    for (int kb_ = 0; kb_ < KB; ++kb_) {
        const int key = wkey0 + 16 * kb_ + lo;
        const int key_c = key < Skv ? key : Skv - 1;
#pragma unroll
        for (int ks = 0; ks < NK; ++ks) {
            kreg[kb_][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(kb + p.kvmap.off(key_c) + 32 * ks + 2 * g4));
            if constexpr (L::kVRegs) vreg[kb_][ks] = as_bf16x8(*reinterpret_cast<const u32x4*>(vb + p.kvmap.off(key_c) + 32 * ks + 2 * g4));
        }
    }
    int wave_hi_min = S, wg_hi_max = S;
    int khi_l[KB] = {};  // packed documents: one past the last row that may see this lane's keys (their document's end)
    if (VARLEN) {
        wave_hi_min = __builtin_amdgcn_readfirstlane(p.row_hi[(wkey0 < S ? wkey0 : S - 1)]);
        wg_hi_max = __builtin_amdgcn_readfirstlane(p.row_hi[(j0 + BNK - 1 < S ? j0 + BNK - 1 : S - 1)]);
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int key = wkey0 + 16 * k + lo;
            khi_l[k] = p.row_hi[key < S ? key : S - 1];
        }
    }

    f32x4 dkacc[KB][NS], dvacc[KB][NS];
#pragma unroll
    for (int k = 0; k < KB; ++k)
#pragma unroll
        for (int db = 0; db < NS; ++db) dkacc[k][db] = dvacc[k][db] = f32x4{0.f, 0.f, 0.f, 0.f};

    // LDS addresses of this lane's operand reads; everything that changes per step is an immediate
    const uint32_t sm = lds_addr(smem);
    uint32_t rb[NK];  // row-major operand (Q, dO rows): row lo (+16 per row block), chunk 4*ks + g
    uint32_t vr[NK];  // the same chunk of this wave's V rows
#pragma unroll
    for (int ks = 0; ks < NK; ++ks) {
        rb[ks] = sm + tile16_off_b128<D>(lo, 4 * ks + (lane >> 4));
        vr[ks] = rb[ks] + VS + wave * VW_B;
    }
    uint32_t tb[NS];  // transposed operand (Q^T, dO^T): rows 4*g + (0..3) (+16), column 16*db + lo
#pragma unroll
    for (int db = 0; db < NS; ++db) tb[db] = sm + tile16_off_tr<D>(16 * db, lane);
    const uint32_t ab = sm + AUX + wave * AUX_W + 4 * g4;  // per-row scalars: rows 4*g .. +3 (+16 per row block)

    const int it_begin = (j0 > p.off ? j0 - p.off : 0) / BMQ;  // tile holding the first row that sees the first key
    const int it_end = (wg_hi_max + BMQ - 1) / BMQ;  // exclusive
    const int n_it = it_end - it_begin;
    // Steps are (head in group, row tile) pairs, heads ascending, rows descending inside a head.  The
    // key tile's step sequence is cut into tile_chunks contiguous chunks, one per workgroup; a chunk may be
    // empty (its workgroup then contributes zeros).
    const int total_all = n_it * p.G;
    const int per_split = (total_all + tile_chunks - 1) / tile_chunks;
    int s_begin = split * per_split < total_all ? split * per_split : total_all;
    const int s_end = s_begin + per_split < total_all ? s_begin + per_split : total_all;
    const int total = s_end - s_begin;
    if (total == 0) s_begin = 0;  // keeps the prologue's loads on valid addresses
    const int head_first = s_begin / n_it;             // first head (inside the group) of this chunk
    const int it_first = it_end - 1 - s_begin % n_it;  // and its first row tile

    // ---- global -> LDS loads of a step: per-row scalars (1), Q rows (PW), dO rows (PW) per wave ----
    using Dma = TileDma<D, BMQ, kWaves>;
    constexpr int PW = Dma::PER_WAVE;
    constexpr int GROUP = 1 + 2 * PW;
    static_assert(GROUP <= NS, "one load per slot of the S phase");
    const uint32_t stride_b = p.qmap.row_stride * 2;
    // byte offset, from the tile's first row, of the 16 bytes this lane fetches in its K-th load; rows past
    // `lim` (tile-relative) re-read row `lim` (they are never used unmasked)
    auto lane_off = [&](int K, int lim) __attribute__((always_inline)) {
        const int row = Dma::RPI * (wave + kWaves * K) + lane / Dma::CH;
        const uint32_t chunk_b = (uint32_t)(((lane % Dma::CH) ^ swz16<D>(row)) * 16);
        return (uint32_t)(row < lim ? row : lim) * stride_b + chunk_b;
    };
    uint32_t voff[PW];
#pragma unroll
    for (int K = 0; K < PW; ++K) voff[K] = lane_off(K, BMQ - 1);
    const uint32_t aux_lane_b = 16 * (lane & 15);  // 256 bytes per tile; lanes 16.. duplicate, their LDS bytes are padding
    const int it_tail = (S % BMQ != 0) ? (S - 1) / BMQ : -1;  // the tile that runs past the last row, if any

    // the step being loaded: scalar byte pointers to its tile in q, dO and the per-row scalars
    struct LoadCursor { const char* q; const char* dO; const char* aux; int it, left; };
    LoadCursor dc;
    // byte offsets of the current head (inside the batch entry) in q/dO and of the current tile's rows
    size_t q_head_b = ((size_t)b * S * p.Hq + (size_t)g * p.G + head_first) * D * 2;
    {
        dc.it = it_first;
        const size_t off = p.qmap.off(dc.it * BMQ) * 2;
        dc.q = reinterpret_cast<const char*>(p.q) + q_head_b + off;
        dc.dO = reinterpret_cast<const char*>(p.dO) + q_head_b + off;
        dc.aux = reinterpret_cast<const char*>(p.aux) + (((size_t)b * p.Hq + (size_t)g * p.G + head_first) * (p.S_pad / 32) + dc.it) * 256;
        dc.left = total - 1;
    }
    const size_t aux_jump_b = ((size_t)(p.S_pad / 32) + (size_t)(n_it - 1)) * 256;
    auto advance_load = [&]() __attribute__((always_inline)) {
        if (SP_LIKELY(dc.left > 0)) {  // past the last step the cursor stays (the padding steps re-read the last tile)
            --dc.left;
            if (SP_RARE(VARLEN, dc.it == it_begin)) {  // first tile of a head -> last tile of the next
                dc.it = it_end - 1; q_head_b += (size_t)D * 2; dc.aux += aux_jump_b;
            } else {
                dc.it -= 1; dc.aux -= 256;
            }
            const size_t off = q_head_b + p.qmap.off(dc.it * BMQ) * 2;
            dc.q = reinterpret_cast<const char*>(p.q) + off;
            dc.dO = reinterpret_cast<const char*>(p.dO) + off;
        }
    };
    auto issue_load = [&](auto KC, int buf) __attribute__((always_inline)) {
        constexpr int K = decltype(KC)::value;
        if constexpr (K == 0) {
            dma16(dc.aux + aux_lane_b, smem + AUX + wave * AUX_W + buf * AUX_SLOT);
        } else {
            constexpr int KK = (K - 1) % PW;
            uint32_t off = voff[KK];
            if (SP_RARE(VARLEN, dc.it == it_tail)) off = lane_off(KK, S - 1 - dc.it * BMQ);  // rare
            const char* src = K <= PW ? dc.q : dc.dO;
            char* dst = smem + (K <= PW ? QS : DOS) + buf * TILE_B + (wave + kWaves * KK) * 1024;
            dma16(src + off, dst);
        }
    };

    // ---- prologue: V (resident), a finite stand-in tile for the deferred dK of "step -1", steps 0 and 1 ----
    int cur_it = it_first;    // row tile of the step being computed
    int step_no = 0;          // its number (the step count is padded to a multiple of four: steps >= total are not real)
    // row tiles whose S' needs masking: those holding a row that does not see the wave's last key, and those
    // reaching the end of the first key's document (dense: the end of the sequence)
    const int last_hidden = wkey0 + KPW - 2 - p.off;  // last row that does not see all the wave's keys
    const int it_mask_lo = last_hidden >= 0 ? last_hidden / BMQ : -1;
    const int it_mask_hi = (wave_hi_min - 31 + BMQ - 1) / BMQ;
    // ... there, the keys (their lanes) that no row of the tiles end_it + 1 .. dead_it sees: kept from step to step until a tile
    // in which some key's document ends, or the next head's last tile
    uint64_t dead[KB] = {};
    int end_it = -1, dead_it = -1;
    {
        if constexpr (!L::kVRegs) {
            TileDma<D, BNK, kWaves, true> vdma;
            vdma.init(wave, lane, p.kvmap.row_stride);
            vdma.issue(vb + p.kvmap.off(j0), Skv - 1 - j0, reinterpret_cast<__bf16*>(smem + VS), wave);
        }
        static_for<1, PW + 1>([&](auto K) { issue_load(K, 3); });  // Q rows of step 0 again, as the stand-in
        static_for<0, GROUP>([&](auto K) { issue_load(K, 0); });
        advance_load();
        static_for<0, GROUP>([&](auto K) { issue_load(K, 1); });
        advance_load();
        vmem_wait<GROUP>();  // everything but the loads of step 1 has landed (this wave's share) ...
        __builtin_amdgcn_s_barrier();  // ... and everybody else's
    }

    f32x4 sacc[2][KB], pacc[2][KB];  // [16-row block][key block]
    u32x4 pp[KB], dsp[KB];  // bf16 A operands [key block]: P of the step, dS of the previous step
#pragma unroll
    for (int k = 0; k < KB; ++k) pp[k] = dsp[k] = u32x4{0, 0, 0, 0};

    // The operand slots of a body, x = 0 .. 4*NS-1 in the phases S | dK | dP | dV.  Reads of slot x are issued
    // ahead(x) slots early, possibly from the previous body (slots x >= 4*NS name slots of the next body).
    // Waits happen once per pair of slots, at the even one.  The dP phase takes both row blocks of a contraction step
    // behind each other: the V operands are read with the first and serve both.
    constexpr int P4 = 4 * NS;
    auto nreads = [](int x) constexpr {  // LDS reads of slot x (first slot of a row block: plus the per-row scalars)
        const int s = x % P4;
        if (s < NS) return s % NK == 0 ? 2 : 1;
        if (s >= 2 * NS && s < 3 * NS) return 1 + (s < 2 * NS + 2 ? 1 : 0) + (s % 2 == 0 && !L::kVRegs ? KB : 0);
        return 2;
    };
    auto ahead = [](int x) constexpr {
        const int s = x % P4;
        return (s >= 2 * NS && s < 3 * NS) ? 3 : 4;
    };
    constexpr int kMaxAhead = 4;
    // reads issued after those of slot s+1 by the time (even) slot s waits, which is before slot s issues
    // its own (none for the next body if `last`)
    auto young_reads = [=](int s, bool last) constexpr {
        int n = 0;
        for (int x = s + 2; x <= s + kMaxAhead; ++x)
            if (x - ahead(x) <= s - 1 && !(last && x >= P4)) n += nreads(x);
        return n;
    };

    // in-flight operands (asynchronous reads: see the rule in attn_common.h)
    u32x4 aq[NS], ad[NS], bv[NK][KB], sds[2], sdp[2];
    u32x2 bq0[NS], bq1[NS], bd0[NS], bd1[NS];

    // reads of slot s (0 .. 4*NS-1) of the body at ring position BUF, in KB parts (one behind each MFMA of the slot that
    // issues them)
    auto issue_reads = [&](auto BUFC, auto SC, auto PARTC) __attribute__((always_inline)) {
        constexpr int BUF = decltype(BUFC)::value, PBUF = (BUF + 3) % NBUF, s = decltype(SC)::value, part = decltype(PARTC)::value;
        if constexpr (s < NS) {
            if constexpr (part == 0) {
                if constexpr (s % NK == 0) sds[s / NK] = lds_async_b128<BUF * AUX_SLOT + 64 * (s / NK)>(ab);
                aq[s] = lds_async_b128<QS + BUF * TILE_B + (s / NK) * HALF_B>(rb[s % NK]);
            }
        } else if constexpr (s < 2 * NS) {
            constexpr int t = s - NS;
            if constexpr (part == 0) bq0[t] = lds_async_tr16<QS + PBUF * TILE_B>(tb[t]);
            if constexpr (part == 1) bq1[t] = lds_async_tr16<QS + PBUF * TILE_B + HALF_B>(tb[t]);
        } else if constexpr (s < 3 * NS) {
            constexpr int kk = s - 2 * NS, ks = kk / 2, r = kk % 2;
            if constexpr (part == 0) {
                if constexpr (kk < 2) sdp[r] = lds_async_b128<BUF * AUX_SLOT + 128 + 64 * r>(ab);
                ad[kk] = lds_async_b128<DOS + BUF * TILE_B + r * HALF_B>(rb[ks]);
            }
            if constexpr (r == 0 && !L::kVRegs) bv[ks][part] = lds_async_b128<part * HALF_B>(vr[ks]);
        } else {
            constexpr int t = s - 3 * NS;
            if constexpr (part == 0) bd0[t] = lds_async_tr16<DOS + BUF * TILE_B>(tb[t]);
            if constexpr (part == 1) bd1[t] = lds_async_tr16<DOS + BUF * TILE_B + HALF_B>(tb[t]);
        }
    };

    // One body = step u at ring position BUF: (BUF+3)%4 holds step u-1 (its dK is done here), (BUF+1)%4 step
    // u+1, (BUF+2)%4 receives step u+2.  FIRST: nothing was prefetched for this body (it follows the loop
    // back-edge, which asynchronous values must not cross); LAST: it prefetches nothing for the next body.
    // In the very first body the deferred dK multiplies zeros by the stand-in tile.
    auto body = [&](auto BUFC, auto FIRSTC, auto LASTC) __attribute__((always_inline)) {
        constexpr int BUF = decltype(BUFC)::value, DBUF = (BUF + 2) % NBUF;
        constexpr bool FIRST = decltype(FIRSTC)::value, LAST = decltype(LASTC)::value;
        using NextBuf = std::integral_constant<int, (BUF + 1) % NBUF>;
        // Where the vector-ALU work goes: behind the MFMAs of the dK, dP and dV phases, numbered 0 .. 3*G-1, evenly.  The
        // exponentials begin behind the second MFMA of the dK phase (two have then issued since the last write of S') and
        // end a slot before the dV phase; P is packed one place behind them (an operand is at least two instructions old
        // when an MFMA reads it).  Eight other spreads (fewer in the dP phase with its many reads, none behind the MFMAs
        // that a read follows) were the same or up to 1.5 % slower.
        constexpr int G = NS * KB, N_EXP = 8 * KB, N_PAIR = 4 * KB, kExpL = 2 * G - KB - 1;
        auto exps_done = [](int x) constexpr { return x < 1 ? 0 : x >= kExpL ? N_EXP : x * N_EXP / kExpL; };
        auto packs_done = [=](int x) constexpr { return exps_done(x - 1) / 2; };
        auto pairs_done = [](int x) constexpr { return x < 2 * G ? 0 : (x - 2 * G + 1) * N_PAIR / G; };
        // The step's elements in the order in which the S phase finishes them: element i = row block i / (4*KB), then
        // key block, then register.  P stays in the S' registers; arguments are computed one place ahead, so that no
        // exponential waits for its own product.
        float arg[N_EXP];
        auto exp_args = [&](auto XC) __attribute__((always_inline)) {
            constexpr int x = decltype(XC)::value;
            static_for<exps_done(x - 1), exps_done(x)>([&](auto I) {
                constexpr int i = decltype(I)::value;
                arg[i] = sacc[i / (4 * KB)][i / 4 % KB][i % 4] * p.scale_log2;
            });
        };
        auto valu_at = [&](auto XC) __attribute__((always_inline)) {
            constexpr int x = decltype(XC)::value;
            if constexpr (x < 2 * G) {
                static_for<packs_done(x - 1), packs_done(x)>([&](auto J) {
                    constexpr int i = 2 * decltype(J)::value, r = i / (4 * KB), k = i / 4 % KB, e = i % 4;
                    pp[k][2 * r + e / 2] = pack_bf16(sacc[r][k][e], sacc[r][k][e + 1]);
                });
                static_for<exps_done(x - 1), exps_done(x)>([&](auto I) {
                    constexpr int i = decltype(I)::value;
                    sacc[i / (4 * KB)][i / 4 % KB][i % 4] = __builtin_amdgcn_exp2f(arg[i]);
                });
                if constexpr (x >= 1) exp_args(Int<x + 1>{});
            } else {
                static_for<pairs_done(x - 1), pairs_done(x)>([&](auto J) {  // dS, for the dK of the next body
                    constexpr int i = 2 * decltype(J)::value, r = i / (4 * KB), k = i / 4 % KB, e = i % 4;
                    uint32_t w = pack_bf16(sacc[r][k][e] * pacc[r][k][e], sacc[r][k][e + 1] * pacc[r][k][e + 1]);
                    asm volatile("" : "+v"(w));  // pins the arithmetic here: its only consumers are in the next body
                    dsp[k][2 * r + e / 2] = w;
                });
            }
        };

        if constexpr (FIRST) {
            static_for<0, kMaxAhead>([&](auto XC) {
                if constexpr (decltype(XC)::value - ahead(decltype(XC)::value) < 0) static_for<0, KB>([&](auto PART) { issue_reads(BUFC, XC, PART); });
            });
        }
        static_for<0, P4>([&](auto SC) {
            constexpr int s = decltype(SC)::value;
            constexpr bool even = s % 2 == 0;
            constexpr int W = even ? young_reads(s, LAST) : -1;  // reads allowed to stay in flight at the pair's wait
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (s == 2 * NS) {
                // Everybody is past the dK phase: nobody reads ring position (BUF+3)%4 any more.  This wave's
                // loads of step u+1 have landed (those of step u+2, issued in this body, may be in flight);
                // after the barrier so have everybody's.
                vmem_wait<GROUP>();
                __builtin_amdgcn_s_barrier();
            }
            // the reads this slot issues go out behind its MFMAs
            auto issue_slot = [&](auto PART) __attribute__((always_inline)) {
                static_for<1, kMaxAhead + 1>([&](auto AC) {
                    constexpr int x = s + decltype(AC)::value;
                    if constexpr (x - ahead(x) == s) {
                        if constexpr (x < P4) issue_reads(BUFC, Int<x>{}, PART);
                        else if constexpr (!LAST) issue_reads(NextBuf{}, Int<x - P4>{}, PART);
                    }
                });
                __builtin_amdgcn_sched_barrier(0);
            };
            // The slot's MFMAs, one per key block, each followed by its share of the other work: a lone wave that issues
            // two MFMAs in a row stands still while the first one runs.
            static_for<0, KB>([&](auto N) {
                constexpr int n = decltype(N)::value, w = n == 0 ? W : -1;
                if constexpr (s < NS) {
                    // ---- S(u); the loads of step u+2 ----
                    constexpr int r = s / NK, ks = s % NK;
                    if constexpr (n == 0 && ks == 0) lds_wait<w>(sds[r]);
                    if constexpr (ks == 0) mfma16_vc<n == 0 ? -1 : w>(sacc[r][n], aq[s], kreg[n][ks], __builtin_bit_cast(f32x4, sds[r]));
                    else mfma16_v<w>(sacc[r][n], aq[s], kreg[n][ks]);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_slot(N);
                    if constexpr (n == 1 && s < GROUP) issue_load(SC, DBUF);
                } else if constexpr (s < 2 * NS) {
                    // ---- dK(u-1), exponentials ----
                    // (key blocks forth in even slots, back in odd ones: each MFMA keeps an operand of the one before it)
                    constexpr int t = s - NS, k = even ? n : KB - 1 - n;
                    const u32x4 bqt = {bq0[t][0], bq0[t][1], bq1[t][0], bq1[t][1]};
                    mfma16_a<w>(dkacc[k][t], dsp[k], bqt);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_slot(N);
                    if constexpr (s == NS && n == 1) {  // two MFMAs have issued since the last write of S'
                        // Causal / document mask: hidden positions get S' = -inf, i.e. P = 0.  Register r of row
                        // block b is row q0 + 4*g + 16*b + r, so "hidden" is one compare of a compile-time number
                        // with a per-lane limit and one select.  A step none of whose rows sees any of
                        // the wave's keys (above the wave's diagonal while the rest of the workgroup is still on
                        // theirs, and padding) is overwritten outright: a wave is in that state for up to six of the
                        // eight steps of a tile's diagonal, and the whole workgroup waits for it at each barrier.
                        // With packed documents, a key whose document ends before the row tile is seen by none of
                        // its rows: all its S' take one select on a per-lane flag (a select, not arithmetic: S'
                        // of such a pair may be anything, a NaN included); upper limits are compared element by
                        // element only on the row tile in which some key's document (dense: the sequence) ends.
                        if (SP_RARE(VARLEN, cur_it <= it_mask_lo || step_no >= total)) {
                            const int q0 = cur_it * BMQ;
                            if (step_no >= total || q0 + BMQ - 1 + p.off < wkey0) {
                                asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                                for (int k = 0; k < KB; ++k)
#pragma unroll
                                    for (int i = 0; i < 8; ++i) sacc[i / 4][k][i % 4] = -__builtin_inff();
                            } else {
                                asm volatile("" ::: "memory");  // keeps this a branch (not selects executed on every step)
#pragma unroll
                                for (int k = 0; k < KB; ++k) {
                                    const int key = wkey0 + 16 * k + (int)(__lane_id() & 15);
                                    const int lim = key - p.off - q0 - 4 * (int)(__lane_id() >> 4);  // first row that sees the key
#pragma unroll
                                    for (int i = 0; i < 8; ++i) sacc[i / 4][k][i % 4] = 16 * (i / 4) + i % 4 >= lim ? sacc[i / 4][k][i % 4] : -__builtin_inff();
                                }
                            }
                        }
                        if (SP_RARE(VARLEN, cur_it >= it_mask_hi)) {  // rows at or past the end of the first key's document or of the sequence
                            const int q0 = cur_it * BMQ;
                            bool inside = !VARLEN;
                            if (VARLEN && (cur_it <= end_it || cur_it > dead_it)) {
                                dead_it = cur_it;
                                bool ends = false;
#pragma unroll
                                for (int k = 0; k < KB; ++k) ends = ends || (khi_l[k] > q0 && khi_l[k] < q0 + BMQ);
                                inside = __builtin_amdgcn_ballot_w64(ends) != 0;
                                // keys ascend, and so do their documents' ends: the next one, going down, is that of the last hidden key
                                end_it = inside ? cur_it : -1;
#pragma unroll
                                for (int k = 0; k < KB; ++k) {
                                    dead[k] = inside ? 0 : __builtin_amdgcn_ballot_w64(khi_l[k] <= q0);
                                    if (dead[k] != 0) end_it = (__builtin_amdgcn_readlane(khi_l[k], 63 - __builtin_clzll(dead[k])) - 1) / BMQ;
                                }
                            }
                            if (inside) {
                                asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                                for (int k = 0; k < KB; ++k) {
                                    const int lim = (VARLEN ? khi_l[k] : S) - q0 - 4 * (int)(__lane_id() >> 4);
#pragma unroll
                                    for (int i = 0; i < 8; ++i) sacc[i / 4][k][i % 4] = 16 * (i / 4) + i % 4 < lim ? sacc[i / 4][k][i % 4] : -__builtin_inff();
                                }
                            } else {
                                uint64_t any = 0;
#pragma unroll
                                for (int k = 0; k < KB; ++k) any |= dead[k];
                                if (any != 0) {
                                    asm volatile("" ::: "memory");  // keeps this a branch
#pragma unroll
                                    for (int k = 0; k < KB; ++k) hide_lanes(sacc[0][k], sacc[1][k], dead[k]);
                                }
                            }
                        }
                        exp_args(Int<1>{});
                    }
                    valu_at(Int<t * KB + n>{});
                } else if constexpr (s < 3 * NS) {
                    // ---- dP(u), exponentials ----
                    constexpr int kk = s - 2 * NS, ks = kk / 2, r = kk % 2;
                    const u32x4 bvk = [&]() { if constexpr (L::kVRegs) return as_u32x4(vreg[n][ks]); else return bv[ks][n]; }();
                    if constexpr (n == 0 && kk == 0) lds_wait<w>(sdp[0]);
                    if constexpr (ks == 0) mfma16_vc<(kk == 0 ? -1 : w)>(pacc[r][n], ad[kk], bvk, __builtin_bit_cast(f32x4, sdp[r]));
                    else mfma16_v<w>(pacc[r][n], ad[kk], bvk);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_slot(N);
                    valu_at(Int<G + kk * KB + n>{});
                } else {
                    // ---- dV(u), dS products ----
                    constexpr int t = s - 3 * NS, k = even ? n : KB - 1 - n;
                    const u32x4 bdo = {bd0[t][0], bd0[t][1], bd1[t][0], bd1[t][1]};
                    mfma16_a<w>(dvacc[k][t], pp[k], bdo);
                    __builtin_amdgcn_sched_barrier(0);
                    issue_slot(N);
                    valu_at(Int<2 * G + t * KB + n>{});
                }
                __builtin_amdgcn_sched_barrier(0);
            });
        });
        __builtin_amdgcn_sched_barrier(0);
        ++step_no;
        if (step_no < total) cur_it = (cur_it == it_begin) ? it_end - 1 : cur_it - 1;
        advance_load();
    };

    // Four steps per iteration, one per ring position; the step count is rounded up to a multiple of four
    // with steps whose P is all zero (they re-read the last tile).
    for (int u = 0; u < total; u += NBUF) {
        body(std::integral_constant<int, 0>{}, std::true_type{}, std::false_type{});
        body(std::integral_constant<int, 1>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 2>{}, std::false_type{}, std::false_type{});
        body(std::integral_constant<int, 3>{}, std::false_type{}, std::true_type{});
    }

    // ---- the deferred dK of the last step ----
    {
        static_for<0, NS>([&](auto TC) {
            constexpr int t = decltype(TC)::value;
            u32x2 h0 = lds_async_tr16<QS + (NBUF - 1) * TILE_B>(tb[t]);
            u32x2 h1 = lds_async_tr16<QS + (NBUF - 1) * TILE_B + HALF_B>(tb[t]);
            lds_wait<0>(h0, h1);
            const u32x4 bqt = {h0[0], h0[1], h1[0], h1[1]};
#pragma unroll
            for (int k = 0; k < KB; ++k) dkacc[k][t] = mfma16(as_bf16x8(dsp[k]), as_bf16x8(bqt), dkacc[k][t]);
        });
    }
    wait_vmem();  // no direct-to-LDS load may outlive the workgroup's LDS allocation

    // ---- write dK and dV: accumulator rows = keys, column = d ----
    if constexpr (SPLIT) {
        // fp32 partial sums of this chunk (dK unscaled); the reduction kernel adds the chunks in a fixed order.  A
        // lane holds four consecutive keys of one column in four registers, and the sums are laid out like that, so a
        // store is 16 bytes per lane and 256 contiguous bytes per 16 lanes: 64 stores per wave where key-major sums
        // took 256 of 4 bytes per lane (5.5 us per workgroup).
        const int keys = Skv - j0 < BNK ? Skv - j0 : BNK;
        float* pk = p.part + part_offset((int64_t)b * p.Hkv + g, p.chunks.nsplit, Skv, first_chunk, split, keys, D);
        float* pv = pk + (size_t)p.B * p.Hkv * p.chunks.nsplit * Skv * D;
#pragma unroll
        for (int k = 0; k < KB; ++k) {
            const int k0 = wkey0 - j0 + 16 * k + g4;  // first of the lane's four keys, in the tile
            if (k0 + 4 <= keys) {
#pragma unroll
                for (int db = 0; db < NS; ++db) {
                    const size_t at = (size_t)k0 * D + 4 * (16 * db + lo);
                    *reinterpret_cast<f32x4*>(pk + at) = dkacc[k][db];
                    *reinterpret_cast<f32x4*>(pv + at) = dvacc[k][db];
                }
            } else if (k0 < keys) {  // the last one to three keys
#pragma unroll
                for (int db = 0; db < NS; ++db)
#pragma unroll
                    for (int e = 0; e < 3; ++e)
                        if (k0 + e < keys) {
                            const size_t at = (size_t)k0 * D + (size_t)(keys - k0) * (16 * db + lo) + e;
                            pk[at] = dkacc[k][db][e];
                            pv[at] = dvacc[k][db][e];
                        }
            }
        }
    } else {
#pragma unroll
        for (int k = 0; k < KB; ++k)
#pragma unroll
            for (int db = 0; db < NS; ++db)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int krow = wkey0 + 16 * k + g4 + e;
                    if (krow < Skv) {
                        const size_t off = ((size_t)b * Skv * p.Hkv + g) * D + p.kvmap.off(krow) + 16 * db + lo;
                        p.dk[off] = (__bf16)(dkacc[k][db][e] * p.scale);
                        p.dv[off] = (__bf16)dvacc[k][db][e];
                    }
                }
    }
}

}  // namespace dkdv16
}  // namespace sp
