// The kernel of the backward's two matrix stages, and its launcher.
//
// dK/dV (attn_bwd_dkdv.h) and dQ (attn_bwd_dq.h) read the same inputs and write different outputs, so one launch
// holds the workgroups of both.  Either stage alone ends with compute units idle (each unit holds one workgroup,
// and the longest walk of a stage is twice the mean or more), and a short problem fills the chip with neither.
// Whole backward, one launch against one per stage (with equal programs, 4 query heads, D = 128): 512 rows 71 -> 35
// us, 4096 rows 218 -> 124, 8192 398 -> 267, 16384 890 -> 753, 32768 2.80 -> 2.77 ms, 16 x 4096 rows 857 -> 815 us.
// Both programs keep a wave's whole register file, so sharing a kernel costs neither of them occupancy.
#pragma once
#include "attn_bwd_dkdv16.h"
#include "attn_bwd_dq16.h"

namespace {

using namespace sp;

struct MatrixParams {
    dkdv::DkdvParams kv;
    dq::DqParams q;
    uint32_t base;         // first workgroup of this launch
    // Order of dispatch: n_lead workgroups of one stage, then the remaining mix_kv and mix_q of the two in even
    // alternation, each stage longest first.
    uint32_t n_lead, mix_kv, mix_q;
    bool lead_is_q;
};

// LONG: the programs with 16x16x32 MFMAs (bwd_long_launch()).
template <int D, bool VARLEN, bool SPLIT, int NQ, bool LONG>
__global__ __launch_bounds__(dkdv::kThreads) void attn_bwd_matrix_kernel(MatrixParams p) {
    static_assert(dkdv::kThreads == dq::kThreads, "one block size");
    constexpr int kKv = LONG ? dkdv16::Lds<D>::BYTES : dkdv::Lds<D>::BYTES, kLds = kKv > dq::Lds<D>::BYTES ? kKv : dq::Lds<D>::BYTES;
    __shared__ __attribute__((aligned(1024))) char smem[kLds];
    const uint32_t i = p.base + blockIdx.x;
    bool is_q = p.lead_is_q;
    uint32_t wg = i;
    if (i >= p.n_lead) {
        const uint32_t r = i - p.n_lead;
        uint32_t q_before = 0;  // dQ workgroups among the first r of the alternation
        if (p.mix_kv == 0) { is_q = true; q_before = r; }
        else if (p.mix_q == 0) is_q = false;
        else {  // short launches only: the products fit 32 bits
            q_before = r * p.mix_q / (p.mix_kv + p.mix_q);
            is_q = (r + 1) * p.mix_q / (p.mix_kv + p.mix_q) > q_before;
        }
        wg = is_q ? q_before : r - q_before;
        if (is_q == p.lead_is_q) wg += p.n_lead;
    }
    if constexpr (LONG) {
        if (is_q) dq16::run<D, VARLEN, NQ>(p.q, wg, smem);
        else dkdv16::run<D, VARLEN, SPLIT>(p.kv, wg, smem);
    } else {
        if (is_q) dq::run<D, VARLEN, NQ>(p.q, wg, smem);
        else dkdv::run<D, VARLEN, SPLIT>(p.kv, wg, smem);
    }
}

// In which order the workgroups of the two stages go out (speed only: every order gives the same bits).  Each stage
// hands out its longest walks first; what they take is estimated with the costs of sp_common.h (at D = 64 both are a third
// shorter, and it is their ratio that counts).
//   Even walks beyond one round (even_walks()): the stage with the longer workgroups first, the other fills its last
// round.
//   Up to three rounds of the chip (768 workgroups; five with packed documents, whose work is uneven): the two are
// merged by expected length, i.e. the stage with the longer walks leads until its remaining ones are as long as the
// other's, and from there they alternate.  Measured against dK/dV first / dQ first, us: 64 x 512 rows 130 against 132 /
// 139, packed documents of 32768 rows at D = 64 (longest 12877) 448 against 572 / 506; where dQ's walks are the longer
// ones the merged order is as good as dQ first: 8192 rows of 5 heads, full attention, 286 against 345 / 284, 16384 rows,
// 4 heads, 780 against 886 / 780.
//   Beyond that whole stages follow each other: alternating mixes two access patterns that each share their stream
// through L2 (131072 rows 47.0 ms against 41.9; 16384 rows of 8 heads 1572 us against 1490).  dQ first, since the
// chunks of dK/dV are the finer ones to fill the end with (16 x 4096 rows 821 us against 838), unless a dK/dV walk
// started last would outlast the rest (24576 rows, 8 query and 2 KV heads, dQ first 3434 us, dK/dV first 3238; 65536
// rows in documents of 512, longest 4364, 625 and 497).
inline void dispatch_order(const AttnArgs& a, int64_t n_kv, int64_t n_q, MatrixParams& p) {
    const int64_t longest = a.longest > 0 && a.longest < a.S ? a.longest : a.S;
    const double steps = (double)((longest + 31) / 32);
    const int q_rows = 128 * dq_row_blocks(a.B, a.S, a.Hq);
    const double q_step = dq_step(q_rows), t_q = q_step * steps + kDqFixed;
    const double t_kv = kDkdvStep * (a.chunks.len > 0 ? a.chunks.len : steps * (a.Hq / a.Hkv) / a.chunks.nsplit) + kDkdvFixed;
    bool lead_q;
    int64_t lead;
    if (!a.row_lo && (a.off >= a.Skv || (even_walks(a.S, a.Skv, a.off) && n_kv + n_q > kComputeUnits))) {  // the longer workgroups first
        lead_q = even_dq_first(a.S, a.Skv, a.off, a.Hq, a.Hkv, q_rows, a.chunks.nsplit, a.D);
        lead = lead_q ? n_q : n_kv;
    } else if (n_kv + n_q <= (a.row_lo ? 1280 : 768)) {
        // walks fall evenly from the longest to the shortest (a short document's, or that of the first rows resp.
        // the last keys)
        double short_q = kDqFixed, short_kv = kDkdvFixed;
        if (!a.row_lo) {
            short_q += q_step * (double)((a.off + q_rows < a.Skv ? a.off + q_rows : a.Skv) / 32);
            short_kv = a.chunks.len > 0 ? t_kv : short_kv + kDkdvStep * dkdv_tile_steps(order_tiles(a.Skv) - 1, a.S, a.off, a.Hq / a.Hkv) / a.chunks.nsplit;
        }
        lead_q = t_q >= t_kv;
        const double longer = lead_q ? t_q : t_kv, other = lead_q ? t_kv : t_q, least = lead_q ? short_q : short_kv;
        const double share = longer > least ? (longer - other) / (longer - least) : 1.;
        lead = (int64_t)((double)(lead_q ? n_q : n_kv) * (share < 1. ? share : 1.));
    } else {
        // dQ first unless the longest dK/dV walk, started last, would outlast the rest of its stage
        double kv_all;  // dK/dV work per compute unit; packed documents: as if all were of the mean length
        if (a.row_lo) {
            kv_all = t_kv * (double)n_kv * (double)(a.S / (a.n_docs > 0 ? a.n_docs : 1)) / (double)longest / (double)kComputeUnits;
        } else {
            const int32_t tiles = order_tiles(a.Skv), G = a.Hq / a.Hkv;
            const double mean = ((double)dkdv_tile_steps(0, a.S, a.off, G) + (double)dkdv_tile_steps(tiles - 1, a.S, a.off, G)) / 2.;
            kv_all = (kDkdvStep * mean * tiles * (double)a.Hkv * a.B + kDkdvFixed * (double)n_kv) / (double)kComputeUnits;
        }
        lead_q = t_kv <= kv_all;
        lead = lead_q ? n_q : n_kv;
    }
    p.lead_is_q = lead_q;
    p.n_lead = (uint32_t)lead;
    p.mix_q = (uint32_t)(lead_q ? n_q - lead : n_q);
    p.mix_kv = (uint32_t)(lead_q ? n_kv : n_kv - lead);
}

template <int D, bool VARLEN, int NQ, bool LONG>
void launch_grid(const MatrixParams& p, unsigned n, hipStream_t st) {
    if (p.kv.chunks.nsplit > 1) hipLaunchKernelGGL((attn_bwd_matrix_kernel<D, VARLEN, true, NQ, LONG>), dim3(n), dim3(dkdv::kThreads), 0, st, p);
    else hipLaunchKernelGGL((attn_bwd_matrix_kernel<D, VARLEN, false, NQ, LONG>), dim3(n), dim3(dkdv::kThreads), 0, st, p);
}

template <int D, bool VARLEN, bool LONG>
sp_status launch_matrix(const AttnArgs& a, hipStream_t st) {
    MatrixParams p{};
    int nq;  // row blocks of a dQ wave
    const bool kv = (a.stages & SP_BWD_STAGE_DKDV) != 0, qs = (a.stages & SP_BWD_STAGE_DQ) != 0;
    static_assert(dkdv::BNK == kOrderTile && dq::kRows<2> == kOrderTile, "the tile orders are made for this tile size");
    {
        dkdv::DkdvParams& k = p.kv;
        k.q = (const __bf16*)a.q; k.k = (const __bf16*)a.k; k.v = (const __bf16*)a.v; k.dO = (const __bf16*)a.dO;
        k.aux = a.aux; k.dk = (__bf16*)a.dk; k.dv = (__bf16*)a.dv; k.row_hi = a.row_hi; k.order = a.order_k;
        k.S = a.S; k.Skv = a.Skv; k.off = a.off; k.S_pad = a.S_pad; k.Hq = a.Hq; k.Hkv = a.Hkv; k.G = a.Hq / a.Hkv;
        k.qmap = a.qmap; k.kvmap = a.kvmap;
        k.n_ktiles = (a.Skv + dkdv::BNK - 1) / dkdv::BNK;
        k.chunks = a.chunks; k.part = a.dkdv_part;
        k.scale = a.scale; k.scale_log2 = a.scale * kLog2e;
        k.B = a.B;
        if (kv && (k.chunks.nsplit < 1 || (k.chunks.nsplit > 1 && !k.part))) return SP_ERR_WORKSPACE;
    }
    {
        dq::DqParams& q = p.q;
        q.q = (const __bf16*)a.q; q.k = (const __bf16*)a.k; q.v = (const __bf16*)a.v; q.dO = (const __bf16*)a.dO;
        q.lse = a.lse; q.delta = a.delta; q.dq = (__bf16*)a.dq; q.row_lo = a.row_lo; q.order = a.order_q;
        q.B = a.B; q.S = a.S; q.Skv = a.Skv; q.off = a.off; q.Hq = a.Hq; q.Hkv = a.Hkv; q.G = a.Hq / a.Hkv;
        q.qmap = a.qmap; q.kvmap = a.kvmap;
        nq = dq_row_blocks(a.B, a.S, a.Hq);
        const int rows = nq == 1 ? dq::kRows<1> : dq::kRows<2>;
        q.n_qtiles = (a.S + rows - 1) / rows;
        q.n_ranks = VARLEN && q.order ? order_tiles(a.S) * (kOrderTile / rows) : q.n_qtiles;
        q.scale = a.scale; q.scale_log2 = a.scale * kLog2e;
    }
    const int64_t n_kv = kv ? (int64_t)p.kv.chunks.n_chunks * a.Hkv * a.B : 0;
    const int64_t n_q = qs ? (int64_t)p.q.n_ranks * a.Hq * a.B : 0;
    if (n_kv + n_q > 0x7fffffff) return SP_ERR_SHAPE;
    dispatch_order(a, n_kv, n_q, p);
    constexpr int64_t kMaxGrid = 1 << 23;  // workgroups per launch (a grid holds fewer than 2^32 threads)
    for (int64_t base = 0; base < n_kv + n_q; base += kMaxGrid) {
        const int64_t n = n_kv + n_q - base < kMaxGrid ? n_kv + n_q - base : kMaxGrid;
        p.base = (uint32_t)base;
        if (nq == 1) launch_grid<D, VARLEN, 1, LONG>(p, (unsigned)n, st);
        else launch_grid<D, VARLEN, 2, LONG>(p, (unsigned)n, st);
        if (launch_status() != SP_OK) return SP_ERR_LAUNCH;
    }
    return SP_OK;
}

}  // namespace
