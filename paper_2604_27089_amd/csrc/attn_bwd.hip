// Causal grouped-query attention, backward, for one device's head shard
// (paper Section 3.1: the rewritten graph must stay correct in the backward
// pass, each inserted operator having a gradient; Section 4.2 (breakdown analysis): under
// activation checkpointing the backward is where the extra time goes).
//
// Three stages, no atomics (bitwise reproducible):
//   delta : Delta_i = dO_i . O_i and the per-row seeds -LSE_i/scale, -Delta_i
//           (this file; HBM-bound, fp32 out)
//   dkdv  : attn_bwd_dkdv.h (long launches: attn_bwd_dkdv16.h), and the sum of its partial results here
//   dq    : attn_bwd_dq.h (attn_bwd_dq16.h)
// The last two are launched together (attn_bwd_matrix.h).
// P is rebuilt from the saved LSE: P_ij = exp(scale*s_ij - LSE_i); S and dP
// are evaluated in both matrix kernels.
#include "attn_bwd_dkdv.h"

namespace {

using namespace sp;

#ifdef SP_BWD_ALWAYS_LONG  // a build for tests: small shapes reach the edges of the long launches' programs
constexpr bool kAlwaysLong = true;
#else
constexpr bool kAlwaysLong = false;
#endif

// ------------------------------------------------------------------ delta
// One 16-byte vector of O and dO per lane, D/8 lanes per (row, head).  The grid covers the padded row range
// [0, S_pad): rows past the sequence only zero their slots of the per-row scalars (they are fetched by the
// dK/dV kernel, never used unmasked).
template <int D>
__global__ __launch_bounds__(256) void delta_kernel(const __bf16* __restrict__ o,
                                                   const __bf16* __restrict__ dO,
                                                   const float* __restrict__ lse,
                                                   float* __restrict__ delta, float* __restrict__ aux,
                                                   int32_t B, int32_t S, int32_t S_pad, int32_t Hq,
                                                   float inv_scale, RowMap map) {
    constexpr int LPV = D / 8;  // lanes per (row, head) vector, 16 bytes each
    const int64_t n_vec = (int64_t)B * S_pad * Hq;
    const int64_t vec = ((int64_t)blockIdx.x * 256 + threadIdx.x) / LPV;  // (b*S_pad + i)*Hq + h
    const int part = threadIdx.x % LPV;
    if (vec >= n_vec) return;  // whole (row, head) groups of lanes leave together: LPV divides 64
    const int64_t bi = vec / Hq, b = bi / S_pad;
    const int32_t h = (int32_t)(vec - bi * Hq), i = (int32_t)(bi - b * S_pad);
    // the per-row accumulator seeds of the dK/dV kernel: per 32-row tile, 32 x -LSE/scale then 32 x -Delta
    float* t = aux + ((b * Hq + h) * (S_pad / 32) + i / 32) * 64 + i % 32;
    if (i >= S) {
        if (part == 0) { t[0] = 0.f; t[32] = 0.f; }
        return;
    }
    const size_t at = (size_t)b * S * Hq * D + map.off(i) + (size_t)h * D + 8 * part;
    const bf16x8 x = as_bf16x8(*reinterpret_cast<const u32x4*>(o + at));
    const bf16x8 y = as_bf16x8(*reinterpret_cast<const u32x4*>(dO + at));
    float acc = 0.f;
#pragma unroll
    for (int e = 0; e < 8; ++e) acc += (float)x[e] * (float)y[e];
#pragma unroll
    for (int off = LPV / 2; off >= 1; off >>= 1) acc += __shfl_xor(acc, off, 64);
    if (part == 0) {
        delta[(b * Hq + h) * S + i] = acc;
        t[0] = -lse[(b * Hq + h) * S + i] * inv_scale;
        t[32] = -acc;
    }
}

// dK = scale * sum of the chunks' partial sums, dV = sum of theirs (layout: dkdv::part_offset); the outputs follow
// `map`.  A block takes 16 (D = 128) or 32 keys of one tile, a thread four keys of two columns.
template <int D>
__global__ __launch_bounds__(256) void dkdv_reduce_kernel(const float* __restrict__ part, __bf16* __restrict__ dk,
                                                         __bf16* __restrict__ dv, DkdvChunks chunks, int32_t n_tiles,
                                                         float scale, RowMap map, int32_t S, int32_t Skv, int32_t off,
                                                         int32_t G, int32_t Hkv, int64_t n_bg) {
    constexpr int CP = D / 2;                            // column pairs
    constexpr int BPT = kOrderTile / 4 / (256 / CP);     // blocks per tile
    const int64_t tile = blockIdx.x / BPT, bg = tile / n_tiles, b = bg / Hkv;
    const int jt = (int)(tile - bg * n_tiles), g = (int)(bg - b * Hkv);
    int n_split = chunks.nsplit, first = jt * n_split;
    if (chunks.len > 0) {  // uniform
        int count, upto;
        dkdv::scan_chunks(n_tiles, S, off, G, chunks.len, count, upto);
        n_split = __builtin_amdgcn_readlane(count, jt);
        first = __builtin_amdgcn_readlane(upto, jt) - n_split;
    }
    const int c = (int)(threadIdx.x % CP) * 2;
    const int k0 = ((int)(blockIdx.x % BPT) * (256 / CP) + (int)(threadIdx.x / CP)) * 4;  // in the tile
    const int keys = Skv - jt * kOrderTile < kOrderTile ? Skv - jt * kOrderTile : kOrderTile;
    if (k0 >= keys) return;
    const int n = keys - k0 < 4 ? keys - k0 : 4;
    const size_t chunk = (size_t)keys * D;  // floats from one chunk of the tile to the next
    const float* sk_ = part + dkdv::part_offset(bg, chunks.nsplit, Skv, first, 0, keys, D) + (size_t)k0 * D + (size_t)n * c;
    const float* sv_ = sk_ + (size_t)n_bg * chunks.nsplit * Skv * D;
    float sk[2][4] = {}, sv[2][4] = {};
    if (n == 4) {
#pragma unroll 4
        for (int32_t s = 0; s < n_split; ++s) {
            const f32x4 ka = *reinterpret_cast<const f32x4*>(sk_ + s * chunk), kb = *reinterpret_cast<const f32x4*>(sk_ + s * chunk + 4);
            const f32x4 va = *reinterpret_cast<const f32x4*>(sv_ + s * chunk), vb = *reinterpret_cast<const f32x4*>(sv_ + s * chunk + 4);
#pragma unroll
            for (int e = 0; e < 4; ++e) { sk[0][e] += ka[e]; sk[1][e] += kb[e]; sv[0][e] += va[e]; sv[1][e] += vb[e]; }
        }
    } else {
        for (int32_t s = 0; s < n_split; ++s)
            for (int x = 0; x < 2; ++x)
                for (int e = 0; e < 3; ++e)
                    if (e < n) {
                        sk[x][e] += sk_[s * chunk + x * n + e];
                        sv[x][e] += sv_[s * chunk + x * n + e];
                    }
    }
    const size_t base = ((size_t)b * Skv * Hkv + g) * D + c;
#pragma unroll
    for (int e = 0; e < 4; ++e)
        if (e < n) {
            const size_t o = base + map.off(jt * kOrderTile + k0 + e);
            *reinterpret_cast<uint32_t*>(dk + o) = pack_bf16(sk[0][e] * scale, sk[1][e] * scale);
            *reinterpret_cast<uint32_t*>(dv + o) = pack_bf16(sv[0][e], sv[1][e]);
        }
}

template <int D>
sp_status launch(const AttnArgs& a, hipStream_t st) {
    if (a.stages & SP_BWD_STAGE_DELTA) {
        const int64_t lanes = (int64_t)a.B * a.S_pad * a.Hq * (D / 8);
        const int64_t blocks = (lanes + 255) / 256;
        if (blocks > 0x7fffffff) return SP_ERR_SHAPE;
        hipLaunchKernelGGL((delta_kernel<D>), dim3((unsigned)blocks), dim3(256), 0, st, (const __bf16*)a.o,
                           (const __bf16*)a.dO, a.lse, a.delta, a.aux, a.B, a.S, a.S_pad, a.Hq,
                           1.0f / a.scale, a.qmap);
        if (hipGetLastError() != hipSuccess) return SP_ERR_LAUNCH;
    }
    if (a.stages & (SP_BWD_STAGE_DKDV | SP_BWD_STAGE_DQ)) {
        const bool long_launch = kAlwaysLong || bwd_long_launch(a.B, a.S, a.Skv, a.off, a.Hq, a.Hkv, a.D, a.row_lo ? a.n_docs : 0);
        const sp_status r = D == 64 ? (long_launch ? launch_attn_bwd_matrix_long_d64(a, st) : launch_attn_bwd_matrix_d64(a, st))
                                    : (long_launch ? launch_attn_bwd_matrix_long_d128(a, st) : launch_attn_bwd_matrix_d128(a, st));
        if (r != SP_OK) return r;
    }
    if ((a.stages & SP_BWD_STAGE_DKDV) && a.chunks.nsplit > 1) {
        const int32_t tiles = order_tiles(a.Skv);
        const int64_t blocks = (int64_t)a.B * a.Hkv * tiles * (kOrderTile / 4 / (256 / (D / 2)));
        if (blocks > 0x7fffffff) return SP_ERR_SHAPE;
        hipLaunchKernelGGL((dkdv_reduce_kernel<D>), dim3((unsigned)blocks), dim3(256), 0, st, a.dkdv_part, (__bf16*)a.dk,
                           (__bf16*)a.dv, a.chunks, tiles, a.scale, a.kvmap, a.S, a.Skv, a.off, a.Hq / a.Hkv, a.Hkv,
                           (int64_t)a.B * a.Hkv);
        if (launch_status() != SP_OK) return SP_ERR_LAUNCH;
    }
    return SP_OK;
}

}  // namespace

namespace sp {

sp_status launch_attn_bwd(const AttnArgs& a, hipStream_t st) {
    if (a.Hq > 65535 || a.B > 65535) return SP_ERR_SHAPE;
    if (a.D == 128) return launch<128>(a, st);
    if (a.D == 64) return launch<64>(a, st);
    return SP_ERR_UNSUPPORTED;
}

}  // namespace sp
