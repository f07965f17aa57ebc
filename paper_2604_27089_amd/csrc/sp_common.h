// Shared host-side declarations of the C-ABI layer (validation helpers and the
// kernel launchers implemented in the .hip files).
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include "../../include/sp_hotpath.h"

namespace sp {

inline bool aligned16(const void* p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

inline sp_status launch_status() {
    return hipGetLastError() == hipSuccess ? SP_OK : SP_ERR_LAUNCH;
}

// Where row r (0 <= r < S) of an attention-side [S, H, D] tensor lives, in elements from the start of
// its batch entry (the head offset h*D comes on top).  Two layouts are served by the same kernels:
//   attention-side  [S, H, D]        : r * H*D
//   sequence-side   [S_l, P*H, D]    : (r % S_l) * P*H*D + (r / S_l) * H*D
// the second being the tensor whose pack (seq -> head re-layout) is the first: reading through this map
// folds the pack into the attention kernels' loads and the unpack into their stores.  S_l is a power
// of two there (mask/shift); the attention-side case uses shift 31, so r >> shift is 0 for every row.
// A batch entry spans S*H*D elements in both layouts.
struct RowMap {
    uint32_t mask;          // S_l - 1, or 0x7fffffff
    int32_t shift;          // log2(S_l), or 31
    uint32_t row_stride;    // elements between consecutive rows of a chunk
    uint32_t chunk_stride;  // elements between chunk p and chunk p+1 (H*D, or 0)
    __host__ __device__ size_t off(int32_t r) const {
        return (size_t)((uint32_t)r & mask) * row_stride + (size_t)((uint32_t)r >> shift) * chunk_stride;
    }
    static RowMap attention_side(int32_t H, int32_t D) { return RowMap{0x7fffffffu, 31, (uint32_t)(H * D), 0u}; }
    static RowMap sequence_side(int32_t S_l_log2, int32_t H, int32_t D, int32_t P) {
        return RowMap{(1u << S_l_log2) - 1u, S_l_log2, (uint32_t)(P * H * D), (uint32_t)(H * D)};
    }
};

// How the dK/dV work of the key tiles of one sequence and KV head is cut into chunks, one workgroup each.
struct DkdvChunks {
    int32_t nsplit;    // chunks per key tile, and (times the keys) the room there is for partial sums
    int32_t len;       // > 0: instead, every tile gets as many chunks of about this many steps as it needs
    int32_t n_chunks;  // over all key tiles
};

// One attention problem as the kernels see it.  Dense calls are B independent
// sequences of S rows; packed-document calls are B = 1, S = T rows with a
// per-row visibility window taken from `row_lo` / `row_hi`.  In general the S
// query rows face Skv keys and row i sees keys j <= i + off (one step of a ring
// schedule); every key must be seen by some row (Skv <= S + off, off >= 0).
// Causal attention over one sequence is Skv = S, off = 0.
struct AttnArgs {
    const void* q; const void* k; const void* v;   // bf16
    void* o; float* lse;                           // fwd outputs (bwd: inputs)
    const void* dO; void* dq; void* dk; void* dv;  // bwd only
    float* delta;                                  // bwd workspace, [B, Hq, S] fp32
    float* aux;                                    // bwd workspace, [B*Hq, S_pad/32, 2, 32] fp32: per 32-row
                                                   // tile, 32 x -LSE/scale then 32 x -Delta
    int32_t S_pad;                                 // rows per head in aux (S rounded up to 64, plus 64)
    const int32_t* row_lo;  // varlen: first row of the row's document, [S]; null if dense
    const int32_t* row_hi;  // varlen: one past the last row of the row's document, [S]
    const int32_t* order_q; // varlen: query tiles (256 rows) in the order workgroups take them; null = last first
    const int32_t* order_k; // varlen: key tiles (256 keys) likewise; null = first first
    int32_t B, S, Hq, Hkv, D;
    int32_t Skv, off;       // keys per sequence; causal offset
    RowMap qmap, kvmap;     // layout of q, o, dO, dq and of k, v, dk, dv
    float scale;            // softmax scale (already defaulted)
    int32_t stages;         // bwd: bit mask of SP_BWD_STAGE_*
    int32_t n_docs;         // varlen: number of documents (else 0)
    int32_t longest;        // bwd: upper bound of the longest document, when the caller knows one (else 0)
    DkdvChunks chunks;      // bwd: the work split of the dK/dV stage (dkdv_split_count, dkdv_chunks)
    float* dkdv_part;       // bwd workspace: the chunks' fp32 partial sums (null when chunks.nsplit == 1)
};

sp_status launch_relayout(const void* in, void* out, int64_t B, int64_t S_l, int64_t H, int64_t D,
                          int32_t P, int32_t elem_bytes, bool to_head, hipStream_t st);
// Longest-first tile orders for packed documents (doc_bounds.hip).  All three attention kernels use tiles
// of kOrderTile rows resp. keys per workgroup.  Above kMaxOrderTiles tiles the quadratic ranking is not
// worth its time and callers pass null orders.
constexpr int32_t kOrderTile = 256;
constexpr int32_t kMaxOrderTiles = 16384;
constexpr int64_t kComputeUnits = 256;
inline int32_t order_tiles(int64_t T) { return (int32_t)((T + kOrderTile - 1) / kOrderTile); }
// Per-row document windows, and (if `work` is not null) the tile orders: `work` is scratch of
// 2*order_tiles(T) int32, `order_q`, `order_k` receive order_tiles(T) int32 each.
sp_status launch_doc_bounds(const int32_t* cu_seqlens, int32_t n_docs, int32_t T, int32_t* row_lo,
                            int32_t* row_hi, int32_t* work, int32_t* order_q, int32_t* order_k, hipStream_t st);
// Debug aid: writes 0 to *flag if cu_seqlens is well formed for T rows, else a bit mask (doc_bounds.hip).
sp_status launch_check_cu_seqlens(const int32_t* cu_seqlens, int32_t n_docs, int32_t T, int32_t* flag, hipStream_t st);
// Grid of the forward and dQ kernels: x = head + Hq * batch, (y, z) = rank of the query tile in the order the
// tiles are taken (rank = y + kRankY * z).  Workgroups are dispatched x first, so all heads and batch entries
// of the longest tile go out before any shorter tile (a batch-major order would end with the long tiles of
// the last batch entry).
constexpr uint32_t kRankY = 32768;
inline dim3 tile_rank_grid(int32_t Hq, int32_t B, int32_t n_tiles) {
    return dim3((uint32_t)Hq * (uint32_t)B, (uint32_t)n_tiles < kRankY ? (uint32_t)n_tiles : kRankY,
                ((uint32_t)n_tiles + kRankY - 1) / kRankY);
}
// How many key groups share a forward workgroup (attn_fwd.hip): its 8 waves cover 256 / KS rows, and every KS-th
// key tile goes to the same group.  A compute unit holds one workgroup, and a workgroup walks its keys tile by
// tile, so a launch of few 256-row tiles leaves most units idle while the longest tile is walked alone: KS groups
// give KS times the workgroups, each with 1/KS of the walk, for KS times the K/V bytes staged per product.  The
// count is taken whose estimate is least: no launch ends before its longest workgroup, nor before the work shared
// out evenly plus the units' idle time in a last round of (at least) the shortest workgroups, a fifth slower than
// a workgroup alone (clock and shared paths); a workgroup takes 1.6 us per 64 keys of its walk, 8 and 38 % more
// per key with 2 and 4 groups, and 9 to 10.5 us beyond.
// Measured, 4 query heads of D = 128, KS = 1 / 2 / 4, us: 512 rows (8 tiles of 256) 23 / 17 / 15, 4096 rows (64) 106 /
// 61 / 49, 8192 rows (128) 196 / 116 / 114, 12288 rows (192) 310 / 192 / 247, 16384 rows (256) 405 / 292 / 379, 24576
// rows (384) 654 / 639 / 793, 32768 rows (512) 1000 / 1057 / 1365; 8 x 2048 rows (256) 64 / 52 / 73; 64 x 512 rows (512)
// 49 / 66 / 86; D = 64: 8192 rows 164 / 90 / 64, 16384 rows 318 / 204 / 216; rows that see every key (a past block of a
// ring): 2048 rows, 32 heads 72 / 76 / -, 700 rows, 24 heads 29 / 20 / 31.  A function of the extents only, so that every
// layout and entry point of one problem gives the same bits (one packed document included).
constexpr double kGroupWork[3] = {1., 1.08, 1.38}, kGroupFixed[3] = {9., 10., 10.5};  // by log2 of the groups
inline double key_group_per_key(int i) { return 1.6 / 64. * kGroupWork[i] / (1 << i); }  // us per key of a workgroup's walk
// When `workgroups` of `work` us in all are done, the first (shortest) and last of which take t_first and t_last.
inline double key_groups_end(double workgroups, double work, double t_first, double t_last) {
    const double rounds = workgroups / (double)kComputeUnits;
    const double spread = 1.2 * (work / (double)kComputeUnits + t_first * ((double)(int64_t)(rounds + 0.999999) - rounds));
    return rounds > 1. && spread > t_last ? spread : t_last;
}
inline int fwd_key_groups(int64_t B, int64_t S, int64_t Skv, int64_t off, int32_t Hq) {
    const double heads = (double)Hq * (double)B;
    if (heads * (double)S > 1024. * kOrderTile) return 1;  // many rounds
    int best = 1;
    double best_time = 0.;
    for (int i = 0; i < 3; ++i) {
        const int64_t rows = kOrderTile >> i, ranks = (S + rows - 1) / rows;
        const double per_key = key_group_per_key(i);
        const int64_t ramp_end = off < Skv ? (Skv - off) / rows : 0;  // tiles whose last row does not see every key yet
        const double ramp = (double)(ramp_end < ranks ? ramp_end : ranks);
        const double keys = ramp * (double)off + (double)rows * ramp * (ramp + 1.) / 2. + ((double)ranks - ramp) * (double)Skv;
        const int64_t first = off + rows < Skv ? off + rows : Skv, last = off + S < Skv ? off + S : Skv;
        const int64_t least = 32 << i;
        const double t_first = per_key * (double)(first > least ? first : least) + kGroupFixed[i], t_last = per_key * (double)last + kGroupFixed[i];
        const double time = key_groups_end(heads * (double)ranks, heads * (per_key * keys + kGroupFixed[i] * (double)ranks), t_first, t_last);
        if (i == 0 || time < best_time) { best = 1 << i; best_time = time; }
    }
    return best;
}
// The same for packed documents, of which the host knows only how many there are.  Taken as one sequence, short documents
// got more groups than their walks are long enough for: documents of 256 rows, 4 heads of D = 128, 14272 rows 30 us with
// one group, 36 with two; of 512 rows, 17615 rows 44 / 52; of 1024 rows, 8 heads, 9399 rows 48 / 54.  So they count as
// documents of (nearly) the mean length: a tile walks from the start of its first row's document, 0.6 of a mean length
// before it, at most 1.5 (0.5 and 1 if all are equally long; lengths that differ lengthen both, and documents much longer
// than that gain from groups that this rule does not give: 8627 rows in 44 documents, the longest 963, 8 heads, 52 us
// with one group, 48 with two).  Over 17911 packed batches of 256 to 66000 rows, equal and lognormal lengths, a mean of
// 0.81 of the time with one group and two batches more than 4 % above it; as one sequence 0.78, and 451, by up to 34 %.
inline int packed_key_groups(int64_t T, int64_t n_docs, int32_t Hq) {
    if (n_docs <= 1) return fwd_key_groups(1, T, T, 0, Hq);
    if ((double)Hq * (double)T > 1024. * kOrderTile) return 1;
    const double mean = (double)((T + n_docs - 1) / n_docs);
    int best = 1;
    double best_time = 0.;
    for (int i = 0; i < 3; ++i) {
        const int64_t rows = kOrderTile >> i, ranks = (T + rows - 1) / rows;
        const double per_key = key_group_per_key(i), most = (double)T;
        const double walk = 0.6 * mean + (double)rows, longest = 1.5 * mean + (double)rows, workgroups = (double)Hq * (double)ranks;
        const double work = workgroups * (per_key * (walk < most ? walk : most) + kGroupFixed[i]);
        const double time = key_groups_end(workgroups, work, per_key * (double)rows + kGroupFixed[i], per_key * (longest < most ? longest : most) + kGroupFixed[i]);
        if (i == 0 || time < best_time) { best = 1 << i; best_time = time; }
    }
    return best;
}
// Row blocks of 32 query rows per wave of the dQ stage: 2 (256 rows per workgroup) unless the launch has few tiles
// and is bound by the walk of the longest one.  With one block a wave's step takes 0.4 us instead of 0.75 and there are
// twice the workgroups, but every K/V operand read from LDS feeds one MFMA instead of two (16x16x32: two
// instead of four).  Same bits.  Backward
// with 2 / 1 blocks, 4 heads of D = 128, us: 2048 rows (32 tiles of 256) 75 / 59, 4096 rows (64) 127 / 103, 8192 rows
// (128) 280 / 246, 10007 rows of 3 heads (120) 330 / 277, 12288 rows (192) 483 / 509, 16384 rows (256) 835 / 855;
// 8192 rows of 5 heads (160) 347 / 354; D = 64: 4096 rows 87 / 70, 8192 rows 173 / 150.
inline int dq_row_blocks(int64_t B, int64_t S, int32_t Hq) {
    return (S + kOrderTile - 1) / kOrderTile * Hq * B <= 128 ? 1 : 2;
}
sp_status launch_attn_fwd(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_bwd(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_bwd_matrix_d64(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_bwd_matrix_d128(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_bwd_matrix_long_d64(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_bwd_matrix_long_d128(const AttnArgs& a, hipStream_t st);
sp_status launch_attn_merge(float* o_acc, float* lse_acc, const void* o_blk, const float* lse_blk, void* o_out,
                            int64_t B, int64_t S, int32_t Hq, int32_t D, hipStream_t st);

// How many workgroups share one 256-key tile of the dK/dV kernel.  A key tile's work is every row from
// its diagonal to the end of the sequence (or document), for every query head of the group: with one KV
// head that is one workgroup per 256 keys, far too few to fill and balance 256 compute units below a
// few hundred thousand rows (at 32K rows: 128 workgroups, the longest doing 1/64 of all the work).  The
// (head, row tile) steps of a key tile are therefore cut into this many contiguous chunks, one workgroup
// each, whose fp32 partial sums a second kernel adds in a fixed order (measured: 4.36 -> 1.65 ms at 32K
// rows, 10.1 -> 6.3 ms at 64K, 25.3 -> 24.7 ms at 128K).
// n chunks per tile cost (tiles * n / 256) times what a workgroup takes beyond its steps, and leave a longest chunk of
// steps_first / n steps, a fraction of which is exposed at the end.  The sum is smallest near n = sqrt(2.1 * steps_first /
// tiles); at most 8 chunks, and no more than about 2048 workgroups.  (The constant was fitted to sequences of 1K to 128K
// rows, dense and packed, when a workgroup stored its sums 4 bytes per lane and took 27 us beyond its steps; it is 20 now,
// and the count is still within a few percent of the best: 16384 rows, 4 heads, 5 chunks instead of 8 are 4 % faster at
// D = 128 and slower at D = 64, 32768 rows 4 instead of 8 1 %.)  It is also the room for partial sums: the rules below
// take at most as many.  `longest` = the longest sequence in the call when the caller knows it (packed documents: the
// max_seqlen hint), else S.  The counts depend on extents only, so one packed document and a dense call of equal extents
// agree bitwise.
inline int32_t dkdv_split_count(int64_t B, int64_t S, int64_t Skv, int32_t Hq, int32_t Hkv, int64_t longest = 0) {
    if (B <= 0 || S <= 0 || Skv <= 0 || Hkv <= 0) return 1;
    if (longest <= 0 || longest > S) longest = S;
    const int64_t tiles = (Skv + 255) / 256 * Hkv * B;
    const int64_t steps_first = (longest + 31) / 32 * (Hq / Hkv);  // steps of the longest key tile
    int64_t n = 1;
    while (n < 8 && (2 * n + 1) * (2 * n + 1) * tiles * 10 <= 4 * 21 * steps_first) ++n;  // n <= sqrt(2.1 x) + 0.5
    // Several sequences are dispatched batch entry fastest, longest tiles of every sequence first: with few tiles two
    // chunks each, and at least a workgroup per compute unit, balance better than the rule above (backward, chunks 1 /
    // 2 / 4 / 8, us: 32 x 2048 rows, 256 tiles, 571 / 510 / 508 / 506; 64 x 512 rows, 128 tiles, 153 / 152 / 165 / 163;
    // 4 x 4096 rows, 64 tiles, 614 / 342 / 237 / 255; 8 x 2048 rows, 64 tiles, 323 / 187 / 147 / 164).
    if (B > 1 && n * tiles < 512) {
        const int64_t fill = (256 + tiles - 1) / tiles < 8 ? (256 + tiles - 1) / tiles : 8;
        const int64_t least = fill > 2 ? fill : 2;
        if (n < least) n = least;
    }
    const int64_t cap = (2048 + tiles - 1) / tiles;
    if (n > cap) n = cap;
    return n < 1 ? 1 : (int32_t)n;
}
// What the estimates take a workgroup of the two matrix stages to cost in a full chip, in us: per 32-row step of dK/dV, per
// 32-key step of dQ with one or two row blocks (D = 128; D = 64 takes two thirds), and beyond the steps (resident operands
// and first tiles, the pipeline's fill, the results).  Fitted to the 32x32x16 programs, which run wherever a count or an
// order is worth more than a few percent; the 16x16x32 ones of long launches take 4 to 7 % less for either stage (D = 64:
// 0.58 of D = 128 for dK/dV, 0.61 for dQ), and what decides is the ratio of the two.
constexpr double kDkdvStep = 1.5, kDkdvFixed = 20., kDqFixed = 10.;
inline double dq_step(int64_t q_rows) { return q_rows == 128 ? 0.5 : 0.95; }
inline double step_share(int32_t D) { return D == 64 ? 2. / 3. : 1.; }
// What the kernel that adds the chunks' partial sums takes, in us: written once and read once at 12 TB/s (they stay in the
// memory-side cache), and a launch.
inline double dkdv_reduce_time(int64_t B, int64_t Skv, int32_t Hkv, int32_t D, int32_t nsplit) {
    return 4. + (double)nsplit * (double)B * (double)Skv * Hkv * D * 16. / 12e6;
}
// (head, row tile) steps of the 256 keys of tile jt when the whole sequence is one document
__host__ __device__ inline int32_t dkdv_tile_steps(int32_t jt, int32_t S, int32_t off, int32_t G) {
    const int32_t j0 = jt * kOrderTile;
    return ((S + 31) / 32 - (j0 > off ? j0 - off : 0) / 32) * G;
}
// Where the work of every tile is known on the host (one document per sequence), there are several sequences or KV
// heads and at most as many key tiles as compute units, the number of chunks follows from an estimate of when dK/dV and
// dQ, launched together, are done: not before the longest workgroup of either, nor before all work shared out evenly,
// plus an eighth of the longest dK/dV workgroup for the uneven end and the reduction of the partial sums.  Of 1 ..
// `most`, the count that the rule above gives and the workspace is sized for.  Backward, rule / estimate (with the order
// of dispatch of attn_bwd_matrix.h), us: 16 x 1024 rows of 4 heads, full attention, 129 / 96; 32 x 2048 rows, 4 query
// heads and one KV head, 499 / 461; 4096 rows, 32 and 8 heads, 566 / 436; 2500 rows, the same, 280 / 198.  For a single
// KV head the estimate gives no more than the rule (16384 rows 765 / 765 us, D = 64 458 / 467; 65536 rows 10.8 / 11.0 ms).
inline int32_t dkdv_causal_splits(int64_t B, int32_t S, int32_t Skv, int32_t off, int32_t Hq, int32_t Hkv, int32_t D, int32_t most) {
    const int32_t tiles = order_tiles(Skv), G = Hq / Hkv, q_rows = 128 * dq_row_blocks(B, S, Hq);
    const double head_b = (double)Hkv * (double)B, scale = step_share(D), kv_step = scale * kDkdvStep, q_step = scale * dq_step(q_rows);
    double steps = 0.;
    for (int32_t t = 0; t < tiles; ++t) steps += dkdv_tile_steps(t, S, off, G);
    const double longest = dkdv_tile_steps(0, S, off, G);
    const double ranks = (double)(((int64_t)S + q_rows - 1) / q_rows), n_q = ranks * Hq * (double)B;
    const double q_last = (double)((Skv + 31) / 32), q_first = (double)((off < Skv ? off : Skv) / 32);
    const double t_q = q_step * q_last + kDqFixed, work_q = n_q * (q_step * (q_first + q_last) / 2. + kDqFixed);
    int32_t best = 1;
    double best_time = 0.;
    for (int32_t n = 1; n <= most; ++n) {
        const double jobs = (double)tiles * n * head_b;
        double t_kv = kv_step * longest / n + kDkdvFixed;
        if (n > 1 && jobs + n_q <= (double)kComputeUnits) t_kv = kv_step * 1.1 * steps * head_b / jobs + kDkdvFixed;  // equal chunks
        const double shared = (kv_step * steps * head_b + kDkdvFixed * jobs + work_q) / (double)kComputeUnits + 10.;
        double time = t_kv > t_q ? t_kv : t_q;
        if (shared > time) time = shared;
        time += t_kv / 8.;
        if (n > 1) time += dkdv_reduce_time(B, Skv, Hkv, D, n);
        if (n == 1 || time < best_time) { best = n; best_time = time; }
    }
    return best;
}
// Equal chunks.  A causal key tile's steps fall linearly from the first tile to the last, so the same number of
// chunks for every tile makes the first tile's twice as long as the mean.  A launch whose workgroups all run at once
// (dK/dV and dQ together at most one per compute unit) ends with those, so there, if the work of each tile is known
// on the host (`causal`: one document per sequence), tiles get chunks of one length instead, as short as the room
// for partial sums allows (a tile's chunks times its keys, summed, at most nsplit * Skv).  A workgroup finds its
// tile with one scan over the tiles' chunk counts, a tile per lane of a wave.  Launches of several rounds keep the
// unequal chunks: the short ones fill the end.  Backward with unequal / equal chunks, us, 4 heads of D = 128: 2048
// rows 59 / 53, 3000 rows 79 / 69, 4096 rows 100 / 89; two rounds, 8192 rows, 233 / 250; four, 16384 rows, 786 / 839.
constexpr int32_t kMaxEqualTiles = 64;
inline DkdvChunks dkdv_chunks(int64_t B, int32_t S, int32_t Skv, int32_t off, int32_t Hq, int32_t Hkv, int32_t D, int32_t nsplit, bool causal) {
    const int32_t n = order_tiles(Skv), G = Hq / Hkv, q_rows = 128 * dq_row_blocks(B, S, Hq);
    const int64_t n_q = ((int64_t)S + q_rows - 1) / q_rows * Hq * B;
    if (causal && (int64_t)Hkv * B > 1 && (int64_t)n * Hkv * B <= kComputeUnits) nsplit = dkdv_causal_splits(B, S, Skv, off, Hq, Hkv, D, nsplit);
    const int64_t workgroups = (int64_t)n * nsplit * Hkv * B + n_q;
    DkdvChunks c{nsplit, 0, n * nsplit};
    if (!causal || workgroups > kComputeUnits || nsplit < 2 || n < 2 || n > kMaxEqualTiles || (int64_t)S * G > (int64_t)1 << 30) return c;
    int64_t total = 0;
    for (int32_t t = 0; t < n; ++t) total += dkdv_tile_steps(t, S, off, G);
    // steps are taken four at a time, so lengths are multiples of four; the smallest one (up to 1/16) that fits
    for (int64_t len = (total / ((int64_t)n * nsplit) + 4) & ~(int64_t)3;; len += (len / 16 + 4) & ~(int64_t)3) {
        int64_t rows = 0;
        int32_t chunks = 0;
        for (int32_t t = 0; t < n; ++t) {
            const int32_t k = (int32_t)((dkdv_tile_steps(t, S, off, G) + len - 1) / len);
            const int32_t keys = Skv - t * kOrderTile;
            chunks += k;
            rows += (int64_t)k * (keys < kOrderTile ? keys : kOrderTile);
        }
        if (rows <= (int64_t)nsplit * Skv) return DkdvChunks{nsplit, (int32_t)len, chunks};
    }
}
// When the chip is done with n workgroups that take walk(0), walk(1), .. us in the order of dispatch.  Workgroups are dealt
// to the shader engines in turn and stay there, on whichever unit of the engine comes free first; the first engine, which
// has as many as any, stands for all.  (Counted over the whole chip, 224 workgroups of dQ just fit twice on the 116 units
// that 140 of dK/dV leave; they took a third round, 553 us of dK/dV alone, 688 together.)
constexpr int64_t kEngines = 32, kEngineUnits = kComputeUnits / kEngines;
template <typename WALK>
inline double dispatch_end(int64_t n, WALK&& walk) {
    double unit[kEngineUnits] = {}, end = 0.;
    for (int64_t i = 0; i < n; i += kEngines) {
        int u = 0;
        for (int j = 1; j < kEngineUnits; ++j) u = unit[j] < unit[u] ? j : u;
        unit[u] += walk(i);
        if (unit[u] > end) end = unit[u];
    }
    return end;
}
// Even walks: the shortest walk of either stage is at least a third of the longest (a block from the past in a ring
// schedule, or any causal offset from a third of the keys on).  Beyond one round of the chip such workgroups end in whole
// rounds, like those of a block that hides nothing, and the estimates for a causal ramp do not see that: with them an
// offset one below "hides nothing" got another chunk count and order, and times up to 17 % above those of one stage
// after the other (backward, us, one stage after the other / causal estimate / this rule: 7039 rows of 16 and 4 heads,
// D = 64, offset 7038, 685 / 805 / 678; 9224 rows, 20 and 5 heads, offset 9106, 1430 / 1602 / 1392).  1356 shapes with
// offsets above half: 0.690 of the time of one stage after the other with the causal estimates, 17 of them more than 3 %
// above it; with this rule 0.671 and 4 (5 % in one round of dK/dV beside one of dQ: 5860 rows of 8 heads 435 / 456).
// Offsets of a third to half of the keys, 182 shapes: 0.758 and 0.736.  Below a third the causal estimates stay: none of
// 363 shapes was slower with them than one stage after the other.
inline bool even_walks(int64_t S, int64_t Skv, int64_t off) { return 3 * off >= Skv && 3 * (Skv - off) <= 2 * S; }
// The share of the (row, key) pairs that are visible there, and what a workgroup of either stage takes on average, in us.
inline double even_share(int64_t S, int64_t Skv, int64_t off) {
    const double hidden = off < Skv ? (double)(Skv - off) : 0.;
    return 1. - hidden * hidden / (2. * (double)S * (double)Skv);
}
inline double even_dq_time(int64_t S, int64_t Skv, int64_t off, int64_t q_rows, int32_t D) {
    return step_share(D) * dq_step(q_rows) * (double)((Skv + 31) / 32) * even_share(S, Skv, off) + kDqFixed;
}
inline double even_dkdv_time(int64_t S, int64_t Skv, int64_t off, int32_t G, int32_t nsplit, int32_t D) {
    return step_share(D) * kDkdvStep * (double)((S + 31) / 32 * G) * even_share(S, Skv, off) / nsplit + kDkdvFixed;
}
// The stage with the longer workgroups goes first, the other fills its last round.
inline bool even_dq_first(int64_t S, int64_t Skv, int64_t off, int32_t Hq, int32_t Hkv, int64_t q_rows, int32_t nsplit, int32_t D) {
    return even_dq_time(S, Skv, off, q_rows, D) > even_dkdv_time(S, Skv, off, Hq / Hkv, nsplit, D);
}
// Work split for even walks: of 1 .. `most` chunks per tile (what the workspace has room for) the one is taken with which
// both stages, every workgroup with its own walk, and the reduction of the partial sums end soonest.  (With the mean walk
// for all, offsets below half the keys got too few chunks: 4 x 8695 rows of 4 heads, D = 64, offset 3007, one chunk
// instead of two or three, 914 us instead of 819.)  A few microseconds of host time; beyond 2^20 workgroups it is not spent.
inline int32_t dkdv_full_splits(int64_t B, int64_t S, int64_t Skv, int32_t Hq, int32_t Hkv, int32_t D, int32_t most, int64_t off = INT32_MAX) {
    if (off > Skv) off = Skv;
    const int32_t G = Hq / Hkv;
    const int64_t heads_kv = Hkv * B, heads_q = Hq * B, q_rows = 128 * dq_row_blocks(B, S, Hq), ranks = (S + q_rows - 1) / q_rows, n_q = ranks * heads_q;
    const int64_t tiles = (Skv + kOrderTile - 1) / kOrderTile * heads_kv;
    if (most <= 1 || tiles * most + n_q > (int64_t)1 << 20) return most;
    const double q_step = step_share(D) * dq_step(q_rows);
    int32_t best = 1;
    double best_end = 0.;
    for (int32_t n = 1; n <= most; ++n) {
        const bool q_first = even_dq_first(S, Skv, off, Hq, Hkv, q_rows, n, D);
        const double kv_step = step_share(D) * kDkdvStep / n;
        const int64_t n_kv = tiles * n, first = q_first ? n_q : n_kv;
        double end = dispatch_end(n_kv + n_q, [&](int64_t i) {
            const int64_t wg = i < first ? i : i - first;
            if ((i < first) != q_first) return kv_step * dkdv_tile_steps((int32_t)(wg / heads_kv / n), (int32_t)S, (int32_t)off, G) + kDkdvFixed;
            const int64_t rows = (ranks - wg / heads_q) * q_rows, keys = (rows < S ? rows : S) + off;  // longest tile first
            return q_step * (double)(((keys < Skv ? keys : Skv) + 31) / 32) + kDqFixed;
        });
        if (n > 1) end += dkdv_reduce_time(B, Skv, Hkv, D, n);
        if (n == 1 || end < best_end) { best = n; best_end = end; }
    }
    return best;
}
// The work split of a dense call.
inline DkdvChunks dense_chunks(int64_t B, int32_t S, int32_t Skv, int32_t off, int32_t Hq, int32_t Hkv, int32_t D) {
    const int32_t most = dkdv_split_count(B, S, Skv, Hq, Hkv);
    if (off < Skv) {
        const DkdvChunks c = dkdv_chunks(B, S, Skv, off, Hq, Hkv, D, most, true);
        const int64_t q_rows = 128 * dq_row_blocks(B, S, Hq), n_q = (S + q_rows - 1) / q_rows * Hq * B;
        if (!even_walks(S, Skv, off) || (int64_t)c.n_chunks * Hkv * B + n_q <= kComputeUnits) return c;
    }
    const int32_t n = dkdv_full_splits(B, S, Skv, Hq, Hkv, D, most, off);
    return DkdvChunks{n, 0, n * order_tiles(Skv)};
}
// Which MFMA shape the backward's matrix stages run with: 32x32x16 (false), or in long launches 16x16x32 (true).  Where the
// chip is full for long enough the board's power sets the clock, and 16x16x32 takes less energy per product; elsewhere the
// clock is at its limit and what counts is instructions, of which that shape has twice the MFMAs, masks for twice the
// blocks and a quarter more code to fetch.  The two part at the matrix work per compute unit, in us by the costs above;
// packed documents count as all of the mean length (the caller's longest may be anything).  Measured, backward, 4 query
// heads and 1 KV head unless said otherwise, (work) 32x32x16 / 16x16x32, us:
//   D = 128, from 90: 1024 rows (2) 35.3 / 37.4, of 8 heads (5) 50.7 / 56.0, 4096 rows of 8 heads (78) 178 / 185, 6000 rows (84)
//     153 / 154, 8192 rows of 3 heads (118) 177 / 173, of 4 (157) 221 / 212, 16384 rows (627) 744 / 708, 32768 (2509) 2752 / 2608
//   D = 64, from 125: 2048 rows (7) 37.4 / 38.9, 8192 rows (105) 137 / 139, 4 x 5207 rows (169) 216 / 211, 16384 rows of 2 heads
//     (209) 249 / 253 and 258 / 257 on two cards, 11332 rows (200) 238 / 227, 32768 rows (1673) 1605 / 1525
//   rows that see every key, 8 KV heads, from 70 and 90: D = 128, 24 heads, 1470 rows (61) 115 / 118, 1660 rows (77) 134 / 131,
//     32 heads, 4096 rows (627) 696 / 659; D = 64, 32 heads, 1563 rows (61) 100 / 101, 2048 rows (105) 125 / 120
//   packed, D = 128, from 100: 5000 rows in documents of 600 (6) 75 / 84, 20000 in documents of 1024 (28) 177 / 189, 131072 in
//     documents of 256 (83) 638 / 669, of 600 (175) 976 / 961, 65536 in documents of 4096 (446) 1346 / 1311
//   packed, D = 64, from 400: 20000 rows in documents of 1024 (18) 121 / 132, 131072 in documents of 600 (117) 593 / 634, of 2000
//     (330) 912 / 940, 40000 in 6 documents (415) 1210 / 1154
// At D = 128 the chip is also full in a launch whose workgroups all run at once and end together: from work of 0.475 of its
// longest workgroup on (4096 rows, 39 of 74 us: 84.5 / 82.0 and 81.7 / 80.8 on two cards; 158 shapes below that 0.98 to 1.10
// of the time of 32x32x16, 24 from there on 0.975 to 0.99; D = 64 1.04 to 1.10 throughout).
// A function of the extents only, and the same for one packed document as for a dense call: both give the same bits.
constexpr double kLongLaunch[2][3] = {{125., 90., 400.}, {90., 70., 100.}};  // [D = 64, 128][dense, every key seen, packed]
inline bool bwd_long_launch(int64_t B, int64_t S, int64_t Skv, int64_t off, int32_t Hq, int32_t Hkv, int32_t D, int64_t n_docs) {
    const bool packed = n_docs > 1;
    const double pairs = packed ? (double)S * ((double)S / (double)n_docs) / 2. : even_share(S, Skv, off) * (double)S * (double)Skv * (double)B;
    const double work = step_share(D) * (kDkdvStep + dq_step(2 * 128)) * pairs * Hq / (32. * 256.) / (double)kComputeUnits;
    if (work >= kLongLaunch[D == 128][packed ? 2 : off >= Skv]) return true;
    if (packed || D != 128 || off != 0 || Skv != S || work < 30.) return false;
    const DkdvChunks c = dense_chunks(B, (int32_t)S, (int32_t)S, 0, Hq, Hkv, D);
    const int64_t q_rows = 128 * dq_row_blocks(B, S, Hq), n_q = (S + q_rows - 1) / q_rows * Hq * B;
    if ((int64_t)c.n_chunks * Hkv * B + n_q > kComputeUnits) return false;
    const double steps = c.len > 0 ? (double)c.len : (double)dkdv_tile_steps(0, (int32_t)S, 0, Hq / Hkv) / c.nsplit;
    const double t_kv = kDkdvStep * steps + kDkdvFixed, t_q = dq_step(q_rows) * (double)((S + 31) / 32) + kDqFixed;
    return work >= 0.475 * (t_kv > t_q ? t_kv : t_q);
}
inline size_t dkdv_part_bytes(int64_t B, int64_t Skv, int32_t Hkv, int32_t D, int32_t nsplit) {
    return nsplit > 1 ? (size_t)2 * nsplit * B * Skv * Hkv * D * sizeof(float) : 0;
}

// pointwise operators outside attention (pointwise.hip)
sp_status launch_rmsnorm_fwd(const void* x, const void* w, void* y, float* rstd, int64_t T, int32_t C, float eps,
                             hipStream_t st);
sp_status launch_rmsnorm_bwd(const void* x, const void* w, const float* rstd, const void* dy, void* dx, void* dw,
                             float* part, int64_t T, int32_t C, hipStream_t st);
int32_t rmsnorm_bwd_groups(int64_t T);  // partial rows of dw the backward writes to its workspace
sp_status launch_rope(const void* x, const float* cs, const float* sn, void* out, int64_t T, int32_t H, int32_t D,
                      bool conjugate, hipStream_t st);
sp_status launch_swiglu_fwd(const void* g, const void* u, void* y, int64_t n, hipStream_t st);
sp_status launch_swiglu_bwd(const void* g, const void* u, const void* dy, void* dg, void* du, int64_t n, hipStream_t st);

// row pitch of the per-row backward scalars
inline int32_t aux_pitch(int64_t S) { return (int32_t)((S + 63) / 64 * 64 + 64); }

}  // namespace sp
