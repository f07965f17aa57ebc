// Device-side building blocks shared by the attention kernels: vector types,
// the bf16 MFMA wrapper and its operand / accumulator lane layouts.
//
// v_mfma_f32_32x32x16_bf16 computes C[32x32] += A[32x16] * B[16x32] per wave.
// With lane l, lo = l % 32, hi = l / 32:
//   A operand: lane holds A[lo][8*hi + e], e = 0..7   (8 bf16 = 16 bytes)
//   B operand: lane holds B[8*hi + e][lo], e = 0..7
//   C/D      : lane holds C[8*(r/4) + 4*hi + r%4][lo] in register r = 0..15
// The contraction index only has to be paired consistently between A and B,
// which the kernels use to feed an accumulator straight back in as an operand:
// registers r = 8c .. 8c+7 of a C tile are rows {16c + 4*hi + e, 16c + 8 + 4*hi + e}.
#pragma once
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>
#include <utility>

namespace sp {

typedef __bf16 bf16x8 __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x4 __attribute__((ext_vector_type(4)));
typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef float f32x2 __attribute__((ext_vector_type(2)));
typedef uint32_t u32x4 __attribute__((ext_vector_type(4)));
typedef uint32_t u32x2 __attribute__((ext_vector_type(2)));

// Branches of the hand-scheduled loops: the rare side goes out of line, so that the usual path takes no jump.
#define SP_LIKELY(x) __builtin_expect(!!(x), 1)
#define SP_UNLIKELY(x) __builtin_expect(!!(x), 0)
// ... unless the walks are short: packed documents take the rare sides in a few steps of many walks, each time from cold
// code far from the loop (backward, out of line / in line, us: 20000 rows in documents of 4096, 390 / 375, 9000 in documents
// of 2000, 172 / 166; dense 16384 rows, D = 64, 421 / 429).
#define SP_RARE(VARLEN, x) ((VARLEN) ? !!(x) : SP_UNLIKELY(x))
template <int N> using Int = std::integral_constant<int, N>;

// compile-time loop: f(std::integral_constant<int, I>{}) for I in [B, E)
template <int B, int E, typename F>
__device__ __forceinline__ void static_for(F&& f) {
    if constexpr (B < E) {
        f(std::integral_constant<int, B>{});
        static_for<B + 1, E>(static_cast<F&&>(f));
    }
}

constexpr float kLog2e = 1.4426950408889634f;
constexpr float kLn2 = 0.6931471805599453f;

__device__ __forceinline__ f32x16 mfma32(bf16x8 a, bf16x8 b, f32x16 c) {
    return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0);
}

__device__ __forceinline__ bf16x8 as_bf16x8(u32x4 v) { return __builtin_bit_cast(bf16x8, v); }
__device__ __forceinline__ u32x4 as_u32x4(bf16x8 v) { return __builtin_bit_cast(u32x4, v); }

// two fp32 -> packed bf16 pair, round to nearest even (one v_cvt_pk_bf16_f32)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi) {
    f32x2 f = {lo, hi};
    bf16x2 b = __builtin_convertvector(f, bf16x2);
    return __builtin_bit_cast(uint32_t, b);
}

// registers [first, first+8) of an accumulator tile as a bf16 MFMA operand
__device__ __forceinline__ bf16x8 acc_to_operand(const f32x16& c, int first) {
    u32x4 r;
    r[0] = pack_bf16(c[first + 0], c[first + 1]);
    r[1] = pack_bf16(c[first + 2], c[first + 3]);
    r[2] = pack_bf16(c[first + 4], c[first + 5]);
    r[3] = pack_bf16(c[first + 6], c[first + 7]);
    return as_bf16x8(r);
}

// Position of a 4-row group inside its 16-row block in the "operand order" used
// for transposed LDS tiles: [0-3, 8-11, 4-7, 12-15], so that lane half `hi`
// reads its 8 contraction slots {4*hi + e, 8 + 4*hi + e} as one 16-byte load at
// offset 8*hi.
__device__ __forceinline__ int operand_pos4(int group4) {  // group4 = row/4
    const int blk = group4 >> 2, q4 = group4 & 3;
    const int pb = (q4 == 1) ? 2 : (q4 == 2) ? 1 : q4;
    return 16 * blk + 4 * pb;
}

// value held by the same lane of the other 32-lane half of the wave (v_permlane32_swap)
__device__ __forceinline__ float xhalf(float x) {
    const uint32_t u = __builtin_bit_cast(uint32_t, x);
    // swaps the upper half of the first operand with the lower half of the second
    const auto r = __builtin_amdgcn_permlane32_swap(u, u, false, false);
    // r[0]: lanes 0-31 keep x, lanes 32-63 receive the lower half; r[1]: lanes 0-31 receive the upper half
    const uint32_t other = (__lane_id() < 32) ? r[1] : r[0];
    return __builtin_bit_cast(float, other);
}

// Transpose a 4 (rows) x 8 (cols) bf16 block held as four 16-byte row vectors
// into eight 8-byte column vectors (4 rows each).
__device__ __forceinline__ void transpose4x8(const u32x4 (&row)[4], u32x2 (&col)[8]) {
#pragma unroll
    for (int w = 0; w < 4; ++w) {
        col[2 * w][0] = (row[0][w] & 0xffffu) | (row[1][w] << 16);
        col[2 * w][1] = (row[2][w] & 0xffffu) | (row[3][w] << 16);
        col[2 * w + 1][0] = (row[0][w] >> 16) | (row[1][w] & 0xffff0000u);
        col[2 * w + 1][1] = (row[2][w] >> 16) | (row[3][w] & 0xffff0000u);
    }
}

}  // namespace sp

// ---------------------------------------------------------------------------
// Unpadded, XOR-swizzled LDS tiles filled by direct global->LDS loads.
//
// A tile holds ROWS rows of D bf16 (D*2 bytes, CH = D/8 chunks of 16 bytes).
// Chunk c of row r is stored at chunk position c ^ swz<D>(r).  The swizzle is
// chosen so that both access patterns of the attention kernels are free of
// bank conflicts (64 banks x 4 bytes):
//   - row-major operand reads (ds_read_b128): 16 consecutive rows, same chunk;
//   - transposing reads (ds_read_b64_tr_b16): 4 consecutive rows (row % 4 = 0..3)
//     x 4 consecutive chunks per half-wave.
// ---------------------------------------------------------------------------
namespace sp {

template <int D>
__device__ __forceinline__ int swz(int row);
template <>
__device__ __forceinline__ int swz<128>(int row) { return ((row & 3) << 2) | ((row >> 2) & 3); }
template <>
__device__ __forceinline__ int swz<64>(int row) { return (((row >> 1) & 1) << 2) | ((row >> 2) & 3); }

#define SP_GPTR(p) ((const __attribute__((address_space(1))) void*)(p))
#define SP_LPTR(p) ((__attribute__((address_space(3))) void*)(p))

// One wave copies 1024 contiguous LDS bytes: lane l supplies the 16 global bytes
// that land at lds_base + 16*l (lds_base must be wave-uniform).
__device__ __forceinline__ void dma16(const void* gsrc, void* lds_base) {
    __builtin_amdgcn_global_load_lds(SP_GPTR(gsrc), SP_LPTR(lds_base), 16, 0, 0);
}

// All of this wave's outstanding global loads (register and LDS destinations) have landed.
__device__ __forceinline__ void wait_vmem() { asm volatile("s_waitcnt vmcnt(0)" ::: "memory"); }

typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

// Transposing LDS read: within each 16-lane block, lane i receives element i%4... see
// tile_dma_rows/tr_operand below for how the kernels use it.
__device__ __forceinline__ s16x4 lds_read_tr16(const void* p) {
    return __builtin_amdgcn_ds_read_tr16_b64_v4i16((s16x4 __attribute__((address_space(3)))*)(p));
}

// ---------------------------------------------------------------------------
// Hazard-proof build (-DSP_PADDED_MFMA): every assembly MFMA below is preceded by
// a full wait for outstanding LDS reads plus the two wait states a vector-ALU
// write needs before an MFMA reads it, and followed by the wait states after
// which any instruction may read its result; every partial LDS wait becomes a
// full one.  Every select on a lane mask is preceded by the wait states a
// mask needs between the compare that writes it and its use.  The arithmetic and its order are unchanged, so the padded build
// must give the regular build's bits: a test compares the two, which checks the
// hand-counted waits and instruction spacing of the regular build.
// ---------------------------------------------------------------------------
#ifdef SP_PADDED_MFMA
#define SP_MFMA_PRE "s_waitcnt lgkmcnt(0)\n\ts_nop 1\n\t"
#define SP_MFMA_POST "\n\ts_nop 15\n\ts_nop 7"
#define SP_MASK_PRE "s_nop 1\n\t"
#define SP_LGKM(N) 0
#else
#define SP_MFMA_PRE ""
#define SP_MFMA_POST ""
#define SP_MASK_PRE ""
#define SP_LGKM(N) (N)
#endif

// ---------------------------------------------------------------------------
// Asynchronous LDS operand reads with explicit waits.
//
// The compiler waits for ALL outstanding LDS reads before the first use of any
// of them; a software pipeline that keeps several operand reads in flight needs
// partial waits.  These helpers issue the read as opaque assembly (the compiler
// then tracks nothing) and lds_wait<N>(x) blocks until at most N younger LDS
// reads are outstanding, tying x to the wait so no use of x can be placed before
// it.  LDS reads of a wave complete in order, which makes the count exact.
// Rule: every value produced by lds_async_* must pass through lds_wait before
// it is used in any way, a register copy included: so such values never cross a
// control-flow join and are never packed into wider vectors before the wait.
// ---------------------------------------------------------------------------
__device__ __forceinline__ uint32_t lds_addr(const void* p) {
    return (uint32_t)(uintptr_t)(__attribute__((address_space(3))) const char*)(p);
}
template <int OFF>
__device__ __forceinline__ u32x4 lds_async_b128(uint32_t addr) {
    u32x4 r;
    asm volatile("ds_read_b128 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
    return r;
}
template <int OFF>
__device__ __forceinline__ u32x2 lds_async_tr16(uint32_t addr) {
    u32x2 r;
    asm volatile("ds_read_b64_tr_b16 %0, %1 offset:%2" : "=v"(r) : "v"(addr), "n"(OFF));
    return r;
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x4& x) {
    asm volatile("s_waitcnt lgkmcnt(%1)" : "+v"(x) : "n"(SP_LGKM(N)));
}
template <int N>
__device__ __forceinline__ void lds_wait(u32x2& x, u32x2& y) {
    asm volatile("s_waitcnt lgkmcnt(%2)" : "+v"(x), "+v"(y) : "n"(SP_LGKM(N)));
}

// ---------------------------------------------------------------------------
// Assembly MFMAs for the hand-scheduled backward kernels.
//
// In a kernel that may use more than 256 registers the compiler is free to put
// any MFMA accumulator into the accumulation registers, and does so even for
// tiles the vector ALU has to read and seed, paying a move per register each
// way; issued as assembly, the accumulator is constrained to the register file
// the kernel wants it in.  The compiler then no longer knows the instruction is
// an MFMA, so the caller owns the data hazards.  Those kernels run one wave per
// SIMD and are bound by how many instructions that lone wave can issue, so the
// helpers carry no padding in the regular build; the callers guarantee that
//   - no vector-ALU instruction writes an operand within the two instructions
//     before the MFMA (operands come from LDS reads, from earlier MFMAs, or from
//     arithmetic done at least one operand slot earlier);
//   - the vector ALU reads an MFMA's result only after enough later instructions
//     have issued to cover the MFMA's result latency, 8 passes for 32x32x16 and 4
//     for 16x16x32 (in the kernels: two independent MFMAs, or the vector-ALU chunk
//     of an earlier step);
//   - back-to-back MFMAs on the same accumulator are interlocked by hardware.
// MFMAs ignore the EXEC mask: code that contains them must only be skipped by a
// truly scalar branch, so every wave-uniform condition guarding such code has
// to be built from scalar values (readfirstlane anything loaded per lane).
// Volatile assembly statements keep their order, which is what orders an MFMA
// after the wait that covers its operands.  W >= 0: that wait rides in the same
// statement.
//   mfma_v  : accumulator in vector registers       mfma_vc : ... starting from another tile
//   mfma_a  : accumulator in accumulation registers
//   *_ab    : the B operand lives in accumulation registers (resident operands)
// (32x32x16; the forms of 16x16x32 are further down)
// ---------------------------------------------------------------------------
template <int W>
__device__ __forceinline__ void mfma_v(f32x16& acc, const u32x4& a, const bf16x8& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b));
}
template <int W>
__device__ __forceinline__ void mfma_v(f32x16& acc, const u32x4& a, const u32x4& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b));
}
__device__ __forceinline__ void mfma_vc(f32x16& acc, const u32x4& a, const bf16x8& b, const f32x16& c) {
    asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "v"(b), "v"(c));
}
__device__ __forceinline__ void mfma_vc(f32x16& acc, const u32x4& a, const u32x4& b, const f32x16& c) {
    asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "v"(b), "v"(c));
}
__device__ __forceinline__ void mfma_a(f32x16& acc, const u32x4& a, const u32x4& b) {
    asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+a"(acc) : "v"(a), "v"(b));
}
template <int W>
__device__ __forceinline__ void mfma_a_w(f32x16& acc, const u32x4& a, const u32x4& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+a"(acc) : "v"(a), "v"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+a"(acc) : "v"(a), "v"(b));
}
template <int W>
__device__ __forceinline__ void mfma_v_ab(f32x16& acc, const u32x4& a, const bf16x8& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "a"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "a"(b));
}
template <int W>
__device__ __forceinline__ void mfma_vc_ab(f32x16& acc, const u32x4& a, const bf16x8& b, const f32x16& c) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%4)\n\t" SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "a"(b), "v"(c), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_32x32x16_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "a"(b), "v"(c));
}
// x = the lane's bit of `lanes` ? -inf : x.  One select per register as assembly: written in C++, a run of selects on one
// flag becomes a branch around moves, and its copies of whole accumulator tiles took the dQ stage with one row block
// (packed documents) from 241 to 256 vector registers and moves between the register files.  The compiler does not see
// that the selects read a mask that a compare may just have written: two wait states, in a statement that hands the mask
// on, so that no select can be placed before it.
template <typename TILE>
__device__ __forceinline__ void select_hidden(TILE& x, uint64_t lanes) {
    const float hidden = -__builtin_inff();
#pragma unroll
    for (int r = 0; r < (int)(sizeof(TILE) / 4); ++r) {
        float v = x[r];
        asm(SP_MASK_PRE "v_cndmask_b32 %0, %0, %1, %2" : "+v"(v) : "v"(hidden), "s"(lanes));
        x[r] = v;
    }
}
template <typename TILE>
__device__ __forceinline__ void hide_lanes(TILE& x, uint64_t lanes) {
    asm("s_nop 1" : "+s"(lanes));
    select_hidden(x, lanes);
}
template <typename TILE>
__device__ __forceinline__ void hide_lanes(TILE& x, TILE& y, uint64_t lanes) {  // two tiles, one wait
    asm("s_nop 1" : "+s"(lanes));
    select_hidden(x, lanes);
    select_hidden(y, lanes);
}
// at most N of this wave's global loads (register and LDS destinations) are still in flight
template <int N>
__device__ __forceinline__ void vmem_wait() { asm volatile("s_waitcnt vmcnt(%0)" ::"n"(N) : "memory"); }
// Waits that tie the values they cover: used where the awaited registers are then combined into wider
// operands (the combination must not be scheduled before the wait).
template <int N>
__device__ __forceinline__ void lds_wait4(u32x4& a, u32x4& b, u32x4& c, u32x4& d) {
    asm volatile("s_waitcnt lgkmcnt(%4)" : "+v"(a), "+v"(b), "+v"(c), "+v"(d) : "n"(SP_LGKM(N)));
}
// ---------------------------------------------------------------------------
// v_mfma_f32_16x16x32_bf16: C[16x16] += A[16x32] * B[32x16] per wave.  With lane l, lo = l % 16, g = l / 16:
//   A operand: lane holds A[lo][8*g + e], e = 0..7;   B operand: lane holds B[8*g + e][lo]
//   C/D      : lane holds C[4*g + r][lo] in register r = 0..3
// Two C tiles (rows 0-15 and 16-31), rounded to bf16, are together an operand over a contraction index of 32 in the
// order {4*g + e, 16 + 4*g + e}, e = 0..3; the other operand follows that order with two transposing reads.
//
// Why this shape: the long kernels run at the clock that the board's power leaves them (1.65 to 2.0 of 2.4 GHz), so what
// counts is energy per product, and per product this shape moves half as many accumulator registers as 32x32x16.
// Register-only loops on random data, every unit busy: 32x32x16 1.78-1.81 PFLOP/s at 1.77 GHz, 16x16x32 2.00-2.06
// PFLOP/s at 2.07 GHz, 2.09 where each instruction keeps one operand of the one before (both shapes keep the matrix
// pipe 93 to 97 % busy; on zeros, at the full clock, both reach 2.4).
//
// The assembly forms follow the rules above.
// ---------------------------------------------------------------------------
__device__ __forceinline__ f32x4 mfma16(bf16x8 a, bf16x8 b, f32x4 c) {
    return __builtin_amdgcn_mfma_f32_16x16x32_bf16(a, b, c, 0, 0, 0);
}
template <int W, typename B>
__device__ __forceinline__ void mfma16_v(f32x4& acc, const u32x4& a, const B& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "v"(b));
}
template <int W, typename B>
__device__ __forceinline__ void mfma16_vc(f32x4& acc, const u32x4& a, const B& b, const f32x4& c) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%4)\n\t" SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "v"(b), "v"(c), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "v"(b), "v"(c));
}
template <int W, typename B>
__device__ __forceinline__ void mfma16_v_ab(f32x4& acc, const u32x4& a, const B& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "a"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+v"(acc) : "v"(a), "a"(b));
}
template <int W, typename B>
__device__ __forceinline__ void mfma16_vc_ab(f32x4& acc, const u32x4& a, const B& b, const f32x4& c) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%4)\n\t" SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "a"(b), "v"(c), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %3" SP_MFMA_POST : "=&v"(acc) : "v"(a), "a"(b), "v"(c));
}
template <int W>
__device__ __forceinline__ void mfma16_a(f32x4& acc, const u32x4& a, const u32x4& b) {
    if constexpr (W >= 0) asm volatile("s_waitcnt lgkmcnt(%3)\n\t" SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+a"(acc) : "v"(a), "v"(b), "n"(W));
    else asm volatile(SP_MFMA_PRE "v_mfma_f32_16x16x32_bf16 %0, %1, %2, %0" SP_MFMA_POST : "+a"(acc) : "v"(a), "v"(b));
}

// The swizzle of tiles read for these shapes: chunk c of row r at chunk position c ^ swz16<D>(r).  Free of bank
// conflicts for row-major operand reads (16 consecutive rows, same chunk) and for transposing reads (8 consecutive rows
// x 2 consecutive chunks per half-wave).  It depends on row % 16 only, so blocks of 16 rows are a constant apart.
template <int D>
__device__ __forceinline__ int swz16(int row) {
    return D == 128 ? ((row & 7) << 1) | ((row >> 3) & 1) : ((row & 6)) | ((row >> 3) & 1);
}
// Byte offset of the 16-byte operand chunk (row, chunk) in such a tile.
template <int D>
__device__ __forceinline__ int tile16_off_b128(int row, int chunk) {
    return row * (D * 2) + ((chunk ^ swz16<D>(row)) * 16);
}
// Byte offset that lane `lane` passes to the transposing read so that it receives rows 4*g .. 4*g+3 of column col0 + lo.
template <int D>
__device__ __forceinline__ int tile16_off_tr(int col0, int lane) {
    const int row = 4 * (lane >> 4) + ((lane >> 2) & 3), col = col0 + 4 * (lane & 3);
    return row * (D * 2) + (((col >> 3) ^ swz16<D>(row)) * 16) + (col & 7) * 2;
}

// Per-lane description of the DMA loads that fill one ROWS x D tile with NW waves.
// (NW waves).  Instruction i (0 .. ROWS*CH/64-1) covers 64/CH rows; wave w issues i = w, w+NW, ...
// `wave` must be wave-uniform in the scalar sense (readfirstlane) so that LDS
// destinations are scalar.  Global addresses are a scalar tile base plus a 32-bit
// per-lane byte offset (rows of a tile span far less than 4 GiB).
template <int D, int ROWS, int NW = 4, bool S16 = false>
struct TileDma {
    static constexpr int CH = D / 8;
    static constexpr int RPI = 64 / CH;             // rows per instruction
    static constexpr int N_INSTR = ROWS * CH / 64;  // per tile, all waves
    static constexpr int PER_WAVE = N_INSTR / NW;
    static_assert(N_INSTR % NW == 0, "tile must split evenly over the waves");
    int row[PER_WAVE];          // row inside the tile this lane fetches for its k-th instruction
    uint32_t chunk_b[PER_WAVE]; // byte offset of the (swizzled) chunk this lane fetches inside that row
    uint32_t stride_b;          // global row stride in bytes
    __device__ __forceinline__ void init(int wave, int lane, size_t row_stride_elems) {
        stride_b = (uint32_t)(row_stride_elems * 2);
#pragma unroll
        for (int k = 0; k < PER_WAVE; ++k) {
            const int i = wave + NW * k;
            row[k] = RPI * i + lane / CH;
            chunk_b[k] = (uint32_t)(((lane % CH) ^ (S16 ? swz16<D>(row[k]) : swz<D>(row[k]))) * 16);
        }
    }
    // The K-th of this wave's PER_WAVE loads for the tile whose first row is at `tile` (a scalar
    // address); rows past the tile-relative row `lim` re-read row `lim` (their values are never used
    // unmasked).  Branch-free, so it can sit inside software-pipelined code.
    template <int K>
    __device__ __forceinline__ void issue_one(const __bf16* tile, int lim, __bf16* lds, int wave) const {
        const int r = row[K] < lim ? row[K] : lim;
        dma16(reinterpret_cast<const char*>(tile) + ((uint32_t)r * stride_b + chunk_b[K]), lds + (wave + NW * K) * 512);
    }
    __device__ __forceinline__ void issue(const __bf16* tile, int lim, __bf16* lds, int wave) const {
        static_for<0, PER_WAVE>([&](auto K) { issue_one<decltype(K)::value>(tile, lim, lds, wave); });
    }
};

// Byte offset, inside a swizzled tile, of the 16-byte row-major operand chunk (row, chunk).
template <int D>
__device__ __forceinline__ int tile_off_b128(int row, int chunk) {
    return row * (D * 2) + ((chunk ^ swz<D>(row)) * 16);
}

// Byte offset this lane passes to the transposing read so that, together with the other
// lanes of its 16-lane block, it receives rows {row0 .. row0+3} of column (col0 + i) where i
// is its index in the block: lane i supplies row row0 + i/4, columns col0 + 4*(i%4) .. +3.
template <int D>
__device__ __forceinline__ int tile_off_tr(int row0, int col0, int i16) {
    const int row = row0 + (i16 >> 2);
    const int col = col0 + 4 * (i16 & 3);
    return row * (D * 2) + (((col >> 3) ^ swz<D>(row)) * 16) + (col & 7) * 2;
}

// Stores 32 result rows of D columns as bf16, from a transposed accumulator (lane = row lo, register r of block db =
// column 32*db + 8*(r/4) + 4*hi + r%4), through `buf`: 32 * D * 2 bytes of LDS that no other wave touches.  Straight
// from the registers a store instruction would write 16 bytes to each of 32 rows, an eighth of a cache line each; from
// LDS it writes whole rows, 1 KB per instruction.  16-byte chunk c of row r sits at position c ^ (r or r/2) of its row,
// which spreads both the 8-byte writes (32 rows, one chunk) and the 16-byte reads (whole rows) over the banks.
// address(row) is where row `row` (0 .. 31) goes; rows from `rows` on are left out.
template <int D, typename ADDR>
__device__ __forceinline__ void store_rows(const f32x16 (&acc)[D / 32], float scale, char* buf, int rows, ADDR&& address) {
    constexpr int CH = D / 8, RPI = 64 / CH;  // chunks per row, rows per store instruction
    const int lane = __lane_id(), lo = lane & 31, hi = lane >> 5;
    auto at = [](int row, int chunk) __attribute__((always_inline)) { return row * (D * 2) + ((chunk ^ ((D == 128 ? row : row >> 1) & (CH - 1))) * 16); };
#pragma unroll
    for (int db = 0; db < D / 32; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            u32x2 w;
            w[0] = pack_bf16(acc[db][4 * g + 0] * scale, acc[db][4 * g + 1] * scale);
            w[1] = pack_bf16(acc[db][4 * g + 2] * scale, acc[db][4 * g + 3] * scale);
            *reinterpret_cast<u32x2*>(buf + at(lo, 4 * db + g) + 8 * hi) = w;
        }
    asm volatile("" ::: "memory");  // LDS accesses of a wave execute in order: keeping the order is all it takes
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int row = RPI * i + lane / CH, chunk = lane % CH;
        const u32x4 v = *reinterpret_cast<const u32x4*>(buf + at(row, chunk));
        if (row < rows) *reinterpret_cast<u32x4*>(address(row) + 8 * chunk) = v;
    }
    asm volatile("" ::: "memory");
}

// The same for accumulators of 16x16x32: acc[rb][db] holds rows 16*rb + lo, columns 16*db + 4*g + r.
template <int D, typename ADDR>
__device__ __forceinline__ void store_rows16(const f32x4 (&acc0)[D / 16], const f32x4 (&acc1)[D / 16], float scale, char* buf, int rows, ADDR&& address) {
    constexpr int CH = D / 8, RPI = 64 / CH;  // chunks per row, rows per store instruction
    const int lane = __lane_id(), lo = lane & 15, g = lane >> 4;
    auto at = [](int row, int chunk) __attribute__((always_inline)) { return row * (D * 2) + ((chunk ^ ((D == 128 ? row : row >> 1) & (CH - 1))) * 16); };
#pragma unroll
    for (int rb = 0; rb < 2; ++rb)
#pragma unroll
        for (int db = 0; db < D / 16; ++db) {
            const f32x4& a = rb == 0 ? acc0[db] : acc1[db];
            u32x2 w;
            w[0] = pack_bf16(a[0] * scale, a[1] * scale);
            w[1] = pack_bf16(a[2] * scale, a[3] * scale);
            *reinterpret_cast<u32x2*>(buf + at(16 * rb + lo, 2 * db + (g >> 1)) + 8 * (g & 1)) = w;
        }
    asm volatile("" ::: "memory");  // LDS accesses of a wave execute in order: keeping the order is all it takes
#pragma unroll
    for (int i = 0; i < 32 / RPI; ++i) {
        const int row = RPI * i + lane / CH, chunk = lane % CH;
        const u32x4 v = *reinterpret_cast<const u32x4*>(buf + at(row, chunk));
        if (row < rows) *reinterpret_cast<u32x4*>(address(row) + 8 * chunk) = v;
    }
    asm volatile("" ::: "memory");
}

}  // namespace sp
