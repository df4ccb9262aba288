// Device-side building blocks shared by the forward kernels of libbsfa.so (gfx950, wave64):
// element types and MFMA wrappers, the LDS tile layout with its direct HBM -> LDS copies,
// counters and barriers that leave those copies in flight, wave-level maxima, work decomposition.
#pragma once
#include "bsfa_internal.h"

#include <math.h>

#include <type_traits>
#include <utility>

namespace bsfa {

// The 16-bit element type of Q, K, V, P and O: bf16 or fp16 (the paper's kernel is fp16
// throughout, Section 5.1).  Same storage size, same MFMA shape, same LDS layout; only the
// matrix instruction, the pack and the pair sum differ.
template <bool F16> struct Elem;
template <> struct Elem<false> {
    typedef __bf16 T;
    typedef __bf16 x8 __attribute__((ext_vector_type(8)));
    typedef __bf16 x4 __attribute__((ext_vector_type(4)));
    typedef __bf16 x2 __attribute__((ext_vector_type(2)));
};
template <> struct Elem<true> {
    typedef _Float16 T;
    typedef _Float16 x8 __attribute__((ext_vector_type(8)));
    typedef _Float16 x4 __attribute__((ext_vector_type(4)));
    typedef _Float16 x2 __attribute__((ext_vector_type(2)));
};
typedef float f32x16 __attribute__((ext_vector_type(16)));
typedef __bf16 bf16x8_t __attribute__((ext_vector_type(8)));
typedef __bf16 bf16x2_t __attribute__((ext_vector_type(2)));
typedef _Float16 f16x8_t __attribute__((ext_vector_type(8)));
typedef _Float16 f16x2_t __attribute__((ext_vector_type(2)));
// 32x32x16 MFMA, fp32 accumulate, and p0 + p1 + acc on a packed pair: one overload per element type
__device__ __forceinline__ f32x16 mfma16(bf16x8_t a, bf16x8_t b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_bf16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ f32x16 mfma16(f16x8_t a, f16x8_t b, f32x16 c) { return __builtin_amdgcn_mfma_f32_32x32x16_f16(a, b, c, 0, 0, 0); }
__device__ __forceinline__ float pair_sum(bf16x2_t pp, float acc)
{
    const bf16x2_t ones = {(__bf16)1.0f, (__bf16)1.0f};
    return __builtin_amdgcn_fdot2_f32_bf16(pp, ones, acc, false);
}
__device__ __forceinline__ float pair_sum(f16x2_t pp, float acc)
{
    const f16x2_t ones = {(_Float16)1.0f, (_Float16)1.0f};
    return __builtin_amdgcn_fdot2(pp, ones, acc, false);
}
// 32x32x64 MFMA on fp8 (e4m3) operands, fp32 accumulate: a lane holds 32 consecutive bytes of the
// contraction dimension of its row (A) or column (B); block scales fixed at 2^0
typedef int i32x8 __attribute__((ext_vector_type(8)));
typedef int i32x4 __attribute__((ext_vector_type(4)));
__device__ __forceinline__ f32x16 mfma64_fp8(i32x8 a, i32x8 b, f32x16 c)
{
    return __builtin_amdgcn_mfma_scale_f32_32x32x64_f8f6f4(a, b, c, 0, 0, 0, 127, 0, 127);
}
// eight fp32 -> two dwords of fp8 (e4m3), round to nearest even
__device__ __forceinline__ void cvt8_fp8(const float (&f)[8], int &w0, int &w1)
{
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(f[0], f[1], 0, false);
    w0 = __builtin_amdgcn_cvt_pk_fp8_f32(f[2], f[3], w0, true);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(f[4], f[5], 0, false);
    w1 = __builtin_amdgcn_cvt_pk_fp8_f32(f[6], f[7], w1, true);
}
typedef short s16x4 __attribute__((ext_vector_type(4)));
typedef short s16x8 __attribute__((ext_vector_type(8)));

#define LDS_PTR(T, p) ((__attribute__((address_space(3))) T *)(uintptr_t)(p))
#define GLB_PTR(T, p) ((const __attribute__((address_space(1))) T *)(p))

// ---- LDS tile layout --------------------------------------------------------------------
// A tile is stored as units of 1024 bytes, what one direct copy instruction of a wave writes (64 lanes x 16 bytes, in
// lane order: the LDS side of a direct copy is linear), `pitch` bytes apart.  Of the tile's R rows, U units hold R / U
// rows each: unit u the rows u, u + U, u + 2U, ...  So
//     address(row, byte) = (row % U) * pitch + (row / U) * row_bytes + byte
// is a per-lane base plus a constant for every operand a wave reads: all gathers are one base register and immediate
// offsets.  The bytes a unit is longer than 1024 spread the rows that are read together over the banks: 16 for reads
// of 16 bytes per row (16 rows at a time), 32 and 64 for the transposing reads of V (4 rows x 32 bytes from two places
// 128 bytes apart at head_dim 128, 4 rows x 64 bytes at head_dim 64).
// (An XOR of the chunk index with the row spreads them as well, but costs a vector instruction per operand address:
// 14 a key block, and the registers for them.)
constexpr int kUnit = 1024;
constexpr int kPitch16 = kUnit + 16;                                   // K, transposed V, fp8 K
constexpr int v_pitch(int d) { return d == 128 ? kUnit + 32 : kUnit + 64; }   // V in place

// Byte offset (relative to the tile's first row) of the 16 bytes that a lane copies of unit `unit` of a tile of rows
// of D elements; a unit `n` further starts n rows further.
template <int D>
__device__ __forceinline__ uint32_t unit_src_offset(int unit, int lane, int stride_n)
{
    constexpr int CPR = D / 8;          // 16-byte chunks of a row; rows of a unit: 64 / CPR; units: D / 8
    return (uint32_t)((unit + (D / 8) * (lane / CPR)) * stride_n + 8 * (lane % CPR)) * 2u;
}

// Buffer descriptor of one tile: bytes at and beyond `bytes` are not read, their LDS bytes become 0.  That is all the
// last key block of a sequence needs that does not fill it: its absent keys are hidden from every real row by the
// causal mask and meet probabilities of 0 in the second product (Section 4.3's padding never shows).
constexpr uint32_t kWholeTile = 0x7fffffffu;                           // (a tile is shorter: see launch_forward)
__device__ __forceinline__ i32x4 tile_rsrc(const unsigned char *tile, uint32_t bytes)
{
    const uint64_t a = reinterpret_cast<uint64_t>(tile);
    return i32x4{(int)(uint32_t)a, (int)((uint32_t)(a >> 32) & 0xffffu), (int)bytes, 0x00020000};
}
// bytes of the first `rows` rows of a tile
template <int D> __device__ __forceinline__ uint32_t row_bytes(int rows, int stride_n) { return (uint32_t)((rows - 1) * stride_n + D) * 2u; }

// One unit of an asynchronous HBM -> LDS copy: each lane fetches 16 bytes, the hardware writes them at M0 + lane * 16.
// Repetition r of a wave's share of a tile goes to lds + r * LDS_STEP (lds: the wave's first unit) and is fetched `rep`
// bytes behind the one before; `off` is this lane's running offset.  The instruction is emitted through inline asm so
// that the compiler does not serialise every later LDS read behind all copies in flight: completion is tracked by
// vmcnt, which the kernel manages itself (wait_vmcnt).  The one wait state between a write of M0 and the load is the
// addition of `rep`, or a nop.
template <int R, int LDS_STEP>
__device__ __forceinline__ void unit_copy_async(uint32_t &off, uint32_t rep, i32x4 rsrc, uint32_t lds)
{
    const uint32_t dst = __builtin_amdgcn_readfirstlane(lds);
    if constexpr (R == 0)
        asm volatile("s_mov_b32 m0, %1\n\ts_nop 0\n\tbuffer_load_dwordx4 %0, %2, 0 offen lds" : : "v"(off), "s"(dst), "s"(rsrc) : "memory", "m0");
    else
        asm volatile("s_add_u32 m0, %1, %2\n\tv_add_u32 %0, %3, %0\n\tbuffer_load_dwordx4 %0, %4, 0 offen lds"
                     : "+v"(off) : "s"(dst), "n"(R * LDS_STEP), "s"(rep), "s"(rsrc) : "memory", "m0", "scc");
}

// s_waitcnt vmcnt(N) only (gfx9 encoding: vmcnt in bits 3:0 and 15:14, no wait on the others)
template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt range");
    __builtin_amdgcn_s_waitcnt((N & 15) | ((N >> 4) << 14) | 0x0F70);
}

// Workgroup barrier that orders LDS traffic only: the global -> LDS copies in flight are tracked
// separately with wait_vmcnt, so the barrier must not drain them.
__device__ __forceinline__ void wg_barrier()
{
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "workgroup", "local");
    __builtin_amdgcn_s_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "workgroup", "local");
}

// max over lanes l and l^32, result in both lanes.  v_permlane32_swap exchanges the upper half
// of its first operand with the lower half of its second: with two copies of x the first
// register ends up holding x[l & 31] and the second x[32 + (l & 31)] in every lane.  Written as
// one asm block so that the two copies are guaranteed to live in different registers.
__device__ __forceinline__ float pair_max(float x)
{
    float a = x, b;
    asm volatile("v_mov_b32 %1, %0\n\ts_nop 1\n\tv_permlane32_swap_b32 %0, %1\n\ts_nop 1\n\tv_max_f32 %0, %0, %1"
                 : "+v"(a), "=&v"(b));
    return a;
}

// max over the wave of a value that is already equal in lanes l and l^32 (wave-uniform result):
// four DPP steps inside each row of 16 lanes, then rows 0 and 1 are combined through SGPRs.
__device__ __forceinline__ float wave_max_paired(float x)
{
    asm volatile("s_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_max_f32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1"
                 : "+v"(x));
    const int xi = __builtin_bit_cast(int, x);
    return fmaxf(__builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 0)),
                 __builtin_bit_cast(float, __builtin_amdgcn_readlane(xi, 16)));
}

// The same scalar, unknown to the compiler.  Where both sides of a decision work on the accumulators, two one-sided
// branches on values it cannot relate keep every accumulator in its registers; as two sides of one branch (or threaded
// into one path with the next decision) they are given registers of their own, and hundreds are spilled.
template <class T> __device__ __forceinline__ T opaque(T x)
{
    asm("" : "+s"(x));
    return x;
}

// f(integral_constant<int, 0>) ... f(integral_constant<int, N - 1>), in order: a fully unrolled loop
// whose body sees its index as a constant expression
template <int... I, class F>
__device__ __forceinline__ void static_for_impl(std::integer_sequence<int, I...>, F &&f)
{
    (f(std::integral_constant<int, I>{}), ...);
}
template <int N, class F> __device__ __forceinline__ void static_for(F &&f)
{
    static_for_impl(std::make_integer_sequence<int, N>{}, f);
}
// the same for LO .. HI - 1
template <int LO, int HI, class F> __device__ __forceinline__ void static_range(F &&f)
{
    static_for<HI - LO>([&](auto n) { f(std::integral_constant<int, LO + decltype(n)::value>{}); });
}

// sum over the 16 lanes of a row (all other rows of the wave: zero or unused), wave-uniform
__device__ __forceinline__ int row_sum16(int x)
{
    asm volatile("s_nop 1\n\t"
                 "v_add_u32_dpp %0, %0, %0 quad_perm:[1,0,3,2] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_u32_dpp %0, %0, %0 quad_perm:[2,3,0,1] row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_u32_dpp %0, %0, %0 row_half_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1\n\t"
                 "v_add_u32_dpp %0, %0, %0 row_mirror row_mask:0xf bank_mask:0xf\n\ts_nop 1"
                 : "+v"(x));
    return __builtin_amdgcn_readlane(x, 0);
}

// Work decomposition: a work item is (batch b, KV head, group of HP query heads, QT query tiles from i on).
// With at least 8 (batch, KV head) pairs the pair is chosen by the low three bits of the
// workgroup id, which is the XCD the hardware dispatches the group to, so that all groups
// streaming one K/V sequence share one L2.  Heavy (late) query tiles first; which places the first workgroups share a
// CU in, turned_places says.
//
// Where batch elements have lengths of their own, only the work items that exist are counted off, late tiles first
// (the others follow, for their empty statistics): consecutive workgroups are dealt to the parts of an XCD in turn, and
// with gaps of a regular distance between them all of the longest element's late tiles fell to the same part (4 x up to
// 4000 tokens of 16 heads of width 64 over 8, heads in pairs: 107 us, 63 this way; 2 x up to 5000 of 32 heads: 166, 139).
// (Up to 256 workgroups, one to a CU, there is nothing to deal, and the counting takes half a microsecond: 4 x up to 54
// tokens of 28 heads over 4 9.2 us with, 8.7 without.  More than 16 pairs to an XCD do not fit a row of lanes.)
// With c the tiles of each pair, S(t) = sum of max(0, c - t) items lie in the rows of tiles from t up.  Item x is in row
// t = the last with S(t) > x; the pairs that row holds are those with S(c) <= x (a lane each), and with their number k
// S(t) = sum of their c - k t.
template <int HP, int QT, int ROWS, int PLACES>
__device__ __forceinline__ bool decode_work(const FwdParams &p, uint32_t w, int &b, int &g, int &h0, int &i, int &n_tok)
{
    const int pairs = p.batch * p.hkv;
    const int gsub = p.group / HP;               // head groups per KV head (HP: 1, 2 or 4)
    const int npx = pairs >= 8 ? (pairs + 7) >> 3 : pairs;                               // pairs of an XCD
    uint32_t v = pairs >= 8 ? w >> 3 : w;
    if constexpr (PLACES > 1) {                  // (selects: branches would put a load's way in front of the loads below)
        uint32_t to = p.turn[0] + p.turn[1] - 1 - v;
        if constexpr (PLACES > 2) to = v < p.turn[1] ? to : p.turn[1] + p.turn[2] - 1 - v;
        v = ((v >= p.turn[0]) & (v < p.turn[PLACES - 1])) ? to : v;
    }
    const int tiles = (p.mq + QT - 1) / QT;
    int pl, t;
    uint32_t sub;
    if (p.counted) {
        const int lane = threadIdx.x & 63, mine = pairs >= 8 ? (int)(w & 7) + 8 * lane : lane;
        const bool valid = lane < npx && mine < pairs;
        const int n = valid ? min(max(p.seqlens[p.div_hkv.of((uint32_t)mine)], 0), p.seqlen) : 0;
        int c = (n + ROWS - 1) / ROWS;
        const uint32_t item = p.div_gsub.of(v);
        sub = v - item * (uint32_t)gsub;
        int x = (int)item;
        const int total = row_sum16(c);
        const bool empty = x >= total;
        if (empty) {                             // the tiles beyond the elements' ends, in the same way
            x -= total;
            c = valid ? tiles - c : 0;
        }
        int above = 0;                           // S(c)
        for (int e = 0; e < npx; e += 4)
#pragma unroll
            for (int f = 0; f < 4; ++f) above += max(__builtin_amdgcn_readlane(c, e + f) - c, 0);
        const bool in_row = valid && above <= x;
        const int k = __builtin_popcountll(__builtin_amdgcn_ballot_w64(in_row)), sum = row_sum16(in_row ? c : 0);
        if (sum <= x) return false;              // (only where pairs do not fill the XCDs)
        t = counted_row(sum, x, k);
        const int at = x - (sum - k * (t + 1));  // which of the row's pairs: those longer than t, in order
        const bool longer = in_row && c > t;
        const uint64_t m = __builtin_amdgcn_ballot_w64(longer);
        const int before = (int)__builtin_amdgcn_mbcnt_lo((uint32_t)m, 0u);      // (at most 16 lanes)
        pl = __builtin_ctzll(__builtin_amdgcn_ballot_w64(longer && before == at));
        n_tok = __builtin_amdgcn_readlane(n, pl);
        if (empty) t = tiles - 1 - t;
    } else {
        const uint32_t idesc = p.div_tile.of(v), rest = v - idesc * (uint32_t)(npx * gsub);
        pl = (int)p.div_gsub.of(rest);
        sub = rest - (uint32_t)(pl * gsub);
        t = tiles - 1 - (int)idesc;
    }
    g = pairs >= 8 ? (int)(w & 7) + 8 * pl : pl;
    if (g >= pairs) return false;
    b = (int)p.div_hkv.of((uint32_t)g);
    if (!p.seqlens) n_tok = p.seqlen;
    else if (!p.counted) n_tok = min(max(__builtin_amdgcn_readfirstlane(p.seqlens[b]), 0), p.seqlen);
    g -= b * p.hkv;
    h0 = g * p.group + (int)sub * HP;
    i = t * QT;
    return true;
}

}  // namespace bsfa
