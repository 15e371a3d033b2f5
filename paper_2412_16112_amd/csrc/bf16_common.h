// Device-side building blocks shared by the bf16 kernels (forward and backward) for gfx950, head_dim
// CLEAR_HEAD_DIM (128 unless the including file sets 64):
// vector types, LDS-direct staging loads, the element masks of Eq. 3, the LDS layout of a staged 64-token tile and the MFMA
// operand reads from it (row-wise and transposed).
#pragma once
#include <hip/hip_runtime.h>

#include <mutex>
#include <type_traits>
#include <utility>

#include "block_class.h"
#include "clear_internal.h"

namespace clear {
namespace {

typedef __attribute__((ext_vector_type(8))) __bf16 bf16x8;
typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
typedef __attribute__((ext_vector_type(2))) __bf16 bf16x2;
typedef __attribute__((ext_vector_type(4))) short short4v;
typedef __attribute__((ext_vector_type(16))) float f32x16;
typedef __attribute__((ext_vector_type(4))) float f32x4;
typedef __attribute__((ext_vector_type(4), aligned(4))) float f32x4_any;  // in callers' fp32 tensors, which need only be 4-byte aligned

#ifndef CLEAR_HEAD_DIM
#define CLEAR_HEAD_DIM 128
#endif
constexpr int D = CLEAR_HEAD_DIM;    // head_dim
static_assert(D == 128 || D == 64, "row layout, swizzle and operand addresses are worked out for 128 and 64 channels");
constexpr int KS = D / 16;           // contraction steps of Q K^T (16 channels per matrix instruction)
constexpr int NDB = D / 32;          // 32-channel slices of O
constexpr int CHUNKS = D / 8;        // 16-byte chunks per token row
constexpr int ROW_BYTES = D * 2;     // one token row of K or V
constexpr int ROWS_PER_STORE = 1024 / ROW_BYTES;  // token rows a wave stores with 16 bytes per lane
constexpr int TILE_KEYS = kKeyTileKeys;
constexpr int TILE_BYTES = TILE_KEYS * ROW_BYTES;  // 16 KB for K, same for V
// How many matrix instructions ahead the forward block pipeline reads its LDS operands.  At 128 channels the image-query
// kernel sits at its 168-register limit (three waves per SIMD with the loading waves) and spills a few registers outside the loop of
// steps; a second slot ahead needs the fourth operand buffer.  (On the pipeline by 64-key tiles before this one two slots cost 4 % of the
// kernel's time in reloads of a query fragment.)  64 channels have the registers for two.
#ifndef CLEAR_OPERAND_PREFETCH
#if CLEAR_HEAD_DIM == 128
#define CLEAR_OPERAND_PREFETCH 1
#else
#define CLEAR_OPERAND_PREFETCH 2
#endif
#endif
#ifndef CLEAR_TILES_PER_STAGE
#define CLEAR_TILES_PER_STAGE 2
#endif
constexpr int TPS = CLEAR_TILES_PER_STAGE;           // key tiles (K + V = 32 KB each) staged per barrier
#ifndef CLEAR_NBUF
#define CLEAR_NBUF 2
#endif
constexpr int NBUF = CLEAR_NBUF;                     // stage buffers: one being computed on, the others being filled
constexpr int STAGE_BYTES = TPS * 2 * TILE_BYTES;
constexpr float FAST_SUM_LIMIT = 1.0e30f;  // the fast pass is discarded when a query's sums leave [0, 1e30)
constexpr float M_INIT = -1.0e30f;         // finite "no key seen yet" (keeps exp2 arguments free of inf - inf)

__device__ __forceinline__ float wave_pair_max(float x)
{
    // lanes l and l ^ 32 hold the two halves of one query's scores
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return fmaxf(__uint_as_float(r[0]), __uint_as_float(r[1]));
}

__device__ __forceinline__ float wave_pair_sum(float x)
{
    auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return __uint_as_float(r[0]) + __uint_as_float(r[1]);
}

// One 16-byte-per-lane load from global memory straight into LDS: the wave writes 1 KB starting at
// lds_addr (wave-uniform), lane i at lds_addr + 16 i; lane i reads gbase + voff.  Counted by vmcnt.
// Written as asm so that the compiler does not serialise later LDS reads behind it; the kernel waits
// with explicit s_waitcnt vmcnt before the barrier that publishes the tile.
// The compiler puts no wait states into asm, so they are written out: the load needs one after the write of M0 and five
// after a vector instruction that wrote its scalar base (v_readlane, where the base had been spilled), which may stand right in
// front of the asm: the write of M0 and four more.
__device__ __forceinline__ void load_to_lds_16B(const void* gbase, unsigned voff, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dwordx4 %1, %2" ::"s"(lds_addr), "v"(voff), "s"(gbase) : "memory", "m0");
}
// The same with 4 bytes per lane: 256 bytes starting at lds_addr.
__device__ __forceinline__ void load_to_lds_4B(const void* gbase, unsigned voff, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 3\n\tglobal_load_lds_dword %1, %2" ::"s"(lds_addr), "v"(voff), "s"(gbase) : "memory", "m0");
}

// This lane's index in its wave from the hardware's lane count (two instructions, no register kept live for it).
__device__ __forceinline__ int fresh_lane_id()
{
    int l;
    asm volatile("v_mbcnt_lo_u32_b32 %0, -1, 0\n\tv_mbcnt_hi_u32_b32 %0, -1, %0" : "=v"(l));
    return l;
}

template <int N>
__device__ __forceinline__ void wait_vmcnt()
{
    static_assert(N >= 0 && N < 64, "vmcnt is 6 bits");
    __builtin_amdgcn_s_waitcnt((N & 0xF) | (7 << 4) | (15 << 8) | ((N >> 4) << 14));  // expcnt, lgkmcnt unconstrained
}

// Query/key prologue on 8 consecutive channels (4 rotary pairs) of one token, in fp32: RMS-norm gain, then
// the rotation by the sum of the row angle and the column angle (tables hold (cos, sin) per pair).
// g0, g1: this chunk's 8 gains; a0, a1 / b0, b1: its 8 floats of the token's row / column table rows.
__device__ __forceinline__ void prologue_chunk_values(float (&x)[8], float inv_rms, bool has_gain, const f32x4& g0, const f32x4& g1,
                                                      bool turn, const f32x4& a0, const f32x4& a1, const f32x4& b0, const f32x4& b1)
{
    if (has_gain) {
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            x[j] = x[j] * inv_rms * g0[j];
            x[4 + j] = x[4 + j] * inv_rms * g1[j];
        }
    }
    if (turn) {
        const float cy[4] = {a0[0], a0[2], a1[0], a1[2]}, sy[4] = {a0[1], a0[3], a1[1], a1[3]};
        const float cx[4] = {b0[0], b0[2], b1[0], b1[2]}, sx[4] = {b0[1], b0[3], b1[1], b1[3]};
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const float c = cy[t] * cx[t] - sy[t] * sx[t];
            const float s = sy[t] * cx[t] + cy[t] * sx[t];
            const float e = x[2 * t], o = x[2 * t + 1];
            x[2 * t] = c * e - s * o;
            x[2 * t + 1] = s * e + c * o;
        }
    }
}

struct WaveState {
    f32x16 oacc[NDB];  // O^T tiles: channel 32*db + 8*(reg/4) + 4*hh + reg%4 of this lane's query
    float m_run;     // running maximum, raw logits (may lag the true maximum by < 2^8 in the exponent)
    float l_run;     // this lane's share of the denominator
    float c;         // log2(e) / sqrt(head_dim)
};

enum MaskMode : int { kMaskNone = 0, kMaskLinear = 1, kMaskImage = 2, kMaskTable = 3 };

// Which family of image masks a kernel instance is compiled for.  The disc of Eq. 3 is the product path and
// gets a kernel of its own, so that the code of the compared masks (integer divisions per element for the
// Swin windows, strided token addresses) neither lengthens it nor shares its instruction cache.
enum MaskCode : int { kCodeDisc = 0, kCodeGeneric = 1, kCodeFull = 2 };
__host__ __device__ constexpr int mask_code_of(int mask_kind)
{
    return mask_kind == kMaskDisc ? kCodeDisc : (mask_kind == kMaskFull ? kCodeFull : kCodeGeneric);
}

// Read-only tables (tile lists, lane masks) are addressed through the constant address space so that
// they are fetched with scalar loads: wave-uniform, and not counted among the vector loads whose
// completion the tile prefetch waits on.
typedef const __attribute__((address_space(4))) int* const_int_ptr;
typedef const __attribute__((address_space(4))) unsigned long long* const_u64_ptr;
typedef const __attribute__((address_space(4))) unsigned* const_u32_ptr;

struct MaskArgs {
    int a, b;  // linear: first token of the tile, token limit; image: tile origin (row, col)
    int hh, qy, qx, gridH, gridW, r2;
    int kind, r, shift;    // MaskKind; for kinds other than the disc: radius / window size and Swin shift
    const_u64_ptr row[2];  // kMaskTable: 16 lane masks per key block (one per score register)
    bool masked[2];        // kMaskTable: whether they admit less than everything
};

// Lane masks of a block: 16 words, one per score register, kept in scalar registers from the block's S product to its
// exponentials.
struct MaskWords {
    unsigned long long w[16];
};
__device__ __forceinline__ void mask_scores(f32x16& s, const MaskWords& mw)
{
#pragma unroll
    for (int r = 0; r < 16; ++r) s[r] = __builtin_amdgcn_inverse_ballot_w64(mw.w[r]) ? s[r] : -INFINITY;
}

// Sets the scores of inadmissible (query, key) pairs of key block kb to -inf.  Register r of this lane
// is key slot 8*(r/4) + 4*hh + r%4 of the block (Eq. 3 for image keys; the token limit for linear tiles).
template <int MASK, int CODE>
__device__ __forceinline__ void apply_mask(f32x16& s, int kb, const MaskArgs& ma)
{
    if (MASK == kMaskLinear) {
        const int base = ma.a + 32 * kb + 4 * ma.hh;
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (base + 8 * (r >> 2) + (r & 3) >= ma.b) s[r] = -INFINITY;
    } else if (MASK == kMaskImage && CODE != kCodeDisc) {
        // The other local masks.  Square and Swin windows are products of a row condition and a column condition:
        // 4 + 4 tests per block instead of 16 pair tests (kCodeFull: only the grid's edge).
        const int ky0 = ma.a + kKeyBlockH * kb, kx0 = ma.b + 4 * ma.hh;
        bool row_ok[4], col_ok[4];
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int ky = ky0 + g, kx = kx0 + g;
            row_ok[g] = ky < ma.gridH && (CODE == kCodeFull || axis_admits(ma.kind, ma.r, ma.shift, ma.qy, ky));
            col_ok[g] = kx < ma.gridW && (CODE == kCodeFull || axis_admits(ma.kind, ma.r, ma.shift, ma.qx, kx));
        }
#pragma unroll
        for (int e = 0; e < 16; ++e) {
            const bool keep = row_ok[e >> 2] && col_ok[e & 3];
            s[e] = keep ? s[e] : -INFINITY;
        }
    } else if (MASK == kMaskImage) {
        const int ky0 = ma.a + kKeyBlockH * kb, kx0 = ma.b + 4 * ma.hh;
        int dx2[4];
#pragma unroll
        for (int t = 0; t < 4; ++t) {
            const int dx = kx0 + t - ma.qx;
            dx2[t] = (kx0 + t < ma.gridW) ? dx * dx : 0x7fffffff;  // columns beyond the grid never pass
        }
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            const int dy = ky0 + g - ma.qy;
            const int lim = (ky0 + g < ma.gridH) ? ma.r2 - dy * dy : 0;  // dx^2 must stay below lim
#pragma unroll
            for (int t = 0; t < 4; ++t)
                if (!(dx2[t] < lim)) s[4 * g + t] = -INFINITY;
        }
    }
}

// p = 2^{(s - m) c} for the 16 scores of one block; returns their sum; packs them as the B operand of P V.
__device__ __forceinline__ float exp_block(const f32x16& s, float c, float mc, bf16x8 (&pf)[2])
{
    float sum = 0.f;
#pragma unroll
    for (int r = 0; r < 16; ++r) {
        const float pv = __builtin_amdgcn_exp2f(__builtin_fmaf(s[r], c, -mc));
        sum += pv;
        pf[r >> 3][r & 7] = (__bf16)pv;
    }
    return sum;
}

__device__ __forceinline__ float max_block(const f32x16& s)
{
    float mx = fmaxf(s[0], s[1]);
#pragma unroll
    for (int r = 2; r < 16; ++r) mx = fmaxf(mx, s[r]);
    return mx;
}

typedef const __attribute__((address_space(3))) bf16x8* lds_bf16x8_ptr;
typedef __attribute__((address_space(3))) short4v* lds_short4_ptr;

// LDS layout of a staged tile (64 tokens x D channels): planes of 32 channels (64 bytes), each 64 rows x 64 bytes = 4 KB,
// filled by 1 KB load instructions of 16 rows x 64 bytes (lane i: slot i % 4 of row i / 4; four neighbouring lanes read 64
// contiguous bytes).  Inside a row of 64 bytes the 16-byte chunk q sits in slot q ^ plane_swz(row).  Both operand reads
// are then free of bank conflicts, and their addresses are one of two per-lane offsets plus a constant that fits
// the instruction: no address arithmetic per operand.
__device__ __forceinline__ int plane_swz(int row) { return (((row >> 2) & 1) << 1) | ((row >> 3) & 1); }
constexpr int PLANE_BYTES = TILE_KEYS * 64;
constexpr int NPLANE = D / 32;
constexpr int BLOCK_BYTES = 32 * 64;  // from the first 32-token block of a tile to the second, inside every plane
static_assert(NPLANE * PLANE_BYTES == TILE_BYTES, "a tile is NPLANE planes");

// Lane offsets of the two operand reads inside a block: [0] for even contraction steps / the first half of a step's keys, [1] for odd / the second.
__device__ __forceinline__ unsigned k_lane_offset(int lane, int e)
{
    const int qi = lane & 31, hh = lane >> 5;
    return (unsigned)((qi >> 4) * 1024 + (qi & 15) * 64 + (((2 * e + hh) ^ plane_swz(qi & 15)) << 4));
}
__device__ __forceinline__ unsigned v_lane_offset(int lane, int e)
{
    const int j = lane & 15, row = 4 * (lane >> 5) + (j >> 2) + 8 * e;
    return (unsigned)(row * 64 + (((2 * ((lane >> 4) & 1) + ((j & 3) >> 1)) ^ plane_swz(row)) << 4) + 8 * (j & 1));
}
constexpr unsigned K_LANE_ODD = 32, V_LANE_ODD = 512 | 16;  // [1] is [0] with these bits turned over (block addresses are multiples of 1 KB)

// K operand, contraction step ks: chunk 2 ks + hh of key row qi.  `base`: lane offset for even / odd ks + block address.
// (extra: a constant byte offset on top, e.g. TILE_BYTES for the second tile of a staged pair)
__device__ __forceinline__ bf16x8 read_k(const unsigned (&base)[2], int ks, unsigned extra = 0)
{
    return *(lds_bf16x8_ptr)(size_t)(base[ks & 1] + (unsigned)((ks >> 1) * PLANE_BYTES) + extra);
}
// V^T operand for keys 16 s2 + 4 hh + {0..3} and 16 s2 + 8 + 4 hh + {0..3} of the block, channels 32 db .. 32 db + 31: two 16-bit
// transpose reads.  Within 16 lanes, lane j addresses row j / 4 and channels 4 (j % 4) .. + 3 of the group's 16-channel slice.
__device__ __forceinline__ bf16x8 read_v(const unsigned (&base)[2], int s2, int db, unsigned extra = 0)
{
    const unsigned imm = (unsigned)(db * PLANE_BYTES + s2 * 1024) + extra;
    union { struct { short4v lo, hi; } h; bf16x8 v; } u;
    u.h.lo = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(size_t)(base[0] + imm));
    u.h.hi = __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_short4_ptr)(size_t)(base[1] + imm));
    return u.v;
}

// Raises a kernel's dynamic-LDS limit once per device (function attributes belong to the device's copy of the
// kernel), safely from several host threads: one slot per kernel instantiation, which the caller keeps in a
// function-local static.
struct LdsLimitOnce {
    static constexpr int kDevices = 64;
    std::once_flag once[kDevices];
    hipError_t result[kDevices] = {};
    hipError_t ensure(const void* kernel, int bytes)
    {
        int dev = 0;
        hipError_t e = hipGetDevice(&dev);
        if (e != hipSuccess) return e;
        if (dev < 0 || dev >= kDevices) return hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes);
        std::call_once(once[dev], [&] { result[dev] = hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, bytes); });
        return result[dev];
    }
};

// Pins the instruction order: nothing is scheduled across this point.
#define SCHED_FENCE() __builtin_amdgcn_sched_barrier(0)

// f(integral_constant<int, 0>{}), ..., f(integral_constant<int, N - 1>{}), in order.
template <typename F, int... Is>
__device__ __forceinline__ void static_for_impl(F& f, std::integer_sequence<int, Is...>)
{
    (f(std::integral_constant<int, Is>{}), ...);
}
template <int N, typename F>
__device__ __forceinline__ void static_for(F& f)
{
    static_for_impl(f, std::make_integer_sequence<int, N>{});
}

}  // namespace
}  // namespace clear
