// Backward pass of the CLEAR local attention for gfx950 (bf16, head_dim 128; kernels_bf16_bwd_d64.hip compiles
// this file a second time for head_dim 64): dQ, dK, dV of Eq. 1 under the
// mask of Eq. 3, given dO and the per-row log-sum-exp the forward pass can return.  With
//   s_ij = q_i.k_j / sqrt(d),  p_ij = exp(s_ij - lse_i) for M_ij = 1 (else 0),  delta_i = dO_i . O_i,
//   dp_ij = dO_i . v_j,        ds_ij = p_ij (dp_ij - delta_i):
//   dQ_i = sum_j ds_ij k_j / sqrt(d),   dK_j = sum_i ds_ij q_i / sqrt(d),   dV_j = sum_i p_ij dO_i.
//
// One kernel template computes either half.  Its "rows" are the tokens whose gradient a workgroup
// produces (queries for dQ, keys for dK and dV), held one per lane as MFMA B operands like Q in the forward
// kernel; its "columns" are the tokens summed over, staged in LDS tiles exactly like K and V in the forward
// kernel, in tiles of 64 (the mask is symmetric, so the key tiles a query tile reaches
// are also the query tiles that reach a key tile at its place):
//   mode   rows      column tiles (C1 | C2)   S = C1 r1^T   dP = C2 r2^T   accumulators
//   dQ     queries   K | V                    K q^T         V dO^T         dQ += K^T dS
//   dK+dV  keys      Q | dO                   Q k^T         dO v^T         dK += Q^T dS, dV += dO^T P, from one S and one dP
// lse and delta belong to the query: a per-lane scalar for dQ, a per-column vector (staged next to the tile, by LDS-direct loads
// like the tile, in the form in which S and dP start from it: neg_lse, neg_delta) for dK and dV.  Text rows sum over every token: they are split along the columns into partial sums that a
// small kernel adds up, like the text-query rows of the forward pass; with one range of columns they store their gradients themselves.
// Both are formed by the dQ kernels on their way when they run before the dK / dV kernels (BwdParams::O given),
// otherwise by clear_bwd_delta_kernel.
//
// What bounds it: a 32 x 32 block is 24 (dQ) or 32 (dK + dV) matrix instructions of 32 cycles, each of which holds the SIMD's vector issue
// port for about 20 of them, and the vector work of the block fits into the rest only if it is spread evenly and is little:
// an operand's address is one of two lane offsets plus an immediate (planes, as in the forward kernel; rows of
// 256 bytes took an XOR per operand), lse and delta go in as the initial accumulators of S and dP (16 subtractions of delta less; lse was the
// addend of a multiply-add that is a multiplication now), blocks that are admitted whole take no mask, and P and dS are formed under the matrix
// instructions of the products between.
// 24 heads of 128 channels, 512 text tokens, 64 x 64 grid, r = 16, forward and backward, on one card: 557 -> 518 us; 128 x 128, 333 text tokens:
// 1 991 -> 1 858 us; 38 heads of 64 channels, 64 x 64: 489 -> 455 us.
// (S rounds at the size of lse from its first product on, where it used to grow to it.  Error of P from its exponent, emulated in fp32 at 128 channels:
// 3.1e-7 -> 6.2e-7 of itself for logits of deviation 1, 4.9e-7 -> 5.1e-7 for 2, 2.7e-6 -> 2.1e-6 for 12; P's rounding to bf16 is 1.7e-3, and the error of dQ, dK and
// dV against 64 bits is unchanged to 1e-4 of itself.)
// Matrix pipe busy 52 % (dQ) and 56 % (dK + dV) of the CUs' time in image rows at 512 x 512, 70 and 73 % in text rows, 57 % in the one launch at 64 x 64; no
// cycle lost to LDS bank conflicts in any of them.
#include <hip/hip_runtime.h>

#include "bf16_common.h"
#include "block_class.h"
#include "clear_internal.h"

#if CLEAR_HEAD_DIM == 64
// second compilation of this file: its own kernel and launcher names
#define clear_bwd_bf16_kernel clear_bwd_bf16_d64_kernel
#define clear_bwd_delta_kernel clear_bwd_delta_d64_kernel
#define clear_bwd_reduce_kernel clear_bwd_reduce_d64_kernel
#define clear_bwd_bf16_all_kernel clear_bwd_bf16_d64_all_kernel
#define launch_bf16_backward launch_bf16_d64_backward
#else
#define launch_bf16_backward launch_bf16_d128_backward
#endif

namespace clear {
namespace {

typedef __attribute__((ext_vector_type(4))) unsigned u32x4;

enum BwdMode : int { kBwdQ = 0, kBwdKV = 1 };
enum BwdPart : int { kPartQ = 0, kPartK = 1, kPartV = 2 };  // partial sums of the text rows, in this order in the workspace

constexpr int STATS_BYTES = TILE_KEYS * 2 * 4;                           // per staged tile: neg_lse and neg_delta of its 64 columns
constexpr int BWD_LDS_BYTES = NBUF * STAGE_BYTES + NBUF * TPS * STATS_BYTES;

// One workgroup of a backward launch: workgroup `bid` of `nblk`.
template <int MODE, bool LINROWS, int CODE>
__device__ __forceinline__ void clear_bwd_bf16_workgroup(const BwdParams& p, const int bid, const int nblk)
{
    constexpr int NWY = kBf16NWY, NWX = kBf16NWX, NW = NWY * NWX;
    constexpr int STAGERS = NW / 2;  // the waves take turns, half of them staging a whole stage
    constexpr bool COLSTAT = MODE != kBwdQ;  // lse / delta indexed by column
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // [NBUF][TPS][C1 tile | C2 tile], then the column statistics
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    float* const stats = (float*)(smem + NBUF * STAGE_BYTES);  // [NBUF][TPS][2][64]

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31;
    const int hh = lane >> 5;

    // ---- workgroup -> (batch*head, row tile[, column split]); XCD-aware like the forward kernel
    int vid;
    {
        const int xcd = bid & 7, idx = bid >> 3;
        const int q = nblk >> 3, rem = nblk & 7;
        vid = xcd * q + imin(xcd, rem) + idx;
    }
    int bh, rt, split = 0;
    if (LINROWS) {
        split = vid % p.n_splits;
        const int t = vid / p.n_splits;
        rt = t % p.n_tq_tiles;
        bh = t / p.n_tq_tiles;
    } else {
        rt = vid % p.n_q_tiles;
        if (p.qt_order) rt = ((const_int_ptr)p.qt_order)[rt];  // the order in which a head's row tiles are dealt out
        bh = vid / p.n_q_tiles;
    }
    // Image rows live on an rH x rW grid and image columns on a cH x cW grid; grid point (y, x) is image token
    // (y * stride + oy, x * stride + ox) of the raster.  Plain masks: both are the raster.  Strided mask: the
    // workgroup belongs to one residue class of its rows; queries of class c meet the keys of class c + (ry, rx),
    // so the columns of a key class are the queries of class c - (ry, rx).
    int stride = 1, r_oy = 0, r_ox = 0, c_oy = 0, c_ox = 0;
    int rH = p.gridH, rW = p.gridW, cH = p.gridH, cW = p.gridW;
    if (!LINROWS && CODE == kCodeFull) {
        const int cls = bh % p.n_classes;
        bh /= p.n_classes;
        stride = p.stride;
        r_oy = cls / stride;
        r_ox = cls % stride;
        const int dy = MODE == kBwdQ ? p.stride_ry : stride - p.stride_ry, dx = MODE == kBwdQ ? p.stride_rx : stride - p.stride_rx;
        c_oy = (r_oy + dy) % stride;
        c_ox = (r_ox + dx) % stride;
        rH = (p.gridH - r_oy + stride - 1) / stride;  // >= 1: the host requires gridH, gridW >= stride
        rW = (p.gridW - r_ox + stride - 1) / stride;
        cH = (p.gridH - c_oy + stride - 1) / stride;
        cW = (p.gridW - c_ox + stride - 1) / stride;
    }
    const int batch = bh / p.H, head = bh % p.H;
    auto head_of = [&](const void* ptr, const TensorStrides& st) { return (const __bf16*)ptr + batch * st.sb + head * st.sh; };
    const TensorStrides& r1s = MODE == kBwdQ ? p.qs : p.ks;
    const TensorStrides& r2s = MODE == kBwdQ ? p.dos : p.vs;
    const TensorStrides& c1s = MODE == kBwdQ ? p.ks : p.qs;
    const TensorStrides& c2s = MODE == kBwdQ ? p.vs : p.dos;
    const __bf16* const R1 = head_of(MODE == kBwdQ ? p.Q : p.K, r1s);
    const __bf16* const R2 = head_of(MODE == kBwdQ ? p.dO : p.V, r2s);
    const unsigned char* const C1 = (const unsigned char*)head_of(MODE == kBwdQ ? p.K : p.Q, c1s);
    const unsigned char* const C2 = (const unsigned char*)head_of(MODE == kBwdQ ? p.V : p.dO, c2s);
    const unsigned c1_pitch = (unsigned)c1s.sn * 2, c2_pitch = (unsigned)c2s.sn * 2;  // bytes from one token row to the next
    float* const neg_lse = p.neg_lse + (long long)bh * p.N;
    float* const neg_delta = p.neg_delta + (long long)bh * p.N;

    // ---- this wave's rows, and this lane's one among them.  What depends on the lane (row coordinates, token, validity,
    // the half of the wave) is worked out again from the hardware's lane count wherever it is needed (here, per masked
    // tile, in the epilogue) instead of being carried through the tile loop: the fused dK / dV kernel has no register
    // to spare there, and a value spilled to scratch memory costs, on its way back, a wait for every load in flight.
    int wy0 = 0, wx0 = 0, r0 = 0;
    bool wave_has_rows;
    if (LINROWS) {
        r0 = rt * (NW * 32) + wave * 32;
        wave_has_rows = r0 < p.n_text;
    } else {
        wy0 = (rt / p.n_qtx) * (NWY * kWaveQH) + (wave / NWX) * kWaveQH;
        wx0 = (rt % p.n_qtx) * (NWX * kWaveQW) + (wave % NWX) * kWaveQW;
        wave_has_rows = wy0 < rH && wx0 < rW;
    }
    struct LaneRow {
        int hh, ry, rx, token;
        bool valid;
    };
    auto lane_row = [&]() {
        LaneRow L;
        const int ln = fresh_lane_id();
        const int q = ln & 31;
        L.hh = ln >> 5;
        L.ry = L.rx = 0;
        if (LINROWS) {
            L.token = r0 + q;
            L.valid = L.token < p.n_text;
            if (!L.valid) L.token = p.n_text - 1;
        } else {
            L.ry = wy0 + (q >> 3);
            L.rx = wx0 + (q & 7);
            L.valid = L.ry < rH && L.rx < rW;
            L.token = p.n_text + (imin(L.ry, rH - 1) * stride + r_oy) * p.gridW + imin(L.rx, rW - 1) * stride + r_ox;
        }
        return L;
    };
    const int r_token = lane_row().token;
    // B operands: KS contraction steps of 16 channels, this lane supplying channels 16 s + 8 hh .. + 7
    bf16x8 r1f[KS], r2f[KS];
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        r1f[s] = *(const bf16x8*)(R1 + (long long)r_token * r1s.sn + 8 * hh + 16 * s);
        r2f[s] = *(const bf16x8*)(R2 + (long long)r_token * r2s.sn + 8 * hh + 16 * s);
    }
    // dQ: what S and dP of this lane's query start from
    float s_from = 0.f, dp_from = 0.f;
    if (!COLSTAT) {
        if (p.O) {
            // delta of this lane's row from the dO fragments it holds and the matching pieces of its O row; the other half
            // of the row's channels sits 32 lanes away
            const __bf16* orow = head_of(p.O, p.os) + (long long)r_token * p.os.sn + 8 * (fresh_lane_id() >> 5);
            float part = 0.f;
#pragma unroll
            for (int s = 0; s < KS; ++s) {
                const bf16x8 o = *(const bf16x8*)(orow + 16 * s);
#pragma unroll
                for (int j = 0; j < 8; ++j) part += (float)o[j] * (float)r2f[s][j];
            }
            dp_from = -(part + __shfl_xor(part, 32, 64));
            s_from = p.lse[(long long)bh * p.N + r_token] * p.neg_inv_scale;
            const LaneRow own = lane_row();
            if (own.valid && own.hh == 0 && split == 0) {
                neg_lse[own.token] = s_from;
                neg_delta[own.token] = dp_from;
            }
        } else {
            s_from = neg_lse[r_token];
            dp_from = neg_delta[r_token];
        }
    }
#pragma unroll
    for (int s = 0; s < KS; ++s) {
        asm volatile("" : "+v"(r1f[s]));
        asm volatile("" : "+v"(r2f[s]));
    }
    asm volatile("" : "+v"(s_from), "+v"(dp_from));

    const const_int_ptr row_ptr = (const_int_ptr)p.row_ptr, col_idx = (const_int_ptr)p.col_idx, n_plain = (const_int_ptr)p.n_plain;
    const const_u64_ptr mask_tbl = (const_u64_ptr)p.mask_tbl;

    // ---- column tile list: tokens [lin_begin, lin_limit) in 64-token tiles, then (image rows) the CSR row:
    //   [0, cb1) whole linear tiles   [cb1, cb2) the ragged linear tile   [cb2, cb3) image tiles inside the grid
    //   [cb3, cb4) image tiles cut by the border
    int n_tiles, n_lin_tiles, csr_begin = 0;
    int lin_begin = 0, lin_limit = 0;
    if (LINROWS) {
        lin_begin = split * p.split_keys;
        lin_limit = (long long)lin_begin + p.split_keys < p.N ? lin_begin + p.split_keys : (int)p.N;
        n_lin_tiles = (lin_limit - lin_begin + TILE_KEYS - 1) / TILE_KEYS;
        n_tiles = n_lin_tiles;
    } else {
        lin_limit = p.n_text;
        n_lin_tiles = (p.n_text + TILE_KEYS - 1) / TILE_KEYS;
        csr_begin = row_ptr[rt];
        n_tiles = n_lin_tiles + (row_ptr[rt + 1] - csr_begin);
    }
    const int cb1 = (lin_limit - lin_begin) / TILE_KEYS, cb2 = n_lin_tiles;
    constexpr bool dense_image = !LINROWS && CODE == kCodeFull;  // strided: tiles inside the class grid need no mask
    const int cb3 = LINROWS ? n_lin_tiles : ((p.mask_tbl || dense_image) ? n_lin_tiles + n_plain[rt] : n_lin_tiles);
    const int cb4 = n_tiles;
    auto stage_len = [&](int t) {
        const int e = t < cb1 ? cb1 : (t < cb2 ? cb2 : (t < cb3 ? cb3 : cb4));
        return imin(TPS, e - t);
    };
    auto tile_origin = [&](int i, int& a, int& b) {  // linear -> (first token, -1); image -> (row, col) of the 8 x 8 tile
        if (i < n_lin_tiles) {
            a = lin_begin + i * TILE_KEYS;
            b = -1;
        } else {
            const int packed = col_idx[csr_begin + i - n_lin_tiles];
            a = packed >> 16;
            b = packed & 0xffff;
        }
    };
    auto slot_token = [&](int a, int b, int slot) {  // token staged in slot `slot` (0..63) of the tile with origin (a, b)
        if (b < 0) return imin(a + slot, lin_limit - 1);
        const int ky = imin(a + (slot >> 3), cH - 1);
        const int kx = imin(b + (slot & 7), cW - 1);
        return p.n_text + (ky * stride + c_oy) * p.gridW + kx * stride + c_ox;
    };

    // ---- staging: LDS-direct loads of the two column tiles (same layout and swizzle as K and V in the
    // forward kernel), and for dK / dV neg_lse and neg_delta of the tile's 64 queries (wave j of the first TPS waves
    // for tile j of the stage)
    // A staging wave takes 16 rows of both tiles, all their planes: one token address per tile.
    static_assert(STAGERS == TILE_KEYS / 16, "the waves that stage a tile cover its rows");
    auto issue_tile = [&](int i, unsigned lds_tile) {
        int a, b;
        tile_origin(i, a, b);
        // The lane's place in the tile is worked out again from the hardware's lane count: values kept in registers
        // since the kernel's start get spilled in the fused dK / dV kernel, and their reload from scratch memory would
        // wait for every load issued before it, the staged tile in front included.
        const int ln = fresh_lane_id();
        const int part = wave % STAGERS, row = 16 * part + (ln >> 2);
        const unsigned token = (unsigned)slot_token(a, b, row);
        const unsigned chunk_off = (unsigned)(((ln & 3) ^ plane_swz(row)) << 4);
        const unsigned o1 = token * c1_pitch + chunk_off, o2 = token * c2_pitch + chunk_off;
        auto load_plane = [&](auto pl_tag) __attribute__((always_inline)) {
            constexpr int pl = decltype(pl_tag)::value;
            load_to_lds_16B(C1, o1 + pl * 64, lds_tile + pl * PLANE_BYTES + part * 1024);
            load_to_lds_16B(C2, o2 + pl * 64, lds_tile + TILE_BYTES + pl * PLANE_BYTES + part * 1024);
        };
        static_for<NPLANE>(load_plane);
    };
    // Half of the waves stage a whole stage, the other half the next one (each SIMD holds one wave of either half): while
    // one wave of a SIMD stands at its load instructions the other one is already at its matrix products.
    int issue_turn = 0;
    auto issue_stage = [&](int t, int buf) {
        const int len = stage_len(t);
        const bool mine = wave / STAGERS == (issue_turn & 1);
        ++issue_turn;
#pragma unroll
        for (int j = 0; j < TPS; ++j)
            if (j < len && mine) issue_tile(t + j, lds_base + (unsigned)buf * STAGE_BYTES + (unsigned)j * (2 * TILE_BYTES));
        // (Not through registers: a value in flight there is one more to hold through the blocks, and where the allocator spilled it, the store
        // to scratch waited for the stage that had just been requested.)
        if (COLSTAT && wave < len) {
            int a, b;
            tile_origin(t + wave, a, b);
            const unsigned offset = 4 * (unsigned)slot_token(a, b, fresh_lane_id());
            const unsigned at = lds_base + NBUF * STAGE_BYTES + (unsigned)((buf * TPS + wave) * STATS_BYTES);
            load_to_lds_4B(neg_lse, offset, at);
            load_to_lds_4B(neg_delta, offset, at + TILE_KEYS * 4);
        }
    };

    // Lane offsets of the two operand reads, both below 2 KB, in one register: the dK / dV kernel of the square and Swin masks has no second one.
    const unsigned kv_lane = k_lane_offset(lane, 0) | v_lane_offset(lane, 0) << 16;

    f32x16 acc[NDB];  // gradient^T tiles: channel 32 db + 8 (reg / 4) + 4 hh + reg % 4 of this lane's row
    f32x16 acc_v[MODE == kBwdKV ? NDB : 1];  // keys: acc holds dK, acc_v holds dV
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            acc[db][r] = 0.f;
            if constexpr (MODE == kBwdKV) acc_v[db][r] = 0.f;
        }
    const float c = p.scale_log2e;

    // Both products that make P and dS start from what would be subtracted from them: S from -lse / scale and dP from -delta, so that
    // P = 2^(S c) and dS = P dP with no subtraction per pair.  dQ: lse and delta are the lane's own; keys: four 16-byte reads each.
    f32x16 s_init, dp_init;
    if (!COLSTAT) {
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            s_init[r] = s_from;
            dp_init[r] = dp_from;
        }
        asm volatile("" : "+v"(s_init), "+v"(dp_init));
    }
    struct Block {
        unsigned kb[2], vb[2];   // operand addresses of its tile pair
        const float* stats;      // of its tile
        MaskArgs ma;
    };

    // One 32-column block as a hand-ordered pipeline in the manner of the forward kernel: matrix instructions in program order, each LDS
    // operand read PD slots ahead of the instruction that takes it; two slots after a product's last instruction its results can be
    // read without a wait, and from there the vector work is dealt out two scores at a time:
    //   dQ:   slots [0, KS)    S = K q^T            keys:  slots [0, KS)    S = Q k^T
    //         next KS          dP = V dO^T                 next KS          dP = dO v^T
    //                                                      next 2 NDB       dV^T += dO^T P^T
    //         last 2 NDB       dQ^T += K^T dS^T            last 2 NDB       dK^T += Q^T dS^T
    // Keys at 128 channels: dS is taken from the probabilities as rounded to bf16 for the dV product, so that the fp32 ones need not live beside
    // dP (251 to 256 of 256 registers as it is).
    auto do_block = [&](auto mask_tag, auto blk_tag, const Block& b) __attribute__((always_inline)) {
        constexpr int MASK = decltype(mask_tag)::value, blk = decltype(blk_tag)::value;
        constexpr bool KV = MODE == kBwdKV, ROUNDED_P = KV && D == 128;
        constexpr int S_END = KS, DP_END = 2 * KS, DV_END = DP_END + (KV ? 2 * NDB : 0), NSLOT = DV_END + 2 * NDB;
        constexpr unsigned AT = blk * BLOCK_BYTES;
        auto operand = [&](int slot) {
            if (slot < S_END) return read_k(b.kb, slot, AT);
            if (slot < DP_END) return read_k(b.kb, slot - S_END, AT + TILE_BYTES);
            if (slot < DV_END) return read_v(b.vb, (slot - DP_END) / NDB, (slot - DP_END) % NDB, AT + TILE_BYTES);  // (consecutive instructions write different accumulators)
            return read_v(b.vb, (slot - DV_END) / NDB, (slot - DV_END) % NDB, AT);
        };
        constexpr int PD = 2, RING = KV && D == 128 ? PD + 1 : PD + 2;
        bf16x8 op[RING];
        const float* const st = b.stats + 32 * blk + 4 * (fresh_lane_id() >> 5);  // statistics of this lane's 16 columns: 4 groups of 4
        auto column_stats = [&](int offset) __attribute__((always_inline)) {
            f32x16 v;
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                const f32x4 w = *(const f32x4*)(st + offset + 8 * g);
#pragma unroll
                for (int u = 0; u < 4; ++u) v[4 * g + u] = w[u];
            }
            return v;
        };
        f32x16 sc = COLSTAT ? column_stats(0) : s_init, dp = dp_init;
#pragma unroll
        for (int i = 0; i < PD; ++i) op[i] = operand(i);
        bf16x8 pf[2], xf[2];
        MaskWords mw;
        auto p_pair = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 2 * i; r < 2 * i + 2; ++r) {
                sc[r] = __builtin_amdgcn_exp2f(sc[r] * c);
                if (KV) pf[r >> 3][r & 7] = (__bf16)sc[r];
            }
        };
        auto ds_pair = [&](int i) __attribute__((always_inline)) {
#pragma unroll
            for (int r = 2 * i; r < 2 * i + 2; ++r) {
                float pr = sc[r];
                if (ROUNDED_P) {  // back from the packed operand registers: an even element is the low half of its word
                    const unsigned w = __builtin_bit_cast(u32x4, pf[r >> 3])[(r & 7) >> 1];
                    pr = __builtin_bit_cast(float, (r & 1) ? (w & 0xffff0000u) : (w << 16));
                }
                xf[r >> 3][r & 7] = (__bf16)(pr * dp[r]);
            }
        };
        auto run_slot = [&](auto slot_tag) __attribute__((always_inline)) {
            constexpr int slot = decltype(slot_tag)::value;
            if (slot + PD < NSLOT) op[(slot + PD) % RING] = operand(slot + PD);
            if (MASK == kMaskTable && slot == 0 && b.ma.masked[blk]) {
#pragma unroll
                for (int r = 0; r < 16; ++r) mw.w[r] = b.ma.row[blk][r];
            }
            if (COLSTAT && slot == S_END - 2) dp = column_stats(TILE_KEYS);
            if (!KV && slot == DP_END) {
#pragma unroll
                for (int i = 0; i < 8; ++i) ds_pair(i);
            }
            if (slot < S_END)
                sc = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], r1f[slot], sc, 0, 0, 0);
            else if (slot < DP_END)
                dp = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], r2f[slot - S_END], dp, 0, 0, 0);
            else if (slot < DV_END) {
                constexpr int i = slot >= DP_END && slot < DV_END ? slot - DP_END : 0;
                if constexpr (KV) acc_v[i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], pf[i / NDB], acc_v[i % NDB], 0, 0, 0);
            } else {
                constexpr int i = slot >= DV_END ? slot - DV_END : 0;
                acc[i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], xf[i / NDB], acc[i % NDB], 0, 0, 0);
            }
            constexpr int WAIT = KS == 8 ? 2 : 1;
            if (slot == S_END + WAIT) {
                if (MASK == kMaskTable) {
                    if (b.ma.masked[blk]) mask_scores(sc, mw);
                } else {
                    apply_mask<MASK, CODE>(sc, blk, b.ma);
                }
            }
#pragma unroll
            for (int i = 0; i < 8; ++i) {
                // (dQ: all of P is due before the dS products, so it is done KS / 8 slots earlier per pair)
                if (slot == S_END + WAIT + (KV ? i * KS / 8 : i * (KS - WAIT) / 8)) p_pair(i);
                if (KV && slot == DP_END + WAIT + (KS == 8 && i > 0 ? 1 : 0) + i * KS / 8) ds_pair(i);
            }
            SCHED_FENCE();
        };
        static_for<NSLOT>(run_slot);
    };

    int pf_tile = 0;
    auto begin_stage = [&](int buf) {
        wait_vmcnt<0>();
        __syncthreads();
        if (pf_tile < n_tiles) {
            const int len = stage_len(pf_tile);
            issue_stage(pf_tile, buf ^ 1);
            pf_tile += len;
        }
    };
    const const_int_ptr wave_desc = (const_int_ptr)p.wave_desc;
    // Runs the reachable blocks of one staged tile.
    auto run_blocks = [&](auto mask_tag, bool run0, bool run1, const MaskArgs& ma, int buf, int j) __attribute__((always_inline)) {
        Block b;
        const unsigned tile_at = lds_base + (unsigned)buf * STAGE_BYTES + (unsigned)j * (2 * TILE_BYTES);
        unsigned kv = kv_lane;
        asm volatile("" : "+v"(kv));  // (taken apart here, not in front of the loop)
        b.kb[0] = tile_at + (kv & 0xffff);
        b.vb[0] = tile_at + (kv >> 16);
        b.kb[1] = b.kb[0] ^ K_LANE_ODD;
        b.vb[1] = b.vb[0] ^ V_LANE_ODD;
        b.stats = stats + ((buf * TPS + j) * 2) * TILE_KEYS;
        b.ma = ma;
        if (run0) do_block(mask_tag, std::integral_constant<int, 0>{}, b);
        if (run1) do_block(mask_tag, std::integral_constant<int, 1>{}, b);
    };
    auto run_tile = [&](auto mask_tag, int t, int buf, int j) __attribute__((always_inline)) {
        if constexpr (decltype(mask_tag)::value == kMaskTable) {
            // image tiles inside the grid: what this wave does with the tile was worked out on the host (the mask-table
            // entries of its two blocks, the all-zeros entry for a block out of reach, or kWaveSkipsTile)
            const int d = wave_desc[(long long)(csr_begin + t - n_lin_tiles) * NW + wave];
            if (d == kWaveSkipsTile || !wave_has_rows) return;
            const int zeros = (2 * p.mask_ry + 1) * (2 * p.mask_rx + 1) + 1;
            const int i0 = d & 0xffff, i1 = (int)((unsigned)d >> 16);
            MaskArgs ma;
            ma.row[0] = mask_tbl + 16 * i0;
            ma.row[1] = mask_tbl + 16 * i1;
            ma.masked[0] = i0 != zeros - 1;  // (the entry in front of the all-zeros one is all ones)
            ma.masked[1] = i1 != zeros - 1;
            run_blocks(mask_tag, i0 != zeros, i1 != zeros, ma, buf, j);
            return;
        }
        int ta, tb;
        tile_origin(t, ta, tb);
        const bool linear = tb < 0;
        int cls0, cls1;
        if (!wave_has_rows) {
            cls0 = cls1 = kBlockSkip;
        } else if (linear) {
            cls0 = classify_linear_block(ta, 32, lin_limit);
            cls1 = classify_linear_block(ta + 32, 32, lin_limit);
        } else if (CODE == kCodeFull) {
            cls0 = classify_full_block(wy0, wx0, rH, rW, ta, tb, kKeyBlockH, kKeyBlockW, cH, cW);
            cls1 = classify_full_block(wy0, wx0, rH, rW, ta + kKeyBlockH, tb, kKeyBlockH, kKeyBlockW, cH, cW);
        } else if (CODE == kCodeDisc) {
            cls0 = classify_image_block(wy0, wx0, kWaveQH, kWaveQW, ta, tb, kKeyBlockH, kKeyBlockW, p.gridH, p.gridW, p.r2);
            cls1 = classify_image_block(wy0, wx0, kWaveQH, kWaveQW, ta + kKeyBlockH, tb, kKeyBlockH, kKeyBlockW, p.gridH, p.gridW, p.r2);
        } else {
            const MaskSpec spec = {p.mask_kind, p.mask_r, p.mask_shift};
            cls0 = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, ta, tb, kKeyBlockH, kKeyBlockW, p.gridH, p.gridW);
            cls1 = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, ta + kKeyBlockH, tb, kKeyBlockH, kKeyBlockW, p.gridH, p.gridW);
        }
        MaskArgs ma;
        const LaneRow tile_row = lane_row();
        ma.hh = tile_row.hh;
        ma.a = ta;
        ma.b = linear ? lin_limit : tb;
        ma.qy = tile_row.ry; ma.qx = tile_row.rx; ma.gridH = cH; ma.gridW = cW; ma.r2 = p.r2;
        ma.kind = p.mask_kind; ma.r = p.mask_r; ma.shift = p.mask_shift;
        run_blocks(mask_tag, cls0 != kBlockSkip, cls1 != kBlockSkip, ma, buf, j);
    };
    auto run_category = [&](auto mask_tag, int& t, int end, int& buf) __attribute__((always_inline)) {
        for (; t < end; t += TPS, buf ^= 1) {
            begin_stage(buf);
#pragma unroll 1
            for (int j = 0; j < imin(TPS, end - t); ++j) run_tile(mask_tag, t + j, buf, j);
        }
        t = end;
    };

    // prologue: the first stage is in flight
    if (n_tiles > 0) {
        pf_tile = stage_len(0);
        issue_stage(0, 0);
    }
    int buf = 0, t = 0;
    run_category(std::integral_constant<int, kMaskNone>{}, t, cb1, buf);
    run_category(std::integral_constant<int, kMaskLinear>{}, t, cb2, buf);
    if (!LINROWS) {
        if constexpr (dense_image)
            run_category(std::integral_constant<int, kMaskNone>{}, t, cb3, buf);
        else
            run_category(std::integral_constant<int, kMaskTable>{}, t, cb3, buf);
        run_category(std::integral_constant<int, kMaskImage>{}, t, cb4, buf);
    }
    // ---- epilogue
    const LaneRow out_row = lane_row();
    if (!out_row.valid) return;
    const int out_token = out_row.token, out_hh = out_row.hh;
    const float out_scale = p.scale;  // dQ and dK carry the 1 / sqrt(d) of the logits
    if (LINROWS && p.n_splits > 1) {
        // partial sums of this column split: [mode][bh][split][row][d] fp32 (one range of columns is the whole sum: stored below)
        constexpr int slot0 = MODE == kBwdKV ? kPartK : kPartQ;
        float* wo = p.ws + ((((long long)slot0 * p.B * p.H + bh) * p.n_splits + split) * p.n_text + out_token) * D;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 v = {acc[db][4 * g] * out_scale, acc[db][4 * g + 1] * out_scale, acc[db][4 * g + 2] * out_scale, acc[db][4 * g + 3] * out_scale};
                *(f32x4*)(wo + 32 * db + 8 * g + 4 * out_hh) = v;
            }
        if constexpr (MODE == kBwdKV) {
            float* wv = p.ws + ((((long long)kPartV * p.B * p.H + bh) * p.n_splits + split) * p.n_text + out_token) * D;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v = {acc_v[db][4 * g], acc_v[db][4 * g + 1], acc_v[db][4 * g + 2], acc_v[db][4 * g + 3]};
                    *(f32x4*)(wv + 32 * db + 8 * g + 4 * out_hh) = v;
                }
        }
    } else {
        const TensorStrides& outs = MODE == kBwdQ ? p.dqs : p.dks;
        __bf16* orow = (__bf16*)(MODE == kBwdQ ? p.dQ : p.dK) + batch * outs.sb + head * outs.sh + (long long)out_token * outs.sn;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                bf16x4 v;
#pragma unroll
                for (int u = 0; u < 4; ++u) v[u] = (__bf16)(acc[db][4 * g + u] * out_scale);
                *(bf16x4*)(orow + 32 * db + 8 * g + 4 * out_hh) = v;
            }
        if constexpr (MODE == kBwdKV) {
            __bf16* vrow = (__bf16*)p.dV + batch * p.dvs.sb + head * p.dvs.sh + (long long)out_token * p.dvs.sn;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    bf16x4 v;
#pragma unroll
                    for (int u = 0; u < 4; ++u) v[u] = (__bf16)acc_v[db][4 * g + u];
                    *(bf16x4*)(vrow + 32 * db + 8 * g + 4 * out_hh) = v;
                }
        }
    }
}

template <int MODE, bool LINROWS, int CODE>
__global__ void __launch_bounds__(512, 1) clear_bwd_bf16_kernel(const BwdParams p)
{
    clear_bwd_bf16_workgroup<MODE, LINROWS, CODE>(p, (int)blockIdx.x, (int)gridDim.x);
}

// The four independent kernels of a backward pass in one launch of 2 n_image + 2 n_text_wgs workgroups, in one of two orders:
//   image rows first   dK and dV of the image keys, dQ of the image queries, dK and dV of the text keys, dQ of the text queries
//   p.text_first       dK and dV of the text keys, of the image keys, dQ of the text queries, of the image queries
// For problems of a few rounds of workgroups, where four launches, one after the other or on two streams, leave CUs idle between them, and
// where it is the kind that runs last that decides how evenly the CUs finish (choose_backward_shape, which states what that is
// worth).  (delta comes from clear_bwd_delta_kernel here.)
template <int CODE>
__global__ void __launch_bounds__(512, 1) clear_bwd_bf16_all_kernel(const BwdParams p, const int n_image, const int n_text_wgs)
{
    int bid = (int)blockIdx.x;
    bool text, kv;
    if (p.text_first) {
        kv = bid < n_text_wgs + n_image;
        if (!kv) bid -= n_text_wgs + n_image;
        text = bid < n_text_wgs;
        if (!text) bid -= n_text_wgs;
    } else {
        text = bid >= 2 * n_image;
        if (text) bid -= 2 * n_image;
        const int n = text ? n_text_wgs : n_image;
        kv = bid < n;
        if (!kv) bid -= n;
    }
    // Each kind reads its parameters for itself: read once for all four, they fill the scalar registers of every one of them (122 spilled
    // for the disc at 128 channels, now 10), and what is spilled takes vector registers that dK and dV need.  (The kernel's first argument
    // is at the start of its argument segment.)
    auto params = []() -> const BwdParams& {
        auto at = (const __attribute__((address_space(4))) BwdParams*)__builtin_amdgcn_kernarg_segment_ptr();
        asm volatile("" : "+s"(at));
        return *(const BwdParams*)at;
    };
    if (!text) {
        if (kv) return clear_bwd_bf16_workgroup<kBwdKV, false, CODE>(params(), bid, n_image);
        return clear_bwd_bf16_workgroup<kBwdQ, false, CODE>(params(), bid, n_image);
    }
    if (kv) return clear_bwd_bf16_workgroup<kBwdKV, true, kCodeDisc>(params(), bid, n_text_wgs);
    clear_bwd_bf16_workgroup<kBwdQ, true, kCodeDisc>(params(), bid, n_text_wgs);
}

// delta_i = dO_i . O_i for every row: D / 8 lanes per row (8 channels = 16 bytes each).  A workgroup takes 256 / CHUNKS
// neighbouring tokens of kDeltaHeads heads, so that a lane has 2 kDeltaHeads loads in flight and the head's place is
// uniform: with one row a lane, 64-bit divisions that found its place stood in front of its only two loads.  24 heads,
// 4 608 tokens, head_dim 128: 11.8 us, 4.8 TB/s.  With the reduction below, a training step's call 576 -> 564 us.
constexpr int kDeltaHeads = 4, kDeltaTokens = 256 / CHUNKS;
__global__ void __launch_bounds__(256) clear_bwd_delta_kernel(const __bf16* O, TensorStrides os, const __bf16* dO, TensorStrides dos, int H, int BH,
                                                              long long N, unsigned n_token_blocks, const float* lse, float neg_inv_scale, float* neg_lse, float* neg_delta)
{
    const long long t = (long long)(blockIdx.x % n_token_blocks) * kDeltaTokens + threadIdx.x / CHUNKS;
    const int bh0 = (int)(blockIdx.x / n_token_blocks) * kDeltaHeads;
    const int part = threadIdx.x % CHUNKS;
    const long long tc = t < N ? t : N - 1;
    const int n_heads = imin(kDeltaHeads, BH - bh0);
    bf16x8 o[kDeltaHeads], g[kDeltaHeads];
    float l[kDeltaHeads];
#pragma unroll
    for (int i = 0; i < kDeltaHeads; ++i) {
        if (i < n_heads) {
            const int b = (bh0 + i) / H, h = (bh0 + i) % H;
            o[i] = *(const bf16x8*)(O + b * os.sb + h * os.sh + tc * os.sn + 8 * part);
            g[i] = *(const bf16x8*)(dO + b * dos.sb + h * dos.sh + tc * dos.sn + 8 * part);
            l[i] = lse[(long long)(bh0 + i) * N + tc];
        }
    }
#pragma unroll
    for (int i = 0; i < kDeltaHeads; ++i) {
        if (i < n_heads) {
            float s = 0.f;
#pragma unroll
            for (int j = 0; j < 8; ++j) s += (float)o[i][j] * (float)g[i][j];
#pragma unroll
            for (int off = CHUNKS / 2; off > 0; off >>= 1) s += __shfl_xor(s, off, 64);
            if (t < N && part == 0) {
                neg_lse[(long long)(bh0 + i) * N + t] = l[i] * neg_inv_scale;
                neg_delta[(long long)(bh0 + i) * N + t] = -s;
            }
        }
    }
}

// Adds up the column-split partial sums of the text rows and stores them as bf16: 4 channels a thread, 1024 / D rows
// (mode, batch*head, text row) a workgroup.  Four partial sums are read at a time; they are added in the order of the splits.
// (One channel a thread and one row a workgroup before: 36 864 workgroups of 128 threads at 24 heads and 512 text tokens.)
constexpr int kReduceRows = 1024 / D;
__global__ void __launch_bounds__(256) clear_bwd_reduce_kernel(const BwdParams p)
{
    typedef __attribute__((ext_vector_type(4))) __bf16 bf16x4;
    const unsigned ch = 4 * (threadIdx.x % (D / 4));
    const long long BHn = (long long)p.B * p.H * p.n_text;
    const long long gr = (long long)blockIdx.x * kReduceRows + threadIdx.x / (D / 4);
    if (gr >= 3 * BHn) return;
    const int mode = gr >= 2 * BHn ? 2 : (gr >= BHn ? 1 : 0);
    const long long row = gr - mode * BHn;
    int bh, q;
    if (BHn <= 0x7fffffffLL) {  // (64-bit divisions are long)
        bh = (int)((unsigned)row / (unsigned)p.n_text);
        q = (int)((unsigned)row % (unsigned)p.n_text);
    } else {
        bh = (int)(row / p.n_text);
        q = (int)(row % p.n_text);
    }
    const float* part = p.ws + ((((long long)mode * p.B * p.H + bh) * p.n_splits) * p.n_text + q) * D + ch;
    const long long pitch = (long long)p.n_text * D;  // from one split to the next
    f32x4 s = {0.f, 0.f, 0.f, 0.f};
    int k = 0;
    for (; k + 4 <= p.n_splits; k += 4, part += 4 * pitch) {
        const f32x4 v0 = *(const f32x4*)part, v1 = *(const f32x4*)(part + pitch), v2 = *(const f32x4*)(part + 2 * pitch), v3 = *(const f32x4*)(part + 3 * pitch);
        s += v0;
        s += v1;
        s += v2;
        s += v3;
    }
    for (; k < p.n_splits; ++k, part += pitch) s += *(const f32x4*)part;
    __bf16* const out = (__bf16*)(mode == kPartQ ? p.dQ : (mode == kPartK ? p.dK : p.dV));
    const TensorStrides& st = mode == kPartQ ? p.dqs : (mode == kPartK ? p.dks : p.dvs);
    bf16x4 r;
#pragma unroll
    for (int j = 0; j < 4; ++j) r[j] = (__bf16)s[j];
    *(bf16x4*)(out + (bh / p.H) * st.sb + (bh % p.H) * st.sh + q * st.sn + ch) = r;
}

template <int MODE, bool LINROWS, int CODE>
hipError_t launch_bwd_code(const BwdParams& p, int nblk, hipStream_t stream)
{
    auto kern = clear_bwd_bf16_kernel<MODE, LINROWS, CODE>;
    static LdsLimitOnce lds_limit;  // one per kernel instantiation
    hipError_t e = lds_limit.ensure((const void*)kern, BWD_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(nblk), dim3(512), BWD_LDS_BYTES, stream, p);
    return hipGetLastError();
}

template <int CODE>
hipError_t launch_bwd_all(const BwdParams& p, int n_image, int n_text_wgs, hipStream_t stream)
{
    auto kern = clear_bwd_bf16_all_kernel<CODE>;
    static LdsLimitOnce lds_limit;  // one per kernel instantiation
    hipError_t e = lds_limit.ensure((const void*)kern, BWD_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(2 * n_image + 2 * n_text_wgs), dim3(512), BWD_LDS_BYTES, stream, p, n_image, n_text_wgs);
    return hipGetLastError();
}

// One kernel per family of image masks for the image rows; text rows meet every token and need none.
template <int MODE, bool LINROWS>
hipError_t launch_bwd(const BwdParams& p, int nblk, hipStream_t stream)
{
    if constexpr (LINROWS) {
        return launch_bwd_code<MODE, LINROWS, kCodeDisc>(p, nblk, stream);
    } else {
        const int code = mask_code_of(p.mask_kind);
        return code == kCodeDisc   ? launch_bwd_code<MODE, LINROWS, kCodeDisc>(p, nblk, stream)
               : code == kCodeFull ? launch_bwd_code<MODE, LINROWS, kCodeFull>(p, nblk, stream)
                                   : launch_bwd_code<MODE, LINROWS, kCodeGeneric>(p, nblk, stream);
    }
}

}  // namespace

hipError_t launch_bf16_backward(const BwdParams& p, const void* O, float* stats, hipStream_t stream, int phase)
{
    const int BH = p.B * p.H;
    const bool all = phase == kBwdPhaseAll;
    hipError_t e = hipSuccess;
    // (kBwdPhaseAll: no delta kernel; the dQ kernels form delta and run before the dK / dV kernels, which read it)
    if (phase == kBwdPhaseDelta) {
        const unsigned token_blocks = (unsigned)((p.N + kDeltaTokens - 1) / kDeltaTokens), head_blocks = (unsigned)((BH + kDeltaHeads - 1) / kDeltaHeads);
        hipLaunchKernelGGL(clear_bwd_delta_kernel, dim3(token_blocks * head_blocks), dim3(256), 0, stream, (const __bf16*)O, p.os, (const __bf16*)p.dO, p.dos, p.H, BH, p.N, token_blocks, p.lse, p.neg_inv_scale, stats, stats + BH * p.N);
        e = hipGetLastError();
    }
    const long long per_head = (long long)p.n_classes * p.n_q_tiles;
    if (phase == kBwdPhaseFour) {
        const int nlin4 = p.n_text > 0 ? BH * p.n_tq_tiles * p.n_splits : 0, nimg = (int)(BH * per_head);  // (64 image workgroups per CU at most)
        const int code = mask_code_of(p.mask_kind);
        return code == kCodeDisc   ? launch_bwd_all<kCodeDisc>(p, nimg, nlin4, stream)
               : code == kCodeFull ? launch_bwd_all<kCodeFull>(p, nimg, nlin4, stream)
                                   : launch_bwd_all<kCodeGeneric>(p, nimg, nlin4, stream);
    }
    const int nlin = p.n_text > 0 ? BH * p.n_tq_tiles * p.n_splits : 0;
    BwdParams pq = p;  // for the dQ kernels
    if (all) pq.O = O;
    auto shift = [&](BwdParams* q, int b, int h) {
        auto at = [&](const void* t, const TensorStrides& st) { return (const __bf16*)t + b * st.sb + h * st.sh; };
        const long long row = ((long long)b * p.H + h) * p.N;
        q->Q = at(p.Q, p.qs);
        q->K = at(p.K, p.ks);
        q->V = at(p.V, p.vs);
        q->dO = at(p.dO, p.dos);
        q->dQ = (void*)at(p.dQ, p.dqs);
        q->dK = (void*)at(p.dK, p.dks);
        q->dV = (void*)at(p.dV, p.dvs);
        if (q->O) q->O = at(q->O, p.os);
        q->lse = p.lse + row;
        q->neg_lse = p.neg_lse + row;
        q->neg_delta = p.neg_delta + row;
    };
    auto launch_image = [&](const BwdParams& params, auto mode_tag) {
        return launch_by_heads(params, per_head, 0xffffffffLL / 512, shift, [&](const BwdParams& q, int n) { return launch_bwd<decltype(mode_tag)::value, false>(q, n, stream); });
    };
    if (e == hipSuccess && (all || phase == kBwdPhaseImageQ)) e = launch_image(pq, std::integral_constant<int, kBwdQ>{});
    if (e == hipSuccess && nlin > 0 && (all || phase == kBwdPhaseTextQ)) e = launch_bwd<kBwdQ, true>(pq, nlin, stream);
    if (e == hipSuccess && (all || phase == kBwdPhaseImageKV)) {
        e = launch_image(p, std::integral_constant<int, kBwdKV>{});
    }
    if (e != hipSuccess || p.n_text == 0) return e;
    if (e == hipSuccess && (all || phase == kBwdPhaseTextKV)) {
        e = launch_bwd<kBwdKV, true>(p, nlin, stream);
    }
    if (e == hipSuccess && p.n_splits > 1 && (all || phase == kBwdPhaseReduce)) {
        hipLaunchKernelGGL(clear_bwd_reduce_kernel, dim3((unsigned)((3LL * BH * p.n_text + kReduceRows - 1) / kReduceRows)), dim3(256), 0, stream, p);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace clear
