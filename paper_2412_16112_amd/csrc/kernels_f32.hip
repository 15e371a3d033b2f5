// fp32 path of the CLEAR local-attention forward pass (head_dim 64): fp32 matrix instructions (products and sums in
// fp32), exact online softmax (Eq. 1) over the keys the mask of Eq. 3 admits, on the tile schedule of the bf16 path.
//
// As in the bf16 kernels everything is computed transposed, so that a lane owns one query: S^T = K Q^T and O^T += V^T P^T
// on v_mfma_f32_16x16x4_f32.  A wave owns a 4 x 4 patch of queries (or 16 text queries), four lanes per query, and
// takes the keys in cells of 16 (4 x 4 image tokens, or 16 consecutive ones), of which it skips those out of its
// reach: 16 rather than 32 on a side because this path is bound by the fp32 matrix rate (1/16 of the bf16 one, so
// that operand reads from LDS and the vector work of the softmax hide behind it), and the smaller the patch and the
// cell, the fewer masked pairs are multiplied (r = 16: 1 150 keys per query for 793 admitted ones, 1 440 with 32).
//
// A workgroup is four waves and walks the text keys, then the image tiles of its schedule row that its own
// queries reach, staged in LDS half a tile at a time and double-buffered.  The waves hold 4, 2 or 1 patches (`groups` = 1,
// 2, 4 waves per patch): with several waves per patch each takes a share of every tile's cells and the partial softmax sums are joined
// in LDS at the end, which gives small problems as many workgroups as the chip has CUs and shorter key walks.
// A 38-head 64 x 64 grid with 333 text tokens, r = 16: 2.98 -> 0.72 ms
// (74 TFLOP/s of admitted pairs, 110 where nothing is masked; a large fp32 matrix product reaches 154); one head of 16 x 16
// tokens with 8 text tokens 0.43 ms -> 12 us.  (Before: vector arithmetic, a thread per query, the whole list of every
// 16 x 16 tile.  A single 32 KB stage per workgroup: 0.73 ms; two whole-tile stages, two workgroups per CU: 1.17 ms.)
#include <hip/hip_runtime.h>

#include <cfloat>

#include "bf16_common.h"
#include "block_class.h"
#include "clear_internal.h"

namespace clear {
namespace {

constexpr int HD = 64;                     // head_dim
constexpr int kWaves = 4;
constexpr int kCell = 16;  // keys per cell, queries per wave

// LDS rows are 256 bytes, one sweep over the banks, 16-byte chunks permuted: logical chunk c of row k sits in slot
// c ^ (k & 15).  The 16 rows of a K read (one chunk each) and the 4 rows x 64 bytes of a V read then use all banks once.
__device__ __forceinline__ int f32_swz(int row) { return row & 15; }

// 16 bytes per lane from global memory into LDS at lds_addr + 16 * lane (see load_to_lds_16B; 64-bit addresses, as a head
// of an fp32 context may exceed 4 GB).  One wait state after the write of M0; there is no scalar base to wait for.
__device__ __forceinline__ void load_to_lds_16B_far(const void* src, unsigned lds_addr)
{
    asm volatile("s_mov_b32 m0, %0\n\ts_nop 0\n\tglobal_load_lds_dwordx4 %1, off" ::"s"(lds_addr), "v"(src) : "memory", "m0");
}

// max / sum over the four lanes that share a query (lanes l, l ^ 16, l ^ 32, l ^ 48)
__device__ __forceinline__ float quad_max(float x)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return wave_pair_max(fmaxf(__uint_as_float(a[0]), __uint_as_float(a[1])));
}
__device__ __forceinline__ float quad_sum(float x)
{
    auto a = __builtin_amdgcn_permlane16_swap(__float_as_uint(x), __float_as_uint(x), false, false);
    return wave_pair_sum(__uint_as_float(a[0]) + __uint_as_float(a[1]));
}

typedef __attribute__((address_space(3))) const f32x4* lds_f32x4_ptr;
typedef __attribute__((address_space(3))) const float* lds_f32_ptr;

// DISC: the mask of Eq. 3 (its element test is a few instructions); otherwise whichever mask p.mask_kind names.
// CELLS: key cells per stage; half a tile (2, 32 KB of LDS for two stages: five workgroups per CU) unless four waves share a patch.
template <bool DISC, int CELLS>
__global__ void __launch_bounds__(kWaves * 64, CELLS == 2 ? 5 : 2) clear_fwd_f32_kernel(const FwdParams p, const int image_first, const int n_image)
{
    constexpr int STAGE_KEYS = CELLS * kCell, HALF_BYTES = STAGE_KEYS * HD * 4;
    constexpr int PARTS = TILE_KEYS / STAGE_KEYS, PART_H = kKeyTileH / PARTS;  // stages per key tile; rows of an image tile in one
    __shared__ __attribute__((aligned(1024))) unsigned char smem[2 * 2 * HALF_BYTES];  // [stage buffer][K | V]
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;
    const int lane = threadIdx.x & 63, qi = lane & 15, g = lane >> 4;
    const int wave = __builtin_amdgcn_readfirstlane(threadIdx.x >> 6);
    const int groups = p.f32_groups, patches = kWaves / groups;
    const int patch = wave / groups, group = wave % groups;

    // ---- workgroup -> (batch*head, query tile); image-query workgroups first, each XCD a contiguous range of either kind
    const bool textq = (int)blockIdx.x >= n_image;
    int vid;
    {
        const int bid = textq ? (int)blockIdx.x - n_image : (int)blockIdx.x, nblk = textq ? (int)gridDim.x - n_image : n_image;
        const int xcd = bid & 7, idx = bid >> 3, q = nblk >> 3, rem = nblk & 7;
        vid = (textq ? 0 : image_first) + xcd * q + imin(xcd, rem) + idx;
    }
    int bh, qt = 0, split = 0;
    int ty0 = 0, tx0 = 0, th = 0, tw = 0;  // image: the rectangle of queries of this workgroup
    int wy0 = 0, wx0 = 0, q0 = 0;  // first query of this wave
    bool wave_has_queries;
    if (textq) {
        split = vid % p.n_splits;
        const int t = vid / p.n_splits;
        bh = t / p.n_tq_tiles;
        q0 = (t % p.n_tq_tiles) * (patches * kCell) + patch * kCell;
        wave_has_queries = q0 < p.n_text;
    } else {
        // 16 x 16 query tiles of the schedule, cut into 8 x 8, 4 x 8 or 4 x 4 ones
        th = groups == 1 ? 8 : 4;
        tw = groups == 4 ? 4 : 8;
        const int sx = kF32QTileW / tw, subs = (kF32QTileH / th) * sx;
        const int sub = vid % subs, t = vid / subs;
        qt = p.qt_begin + t % p.n_q_tiles_launch;
        bh = t / p.n_q_tiles_launch;
        ty0 = (qt / p.n_qtx) * kF32QTileH + (sub / sx) * th;
        tx0 = (qt % p.n_qtx) * kF32QTileW + (sub % sx) * tw;
        if (ty0 >= p.gridH || tx0 >= p.gridW || ty0 >= p.own_y1 || ty0 + th <= p.own_y0) return;  // no query here
        wy0 = ty0 + 4 * (patch >> 1);
        wx0 = tx0 + 4 * (patch & 1);
        wave_has_queries = wy0 < p.gridH && wx0 < p.gridW;
    }
    auto query_token = [&](int i) -> long long {  // query i of this wave (a valid token also where there is none)
        if (textq) return imin(q0 + i, p.n_text - 1);
        return (long long)p.n_text + (long long)imin(wy0 + (i >> 2), p.gridH - 1) * p.gridW + imin(wx0 + (i & 3), p.gridW - 1);
    };
    const int qy = wy0 + (qi >> 2), qx = wx0 + (qi & 3);
    const long long head_off = (long long)bh * p.N * HD;
    const float* const Kh = (const float*)p.K + head_off;
    const float* const Vh = (const float*)p.V + head_off;

    // ---- stage list: the key range in stages of STAGE_KEYS tokens, then (image) the parts of the schedule row's tiles that
    // this workgroup reaches
    int n_lin, n_stages, csr_begin = 0;
    long long lin_begin = 0, lin_limit;
    const const_int_ptr row_ptr = (const_int_ptr)p.row_ptr, col_idx = (const_int_ptr)p.col_idx;
    if (textq) {
        lin_begin = (long long)split * p.split_keys;
        lin_limit = lin_begin + p.split_keys < p.NV ? lin_begin + p.split_keys : p.NV;
        n_stages = n_lin = (int)((lin_limit - lin_begin + STAGE_KEYS - 1) / STAGE_KEYS);
    } else {
        lin_limit = p.n_text;
        n_lin = (p.n_text + STAGE_KEYS - 1) / STAGE_KEYS;
        csr_begin = row_ptr[qt];
        n_stages = n_lin + (row_ptr[qt + 1] - csr_begin) * PARTS;
    }
    const MaskSpec spec = {DISC ? (int)kMaskDisc : p.mask_kind, p.mask_r, p.mask_shift};
    struct Stage {
        int i;     // index in the list; n_stages: the end
        int a, b;  // image: origin (row, col)
    };
    auto next_stage = [&](int i) {  // the first stage at or after i that holds a key for this workgroup
        Stage t = {i, 0, 0};
        for (; t.i < n_stages; ++t.i) {
            if (t.i < n_lin) break;
            const int e = t.i - n_lin, packed = col_idx[csr_begin + e / PARTS];
            t.a = (packed >> 16) + PART_H * (e % PARTS);
            t.b = packed & 0xffff;
            if (classify_image_block_spec(spec, ty0, tx0, th, tw, t.a, t.b, PART_H, kKeyTileW, p.gridH, p.gridW) != kBlockSkip) break;
        }
        return t;
    };
    // LDS row 16 c + i of a stage is key i of cell c: linear stages in token order, image stages as rows of two 4 x 4 cells
    auto issue_stage = [&](const Stage& t, int buf) {
        const unsigned dst = lds_base + (unsigned)buf * (2 * HALF_BYTES);
#pragma unroll
        for (int n = 0; n < STAGE_KEYS / 4 / kWaves; ++n) {
            const int ii = wave * (STAGE_KEYS / 4 / kWaves) + n;  // 1 KB = 4 rows per load instruction
            const int row = 4 * ii + g;
            long long token;
            if (t.i < n_lin) {
                token = lin_begin + (long long)t.i * STAGE_KEYS + row;
                token = token < lin_limit ? token : lin_limit - 1;
                if (textq && token >= p.vkeys_text) token += p.vshift;  // position in the key list -> token
            } else {
                const int c = row >> 4, i = row & 15;
                const int ky = imin(t.a + 4 * (c >> 1) + (i >> 2), p.gridH - 1), kx = imin(t.b + 4 * (c & 1) + (i & 3), p.gridW - 1);
                token = (long long)p.n_text + (long long)ky * p.gridW + kx;
            }
            const long long off = token * HD + 4 * (qi ^ f32_swz(row));
            load_to_lds_16B_far(Kh + off, dst + ii * 1024);
            load_to_lds_16B_far(Vh + off, dst + HALF_BYTES + ii * 1024);
        }
    };

    Stage cur = next_stage(0);
    if (cur.i < n_stages) issue_stage(cur, 0);

    // Q as B operand: contraction step 4 j + t takes channel 4 (4 j + g) + t from lane group g
    f32x4 qf[4];
#pragma unroll
    for (int j = 0; j < 4; ++j) qf[j] = *(const f32x4*)((const float*)p.Q + head_off + query_token(qi) * HD + 4 * (4 * j + g));

    const f32x4 zero = {0.f, 0.f, 0.f, 0.f};
    f32x4 o[4] = {zero, zero, zero, zero};  // channel 16 cb + 4 g + reg of this lane's query
    float m = -FLT_MAX, l = 0.f;            // running maximum (finite, so that no difference below is inf - inf); this lane's share of the sum
    const float sc = p.scale_log2e;
    // LDS addresses in cell 0 of stage buffer 0 (the other cells follow through the instructions' immediate offsets): chunk
    // 4 j + g of K row qi; channel 16 cb + qi of V row 4 g + t
    unsigned k_addr[4], v_addr[4][4];
#pragma unroll
    for (int j = 0; j < 4; ++j) k_addr[j] = lds_base + (unsigned)(qi * 256 + (((4 * j + g) ^ f32_swz(qi)) << 4));
#pragma unroll
    for (int t = 0; t < 4; ++t)
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
            v_addr[t][cb] = lds_base + (unsigned)(HALF_BYTES + (4 * g + t) * 256 + (((4 * cb + (qi >> 2)) ^ f32_swz(4 * g + t)) << 4) + (qi & 3) * 4);

    auto run_stage = [&](auto buf_tag, auto text_tag) __attribute__((always_inline)) {
        constexpr int buf = decltype(buf_tag)::value;
        constexpr bool TEXT = decltype(text_tag)::value;
        wait_vmcnt<0>();
        __syncthreads();  // the stage has landed, and everyone has left the other buffer
        const Stage nxt = next_stage(cur.i + 1);
        if (nxt.i < n_stages) issue_stage(nxt, buf ^ 1);
        const bool linear = TEXT || cur.i < n_lin;
        const long long lin_left = lin_limit - lin_begin - (long long)cur.i * STAGE_KEYS;  // keys of the range from this stage on
        const int left = lin_left < STAGE_KEYS ? (int)lin_left : STAGE_KEYS;
        const bool cut = cur.a + PART_H > p.gridH || cur.b + kKeyTileW > p.gridW;
        auto run_cell = [&](auto c_tag) __attribute__((always_inline)) {
            constexpr int c = decltype(c_tag)::value;
            if ((c & (groups - 1)) != group || !wave_has_queries) return;
            const int ky0 = cur.a + 4 * (c >> 1), kx0 = cur.b + 4 * (c & 1);
            const int cls = linear ? classify_linear_block(c * kCell, kCell, left)
                                   : classify_image_block_spec(spec, wy0, wx0, 4, 4, ky0, kx0, 4, 4, p.gridH, p.gridW);
            if (cls == kBlockSkip) return;
            constexpr unsigned at = buf * 2 * HALF_BYTES + c * kCell * 256;
            f32x4 k4[4], s = zero;
#pragma unroll
            for (int j = 0; j < 4; ++j) k4[j] = *(lds_f32x4_ptr)(size_t)(k_addr[j] + at);
#pragma unroll
            for (int j = 0; j < 4; ++j)
#pragma unroll
                for (int t = 0; t < 4; ++t) s = __builtin_amdgcn_mfma_f32_16x16x4f32(k4[j][t], qf[j][t], s, 0, 0, 0);
            // register t of lane group g is key 4 g + t of the cell
            if (cls == kBlockPartial) {
                if (linear) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) s[t] = c * kCell + 4 * g + t < left ? s[t] : -INFINITY;
                } else if (DISC) {
                    const int dy = ky0 + g - qy, dx0 = kx0 - qx;
                    const int lim = p.r2 - __mul24(dy, dy);  // dx^2 has to stay below this
#pragma unroll
                    for (int t = 0; t < 4; ++t) s[t] = __mul24(dx0 + t, dx0 + t) < lim ? s[t] : -INFINITY;
                } else {
#pragma unroll
                    for (int t = 0; t < 4; ++t) s[t] = mask_admits(spec, qy, qx, ky0 + g, kx0 + t) ? s[t] : -INFINITY;
                }
                if (cut && !linear) {
#pragma unroll
                    for (int t = 0; t < 4; ++t) s[t] = ky0 + g < p.gridH && kx0 + t < p.gridW ? s[t] : -INFINITY;
                }
            }
            const float mx = quad_max(fmaxf(fmaxf(s[0], s[1]), fmaxf(s[2], s[3])));
            if (__builtin_amdgcn_ballot_w64(mx > m) != 0) {  // some query of the wave has a new maximum
                const float m_new = fmaxf(m, mx), alpha = __builtin_amdgcn_exp2f((m - m_new) * sc);
                m = m_new;
                l *= alpha;
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) o[cb] *= alpha;
            }
            f32x4 pr;
#pragma unroll
            for (int t = 0; t < 4; ++t) pr[t] = __builtin_amdgcn_exp2f((s[t] - m) * sc);
            l += (pr[0] + pr[1]) + (pr[2] + pr[3]);
            if constexpr (TEXT) {
                // Over all the keys of a range a sum that takes a rounding per key loses more than the shorter walks of the image rows:
                // the cell's products are summed on their own and added in one step.  (38 heads, 64 x 64 grid, 333 text tokens, relative
                // error of the text rows against 64 bits: 8.6e-7 -> 6.5e-7; for image rows too it would be 7.6e-7 -> 5.5e-7 at 3 % of the time.)
                f32x4 oc[4] = {zero, zero, zero, zero};
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb)
                        oc[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(*(lds_f32_ptr)(size_t)(v_addr[t][cb] + at), pr[t], oc[cb], 0, 0, 0);
#pragma unroll
                for (int cb = 0; cb < 4; ++cb) o[cb] += oc[cb];
            } else {
#pragma unroll
                for (int t = 0; t < 4; ++t)
#pragma unroll
                    for (int cb = 0; cb < 4; ++cb)
                        o[cb] = __builtin_amdgcn_mfma_f32_16x16x4f32(*(lds_f32_ptr)(size_t)(v_addr[t][cb] + at), pr[t], o[cb], 0, 0, 0);
            }
        };
        static_for<CELLS>(run_cell);
        cur = nxt;
    };
    auto walk = [&](auto text_tag) __attribute__((always_inline)) {
        while (cur.i < n_stages) {
            run_stage(std::integral_constant<int, 0>{}, text_tag);
            if (cur.i >= n_stages) break;
            run_stage(std::integral_constant<int, 1>{}, text_tag);
        }
    };
    if (textq)
        walk(std::true_type{});
    else
        walk(std::false_type{});

    // (formed again rather than held through the walk)
    const int end_lane = fresh_lane_id(), end_qi = end_lane & 15, end_g = end_lane >> 4, end_qy = wy0 + (end_qi >> 2), end_qx = wx0 + (end_qi & 3);
    const long long q_token = query_token(end_qi);
    const bool q_valid = textq ? q0 + end_qi < p.n_text
                               : end_qy < p.gridH && end_qx < p.gridW && end_qy >= p.own_y0 && end_qy < p.own_y1;  // (row-band mode: owned rows only)
    l = quad_sum(l);
    if (groups > 1) {
        // join the partial sums of the waves that share a patch: wave by wave in LDS, 18 floats per lane
        __syncthreads();
        float* const mine = (float*)smem + wave * (18 * 64) + end_lane;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb)
#pragma unroll
            for (int t = 0; t < 4; ++t) mine[(4 * cb + t) * 64] = o[cb][t];
        mine[16 * 64] = m;
        mine[17 * 64] = l;
        __syncthreads();
        if (group != 0) return;
        for (int k = 1; k < groups; ++k) {
            const float* const other = mine + k * (18 * 64);
            const float mo = other[16 * 64], m_new = fmaxf(m, mo);
            const float wa = __builtin_amdgcn_exp2f((m - m_new) * sc), wb = __builtin_amdgcn_exp2f((mo - m_new) * sc);
            m = m_new;
            l = l * wa + other[17 * 64] * wb;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb)
#pragma unroll
                for (int t = 0; t < 4; ++t) o[cb][t] = o[cb][t] * wa + other[(4 * cb + t) * 64] * wb;
        }
    }
    // A masked pair is multiplied like the others, by a weight of zero: an infinity or NaN in V then reaches queries that do not see it.  Where a sum is
    // not finite, the wave goes through its keys once more, one by one, and leaves the masked ones out (maximum and sum of the weights stand).
    float finite = 0.f;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb)
#pragma unroll
        for (int t = 0; t < 4; ++t) finite += 0.f * o[cb][t];
    if (__builtin_amdgcn_ballot_w64(!(finite == 0.f)) != 0) {
        const float* const Qr = (const float*)p.Q + head_off + q_token * HD + 4 * end_g;  // this lane's channels, of Q, K and V: 16 cb + 4 g + reg
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) o[cb] = zero;
        auto visit = [&](long long token, bool admitted) {
            float s = 0.f;
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                const f32x4 a = *(const f32x4*)(Qr + 16 * cb), b = *(const f32x4*)(Kh + token * HD + 16 * cb + 4 * end_g);
#pragma unroll
                for (int t = 0; t < 4; ++t) s = __builtin_fmaf(a[t], b[t], s);
            }
            const float w = __builtin_amdgcn_exp2f((quad_sum(s) - m) * sc);
#pragma unroll
            for (int cb = 0; cb < 4; ++cb) {
                const f32x4 v = *(const f32x4*)(Vh + token * HD + 16 * cb + 4 * end_g);
#pragma unroll
                for (int t = 0; t < 4; ++t) o[cb][t] = admitted ? __builtin_fmaf(w, v[t], o[cb][t]) : o[cb][t];
            }
        };
#pragma unroll 1
        for (long long i = lin_begin; i < lin_limit; ++i) visit(textq && i >= p.vkeys_text ? i + p.vshift : i, true);
        if (!textq) {
            const int n_img = (n_stages - n_lin) / PARTS;
#pragma unroll 1
            for (int e = 0; e < n_img * TILE_KEYS; ++e) {
                const int packed = col_idx[csr_begin + e / TILE_KEYS], ky = (packed >> 16) + e % TILE_KEYS / kKeyTileW, kx = (packed & 0xffff) + e % kKeyTileW;
                if (ky >= p.gridH || kx >= p.gridW) continue;
                const bool admitted = mask_admits(spec, end_qy, end_qx, ky, kx);
                if (__builtin_amdgcn_ballot_w64(admitted) != 0) visit((long long)p.n_text + (long long)ky * p.gridW + kx, admitted);
            }
        }
    }
    if (!q_valid) return;
    if (textq && p.n_splits > 1) {
        const long long row = ((long long)bh * p.n_splits + split) * p.n_text + q_token;
#pragma unroll
        for (int cb = 0; cb < 4; ++cb) *(f32x4*)(p.ws_o + row * HD + 16 * cb + 4 * end_g) = o[cb];
        if (end_g == 0) {
            p.ws_ml[row * 2] = m;
            p.ws_ml[row * 2 + 1] = l;
        }
        return;
    }
    const float inv = 1.0f / l, lse = logf(l) + m * sc * 0.6931471805599453f;
    float* orow = (float*)p.O + head_off + q_token * HD;
    float* lse_out = p.lse ? p.lse + (long long)bh * p.N + q_token : nullptr;
    if (textq && p.band_o) {
        orow = p.band_o + ((long long)bh * p.n_text + q_token) * HD;
        lse_out = p.band_lse + (long long)bh * p.n_text + q_token;
    }
    if (lse_out && end_g == 0) *lse_out = lse;
#pragma unroll
    for (int cb = 0; cb < 4; ++cb) *(f32x4_any*)(orow + 16 * cb + 4 * end_g) = o[cb] * inv;
}

// Log-sum-exp combination of the key-split partial results of the text-query rows: 16 lanes per row, 4 channels each.
__global__ void __launch_bounds__(256) clear_text_merge_f32_kernel(const FwdParams p)
{
    const long long row = (long long)blockIdx.x * 16 + threadIdx.x / 16;
    if (row >= (long long)p.B * p.H * p.n_text) return;
    const int bh = (int)(row / p.n_text), q = (int)(row % p.n_text);
    const int ch = 4 * (threadIdx.x % 16);
    float m = -INFINITY;
    for (int s = 0; s < p.n_splits; ++s) m = fmaxf(m, p.ws_ml[(((long long)bh * p.n_splits + s) * p.n_text + q) * 2]);
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    for (int s = 0; s < p.n_splits; ++s) {
        const long long r = ((long long)bh * p.n_splits + s) * p.n_text + q;
        const float w = __builtin_amdgcn_exp2f((p.ws_ml[r * 2] - m) * p.scale_log2e);
        den += w * p.ws_ml[r * 2 + 1];
        num += w * *(const f32x4*)(p.ws_o + r * HD + ch);
    }
    const float lse = logf(den) + m * p.scale_log2e * 0.6931471805599453f;
    float* out = p.band_o ? p.band_o + row * HD : (float*)p.O + ((long long)bh * p.N + q) * HD;
    *(f32x4_any*)(out + ch) = num / den;
    if (ch == 0) {
        if (p.band_o)
            p.band_lse[row] = lse;
        else if (p.lse)
            p.lse[(long long)bh * p.N + q] = lse;
    }
}

}  // namespace

hipError_t launch_f32_d64(const FwdParams& p, hipStream_t stream, int phase)
{
    const int BH = p.B * p.H;
    hipError_t e = hipSuccess;
    const bool all = phase == kPhaseAll || phase == kPhaseImageAndTextQuery;
    const int subs = 4 * p.f32_groups;  // workgroups per 16 x 16 query tile
    const long long n_image = all || phase == kPhaseImage ? (long long)BH * p.n_q_tiles_launch * subs : 0;
    const long long n_text = p.n_text > 0 && (all || phase == kPhaseTextQuery) ? (long long)BH * p.n_tq_tiles * p.n_splits : 0;
    constexpr long long kMost = 0xffffffffLL / (kWaves * 64);  // workgroups a launch can have
    if (n_image > 0x7fffffffLL || n_text > kMost) return hipErrorInvalidConfiguration;
    const bool disc = p.mask_kind == kMaskDisc, wide = p.f32_groups == 4;
    auto kern = disc ? (wide ? clear_fwd_f32_kernel<true, 4> : clear_fwd_f32_kernel<true, 2>)
                     : (wide ? clear_fwd_f32_kernel<false, 4> : clear_fwd_f32_kernel<false, 2>);
    auto run = [&](long long first, long long n_img, long long n_txt) {
        if (n_img + n_txt == 0) return hipSuccess;
        hipLaunchKernelGGL(kern, dim3((unsigned)(n_img + n_txt)), dim3(kWaves * 64), 0, stream, p, (int)first, (int)n_img);
        return hipGetLastError();
    };
    long long first = 0;
    for (; e == hipSuccess && n_image - first + n_text > kMost; first += kMost < n_image - first ? kMost : n_image - first)  // (thin grids of many heads)
        e = run(first, kMost < n_image - first ? kMost : n_image - first, 0);
    if (e == hipSuccess) e = run(first, n_image - first, n_text);
    if (e != hipSuccess) return e;
    if (p.n_text > 0 && p.n_splits > 1 && (phase == kPhaseAll || phase == kPhaseTextMerge)) {
        hipLaunchKernelGGL(clear_text_merge_f32_kernel, dim3((unsigned)(((long long)BH * p.n_text + 15) / 16)), dim3(256), 0, stream, p);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace clear
