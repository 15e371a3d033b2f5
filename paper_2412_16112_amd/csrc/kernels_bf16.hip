// bf16 MFMA kernels for the CLEAR local-attention forward pass on gfx950 (head_dim 128; kernels_bf16_d64.hip
// compiles this file a second time for head_dim 64).
//
// Everything is computed "transposed" so that one lane owns one query for the whole pass:
//   S^T = K_blk * Q^T   (32 keys x 32 queries per MFMA tile, A = keys from LDS, B = queries in VGPRs)
//   O^T += V_blk^T * P^T (A = V read from LDS with the 16-bit transpose load, B = P^T straight from
//                         the S^T accumulators: the accumulator layout of one MFMA is the B-operand
//                         layout of the next, up to a fixed permutation of the contraction index
//                         that the V loads follow)
// With v_mfma_f32_32x32x16_bf16, lane l holds column n = l % 32 (its query) and rows
// 8*(reg/4) + 4*(l/32) + reg%4 of every 32 x 32 accumulator tile, so the row maximum and the
// softmax denominator of Eq. 1 need one exchange with lane l ^ 32 and no LDS round trip.
//
// A workgroup of 8 computing waves owns a 16 x 16 patch of image queries (or 256 text queries), 32 queries per wave, and
// walks a list of 64-key tiles: the text keys, then the 8 x 8 image key tiles its schedule row lists (Sec. 3.2: text
// keys for every query, image keys inside the radius-r disc).  K and V tiles are staged in LDS once per workgroup, by
// four further waves that do nothing else (one per SIMD, one stage ahead of the computing waves, one workgroup
// barrier per stage).
//
// Every computing wave follows a program of its own, made on the host (build_block_programs): one word per 32-key
// block its queries reach, with the block's place in the stage and its lane masks.  The blocks run as one software
// pipeline across stages and barriers: the S product of a block is issued together with the exponentials and the P V
// product of the block before it.
//
// What bounds it: for one or two rounds of workgroups, cycles - by the cost model of the launch shapes a workgroup takes about 16 000 and 900 a
// stage beside 520 for every block of a SIMD's two waves, 512 of them matrix cycles (16 instructions of 32) -; for large grids the chip's power
// budget, so bytes and instructions count there and waiting hardly does (order_forward_tiles: a third less L2 misses took 5 % of the
// time; 9 % fewer cycles of waiting took none).
// Against the version that worked by 64-key tiles inside a stage, with index arithmetic and masks per element at the grid's border,
// and a launch and a merge pass of its own for the text queries (24 heads, head_dim 128, 512 text tokens): 32 x 32 grid, r = 8:
// 48.6 -> 31.6 us; 64 x 64, r = 16: 132 -> 114 us; 512 x 512, r = 16: 8.00 -> 7.67 ms; 192 x 320, r = 32: 3.66 -> 3.46 ms.
#include <hip/hip_runtime.h>

#include "bf16_common.h"
#include "block_class.h"
#include "clear_internal.h"

#if CLEAR_HEAD_DIM == 64
// second compilation of this file: its own kernel and launcher names
#define clear_fwd_bf16_kernel clear_fwd_bf16_d64_kernel
#define clear_fwd_bf16_both_kernel clear_fwd_bf16_d64_both_kernel
#define clear_text_merge_kernel clear_text_merge_d64_kernel
#define launch_bf16 launch_bf16_d64
#else
#define launch_bf16 launch_bf16_d128
#endif

namespace clear {
namespace {

constexpr int NW = kBf16NWY * kBf16NWX;  // computing waves
constexpr int NLW = 4;                   // loading waves
constexpr int STAGE_HALF = TPS * TILE_BYTES;  // K (or V) of one stage: 32 KB
// K is double-buffered.  V is needed one block longer than K, past the barrier that ends its stage, and has three buffers:
// 160 KB together, all the LDS of a CU.
constexpr int NKBUF = 2, NVBUF = 3;
constexpr int FWD_LDS_BYTES = (NKBUF + NVBUF) * STAGE_HALF;
constexpr int FLAG_BYTES = 64;  // at the end of the LDS, used between passes only
constexpr int BLOCKS_PER_STAGE = 2 * TPS;

// Reference maximum of the fast pass: a query adopts the maximum of the first block in which it sees an
// admissible key (nothing has been accumulated for it before, so nothing needs rescaling) and keeps it:
// all later exponentials are taken relative to it, 2^{(s - m_ref) c}, whatever their size.  Whether that
// stayed within the range of fp32 is checked once, on the finished sums.
__device__ __forceinline__ void adopt_reference(WaveState& ws, float mx_pair)
{
    ws.m_run = (ws.m_run == M_INIT) ? fmaxf(mx_pair, M_INIT) : ws.m_run;
}

// One workgroup of a forward launch: workgroup `bid` of `nblk` (image-query rows, or with TEXTQ the text-query rows).
template <bool TEXTQ>
__device__ __forceinline__ void clear_fwd_bf16_workgroup(const FwdParams& p, const int bid, const int nblk)
{
    extern __shared__ __attribute__((aligned(1024))) unsigned char smem[];  // [NKBUF][TPS] K tiles, [NVBUF][TPS] V tiles
    const unsigned lds_base = (unsigned)(size_t)(__attribute__((address_space(3))) unsigned char*)smem;

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int qi = lane & 31;   // query slot inside the wave's patch
    const int hh = lane >> 5;   // which half of the contraction slice this lane feeds
    const bool loader = wave >= NW;

    // ---- workgroup -> (batch*head, query tile[, key split]); XCD-aware: workgroups are dealt
    // round-robin to the 8 XCDs, so give each XCD one contiguous range of the logical index.
    int vid;
    {
        const int xcd = bid & 7, idx = bid >> 3;
        const int q = nblk >> 3, rem = nblk & 7;
        vid = xcd * q + imin(xcd, rem) + idx;
    }
    int bh, qt, split = 0, variant = 0;
    // Image queries live on a qH x qW grid and their image keys on a kH x kW grid; grid point (y, x) is image
    // token (y * stride + oy, x * stride + ox) of the raster.  Plain masks: both are the raster itself.
    // Strided mask: the workgroup belongs to one residue class of the queries, (q_oy, q_ox) = (y % stride,
    // x % stride), and reads the keys of the class moved by (stride_ry, stride_rx); the wave programs come in four
    // variants, as the key class has the larger or the smaller extent on either axis.
    // Row bands may move the grid down by y_shift rows in these coordinates (so that a query tile starts at the first
    // owned row): grid rows then start at y_shift, and only where a token's address is formed is the shift taken off.
    const int stride = TEXTQ ? 1 : p.stride;
    int q_oy = 0, q_ox = 0, k_oy = 0, k_ox = 0;
    const int y_shift = TEXTQ ? 0 : p.y_shift;
    int qH = p.gridH + y_shift, qW = p.gridW, kH = qH, kW = qW;
    // `groups` waves share a patch of 32 queries and deal its key blocks out among themselves
    const int groups = TEXTQ ? p.tq_groups : p.groups, patches = NW / groups;
    const int patch = wave % patches, group = wave / patches;
    if (TEXTQ) {
        split = vid % p.n_splits;
        const int t = vid / p.n_splits;
        qt = t % p.n_tq_tiles;
        bh = t / p.n_tq_tiles;
    } else {
        qt = p.qt_begin + vid % p.n_q_tiles_launch;
        if (p.qt_order) qt = ((const_int_ptr)p.qt_order)[qt];  // the order in which a head's query tiles are dealt out
        bh = vid / p.n_q_tiles_launch;
        if (stride > 1) {
            const int cls = bh % p.n_classes;
            bh /= p.n_classes;
            q_oy = cls / stride;
            q_ox = cls % stride;
            k_oy = (q_oy + p.stride_ry) % stride;
            k_ox = (q_ox + p.stride_rx) % stride;
            qH = (p.gridH - q_oy + stride - 1) / stride;  // >= 1: the host requires gridH, gridW >= stride
            qW = (p.gridW - q_ox + stride - 1) / stride;
            kH = (p.gridH - k_oy + stride - 1) / stride;
            kW = (p.gridW - k_ox + stride - 1) / stride;
            variant = 2 * (kH > p.gridH / stride) + (kW > p.gridW / stride);
        }
    }
    const int batch = bh / p.H, head = bh % p.H;
    const __bf16* const Qh = (const __bf16*)p.Q + batch * p.qs.sb + head * p.qs.sh;

    // ---- stage list: the linear tiles (tokens [lin_begin, lin_limit), 64 a tile), then the image tiles of the CSR row, TPS to a
    // stage; linear and image tiles do not share a stage
    int n_lin_tiles, n_img_tiles = 0, csr_begin = 0;
    int lin_begin = 0, lin_limit = 0;
    if (TEXTQ) {
        lin_begin = split * p.split_keys;
        lin_limit = (long long)lin_begin + p.split_keys < p.NV ? lin_begin + p.split_keys : (int)p.NV;
    } else {
        const const_int_ptr row_ptr = (const_int_ptr)p.row_ptr;
        lin_limit = p.n_text;
        csr_begin = row_ptr[qt];
        n_img_tiles = row_ptr[qt + 1] - csr_begin;
    }
    n_lin_tiles = (lin_limit - lin_begin + TILE_KEYS - 1) / TILE_KEYS;
    const int n_lin_stages = (n_lin_tiles + TPS - 1) / TPS;
    const int n_stages = n_lin_stages + (n_img_tiles + TPS - 1) / TPS;

    unsigned* const flags = (unsigned*)(smem + FWD_LDS_BYTES - FLAG_BYTES);
    if (loader) {
        // A loading wave stays one stage ahead of the computing waves: after the barrier that hands stage s over, everyone has
        // left K of stage s - 1 and V of stage s - 2, whose buffers take stage s + 1.  It covers 16 rows of every tile.
        const int ldw = wave - NW;
        const unsigned char* const Kh = (const unsigned char*)((const __bf16*)p.K + batch * p.ks.sb + head * p.ks.sh);
        const unsigned char* const Vh = (const unsigned char*)((const __bf16*)p.V + batch * p.vs.sb + head * p.vs.sh);
        const unsigned k_pitch = (unsigned)p.ks.sn * 2, v_pitch = (unsigned)p.vs.sn * 2;  // bytes from one token row to the next
        const int row = 16 * ldw + (lane >> 2);
        const unsigned chunk_off = (unsigned)(((lane & 3) ^ plane_swz(row)) << 4);
        const const_int_ptr col_idx = (const_int_ptr)p.col_idx;
        auto issue_tile = [&](int token, unsigned k_tile, unsigned v_tile) __attribute__((always_inline)) {
            const unsigned ko = (unsigned)token * k_pitch + chunk_off, vo = (unsigned)token * v_pitch + chunk_off;
            auto load_plane = [&](auto pl_tag) __attribute__((always_inline)) {
                constexpr int pl = decltype(pl_tag)::value;
                load_to_lds_16B(Kh, ko + pl * 64, k_tile + pl * PLANE_BYTES + ldw * 1024);
                load_to_lds_16B(Vh, vo + pl * 64, v_tile + pl * PLANE_BYTES + ldw * 1024);
            };
            static_for<NPLANE>(load_plane);  // (not a loop: one that contains inline asm is not unrolled)
        };
        auto issue_stage = [&](int s, int kb, int vb) {
            auto load_tile = [&](auto j_tag) __attribute__((always_inline)) {
                constexpr int j = decltype(j_tag)::value;
                const unsigned k_tile = lds_base + (unsigned)(kb * STAGE_HALF + j * TILE_BYTES), v_tile = lds_base + (unsigned)((NKBUF + vb) * STAGE_HALF + j * TILE_BYTES);
                // addresses are clamped to valid tokens: slots beyond the range or the grid are masked in the compute
                if (s < n_lin_stages) {
                    const int i = s * TPS + j;
                    if (i >= n_lin_tiles) return;
                    int token = imin(lin_begin + i * TILE_KEYS + row, lin_limit - 1);
                    if (TEXTQ && token >= p.vkeys_text) token += p.vshift;  // position in the key list -> token
                    issue_tile(token, k_tile, v_tile);
                } else {
                    const int i = (s - n_lin_stages) * TPS + j;
                    if (i >= n_img_tiles) return;
                    const int packed = col_idx[csr_begin + i];  // tile origin, row << 16 | col
                    const int ky = imax(imin((packed >> 16) + (row >> 3), kH - 1) - y_shift, 0);  // (rows above the grid: out of every owned query's reach)
                    const int kx = imin((packed & 0xffff) + (row & 7), kW - 1);
                    issue_tile(p.n_text + (ky * stride + k_oy) * p.gridW + kx * stride + k_ox, k_tile, v_tile);
                }
            };
            static_for<TPS>(load_tile);
        };
        auto loader_pass = [&]() {
            int kb = 0, vb = 0;
            if (n_stages > 0) issue_stage(0, 0, 0);
            for (int s = 0; s < n_stages; ++s) {
                wait_vmcnt<0>();
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                kb ^= 1;
                vb = vb + 1 == NVBUF ? 0 : vb + 1;
                if (s + 1 < n_stages) issue_stage(s + 1, kb, vb);
            }
        };
        loader_pass();
        __syncthreads();
        __syncthreads();
        unsigned redo = 0;
#pragma unroll
        for (int i = 0; i < NW; ++i) redo |= flags[i];
        if (__builtin_amdgcn_readfirstlane(redo) != 0) {
            __syncthreads();
            loader_pass();
            __syncthreads();
        }
        if (groups > 1) __syncthreads();
        return;
    }

    // ---- this lane's query
    int wy0 = 0, wx0 = 0;  // origin of the wave's 4 x 8 query patch (image mode)
    int qy = 0, qx = 0;
    int q_token;
    bool q_valid, wave_has_queries;
    if (TEXTQ) {
        const int q0 = (qt * patches + patch) * kTextQueriesPerWave;
        q_token = q0 + qi;
        q_valid = q_token < p.n_text;
        wave_has_queries = q0 < p.n_text;
        if (!q_valid) q_token = p.n_text - 1;
    } else {
        wy0 = ((qt / p.n_qtx) * (patches / kBf16NWX) + patch / kBf16NWX) * kWaveQH;
        wx0 = (qt % p.n_qtx) * (kBf16NWX * kWaveQW) + (patch % kBf16NWX) * kWaveQW;
        qy = wy0 + (qi >> 3);
        qx = wx0 + (qi & 7);
        // (row-band mode: only the rows [own_y0, own_y1) carry queries; the halo rows are keys only)
        q_valid = qy < qH && qx < qW && qy >= p.own_y0 && qy < p.own_y1;
        wave_has_queries = wy0 < qH && wx0 < qW && wy0 < p.own_y1 && wy0 + kWaveQH > p.own_y0;
        q_token = p.n_text + (imax(imin(qy, qH - 1) - y_shift, 0) * stride + q_oy) * p.gridW + imin(qx, qW - 1) * stride + q_ox;
    }

    // Q^T as MFMA B operand: KS contraction steps of 16 channels; this lane supplies channels 16*s + 8*hh .. +7
    bf16x8 qf[KS];
    {
        const __bf16* qrow = Qh + (long long)q_token * p.qs.sn + 8 * hh;
#pragma unroll
        for (int s = 0; s < KS; ++s)  // (read once: non-temporal, so that the rows do not push K and V tiles out of the L2)
            qf[s] = __builtin_nontemporal_load((const bf16x8*)(qrow + 16 * s));
    }

    // ---- the wave's program.  Image-query rows: its own words.  Text-query rows: every stage but the last takes the same words again.
    // Scalar loads return out of order with LDS reads, so that a wait for an operand with one of them in flight waits for it too.  At 64 channels,
    // where a step is half as long, the words come in with a vector load, one to a lane, 64 at a time, and a step reads its own with
    // v_readlane (38 heads, 128 x 128: 461 -> 454 us); at 128 the second round trip at the start costs small calls more (32 x 32: 31.8 -> 32.6 us).
    constexpr bool LANE_WORDS = D == 64;
    constexpr int STAGE_KEYS = TPS * TILE_KEYS, TAIL = 32;  // (text: lanes from TAIL on hold the last stage's words)
    const const_u64_ptr mask_words = (const_u64_ptr)p.block_masks;
    const const_u32_ptr words = (const_u32_ptr)p.program;
    const unsigned per_stage = (unsigned)(BLOCKS_PER_STAGE / groups);
    unsigned pc_first, pc_tail = 0;            // where the program starts (text: and the words of the last stage)
    unsigned pc = 0, pc_wrap = ~0u, prog = 0;  // next word; where the text words start again; LANE_WORDS: lane i has word i of this 64
    const unsigned* next_words = nullptr;      // image, LANE_WORDS: the 64 words after those
    int whole_left = 0;                        // text: stages before the last one
    if (TEXTQ) {
        pc_first = p.text_words + (unsigned)(group * (STAGE_KEYS + 1)) * per_stage;
        pc_tail = pc_first + (unsigned)(lin_limit - lin_begin - (n_stages - 1) * STAGE_KEYS) * per_stage;
        if (LANE_WORDS) {
            prog = p.program[(lane < TAIL ? pc_first : pc_tail) + (lane & (BLOCKS_PER_STAGE - 1))];
            pc_first = 0;
            pc_tail = TAIL;
        }
    } else {
        pc_first = ((const_u32_ptr)p.program_ptr)[((long long)variant * p.n_q_tiles + qt) * NW + wave];
    }
    auto start_program = [&]() {
        pc = pc_first;
        if (TEXTQ) {
            whole_left = n_stages - 1;
            if (whole_left == 0) pc = pc_tail;
            pc_wrap = whole_left == 0 ? ~0u : pc_first + per_stage;
        } else if (LANE_WORDS) {
            prog = p.program[pc_first + lane];
            next_words = p.program + pc_first + 64;
            pc = 0;
        }
    };
    auto word = [&]() -> unsigned {
        const unsigned w = LANE_WORDS ? (unsigned)__builtin_amdgcn_readlane((int)prog, (int)(pc & 63)) : words[pc];
        ++pc;
        if (TEXTQ && pc == pc_wrap) {
            const bool last = --whole_left == 0;
            pc = last ? pc_tail : pc_first;
            pc_wrap = last ? ~0u : pc_wrap;
        }
        if (LANE_WORDS && !TEXTQ && (pc & 63) == 0) {
            prog = next_words[lane];
            next_words += 64;
        }
        return w;
    };

    // ---- running softmax state: one query per lane (shared with lane ^ 32)
    WaveState ws;
    ws.c = p.scale_log2e;

    // ---- per-lane LDS read offsets inside a staged block
    unsigned k_lane[2], v_lane[2];
#pragma unroll
    for (int e = 0; e < 2; ++e) {
        k_lane[e] = lds_base + k_lane_offset(lane, e);
        v_lane[e] = lds_base + (unsigned)(NKBUF * STAGE_HALF) + v_lane_offset(lane, e);
    }
    auto block_offset = [](unsigned w) { return (w & kProgramPlaceMask) << 11; };
    auto mask_id = [](unsigned w) { return (w & ~kProgramFlags) >> kProgramMaskShift; };

    // Prologue of the block on the query row (RMS norm over the head's channels - this lane holds half of them,
    // lane ^ 32 the others -, rotary embedding for image queries, back to bf16).  Runs once, after the first
    // stage's loads have been issued, so that the wait for the row and for the tables overlaps them.
    auto query_prologue = [&]() __attribute__((always_inline)) {
    if (p.q_gain || p.rope_y) {
        float ss = 0.f;
#pragma unroll
        for (int s = 0; s < KS; ++s)
#pragma unroll
            for (int j = 0; j < 8; ++j) ss += (float)qf[s][j] * (float)qf[s][j];
        ss = wave_pair_sum(ss);
        const float inv_rms = 1.0f / sqrtf(ss * (1.0f / D) + p.norm_eps);
        const bool has_gain = p.q_gain != nullptr;
        const bool turn = !TEXTQ && p.rope_y;
        // Table entries are fetched without branches, half of the chunks at a time, so that the loads of a half
        // are in flight together (one memory round trip per half, not one per chunk).  A step that is switched
        // off reads the other step's table instead (any D readable floats) and ignores what it read.
        const float* const any_table = has_gain ? p.q_gain : p.rope_y;
        const float* const ysrc = turn ? p.rope_y + (size_t)(imax(imin(qy, qH - 1) - y_shift, 0) * stride + q_oy) * D : any_table;
        const float* const xsrc = turn ? p.rope_x + (size_t)(imin(qx, qW - 1) * stride + q_ox) * D : any_table;
        constexpr int HALF = KS / 2;
#pragma unroll
        for (int h0 = 0; h0 < KS; h0 += HALF) {
            f32x4 g[HALF][2], a[HALF][2], b[HALF][2];
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
                const int c0 = 16 * (h0 + i) + 8 * hh;
                g[i][0] = *(const f32x4*)(any_table + c0);
                g[i][1] = *(const f32x4*)(any_table + c0 + 4);
                a[i][0] = *(const f32x4*)(ysrc + c0);
                a[i][1] = *(const f32x4*)(ysrc + c0 + 4);
                b[i][0] = *(const f32x4*)(xsrc + c0);
                b[i][1] = *(const f32x4*)(xsrc + c0 + 4);
            }
#pragma unroll
            for (int i = 0; i < HALF; ++i) {
                const int s = h0 + i;
                float x[8];
#pragma unroll
                for (int j = 0; j < 8; ++j) x[j] = (float)qf[s][j];
                prologue_chunk_values(x, inv_rms, has_gain, g[i][0], g[i][1], turn, a[i][0], a[i][1], b[i][0], b[i][1]);
#pragma unroll
                for (int j = 0; j < 8; ++j) qf[s][j] = (__bf16)x[j];
            }
        }
    }

    };

    // One pass over the program.  CAREFUL = false: fast pass (fixed reference maximum); returns the
    // lanes that ran out of headroom.  CAREFUL = true: exact online softmax, block by block, slow.
    auto run_pass = [&](auto careful_tag) -> unsigned long long {
        constexpr bool CAREFUL = decltype(careful_tag)::value;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int r = 0; r < 16; ++r) ws.oacc[db][r] = 0.f;
        ws.m_run = M_INIT;
        ws.l_run = 0.f;
        // The Q fragments are waited for here, once, with the first tiles already on their way.
#pragma unroll
        for (int s = 0; s < KS; ++s) asm volatile("" : "+v"(qf[s]));
        if (!CAREFUL) query_prologue();  // the fast pass always comes first
        auto barrier = [&]() {
            __builtin_amdgcn_s_barrier();
            asm volatile("" ::: "memory");
        };
        if (!wave_has_queries) {
            for (int s = 0; s < n_stages; ++s) barrier();
            return 0;
        }
        if (n_stages == 0) return 0;
        int stage = 0;
        unsigned k_at = 0, v_at = 0;  // stage buffers in use, bytes
        auto next_stage = [&]() {
            ++stage;
            k_at ^= STAGE_HALF;
            v_at = v_at + STAGE_HALF == NVBUF * STAGE_HALF ? 0 : v_at + STAGE_HALF;
            barrier();
        };
        start_program();

        if constexpr (CAREFUL) {
            barrier();
            for (;;) {
                const unsigned w = word();
                const unsigned off = block_offset(w), id = mask_id(w);
                if (id != kMaskIdNothing && !(w & kProgramNoBlock)) {
                    const unsigned kb[2] = {k_lane[0] + k_at + off, k_lane[1] + k_at + off}, vb[2] = {v_lane[0] + v_at + off, v_lane[1] + v_at + off};
                    f32x16 s = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};
#pragma unroll
                    for (int ks = 0; ks < KS; ++ks) s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_k(kb, ks), qf[ks], s, 0, 0, 0);
                    if (id != kMaskIdNone) {
                        MaskWords mw;
#pragma unroll
                        for (int r = 0; r < 16; ++r) mw.w[r] = mask_words[16 * (size_t)id + r];
                        mask_scores(s, mw);
                    }
                    const float m_new = fmaxf(ws.m_run, wave_pair_max(max_block(s)));
                    const float alpha = __builtin_amdgcn_exp2f((ws.m_run - m_new) * ws.c);
                    ws.l_run *= alpha;
#pragma unroll
                    for (int db = 0; db < NDB; ++db)
#pragma unroll
                        for (int r = 0; r < 16; ++r) ws.oacc[db][r] *= alpha;
                    ws.m_run = m_new;
                    bf16x8 pf[2];
                    ws.l_run += exp_block(s, ws.c, m_new * ws.c, pf);
#pragma unroll
                    for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                        for (int db = 0; db < NDB; ++db) ws.oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_v(vb, s2, db), pf[s2], ws.oacc[db], 0, 0, 0);
                }
                if (w & kProgramStageEnd) {
                    if (stage + 1 == n_stages) break;
                    next_stage();
                }
            }
            return 0;
        } else {
            // Fast pass: a software pipeline over blocks.  One step issues KS matrix instructions of S = K Q^T for block n and
            // 2 NDB of O += V P for the block before it, in program order, each LDS operand read PD instructions ahead; the
            // vector work rides along:
            //   slots [0, KS)          S of block n        | exponentials, sum, P of block n - 1 (from `t`)
            //   slots [KS, NSLOT)      P V of block n - 1  | the last of them; then scale and mask the scores of block n into `t`
            // The reference maximum of a query never moves once set, so O is only ever touched by the matrix pipeline.
            constexpr int PD = CLEAR_OPERAND_PREFETCH, RING = PD == 1 ? 2 : 4, NSLOT = KS + 2 * NDB;
            static_assert(NSLOT % RING == 0 && PD <= KS && PD < RING, "the operand ring carries over from step to step");
            bf16x8 op[RING];
            float t[16];  // (s - m) c of the block whose exponentials are due
#pragma unroll
            for (int r = 0; r < 16; ++r) t[r] = -INFINITY;  // (nothing before the first block: P = 0)
            const float c = ws.c;
            unsigned w = word(), w_next = word();  // (a program is followed by two more readable words)
            barrier();
            unsigned kb[2], vb[2], v_old = v_at + block_offset(w);
#pragma unroll
            for (int e = 0; e < 2; ++e) kb[e] = k_lane[e] + k_at + block_offset(w);
#pragma unroll
            for (int i = 0; i < PD; ++i) op[i] = read_k(kb, i);
            const f32x16 zero = {0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f, 0.f};

            // returns whether this was the last block
            auto step = [&](auto adopt_tag) __attribute__((always_inline)) -> bool {
                constexpr bool ADOPT = decltype(adopt_tag)::value;
                const unsigned id = mask_id(w);
                const unsigned v_new = v_at + block_offset(w);
#pragma unroll
                for (int e = 0; e < 2; ++e) vb[e] = v_lane[e] + v_old;
                unsigned kn[2];  // block n + 1, if it is in the same stage (otherwise what is read there is read again after the barrier)
#pragma unroll
                for (int e = 0; e < 2; ++e) kn[e] = k_lane[e] + k_at + block_offset(w_next);
                const unsigned w_after = word();
                float mc = ws.m_run * c, sum = 0.f;
                bf16x8 pf[2];
                f32x16 s;
                MaskWords mw;
                auto operand = [&](int slot) { return slot < KS ? read_k(kb, slot) : slot < NSLOT ? read_v(vb, (slot - KS) / NDB, (slot - KS) % NDB) : read_k(kn, slot - NSLOT); };
                auto run_slot = [&](auto slot_tag) __attribute__((always_inline)) {
                    constexpr int slot = decltype(slot_tag)::value;
                    op[(slot + PD) % RING] = operand(slot + PD);
                    // The read stays in front of the matrix instruction, which then waits for older reads only.  (At 64 channels, with twice the vector
                    // work to a matrix instruction, the order inside a slot is better left to the compiler: 256 heads, 64 x 64, 473 -> 459 us.)
                    if (D != 64) SCHED_FENCE();
                    constexpr int i = slot >= KS ? slot - KS : 0;
                    if (slot == 0 && id != kMaskIdNone) {
#pragma unroll
                        for (int r = 0; r < 16; ++r) mw.w[r] = mask_words[16 * (size_t)id + r];
                    }
                    if (slot < KS)
                        s = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], qf[slot < KS ? slot : 0], slot == 0 ? zero : s, 0, 0, 0);
                    else
                        ws.oacc[i % NDB] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(op[slot % RING], pf[i / NDB], ws.oacc[i % NDB], 0, 0, 0);
                    // exponentials as a vector pipeline over pairs of scores: exponentiated in slot a, summed and packed in slot a + 1
#pragma unroll
                    for (int g = 0; g < 8; ++g) {
                        const int a = KS == 8 ? (g < 4 ? g + g / 2 : g + 2) : (g < 4 ? g / 2 : g / 2 + 1);
                        if (slot == a) {
                            t[2 * g] = __builtin_amdgcn_exp2f(t[2 * g]);
                            t[2 * g + 1] = __builtin_amdgcn_exp2f(t[2 * g + 1]);
                        }
                        if (slot == a + 1) {
                            sum += t[2 * g] + t[2 * g + 1];
                            pf[g >> 2][2 * (g & 3)] = (__bf16)t[2 * g];
                            pf[g >> 2][2 * (g & 3) + 1] = (__bf16)t[2 * g + 1];
                            asm volatile("" : "+v"(sum));  // (the sum is formed here, not where it is used)
                        }
                    }
                    constexpr int FIRST = KS == 8 ? KS + 3 : KS + 2;  // the scores of block n are complete; four of them per slot, or eight
                    constexpr int PER = KS == 8 ? 4 : 8;
                    if (!ADOPT && slot >= FIRST && (slot - FIRST) * PER < 16) {
#pragma unroll
                        for (int u = 0; u < PER; ++u) {
                            const int r = slot >= FIRST ? (slot - FIRST) * PER + u : 0;
                            t[r & 15] = __builtin_fmaf(s[r & 15], c, -mc);
                        }
                    }
                    SCHED_FENCE();
                };
                static_for<NSLOT>(run_slot);  // (not a loop: one that contains inline asm is not unrolled)
                if (ADOPT) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] = s[r];
                }
                if (id != kMaskIdNone) {
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] = __builtin_amdgcn_inverse_ballot_w64(mw.w[r]) ? t[r] : -INFINITY;
                }
                if (ADOPT) {
                    float mx = t[0];
#pragma unroll
                    for (int r = 1; r < 16; ++r) mx = fmaxf(mx, t[r]);
                    adopt_reference(ws, wave_pair_max(mx));
                    mc = ws.m_run * c;
#pragma unroll
                    for (int r = 0; r < 16; ++r) t[r] = __builtin_fmaf(t[r], c, -mc);
                }
                ws.l_run += sum;
                v_old = v_new;
                unsigned ended = w;
                w = w_next;
                w_next = w_after;
#pragma unroll
                for (int e = 0; e < 2; ++e) kb[e] = kn[e];
                if (ended & kProgramStageEnd) {
                    for (;;) {
                        if (stage + 1 == n_stages) return true;
                        next_stage();
                        if (!(w & kProgramNoBlock)) break;  // a stage without a block of this wave, and nothing left over from before
                        w = w_next;
                        w_next = word();
                    }
#pragma unroll
                    for (int e = 0; e < 2; ++e) kb[e] = k_lane[e] + k_at + block_offset(w);
#pragma unroll
                    for (int i = 0; i < PD; ++i) op[i] = read_k(kb, i);
                }
                return false;
            };
            // While some query of the wave has no reference maximum yet (the first blocks), the block maxima are formed and
            // adopted; after that no maximum is needed at all.
            bool done = false, adopting = true;
            while (!done && adopting) {
                done = step(std::true_type{});
                adopting = __builtin_amdgcn_ballot_w64(ws.m_run == M_INIT) != 0;
            }
            while (!done) done = step(std::false_type{});
            // the last block's P V
#pragma unroll
            for (int e = 0; e < 2; ++e) vb[e] = v_lane[e] + v_old;
            bf16x8 pf[2];
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const float pv = __builtin_amdgcn_exp2f(t[r]);
                ws.l_run += pv;
                pf[r >> 3][r & 7] = (__bf16)pv;
            }
#pragma unroll
            for (int s2 = 0; s2 < 2; ++s2)
#pragma unroll
                for (int db = 0; db < NDB; ++db) ws.oacc[db] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(read_v(vb, s2, db), pf[s2], ws.oacc[db], 0, 0, 0);
            // the fast pass stands only if every sum stayed finite and moderate
            float chk = ws.l_run;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) chk += __builtin_fabsf(ws.oacc[db][r]);
            return __builtin_amdgcn_ballot_w64(!(chk < FAST_SUM_LIMIT));
        }
    };

    // Fast pass first.  If a query of the workgroup ran out of the range of fp32 on its fixed reference, the whole workgroup repeats
    // the walk with the careful pass.
    const unsigned long long bad = run_pass(std::false_type{});
    __syncthreads();  // every wave has left the stage buffers
    if (lane == 0) flags[wave] = bad != 0;
    __syncthreads();
    unsigned redo = 0;
#pragma unroll
    for (int i = 0; i < NW; ++i) redo |= flags[i];
    if (__builtin_amdgcn_readfirstlane(redo) != 0) {
        __syncthreads();  // every wave has read the flags
        run_pass(std::true_type{});
        __syncthreads();  // the epilogue reuses the stage buffers
    }

    float m_run = ws.m_run;
    f32x16(&oacc)[NDB] = ws.oacc;
    // ---- epilogue
    float l_tot = wave_pair_sum(ws.l_run);
    if (groups > 1) {
        // Join the waves of a patch: the others leave maximum, sum and O in LDS, lane by lane, the first adds them up.
        constexpr int FLOATS = NDB * 16 + 2;
        float* const area = (float*)smem + ((group - 1) * patches + patch) * (FLOATS * 64) + lane;
        if (group > 0) {
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) area[(16 * db + r) * 64] = oacc[db][r];
            area[NDB * 16 * 64] = m_run;
            area[(NDB * 16 + 1) * 64] = l_tot;
        }
        __syncthreads();
        if (group > 0) return;
#pragma unroll 1
        for (int g = 1; g < groups; ++g) {
            const float* const other = (const float*)smem + ((g - 1) * patches + patch) * (FLOATS * 64) + lane;
            const float mo = other[NDB * 16 * 64], m_new = fmaxf(m_run, mo);
            const float wa = __builtin_amdgcn_exp2f((m_run - m_new) * ws.c), wb = __builtin_amdgcn_exp2f((mo - m_new) * ws.c);
            m_run = m_new;
            l_tot = l_tot * wa + other[(NDB * 16 + 1) * 64] * wb;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int r = 0; r < 16; ++r) oacc[db][r] = oacc[db][r] * wa + other[(16 * db + r) * 64] * wb;
        }
    }
    if (TEXTQ && p.n_splits > 1) {
        if (q_valid) {
            const long long row = ((long long)bh * p.n_splits + split) * p.n_text + q_token;
            float* wo = p.ws_o + row * D;
#pragma unroll
            for (int db = 0; db < NDB; ++db)
#pragma unroll
                for (int g = 0; g < 4; ++g) {
                    f32x4 v = {oacc[db][4 * g], oacc[db][4 * g + 1], oacc[db][4 * g + 2], oacc[db][4 * g + 3]};
                    *(f32x4*)(wo + 32 * db + 8 * g + 4 * hh) = v;
                }
            if (hh == 0) {
                p.ws_ml[row * 2] = m_run;
                p.ws_ml[row * 2 + 1] = l_tot;
            }
        }
        return;
    }
    const float inv = 1.0f / l_tot;
    const float lse = __logf(l_tot) + m_run * p.scale_log2e * 0.6931471805599453f;
    if (TEXTQ && p.band_o) {
        if (!q_valid) return;
        const long long row = (long long)bh * p.n_text + q_token;
        if (hh == 0) p.band_lse[row] = lse;
#pragma unroll
        for (int db = 0; db < NDB; ++db)
#pragma unroll
            for (int g = 0; g < 4; ++g) {
                f32x4 v = {oacc[db][4 * g] * inv, oacc[db][4 * g + 1] * inv, oacc[db][4 * g + 2] * inv, oacc[db][4 * g + 3] * inv};
                *(f32x4_any*)(p.band_o + row * D + 32 * db + 8 * g + 4 * hh) = v;
            }
        return;
    }
    // The wave's 32 x D output tile is turned round in LDS (the stage buffers are idle by now: every wave
    // has passed the barrier above) so that it leaves as whole rows: a lane owns a query, and
    // storing from that layout would scatter 8-byte pieces over 32 rows per instruction.
    if (p.lse && q_valid && hh == 0) p.lse[(long long)bh * p.N + q_token] = lse;
    constexpr int OROW = ROW_BYTES + 16;  // padded row pitch in LDS
    static_assert(NW * 32 * OROW <= FWD_LDS_BYTES - FLAG_BYTES, "the output tiles leave the flags alone");
    unsigned char* const wbase = smem + (groups > 1 ? (NW * (NDB * 16 + 2) * 64 * 4 * 3) / 4 : 0) + patch * (32 * OROW);
#pragma unroll
    for (int db = 0; db < NDB; ++db)
#pragma unroll
        for (int g = 0; g < 4; ++g) {
            bf16x4 v;
#pragma unroll
            for (int t = 0; t < 4; ++t) v[t] = (__bf16)(oacc[db][4 * g + t] * inv);
            *(bf16x4*)(wbase + qi * OROW + (32 * db + 8 * g + 4 * hh) * 2) = v;
        }
    // CHUNKS lanes per row, ROWS_PER_STORE rows per store instruction
#pragma unroll
    for (int i = 0; i < 32 / ROWS_PER_STORE; ++i) {
        const int row = ROWS_PER_STORE * i + lane / CHUNKS;  // query slot of the patch
        const f32x4 chunk = *(const f32x4*)(wbase + row * OROW + (lane % CHUNKS) * 16);
        long long token;
        bool store;
        if (TEXTQ) {
            token = (qt * patches + patch) * kTextQueriesPerWave + row;
            store = token < p.n_text;
        } else {
            const int oy = wy0 + (row >> 3), ox = wx0 + (row & 7);
            token = (long long)p.n_text + (long long)((oy - y_shift) * stride + q_oy) * p.gridW + ox * stride + q_ox;
            store = oy < qH && ox < qW && oy >= p.own_y0 && oy < p.own_y1;
        }
        if (store) {
            __bf16* orow = (__bf16*)p.O + batch * p.os.sb + head * p.os.sh + token * p.os.sn;
            __builtin_nontemporal_store(chunk, (f32x4*)(orow + (lane % CHUNKS) * 8));  // whole rows, never read again here
        }
    }
}

template <bool TEXTQ>
__global__ void __launch_bounds__((NW + NLW) * 64, 1) clear_fwd_bf16_kernel(const FwdParams p)
{
    clear_fwd_bf16_workgroup<TEXTQ>(p, (int)blockIdx.x, (int)gridDim.x);
}

// Image-query and text-query rows in one launch: workgroups [0, n_first) are the ones of one kind (p.text_first), the rest those of
// the other.  For problems of a few rounds of workgroups, where a launch of image-query rows alone leaves CUs idle
// at its end and a launch of its own for the text-query rows costs more than it computes.
__global__ void __launch_bounds__((NW + NLW) * 64, 1) clear_fwd_bf16_both_kernel(const FwdParams p, const int n_first)
{
    const int bid = (int)blockIdx.x, rest = (int)gridDim.x - n_first;
    const bool first = bid < n_first;
    if (first != p.text_first)
        clear_fwd_bf16_workgroup<false>(p, first ? bid : bid - n_first, first ? n_first : rest);
    else
        clear_fwd_bf16_workgroup<true>(p, first ? bid : bid - n_first, first ? n_first : rest);
}

// Combines the key-split partial results of the text-query rows: with m the largest running
// maximum, O = sum_i 2^{(m_i - m) c} O_i / sum_i 2^{(m_i - m) c} l_i.
// Bound by reading the partial results.  A thread takes four channels of a row, 1024 / D rows a workgroup, and has the
// loads of four splits in flight; they are added in the order of the splits.
// 24 heads, 512 text tokens, 512 x 512 grid, 16 splits: 48.6 us with one channel a thread -> 25.9 us (4 TB/s).
constexpr int kMergeRows = 1024 / D;
__global__ void __launch_bounds__(256) clear_text_merge_kernel(const FwdParams p)
{
    const unsigned row = blockIdx.x * kMergeRows + threadIdx.x / (D / 4);  // bh * n_text + q
    if (row >= (unsigned)(p.B * p.H * p.n_text)) return;
    const int bh = (int)(row / (unsigned)p.n_text), q = (int)(row % (unsigned)p.n_text);
    const int ch = 4 * (threadIdx.x % (D / 4));
    const long long first = (long long)bh * p.n_splits * p.n_text + q;
    typedef __attribute__((ext_vector_type(2))) float f32x2;
    const f32x2* ml = (const f32x2*)p.ws_ml + first;  // (maximum, denominator), n_text entries from one split to the next
    const float* part = p.ws_o + first * D + ch;
    const long long pitch = (long long)p.n_text * D;
    float m = -INFINITY;
    for (int s = 0; s < p.n_splits; ++s) m = fmaxf(m, ml[(long long)s * p.n_text].x);
    f32x4 num = {0.f, 0.f, 0.f, 0.f};
    float den = 0.f;
    auto add = [&](const f32x2 e, const f32x4 o) __attribute__((always_inline)) {
        const float w = __builtin_amdgcn_exp2f((e.x - m) * p.scale_log2e);
        den += w * e.y;
        num += w * o;
    };
    int s = 0;
    for (; s + 4 <= p.n_splits; s += 4, part += 4 * pitch, ml += 4LL * p.n_text) {
        f32x4 o[4];
        f32x2 e[4];
#pragma unroll
        for (int i = 0; i < 4; ++i) {
            o[i] = *(const f32x4*)(part + i * pitch);
            e[i] = ml[(long long)i * p.n_text];
        }
#pragma unroll
        for (int i = 0; i < 4; ++i) add(e[i], o[i]);
    }
    for (; s < p.n_splits; ++s, part += pitch, ml += p.n_text) add(*ml, *(const f32x4*)part);
    // sum_j exp(s_j / sqrt(d)) = den * 2^{m c}
    const float lse = __logf(den) + m * p.scale_log2e * 0.6931471805599453f;
    const f32x4 out = num / den;
    if (p.band_o) {
        *(f32x4_any*)(p.band_o + (long long)row * D + ch) = out;
        if (ch == 0) p.band_lse[row] = lse;
    } else {
        bf16x4 v;
#pragma unroll
        for (int i = 0; i < 4; ++i) v[i] = (__bf16)out[i];
        *(bf16x4*)((__bf16*)p.O + (bh / p.H) * p.os.sb + (bh % p.H) * p.os.sh + q * p.os.sn + ch) = v;
        if (p.lse && ch == 0) p.lse[(long long)bh * p.N + q] = lse;
    }
}

template <bool TEXTQ>
hipError_t launch_fwd(const FwdParams& p, int nblk, hipStream_t stream)
{
    auto kern = clear_fwd_bf16_kernel<TEXTQ>;
    static LdsLimitOnce lds_limit;  // one per kernel instantiation
    hipError_t e = lds_limit.ensure((const void*)kern, FWD_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(kern, dim3(nblk), dim3((NW + NLW) * 64), FWD_LDS_BYTES, stream, p);
    return hipGetLastError();
}

hipError_t launch_fwd_both(const FwdParams& p, int n_image, int n_text_wgs, hipStream_t stream)
{
    static LdsLimitOnce lds_limit;
    hipError_t e = lds_limit.ensure((const void*)clear_fwd_bf16_both_kernel, FWD_LDS_BYTES);
    if (e != hipSuccess) return e;
    hipLaunchKernelGGL(clear_fwd_bf16_both_kernel, dim3(n_image + n_text_wgs), dim3((NW + NLW) * 64), FWD_LDS_BYTES, stream, p,
                       p.text_first ? n_text_wgs : n_image);
    return hipGetLastError();
}

}  // namespace

#if CLEAR_HEAD_DIM == 128
int bf16_text_queries_per_block() { return kBf16NWY * kBf16NWX * kTextQueriesPerWave; }

#endif  // CLEAR_HEAD_DIM == 128

hipError_t launch_bf16(const FwdParams& p, hipStream_t stream, int phase)
{
    const int BH = p.B * p.H;
    hipError_t e = hipSuccess;
    const int n_text_wgs = p.n_text > 0 ? BH * p.n_tq_tiles * p.n_splits : 0;
    const long long per_head = (long long)p.n_classes * p.n_q_tiles_launch;
    if (phase == kPhaseImageAndTextQuery) return launch_fwd_both(p, (int)(BH * per_head), n_text_wgs, stream);  // (64 image workgroups per CU at most)
    if (phase == kPhaseAll || phase == kPhaseImage) {
        auto shift = [&](FwdParams* q, int b, int h) {
            q->Q = (const __bf16*)p.Q + b * p.qs.sb + h * p.qs.sh;
            q->K = (const __bf16*)p.K + b * p.ks.sb + h * p.ks.sh;
            q->V = (const __bf16*)p.V + b * p.vs.sb + h * p.vs.sh;
            q->O = (__bf16*)p.O + b * p.os.sb + h * p.os.sh;
            if (p.lse) q->lse = p.lse + ((long long)b * p.H + h) * p.N;
        };
        e = launch_by_heads(p, per_head, 0xffffffffLL / ((NW + NLW) * 64), shift, [&](const FwdParams& q, int n) { return launch_fwd<false>(q, n, stream); });
        if (e != hipSuccess) return e;
    }
    if (n_text_wgs > 0 && (phase == kPhaseAll || phase == kPhaseTextQuery)) {
        e = launch_fwd<true>(p, n_text_wgs, stream);
        if (e != hipSuccess) return e;
    }
    if (n_text_wgs > 0 && p.n_splits > 1 && (phase == kPhaseAll || phase == kPhaseTextMerge)) {
        hipLaunchKernelGGL(clear_text_merge_kernel, dim3((BH * p.n_text + kMergeRows - 1) / kMergeRows), dim3(256), 0, stream, p);
        e = hipGetLastError();
    }
    return e;
}

}  // namespace clear
