// Host-side entry points of the library run under the host sanitizers (AddressSanitizer + UndefinedBehaviorSanitizer),
// on a machine without a GPU: the schedule builder on ragged, thin, tiny and large shapes and every mask kind, the
// lattice counts, the lane-mask tables, the per-wave tile descriptors, the band layout, and the argument checks of the calls that need a device
// (each must return an error code before any launch), the wave
// programs (block_programs.cpp), the launch shapes, and contexts over a stand-in for the HIP runtime that can be made to fail (fake_hip.cpp).  Results are cross-checked where a second way to get them
// exists; the point of the run is that no sanitizer report appears.  Exit code 0 = clean.
#include <algorithm>
#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <vector>

#include "../../include/clear_attn.h"
#include "../../paper_2412_16112_amd/csrc/block_class.h"
#include "../../paper_2412_16112_amd/csrc/clear_internal.h"
#include "../../paper_2412_16112_amd/csrc/launch_shape.h"
#include "fake_hip.h"

int check_block_programs();  // block_programs.cpp

static int failures = 0;
#define EXPECT(cond)                                                       \
    do {                                                                   \
        if (!(cond)) {                                                     \
            std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); \
            ++failures;                                                    \
        }                                                                  \
    } while (0)

static void schedules()
{
    const int shapes[][3] = {{16, 16, 4},   {20, 28, 4}, {64, 64, 16}, {33, 17, 9}, {24, 40, 16}, {7, 5, 1},
                             {9, 70, 32},   {1, 1, 3},   {1, 200, 5},  {200, 1, 5}, {128, 128, 8}, {192, 320, 32},
                             {40, 40, 1000}, {17, 3, 2}};
    const int tiles[][4] = {{16, 16, 8, 8}, {4, 8, 4, 8}, {2, 2, 1, 2}, {8, 16, 8, 8}, {3, 5, 7, 2}};
    const int kinds[][2] = {{CLEAR_MASK_DISC, 0}, {CLEAR_MASK_SQUARE, 0}, {CLEAR_MASK_SWIN, 0}, {CLEAR_MASK_SWIN, 1}};
    for (const auto& sh : shapes)
        for (const auto& tl : tiles)
            for (const auto& kd : kinds) {
                const int r = sh[2], shift = kd[1] < r ? kd[1] : 0;
                int nq = 0;
                long long np = 0;
                int rc = clear_attn_schedule_host_masked(sh[0], sh[1], r, kd[0], shift, tl[0], tl[1], tl[2], tl[3], &nq, &np, nullptr, nullptr, nullptr);
                EXPECT(rc == CLEAR_OK);
                std::vector<int> row_ptr((size_t)nq + 1), col((size_t)np + 1);
                std::vector<unsigned char> flags((size_t)np + 1);
                rc = clear_attn_schedule_host_masked(sh[0], sh[1], r, kd[0], shift, tl[0], tl[1], tl[2], tl[3], &nq, &np, row_ptr.data(), col.data(),
                                                     flags.data());
                EXPECT(rc == CLEAR_OK);
                EXPECT(row_ptr[0] == 0 && row_ptr[(size_t)nq] == np);
                const int n_kt = ((sh[0] + tl[2] - 1) / tl[2]) * ((sh[1] + tl[3] - 1) / tl[3]);
                for (long long e = 0; e < np; ++e) EXPECT(col[(size_t)e] >= 0 && col[(size_t)e] < n_kt && flags[(size_t)e] <= 1);
                for (int q = 0; q < nq; ++q)
                    for (int e = row_ptr[(size_t)q] + 1; e < row_ptr[(size_t)q + 1]; ++e) EXPECT(col[(size_t)e - 1] < col[(size_t)e]);
            }
    // the pair bound is an upper bound, and refuses what would not fit int indices
    EXPECT(clear::schedule_pair_bound(64, 64, 16, 16, 16, 8, 8) >= 4 * 4 * 36 - 200);
    int nq = 0;
    long long np = 0;
    EXPECT(clear_attn_schedule_host(32767, 32767, 32768, 16, 16, 8, 8, &nq, &np, nullptr, nullptr, nullptr) == CLEAR_ERR_UNSUPPORTED);
    EXPECT(clear_attn_schedule_host(0, 4, 1, 16, 16, 8, 8, &nq, &np, nullptr, nullptr, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_schedule_host(4, 4, 1, 16, 16, 8, 0, &nq, &np, nullptr, nullptr, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_schedule_host(4, 4, 1, 16, 16, 8, 8, nullptr, &np, nullptr, nullptr, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_schedule_host_masked(32, 32, 4, CLEAR_MASK_STRIDED, 0, 16, 16, 8, 8, &nq, &np, nullptr, nullptr, nullptr) == CLEAR_ERR_UNSUPPORTED);
}

static void counts()
{
    // sum(M) against a visit of every pair, on shapes small enough for that
    const int shapes[][4] = {{8, 16, 16, 4}, {0, 9, 13, 3}, {5, 7, 5, 1}, {3, 12, 10, 40}, {2, 20, 28, 6}};
    for (const auto& sh : shapes) {
        const int n_text = sh[0], gh = sh[1], gw = sh[2], r = sh[3];
        for (int kind = 0; kind < 4; ++kind) {
            const int shift = kind == CLEAR_MASK_SWIN ? r / 2 : (kind == CLEAR_MASK_STRIDED ? r + 1 : 0);
            if (kind == CLEAR_MASK_SWIN && shift >= r) continue;
            unsigned long long got = 0;
            EXPECT(clear_attn_mask_count_masked(n_text, gh, gw, r, kind, shift, &got) == CLEAR_OK);
            const clear::MaskSpec spec = {kind, r, shift};
            const long long N = n_text + (long long)gh * gw;
            unsigned long long want = (unsigned long long)n_text * N + (unsigned long long)gh * gw * n_text;
            for (int qy = 0; qy < gh; ++qy)
                for (int qx = 0; qx < gw; ++qx)
                    for (int ky = 0; ky < gh; ++ky)
                        for (int kx = 0; kx < gw; ++kx) want += clear::mask_admits(spec, qy, qx, ky, kx) ? 1 : 0;
            EXPECT(got == want);
        }
    }
    unsigned long long v = 0;
    EXPECT(clear_attn_mask_count(512, 512, 512, 16, &v) == CLEAR_OK && v == 471125568ull);
    EXPECT(clear_attn_mask_count(512, 32767, 32767, 32768, &v) == CLEAR_OK);
    EXPECT(clear_attn_mask_count(-1, 4, 4, 1, &v) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_mask_count(1, 4, 4, 1, nullptr) == CLEAR_ERR_INVALID_ARG);
}

static void mask_tables()
{
    for (int r : {1, 2, 5, 8, 16, 33})
        for (int kind : {CLEAR_MASK_DISC, CLEAR_MASK_SQUARE}) {
            const int ry = (r + 2) / 4, rx = (r + 6) / 8;
            std::vector<unsigned long long> tbl;
            clear::build_bf16_mask_table(r, ry, rx, kind, &tbl);
            EXPECT(tbl.size() == (size_t)((2 * ry + 1) * (2 * rx + 1) + 2) * 16);
            // entry (0, 0), register 0: lane l keeps key slot 4 (l / 32) of the block against query l % 32
            const unsigned long long w = tbl[(size_t)(ry * (2 * rx + 1) + rx) * 16];
            for (int l = 0; l < 64; ++l) {
                const int dy = -((l & 31) >> 3), dx = 4 * (l >> 5) - (l & 7);
                const bool want = kind == CLEAR_MASK_DISC ? dx * dx + dy * dy < r * r : (dx < r && -dx < r && -dy < r);
                EXPECT(((w >> l) & 1) == (want ? 1u : 0u));
            }
            EXPECT(tbl[tbl.size() - 32] == ~0ull && tbl[tbl.size() - 1] == 0ull);
        }
}

// The per-wave tile descriptors that the backward kernels follow against the classification they replace.
static void wave_descriptors()
{
    using namespace clear;
    const int shapes[][4] = {{64, 64, 16, 512}, {40, 56, 8, 300}, {33, 17, 9, 0}, {128, 128, 16, 70}, {24, 40, 100, 5}, {7, 5, 1, 8}, {96, 96, 32, 512}};
    for (const auto& sh : shapes)
        for (int kind : {CLEAR_MASK_DISC, CLEAR_MASK_SQUARE}) {
            const int gh = sh[0], gw = sh[1], r = sh[2], n_text = sh[3];
            Schedule sc;
            build_schedule(gh, gw, r, kBf16QTileH, kBf16QTileW, kKeyTileH, kKeyTileW, &sc, kind, 0);
            // kernel order of the tile lists: tiles inside the grid first (any order will do here), then the cut ones
            std::vector<int> k_col(sc.col_idx.size()), n_plain(sc.row_ptr.size() - 1, 0);
            auto cut = [&](int id) { return (id / sc.n_ktx + 1) * sc.kth > gh || (id % sc.n_ktx + 1) * sc.ktw > gw; };
            auto origin = [&](int id) { return ((id / sc.n_ktx) * sc.kth) << 16 | ((id % sc.n_ktx) * sc.ktw); };
            for (size_t qt = 0; qt + 1 < sc.row_ptr.size(); ++qt) {
                int w = sc.row_ptr[qt];
                for (int e = sc.row_ptr[qt]; e < sc.row_ptr[qt + 1]; ++e)
                    if (!cut(sc.col_idx[e])) k_col[(size_t)w++] = origin(sc.col_idx[e]);
                n_plain[qt] = w - sc.row_ptr[qt];
                for (int e = sc.row_ptr[qt]; e < sc.row_ptr[qt + 1]; ++e)
                    if (cut(sc.col_idx[e])) k_col[(size_t)w++] = origin(sc.col_idx[e]);
            }
            const int ry = std::min((r + 2) / 4, (gh + 3) / 4), rx = std::min((r + 6) / 8, (gw + 7) / 8);
            const int ncol = 2 * rx + 1, ones = (2 * ry + 1) * ncol, zeros = ones + 1;
            std::vector<int> desc;
            build_wave_descriptors(sc, k_col, n_plain, ry, rx, &desc);
            const int waves = kBf16NWY * kBf16NWX;
            EXPECT(desc.size() == k_col.size() * (size_t)waves);
            const MaskSpec spec = {kind, r, 0};
            for (size_t qt = 0; qt + 1 < sc.row_ptr.size(); ++qt)
                for (int e = sc.row_ptr[qt]; e < sc.row_ptr[qt + 1]; ++e)
                    for (int w = 0; w < waves; ++w) {
                        const int wy0 = (int)(qt / sc.n_qtx) * sc.qth + (w / kBf16NWX) * kWaveQH, wx0 = (int)(qt % sc.n_qtx) * sc.qtw + (w % kBf16NWX) * kWaveQW;
                        const int ta = k_col[(size_t)e] >> 16, tb = k_col[(size_t)e] & 0xffff;
                        const int c0 = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, ta, tb, kKeyBlockH, kKeyBlockW, gh, gw);
                        const int c1 = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, ta + kKeyBlockH, tb, kKeyBlockH, kKeyBlockW, gh, gw);
                        const bool any = c0 != kBlockSkip || c1 != kBlockSkip;
                        const int d = desc[(size_t)e * waves + w];
                        if (e < sc.row_ptr[qt] + n_plain[qt]) {
                            EXPECT((d != kWaveSkipsTile) == any);
                            if (d != kWaveSkipsTile) {
                                const int i0 = d & 0xffff, i1 = (int)((unsigned)d >> 16);
                                EXPECT((i0 == zeros) == (c0 == kBlockSkip) && (i0 == ones) == (c0 == kBlockFull));
                                EXPECT((i1 == zeros) == (c1 == kBlockSkip) && (i1 == ones) == (c1 == kBlockFull));
                                EXPECT(i0 >= 0 && i0 <= zeros && i1 >= 0 && i1 <= zeros);
                                if (c0 == kBlockPartial) EXPECT(i0 == (((ta - wy0) >> 2) + ry) * ncol + ((tb - wx0) >> 3) + rx);
                            }
                        } else {
                            EXPECT(d == kWaveSkipsTile);  // cut tiles are classified in the kernel
                        }
                    }
        }
}

// The launch shapes: key ranges of the text-query rows cover the keys, fit the workspace, and fit the static scratch array wherever
// the plain rule (whole rounds of workgroups of 256 text queries) would, so that clear_attn_forward_noalloc serves those calls.
static void launch_shapes()
{
    using namespace clear;
    const int cus = 256, per_block = bf16_text_queries_per_block();
    auto check_ranges = [&](long long NV, int n_splits, int split_keys) {
        EXPECT(n_splits >= 1 && n_splits <= max_text_splits(NV) && split_keys % kKeyTileKeys == 0);
        EXPECT((long long)(n_splits - 1) * split_keys < NV && NV <= (long long)n_splits * split_keys);
    };
    for (int BH : {1, 2, 3, 7, 24, 38, 76, 152, 1000})
        for (int n_text : {1, 8, 77, 333, 512, 2048})
            for (int side : {1, 7, 16, 20, 33, 64, 80, 128, 144, 256, 512, 1024}) {
                const long long NV = n_text + (long long)side * side;
                const int n_q_tiles = ((side + 15) / 16) * ((side + 15) / 16), n_tq = (n_text + per_block - 1) / per_block;
                for (int f32 = 0; f32 < 2; ++f32)
                    for (int head_dim : {64, 128}) {
                        if (f32 && head_dim != 64) continue;
                        int plain = 0, plain_keys = 0, n_splits, split_keys;
                        choose_text_splits(NV, BH, n_tq, cus, !f32 && (long long)BH * n_q_tiles <= 64LL * cus, &plain, &plain_keys);
                        if (f32) {
                            const F32Shape sh = choose_f32_shape(NV, BH, n_text, head_dim, n_q_tiles, cus);
                            EXPECT(sh.groups == 1 || sh.groups == 2 || sh.groups == 4);
                            EXPECT(sh.n_tq_tiles == (n_text * sh.groups + 63) / 64);
                            n_splits = sh.n_splits;
                            split_keys = sh.split_keys;
                        } else {
                            ForwardProblem fp = {n_text, head_dim, BH, NV, 1, cus, {}};
                            for (int i = 0; i < (n_q_tiles <= 64 ? 3 : 1); ++i) fp.sets[i] = {n_q_tiles << i, 20.0, 25.0 / (1 << i)};
                            const ForwardShape sh = choose_forward_shape(fp);
                            EXPECT((sh.groups == 1 || sh.groups == 2 || sh.groups == 4) && (sh.tq_groups == 1 || sh.tq_groups == 2 || sh.tq_groups == 4));
                            EXPECT(fp.sets[sh.groups / 2].n_image_tiles > 0);
                            n_splits = sh.n_splits;
                            split_keys = sh.split_keys;
                        }
                        if (!f32) {
                            const BackwardProblem bp = {n_text, head_dim, BH, cus, NV, (long long)BH * n_q_tiles, 20.0, 25.0, 40.0};
                            const BackwardShape bwd = choose_backward_shape(bp);
                            check_ranges(NV, bwd.n_splits, bwd.split_keys);
                            // every (workgroup) index of the one launch is 31 bits and its threads 32
                            if ((long long)BH * n_q_tiles <= 64LL * cus) EXPECT(2LL * BH * (n_q_tiles + (long long)n_tq * bwd.n_splits) * 512 <= 0xffffffffLL);
                        }
                        check_ranges(NV, n_splits, split_keys);
                        if (text_partial_bytes(BH, plain, n_text, head_dim) <= kScratchBytes) EXPECT(text_partial_bytes(BH, n_splits, n_text, head_dim) <= kScratchBytes);
                    }
            }
}

static void bands_and_argument_checks()
{
    int y0, y1, ht, hb;
    int covered = 0;
    for (int b = 0; b < 8; ++b) {
        EXPECT(clear_attn_band_layout(512, 16, 8, b, &y0, &y1, &ht, &hb) == CLEAR_OK);
        EXPECT(y0 == covered && y1 - y0 == 64);
        covered = y1;
    }
    EXPECT(clear_attn_band_layout(64, 16, 8, 0, &y0, &y1, &ht, &hb) == CLEAR_ERR_UNSUPPORTED);
    EXPECT(clear_attn_band_layout(8, 4, 2, 2, &y0, &y1, &ht, &hb) == CLEAR_ERR_INVALID_ARG);
    int a, b2, c, d;
    EXPECT(clear_attn_tile_shape(128, CLEAR_BF16, &a, &b2, &c, &d) == CLEAR_OK && a == 16 && b2 == 16 && c == 8 && d == 8);
    EXPECT(clear_attn_tile_shape(128, CLEAR_F32, &a, &b2, &c, &d) == CLEAR_ERR_UNSUPPORTED);
    // calls that need a device: every argument error is found first
    clear_attn_ctx* ctx = nullptr;
    EXPECT(clear_attn_create(nullptr, 8, 16, 16, 128, 4, CLEAR_BF16) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_create(&ctx, 8, 0, 16, 128, 4, CLEAR_BF16) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_create(&ctx, 8, 16, 16, 96, 4, CLEAR_BF16) == CLEAR_ERR_UNSUPPORTED);
    EXPECT(clear_attn_create(&ctx, 8, 16, 16, 128, 0, CLEAR_BF16) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_create(&ctx, 512, 8192, 8192, 128, 16, CLEAR_BF16) == CLEAR_ERR_UNSUPPORTED);  // N >= 2^24
    EXPECT(clear_attn_create_masked(&ctx, 8, 16, 16, 128, 4, CLEAR_BF16, 9, 0) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_create_masked(&ctx, 8, 16, 16, 128, 4, CLEAR_BF16, CLEAR_MASK_SWIN, 4) == CLEAR_ERR_INVALID_ARG);
    EXPECT(ctx == nullptr);
    EXPECT(clear_attn_last_error(nullptr) != nullptr);
    float dummy[4] = {0};
    EXPECT(clear_attn_forward(nullptr, dummy, dummy, dummy, dummy, 1, 1, 8, 16, 16, 128, 4, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_forward_noalloc(nullptr, dummy, dummy, dummy, dummy, 1, 1, 8, 16, 16, 128, 4, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_reserve(nullptr, 1) == CLEAR_ERR_INVALID_ARG);
    const float* parts[1] = {dummy};
    EXPECT(clear_attn_merge_text(0, parts, parts, 1, 1, 8, 264, 128, CLEAR_MERGE_EXACT, dummy, CLEAR_BF16, nullptr) == CLEAR_ERR_INVALID_ARG);
    EXPECT(clear_attn_merge_text(1, parts, parts, 1, 1, 8, 4, 128, CLEAR_MERGE_EXACT, dummy, CLEAR_BF16, nullptr) == CLEAR_ERR_INVALID_ARG);
    clear_attn_destroy(nullptr);
}

// Contexts over the stand-in runtime (fake_hip.cpp): what a call does when the runtime fails in the middle of it.
static void contexts()
{
    const int n_text = 40, gh = 33, gw = 45, d = 128, r = 8;
    const size_t N = n_text + (size_t)gh * gw;
    std::vector<float> buffers[9];
    void* t[9];  // Q, K, V, O, dO, dQ, dK, dV, lse
    for (int i = 0; i < 9; ++i) {
        buffers[i].assign(N * d + 16, 0.f);
        t[i] = (void*)(((uintptr_t)buffers[i].data() + 15) & ~(uintptr_t)15);
    }
    const long long before = fake::live;
    clear_attn_ctx* ctx = nullptr;
    EXPECT(clear_attn_create(&ctx, n_text, gh, gw, d, r, CLEAR_BF16) == CLEAR_OK);
    auto backward = [&]() {
        return clear_attn_backward(ctx, t[0], t[1], t[2], t[3], t[4], (const float*)t[8], t[5], t[6], t[7], 1, 1, n_text, gh, gw, d, r, nullptr);
    };
    // the backward tile lists are made with the first backward call: one that fails halfway leaves nothing behind
    for (int good = 0; good < 2; ++good) {
        const long long live = fake::live;
        fake::backward_launches = 0;
        fake::copies_until_error = good ? -1 : 0;
        EXPECT(backward() == (good ? CLEAR_OK : CLEAR_ERR_HIP));
        fake::copies_until_error = -1;
        if (!good) EXPECT(fake::live == live && fake::backward_launches == 0);
    }
    EXPECT(fake::backward_launches > 0 && fake::backward.row_ptr && fake::backward.col_idx && fake::backward.n_plain);
    EXPECT(clear_attn_forward(ctx, t[0], t[1], t[2], t[3], 1, 1, n_text, gh, gw, d, r, nullptr) == CLEAR_OK);
    EXPECT(fake::forward.program && fake::forward.program_ptr && fake::forward.block_masks && fake::forward.row_ptr);
    clear_attn_destroy(ctx);
    EXPECT(fake::live == before);
    // a context whose upload fails leaves nothing behind either
    fake::copies_until_error = 0;
    EXPECT(clear_attn_create(&ctx, n_text, gh, gw, d, r, CLEAR_BF16) == CLEAR_ERR_HIP);
    fake::copies_until_error = -1;
    fake::no_memory = true;
    EXPECT(clear_attn_create(&ctx, n_text, gh, gw, d, r, CLEAR_BF16) == CLEAR_ERR_ALLOC);
    fake::no_memory = false;
    EXPECT(fake::live == before);
}

// The orders in which a head's tiles are dealt to the workgroups: permutations in blocks of 4 x 8 tiles (forward) and 2 x 16 (backward), of which
// grids no wider than a block need none.
static void tile_orders()
{
    const int grids[][2] = {{64, 64}, {96, 160}, {144, 176}, {100, 272}, {70, 300}};
    for (const auto& g : grids) {
        const int n_qty = (g[0] + 15) / 16, n_qtx = (g[1] + 15) / 16;
        std::vector<float> buffer(16);
        clear_attn_ctx* ctx = nullptr;
        EXPECT(clear_attn_create(&ctx, 0, g[0], g[1], 64, 4, CLEAR_BF16) == CLEAR_OK);
        const size_t bytes = (size_t)g[0] * g[1] * 64 * 2 * 24;
        auto at = [&](int i) { return (void*)(uintptr_t)((i + 1) * ((bytes + 4095) & ~(size_t)4095)); };  // (never read: the launchers are stand-ins)
        EXPECT(clear_attn_forward(ctx, at(0), at(1), at(2), at(3), 1, 24, 0, g[0], g[1], 64, 4, nullptr) == CLEAR_OK);
        EXPECT(clear_attn_backward(ctx, at(0), at(1), at(2), at(3), at(4), (const float*)at(8), at(5), at(6), at(7), 1, 24, 0, g[0], g[1], 64, 4, nullptr) == CLEAR_OK);
        const int* const orders[2] = {fake::forward.groups == 1 ? fake::forward.qt_order : nullptr, fake::backward.qt_order};
        const int rows[2] = {4, 2}, cols[2] = {8, 16}, widest_plain[2] = {10, 16};
        for (int k = 0; k < 2; ++k) {
            if (k == 1 || fake::forward.groups == 1) EXPECT((orders[k] != nullptr) == (n_qtx > widest_plain[k]));
            if (!orders[k]) continue;
            std::vector<char> seen((size_t)n_qty * n_qtx, 0);
            for (int i = 0; i < n_qty * n_qtx; ++i) {
                EXPECT(orders[k][i] >= 0 && orders[k][i] < n_qty * n_qtx && !seen[(size_t)orders[k][i]]);
                seen[(size_t)orders[k][i]] = 1;
            }
            for (int i = 0; i < std::min(rows[k], n_qty) * cols[k]; ++i) EXPECT(orders[k][i] == i / cols[k] * n_qtx + i % cols[k]);
        }
        clear_attn_destroy(ctx);
    }
}

// The launch shapes that the cases of tests/test_gpu_backward.py are named for: how many column ranges the text rows take and whether they
// go first.  A change of the cost model that moves one of them leaves an order or a kernel without its test.
static void backward_orders()
{
    const struct {
        int d, B, H, n_text, gh, gw, r, kind, shift, n_splits;
        bool text_first;
    } cases[] = {
        // test_backward_orders_of_the_one_launch
        {128, 1, 24, 333, 96, 96, 8, CLEAR_MASK_DISC, 0, 3, true},    {128, 1, 24, 441, 43, 80, 16, CLEAR_MASK_DISC, 0, 1, true},
        {64, 1, 38, 333, 64, 64, 16, CLEAR_MASK_DISC, 0, 1, true},    {128, 1, 38, 512, 36, 20, 16, CLEAR_MASK_DISC, 0, 1, false},
        {128, 1, 24, 77, 48, 85, 16, CLEAR_MASK_DISC, 0, 3, false},   {64, 1, 13, 300, 96, 96, 32, CLEAR_MASK_DISC, 0, 10, false},
        {64, 1, 38, 333, 64, 64, 16, CLEAR_MASK_SWIN, 8, 2, true},    {128, 1, 24, 512, 43, 80, 8, CLEAR_MASK_SWIN, 4, 2, true},
        {64, 1, 24, 512, 43, 80, 8, CLEAR_MASK_SQUARE, 0, 2, true},   {128, 1, 24, 512, 43, 80, 8, CLEAR_MASK_SQUARE, 0, 3, false},
        {64, 1, 24, 333, 32, 32, 3, CLEAR_MASK_STRIDED, 1, 1, true},  {128, 1, 24, 333, 43, 80, 4, CLEAR_MASK_STRIDED, 5, 2, false},
        // test_backward_small_passes
        {128, 1, 1, 1, 64, 33, 4, CLEAR_MASK_DISC, 0, 4, false},      {128, 1, 5, 33, 80, 131, 4, CLEAR_MASK_DISC, 0, 15, false},
        {128, 2, 3, 19, 100, 83, 4, CLEAR_MASK_DISC, 0, 15, false},
    };
    for (const auto& c : cases) {
        clear_attn_ctx* ctx = nullptr;
        EXPECT(clear_attn_create_masked(&ctx, c.n_text, c.gh, c.gw, c.d, c.r, CLEAR_BF16, c.kind, c.shift) == CLEAR_OK);
        const size_t bytes = (size_t)(c.n_text + c.gh * c.gw) * c.d * 2 * c.B * c.H;
        auto at = [&](int i) { return (void*)(uintptr_t)((i + 1) * ((bytes + 4095) & ~(size_t)4095)); };  // (never read: the launchers are stand-ins)
        EXPECT(clear_attn_backward(ctx, at(0), at(1), at(2), at(3), at(4), (const float*)at(8), at(5), at(6), at(7), c.B, c.H, c.n_text, c.gh, c.gw, c.d, c.r, nullptr) == CLEAR_OK);
        EXPECT(fake::backward.n_splits == c.n_splits && fake::backward.text_first == c.text_first);
        clear_attn_destroy(ctx);
    }
}

int main()
{
    schedules();
    counts();
    mask_tables();
    wave_descriptors();
    failures += check_block_programs();
    launch_shapes();
    backward_orders();
    bands_and_argument_checks();
    contexts();
    tile_orders();
    if (failures) {
        std::printf("%d check(s) failed\n", failures);
        return 1;
    }
    std::printf("host entry points clean under the sanitizers\n");
    return 0;
}
