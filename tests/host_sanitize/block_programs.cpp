// The wave programs of the bf16 forward kernels (build_block_programs) against the mask itself: every program is walked as
// a computing wave walks it, its lane masks are expanded, and each valid query of the wave's patch must meet every admitted key
// exactly once, over all the waves that share the patch, and no other.  Every word must name a block of a tile that the
// loading waves have staged: the fast pass multiplies what the word names, also where the word masks everything out.
#include <algorithm>
#include <cstdio>
#include <vector>

#include "../../include/clear_attn.h"
#include "../../paper_2412_16112_amd/csrc/block_class.h"
#include "../../paper_2412_16112_amd/csrc/clear_internal.h"

using namespace clear;

static int failures = 0;
#define EXPECT(cond)                                                                             \
    do {                                                                                         \
        if (!(cond) && ++failures <= 20) std::printf("FAILED %s:%d: %s\n", __FILE__, __LINE__, #cond); \
    } while (0)

namespace {

constexpr int kWaves = kBf16NWY * kBf16NWX;

struct Word {
    int tile, half;  // staged tile of the stage, which 32 keys of it
    unsigned id;
    bool stage_end, no_block;
};
Word decode(unsigned w, int tile_units)
{
    const int place = (int)(w & kProgramPlaceMask);
    return {place / tile_units, place % tile_units, (w & ~kProgramFlags) >> kProgramMaskShift, (w & kProgramStageEnd) != 0, (w & kProgramNoBlock) != 0};
}
// whether the lane masks `id` keep key slot `key` for query slot `q`
bool kept(const std::vector<unsigned long long>& masks, unsigned id, int q, int key)
{
    const int reg = 4 * (key >> 3) + (key & 3), lane = q + 32 * ((key >> 2) & 1);
    return masks[(size_t)id * 16 + reg] >> lane & 1;
}

// Text-query rows: the words of a stage with `keys` keys, for 1, 2 and 4 waves per patch.
void check_text_words(const BlockPrograms& prog, const std::vector<unsigned long long>& masks, int head_dim)
{
    const int tps = bf16_tiles_per_stage(head_dim), tile_units = kKeyTileKeys * head_dim * 2 / 2048, stage_keys = tps * kKeyTileKeys;
    for (int i = 0; i < 3; ++i) {
        const int waves = 1 << i, per = 2 * tps / waves;
        for (int keys = 0; keys <= stage_keys; ++keys) {
            const int real = keys == 0 ? stage_keys : keys, staged = (real + kKeyTileKeys - 1) / kKeyTileKeys;
            std::vector<int> seen((size_t)stage_keys, 0);
            for (int g = 0; g < waves; ++g) {
                const size_t at = prog.text_words[i] + ((size_t)g * (stage_keys + 1) + keys) * per;
                bool ended = false;
                for (int k = 0; k < per && !ended; ++k) {
                    const Word w = decode(prog.words[at + k], tile_units);
                    ended = w.stage_end;
                    EXPECT(!w.no_block);
                    EXPECT(w.half < 2 && w.tile < staged);  // (a tile that holds a key: the others are not loaded)
                    EXPECT((size_t)w.id * 16 + 16 <= masks.size());
                    for (int key = 0; key < 32; ++key) {
                        EXPECT(kept(masks, w.id, 0, key) == kept(masks, w.id, 31, key));
                        if (kept(masks, w.id, 0, key)) ++seen[(size_t)(w.tile * kKeyTileKeys + w.half * 32 + key)];
                    }
                }
                EXPECT(ended);
            }
            for (int key = 0; key < stage_keys; ++key) EXPECT(seen[(size_t)key] == (key < real));
        }
    }
}

struct Shape {
    int n_text, gridH, gridW, r, kind, shift;
};

// Image-query rows of one table set.
void check_image_programs(const Shape& sh, const Schedule& s, const std::vector<int>& k_col, const BlockPrograms& prog,
                          const std::vector<unsigned long long>& masks, int head_dim, int groups)
{
    unsigned long long ran[4][4] = {};  // blocks run: by key class and query class
    const bool strided = sh.kind == CLEAR_MASK_STRIDED && sh.r > 1;  // (r = 1 admits every pair: one class)
    const MaskSpec spec = {sh.kind, sh.r, sh.shift};
    const int tps = bf16_tiles_per_stage(head_dim), tile_units = kKeyTileKeys * head_dim * 2 / 2048;
    const int n_lin_tiles = (sh.n_text + kKeyTileKeys - 1) / kKeyTileKeys, n_lin_stages = (n_lin_tiles + tps - 1) / tps;
    const size_t n_q_tiles = s.row_ptr.size() - 1;
    const int patches = kWaves / groups;
    EXPECT(prog.ptr.size() == (strided ? 4 : 1) * n_q_tiles * kWaves);
    for (int v = 0; v < (strided ? 4 : 1); ++v) {
        // a residue class has gridH / r or one more rows, gridW / r or one more columns; the larger class exists where r does not divide
        if (((v >> 1) && sh.gridH % sh.r == 0) || ((v & 1) && sh.gridW % sh.r == 0)) continue;
        const int kH = strided ? sh.gridH / sh.r + (v >> 1) : sh.gridH, kW = strided ? sh.gridW / sh.r + (v & 1) : sh.gridW;
        for (size_t qt = 0; qt < n_q_tiles; ++qt) {
            const int begin = s.row_ptr[qt], n_img = s.row_ptr[qt + 1] - begin, n_stages = n_lin_stages + (n_img + tps - 1) / tps;
            for (int patch = 0; patch < patches; ++patch) {
                const int wy0 = (int)(qt / s.n_qtx) * s.qth + (patch / kBf16NWX) * kWaveQH, wx0 = (int)(qt % s.n_qtx) * s.qtw + (patch % kBf16NWX) * kWaveQW;
                if (wy0 >= s.gridH || wx0 >= s.gridW) continue;  // a wave without queries runs no program
                std::vector<unsigned char> text((size_t)32 * (sh.n_text + 1), 0), image((size_t)32 * kH * kW, 0);
                for (int g = 0; g < groups; ++g) {
                    size_t pc = prog.ptr[((size_t)v * n_q_tiles + qt) * kWaves + g * patches + patch];
                    bool flushed = false;  // the word before masks everything out
                    for (int st = 0; st < n_stages;) {
                        if (pc + kProgramSpareWords >= prog.words.size()) {  // (the kernels read ahead)
                            EXPECT(pc + kProgramSpareWords < prog.words.size());
                            return;
                        }
                        const Word w = decode(prog.words[pc++], tile_units);
                        const bool linear = st < n_lin_stages;
                        const int i = (linear ? st : st - n_lin_stages) * tps + w.tile;
                        if (w.no_block) {
                            EXPECT(flushed && w.stage_end);  // (nothing may be left over from the stage before)
                        } else {
                            EXPECT(w.half < 2 && w.tile < tps && i < (linear ? n_lin_tiles : n_img));
                            EXPECT((size_t)w.id * 16 + 16 <= masks.size());
                        }
                        flushed = w.no_block || w.id == kMaskIdNothing;
                        for (int u = 0; u < (strided ? 4 : 1) && !w.no_block; ++u)
                            if (!strided || (wy0 < sh.gridH / sh.r + (u >> 1) && wx0 < sh.gridW / sh.r + (u & 1))) ++ran[v][u];
                        if (!w.no_block && i < (linear ? n_lin_tiles : n_img) && (size_t)w.id * 16 + 16 <= masks.size())
                            for (int q = 0; q < 32; ++q) {
                                const int qy = wy0 + (q >> 3), qx = wx0 + (q & 7);
                                if (qy >= s.gridH || qx >= s.gridW) continue;
                                for (int key = 0; key < 32; ++key) {
                                    if (!kept(masks, w.id, q, key)) continue;
                                    if (linear) {
                                        const int token = i * kKeyTileKeys + w.half * 32 + key;
                                        EXPECT(token < sh.n_text);
                                        if (token < sh.n_text) ++text[(size_t)q * sh.n_text + token];
                                    } else {
                                        const int ky = (k_col[(size_t)begin + i] >> 16) + kKeyBlockH * w.half + (key >> 3), kx = (k_col[(size_t)begin + i] & 0xffff) + (key & 7);
                                        EXPECT(ky < kH && kx < kW);
                                        if (ky < kH && kx < kW) ++image[((size_t)q * kH + ky) * kW + kx];
                                    }
                                }
                            }
                        st += w.stage_end;
                    }
                }
                for (int q = 0; q < 32; ++q) {
                    const int qy = wy0 + (q >> 3), qx = wx0 + (q & 7);
                    if (qy >= s.gridH || qx >= s.gridW) continue;
                    int wrong = 0;
                    for (int t = 0; t < sh.n_text; ++t) wrong += text[(size_t)q * sh.n_text + t] != 1;
                    for (int ky = 0; ky < kH; ++ky)
                        for (int kx = 0; kx < kW; ++kx) wrong += image[((size_t)q * kH + ky) * kW + kx] != (sh.kind == CLEAR_MASK_STRIDED || mask_admits(spec, qy, qx, ky, kx));
                    EXPECT(wrong == 0);
                }
            }
        }
    }
    if (groups > 1) return;
    // the count the library reports: what the classes' waves run, and every 32-key block for every 32 text queries
    unsigned long long want = 0;
    const int stride = strided ? sh.r : 1;
    for (int b = 0; b < stride; ++b)
        for (int a = 0; a < stride; ++a) {
            auto extra = [&](int n, int c) { return (n - c + stride - 1) / stride - n / stride; };  // rows (columns) of class c beyond n / stride
            const int ky = (b + sh.shift / stride) % stride, kx = (a + sh.shift) % stride;
            want += strided ? ran[2 * extra(sh.gridH, ky) + extra(sh.gridW, kx)][2 * extra(sh.gridH, b) + extra(sh.gridW, a)] : ran[0][0];
        }
    want += (unsigned long long)((sh.n_text + 31) / 32) * ((sh.n_text + (unsigned long long)sh.gridH * sh.gridW + 31) / 32);
    EXPECT(executed_pairs_bf16(prog, sh.n_text, sh.gridH, sh.gridW, stride, strided ? sh.shift : 0) == want * 1024);
}

void check_shape(const Shape& sh, int head_dim)
{
    const bool strided = sh.kind == CLEAR_MASK_STRIDED && sh.r > 1;  // (r = 1 admits every pair: one class)
    const bool dense = sh.kind == CLEAR_MASK_STRIDED;  // within a class
    const int n = strided ? 1 : 3, schedH = strided ? (sh.gridH + sh.r - 1) / sh.r : sh.gridH, schedW = strided ? (sh.gridW + sh.r - 1) / sh.r : sh.gridW;
    Schedule sched[3];
    QueryTilePatterns pat[3];
    std::vector<int> k_col[3];
    std::vector<ProgramInput> in;
    for (int i = 0; i < n; ++i) {
        build_schedule(schedH, schedW, dense ? schedH + schedW : sh.r, kBf16QTileH >> i, kBf16QTileW, kKeyTileH, kKeyTileW, &sched[i],
                       dense ? (int)kMaskDisc : sh.kind, dense ? 0 : sh.shift);
        pat[i] = query_tile_patterns(sched[i]);
        order_forward_tiles(sched[i], pat[i], &k_col[i]);
        // the ordered list is the scheduled one
        for (size_t qt = 0; qt + 1 < sched[i].row_ptr.size(); ++qt) {
            std::vector<int> a, b;
            for (int e = sched[i].row_ptr[qt]; e < sched[i].row_ptr[qt + 1]; ++e) {
                a.push_back((sched[i].col_idx[e] / sched[i].n_ktx) * kKeyTileH << 16 | (sched[i].col_idx[e] % sched[i].n_ktx) * kKeyTileW);
                b.push_back(k_col[i][e]);
            }
            std::sort(a.begin(), a.end());
            std::sort(b.begin(), b.end());
            EXPECT(a == b);
        }
        in.push_back({&sched[i], &pat[i], &k_col[i], 1 << i});
    }
    std::vector<BlockPrograms> prog;
    std::vector<unsigned long long> masks;
    build_block_programs(in, sh.n_text, head_dim, strided ? sh.r : 1, sh.gridH, sh.gridW, &prog, &masks);
    const int before = failures;
    for (int i = 0; i < n; ++i) {
        check_text_words(prog[i], masks, head_dim);
        check_image_programs(sh, sched[i], k_col[i], prog[i], masks, head_dim, 1 << i);
    }
    if (failures != before)
        std::printf("  in: n_text %d, grid %d x %d, r %d, mask %d, shift %d, head_dim %d\n", sh.n_text, sh.gridH, sh.gridW, sh.r, sh.kind, sh.shift, head_dim);
}

}  // namespace

// Waves and query tiles whose programs are the same share one: without that a window that holds the whole grid took 16 words a
// (query tile, key tile) pair.
static void check_sharing()
{
    const Shape shapes[] = {{64, 256, 256, 400, CLEAR_MASK_DISC, 0}, {0, 253, 251, 400, CLEAR_MASK_DISC, 0}, {10, 200, 203, 300, CLEAR_MASK_SQUARE, 0},
                            {10, 200, 203, 512, CLEAR_MASK_SWIN, 0}, {10, 256, 254, 2, CLEAR_MASK_STRIDED, 1}};
    for (const Shape& sh : shapes) {
        const int stride = sh.kind == CLEAR_MASK_STRIDED ? sh.r : 1;
        Schedule s;
        build_schedule((sh.gridH + stride - 1) / stride, (sh.gridW + stride - 1) / stride, stride > 1 ? sh.gridH + sh.gridW : sh.r, kBf16QTileH, kBf16QTileW,
                       kKeyTileH, kKeyTileW, &s, stride > 1 ? (int)kMaskDisc : sh.kind, 0);
        const QueryTilePatterns pat = query_tile_patterns(s);
        std::vector<int> k_col;
        order_forward_tiles(s, pat, &k_col);
        std::vector<BlockPrograms> prog;
        std::vector<unsigned long long> masks;
        build_block_programs({{&s, &pat, &k_col, 1}}, sh.n_text, 128, stride, sh.gridH, sh.gridW, &prog, &masks);
        const size_t text_words = 257 + 2 * 129 * 2 + 4 * 129 + 2048;
        EXPECT(prog[0].words.size() <= 2 * s.col_idx.size() * (stride > 1 ? 2 : 1) + s.row_ptr.size() * 8 + text_words);
    }
}

int check_block_programs()
{
    check_sharing();
    const Shape shapes[] = {{8, 16, 16, 4, CLEAR_MASK_DISC, 0},     {0, 1, 1, 1, CLEAR_MASK_DISC, 0},       {77, 48, 85, 16, CLEAR_MASK_DISC, 0},
                            {130, 37, 29, 9, CLEAR_MASK_DISC, 0},   {5, 7, 70, 32, CLEAR_MASK_DISC, 0},     {31, 80, 3, 11, CLEAR_MASK_DISC, 0},
                            {40, 33, 45, 100, CLEAR_MASK_DISC, 0},  {64, 72, 104, 5, CLEAR_MASK_DISC, 0},   {1, 50, 66, 12, CLEAR_MASK_SWIN, 5},
                            {33, 48, 64, 16, CLEAR_MASK_SWIN, 8},   {0, 41, 39, 7, CLEAR_MASK_SWIN, 0},     {65, 20, 23, 64, CLEAR_MASK_SWIN, 1},
                            {12, 43, 39, 7, CLEAR_MASK_SQUARE, 0},  {129, 64, 48, 16, CLEAR_MASK_SQUARE, 0}, {3, 21, 90, 200, CLEAR_MASK_SQUARE, 0},
                            {50, 38, 45, 5, CLEAR_MASK_STRIDED, 17}, {0, 64, 64, 2, CLEAR_MASK_STRIDED, 1},  {9, 35, 36, 1, CLEAR_MASK_STRIDED, 0},
                            {70, 96, 80, 3, CLEAR_MASK_STRIDED, 4}, {2, 24, 17, 16, CLEAR_MASK_STRIDED, 200}};
    for (const Shape& sh : shapes)
        for (int head_dim : {64, 128}) check_shape(sh, head_dim);
    unsigned state = 12345;
    auto draw = [&](int lo, int hi) { return lo + (int)((state = state * 1664525u + 1013904223u) >> 8) % (hi - lo + 1); };
    for (int i = 0; i < 40; ++i) {
        Shape sh = {draw(0, 150), draw(1, 70), draw(1, 70), draw(1, draw(1, 40)), draw(0, 3), 0};
        if (sh.kind == CLEAR_MASK_SWIN) sh.shift = draw(0, sh.r - 1);
        if (sh.kind == CLEAR_MASK_STRIDED) {
            sh.r = std::min(sh.r, std::min(sh.gridH, sh.gridW));
            sh.shift = draw(0, 2 * sh.r * sh.r);
        }
        check_shape(sh, draw(0, 1) ? 64 : 128);
    }
    return failures;
}
