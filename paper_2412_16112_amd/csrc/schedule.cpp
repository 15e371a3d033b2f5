// Host-side integer geometry of the CLEAR mask (Eq. 3, Sec. 3.2): tile schedule, sum(M), and the
// count of pairs the kernels execute.  No device code here.
#include "block_class.h"
#include "clear_internal.h"

#include <algorithm>
#include <array>
#include <map>
#include <new>
#include <cstddef>
#include <unordered_map>
#include <utility>

namespace clear {

static inline int ceil_div(int a, int b) { return (a + b - 1) / b; }
static inline long long imin_ll(long long a, long long b) { return a < b ? a : b; }

// Smallest |a - b| for a in [a0, a1], b in [b0, b1].
static inline int interval_gap(int a0, int a1, int b0, int b1)
{
    if (b0 > a1) return b0 - a1;
    if (a0 > b1) return a0 - b1;
    return 0;
}

long long schedule_pair_bound(int gridH, int gridW, int r, int qth, int qtw, int kth, int ktw)
{
    // per query tile: the rectangle of key tiles that come within r - 1 on each axis (what build_schedule scans)
    const int n_qty = ceil_div(gridH, qth), n_qtx = ceil_div(gridW, qtw), n_kty = ceil_div(gridH, kth), n_ktx = ceil_div(gridW, ktw);
    long long rows = 0, cols = 0;  // the count factorises over the two axes
    for (int ty = 0; ty < n_qty; ++ty) {
        const int qy0 = ty * qth, qy1 = imin(qy0 + qth, gridH) - 1;
        const long long lo = imax(0, (int)(((long long)qy0 - (r - 1)) / kth) - 1), hi = imin(n_kty - 1, (int)imin_ll(((long long)qy1 + r - 1) / kth, n_kty));
        rows += hi >= lo ? hi - lo + 1 : 0;
    }
    for (int tx = 0; tx < n_qtx; ++tx) {
        const int qx0 = tx * qtw, qx1 = imin(qx0 + qtw, gridW) - 1;
        const long long lo = imax(0, (int)(((long long)qx0 - (r - 1)) / ktw) - 1), hi = imin(n_ktx - 1, (int)imin_ll(((long long)qx1 + r - 1) / ktw, n_ktx));
        cols += hi >= lo ? hi - lo + 1 : 0;
    }
    return rows * cols;
}

void build_schedule(int gridH, int gridW, int r, int qth, int qtw, int kth, int ktw, Schedule* s, int mask_kind, int mask_shift)
{
    s->gridH = gridH; s->gridW = gridW; s->r = r;
    s->mask_kind = mask_kind; s->mask_shift = mask_shift;
    s->qth = qth; s->qtw = qtw; s->kth = kth; s->ktw = ktw;
    s->n_qty = ceil_div(gridH, qth); s->n_qtx = ceil_div(gridW, qtw);
    s->n_kty = ceil_div(gridH, kth); s->n_ktx = ceil_div(gridW, ktw);
    s->row_ptr.assign(1, 0);
    s->col_idx.clear();
    s->flags.clear();
    const long long r2 = (long long)r * r;
    for (int ty = 0; ty < s->n_qty; ++ty)
        for (int tx = 0; tx < s->n_qtx; ++tx) {
            // extent of the query tile inside the grid
            const int qy0 = ty * qth, qy1 = imin(qy0 + qth, gridH) - 1;
            const int qx0 = tx * qtw, qx1 = imin(qx0 + qtw, gridW) - 1;
            const bool q_inside = (qy0 + qth <= gridH) && (qx0 + qtw <= gridW);
            // key tiles that can come within distance r-1 on each axis
            const int kty_lo = imax(0, (qy0 - (r - 1)) / kth - 1), kty_hi = imin(s->n_kty - 1, (qy1 + r - 1) / kth);
            const int ktx_lo = imax(0, (qx0 - (r - 1)) / ktw - 1), ktx_hi = imin(s->n_ktx - 1, (qx1 + r - 1) / ktw);
            for (int ky = kty_lo; ky <= kty_hi; ++ky)
                for (int kx = ktx_lo; kx <= ktx_hi; ++kx) {
                    const int ky0 = ky * kth, ky1 = imin(ky0 + kth, gridH) - 1;
                    const int kx0 = kx * ktw, kx1 = imin(kx0 + ktw, gridW) - 1;
                    const long long dy = interval_gap(qy0, qy1, ky0, ky1), dx = interval_gap(qx0, qx1, kx0, kx1);
                    const bool k_inside = (ky0 + kth <= gridH) && (kx0 + ktw <= gridW);
                    const long long fy = imax(qy1 - ky0, ky1 - qy0), fx = imax(qx1 - kx0, kx1 - qx0);
                    bool full;
                    if (mask_kind == kMaskSquare) {
                        if (dy >= r || dx >= r) continue;  // no pair inside the square window: not listed
                        full = q_inside && k_inside && fy < r && fx < r;
                    } else if (mask_kind == kMaskSwin) {
                        // windows (per axis) that the two tiles touch: listed iff they share one
                        const int wq0 = (qy0 + mask_shift) / r, wq1 = (qy1 + mask_shift) / r, wk0 = (ky0 + mask_shift) / r, wk1 = (ky1 + mask_shift) / r;
                        const int vq0 = (qx0 + mask_shift) / r, vq1 = (qx1 + mask_shift) / r, vk0 = (kx0 + mask_shift) / r, vk1 = (kx1 + mask_shift) / r;
                        if (wq1 < wk0 || wk1 < wq0 || vq1 < vk0 || vk1 < vq0) continue;
                        full = q_inside && k_inside && wq0 == wq1 && wk0 == wk1 && wq0 == wk0 && vq0 == vq1 && vk0 == vk1 && vq0 == vk0;
                    } else {
                        if (dy * dy + dx * dx >= r2) continue;  // no pair closer than r: not listed
                        full = q_inside && k_inside && fy * fy + fx * fx < r2;
                    }
                    s->col_idx.push_back(ky * s->n_ktx + kx);
                    s->flags.push_back(full ? 1 : 0);
                }
            s->row_ptr.push_back((int)s->col_idx.size());
        }
}

unsigned long long mask_count(int n_text, int gridH, int gridW, int r, int mask_kind, int mask_shift)
{
    if (mask_kind == kMaskStrided) {
        // a query in column residue a sees the columns of residue (a + r_x) % r; rows likewise; the two axes factorise
        const unsigned long long n_img = (unsigned long long)gridH * gridW, N = n_img + n_text;
        const int rx = mask_shift % r, ry = (mask_shift / r) % r;
        auto count = [&](int n, int a) -> unsigned long long { return a < n ? (unsigned long long)((n - a + r - 1) / r) : 0ull; };
        unsigned long long sx = 0, sy = 0;
        for (int a = 0; a < r; ++a) sx += count(gridW, a) * count(gridW, (a + rx) % r);
        for (int b = 0; b < r; ++b) sy += count(gridH, b) * count(gridH, (b + ry) % r);
        return (unsigned long long)n_text * N + n_img * n_text + sx * sy;
    }
    if (mask_kind == kMaskSwin) {
        // every window of h x w tokens contributes (h w)^2 pairs; windows are the cells of the shifted partition
        const unsigned long long n_img = (unsigned long long)gridH * gridW, N = n_img + n_text;
        unsigned long long sy = 0, sx = 0, img = 0;
        // sum over window rows of h^2 ... the count factorises: sum_{wy, wx} (h_wy w_wx)^2 = (sum h^2)(sum w^2)
        for (int y = 0; y < gridH;) {
            const int end = imin(gridH, ((y + mask_shift) / r + 1) * r - mask_shift);
            sy += (unsigned long long)(end - y) * (end - y);
            y = end;
        }
        for (int x = 0; x < gridW;) {
            const int end = imin(gridW, ((x + mask_shift) / r + 1) * r - mask_shift);
            sx += (unsigned long long)(end - x) * (end - x);
            x = end;
        }
        img = sy * sx;
        return (unsigned long long)n_text * N + n_img * n_text + img;
    }
    // Each offset (dy, dx) of the open disc occurs (gridH - |dy|)(gridW - |dx|) times on the raster.
    const unsigned long long n_img = (unsigned long long)gridH * gridW, N = n_img + n_text;
    unsigned long long img = 0;
    const long long r2 = (long long)r * r;
    for (long long dy = -(r - 1); dy <= r - 1; ++dy) {
        const long long ady = dy < 0 ? -dy : dy;
        if (ady >= gridH) continue;
        for (long long dx = -(r - 1); dx <= r - 1; ++dx) {
            const long long adx = dx < 0 ? -dx : dx;
            if (adx >= gridW || (mask_kind == kMaskDisc && dx * dx + dy * dy >= r2)) continue;  // (square: every |dx|, |dy| < r)
            img += (unsigned long long)(gridH - ady) * (unsigned long long)(gridW - adx);
        }
    }
    return (unsigned long long)n_text * N + n_img * n_text + img;
}

// Lane masks of the bf16 kernels for a (4 x 8 query patch, 4 x 8 key block) pair whose origins differ by
// (4 dby, 8 dbx), |dby| <= ry, |dbx| <= rx: entry (dby + ry) * (2 rx + 1) + dbx + rx holds 16 words, one per
// score register r; bit l is set iff lane l (query l % 32 of the patch, key slot 8 (r/4) + 4 (l/32) + r % 4
// of the block) is admitted by the mask: Eq. 3, dx^2 + dy^2 < r^2, or the square window |dx| < r and |dy| < r
// (the two kinds that depend on the offset alone).  Two more entries follow: all ones, all zeros.
void build_bf16_mask_table(int r, int ry, int rx, int mask_kind, std::vector<unsigned long long>* tbl)
{
    const MaskSpec spec = {mask_kind, r, 0};
    const long long r2 = (long long)r * r;
    const int ncol = 2 * rx + 1;
    tbl->assign((size_t)((2 * ry + 1) * ncol + 2) * 16, 0ull);
    for (int dby = -ry; dby <= ry; ++dby)
        for (int dbx = -rx; dbx <= rx; ++dbx) {
            unsigned long long* e = tbl->data() + (size_t)((dby + ry) * ncol + dbx + rx) * 16;
            for (int reg = 0; reg < 16; ++reg)
                for (int l = 0; l < 64; ++l) {
                    const int qi = l & 31, hh = l >> 5;
                    const long long dy = 4 * dby + (reg >> 2) - (qi >> 3);
                    const long long dx = 8 * dbx + 4 * hh + (reg & 3) - (qi & 7);
                    const bool in_reach = dx > -r && dx < r && dy > -r && dy < r;  // (also keeps the products below in range)
                    if (in_reach && (mask_kind == kMaskDisc ? dx * dx + dy * dy < r2 : mask_admits(spec, 0, 0, (int)dy, (int)dx))) e[reg] |= 1ull << l;
                }
        }
    unsigned long long* ones = tbl->data() + tbl->size() - 32;
    for (int reg = 0; reg < 16; ++reg) ones[reg] = ~0ull;
}

void build_wave_descriptors(const Schedule& s, const std::vector<int>& k_col, const std::vector<int>& n_plain, int mask_ry, int mask_rx,
                            std::vector<int>* desc)
{
    const int nwy = s.qth / kWaveQH, nwx = s.qtw / kWaveQW, waves = nwy * nwx;
    const MaskSpec spec = {s.mask_kind, s.r, s.mask_shift};
    const int ncol = 2 * mask_rx + 1;
    const int ones = (2 * mask_ry + 1) * ncol, zeros = ones + 1;
    desc->assign(k_col.size() * (size_t)waves, kWaveSkipsTile);
    for (size_t qt = 0; qt + 1 < s.row_ptr.size(); ++qt) {
        const int qy0 = (int)(qt / s.n_qtx) * s.qth, qx0 = (int)(qt % s.n_qtx) * s.qtw;
        for (int e = s.row_ptr[qt]; e < s.row_ptr[qt] + n_plain[qt]; ++e) {
            const int ta = k_col[e] >> 16, tb = k_col[e] & 0xffff;
            for (int w = 0; w < waves; ++w) {
                const int wy0 = qy0 + (w / nwx) * kWaveQH, wx0 = qx0 + (w % nwx) * kWaveQW;
                int idx[2];
                bool any = false;
                for (int kb = 0; kb < 2; ++kb) {
                    const int cls = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, ta + kKeyBlockH * kb, tb, kKeyBlockH, kKeyBlockW,
                                                              s.gridH, s.gridW);
                    any |= cls != kBlockSkip;
                    const int dby = ((ta - wy0) >> 2) + kb, dbx = (tb - wx0) >> 3;  // relative block offset in blocks (exact: both are aligned)
                    idx[kb] = cls == kBlockPartial ? (dby + mask_ry) * ncol + dbx + mask_rx : (cls == kBlockFull ? ones : zeros);
                }
                if (any) (*desc)[(size_t)e * waves + w] = idx[0] | (idx[1] << 16);
            }
        }
    }
}

namespace {

// Lane masks of (4 x 8 query patch, 4 x 8 key block) pairs, each distinct one kept once.
class BlockMasks {
  public:
    BlockMasks(const MaskSpec& spec, std::vector<unsigned long long>* words) : spec_(spec), words_(words)
    {
        words_->assign((size_t)kMaskIdFree * 16, 0ull);
        for (int reg = 0; reg < 16; ++reg) (*words_)[(size_t)kMaskIdNone * 16 + reg] = ~0ull;
        for (int k = 1; k < 32; ++k)
            for (int reg = 0; reg < 16; ++reg) {
                const int key = 8 * (reg >> 2) + (reg & 3);  // of the lower lanes; the upper lanes hold the key 4 further on
                (*words_)[(size_t)(kMaskIdFirstKeys + k) * 16 + reg] = (key < k ? 0xffffffffull : 0) | (key + 4 < k ? 0xffffffffull << 32 : 0);
            }
    }
    const MaskSpec& spec() const { return spec_; }
    // The disc: a patch at (wy0, wx0) against a block at (ky0, kx0) of which the first `rows` rows and `cols` columns are keys.
    unsigned of_disc(int wy0, int wx0, int ky0, int kx0, int rows, int cols)
    {
        // depends on the offset alone
        const unsigned long long key = ((unsigned long long)(unsigned)(ky0 - wy0) << 32) ^ ((unsigned long long)(unsigned)(kx0 - wx0) << 8) ^ (unsigned)(rows << 4 | cols);
        auto it = by_offset_.find(key);
        if (it != by_offset_.end()) return it->second;
        // one byte (8 query columns) per row offset and key column
        unsigned char byte[kWaveQH + kKeyBlockH - 1][kKeyBlockW];
        for (int d = 0; d < kWaveQH + kKeyBlockH - 1; ++d) {
            const long long dy = (long long)ky0 - wy0 + d - (kWaveQH - 1), lim = (long long)spec_.r * spec_.r - dy * dy;
            unsigned near = 0;  // bit t: dx = kx0 - wx0 + t - 7 is close enough
            for (int t = 0; t < kWaveQW + kKeyBlockW - 1; ++t) {
                const long long dx = (long long)kx0 - wx0 + t - (kWaveQW - 1);
                near |= (unsigned)(dx * dx < lim) << t;
            }
            for (int kx = 0; kx < kKeyBlockW; ++kx) {
                unsigned v = 0;
                for (int qx = 0; qx < kWaveQW; ++qx) v |= (near >> (kx - qx + kWaveQW - 1) & 1) << qx;
                byte[d][kx] = (unsigned char)v;
            }
        }
        // far inside a large disc the offset does not matter: then one mask per cut
        bool all = true;
        for (const auto& row : byte)
            for (unsigned char v : row) all &= v == 0xff;
        if (all) return by_offset_.emplace(key, of_axes(0x1111u * ((1u << rows) - 1), 0x0101010101010101ull * ((1u << cols) - 1))).first->second;
        const unsigned id = add();
        for (int reg = 0; reg < 16; ++reg) {
            unsigned long long w = 0;
            const int ky = reg >> 2;
            for (int hh = 0; hh < 2; ++hh) {
                const int kx = 4 * hh + (reg & 3);
                if (ky < rows && kx < cols)
                    for (int qy = 0; qy < kWaveQH; ++qy) w |= (unsigned long long)byte[ky - qy + kWaveQH - 1][kx] << (32 * hh + 8 * qy);
            }
            (*words_)[(size_t)id * 16 + reg] = w;
        }
        by_offset_.emplace(key, id);
        return id;
    }
    // The other masks, a condition per axis: bit 4 qy + ky of row_ok, bit 8 qx + kx of col_ok.
    unsigned of_axes(unsigned row_ok, unsigned long long col_ok)
    {
        const auto key = std::make_pair(col_ok, row_ok);
        auto it = by_axis_.find(key);
        if (it != by_axis_.end()) return it->second;
        // score register `reg` of lane l is query l % 32 of the patch against key 8 (reg / 4) + 4 (l / 32) + reg % 4 of the block
        unsigned queries[kKeyBlockW] = {};  // per key column: the query columns that have it
        for (int kx = 0; kx < kKeyBlockW; ++kx)
            for (int qx = 0; qx < kWaveQW; ++qx) queries[kx] |= (unsigned)(col_ok >> (8 * qx + kx) & 1) << qx;
        const unsigned id = add();
        for (int reg = 0; reg < 16; ++reg) {
            unsigned long long w = 0;
            const int ky = reg >> 2;
            for (int hh = 0; hh < 2; ++hh)
                for (int qy = 0; qy < kWaveQH; ++qy)
                    if (row_ok >> (4 * qy + ky) & 1) w |= (unsigned long long)queries[4 * hh + (reg & 3)] << (32 * hh + 8 * qy);
            (*words_)[(size_t)id * 16 + reg] = w;
        }
        by_axis_.emplace(key, id);
        return id;
    }

  private:
    unsigned add()
    {
        words_->resize(words_->size() + 16);
        return (unsigned)(words_->size() / 16 - 1);
    }
    MaskSpec spec_;
    std::vector<unsigned long long>* words_;
    std::unordered_map<unsigned long long, unsigned> by_offset_;
    std::map<std::pair<unsigned long long, unsigned>, unsigned> by_axis_;
};

// What a patch has to do with the blocks of its query tile's list: per block kOutOfReach, or 1 + the id of its lane masks.  That is
// asked for every patch and listed block (100 x 117 tokens, r = 31: 240 000 times), so a tile's own part of an answer is worked out once
// for all patches (Tile), and answers() is a loop of table reads without branches.
constexpr unsigned kOutOfReach = 0, kUnknown = ~0u;

// The disc.  An answer depends on the offset between patch and block and on how much of either the grid's border cuts off, of which
// there is one amount per axis: a table by offset for each combination of the two cuts, filled as they are met.
class DiscBlocks {
  public:
    struct Tile {
        int at[2];   // of the tile's two blocks: place in a patch's tables for a patch at the origin
        int y0, x0;
    };
    // `questions`: how many there will be
    DiscBlocks(BlockMasks* masks, int gridH, int gridW, long long questions) : masks_(masks), gridH_(gridH), gridW_(gridW)
    {
        const int r = masks->spec().r;
        reach_y_ = imin((r + kWaveQH + kKeyTileH) / kKeyBlockH, ceil_div(gridH, kKeyBlockH)) + 2;
        reach_x_ = imin((r + kWaveQW + kKeyBlockW) / kKeyBlockW, ceil_div(gridW, kKeyBlockW)) + 2;
        pitch_ = 2 * reach_x_ + 1;
        size_ = (2LL * reach_y_ + 1) * pitch_;
        tabled_ = size_ * kTables <= std::max(1LL << 16, questions) && size_ * kTables < (1LL << 30);  // (filling more costs more than it saves)
    }
    Tile tile(int ky0, int kx0) const
    {
        Tile t = {{0, 0}, ky0, kx0};
        for (int kb = 0; kb < 2 && tabled_; ++kb) {
            const int by = ky0 + kKeyBlockH * kb;
            const int table = by >= gridH_ || kx0 >= gridW_ ? kOutside : (by + kKeyBlockH > gridH_ ? 1 : 0) | (kx0 + kKeyBlockW > gridW_ ? 2 : 0);
            t.at[kb] = (int)(table * size_) + by / kKeyBlockH * pitch_ + kx0 / kKeyBlockW;
        }
        return t;
    }
    // for a patch with queries
    void answers(int wy0, int wx0, const std::vector<Tile>& tiles, unsigned* out)
    {
        const MaskSpec& spec = masks_->spec();
        auto ask = [&](const Tile& t, int kb) {
            const int by = t.y0 + kKeyBlockH * kb;
            const int cls = classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, by, t.x0, kKeyBlockH, kKeyBlockW, gridH_, gridW_);
            if (cls == kBlockSkip) return kOutOfReach;
            if (cls == kBlockFull) return 1 + kMaskIdNone;
            return 1 + masks_->of_disc(wy0, wx0, by, t.x0, imin(gridH_ - by, kKeyBlockH), imin(gridW_ - t.x0, kKeyBlockW));
        };
        const size_t n = tiles.size();
        if (!tabled_) {
            for (size_t i = 0; i < n; ++i)
                for (int kb = 0; kb < 2; ++kb) out[2 * i + kb] = ask(tiles[i], kb);
            return;
        }
        std::vector<unsigned>& mine = tables_[(wy0 + kWaveQH > gridH_ ? 1 : 0) | (wx0 + kWaveQW > gridW_ ? 2 : 0)];
        if (mine.empty()) {
            mine.assign((size_t)(kTables * size_), kUnknown);
            std::fill(mine.begin() + (std::ptrdiff_t)(kOutside * size_), mine.end(), kOutOfReach);
        }
        unsigned* const table = mine.data() + (reach_y_ - wy0 / kWaveQH) * pitch_ + reach_x_ - wx0 / kWaveQW;
        const Tile* const tile = tiles.data();
        bool unknown = false;
        for (size_t i = 0; i < n; ++i)
            for (int kb = 0; kb < 2; ++kb) {
                const unsigned answer = table[tile[i].at[kb]];
                out[2 * i + kb] = answer;
                unknown |= answer == kUnknown;
            }
        if (!unknown) return;
        for (size_t i = 0; i < n; ++i)
            for (int kb = 0; kb < 2; ++kb)
                if (out[2 * i + kb] == kUnknown) out[2 * i + kb] = table[tile[i].at[kb]] = ask(tile[i], kb);
    }

  private:
    static_assert(kWaveQH == kKeyBlockH && kWaveQW == kKeyBlockW, "patches and blocks lie on one lattice");
    static constexpr int kOutside = 4, kTables = 5;  // a block's cut: bit 0 rows, bit 1 columns; or wholly outside
    BlockMasks* masks_;
    int gridH_, gridW_, reach_y_, reach_x_, pitch_;
    long long size_;
    bool tabled_;
    std::vector<unsigned> tables_[4];  // by the patch's cut
};

// Masks that are a condition per axis: square, Swin, and the residue classes of the strided mask, in which every pair is admitted (there the
// query grid, qH x qW, and the key grid, kH x kW, may differ by a row or a column).
class AxisBlocks {
  public:
    struct Tile {
        int y, x;  // the tile's first block row, its block column
    };
    AxisBlocks(BlockMasks* masks, int qH, int qW, int kH, int kW) : masks_(masks)
    {
        rows_.build(masks->spec(), qH, kH, kWaveQH, kKeyBlockH);
        cols_.build(masks->spec(), qW, kW, kWaveQW, kKeyBlockW);
        ids_.assign(rows_.bits.size() * cols_.bits.size(), kUnknown);
        for (size_t i = 0; i < rows_.bits.size(); ++i) ids_[i * cols_.bits.size()] = kOutOfReach;
        for (size_t j = 0; j < cols_.bits.size(); ++j) ids_[j] = kOutOfReach;
    }
    Tile tile(int ky0, int kx0) const { return {ky0 / kKeyBlockH, kx0 / kKeyBlockW}; }
    void answers(int wy0, int wx0, const std::vector<Tile>& tiles, unsigned* out)
    {
        const unsigned *const row = rows_.of(wy0 / kWaveQH), *const col = cols_.of(wx0 / kWaveQW);
        const size_t n = tiles.size(), pitch = cols_.bits.size();
        const Tile* const tile = tiles.data();
        unsigned* const ids = ids_.data();
        bool unknown = false;
        for (size_t i = 0; i < n; ++i)
            for (int kb = 0; kb < 2; ++kb) {
                const unsigned answer = ids[row[tile[i].y + kb] * pitch + col[tile[i].x]];
                out[2 * i + kb] = answer;
                unknown |= answer == kUnknown;
            }
        if (!unknown) return;
        for (size_t i = 0; i < n; ++i)
            for (int kb = 0; kb < 2; ++kb) {
                if (out[2 * i + kb] != kUnknown) continue;
                const unsigned ry = row[tile[i].y + kb], rx = col[tile[i].x];
                unsigned& answer = ids[ry * pitch + rx];
                if (answer == kUnknown) {
                    const unsigned long long row_ok = rows_.bits[ry], col_ok = cols_.bits[rx];
                    answer = 1 + (row_ok == 0xffff && col_ok == ~0ull ? kMaskIdNone : masks_->of_axes((unsigned)row_ok, col_ok));
                }
                out[2 * i + kb] = answer;
            }
    }

  private:
    // One axis: per patch and block which condition holds between them, as its place in `bits` (0: no pair is admitted).
    class Axis {
      public:
        std::vector<unsigned long long> bits;  // the distinct conditions: bit (block size) q + k
        void build(const MaskSpec& m, int q_end, int k_end, int q_size, int k_size)
        {
            all_ = m.kind == kMaskFull;  // (the same for every patch)
            const int n_a = all_ ? 1 : ceil_div(q_end, q_size), n_b = ceil_div(k_end, k_size);
            std::vector<int> window;  // Swin
            if (m.kind == kMaskSwin)
                for (int y = 0; y < imax(q_end, k_end) + q_size; ++y) window.push_back((y + m.shift) / m.r);
            auto admits = [&](int q, int k) { return all_ || (m.kind == kMaskSwin ? window[q] == window[k] : axis_admits(m.kind, m.r, m.shift, q, k)); };
            span_ = all_ ? n_b : imin(n_b, (2 * (imin(m.r, q_end + k_end) - 1) + q_size - 1) / k_size + 2);
            first_.assign(n_a, 0);
            code_.assign((size_t)n_a * span_, 0);
            dense_.assign((size_t)n_b + 2, 0);  // (a listed tile may lie in the one row or column that only the larger classes have)
            bits.assign(1, 0);
            std::map<unsigned long long, unsigned> seen;
            for (int a = 0; a < n_a; ++a) {
                const int q0 = a * q_size;
                first_[a] = all_ ? 0 : imin(imax(0, q0 - m.r + 1) / k_size, n_b - span_);
                for (int i = 0; i < span_; ++i) {
                    const int k0 = (first_[a] + i) * k_size;
                    unsigned long long ok = 0;
                    bool any = false;  // a query of the grid has a key
                    for (int q = 0; q < q_size; ++q)
                        for (int k = 0; k < k_size && k0 + k < k_end; ++k)
                            if (admits(q0 + q, k0 + k)) {
                                ok |= 1ull << (k_size * q + k);
                                any |= q0 + q < q_end;
                            }
                    if (!any) continue;
                    const auto known = seen.emplace(ok, (unsigned)bits.size());
                    if (known.second) bits.push_back(ok);
                    code_[(size_t)a * span_ + i] = known.first->second;
                }
            }
        }
        // the conditions of patch a, by block
        const unsigned* of(int a)
        {
            if (all_) a = 0;
            if (a != shown_) {
                if (shown_ >= 0) std::fill_n(dense_.begin() + first_[shown_], span_, 0);
                std::copy_n(code_.begin() + (std::ptrdiff_t)a * span_, span_, dense_.begin() + first_[a]);
                shown_ = a;
            }
            return dense_.data();
        }

      private:
        bool all_ = false;
        int span_ = 0, shown_ = -1;   // blocks kept per patch
        std::vector<int> first_;      // the first of them
        std::vector<unsigned> code_, dense_;
    };
    BlockMasks* masks_;
    Axis rows_, cols_;
    std::vector<unsigned> ids_;  // by the two conditions
};

}  // namespace

QueryTilePatterns query_tile_patterns(const Schedule& s)
{
    // What a query tile's list looks like from its origin depends on where the grid ends, as far as its window or a margin of two key
    // tiles reaches, on its place modulo 4 key tiles (order_forward_tiles) and, for Swin windows, on its place in a window.
    QueryTilePatterns out;
    out.id.resize(s.row_ptr.size() - 1);
    auto axis = [&](int q0, int qt, int kt, int grid) {
        const int margin = s.r + 2 * kt;
        const bool swin = s.mask_kind == kMaskSwin;
        return std::array<int, 4>{imin(q0, margin), imin(grid - q0, qt + margin), q0 % (4 * kt), swin ? (q0 + s.mask_shift) % s.r : 0};
    };
    std::map<std::array<int, 4>, int> rows, cols;
    std::vector<int> row_id(s.n_qty), col_id(s.n_qtx);
    for (int ty = 0; ty < s.n_qty; ++ty) row_id[ty] = rows.emplace(axis(ty * s.qth, s.qth, s.kth, s.gridH), (int)rows.size()).first->second;
    for (int tx = 0; tx < s.n_qtx; ++tx) col_id[tx] = cols.emplace(axis(tx * s.qtw, s.qtw, s.ktw, s.gridW), (int)cols.size()).first->second;
    std::vector<int> seen(rows.size() * cols.size(), -1);
    for (int ty = 0; ty < s.n_qty; ++ty)
        for (int tx = 0; tx < s.n_qtx; ++tx) {
            int& id = seen[(size_t)row_id[ty] * cols.size() + col_id[tx]];
            if (id < 0) {
                id = (int)out.first.size();
                out.first.push_back(ty * s.n_qtx + tx);
            }
            out.id[(size_t)ty * s.n_qtx + tx] = id;
        }
    return out;
}

void order_forward_tiles(const Schedule& s, const QueryTilePatterns& pat, std::vector<int>* k_col)
{
    struct Pair {
        int key, a, b;  // b: -1 without a partner
    };
    constexpr int kKeys = 16;  // places modulo 4 x 4; tiles without a partner follow, by the same key
    std::vector<Pair> pairs;
    std::vector<unsigned char> listed((size_t)s.n_kty * s.n_ktx, 0);
    k_col->assign(s.col_idx.size(), 0);
    auto mod4 = [](int a) { return a & 3; };
    for (int qt : pat.first) {
        const int begin = s.row_ptr[qt], end = s.row_ptr[qt + 1];
        for (int e = begin; e < end; ++e) listed[s.col_idx[e]] = 1;
        // twice the centre of the query tile, in key tiles, less one: a tile (y, x) and its mirror add up to it
        const int cy2 = 2 * (qt / s.n_qtx) * s.qth + s.qth - s.kth, cx2 = 2 * (qt % s.n_qtx) * s.qtw + s.qtw - s.ktw;
        const bool on_tiles = cy2 % s.kth == 0 && cx2 % s.ktw == 0;
        pairs.clear();
        int place[2 * kKeys + 1] = {};  // where the tiles of a key go
        for (int e = begin; e < end; ++e) {
            const int id = s.col_idx[e];
            if (listed[id] != 1) continue;
            const int y = id / s.n_ktx, x = id - y * s.n_ktx, my = cy2 / s.kth - y, mx = cx2 / s.ktw - x;
            const int mirror = on_tiles && my >= 0 && mx >= 0 && my < s.n_kty && mx < s.n_ktx ? my * s.n_ktx + mx : -1;
            Pair p = {0, id, -1};
            listed[id] = 2;
            if (mirror >= 0 && listed[mirror] == 1) {
                listed[mirror] = 2;
                p.b = mirror;
            }
            p.key = imin(mod4(y) * 4 + mod4(x), mod4(1 - y) * 4 + mod4(1 - x)) + (p.b < 0 ? kKeys : 0);
            place[p.key + 1] += p.b >= 0 ? 2 : 1;
            pairs.push_back(p);
        }
        for (int k = 0; k < 2 * kKeys; ++k) place[k + 1] += place[k];
        auto origin = [&](int id) { return (id / s.n_ktx) * s.kth << 16 | (id % s.n_ktx) * s.ktw; };
        for (const Pair& p : pairs) {
            int* const to = k_col->data() + begin + place[p.key];
            to[0] = origin(p.a);
            if (p.b >= 0) to[1] = origin(p.b);
            place[p.key] += p.b >= 0 ? 2 : 1;
        }
        for (int e = begin; e < end; ++e) listed[s.col_idx[e]] = 0;
    }
    for (size_t qt = 0; qt + 1 < s.row_ptr.size(); ++qt) {
        const int rep = pat.first[pat.id[qt]];
        if ((int)qt == rep) continue;
        // the same list, moved (rows and columns in one addition: neither half leaves its 16 bits)
        const int by = ((int)(qt / s.n_qtx) - rep / s.n_qtx) * s.qth * 65536 + ((int)(qt % s.n_qtx) - rep % s.n_qtx) * s.qtw;
        for (int e = s.row_ptr[qt], f = s.row_ptr[rep]; e < s.row_ptr[qt + 1]; ++e, ++f) (*k_col)[e] = (*k_col)[f] + by;
    }
}

namespace {

// The image-query programs of one table set and variant (of the key grid's extents), appended to out->words; out->ptr of the variant, and the
// words of a pattern's waves.
template <int GROUPS, class Blocks>
void build_image_programs(const ProgramInput& in, int n_text, int head_dim, Blocks& blocks, unsigned* ptr, std::vector<unsigned>* words, std::vector<double>* steps_of,
                          std::vector<unsigned>* blocks_of)
{
    const Schedule& s = *in.sched;
    const int waves = kBf16NWY * kBf16NWX, patches = waves / GROUPS, tps = bf16_tiles_per_stage(head_dim);
    const int tile_units = kKeyTileKeys * head_dim * 2 / 2048;  // a staged K (or V) tile in the units of kProgramPlaceMask
    const int n_lin_stages = ceil_div(ceil_div(n_text, kKeyTileKeys), tps);
    int most = 0;  // the longest list
    size_t at_most = 0;  // words
    for (int qt : in.pat->first) {
        const int n_img = s.row_ptr[qt + 1] - s.row_ptr[qt];
        most = imax(most, n_img);
        at_most += (size_t)(n_lin_stages + ceil_div(n_img, tps)) * 2 * tps * waves;
    }
    words->reserve(words->size() + std::min<size_t>(at_most, 1u << 22));
    std::vector<typename Blocks::Tile> tiles;
    std::vector<unsigned> answers((size_t)most * 2);
    const size_t room = (size_t)(n_lin_stages + ceil_div(most, tps)) * 2 * tps + 1;  // (a word may be written past the last and not kept)
    std::vector<unsigned> scratch(room * GROUPS);                                    // the programs of the waves that share a patch
    unsigned *end[GROUPS], *had[GROUPS];
    for (int g = 0; g < GROUPS; ++g) end[g] = scratch.data() + (size_t)g * room;
    unsigned turn = 0;  // the waves of a patch take its blocks in turn
    int idle_words[GROUPS] = {};
    auto put = [&](unsigned word, bool reached) __attribute__((always_inline)) {
        *end[turn] = word;  // (without a branch: the edge of a disc cannot be foreseen)
        end[turn] += reached;
        turn = (turn + reached) % GROUPS;
    };
    auto begin_stage = [&]() __attribute__((always_inline)) {
        for (int g = 0; g < GROUPS; ++g) had[g] = end[g];
    };
    auto end_stage = [&]() __attribute__((always_inline)) {
        for (int g = 0; g < GROUPS; ++g) {
            if (end[g] == had[g]) {
                // no block here: one that masks everything finishes what the wave has pending, after that nothing is left to do
                const bool idle = had[g] > scratch.data() + (size_t)g * room && ((had[g][-1] & ~kProgramFlags) >> kProgramMaskShift) == kMaskIdNothing;
                *end[g]++ = kMaskIdNothing << kProgramMaskShift | (idle ? kProgramNoBlock : 0);
                idle_words[g] += idle;
            }
            end[g][-1] |= kProgramStageEnd;
        }
    };
    // the text keys' stages, the same for every patch
    for (int st = 0; st < n_lin_stages; ++st) {
        begin_stage();
        for (int j = 0; j < tps; ++j)
            for (int kb = 0; kb < 2; ++kb) {
                const int left = n_text - ((st * tps + j) * 2 + kb) * 32;
                if (left > 0) put((unsigned)(j * tile_units + kb) | (left >= 32 ? kMaskIdNone : kMaskIdFirstKeys + (unsigned)left) << kProgramMaskShift, true);
            }
        end_stage();
    }
    unsigned* text_end[GROUPS];
    int text_idle[GROUPS];
    for (int g = 0; g < GROUPS; ++g) {
        text_end[g] = end[g];
        text_idle[g] = idle_words[g];
    }
    const unsigned text_turn = turn;
    struct Piece {
        size_t at, size;
    };
    std::vector<Piece> last((size_t)waves, Piece{0, 0});  // the waves' programs before this one
    for (size_t k = 0; k < in.pat->first.size(); ++k) {
        const size_t qt = in.pat->first[k];
        const int begin = s.row_ptr[qt], n_img = s.row_ptr[qt + 1] - begin;
        tiles.clear();
        for (int e = begin; e < begin + n_img; ++e) tiles.push_back(blocks.tile((*in.k_col)[e] >> 16, (*in.k_col)[e] & 0xffff));
        for (int patch = 0; patch < patches; ++patch) {
            const int wy0 = (int)(qt / s.n_qtx) * s.qth + (patch / kBf16NWX) * kWaveQH, wx0 = (int)(qt % s.n_qtx) * s.qtw + (patch % kBf16NWX) * kWaveQW;
            const bool queries = wy0 < s.gridH && wx0 < s.gridW;  // (a wave without any follows no program; the mean of the steps counts it as out of reach of every block)
            if (queries)
                blocks.answers(wy0, wx0, tiles, answers.data());
            else
                std::fill(answers.begin(), answers.end(), kOutOfReach);
            for (int g = 0; g < GROUPS; ++g) {
                end[g] = text_end[g];
                idle_words[g] = text_idle[g];
            }
            turn = text_turn;
            const unsigned* answer = answers.data();
            for (int first = 0; first < n_img; first += tps) {
                begin_stage();
                const int n = imin(tps, n_img - first);
                for (int j = 0; j < n; ++j)
                    for (int kb = 0; kb < 2; ++kb, ++answer) put((unsigned)(j * tile_units + kb) | (*answer - 1) << kProgramMaskShift, *answer != kOutOfReach);
                end_stage();
            }
            for (int g = 0; g < GROUPS; ++g) {
                const unsigned *const from = scratch.data() + (size_t)g * room, *const to = end[g];
                const int wave = g * patches + patch;
                const size_t size = (size_t)(to - from);
                (*steps_of)[k] += (double)size;
                if (!queries) continue;
                (*blocks_of)[k * waves + wave] = (unsigned)size - (unsigned)idle_words[g];
                // Waves whose programs are the same share one: those of a class of the strided mask, or of a window that holds the whole grid.
                const Piece candidates[2] = {last[wave], last[wave > 0 ? wave - 1 : 0]};
                const Piece* same = nullptr;
                for (const Piece& c : candidates)
                    if (!same && c.size == size && std::equal(from, to, words->begin() + (std::ptrdiff_t)c.at)) same = &c;
                if (same) {
                    last[wave] = *same;
                } else {
                    last[wave] = {words->size(), size};
                    words->insert(words->end(), from, to);
                    if (words->size() > kMaxProgramWords) throw std::bad_alloc();  // (places in it are 32-bit numbers)
                }
                ptr[qt * waves + wave] = (unsigned)last[wave].at;
            }
        }
    }
}

// The words of a text-query stage, for every number of keys left and wave of a patch.
void build_text_words(int head_dim, BlockPrograms* out)
{
    const int tps = bf16_tiles_per_stage(head_dim), tile_units = kKeyTileKeys * head_dim * 2 / 2048;
    // text-query rows: every stage holds the same blocks, the last one as many as there are keys left
    const int stage_blocks = 2 * tps;
    for (int i = 0; i < 3; ++i) {
        const int waves_per_patch = 1 << i, per = stage_blocks / waves_per_patch;
        out->text_words[i] = (unsigned)out->words.size();
        for (int g = 0; g < waves_per_patch; ++g)
            for (int keys = 0; keys <= tps * kKeyTileKeys; ++keys) {
                int used = 0;
                for (int k = 0; k < per; ++k) {
                    const int b = k * waves_per_patch + g, left = keys == 0 ? 32 : keys - 32 * b;
                    if (left <= 0 && k > 0) break;
                    // (a wave without a key left names the stage's first block: its own lies in a tile that is not staged)
                    const unsigned id = left >= 32 ? kMaskIdNone : left > 0 ? kMaskIdFirstKeys + (unsigned)left : kMaskIdNothing;
                    const unsigned place = left > 0 ? (unsigned)((b >> 1) * tile_units + (b & 1)) : 0;
                    out->words.push_back(place | id << kProgramMaskShift);
                    ++used;
                }
                out->words.back() |= kProgramStageEnd;
                for (; used < per; ++used) out->words.push_back(0);
            }
    }
    out->words.insert(out->words.end(), kProgramSpareWords, 0u);
}

}  // namespace

void build_block_programs(const std::vector<ProgramInput>& in, int n_text, int head_dim, int stride, int gridH, int gridW,
                          std::vector<BlockPrograms>* out, std::vector<unsigned long long>* masks)
{
    const Schedule& s = *in[0].sched;  // (the sets differ in the height of their query tiles only)
    const bool strided = stride > 1;
    const int waves = kBf16NWY * kBf16NWX, tps = bf16_tiles_per_stage(head_dim), n_variants = strided ? 4 : 1;
    BlockMasks set({strided ? (int)kMaskFull : s.mask_kind, s.r, s.mask_shift}, masks);
    out->resize(in.size());
    std::vector<double> steps(in.size(), 0.0);
    for (size_t i = 0; i < in.size(); ++i) {
        (*out)[i].words.clear();
        (*out)[i].ptr.assign((size_t)n_variants * (in[i].sched->row_ptr.size() - 1) * waves, 0);
    }
    int n_built = 0;
    for (int v = 0; v < n_variants; ++v) {
        // (the larger class of an axis exists where the stride does not divide it)
        if (strided && (((v >> 1) && gridH % stride == 0) || ((v & 1) && gridW % stride == 0))) continue;
        ++n_built;
        auto run = [&](auto&& blocks) {
            for (size_t i = 0; i < in.size(); ++i) {
                BlockPrograms& o = (*out)[i];
                const QueryTilePatterns& pat = *in[i].pat;
                const size_t n_q_tiles = in[i].sched->row_ptr.size() - 1;
                unsigned* const ptr = o.ptr.data() + (size_t)v * n_q_tiles * waves;
                std::vector<double> steps_of(pat.first.size(), 0);
                std::vector<unsigned> blocks_of(pat.first.size() * waves, 0);
                if (in[i].groups == 1) build_image_programs<1>(in[i], n_text, head_dim, blocks, ptr, &o.words, &steps_of, &blocks_of);
                if (in[i].groups == 2) build_image_programs<2>(in[i], n_text, head_dim, blocks, ptr, &o.words, &steps_of, &blocks_of);
                if (in[i].groups == 4) build_image_programs<4>(in[i], n_text, head_dim, blocks, ptr, &o.words, &steps_of, &blocks_of);
                for (size_t qt = 0; qt < n_q_tiles; ++qt) {
                    const size_t first = pat.first[pat.id[qt]];
                    if (first != qt) std::copy(ptr + first * waves, ptr + (first + 1) * waves, ptr + qt * waves);
                    steps[i] += steps_of[pat.id[qt]];
                }
                // executed blocks, of the waves that have queries (of a class of either extent)
                if (in[i].groups > 1) continue;
                std::vector<unsigned long long> blocks_in(pat.first.size(), 0);
                for (size_t j = 0; j < blocks_of.size(); ++j) blocks_in[j / waves] += blocks_of[j];
                for (int u = 0; u < n_variants; ++u)
                    for (size_t qt = 0; qt < n_q_tiles; ++qt) {
                        if (!strided) {
                            o.blocks[v][u] += blocks_in[pat.id[qt]];
                            continue;
                        }
                        const Schedule& sc = *in[i].sched;
                        for (int w = 0; w < waves; ++w) {
                            const int wy0 = (int)(qt / sc.n_qtx) * sc.qth + (w / kBf16NWX) * kWaveQH, wx0 = (int)(qt % sc.n_qtx) * sc.qtw + (w % kBf16NWX) * kWaveQW;
                            if (wy0 < gridH / stride + (u >> 1) && wx0 < gridW / stride + (u & 1)) o.blocks[v][u] += blocks_of[(size_t)pat.id[qt] * waves + w];
                        }
                    }
            }
        };
        if (set.spec().kind == kMaskDisc) {
            long long questions = 0;
            for (const ProgramInput& p : in)
                for (int qt : p.pat->first) questions += (p.sched->row_ptr[qt + 1] - p.sched->row_ptr[qt]) * 2LL * (waves / p.groups);
            run(DiscBlocks(&set, s.gridH, s.gridW, questions));
        } else {
            run(AxisBlocks(&set, s.gridH, s.gridW, strided ? gridH / stride + (v >> 1) : s.gridH, strided ? gridW / stride + (v & 1) : s.gridW));
        }
    }
    for (size_t i = 0; i < in.size(); ++i) {
        const std::vector<int>& row_ptr = in[i].sched->row_ptr;
        const size_t n_q_tiles = row_ptr.size() - 1;
        double stages = 0;
        for (size_t qt = 0; qt < n_q_tiles; ++qt) stages += ceil_div(ceil_div(n_text, kKeyTileKeys), tps) + ceil_div(row_ptr[qt + 1] - row_ptr[qt], tps);
        (*out)[i].mean_stages = stages / (double)n_q_tiles;
        (*out)[i].mean_steps = steps[i] / ((double)n_built * n_q_tiles * waves);
        build_text_words(head_dim, &(*out)[i]);
    }
}

unsigned long long executed_pairs_bf16(const BlockPrograms& prog, int n_text, int gridH, int gridW, int stride, int layer)
{
    const long long N = (long long)n_text + (long long)gridH * gridW;
    unsigned long long blocks = 0;  // (32 query x 32 key) blocks
    if (stride == 1) {
        blocks = prog.blocks[0][0];
    } else {
        const int rx = layer % stride, ry = (layer / stride) % stride;
        auto larger = [&](int n, int a) { return a < n % stride; };  // whether class a of an axis has the larger extent
        for (int b = 0; b < stride; ++b)
            for (int a = 0; a < stride; ++a)
                blocks += prog.blocks[2 * larger(gridH, (b + ry) % stride) + larger(gridW, (a + rx) % stride)][2 * larger(gridH, b) + larger(gridW, a)];
    }
    // text-query rows: every wave that holds at least one text query visits every 32-key block of [0, N)
    blocks += (unsigned long long)ceil_div(n_text, kTextQueriesPerWave) * (unsigned long long)((N + 31) / 32);
    return blocks * 1024ull;
}

unsigned long long executed_pairs_f32(const Schedule& s, int n_text)
{
    const long long N = (long long)n_text + (long long)s.gridH * s.gridW;
    const MaskSpec spec = {s.mask_kind, s.r, s.mask_shift};
    constexpr int kSide = 4, kCell = kSide * kSide;  // 4 x 4 query patches against cells of 16 keys
    const unsigned long long text_cells = (unsigned long long)ceil_div(n_text, kCell);
    unsigned long long cells = text_cells * (unsigned long long)((N + kCell - 1) / kCell);  // text queries meet every cell of [0, N)
    for (size_t qt = 0; qt + 1 < s.row_ptr.size(); ++qt)
        for (int y0 = (int)(qt / s.n_qtx) * s.qth, ye = imin(y0 + s.qth, s.gridH); y0 < ye; y0 += kSide)
            for (int x0 = (int)(qt % s.n_qtx) * s.qtw, xe = imin(x0 + s.qtw, s.gridW); x0 < xe; x0 += kSide) {
                cells += text_cells;
                for (int e = s.row_ptr[qt]; e < s.row_ptr[qt + 1]; ++e)
                    for (int c = 0; c < kKeyTileKeys / kCell; ++c) {
                        const int ky0 = (s.col_idx[e] / s.n_ktx) * s.kth + kSide * (c >> 1), kx0 = (s.col_idx[e] % s.n_ktx) * s.ktw + kSide * (c & 1);
                        cells += classify_image_block_spec(spec, y0, x0, kSide, kSide, ky0, kx0, kSide, kSide, s.gridH, s.gridW) != kBlockSkip;
                    }
            }
    return cells * kCell * kCell;
}

}  // namespace clear
