// Host-side integer geometry of the CLEAR mask (Eq. 3, Sec. 3.2): tile schedule, sum(M), and the
// count of pairs the kernels execute.  No device code here.
#include "block_class.h"
#include "clear_internal.h"

#include <algorithm>
#include <array>
#include <map>
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

unsigned long long executed_pairs_bf16(const Schedule& s, int n_text, int text_split_keys, bool whole_tiles)
{
    (void)text_split_keys;  // splits are multiples of the 64-key stage: the block count does not depend on them
    const long long N = (long long)n_text + (long long)s.gridH * s.gridW;
    unsigned long long blocks = 0;  // executed (32 query x 32 key) blocks
    const int n_text_tiles = ceil_div(n_text, kKeyTileKeys);
    const int nwy = s.qth / kWaveQH, nwx = s.qtw / kWaveQW;
    const MaskSpec spec = {s.mask_kind, s.r, s.mask_shift};
    for (int ty = 0; ty < s.n_qty; ++ty)
        for (int tx = 0; tx < s.n_qtx; ++tx) {
            const int qt = ty * s.n_qtx + tx;
            for (int wy = 0; wy < nwy; ++wy)
                for (int wx = 0; wx < nwx; ++wx) {
                    const int y0 = ty * s.qth + wy * kWaveQH, x0 = tx * s.qtw + wx * kWaveQW;
                    if (y0 >= s.gridH || x0 >= s.gridW) continue;  // wave has no query: it computes nothing
                    if (whole_tiles)
                        blocks += 2ull * n_text_tiles;
                    else
                        blocks += ceil_div(n_text, 32);
                    for (int e = s.row_ptr[qt]; e < s.row_ptr[qt + 1]; ++e) {
                        const int ky0 = (s.col_idx[e] / s.n_ktx) * s.kth, kx0 = (s.col_idx[e] % s.n_ktx) * s.ktw;
                        int reached = 0;
                        for (int kb = 0; kb < 2; ++kb)
                            reached += classify_image_block_spec(spec, y0, x0, kWaveQH, kWaveQW, ky0 + kKeyBlockH * kb, kx0, kKeyBlockH,
                                                                 kKeyBlockW, s.gridH, s.gridW) != kBlockSkip;
                        blocks += whole_tiles ? 2 * (reached > 0) : reached;
                    }
                }
        }
    // text-query pass: every wave that holds at least one text query visits every 32-key block of [0, N)
    const unsigned long long text_waves = (unsigned long long)ceil_div(n_text, kTextQueriesPerWave);
    blocks += whole_tiles ? text_waves * 2ull * (unsigned long long)((N + kKeyTileKeys - 1) / kKeyTileKeys) : text_waves * (unsigned long long)((N + 31) / 32);
    return blocks * 1024ull;
}

namespace {

// Lane masks of (4 x 8 query patch, 4 x 8 key block) pairs, each distinct one kept once.
class BlockMasks {
  public:
    BlockMasks(const MaskSpec& spec, std::vector<unsigned long long>* words) : spec_(spec), words_(words)
    {
        words_->assign((size_t)kMaskIdFree * 16, 0ull);
        for (int reg = 0; reg < 16; ++reg) (*words_)[(size_t)kMaskIdNone * 16 + reg] = ~0ull;
        // block offsets that a patch and a block of a listed tile can have
        reach_y_ = (spec.r + kWaveQH + kKeyTileKeys / kKeyBlockW) / kKeyBlockH + 1;
        reach_x_ = (spec.r + kWaveQW + kKeyBlockW) / kKeyBlockW;
        const size_t offsets = (size_t)(2 * reach_y_ + 1) * (2 * reach_x_ + 1);
        if (spec.kind == kMaskDisc && offsets <= (1u << 16)) whole_.assign(offsets, 0);
        for (int k = 1; k < 32; ++k)
            for (int reg = 0; reg < 16; ++reg) {
                const int key = 8 * (reg >> 2) + (reg & 3);  // of the lower lanes; the upper lanes hold the key 4 further on
                (*words_)[(size_t)(kMaskIdFirstKeys + k) * 16 + reg] = (key < k ? 0xffffffffull : 0) | (key + 4 < k ? 0xffffffffull << 32 : 0);
            }
    }
    // The disc's mask id for a patch and a block that lie inside the grid, by the offset between them (both are aligned to blocks), or
    // kOutOfReach; has_table(): whether that offset, and the one of the block below it, have a place in the table.
    static constexpr unsigned kOutOfReach = ~0u;
    bool has_table(int dy, int dx) const
    {
        return !whole_.empty() && abs(dy) < (reach_y_ - 1) * kKeyBlockH && abs(dx) < reach_x_ * kKeyBlockW;
    }
    unsigned of_whole(int dy, int dx)
    {
        unsigned& slot = whole_[(size_t)(dy / kKeyBlockH + reach_y_) * (2 * reach_x_ + 1) + dx / kKeyBlockW + reach_x_];
        if (slot == 0) {
            constexpr int far = 1 << 20;  // a grid without borders
            const int cls = classify_image_block(far / 2, far / 2, kWaveQH, kWaveQW, far / 2 + dy, far / 2 + dx, kKeyBlockH, kKeyBlockW, far, far, spec_.r * spec_.r);
            slot = cls == kBlockSkip ? kOutOfReach : 1 + (cls == kBlockFull ? kMaskIdNone : id(far / 2, far / 2, far / 2 + dy, far / 2 + dx, kKeyBlockH, kKeyBlockW));
        }
        return slot == kOutOfReach ? kOutOfReach : slot - 1;
    }
    // The mask of a patch at (wy0, wx0) against a block at (ky0, kx0) of which the first `rows` rows and `cols` columns are keys.
    unsigned id(int wy0, int wx0, int ky0, int kx0, int rows, int cols)
    {
        if (spec_.kind == kMaskDisc) {
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
        // the other masks are a condition per axis
        unsigned row_ok = 0;
        unsigned long long col_ok = 0;
        const bool all = spec_.kind == kMaskFull;
        for (int q = 0; q < kWaveQH; ++q)
            for (int k = 0; k < rows; ++k)
                if (all || axis_admits(spec_.kind, spec_.r, spec_.shift, wy0 + q, ky0 + k)) row_ok |= 1u << (4 * q + k);
        for (int q = 0; q < kWaveQW; ++q)
            for (int k = 0; k < cols; ++k)
                if (all || axis_admits(spec_.kind, spec_.r, spec_.shift, wx0 + q, kx0 + k)) col_ok |= 1ull << (8 * q + k);
        const auto key = std::make_pair(col_ok, row_ok);
        auto it = by_axis_.find(key);
        if (it != by_axis_.end()) return it->second;
        const unsigned id = add();
        fill(id, [&](int qy, int qx, int ky, int kx) { return (row_ok >> (4 * qy + ky) & 1) && (col_ok >> (8 * qx + kx) & 1); });
        by_axis_.emplace(key, id);
        return id;
    }

  private:
    unsigned add()
    {
        words_->resize(words_->size() + 16);
        return (unsigned)(words_->size() / 16 - 1);
    }
    // Score register `reg` of lane l is query l % 32 of the patch against key 8 (reg / 4) + 4 (l / 32) + reg % 4 of the block.
    template <typename F>
    void fill(size_t id, F admits)
    {
        for (int reg = 0; reg < 16; ++reg) {
            unsigned long long w = 0;
            for (int l = 0; l < 64; ++l)
                if (admits((l & 31) >> 3, l & 7, reg >> 2, 4 * (l >> 5) + (reg & 3))) w |= 1ull << l;
            (*words_)[id * 16 + reg] = w;
        }
    }
    MaskSpec spec_;
    std::vector<unsigned long long>* words_;
    int reach_y_, reach_x_;
    std::vector<unsigned> whole_;
    std::unordered_map<unsigned long long, unsigned> by_offset_;
    std::map<std::pair<unsigned long long, unsigned>, unsigned> by_axis_;
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
        for (int e = begin; e < end; ++e) {
            const int id = s.col_idx[e];
            if (listed[id] != 1) continue;
            const int y = id / s.n_ktx, x = id % s.n_ktx, my = cy2 / s.kth - y, mx = cx2 / s.ktw - x;
            const int mirror = on_tiles && my >= 0 && mx >= 0 && my < s.n_kty && mx < s.n_ktx ? my * s.n_ktx + mx : -1;
            Pair p = {0, id, -1};
            listed[id] = 2;
            if (mirror >= 0 && listed[mirror] == 1) {
                listed[mirror] = 2;
                p.b = mirror;
            }
            p.key = imin(mod4(y) * 4 + mod4(x), mod4(1 - y) * 4 + mod4(1 - x));
            pairs.push_back(p);
        }
        std::stable_sort(pairs.begin(), pairs.end(), [](const Pair& p, const Pair& q) { return (p.b < 0) != (q.b < 0) ? q.b < 0 : p.key < q.key; });
        int w = begin;
        auto put = [&](int id) { (*k_col)[w++] = (id / s.n_ktx) * s.kth << 16 | (id % s.n_ktx) * s.ktw; };
        for (const Pair& p : pairs) {
            put(p.a);
            if (p.b >= 0) put(p.b);
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

static void build_block_programs_for(const Schedule& s, const QueryTilePatterns& pat, const std::vector<int>& k_col, int n_text, int head_dim, int groups,
                                     int stride, int gridH, int gridW, BlockMasks& masks, BlockPrograms* out)
{
    const bool strided = stride > 1;
    const int waves = kBf16NWY * kBf16NWX, patches = waves / groups, tps = bf16_tiles_per_stage(head_dim);
    const int tile_units = kKeyTileKeys * head_dim * 2 / 2048;  // a staged K (or V) tile in the units of kProgramPlaceMask
    const size_t n_q_tiles = s.row_ptr.size() - 1;
    const MaskSpec spec = {strided ? (int)kMaskFull : s.mask_kind, s.r, s.mask_shift};
    const int n_variants = strided ? 4 : 1;
    out->ptr.resize((size_t)n_variants * n_q_tiles * waves);
    out->words.clear();
    std::vector<unsigned> scratch;
    const int n_lin_tiles = ceil_div(n_text, kKeyTileKeys), n_lin_stages = ceil_div(n_lin_tiles, tps);
    double all_stages = 0, all_steps = 0;
    for (int v = 0; v < n_variants; ++v) {
        const int kH = strided ? gridH / stride + (v >> 1) : s.gridH, kW = strided ? gridW / stride + (v & 1) : s.gridW;
        std::vector<double> steps_of(pat.first.size(), 0);
        for (size_t k = 0; k < pat.first.size(); ++k) {
            const size_t qt = pat.first[k];
            const int n_img = s.row_ptr[qt + 1] - s.row_ptr[qt], n_stages = n_lin_stages + ceil_div(n_img, tps);
            const size_t room = (size_t)n_stages * 2 * tps;
            scratch.resize(room * groups);
            for (int patch = 0; patch < patches; ++patch) {
                const int wy0 = (int)(qt / s.n_qtx) * s.qth + (patch / kBf16NWX) * kWaveQH, wx0 = (int)(qt % s.n_qtx) * s.qtw + (patch % kBf16NWX) * kWaveQW;
                const bool inside_patch = wy0 + kWaveQH <= s.gridH && wx0 + kWaveQW <= s.gridW;
                unsigned* end[4];
                for (int g = 0; g < groups; ++g) end[g] = scratch.data() + (size_t)g * room;
                unsigned turn = 0;
                auto put = [&](unsigned place, unsigned id) { *end[turn++ & (unsigned)(groups - 1)]++ = place | id << kProgramMaskShift; };
                for (int st = 0; st < n_stages; ++st) {
                    unsigned* const had[4] = {end[0], end[1], end[2], end[3]};
                    const int first = st < n_lin_stages ? st * tps : (st - n_lin_stages) * tps, last = imin(first + tps, st < n_lin_stages ? n_lin_tiles : n_img);
                    for (int i = first; i < last; ++i) {
                        const unsigned place = (unsigned)((i - first) * tile_units);
                        if (st < n_lin_stages) {
                            for (int kb = 0; kb < 2; ++kb) {
                                const int left = n_text - (i * 2 + kb) * 32;
                                if (left > 0) put(place + kb, left >= 32 ? kMaskIdNone : kMaskIdFirstKeys + (unsigned)left);
                            }
                            continue;
                        }
                        const int packed = k_col[s.row_ptr[qt] + i], ky0 = packed >> 16, kx0 = packed & 0xffff;
                        if (inside_patch && ky0 + s.kth <= kH && kx0 + s.ktw <= kW && masks.has_table(ky0 - wy0, kx0 - wx0)) {
                            for (int kb = 0; kb < 2; ++kb) {
                                const unsigned id = masks.of_whole(ky0 - wy0 + kKeyBlockH * kb, kx0 - wx0);
                                if (id != BlockMasks::kOutOfReach) put(place + kb, id);
                            }
                            continue;
                        }
                        for (int kb = 0; kb < 2; ++kb) {
                            const int by = ky0 + kKeyBlockH * kb;
                            const int cls = strided ? classify_full_block(wy0, wx0, s.gridH, s.gridW, by, kx0, kKeyBlockH, kKeyBlockW, kH, kW)
                                                    : classify_image_block_spec(spec, wy0, wx0, kWaveQH, kWaveQW, by, kx0, kKeyBlockH, kKeyBlockW, kH, kW);
                            if (cls == kBlockSkip) continue;
                            put(place + kb, cls == kBlockFull ? kMaskIdNone : masks.id(wy0, wx0, by, kx0, imin(kH - by, kKeyBlockH), imin(kW - kx0, kKeyBlockW)));
                        }
                    }
                    for (int g = 0; g < groups; ++g) {
                        if (end[g] == had[g]) {
                            // no block here: one that masks everything finishes what the wave has pending, after that nothing is left to do
                            const bool idle = had[g] > scratch.data() + (size_t)g * room && ((had[g][-1] & ~kProgramFlags) >> kProgramMaskShift) == kMaskIdNothing;
                            *end[g]++ = kMaskIdNothing << kProgramMaskShift | (idle ? kProgramNoBlock : 0);
                        }
                        end[g][-1] |= kProgramStageEnd;
                    }
                }
                for (int g = 0; g < groups; ++g) {
                    const unsigned* const begin = scratch.data() + (size_t)g * room;
                    steps_of[k] += (double)(end[g] - begin);
                    out->ptr[((size_t)v * n_q_tiles + qt) * waves + g * patches + patch] = (unsigned)out->words.size();
                    out->words.insert(out->words.end(), begin, (const unsigned*)end[g]);
                }
            }
        }
        for (size_t qt = 0; qt < n_q_tiles; ++qt) {
            const int k = pat.id[qt];
            unsigned* const of_variant = out->ptr.data() + (size_t)v * n_q_tiles * waves;
            if (pat.first[k] != (int)qt) std::copy(of_variant + (size_t)pat.first[k] * waves, of_variant + (size_t)(pat.first[k] + 1) * waves, of_variant + qt * waves);
            all_stages += n_lin_stages + ceil_div(s.row_ptr[qt + 1] - s.row_ptr[qt], tps);
            all_steps += steps_of[k];
        }
    }
    out->mean_stages = all_stages / (double)(n_variants * n_q_tiles);
    out->mean_steps = all_steps / (double)(n_variants * n_q_tiles * waves);
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
    out->words.push_back(0);
    out->words.push_back(0);
}

void build_block_programs(const std::vector<ProgramInput>& in, int n_text, int head_dim, int stride, int gridH, int gridW,
                          std::vector<BlockPrograms>* out, std::vector<unsigned long long>* masks)
{
    const Schedule& s = *in[0].sched;
    BlockMasks set({stride > 1 ? (int)kMaskFull : s.mask_kind, s.r, s.mask_shift}, masks);
    out->resize(in.size());
    for (size_t i = 0; i < in.size(); ++i)
        build_block_programs_for(*in[i].sched, *in[i].pat, *in[i].k_col, n_text, head_dim, in[i].groups, stride, gridH, gridW, set, &(*out)[i]);
}

unsigned long long executed_pairs_bf16_strided(const Schedule& s, int n_text, int gridH, int gridW, int stride, int layer)
{
    const long long N = (long long)n_text + (long long)gridH * gridW;
    const int rx = layer % stride, ry = (layer / stride) % stride;
    const int n_text_tiles = ceil_div(n_text, kKeyTileKeys);
    const int nwy = s.qth / kWaveQH, nwx = s.qtw / kWaveQW;
    auto extent = [&](int n, int a) { return a < n ? (n - a + stride - 1) / stride : 0; };
    unsigned long long blocks = 0;
    for (int b = 0; b < stride; ++b)
        for (int a = 0; a < stride; ++a) {
            const int qH = extent(gridH, b), qW = extent(gridW, a);
            const int kH = extent(gridH, (b + ry) % stride), kW = extent(gridW, (a + rx) % stride);
            for (int ty = 0; ty < s.n_qty; ++ty)
                for (int tx = 0; tx < s.n_qtx; ++tx) {
                    const int qt = ty * s.n_qtx + tx;
                    for (int wy = 0; wy < nwy; ++wy)
                        for (int wx = 0; wx < nwx; ++wx) {
                            const int y0 = ty * s.qth + wy * kWaveQH, x0 = tx * s.qtw + wx * kWaveQW;
                            if (y0 >= qH || x0 >= qW) continue;
                            for (int t = 0; t < n_text_tiles; ++t)
                                blocks += 2 * (classify_linear_block((long long)t * kKeyTileKeys, 32, n_text) != kBlockSkip);
                            for (int e = s.row_ptr[qt]; e < s.row_ptr[qt + 1]; ++e) {
                                const int ky0 = (s.col_idx[e] / s.n_ktx) * s.kth, kx0 = (s.col_idx[e] % s.n_ktx) * s.ktw;
                                bool any = false;
                                for (int kb = 0; kb < 2; ++kb)
                                    any |= classify_full_block(y0, x0, qH, qW, ky0 + kKeyBlockH * kb, kx0, kKeyBlockH, kKeyBlockW, kH, kW) != kBlockSkip;
                                blocks += 2 * any;
                            }
                        }
                }
        }
    const unsigned long long text_waves = (unsigned long long)ceil_div(n_text, kTextQueriesPerWave);
    blocks += text_waves * 2ull * (unsigned long long)((N + kKeyTileKeys - 1) / kKeyTileKeys);
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
