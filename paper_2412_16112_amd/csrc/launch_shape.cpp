// Launch shapes (see launch_shape.h).  No device code here.
#include "launch_shape.h"

#include <algorithm>
#include <cmath>

namespace clear {

// The maximum number of key splits of the text-query pass; the workspace is sized for it.
int max_text_splits(long long N)
{
    // at least 512 keys per split, at most 64 splits
    long long s = (N + 511) / 512;
    if (s < 1) s = 1;
    if (s > 64) s = 64;
    return (int)s;
}

// Splits for a given batch*heads: at least two workgroups per CU when the keys allow it, and a workgroup
// count that fills whole rounds of the CUs (a partial last round idles most of the chip).
// `together`: the text-query workgroups go out in one launch with the image-query ones (launch_all) and fill the CUs
// that those leave idle, so whole rounds do not matter; what then costs is the number of splits (partial results
// written, read back and merged) and the length of a text-query workgroup when it is the last to finish: one round
// of workgroups at most, of at least 2 048 keys each.  (Measured over 1 - 32 splits, 24 heads: 2 splits at a 64 x 64
// grid and 5 at 128 x 128 and 256 x 256 beat the whole-rounds choice of 5, 16 and 16 by 6 %, 8 % and 2 %.)
void choose_text_splits(long long N, int BH, int n_tq_tiles, int num_cus, bool together, int* n_splits, int* split_keys)
{
    const int max_s = max_text_splits(N);
    const long long units = (long long)BH * n_tq_tiles;
    int best = 1;
    double best_score = -1.0;
    if (together && units < num_cus) {
        best = (int)std::min<long long>(max_s, num_cus / units);
        while (best > 1 && N / best < 2048) --best;
    } else {
        for (int s = 1; s <= max_s; ++s) {
            long long keys = (N + s - 1) / s;
            keys = ((keys + kKeyTileKeys - 1) / kKeyTileKeys) * kKeyTileKeys;
            const long long real = (N + keys - 1) / keys;  // splits that actually hold keys
            const long long wgs = units * real;
            const long long rounds = (wgs + num_cus - 1) / num_cus;
            double score = (double)wgs / (double)(rounds * num_cus);  // fraction of the rounds that is busy
            if (wgs < 2LL * num_cus) score *= 0.5;                    // too few workgroups to hide a workgroup's start-up
            if (score > best_score + 1e-9) {
                best_score = score;
                best = s;
            }
        }
    }
    long long keys = (N + best - 1) / best;
    keys = ((keys + kKeyTileKeys - 1) / kKeyTileKeys) * kKeyTileKeys;  // whole 64-key stages
    *split_keys = (int)keys;
    *n_splits = (int)((N + keys - 1) / keys);
}

// Launch shape of the fp32 kernel.  A workgroup is four waves of 16 queries, all on one 8 x 8 patch of queries (64 text
// queries); with `groups` = 2 or 4 waves on every 16 queries a patch of 4 x 8 or 4 x 4 (32 or 16 text queries) walks its
// keys in a half or a quarter of the steps, at two or four times the staging traffic per pair.  So: as many waves per
// patch as it takes to have two workgroups for every CU.  Text-query
// rows: key ranges of 1 024 and more, about the length of an image query's walk, so that no text workgroup is the
// last one running by far; shorter ones, down to 256, where that leaves CUs without work.
F32Shape choose_f32_shape(long long NV, int BH, int n_text, int head_dim, int n_q_tiles, int num_cus)
{
    const long long image = (long long)BH * n_q_tiles * 4;
    auto text_units = [&](int groups) { return BH * (((long long)n_text * groups + 63) / 64); };
    int groups = 1;
    while (groups < 4 && image * groups + text_units(groups) < 2LL * num_cus) groups *= 2;
    F32Shape shape = {groups, (int)(((long long)n_text * groups + 63) / 64), 0, 0};
    if (n_text == 0) return shape;
    long long splits = NV / 1024;
    const long long idle = 2LL * num_cus - image * groups;
    if (idle > 0) splits = std::max(splits, std::min(NV / (256 * groups), idle / text_units(groups)));
    splits = std::max(1LL, std::min<long long>(splits, max_text_splits(NV)));
    while (splits > 1 && text_partial_bytes(BH, (int)splits, n_text, head_dim) > kScratchBytes) --splits;  // (clear_attn_forward_noalloc takes the same shape)
    long long keys = (NV + splits - 1) / splits;
    keys = ((keys + kKeyTileKeys - 1) / kKeyTileKeys) * kKeyTileKeys;
    shape.split_keys = (int)keys;
    shape.n_splits = (int)((NV + keys - 1) / keys);
    return shape;
}

// Launch shape of a bf16 forward call: how many waves share 32 image queries (`groups`) and 32 text queries (`tq_groups`), the key
// ranges of the text queries, and which rows' workgroups go out first.
//
// One workgroup fills a CU, so what a call of a few workgroups per CU takes is decided by how evenly they fill the CUs and by the length of
// the longest.  Waves that share queries halve or quarter a workgroup's walk over its keys and double or quadruple the number
// of workgroups, at the price of staging every key tile twice or four times; key ranges do the same for the text queries at the price of
// partial results and a kernel that merges them.  Every combination is priced with the cost of a workgroup - a fixed part
// (dispatch, query rows and first tiles, output), a part per stage (barrier and refill of the pipeline) and a part per 32-key block of either of
// the two waves of a SIMD, fitted to measured calls - and the time at which the last CU finishes, longest workgroups first; the cheapest is
// taken.  (128 channels, 10 shapes from 1 head of 64 x 64 to 24 of 128 x 128: the predicted cycles are 1.44 to 1.96 times the measured
// nanoseconds; few workgroups at the upper end, where the clock is high, cut tiles at the lower.  64 channels, fitted to 24 calls in each of their
// shapes: the picks take 1.4 % more than the fastest on average, with the numbers of 128 channels about 4; 38 heads, 64 x 64, 333 text tokens
// 127 -> 112 us, 96 x 96 240 -> 235, 24 heads, 128 x 128 271 -> 260.)  (24 heads,
// 32 x 32 grid, 512 text tokens, r = 8: 40 -> 32 us against one wave per patch throughout; 2 heads: 36 -> 20 us.)  Beyond 16 workgroups
// per CU the evenness takes care of itself: one wave per patch, and choose_text_splits.
ForwardShape choose_forward_shape(const ForwardProblem& fp)
{
    const int n_text = fp.n_text, BH = fp.BH, n_classes = fp.n_classes, num_cus = fp.num_cus, per_block = bf16_text_queries_per_block();
    const long long NV = fp.NV, image_wgs = (long long)BH * n_classes * fp.sets[0].n_image_tiles;
    ForwardShape best = {1, 1, 1, kKeyTileKeys, false};
    auto text_tiles = [&](int groups) { return (n_text * groups + per_block - 1) / per_block; };
    if (image_wgs > 16LL * num_cus) {
        if (n_text > 0) choose_text_splits(NV, BH, text_tiles(1), num_cus, image_wgs <= 64LL * num_cus, &best.n_splits, &best.split_keys);
        return best;
    }
    // cycles; a SIMD takes `block` for every block of its two waves (at 128 channels 512 of them are matrix cycles)
    const bool d64 = fp.head_dim == 64;
    const double fixed = d64 ? 12e3 : 16e3, stage = d64 ? 700 : 900, block = d64 ? 480 : 520, in_doubt = d64 ? 0.99 : 0.98;
    const int stage_keys = bf16_tiles_per_stage(fp.head_dim) * kKeyTileKeys;
    double best_time = 1e300;
    for (int gi = 0; gi < 3; ++gi) {
        const ForwardProblem::Set& f = fp.sets[gi];
        if (f.n_image_tiles == 0) continue;  // not built
        const double n_image = (double)BH * n_classes * f.n_image_tiles, c_image = fixed + f.stages * stage + 2 * f.steps * block;
        for (int ti = 0; ti < (n_text > 0 ? 3 : 1); ++ti) {
            const int tg = 1 << ti;
            long long last_keys = -1;
            for (int s = 1; s <= (n_text > 0 ? std::min(max_text_splits(NV), 16) : 1); ++s) {
                double n_text_wgs = 0, c_text = 0, merge = 0;
                long long keys = (NV + s - 1) / s;
                keys = (keys + kKeyTileKeys - 1) / kKeyTileKeys * kKeyTileKeys;
                const int real = (int)((NV + keys - 1) / keys);
                if (n_text > 0) {
                    if (keys == last_keys) continue;
                    last_keys = keys;
                    const size_t partial = text_partial_bytes(BH, real, n_text, fp.head_dim);
                    const double bytes = (double)partial;
                    if (real > 1 && partial > kScratchBytes) break;  // (clear_attn_forward_noalloc takes the same shape)
                    const double stages = std::ceil((double)keys / stage_keys);
                    n_text_wgs = (double)BH * text_tiles(tg) * real;
                    c_text = fixed + stages * stage + 2 * block * stages * std::max(1.0, (double)stage_keys / 32 / tg) * std::min(1.0, (double)keys / (stages * stage_keys));
                    if (real > 1) merge = 12e3 + 2 * bytes / 2000;  // a kernel of its own; partial results written and read back
                }
                // longest first: c1 n1, then c2 n2
                const bool text_first = c_text > c_image;
                const double c1 = text_first ? c_text : c_image, c2 = text_first ? c_image : c_text, n1 = text_first ? n_text_wgs : n_image, n2 = text_first ? n_image : n_text_wgs;
                // (no shape takes less than its longest workgroup, or than its work spread evenly)
                if ((std::max(c1, (n1 * c1 + n2 * c2) / num_cus) + merge) * (1 - 1e-9) >= best_time * in_doubt) continue;
                const double q = std::floor(n1 / num_cus), r = n1 - q * num_cus;
                double lo = (q + (r > 0)) * c1, hi = lo + (n2 > 0 ? (std::ceil(n2 / num_cus) + 1) * c2 : 0);
                auto fits = [&](double t) { return r * std::floor((t - (q + 1) * c1) / c2) + (num_cus - r) * std::floor((t - q * c1) / c2) >= n2; };
                if (n2 == 0 || fits(lo)) hi = lo;
                for (int i = 0; i < 24 && hi > lo; ++i) {
                    const double mid = 0.5 * (lo + hi);
                    (fits(mid) ? hi : lo) = mid;
                }
                const double time = hi + merge;
                if (time < best_time * in_doubt) {  // (in doubt the simpler shape)
                    best_time = time;
                    best = {1 << gi, tg, real, (int)keys, text_first};
                }
            }
        }
    }
    return best;
}

// When the last of num_cus CUs finishes, if every workgroup starts on the CU that is free first: n[i] workgroups of cost[i], in this order.
static double finish_time(int num_cus, const double (&n)[4], const double (&cost)[4])
{
    struct Group {
        double free_at, cus;
    } g[6] = {{0.0, (double)num_cus}};  // by time; a kind adds one group at most
    int ng = 1;
    for (int i = 0; i < 4; ++i)
        for (double left = n[i]; left > 0;) {
            if (left >= num_cus && g[ng - 1].free_at - g[0].free_at <= cost[i]) {  // whole rounds: every CU takes one
                const double rounds = std::floor(left / num_cus);
                for (int k = 0; k < ng; ++k) g[k].free_at += rounds * cost[i];
                left -= rounds * num_cus;
                continue;
            }
            const double take = std::min(left, g[0].cus), at = g[0].free_at + cost[i];
            left -= take;
            g[0].cus -= take;
            if (g[0].cus == 0) std::copy(g + 1, g + ng--, g);
            int k = ng;
            while (k > 0 && g[k - 1].free_at > at) --k;
            if (k > 0 && g[k - 1].free_at == at) {
                g[k - 1].cus += take;
            } else {
                std::copy_backward(g + k, g + ng, g + ng + 1);
                g[k] = {at, take};
                ++ng;
            }
        }
    return g[ng - 1].free_at;
}

// Launch shape of a backward pass in one launch: column ranges of the text rows and the order of its four kinds of workgroups.
//
// As in the forward pass one workgroup fills a CU, and the time of a few rounds is how evenly they fill the CUs.  Long text rows go first, or
// they are the last to run; short ones go last and fill the gaps that image rows of unequal length leave.  Each pair of a split count and an order
// is priced with a cost per workgroup (a fixed part, one per stage, one per block of either of the two waves of a SIMD; a text workgroup of four
// waves or fewer has one wave to a SIMD) and two times for the launch: that of finish_time with all image rows as long as those whose waves
// all have rows, and the evenly spread work plus half a workgroup of the last kind.  Their mean is taken, 4 % more where image rows come last (they differ
// in length, which finish_time does not see).  Several ranges cost the kernel that adds them up.  A range of over four times an image row's walk that takes more than
// a quarter of the evenly spread work is not considered: the mean misses how such workgroups outlast the others (24 heads, 128 x 128, 333 text tokens: one
// range 1 433 us, four 1 360).
// (Fitted to 16 calls at 128 channels and 10 at 64, 1 to 8 ranges in both orders.  Training steps against image rows first with choose_text_splits and a
// reduction always, forward included, on one card: 24 heads of 128 channels, 512 text tokens, 64 x 64, r = 16 518 -> 500 us, 32 x 32, r = 8 151 -> 141; 43 x 80, 441 text
// tokens 468 -> 440; 48 x 85, 77 text tokens 369 -> 365; 128 x 128, 333 text tokens 1 865 -> 1 873, its runs 0.8 % apart; 38 heads, 36 x 20 214 -> 204; 38 heads of 64,
// 333 text tokens, 64 x 64 455 -> 442; 4 x 28 heads of 64, 104 x 72, r = 8 1 869 -> 1 815.)
// Beyond 16 image workgroups per CU the evenness takes care of itself: image rows first, and choose_text_splits.
BackwardShape choose_backward_shape(const BackwardProblem& bp)
{
    const int per_block = bf16_text_queries_per_block(), n_tiles = (bp.n_text + per_block - 1) / per_block;
    BackwardShape best = {1, kKeyTileKeys, false};
    if (bp.n_text == 0) return best;
    choose_text_splits(bp.N, bp.BH, n_tiles, bp.num_cus, true, &best.n_splits, &best.split_keys);
    if (bp.image_wgs > 16LL * bp.num_cus) return best;
    const bool d64 = bp.head_dim == 64;
    // cycles
    const double fixed = d64 ? 8e3 : 18e3, stage = d64 ? 1900 : 1200, block_kv = d64 ? 920 : 1140, block_q = d64 ? 720 : 1020, lone_wave = d64 ? 0.57 : 0.5;
    const int stage_keys = bf16_tiles_per_stage(bp.head_dim) * kKeyTileKeys;
    const double image = fixed + bp.stages * stage, image_kv = image + 2 * bp.steps * block_kv, image_q = image + 2 * bp.steps * block_q;
    const double full_kv = image + 2 * bp.full_steps * block_kv, full_q = image + 2 * bp.full_steps * block_q;
    const int last_rows = bp.n_text - (n_tiles - 1) * per_block;
    const double waves = last_rows * 2 > per_block ? 1.0 : (n_tiles - 1 + lone_wave) / n_tiles;  // cost of a text block, mean of the tiles
    const int most = std::min(max_text_splits(bp.N), 16);
    const double units = (double)bp.BH * n_tiles;
    double best_time = 1e300;
    long long last_keys = -1;
    for (int s = 1; s <= most; ++s) {
        long long keys = (bp.N + s - 1) / s;
        keys = (keys + kKeyTileKeys - 1) / kKeyTileKeys * kKeyTileKeys;
        if (keys == last_keys) continue;
        last_keys = keys;
        const int real = (int)((bp.N + keys - 1) / keys);
        const double n_text_wgs = units * real, n_image = (double)bp.image_wgs;
        if (n_text_wgs > std::max(units, 64.0 * bp.num_cus)) break;
        const double text = fixed + std::ceil((double)keys / stage_keys) * stage, blocks = 2 * (double)keys / 32 * waves;
        const double text_kv = text + blocks * block_kv, text_q = text + blocks * block_q;
        const double reduce = real == 1 ? 0 : 12e3 + 3e-4 * 2 * 3 * sizeof(float) * bp.BH * real * (double)bp.n_text * bp.head_dim;  // a kernel of its own; partial sums written and read back
        const double even = (n_image * (image_kv + image_q) + n_text_wgs * (text_kv + text_q)) / bp.num_cus, longest = std::max(full_kv, text_kv);
        if (keys > 4 * 32 * bp.steps && text_kv > 0.25 * even && s < most) continue;
        for (int text_first = 0; text_first < 2; ++text_first) {
            const double n[2][4] = {{n_image, n_image, n_text_wgs, n_text_wgs}, {n_text_wgs, n_image, n_text_wgs, n_image}};
            const double c[2][4] = {{full_kv, full_q, text_kv, text_q}, {text_kv, full_kv, text_q, full_q}};
            const double spread = std::max(longest, even + 0.5 * c[text_first][3]);
            const double time = (0.5 * (finish_time(bp.num_cus, n[text_first], c[text_first]) + spread) + reduce) * (text_first ? 1.04 : 1.0);
            if (time < best_time) {
                best_time = time;
                best = {real, (int)keys, text_first != 0};
            }
        }
    }
    return best;
}

}  // namespace clear
