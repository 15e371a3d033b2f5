// Internal declarations shared by the host API and the kernel launchers (not part of the C ABI).
#pragma once
#include <hip/hip_runtime.h>
#include <cstdint>
#include <vector>

namespace clear {

// Geometry of the bf16 MFMA kernels: a wave owns a 4 x 8 patch of queries (32 = one MFMA N
// dimension); a workgroup owns NWY x NWX such patches; a key tile is 8 x 8 image tokens staged as
// two 4 x 8 blocks of 32 keys (one MFMA M dimension each).
constexpr int kWaveQH = 4, kWaveQW = 8;
constexpr int kKeyBlockH = 4, kKeyBlockW = 8;
constexpr int kKeyTileH = 8, kKeyTileW = 8;
constexpr int kKeyTileKeys = kKeyTileH * kKeyTileW;  // 64 keys per staged tile
#ifndef CLEAR_NWY
#define CLEAR_NWY 4
#endif
constexpr int kBf16NWY = CLEAR_NWY, kBf16NWX = 2;    // workgroup = (4 NWY) x 16 queries, 2 NWY waves
constexpr int kBf16QTileH = kBf16NWY * kWaveQH, kBf16QTileW = kBf16NWX * kWaveQW;
constexpr int kTextQueriesPerWave = 32;

// fp32 path: 16 x 16 query tiles in the schedule (the workgroups take parts of them), same key tiles.
constexpr int kF32QTileH = 16, kF32QTileW = 16;

struct Schedule {
    int gridH = 0, gridW = 0, r = 0;
    int mask_kind = 0, mask_shift = 0;  // MaskKind of block_class.h; shift: Swin windows only
    int qth = 0, qtw = 0, kth = 0, ktw = 0;
    int n_qty = 0, n_qtx = 0, n_kty = 0, n_ktx = 0;
    std::vector<int> row_ptr;        // n_q_tiles + 1
    std::vector<int> col_idx;        // key tile ids, ascending per query tile
    std::vector<unsigned char> flags;  // CLEAR_TILE_FULL / CLEAR_TILE_PARTIAL
};

// Host-side integer geometry (schedule.cpp)
void build_schedule(int gridH, int gridW, int r, int qth, int qtw, int kth, int ktw, Schedule* s, int mask_kind = 0, int mask_shift = 0);
// Upper bound, in 64 bits, on the (query tile, key tile) pairs build_schedule would list (it stores them with int indices).
long long schedule_pair_bound(int gridH, int gridW, int r, int qth, int qtw, int kth, int ktw);
// (query tile, key tile) pairs a context may have; create refuses more.  A pair takes 9 bytes of tile lists and, in a bf16 context, up to 16
// words of wave programs (typically 14: 0.7 GB at 768 x 768, r = 400, 13 million pairs) where neither query tiles nor waves
// share any, as with r about half of a large grid.  Windows that hold the whole grid share nearly all of them.
constexpr long long kMaxSchedulePairs = 1LL << 28;
unsigned long long mask_count(int n_text, int gridH, int gridW, int r, int mask_kind = 0, int mask_shift = 0);
// Pairs the fp32 path multiplies: 4 x 4 query patches against the cells of 16 keys they reach.
unsigned long long executed_pairs_f32(const Schedule& s, int n_text);

// Where element (b, h, n, c) of a [B, H, N, head_dim] tensor lives: base + b * sb + h * sh + n * sn + c (in
// elements; channels are contiguous).  The plain layout is sn = head_dim, sh = N * head_dim, sb = H * N * head_dim.
struct TensorStrides {
    long long sb, sh, sn;
};

// Programs of the bf16 forward kernels' computing waves: a word per 32-key block of the wave's key list, in stage order
// (a stage: 2 tiles at head_dim 128, 4 at 64; the text tiles first, then the listed image tiles).
constexpr unsigned kProgramPlaceMask = 15;       // where the block lies in its stage buffer, in units of 2 KB
constexpr int kProgramMaskShift = 4;             // bits 4 .. 29: its lane masks (an id)
constexpr unsigned kProgramStageEnd = 1u << 31;  // the wave's last word of this stage
constexpr unsigned kProgramNoBlock = 1u << 30;   // nothing to do in this stage (only where the word before it masks everything out)
constexpr unsigned kProgramFlags = kProgramStageEnd | kProgramNoBlock | kProgramPlaceMask;
constexpr unsigned kMaskIdNone = 0;       // every pair of the block is admitted
constexpr unsigned kMaskIdNothing = 1;    // none is
constexpr unsigned kMaskIdFirstKeys = 1;  // + k, 1 <= k < 32: the first k keys of the block are
constexpr int kProgramSpareWords = 128;   // readable words behind the last program: the kernels fetch 64 at a time and read two ahead
constexpr size_t kMaxProgramWords = 0xffff0000u;  // places among them are 32-bit numbers; more are refused as out of memory
constexpr unsigned kMaskIdFree = 33;      // masks of image blocks from here on
constexpr int bf16_tiles_per_stage(int head_dim) { return head_dim == 64 ? 4 : 2; }
struct BlockPrograms {
    std::vector<unsigned> words;               // kProgramSpareWords at the end
    std::vector<unsigned> ptr;                 // [variants][n_q_tiles][kBf16NWY * kBf16NWX]: where a wave's program starts
    double mean_stages, mean_steps;            // of a query tile: stages, blocks per wave
    unsigned text_words[3];                    // for 1, 2, 4 waves per patch of text queries: [wave][keys of the stage][blocks per stage / waves]
                                               // words of a stage with that many keys (0: a whole stage that is not the last)
    unsigned long long blocks[4][4] = {};      // [variant of the key class][of the query class]: blocks that the waves of a head (of a class of it) run
                                               // (one wave per patch only)
};
// Query tiles whose lists and programs are the same but for their place: interior ones, mostly.
struct QueryTilePatterns {
    std::vector<int> id;     // per query tile: its pattern
    std::vector<int> first;  // per pattern: the first query tile that has it
};
QueryTilePatterns query_tile_patterns(const Schedule& s);
// Tile lists of the bf16 forward kernels (per query tile, origins row << 16 | col): pairs of a tile and its point mirror through the
// centre of the query tile (a stage at head_dim 128: what one wave's queries do not reach of it another's do), in the order of
// their place on the raster modulo 4 x 4 tiles, which is the same for both of a pair, whatever query tile it is seen from:
// query tiles whose windows overlap then need a key tile at about the same step of their lists.
void order_forward_tiles(const Schedule& s, const QueryTilePatterns& pat, std::vector<int>* k_col);
struct ProgramInput {
    const Schedule* sched;  // query tiles of 16 / groups rows
    const QueryTilePatterns* pat;
    const std::vector<int>* k_col;  // its tile lists (order_forward_tiles)
    int groups;                     // waves a query patch's blocks are dealt to, in turn
};
// Programs for one or several numbers of waves per patch; masks, for all of them: [mask id][16 score registers], bit l = lane l keeps the
// score.  stride > 1 (strided mask): the schedule is that of a residue class on its larger extents, and there are four variants, as the
// keys' class has gridH / stride or one more rows, gridW / stride or one more columns.
void build_block_programs(const std::vector<ProgramInput>& in, int n_text, int head_dim, int stride, int gridH, int gridW,
                          std::vector<BlockPrograms>* out, std::vector<unsigned long long>* masks);

// Pairs fed to the matrix pipeline per (batch, head) by the bf16 forward kernels with one wave per patch: every block that a wave runs, those
// included that mask everything and only finish what is pending.
unsigned long long executed_pairs_bf16(const BlockPrograms& prog, int n_text, int gridH, int gridW, int stride, int layer);

struct FwdParams {
    const void* Q;
    const void* K;
    const void* V;
    void* O;
    TensorStrides qs, ks, vs, os;  // bf16 kernels only; the fp32 kernel takes the plain layout
    int B, H, n_text, gridH, gridW, r2;
    long long N;       // tokens per (batch, head)
    int n_q_tiles;     // image query tiles per head
    int n_qtx;         // query tiles per tile row
    const int* row_ptr;  // device CSR
    const int* col_idx;  // per query tile: key tile origins (row << 16 | col)
    const int* qt_order;  // bf16 image-query kernel, whole-grid launches: the query tile that the i-th workgroup of a head takes (null: i)
    const unsigned* program;      // bf16 kernels: the wave programs (BlockPrograms on the device)
    const unsigned* program_ptr;
    const unsigned long long* block_masks;
    unsigned text_words;          // where the text-query rows' words lie among the programs, for tq_groups
    bool text_first;              // bf16, one launch for both: the text-query workgroups go first
    int groups, tq_groups;  // bf16 kernels: waves that share a patch of 32 queries (1, 2 or 4), image and text-query rows
    float scale_log2e;  // log2(e) / sqrt(head_dim)
    // text-query pass: dense rows split along the keys, partial results merged afterwards
    int n_tq_tiles;   // text query tiles per head
    int n_splits;     // key splits
    int split_keys;   // keys per split, multiple of 64
    float* ws_o;      // [B*H][n_splits][n_text][head_dim] un-normalised partial outputs
    float* ws_ml;     // [B*H][n_splits][n_text][2]        running max (raw logit) and denominator
    // Row-band mode (one band of image rows with its halo; Sec. 3.4).  Whole grid: own_y0 = 0, own_y1 = gridH,
    // qt_begin = 0, n_q_tiles_launch = n_q_tiles, NV = N, vkeys_text = INT_MAX, vshift = 0, y_shift = 0, band_o = null.
    int own_y0, own_y1;    // image rows whose queries are computed; the other rows are halo: keys only
    int qt_begin;          // first query tile launched (tile rows covering the owned rows)
    int n_q_tiles_launch;  // query tiles launched per (batch, head)
    // key list of the text-query pass by "virtual" index v in [0, NV): token v for v < vkeys_text, else v + vshift
    long long NV;
    int vkeys_text;
    int vshift;
    int y_shift;      // tile coordinates (own_y0, own_y1, the tile lists) = image row + y_shift; the grid then spans rows [y_shift, y_shift + gridH)
    float* band_o;    // when set, the text merge writes fp32 softmax outputs [B*H][n_text][head_dim] here ...
    float* band_lse;  // ... and the natural log of the softmax denominators [B*H][n_text] here, not O's text rows
    int mask_kind, mask_r, mask_shift;  // MaskKind, radius / window size, Swin shift
    float* lse;       // optional [B*H][N]: natural log of every row's softmax denominator sum_j exp(q.k_j / sqrt(d))
    // Strided mask: n_classes = stride^2 dense problems per (batch, head), one per residue class (y % stride,
    // x % stride) of the queries; class (a, b) takes its keys from class ((a + stride_rx) % stride, (b + stride_ry)
    // % stride).  The tile lists then describe the class sub-grid.  Otherwise n_classes = 1, stride = 1.
    int n_classes, stride, stride_rx, stride_ry;
    // Query prologue applied while the query rows are loaded (bf16 kernels; all null: Q is used as it is).
    const float* q_gain;  // [head_dim] RMS-norm gain, or null: no normalisation
    const float* rope_y;  // [gridH][head_dim/2][2] (cos, sin) per row, or null: no rotation
    const float* rope_x;  // [gridW][head_dim/2][2] (cos, sin) per column
    float norm_eps;
    int f32_groups;  // fp32 kernel: waves per 16-query patch (1, 2 or 4 of a workgroup's 4)
};

// Launches `per_head` workgroups for every (batch, head) of p, in one launch or, where they are more than the `most` that one can have (2^32
// threads: beyond that the runtime drops the excess without an error), in one for several batch items or heads at a time: shift(&q, b, h) moves
// the pointers of q to batch item b, head h; launch(q, n) launches n workgroups.
template <class Params, class Shift, class Launch>
hipError_t launch_by_heads(const Params& p, long long per_head, long long most, Shift shift, Launch launch)
{
    if (per_head * p.B * p.H <= most) return launch(p, (int)(per_head * p.B * p.H));
    if (per_head > most) return hipErrorInvalidConfiguration;
    const bool whole = per_head * p.H <= most;  // a launch takes all heads of several batch items, or several heads of one
    const int nb = whole ? (int)(most / (per_head * p.H)) : 1, nh = whole ? p.H : (int)(most / per_head);
    hipError_t e = hipSuccess;
    for (int b = 0; b < p.B && e == hipSuccess; b += nb)
        for (int h = 0; h < p.H && e == hipSuccess; h += nh) {
            Params q = p;
            q.B = p.B - b < nb ? p.B - b : nb;
            q.H = p.H - h < nh ? p.H - h : nh;
            shift(&q, b, h);
            e = launch(q, (int)(per_head * q.B * q.H));
        }
    return e;
}

// Launchers (kernels_bf16.hip, kernels_f32.hip).  Each returns the first HIP error met.
// phase: kPhaseAll, or one of the three kernels of a forward pass (used to time them one by one).
// kPhaseImageAndTextQuery (bf16 only): the first two in one launch.
enum Phase : int { kPhaseAll = -1, kPhaseImage = 0, kPhaseTextQuery = 1, kPhaseTextMerge = 2, kPhaseImageAndTextQuery = 3 };
hipError_t launch_bf16_d128(const FwdParams& p, hipStream_t stream, int phase);
hipError_t launch_bf16_d64(const FwdParams& p, hipStream_t stream, int phase);
hipError_t launch_f32_d64(const FwdParams& p, hipStream_t stream, int phase);
int bf16_text_queries_per_block();
// What each wave of a bf16 backward workgroup does with each listed tile that lies inside the grid (those are masked from the
// table): desc[e * waves + w] for entry e of the kernel-order tile list `k_col` (origins row << 16 | col) and wave w
// (patch row w / 2, patch column w % 2 of the query tile) = table entry of block 0 | table entry of block 1 << 16,
// where a block that is wholly admitted takes the all-ones entry and one out of reach the all-zeros entry; or
// kWaveSkipsTile when neither block can be reached.  Entries of tiles cut by the border hold kWaveSkipsTile (not used).
constexpr int kWaveSkipsTile = -1;
void build_wave_descriptors(const Schedule& s, const std::vector<int>& k_col, const std::vector<int>& n_plain, int mask_ry, int mask_rx,
                            std::vector<int>* desc);
void build_bf16_mask_table(int r, int ry, int rx, int mask_kind, std::vector<unsigned long long>* tbl);
// Backward pass (kernels_bf16_bwd.hip).
struct BwdParams {
    const void* Q;
    const void* K;
    const void* V;
    const void* dO;
    const float* lse;    // [B*H][N] natural log of the softmax denominators (from the forward pass)
    // What the columns of dK and dV start S and dP from, both [B*H][N] in the context's workspace: -lse / scale and -delta, with
    // delta_i = dO_i . O_i.  Stored by the delta kernel, or, where O is given here, by the dQ kernels for the dK / dV kernels launched
    // after them.
    float* neg_lse;
    float* neg_delta;
    const void* O;  // the forward output: the dQ kernels form both for their own rows (null: every kernel reads them)
    void* dQ;
    void* dK;
    void* dV;
    TensorStrides qs, ks, vs, os, dos, dqs, dks, dvs;  // lse, neg_lse and neg_delta are plain [B*H][N]
    int B, H, n_text, gridH, gridW, r2;
    long long N;
    int n_q_tiles, n_qtx;
    const int* row_ptr;
    const int* col_idx;  // tiles inside the grid first, then the ones cut by the border
    const int* n_plain;  // per row tile: how many of its tiles lie inside the grid
    const int* qt_order;  // the row tile that the i-th workgroup of a head takes (null: i)
    const unsigned long long* mask_tbl;  // lane masks per relative block offset (may be null)
    int mask_ry, mask_rx;
    const int* wave_desc;  // with mask_tbl: per listed tile inside the grid (kernel order) and wave of the workgroup, the mask-table
                           // entries of the tile's two blocks (low / high 16 bits), or kWaveSkipsTile (build_wave_descriptors; rows
                           // and columns swap roles for dK and dV: the masks with a table are symmetric)
    int mask_kind, mask_r, mask_shift;  // MaskKind, radius / window size, Swin shift
    int n_classes, stride, stride_rx, stride_ry;  // strided mask, as in FwdParams (otherwise 1, 1, 0, 0)
    float scale_log2e;  // log2(e) / sqrt(head_dim)
    float scale;        // 1 / sqrt(head_dim)
    float neg_inv_scale;  // -1 / scale
    // text rows: sums over every token, split along the columns, partial sums added up afterwards (one split: stored as they are)
    int n_tq_tiles, n_splits, split_keys;
    bool text_first;  // one launch for all rows (kBwdPhaseFour): see BackwardShape
    float* ws;  // [3 (dQ, dK, dV)][B*H][n_splits][n_text][head_dim]
};
// phase: kBwdPhaseAll (the dQ kernels, which form neg_lse and neg_delta on their way, then the dK / dV kernels, then the reduction),
// or one kernel of the pass: delta first; the image-row and text-row kernels are independent
// of each other; the reduction of the text-row partial sums, if there are several, comes after the two text-row kernels.
// kBwdPhaseFour: the four kernels between delta and the reduction in one launch.
// O: the forward output; stats: [2][B*H][N], where the delta kernel stores neg_lse and neg_delta.
enum BwdPhase : int { kBwdPhaseAll = -1, kBwdPhaseDelta = 0, kBwdPhaseImageQ = 1, kBwdPhaseImageKV = 2, kBwdPhaseTextQ = 3, kBwdPhaseTextKV = 4, kBwdPhaseReduce = 5, kBwdPhaseFour = 6 };
hipError_t launch_bf16_d128_backward(const BwdParams& p, const void* O, float* stats, hipStream_t stream, int phase);
hipError_t launch_bf16_d64_backward(const BwdParams& p, const void* O, float* stats, hipStream_t stream, int phase);

// band_merge.hip: combination of the text-query outputs of several row bands.
constexpr int kMaxMergeParts = 64;
struct MergeParts {
    int n;
    const float* o[kMaxMergeParts];    // [B*H][n_text][head_dim] softmax outputs
    const float* lse[kMaxMergeParts];  // [B*H][n_text] natural log of the softmax denominators
};
hipError_t launch_merge_text(const MergeParts& parts, int BH, int n_text, long long N, int head_dim, int mode, void* O, int dtype,
                             hipStream_t stream);
// prologue.hip: RMS norm + rotary embedding of whole [BH][N][head_dim] bf16 tensors (the keys of a fused
// forward pass; also the stand-alone pass).  X == Y is allowed.
hipError_t launch_qk_prologue(const void* X, const TensorStrides& xs, void* Y, const TensorStrides& ys, int B, int H, int n_text, int gridH,
                              int gridW, int head_dim, const float* gain, float eps, const float* rope_y, const float* rope_x,
                              hipStream_t stream);
// mfma_peak.hip: sustained rate of back-to-back bf16 MFMAs on every SIMD, and the shader clock it ran at.
hipError_t measure_mfma_peak(int num_cus, double seconds, double* tflops, double* shader_mhz);

}  // namespace clear
