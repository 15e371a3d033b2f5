// How a call's work is cut into workgroups (host only): waves per query patch, key ranges of the text-query rows, order.
#pragma once
#include "clear_internal.h"

namespace clear {

// The static array clear_attn_forward_noalloc puts the partial results of the text-query rows into, and what they take:
// partial outputs (rounded up to 256 bytes), then (maximum, denominator) pairs.  The shapes below respect it for every
// entry point, so that all of them run the same key ranges.
constexpr size_t kScratchBytes = (size_t)112 << 20;
inline size_t text_partial_o_bytes(int BH, int n_splits, int n_text, int head_dim)
{
    return ((size_t)BH * n_splits * n_text * head_dim * sizeof(float) + 255) & ~(size_t)255;
}
inline size_t text_partial_bytes(int BH, int n_splits, int n_text, int head_dim)
{
    return text_partial_o_bytes(BH, n_splits, n_text, head_dim) + (size_t)BH * n_splits * n_text * 2 * sizeof(float);
}

int max_text_splits(long long N);
void choose_text_splits(long long N, int BH, int n_tq_tiles, int num_cus, bool together, int* n_splits, int* split_keys);

struct F32Shape {
    int groups;      // waves per 16-query patch (1, 2, 4)
    int n_tq_tiles;  // text-query workgroups per head and key range
    int n_splits, split_keys;
};
F32Shape choose_f32_shape(long long NV, int BH, int n_text, int head_dim, int n_q_tiles, int num_cus);

struct ForwardProblem {
    int n_text, head_dim, BH;
    long long NV;  // keys of the text-query rows
    int n_classes, num_cus;
    struct Set {  // 1, 2, 4 waves per patch
        int n_image_tiles;     // query tiles to launch; 0: no such tables
        double stages, steps;  // of a query tile, on average: stages, blocks per wave
    } sets[3];
};
struct ForwardShape {
    int groups, tq_groups, n_splits, split_keys;
    bool text_first;
};
ForwardShape choose_forward_shape(const ForwardProblem& fp);

struct BackwardProblem {  // of a backward pass whose four kinds of workgroups go out in one launch
    int n_text, head_dim, BH, num_cus;
    long long N, image_wgs;  // image row tiles, each once for dQ and once for dK and dV
    double stages, steps;    // of an image row tile, on average: stages, blocks per wave
    double full_steps;       // blocks per wave that has rows
};
struct BackwardShape {
    int n_splits, split_keys;  // column ranges of the text rows
    bool text_first;           // text rows before image rows, dK + dV of both before dQ; otherwise the image rows first
};
BackwardShape choose_backward_shape(const BackwardProblem& bp);

}  // namespace clear
