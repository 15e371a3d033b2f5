// Row-band ("patch-parallel") inference, Sec. 3.4: combines the text-query outputs that each band computed
// over its own keys.
//   exact:   O = sum_p w_p O_p,  w_p = exp(lse_p) / sum_p exp(lse_p)   (softmax over the union of disjoint key sets)
//   average: O = (1/n) sum_p O_p                                         (Eq. 7)
#include "../../include/clear_attn.h"

#include <hip/hip_runtime.h>

#include "clear_internal.h"

namespace clear {
namespace {

// Bound by reading the parts.  A thread takes VEC channels of a row (four, or one where head_dim is not a multiple of
// four) and has four parts' loads in flight; the parts are added in their order.
// 8 parts, 24 heads, 512 text tokens, head_dim 128: 20.9 us with a row a workgroup and one channel a thread -> 11.2 us
// (4.8 TB/s); a band of a 512 x 512 grid with its merge 1018 -> 1012 us.
template <typename OutT, int VEC>
__global__ void __launch_bounds__(256) merge_text_kernel(const MergeParts parts, unsigned n_threads, int n_text, long long N, int d, int mode, OutT* O)
{
    // the callers' tensors are as aligned as their elements
    typedef float vec __attribute__((ext_vector_type(VEC)));
    typedef float vec_in __attribute__((ext_vector_type(VEC), aligned(4)));
    typedef OutT vec_out __attribute__((ext_vector_type(VEC), aligned(sizeof(OutT))));
    const unsigned t = blockIdx.x * 256 + threadIdx.x;
    if (t >= n_threads) return;
    const unsigned per_row = (unsigned)d / VEC, row = t / per_row;  // bh * n_text + q
    const int ch = (int)(VEC * (t % per_row));
    const long long at = (long long)row * d + ch;
    float mx = -INFINITY, den = 0.f;
    if (mode == CLEAR_MERGE_EXACT)
        for (int i = 0; i < parts.n; ++i) mx = fmaxf(mx, parts.lse[i][row]);
    vec acc = 0.f;
    auto add = [&](const float lse, const vec o) __attribute__((always_inline)) {
        if (mode == CLEAR_MERGE_AVERAGE) {
            acc += o;
        } else {
            const float w = __expf(lse - mx);
            den += w;
            acc += w * o;
        }
    };
    const bool weighted = mode == CLEAR_MERGE_EXACT;
    int i = 0;
    for (; i + 4 <= parts.n; i += 4) {
        vec o[4];
        float lse[4];
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            o[j] = *(const vec_in*)(parts.o[i + j] + at);
            lse[j] = weighted ? parts.lse[i + j][row] : 0.f;
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) add(lse[j], o[j]);
    }
    for (; i < parts.n; ++i) add(weighted ? parts.lse[i][row] : 0.f, *(const vec_in*)(parts.o[i] + at));
    acc /= weighted ? den : (float)parts.n;
    const unsigned bh = row / (unsigned)n_text, q = row % (unsigned)n_text;
    vec_out out;
#pragma unroll
    for (int j = 0; j < VEC; ++j) out[j] = (OutT)acc[j];
    *(vec_out*)(O + ((long long)bh * N + q) * d + ch) = out;
}

template <typename OutT>
hipError_t launch(const MergeParts& parts, int BH, int n_text, long long N, int d, int mode, OutT* O, hipStream_t stream)
{
    const int vec = d % 4 == 0 ? 4 : 1;
    const unsigned long long n_threads = (unsigned long long)BH * n_text * (d / vec), blocks = (n_threads + 255) / 256;
    if (n_threads > 0xffffff00ULL) return hipErrorInvalidConfiguration;  // (more than a launch can have)
    if (vec == 4)
        hipLaunchKernelGGL((merge_text_kernel<OutT, 4>), dim3((unsigned)blocks), dim3(256), 0, stream, parts, (unsigned)n_threads, n_text, N, d, mode, O);
    else
        hipLaunchKernelGGL((merge_text_kernel<OutT, 1>), dim3((unsigned)blocks), dim3(256), 0, stream, parts, (unsigned)n_threads, n_text, N, d, mode, O);
    return hipGetLastError();
}

}  // namespace

hipError_t launch_merge_text(const MergeParts& parts, int BH, int n_text, long long N, int head_dim, int mode, void* O, int dtype,
                             hipStream_t stream)
{
    if (dtype == CLEAR_BF16) return launch(parts, BH, n_text, N, head_dim, mode, (__bf16*)O, stream);
    return launch(parts, BH, n_text, N, head_dim, mode, (float*)O, stream);
}

}  // namespace clear
