// Stand-ins for the kernel launchers, so that the host side of the library (argument checks, schedule builder,
// band layout, contexts and the parameters of a launch) links without any kernel and can run under the host sanitizers on a machine
// without a GPU.  The launchers of the forward and backward kernels record what they are given.
#include <algorithm>

#include "../../paper_2412_16112_amd/csrc/block_class.h"
#include "fake_hip.h"

namespace fake {
int forward_launches = 0, backward_launches = 0;
clear::FwdParams forward;
clear::BwdParams backward;
static hipError_t record(const clear::FwdParams& p)
{
    ++forward_launches;
    forward = p;
    return hipSuccess;
}
static hipError_t record(const clear::BwdParams& p)
{
    ++backward_launches;
    backward = p;
    return hipSuccess;
}
}  // namespace fake

namespace clear {
hipError_t launch_bf16_d128(const FwdParams& p, hipStream_t, int) { return fake::record(p); }
hipError_t launch_bf16_d64(const FwdParams& p, hipStream_t, int) { return fake::record(p); }
hipError_t launch_f32_d64(const FwdParams& p, hipStream_t, int) { return fake::record(p); }
hipError_t launch_bf16_d128_backward(const BwdParams& p, const void*, float*, hipStream_t, int) { return fake::record(p); }
hipError_t launch_bf16_d64_backward(const BwdParams& p, const void*, float*, hipStream_t, int) { return fake::record(p); }
hipError_t launch_merge_text(const MergeParts&, int, int, long long, int, int, void*, int, hipStream_t) { return hipErrorNotSupported; }
hipError_t measure_mfma_peak(int, double, double*, double*) { return hipErrorNotSupported; }
hipError_t launch_qk_prologue(const void*, const TensorStrides&, void*, const TensorStrides&, int, int, int, int, int, int, const float*, float,
                              const float*, const float*, hipStream_t)
{
    return hipErrorNotSupported;
}
int bf16_text_queries_per_block() { return kBf16NWY * kBf16NWX * kTextQueriesPerWave; }
}  // namespace clear
