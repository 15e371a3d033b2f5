// What the stand-ins for the HIP runtime (fake_hip.cpp) and the kernel launchers (launch_stubs.cpp) are told and report.
#pragma once
#include "../../paper_2412_16112_amd/csrc/clear_internal.h"

namespace fake {
extern int device;             // the current device
extern bool no_memory;         // hipMalloc fails
extern int copies_until_error; // hipMemcpy fails once this many have succeeded (-1: never)
extern bool capturing;         // every stream is being captured
extern long long live;         // device allocations not yet freed
extern int copies;             // hipMemcpy calls
// the kernel launches since the last reset
extern int forward_launches, backward_launches;
extern clear::FwdParams forward;   // the last one's parameters
extern clear::BwdParams backward;
}  // namespace fake
