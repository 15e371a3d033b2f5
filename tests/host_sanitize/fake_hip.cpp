// Stand-ins for the HIP runtime calls of the library's host side: device memory is host memory, so that contexts can be made, calls
// run up to their launches, and failures of the runtime forced, on a machine without a GPU and under the host sanitizers.
#include "fake_hip.h"

#include <cstdlib>
#include <cstring>

namespace fake {
int device = 0;
bool no_memory = false;
int copies_until_error = -1;
bool capturing = false;
long long live = 0;
int copies = 0;
static unsigned char scratch_array[1];
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void** ptr, size_t size)
{
    if (fake::no_memory) return hipErrorOutOfMemory;
    *ptr = malloc(size ? size : 1);
    ++fake::live;
    return *ptr ? hipSuccess : hipErrorOutOfMemory;
}
hipError_t hipFree(void* ptr)
{
    if (ptr) --fake::live;
    free(ptr);
    return hipSuccess;
}
hipError_t hipMemcpy(void* dst, const void* src, size_t size, hipMemcpyKind)
{
    if (fake::copies_until_error == 0) return hipErrorUnknown;
    if (fake::copies_until_error > 0) --fake::copies_until_error;
    ++fake::copies;
    memcpy(dst, src, size);
    return hipSuccess;
}
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipGetDevice(int* d)
{
    *d = fake::device;
    return hipSuccess;
}
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* prop, int)
{
    memset(prop, 0, sizeof(*prop));
    prop->multiProcessorCount = 256;
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** ptr, const void*)
{
    *ptr = fake::scratch_array;
    return hipSuccess;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* status)
{
    *status = fake::capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "fake error"; }
}
