// Test aid: leaves one 32-bit word all over the LDS of every CU, so that a kernel that reads a word it has not written
// reads this one and not whatever an earlier kernel happened to leave.
#include <hip/hip_runtime.h>

constexpr int kLdsBytes = 160 * 1024;  // all of a CU's: one workgroup fits at a time, so neighbours go to other CUs

__global__ __launch_bounds__(1024) void lds_fill_kernel(unsigned word) {
    extern __shared__ unsigned lds[];
    volatile unsigned* p = lds;  // nothing reads it back
    for (int i = threadIdx.x; i < kLdsBytes / 4; i += 1024) p[i] = word;
}

// Fills on `stream`, several workgroups per CU (each XCD deals its share out to its CUs in turn). 0, or a HIP error code.
extern "C" int lds_fill(unsigned word, void* stream) {
    int dev = 0, cus = 0;
    hipError_t rc = hipGetDevice(&dev);
    if (rc == hipSuccess) rc = hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (rc == hipSuccess)
        rc = hipFuncSetAttribute((const void*)lds_fill_kernel, hipFuncAttributeMaxDynamicSharedMemorySize, kLdsBytes);
    if (rc != hipSuccess) return (int)rc;
    hipLaunchKernelGGL(lds_fill_kernel, dim3(4 * cus), dim3(1024), kLdsBytes, (hipStream_t)stream, word);
    return (int)hipGetLastError();
}
