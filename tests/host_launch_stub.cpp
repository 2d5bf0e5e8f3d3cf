// What the launchers of binsort.hip ask of the GPU, on the CPU: the last launch's workgroups and threads, and no launch.
#include <hip/hip_runtime.h>

extern "C" {
long long stub_blocks = 0, stub_threads = 0;

hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t, hipStream_t)
{
    stub_blocks = (long long)grid.x * grid.y * grid.z;
    stub_threads = (long long)block.x * block.y * block.z;
    return hipErrorUnknown;   // (the kernel is not called)
}
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipErrorUnknown; }
hipError_t hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t) { return hipErrorUnknown; }
hipError_t hipGetLastError() { return hipSuccess; }
void** __hipRegisterFatBinary(const void*) { return nullptr; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
}
