// Which kernels a call launches, on the CPU, also where device memory cannot be had: libsig's host code over a HIP runtime of its own,
// which refuses allocations above a limit and writes launches down.  Built and driven by tests/test_host_sanitized.py.
//   host_launches REGISTERS < calls       REGISTERS: lines "kernel registers", as the compiler reported them
// A call is a line "BYTES f|b B L D DEPTH STREAM" (forward or backward, with BYTES to be had); the answer "STATUS REFUSED kernel kernel ...".
// The context is a new one for each.  A call that never returns ends in SIGALRM.
#include <unistd.h>

#include <cstdint>
#include <cstdlib>
#include <fstream>
#include <iostream>
#include <map>
#include <string>
#include <thread>
#include <vector>

#include <hip/hip_runtime_api.h>

#include "sig.h"

static size_t most_bytes = 0, refused = 0;
static std::vector<std::string> launched;
static std::map<const void *, std::string> &kernels()
{
    static std::map<const void *, std::string> names;
    return names;
}
static std::map<std::string, int> registers;
struct Launch { dim3 grid, block; size_t lds; hipStream_t stream; };
static thread_local Launch pushed;
static char storage[1 << 16];

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterFunction(void **, const void *host, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { kernels()[host] = name; }
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t lds, hipStream_t stream)
{
    pushed = Launch{grid, block, lds, stream};
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *lds, hipStream_t *stream)
{
    *grid = pushed.grid;
    *block = pushed.block;
    *lds = pushed.lds;
    *stream = pushed.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *host, dim3, dim3, void **, size_t, hipStream_t) { launched.push_back(kernels()[host]); return hipSuccess; }
hipError_t hipGetDevice(int *device) { *device = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t, int) { *value = 256; return hipSuccess; }
hipError_t hipGetSymbolAddress(void **address, const void *) { *address = storage; return hipSuccess; }
hipError_t hipFuncGetAttributes(hipFuncAttributes *attributes, const void *host)
{
    *attributes = hipFuncAttributes{};
    attributes->numRegs = registers[kernels()[host]];
    return attributes->numRegs > 0 ? hipSuccess : hipErrorInvalidValue;
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status) { *status = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipMalloc(void **p, size_t bytes)
{
    *p = nullptr;
    if (bytes > most_bytes) { ++refused; return hipErrorOutOfMemory; }
    *p = std::malloc(64);   // (nothing is launched, so nothing writes to it)
    return hipSuccess;
}
hipError_t hipFree(void *p) { std::free(p); return hipSuccess; }
hipError_t hipDeviceSynchronize() { return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
}

int main(int argc, char **argv)
{
    alarm(60);
    if (argc > 1) {
        std::ifstream file(argv[1]);
        std::string kernel;
        for (int count; file >> kernel >> count;) registers[kernel] = count;
    }
    float x = 0.0f;   // every pointer of a call: nothing is read or written
    size_t bytes;
    char direction;
    int64_t B, L;
    int d, depth, stream;
    while (std::cin >> bytes >> direction >> B >> L >> d >> depth >> stream) {
        sig_ctx *ctx = nullptr;
        if (sig_create(&ctx) != SIG_OK) return 1;
        launched.clear();
        refused = 0;
        most_bytes = bytes;
        const int rc = direction == 'b' ? sig_backward(ctx, &x, B, L, d, depth, stream, &x, &x, &x, nullptr)
                                        : sig_compute(ctx, &x, B, L, d, depth, stream, &x, nullptr);
        std::cout << rc << ' ' << refused;
        for (const std::string &kernel : launched) std::cout << ' ' << kernel;
        std::cout << std::endl;
        // the context is free for other threads
        most_bytes = (size_t)1 << 40;
        int other = -1;
        std::thread([&] { other = sig_backward(ctx, &x, 2, 40, 13, 3, 1, &x, &x, &x, nullptr); }).join();
        sig_destroy(ctx);
        if (other != SIG_OK) return 1;
    }
    return 0;
}
