// Calls whose device memory cannot be had, on the CPU: libsig's host code over a HIP runtime of its own, which refuses allocations
// above a limit and writes down which kernels would have been launched.  Built by tests/test_host_sanitized.py.  A call that never
// returns ends in SIGALRM.
#include <unistd.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
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
hipError_t hipFuncGetAttributes(hipFuncAttributes *attributes, const void *) { *attributes = hipFuncAttributes{}; return hipErrorInvalidValue; }
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

static long failures = 0;
#define EXPECT(cond, ...) do { if (!(cond)) { ++failures; std::printf("FAILED %s: ", #cond); std::printf(__VA_ARGS__); std::printf("\n"); } } while (0)

static bool ran(const char *kernel)
{
    for (const std::string &name : launched)
        if (name.find(kernel) != std::string::npos) return true;
    return false;
}

int main()
{
    alarm(20);
    float x = 0.0f;   // every pointer of a call: nothing is read or written
    sig_ctx *ctx = nullptr;
    EXPECT(sig_create(&ctx) == SIG_OK, "sig_create");

    struct Call {
        const char *what;
        bool backward;
        int64_t B, L;
        int d, depth, stream;
        size_t most;           // bytes that can be had
        const char *kernel;    // runs with them
        int status;            // ... and the call's status
    };
    const Call calls[] = {
        // the reduced rows of the first: 2 * 39 * 12 * 14 floats; the general sweep needs less
        {"gradient at depth 3, twelve channels", true, 2, 40, 12, 3, 1, 48000, "sig_backward_general", SIG_OK},
        {"... with enough", true, 2, 40, 12, 3, 1, (size_t)1 << 30, "sig_stream_depth3", SIG_OK},
        {"... with nothing", true, 2, 40, 11, 3, 1, 0, nullptr, SIG_ERR_ALLOC},
        {"gradient at depth 2, a long path", true, 1, 1500, 6, 2, 1, 0, "sig_stream_depth2", SIG_OK},
        {"rows split across workgroups, in stretches", false, 1, 1400, 10, 4, 1, 0, "sig_split_rows", SIG_OK},
        {"few long paths in segments", false, 1, 2000, 6, 5, 0, 0, nullptr, SIG_ERR_ALLOC},
        {"gradient cut in time", true, 1, 600, 5, 4, 1, 0, nullptr, SIG_ERR_ALLOC},
    };
    for (const Call &c : calls) {
        sig_destroy(ctx);
        ctx = nullptr;
        EXPECT(sig_create(&ctx) == SIG_OK, "%s: sig_create", c.what);
        for (int again = 0; again < 2; ++again) {
            std::printf("%s, %zu bytes\n", c.what, c.most);
            std::fflush(stdout);
            launched.clear();
            refused = 0;
            most_bytes = c.most;
            const int rc = c.backward ? sig_backward(ctx, &x, c.B, c.L, c.d, c.depth, c.stream, &x, &x, &x, nullptr)
                                      : sig_compute(ctx, &x, c.B, c.L, c.d, c.depth, c.stream, &x, nullptr);
            EXPECT(rc == c.status, "%s: status %d", c.what, rc);
            EXPECT(again || (refused > 0) == (c.most < (size_t)1 << 30), "%s: %zu allocations refused", c.what, refused);
            EXPECT(c.kernel ? ran(c.kernel) : launched.empty(), "%s: %zu launches, first %s", c.what, launched.size(), launched.empty() ? "-" : launched[0].c_str());
            // the context is free for other threads
            most_bytes = (size_t)1 << 30;
            std::thread other([&] {
                float y = 0.0f;
                EXPECT(sig_backward(ctx, &y, 2, 40, 13, 3, 1, &y, &y, &y, nullptr) == SIG_OK, "%s: the call behind it", c.what);
            });
            other.join();
            sig_destroy(ctx);
            EXPECT(sig_create(&ctx) == SIG_OK, "sig_create");
        }
    }
    sig_destroy(ctx);
    std::printf("%s\n", failures ? "failed" : "no scratch ok");
    return failures ? 1 : 0;
}
