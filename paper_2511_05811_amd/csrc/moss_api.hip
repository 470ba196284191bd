// Status strings, cached device properties and call numbers of libmoss_hip.so.
#include <atomic>
#include <chrono>

#include <unistd.h>

#include "moss_internal.h"
#include "moss_producer.h"

static std::atomic<int> g_cu_count[64];   // per device, 0 = not asked yet; racing first calls store the same value

int moss_internal_cu_count()
{
    int dev = 0;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= 64) return 0;
    int n = g_cu_count[dev].load();
    if (n == 0) {
        if (hipDeviceGetAttribute(&n, hipDeviceAttributeMultiprocessorCount, dev) != hipSuccess) return 0;
        g_cu_count[dev].store(n);
    }
    return n;
}

// The numbers start at a place that depends on time and process (mixed as in splitmix64), so that memory which another
// process left behind does not hold them.
uint64_t moss_next_call()
{
    static std::atomic<uint64_t> last{[] {
        uint64_t z = (uint64_t)std::chrono::system_clock::now().time_since_epoch().count() + ((uint64_t)getpid() << 40);
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull;
        z = (z ^ (z >> 27)) * 0x94D049BB133111EBull;
        return z ^ (z >> 31);
    }()};
    uint64_t c;
    do c = (last.fetch_add(1) + 1) & 0xFFFFFFFFFFFFull;
    while (c == 0);
    return c;
}

bool moss_may_number_calls(hipStream_t st)
{
    hipStreamCaptureStatus status;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();
        return false;
    }
    return status == hipStreamCaptureStatusNone;
}

extern "C" uint32_t moss_internal_interface(void) { return MOSS_INTERFACE; }

extern "C" int moss_device_cu_count(void) { return moss_internal_cu_count(); }

extern "C" const char *moss_status_string(int status)
{
    switch (status) {
        case MOSS_OK: return "ok";
        case MOSS_ERR_NULL: return "a required pointer is NULL";
        case MOSS_ERR_SHAPE: return "bad shape (non-positive, not a multiple of the group size, or too large)";
        case MOSS_ERR_ALIGN: return "pointer or leading dimension not aligned";
        case MOSS_ERR_WORKSPACE: return "workspace missing or too small";
        case MOSS_ERR_UNSUPPORTED: return "unsupported flag or dtype combination";
        case MOSS_ERR_HIP: return "HIP runtime error";
        default: return "unknown status";
    }
}
