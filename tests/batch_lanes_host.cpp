// The batch's lanes on the CPU: the HIP runtime and the solve are stand-ins that
// record which stream solved which problem, and the wait for one stream fails.
#include <atomic>
#include <chrono>
#include <cstdarg>
#include <cstdio>
#include <cstring>
#include <thread>

#include "cp_internal.h"

static char g_error[512] = "";
static std::atomic<int> g_streams{0};
static hipStream_t g_lost = nullptr;
static hipStream_t g_solved_on[16];

namespace cp {
void set_error(const char* fmt, ...) {
    va_list ap;
    va_start(ap, fmt);
    std::vsnprintf(g_error, sizeof g_error, fmt, ap);
    va_end(ap);
}
}  // namespace cp

extern "C" {
const char* cylpoisson_last_error(void) { return "text of an earlier failure"; }
// problem i's plan has nr = 100 - i; the lost stream's lane ends first
int cylpoisson_solve(cylpoisson_plan* p, const double*, double*, double, void* stream) {
    const int i = 100 - p->nr;
    g_solved_on[i] = static_cast<hipStream_t>(stream);
    std::this_thread::sleep_for(std::chrono::milliseconds(stream == g_lost ? 20 : 60));
    return CYLPOISSON_OK;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) {
    *e = reinterpret_cast<hipEvent_t>(1);
    return hipSuccess;
}
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "the stream was lost"; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) {
    *s = reinterpret_cast<hipStream_t>(static_cast<size_t>(0x100 * ++g_streams));
    if (g_streams == 2) g_lost = *s;
    return hipSuccess;
}
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t s) { return s == g_lost ? hipErrorUnknown : hipSuccess; }
}

int main() {
    constexpr int n = 7;
    cylpoisson_plan plans[n];
    cylpoisson_plan* pp[n];
    const double* rho[n] = {};
    double* phi[n] = {};
    int st[n], bad = 0;
    for (int i = 0; i < n; ++i) {
        plans[i].nr = 100 - i;
        plans[i].nt = plans[i].nz = 1;
        pp[i] = &plans[i];
    }
    const int status = cylpoisson_solve_batch(pp, rho, phi, n, 1e-12, nullptr, st);
    int lost = 0;
    for (int i = 0; i < n; ++i) {
        const bool on_lost = g_solved_on[i] == g_lost;
        lost += on_lost;
        std::printf("problem %d: status %d, lost stream %d\n", i, st[i], on_lost);
        if (st[i] != (on_lost ? CYLPOISSON_EHIP : CYLPOISSON_OK)) ++bad;
    }
    std::printf("batch status %d: %s\n", status, g_error);
    if (lost == 0 || lost == n || status != CYLPOISSON_EHIP) ++bad;
    if (!std::strstr(g_error, "the stream was lost")) ++bad;
    for (int i = 0; i < n; ++i)
        if (plans[i].share != 1) ++bad;
    return bad != 0;
}
