// Stand-ins for the HIP runtime calls and the kernel launchers that api.cpp makes, for host-only
// checks of its calls: device memory is heap memory, asynchronous copies run when their stream is
// waited for (a source that has gone by then is found by the address sanitizer), launches are
// recorded, and events read a clock that the launches advance.
#include "fake_runtime.h"

#include <cstdlib>
#include <cstring>

#include "dsx_internal.h"

namespace fake {
std::vector<Launch> launches;
double clock_ms = 0.0;
double (*cost)(const Launch&) = nullptr;
size_t pending = 0;
size_t fail_copy_bytes = 0;
std::string fail_launch;

struct Copy { void* dst; const void* src; size_t n; };
static std::vector<Copy> copies;

static void flush()
{
    for (const Copy& c : copies) std::memcpy(c.dst, c.src, c.n);
    copies.clear();
    pending = 0;
}

void reset()
{
    flush();
    launches.clear();
    cost = nullptr;
    fail_copy_bytes = 0;
    fail_launch.clear();
}

static hipError_t launch(const char* name, int tc = 0)
{
    if (fail_launch == name) return hipErrorUnknown;
    launches.push_back({name, tc});
    if (cost) clock_ms += cost(launches.back());
    return hipSuccess;
}
}  // namespace fake

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { fake::flush(); std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind)
{
    fake::flush();
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    if (n == fake::fail_copy_bytes) return hipErrorUnknown;
    fake::copies.push_back({d, s, n});
    ++fake::pending;
    return hipSuccess;
}
hipError_t hipStreamSynchronize(hipStream_t) { fake::flush(); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { *s = nullptr; return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { *e = reinterpret_cast<hipEvent_t>(new double(0.0)); return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipEventCreate(e); }
hipError_t hipEventDestroy(hipEvent_t e) { delete reinterpret_cast<double*>(e); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t) { *reinterpret_cast<double*>(e) = fake::clock_ms; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { fake::flush(); return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t a, hipEvent_t b)
{
    *ms = (float)(*reinterpret_cast<double*>(b) - *reinterpret_cast<double*>(a));
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
}

namespace dsx {
hipError_t launch_sums(const SumsParams&, int, hipStream_t) { return fake::launch("sums"); }
hipError_t launch_fft_planes(const PlaneParams&, hipStream_t) { return fake::launch("fft_planes"); }
hipError_t launch_fft_axis1(const Axis1Params& p, hipStream_t) { return fake::launch("fft_axis1", p.tc); }
hipError_t launch_recombine_nuclear(const RecombParams&, int, int, int, size_t, hipStream_t) { return fake::launch("nuclear"); }
hipError_t launch_recombine_magnetic(const RecombParams&, int, int, size_t, hipStream_t) { return fake::launch("magnetic"); }
hipError_t launch_recombine_direct(const RecombParams&, hipStream_t) { return fake::launch("direct"); }
hipError_t launch_recombine_magnetic_rows(const RecombParams&, int, size_t, hipStream_t) { return fake::launch("magnetic_rows"); }
hipError_t launch_bragg(const BraggParams&, int, hipStream_t) { return fake::launch("bragg"); }
hipError_t launch_dw_mean(const DwParams&, hipStream_t) { return fake::launch("dw_mean"); }
hipError_t launch_lanczos(const LanczosParams&, hipStream_t) { return fake::launch("lanczos"); }
hipError_t launch_lanczos_points(const PointsParams&, hipStream_t) { return fake::launch("points"); }
hipError_t launch_lanczos_stencil(const LanczosParams&, hipStream_t) { return fake::launch("stencil"); }
int recombine_max_threads(int, int) { return 512; }
size_t planes_lds_bytes(const PlaneParams&) { return 0; }
size_t axis1_lds_bytes(const Axis1Params&) { return 0; }
size_t lanczos_lds_bytes(const LanczosParams&) { return 0; }
}  // namespace dsx
