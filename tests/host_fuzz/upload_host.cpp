// svo_upload where host memory runs out, on the CPU (test infrastructure:
// tests/test_host_upload.py compiles and runs it): the host source is included
// whole over a stubbed HIP runtime that counts what is allocated, and each
// run lets one host allocation more succeed before the next one fails.
#include "../../paper_1911_06001_amd/csrc/svo_host.cpp"

#include <cstdlib>

namespace {
long allow = -1;      // host allocations left (-1: no limit)
int held = 0;         // device and pinned blocks, and events
}

void* operator new(size_t n) {
    if (allow == 0) throw std::bad_alloc();
    if (allow > 0) --allow;
    if (void* p = std::malloc(n ? n : 1)) return p;
    throw std::bad_alloc();
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

namespace svo {
hipError_t launch_primary_rays(const CameraArgs&, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_ao_rays(const AoArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_shade(const ShadeArgs&, hipStream_t) { return hipSuccess; }
hipError_t static_scratch(int, unsigned char**) { return hipErrorNoDevice; }
hipError_t launch_zero_words(uint32_t*, uint32_t, hipStream_t) { return hipSuccess; }
size_t trace_lds_bytes(const TraceArgs&, uint32_t) { return 0; }
hipError_t prepare_trace(size_t) { return hipSuccess; }
hipError_t launch_trace(const TraceArgs&, const LaunchCfg&, hipStream_t, const unsigned char*, size_t) { return hipSuccess; }
}  // namespace svo

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { ++held; return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { --held; std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return hipMalloc((void**)e, 1); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return hipMalloc((void**)e, 1); }
hipError_t hipEventDestroy(hipEvent_t e) { return hipFree((void*)e); }
hipError_t hipEventRecord(hipEvent_t, hipStream_t) { return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* s) { *s = hipStreamCaptureStatusNone; return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t, hipEvent_t, unsigned) { return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipGetDeviceCount(int* n) { *n = 1; return hipSuccess; }
hipError_t hipDeviceSynchronize(void) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 163840; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "stub"; }
}

int main() {
    // a world root over two leaves and a transformed node over one
    const uint64_t nodes[] = {7ull | (1ull << 8), 1ull << 32, 2ull << 32, 1ull | (0x80000000ull << 32), 3ull << 32};
    const uint32_t child[] = {4};
    const float cell[] = {0.f, 0.f, 0.f, 1.f}, lo[] = {0.f, 0.f, 0.f};
    svo_ctx ctx;
    ctx.n_cu = 256;
    ctx.max_lds = ctx.lds_per_cu = 163840;
    ctx.cfg = default_config();
    for (long n = 0;; ++n) {
        svo_scene h = 0;
        allow = n;
        const int rc = svo_upload(&ctx, nodes, 5, 0, lo, 2.f, 20, child, cell, 1, &h);
        allow = -1;
        if (rc == SVO_OK) {
            svo_free_scene(&ctx, h);
            std::printf("failures %ld held %d\n", n, held);
            return held ? 1 : 0;
        }
        if (rc != SVO_ENOMEM || held || !ctx.scenes.empty()) {
            std::printf("allocation %ld: code %d, %d blocks held\n", n, rc, held);
            return 1;
        }
    }
}
