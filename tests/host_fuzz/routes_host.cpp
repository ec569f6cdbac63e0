// Which candidate path and shape the library's host code picks for a launch,
// on the CPU (test infrastructure: tests/test_host_routes.py compiles and runs it).  The
// host source is included whole and the HIP runtime and the kernels' launch
// functions are stubs, so a launch ends in a look at its arguments.
#include "../../paper_1911_06001_amd/csrc/svo_host.cpp"

#include <cstdlib>

namespace {
svo::TraceArgs launched;
svo::LaunchCfg shape;
}

namespace svo {
hipError_t launch_primary_rays(const CameraArgs&, float*, hipStream_t) { return hipSuccess; }
hipError_t launch_ao_rays(const AoArgs&, hipStream_t) { return hipSuccess; }
hipError_t launch_shade(const ShadeArgs&, hipStream_t) { return hipSuccess; }
hipError_t static_scratch(int, unsigned char**) { return hipErrorNoDevice; }
hipError_t launch_zero_words(uint32_t*, uint32_t, hipStream_t) { return hipSuccess; }
size_t trace_lds_bytes(const TraceArgs& a, uint32_t waves) {   // tables and per-wave state, to the kilobyte
    return (size_t)a.n_frames * 64 + (size_t)a.n_bvh_total * sizeof(BvhNode) + (size_t)waves * 5632;
}
hipError_t prepare_trace(size_t) { return hipSuccess; }
hipError_t launch_trace(const TraceArgs& a, const LaunchCfg& c, hipStream_t, const unsigned char*, size_t) {
    launched = a;
    shape = c;
    return hipSuccess;
}
}  // namespace svo

extern "C" {
hipError_t hipMalloc(void** p, size_t n) { return (*p = std::malloc(n)) ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemset(void* p, int v, size_t n) { std::memset(p, v, n); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t*) { return hipSuccess; }
hipError_t hipEventCreateWithFlags(hipEvent_t*, unsigned) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
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

namespace {

// A world of 64 transformed cells, every part twice its cell's size: `n` of
// them in use, all candidates.
svo_scene upload(svo_ctx& ctx, uint32_t n) {
    std::vector<uint64_t> nodes;
    const uint32_t groups = (n + 7) / 8, leaf = 1 + groups + n;
    nodes.push_back((uint64_t)((1u << groups) - 1u) | (1ull << 8));
    for (uint32_t g = 0; g < groups; ++g) {
        const uint32_t cnt = std::min(8u, n - 8 * g);
        nodes.push_back((uint64_t)((1u << cnt) - 1u) | ((uint64_t)(groups - g + 8 * g) << 8));
    }
    for (uint32_t s = 0; s < n; ++s) nodes.push_back(1ull | ((uint64_t)(0x80000000u | s) << 32));
    nodes.push_back(0xFF0000FFull << 32);
    std::vector<uint32_t> child(n, leaf);
    std::vector<float> cell, fwd;
    for (uint32_t s = 0; s < n; ++s) {
        cell.insert(cell.end(), {0.f, 0.f, 0.f, 1.f});
        fwd.insert(fwd.end(), {2.f, 0, 0, 0, 0, 2.f, 0, 0, 0, 0, 2.f, (float)(10 + s)});
    }
    const float lo[3] = {0, 0, 0};
    svo_scene h = 0;
    if (svo_upload(&ctx, nodes.data(), nodes.size(), 0, lo, 4.f, 20, child.data(), cell.data(), n, &h) ||
        svo_set_transforms(&ctx, h, 0, n, fwd.data(), nullptr)) {
        std::printf("upload: %s\n", svo_last_error());
        std::exit(2);
    }
    return h;
}

}  // namespace

// routes_host CONTEXT TUNED CANDIDATES JOBS [WAVES BLOCKS]: sorted_candidates of
// the context and of the scene's tuning (-1: not tuned), and the configured
// shape; prints the path, the hierarchy nodes and the shape of a batch and of
// a plan, or what refused them.
int main(int argc, char** argv) {
    if (argc != 5 && argc != 7) return 2;
    const int tuned = std::atoi(argv[2]);
    const uint32_t n = (uint32_t)std::atoi(argv[3]), jobs = (uint32_t)std::atoi(argv[4]);
    svo_ctx ctx;
    ctx.n_cu = 256;
    ctx.max_lds = ctx.lds_per_cu = 163840;
    ctx.cfg = default_config();
    ctx.cfg.sorted_candidates = (uint32_t)std::atoi(argv[1]);
    if (argc == 7) {
        ctx.cfg.waves_per_block = (uint32_t)std::atoi(argv[5]);
        ctx.cfg.blocks_per_cu = (uint32_t)std::atoi(argv[6]);
    }
    std::vector<uint32_t> queue(svo::kQueueWords * kMaxStreams);
    ctx.d_queue = queue.data();
    const svo_scene h = upload(ctx, n);
    Scene* S = find_scene(&ctx, h);
    if (S->n_cand != n) return 3;
    if (tuned >= 0) {
        S->tuned = true;
        S->cfg = ctx.cfg;
        S->cfg.sorted_candidates = (uint32_t)tuned;
    }
    alignas(16) float rays[8] = {};
    uint32_t id[1];
    float t[1];
    std::vector<svo_job> J(jobs);
    for (svo_job& j : J) {
        j = svo_job{};
        j.scene = h;
        j.rays = rays;
        j.n = 1;
        j.out_id = id;
        j.out_t = t;
    }
    if (svo_trace_batch(&ctx, J.data(), jobs, nullptr))
        std::printf("batch refused: %s\n", svo_last_error());
    else
        std::printf("batch %s %u %ux%u\n", launched.sort_cand ? "one-by-one" : "hierarchy", launched.n_bvh_total,
                    shape.waves_per_block, launched.max_blocks / (uint32_t)ctx.n_cu);
    svo_plan_limits lim{};
    lim.max_jobs = jobs;
    lim.max_frames = jobs * (1 + n);
    svo_plan* p = nullptr;
    if (svo_plan_create(&ctx, &h, 1, &lim, &p) || svo_plan_set_jobs(&ctx, p, J.data(), jobs) || svo_plan_launch(&ctx, p, nullptr))
        std::printf("plan refused: %s\n", svo_last_error());
    else
        std::printf("plan %s %u %ux%u\n", launched.sort_cand ? "one-by-one" : "hierarchy", launched.n_bvh_total,
                    shape.waves_per_block, launched.max_blocks / (uint32_t)ctx.n_cu);
    svo_plan_destroy(&ctx, p);
    svo_free_scene(&ctx, h);
    for (auto& b : ctx.batch) {
        (void)hipFree(b.dev);
        (void)hipHostFree(b.host);
    }
    return 0;
}
