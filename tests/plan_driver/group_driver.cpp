// Runs groups and a server of the library on a device that is not there: the
// HIP calls and kernel launches that they make are defined here, take the place
// of the real ones, and print what matters for the launches:
//   capture N F   a graph of N launches with store policy F (1 non-temporal) begun
//   tile W H Z    tile and planes per block of a domain in an uploaded table
//   time          a timing event recorded
//   graph F       a captured graph of policy F launched
//   launch F      a single batched launch of policy F
// Usage: group_driver group STORAGE NCOMP C_NS STEPS NX NY NZ [NX NY NZ ...]
//        group_driver server STORAGE NCOMP C_NS TILE_X TILE_Y NX NY NZ [...]
// FAKE_FAIL_CAPTURE=K lets the K-th capture fail.  Exit code 3: a call that has to
// succeed did not; 4: create refused.
#include <hip/hip_runtime_api.h>

#include <atomic>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <mutex>
#include <set>
#include <string>
#include <vector>

#include "lbm_internal.h"

namespace {

std::recursive_mutex mu;
std::set<hipEvent_t> timing;
std::map<void*, int> graph_policy;  // of graphs and their executables
bool capturing = false;
int captured = 0, captured_nt = -1, captures = 0;
int next_handle = 1;

template <typename H>
H handle()
{
    return reinterpret_cast<H>(static_cast<uintptr_t>(0x1000 + 64 * next_handle++));
}

struct Lock {
    std::lock_guard<std::recursive_mutex> l{mu};
};

}  // namespace

extern "C" {

hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
hipError_t hipMemGetInfo(size_t* f, size_t* t) { *f = *t = size_t(1) << 30; return hipSuccess; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::malloc(n ? n : 1); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipHostMalloc(void** p, size_t n, unsigned) { return hipMalloc(p, n); }
hipError_t hipHostFree(void* p) { return hipFree(p); }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind) { std::memcpy(d, s, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind, hipStream_t)
{
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipStreamCreate(hipStream_t* s) { Lock l; *s = handle<hipStream_t>(); return hipSuccess; }
hipError_t hipStreamDestroy(hipStream_t) { return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e)
{
    Lock l;
    *e = handle<hipEvent_t>();
    timing.insert(*e);
    return hipSuccess;
}
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { Lock l; *e = handle<hipEvent_t>(); return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t)
{
    Lock l;
    if (timing.count(e)) std::printf("time\n");
    return hipSuccess;
}
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventQuery(hipEvent_t) { return hipSuccess; }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode)
{
    Lock l;
    const char* f = std::getenv("FAKE_FAIL_CAPTURE");
    if (++captures == (f ? std::atoi(f) : 0)) return hipErrorUnknown;
    capturing = true;
    captured = 0;
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    Lock l;
    capturing = false;
    *g = handle<hipGraph_t>();
    graph_policy[*g] = captured_nt;
    std::printf("capture %d %d\n", captured, captured_nt);
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* x, hipGraph_t g, hipGraphNode_t*, char*, size_t)
{
    Lock l;
    *x = handle<hipGraphExec_t>();
    graph_policy[*x] = graph_policy[g];
    return hipSuccess;
}
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
hipError_t hipGraphLaunch(hipGraphExec_t x, hipStream_t)
{
    Lock l;
    if (!graph_policy.count(x)) std::exit(3);
    std::printf("graph %d\n", graph_policy[x]);
    return hipSuccess;
}

}  // extern "C"

namespace hm {

hipError_t launch_init(const Problem&, const double*, void*, hipStream_t) { return hipSuccess; }
hipError_t launch_diagnostics(const Problem&, const void*, const float*, bool, double*, double*, double*, double*,
                              double* out, hipStream_t)
{
    for (int k = 0; k < 5; ++k) out[k] = 0.0;
    return hipSuccess;
}
int batch_blocks_per_cu(int storage, int ncomp, int) { return ncomp == 1 && storage != kF64 ? 2 : 1; }
int batch_encode(int, const BatchDomain* d, int n, void*)
{
    Lock l;
    for (int i = 0; i < n; ++i) std::printf("tile %d %d %d\n", d[i].tile_x, d[i].tile_y, d[i].zchunk);
    return n;
}
hipError_t launch_step_batch(int, int, int, const void*, int, int, bool nt, hipStream_t)
{
    Lock l;
    if (capturing) {
        ++captured;
        captured_nt = nt ? 1 : 0;
    } else {
        std::printf("launch %d\n", nt ? 1 : 0);
    }
    return hipSuccess;
}

}  // namespace hm

int main(int argc, char** argv)
{
    if (argc < 9) return 2;
    const bool group = std::string(argv[1]) == "group";
    lbm_params p{};
    p.storage = std::atoi(argv[2]);
    p.ncomp = std::atoi(argv[3]);
    p.c_ns = std::atoi(argv[4]);
    p.tau[0] = p.tau[1] = 1.0;
    p.g_scale = 1.0;
    std::vector<lbm_domain> doms;
    int64_t most = 0;
    for (int k = group ? 6 : 7; k + 2 < argc; k += 3) {
        doms.push_back({std::atoi(argv[k]), std::atoi(argv[k + 1]), std::atoi(argv[k + 2])});
        const lbm_domain& d = doms.back();
        most = std::max(most, static_cast<int64_t>(d.nx) * d.ny * d.nz);
    }
    const std::vector<float> ns(static_cast<size_t>(2 * most), 0.0f);
    const std::vector<double> rho(static_cast<size_t>(2 * most), 0.5);
    if (group) {
        std::vector<lbm_ctx*> ctx(doms.size(), nullptr);
        for (size_t i = 0; i < doms.size(); ++i)
            if (lbm_create(&doms[i], ns.data(), rho.data(), &p, nullptr, nullptr, &ctx[i])) return 3;
        lbm_group* g = nullptr;
        if (lbm_group_create(ctx.data(), static_cast<int32_t>(ctx.size()), &g)) return 4;
        std::printf("created\n");
        if (lbm_group_step(g, std::atoi(argv[5]))) return 3;
        lbm_group_destroy(g);
        for (lbm_ctx* c : ctx) lbm_destroy(c);
    } else {
        lbm_server_cfg cfg{};
        cfg.max_slots = 8;
        cfg.steps_per_tick = 4;
        cfg.storage = p.storage;
        cfg.ncomp = p.ncomp;
        cfg.c_ns = p.c_ns;
        cfg.max_cells = most;
        cfg.tile_x = std::atoi(argv[5]);
        cfg.tile_y = std::atoi(argv[6]);
        lbm_server* s = nullptr;
        if (lbm_server_create(&cfg, nullptr, &s)) return 4;
        {
            Lock l;
            std::printf("created\n");
        }
        for (const lbm_domain& d : doms) {  // one after the other, each alone
            lbm_request rq{};
            rq.dom = d;
            rq.n_s = ns.data();
            rq.rho_init = rho.data();
            rq.params = p;
            rq.max_steps = 8;
            uint64_t t = 0;
            lbm_result r{};
            if (lbm_batch_submit(s, &rq, &t) || lbm_batch_wait(s, t, 30.0, &r) || r.status) return 3;
        }
        lbm_server_destroy(s);
    }
    return 0;
}
