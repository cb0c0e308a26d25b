// liblbmd.so's host side without a GPU: this program defines the HIP entry
// points the library imports.  Memory is host memory, kernels do nothing, and
// every launch, event and graph call is printed in order.  Test code only.
//
//   hip_record <precision> <mode> <graph_steps> <steps,steps,...> <L:N:chain_len,...> [shared]
//
// shared: that many streams after the first share its hardware queue.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <map>
#include <string>
#include <vector>

#include "../../include/lbmd.h"

namespace {
// the library registers its kernels before this program's own statics exist
std::map<const void*, std::string>& kernels() { static std::map<const void*, std::string> k; return k; }
std::map<const void*, int> ids;   // streams, events, graphs: small numbers in order of appearance
int id(const void* p) { return ids.emplace(p, (int)ids.size()).first->second; }
uintptr_t next_handle = 0x1000;
template <typename T> hipError_t make(T* out) { *out = (T)(next_handle += 16); id(*out); return hipSuccess; }
bool capture = false;
int shared = 0;
struct Config { dim3 grid, block; size_t lds; hipStream_t stream; };
std::vector<Config> configs;
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* m; return &m; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*)
{
    int st;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string s = st == 0 ? d : name;
    std::free(d);
    s = s.substr(0, s.find('('));
    s = s.substr(s.find("lbd::") == std::string::npos ? 0 : s.find("lbd::") + 5);
    for (size_t k; (k = s.find(' ')) != std::string::npos;) s.erase(k, 1);
    kernels()[host] = s;
}
void __hipRegisterVar(void**, void*, char*, char* name, int, size_t size, int, int) { std::printf("var %s %zu\n", name, size); }
hipError_t __hipPushCallConfiguration(dim3 g, dim3 b, size_t lds, hipStream_t s)
{
    configs.push_back({g, b, lds, s});
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3* g, dim3* b, size_t* lds, hipStream_t* s)
{
    const Config c = configs.back();
    configs.pop_back();
    *g = c.grid; *b = c.block; *lds = c.lds; *s = c.stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t s)
{
    if (kernels()[f] == "k_probe_wait") (*(uint32_t**)args[0])[1] = id(s) > shared ? 1u : 0u;
    std::printf("launch %s stream %d grid %u,%u block %u\n", kernels()[f].c_str(), id(s), g.x, g.y, b.x);
    return hipSuccess;
}
hipError_t hipGetDevice(int* d) { *d = 0; return hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { *v = 256; return hipSuccess; }
const char* hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipGetSymbolAddress(void** p, const void* s) { *p = (void*)s; return hipSuccess; }
hipError_t hipMalloc(void** p, size_t n) { *p = std::calloc(n, 1); return hipSuccess; }
hipError_t hipFree(void* p) { std::free(p); return hipSuccess; }
hipError_t hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k)
{
    std::printf("copy %s %zu\n", k == hipMemcpyDeviceToHost ? "out" : "in", n);
    std::memcpy(d, s, n);
    return hipSuccess;
}
hipError_t hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t) { return hipMemcpy(d, s, n, k); }
hipError_t hipMemsetAsync(void* d, int v, size_t n, hipStream_t) { std::memset(d, v, n); return hipSuccess; }
hipError_t hipStreamCreateWithFlags(hipStream_t* s, unsigned) { return make(s); }
hipError_t hipStreamDestroy(hipStream_t s) { std::printf("destroy %d\n", id(s)); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipEventCreate(hipEvent_t* e) { return make(e); }
hipError_t hipEventCreateWithFlags(hipEvent_t* e, unsigned) { return make(e); }
hipError_t hipEventDestroy(hipEvent_t) { return hipSuccess; }
hipError_t hipEventElapsedTime(float* ms, hipEvent_t, hipEvent_t) { *ms = 1.f; return hipSuccess; }
hipError_t hipEventSynchronize(hipEvent_t) { return hipSuccess; }
hipError_t hipEventRecord(hipEvent_t e, hipStream_t s) { std::printf("record %d stream %d\n", id(e), id(s)); return hipSuccess; }
hipError_t hipStreamWaitEvent(hipStream_t s, hipEvent_t e, unsigned) { std::printf("wait %d stream %d\n", id(e), id(s)); return hipSuccess; }
hipError_t hipStreamBeginCapture(hipStream_t s, hipStreamCaptureMode)
{
    capture = true;
    std::printf("capture stream %d\n", id(s));
    return hipSuccess;
}
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t* g)
{
    capture = false;
    std::printf("captured\n");
    return make(g);
}
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus* st)
{
    *st = capture ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipGraphInstantiate(hipGraphExec_t* e, hipGraph_t, hipGraphNode_t*, char*, size_t) { return make(e); }
hipError_t hipGraphLaunch(hipGraphExec_t e, hipStream_t s) { std::printf("replay %d stream %d\n", id(e), id(s)); return hipSuccess; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

#define CHECK(call) do { if ((call) != LB_OK) { std::printf("failed: %s: %s\n", #call, lb_last_error(h)); return 1; } } while (0)

int main(int argc, char** argv)
{
    if (argc < 6) return 2;
    shared = argc > 6 ? std::atoi(argv[6]) : 0;
    lb_handle* h = nullptr;
    std::vector<lb_box_desc> boxes;
    std::vector<double> x0;
    for (char* t = std::strtok(argv[5], ","); t; t = std::strtok(nullptr, ",")) {
        lb_box_desc d{};
        if (std::sscanf(t, "%d:%d:%d", &d.L, &d.n_beads, &d.chain_len) != 3) return 2;
        d.rho0 = d.omega_shear = d.omega_bulk = d.omega_ghost = d.bead_mass = d.eps_wca = d.sigma_wca = 1.0;
        d.kT = 1e-2; d.thermalize = 2; d.tau_lb = 0.1; d.md_dt = 0.01; d.md_substeps = 10;
        d.zeta = 20.0; d.k_fene = 30.0; d.r0_fene = 1.5; d.seed = 1; d.box_id = (uint32_t)boxes.size();
        for (int b = 0; b < d.n_beads; ++b) { x0.push_back(0.97 * b); x0.push_back(1.0); x0.push_back(1.0); }
        boxes.push_back(d);
    }
    size_t sb, cb;
    CHECK(lb_query_sizes(boxes.data(), (int)boxes.size(), std::atoi(argv[1]), 0, &sb, &cb));
    auto alloc = [](size_t n) { return std::aligned_alloc(256, (n + 255) / 256 * 256); };
    CHECK(lb_init(boxes.data(), (int)boxes.size(), std::atoi(argv[1]), 0, x0.data(), alloc(sb), alloc(cb), nullptr, &h));
    std::printf("launch mode\n");
    CHECK(lb_set_launch(h, std::atoi(argv[2]), std::atoi(argv[3])));
    for (char* t = std::strtok(argv[4], ","); t; t = std::strtok(nullptr, ",")) {
        std::printf("step %s\n", t);
        CHECK(lb_step(h, std::atoi(t)));
    }
    std::printf("export\n");
    std::vector<char> state(lb_state_host_bytes(h));
    CHECK(lb_export_state(h, state.data(), state.size()));
    std::printf("free\n");
    lb_free(h);
    return 0;
}
