// Which kernels the library launches, and how, without a GPU: this program stands in for the HIP runtime (its definitions come before those of
// the shared library), so that calls of the C ABI run their host code, device memory is host memory and launches are printed.
//   launch_routes_driver libnetmax.so < cases
// A case is a line: iterations, workers, batch, bytes by which the features miss an aligned address, 1 for a stream under capture, 1 for a
// device with cooperative launches, 1 for bfloat16 operands, 1 for the fusion switch, layer widths.  A line of output:
// "plain:kernel:arguments:workgroups" or "cooperative:..." in order: netmax_init, '|', one iteration by separate calls, '|', netmax_run.
// Arguments: the template's, without spaces.
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <cxxabi.h>
#include <dlfcn.h>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "../include/netmax.h"

static std::map<const void *, std::pair<std::string, std::string>> g_names;
static bool g_capturing, g_cooperative;
static dim3 g_grid, g_block;
static size_t g_shared;
static hipStream_t g_stream;
static std::ostringstream g_out;

// netmax::name<...>(...) of a mangled name: the last part of the nested name
static std::string short_name(const std::string &mangled)
{
    size_t at = mangled.find("_ZN6netmax");
    at = at == std::string::npos ? 2 : at + 10;
    const int n = std::atoi(mangled.c_str() + at);
    while (at < mangled.size() && isdigit(mangled[at])) ++at;
    return n > 0 ? mangled.substr(at, n) : mangled;
}

// its template arguments
static std::string arguments(const std::string &mangled)
{
    int status = 0;
    char *whole = abi::__cxa_demangle(mangled.c_str(), nullptr, nullptr, &status);
    if (!whole) return "";
    const std::string s(whole);
    free(whole);
    std::string of;
    const size_t from = s.find('<'), to = s.find('>');
    for (size_t k = from; from < s.find('(') && k < to; ++k)
        if (k > from && s[k] != ' ') of += s[k];
    return of;
}
static void launched(const char *how, const void *function, dim3 grid)
{
    g_out << ' ' << how << ':' << g_names[function].first << ':' << g_names[function].second << ':' << (uint64_t)grid.x * grid.y * grid.z;
}

extern "C" {
void **__hipRegisterFatBinary(const void *) { static void *handle; return &handle; }
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *function, char *, const char *name, unsigned, void *, void *, dim3 *, dim3 *, int *) { g_names[function] = {short_name(name), arguments(name)}; }
hipError_t __hipPushCallConfiguration(dim3 grid, dim3 block, size_t shared, hipStream_t s)
{
    g_grid = grid; g_block = block; g_shared = shared; g_stream = s;
    return hipSuccess;
}
hipError_t __hipPopCallConfiguration(dim3 *grid, dim3 *block, size_t *shared, hipStream_t *s)
{
    *grid = g_grid; *block = g_block; *shared = g_shared; *s = g_stream;
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void *function, dim3 grid, dim3, void **, size_t, hipStream_t) { launched("plain", function, grid); return hipSuccess; }
hipError_t hipLaunchCooperativeKernel(const void *function, dim3 grid, dim3, void **, unsigned, hipStream_t) { launched("cooperative", function, grid); return hipSuccess; }
hipError_t hipGetDevice(int *dev) { *dev = 0; return hipSuccess; }
hipError_t hipSetDevice(int) { return hipSuccess; }
hipError_t hipDeviceGetAttribute(int *value, hipDeviceAttribute_t what, int)
{
    *value = what == hipDeviceAttributeCooperativeLaunch ? g_cooperative : 256;            // else: the number of compute units
    return hipSuccess;
}
// one workgroup a compute unit: what the registers of the whole-iteration kernels leave room for
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int *blocks, const void *, int, size_t shared) { *blocks = shared <= 160 * 1024; return hipSuccess; }
hipError_t hipFuncSetAttribute(const void *, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipGetSymbolAddress(void **p, const void *) { static char place[8]; *p = place; return hipSuccess; }
const char *hipGetErrorString(hipError_t) { return "error"; }
hipError_t hipGetLastError() { return hipSuccess; }
hipError_t hipMalloc(void **p, size_t n) { *p = calloc(1, n); return *p ? hipSuccess : hipErrorOutOfMemory; }
hipError_t hipFree(void *p) { free(p); return hipSuccess; }
hipError_t hipMemcpy(void *to, const void *from, size_t n, hipMemcpyKind) { memcpy(to, from, n); return hipSuccess; }
hipError_t hipMemcpyAsync(void *to, const void *from, size_t n, hipMemcpyKind, hipStream_t) { memcpy(to, from, n); return hipSuccess; }
// on the null stream: not ordered ahead of what a context's own stream does, so not for its memory
hipError_t hipMemset(void *, int, size_t) { return hipErrorNotSupported; }
hipError_t hipMemsetAsync(void *p, int v, size_t n, hipStream_t) { memset(p, v, n); return hipSuccess; }
hipError_t hipStreamSynchronize(hipStream_t) { return hipSuccess; }
hipError_t hipStreamIsCapturing(hipStream_t, hipStreamCaptureStatus *status)
{
    *status = g_capturing ? hipStreamCaptureStatusActive : hipStreamCaptureStatusNone;
    return hipSuccess;
}
hipError_t hipStreamBeginCapture(hipStream_t, hipStreamCaptureMode) { return hipErrorNotSupported; }
hipError_t hipStreamEndCapture(hipStream_t, hipGraph_t *) { return hipErrorNotSupported; }
hipError_t hipGraphInstantiate(hipGraphExec_t *, hipGraph_t, hipGraphNode_t *, char *, size_t) { return hipErrorNotSupported; }
hipError_t hipGraphLaunch(hipGraphExec_t, hipStream_t) { return hipErrorNotSupported; }
hipError_t hipGraphDestroy(hipGraph_t) { return hipSuccess; }
hipError_t hipGraphExecDestroy(hipGraphExec_t) { return hipSuccess; }
}

int main(int argc, char **argv)
{
    void *lib = argc == 2 ? dlopen(argv[1], RTLD_NOW) : nullptr;
    if (!lib) {
        fprintf(stderr, "%s\n", argc == 2 ? dlerror() : "usage: launch_routes_driver libnetmax.so < cases");
        return 2;
    }
#define ENTRY(name) const auto name##_ = reinterpret_cast<decltype(&name)>(dlsym(lib, #name))
    ENTRY(netmax_init); ENTRY(netmax_bind_state); ENTRY(netmax_bind_data); ENTRY(netmax_run); ENTRY(netmax_sample_peers); ENTRY(netmax_local_step);
    ENTRY(netmax_mix); ENTRY(netmax_set_fusion); ENTRY(netmax_destroy); ENTRY(netmax_last_error);
#undef ENTRY
    for (std::string line; std::getline(std::cin, line);) {
        std::istringstream in(line);
        int iters, offset, capture, cooperative, bf16, fused;
        netmax_config c{};
        in >> iters >> c.M >> c.batch >> offset >> capture >> cooperative >> bf16 >> fused;
        int widths = 0;
        while (widths <= NETMAX_MAX_LAYERS && in >> c.dims[widths]) ++widths;
        c.n_layers = widths - 1;
        for (int l = 0; l < c.n_layers; ++l) c.D += c.dims[l] * c.dims[l + 1] + c.dims[l + 1];
        c.ld = (c.D + NETMAX_TILE - 1) / NETMAX_TILE * NETMAX_TILE;
        c.model = NETMAX_MLP;
        c.gemm_in = bf16 ? NETMAX_BF16 : NETMAX_F32;
        c.lr = 0.1f; c.rho = 0.001f; c.momentum = 0.9f; c.seed = 1;
        c.stream = &c;                                       // any: a stream of its own
        std::vector<double> P((size_t)c.M * c.M, 1.0 / (c.M - 1));
        for (int i = 0; i < c.M; ++i) P[(size_t)i * c.M + i] = 0.0;
        c.P = P.data();
        std::vector<int64_t> off(c.M + 1);
        for (int i = 0; i <= c.M; ++i) off[i] = 10 * i;
        // addresses only: nothing but kernels looks behind them
        auto at = [](uintptr_t a) { return reinterpret_cast<float *>(a << 32); };
        std::vector<int32_t> peers(c.M);
        netmax_ctx *ctx = nullptr;
        g_capturing = false;
        g_cooperative = cooperative;
        g_out.str("");
        int rc = netmax_init_(&ctx, &c);
        if (rc == NETMAX_OK) rc = netmax_bind_state_(ctx, at(1), at(2), at(3), at(4));
        if (rc == NETMAX_OK) rc = netmax_bind_data_(ctx, reinterpret_cast<char *>(at(5)) + offset, reinterpret_cast<int32_t *>(at(6)), off.data());
        if (rc == NETMAX_OK && fused) rc = netmax_set_fusion_(ctx, 1);
        g_capturing = capture;
        g_out << " |";
        if (rc == NETMAX_OK) rc = netmax_sample_peers_(ctx, 0, peers.data());
        if (rc == NETMAX_OK) rc = netmax_local_step_(ctx, 0);
        if (rc == NETMAX_OK) rc = netmax_mix_(ctx, 0, peers.data());
        g_out << " |";
        if (rc == NETMAX_OK) rc = netmax_run_(ctx, 0, iters, peers.data(), 0);
        if (rc != NETMAX_OK) {
            fprintf(stderr, "%s: %s\n", line.c_str(), netmax_last_error_(ctx));
            return 1;
        }
        g_capturing = false;
        netmax_destroy_(ctx);
        printf("%s\n", g_out.str().c_str());
    }
    return 0;
}
