// The library's host code on a stand-in for the HIP runtime (no GPU): allocations are
// addresses only, copies do nothing, kernel launches are recorded. Linked with
// libipoisson.so into a program whose runtime functions replace the real ones. Reads
// one request per line, d n0 .. n_{d-1} order precision flags call, and prints
//   call = size:    the plan's workspace bytes
//   call = execute, adjoint: the launches of one call, one "kernel grid-blocks threads"
//   each, and a line "end"
#include <cxxabi.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <iostream>
#include <map>
#include <sstream>
#include <string>
#include <vector>

#include "ipoisson.h"

struct Dim {
    uint32_t x, y, z;
};
struct Config {
    Dim grid, block;
    size_t lds;
    void *stream;
};

static std::map<const void *, std::string> &names()
{
    static std::map<const void *, std::string> m;
    return m;
}
static std::vector<std::string> g_launches;
static std::vector<Config> g_config;
static uintptr_t g_next = (uintptr_t)1 << 40;

extern "C" {
void **__hipRegisterFatBinary(const void *)
{
    static void *h;
    return &h;
}
void __hipUnregisterFatBinary(void **) {}
void __hipRegisterVar(void **, void *, char *, char *, int, size_t, int, int) {}
void __hipRegisterFunction(void **, const void *f, char *, const char *name, unsigned, void *, void *, void *, void *,
                           int *)
{
    int st = 0;
    char *s = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    std::string n = s ? s : name;
    std::free(s);
    n = n.substr(0, n.find("(ips::"));
    for (size_t at; (at = n.find(' ')) != std::string::npos;) n.erase(at, 1);
    for (size_t at; (at = n.find("ips::")) != std::string::npos;) n.erase(at, 5);
    if (n.compare(0, 5, "voidk") == 0) n.erase(0, 4);
    names()[f] = n;
}
int __hipPushCallConfiguration(Dim g, Dim b, size_t lds, void *st)
{
    g_config.push_back({g, b, lds, st});
    return 0;
}
int __hipPopCallConfiguration(Dim *g, Dim *b, size_t *lds, void **st)
{
    const Config c = g_config.back();
    g_config.pop_back();
    *g = c.grid, *b = c.block, *lds = c.lds, *st = c.stream;
    return 0;
}
int hipLaunchKernel(const void *f, Dim g, Dim b, void **, size_t, void *)
{
    g_launches.push_back(names()[f] + " " + std::to_string((uint64_t)g.x * g.y * g.z) + " " + std::to_string(b.x));
    return 0;
}
int hipMalloc(void **p, size_t n)
{
    *p = reinterpret_cast<void *>(g_next);
    g_next += (n + 4095) & ~(size_t)4095;
    return 0;
}
int hipFree(void *) { return 0; }
int hipMemcpy(void *, const void *, size_t, int) { return 0; }
int hipMemset(void *, int, size_t) { return 0; }
int hipGetDevice(int *d) { return *d = 0; }
int hipSetDevice(int) { return 0; }
int hipDeviceSynchronize() { return 0; }
int hipStreamSynchronize(void *) { return 0; }
int hipDeviceGetAttribute(int *v, int, int)
{
    *v = 256;
    return 0;
}
int hipFuncSetAttribute(const void *, int, int) { return 0; }
int hipOccupancyMaxActiveBlocksPerMultiprocessor(int *n, const void *, int, size_t)
{
    *n = 2;
    return 0;
}
int hipGetLastError() { return 0; }
const char *hipGetErrorString(int) { return "stub"; }
}

int main()
{
    std::string line;
    while (std::getline(std::cin, line)) {
        std::istringstream in(line);
        int d = 0, order = 0, precision = 0;
        unsigned flags = 0;
        int64_t n[3] = {1, 1, 1};
        const double h[3] = {0.1, 0.1, 0.1};
        std::string call;
        in >> d;
        for (int a = 0; a < d && a < 3; ++a) in >> n[a];
        in >> order >> precision >> flags >> call;
        ips_plan p = nullptr;
        int rc = ips_plan_create(&p, d, n, h, order, precision, flags);
        if (rc) {
            std::printf("error %d\nend\n", rc);
            continue;
        }
        if (call == "size") {
            size_t bytes = 0;
            ips_plan_workspace_size(p, &bytes);
            std::printf("%zu\n", bytes);
        } else {
            g_launches.clear();
            double *in_arr = reinterpret_cast<double *>((uintptr_t)3 << 44);
            double *out_arr = reinterpret_cast<double *>((uintptr_t)5 << 44);
            rc = call == "adjoint" ? ips_execute_adjoint(p, in_arr, out_arr, nullptr)
                                   : ips_execute(p, in_arr, out_arr, nullptr);
            if (rc) std::printf("error %d\n", rc);
            for (const std::string &s : g_launches) std::printf("%s\n", s.c_str());
            std::printf("end\n");
        }
        ips_plan_destroy(p);
    }
    return 0;
}
