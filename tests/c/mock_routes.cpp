// Hooks around the CPU stand-in of the HIP runtime (mock_hip.cpp), linked with
// -Wl,--wrap for each, for tests/test_host_routes.py: device allocations
// counted or refused, uploads kept, downloads filled with a value, and every
// kernel launch seen by its name.  Test infrastructure, never linked into the
// library.
#include "../../paper_2607_00488_amd/csrc/shared.h"
#include <atomic>
#include <chrono>
#include <cstring>
#include <map>
#include <string>
#include <thread>
#include <vector>

namespace {
long g_mallocs = 0, g_fail_at = 0;
size_t g_keep = 0;
std::vector<char> g_kept;
bool g_fill_on = false;
double g_fill = 0.0;
std::atomic<long> g_launches{0};
int g_launch_us = 0;
// what the entries of the last grouped launch of points read and write
struct Range {
    unsigned long long entry, kind, at, bytes;
};
std::vector<Range> g_ranges;
void see_points(const nr::ShEval& e, int d) {
    const unsigned long long p = e.n_pts;
    g_ranges.push_back({(unsigned long long)d, 0, (unsigned long long)e.theta, p * 56});
    g_ranges.push_back({(unsigned long long)d, 1, (unsigned long long)e.rec, 8});
    g_ranges.push_back({(unsigned long long)d, 2, (unsigned long long)e.dpart, p * e.n_slice * 8});
    if (e.hpart)
        g_ranges.push_back({(unsigned long long)d, 3, (unsigned long long)e.hpart,
                            p * e.n_slice * nr::kShAcc * 8});
}
std::map<const void*, std::string>& names() {
    static std::map<const void*, std::string> m;
    return m;
}
}  // namespace

extern "C" {

// device allocations so far; the one of the given number (0: none) is refused
long mock_mallocs() { return g_mallocs; }
void mock_fail_at(long n) { g_fail_at = n; }
long mock_launches() { return g_launches; }
// a launch takes this long on the host (a full queue)
void mock_launch_time(int us) { g_launch_us = us; }
// keeps the last upload of exactly n bytes
void mock_keep(size_t n) { g_keep = n; g_kept.clear(); }
size_t mock_kept(void* out) {
    if (!g_kept.empty()) std::memcpy(out, g_kept.data(), g_kept.size());
    return g_kept.size();
}
// (entry, kind, address, bytes) of theta (0), records (1), deviance (2) and
// gradient sums (3) of every entry of the last grouped launch
long mock_ranges(unsigned long long* out, long cap) {
    for (size_t i = 0; i < g_ranges.size() && (long)(4 * i + 4) <= cap; ++i)
        std::memcpy(out + 4 * i, &g_ranges[i], 32);
    return (long)g_ranges.size();
}
// asynchronous downloads deliver doubles of this value
void mock_fill(int on, double v) { g_fill_on = on != 0; g_fill = v; }

hipError_t __real_hipMalloc(void**, size_t);
hipError_t __wrap_hipMalloc(void** p, size_t n) {
    if (++g_mallocs == g_fail_at) return hipErrorOutOfMemory;
    return __real_hipMalloc(p, n);
}

hipError_t __real_hipMemcpy(void*, const void*, size_t, hipMemcpyKind);
hipError_t __wrap_hipMemcpy(void* d, const void* s, size_t n, hipMemcpyKind k) {
    if (k == hipMemcpyHostToDevice && n && n == g_keep)
        g_kept.assign((const char*)s, (const char*)s + n);
    return __real_hipMemcpy(d, s, n, k);
}

hipError_t __real_hipMemcpyAsync(void*, const void*, size_t, hipMemcpyKind, hipStream_t);
hipError_t __wrap_hipMemcpyAsync(void* d, const void* s, size_t n, hipMemcpyKind k, hipStream_t st) {
    hipError_t e = __real_hipMemcpyAsync(d, s, n, k, st);
    if (k == hipMemcpyDeviceToHost && g_fill_on)
        for (size_t i = 0; i < n / sizeof(double); ++i) ((double*)d)[i] = g_fill;
    return e;
}

void __real___hipRegisterFunction(void**, const void*, char*, const char*, unsigned int, uint3*,
                                  uint3*, dim3*, dim3*, int*);
void __wrap___hipRegisterFunction(void** m, const void* f, char* d, const char* name,
                                  unsigned int l, uint3* a, uint3* b, dim3* c, dim3* e, int* w) {
    names()[f] = name;
    __real___hipRegisterFunction(m, f, d, name, l, a, b, c, e, w);
}

hipError_t __real_hipLaunchKernel(const void*, dim3, dim3, void**, size_t, hipStream_t);
hipError_t __wrap_hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t sh,
                                  hipStream_t s) {
    ++g_launches;
    if (g_launch_us) std::this_thread::sleep_for(std::chrono::microseconds(g_launch_us));
    const std::string& n = names()[f];
    if (n.find("ELi16EE") != std::string::npos || n.find("ILi16EE") != std::string::npos) {
        if (n.find("k_sh_eval") != std::string::npos) {
            g_ranges.clear();
            const auto& q = *(const nr::ShGroup<nr::ShEval, nr::kShGroup>*)args[0];
            for (int d = 0; d < q.n; ++d) see_points(q.p[d], d);
        } else if (n.find("k_sh_tail") != std::string::npos) {
            g_ranges.clear();
            const auto& q = *(const nr::ShGroup<nr::ShTail, nr::kShGroup>*)args[0];
            for (int d = 0; d < q.n; ++d) see_points(q.p[d].e, d);
        }
    }
    return __real_hipLaunchKernel(f, g, b, args, sh, s);
}
}
