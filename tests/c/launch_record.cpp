// Runs libnoble's calls without a GPU and prints the kernel launches they make.
//
// The HIP functions that the library calls are defined here, in the
// executable, which the dynamic linker prefers over libamdhip64: a launch is
// recorded instead of made, and the device is said to be a gfx950.  Device
// pointers are made-up addresses that nothing reads.
//
// Reads lines "CALL T d_in d_out r dtype activation groups scratch" from
// standard input (CALL: fwd, static, bwd or storage; scratch: bytes, -1: what
// the size query gives) and prints for each "call <status>", its launches
// as "launch <gx> <gy> <block> <kernel>" and the arrays that a launch clears
// as "zero <argument> <bytes>" (argument: its name, or an address).
#include <cxxabi.h>
#include <stdint.h>

#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <map>
#include <string>

#include <hip/hip_runtime.h>

#include "noble.h"
#include "noble_binding.h"
#include "noble_skinny.hpp"

namespace {
std::map<const void*, std::string>& kernels() {
    static std::map<const void*, std::string> m;
    return m;
}
// Argument i of a call: 2^44 bytes apart, beyond any buffer of the calls.
const char* const kNames[] = {"x",  "W",  "b",  "W_down", "omega1", "phi1", "M",     "omega2",  "phi2",  "W_up",    "y",      "reserve",
                              "scratch", "dy", "dx", "dW", "db", "dW_down", "dM", "dW_up", "domega1", "dphi1", "domega2", "dphi2"};
enum { X, W, B, WD, O1, P1, M, O2, P2, WU, Y, RES, SCR, DY, DX, DW, DB, DWD, DM, DWU, DO1, DP1, DO2, DP2 };
void* ptr(int i) { return reinterpret_cast<void*>((uint64_t)(i + 1) << 44); }
float* fptr(int i) { return static_cast<float*>(ptr(i)); }
std::string where(const void* p) {
    const uint64_t a = reinterpret_cast<uint64_t>(p), i = a >> 44;
    char off[40];
    snprintf(off, sizeof off, "+%llu", (unsigned long long)(a & ((1ull << 44) - 1)));
    if (i < 1 || i > sizeof kNames / sizeof kNames[0]) return off;
    return (a & ((1ull << 44) - 1)) ? kNames[i - 1] + std::string(off) : kNames[i - 1];
}
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) {
    static void* h = nullptr;
    return &h;
}
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void* host, char*, const char* name, unsigned, void*, void*, void*, void*, int*) {
    int st = 0;
    char* d = abi::__cxa_demangle(name, nullptr, nullptr, &st);
    kernels()[host] = d ? d : name;
    free(d);
}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
hipError_t hipGetDevice(int* d) {
    *d = 0;
    return hipSuccess;
}
#undef hipGetDeviceProperties
hipError_t hipGetDevicePropertiesR0600(hipDeviceProp_tR0600* p, int) {
    memset(p, 0, sizeof *p);
    strcpy(p->gcnArchName, "gfx950:sramecc+:xnack-");
    return hipSuccess;
}
hipError_t hipGetSymbolAddress(void** p, const void*) {
    *p = ptr(SCR);
    return hipSuccess;
}
hipError_t hipLaunchKernel(const void* f, dim3 g, dim3 b, void** args, size_t, hipStream_t) {
    const auto it = kernels().find(f);
    const std::string name = it == kernels().end() ? "?" : it->second;
    printf("launch %u %u %u %s\n", g.x, g.y, b.x * b.y * b.z, name.c_str());
    noble::ZeroList z{};
    if (name.find("proj_kernel") != std::string::npos) z = static_cast<const noble::ProjArgs*>(args[0])->z;
    if (name.find("zero_kernel") != std::string::npos) z = *static_cast<const noble::ZeroList*>(args[0]);
    for (int i = 0; i < z.count; ++i) printf("zero %s %lld\n", where(z.ptr[i]).c_str(), (long long)z.n[i] * 4);
    return hipSuccess;
}
}

int main() {
    char call[16];
    long long T, di, do_, r, dt, act, G, scr;
    while (scanf("%15s %lld %lld %lld %lld %lld %lld %lld %lld", call, &T, &di, &do_, &r, &dt, &act, &G, &scr) == 9) {
        noble_linear_desc d{T, di, do_, r, (int32_t)dt, (int32_t)act, (int32_t)G, 0};
        const bool fwd = !strcmp(call, "fwd"), br = r > 0;
        size_t n = (size_t)scr;
        int st = NOBLE_OK;
        if (scr < 0)
            st = fwd ? noble_linear_fwd_scratch_size(&d, &n) : noble_linear_workspace_size(&d, nullptr, &n);
        auto p = [&](int i) { return br ? ptr(i) : nullptr; };
        auto f = [&](int i) { return br ? fptr(i) : nullptr; };
        if (st != NOBLE_OK) {
        } else if (fwd) {
            st = noble_linear_fwd(&d, ptr(X), ptr(W), fptr(B), p(WD), f(O1), f(P1), p(M), f(O2), f(P2), p(WU), ptr(Y), p(RES),
                                  p(SCR), n, nullptr);
        } else if (!strcmp(call, "static")) {
            st = noble_linear_fwd_static(&d, ptr(X), ptr(W), fptr(B), p(WD), f(O1), f(P1), p(M), f(O2), f(P2), p(WU), ptr(Y),
                                         p(RES), nullptr);
        } else if (!strcmp(call, "bwd")) {
            st = noble_linear_bwd(&d, ptr(DY), ptr(X), ptr(W), p(WD), f(O1), f(P1), p(M), f(O2), f(P2), p(WU), p(RES), ptr(DX),
                                  fptr(DW), fptr(DB), f(DWD), f(DM), f(DWU), f(DO1), f(DP1), f(DO2), f(DP2), ptr(SCR), n, nullptr);
        } else {
            st = noble_linear_bwd_storage(&d, ptr(DY), ptr(X), ptr(W), p(WD), f(O1), f(P1), p(M), f(O2), f(P2), p(WU), p(RES),
                                          ptr(DX), ptr(DW), fptr(DB), p(DWD), p(DM), p(DWU), f(DO1), f(DP1), f(DO2), f(DP2),
                                          ptr(SCR), n, nullptr);
        }
        printf("call %d\n", st);
    }
    return 0;
}
