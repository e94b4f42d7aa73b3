// Calls the library's state entry points with the HIP runtime replaced by the functions
// below (the executable's definitions come before the runtime's), so that no device is
// needed and no pointer is followed: every copy and kernel launch is only recorded.  The
// caller's pointer P is said to lie where the first argument tells; printed per call are
// the copies that have P as an operand and the order of copies and launches.
//   usage: caller_memory <library> <own|other|host|managed|unknown> <offset of P in bytes>
#include <dlfcn.h>

#include <cstdint>
#include <cstdio>
#include <cstdlib>
#include <cstring>
#include <string>

#include "../include/mhd950.h"

namespace {
constexpr uintptr_t kCaller = uintptr_t(1) << 44, kWork = uintptr_t(1) << 45;
const char* kind = "own";
uintptr_t P = kCaller;
std::string trace;

struct Attributes {  // hipPointerAttribute_t
    int type, device;
    void *dev, *host;
    int managed;
    unsigned flags;
};
struct Dim3 {
    unsigned x, y, z;
};
}  // namespace

extern "C" {
void** __hipRegisterFatBinary(const void*) { static void* h; return &h; }
void __hipUnregisterFatBinary(void**) {}
void __hipRegisterFunction(void**, const void*, char*, const char*, unsigned, void*, void*, void*, void*, int*) {}
void __hipRegisterVar(void**, void*, char*, char*, int, size_t, int, int) {}
int __hipPushCallConfiguration(Dim3, Dim3, size_t, void*) { return 0; }
int __hipPopCallConfiguration(Dim3* g, Dim3* b, size_t* m, void** s)
{
    *g = *b = Dim3{1, 1, 1};
    *m = 0;
    *s = nullptr;
    return 0;
}
int hipLaunchKernel(const void*, Dim3, Dim3, void**, size_t, void*) { trace += 'k'; return 0; }
int hipGetLastError() { return 0; }
int hipGetDevice(int* d) { *d = 0; return 0; }
int hipStreamGetDevice(void*, int* d) { *d = 0; return 0; }
int hipDeviceGetAttribute(int*, int, int) { return 1; }
int hipStreamSynchronize(void*) { return 0; }
int hipMemsetAsync(void*, int, size_t, void*) { return 0; }
int hipMemcpyAsync(void* dst, const void* src, size_t bytes, int, void*)
{
    if ((uintptr_t)src == P || (uintptr_t)dst == P) {
        trace += (uintptr_t)src == P ? "[in " : "[out ";
        trace += std::to_string(bytes) + "]";
    }
    return 0;
}
int hipPointerGetAttributes(Attributes* a, const void* p)
{
    std::memset(a, 0, sizeof *a);
    if ((uintptr_t)p < kCaller || (uintptr_t)p >= kWork) {
        a->type = 2;
        return 0;
    }
    if (!std::strcmp(kind, "unknown")) return 1;
    const bool device = !std::strcmp(kind, "own") || !std::strcmp(kind, "other");
    a->type = device ? 2 : std::strcmp(kind, "host") ? 3 : 1;
    a->device = !std::strcmp(kind, "other") ? 1 : 0;
    a->managed = !std::strcmp(kind, "managed");
    return 0;
}
}

namespace {
void* lib;
void* fn(const char* name)
{
    void* f = dlsym(lib, name);
    if (!f) {
        std::fprintf(stderr, "no symbol %s\n", name);
        std::exit(2);
    }
    return f;
}
#define CALL(name) ((decltype(&name))fn(#name))

void check(mhd_status st, const char* what)
{
    if (st != MHD_OK) {
        std::fprintf(stderr, "%s: status %d\n", what, (int)st);
        std::exit(2);
    }
}
void say(const std::string& name, mhd_status st)
{
    check(st, name.c_str());
    std::printf("%s %s\n", name.c_str(), trace.c_str());
    trace.clear();
}
}  // namespace

int main(int argc, char** argv)
{
    if (argc != 4) return 2;
    kind = argv[2];
    P = kCaller + (uintptr_t)std::atoi(argv[3]);
    lib = dlopen(argv[1], RTLD_NOW | RTLD_LOCAL);
    if (!lib) {
        std::fprintf(stderr, "%s\n", dlerror());
        return 2;
    }
    void* work = (void*)kWork;
    const size_t big = size_t(1) << 40;
    double* caller = (double*)P;
    const mhd_grid g = {16, 4, 4, {1.0, 1.0, 1.0}};
    for (int fp32 = 0; fp32 < 2; ++fp32) {
        const std::string prec = fp32 ? "fp32 " : "fp64 ";
        mhd_physics mhd = {};
        mhd.eos = MHD_EOS_ADIABATIC_MHD;
        mhd.gamma = 5.0 / 3.0;
        mhd_physics dust = {};
        dust.eos = MHD_EOS_ISOTHERMAL_HYDRO;
        dust.cs_iso = 1.0;
        dust.ndust = 1;
        dust.t_stop[0] = 1.0;
        const mhd_scheme sm = {MHD_RECON_PLM, MHD_RS_HLLE, MHD_INT_RK2, 0.3, fp32, 1e-12};
        const mhd_scheme sd = {MHD_RECON_PLM, MHD_RS_HLLE, MHD_INT_IMEX2P, 0.3, fp32, 1e-12};
        for (int d = 0; d < 2; ++d) {
            mhd_ctx* c = nullptr;
            check(CALL(mhd_create)(&g, d ? &dust : &mhd, d ? &sd : &sm, work, big, nullptr, &c), "create");
            const std::string who = prec + (d ? "dust " : "mhd ");
            trace.clear();
            say(who + "set", CALL(mhd_set_state)(c, caller, 1));
            say(who + "get", CALL(mhd_get_state)(c, caller, 1));
            CALL(mhd_destroy)(c);
        }
        for (int nb = 1; nb <= 2; ++nb) {
            const mhd_grid both[2] = {g, g};
            const std::string who = prec + (nb == 1 ? "block " : "batch ");
            mhd_batch* b = nullptr;
            check(CALL(mhd_batch_create)(nb, both, &mhd, &sm, work, big, nullptr, &b), "batch");
            trace.clear();
            say(who + "set", CALL(mhd_batch_set_state)(b, caller, 1));
            say(who + "get", CALL(mhd_batch_get_state)(b, caller, 1));
            CALL(mhd_batch_destroy)(b);
        }
        if (!fp32) {
            mhd_cnn* n = nullptr;
            check(CALL(mhd_cnn_create)(&g, &mhd, work, big, nullptr, &n), "network");
            trace.clear();
            const double* own = (const double*)(kWork + (uintptr_t(1) << 41));
            say(prec + "closure coarse", CALL(mhd_cnn_accumulate)(n, own, caller, own, 0.1, nullptr));
            CALL(mhd_cnn_destroy)(n);
        }
    }
    return 0;
}
