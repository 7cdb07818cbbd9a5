// Which kernel a convolution call launches, without a GPU: librtoss.so linked against stand-ins for the few runtime calls it
// makes, on a device of 256 compute units.  Reads calls, one a line,
//     coherent Co Ci ksize k rule dt  N H W stride out_dt  fused
// (fused: 1 a whole output stage into a channel slice, more the same at that pitch, less than 0 a pitch and nothing else; dt + 16: packs
// the layer instead, with every allocation refused)
// and prints the status, the launched kernel's handle (its offset in the library), the dynamic LDS it was launched with and the
// limit that was set for it.
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <cstdlib>
#include <map>
#include <new>

#include "rtoss.h"

static const void* g_kernel;
static size_t g_lds;
static std::map<const void*, int> g_limit;

// the library's allocations come here too
static bool g_refuse;
void* operator new(size_t n)
{
    void* p = g_refuse ? nullptr : std::malloc(n);
    if (!p) throw std::bad_alloc();
    return p;
}
void operator delete(void* p) noexcept { std::free(p); }
void operator delete(void* p, size_t) noexcept { std::free(p); }

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipFuncSetAttribute(const void* kernel, hipFuncAttribute, int bytes) { return g_limit[kernel] = bytes, hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, hipSuccess; }
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t lds, hipStream_t) { return g_kernel = kernel, g_lds = lds, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
static size_t g_call_lds;
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t lds, hipStream_t) { return g_call_lds = lds, hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t* lds, hipStream_t*) { return *lds = g_call_lds, hipSuccess; }
}

int main()
{
    rtoss_wdesc d;
    rtoss_cdesc c{};
    int coherent, rule, dt, out_dt, fused;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d", &coherent, &d.Co, &d.Ci, &d.ksize, &d.k, &rule, &dt, &c.N, &c.H, &c.W, &c.stride,
                 &out_dt, &fused) == 13) {
        d.dt = (rtoss_dtype)(dt & 15);
        c.out_dt = (rtoss_dtype)out_dt;
        c.pad = d.ksize / 2;
        c.layout = RTOSS_NHWC;
        uint16_t masks[256];
        int P = 0;
        if (rtoss_pattern_dict(d.k, (rtoss_rule)rule, masks, 256, &P)) return 1;
        char* const base = (char*)((size_t)1 << 44);  // addresses that nothing reads
        char *const x = base + ((size_t)1 << 42), *const y = base + ((size_t)2 << 42);
        rtoss_epilogue e{};
        e.scale_dev = e.bias_dev = (const float*)base;
        e.residual_dev = y + ((size_t)1 << 42);
        e.act = RTOSS_ACT_SILU;
        e.y_ld = e.residual_ld = fused > 1 ? fused : (d.Co + 7) / 8 * 8 + 16;
        if (fused < 0) {
            e = rtoss_epilogue{};
            e.y_ld = -fused;
        }
        g_kernel = nullptr;
        g_lds = 0;
        g_refuse = dt & 16;
        const rtoss_status st = dt & 16    ? rtoss_pack(&d, x, (const uint8_t*)x, masks, P, base, (size_t)1 << 40, nullptr, 0, nullptr)
                                : coherent ? rtoss_conv2d_pattern_coherent(&d, &c, fused ? &e : nullptr, masks, P, base, x, y, nullptr)
                                : fused    ? rtoss_conv2d_pattern_fused(&d, &c, &e, masks, P, base, x, y, nullptr)
                                           : rtoss_conv2d_pattern(&d, &c, masks, P, base, x, y, nullptr);
        g_refuse = false;
        Dl_info info{};
        size_t at = 0;
        if (g_kernel && dladdr(g_kernel, &info)) at = (size_t)((const char*)g_kernel - (const char*)info.dli_fbase);
        const auto limit = g_limit.find(g_kernel);
        printf("%d %zx %zu %d\n", (int)st, at, g_lds, limit == g_limit.end() ? 64 * 1024 : limit->second);  // (64 KB: the runtime's default)
    }
    return 0;
}
