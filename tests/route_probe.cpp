// Which kernel a convolution call launches, without a GPU: librtoss.so linked against stand-ins for the few runtime calls it
// makes, on a device of 256 compute units.  Reads calls, one a line,
//     coherent Co Ci ksize k rule dt  N H W stride out_dt  fused
// and prints the status and the launched kernel's handle (its offset in the library).
#include <dlfcn.h>
#include <hip/hip_runtime_api.h>

#include <cstdio>
#include <vector>

#include "rtoss.h"

static const void* g_kernel;

extern "C" {
hipError_t hipGetDevice(int* d) { return *d = 0, hipSuccess; }
hipError_t hipDeviceGetAttribute(int* v, hipDeviceAttribute_t, int) { return *v = 256, hipSuccess; }
hipError_t hipFuncSetAttribute(const void*, hipFuncAttribute, int) { return hipSuccess; }
hipError_t hipOccupancyMaxActiveBlocksPerMultiprocessor(int* n, const void*, int, size_t) { return *n = 2, hipSuccess; }
hipError_t hipLaunchKernel(const void* kernel, dim3, dim3, void**, size_t, hipStream_t) { return g_kernel = kernel, hipSuccess; }
hipError_t hipGetLastError(void) { return hipSuccess; }
hipError_t __hipPushCallConfiguration(dim3, dim3, size_t, hipStream_t) { return hipSuccess; }
hipError_t __hipPopCallConfiguration(dim3*, dim3*, size_t*, hipStream_t*) { return hipSuccess; }
}

int main()
{
    rtoss_wdesc d;
    rtoss_cdesc c{};
    int coherent, rule, dt, out_dt, fused;
    while (scanf("%d %d %d %d %d %d %d %d %d %d %d %d %d", &coherent, &d.Co, &d.Ci, &d.ksize, &d.k, &rule, &dt, &c.N, &c.H, &c.W, &c.stride,
                 &out_dt, &fused) == 13) {
        d.dt = (rtoss_dtype)dt;
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
        e.y_ld = e.residual_ld = (d.Co + 7) / 8 * 8 + 16;  // a channel slice
        g_kernel = nullptr;
        const rtoss_status st = coherent ? rtoss_conv2d_pattern_coherent(&d, &c, fused ? &e : nullptr, masks, P, base, x, y, nullptr)
                                : fused  ? rtoss_conv2d_pattern_fused(&d, &c, &e, masks, P, base, x, y, nullptr)
                                         : rtoss_conv2d_pattern(&d, &c, masks, P, base, x, y, nullptr);
        Dl_info info{};
        size_t at = 0;
        if (g_kernel && dladdr(g_kernel, &info)) at = (size_t)((const char*)g_kernel - (const char*)info.dli_fbase);
        printf("%d %zx\n", (int)st, at);
    }
    return 0;
}
