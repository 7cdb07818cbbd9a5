// Internal declarations shared by the host API and the kernel launchers.
#pragma once

#include <hip/hip_runtime.h>
#include <stddef.h>
#include <stdint.h>

#include <atomic>

#include "rtoss.h"

namespace rtoss {

struct ConvParams;  // rtoss_cdesc + the fused output stage (epilogue.h)

constexpr int kMaxPatterns = 255;

// A dictionary travels to every kernel by value in the launch arguments, so the host
// array can be released as soon as the call returns and no device copy is needed.
struct Dict {
    uint16_t mask[256];
    int P;
    int k;
    int layout;  // tap layout of the 2-of-4 fragments (sparse_frag.h) that fits every pattern, cheapest first; -1: none
    bool repeats;  // ... for some of them with the layout's repeated taps only
};

// Decoded dictionary for the convolution kernels: tap[p][j] = j-th live tap of pattern p
// in ascending order (unused entries 0).
struct TapTable {
    uint8_t tap[256][9];
};

// Most workgroups in the first dimension of a grid, rounded down to a multiple of the 8 XCDs: the runtime refuses launches
// with 2^32 or more work items in a dimension, and no kernel with this limit has more than 256 lanes.
constexpr int64_t kMaxGridGroups = 0xffffffff / 256 / 8 * 8;
// Most 16-byte chunks of an input whose copy sources are 32-bit chunk offsets.
constexpr int64_t kMaxChunks = 0x7fffffff;

inline int elem_bytes(rtoss_dtype dt) { return dt == RTOSS_F32 ? 4 : 2; }
inline size_t align_up(size_t v, size_t a) { return (v + a - 1) / a * a; }

// ----- packed blob geometry (host side; the kernels receive section pointers) -----
enum MatrixFormat {
    kFormatNone = 0,     // only the live list (section 0): direct kernels
    kFormatDense = 1,    // 1x1, rows of any multiple of 4 bytes: zero-filled matrix-core fragments
    kFormatSparse24 = 2, // 3x3: 2-of-4 compressed fragments + indices
    kFormatStem = 3,     // 3x3 with <= 3 input channels: one zero-filled fragment per 16 output channels
    kFormatDenseStream = 4,  // 1x1 with Ci = 32 * 2^n <= 1024 (fp32: 16 * 2^n <= 512): zero-filled fragments in the streaming kernel's order
    kFormatDense3x3 = 5,     // 3x3 whose dictionary has no 2-of-4 shape: zero-filled fragments, one per tap
    kFormatGather3x3 = 6     // 3x3, on request (rtoss_pack_coherent): per-block tap lists on the dense instruction
};

struct BlobGeometry {
    int64_t G;          // number of groups of 9
    int64_t n_elems;    // Co*Ci*ksize*ksize
    size_t live_off;    // [G][k] values
    size_t idx_off;     // [G] bytes
    MatrixFormat format;
    size_t mat_off;     // matrix-core section (0 if none)
    size_t mat_bytes;
    size_t dense_off;   // the same weights in the dense mode's format beside kFormatSparse24 (0: not); with kFormatDense3x3: that section alone
    size_t total;
};

// Filled by host code in api.cpp.
rtoss_status blob_geometry(const rtoss_wdesc* d, const Dict& dict, BlobGeometry* out, bool coherent = false);

// ----- error plumbing -----
rtoss_status fail(rtoss_status st, const char* fmt, ...);
rtoss_status check_hip(hipError_t e, const char* what);

// ----- per-device launch state (api.hip) -----
// The current device's ordinal and its number of compute units (queried once per device).
struct DeviceInfo {
    int device;
    int cus;
};
rtoss_status current_device(DeviceInfo* out);
// Raises a kernel's dynamic-LDS limit to `bytes` on device `dev` (the current one), once per (kernel instantiation,
// device): `done` is the instantiation's own word, bit d = done on device d.  Safe to call from several
// threads (the attribute call is idempotent; the word only saves repeating it).
struct LaunchOnce {
    std::atomic<uint64_t> done{0};
};
rtoss_status ensure_dynamic_lds(const void* kernel, size_t bytes, LaunchOnce& once, int dev, const char* what);

// ----- launchers (one per kernel family; defined next to the kernels) -----
rtoss_status launch_select(const void* w, rtoss_dtype dt, int64_t G, const Dict& dict, uint8_t* idx, hipStream_t s);

constexpr int kSelectBatchMax = 64;  // tensors per batched selection launch
rtoss_status launch_select_batch(const rtoss_select_item* items, int n, rtoss_dtype dt, const Dict& dict, hipStream_t s);

// counts of each pattern index (select.hip; counts.h: zeroing them)
rtoss_status launch_histogram(const uint8_t* idx, int64_t G, int P, uint32_t* hist, hipStream_t s);

rtoss_status launch_conv_direct(const rtoss_wdesc& d, const ConvParams& c, const Dict& dict, const void* live_values,
                                const uint8_t* live_idx, const void* x, void* y, hipStream_t s);

// Prune and pack layers of one dictionary, as few launches as possible (pack.hip).
struct PackItem {
    rtoss_wdesc d;
    const void* w;
    const uint8_t* idx;
    void* section;      // private section of the blob
    void* live;         // public section: values (the blob's start)
    uint8_t* live_idx;  // public section: indices
};
rtoss_status launch_pack(const PackItem* items, const BlobGeometry* geo, int n, const Dict& dict, hipStream_t s);

// The matrix-core kernels took over shapes that the element-wise kernel serves at any size.  *_launch_ok: the launch is
// within the kernel's limits, or of a shape that the kernel alone serves (which then reports the error).

// 3x3 convolution on the sparse matrix instruction (conv3x3_sparse.hip)
bool sparse3x3_launch_ok(const rtoss_wdesc& d, const Dict& dict, const ConvParams& c);
bool sparse3x3_shape_ok(const rtoss_wdesc& d, const Dict& dict);
bool sparse3x3_is_faster(const rtoss_wdesc& d, const Dict& dict, const ConvParams& c);  // (of a layer with both sections)
size_t sparse3x3_section_bytes(const rtoss_wdesc& d, int layout);
rtoss_status launch_conv3x3_sparse(const rtoss_wdesc& d, const ConvParams& c, int layout, const void* section, const void* x,
                                   void* y, hipStream_t s);

// ... large stride-1 layers: pipelined kernel over strips of output rows (conv3x3_rows.hip); same packed section
// planned: its cut where the caller has it (rows_plan.h), or nullptr
struct RowsLaunch;
rtoss_status launch_conv3x3_rows(const rtoss_wdesc& d, const ConvParams& c, int layout, const RowsLaunch* planned, const void* section,
                                 const void* x, void* y, hipStream_t s);
rtoss_status launch_conv3x3_rows_groups(const rtoss_wdesc& d, const ConvParams& c, const RowsLaunch* planned, const void* section, const void* x,
                                        void* y, hipStream_t s);  // (its part for layout 1)
bool rows3x3_needs_fused_stage(const ConvParams& c);

// ... launches too small to fill the chip: input channels split over the waves of a workgroup (conv3x3_ksplit.hip).  Reads
// the packed sections of the sparse kernels (layout 0 or 1) and of the dense-mode kernel (layout 2).
// ksplit3x3_plan: variant to launch, 0 = another kernel serves the launch better.
int ksplit3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout);
rtoss_status launch_conv3x3_ksplit(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                   const void* x, void* y, hipStream_t s);
// the same for the section of conv3x3_gather.hip (layout 3)
rtoss_status launch_conv3x3_ksplit_gather(const rtoss_wdesc& d, const ConvParams& c, int plan, const void* headers, const void* frags,
                                          const void* zeros, const void* x, void* y, hipStream_t s);

// ... stride 1, launches of medium size: strips of output rows (conv3x3_strip.hip); same sections and layouts.
// strip3x3_plan: variant to launch, 0 = another kernel serves the launch better.
int strip3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout);
int strip3x3_rows(int plan);  // output rows of a workgroup
rtoss_status launch_conv3x3_strip(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                  const void* x, void* y, hipStream_t s);

// ... with helper waves (conv3x3_ring.hip): rows of a wave, 0 = another kernel serves the launch better
int ring3x3_plan(const rtoss_wdesc& d, const ConvParams& c, int layout);
rtoss_status launch_conv3x3_ring(const rtoss_wdesc& d, const ConvParams& c, int layout, int plan, const void* section, const void* zeros,
                                 const void* x, void* y, hipStream_t s);

// 3x3 convolution with live taps gathered onto the dense matrix instruction, for block-shared patterns
// (conv3x3_gather.hip); its own blob format, chosen by the caller (rtoss_pack_coherent)
bool gather3x3_shape_ok(const rtoss_wdesc& d);
size_t gather3x3_header_bytes(const rtoss_wdesc& d);
size_t gather3x3_section_bytes(const rtoss_wdesc& d);
rtoss_status launch_pack_gather3x3(const rtoss_wdesc& d, const void* w, const uint8_t* idx, const Dict& dict, void* section,
                                   void* live_values, uint8_t* live_idx, hipStream_t s);
rtoss_status launch_conv3x3_gather(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                   hipStream_t s);

// 3x3 convolution in dense mode on the matrix cores (conv3x3_dense.hip)
bool dense3x3_launch_ok(const rtoss_wdesc& d, const ConvParams& c);
bool dense3x3_shape_ok(const rtoss_wdesc& d);
size_t dense3x3_section_bytes(const rtoss_wdesc& d);
rtoss_status launch_conv3x3_dense(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                  hipStream_t s);

// 1x1 convolution on the dense matrix instruction (conv1x1_mma.hip)
bool dense1x1_launch_ok(const rtoss_wdesc& d, const ConvParams& c);
bool dense1x1_shape_ok(const rtoss_wdesc& d);
size_t dense1x1_section_bytes(const rtoss_wdesc& d);
rtoss_status launch_conv1x1_mma(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                hipStream_t s);

// 1x1 convolution, streaming kernel with register-resident weights (conv1x1_stream.hip)
bool stream1x1_launch_ok(const rtoss_wdesc& d, const ConvParams& c);
bool stream1x1_shape_ok(const rtoss_wdesc& d);
size_t stream1x1_section_bytes(const rtoss_wdesc& d);
rtoss_status launch_conv1x1_stream(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                   hipStream_t s);

// ... launches too small for it: input channels split over the waves of a workgroup (conv1x1_ksplit.hip); same packed section.
// ksplit1x1_plan: variant to launch, 0 = the streaming kernel serves the launch better.
int ksplit1x1_plan(const rtoss_wdesc& d, const ConvParams& c);
rtoss_status launch_conv1x1_ksplit(const rtoss_wdesc& d, const ConvParams& c, int plan, const void* section, const void* x, void* y,
                                   hipStream_t s);

// 3x3 convolution with <= 3 input channels (conv3x3_stem.hip)
bool stem3x3_shape_ok(const rtoss_wdesc& d);
bool stem3x3_launch_ok(const rtoss_wdesc& d, const ConvParams& c);
size_t stem3x3_section_bytes(const rtoss_wdesc& d);
rtoss_status launch_conv3x3_stem(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                 hipStream_t s);

}  // namespace rtoss
