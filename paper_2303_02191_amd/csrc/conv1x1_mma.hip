// 1x1 pattern-pruned convolution on the CDNA4 matrix cores (fp16 / bf16 / fp32, fp32 accumulate):
// the general kernels, for any channel counts whose input rows are a multiple of 4 bytes: a ring of LDS buffers for large
// launches of whole stages and channel tiles, and whole output rows for everything else (second half of this comment).
// (64-byte multiples of 2^n stages with whole channel tiles take conv1x1_stream.hip and conv1x1_ksplit.hip instead.)
//
// Section IV.D prunes a 1x1 layer by cutting the flattened [Co][Ci] weight matrix into groups
// of 9 and keeping k weights per group, so the pruned layer is a GEMM
//     Y[p][co] = sum_ci W'[co][ci] * X[p][ci]          (p runs over all N*H*W positions)
// whose weight matrix has k-of-9 sparsity along its flattened axis.  That sparsity has no
// structure a matrix instruction could skip (groups straddle rows and have no 2-of-4 shape),
// and the layer is bound by HBM traffic anyway: activations in, activations out, every byte
// once.  So the weights are expanded to zero-filled dense fragments (they are tiny and stay in
// L2), and the ring is built to stream activations: channels-last rows are contiguous, a
// workgroup owns 128 consecutive positions x up to 128 output channels, and K runs over stages
// of 64 bytes of input channels through a 5-deep ring of LDS buffers filled by global -> LDS copies
// four stages ahead (an HBM-bound kernel lives on bytes in flight: two resident workgroups per CU x
// four stages x 8 KB of activations).  Activation rows sit in LDS at a 64-byte pitch with their
// four 16-byte chunks XOR-swizzled by (position / 2) % 4, which makes the 16-byte operand reads
// of 8 neighbouring positions hit 8 different bank groups without any padding.
//
// Ragged channel counts, and small launches of the others, take a kernel of their own (the second one here): with a
// handful of stages the ring never fills, and rows of 255 channels have no alignment to store by.  There operands go
// straight from memory into registers and the output tile is laid out in LDS as it lies in memory -- rows without gaps,
// all channels of the positions -- so that it leaves in whole 16-byte pieces whatever the channel count.  72 -> 255
// channels on 28 028 positions in fp16: 13.9 us with the ring and 4-byte stores, now 8.6 (the write alone takes 3); on 600
// positions 10.7 and 4.1.  What bounds it: one round of workgroups, so loads, products and stores follow each other.
//
// Operand layout of v_mfma_f32_16x16x32 (wave64; r = lane % 16, q = lane / 16): A lane holds
// row r, K = 8q..8q+7; B lane holds column r, K = 8q..8q+7; D lane holds column r, rows 4q..4q+3.
// fp32 in the ring: four v_mfma_f32_16x16x4_f32 per step, instruction s on element s of every lane's 16 bytes.
#include <algorithm>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "fp32_split.h"
#include "mma.h"
#include "work_order.h"
#include "pack_plan.h"

namespace rtoss {

namespace {

constexpr int kFrag = 1024;      // one A fragment: 64 lanes x 16 bytes = 16 output channels x 64 bytes of input channels
constexpr int kTilePos = 128;    // positions per workgroup
constexpr int kRing = 5;

inline size_t frag_bytes(const rtoss_wdesc& d) { return (size_t)stage_count(d) * ring_padded_tiles(d.Co) * kFrag; }

template <typename T, typename TO, int TM>
__global__ __launch_bounds__(256) void conv1x1_mma_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                          const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                          int64_t P, int Ci, int Co, int m_tiles_total, Divisor co_blocks,
                                                          int total_work, int work_per_xcd, Epilogue ep)
{
    constexpr int TN = 2;                                // 16-position blocks per wave
    constexpr int A_PER_WAVE = (TM + 3) / 4;             // copy instructions per wave and stage (64 lanes x 16 B each)
    constexpr int A_AREA = A_PER_WAVE * 4 * 1024;
    constexpr int X_PER_WAVE = 2;                        // 128 positions x 64 bytes
    constexpr int X_AREA = 4 * X_PER_WAVE * 1024;
    constexpr int STAGE = A_AREA + X_AREA;
    constexpr int CPW = A_PER_WAVE + X_PER_WAVE;         // copies one wave has in flight per stage
    extern __shared__ __attribute__((aligned(16))) char smem[];  // kRing stages

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD-contiguous work order (channel blocks of one position tile, and neighbouring tiles, share an L2)
    const int work = (blockIdx.x % 8) * work_per_xcd + blockIdx.x / 8;
    if (work >= total_work) return;
    const int all_tile = co_blocks.quotient(work), cblk = co_blocks.remainder(work, all_tile);
    const int64_t p0 = (int64_t)all_tile * kTilePos;
    const int mt0 = cblk * TM;
    const int row_bytes = Ci * (int)sizeof(T);
    const int stages = row_bytes / 64;

    // ---- copy sources: every lane copies 16 bytes in every copy instruction (no branches); lanes
    // whose slot is padding read the packer's block of zeros ----
    const char* x_ptr[X_PER_WAVE];
#pragma unroll
    for (int k = 0; k < X_PER_WAVE; ++k) {
        const int c = (k * 4 + wave) * 64 + lane;                // LDS chunk this lane fills
        const int pos = c >> 2, q = (c & 3) ^ ((pos >> 1) & 3);  // ... holds channel chunk q of position pos
        const bool real = p0 + pos < P;
        x_ptr[k] = real ? (const char*)x + (p0 + pos) * row_bytes + q * 16 : zeros;
    }
    const char* a_ptr[A_PER_WAVE];
#pragma unroll
    for (int k = 0; k < A_PER_WAVE; ++k) {
        const int kk = k * 4 + wave;
        a_ptr[k] = kk < TM ? wfrag + (int64_t)(mt0 + kk) * kFrag + lane * 16 : zeros;
    }
    const int64_t a_stage_stride = (int64_t)m_tiles_total * kFrag;
    auto issue_stage = [&](int stage, int buf) {
        char* base = smem + buf * STAGE;
#pragma unroll
        for (int k = 0; k < A_PER_WAVE; ++k) {
            const int kk = k * 4 + wave;
            // (the zero block is shorter than a stage stride; padding lanes re-read its start every stage)
            copy16_to_lds(kk < TM ? a_ptr[k] + stage * a_stage_stride : a_ptr[k], base + kk * 1024);
        }
#pragma unroll
        for (int k = 0; k < X_PER_WAVE; ++k) copy16_to_lds(x_ptr[k] + stage * 64, base + A_AREA + (k * 4 + wave) * 1024);
    };

    const int nn = lane & 15, qq = lane >> 4;
    f32x4 acc[TM][TN];
#pragma unroll
    for (int m = 0; m < TM; ++m)
#pragma unroll
        for (int j = 0; j < TN; ++j) acc[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};

    // kRing-1 stages are always in flight or being multiplied.  Past the end the last stage is
    // fetched again into a free buffer, so that every wave has issued exactly CPW copies per
    // stage and the wait below can count them.
    constexpr int AHEAD = kRing - 2;  // stages still in flight when a stage must have landed
    static_assert(AHEAD * CPW < 64, "outstanding copies must fit the counter");
#pragma unroll
    for (int s = 0; s < kRing - 1; ++s) issue_stage(min(s, stages - 1), s);
    int buf = 0;
    for (int s = 0; s < stages; ++s) {
        // all but the AHEAD newest stages' copies of this wave have landed ...
        // (a bare barrier: __syncthreads() would add a fence that waits for ALL outstanding copies)
        asm volatile("" ::: "memory");
        __builtin_amdgcn_s_waitcnt(0x0070 | ((AHEAD * CPW) & 15) | (((AHEAD * CPW) >> 4) << 14));  // + lgkmcnt(0)
        __builtin_amdgcn_s_barrier();  // ... and everybody's; everybody is done with the buffer refilled next
        asm volatile("" ::: "memory");
        issue_stage(min(s + kRing - 1, stages - 1), buf == 0 ? kRing - 1 : buf - 1);
        const char* A = smem + buf * STAGE + lane * 16;
        // position block j of this wave starts at wave*32 + 16 j; the swizzle depends on n only
        const char* X = smem + buf * STAGE + A_AREA + (wave * TN * 16 + nn) * 64 + ((qq ^ ((nn >> 1) & 3)) * 16);
        u32x4 b[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) b[j] = *(const u32x4*)(X + j * 16 * 64);
#pragma unroll
        for (int m = 0; m < TM; ++m) {
            const u32x4 a = *(const u32x4*)(A + m * kFrag);
#pragma unroll
            for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(a, b[j], acc[m][j]);
        }
        buf = buf + 1 == kRing ? 0 : buf + 1;
    }
    __builtin_amdgcn_s_waitcnt(0x0f70);  // the surplus copies have landed: LDS may be reused
    __syncthreads();

    // ---- epilogue: transpose through LDS so that whole channel rows are written, 16 bytes per lane ----
    {
        constexpr int EB = (int)sizeof(TO);
        constexpr int HALVES = (EB == 4 && TM >= 2) ? 2 : 1;
        constexpr int TMH = TM / HALVES;
        constexpr int ROW = TMH * 16 * EB + (EB == 2 ? 8 : 16);
        static_assert(4 * 16 * TN * ROW <= kRing * STAGE, "epilogue staging must fit in the ring");
        char* stage_out = smem + wave * (16 * TN * ROW);
#pragma unroll
        for (int h = 0; h < HALVES; ++h) {
#pragma unroll
            for (int j = 0; j < TN; ++j)
#pragma unroll
                for (int mm = 0; mm < TMH; ++mm) {
                    f32x4 v = acc[h * TMH + mm][j];
                    {  // output stage on this lane's 4 consecutive channels of position p_f
                        const int co4 = 16 * (mt0 + h * TMH + mm) + 4 * qq;
                        const int64_t p_f = p0 + wave * (TN * 16) + j * 16 + nn;
                        if (p_f < P && co4 < Co) {
                            float vv[4] = {v.x, v.y, v.z, v.w};
                            epi_scale_bias_act<4>(vv, ep, co4);
                            epi_residual<TO, 4>(vv, ep, p_f, co4);
                            v = f32x4{vv[0], vv[1], vv[2], vv[3]};
                        }
                    }
                    char* dst = stage_out + (j * 16 + nn) * ROW + (16 * mm + 4 * qq) * EB;
                    if constexpr (EB == 4) {
                        *(f32x4*)dst = v;
                    } else {
                        uint2 o;
                        o.x = pack2_from_f32<TO>(v.x, v.y);
                        o.y = pack2_from_f32<TO>(v.z, v.w);
                        *(uint2*)dst = o;
                    }
                }
            constexpr int CH = TMH * 16 * EB / 16;  // 16-byte chunks per row
            static_assert(64 % CH == 0, "row chunks must tile the wave");
            constexpr int POS_PER_PASS = 64 / CH;
            constexpr int PASSES = (16 * TN) / POS_PER_PASS;
            const int co_first = 16 * (mt0 + h * TMH);
#pragma unroll
            for (int ps = 0; ps < PASSES; ++ps) {
                const int pl = ps * POS_PER_PASS + lane / CH;  // position within the wave's 32
                const int chunk = lane % CH;
                const int64_t p = p0 + wave * (TN * 16) + pl;
                const int co = co_first + chunk * (16 / EB);
                const u32x4 v = *(const u32x4*)(stage_out + pl * ROW + chunk * 16);
                if (p < P && co < Co) *(u32x4*)(y + p * ep.ldy + co) = v;
            }
        }
    }
}

// The kernel without a ring.  A workgroup owns 16*TN positions and all output channels (blocks of `span` where a row is too long
// for LDS), 64*TM at a time, wave v tiles v*TM ...; the next step's operands are loaded while the current one's are multiplied.
// ROW16: input rows are multiples of 16 bytes, else of 4.  fp32 goes through the bf16 instruction (fp32_split.h): 80 -> 120 channels
// on 48 000 positions 23.0 us on the fp32 instruction, now 18.5.
// Column n of position block j is position TN*n + j of the tile: neighbouring lanes write rows TN apart, whose LDS addresses spread
// over the banks (512-byte rows, as 16 neighbouring positions, would all meet in one).
template <typename T, typename TO, int TM, int TN, bool ROW16, int STEPS>
__device__ __forceinline__ void whole_rows(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                           int64_t P, int Ci, int Co, int m_tiles_total, int work_total, int work_per_xcd, int pitch, int span,
                                           int blocks, uint32_t per_chunks, uint32_t per_last_chunks, const Epilogue& ep)
{
    constexpr int EB = (int)sizeof(TO), PT = 16 * TN;
    extern __shared__ __attribute__((aligned(16))) char smem[];  // [position][channel] of the tile, rows `pitch` bytes apart
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int nn = lane & 15, qq = lane >> 4;
    const int row_bytes = Ci * (int)sizeof(T), stages = (row_bytes + 63) / 64;
    const int64_t a_stage = (int64_t)m_tiles_total * kFrag;
    float* const lds_ep = (float*)(smem + PT * pitch + 16);
    // XCD-contiguous order, channel block fastest; more work than workgroups only past the grid's limit
    for (int t = blockIdx.x / 8; t < work_per_xcd; t += gridDim.x / 8) {
        const int work = (blockIdx.x % 8) * work_per_xcd + t;
        if (work >= work_total) return;
        const int64_t p0 = (int64_t)(work / blocks) * PT;
        const int first = (int)(work % blocks) * span, end = min(first + span, Co);  // this workgroup's channels
        const char* src[TN];
#pragma unroll
        for (int j = 0; j < TN; ++j) src[j] = (const char*)x + std::min<int64_t>(p0 + TN * nn + j, P - 1) * row_bytes;  // (past the end: not stored)
        if (t != (int)(blockIdx.x / 8)) __syncthreads();  // everybody is done reading the tile before
        for (int c0 = first + (end - first - 1) / (64 * TM) * (64 * TM); c0 >= first; c0 -= 64 * TM) {  // (from the last: see below)
            EpiScaleBias<64 * TM> scale_bias;
            scale_bias.load(ep, c0, Co, tid);
            const char* a_src[TM];
#pragma unroll
            for (int m = 0; m < TM; ++m) a_src[m] = wfrag + (int64_t)min(c0 / 16 + wave * TM + m, m_tiles_total - 1) * kFrag + lane * 16;
            constexpr int ST = sizeof(T) == 4 ? 2 : 1;  // stages of a step: fp32 takes 32 channels at a time too (fp32_split.h)
            struct Operands {
                u32x4 a[TM][ST], b[TN][ST];
            } next;
            auto load_stage = [&](int stage, Operands& o, int h) {
                const bool none = ST == 2 && stage >= stages;  // uniform: the second half of an odd last step
#pragma unroll
                for (int m = 0; m < TM; ++m) o.a[m][h] = *(const u32x4*)(none ? zeros : a_src[m] + stage * a_stage);
                const int at = stage * 64 + qq * 16, left = row_bytes - at;  // (bytes of the row from this lane's 16 on)
                if (ROW16 || (stage + 1) * 64 <= row_bytes) {  // uniform
#pragma unroll
                    for (int j = 0; j < TN; ++j) __builtin_memcpy(&o.b[j][h], ROW16 && left <= 0 ? zeros : src[j] + at, 16);
                } else {
#pragma unroll
                    for (int j = 0; j < TN; ++j)
#pragma unroll
                        for (int w = 0; w < 4; ++w) {
                            uint32_t d;
                            __builtin_memcpy(&d, left > 4 * w ? src[j] + at + 4 * w : zeros, 4);
                            o.b[j][h][w] = d;
                        }
                }
            };
            auto load = [&](int step, Operands& o) {
#pragma unroll
                for (int h = 0; h < ST; ++h) load_stage(step * ST + h, o, h);
                __builtin_amdgcn_sched_barrier(0);  // (the scheduler would move the loads down to where they are used)
            };
            f32x4 acc[TM][TN], small[TM][TN];  // (small: fp32 only)
#pragma unroll
            for (int m = 0; m < TM; ++m)
#pragma unroll
                for (int j = 0; j < TN; ++j) acc[m][j] = small[m][j] = f32x4{0.f, 0.f, 0.f, 0.f};
            auto multiply = [&](const Operands& o) {
                if constexpr (ST == 2) {
                    Split8 b[TN];
#pragma unroll
                    for (int j = 0; j < TN; ++j) b[j] = split8(o.b[j][0], o.b[j][1]);
#pragma unroll
                    for (int m = 0; m < TM; ++m) {
                        const Split8 a = split8(o.a[m][0], o.a[m][1]);
                        split_steps<STEPS>([&](auto step) {
#pragma unroll
                            for (int j = 0; j < TN; ++j) split_step<decltype(step)::value>(a, b[j], acc[m][j], small[m][j]);
                        });
                    }
                } else {
#pragma unroll
                    for (int m = 0; m < TM; ++m)
#pragma unroll
                        for (int j = 0; j < TN; ++j) acc[m][j] = Dense16<T>::mma(o.a[m][0], o.b[j][0], acc[m][j]);
                }
            };
            load(0, next);
            for (int step = 1; step * ST < stages; ++step) {
                const Operands o = next;
                load(step, next);
                multiply(o);
            }
            multiply(next);
            // output stage: value (m, j, e) is channel co + 16 m + e of position p0 + TN nn + j
            const int co = c0 + 16 * wave * TM + 4 * qq;
            float v[4 * TM * TN];
#pragma unroll
            for (int i = 0; i < TM * TN; ++i) {
                const f32x4 sum = sizeof(T) == 4 ? split_sum(acc[i / TN][i % TN], small[i / TN][i % TN]) : acc[i / TN][i % TN];
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * i + e] = sum[e];
            }
            if (ep.scale || ep.bias) {
                scale_bias.store(lds_ep, ep, tid);
                __syncthreads();
                const float* at = lds_ep + co - c0;
                if (ep.scale)
#pragma unroll
                    for (int i = 0; i < 4 * TM * TN; ++i) v[i] *= at[16 * (i / 4 / TN) + i % 4];
                if (ep.bias)
#pragma unroll
                    for (int i = 0; i < 4 * TM * TN; ++i) v[i] += at[64 * TM + 16 * (i / 4 / TN) + i % 4];
            }
            epi_act<4 * TM * TN>(v, ep.act);
            if (ep.residual)
#pragma unroll
                for (int j = 0; j < TN; ++j) {
                    const TO* r = (const TO*)ep.residual + std::min<int64_t>(p0 + TN * nn + j, P - 1) * ep.ldr;
#pragma unroll
                    for (int i = 0; i < 4 * TM; ++i) v[4 * (i / 4 * TN + j) + i % 4] += to_f32(r[min(co + 16 * (i / 4) + i % 4, Co - 1)]);
                }
            // Into the tile, four channels at a time.  The last four of a ragged row run over into the next row's first ones, so
            // they are written in front of a barrier, and the blocks of channels from the last to the first.
            // (an access that is not aligned to its size stalls LDS for some 45 cycles.  TN is even: the rows of a step j start at
            // multiples of 4 bytes, or all 2 bytes behind one.)
            const bool odd_rows = pitch % 4 != 0;
            auto write = [&](int m) {
                char* at = smem + TN * nn * pitch + (co - first + 16 * m) * EB;
#pragma unroll
                for (int j = 0; j < TN; ++j, at += pitch) {
                    const float* f = v + 4 * (m * TN + j);
                    if constexpr (EB == 4) {
#pragma unroll
                        for (int e = 0; e < 4; ++e) ((float*)at)[e] = f[e];
                    } else if (j % 2 == 0 || !odd_rows) {
                        ((uint32_t*)at)[0] = pack2_from_f32<TO>(f[0], f[1]);
                        ((uint32_t*)at)[1] = pack2_from_f32<TO>(f[2], f[3]);
                    } else {
                        const uint32_t ends = pack2_from_f32<TO>(f[0], f[3]);
                        *(uint16_t*)at = (uint16_t)ends;
                        *(uint32_t*)(at + 2) = pack2_from_f32<TO>(f[1], f[2]);
                        *(uint16_t*)(at + 6) = (uint16_t)(ends >> 16);
                    }
                }
            };
            const int whole = min(max((end - c0) / 16 - wave * TM, 0), TM);  // this wave's tiles without a channel past the last
#pragma unroll
            for (int m = 0; m < TM; ++m)
                if (m >= whole && co + 16 * m < end) write(m);
            __syncthreads();
#pragma unroll
            for (int m = 0; m < TM; ++m)
                if (m < whole) write(m);
        }
        __syncthreads();
        const int live = (int)std::min<int64_t>(PT, P - p0), row = (end - first) * EB;
        // (past the L2's write-back, which would end the launch with writing the tensor a second time: 72 -> 255 on 28 028
        // positions 8.9 -> 6.7 us, 72 -> 240 likewise, on 112 112 positions 24.6 -> 22.3)
        if (pitch == row) {  // the tile is one piece of the output, and starts at a multiple of 16 bytes
            char* out = (char*)(y + p0 * Co);
            const auto base = store_base(out);
            const int bytes = live * row;
            int i = tid * 16;
            for (; i + 3 * 4096 + 16 <= bytes; i += 4 * 4096) {
                u32x4 r[4];
#pragma unroll
                for (int k = 0; k < 4; ++k) r[k] = *(const u32x4*)(smem + i + 4096 * k);
#pragma unroll
                for (int k = 0; k < 4; ++k) store16_through(base, i + 4096 * k, r[k]);
            }
            for (; i + 16 <= bytes; i += 4096) store16_through(base, i, *(const u32x4*)(smem + i));
            const int tail = bytes & ~15;
            if (tid < (bytes - tail) / EB) ((TO*)(out + tail))[tid] = ((const TO*)(smem + tail))[tid];
        } else {
            const int chunks = (row + 15) / 16;
            const uint32_t reciprocal = end == Co ? per_last_chunks : per_chunks;
            // piece(row of the tile, byte of the row, in LDS)
            auto pieces = [&](auto&& piece) {
                for (int i = tid; i < live * chunks; i += 256) {
                    const int r = chunks == 1 ? i : (int)__umulhi((uint32_t)i, reciprocal), at = (i - r * chunks) * 16;  // (i / chunks)
                    piece(r, at, smem + r * pitch + at);
                }
            };
            // (whole sectors; else as the L2 puts them together, and rows may be aligned to an element only)
            const int64_t apart = (int64_t)ep.ldy * EB;
            if (aligned_pieces((uintptr_t)y, row, first * EB, apart, blocks == 1 && ep.ldy == Co ? 16 : kSector) && PT * apart < kNoStore) {
                const auto base = store_base(y + p0 * ep.ldy + first);
                pieces([&](int r, int at, const char* in) { store16_through(base, (uint32_t)r * ep.ldy * EB + at, *(const u32x4*)in); });
            } else {
                pieces([&](int r, int at, const char* in) {
                    char* out = (char*)(y + (p0 + r) * ep.ldy + first) + at;
                    if (at + 16 <= row) __builtin_memcpy(out, in, 16);
                    else
                        for (int e = 0; e < (row - at) / EB; ++e) ((TO*)out)[e] = ((const TO*)in)[e];
                });
            }
        }
    }
}

template <typename T, typename TO, int TM, int TN, bool ROW16>
__global__ __launch_bounds__(256, 2) void conv1x1_mma_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                          const char* __restrict__ zeros, int64_t P, int Ci, int Co, int m_tiles_total,
                                                          int work_total, int work_per_xcd, int pitch, int span, int blocks,
                                                          uint32_t per_chunks, uint32_t per_last_chunks, Epilogue ep)
{
    whole_rows<T, TO, TM, TN, ROW16, kSplitSix>(x, y, wfrag, zeros, P, Ci, Co, m_tiles_total, work_total, work_per_xcd, pitch, span, blocks,
                                                per_chunks, per_last_chunks, ep);
}
// (fp32 sums of few products: fp32_split.h.  A kernel of its own, 36 -> 120 channels on 28 028 positions 10.1 us; one for both with a branch 11.6)
template <typename T, typename TO, int TM, int TN, bool ROW16, int STEPS>
__global__ __launch_bounds__(256, 2) void conv1x1_mma_kernel(const T* __restrict__ x, TO* __restrict__ y, const char* __restrict__ wfrag,
                                                          const char* __restrict__ zeros, int64_t P, int Ci, int Co, int m_tiles_total,
                                                          int work_total, int work_per_xcd, int pitch, int span, int blocks,
                                                          uint32_t per_chunks, uint32_t per_last_chunks, Epilogue ep)
{
    whole_rows<T, TO, TM, TN, ROW16, STEPS>(x, y, wfrag, zeros, P, Ci, Co, m_tiles_total, work_total, work_per_xcd, pitch, span, blocks,
                                            per_chunks, per_last_chunks, ep);
}

template <typename T, typename TO, int TM, int TN, bool ROW16, int... STEPS>
rtoss_status launch_whole_rows_tile(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    constexpr int EB = (int)sizeof(TO), PT = 16 * TN, kTileBytes = 64 * 1024;
    constexpr int kSpan = (kTileBytes / PT - 32) / EB / (64 * TM) * (64 * TM);  // channels of a block, where a row is too long for the tile
    static_assert(kSpan > 0, "a block is at least one step of the channel loop");
    const int64_t P = (int64_t)c.N * c.H * c.W;
    // The output rows of a tile without gaps where rows are not aligned to 16 bytes and the tile is one piece of the output; else a
    // pitch that keeps them aligned.
    const auto padded = [](int64_t bytes) { return (bytes + 15) / 16 * 16 + 16; };
    int span = d.Co;
    int64_t pitch = (int64_t)d.Co * EB;
    if (pitch % 16 == 0 || c.ep.ldy != d.Co || d.Co < 16) pitch = padded(pitch);  // (fewer: a row's end runs over into an unordered one)
    if (pitch * PT > kTileBytes) {
        span = kSpan;
        pitch = padded(span * EB);
    }
    const int blocks = (d.Co + span - 1) / span;
    const auto reciprocal = [](int channels) { return (uint32_t)(((uint64_t)1 << 32) / (unsigned)((channels * EB + 15) / 16) + 1); };  // (exact: < 2^16 chunks a tile)
    const int64_t total = (P + PT - 1) / PT * blocks, per_xcd = (total + 7) / 8;
    if (total > 0x7ffffff0) return fail(RTOSS_ESHAPE, "conv1x1: too many tiles");  // (not within the limit of dense1x1_launch_ok)
    constexpr int extra = 16 + EpiScaleBias<64 * TM>::kBytes;
    auto kern = conv1x1_mma_kernel<T, TO, TM, TN, ROW16, STEPS...>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, kTileBytes + extra, lds_once, c.dev.device, "conv1x1 shared memory attribute")) return st;
    const int64_t groups = std::min<int64_t>(8 * per_xcd, kMaxGridGroups);
    kern<<<dim3((unsigned)groups), dim3(256), (size_t)pitch * PT + extra, s>>>(
        (const T*)x, (TO*)y, wfrag, wfrag + frag_bytes(d), P, d.Ci, d.Co, ring_padded_tiles(d.Co), (int)total, (int)per_xcd, (int)pitch, span, blocks,
        reciprocal(span), reciprocal(d.Co - (blocks - 1) * span), c.ep);
    return check_hip(hipGetLastError(), "conv1x1 launch");
}

template <typename T, typename TO, bool ROW16, int... STEPS>
rtoss_status launch_whole_rows_steps(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    // Tiles of 32 positions; of 64 where that still leaves more than one workgroup per compute unit and a workgroup's weights are
    // many (72 -> 255, 28 028 positions: 8.6 us and 9.3; 80 -> 85, 48 000: 8.1 and 7.6).  fp32 has no registers for that, and fp32
    // output no room in LDS: 64 positions of a step's 256 channels are the whole tile (72 -> 240, where they fit: 11.6 us, 32 positions 9.4).
    const int tiles = (d.Co + 15) / 16;
    if (tiles <= 4) return launch_whole_rows_tile<T, TO, 1, 2, ROW16, STEPS...>(d, c, wfrag, x, y, s);
    if (tiles <= 8) return launch_whole_rows_tile<T, TO, 2, 2, ROW16, STEPS...>(d, c, wfrag, x, y, s);
    if constexpr (sizeof(T) == 2 && sizeof(TO) == 2) {
        const DeviceInfo& dev = c.dev;
        if ((int64_t)c.N * c.H * c.W > 64 * (int64_t)dev.cus) return launch_whole_rows_tile<T, TO, 4, 4, ROW16>(d, c, wfrag, x, y, s);
    }
    return launch_whole_rows_tile<T, TO, 4, 2, ROW16, STEPS...>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO, bool ROW16>
rtoss_status launch_whole_rows(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    if constexpr (sizeof(T) == 4)
        if (few_live_products(d)) return launch_whole_rows_steps<T, TO, ROW16, kSplitAll>(d, c, wfrag, x, y, s);
    return launch_whole_rows_steps<T, TO, ROW16>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO, int TM>
rtoss_status launch_tm(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int64_t P = (int64_t)c.N * c.H * c.W;
    const int64_t pos_tiles = (P + kTilePos - 1) / kTilePos;
    const int co_blocks = ((d.Co + 15) / 16 + TM - 1) / TM;
    const int64_t total = pos_tiles * co_blocks;
    if (total > 0x3fffffff) return fail(RTOSS_ESHAPE, "conv1x1: too many tiles");
    const int work_per_xcd = (int)((total + 7) / 8);
    constexpr int stage_bytes = ((TM + 3) / 4) * 4096 + 2 * 4096;
    const size_t smem = (size_t)kRing * stage_bytes;
    auto kern = conv1x1_mma_kernel<T, TO, TM>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, c.dev.device, "conv1x1 shared memory attribute")) return st;
    dim3 grid((unsigned)(work_per_xcd * 8)), block(256);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + frag_bytes(d), P, d.Ci, d.Co, ring_padded_tiles(d.Co),
                                   Divisor(co_blocks), (int)total, work_per_xcd, c.ep);
    return check_hip(hipGetLastError(), "conv1x1 launch");
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    // the fragment section is padded to a multiple of 8 channel tiles, so a block of TM <= 8 tiles never reads past it
    const int tiles = (d.Co + 15) / 16;
    const int row_bytes = d.Ci * (int)sizeof(T);
    if (row_bytes % 16) return launch_whole_rows<T, TO, false>(d, c, wfrag, x, y, s);
    if (row_bytes % 64 || d.Co % 16) return launch_whole_rows<T, TO, true>(d, c, wfrag, x, y, s);
    // Whole tiles: while there are no more tiles of 32 positions than compute units, and the ring's blocks of 128 channels are
    // not the better split (us, ring and registers; positions in brackets):
    //     fp16  96 -> 128 (6400) 6.6 4.6   192 -> 256 (6400) 7.9 6.1   384 -> 256 (6400) 10.0 7.7   192 -> 256 (12 800) 8.3 8.4  stays
    //     fp16 192 ->  48 (6400) 5.2 5.1  stays   384 -> 512 (6400) 10.6 13.1  stays
    //     fp32  96 -> 128 (6400) 11.9 6.2  240 ->  48 (6400) 12.2 7.0  240 -> 256 (400) 21.1 12.2   240 -> 48 (25 600) 13.0 19.5  stays
    const DeviceInfo& dev = c.dev;
    if ((int64_t)c.N * c.H * c.W <= 32 * (int64_t)dev.cus && tiles <= 16 && (tiles > 4 || sizeof(T) == 4))
        return launch_whole_rows<T, TO, true>(d, c, wfrag, x, y, s);
    if (tiles <= 2) return launch_tm<T, TO, 2>(d, c, wfrag, x, y, s);
    if (tiles <= 4) return launch_tm<T, TO, 4>(d, c, wfrag, x, y, s);
    return launch_tm<T, TO, 8>(d, c, wfrag, x, y, s);
}

}  // namespace

bool dense1x1_shape_ok(const rtoss_wdesc& d)
{
    return d.ksize == 1 && d.Ci * elem_bytes(d.dt) % 4 == 0;
}

bool dense1x1_launch_ok(const rtoss_wdesc& d, const ConvParams& c)
{
    if (d.dt != RTOSS_F32 && d.Ci % 32 == 0 && d.Co % 16 == 0) return true;
    const int tiles = (d.Co + 15) / 16, per_block = tiles <= 4 ? 4 : 8;  // (a smaller block of a few-channel layer: the same number of them)
    return ((int64_t)c.N * c.H * c.W + kTilePos - 1) / kTilePos * ((tiles + per_block - 1) / per_block) <= kMaxGridGroups;
}

size_t dense1x1_section_bytes(const rtoss_wdesc& d) { return frag_bytes(d) + zero_section_bytes(stage_count(d)); }

rtoss_status launch_conv1x1_mma(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (d.dt == RTOSS_F32) return launch_typed<float, float>(d, c, wf, x, y, s);
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, wf, x, y, s);
}

}  // namespace rtoss
