// 1x1 pattern-pruned convolution on the CDNA4 matrix cores (fp16 / bf16 / fp32, fp32 accumulate):
// the general kernel, for any channel counts whose
// input rows are a multiple of 4 bytes.  (64-byte multiples of 2^n stages with whole channel tiles
// take the streaming kernel with register-resident weights instead.)
//
// Section IV.D prunes a 1x1 layer by cutting the flattened [Co][Ci] weight matrix into groups
// of 9 and keeping k weights per group, so the pruned layer is a GEMM
//     Y[p][co] = sum_ci W'[co][ci] * X[p][ci]          (p runs over all N*H*W positions)
// whose weight matrix has k-of-9 sparsity along its flattened axis.  That sparsity has no
// structure a matrix instruction could skip (groups straddle rows and have no 2-of-4 shape),
// and the layer is bound by HBM traffic anyway: activations in, activations out, every byte
// once.  So the weights are expanded to zero-filled dense fragments (they are tiny and stay in
// L2), and the kernel is built to stream activations: channels-last rows are contiguous, a
// workgroup owns 128 consecutive positions x up to 128 output channels, and K runs over stages
// of 64 bytes of input channels through a 5-deep ring of LDS buffers filled by global -> LDS copies
// four stages ahead (an HBM-bound kernel lives on bytes in flight: two resident workgroups per CU x
// four stages x 8 KB of activations).  Activation rows sit in LDS at a 64-byte pitch with their
// four 16-byte chunks XOR-swizzled by (position / 2) % 4, which makes the 16-byte operand reads
// of 8 neighbouring positions hit 8 different bank groups without any padding.
//
// Ragged channel counts (RAG): the last stage's lanes past the row end copy the block of zeros, rows that are
// not 16-byte aligned are copied 4 bytes per lane (COPY), and output rows that are not leave LDS 4 bytes per lane
// too, consecutive lanes on consecutive channels (a row of 255 16-bit channels has no alignment to exploit, but a
// store instruction covers 256 neighbouring bytes).  On the vector ALUs 72 -> 255 channels on 28 028 positions took
// 74 us, here 13; the stores' address processing is most of what is left.
//
// Operand layout of v_mfma_f32_16x16x32 (wave64; r = lane % 16, q = lane / 16): A lane holds
// row r, K = 8q..8q+7; B lane holds column r, K = 8q..8q+7; D lane holds column r, rows 4q..4q+3.
// fp32: four v_mfma_f32_16x16x4_f32 per step, instruction s on element s of every lane's 16 bytes.
#include <algorithm>

#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "pack_plan.h"

namespace rtoss {

namespace {

constexpr int kFrag = 1024;      // one A fragment: 64 lanes x 16 bytes = 16 output channels x 64 bytes of input channels
constexpr int kTilePos = 128;    // positions per workgroup
constexpr int kRing = 5;

inline size_t frag_bytes(const rtoss_wdesc& d) { return (size_t)stage_count(d) * ring_padded_tiles(d.Co) * kFrag; }

template <typename T, typename TO, int TM, bool RAG, int COPY>
__global__ __launch_bounds__(256) void conv1x1_mma_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                          const char* __restrict__ wfrag, const char* __restrict__ zeros,
                                                          int64_t P, int Ci, int Co, int m_tiles_total, int co_blocks,
                                                          int total_work, int work_per_xcd, Epilogue ep)
{
    constexpr int TN = 2;                                // 16-position blocks per wave
    constexpr int A_PER_WAVE = (TM + 3) / 4;             // copy instructions per wave and stage (64 lanes x 16 B each)
    constexpr int A_AREA = A_PER_WAVE * 4 * 1024;
    constexpr int X_PER_WAVE = 32 / COPY;                // 128 positions x 64 bytes, 64 * COPY bytes per copy instruction
    constexpr int X_AREA = 4 * X_PER_WAVE * 64 * COPY;
    constexpr int STAGE = A_AREA + X_AREA;
    constexpr int CPW = A_PER_WAVE + X_PER_WAVE;         // copies one wave has in flight per stage
    extern __shared__ __attribute__((aligned(16))) char smem[];  // kRing stages

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    // XCD-contiguous work order (channel blocks of one position tile, and neighbouring tiles, share an L2)
    const int work = (blockIdx.x % 8) * work_per_xcd + blockIdx.x / 8;
    if (work >= total_work) return;
    const int cblk = work % co_blocks;
    const int64_t p0 = (int64_t)(work / co_blocks) * kTilePos;
    const int mt0 = cblk * TM;
    const int row_bytes = Ci * (int)sizeof(T);
    const int stages = (row_bytes + 63) / 64;

    // ---- copy sources: every lane copies 16 bytes in every copy instruction (no branches); lanes
    // whose slot is padding read the packer's block of zeros ----
    const char* x_ptr[X_PER_WAVE];
    unsigned tail_ok = 0;  // RAG: bit k = the last stage still has channels at this lane's copy k
#pragma unroll
    for (int k = 0; k < X_PER_WAVE; ++k) {
        const int e = ((k * 4 + wave) * 64 + lane) * COPY, c = e / 16;  // LDS byte, and chunk, this lane fills
        const int pos = c >> 2, q = (c & 3) ^ ((pos >> 1) & 3);         // ... holds channel chunk q of position pos
        const int at = q * 16 + e % 16;                                 // byte within the stage
        const bool real = p0 + pos < P;
        x_ptr[k] = real ? (const char*)x + (p0 + pos) * row_bytes + at : zeros;
        if (RAG && (stages - 1) * 64 + at < row_bytes) tail_ok |= 1u << k;
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
        for (int k = 0; k < X_PER_WAVE; ++k) {
            const char* src = x_ptr[k] + stage * 64;
            if (RAG && stage == stages - 1 && !(tail_ok >> k & 1u)) src = zeros;
            char* dst = base + A_AREA + (k * 4 + wave) * 64 * COPY;
            if constexpr (COPY == 16) copy16_to_lds(src, dst);
            else copy4_to_lds(src, dst);
        }
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
    static_assert(AHEAD * CPW < 64 && X_PER_WAVE <= 32, "outstanding copies must fit the counter");
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
                            if constexpr (RAG) {
                                epi_ragged<TO, 4>(vv, ep, p_f, co4, Co);
                            } else {
                                epi_scale_bias_act<4>(vv, ep, co4);
                                epi_residual<TO, 4>(vv, ep, p_f, co4);
                            }
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
            if constexpr (RAG) {
                if (Co * EB % 16 != 0 || ep.ldy * EB % 16 != 0) {  // uniform: rows without a 16-byte alignment
                    // a lane takes 4 bytes of a row (two 16-bit channels: the store need not be aligned), eight rows at a
                    // time so that their LDS reads are in flight together
                    constexpr int PER = 4 / EB, LANES = TMH * 16 / PER;  // lanes a row of this block occupies
                    constexpr int ROWS = LANES >= 64 ? 1 : 64 / LANES;   // rows per instruction
                    static_assert(LANES <= 64 && 64 % LANES == 0 && (16 * TN) % (8 * ROWS) == 0, "rows tile the wave");
                    const int c = (lane % LANES) * PER, live = min(PER, Co - co_first - c);
                    const int64_t first = p0 + wave * (TN * 16) + lane / LANES;
                    TO* yp = y + first * ep.ldy + co_first + c;
                    for (int r0 = 0; r0 < 16 * TN; r0 += 8 * ROWS) {
                        uint32_t v[8];
#pragma unroll
                        for (int i = 0; i < 8; ++i)
                            v[i] = *(const uint32_t*)(stage_out + (r0 + i * ROWS + lane / LANES) * ROW + c * EB);
#pragma unroll
                        for (int i = 0; i < 8; ++i) {
                            const int r = r0 + i * ROWS;
                            if (first + r >= P || live <= 0) continue;
                            char* at = (char*)(yp + (int64_t)r * ep.ldy);
                            if (live == PER) __builtin_memcpy(at, &v[i], 4);
                            else __builtin_memcpy(at, &v[i], EB);
                        }
                    }
                    continue;
                }
            }
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

template <typename T, typename TO, int TM, bool RAG = false, int COPY = 16>
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
    auto kern = conv1x1_mma_kernel<T, TO, TM, RAG, COPY>;
    static LaunchOnce lds_once;  // per instantiation
    if (rtoss_status st = ensure_dynamic_lds((const void*)kern, smem, lds_once, "conv1x1 shared memory attribute")) return st;
    dim3 grid((unsigned)(work_per_xcd * 8)), block(256);
    kern<<<grid, block, smem, s>>>((const T*)x, (TO*)y, wfrag, wfrag + frag_bytes(d), P, d.Ci, d.Co, ring_padded_tiles(d.Co),
                                   co_blocks, (int)total, work_per_xcd, c.ep);
    return check_hip(hipGetLastError(), "conv1x1 launch");
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    // the fragment section is padded to a multiple of 8 channel tiles, so a block of TM <= 8 tiles never reads past it
    const int tiles = (d.Co + 15) / 16;
    const int row_bytes = d.Ci * (int)sizeof(T);
    if (row_bytes % 16) {  // input rows are 4-byte aligned only
        if (tiles <= 4) return launch_tm<T, TO, 4, true, 4>(d, c, wfrag, x, y, s);
        return launch_tm<T, TO, 8, true, 4>(d, c, wfrag, x, y, s);
    }
    if (row_bytes % 64 || d.Co % 16) {
        if (tiles <= 4) return launch_tm<T, TO, 4, true>(d, c, wfrag, x, y, s);
        return launch_tm<T, TO, 8, true>(d, c, wfrag, x, y, s);
    }
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
