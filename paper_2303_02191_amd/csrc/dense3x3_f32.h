// 3x3 dense mode of fp32 tensors: one workgroup's tile of 64 output channels x R rows x 16 columns on the bf16 matrix
// instruction (fp32_split.h).  Reads the dense-mode section (pack_plan.h).  The kernels around it: conv3x3_dense.hip (two and
// four rows: medium launches, stride 2, ragged channel counts), conv3x3_strip.hip (eight rows: large launches).
#pragma once
#include "common.h"
#include "epilogue.h"
#include "fp32_split.h"
#include "pack_plan.h"

namespace rtoss {

template <int S, int R> struct F32Tile {
    static constexpr int IH = (R - 1) * S + 3, LW = 15 * S + 3;  // input rows and columns
    static constexpr int POS = IH * LW;
    static constexpr int PLANE = POS * 64;                       // 32 channels of one bf16 part
    static constexpr int BUF = 3 * PLANE;
    static constexpr int LDS = 2 * BUF;
    static constexpr int U = (POS * 4 + 255) / 256;              // 32-byte pieces of the input a lane splits per stage
};

// A stage is 32 input channels: two 16-channel stages of the section.  All four waves split the stage's activations into
// LDS, once for the nine taps and the four waves that read them; a wave owns 16 of the 64 channels and all positions, so its
// weights go straight from memory into its registers and are split there.  The next stage's activations and the next column
// of taps' weights are on their way while the current ones are multiplied.
// The 16 columns of a matrix instruction are 16 positions of one output row, and input row i at column shift kw serves up to
// three output rows: a stage is three columns of taps (kw), and in each a wave reads every input row once.  At stride 2 the
// even and odd columns lie apart in LDS, so that these reads are contiguous too.
//
// What bounds it: the matrix pipes in part (256 -> 256 channels on 4x80x80, eight rows: 135 us where the six products take 79 at
// the instruction's peak; the fp32 instruction took 274), and in part the splitting.  A SIMD issues two vector instructions in
// the shadow of a matrix instruction and adds four cycles for every further one; a stage has 108 matrix instructions per two
// rows and 400 vector instructions for the wave's weights whatever the rows.  Dealing the vector instructions evenly between
// the matrix instructions gained nothing over leaving them to a second resident workgroup.
template <int S, int R, bool RAG>
__device__ __forceinline__ void dense3x3_f32_tile(const float* __restrict__ x, float* __restrict__ y, const char* __restrict__ wfrag,
                                                  const char* __restrict__ zeros, int H, int W, int Ci, int Co, int Ho, int Wo,
                                                  int cblocks, int cb, int n_img, int oh0, int ow0, const Epilogue& ep, char* smem)
{
    using P = F32Tile<S, R>;
    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int half_stages = (Ci + 15) / 16, stages = (half_stages + 1) / 2;

    // ---- activations: piece = (position, quarter): 4 channels of either half of the stage ----
    const char* src[P::U];
    int q_of[P::U];
#pragma unroll
    for (int u = 0; u < P::U; ++u) {
        const int c = u * 256 + tid, pos = c >> 2, q = c & 3;
        const int r = pos / P::LW, i = pos % P::LW, col = S == 1 ? i : (i < 17 ? 2 * i : 2 * (i - 17) + 1);
        const int ih = oh0 * S - 1 + r, iw = ow0 * S - 1 + col;
        const bool inside = pos < P::POS && (unsigned)ih < (unsigned)H && (unsigned)iw < (unsigned)W;
        src[u] = inside ? (const char*)(x + (((int64_t)n_img * H + ih) * W + iw) * Ci + 4 * q) : zeros;
        q_of[u] = q;
    }
    u32x4 raw[P::U][2];
    auto load_activations = [&](int stage) {
#pragma unroll
        for (int u = 0; u < P::U; ++u) {
            const char* p = src[u] + stage * 128;
            const int left = Ci - 32 * stage - 4 * q_of[u];  // channels the row still has at this piece (Ci is a multiple of 4)
            raw[u][0] = *(const u32x4*)(!RAG || left > 0 ? p : zeros);
            raw[u][1] = *(const u32x4*)(left > 16 ? p + 64 : zeros);
        }
    };
    // ---- weights: this wave's tile of the block, one column of taps at a time ----
    const char* a_src = wfrag + (int64_t)(4 * cb + wave) * kDenseTileBytes + lane * 16;
    const int64_t a_half = (int64_t)cblocks * (4 * kDenseTileBytes);
    u32x4 araw[3][2];
    auto load_weights = [&](int stage, int kw) {
        const char* p = a_src + 2 * stage * a_half + kw * kFragBytes;
        const bool second = 2 * stage + 1 < half_stages;  // uniform
#pragma unroll
        for (int kh = 0; kh < 3; ++kh) {
            araw[kh][0] = *(const u32x4*)(p + 3 * kh * kFragBytes);
            araw[kh][1] = *(const u32x4*)(second ? p + a_half + 3 * kh * kFragBytes : zeros);
        }
    };
    load_weights(0, 0);
    load_activations(0);
    const int nn = lane & 15, qq = lane >> 4;
    const int co = 64 * cb + 16 * qq + 4 * wave, ow = ow0 + nn;  // this lane's 4 channels and column
    // (asked for here: behind the last product they would be a wait of their own)
    f32x4 scale, bias;
    if (!RAG && co < Co) {
        if (ep.scale) scale = *(const f32x4*)(ep.scale + co);
        if (ep.bias) bias = *(const f32x4*)(ep.bias + co);
    }

    f32x4 main[R], small[R];
#pragma unroll
    for (int j = 0; j < R; ++j) main[j] = small[j] = f32x4{0.f, 0.f, 0.f, 0.f};
    for (int stage = 0; stage < stages; ++stage) {
        const int next = min(stage + 1, stages - 1);  // (behind the last stage: loaded again, not used; a branch would make the waits coarser)
        char* buf = smem + (stage & 1) * P::BUF;
#pragma unroll
        for (int u = 0; u < P::U; ++u) {
            const int c = u * 256 + tid;
            const Split8 s = split8(raw[u][0], raw[u][1]);
            if ((u + 1) * 256 > P::POS * 4 && c >= P::POS * 4) break;
            *(u32x4*)(buf + c * 16) = s.h;
            *(u32x4*)(buf + P::PLANE + c * 16) = s.m;
            *(u32x4*)(buf + 2 * P::PLANE + c * 16) = s.l;
        }
        const char* X = buf + nn * 64 + qq * 16;
#pragma unroll
        for (int kw = 0; kw < 3; ++kw) {
            Split8 a[3];
#pragma unroll
            for (int kh = 0; kh < 3; ++kh) a[kh] = split8(araw[kh][0], araw[kh][1]);
            __builtin_amdgcn_sched_barrier(0);  // (the scheduler would move the loads down to where they are used)
            load_weights(kw < 2 ? stage : next, kw < 2 ? kw + 1 : 0);
            if (kw == 0) {
                load_activations(next);
                __syncthreads();  // the stage is in LDS; everybody is done with the other buffer, which the next one takes
            }
            const int shift = S == 1 ? kw : (kw & 1) * 17 + (kw >> 1);  // (stride 2: even columns first, odd ones from 17 on)
            auto row = [&](int i) {
                const char* at = X + (i * P::LW + shift) * 64;
                return Split8{*(const u32x4*)at, *(const u32x4*)(at + P::PLANE), *(const u32x4*)(at + 2 * P::PLANE)};
            };
            Split8 b = row(0);
#pragma unroll
            for (int i = 0; i < P::IH; ++i) {
                Split8 coming;
                if (i + 1 < P::IH) coming = row(i + 1);
                __builtin_amdgcn_sched_barrier(0);  // (likewise)
                split_steps<kSplitSix>([&](auto step) {
#pragma unroll
                    for (int kh = 0; kh < 3; ++kh) {
                        const int j = (i - kh) / S;
                        if (i < kh || (i - kh) % S || j >= R) continue;
                        split_step<decltype(step)::value>(a[kh], b, main[j], small[j]);
                    }
                });
                if (i + 1 < P::IH) b = coming;
            }
        }
    }

    // ---- store: a lane holds 4 consecutive channels of one position per row ----
    const bool live = co < Co && ow < Wo;
    const int64_t pos0 = ((int64_t)n_img * Ho + oh0) * Wo + ow;
    if constexpr (RAG) {
        if (!live) return;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (oh0 + j >= Ho) break;
            const int64_t pos = pos0 + (int64_t)j * Wo;
            const f32x4 sum = split_sum(main[j], small[j]);
            float v[4] = {sum.x, sum.y, sum.z, sum.w};
            epi_ragged<float, 4>(v, ep, pos, co, Co);
            store_ragged<float, 4>(y + pos * ep.ldy, v, co, Co, ep.ldy);
        }
    } else {
        EpiResidual<float, 4> shortcut[R];
        if (ep.residual && live)
#pragma unroll
            for (int j = 0; j < R; ++j)
                if (oh0 + j < Ho) shortcut[j].load(ep, pos0 + (int64_t)j * Wo, co);
        float v[4 * R];
#pragma unroll
        for (int j = 0; j < R; ++j) {
            f32x4 t = split_sum(main[j], small[j]);
            if (ep.scale) t *= scale;
            if (ep.bias) t += bias;
#pragma unroll
            for (int e = 0; e < 4; ++e) v[4 * j + e] = t[e];
        }
        epi_act<4 * R>(v, ep.act);
        // whole rows of 64 channels past the L2's write-back, through the buffer that the last stage does not read (64 -> 64 on
        // 4x40x40 8.5 -> 8.1 us, 256 -> 256 on 4x80x80 139.8 -> 137.9)
        static_assert(R * 4096 <= P::BUF, "the outputs fit a buffer");
        char* out = smem + (stages & 1) * P::BUF;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            float o[4] = {v[4 * j], v[4 * j + 1], v[4 * j + 2], v[4 * j + 3]};
            if (ep.residual) shortcut[j].add(o);
            *(f32x4*)(out + j * 4096 + nn * 256 + ((co / 4 % 16) ^ nn) * 16) = f32x4{o[0], o[1], o[2], o[3]};
        }
        __syncthreads();
        const int col = tid >> 4, chunk = tid & 15;
        const bool inside = ow0 + col < Wo && 64 * cb + 4 * chunk < Co;
#pragma unroll
        for (int j = 0; j < R; ++j) {
            if (oh0 + j >= Ho) break;
            const auto base = store_base(y + (((int64_t)n_img * Ho + oh0 + j) * Wo + ow0) * ep.ldy + 64 * cb);
            store16_through(base, inside ? (uint32_t)col * ep.ldy * 4 + chunk * 16 : kNoStore,
                            *(const u32x4*)(out + j * 4096 + col * 256 + (chunk ^ col) * 16));
        }
    }
}

}  // namespace rtoss
