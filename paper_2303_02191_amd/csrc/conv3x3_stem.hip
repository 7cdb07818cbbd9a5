// 3x3 convolution for very small input channel counts (the 3-channel image stem) on the dense
// matrix instruction (fp16 / bf16, fp32 accumulate).
//
// With Ci <= 3 the whole reduction, K = 9*Ci <= 27, fits one v_mfma_f32_16x16x32 step: a block
// of 16 output positions x 16 output channels is one instruction, pruned taps are explicit
// zeros in the weight fragment (there is nothing to skip in a single instruction), and the
// layer is bound by the output write.  K index k = kh*(3*Ci) + kw*Ci + ci, which is the memory
// order of a channels-last patch row, so a lane's 8 consecutive K values are short contiguous
// runs of the input tile staged in LDS.
//
// What bounds it: the vector instructions of the output stage (3 -> 32 channels on 16x640x640 with SiLU: 38.3 us, 30 of them the
// time of its 144 MB).  So what surrounds that stage is kept small: the tile comes in aligned words, with uniform row
// arithmetic, instead of halves (52.2 -> 42.4 us), scale and bias stay in registers, addresses advance by uniform steps.
//
// Operand layout (wave64; r = lane % 16, q = lane / 16): A lane holds row r, K = 8q..8q+7; B lane
// holds column r, K = 8q..8q+7; D lane holds column r, rows 4q..4q+3.
#include "common.h"
#include "dtypes.h"
#include "epilogue.h"
#include "mma.h"
#include "work_order.h"
#include "stem_rows.h"

namespace rtoss {

namespace {

constexpr int kTH = 8, kTW = 32;  // output tile: 8 rows x 32 columns = 16 blocks of 16 positions


// Ci is a template parameter: the index arithmetic below divides by it (and by 3 * Ci) per element, which
// as run-time divisions made the kernel bound by integer ALU work.
template <typename T, typename TO, int S, int TM, int Ci>
__global__ __launch_bounds__(256, TM == 2 ? 6 : 4) void conv3x3_stem_kernel(const T* __restrict__ x, TO* __restrict__ y,
                                                           const char* __restrict__ wfrag, int H, int W, int Co,
                                                           int Ho, int Wo, Divisor tiles_c, int odd_image, Epilogue ep)
{
    constexpr int IH = (kTH - 1) * S + 3, IW = (kTW - 1) * S + 3;
    constexpr int kRow = IW * Ci;                 // halves of an input row of the tile
    constexpr int kPer = (kRow / 2 + 64) / 64;    // rounds of 64 aligned words that cover such a row, wherever it begins
    constexpr int kPitch = 128 * kPer;            // halves of a row in LDS: whole rounds
    constexpr int kRows = (IH + 3) / 4;
    // Behind the tile: the zeros of the K slots past the reduction, one half for each of a lane's four blocks below.
    constexpr int kNone = IH * kPitch, kDown = S * kPitch, kRight = 16 * S * Ci;
    __shared__ __attribute__((aligned(16))) uint16_t smem[2 + kNone + kDown + kRight + 1];
    uint16_t* const xs = smem + 2;

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int tile_r = tiles_c.quotient(blockIdx.x), tile_c = tiles_c.remainder(blockIdx.x, tile_r);
    const int n_img = blockIdx.y;
    const int oh0 = tile_r * kTH, ow0 = tile_c * kTW;
    const int ih0 = oh0 * S - 1, iw0 = ow0 * S - 1;

    // ---- stage the input tile (with halo, zero padded): wave w takes rows w, w + 4, ... as aligned words, all of them asked for
    // before the first one is used.  Of a tensor of an odd number of halves the last one is read by itself, below. ----
    const int lo = iw0 < 0 ? Ci : 0, hi = min(IW, W - iw0) * Ci;  // halves of a row inside the image
    const bool edge = lo > 0 || hi < kRow;                        // uniform, and so is the next
    const bool alternate = (W & Ci & 1) != 0;                     // rows begin in the lower and the upper half of a word in turn
    const int cut_row = n_img == odd_image && W - iw0 <= IW ? H - 1 : -1;  // input row of the tile that ends a tensor of an odd number of halves
    uint32_t word[kRows][kPer];
    int odd[kRows];  // uniform: the row begins in the upper half of its first word
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int ih = min(max(ih0 + wave + 4 * i, 0), H - 1);
        const int64_t at = (((int64_t)n_img * H + ih) * W + iw0) * Ci;
        const StemRow row((int)at & 1, lo, hi, ih == cut_row);
        odd[i] = row.odd;
        const char* src = (const char*)x + (at - row.odd) * 2;
#pragma unroll
        for (int k = 0; k < kPer; ++k) word[i][k] = *(const uint32_t*)(src + 4 * row.word(k * 64 + lane));
    }
    // weight fragments stay in registers: TM tiles of 16 output channels; so do scale and bias of this lane's channels
    u32x4 afrag[TM];
#pragma unroll
    for (int m = 0; m < TM; ++m) afrag[m] = *(const u32x4*)(wfrag + (m * 64 + lane) * 16);
    const int nn = lane & 15, qq = lane >> 4;
    float scale[4 * TM], bias[4 * TM];
#pragma unroll
    for (int mp = 0; mp < TM; mp += 2) {
        const int co = 16 * mp + 8 * qq;  // this lane's 8 consecutive channels of a pair of tiles
#pragma unroll
        for (int g = 0; g < 2; ++g) {
            if (ep.scale && co < Co) *(f32x4*)(scale + 4 * mp + 4 * g) = *(const f32x4*)(ep.scale + co + 4 * g);
            if (ep.bias && co < Co) *(f32x4*)(bias + 4 * mp + 4 * g) = *(const f32x4*)(ep.bias + co + 4 * g);
        }
    }
#pragma unroll
    for (int i = 0; i < kRows; ++i) {
        const int r = wave + 4 * i, ih = ih0 + r;
        if (r >= IH) continue;  // uniform
        const bool outside = (unsigned)ih >= (unsigned)H;  // uniform
        uint16_t* row = xs + r * kPitch;
#pragma unroll
        for (int k = 0; k < kPer; ++k) {
            const int d = k * 64 + lane, h = 2 * d - odd[i];  // the word's first half
            uint32_t w = outside ? 0 : word[i][k];
            if (edge) {
                if (h < lo || h >= hi) w &= 0xffff0000u;
                if (h + 1 < lo || h + 1 >= hi) w &= 0xffffu;
            }
            if (alternate && odd[i]) {
                row[2 * d - 1] = (uint16_t)w;
                row[2 * d] = (uint16_t)(w >> 16);
            } else {
                *(uint32_t*)(row + 2 * d) = w;
            }
        }
    }
    if (cut_row >= 0) {  // uniform: the tensor's last half
        const int r = cut_row - ih0;
        asm volatile("" ::: "memory");  // (behind the wave's own write of that row)
        if (r < IH && wave == (r & 3) && lane == 0) xs[r * kPitch + hi - 1] = ((const uint16_t*)x)[(((int64_t)n_img + 1) * H * W) * Ci - 1];
    }
    if (tid < 4) xs[kNone + (tid >> 1) * kDown + (tid & 1) * kRight] = 0;
    const int begin = alternate ? 0 : odd[0];  // of a row in LDS
    __syncthreads();

    // LDS offset of each of this lane's 8 K values relative to the block's first position (same for all blocks).  Those past the
    // reduction weigh 0 and read zeros (a value of the tile may be infinite).
    constexpr int k3 = 3 * Ci, K = 9 * Ci;
    int koff[8];
#pragma unroll
    for (int j = 0; j < 8; ++j) {
        const int k = 8 * qq + j, kh = k / k3;
        koff[j] = k < K ? kh * kPitch + k - kh * k3 + 2 * wave * S * kPitch + nn * S * Ci + begin : kNone;
    }
    // (position and address of this lane's first output; a block's distance from it is uniform)
    const int64_t pos0 = ((int64_t)n_img * Ho + oh0 + 2 * wave) * Wo + ow0 + nn;
    TO* const y0 = y + pos0 * ep.ldy + 8 * qq;
    const int left = Wo - ow0 - nn, below = Ho - oh0 - 2 * wave;
    static_assert(TM % 2 == 0, "pairs of channel tiles");
    epi_by_form(ep, [&](auto form) {
#pragma unroll 1
        for (int jb = 0; jb < 4; ++jb) {  // 16 blocks: 8 rows x 2 half-rows of 16 columns
            const int r = jb >> 1, c = (jb & 1) * 16;
            const uint16_t* at = xs + r * kDown + (jb & 1) * kRight;
            u32x4 b;
#pragma unroll
            for (int j = 0; j < 4; ++j) b[j] = at[koff[2 * j]] | ((uint32_t)at[koff[2 * j + 1]] << 16);
            if (r >= below) break;  // uniform
            const bool inside = c < left;
            const int64_t step = (int64_t)r * Wo + c;
            TO* yp = y0 + step * ep.ldy;
#pragma unroll
            for (int mp = 0; mp < TM; mp += 2) {
                const f32x4 d0 = Dense16<T>::mma(afrag[mp], b, f32x4{0.f, 0.f, 0.f, 0.f});
                const f32x4 d1 = Dense16<T>::mma(afrag[mp + 1], b, f32x4{0.f, 0.f, 0.f, 0.f});
                const int co = 16 * mp + 8 * qq;
                if (inside && co < Co) {
                    float vv[8] = {d0.x, d0.y, d0.z, d0.w, d1.x, d1.y, d1.z, d1.w};
                    epi_scale_bias_act_of<decltype(form)::value, 8>(vv, ep, scale + 4 * mp, bias + 4 * mp);
                    epi_residual<TO, 8>(vv, ep, pos0 + step, co);
                    if constexpr (sizeof(TO) == 4) {
                        *(f32x4*)(yp + 16 * mp) = f32x4{vv[0], vv[1], vv[2], vv[3]};
                        *(f32x4*)(yp + 16 * mp + 4) = f32x4{vv[4], vv[5], vv[6], vv[7]};
                    } else {
                        *(u32x4*)(yp + 16 * mp) = pack8_from_f32<TO>(vv);
                    }
                }
            }
        }
    });
}

template <typename T, typename TO, int S, int TM, int Ci>
rtoss_status launch_stem_ci(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int Ho = (c.H + 2 - 3) / S + 1, Wo = (c.W + 2 - 3) / S + 1;
    const int tiles_r = (Ho + kTH - 1) / kTH, tiles_c = (Wo + kTW - 1) / kTW;
    if (c.N > 65535) return fail(RTOSS_ESHAPE, "conv: batch too large");
    dim3 grid((unsigned)(tiles_r * tiles_c), (unsigned)c.N), block(256);
    conv3x3_stem_kernel<T, TO, S, TM, Ci><<<grid, block, 0, s>>>((const T*)x, (TO*)y, wfrag, c.H, c.W, d.Co, Ho, Wo, Divisor(tiles_c),
                                                                 c.N & c.H & c.W & Ci & 1 ? c.N - 1 : -1, c.ep);
    return check_hip(hipGetLastError(), "conv3x3 stem launch");
}

template <typename T, typename TO, int S, int TM>
rtoss_status launch_stem(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    if (d.Ci == 3) return launch_stem_ci<T, TO, S, TM, 3>(d, c, wfrag, x, y, s);
    if (d.Ci == 2) return launch_stem_ci<T, TO, S, TM, 2>(d, c, wfrag, x, y, s);
    return launch_stem_ci<T, TO, S, TM, 1>(d, c, wfrag, x, y, s);
}

template <typename T, typename TO>
rtoss_status launch_typed(const rtoss_wdesc& d, const ConvParams& c, const char* wfrag, const void* x, void* y, hipStream_t s)
{
    const int tiles = (d.Co + 15) / 16;
    if (c.stride == 1) {
        if (tiles <= 2) return launch_stem<T, TO, 1, 2>(d, c, wfrag, x, y, s);
        return launch_stem<T, TO, 1, 4>(d, c, wfrag, x, y, s);
    }
    if (tiles <= 2) return launch_stem<T, TO, 2, 2>(d, c, wfrag, x, y, s);
    return launch_stem<T, TO, 2, 4>(d, c, wfrag, x, y, s);
}

}  // namespace

bool stem3x3_shape_ok(const rtoss_wdesc& d)
{
    return d.ksize == 3 && (d.dt == RTOSS_F16 || d.dt == RTOSS_BF16) && d.Ci <= 3 && d.Co % 16 == 0 && d.Co <= 64;
}

// (rows are read as words of two values: stem_rows.h)
bool stem3x3_launch_ok(const rtoss_wdesc& d, const ConvParams& c) { return (int64_t)c.N * c.H * c.W * d.Ci > 1; }

size_t stem3x3_section_bytes(const rtoss_wdesc& d) { return (size_t)4 * 1024; }  // 4 tiles, unused ones zero

rtoss_status launch_conv3x3_stem(const rtoss_wdesc& d, const ConvParams& c, const void* section, const void* x, void* y,
                                 hipStream_t s)
{
    const char* wf = (const char*)section;
    const bool f32out = c.out_dt == RTOSS_F32;
    if (d.dt == RTOSS_F16)
        return f32out ? launch_typed<f16_t, float>(d, c, wf, x, y, s) : launch_typed<f16_t, f16_t>(d, c, wf, x, y, s);
    return f32out ? launch_typed<bf16_t, float>(d, c, wf, x, y, s) : launch_typed<bf16_t, bf16_t>(d, c, wf, x, y, s);
}

}  // namespace rtoss
