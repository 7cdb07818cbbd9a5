// Output stage of the 3x3 kernels over strips of output rows (conv3x3_strip.hip, conv3x3_ring.hip).
#pragma once
#include "epilogue.h"

namespace rtoss {

constexpr int kStripTM = 4;               // channel tiles of a workgroup (64 channels)
constexpr int kStripCols = 16;            // output columns of a workgroup
constexpr int kStripLW = kStripCols + 2;  // input columns

// A wave's TN rows of 16 columns x 64 channels, from its accumulators: a lane holds column lane % 16 and the 16 consecutive channels 16 * (lane / 16)
// of every row.  oh0: the wave's first row; cb: block of 64 channels; lds_ep: scale and bias (EpiScaleBias).  ROWS_OUT: in rows of 128
// bytes, past the L2's write-back, through `area` (TN row tiles of LDS that nothing else uses).
template <typename TO, int TN, bool ROWS_OUT>
__device__ __forceinline__ void strip_output(const f32x4 (&acc)[kStripTM][TN], char* area, const float* lds_ep, TO* __restrict__ y, int H, int W,
                                             int Co, int cb, int n_img, int oh0, int ow0, int lane, const Epilogue& ep)
{
    const int nn = lane & 15, qq = lane >> 4;
    const int co = 64 * cb + 16 * qq, ow = ow0 + nn;
    const bool live = co < Co && ow < W;  // (Co is a multiple of 16: a run of 16 channels is all in or all out)
    if (!ROWS_OUT && !live) return;
    auto finish = [&](auto shortcut_tag, auto form) {
        constexpr bool SHORTCUT = decltype(shortcut_tag)::value;
        EpiResidual<TO, 16> shortcut[TN];
        const int64_t pos0 = ((int64_t)n_img * H + oh0) * W + ow;
        if constexpr (SHORTCUT) {  // its loads go out together, before any of them is needed
#pragma unroll
            for (int j = 0; j < TN; ++j)
                if (live && oh0 + j < H) shortcut[j].load(ep, pos0 + (int64_t)j * W, co);
        }
#pragma unroll
        for (int j = 0; j < TN; ++j) {
            if (oh0 + j >= H) break;
            TO* yp = y + (pos0 + (int64_t)j * W) * ep.ldy + co;
            float v[16];
#pragma unroll
            for (int m = 0; m < kStripTM; ++m)
#pragma unroll
                for (int e = 0; e < 4; ++e) v[4 * m + e] = acc[m][j][e];
            epi_scale_bias_act_of<decltype(form)::value, 16>(v, ep, lds_ep + 16 * qq, lds_ep + 64 + 16 * qq);
            if constexpr (SHORTCUT) shortcut[j].add(v);
            if constexpr (sizeof(TO) == 4) {
#pragma unroll
                for (int g = 0; g < 4; ++g) *(f32x4*)(yp + 4 * g) = f32x4{v[4 * g], v[4 * g + 1], v[4 * g + 2], v[4 * g + 3]};
            } else {
                const Run16<TO> o(v);
                if constexpr (!ROWS_OUT) {
                    o.store(yp);
                    continue;
                }
                RowTile<TO>::put(area + j * RowTile<TO>::kBytes, lane, o);
                const auto base = store_base(y + (((int64_t)n_img * H + oh0 + j) * W + ow0) * ep.ldy + 64 * cb);
                RowTile<TO>::store(area + j * RowTile<TO>::kBytes, lane, base, [&](int row, int c) {
                    return ow0 + row < W && 64 * cb + 8 * c < Co ? (uint32_t)row * ep.ldy * 2 + c * 16 : kNoStore;
                });
            }
        }
    };
    if (ep.residual) epi_by_form<false>(ep, [&](auto form) { finish(std::true_type{}, form); });
    else epi_by_form<false>(ep, [&](auto form) { finish(std::false_type{}, form); });
}

}  // namespace rtoss
