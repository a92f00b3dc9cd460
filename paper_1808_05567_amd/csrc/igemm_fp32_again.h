// Sums of fp32 tensors that the bf16 instructions could not form (split_bf16.h), again on the fp32 instructions by the wave that has
// them: a fragment of 32 channels x 32 pixels, operands straight from memory.
//
// What bounds it: the fp32 MFMAs, 512 clocks a step of 16 channels, beside which the next two steps are on their way.  All of a tensor NaN,
// the whole launch: 28 images 3x3 128 -> 128 at 28x28 156 us, 69 on the fp32 instructions alone (1 404 one product at a time); 64 images
// 512 -> 1024 1x1 stride 2 at 28x28 278 and 114 (3 671); one NaN in it 127 (1 032).
#pragma once
#include "igemm_exchange.h"

namespace convmi {

constexpr int kAgainSteps = 4;  // steps of 16 products that are summed apart (chains of 64)

// The lane's pixel is (n, oj, oi) (none: not `ok`), its row of the weights k; steps [u0, u1) of the reduction, a step is one tap of four
// channel blocks.  FW: the forward pass's weights.
template <bool FW>
static __device__ __forceinline__ f32x16 fragment_in_fp32(const IgemmArgs &a, int n, int oj, int oi, bool ok, int k, int u0, int u1)
{
    const int h = (threadIdx.x >> 5) & 1, HW = a.H * a.W, RS = a.R * a.S;
    const int taps = FW ? a.wt_taps : RS;
    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * taps * a.Kp * 16);
    const int y0 = oj * a.stride - a.pad_h, x0 = oi * a.cstride - a.pad_w;
    f32x16 sum{}, part{};
    auto load = [&](int u, f32x4 (&w)[2], f32x4 (&x)[2]) {
        const int cq = u / RS, tap = u - cq * RS, r = tap / a.S, s = tap - r * a.S, y = y0 + r, xx = x0 + s;
        const bool in = ok && (unsigned)y < (unsigned)a.H && (unsigned)xx < (unsigned)a.W;
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int cb = 4 * cq + 2 * h + b;
            const bool live = u < u1 && cb < a.Cb;
            const unsigned at = (((unsigned)n * (unsigned)a.Cb + (unsigned)cb) * (unsigned)HW + (unsigned)y * (unsigned)a.W + (unsigned)xx) * 16u;
            x[b] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, live && in ? at : kOutOfRange, 0, 0));
            const bool row = live && k < a.Kp;
            if constexpr (FW) {
                const unsigned ft = (unsigned)(a.wt_tap0 - r * a.wt_dr - s * a.wt_ds);
                const unsigned wt = (((unsigned)(k >> 2) * (unsigned)taps + ft) * (unsigned)a.Cb + (unsigned)cb) * 64u + (unsigned)(k & 3) * 4u;
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    w[b][t] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_wt, row ? wt + 16u * t : kOutOfRange, 0, 0));
            } else {
                const unsigned wt = (((unsigned)cb * (unsigned)RS + (unsigned)tap) * (unsigned)a.Kp + (unsigned)k) * 16u;
                w[b] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, row ? wt : kOutOfRange, 0, 0));
            }
        }
    };
    auto multiply = [&](const f32x4 (&w)[2], const f32x4 (&x)[2]) {
#pragma unroll
        for (int b = 0; b < 2; ++b)
#pragma unroll
            for (int t = 0; t < 4; ++t) part = __builtin_amdgcn_mfma_f32_32x32x2f32(w[b][t], x[b][t], part, 0, 0, 0);
    };
    if (a.no_taps) return sum;
    f32x4 w[2][2], x[2][2];
    load(u0, w[0], x[0]);
    for (int u = u0, g = 0; u < u1; u += 2) {
        load(u + 1, w[1], x[1]);
        multiply(w[0], x[0]);
        load(u + 2, w[0], x[0]);
        multiply(w[1], x[1]);  // (past the end: zeros)
        if ((g += 2) == kAgainSteps || u + 2 >= u1) {
            sum += part;
            part = f32x16{};
            g = 0;
        }
    }
    return sum;
}

}  // namespace convmi
