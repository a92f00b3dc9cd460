// The register-operand kernel (igemm_reg.hip) for fp32 tensors on the bf16 matrix instructions (split_bf16.h): results of few
// tiles, the waves of a workgroup split the reduction.
//
// A step is one tap of four channel blocks, two to a lane half; its operands come from memory straight into registers
// and are converted there by the wave that multiplies them.  What bounds it: conversions, four pairs (about 280 clocks) for
// each of the FK + FM operands of a step next to FK * FM * 192 clocks of MFMAs, which the waves of a SIMD take in
// turns; the fp32 instructions take FK * FM * 512.
#include <algorithm>

#include "igemm_fp32_again.h"
#include "split_bf16.h"

namespace convmi {

// FK x FM accumulator tiles per wave, NW waves that split the reduction, D steps in flight.
// FW (backward by data): the weights as the forward pass has them (put_weights).
template <int FK, int FM, int NW, int D, bool FW>
__global__ __launch_bounds__(NW * 64, FK * FM == 1 ? 4 : FK * FM == 2 ? 3 : 2) void igemm_reg_split_kernel(const IgemmArgs a)
{
    constexpr int TK = FK * 32, TM = FM * 32;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;

    int kt, mt, sp;
    if (!small_tile(a, blockIdx.x, kt, mt, sp)) return;
    const int k0 = kt * TK, m0 = mt * TM;
    const int PQ = a.P * a.Q, npix = a.N * PQ, HW = a.H * a.W, RS = a.R * a.S;
    const float inv_PQ = a.inv_P, inv_Q = a.inv_TQ;

    // (operand addresses as in igemm_reg.hip: the input's buffer starts pad_h rows and pad_w pixels early)
    const long long shift = ((long long)a.pad_h * a.W + a.pad_w) * 16;
    const rsrc_t rsrc_in = make_rsrc(static_cast<const char *>(a.in) - shift, 0, (size_t)((long long)a.N * a.Cb * HW * 16 + shift));
    const int taps = FW ? a.wt_taps : RS;
    const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * taps * a.Kp * 16);
    const unsigned row_block = (unsigned)taps * (unsigned)a.Cb * 64u;  // (FW) bytes of a block of rows
    unsigned b_off[FM], a_off[FK][2];
    int ih0[FM], iw0[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int m = m0 + j * 32 + l32;
        const int n = fast_div(m, inv_PQ);
        const int rem = m - mul24(n, PQ);
        const int oj = fast_div(rem, inv_Q);
        const int oi = rem - mul24(oj, a.Q);
        const int y = mul24(oj, a.stride), x = mul24(oi, a.cstride);
        b_off[j] = (unsigned)(mul24(mul24(mul24(n, a.Cb) + 2 * h, a.H) + y, a.W) + x) * 16u;
        // (a pixel beyond the last one: no row is inside the image)
        ih0[j] = m < npix ? y - a.pad_h : 0x40000000;
        iw0[j] = x - a.pad_w;
    }
#pragma unroll
    for (int i = 0; i < FK; ++i) {
        if constexpr (FW) {
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int blk = (k0 >> 2) + 8 * i + 4 * b + wt_block(lane);
                a_off[i][b] = blk < a.Kp >> 2 ? (unsigned)blk * row_block + (unsigned)wt_channel(lane) * 16u : kOutOfRange;
            }
        } else {
            const int k = k0 + i * 32 + l32;
            a_off[i][0] = a_off[i][1] = k < a.Kp ? (unsigned)(mul24(2 * h, RS * a.Kp) + k) * 16u : kOutOfRange;
        }
    }

    // This wave's share of the reduction: steps [u0, u1), step u = (four channel blocks, r, s).
    const int steps = ((a.Cb + 3) >> 2) * RS;
    const int sbeg = sp * a.st_per;
    const int nst = min(steps - sbeg, a.st_per);
    const int per = (nst + NW - 1) / NW;
    const int u0 = sbeg + min(wave * per, nst), u1 = sbeg + min(wave * per + per, nst);
    int cq = u0 / RS;
    int tap = u0 - cq * RS;
    int r = tap / a.S;
    int s = tap - r * a.S;
    int u = u0;  // next step to load

    u32x4 A[D][FK][2], B[D][FM][2];
    auto load = [&](u32x4(&av)[FK][2], u32x4(&bv)[FM][2]) {
        // (past the wave's share, and blocks beyond the last one: zeros on both sides)
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const bool live = u < u1 && 4 * cq + 2 * h + b < a.Cb;
            const unsigned sa = u < u1 ? (unsigned)((4 * cq + b) * RS + r * a.S + s) * (unsigned)a.Kp * 16u : 0u;
            const unsigned sb = u < u1 ? (unsigned)((4 * cq + b) * HW + r * a.W + s) * 16u : 0u;
#pragma unroll
            for (int j = 0; j < FM; ++j) {
                const bool in = live && (unsigned)(ih0[j] + r) < (unsigned)a.H && (unsigned)(iw0[j] + s) < (unsigned)a.W;
                bv[j][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, in ? b_off[j] : kOutOfRange, sb, 0);
            }
            if constexpr (!FW)
#pragma unroll
                for (int i = 0; i < FK; ++i)
                    av[i][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, live ? a_off[i][b] : kOutOfRange, sa, 0);
        }
        if constexpr (FW) {
            const bool mine = u < u1 && 16 * cq + wt_channel(lane) < 4 * a.Cb;
            const unsigned sf = u < u1 ? ((unsigned)(a.wt_tap0 - r * a.wt_dr - s * a.wt_ds) * (unsigned)a.Cb + 4u * cq) * 64u : 0u;
#pragma unroll
            for (int i = 0; i < FK; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    av[i][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, mine ? a_off[i][b] : kOutOfRange, sf, 0);
        }
        ++u;
        if (++s == a.S) {
            s = 0;
            if (++r == a.R) {
                r = 0;
                ++cq;
            }
        }
    };

    unsigned lost = 0;  // bits of the operands that no bf16 number holds
    f32x16 big[FK][FM], small[FK][FM];
#pragma unroll
    for (int i = 0; i < FK; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) big[i][j] = small[i][j] = f32x16{};
    unsigned char *const area = lds + wave * (FK * kWtBytes);
    if (u0 < u1) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(A[d], B[d]);
        // (loads past u1 ask for nothing: their lanes are out of range)
        for (int g = u0; g < u1; g += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                Bf16x3 as[FK], bs[FM];
#pragma unroll
                for (int i = 0; i < FK; ++i) {
                    as[i] = split8<false>(A[d][i], lost);
                    if constexpr (FW) put_weights(area + i * kWtBytes, lane, as[i]);
                }
#pragma unroll
                for (int j = 0; j < FM; ++j) bs[j] = split8<false>(B[d][j], lost);
                load(A[d], B[d]);
                if constexpr (FW) {
#pragma unroll
                    for (int i = 0; i < FK; ++i) as[i] = get_weights(area + i * kWtBytes, lane);
                }
                static_for<0, kSplitProducts>([&](auto t) {
#pragma unroll
                    for (int i = 0; i < FK; ++i)
#pragma unroll
                        for (int j = 0; j < FM; ++j) mma_split<decltype(t)::value>(as[i], bs[j], big[i][j], small[i][j]);
                });
                __builtin_amdgcn_sched_barrier(0);
            }
        }
    }
    mark_if_lost(lost, big[0]);
    float most = 0.0f;
#pragma unroll
    for (int i = 0; i < FK; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            big[i][j] += small[i][j];
            most = max_magnitude(most, big[i][j]);
        }
    // Infinite or NaN sums: the wave's share again.
    if (__builtin_expect(sums_need_fp32(most), 0)) {
        static_for<0, FK * FM>([&](auto fc) {
            constexpr int i = decltype(fc)::value / FM, j = decltype(fc)::value % FM;
            const int m = m0 + j * 32 + l32, n = fast_div(m, inv_PQ), rem = m - mul24(n, PQ), oj = fast_div(rem, inv_Q);
            big[i][j] = fragment_in_fp32<FW>(a, n, oj, rem - mul24(oj, a.Q), m < npix, k0 + i * 32 + l32, u0, u1);
        });
    }
    if constexpr (FW) __syncthreads();  // (the weights are done with before the sums take their place)
    add_and_store<CONV_F32, FK, FM, NW, true>(a, big, lds, k0, m0, sp, [&](int n, int oj, int oi, int krow) {
        return sum_inside_image<CONV_F32, 4, FW>(a, n, oj, oi, krow, sbeg, sbeg + nst);
    });
}

#define REG_SPLIT_ENTRY(FK, FM, NW, D) \
    {FK, FM, NW, igemm_reg_split_kernel<FK, FM, NW, D, false>, igemm_reg_split_kernel<FK, FM, NW, D, true>}
static const struct RegSplitEntry {
    int fk, fm, nw;
    igemm_fn_t fn, fwd_wt_fn;
} g_reg_split[] = {
    REG_SPLIT_ENTRY(1, 1, 4, 2), REG_SPLIT_ENTRY(1, 1, 8, 2), REG_SPLIT_ENTRY(2, 1, 4, 2), REG_SPLIT_ENTRY(2, 1, 8, 2),
    REG_SPLIT_ENTRY(1, 2, 4, 2), REG_SPLIT_ENTRY(2, 2, 4, 1), REG_SPLIT_ENTRY(2, 2, 8, 1), REG_SPLIT_ENTRY(1, 1, 16, 2),
};

bool igemm_reg_split_exists(int fk, int fm, int nw)
{
    for (const RegSplitEntry &e : g_reg_split)
        if (e.fk == fk && e.fm == fm && e.nw == nw) return true;
    return false;
}

size_t igemm_reg_split_lds_bytes(int fk, int fm, int nw, bool fwd_wt)
{
    return std::max((size_t)std::min(nw / 4, fk * fm) * nw * 4096, fwd_wt ? (size_t)nw * fk * kWtBytes : 0);
}

hipError_t launch_igemm_reg_split(int fk, int fm, int nw, const IgemmArgs &a, int grid, hipStream_t stream)
{
    for (const RegSplitEntry &e : g_reg_split) {
        if (e.fk != fk || e.fm != fm || e.nw != nw) continue;
        const size_t lds = igemm_reg_split_lds_bytes(fk, fm, nw, a.fwd_wt != 0);
        const igemm_fn_t fn = a.fwd_wt ? e.fwd_wt_fn : e.fn;
        if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(fn), lds); err != hipSuccess) return err;
        hipLaunchKernelGGL(fn, dim3(grid), dim3(nw * 64), lds, stream, a);
        return hipGetLastError();
    }
    return hipErrorInvalidDeviceFunction;
}

}  // namespace convmi
