// The end of a kernel whose waves split the reduction of one small tile: their sums meet in LDS, and the
// result is stored with what is fused into it.  Shared by the register-operand kernel and the patch kernel.
#pragma once
#include "igemm_kernel.h"

namespace convmi {

static __device__ __forceinline__ bool any_nan(const f32x4 &v) { return v[0] != v[0] || v[1] != v[1] || v[2] != v[2] || v[3] != v[3]; }

// Workgroup -> tile (channel tile kt, pixel tile mt) and, where the reduction is split over workgroups, copy sp:
// dealt over the XCDs as in igemm_kernel.  False: nothing to do.
static __device__ __forceinline__ bool small_tile(const IgemmArgs &a, int bid, int &kt, int &mt, int &sp)
{
    const int x = bid & 7, jx = bid >> 3;
    sp = 0;
    if (a.gk == 1) {
        int lin = x * a.per_xcd + jx;
        if (lin >= a.total * a.ksplit) return false;
        sp = lin / a.total;
        lin -= sp * a.total;
        mt = lin / a.n_kt;
        kt = lin - mt * a.n_kt;
        return true;
    }
    const int kg = x % a.gk, mg = x / a.gk;
    const int mql = jx / a.kt_per;
    kt = kg * a.kt_per + (jx - mql * a.kt_per);
    mt = mg * a.mq_per + mql;
    return kt < a.n_kt && mql < a.mq_per && mt < a.n_mt;
}

template <int DT>
static __device__ __forceinline__ float widened(const void *base, size_t i)
{
    if constexpr (DT == CONV_BF16)
        return __builtin_bit_cast(float, (unsigned)static_cast<const unsigned short *>(base)[i] << 16);
    else
        return static_cast<const float *>(base)[i];
}

// Four consecutive channels of one pixel, krow .. krow + 3 at (n, oj, oi), summed over steps [u0, u1) one product at a time;
// a step is a tap of CBS channel blocks.  Taps outside the image are left out.  FW: the forward pass's weights.
template <int DT, int CBS, bool FW = false>
static __device__ __forceinline__ f32x4 sum_inside_image(const IgemmArgs &a, int n, int oj, int oi, int krow, int u0, int u1)
{
    constexpr int V = Elem<DT>::V;
    f32x4 sum = {0.f, 0.f, 0.f, 0.f};
    if (a.no_taps) return sum;
    const int RS = a.R * a.S;
    for (int u = u0; u < u1; ++u) {
        const int cp = u / RS, tap = u - cp * RS, r = tap / a.S, s = tap - r * a.S;
        const int y = oj * a.stride - a.pad_h + r, x = oi * a.cstride - a.pad_w + s;
        if (y < 0 || y >= a.H || x < 0 || x >= a.W) continue;
        for (int cb = CBS * cp; cb < min(CBS * cp + CBS, a.Cb); ++cb) {
            const size_t in = ((size_t)n * a.Cb + cb) * a.H * a.W + (size_t)y * a.W + x;
            const size_t wt = FW ? ((size_t)(krow / V) * a.wt_taps + (a.wt_tap0 - r * a.wt_dr - s * a.wt_ds)) * a.Cb * V + (size_t)cb * V
                                 : ((size_t)cb * RS + tap) * a.Kp + krow;
            for (int c = 0; c < V; ++c) {
                const float v = widened<DT>(a.in, in * V + c);
#pragma unroll
                for (int t = 0; t < 4; ++t)
                    sum[t] = fmaf(v, widened<DT>(a.wt, FW ? (wt + c) * V + krow % V + t : (wt + t) * V + c), sum[t]);
            }
        }
    }
    return sum;
}

// FK x FM fragments of NW waves.  EXACT: a sum that is NaN is replaced by again(n, oj, oi, krow) in plans that ask for it
// (IgemmArgs::exact).
template <int DT, int FK, int FM, int NW, bool EXACT, class F>
static __device__ __forceinline__ void add_and_store(const IgemmArgs &a, const f32x16 (&acc)[FK][FM], unsigned char *lds,
                                                     int k0, int m0, int sp, F &&again)
{
    using E_ = Elem<DT>;
    constexpr int V = E_::V;
    constexpr int NF = FK * FM, NT = NW * 64;
    // fragments summed per round through LDS: as many as give every thread a 4-channel chunk
    constexpr int G = (NT / 256 < NF) ? NT / 256 : NF;
    static_assert(NF % G == 0, "whole rounds");
    f32x4 *const xch = reinterpret_cast<f32x4 *>(lds);  // [G][NW][256] chunks of 4 channels
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;
    const int PQ = a.P * a.Q, npix = a.N * PQ;
    const float inv_PQ = a.inv_P, inv_Q = a.inv_TQ;  // (1 / (P*Q), 1 / Q in these kernels' plans)
    // The waves' sums, G fragments per round: every wave writes its own, then each thread adds
    // one chunk of 4 consecutive channels of one pixel over the waves, pairwise.
    constexpr int NR = NF / G;
    const size_t oplane = (size_t)a.OH * a.OW * 16;
    const size_t out_bytes = (size_t)a.N * a.out_kb * oplane;
    constexpr unsigned SC = (V == 8) ? 2u : 1u;  // a partial result is fp32 whatever the type
    const rsrc_t ro = a.ksplit > 1 ? make_rsrc(static_cast<char *>(a.out) + (size_t)sp * out_bytes * SC, 0, out_bytes * SC)
                                   : make_rsrc(a.out, 0, out_bytes);
    const int tg = tid >> 8, ch = tid & 255;  // (wave-uniform: 4 waves per fragment)
    // Where the thread's chunk of round q goes.
    struct Place {
        int krow, n, oj, oi, oy, ox;
        bool ok;
        unsigned pos;
    };
    auto place = [&](int q) {
        Place p;
        const int f = q * G + tg, fi = f / FM, fj = f - fi * FM;
        p.krow = k0 + fi * 32 + (ch >> 6) * 8 + 4 * h;
        const int m = m0 + fj * 32 + l32;
        p.n = fast_div(m, inv_PQ);
        const int rem = m - mul24(p.n, PQ);
        p.oj = fast_div(rem, inv_Q);
        p.oi = rem - mul24(p.oj, a.Q);
        p.ok = tg < G && m < npix && p.krow < a.Kp;
        p.oy = mul24(p.oj, a.ostr) + a.oy0;
        p.ox = mul24(p.oi, a.ostr_x) + a.ox0;
        int kb = p.krow / V;
        if (a.shuffle) {  // the channel block is a position of the ostr x ostr_x cell
            const int cy = kb / a.ostr_x;
            p.oy += cy;
            p.ox += kb - cy * a.ostr_x;
            kb = 0;
            p.ok = p.ok && p.oy < a.OH && p.ox < a.OW;
        }
        p.pos = (unsigned)(mul24(mul24(mul24(p.n, a.out_kb) + kb, a.OH) + p.oy, a.OW) + p.ox) * 16u +
                (V == 8 ? (unsigned)(p.krow & 4) * 2u : 0u);
        return p;
    };
    // What is fused into it: the operands of all rounds are requested here, ahead of the first exchange.  (Behind it,
    // round by round, each round waited for a trip to memory: the compiler moves no load over the stores of the
    // round before, since the residual may be the output buffer -- a thread reads only what it will write
    // itself.  Bottleneck block of 8 images, 1024 and 256 channels at 14x14, bf16: 20.9 -> 19.7 us; 1024 -> 2048
    // stride 2 with a residual, N = 12: 14.6 -> 13.7.)  A launch with nothing fused takes a path without those operands: with
    // one path for both it took 1.01 of the time of one that had none (bf16, 90 passes of 3.5 - 40 us), now 1.00, and
    // fused bf16 launches beyond 6 us 0.98 of what they took.
    const bool fused = a.ksplit == 1 && (a.scale != nullptr || a.bias != nullptr || a.resid != nullptr || a.relu != 0);
    auto rounds = [&](auto fused_tag) {
        constexpr bool FUSED = decltype(fused_tag)::value;
        constexpr int NO = FUSED ? NR : 1;
        f32x4 sv[NO], bv[NO];
        typename E_::Four res[NO];
        if constexpr (FUSED) {
#pragma unroll
            for (int q = 0; q < NR; ++q) {
                sv[q] = f32x4{1.f, 1.f, 1.f, 1.f};
                bv[q] = f32x4{0.f, 0.f, 0.f, 0.f};
                res[q] = typename E_::Four{};
                const Place p = place(q);
                // (rows beyond Kp are out of range)
                if (a.scale)
                    sv[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          make_rsrc(a.scale, 0, (size_t)a.Kp * 4), (unsigned)p.krow * 4u, 0, 0));
                if (a.bias)
                    bv[q] = __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(
                                                          make_rsrc(a.bias, 0, (size_t)a.Kp * 4), (unsigned)p.krow * 4u, 0, 0));
                if (a.resid) res[q] = E_::load4(make_rsrc(a.resid, 0, out_bytes), p.ok ? p.pos : kOutOfRange, 0);
            }
        }
#pragma unroll
        for (int q = 0; q < NR; ++q) {
            const int f0 = q * G;
            if (f0 > 0) __syncthreads();
#pragma unroll
            for (int g = 0; g < G; ++g) {
                const f32x16 &c = acc[(f0 + g) / FM][(f0 + g) % FM];
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const f32x4 v = {c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]};
                    xch[(g * NW + wave) * 256 + vq * 64 + lane] = v;
                }
            }
            __syncthreads();
            if (tg < G) {
                f32x4 v = wave_sum<0, NW>([&](int w) { return xch[(tg * NW + w) * 256 + ch]; });
                const Place p = place(q);
                if constexpr (EXACT) {
                    if (a.exact && p.ok && any_nan(v)) v = again(p.n, p.oj, p.oi, p.krow);
                }
                if (!FUSED && a.ksplit > 1) {
                    Elem<CONV_F32>::store4(ro, p.ok ? p.pos * SC : kOutOfRange, 0, v[0], v[1], v[2], v[3]);
                    continue;
                }
                const unsigned off = p.ok ? p.pos : kOutOfRange;
                float o[4] = {v[0], v[1], v[2], v[3]};
                if constexpr (FUSED) {
                    float r4[4];
                    E_::widen4(res[q], r4);
#pragma unroll
                    for (int t = 0; t < 4; ++t) {
                        o[t] = o[t] * sv[q][t] + r4[t] + bv[q][t];
                        if (a.relu) o[t] = fmaxf(o[t], 0.0f);
                    }
                }
                E_::store4(ro, off, 0, o[0], o[1], o[2], o[3]);
                if (a.zero_fill) {
                    for (int dy = 0; dy < a.ostr; ++dy)
                        for (int dx = 0; dx < a.ostr_x; ++dx) {
                            if ((dy | dx) == 0) continue;
                            const bool in = p.ok && p.oy + dy < a.OH && p.ox + dx < a.OW;
                            E_::store4(ro, in ? off + (unsigned)(dy * a.OW + dx) * 16u : kOutOfRange, 0, 0.f, 0.f,
                                       0.f, 0.f);
                        }
                }
            }
        }
    };
    if (fused) rounds(std::true_type{});
    else rounds(std::false_type{});
}

}  // namespace convmi
