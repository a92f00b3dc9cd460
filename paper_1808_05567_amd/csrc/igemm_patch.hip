// Implicit-GEMM direct convolution for results of few tiles under a filter of several taps, bf16: the
// register-operand kernel (igemm_reg.hip) with the pixels in LDS.
//
// What bounds that kernel there are the bytes that go through a CU's vector L1, 64 a clock: per tap a wave
// loads FK weight operands and FM pixel operands of 1 KiB for FK * FM MFMAs of 32 clocks, and the pixels are the
// same for every tap but for a shift (512 -> 512 3x3 at 7x7, N = 32: 16.1 us; 14.2 without its MFMAs, 9.5 without its
// loads).  Here a wave brings the pixels of its tile and the halo around them, two channel blocks at a time, into a
// patch of LDS of its own, once for all taps; the weights, which no two taps share, still go straight
// into registers.  As there, the waves split the reduction (wave w takes the pairs of channel blocks w, w + NW, ...),
// nothing in the main loop waits for another wave, and the sums meet in LDS at the end.
//
// A patch is the run of the input's flat pixel list (image, row, column) from the first tap of the tile's first
// pixel to the last tap of its last one, so it may cross rows and images; every lane keeps the position of its
// pixel for every tap, and where a tap falls outside the image that of a chunk of zeros.  Lanes take
// consecutive pixels, i.e. consecutive 16-byte chunks: no bank conflicts at stride 1.
//
// FWD_WT (backward by data): the weights as the forward pass has them, [channel block of dI][tap][channel of dO][8]. A
// fragment of a tap is 16 channels of dO of four blocks, 1 KiB, which a wave brings into a ring of LDS of its own and
// reads back transposed, the tap flipped: the launch that would transform all weights first is left out.
//
// What bounds it now: the weights through the vector L1, FK KiB a tap and wave, or where a wave has one or two
// pairs of channel blocks the trip of their first loads.  Measured against what these layers ran on before (three
// sets of tensors in turn): 512 -> 512 3x3 at 7x7, N = 32, forward 16.2 -> 12.8 us, backward 23.1 -> 13.4 (6.4 of
// it the transform launch and the cold weights behind it); N = 1 7.9 -> 6.2 and 13.2 -> 7.5; 604 -> 76 3x3 at 9x8,
// N = 64, forward 18.5 -> 10.3; 256 -> 256 3x3 at 14x14, N = 16, 10.5 -> 8.7 and 13.6 -> 9.5; 192 -> 192 1x7 at 17x17,
// N = 16, forward 8.1 -> 7.0.  560 forward and backward passes of such layers, N = 1 ... 256, on average 0.96 and 0.82.
#include <algorithm>

#include "igemm_exchange.h"

namespace convmi {

// NTAP taps (R x S, any way), FK x FM accumulator tiles per wave, NW waves that split the reduction, the weights
// of D taps in flight (D divides NTAP, so that the registers of a tap are known at compile time).
template <int DT, int NTAP, int FK, int FM, int NW, int D, bool FWD_WT>
__global__ __launch_bounds__(NW * 64, FK * FM <= 2 ? 4 : 2) void igemm_patch_kernel(const IgemmArgs a)
{
    using E_ = Elem<DT>;
    constexpr int TK = FK * 32, TM = FM * 32;
    static_assert(FWD_WT ? NTAP > D : NTAP % D == 0, "whole rounds of the weight registers; the ring is shorter than a patch lives");
    constexpr int MAXL = kPatchLoads;  // wave-level loads per channel block

    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;

    int kt, mt, sp;
    if (!small_tile(a, blockIdx.x, kt, mt, sp)) return;
    const int k0 = kt * TK, m0 = mt * TM;
    const int PQ = a.P * a.Q, npix = a.N * PQ, HW = a.H * a.W;
    const float inv_PQ = a.inv_P, inv_Q = a.inv_TQ, inv_HW = a.inv_Hs;

    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * NTAP * a.Kp * 16);
    const int pairs = (a.Cb + 1) >> 1;

    // The pixel of the flat input list under tap (0, 0) of result pixel m (it may lie before the image).
    auto first_tap = [&](int m, int &y, int &x) {
        const int n = fast_div(m, inv_PQ);
        const int rem = m - mul24(n, PQ);
        const int oj = fast_div(rem, inv_Q);
        y = mul24(oj, a.stride) - a.pad_h;
        x = mul24(rem - mul24(oj, a.Q), a.cstride) - a.pad_w;
        return mul24(n, HW) + mul24(y, a.W) + x;
    };
    int y0, x0;
    const int v0 = __builtin_amdgcn_readfirstlane(first_tap(m0, y0, x0));

    // This wave's patch buffers: two channel blocks of PLS positions each and a chunk of zeros.
    const int bufbytes = 2 * a.PLS * 16 + 16;
    unsigned char *const patch = lds + wave * (2 * bufbytes + (FWD_WT ? D * FK * 1024 : 0));
    if (lane < 2) *reinterpret_cast<u32x4 *>(patch + lane * bufbytes + 2 * a.PLS * 16) = u32x4{0, 0, 0, 0};
    unsigned p_off[MAXL];  // where the lane's positions lie in the input (channel block 0)
#pragma unroll
    for (int l = 0; l < MAXL; ++l) {
        const int v = v0 + l * 64 + lane;
        const int n = fast_div(max(v, 0), inv_HW);
        p_off[l] = (unsigned)v < (unsigned)(a.N * HW) ? (unsigned)(mul24(mul24(n, a.Cb), HW) + (v - mul24(n, HW))) * 16u
                                                      : kOutOfRange;
    }
    auto load_patch = [&](int cp, int buf) {
#pragma unroll
        for (int l = 0; l < MAXL; ++l)
            if (l * 64 < a.PLS) {
#pragma unroll
                for (int b = 0; b < 2; ++b)  // (the second block of an odd last pair: zeros)
                    load_to_lds_16(rsrc_in, 2 * cp + b < a.Cb ? p_off[l] : kOutOfRange,
                                   (unsigned)((2 * cp + b) * HW) * 16u, patch + buf * bufbytes + (b * a.PLS + l * 64) * 16);
            }
    };

    // Position of the lane's pixels in the patch for every tap, as an offset from the patch buffer.
    unsigned b_pos[NTAP][FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int m = m0 + j * 32 + l32;
        int y, x;
        const int p = first_tap(m, y, x) - v0;
        int r = 0, s = 0;
#pragma unroll
        for (int t = 0; t < NTAP; ++t) {
            const bool in = m < npix && (unsigned)(y + r) < (unsigned)a.H && (unsigned)(x + s) < (unsigned)a.W;
            b_pos[t][j] = (unsigned)(in ? h * a.PLS + p + r * a.W + s : 2 * a.PLS) * 16u;
            if (++s == a.S) {
                s = 0;
                ++r;
            }
        }
    }
    // Weights: a lane's row and channel block; or, as the forward pass has them, its block of dI and channel of dO, in
    // the order of the LDS (quads of four channels of dO, the quad's four blocks side by side).
    const int wquad = lane >> 4, wblk = (lane >> 2) & 3;
    unsigned a_off[FK];
#pragma unroll
    for (int i = 0; i < FK; ++i) {
        if constexpr (FWD_WT) {
            const int blk = (k0 >> 3) + 4 * i + wblk;
            a_off[i] = blk < a.Kp >> 3 ? ((unsigned)blk * (unsigned)(NTAP * a.Cb * 8) + 4 * wquad + (lane & 3)) * 16u : kOutOfRange;
        } else {
            const int k = k0 + i * 32 + l32;
            a_off[i] = k < a.Kp ? (unsigned)(mul24(h, NTAP * a.Kp) + k) * 16u : kOutOfRange;
        }
    }

    f32x16 acc[FK][FM];
#pragma unroll
    for (int i = 0; i < FK; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j) acc[i][j] = f32x16{};

    u32x4 A[FWD_WT ? 1 : D][FK], bc[FM];
    // weights of tap t of pair cp (beyond the wave's last pair, and the upper half of an odd last one: zeros)
    auto load_weights = [&](u32x4(&av)[FK], int cp, int t) {
        const bool live = cp < pairs;  // (wave-uniform)
        const unsigned at = live ? (unsigned)((2 * cp * NTAP + t) * a.Kp) * 16u : 0u;
        const bool mine = live && 2 * cp + h < a.Cb;
#pragma unroll
        for (int i = 0; i < FK; ++i)
            av[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, mine ? a_off[i] : kOutOfRange, at, 0);
    };
    auto read_pixels = [&](u32x4(&b)[FM], int t, int buf) {
#pragma unroll
        for (int j = 0; j < FM; ++j) b[j] = *reinterpret_cast<const u32x4 *>(patch + buf * bufbytes + b_pos[t][j]);
    };
    // The wave's loads complete in order: with at most the weights on their way that were asked for behind the patch,
    // those of the D newest taps or of all but the last, the patch has landed.
    auto patch_landed = [&]() {
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D < NTAP ? D : NTAP - 1) * FK) : "memory");
        __builtin_amdgcn_sched_barrier(0);
    };

    int cp = wave, buf = 0;
    if constexpr (FWD_WT) {
        unsigned char *const ring = patch + 2 * bufbytes;
        // transposing reads: lanes 4*j + q of a group of 16 address 4 channels of dI of channel j of dO and receive
        // channels 0..3 of dO of their own channel; two reads make the 8 of a lane half
        const int q4 = lane & 3;
        const unsigned read_at = lds_address(ring) +
            (unsigned)(((8 * h + 2 * ((lane >> 4) & 1) + (q4 >> 1)) * 4 + ((lane >> 2) & 3)) * 16 + (q4 & 1) * 8);
        auto load_tap = [&](int pair, int t, int slot) {
            const bool mine = pair < pairs && 2 * pair + (wquad >> 1) < a.Cb;
            const unsigned at = pair < pairs ? (unsigned)((NTAP - 1 - t) * a.Cb * 8 + 16 * pair) * 16u : 0u;
#pragma unroll
            for (int i = 0; i < FK; ++i)
                load_to_lds_16(rsrc_wt, mine ? a_off[i] : kOutOfRange, at, ring + (slot * FK + i) * 1024);
        };
        lds_u32x2 an[2 * FK];
        auto read_tap = [&](int slot) {
            const unsigned at = read_at + (unsigned)(slot * FK * 1024);
            static_for<0, FK>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                an[2 * i] = lds_read_tr16_b64_untracked<i * 1024>(at);
                an[2 * i + 1] = lds_read_tr16_b64_untracked<i * 1024 + 256>(at);
            });
        };
        u32x4 ac[FK];
        auto tap_landed = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            lds_reads_pending<0>();
#pragma unroll
            for (int o = 0; o < 2 * FK; ++o) lds_read_landed(an[o]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < FK; ++i) ac[i] = u32x4{an[2 * i][0], an[2 * i][1], an[2 * i + 1][0], an[2 * i + 1][1]};
        };
        // All but the loads of the D - 1 newest taps have landed, and but for `patch_loads` asked for among them.
        auto loads_landed = [&](int patch_loads) {
            __builtin_amdgcn_sched_barrier(0);
            if (patch_loads == 0) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * FK) : "memory");
            else if (patch_loads == 2) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * FK + 2) : "memory");
            else if (patch_loads == 4) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * FK + 4) : "memory");
            else if (patch_loads == 6) asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * FK + 6) : "memory");
            else asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * FK + 8) : "memory");
            __builtin_amdgcn_sched_barrier(0);
        };
        static_assert(MAXL == 4, "the counts above");
        if (cp < pairs) {
            load_patch(cp, 0);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int d = 0; d < D; ++d) load_tap(cp, d, d);
            loads_landed(0);
            read_tap(0);
            read_pixels(bc, 0, 0);
            tap_landed();
            load_tap(cp, D, 0);
            int slot = 1 % D;  // of the next tap
            for (; cp < pairs; cp += NW, buf ^= 1) {
                const bool more = cp + NW < pairs;  // (wave-uniform)
                if (more) load_patch(cp + NW, buf ^ 1);
                const int patch_loads = more ? a.PLS / 32 : 0;
#pragma unroll
                for (int t = 0; t < NTAP; ++t) {
                    // the next tap's weights and pixels are read while this one's MFMAs issue
                    u32x4 bn[FM];
                    // (the next patch was asked for behind tap D, so the waits for the taps up to there let it be)
                    loads_landed(t + 1 <= D ? patch_loads : 0);
                    read_tap(slot);
                    read_pixels(bn, t + 1 < NTAP ? t + 1 : 0, t + 1 < NTAP ? buf : buf ^ 1);
                    __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                    for (int i = 0; i < FK; ++i)
#pragma unroll
                        for (int j = 0; j < FM; ++j) E_::mma(ac[i], bc[j], acc[i][j]);
                    tap_landed();
                    const int u = t + 1 + D;
                    load_tap(u < NTAP ? cp : cp + NW, u < NTAP ? u : u - NTAP, slot);
                    slot = slot + 1 < D ? slot + 1 : 0;
#pragma unroll
                    for (int j = 0; j < FM; ++j) bc[j] = bn[j];
                }
            }
        }
    } else if (cp < pairs) {
        load_patch(cp, 0);
        __builtin_amdgcn_sched_barrier(0);
#pragma unroll
        for (int d = 0; d < D; ++d) load_weights(A[d], cp, d);
        patch_landed();
        read_pixels(bc, 0, 0);
        for (; cp < pairs; cp += NW, buf ^= 1) {
            const bool more = cp + NW < pairs;  // (wave-uniform)
            if (more) load_patch(cp + NW, buf ^ 1);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int t = 0; t < NTAP; ++t) {
                // the next tap's pixels are read while this one's MFMAs issue
                u32x4 bn[FM];
                if (t + 1 < NTAP) {
                    read_pixels(bn, t + 1, buf);
                } else if (more) {
                    patch_landed();
                    read_pixels(bn, 0, buf ^ 1);
                } else {
#pragma unroll
                    for (int j = 0; j < FM; ++j) bn[j] = bc[j];
                }
#pragma unroll
                for (int i = 0; i < FK; ++i)
#pragma unroll
                    for (int j = 0; j < FM; ++j) E_::mma(A[t % D][i], bc[j], acc[i][j]);
                load_weights(A[t % D], t + D < NTAP ? cp : cp + NW, t + D < NTAP ? t + D : t + D - NTAP);
                __builtin_amdgcn_sched_barrier(0);
#pragma unroll
                for (int j = 0; j < FM; ++j) bc[j] = bn[j];
            }
        }
    }
    // (the patches are done with before the sums take their place)
    wait_all_memory();
    __syncthreads();
    add_and_store<DT, FK, FM, NW, false>(a, acc, lds, k0, m0, sp, [](int, int, int, int) { return f32x4{}; });
}

constexpr int kPatchRing = 3;  // taps of the ring of weights
// (measured as well: nine taps' weights in flight, 0.95 - 0.98 on four waves with one channel fragment and 1.0 - 1.5 else;
// seven taps with one in flight 1.0 - 1.24; 25 taps, 1.0 - 2.6 of the staged kernel)
#define PATCH_ENTRY(NTAP, FK, FM, NW, D) \
    {CONV_BF16, NTAP, FK, FM, NW, igemm_patch_kernel<CONV_BF16, NTAP, FK, FM, NW, D, false>, \
     igemm_patch_kernel<CONV_BF16, NTAP, FK, FM, NW, kPatchRing, true>}
static const struct PatchEntry {
    int dtype, ntap, fk, fm, nw;
    igemm_fn_t fn, fwd_wt_fn;
} g_patch[] = {
    PATCH_ENTRY(9, 1, 1, 8, 3), PATCH_ENTRY(9, 2, 1, 8, 3), PATCH_ENTRY(9, 1, 2, 8, 3), PATCH_ENTRY(9, 1, 2, 4, 9),
    PATCH_ENTRY(9, 2, 2, 4, 3), PATCH_ENTRY(9, 2, 2, 8, 3), PATCH_ENTRY(9, 1, 4, 4, 9), PATCH_ENTRY(9, 2, 4, 4, 3),
    PATCH_ENTRY(9, 1, 4, 8, 3),
    PATCH_ENTRY(7, 1, 1, 8, 7), PATCH_ENTRY(7, 2, 1, 8, 7), PATCH_ENTRY(7, 1, 2, 8, 7), PATCH_ENTRY(7, 1, 2, 4, 7),
    PATCH_ENTRY(7, 2, 2, 4, 7), PATCH_ENTRY(7, 2, 2, 8, 7), PATCH_ENTRY(7, 1, 4, 4, 7), PATCH_ENTRY(7, 2, 4, 4, 7),
    PATCH_ENTRY(7, 1, 4, 8, 7),
};

static const PatchEntry *find_patch(int dtype, int ntap, int fk, int fm, int nw)
{
    for (const PatchEntry &e : g_patch)
        if (e.dtype == dtype && e.ntap == ntap && e.fk == fk && e.fm == fm && e.nw == nw) return &e;
    return nullptr;
}

bool igemm_patch_exists(int dtype, int ntap, int fk, int fm, int nw) { return find_patch(dtype, ntap, fk, fm, nw) != nullptr; }

size_t igemm_patch_lds_bytes(int fk, int fm, int nw, int pls, bool fwd_wt)
{
    return std::max((size_t)nw * (2 * (2 * (size_t)pls * 16 + 16) + (fwd_wt ? kPatchRing * fk * 1024 : 0)),
                    igemm_reg_lds_bytes(fk, fm, nw, false));
}

hipError_t launch_igemm_patch(const IgemmVariant &v, const IgemmArgs &a, int grid, hipStream_t stream)
{
    const PatchEntry *e = find_patch(v.dtype, a.R * a.S, v.fk, v.fm, v.wk);
    if (!e) return hipErrorInvalidDeviceFunction;
    const size_t lds = igemm_patch_lds_bytes(e->fk, e->fm, e->nw, a.PLS, a.fwd_wt != 0);
    const igemm_fn_t fn = a.fwd_wt ? e->fwd_wt_fn : e->fn;
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(fn), lds); err != hipSuccess) return err;
    hipLaunchKernelGGL(fn, dim3(grid), dim3(e->nw * 64), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
