// Implicit-GEMM direct convolution for results of few tiles: small minibatches, small images.
//
// The staged kernel (igemm_kernel.h) wants tiles of 64 x 512 or 128 x 224 results and walks the
// whole reduction of a tile in one workgroup; with a few thousand result pixels that is a
// handful of workgroups on 256 CUs, each a serial chain of up to 64 steps.  Here the chip is
// filled from the other side: a workgroup owns a small tile (FK*32 channels x FM*32 pixels) and
// its waves split the REDUCTION of that tile between them, each with the whole tile in
// its accumulators.  The waves' sums meet in LDS at the end, added pairwise (one fixed
// order), so one launch does it and no partial results go through memory.
//
// Operands go from memory straight into the registers the MFMAs take them from (a pixel's
// channel block and a weight row's channel block are 16 bytes each, consecutive lanes take
// consecutive pixels or rows): no LDS staging, no barrier in the main loop, so a wave only
// waits for its own loads, D steps after they were issued.  The taps of one channel-block
// pair are consecutive steps of a wave, so the pixels that neighbouring taps share come out of
// the CU's vector L1.
//
// What bounds it: the bytes that go through the vector L1, 64 per clock and CU; per step a
// wave loads FK + FM operands of 1 KiB and issues FK * FM MFMAs (bf16: 32 clocks each, fp32:
// 4 x 64 clocks), so a 2 x 2 tile can keep a bf16 matrix core half busy and an fp32 one fully.
// Larger results are better off sharing operands through LDS (see plan_igemm).
//
// Measured against the staged kernel with the reduction split over workgroups (forward, fp32 / bf16): 256 -> 256 3x3
// at 14x14, N = 1: 25 -> 8.6 / 11 -> 5.3 us, N = 8: 29 -> 24 / 13.5 -> 6.4; 512 -> 2048 1x1 at 7x7, N = 1: 15 -> 6.1 / 8.7 -> 3.9.
// (bf16 filters of seven and nine taps run on igemm_patch.hip, which reads their pixels once for all taps, where that is
// the faster one by estimate.)
#include <algorithm>

#include "igemm_exchange.h"

namespace convmi {

// FK x FM accumulator tiles per wave, NW waves that split the reduction, D steps in flight.
// EXACT: for layers that would else run on the untiled loops, which leave the taps outside the image
// out.  Here such a tap multiplies a weight by zero, which an infinite or NaN weight turns into NaN; a
// sum that is NaN is therefore formed again without them.
// GROUPS (fp32): a wave's steps are summed in groups of IgemmArgs::group rounds of D, each from zero, then
// added to the sum of the groups before.  One chain over a wave's share has the larger rounding error
// where the same result used to have its reduction split over more chains.  (It costs 1 - 14 %: 128 -> 128 3x3 at 28x28,
// N = 28, 68.5 us for 66.8; 512 -> 2048 1x1 at 7x7, N = 1, 6.4 for 6.0; 256 -> 1024 1x1 at 14x14, N = 15, 22.9 for 19.6.)
// FWD_WT (bf16, backward by data): the weights as the forward pass has them, through a ring of LDS of the wave's own and
// transposing reads, the tap flipped (as in igemm_patch.hip): no launch that transforms them first.  (1x1 backward passes on
// this kernel, N = 2 ... 192, three sets of tensors in turn: 0.90 of the time with the launch.)
template <int DT, int FK, int FM, int NW, int D, bool EXACT, bool GROUPS, bool FWD_WT = false>
__global__ __launch_bounds__(NW * 64, FK * FM <= 2 ? 4 : 2) void igemm_reg_kernel(const IgemmArgs a)
{
    using E_ = Elem<DT>;
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
    const float inv_PQ = a.inv_P, inv_Q = a.inv_TQ;  // (1 / (P*Q), 1 / Q in this kernel's plans)

    // Operand addresses.  The input's buffer starts pad_h rows and pad_w pixels before the
    // tensor, so that a lane's offset is its pixel's and the tap moves the scalar offset
    // only; taps outside the image never load (their lanes carry kOutOfRange).
    const long long shift = ((long long)a.pad_h * a.W + a.pad_w) * 16;
    const rsrc_t rsrc_in = make_rsrc(static_cast<const char *>(a.in) - shift, 0,
                                     (size_t)((long long)a.N * a.Cb * HW * 16 + shift));
    const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * RS * a.Kp * 16);
    unsigned b_off[FM], a_off[FK];
    int ih0[FM], iw0[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) {
        const int m = m0 + j * 32 + l32;
        const int n = fast_div(m, inv_PQ);
        const int rem = m - mul24(n, PQ);
        const int oj = fast_div(rem, inv_Q);
        const int oi = rem - mul24(oj, a.Q);
        const int y = mul24(oj, a.stride), x = mul24(oi, a.cstride);
        b_off[j] = (unsigned)(mul24(mul24(mul24(n, a.Cb) + h, a.H) + y, a.W) + x) * 16u;
        // (a pixel beyond the last one: no row is inside the image)
        ih0[j] = m < npix ? y - a.pad_h : 0x40000000;
        iw0[j] = x - a.pad_w;
    }
    // (the forward pass's weights: the lane's block of dI and channel of dO, in the order of the LDS)
    const int wquad = lane >> 4, wblk = (lane >> 2) & 3;
    const int kf = a.Cb * 8;  // ... and their rows
#pragma unroll
    for (int i = 0; i < FK; ++i) {
        if constexpr (FWD_WT) {
            const int blk = (k0 >> 3) + 4 * i + wblk;
            a_off[i] = blk < a.Kp >> 3 ? ((unsigned)blk * (unsigned)(RS * kf) + 4 * wquad + (lane & 3)) * 16u : kOutOfRange;
        } else {
            const int k = k0 + i * 32 + l32;
            a_off[i] = k < a.Kp ? (unsigned)(mul24(h, RS * a.Kp) + k) * 16u : kOutOfRange;
        }
    }
    unsigned char *const ring = lds + wave * (D * FK * 1024);

    // This wave's share of the reduction: steps [u0, u1), step u = (channel-block pair, r, s);
    // the lane halves take the two blocks of the pair.
    const int steps = ((a.Cb + 1) >> 1) * RS;
    const int sbeg = sp * a.st_per;
    const int nst = min(steps - sbeg, a.st_per);
    const int per = (nst + NW - 1) / NW;
    const int u0 = sbeg + min(wave * per, nst), u1 = sbeg + min(wave * per + per, nst);
    int cp = u0 / RS;
    int tap = u0 - cp * RS;
    int r = tap / a.S;
    int s = tap - r * a.S;
    int u = u0;  // next step to load

    u32x4 A[FWD_WT ? 1 : D][FK], B[D][FM];
    auto load = [&](u32x4(&av)[FK], u32x4(&bv)[FM], int slot) {
        // (past the wave's share, and the upper half of an odd last pair: zeros on both sides)
        const bool live = u < u1 && 2 * cp + h < a.Cb;
        const unsigned sa = (unsigned)(2 * cp * RS + r * a.S + s) * (unsigned)a.Kp * 16u;
        const unsigned sb = (unsigned)(2 * cp * HW + r * a.W + s) * 16u;
#pragma unroll
        for (int j = 0; j < FM; ++j) {
            const bool in = live && (unsigned)(ih0[j] + r) < (unsigned)a.H && (unsigned)(iw0[j] + s) < (unsigned)a.W;
            bv[j] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, in ? b_off[j] : kOutOfRange, u < u1 ? sb : 0u, 0);
        }
        if constexpr (FWD_WT) {
            const bool mine = u < u1 && 2 * cp + (wquad >> 1) < a.Cb;
            const unsigned sf = (unsigned)((RS - 1 - r * a.S - s) * kf + 16 * cp) * 16u;
#pragma unroll
            for (int i = 0; i < FK; ++i)
                load_to_lds_16(rsrc_wt, mine ? a_off[i] : kOutOfRange, u < u1 ? sf : 0u, ring + (slot * FK + i) * 1024);
        } else {
#pragma unroll
            for (int i = 0; i < FK; ++i)
                av[i] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, live ? a_off[i] : kOutOfRange, u < u1 ? sa : 0u, 0);
        }
        ++u;
        if (++s == a.S) {
            s = 0;
            if (++r == a.R) {
                r = 0;
                ++cp;
            }
        }
    };

    f32x16 acc[FK][FM];
#pragma unroll
    for (int i = 0; i < FK; ++i)
#pragma unroll
        for (int j = 0; j < FM; ++j)
#pragma unroll
            for (int t = 0; t < 16; ++t) acc[i][j][t] = 0.0f;
    auto multiply = [&](const u32x4(&av)[FK], const u32x4(&bv)[FM]) {
#pragma unroll
        for (int i = 0; i < FK; ++i)
#pragma unroll
            for (int j = 0; j < FM; ++j) E_::mma(av[i], bv[j], acc[i][j]);
    };

    if constexpr (FWD_WT) {
        static_assert(D >= 3 && DT == CONV_BF16, "a step's weights are read while the one before multiplies");
        // transposing reads: lanes 4*j + q of a group of 16 address 4 channels of dI of channel j of dO and receive
        // channels 0..3 of dO of their own channel; two reads make the 8 of a lane half
        const int q4 = lane & 3;
        const unsigned read_at = lds_address(ring) +
            (unsigned)(((8 * h + 2 * ((lane >> 4) & 1) + (q4 >> 1)) * 4 + ((lane >> 2) & 3)) * 16 + (q4 & 1) * 8);
        lds_u32x2 an[2 * FK];
        auto read_weights = [&](auto sc) {
            constexpr int slot = decltype(sc)::value;
            static_for<0, FK>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                an[2 * i] = lds_read_tr16_b64_untracked<(slot * FK + i) * 1024>(read_at);
                an[2 * i + 1] = lds_read_tr16_b64_untracked<(slot * FK + i) * 1024 + 256>(read_at);
            });
        };
        auto weights_landed = [&]() {
            __builtin_amdgcn_sched_barrier(0);
            lds_reads_pending<0>();
#pragma unroll
            for (int o = 0; o < 2 * FK; ++o) lds_read_landed(an[o]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < FK; ++i) A[0][i] = u32x4{an[2 * i][0], an[2 * i][1], an[2 * i + 1][0], an[2 * i + 1][1]};
        };
        if (u0 < u1) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                load(A[0], B[d], d);
                __builtin_amdgcn_sched_barrier(0);
            }
            asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * (FK + FM)) : "memory");
            __builtin_amdgcn_sched_barrier(0);
            read_weights(std::integral_constant<int, 0>{});
            weights_landed();
            for (int g = u0; g < u1; g += D)
                static_for<0, D>([&](auto dc) {
                    constexpr int d = decltype(dc)::value;
                    // (a step past the share: zeros on both sides) the loads of the step after this one have landed
                    __builtin_amdgcn_sched_barrier(0);
                    asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 2) * (FK + FM)) : "memory");
                    __builtin_amdgcn_sched_barrier(0);
                    read_weights(std::integral_constant<int, (d + 1) % D>{});
                    multiply(A[0], B[d]);
                    weights_landed();
                    load(A[0], B[d], d);
                });
        }
        wait_all_memory();  // (the rings are done with before the sums take their place)
        __syncthreads();
    } else if (u0 < u1) {
#pragma unroll
        for (int d = 0; d < D; ++d) load(A[d], B[d], d);
        // (loads past u1 ask for nothing: their lanes are out of range)
        // rounds of D steps from g on, up to `end`: the loads of the next round go out behind each step
        auto rounds = [&](int &g, int end) {
            for (; g < end; g += D) {
#pragma unroll
                for (int d = 0; d < D; ++d) {
                    multiply(A[d], B[d]);
                    load(A[d], B[d], d);
                    __builtin_amdgcn_sched_barrier(0);
                }
            }
        };
        int g = u0;
        f32x16 sum[GROUPS ? FK : 1][GROUPS ? FM : 1];  // of the groups so far
        auto end_group = [&]() {
            if constexpr (GROUPS) {
#pragma unroll
                for (int i = 0; i < FK; ++i)
#pragma unroll
                    for (int j = 0; j < FM; ++j) {
                        add_here(sum[i][j], acc[i][j]);
                        acc[i][j] = f32x16{};
                    }
            }
        };
        if constexpr (GROUPS) {
#pragma unroll
            for (int i = 0; i < FK; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) sum[i][j] = f32x16{};
            for (; g + a.group * D < u1; end_group()) rounds(g, g + a.group * D);
        }
        rounds(g, u1 - D);
        // the last 1 .. D steps, already in registers
#pragma unroll
        for (int d = 0; d < D; ++d)
            if (g + d < u1) multiply(A[d], B[d]);
        if constexpr (GROUPS) {
            end_group();
#pragma unroll
            for (int i = 0; i < FK; ++i)
#pragma unroll
                for (int j = 0; j < FM; ++j) acc[i][j] = sum[i][j];
        }
    }
    add_and_store<DT, FK, FM, NW, EXACT>(a, acc, lds, k0, m0, sp, [&](int n, int oj, int oi, int krow) {
        return sum_inside_image<DT, 2>(a, n, oj, oi, krow, sbeg, sbeg + nst);
    });
}

constexpr int kWeightRing = 4;  // steps of the ring of the forward pass's weights
template <int DT, int FK, int FM, int NW>
constexpr igemm_fn_t fwd_wt_kernel()
{
    if constexpr (DT == CONV_BF16) return igemm_reg_kernel<DT, FK, FM, NW, kWeightRing, false, false, true>;
    else return nullptr;
}
#define REG_ENTRY(DT, FK, FM, NW, D) \
    {DT, FK, FM, NW, D, igemm_reg_kernel<DT, FK, FM, NW, D, false, false>, \
     igemm_reg_kernel<DT, FK, FM, NW, D, true, false>, igemm_reg_kernel<DT, FK, FM, NW, D, false, DT == CONV_F32>, fwd_wt_kernel<DT, FK, FM, NW>()}
static const struct RegEntry {
    int dtype, fk, fm, nw, depth;
    igemm_fn_t fn, exact_fn, groups_fn, fwd_wt_fn;
} g_reg[] = {
    REG_ENTRY(CONV_F32, 1, 1, 4, 4),  REG_ENTRY(CONV_F32, 1, 1, 8, 3),  REG_ENTRY(CONV_F32, 2, 1, 8, 3),
    REG_ENTRY(CONV_F32, 1, 2, 4, 3),  REG_ENTRY(CONV_F32, 2, 2, 4, 3),
    REG_ENTRY(CONV_BF16, 1, 1, 4, 3), REG_ENTRY(CONV_BF16, 1, 1, 8, 3), REG_ENTRY(CONV_BF16, 2, 1, 8, 2),
    REG_ENTRY(CONV_BF16, 2, 2, 4, 3),
};
// (dropped after measuring 42 layers at N = 1 ... 256 under every variant: 16 waves, 2 x 4 fragments,
// 1 x 2 and 2 x 2 fragments on eight waves: never more than 2 % ahead of the ones above.  More steps in
// flight: 5 to 12 cost 3 - 30 % against 2 to 4 in bf16, 1 - 5 % in fp32: waves per SIMD cover the loads
// better than a wave's own depth does.)

int igemm_reg_depth(int dtype, int fk, int fm, int nw)
{
    for (const RegEntry &e : g_reg)
        if (e.dtype == dtype && e.fk == fk && e.fm == fm && e.nw == nw) return e.depth;
    return 0;
}

size_t igemm_reg_lds_bytes(int fk, int fm, int nw, bool fwd_wt)
{
    const int per_round = std::min(nw / 4, fk * fm);
    return std::max((size_t)per_round * nw * 4096, fwd_wt ? (size_t)nw * kWeightRing * fk * 1024 : 0);
}

hipError_t launch_igemm_reg(const IgemmVariant &v, const IgemmArgs &a, int grid, hipStream_t stream)
{
    for (const RegEntry &e : g_reg) {
        if (e.dtype != v.dtype || e.fk != v.fk || e.fm != v.fm || e.nw != v.wk) continue;
        const size_t lds = igemm_reg_lds_bytes(e.fk, e.fm, e.nw, a.fwd_wt != 0);
        const igemm_fn_t fn = a.fwd_wt ? e.fwd_wt_fn : a.exact ? e.exact_fn : a.group > 0 ? e.groups_fn : e.fn;
        if (!fn) return hipErrorInvalidDeviceFunction;
        if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(fn), lds); err != hipSuccess)
            return err;
        hipLaunchKernelGGL(fn, dim3(grid), dim3(e.nw * 64), lds, stream, a);
        return hipGetLastError();
    }
    return hipErrorInvalidDeviceFunction;
}

}  // namespace convmi
