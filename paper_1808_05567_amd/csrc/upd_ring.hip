// Weight-gradient update (Algorithm 8 of the paper) for filters with 1, 3, 5 or 7 columns, any
// number of rows, any stride, pads per axis, both types.
//
//   dW[k,c,r,s] = sum over (n,oj,oi) of I[n,c,oj*stride-pad_h+r,oi*stride-pad_w+s] * dO[n,k,oj,oi]
//
// The band kernels give a workgroup a 64 x 64 to 256 x 256 block of dW (all taps of it) and fill
// the chip by splitting the pixel range; every split writes its block as an fp32 partial copy
// and a second launch adds the copies.  Where the pixels are few, those copies ARE the work:
// 256 workgroups x 295 KB for a bf16 3x3 layer of 128+ channels, 75 MB there and back whatever the
// minibatch (N = 8: 25 us + 7 us for 3 us of arithmetic).  Here a workgroup owns a small block (FC*32 input
// channels x FK*32 output channels x the S taps of ONE filter row), so that the blocks
// themselves fill the chip, and its waves split the pixels of the block between them; their
// sums meet in LDS, pairwise.  Few or no partial copies are left, and with one split
// the kernel writes dW itself.
//
// Operands: a stage is PXS pixels of the flat list (n, oj, oi), sixteen in bf16 (one MFMA's reduction) and
// eight in fp32 (four MFMAs'); wave w takes stages w, w + NW, ..., so that the waves of a workgroup read
// the same cache lines.  Per stage a wave loads 1 KiB for every operand -- one per tap and 32-channel
// fragment of the input, one per fragment of dO -- straight into a ring of D patches of LDS of its own
// (padding, the image's edges and the list's end are lanes whose offset is out of range and arrive as
// zeros), so there is no barrier in the main loop: a wave waits for its own loads, D - 1 stages after
// they went out.  Within a patch the lanes take runs of 4 pixels of a channel block (64 bytes, one
// request) and the runs of the blocks that an operand read touches lie side by side, so that the
// reads are free of bank conflicts (fp32: two lanes to a bank).  fp32 reads a float per lane; bf16 reads
// with the transposing read, 8 pixels of one channel per lane.
//
// What bounds it: per stage S*FC + FK KiB through the vector L1 into LDS, and out of LDS again, for
// S*FC*FK MFMAs (x 4 in fp32: there the matrix core, 80 - 85 % of its rate).  The neighbouring taps' and
// the next filter row's pixels are the same lines, which the L1 and the XCD's L2 hold; but a line that
// comes from HBM is waited for by everyone who shares it, and the ring holds two stages: with
// tensors far beyond the last-level cache the bf16 1x1 layers are better off in the large blocks (planner).
// Measured against the kernels these layers ran on before (whole update, reduce launch included; three sets of
// tensors in turn), fp32 / bf16: 256 -> 256 3x3 at 14x14, N = 8: 35 -> 30 / 20 -> 9 us, N = 32: 81 -> 72 /
// 33 -> 19, N = 128: 264 -> 249 / 54 -> 38; 1024 -> 256 1x1 at 14x14, N = 32: 62 -> 37 / 16 -> 12; 288 -> 384 3x3
// stride 2 at 35x35, N = 32: 268 -> 173 / 57 -> 45; 160 -> 192 7x1 at 17x17, N = 128: 249 -> 169 / 59 -> 37.  (A first
// version gathered into registers -- in fp32 a float per lane, 24 clocks of the L1 for each: 296 us
// where this one takes 249; in bf16 through LDS writes with one stage in flight: 54 us for 38.)
#include <algorithm>

#include "igemm_kernel.h"

namespace convmi {

// S taps of a filter row, FC x FK accumulator tiles per tap, NW waves, a ring of D stages each.
// SUM: how a wave adds up its pixels.  0: in one chain.  1: in groups of UpdArgs::group rounds of D stages,
// each summed from zero, then added to the sum of the groups before.  2 (fp32): a stage's eight
// pixels from zero, then added.  One chain has the larger rounding error where the wave has
// more pixels than a wave of the kernel that this one replaces (the planner's upd_sum_error): in fp32
// up to twice the relative error.  1 takes a second set of accumulators, 2 only one or two tiles.
template <int DT, int S, int FC, int FK, int NW, int D, int SUM>
__global__ __launch_bounds__(NW * 64, SUM == 1 && S * FC * FK <= 3 ? 4 : 2) void
upd_ring_kernel(const UpdArgs a)
{
    constexpr bool BF = DT == CONV_BF16;
    constexpr int V = BF ? 8 : 4;
    constexpr int PXS = BF ? 16 : 8;
    constexpr int NA = S * FC, NO = NA + FK;  // operands of a stage: (tap, fragment) of the input, then dO
    constexpr int NF = NA * FK;               // accumulator tiles
    constexpr int NB = 32 / V;                // channel blocks of a fragment
    constexpr int G = NW / 4;                 // tiles summed per round (a thread per chunk)

    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    f32x4 *const xch = reinterpret_cast<f32x4 *>(lds);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;

    // split slowest: the blocks of a pixel range run side by side and share its lines in the L2
    const int bid = blockIdx.x;
    int lin = (bid & 7) * a.per_xcd + (bid >> 3);
    if (lin >= a.total) return;
    const int blocks = a.n_ct * a.n_kt * a.R;
    const int split = lin / blocks;
    lin -= split * blocks;
    const int kt = lin % a.n_kt;
    lin /= a.n_kt;
    const int ct = lin % a.n_ct;
    const int r = lin / a.n_ct;
    const int c0 = ct * FC * 32, k0 = kt * FK * 32;

    const int PQ = a.P * a.Q, npix = a.N * PQ, HW = a.H * a.W;
    const float inv_PQ = 1.0f / (float)PQ, inv_Q = 1.0f / (float)a.Q;
    const int g0 = split * a.rows_per_split;  // (here: pixels per split)
    const int g1 = min(npix, g0 + a.rows_per_split);

    // The input's buffer starts pad rows and pad_w pixels before the tensor (less r rows: this
    // launch's filter row), so that a pixel's offset is non-negative; lanes whose pixel lies
    // outside the image carry kOutOfRange.
    const long long shift = ((long long)a.pad * a.W + a.pad_w) * 16;
    const rsrc_t rsrc_in = make_rsrc(static_cast<const char *>(a.in) - shift, 0,
                                     (size_t)((long long)a.N * a.Cb * HW * 16 + shift));
    const rsrc_t rsrc_out = make_rsrc(a.dout, 0, (size_t)a.N * a.Kb * PQ * 16);
    // Lane -> (run of 4 pixels, channel block, pixel of the run): the runs of one pixel quad are
    // NB consecutive groups of 4 lanes, a block each.
    const int lblk = (lane >> 2) % NB;
    const int lpix = (lane >> 2) / NB * 4 + (lane & 3);
    unsigned in_ch[FC], out_ch[FK];  // channel part of the lane's offsets
#pragma unroll
    for (int i = 0; i < FC; ++i) {
        const int blk = c0 / V + NB * i + lblk;
        in_ch[i] = blk < a.Cb ? (unsigned)blk * (unsigned)HW * 16u : kOutOfRange;
    }
#pragma unroll
    for (int i = 0; i < FK; ++i) {
        const int blk = k0 / V + NB * i + lblk;
        out_ch[i] = blk < a.Kb ? (unsigned)blk * (unsigned)PQ * 16u : kOutOfRange;
    }

    unsigned char *const ring = lds + wave * (D * NO * 1024);
    int m = g0 + wave * PXS + lpix;  // the lane's pixel of the next stage to load
    auto load = [&](int slot) {
        unsigned char *const p = ring + slot * (NO * 1024);
        const int n = fast_div(m, inv_PQ);
        const int rem = m - mul24(n, PQ);
        const int oj = fast_div(rem, inv_Q);
        const int oi = rem - mul24(oj, a.Q);
        const int y = mul24(oj, a.stride), x = mul24(oi, a.stride);
        const bool live = m < g1;
        const bool row = live && (unsigned)(y - a.pad + r) < (unsigned)a.H;
        const unsigned in_pix = (unsigned)(mul24(mul24(n, a.Cb), HW) + mul24(y, a.W) + x) * 16u;
        const unsigned out_pix = (unsigned)(mul24(mul24(n, a.Kb), PQ) + rem) * 16u;
#pragma unroll
        for (int s = 0; s < S; ++s) {
            const bool in = row && (unsigned)(x - a.pad_w + s) < (unsigned)a.W;
#pragma unroll
            for (int i = 0; i < FC; ++i)
                load_to_lds_16(rsrc_in, in && in_ch[i] != kOutOfRange ? in_ch[i] + in_pix : kOutOfRange,
                               (unsigned)(r * a.W + s) * 16u, p + (s * FC + i) * 1024);
        }
#pragma unroll
        for (int i = 0; i < FK; ++i)
            load_to_lds_16(rsrc_out, live && out_ch[i] != kOutOfRange ? out_ch[i] + out_pix : kOutOfRange, 0u,
                           p + (NA + i) * 1024);
        m += NW * PXS;
    };

    f32x16 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[f][t] = 0.0f;

    // Operand reads.  bf16, transposing: lanes 4*j + q of a group of 16 address 4 channels of pixel j and
    // receive pixels 0..3 of their own channel; two reads make the 8 pixels of a lane half.
    // fp32: the lane's channel of pixel 2*q + h.
    const int q4 = lane & 3;
    const int r_lane = BF ? ((2 * h * NB + 2 * ((lane >> 4) & 1) + (q4 >> 1)) * 4 + ((lane >> 2) & 3)) * 16 + (q4 & 1) * 8
                          : (l32 >> 2) * 64 + h * 16 + (l32 & 3) * 4;
    const int steps = (g1 - g0 + NW * PXS - 1) / (NW * PXS);
#pragma unroll
    for (int d = 0; d < D; ++d) load(d);
    f32x16 sum[SUM == 1 ? NF : 1];  // of the groups so far
    if constexpr (SUM == 1) {
#pragma unroll
        for (int f = 0; f < NF; ++f) sum[f] = f32x16{};
    }
    for (int u = 0; u < steps;) {
        // (whole rounds of D stages: what lies past the range's end arrives as zeros)
        for (const int end = SUM == 1 ? min(steps, u + a.group * D) : steps; u < end; u += D) {
#pragma unroll
            for (int d = 0; d < D; ++d) {
                // this stage's loads have landed; the D - 1 later ones may be on their way
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((D - 1) * NO) : "memory");
                __builtin_amdgcn_sched_barrier(0);
                if constexpr (BF) {
                    const unsigned p = lds_address(ring + d * (NO * 1024)) + (unsigned)r_lane;
                    lds_u32x2 t[2 * NO];
                    static_for<0, NO>([&](auto oc) {
                        constexpr int o = decltype(oc)::value;
                        t[2 * o] = lds_read_tr16_b64_untracked<o * 1024>(p);
                        t[2 * o + 1] = lds_read_tr16_b64_untracked<o * 1024 + NB * 64>(p);
                    });
                    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
#pragma unroll
                    for (int o = 0; o < 2 * NO; ++o) lds_read_landed(t[o]);
                    __builtin_amdgcn_sched_barrier(0);
                    load(d);  // (the patch has been read: the stage D further on takes it)
                    auto operand = [&](int o) {
                        const u32x4 v = {t[2 * o][0], t[2 * o][1], t[2 * o + 1][0], t[2 * o + 1][1]};
                        return __builtin_bit_cast(bf16x8, v);
                    };
#pragma unroll
                    for (int o = 0; o < NA; ++o)
#pragma unroll
                        for (int j = 0; j < FK; ++j)
                            acc[o * FK + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(o), operand(NA + j),
                                                                                      acc[o * FK + j], 0, 0, 0);
                } else {
                    const float *p = reinterpret_cast<const float *>(ring + d * (NO * 1024) + r_lane);
                    float t[PXS / 2][NO];
#pragma unroll
                    for (int q = 0; q < PXS / 2; ++q)
#pragma unroll
                        for (int o = 0; o < NO; ++o) t[q][o] = p[(o * 1024 + (q >> 1) * 512 + (q & 1) * 32) / 4];
                    if constexpr (SUM == 2) {
                        // (a tile's sum is added behind the next tile's MFMAs where there are registers for two)
                        constexpr bool LATER = NF > 1 && NF <= 8;
                        f32x16 part[LATER ? 2 : 1];
#pragma unroll
                        for (int f = 0; f < NF; ++f) {
                            f32x16 &now = part[LATER ? f & 1 : 0];
                            now = f32x16{};
#pragma unroll
                            for (int q = 0; q < PXS / 2; ++q)
                                now = __builtin_amdgcn_mfma_f32_32x32x2f32(t[q][f / FK], t[q][NA + f % FK], now, 0, 0, 0);
                            if (f == 0) {
                                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                                __builtin_amdgcn_sched_barrier(0);
                                load(d);
                            }
                            if (LATER && f > 0) add_here(acc[f - 1], part[(f - 1) & 1]);
                            if (!LATER || f == NF - 1) add_here(acc[f], now);
                            __builtin_amdgcn_sched_barrier(0);
                        }
                    } else {
#pragma unroll
                        for (int q = 0; q < PXS / 2; ++q) {
                            if (q == PXS / 2 - 1) {
                                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
                                __builtin_amdgcn_sched_barrier(0);
                                load(d);
                            }
#pragma unroll
                            for (int o = 0; o < NA; ++o)
#pragma unroll
                                for (int j = 0; j < FK; ++j)
                                    acc[o * FK + j] = __builtin_amdgcn_mfma_f32_32x32x2f32(t[q][o], t[q][NA + j],
                                                                                           acc[o * FK + j], 0, 0, 0);
                        }
                    }
                }
            }
        }
        if constexpr (SUM == 1) {
#pragma unroll
            for (int f = 0; f < NF; ++f) {
                add_here(sum[f], acc[f]);
                acc[f] = f32x16{};
            }
        }
    }
    if constexpr (SUM == 1) {
#pragma unroll
        for (int f = 0; f < NF; ++f) acc[f] = sum[f];
    }
    wait_all_memory();  // (the last stages' loads still write zeros into the ring)

    // The waves' sums, G tiles per round, pairwise.  Rows of a tile are input channels: a
    // chunk of four consecutive ones is 16 bytes of dW.
    const int RS = a.R * S;
    float *const dst = a.partial + (size_t)split * ((size_t)a.Cb * RS * a.Kp * V);
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += G) {
        __syncthreads();  // (the patches, or the last round, are done with)
#pragma unroll
        for (int g = 0; g < G; ++g)
            if (f0 + g < NF) {
#pragma unroll
                for (int vq = 0; vq < 4; ++vq) {
                    const f32x16 &c = acc[f0 + g < NF ? f0 + g : 0];
                    const f32x4 v = {c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]};
                    xch[(g * NW + wave) * 256 + vq * 64 + lane] = v;
                }
            }
        __syncthreads();
        const int g = tid >> 8, ch = tid & 255, f = f0 + g;
        if (f < NF) {
            const f32x4 v = wave_sum<0, NW>([&](int w) { return xch[(g * NW + w) * 256 + ch]; });
            const int o = f / FK, j = f - o * FK, s = o / FC, i = o - s * FC;
            const int c = c0 + 32 * i + (ch >> 6) * 8 + 4 * h;
            const int k = k0 + 32 * j + l32;
            const int cb = c / V;
            if (cb < a.Cb && k < a.Kp)
                *reinterpret_cast<f32x4 *>(dst + (((size_t)cb * RS + r * S + s) * a.Kp + k) * V + (c - cb * V)) = v;
        }
    }
}

typedef void (*upd_ring_fn_t)(const UpdArgs);
#define UPD_RING_ENTRY(DT, S, FC, FK, NW, D, SUM) {DT, S, FC, FK, NW, D, SUM, upd_ring_kernel<DT, S, FC, FK, NW, D, SUM>}
static const struct UpdRingEntry {
    int dtype, s, fc, fk, nw, depth, sum;
    upd_ring_fn_t fn;
} g_upd_ring[] = {
#define F32(S, FC, FK, NW, D, SUM) UPD_RING_ENTRY(CONV_F32, S, FC, FK, NW, D, 0), UPD_RING_ENTRY(CONV_F32, S, FC, FK, NW, D, SUM)
#define BF16(S, FC, FK, NW, D) UPD_RING_ENTRY(CONV_BF16, S, FC, FK, NW, D, 0)
#define BF16_SUM(S, FC, FK, NW, D) BF16(S, FC, FK, NW, D), UPD_RING_ENTRY(CONV_BF16, S, FC, FK, NW, D, 1)
    F32(1, 1, 1, 8, 4, 1), F32(1, 2, 2, 8, 2, 1), UPD_RING_ENTRY(CONV_F32, 1, 2, 4, 8, 2, 0),
    F32(3, 1, 1, 8, 2, 1), F32(3, 1, 2, 8, 2, 1), F32(3, 2, 2, 8, 2, 2), F32(3, 2, 2, 4, 4, 2),
    F32(5, 1, 1, 8, 2, 1), F32(7, 1, 1, 8, 2, 2),
    BF16_SUM(1, 1, 1, 8, 4), BF16_SUM(1, 2, 2, 8, 2), BF16(1, 2, 4, 8, 2),
    BF16_SUM(3, 1, 1, 8, 2), BF16_SUM(3, 1, 2, 8, 2), BF16(3, 2, 2, 8, 2), BF16(3, 2, 2, 4, 4),
    BF16_SUM(5, 1, 1, 8, 2), BF16(7, 1, 1, 8, 2),
};

// (dropped after measuring 38 layers at N = 8 ... 256: deeper rings where they fit, 4 x 2 and 4 x 4
// fragments: at most 2 % ahead of these on a few layers)
static const UpdRingEntry *find_ring(int dtype, int s, int fc, int fk, int nw, int depth, int sum)
{
    for (const UpdRingEntry &e : g_upd_ring)
        if (e.dtype == dtype && e.s == s && e.fc == fc && e.fk == fk && e.nw == nw && e.depth == depth && e.sum == sum)
            return &e;
    return nullptr;
}

bool upd_ring_exists(int dtype, int s, int fc, int fk, int nw, int depth, int sum)
{
    return find_ring(dtype, s, fc, fk, nw, depth, sum) != nullptr;
}

size_t upd_ring_lds_bytes(int s, int fc, int fk, int nw, int depth)
{
    // (the exchange holds nw/4 tiles of every wave)
    return std::max((size_t)nw / 4 * nw * 4096, (size_t)nw * depth * (s * fc + fk) * 1024);
}

hipError_t launch_upd_ring(int dtype, int fc, int fk, int nw, int depth, int sum, const UpdArgs &a, int grid,
                           hipStream_t stream)
{
    const UpdRingEntry *e = find_ring(dtype, a.S, fc, fk, nw, depth, sum);
    if (!e) return hipErrorInvalidDeviceFunction;
    const size_t lds = upd_ring_lds_bytes(e->s, fc, fk, nw, depth);
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(e->fn), lds); err != hipSuccess)
        return err;
    hipLaunchKernelGGL(e->fn, dim3(grid), dim3(nw * 64), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
