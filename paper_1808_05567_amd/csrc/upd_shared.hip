// Weight-gradient update of bf16 tensors, any filter and stride 1 or 2 (one tap: any stride), with both operands of a
// workgroup staged once for all its waves.
//
//   dW[k,c,r,s] = sum over (n,oj,oi) of I[n,c,oj*stride-pad_h+r,oi*stride-pad_w+s] * dO[n,k,oj,oi]
//
// A workgroup owns a block of WC*FC*32 input channels x WK*FK*32 output channels under T neighbouring taps of one filter row, over
// a range of the flat pixel list (n, oj, oi); WP groups of waves share its pixels.  Per stage SP pixels of dO and the run of the
// input under them go straight into LDS (loads that write there), up to NB - 1 stages ahead, one barrier per stage.  The
// waves read both with transposing reads, four pixels of a channel each, at any position: a tap is an offset.
//
// The run of the input: padded rows one behind the other, LW positions each, so that the pixels of a row are `stride` positions
// apart and the first of the next row follows after a gap.  With stride 2 the even positions come first, then the odd ones
// (LW is even): the pixels of a tap are neighbours then.  A plane of eight channels is a multiple of 16 positions and 4 more long, so
// that the 16 chunks that a transposing read takes of four neighbouring pixels and four planes lie in different banks.
//
// Against the kernels of one wave to a block (upd_ring.hip, upd_window.hip) an operand comes through the L2 once for a block of up to
// 256 x 256 channels, not of 64 x 64; against the row kernel no row is padded to runs of eight pixels and no tap is made by shifts.
// What bounds it: the way of its operands from the L2, 16 to 20 bytes a clock and CU (288 -> 384 3x3 stride 2, N = 32: 414 MB of lines, 11.5 TB/s,
// 67 MB of them from memory; a loop that only streams gets 32 - 38), for wide blocks the MFMAs, 0.54 of the
// time at 1.7 GHz; LDS a quarter.  Measured, reduce launch included: 288 -> 384 3x3 stride 2 at 35x35, N = 32 / 92, 42 -> 36 and 113 ->
// 89 us; 504 -> 284 1x7 at 23x21, N = 27, 57 -> 41; 632 -> 40 7x1 at 59x60, N = 18, 113 -> 89.
#include <algorithm>

#include "igemm_kernel.h"

namespace convmi {

template <int T, int ST, int FC, int FK, int WC, int WK, int WP, int SP, int PI, int NB>
__global__ __launch_bounds__(WC *WK *WP * 64, 2) void upd_shared_kernel(const UpdArgs a)
{
    constexpr int V = 8;
    constexpr int NW = WC * WK * WP;
    constexpr int PO = (SP + 63) / 64 * 64;               // positions of a plane of dO
    constexpr int GI = PI / 64, GO = PO / 64;             // wave-level loads of a plane
    constexpr int NPI = WC * FC * 4, NPO = WK * FK * 4;   // planes
    constexpr int WI = NW / GI, WO = NW / GO;             // waves that share a position group's planes
    constexpr int NII = (NPI + WI - 1) / WI, NIO = (NPO + WO - 1) / WO;  // loads of a wave per stage
    constexpr int PITCH_I = PI * 16 + 64, PITCH_O = PO * 16 + 64;
    constexpr int IN_BYTES = NPI * PITCH_I, BUF = IN_BYTES + NPO * PITCH_O;
    constexpr int HALF = PI / 2 * 16;                     // (stride 2) where the odd positions start
    constexpr int NQ = SP / 16 / WP;                      // runs of 16 pixels of a wave per stage
    static_assert(NW % GI == 0 && NW % GO == 0 && SP % (16 * WP) == 0 && (T > 1 || ST == 1), "");
    static_assert(FC * 4 * PITCH_I < 65536 && FK * 4 * PITCH_O + SP * 16 < 65536, "offsets of LDS reads");
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const int wave_c = wave % WC, wave_k = wave / WC % WK, wave_p = wave / (WC * WK);

    // split slowest: the blocks of a pixel range run side by side and share its lines in the L2
    const int bid = blockIdx.x;
    int lin = (bid & 7) * a.per_xcd + (bid >> 3);
    if (lin >= a.total) return;
    const int groups = (a.S + T - 1) / T;  // of taps in a filter row
    const int blocks = a.n_ct * a.n_kt * a.R * groups;
    const int split = lin / blocks;
    lin -= split * blocks;
    const int kt = lin % a.n_kt;
    lin /= a.n_kt;
    const int ct = lin % a.n_ct;
    lin /= a.n_ct;
    const int s0 = lin % groups * T, r = lin / groups;
    const int c0 = ct * WC * FC * 32, k0 = kt * WK * FK * 32;

    const int PQ = a.P * a.Q, npix = a.N * PQ, HW = a.H * a.W;
    const float inv_PQ = 1.0f / (float)PQ, inv_Q = 1.0f / (float)a.Q, inv_P = 1.0f / (float)a.P;
    const int g0 = split * a.rows_per_split;  // (here: pixels per split, a whole number of stages)
    const int stages = (min(npix - g0, a.rows_per_split) + SP - 1) / SP;
    // A row of the run, in positions (stride 2: in pairs of them), and what it has behind its last pixel's successor
    const int LW = T == 1 ? a.Q : ST == 1 ? a.Q + T - 1 : a.Q - 1 + (T + 1) / 2;
    const int row_gap = LW - a.Q;
    const float inv_LW = 1.0f / (float)LW;

    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const rsrc_t rsrc_out = make_rsrc(a.dout, 0, (size_t)a.N * a.Kb * PQ * 16);
    // This wave's loads: planes wave / GI + i * WI of position group wave % GI.
    const int grp_i = wave % GI, grp_o = wave % GO;
    const int pl_i = wave / GI, pl_o = wave / GO;
    constexpr int GH = ST == 2 ? GI / 2 : GI;
    const int odd = ST == 2 ? grp_i / GH : 0;  // (stride 2) which of a pair
    const int idx_i = (ST == 2 ? grp_i % GH : grp_i) * 64 + lane, idx_o = grp_o * 64 + lane;
    const unsigned in_ch = (unsigned)(c0 / V) * (unsigned)HW * 16u, out_ch = (unsigned)(k0 / V) * (unsigned)PQ * 16u;
    const int in_blocks = a.Cb - c0 / V, out_blocks = a.Kb - k0 / V;

    // first pixel of the next stage to load: number m0, column oi0 of output row rho0
    int m0 = g0, rho0 = g0 / a.Q, oi0 = g0 - rho0 * a.Q;
    const int step_rho = SP / a.Q, step_oi = SP - step_rho * a.Q;
    auto load_stage = [&](unsigned char *buf) {
        {
            const int x = oi0 + idx_i, row = fast_div(x, inv_LW), col = x - mul24(row, LW);
            const int rho = rho0 + row, n = fast_div(rho, inv_P), oj = rho - mul24(n, a.P);
            const int ih = mul24(oj, a.stride) - a.pad + r;
            const int iw = (T == 1 ? mul24(col, a.stride) : ST * col + odd) - a.pad_w + s0;
            const bool ok = n < a.N && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const unsigned off = ((unsigned)n * (unsigned)a.Cb * (unsigned)HW + (unsigned)(mul24(ih, a.W) + iw)) * 16u + in_ch;
#pragma unroll
            for (int i = 0; i < NII; ++i) {
                const int plane = pl_i + i * WI;
                if (NPI % WI != 0 && plane >= NPI) continue;
                load_to_lds_16(rsrc_in, ok && plane < in_blocks ? off : kOutOfRange, (unsigned)plane * (unsigned)HW * 16u,
                               buf + plane * PITCH_I + grp_i * 1024);
            }
        }
        {
            const int m = m0 + idx_o, n = fast_div(m, inv_PQ);
            const unsigned off = ((unsigned)n * (unsigned)(a.Kb - 1) * (unsigned)PQ + (unsigned)m) * 16u + out_ch;
#pragma unroll
            for (int i = 0; i < NIO; ++i) {
                const int plane = pl_o + i * WO;
                if (NPO % WO != 0 && plane >= NPO) continue;
                load_to_lds_16(rsrc_out, m < npix && plane < out_blocks ? off : kOutOfRange, (unsigned)plane * (unsigned)PQ * 16u,
                               buf + IN_BYTES + plane * PITCH_O + grp_o * 1024);
            }
        }
        m0 += SP;
        rho0 += step_rho;
        oi0 += step_oi;
        if (oi0 >= a.Q) {
            oi0 -= a.Q;
            ++rho0;
        }
    };
    static_assert(NB == 2 || (NPI % WI == 0 && NPO % WO == 0), "every wave's loads of a stage are counted");

    // Transposing reads: lanes 4*j + q of a group of 16 address channels 4q .. 4q + 3 of the group's 16 (planes 2*rows and the
    // next) of pixel j of four, and receive four pixels of their own channel; two reads make the eight pixels of a lane half.
    const int tq = lane & 3, tj = (lane >> 2) & 3, rows = (lane >> 4) & 1;
    const unsigned base = lds_address(lds);
    const unsigned in_lane = base + (unsigned)((wave_c * FC * 4 + 2 * rows + (tq >> 1)) * PITCH_I + (tq & 1) * 8);
    const unsigned out_lane = base + (unsigned)(IN_BYTES + (wave_k * FK * 4 + 2 * rows + (tq >> 1)) * PITCH_O + (tq & 1) * 8 +
                                                (wave_p * NQ * 16 + 8 * h + tj) * 16);
    int c_oi = oi0;  // column of the first pixel of the stage that is computed
    const int first = wave_p * NQ * 16 + 8 * h + tj;

    f32x16 acc[T][FC][FK];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) acc[t][i][j] = f32x16{};

#pragma unroll
    for (int d = 0; d < NB - 1; ++d) load_stage(lds + d * BUF);  // (beyond the range: read and not used)

    auto operand = [&](const lds_u32x2 &x, const lds_u32x2 &y) {
        const u32x4 v = {x[0], x[1], y[0], y[1]};
        return __builtin_bit_cast(bf16x8, v);
    };
    int slot = 0, next = NB - 1;  // buffers of the stage that is computed and of the one that is loaded
    for (int st = 0; st < stages; ++st) {
        // this stage's loads have landed (the NB - 2 later stages' may be on their way); all waves have left the one before
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NB - 2) * (NII + NIO)) : "memory");
        __builtin_amdgcn_s_barrier();
        asm volatile("" ::: "memory");
        __builtin_amdgcn_sched_barrier(0);
        load_stage(lds + next * BUF);
        const unsigned at_i = in_lane + (unsigned)(slot * BUF), at_o = out_lane + (unsigned)(slot * BUF);
        lds_u32x2 ri[2][2 * FC], ro[2][2 * FK];
        unsigned pix[2][2];
        auto place = [&](auto qc) {
            constexpr int q = decltype(qc)::value;
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int j = first + 16 * q + 4 * b;
                pix[q & 1][b] = at_i + (unsigned)((T == 1 ? j : mul24(fast_div(c_oi + j, inv_Q), row_gap) + j) * 16);
            }
        };
        // reads of unit u = run q * T + tap t into operand set u & 1
        auto read_in = [&](auto uc) {
            constexpr int u = decltype(uc)::value, q = u / T, t = u % T;
            constexpr int tap = ST == 1 ? t * 16 : (t & 1) * HALF + (t >> 1) * 16;
            static_for<0, FC>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                ri[u & 1][2 * i] = lds_read_tr16_b64_untracked<i * 4 * PITCH_I + tap>(pix[q & 1][0]);
                ri[u & 1][2 * i + 1] = lds_read_tr16_b64_untracked<i * 4 * PITCH_I + tap>(pix[q & 1][1]);
            });
        };
        auto read_out = [&](auto qc) {
            constexpr int q = decltype(qc)::value;
            static_for<0, FK>([&](auto jc) {
                constexpr int j = decltype(jc)::value;
                ro[q & 1][2 * j] = lds_read_tr16_b64_untracked<j * 4 * PITCH_O + q * 256>(at_o);
                ro[q & 1][2 * j + 1] = lds_read_tr16_b64_untracked<j * 4 * PITCH_O + q * 256 + 64>(at_o);
            });
        };
        place(std::integral_constant<int, 0>{});
        read_out(std::integral_constant<int, 0>{});
        read_in(std::integral_constant<int, 0>{});
        // (the next unit's reads are on their way while a unit's MFMAs issue)
        static_for<0, NQ * T>([&](auto uc) {
            constexpr int u = decltype(uc)::value, q = u / T, t = u % T;
            constexpr bool more = u + 1 < NQ * T, turn = more && t == T - 1;
            if constexpr (turn) {
                place(std::integral_constant<int, q + 1>{});
                read_out(std::integral_constant<int, q + 1>{});
            }
            if constexpr (more) read_in(std::integral_constant<int, u + 1>{});
            __builtin_amdgcn_sched_barrier(0);
            lds_reads_pending<(more ? 2 * FC : 0) + (turn ? 2 * FK : 0)>();
            if constexpr (t == 0) {
#pragma unroll
                for (int o = 0; o < 2 * FK; ++o) lds_read_landed(ro[q & 1][o]);
            }
#pragma unroll
            for (int o = 0; o < 2 * FC; ++o) lds_read_landed(ri[u & 1][o]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j)
                    acc[t][i][j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(operand(ri[u & 1][2 * i], ri[u & 1][2 * i + 1]),
                                                                           operand(ro[q & 1][2 * j], ro[q & 1][2 * j + 1]), acc[t][i][j], 0, 0, 0);
        });
        c_oi += step_oi;
        if (c_oi >= a.Q) c_oi -= a.Q;
        slot = slot + 1 == NB ? 0 : slot + 1;
        next = next + 1 == NB ? 0 : next + 1;
    }
    wait_all_memory();  // (the last stages' loads still write into the buffers)

    // Rows of a tile are input channels: a chunk of four consecutive ones is 16 bytes of dW.
    const int RS = a.R * a.S;
    float *const dst = a.partial + (size_t)split * ((size_t)a.Cb * RS * a.Kp * V);
    auto store = [&](const f32x4 &v, int wc, int wk, int t, int i, int j, int vq, int hh, int l) {
        const int c = c0 + (wc * FC + i) * 32 + vq * 8 + 4 * hh, k = k0 + (wk * FK + j) * 32 + l;
        const int cb = c / V;
        if (s0 + t < a.S && cb < a.Cb && k < a.Kp)
            *reinterpret_cast<f32x4 *>(dst + (((size_t)cb * RS + r * a.S + s0 + t) * a.Kp + k) * V + (c - cb * V)) = v;
    };
    if constexpr (WP == 1) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j)
#pragma unroll
                    for (int vq = 0; vq < 4; ++vq) {
                        const f32x16 &c = acc[t][i][j];
                        store(f32x4{c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]}, wave_c, wave_k, t, i, j, vq, h, l32);
                    }
    } else {
        // the pixel groups' sums, a tile of every wave per round, pairwise
        f32x4 *const xch = reinterpret_cast<f32x4 *>(lds);
        constexpr int CK = WC * WK;
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j) {
                    __syncthreads();  // (the buffers, or the last round, are done with)
#pragma unroll
                    for (int vq = 0; vq < 4; ++vq) {
                        const f32x16 &c = acc[t][i][j];
                        xch[wave * 256 + vq * 64 + lane] = f32x4{c[4 * vq], c[4 * vq + 1], c[4 * vq + 2], c[4 * vq + 3]};
                    }
                    __syncthreads();
#pragma unroll
                    for (int e0 = 0; e0 < CK * 256; e0 += NW * 64) {
                        const int e = e0 + tid;
                        if (CK * 256 >= NW * 64 || e < CK * 256) {
                            const f32x4 v = wave_sum<0, WP>([&](int w) { return xch[w * CK * 256 + e]; });
                            const int ck = e >> 8, ch = e & 255;
                            store(v, ck % WC, ck / WC, t, i, j, ch >> 6, (ch >> 5) & 1, ch & 31);
                        }
                    }
                }
    }
}

typedef void (*upd_fn_t)(const UpdArgs);
#define UPD_SHARED_ENTRY(T, ST, FC, FK, WC, WK, WP, SP, PI, NB) \
    {{T, ST, FC, FK, WC, WK, WP, SP, PI, NB}, upd_shared_kernel<T, ST, FC, FK, WC, WK, WP, SP, PI, NB>}
static const struct UpdSharedEntry {
    UpdSharedVariant v;
    upd_fn_t fn;
} g_upd_shared[] = {
    // one column
    UPD_SHARED_ENTRY(1, 1, 2, 2, 2, 2, 2, 64, 64, 3), UPD_SHARED_ENTRY(1, 1, 2, 2, 1, 2, 4, 128, 128, 3),
    UPD_SHARED_ENTRY(1, 1, 2, 4, 2, 1, 4, 64, 64, 3), UPD_SHARED_ENTRY(1, 1, 2, 4, 2, 2, 2, 64, 64, 3),
    UPD_SHARED_ENTRY(1, 1, 2, 4, 4, 2, 1, 64, 64, 2),
    // seven columns, in one group or three
    UPD_SHARED_ENTRY(7, 1, 1, 1, 2, 4, 1, 64, 128, 3), UPD_SHARED_ENTRY(7, 1, 1, 1, 2, 2, 2, 64, 128, 3),
    UPD_SHARED_ENTRY(7, 1, 1, 1, 1, 2, 4, 64, 128, 3), UPD_SHARED_ENTRY(3, 1, 1, 1, 2, 2, 2, 96, 128, 3),
    UPD_SHARED_ENTRY(3, 1, 1, 1, 2, 2, 1, 96, 128, 2), UPD_SHARED_ENTRY(3, 1, 1, 1, 1, 2, 4, 64, 128, 3),
    // three columns, stride 2
    UPD_SHARED_ENTRY(3, 2, 1, 2, 2, 2, 2, 96, 256, 2), UPD_SHARED_ENTRY(3, 2, 1, 2, 1, 2, 4, 64, 256, 3),
    UPD_SHARED_ENTRY(3, 2, 2, 2, 1, 2, 4, 64, 256, 3), UPD_SHARED_ENTRY(3, 2, 2, 2, 2, 2, 2, 32, 128, 3),
};

static const UpdSharedEntry *find(const UpdSharedVariant &v)
{
    for (const UpdSharedEntry &e : g_upd_shared)
        if (e.v.t == v.t && e.v.st == v.st && e.v.fc == v.fc && e.v.fk == v.fk && e.v.wc == v.wc && e.v.wk == v.wk && e.v.wp == v.wp &&
            e.v.sp == v.sp && e.v.pi == v.pi && e.v.nb == v.nb)
            return &e;
    return nullptr;
}
bool upd_shared_exists(const UpdSharedVariant &v) { return find(v) != nullptr; }
const UpdSharedVariant *upd_shared_variant(int i)
{
    return i >= 0 && i < (int)(sizeof(g_upd_shared) / sizeof(g_upd_shared[0])) ? &g_upd_shared[i].v : nullptr;
}

size_t upd_shared_lds_bytes(const UpdSharedVariant &v)
{
    const size_t buffer = (size_t)4 * (v.wc * v.fc * (v.pi * 16 + 64) + v.wk * v.fk * ((v.sp + 63) / 64 * 1024 + 64));
    return std::max(buffer * v.nb, v.wp > 1 ? (size_t)v.wc * v.wk * v.wp * 4096 : 0);
}

hipError_t launch_upd_shared(const UpdSharedVariant &v, const UpdArgs &a, int grid, hipStream_t stream)
{
    const UpdSharedEntry *e = find(v);
    if (!e) return hipErrorInvalidDeviceFunction;
    const size_t lds = upd_shared_lds_bytes(v);
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(e->fn), lds); err != hipSuccess) return err;
    hipLaunchKernelGGL(e->fn, dim3(grid), dim3(v.wc * v.wk * v.wp * 64), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
