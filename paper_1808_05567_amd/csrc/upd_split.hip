// Weight-gradient update of fp32 tensors on the bf16 matrix instructions (split_bf16.h), any filter and stride.
//
//   dW[k,c,r,s] = sum over (n,oj,oi) of I[n,c,oj*stride-pad_h+r,oi*stride-pad_w+s] * dO[n,k,oj,oi]
//
// A workgroup owns a block of WC*FC*32 input channels x WK*FK*32 output channels under T neighbouring taps of one filter row,
// over a range of the flat pixel list (n, oj, oi).  Per stage it brings SP pixels of dO and the run of the input under them
// through registers into LDS as three bf16 numbers, positions of a plane of eight channels 48 bytes apart, and the waves read both
// operands back with transposing reads: four pixels of a channel each.  The taps' operands are the same staged run, a position
// further each, so an input value is converted once for T taps.
//
// What bounds it: T*FC*FK * 192 clocks of MFMAs a wave and 16 pixels, next to which stand the conversions, 88 vector instructions for
// 16 values of a lane, and the transposing reads, six per operand; two or three waves share a SIMD and take turns.  Measured:
// 28 images of 128 -> 128 3x3 at 28x28 76 -> 45 us; 64 of 256 -> 256 3x3 at 14x14 138 -> 86; 256 of 512 -> 1024 1x1 stride 2 at
// 28x28 415 -> 302; 64 of 192 -> 192 1x7 at 17x17 109 -> 67 (upd_ring.hip and upd_f32_1x1.hip before; the look for bits that are lost,
// 3 % of it, not yet in).
#include <algorithm>

#include "split_bf16.h"

namespace convmi {

constexpr int kPix = 48;  // bytes of a position of a plane
// Positions of a plane in LDS: 4 more than a multiple of 16, so that the 16 chunks that a transposing read takes of four pixels and
// four planes lie in different banks.
constexpr int upd_split_pitch(int positions) { return (positions + 11) / 16 * 16 + 4; }

// PI: positions of a plane of the staged run of the input, 16, 32 or 64 (IgemmArgs has no bound on them beyond that).
template <int T, int FC, int FK, int WC, int WK, int SP, int PI>
__global__ __launch_bounds__(WC *WK * 64, 2) void upd_split_kernel(const UpdArgs a)
{
    constexpr int NW = WC * WK;
    constexpr int NPI = WC * FC * 4, NPO = WK * FK * 4;                   // planes of eight channels
    constexpr int NII = (NPI * PI + NW * 64 - 1) / (NW * 64);             // wave-level shares of a stage
    constexpr int NIO = (NPO * SP + NW * 64 - 1) / (NW * 64);
    constexpr int PPI = 64 / PI, PPO = 64 / SP;                           // planes of a share
    constexpr int PITCH_I = upd_split_pitch(PI) * kPix, PITCH_O = upd_split_pitch(SP) * kPix;
    constexpr int IN_BYTES = NPI * PITCH_I, BUF = IN_BYTES + NPO * PITCH_O;
    constexpr int Q16 = SP / 16;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;
    const int wave_c = wave % WC, wave_k = wave / WC;

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
    const int g0 = split * a.rows_per_split;  // (here: pixels per split)
    const int g1 = min(npix, g0 + a.rows_per_split);
    const int stages = (g1 - g0 + SP - 1) / SP;
    // The run of the input under a stage: padded rows LW positions wide, those of the next output row right behind.  (One tap: just
    // the pixels it reads.)
    const int col_step = T == 1 ? 1 : a.stride, in_step = T == 1 ? a.stride : 1;
    const int LW = (a.Q - 1) * col_step + T;
    const float inv_LW = 1.0f / (float)LW;
    const int row_gap = LW - a.Q * col_step;  // positions between the last pixel's successor in a row and the next row's first

    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const rsrc_t rsrc_out = make_rsrc(a.dout, 0, (size_t)a.N * a.Kb * PQ * 16);
    // Shares: lane -> (plane, position); what of the address does not change from stage to stage.
    const int pos_i = lane % PI, pos_o = lane % SP;
    unsigned in_ch[NII], out_ch[NIO];
    int in_at[NII], out_at[NIO];  // LDS address in a buffer, negative: nothing
#pragma unroll
    for (int i = 0; i < NII; ++i) {
        const int plane = (i * NW + wave) * PPI + lane / PI;
        in_ch[i] = (unsigned)(c0 / 4 + 2 * plane) * (unsigned)HW * 16u;
        in_at[i] = plane < NPI && c0 / 4 + 2 * plane < a.Cb ? plane * PITCH_I + pos_i * kPix : -1;
    }
#pragma unroll
    for (int i = 0; i < NIO; ++i) {
        const int plane = (i * NW + wave) * PPO + lane / SP;
        out_ch[i] = (unsigned)(k0 / 4 + 2 * plane) * (unsigned)PQ * 16u;
        out_at[i] = plane < NPO && k0 / 4 + 2 * plane < a.Kb ? IN_BYTES + plane * PITCH_O + pos_o * kPix : -1;
    }
    // (planes beyond the last block stay zero)
    for (int i = tid * 16; i < 2 * BUF; i += NW * 64 * 16) *reinterpret_cast<u32x4 *>(lds + i) = u32x4{0, 0, 0, 0};

    u32x4 in_raw[NII][2], out_raw[NIO][2];
    // first pixel of the next stage to load: number m0, column oi0 of output row rho0
    int m0 = g0, rho0 = g0 / a.Q, oi0 = g0 - rho0 * a.Q;
    const int step_rho = SP / a.Q, step_oi = SP - step_rho * a.Q;
    auto load_stage = [&]() {
        {
            const int x = oi0 * col_step + pos_i, row = fast_div(x, inv_LW), col = x - mul24(row, LW);
            const int rho = rho0 + row, n = fast_div(rho, inv_P), oj = rho - mul24(n, a.P);
            const int ih = mul24(oj, a.stride) - a.pad + r, iw = col * in_step - a.pad_w + s0;
            const bool ok = m0 < g1 && n < a.N && (unsigned)ih < (unsigned)a.H && (unsigned)iw < (unsigned)a.W;
            const unsigned off = ((unsigned)n * (unsigned)a.Cb * (unsigned)HW + (unsigned)(mul24(ih, a.W) + iw)) * 16u;
#pragma unroll
            for (int i = 0; i < NII; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    in_raw[i][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, ok && in_at[i] >= 0 ? off + in_ch[i] : kOutOfRange,
                                                                         (unsigned)b * (unsigned)HW * 16u, 0);
        }
        {
            const int m = m0 + pos_o, n = fast_div(m, inv_PQ);
            const unsigned off = ((unsigned)n * (unsigned)(a.Kb - 1) * (unsigned)PQ + (unsigned)m) * 16u;
#pragma unroll
            for (int i = 0; i < NIO; ++i)
#pragma unroll
                for (int b = 0; b < 2; ++b)
                    out_raw[i][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_out, m < g1 && out_at[i] >= 0 ? off + out_ch[i] : kOutOfRange,
                                                                          (unsigned)b * (unsigned)PQ * 16u, 0);
        }
        m0 += SP;
        rho0 += step_rho;
        oi0 += step_oi;
        if (oi0 >= a.Q) {
            oi0 -= a.Q;
            ++rho0;
        }
    };
    auto put = [&](int at, unsigned char *buf, const Bf16x3 &v) {
        if (at >= 0) {
            u32x4 *const p = reinterpret_cast<u32x4 *>(buf + at);
            p[0] = v.h;
            p[1] = v.m;
            p[2] = v.l;
        }
    };

    // Transposing reads: lanes 4*j + q of a group of 16 address channels 4q .. 4q + 3 of the group's 16 (planes 2*rows and the
    // next) of pixel j of four, and receive four pixels of their own channel; two reads make the eight pixels of a lane half.
    const int tq = lane & 3, tj = (lane >> 2) & 3, rows = (lane >> 4) & 1;
    const int in_lane = (wave_c * FC * 4 + 2 * rows + (tq >> 1)) * PITCH_I + (tq & 1) * 8;
    const int out_lane = IN_BYTES + (wave_k * FK * 4 + 2 * rows + (tq >> 1)) * PITCH_O + (tq & 1) * 8 + (8 * h + tj) * kPix;
    int in_pix[Q16][2];  // byte offset of the lane's pixel of each read of a stage
    int c_oi = oi0;      // column of the first pixel of the stage that is computed
    auto place_pixels = [&]() {
#pragma unroll
        for (int q = 0; q < Q16; ++q)
#pragma unroll
            for (int b = 0; b < 2; ++b) {
                const int j = 16 * q + 8 * h + 4 * b + tj;
                const int row = T == 1 ? 0 : fast_div(c_oi + j, inv_Q);
                in_pix[q][b] = T == 1 ? j * kPix : (mul24(row, row_gap) + mul24(j, a.stride)) * kPix;
            }
        c_oi += step_oi;
        if (c_oi >= a.Q) c_oi -= a.Q;
    };
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
    auto read8 = [&](const unsigned char *p0, const unsigned char *p1) {
        Bf16x3 v;
        static_for<0, 3>([&](auto pc) {
            constexpr int P = decltype(pc)::value;
            const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)const_cast<unsigned char *>(p0 + P * 16)));
            const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)const_cast<unsigned char *>(p1 + P * 16)));
            (P == 0 ? v.h : P == 1 ? v.m : v.l) = u32x4{x[0], x[1], y[0], y[1]};
        });
        return v;
    };
    auto read_in = [&](const unsigned char *buf, int q, int t, int i) {
        const unsigned char *const p = buf + in_lane + i * 4 * PITCH_I + t * kPix;
        return read8(p + in_pix[q][0], p + in_pix[q][1]);
    };
    auto read_out = [&](const unsigned char *buf, int q, int i) {
        const unsigned char *const p = buf + out_lane + i * 4 * PITCH_O + 16 * q * kPix;
        return read8(p, p + 4 * kPix);
    };

    f32x16 big[T][FC][FK], small[T][FC][FK];
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) big[t][i][j] = small[t][i][j] = f32x16{};

    unsigned lost;
    lds_barrier();  // (the zeros are there)
    load_stage();
    static_for<0, NII>([&](auto i) { put(in_at[i], lds, split8<true>(in_raw[i], lost)); });
    static_for<0, NIO>([&](auto i) { put(out_at[i], lds, split8<true>(out_raw[i], lost)); });
    load_stage();
    place_pixels();
    lds_barrier();

    // A stage is Q16 * T * FC * FK blocks of six MFMAs.  Beside them, pinned: the operands of the block that follows are read, the
    // next stage is converted, one piece behind an MFMA, and the stage after that is requested.
    constexpr int NBLK = Q16 * T * FC * FK, NM = kSplitProducts * NBLK, NITEM = NII + NIO, PIECES = NITEM * kSplitPieces;
    constexpr int NC = NM * 3 / 4;  // MFMAs beside which the pieces stand
    for (int st = 0; st < stages; ++st) {
        const unsigned char *const buf = lds + (st & 1) * BUF;
        unsigned char *const next = lds + (1 - (st & 1)) * BUF;
        Bf16x3 I[2][FC], O[2][FK], item;
        float rest[2];
        O[0][0] = read_out(buf, 0, 0);
        I[0][0] = read_in(buf, 0, 0, 0);
        static_for<0, NM>([&](auto kc) {
            constexpr int k = decltype(kc)::value, b = k / kSplitProducts, m = k % kSplitProducts;
            // blocks of a tap in snake order: (0,0) (0,1) (1,1) (1,0)
            constexpr int u = b / (FC * FK), e = b % (FC * FK), i = e / FK, j = i % 2 == 0 ? e % FK : FK - 1 - e % FK;
            constexpr int q = u / T, t = u % T;
            mma_split<m>(I[u & 1][i], O[q & 1][j], big[t][i][j], small[t][i][j]);
            // (the operands that the next block is the first to use)
            if constexpr (m == 0 && b + 1 < NBLK) {
                constexpr int b2 = b + 1, u2 = b2 / (FC * FK), e2 = b2 % (FC * FK), i2 = e2 / FK,
                              j2 = i2 % 2 == 0 ? e2 % FK : FK - 1 - e2 % FK, q2 = u2 / T, t2 = u2 % T;
                if constexpr (e2 % FK == 0) I[u2 & 1][i2] = read_in(buf, q2, t2, i2);
                if constexpr (t2 == 0 && i2 == 0) O[q2 & 1][j2] = read_out(buf, q2, j2);
            }
            if constexpr (k < NC)
                static_for<k * PIECES / NC, (k + 1) * PIECES / NC>([&](auto pc) {
                    constexpr int piece = decltype(pc)::value % kSplitPieces, it = decltype(pc)::value / kSplitPieces;
                    if constexpr (it < NII) {
                        split_piece<piece, true>(in_raw[it], item, rest, lost);
                        if constexpr (piece == kSplitPieces - 1) put(in_at[it], next, item);
                    } else {
                        split_piece<piece, true>(out_raw[it - NII], item, rest, lost);
                        if constexpr (piece == kSplitPieces - 1) put(out_at[it - NII], next, item);
                    }
                });
            if constexpr (k == NC) load_stage();
            __builtin_amdgcn_sched_barrier(0);
        });
        place_pixels();
        lds_barrier();
    }

    // ---- store: a lane owns one output channel and, per eight rows, four consecutive input channels (a block)
    const int RS = a.R * a.S;
    const size_t copy_bytes = (size_t)a.Cb * RS * a.Kp * 16;
    const rsrc_t rd = make_rsrc(reinterpret_cast<char *>(a.partial) + (size_t)split * copy_bytes, 0, copy_bytes);
    float most = 0.0f;
#pragma unroll
    for (int t = 0; t < T; ++t)
#pragma unroll
        for (int i = 0; i < FC; ++i)
#pragma unroll
            for (int j = 0; j < FK; ++j) {
                big[t][i][j] += small[t][i][j];
                most = max_magnitude(most, big[t][i][j]);
            }
    auto store = [&](const f32x16 &v, int t, int i, int j) {
        const int k = k0 + (wave_k * FK + j) * 32 + l32, c = c0 + (wave_c * FC + i) * 32 + 4 * h;
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            const int cb = c / 4 + 2 * vq;
            const bool live = s0 + t < a.S && k < a.Kp && cb < a.Cb;
            const unsigned at = (((unsigned)cb * (unsigned)RS + (unsigned)(r * a.S + s0 + t)) * (unsigned)a.Kp + (unsigned)k) * 16u;
            Elem<CONV_F32>::store4(rd, live ? at : kOutOfRange, 0, v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]);
        }
    };
    if (__builtin_expect(!sums_need_fp32(most), 1)) {
#pragma unroll
        for (int t = 0; t < T; ++t)
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j) store(big[t][i][j], t, i, j);
        return;
    }
    // Infinite or NaN sums: the wave's block again on the fp32 instructions, a pixel to a lane half, straight from memory, all taps
    // together (five: one by one, for the registers).  All of a tensor NaN, 64 images 64 -> 64 3x3 at 56x56 309 us, 143 on the fp32
    // instructions alone; 512 -> 1024 1x1 stride 2 at 28x28 296 and 110 (fragment by fragment, a pair at a time: 699 and 667).  Four pairs of pixels are on their way while four multiply; chains of 32 pixels are
    // summed apart.
    constexpr int PAIRS = 4, TG = T * FC * FK > 4 ? 1 : T;
    for (int t0 = 0; t0 < T; t0 += TG) {
        float x[2][PAIRS][TG][FC], y[2][PAIRS][FK];
        auto load = [&](int first, float(&xs)[PAIRS][TG][FC], float(&ys)[PAIRS][FK]) {
#pragma unroll
            for (int q = 0; q < PAIRS; ++q) {
                const int m = first + 2 * q + h, n = fast_div(m, inv_PQ), rem = m - mul24(n, PQ), oj = fast_div(rem, inv_Q), oi = rem - mul24(oj, a.Q);
                const int ih = mul24(oj, a.stride) - a.pad + r, iw = mul24(oi, a.stride) - a.pad_w + s0 + t0;
                const bool row = m < g1 && (unsigned)ih < (unsigned)a.H;
#pragma unroll
                for (int t = 0; t < TG; ++t)
#pragma unroll
                    for (int i = 0; i < FC; ++i) {
                        const int c = c0 + (wave_c * FC + i) * 32 + l32;
                        const unsigned at = (((unsigned)n * (unsigned)a.Cb + (unsigned)(c >> 2)) * (unsigned)HW + (unsigned)(mul24(ih, a.W) + iw + t)) * 16u + (c & 3) * 4u;
                        const bool in = row && (unsigned)(iw + t) < (unsigned)a.W && c < a.Cb * 4;
                        xs[q][t][i] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_in, in ? at : kOutOfRange, 0, 0));
                    }
#pragma unroll
                for (int j = 0; j < FK; ++j) {
                    const int k = k0 + (wave_k * FK + j) * 32 + l32;
                    const unsigned at = (((unsigned)n * (unsigned)a.Kb + (unsigned)(k >> 2)) * (unsigned)PQ + (unsigned)rem) * 16u + (k & 3) * 4u;
                    ys[q][j] = __uint_as_float(__builtin_amdgcn_raw_buffer_load_b32(rsrc_out, m < g1 && k < a.Kb * 4 ? at : kOutOfRange, 0, 0));
                }
            }
        };
        f32x16 sum[TG][FC][FK], part[TG][FC][FK];
        auto each = [&](auto &&f) {
            static_for<0, TG * FC * FK>([&](auto fc) {
                constexpr int e = decltype(fc)::value;
                f(std::integral_constant<int, e / (FC * FK)>{}, std::integral_constant<int, e / FK % FC>{}, std::integral_constant<int, e % FK>{});
            });
        };
        auto multiply = [&](const float(&xs)[PAIRS][TG][FC], const float(&ys)[PAIRS][FK]) {
            static_for<0, PAIRS>([&](auto q) {
                each([&](auto t, auto i, auto j) { part[t][i][j] = __builtin_amdgcn_mfma_f32_32x32x2f32(xs[q][t][i], ys[q][j], part[t][i][j], 0, 0, 0); });
            });
        };
        each([&](auto t, auto i, auto j) { sum[t][i][j] = part[t][i][j] = f32x16{}; });
        load(g0, x[0], y[0]);
        for (int m = g0; m < g1; m += 4 * PAIRS) {
            load(m + 2 * PAIRS, x[1], y[1]);
            multiply(x[0], y[0]);
            load(m + 4 * PAIRS, x[0], y[0]);
            multiply(x[1], y[1]);
            if ((m - g0) % 32 != 0 || m + 4 * PAIRS >= g1)
                each([&](auto t, auto i, auto j) {
                    sum[t][i][j] += part[t][i][j];
                    part[t][i][j] = f32x16{};
                });
        }
        each([&](auto t, auto i, auto j) { store(sum[t][i][j], t0 + t, i, j); });
    }
}

typedef void (*upd_fn_t)(const UpdArgs);
#define UPD_SPLIT_ENTRY(T, FC, FK, WC, WK, SP, PI) {{T, FC, FK, WC, WK, SP, PI}, upd_split_kernel<T, FC, FK, WC, WK, SP, PI>}
static const struct UpdSplitEntry {
    UpdSplitVariant v;
    upd_fn_t fn;
} g_upd_split[] = {
    // 1x1 and one column
    UPD_SPLIT_ENTRY(1, 2, 2, 2, 2, 16, 16), UPD_SPLIT_ENTRY(1, 2, 2, 4, 2, 16, 16), UPD_SPLIT_ENTRY(1, 2, 1, 2, 4, 32, 32),
    UPD_SPLIT_ENTRY(1, 2, 1, 2, 2, 32, 32), UPD_SPLIT_ENTRY(1, 1, 2, 2, 2, 32, 32), UPD_SPLIT_ENTRY(1, 1, 1, 2, 2, 32, 32),
    UPD_SPLIT_ENTRY(1, 1, 1, 2, 2, 64, 64), UPD_SPLIT_ENTRY(1, 2, 1, 4, 2, 16, 16), UPD_SPLIT_ENTRY(1, 1, 1, 4, 2, 32, 32),
    // three columns
    UPD_SPLIT_ENTRY(3, 1, 1, 2, 2, 32, 64), UPD_SPLIT_ENTRY(3, 1, 1, 2, 4, 32, 64), UPD_SPLIT_ENTRY(3, 1, 1, 2, 2, 16, 32),
    UPD_SPLIT_ENTRY(3, 1, 1, 2, 2, 16, 64), UPD_SPLIT_ENTRY(3, 1, 1, 2, 4, 16, 64), UPD_SPLIT_ENTRY(3, 1, 1, 2, 4, 16, 32),
    UPD_SPLIT_ENTRY(3, 1, 1, 1, 4, 32, 64), UPD_SPLIT_ENTRY(3, 1, 1, 4, 2, 16, 32),
    // five and seven columns
    UPD_SPLIT_ENTRY(4, 1, 1, 2, 2, 32, 64), UPD_SPLIT_ENTRY(4, 1, 1, 2, 4, 32, 64), UPD_SPLIT_ENTRY(4, 1, 1, 2, 2, 16, 32),
    UPD_SPLIT_ENTRY(5, 1, 1, 2, 2, 16, 32),
};

static const UpdSplitEntry *find(const UpdSplitVariant &v)
{
    for (const UpdSplitEntry &e : g_upd_split)
        if (e.v.t == v.t && e.v.fc == v.fc && e.v.fk == v.fk && e.v.wc == v.wc && e.v.wk == v.wk && e.v.sp == v.sp && e.v.pi == v.pi) return &e;
    return nullptr;
}
bool upd_split_exists(const UpdSplitVariant &v) { return find(v) != nullptr; }
const UpdSplitVariant *upd_split_variant(int i)
{
    return i >= 0 && i < (int)(sizeof(g_upd_split) / sizeof(g_upd_split[0])) ? &g_upd_split[i].v : nullptr;
}

size_t upd_split_lds_bytes(const UpdSplitVariant &v)
{
    return (size_t)2 * 4 * kPix * (v.wc * v.fc * upd_split_pitch(v.pi) + v.wk * v.fk * upd_split_pitch(v.sp));
}

hipError_t launch_upd_split(const UpdSplitVariant &v, const UpdArgs &a, int grid, hipStream_t stream)
{
    const UpdSplitEntry *e = find(v);
    if (!e) return hipErrorInvalidDeviceFunction;
    const size_t lds = upd_split_lds_bytes(v);
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(e->fn), lds); err != hipSuccess) return err;
    hipLaunchKernelGGL(e->fn, dim3(grid), dim3(v.wc * v.wk * 64), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
