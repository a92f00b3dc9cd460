// Implicit-GEMM direct convolution of fp32 tensors on the bf16 matrix instructions (split_bf16.h): forward, and backward by
// data through duality, for results that fill the chip.
//
// A workgroup owns WK*32 channels x WM*FM*32 consecutive pixels of a strip of TQ result columns (as a rule the whole
// width: the pixel list is flat, no slots are lost to row ends).  Each input value is converted once per workgroup: the
// input tile, halo and all, comes through registers into LDS as three bf16 numbers, 16 channels of every position a step,
// and all taps read it from there.  The weights do not go through LDS: a wave's rows are its own, and it converts
// them between the MFMAs that use the ones before.
//
// What bounds it: a round (one tap of 16 channels) is 6 * FM MFMAs a wave, 768 clocks for FM = 4, next to which stand
// 8 pairs of conversions, about 70 clocks of vector instructions each -- hidden behind the MFMAs as long as two
// waves share a SIMD and they take turns -- and, at these operand values, the card's power: the MFMAs alone run at 1.9 of
// 2.47 PFLOP/s on random operands, 1.7 next to this many conversions, 287 TFLOP/s of fp32 products.  (Counters, 256 images: MFMAs busy 55 - 58 %
// of the clocks of 3x3 layers, 38 % of 1x1 ones; a step of 20 layers runs at 1 990 MHz, 2 350 on the fp32 instructions.)
#pragma once
#include <algorithm>

#include "igemm_exchange.h"
#include "igemm_fp32_again.h"
#include "split_address.h"
#include "split_bf16.h"

namespace convmi {

// Bytes of a position of a plane of eight channels: h, m, l.  Lanes 48 bytes apart meet no bank conflict (1x1: none counted); where rows of the
// tile end inside a read, 3x3, conflicts are 46 - 51 % of the LDS cycles, and waits for LDS 3 % of the waves' time.
constexpr int kPosBytes = 48;

// WK x WM waves share a tile (four of them), FM pixel fragments each; KW such sets split the channels between them and add
// their sums in LDS.  G: groups of 16 channels a step.  NI: wave-level shares of the input tile per wave and step.
// FW (backward by data): the weights as the forward pass has them (put_weights).
template <int WK, int WM, int FM, int KW, int G, int NI, bool FW>
__device__ __forceinline__ void igemm_split_tile(const IgemmArgs &a, const int bid, unsigned char *const lds)
{
    static_assert(WK * WM == 4, "four waves a set");
    constexpr int TK = WK * 32, TM = WM * FM * 32;
    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave_all = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int kw = KW == 1 ? 0 : wave_all >> 2, wave = wave_all & 3;
    const int h = lane >> 5, l32 = lane & 31;
    const int wave_k = wave % WK, wave_m = wave / WK;

    int kt, tile, sp;
    if (!small_tile(a, bid, kt, tile, sp)) return;
    const int qt = tile % a.n_qt, q0 = qt * a.TQ;
    const int k0 = kt * TK + wave_k * 32;
    const int RS = a.R * a.S, HW = a.H * a.W;

    // First pixel of the tile: column c0 of row oj0 of image n0 (of the strip).
    const int m0 = (tile / a.n_qt) * TM;
    const int rho0 = m0 / a.TQ, c0 = m0 - rho0 * a.TQ;
    const int n0 = rho0 / a.P, oj0 = rho0 - n0 * a.P;
    struct Pixel {
        int n, oj, oi, pos;  // pos: staged position of its tap (0, 0)
        bool ok;
    };
    auto pixel = [&](int ml) {
        Pixel p;
        const int x = c0 + ml, dr = fast_div(x, a.inv_TQ), col = x - dr * a.TQ;
        const int y = oj0 + dr, dn = fast_div(y, a.inv_P);
        p.n = n0 + dn;
        p.oj = y - dn * a.P;
        p.oi = q0 + col;
        p.ok = p.n < a.N && p.oi < a.Q;
        p.pos = !p.ok ? 0 : a.sampled ? ml : (dn * a.Hs + (p.oj - oj0) * a.stride) * a.LW + col * a.stride;
        return p;
    };

    // Staging of the input: share i of a wave is 64 positions of one plane (two channel blocks).
    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const int cpp = (a.LRW + 63) >> 6;  // shares of a plane
    const int plane_bytes = a.PLS * kPosBytes, buf_bytes = 2 * G * plane_bytes;
    unsigned char *const bufs = lds + kw * 2 * buf_bytes;
    unsigned g_off[NI];
    int item_at[NI], item_cb[NI];  // LDS address in a buffer (negative: nothing), first channel block
#pragma unroll
    for (int i = 0; i < NI; ++i) {
        const int c = i * 4 + wave, plane = c / cpp, pos = (c - plane * cpp) * 64 + lane;
        unsigned off = kOutOfRange;
        if (plane < 2 * G && pos < a.LRW) {
            int n, ih, iw;
            bool ok;
            if (a.sampled) {
                const Pixel p = pixel(pos);
                n = p.n;
                ih = p.oj * a.stride;
                iw = p.oi * a.stride;
                ok = p.ok;
            } else {
                const int row = fast_div(pos, a.inv_LW), lam = oj0 * a.stride + row, dn = fast_div(lam, a.inv_Hs);
                n = n0 + dn;
                ih = lam - dn * a.Hs - a.pad_h;
                iw = q0 * a.stride - a.pad_w + (pos - row * a.LW);
                ok = n < a.N && ih >= 0 && ih < a.H && iw >= 0 && iw < a.W;
            }
            if (ok) off = (((unsigned)n * (unsigned)a.Cb * (unsigned)a.H + (unsigned)ih) * (unsigned)a.W + (unsigned)iw) * 16u;
        }
        g_off[i] = off;
        item_at[i] = plane < 2 * G && pos < a.LRW ? plane * plane_bytes + pos * kPosBytes : -1;
        item_cb[i] = 2 * plane;
    }
    // Channel blocks 4*G*st .. of the set's step s (a step beyond the last one has none).
    const int steps = (a.n_stage + KW - 1) / KW;
    const int rot = (int)(((unsigned)kt * (unsigned)a.rot_k + (unsigned)tile * (unsigned)a.rot_m) % (unsigned)steps);
    auto first_block = [&](int s) {
        int sr = s + rot;
        if (sr >= steps) sr -= steps;
        return (sr * KW + kw) * 4 * G;
    };
    u32x4 in_raw[NI][2];
    auto load_item = [&](int i, int s) {
        const int cb = first_block(s) + item_cb[i];
#pragma unroll
        for (int b = 0; b < 2; ++b)
            in_raw[i][b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_in, s < steps && cb + b < a.Cb ? g_off[i] : kOutOfRange,
                                                                 (unsigned)min(cb + b, a.Cb - 1) * (unsigned)HW * 16u, 0);
    };
    auto stage_item = [&](int i, int buf, const Bf16x3 &v) {
        if (item_at[i] >= 0) {
            u32x4 *const at = reinterpret_cast<u32x4 *>(bufs + buf * buf_bytes + item_at[i]);
            at[0] = v.h;
            at[1] = v.m;
            at[2] = v.l;
        }
    };

    // Weights: rows [k0, k0 + 32) of a round's four blocks, two of them to a lane half.  (FW: see put_weights.)
    const int taps = FW ? a.wt_taps : RS;
    const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * taps * a.Kp * 16);
    unsigned w_off[2];
#pragma unroll
    for (int b = 0; b < 2; ++b)
        w_off[b] = FW ? weight_lane_fwd((k0 >> 2) + wt_block(lane) + 4 * b, wt_channel(lane), a.Cb, taps, a.Kp)
                      : weight_lane(k0 + l32, h, b, a.Cb, RS, a.Kp);
    unsigned char *const w_area = lds + KW * 2 * buf_bytes + wave_all * kWtBytes;
    u32x4 w_raw[2];
    int w_step = 0, w_group = 0, w_tap = 0, w_tr = 0, w_ts = 0;  // of the next load
    auto load_weights = [&]() {
        const int cb = first_block(w_step) + 4 * w_group;
        const bool live = w_step < steps && cb < a.Cb;
        const bool mine = live && (!FW || 4 * cb + wt_channel(lane) < 4 * a.Cb);
        const unsigned shared = !live ? 0u
                                : FW  ? weight_shared_fwd(cb, a.wt_tap0 - w_tr * a.wt_dr - w_ts * a.wt_ds, a.Cb)
                                      : weight_shared(cb, w_tap, RS, a.Kp);
#pragma unroll
        for (int b = 0; b < 2; ++b)
            w_raw[b] = __builtin_amdgcn_raw_buffer_load_b128(rsrc_wt, mine ? w_off[b] : kOutOfRange, shared, 0);
        if constexpr (FW) {
            const bool row_end = w_ts + 1 == a.S;
            w_ts = row_end ? 0 : w_ts + 1;
            w_tr = !row_end ? w_tr : w_tr + 1 == a.R ? 0 : w_tr + 1;
        }
        const bool tap_end = w_tap + 1 == RS, step_end = tap_end && w_group + 1 == G;
        w_tap = tap_end ? 0 : w_tap + 1;
        w_group = step_end ? 0 : w_group + (tap_end ? 1 : 0);
        w_step += step_end ? 1 : 0;
    };
    int bpos[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) bpos[j] = h * plane_bytes + pixel((wave_m * FM + j) * 32 + l32).pos * kPosBytes;

    unsigned lost = 0, lost_in = 0;  // bits of the weights and of the input's share that no bf16 number holds
    f32x16 big[FM], small[FM];
#pragma unroll
    for (int j = 0; j < FM; ++j) big[j] = small[j] = f32x16{};

    load_weights();
    static_for<0, NI>([&](auto ic) { load_item(ic, 0); });
    auto weights_landed = [&](const Bf16x3 &w) {
        if constexpr (FW) {
            put_weights(w_area, lane, w);
            return get_weights(w_area, lane);
        } else {
            return w;
        }
    };
    Bf16x3 A = weights_landed(split8<false>(w_raw, lost));
    load_weights();
    static_for<0, NI>([&](auto ic) {
        stage_item(ic, 0, split8<true>(in_raw[ic], lost_in));
        load_item(ic, 1);
    });
    lds_barrier();

    // One round: the MFMAs of a tap of 16 channels; meanwhile the next round's weights are converted and those of the round
    // after requested, and, in the first NI rounds of a step, a share of the next step's input is staged and the
    // same share of the step after requested.  A fragment of pixels is read while the one before it multiplies, the
    // first one of a round at the end of the round before.
    // (Issue order, pinned: an MFMA, then what of the rest fits beside it.  Left to itself the compiler converts first and
    // multiplies then, and reads each fragment right before it is used.)
    u32x4 B[3], ahead[3];
    auto round = [&](int s, const unsigned char *at, const unsigned char *next_at, auto item_tag) {
        constexpr int ITEM = decltype(item_tag)::value;
        // (the weights first, so that the next ones are requested early: they are wanted a round from here)
        constexpr int NP = kSplitProducts, NM = NP * FM, NW = NM / 2;
        Bf16x3 next, item;
        float rest[2];
        static_for<0, NM>([&](auto kc) {
            constexpr int k = decltype(kc)::value, j = k / NP, i = k % NP;
            mma_split<i>(A, Bf16x3{B[0], B[1], B[2]}, big[j], small[j]);
            if constexpr (i < 3) ahead[i] = reinterpret_cast<const u32x4 *>((j + 1 < FM ? at : next_at) + bpos[(j + 1) % FM])[i];
            if constexpr (k < NW)
                static_for<k * kSplitPieces / NW, (k + 1) * kSplitPieces / NW>([&](auto pc) { split_piece<decltype(pc)::value, false>(w_raw, next, rest, lost); });
            if constexpr (k == NW - 1) {
                load_weights();
                next = weights_landed(next);
            }
            if constexpr (ITEM >= 0 && k >= NW)
                static_for<(k - NW) * kSplitPieces / (NM - NW), (k - NW + 1) * kSplitPieces / (NM - NW)>(
                    [&](auto pc) { split_piece<decltype(pc)::value, true>(in_raw[ITEM], item, rest, lost_in); });
            if constexpr (ITEM >= 0 && k == NM - 1) {
                stage_item(ITEM, (s + 1) & 1, item);
                load_item(ITEM, s + 2);
            }
            if constexpr (i == NP - 1) {
#pragma unroll
                for (int t = 0; t < 3; ++t) B[t] = ahead[t];
            }
            __builtin_amdgcn_sched_barrier(0);
        });
        A = next;
    };
    for (int s = 0; s < steps; ++s) {
        const unsigned char *const buf = bufs + (s & 1) * buf_bytes;
        int q = 0, tr = 0, ts = 0, g = 0;
        const unsigned char *at = buf;
        auto advance = [&]() {
            ++q;
            if (++ts == a.S) {
                ts = 0;
                if (++tr == a.R) {
                    tr = 0;
                    g = G == 1 ? 0 : g + 1;
                }
            }
            return buf + (G == 1 || g < G ? g * 2 * plane_bytes : 0) + (tr * a.LW + ts) * kPosBytes;
        };
#pragma unroll
        for (int t = 0; t < 3; ++t) B[t] = reinterpret_cast<const u32x4 *>(at + bpos[0])[t];
        static_for<0, NI>([&](auto ic) {
            if (decltype(ic)::value < G * RS) {
                const unsigned char *const next_at = advance();
                round(s, at, next_at, ic);
                at = next_at;
            } else {  // (a step of few taps)
                stage_item(ic, (s + 1) & 1, split8<true>(in_raw[ic], lost_in));
                load_item(ic, s + 2);
            }
        });
        while (q < G * RS) {
            const unsigned char *const next_at = advance();
            round(s, at, next_at, std::integral_constant<int, -1>{});
            at = next_at;
        }
        lds_barrier();
    }

    mark_if_lost(lost, big);
    // The sets' sums: each adds and stores half of the fragments.
    constexpr int FO = FM / KW;
    static_assert(FM % KW == 0 && KW <= 2, "two sets take half of the fragments each");
    f32x16 acc[FO];
    if constexpr (KW == 1) {
#pragma unroll
        for (int j = 0; j < FO; ++j) acc[j] = big[j] + small[j];
    } else {
        f32x4 *const xch = reinterpret_cast<f32x4 *>(lds) + wave * (FO * 256) + lane;
        auto swap = [&](auto mine) {
            constexpr int M = decltype(mine)::value;
            f32x4 *const to = xch + (1 - M) * (FO * 1024), *const from = xch + M * (FO * 1024);
#pragma unroll
            for (int j = 0; j < FO; ++j) {
                const f32x16 v = big[(1 - M) * FO + j] + small[(1 - M) * FO + j];
#pragma unroll
                for (int q = 0; q < 4; ++q) to[(j * 4 + q) * 64] = f32x4{v[4 * q], v[4 * q + 1], v[4 * q + 2], v[4 * q + 3]};
            }
            lds_barrier();
#pragma unroll
            for (int j = 0; j < FO; ++j) {
                acc[j] = big[M * FO + j] + small[M * FO + j];
#pragma unroll
                for (int q = 0; q < 4; ++q) {
                    const f32x4 v = from[(j * 4 + q) * 64];
#pragma unroll
                    for (int t = 0; t < 4; ++t) acc[j][4 * q + t] += v[t];
                }
            }
        };
        if (kw == 0) swap(std::integral_constant<int, 0>{});
        else swap(std::integral_constant<int, 1>{});
    }

    // ---- store: a lane owns one pixel and, per eight channel rows, four consecutive channels (a block)
    typedef Elem<CONV_F32> E_;
    const size_t oplane = (size_t)a.OH * a.OW * 16;
    const size_t out_bytes = (size_t)a.N * a.out_kb * oplane;
    const rsrc_t ro = make_rsrc(a.out, 0, out_bytes);
    const rsrc_t rres = make_rsrc(a.resid ? a.resid : a.out, 0, out_bytes);
    const int m_wave = (wave_m * FM + kw * FO) * 32 + l32;
    const bool fused = a.scale != nullptr || a.bias != nullptr || a.resid != nullptr || a.relu != 0;
    auto place = [&](const Pixel &p) {
        return p.ok ? (((unsigned)p.n * (unsigned)a.out_kb * (unsigned)a.OH + (unsigned)(p.oj * a.ostr + a.oy0)) * (unsigned)a.OW +
                       (unsigned)(p.oi * a.ostr + a.ox0)) * 16u + (unsigned)h * (unsigned)oplane
                    : kOutOfRange;
    };
    // (rows beyond the last block of a lane half: nothing)
    auto live_at = [&](unsigned at, int vq) { return k0 + 8 * vq + 4 * h < a.Kp ? at : kOutOfRange; };
    auto skip_of = [&](int vq) { return (unsigned)((k0 + 8 * vq) / 4) * (unsigned)oplane; };
    auto store_fused = [&](const f32x16 &v, unsigned at, const f32x4 (&r)[4]) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            const int row = k0 + 8 * vq + 4 * h;
            f32x4 g = {1.f, 1.f, 1.f, 1.f}, b = {0.f, 0.f, 0.f, 0.f};
            if (a.scale && row < a.Kp) g = *reinterpret_cast<const f32x4 *>(a.scale + row);
            if (a.bias && row < a.Kp) b = *reinterpret_cast<const f32x4 *>(a.bias + row);
            float o[4];
#pragma unroll
            for (int t = 0; t < 4; ++t) {
                o[t] = v[4 * vq + t] * g[t] + r[vq][t] + b[t];
                if (a.relu) o[t] = fmaxf(o[t], 0.0f);
            }
            E_::store4<CONVMI_OUT_POLICY>(ro, live_at(at, vq), skip_of(vq), o[0], o[1], o[2], o[3]);
        }
    };
    auto store_plain = [&](const f32x16 &v, const Pixel &p, unsigned at) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq) {
            const unsigned off = live_at(at, vq);
            if (!a.zero_fill && a.ostr == 1) {
                E_::store4<CONVMI_OUT_POLICY>(ro, off, skip_of(vq), v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]);
                continue;
            }
            E_::store4(ro, off, skip_of(vq), v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]);
            if (a.zero_fill)
                for (int dy = 0; dy < a.ostr; ++dy)
                    for (int dx = 0; dx < a.ostr; ++dx) {
                        if ((dy | dx) == 0) continue;
                        const bool in = off != kOutOfRange && p.oj * a.ostr + a.oy0 + dy < a.OH && p.oi * a.ostr + a.ox0 + dx < a.OW;
                        E_::store4(ro, in ? off + (unsigned)(dy * a.OW + dx) * 16u : kOutOfRange, skip_of(vq), 0.f, 0.f, 0.f, 0.f);
                    }
        }
    };
    auto residual = [&](unsigned at, f32x4 (&r)[4]) {
#pragma unroll
        for (int vq = 0; vq < 4; ++vq)
            r[vq] = a.resid ? __builtin_bit_cast(f32x4, __builtin_amdgcn_raw_buffer_load_b128(rres, live_at(at, vq), skip_of(vq), 0))
                            : f32x4{0.f, 0.f, 0.f, 0.f};
    };

    float most = 0.0f;
#pragma unroll
    for (int j = 0; j < FO; ++j) most = max_magnitude(most, acc[j]);
    if (__builtin_expect(!sums_need_fp32(most), 1)) {
        if (fused) {
            unsigned at[FO];
            f32x4 r[FO][4];  // (all requested before the first store: the residual may be the output)
#pragma unroll
            for (int j = 0; j < FO; ++j) {
                at[j] = place(pixel(m_wave + j * 32));
                residual(at[j], r[j]);
            }
#pragma unroll
            for (int j = 0; j < FO; ++j) store_fused(acc[j], at[j], r[j]);
        } else {
#pragma unroll
            for (int j = 0; j < FO; ++j) {
                const Pixel p = pixel(m_wave + j * 32);
                store_plain(acc[j], p, place(p));
            }
        }
        return;
    }
    // Infinite or NaN sums: all of the wave's again.
    for (int j = 0; j < FO; ++j) {
        const Pixel p = pixel(m_wave + j * 32);
        const unsigned at = place(p);
        f32x16 v = fragment_in_fp32<FW>(a, p.n, p.oj, p.oi, p.ok, k0 + l32, 0, (a.Cb + 3) / 4 * RS);
        if (a.exact && p.ok)
#pragma unroll
            for (int vq = 0; vq < 4; ++vq) {
                const int row = k0 + 8 * vq + 4 * h;
                const f32x4 was = {v[4 * vq], v[4 * vq + 1], v[4 * vq + 2], v[4 * vq + 3]};
                if (row >= a.Kp || !any_nan(was)) continue;
                const f32x4 x = sum_inside_image<CONV_F32, 4, FW>(a, p.n, p.oj, p.oi, row, 0, (a.Cb + 3) / 4 * RS);
#pragma unroll
                for (int t = 0; t < 4; ++t) v[4 * vq + t] = x[t];
            }
        if (fused) {
            f32x4 r[4];
            residual(at, r);
            store_fused(v, at, r);
        } else {
            store_plain(v, p, at);
        }
    }
}

template <int WK, int WM, int FM, int KW, int G, int NI, bool FW>
__global__ __launch_bounds__(256 * KW, KW == 1 ? 2 : 1) void igemm_split_kernel(const IgemmArgs a)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    igemm_split_tile<WK, WM, FM, KW, G, NI, FW>(a, blockIdx.x, lds);
}

// Up to four launches in one: the residue classes of a strided backward pass, on the forward pass's weights.
template <int WK, int WM, int FM, int KW, int G, int NI>
__global__ __launch_bounds__(256 * KW, KW == 1 ? 2 : 1) void igemm_split_classes_kernel(const IgemmSplitClasses c)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    int bid = blockIdx.x, i = 0;
    while (i < 3 && bid >= c.end[i]) ++i;
    if (i > 0) bid -= c.end[i - 1];
    igemm_split_tile<WK, WM, FM, KW, G, NI, true>(c.cls[i], bid, lds);
}

struct SplitEntry {
    int wk, wm, fm, kw, g, ni;
    igemm_fn_t fn;
};
const SplitEntry *igemm_split_fwd_wt_entries(int *count);  // on the forward pass's weights

#define SPLIT_ENTRY(WK, WM, FM, KW, G, NI) {WK, WM, FM, KW, G, NI, igemm_split_kernel<WK, WM, FM, KW, G, NI, SPLIT_FW>}
#define SPLIT_ENTRIES(WK, WM, FM, KW) \
    SPLIT_ENTRY(WK, WM, FM, KW, 1, 1), SPLIT_ENTRY(WK, WM, FM, KW, 1, 2), SPLIT_ENTRY(WK, WM, FM, KW, 1, 3), \
    SPLIT_ENTRY(WK, WM, FM, KW, 1, 4), SPLIT_ENTRY(WK, WM, FM, KW, 2, FM * WM / 2)
#define SPLIT_TABLE \
    SPLIT_ENTRIES(4, 1, 4, 1), SPLIT_ENTRIES(4, 1, 2, 1), SPLIT_ENTRIES(2, 2, 4, 1), SPLIT_ENTRIES(2, 2, 2, 1), \
    SPLIT_ENTRIES(4, 1, 4, 2), SPLIT_ENTRIES(4, 1, 2, 2), SPLIT_ENTRIES(2, 2, 4, 2), SPLIT_ENTRIES(2, 2, 2, 2), \
    SPLIT_ENTRY(4, 1, 2, 1, 1, 5), SPLIT_ENTRY(4, 1, 2, 1, 1, 6), SPLIT_ENTRY(2, 2, 2, 1, 1, 5), SPLIT_ENTRY(2, 2, 2, 1, 1, 6), \
    SPLIT_ENTRY(4, 1, 2, 2, 1, 5)

}  // namespace convmi
