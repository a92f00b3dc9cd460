// C ABI of libconv_mi355x: descriptor validation and per-layer planning (done
// once at conv_create, the analogue of the dryrun phase of Section II-H),
// and the entry points that only enqueue kernels.
#include <stdio.h>
#include <stdlib.h>
#include <string.h>

#include <algorithm>
#include <mutex>
#include <new>
#include <numeric>
#include <unordered_map>

#include "conv_internal.h"

using namespace convmi;

namespace convmi {
hipError_t ensure_dynamic_lds(const void *kernel, size_t bytes)
{
    static std::mutex mu;
    static std::unordered_map<const void *, size_t> have;
    std::lock_guard<std::mutex> lock(mu);
    size_t &cur = have[kernel];
    if (bytes <= cur) return hipSuccess;
    const hipError_t err =
        hipFuncSetAttribute(kernel, hipFuncAttributeMaxDynamicSharedMemorySize, (int)bytes);
    if (err == hipSuccess) cur = bytes;
    return err;
}
}  // namespace convmi

namespace {

// fp32 on the bf16 matrix instructions (igemm_split.hip), in the place of an IgemmPlan's kernel.
struct SplitPlan {
    bool ok = false;
    IgemmSplitVariant v{};
    int fk = 0, fm = 0, nw = 0;  // nw > 0: the register-operand kernel's form of it
    IgemmArgs a{};
    size_t lds = 0;
    int grid = 0;
};

struct IgemmPlan {
    bool ok = false;
    IgemmVariant v{};
    IgemmArgs a{};
    size_t lds = 0;
    int grid = 0;
    bool reg = false;  // the register-operand kernel (v.wk waves split the reduction of a tile)
    bool patch = false;  // ... with the pixels in LDS (reg is set too)
    bool fallback = false;  // ... because no staged tile fits (IgemmGeo::fallback)
};

// The same for a weight update (upd_split.hip).
struct UpdSplitPlan {
    bool ok = false;
    UpdSplitVariant v{};
    UpdArgs a{};
    int grid = 0;
};

// ... and of bf16 tensors (upd_shared.hip).
struct UpdSharedPlan {
    bool ok = false;
    UpdSharedVariant v{};
    UpdArgs a{};
    int grid = 0;
};

// The residue classes of a strided backward pass in one launch on the bf16 instructions.
struct SplitClassesPlan {
    bool ok = false;
    IgemmSplitVariant v{};
    IgemmSplitClasses c{};
    size_t lds = 0;
};

struct BwdClass {  // one stride-parity class of the generic backward pass
    IgemmPlan p;
    WtXformArgs x{};
    WtMergeArgs m{};      // all classes in one launch (merged == true)
    bool merged = false;
    size_t ws_off = 0;
    size_t part_off = 0;  // of the partial results of a split reduction (p.a.ksplit > 1)
};

}  // namespace

struct conv_plan {
    conv_desc_t d;
    int pad_h = 0, pad_w = 0;  // zero padding per axis (d.pad is not used past conv_create)
    conv_info_t info;
    IgemmPlan fwd;
    size_t fwd_ws = 0;  // bytes of fp32 partial results if the forward reduction is split
    SplitPlan fwd_split;      // runs in the place of fwd (fp32)
    size_t fwd_stem_lds = 0;  // > 0: the plain forward pass runs on the resident-filter kernel (its LDS)
    // backward by data
    int bwd_mode = 0;  // 0 unsupported, 1 one launch (duality), 2 parity classes
    int n_bwd = 0;
    bool bwd_quad = false;  // four classes (2x2, 2x1, 1x2, 1x1 taps, in this order) in one launch
    BwdClass bwd[16];
    IgemmStreamPlan fwd_stream, bwd_stream;  // ... (bf16, nothing fused)
    SplitPlan bwd_split;  // runs in the place of a single launch's plan (fp32)
    SplitClassesPlan bwd_classes;  // runs in the place of all that
    size_t bwd_ws = 0;
    // (a backward pass that would run untiled but for the register-operand kernel, which takes a
    // workspace: a caller that brings none still gets the untiled kernel)
    bool bwd_ws_optional = false;
    // weight update
    bool upd_ok = false;
    bool upd_c4 = false;   // few-channel formulation (one input channel block)
    bool upd_c4_bf16 = false; // bf16, one input channel block: (tap, channel) rows on the bf16 MFMA
    bool upd_rows = false; // bf16 row kernel (stride 1)
    int upd_bands_layout = 0;  // fp32 band kernel: 0 = 2x2 channel waves x 2 pixel groups, 1 = 1x2x4, 2 = 1x1x8
    bool upd_bands = false; // fp32 eight-wave band kernel
    bool upd_flat_bf16 = false; // bf16 1x1 eight-wave kernel on the flat pixel list (variant: urv)
    bool upd_flat = false;  // fp32 1x1 eight-wave kernel on the flat pixel list
    int upd_wb = 0;         //   its waves along the narrower tensor's channels
    bool upd_a_is_in = false; //   whether the wider tensor is the input
    UpdRowsVariant urv{};
    bool upd_window = false;  // ... with one window of the input for all taps (bf16)
    bool upd_ring = false;  // small blocks of dW, the waves split the pixels (fragments: urv.fc, urv.fk)
    int upd_copies = 0;    // partial dW copies the reduce kernel sums
    UpdVariant uv{};
    int upd_row_launches = 1;  // > 1: one launch of a 1 x S kernel per filter row
    int upd_strips = 1;        // general kernels: strips of output columns, one launch each
    int upd_strip_w = 0;       // ... their width (the last may be narrower)
    UpdArgs ua{};
    double upd_ring_us = 0;  // what the ring kernel's plan takes by estimate
    UpdSplitPlan upd_split;    // runs in the place of all that (fp32)
    UpdSharedPlan upd_shared;  // ... (bf16)
    size_t upd_lds = 0;
    int upd_grid = 0;
    size_t upd_ws = 0;
    // passes no tiled kernel fits run on the untiled direct kernels (no workspace)
    bool fwd_direct = false, bwd_direct = false, upd_direct = false;
    DirectArgs da{};
    // The minibatch in chunks of chunk_n images (the last chunk has the rest), each a plan of
    // its own run on its slice of the tensors: for tensors beyond the tiled kernels' 32-bit
    // byte offsets, or on request.  n_chunks == 0: none.
    int n_chunks = 0, chunk_n = 0;
    conv_plan *chunk = nullptr, *tail = nullptr;  // owned; tail: the last chunk if it is smaller
    bool fwd_chunked = false, bwd_chunked = false, upd_chunked = false;
    size_t chunk_ws = 0;  // the chunks' own workspace; the per-chunk dW results follow it
    ~conv_plan()
    {
        delete chunk;
        delete tail;
    }
};

namespace {

const int kMaxLds = 160 * 1024;
constexpr size_t kScratchBytes = (size_t)16 << 20;  // conv_noalloc_scratch_bytes

// Largest number of rows of the padded row space (image n occupies rows
// [n*Hs, (n+1)*Hs), output row oj of image n starts at n*Hs + oj*stride) that a
// band of TR consecutive linear output rows touches with an R-tall filter.
int max_band_rows(int N, int P, int TR, int Hs, int stride, int R)
{
    // A band's extent depends on the row it starts at within its image, rho0 % P, and those
    // repeat after at most P bands: the first P bands hold the maximum (the last band of the
    // row space can only be shorter than an earlier one of the same phase).
    const long long NP = (long long)N * P;
    const long long bands = std::min<long long>((NP + TR - 1) / TR, P);
    long long best = 0;
    for (long long b = 0; b < bands; ++b) {
        const long long rho0 = b * TR, rho1 = std::min(NP, rho0 + TR) - 1;
        const long long lam0 = (rho0 / P) * Hs + (rho0 % P) * stride;
        const long long lam1 = (rho1 / P) * Hs + (rho1 % P) * stride + R - 1;
        best = std::max(best, lam1 - lam0 + 1);
    }
    return (int)std::min<long long>(best, 1 << 30);
}

// Rounding error of fp32 sums, as far as comparing two orders of the same sum goes: a chain of n additions of
// random terms has an error variance of n/2 in units of one rounding of its result, and the levels of a
// sum add up.  (A chain's additions are its products in fp32, of which an MFMA rounds each, and its MFMAs in
// bf16, which round once.)  A kernel that takes a launch over from another one may not have the larger error: it sums
// in groups where one chain would be too long, or stays out.  (Measured over 75 layers at N = 1 ... 160 against
// 64 bits: the ratio of two orders' errors is within 20 % of the root of the ratio of these figures, and
// nearer to 1 where both are small, where the result's own rounding counts: a half.  Groups aim
// below the old figure by that much, a plan that cannot reach this is taken up to the old figure.)
constexpr double kErrorMargin = 0.7, kOwnRounding = 0.5;
double chain_error(double n, double group) { return group > 0 && n > group ? group / 2 + n / (2 * group) : n / 2; }
// The largest group, in whole units of `unit` additions, with which n additions stay within `most` (the best
// one if none does); 0 if one chain does.
int group_within(double n, double unit, double most)
{
    if (n / 2 <= most) return 0;
    const double root = most * most - n;
    const double g = root > 0 ? (most + std::sqrt(root)) / unit : std::sqrt(n) / unit + 0.5;
    return std::max(1, (int)g);
}

// Whether the forward and backward kernels' 32-bit byte offsets (and the 32-bit size of a buffer
// resource) reach all of the weights; conv_create takes up to 2^31 of them, 8 GB in fp32.
bool weights_reach(int Cb, int Kp, int R, int S) { return (double)Cb * R * S * Kp * 16 <= 4.0e9; }

// The launch reads the forward pass's weights: a filter of `taps` taps, of which its tap (0, 0) is tap0, dr and ds taps
// up from those of the next row and column.  False, and nothing is set, if they are out of reach: a residue class of a
// strided pass addresses all taps, though its own sub-filter has at most four of nine.
bool forward_weights(IgemmArgs &a, int taps, int tap0, int dr, int ds)
{
    if (!weights_reach(a.Cb, a.Kp, taps, 1)) return false;
    a.fwd_wt = 1;
    a.wt_taps = taps;
    a.wt_tap0 = tap0;
    a.wt_dr = dr;
    a.wt_ds = ds;
    return true;
}

// One candidate plan of the implicit-GEMM kernel: `wk` waves along channels,
// dynamic LDS at most `lds_cap` bytes.  Returns ok=false if nothing fits.
IgemmPlan try_igemm(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S,
                    int stride, int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0,
                    int zero_fill, const IgemmGeo &geo, int wk, int wm, int fk, int fm, size_t lds_cap,
                    int nb = 2, int npl_want = 0, int ppt_only = 0)
{
    IgemmPlan pl;
    // (columns of the result `cstride` input pixels apart, and `ostr_x` output pixels apart)
    const int cstride = geo.cstride > 0 ? geo.cstride : stride;
    const int ostr_x = geo.ostr_x > 0 ? geo.ostr_x : ostr;
    const int V = vlen_of(dtype);
    // (1x1, no padding: only the pixels that are read are staged -- valid where every output
    // pixel has its input pixel; a residue class of a strided backward pass can be one row or
    // column larger than its input, which then needs the zero rows of the padded row space)
    const bool sampled = (R == 1 && S == 1 && pad_h == 0 && pad_w == 0 && (P - 1) * stride < H &&
                          (Q - 1) * stride < W);

    int npl;
    if (R == 1 && S == 1)
        npl = (Cb % 4 == 0) ? 4 : 1;
    else
        npl = (Cb % 2 == 0) ? 2 : 1;
    if (npl_want > 0) {
        if (Cb % npl_want != 0) return pl;
        npl = npl_want;
    }
    // (eight waves: two groups of four, each staging its half of a step's planes)
    if (wk * wm == 8 && npl % 2 != 0) return pl;

    // (NT: threads of one staging group -- the input tile's chunks are dealt per group)
    const int TK = wk * fk * 32, TM = wm * fm * 32, NT = 256;
    const int nent = ((R * S * npl + 1) / 2) * 2;

    // (staged positions per thread that the variant is instantiated for)
    const unsigned have_ppt =
        ppt_only > 0 ? 1u << ppt_only : igemm_variant_ppts(IgemmVariant{dtype, wk, wm, fk, fm, npl, R, S, 0, nb});
    if (have_ppt == 0) return pl;
    int ppt = -1;
    int TQ = std::min(Q, TM);
    int TR = std::max(1, TM / TQ);
    TR = std::min(TR, N * P);
    int Hs = 0, LW = 0, LR = 0;
    for (;; --TR) {
        if (TR < 1) return pl;
        if (sampled) {
            Hs = P;
            LW = TQ;
            LR = TR;
        } else {
            Hs = (P - 1) * stride + R;
            LW = (TQ - 1) * cstride + S;
            LR = max_band_rows(N, P, TR, Hs, stride, R);
        }
        ppt = -1;
        for (int cand = 0; cand <= 16 && ppt < 0; ++cand)
            if ((have_ppt >> cand & 1) && (long long)LR * LW <= (cand == 0 ? NT / 2 : (long long)cand * NT)) ppt = cand;
        if (ppt < 0) continue;
        // the plane pitch is a whole number of wave-level (64-lane) loads
        // (a single-step reduction never touches the second buffer)
        const size_t nbuf = ceil_div(Cb, npl) > 1 ? (size_t)nb : 1;
        const size_t lds = nbuf * ((size_t)nent * TK * 16 + (size_t)npl * ceil_div(LR * LW, 64) * 64 * 16);
        if (lds <= lds_cap) break;
    }

    IgemmArgs &a = pl.a;
    memset(&a, 0, sizeof(a));
    a.N = N; a.Cb = Cb; a.H = H; a.W = W; a.Kp = Kp; a.P = P; a.Q = Q;
    a.stride = stride; a.cstride = cstride; a.pad_h = pad_h; a.pad_w = pad_w;
    a.OH = OH; a.OW = OW; a.ostr = ostr; a.ostr_x = ostr_x; a.oy0 = oy0; a.ox0 = ox0; a.zero_fill = zero_fill;
    a.shuffle = 0; a.out_kb = Kp / V;
    a.ksplit = 1;
    a.scale = nullptr; a.bias = nullptr; a.resid = nullptr; a.relu = 0;
    a.TR = TR; a.TQ = TQ;
    a.n_qt = ceil_div(Q, TQ);
    a.n_mt = ceil_div(N * P, TR);
    a.n_kt = ceil_div(Kp, TK);
    a.Hs = Hs; a.LW = LW; a.LRW = LR * LW; a.PLS = ceil_div(LR * LW, 64) * 64;
    a.sampled = sampled ? 1 : 0;
    a.inv_P = 1.0f / (float)P; a.inv_Hs = 1.0f / (float)Hs;
    a.inv_LW = 1.0f / (float)LW; a.inv_TQ = 1.0f / (float)TQ;
    a.total = a.n_mt * a.n_qt * a.n_kt;
    {
        // Tiles over the XCDs (see the kernel): bytes from beyond the L2s are about
        // gk x input + (8/gk) x weights, provided an XCD's share of the weights (1/gk of
        // them) leaves room in its 4 MB L2 for the input tiles in flight.
        const double in_b = (double)N * Cb * (sampled ? (double)P * Q : (double)H * W) * 16.0;
        const double wt_b = (double)Cb * R * S * Kp * 16.0;
        int best_gk = 1;
        double best = 0;
        for (int gk = 1; gk <= 8; gk *= 2) {
            if (gk > a.n_kt) break;
            if (a.n_kt % gk != 0 && gk > 1) continue;
            double cost = gk * in_b + (8.0 / gk) * wt_b;
            if (wt_b / gk > 2.0e6) cost += 8.0 * in_b;  // the weights would not stay resident
            if (gk == 1 || cost < best) { best = cost; best_gk = gk; }
        }
        if (const char *env = getenv("CONVMI_IGEMM_GK")) {
            const int g = atoi(env);
            if ((g == 1 || g == 2 || g == 4 || g == 8) && g <= a.n_kt && a.n_kt % g == 0) best_gk = g;
        }
        a.gk = best_gk;
        a.kt_per = ceil_div(a.n_kt, a.gk);
        a.mq_per = ceil_div(a.n_mt * a.n_qt, 8 / a.gk);
        a.per_xcd = a.kt_per * a.mq_per;
        // (one channel group: equal shares; whole pixel tiles, which no two XCDs read, for bf16 1x1 without scatter where that
        // costs no CU a tile more -- 512 -> 1024 stride 2 at 28x28, N = 24, 14.0 -> 12.0 us, forward passes 0.86 - 1.01,
        // backward 0.92 - 1.02; else 0.98 - 1.06: 448 -> 384 3x3 at 8x8, N = 224, 41 -> 44)
        const int equal = ceil_div(a.total, 8);
        const bool whole = dtype == CONV_BF16 && R * S == 1 && ostr == 1 && ceil_div(a.per_xcd, 32) == ceil_div(equal, 32);
        if (a.gk == 1 && !whole) a.per_xcd = equal;
    }
    a.n_stage = ceil_div(Cb, npl);
    a.st_per = a.n_stage;
    // (measured at N = 256, bf16, operands not in cache: 6 - 13 % on the forward pass of the deep
    // 1x1 layers, nothing lost elsewhere; CONVMI_IGEMM_ROT="rk,rm" overrides, a tuning aid)
    a.rot_k = 1;
    a.rot_m = 1;
    if (const char *env = getenv("CONVMI_IGEMM_ROT")) {
        int rk = 0, rm = 0;
        if (sscanf(env, "%d,%d", &rk, &rm) == 2 && rk >= 0 && rm >= 0) { a.rot_k = rk; a.rot_m = rm; }
    }
    pl.v = IgemmVariant{dtype, wk, wm, fk, fm, npl, R, S, ppt, nb};
    if (geo.fwd_wt) {
        IgemmVariant w = pl.v;
        w.fw = 1;
        if (igemm_variant_exists(w) && forward_weights(a, R * S, R * S - 1, S, 1)) pl.v = w;
    }
    pl.lds = (a.n_stage > 1 ? nb : 1) * ((size_t)nent * TK * 16 + (size_t)npl * a.PLS * 16);
    pl.grid = a.per_xcd * 8;
    // 32-bit index guards (offsets are kept in 16-byte units / elements)
    // tensors are addressed with 32-bit byte offsets
    const double in_units = (double)N * Cb * H * W, out_units = (double)N * (Kp / V) * OH * OW;
    if (in_units * 16 > 4.0e9 || out_units * 16 > 4.0e9 || !weights_reach(Cb, Kp, R, S)) return pl;
    // the kernels divide small indices through a float reciprocal, exact below 2^22
    if ((double)(N + 1) * std::max(Hs, P) >= 4.0e6 || a.LRW >= (1 << 22)) return pl;
    // ... and multiply row indices (image x channel block x row) as 24-bit integers
    if ((double)(N + 1) * std::max(Cb, Kp / V) * std::max(std::max(H, OH), Hs) >= 8.0e6) return pl;
    pl.ok = true;
    return pl;
}

// MFMA work a plan issues relative to the useful work: padded pixel slots of
// the tiles and padded channel rows both cost full MFMA time.
double igemm_waste(const IgemmPlan &p, int N, int P, int Q, int Kp)
{
    const double TM = p.v.wm * p.v.fm * 32.0, TK = p.v.wk * p.v.fk * 32.0;
    return (p.a.n_mt * p.a.n_qt * TM * p.a.n_kt * TK) / ((double)N * P * Q * Kp);
}

// A plan of the register-operand kernel: fk x fm fragments per workgroup, nw waves (and, with
// ksplit > 1, that many workgroups) that split the reduction.
IgemmPlan try_reg(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S, int stride,
                  int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0, int zero_fill,
                  const IgemmGeo &geo, int fk, int fm, int nw, int ksplit, int patch_fk = 0)
{
    IgemmPlan pl;
    if (patch_fk > 0) fk = patch_fk;  // (the patch kernel's plan: variants of its own)
    else if (igemm_reg_depth(dtype, fk, fm, nw) == 0) return pl;
    const int V = vlen_of(dtype);
    // 32-bit byte offsets, exact small divisions and 24-bit products, as in try_igemm
    const double in_units = (double)N * Cb * H * W, out_units = (double)N * (Kp / V) * OH * OW;
    const double shift = std::max(0.0, (double)pad_h * W + pad_w);
    if ((in_units + shift) * 16 > 4.0e9 || out_units * 16 > 4.0e9 || !weights_reach(Cb, Kp, R, S)) return pl;
    if ((double)N * P * Q + fm * 32 >= 4.0e6 || (double)R * S * Kp >= 8.0e6) return pl;
    if ((double)(N + 1) * std::max(Cb + 1, Kp / V) * std::max(H, OH) >= 8.0e6) return pl;
    IgemmArgs &a = pl.a;
    memset(&a, 0, sizeof(a));
    a.N = N; a.Cb = Cb; a.H = H; a.W = W; a.Kp = Kp; a.P = P; a.Q = Q; a.R = R; a.S = S;
    a.stride = stride; a.cstride = geo.cstride > 0 ? geo.cstride : stride; a.pad_h = pad_h; a.pad_w = pad_w;
    a.OH = OH; a.OW = OW; a.ostr = ostr; a.ostr_x = geo.ostr_x > 0 ? geo.ostr_x : ostr;
    a.oy0 = oy0; a.ox0 = ox0; a.zero_fill = zero_fill;
    a.out_kb = Kp / V;
    a.exact = geo.fallback ? 1 : 0;
    a.no_taps = geo.no_taps ? 1 : 0;
    a.fwd_wt = geo.fwd_wt && dtype == CONV_BF16 && !geo.fallback ? 1 : 0;
    a.inv_P = 1.0f / (float)(P * Q);
    a.inv_TQ = 1.0f / (float)Q;
    a.n_qt = 1;
    a.n_mt = ceil_div(N * P * Q, fm * 32);
    a.n_kt = ceil_div(Kp, fk * 32);
    a.total = a.n_mt * a.n_kt;
    a.n_stage = ceil_div(Cb, 2) * R * S;
    a.st_per = ceil_div(a.n_stage, ksplit);
    a.ksplit = ceil_div(a.n_stage, a.st_per);
    // channel groups over the XCDs, as in try_igemm
    const double in_b = in_units * 16, wt_b = (double)Cb * R * S * Kp * 16.0;
    double best = 0;
    a.gk = 1;
    for (int gk = 1; gk <= 8 && gk <= a.n_kt && a.ksplit == 1; gk *= 2) {
        if (a.n_kt % gk != 0) continue;
        double cost = gk * in_b + (8.0 / gk) * wt_b;
        if (wt_b / gk > 2.0e6) cost += 8.0 * in_b;
        if (gk == 1 || cost < best) { best = cost; a.gk = gk; }
    }
    a.kt_per = ceil_div(a.n_kt, a.gk);
    a.mq_per = ceil_div(a.n_mt, 8 / a.gk);
    a.per_xcd = a.gk == 1 ? ceil_div(a.total * a.ksplit, 8) : a.kt_per * a.mq_per;
    pl.v = IgemmVariant{dtype, nw, 1, fk, fm, 2, R, S, 0};
    pl.lds = igemm_reg_lds_bytes(fk, fm, nw, a.fwd_wt != 0);
    pl.grid = a.per_xcd * 8;
    pl.reg = true;
    pl.fallback = geo.fallback;
    pl.ok = true;
    return pl;
}

// The most input positions from the first to the last of `tile` consecutive pixels of an N x P x Q result whose rows lie
// `row` positions apart, whose columns `col` and whose images HW.  Stops once it is beyond `most`.
// Tiles start at every multiple of the tile in turn, which repeats after P*Q / gcd(P*Q, tile) of them.  Of two tiles, what
// differs is whether they cross one row and one image more, so the walk over the starts ends where one has both that add
// (231 x 165 pixels under 1x7, N = 64: conv_create took 4 ms to divide its way through 36 000 starts for each variant, 0.1 now).
long long longest_run(int N, int P, int Q, long long row, long long col, long long HW, int tile, long long most)
{
    const int PQ = P * Q, npix = N * PQ, tiles = ceil_div(npix, tile);
    const int period = std::min(tiles, PQ / std::gcd(PQ, tile)), whole = std::min(period, npix / tile);
    const int n = (tile - 1) / PQ, rest = (tile - 1) % PQ, a = (tile - 1) / Q, b = (tile - 1) % Q;
    const long long least = a * row + n * (HW - P * row) + b * col, by_row = row - Q * col, by_image = HW - P * row;
    const long long bound = least + (b > 0 ? std::max(by_row, 0LL) : 0) + (rest > 0 ? std::max(by_image, 0LL) : 0);
    long long longest = 0;
    const int step_x = tile % PQ, step_c = tile % Q;
    for (int t = 0, x = 0, c = 0; t < whole && longest < bound && longest <= most; ++t) {
        longest = std::max(longest, least + (c + b >= Q ? by_row : 0) + (x + rest >= PQ ? by_image : 0));
        if ((x += step_x) >= PQ) x -= PQ;
        if ((c += step_c) >= Q) c -= Q;
    }
    if (whole < period) {  // (the last one, which is not whole)
        auto pos = [&](int m) { return m / PQ * HW + m % PQ / Q * row + m % Q * col; };
        longest = std::max(longest, pos(npix - 1) - pos(whole * tile));
    }
    return longest;
}

// The same with the pixels in LDS, for filters of several taps.
IgemmPlan try_patch(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S, int stride,
                    int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0, int zero_fill,
                    const IgemmGeo &geo, int fk, int fm, int nw)
{
    IgemmPlan pl;
    if (geo.fallback || !igemm_patch_exists(dtype, R * S, fk, fm, nw)) return pl;
    IgemmPlan c = try_reg(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0, zero_fill,
                          geo, 0, fm, nw, 1, fk);
    if (!c.ok) return pl;
    IgemmArgs &a = c.a;
    // (the patch is a run of the flat input list: its pixels' order is that of the result's)
    const long long HW = (long long)H * W;
    if ((P - 1) * (long long)stride * W + (Q - 1) * (long long)a.cstride >= HW || (long long)stride * W <= (Q - 1) * (long long)a.cstride)
        return pl;
    // exact small divisions
    if ((double)N * HW >= 4.0e6) return pl;
    // the longest patch
    const int most = 64 * kPatchLoads - ((R - 1) * W + S);
    const long long longest = longest_run(N, P, Q, (long long)stride * W, a.cstride, HW, fm * 32, most);
    if (longest > most) return pl;
    a.PLS = ceil_div((int)longest + (R - 1) * W + S, 64) * 64;
    a.inv_Hs = 1.0f / (float)HW;
    a.fwd_wt = geo.fwd_wt ? 1 : 0;
    c.lds = igemm_patch_lds_bytes(fk, fm, nw, a.PLS, geo.fwd_wt);
    if (c.lds > (size_t)kMaxLds) return pl;
    c.patch = true;
    return c;
}

// What a plan's launch takes, in microseconds, as far as the choice between kernels and tiles goes.
// A workgroup alone on its CU takes `lone` clocks: a fixed part (set-up, first loads, stores) and
// its steps, each bound by what it asks of the matrix cores, of the 64 B/clk into the CU or of
// the LDS reads, whichever is slowest; workgroups that share a CU share those, `busy` clocks
// each, and overlap the rest.  The CU with the most workgroups ends the launch.  The constants
// are a least-squares fit (log of the time) to 4 300 launches: 34 ResNet-50 and Inception-v3
// layers x N = 1 ... 128 x both types x every variant, three sets of tensors in turn; rms error
// 6 - 15 %.  The plan with the lowest estimate was on average 1 % (fp32) and 2 % (bf16) behind the
// fastest variant, and took 0.61 times as long as the large tiles that these sizes ran on before, their
// reduction split through memory (0.55 / 0.29 times as long as those without the split).
double estimate_patch_us(const IgemmPlan &p);
double sums_error(const IgemmPlan &p);
double estimate_us(const IgemmPlan &p, bool scatter)
{
    if (p.patch) return estimate_patch_us(p);
    const IgemmArgs &a = p.a;
    const IgemmVariant &v = p.v;
    const bool bf16 = v.dtype == CONV_BF16;
    const double mfma = bf16 ? 32.0 : 256.0;  // clocks of the MFMAs of one 16-byte operand pair
    const double frags = v.fk * v.fm;
    const int RS = p.reg ? a.R * a.S : v.r * v.s;
    struct Fit { double launch, fixed, step, c_mfma, c_load, c_read, busy; };
    double lone, busy, launch, hbm = 4.8e6;
    int resident;
    bool large = false;  // 224 or more pixels, or 64 x 512: a workgroup or two to a CU
    if (p.reg) {
        // (c_read: the exchange of the waves' sums, clocks per tile and wave)
        const Fit f = bf16 ? Fit{2.6, 0, 256, 0, 1.26, 284, 1480} : Fit{3.9, 0, 441, 1.22, 1.2, 0, 1300};
        const double per = ceil_div(a.st_per, v.wk);  // steps of a wave
        const double simd_waves = v.wk / 4;
        // (the forward pass's weights through LDS: fitted to 1 930 launches, rms error 11 %, whole rounds of its ring)
        const Fit w = {3.0, 0, 400, 1.3, 1.16, 248, 870};
        const double rounds = ceil_div((int)per, 4) * 4;
        const double shared = std::max({frags * mfma * w.c_mfma * simd_waves, v.wk * (v.fk + v.fm) * 16.0 * w.c_load,
                                        v.wk * v.fk * 16.0 * 0.67});
        if (a.fwd_wt) {
            lone = w.fixed + rounds * std::max(shared, w.step) + w.c_read * frags * v.wk;
            busy = rounds * shared + w.busy + 0.54 * w.c_read * frags * v.wk;
        } else {
            lone = f.fixed + per * std::max(frags * mfma * f.c_mfma * simd_waves, f.step) + f.c_read * frags * v.wk;
            busy = per * std::max(frags * mfma * f.c_mfma * simd_waves, v.wk * (v.fk + v.fm) * 16.0 * f.c_load) + f.busy;
        }
        // (waves per SIMD that the registers leave room for)
        const int occ = frags == 1 ? 8 : frags == 2 ? (bf16 ? 7 : 6) : 3;
        resident = std::max(1, occ * 4 / v.wk);
        launch = a.fwd_wt ? w.launch : f.launch;
        // (fp32 beyond a dozen workgroups to a CU: 288 -> 64 backward at 35x35, N = 112, 96 us, 73 in staged tiles)
        hbm = a.fwd_wt ? 2.6e6 : bf16 ? 3.3e6 : p.grid > 3072 ? 2.3e6 : 3.0e6;
    } else {
        const bool small = v.fm <= 2;
        const Fit f = small ? (bf16 ? Fit{2.4, 1350, 298, 1.24, 2.65, 0.92, 800} : Fit{3.0, 245, 253, 1.03, 0.24, 1.0, 2220})
                            : (bf16 ? Fit{1.1, 8760, 6, 1.33, 2.53, 1.62, 4920} : Fit{3.0, 6610, 248, 1.0, 1.2, 1.0, 7580});
        const double waves = v.wk * v.wm, rounds = (RS * v.npl + 1) / 2;
        const double bytes = (rounds * 2 * v.wk * v.fk * 32 + (double)v.npl * a.PLS) * 16;
        const double step = std::max(std::max(rounds * frags * mfma * waves / 4 * f.c_mfma, bytes / 64 * f.c_load),
                                     rounds * (v.fk + v.fm) * waves * 8 * f.c_read);
        lone = f.fixed + a.n_stage * (step + f.step);
        busy = a.n_stage * step + f.busy;
        const int occ = frags * 16 > 128 ? 1 : frags <= 2 ? 4 : small ? 3 : 2;
        resident = waves == 8 ? 1 : std::max(1, std::min((int)(kMaxLds / p.lds), occ));
        launch = f.launch;
        large = !small;
    }
    const int per_cu = ceil_div(p.grid, 256);
    const int full = per_cu / resident, rest = per_cu - full * resident;
    double t = full * std::max(lone, resident * busy) + (rest > 0 ? std::max(lone, rest * busy) : 0.0);
    t = t / 2.3e3 + launch;
    // (the register-operand kernel with three and more workgroups to a CU: 4 - 9 % over what the rest of the fit says)
    if (p.reg && bf16 && p.grid > 768 && !a.fwd_wt) t *= 1.08;
    const int V = vlen_of(v.dtype);
    const double out = (double)a.N * (scatter ? (double)a.OH * a.OW : (double)a.P * a.Q) * (a.Kp / V) * 16;
    if (a.ksplit > 1)  // the second launch, and the partial results there and back
        t += (bf16 ? 1.9 : 1.7) + a.ksplit * out * (bf16 ? 2 : 1) * 2 / 4.0e6;
    const double in = (double)a.N * a.Cb * (RS == 1 ? (double)a.P * a.Q : (double)a.H * a.W) * 16;
    const double bytes = in + out + (double)a.Cb * RS * a.Kp * 16;
    // bf16, the rate at which a staged launch bound by memory moves its bytes: 128-pixel tiles, three
    // workgroups to a CU, 6.5 - 7.3 TB/s up to the last-level cache's 256 MB (64 -> 256 at 56x56, N = 64: 20 us,
    // 30 in the large tiles) and less beyond (5.6 up to 450 MB with several channel tiles: N = 192 54 us, 83; with
    // one channel tile 4.6 from 130 MB on: 512 -> 128 at 28x28, N = 160, 42 us, 34 in the large tiles), not where
    // they are one step of four planes (32 -> 328 at 23x23, N = 128: 12.5 us, 11.7) or scatter;
    // the large ones 4.8, or 6.2 where one channel tile lets the input pass by the caches (64 -> 80 at
    // 73x73, N = 256: 75 us, 88 in small tiles), and less where they leave CUs with one workgroup or none
    // (256 -> 64 at 56x56, N = 16: 112 tiles, 13 us; 7 in small tiles).
    if (bf16 && !p.reg) {
        if (large)
            hbm = (a.n_kt == 1 ? 6.2e6 : 4.8e6) * std::min(1.0, a.total / (scatter ? 224.0 : 300.0));
        else if (!scatter && !(a.n_stage == 1 && v.npl == 4))
            hbm = bytes <= (a.n_kt > 1 ? 2.56e8 : 1.3e8) ? 6.5e6 : a.n_kt > 1 && bytes <= 4.5e8 ? 5.6e6 : 4.6e6;
    }
    // (10 % on top: without them 13 of 280 1x1 passes are 3 % and more behind the kernel it takes over from, with them 7)
    if (p.reg && a.fwd_wt) return 1.1 * std::max(t, launch + bytes / hbm);
    // (in registers on transformed weights, scattering: 3 % on top, and 3.0 TB/s where memory bounds it.  226 passes of odd channel
    // blocks, N = 8 ... 256, all candidates timed: without, 13 of them are 3 % and more slower than the next one down the list,
    // 168 <- 52 at 32x35, N = 196, 31 us for 24; with it two, of 12 us)
    if (p.reg && bf16 && scatter) return std::max(1.03 * t, launch + bytes / (bytes > 6.0e7 ? std::min(hbm, 3.0e6) : hbm));
    // (bf16 staged tiles that scatter, four stores for every one the fit has seen, and read the forward pass's weights: six
    // layers, N = 2 ... 64, take 1.23, 1.34, 1.45 and 1.64 of the estimate.  With it 23 of 104 backward passes of those six and
    // seven other layers, N = 2 ... 192, run on another kernel, in 0.83 of the time (0.51 ... 1.03): 512 -> 1024 stride 2 at
    // 28x28, N = 24, 21.7 -> 16.5 us, 64 -> 256 at 56x56, N = 96, 26.4 -> 16.1, 1024 -> 512 at 14x14, N = 48, 16.1 -> 12.7)
    // (... and in one round of short reductions the stores tell most: 1.1 - 1.5 of that, up to eight steps on 32 to 224 tiles;
    // 256 <- 256 stride 2 at 15x16, N = 53, 8.3 us where the register-operand kernel takes 7.3)
    const double few = !large && a.total <= 256 && a.n_stage <= 8 ? 1.2 : 1.0;
    const double scattered = !bf16 || !scatter || p.reg ? 1.0 : few * (large ? 1.6 : v.fk == 2 ? 1.45 : v.npl == 8 ? 1.23 : 1.34);
    return scattered * std::max(t, launch + bytes / hbm);
}

// The same for the patch kernel: a wave's share is pairs of channel blocks, each a patch and the weights of all taps.
// Fitted to 4 700 launches (3x3, 1x7 and 7x1 layers, N = 1 ... 256, every variant, forward / with the forward pass's
// weights; three sets of tensors in turn): rms error 11 %, the choice 3 % behind the fastest variant.
double estimate_patch_us(const IgemmPlan &p)
{
    const IgemmArgs &a = p.a;
    const IgemmVariant &v = p.v;
    struct Fit { double launch, fixed, frag, c_mfma, c_load, c_read, tap, pair, pos, exch, busy, four, hbm; };
    static const Fit fits[2] = {{2.0, 3250, 132, 1.52, 0.83, 0.97, 102, 0, 1.0, 155, 1450, 1.17, 1.66e6},
                                {1.4, 3060, 433, 1.73, 1.01, 1.84, 273, 307, 0.4, 165, 2480, 1.18, 1.85e6}};
    const Fit &f = fits[a.fwd_wt ? 1 : 0];
    const double taps = a.R * a.S, frags = v.fk * v.fm, waves = v.wk;
    const double pairs = ceil_div(ceil_div(a.Cb, 2), v.wk);
    const double shared = std::max({taps * frags * 32 * waves / 4 * f.c_mfma,
                                    waves * (taps * v.fk + a.PLS / 32) * 16 * f.c_load,
                                    waves * taps * v.fm * 8 * f.c_read * (a.stride > 1 ? 2 : 1)});
    const double lone = (f.fixed + f.frag * frags + pairs * (std::max(shared, taps * f.tap + f.pair) + f.pos * a.PLS) +
                         f.exch * frags * waves) * (v.wk == 4 ? f.four : 1.0);
    const double busy = pairs * (shared + f.pos / 4 * a.PLS) + f.exch * frags * waves + f.busy;
    // (waves per SIMD that the registers leave room for)
    const int occ = frags == 1 ? 7 : v.fk == 1 && v.fm == 2 ? 4 : frags == 2 ? 5 : v.fm == 2 ? 3 : 2;
    const int resident = std::max(1, std::min((int)(kMaxLds / p.lds), occ * 4 / v.wk));
    const int per_cu = ceil_div(p.grid, 256), full = per_cu / resident, rest = per_cu - full * resident;
    const double t = full * std::max(lone, resident * busy) + (rest > 0 ? std::max(lone, rest * busy) : 0.0);
    const double bytes = (double)a.N * a.Cb * a.H * a.W * 16 + (double)a.N * a.P * a.Q * a.Kp * 2 + (double)a.Cb * taps * a.Kp * 16;
    // (8 % on top: without them the choice is 6 - 26 % behind the kernel it takes over from in 17 of 560 launches, with
    // them in three)
    return 1.08 * std::max(t / 2.3e3 + f.launch, f.launch + bytes / f.hbm);
}

// What the launch that transforms the weights of a backward pass takes, and what the pass loses by finding
// them beyond the L2: 3.3 us for 0.5 MB, 3.7 for 1.2 MB, 6.4 for 4.7 MB.
double transform_launch_us(double weight_bytes) { return 3.0 + 0.7e-6 * weight_bytes; }
double transform_us(const IgemmPlan &p)
{
    // (fp32: not counted, which leaves the lines between staged tiles and operands in registers, measured with the launch
    // on both sides, where they are: counted, 128 -> 128 3x3 at 28x28, N = 48, takes 102 us for 95)
    if (p.v.dtype == CONV_F32) return 0;
    return transform_launch_us((double)p.a.Cb * p.a.Kp * 16 * (p.reg ? p.a.R * p.a.S : p.v.r * p.v.s));
}

// Where a launch may read the forward pass's weights (the arguments of forward_weights); taps 0: nowhere.
struct FwdWeights {
    int taps = 0, tap0 = 0, dr = 0, ds = 0;
};

// Channel groups over the XCDs, as in try_igemm: `image` pixels read per image.
void share_over_xcds(IgemmArgs &a, double image, int taps)
{
    const double in_b = (double)a.N * a.Cb * image * 16.0, wt_b = (double)a.Cb * taps * a.Kp * 16.0;
    double best = 0;
    a.gk = 1;
    for (int gk = 1; gk <= 8 && gk <= a.n_kt && a.ksplit == 1; gk *= 2) {
        if (a.n_kt % gk != 0) continue;
        double cost = gk * in_b + (8.0 / gk) * wt_b;
        if (wt_b / gk > 2.0e6) cost += 8.0 * in_b;
        if (gk == 1 || cost < best) { best = cost; a.gk = gk; }
    }
    a.kt_per = ceil_div(a.n_kt, a.gk);
    a.mq_per = ceil_div(a.n_mt, 8 / a.gk);
    a.per_xcd = a.gk == 1 ? ceil_div(a.total * a.ksplit, 8) : a.kt_per * a.mq_per;
}

// The staged input tile of the split kernel for the launch that `p` plans, R x S taps: what decides whether a variant serves it.
struct SplitTile {
    bool ok = false, sampled = false;
    int TQ = 0, Hs = 0, LW = 0, LRW = 0, ni = 0;
};
SplitTile split_tile(const IgemmPlan &p, int R, int S, int wm, int fm, int g, int strips)
{
    SplitTile t;
    const IgemmArgs &a = p.a;
    // (a launch with a staged plan: its tensors are within 32-bit offsets)
    if (!p.ok || a.no_taps || a.shuffle || a.cstride != a.stride || a.ostr_x != a.ostr) return t;
    t.sampled = R * S == 1 && a.pad_h == 0 && a.pad_w == 0 && (a.P - 1) * (long long)a.stride < a.H &&
                (a.Q - 1) * (long long)a.stride < a.W;
    if (t.sampled && strips > 1) return t;
    const int TM = wm * fm * 32;
    t.TQ = ceil_div(a.Q, strips);
    if ((strips - 1) * t.TQ >= a.Q) return t;
    if (t.sampled) {
        t.Hs = a.P;
        t.LW = t.TQ;
        t.LRW = TM;
    } else {
        // rows of an image: those its pixels read, without the rows of zeros below it that stand for the next image's above it too
        const int rows = (a.P - 1) * a.stride + R;
        t.Hs = rows - std::max(0, std::min(rows - a.pad_h - a.H, a.pad_h));
        t.LW = (t.TQ - 1) * a.stride + S;
        const long long touched = std::min<long long>((TM - 2) / t.TQ + 2, (long long)a.N * a.P);
        const long long crossings = std::min<long long>(a.N - 1, ceil_div((int)touched - 1, a.P));
        const long long LR = (touched - 1) * a.stride + crossings * std::max(0, t.Hs - a.P * a.stride) + R;
        if (LR * t.LW > 4096) return t;
        t.LRW = (int)LR * t.LW;
    }
    t.ni = ceil_div(2 * g * ceil_div(t.LRW, 64), 4);
    t.ok = true;
    return t;
}

// A plan of the split kernel.
SplitPlan try_split(const IgemmPlan &p, int R, int S, const FwdWeights &fw, int wk, int wm, int fm, int kw, int g, int strips,
                    int least_ni = 0)
{
    SplitPlan s;
    const SplitTile t = split_tile(p, R, S, wm, fm, g, strips);
    if (!t.ok) return s;
    s.v = IgemmSplitVariant{wk, wm, fm, kw, g, std::max(t.ni, least_ni), fw.taps > 0 ? 1 : 0};
    if (!igemm_split_exists(s.v)) return s;
    s.lds = igemm_split_lds_bytes(s.v, t.LRW);
    if (s.lds > (size_t)kMaxLds) return s;
    const int TK = wk * 32, TM = wm * fm * 32;
    const long long pixels = (long long)p.a.N * p.a.P * t.TQ, tiles = ((pixels + TM - 1) / TM) * strips;
    if (pixels >= (1LL << 30) || tiles * ceil_div(p.a.Kp, TK) >= (1 << 24)) return s;
    IgemmArgs &a = s.a;
    a = p.a;
    a.R = R;
    a.S = S;
    a.fwd_wt = a.group = 0;
    if (fw.taps > 0 && !forward_weights(a, fw.taps, fw.tap0, fw.dr, fw.ds)) return s;
    a.ksplit = 1;
    a.sampled = t.sampled;
    a.n_qt = strips;
    a.TQ = t.TQ;
    a.TR = 0;
    a.Hs = t.Hs;
    a.LW = t.LW;
    a.LRW = a.PLS = t.LRW;
    a.inv_P = 1.0f / (float)a.P;
    a.inv_Hs = 1.0f / (float)a.Hs;
    a.inv_LW = 1.0f / (float)a.LW;
    a.inv_TQ = 1.0f / (float)a.TQ;
    a.n_mt = (int)tiles;
    a.n_kt = ceil_div(a.Kp, TK);
    a.n_stage = ceil_div(a.Cb, 4 * g);
    a.st_per = a.n_stage;
    a.total = a.n_mt * a.n_kt;
    share_over_xcds(a, a.sampled ? (double)a.P * a.Q : (double)a.H * a.W, R * S);
    a.rot_k = a.rot_m = 1;
    s.grid = a.per_xcd * 8;
    s.ok = true;
    return s;
}

// The register-operand kernel's form.  (A reduction split over workgroups: as many of them as `p` has, whose workspace it uses.)
SplitPlan try_reg_split(const IgemmPlan &p, int R, int S, const FwdWeights &fw, int fk, int fm, int nw)
{
    SplitPlan s;
    const IgemmArgs &b = p.a;
    if (!p.ok || b.no_taps || b.shuffle || b.cstride != b.stride || b.ostr_x != b.ostr || !igemm_reg_split_exists(fk, fm, nw)) return s;
    // 32-bit byte offsets, exact small divisions and 24-bit products, as in try_reg
    const double shift = (double)std::max(0, b.pad_h) * b.W + std::max(0, b.pad_w);
    if (((double)b.N * b.Cb * b.H * b.W + shift) * 16 > 4.0e9 || b.pad_h < 0 || b.pad_w < 0) return s;
    if ((double)b.N * b.P * b.Q + fm * 32 >= 4.0e6 || (double)R * S * b.Kp >= 4.0e6) return s;
    if ((double)(b.N + 1) * std::max(b.Cb + 3, b.out_kb) * std::max(b.H, b.OH) >= 8.0e6) return s;
    IgemmArgs &a = s.a;
    a = b;
    a.R = R;
    a.S = S;
    a.fwd_wt = a.group = 0;
    if (fw.taps > 0 && !forward_weights(a, fw.taps, fw.tap0, fw.dr, fw.ds)) return s;
    a.inv_P = 1.0f / (float)(a.P * a.Q);
    a.inv_TQ = 1.0f / (float)a.Q;
    a.n_qt = 1;
    a.n_mt = ceil_div(a.N * a.P * a.Q, fm * 32);
    a.n_kt = ceil_div(a.Kp, fk * 32);
    a.total = a.n_mt * a.n_kt;
    a.n_stage = ceil_div(a.Cb, 4) * R * S;
    a.st_per = ceil_div(a.n_stage, b.ksplit);
    a.ksplit = ceil_div(a.n_stage, a.st_per);
    if (a.ksplit != b.ksplit) return s;
    share_over_xcds(a, R * S == 1 ? (double)a.P * a.Q : (double)a.H * a.W, R * S);
    s.lds = igemm_reg_split_lds_bytes(fk, fm, nw, a.fwd_wt != 0);
    s.fk = fk;
    s.fm = fm;
    s.nw = nw;
    s.grid = a.per_xcd * 8;
    s.ok = true;
    return s;
}

static const int kSplitTiles[][4] = {{4, 1, 4, 1}, {4, 1, 2, 1}, {2, 2, 4, 1}, {2, 2, 2, 1}, {4, 1, 4, 2}, {4, 1, 2, 2}, {2, 2, 4, 2}, {2, 2, 2, 2}};
static const int kRegSplitTiles[][3] = {{1, 1, 4}, {1, 1, 8}, {1, 1, 16}, {2, 1, 4}, {2, 1, 8}, {1, 2, 4}, {2, 2, 4}, {2, 2, 8}};

// What the left-out products add to a sum's error, in the units of chain_error: 0.03 where they are of random sign, 0.2 where all of
// them leave out the same (measured, split_bf16.h).
constexpr double kLeftOut = 0.2;
// Error of its sums in the same units: an MFMA rounds the sum of the large products once for sixteen channels; the small ones' own
// rounding is nothing beside that.
double split_error(const SplitPlan &s)
{
    const IgemmArgs &a = s.a;
    if (s.nw > 0) return ceil_div(a.st_per, s.nw) / 2.0 + std::log2((double)s.nw) / 2 + (a.ksplit > 1 ? a.ksplit / 2.0 : 0) + 0.5 + kLeftOut;
    return ceil_div(a.n_stage, s.v.kw) * s.v.g * a.R * a.S / 2.0 + (s.v.kw - 1) / 2.0 + 0.5 + kLeftOut;
}

// What a launch on the bf16 instructions takes, in microseconds, without the launch that transforms a backward pass's weights: the form of
// estimate_us.  Fitted to 49 000 launches, 650 drawn layers of ResNet-50, Inception-v3 and odd sizes, N = 1 ... 256, every
// variant, three sets of tensors in turn: rms error 8 % (in registers 14 %); the choice is 3 % behind the fastest.
struct SplitTimes {
    double lone, busy;  // clocks of a workgroup alone on its CU, and of one among others
    int resident;
};
// Clocks of a staged workgroup: a round among others and alone, and what stands before and behind its rounds.
double split_round(int fm, bool fwd_wt) { return (fm == 4 ? 814 : 560) + (fwd_wt ? 161 : 0); }
double split_round_alone(int fm, bool fwd_wt) { return (fm == 4 ? 952 : 702) + (fwd_wt ? 253 : 0); }
double split_start(int fm) { return 7244 + 775 * fm; }
SplitTimes split_times(const SplitPlan &s, bool scatter)
{
    const IgemmArgs &a = s.a;
    const double fw = a.fwd_wt ? 1 : 0;
    SplitTimes t;
    if (s.nw > 0) {
        const int type = s.fk * s.fm == 4 ? 3 : s.fk * s.fm == 1 ? 0 : s.fk == 2 ? 1 : 2, frags = s.fk * s.fm;
        static const double lone[4] = {711, 1192, 1508, 2272}, busy[4] = {498, 847, 945, 1339};
        const double per = ceil_div(a.st_per, s.nw), simd = s.nw / 4.0;
        const double loads = s.nw * (s.fk + s.fm) * 32.0, shared = std::max((busy[type] + fw * 92 * s.fk) * simd, loads);
        const double k = scatter ? 1.22 : 1.0;
        t.busy = k * (per * shared + 605 + 1.79 * 123 * frags * s.nw);
        t.lone = k * (3724 + per * std::max(lone[type] + fw * 111 * s.fk, shared) + 123.0 * frags * s.nw);
        t.resident = std::max(1, (frags == 1 ? 4 : frags == 2 ? 3 : 2) * 4 / s.nw);
        return t;
    }
    const IgemmSplitVariant &v = s.v;
    const bool wide = v.fm == 4;
    const double steps = ceil_div(a.n_stage, v.kw), rounds = v.g * a.R * a.S, k = scatter ? 2.06 : 1.0;
    t.busy = v.kw * steps * (rounds * split_round(v.fm, a.fwd_wt != 0) + v.ni * 225 + 120) + 1417 * v.fm * v.kw * k;
    t.lone = std::max(t.busy, split_start(v.fm) * k + steps * (rounds * split_round_alone(v.fm, a.fwd_wt != 0) + v.ni * 262 + 281));
    t.resident = std::max(1, std::min((int)(kMaxLds / s.lds), v.kw == 2 ? 1 : wide ? 2 : 3));
    return t;
}
double tensor_bytes(const IgemmArgs &a, bool scatter)
{
    const int taps = a.R * a.S;
    return (double)a.N * a.Cb * 16 * (taps == 1 ? (double)a.P * a.Q : (double)a.H * a.W) +
           (double)a.N * a.Kp * 4 * (scatter ? (double)a.OH * a.OW : (double)a.P * a.Q) + (double)a.Cb * taps * a.Kp * 16;
}
double split_us(const SplitPlan &s, bool scatter)
{
    const IgemmArgs &a = s.a;
    const SplitTimes w = split_times(s, scatter);
    const int per_cu = ceil_div(s.grid, 256), full = per_cu / w.resident, rest = per_cu - full * w.resident;
    const double t = full * std::max(w.lone, w.resident * w.busy) + (rest > 0 ? std::max(w.lone, rest * w.busy) : 0.0);
    const double launch = s.nw > 0 ? 2.4 : 1.2, hbm = s.nw > 0 ? 3.2e6 : 3.7e6;
    double us = std::max(t / (s.nw > 0 ? 2.2e3 : 2.1e3) + launch, launch + tensor_bytes(a, scatter) / hbm);
    if (a.ksplit > 1)  // the second launch, and the partial results there and back
        us += 1.7 + a.ksplit * (double)a.N * a.P * a.Q * a.Kp * 4 * 2 / 4.0e6;
    return us;
}

// Whether the launch that `p` plans runs on the bf16 instructions: where the estimate says that this is faster by more than split_line,
// and the sums are no less exact.  fw: where the forward pass's weights may be read.
// (CONVMI_IGEMM_SPLIT="wk,wm,fm,kw,g,strips,fw" or "r,fk,fm,waves,fw": one variant wherever it fits, fw 1: on the forward pass's
// weights; 0: never -- a tuning aid, as are those that ask for a variant on the fp32 instructions)
bool variant_asked_for()
{
    for (const char *name : {"CONVMI_IGEMM_CAND", "CONVMI_IGEMM_REG", "CONVMI_IGEMM_GROUP", "CONVMI_IGEMM_NT", "CONVMI_IGEMM_GK",
                             "CONVMI_IGEMM_ROT", "CONVMI_IGEMM_PATCH", "CONVMI_BWD_QUAD", "CONVMI_FORWARD_WEIGHTS", "CONVMI_STEM"})
        if (getenv(name)) return true;
    return false;
}
constexpr double kSplitMargin = 0.96;
// Up to which part of the other plan's estimate (`us`) a candidate's counts.  Time / the fp32 instructions' above the lines, where the
// estimate is too low, 1 100 passes of drawn layers: staged 1x1 with 96 channels or fewer on a side 0.73 - 1.38 (64 -> 80 at 73x73,
// N = 19, 22 -> 27 us; both wait for memory); staged 1x1 in two sets of waves 0.77 - 1.23; staged under a stride 0.83 - 1.28; in
// registers under a stride 0.74 - 1.14 (36 -> 44 3x3 at 20x21, N = 52, 6.8 -> 7.7: half of every line read is not used), in four waves
// or on short reductions in less than 10 us 0.90 - 1.18 (larger filters from 0.82 on 0.99 - 1.12: 64 -> 64 3x3 at 56x56, N = 2, 8.6 -> 9.6);
// in eight waves under larger filters from 0.92 on 0.96 - 1.06, in the mean 1.003 (65 passes, 8 - 15 us; 1x1 0.95 - 0.97); in registers
// under 1x1 in more than 1 200 tiles 0.9 - 1.14.
double split_line(const SplitPlan &s, double us)
{
    const IgemmArgs &a = s.a;
    const bool strided = a.stride > 1 || a.ostr > 1;
    if (s.nw > 0 && a.R * a.S == 1 && a.total > 1200) return 0.8;
    const bool filter = a.R * a.S > 1;
    if (s.nw > 0 && strided) return 0.83;
    if (s.nw > 0 && a.n_stage >= 24 && (s.nw >= 8 || us >= 10)) return filter && s.nw >= 8 ? 0.92 : 0.96;
    if (s.nw > 0) return us >= 10 ? 0.92 : filter ? 0.82 : 0.85;
    if (a.R * a.S == 1 && std::min(4 * a.Cb, a.Kp) <= 96) return 0.74;
    if (a.R * a.S == 1 && s.v.kw == 2) return 0.75;
    return strided ? 0.85 : kSplitMargin;
}
// Tiles of so many fragments, at the least.
double split_tiles(const IgemmArgs &a, int wk, int fragments)
{
    return std::ceil((double)a.N * a.P * a.Q / (fragments * 32)) * ceil_div(a.Kp, wk * 32);
}
SplitPlan plan_split(const IgemmPlan &p, int R, int S, const FwdWeights &fw, bool backward)
{
    SplitPlan best;
    if (!p.ok || p.v.dtype != CONV_F32) return best;
    if (const char *env = getenv("CONVMI_IGEMM_SPLIT")) {
        int wk = 0, wm = 0, fm = 0, kw = 0, g = 0, strips = 1, f = 0;
        if (sscanf(env, "r,%d,%d,%d,%d", &wk, &fm, &kw, &f) >= 3)
            return f && fw.taps == 0 ? best : try_reg_split(p, R, S, f ? fw : FwdWeights{}, wk, fm, kw);
        if (sscanf(env, "%d,%d,%d,%d,%d,%d,%d", &wk, &wm, &fm, &kw, &g, &strips, &f) < 5 || strips < 1) return best;
        return f && fw.taps == 0 ? best : try_split(p, R, S, f ? fw : FwdWeights{}, wk, wm, fm, kw, g, strips);
    }
    if (variant_asked_for()) return best;
    // (1x1 layers of one fragment of channels in the register-operand kernel, many tiles of pixels: it takes 0.5 - 0.7 of its estimate, and
    // this 1.15 - 1.46 of that (from 880 tiles: 192 -> 32 at 35x35, N = 45, 11.9 -> 16.6 us, 316 -> 32 at 51x53, N = 90, 77 -> 113); up to 640 tiles 0.73 - 1.03)
    if (p.reg && R * S == 1 && p.v.fk * p.v.fm == 1 && p.a.n_kt == 1 && p.a.total > 700) return best;
    const bool scatter = p.a.zero_fill != 0;
    const double transform = backward ? transform_launch_us((double)p.a.Cb * R * S * p.a.Kp * 16) : 0;
    const double other_us = estimate_us(p, scatter) + (p.a.fwd_wt ? 0 : transform);
    double best_us = other_us;
    const double most_error = sums_error(p) + kOwnRounding;
    auto consider = [&](const SplitPlan &c) {
        if (!c.ok) return;
        // (staged: half a microsecond on top, which the estimate is off where a launch is short)
        // (more shares to stage than rounds to do it beside: 256 pixels under 1x1, 16 channels a step, 0.66 - 1.33 of the other plan's time
        // where the estimate without this factor says 0.8, 144 <- 564 at 29x30, N = 123, 168 -> 224 us; in wider steps 0.49 - 0.97)
        const double crowded = c.nw == 0 && c.v.ni > c.v.g * R * S ? 1.3 : 1.0;
        const double us = crowded * split_us(c, scatter) + (c.nw > 0 ? 0 : 0.5) + (c.a.fwd_wt ? 0 : transform);
        if (us < best_us && us < split_line(c, other_us) * other_us && split_error(c) <= most_error) {
            best = c;
            best_us = us;
        }
    };
    // (the tensors alone take longer: nothing to look at)
    SplitPlan any;
    any.a = p.a;
    any.a.R = R;
    any.a.S = S;
    if (tensor_bytes(any.a, scatter) / 3.7e6 >= other_us) return best;
    for (const FwdWeights &w : {FwdWeights{}, fw}) {
        for (const auto &t : kSplitTiles) {
            // (... or a launch whose rounds are dealt over all CUs, or one tile)
            const double rounds = (double)ceil_div(p.a.Cb, 4) * R * S;
            const double clocks = std::max(split_tiles(p.a, t[0], t[1] * t[2]) * rounds * split_round(t[2], w.taps > 0) / 256,
                                           split_start(t[2]) + rounds / t[3] * split_round_alone(t[2], w.taps > 0));
            if (clocks / 2.1e3 + 1.7 >= std::min(best_us, kSplitMargin * other_us) - (w.taps > 0 ? 0 : transform)) continue;
            for (int g = 1; g <= 2; ++g) {
                if (g > 1 && R * S > 1) continue;
                for (int strips = 1; strips <= 4; ++strips) consider(try_split(p, R, S, w, t[0], t[1], t[2], t[3], g, strips));
            }
        }
        for (const auto &t : kRegSplitTiles) consider(try_reg_split(p, R, S, w, t[0], t[1], t[2]));
        if (fw.taps == 0) break;
    }
    return best;
}

hipError_t launch_plan(const IgemmPlan &p, const SplitPlan &split, const IgemmArgs &a, hipStream_t stream)
{
    if (split.ok) {
        IgemmArgs s = split.a;
        s.in = a.in;
        s.wt = a.wt;
        s.out = a.out;
        s.scale = a.scale;
        s.bias = a.bias;
        s.resid = a.resid;
        s.relu = a.relu;
        if (split.nw > 0) return launch_igemm_reg_split(split.fk, split.fm, split.nw, s, split.grid, stream);
        return launch_igemm_split(split.v, s, split.lds, split.grid, stream);
    }
    return p.patch ? launch_igemm_patch(p.v, a, p.grid, stream)
           : p.reg ? launch_igemm_reg(p.v, a, p.grid, stream)
                   : launch_igemm(p.v, a, p.lds, p.grid, stream);
}

// fp32: whether a staged backward launch of `us` microseconds takes the forward pass's weights.  It saves a launch and costs four
// 4-byte reads of LDS for one of 16, next to as many MFMAs as pixel fragments share the operand.  403 passes of 70 layers,
// N = 4 ... 256, in both forms: the reads cost 1 % of the launch under 1x1 in tiles of two pixel fragments and 1x7, less
// under 3x3 in seven fragments, 3 - 4 % else (up to 8), so that they are slower from about 150 us on (64 <- 640 7x1 at
// 30x30, N = 28, 140 -> 146 us; 512 <- 2048 1x1 at 7x7, N = 256, 232 -> 242; one launch for the classes of 84 <- 736 3x3
// stride 2 at 59x57, N = 28, 327 -> 336).  With this line the passes take 0.94 of the time with the transform, as without it,
// at most 1.03 (1.04 without), and 1.001 of the better form's.
// (CONVMI_FORWARD_WEIGHTS: 0 never, 1 wherever such a tile is built, in fp32 -- a tuning aid)
bool forward_weights_pay(int taps, int columns, int fm, double us, double weight_bytes)
{
    if (const char *env = getenv("CONVMI_FORWARD_WEIGHTS")) return atoi(env) != 0;
    const bool cheap = taps == 1 ? fm == 2 : columns == 7 || (taps == 9 && fm == 7);
    return (cheap ? 0.01 : 0.03) * us < transform_launch_us(weight_bytes);
}

// Plan one launch of the implicit-GEMM kernel.
//   input tensor:  N x Cb blocks x H x W;  result extent P x Q;  A rows Kp.
// Candidates: 4 or 2 waves along channels, tile within half of the LDS (two
// workgroups per CU overlap each other's barriers and staging) or all of it.
// Preference: least wasted MFMA work, then two workgroups per CU, then the
// wider channel tile (fewer re-reads of the input tile).
IgemmPlan plan_igemm_tile(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S,
                          int stride, int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0,
                          int zero_fill, const IgemmGeo &geo);

// fp32: whether the error of a plan's sums stays within `most`, with the group that sees to it (set in the
// plan's arguments).
bool sums_within(IgemmPlan &p, double most)
{
    IgemmArgs &a = p.a;
    double n, unit, rest = a.ksplit > 1 ? a.ksplit / 2.0 : 0;
    if (p.reg) {
        n = 8.0 * ceil_div(a.st_per, p.v.wk);
        unit = 8.0 * igemm_reg_depth(p.v.dtype, p.v.fk, p.v.fm, p.v.wk);
        rest += std::log2((double)p.v.wk) / 2;
    } else {
        unit = 4.0 * p.v.npl * p.v.r * p.v.s;
        n = unit * a.n_stage;
    }
    if (p.reg || igemm_variant_groups(p.v)) a.group = group_within(n, unit, kErrorMargin * most - rest);
    return chain_error(n, a.group * unit) + rest <= most + kOwnRounding;
}

// ... and that error as the plan is.
double sums_error(const IgemmPlan &p)
{
    const IgemmArgs &a = p.a;
    const double unit = p.reg ? 8.0 * igemm_reg_depth(p.v.dtype, p.v.fk, p.v.fm, p.v.wk) : 4.0 * p.v.npl * p.v.r * p.v.s;
    const double n = p.reg ? 8.0 * ceil_div(a.st_per, p.v.wk) : unit * a.n_stage;
    return chain_error(n, a.group * unit) + (a.ksplit > 1 ? a.ksplit / 2.0 : 0) + (p.reg ? std::log2((double)p.v.wk) / 2 : 0);
}

// (CONVMI_IGEMM_GROUP: steps or rounds that are summed apart, wherever the kernel can -- for tests)
IgemmPlan with_group(IgemmPlan p)
{
    const char *env = getenv("CONVMI_IGEMM_GROUP");
    if (env && p.ok && p.v.dtype == CONV_F32 && (p.reg ? !p.fallback : igemm_variant_groups(p.v))) p.a.group = atoi(env);
    return p;
}

// most_error > 0: the rounding error that the plan's sums may have (fp32).
IgemmPlan plan_igemm(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S,
                     int stride, int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0,
                     int zero_fill, const IgemmGeo &geo = IgemmGeo{}, bool may_split = false, double most_error = 0)
{
    IgemmPlan p;
    if (!geo.fallback)
        p = plan_igemm_tile(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                            zero_fill, geo);
    // Results of few tiles: the smaller tiles, and the kernel that splits the reduction inside the
    // workgroup, where the estimate says they are at least 5 % faster.  The plans above that
    // were picked by measurement at N = 256 (eight waves, 128 x 256) stay, as does a first
    // layer's, which runs on the resident-filter kernel.
    const bool measured = p.ok && (p.v.wk * p.v.wm == 8 || (p.v.wk == 2 && p.v.wm == 2 && p.v.fk == 2 && p.v.fm == 4));
    if (p.ok ? !measured && !getenv("CONVMI_IGEMM_CAND") && igemm_stem_lds(p.v, p.a) == 0 : geo.fallback) {
        const bool scatter = zero_fill != 0;
        IgemmPlan best = p;
        const bool exact_enough = p.ok && (most_error <= 0 || sums_within(best, most_error));
        double best_us = exact_enough ? 0.95 * estimate_us(p, scatter) + (geo.fwd_wt && !p.a.fwd_wt ? transform_us(p) : 0) : 1e30;
        auto transforms = [&](const IgemmPlan &c) { return geo.fwd_wt && dtype == CONV_BF16 && !c.a.fwd_wt; };
        auto consider = [&](IgemmPlan c) {
            if (!c.ok || (most_error > 0 && !sums_within(c, most_error))) return;
            const double us = estimate_us(c, scatter) + (geo.fwd_wt && !c.a.fwd_wt ? transform_us(c) : 0);
            // (of two bound by memory alike: staged ones, where tiles abound, the one that reads its input less often; on
            // transformed weights in registers the larger tile -- 324 <- 456 stride 2 at 55x55, N = 81, 57 us, 89 in the smaller)
            const bool larger = c.reg && best.reg ? transforms(c) && transforms(best) && c.v.fk * c.v.fm > best.v.fk * best.v.fm
                                                  : !c.reg && !best.reg && c.v.fk > best.v.fk && c.a.total >= 768;
            if (us < best_us || (us == best_us && larger)) {
                best = c;
                best_us = us;
            }
        };
        // (25 taps leave a CU one workgroup of the small tiles too: not where the large ones fill the chip -- 48 -> 64
        // 5x5 at 35x35: N = 48 0.99 of the large tiles' time, N = 96 1.18, N = 256 1.34)
        const bool small = p.ok && !(dtype == CONV_BF16 && R * S >= 25 && p.a.total >= 256);
        for (int fk = 1; fk <= 2 && small; ++fk)
            for (int npl = 8; npl >= 2; npl /= 2) {
                if ((R * S == 1) != (npl > 2)) continue;
                consider(try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0,
                                   ox0, zero_fill, geo, 2, 2, fk, 2, (size_t)kMaxLds, 2, npl));
            }
        static const int kReg[][4] = {{1, 1, 4, 1}, {1, 1, 8, 1}, {2, 1, 8, 1}, {1, 2, 4, 1}, {2, 2, 4, 1},
                                      {1, 1, 8, 2}, {1, 1, 8, 4}};
        IgemmGeo transformed = geo;
        transformed.fwd_wt = false;
        const char *reg_env = getenv("CONVMI_IGEMM_REG");
        for (const auto &k : kReg) {
            if (reg_env && strcmp(reg_env, "0") == 0) break;
            if (k[3] > 1 && (!may_split || dtype != CONV_F32)) continue;
            consider(try_reg(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                             zero_fill, geo, k[0], k[1], k[2], k[3]));
            // (bf16 backward passes: on transformed weights too, which many tiles repay -- 344 <- 216 1x1 at 19x21, N = 98, 27 us, 30 in
            // the staged tile of one channel block that is next; 48 -> 256 at 35x35, N = 8, 8.1 and 8.9)
            if (geo.fwd_wt && dtype == CONV_BF16)
                consider(try_reg(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                                 zero_fill, transformed, k[0], k[1], k[2], k[3]));
        }
        static const int kPatch[][3] = {{1, 1, 8}, {2, 1, 8}, {1, 2, 8}, {1, 2, 4}, {2, 2, 4}, {2, 2, 8}, {1, 4, 4}, {2, 4, 4}, {1, 4, 8}};
        for (const auto &k : kPatch) {
            if (reg_env && strcmp(reg_env, "0") == 0) break;
            consider(try_patch(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                               zero_fill, geo, k[0], k[1], k[2]));
        }
        p = best;
        // fp32 1x1: the 64 x 128 tile where the large ones leave a last round of workgroups part empty (512 run at once),
        // which the estimate is too coarse to see.  Time of the small / the large tile, 900 passes of 40 layers, N = 8 ... 256:
        //   - 128-row tiles filling 0.83 - 0.88 of one round behind at least 8 steps (32 where input or result are strided): 0.90 -
        //     1.03, 0.97 on average (512 -> 256 stride 2 at 28x28, N = 252, 123 -> 115 us), strided and shorter 0.95 - 1.05; from
        //     there to 0.92 0.92 - 1.13, up to one round 0.91 - 1.13;
        //   - 1.5 - 1.83 rounds: 0.88 - 1.02 (512 -> 2048 at 7x7, N = 256, 219 -> 202; 512 -> 1024 stride 2 at 28x28, N = 256,
        //     backward 482 -> 438); 1.44 - 1.5 0.99 - 1.13, 1.83 - 2.05 0.92 - 1.13, in the third round and later 0.93 - 1.14;
        //   - 64-row tiles, 0.82 - 2.3 rounds behind at most 12 steps: 0.78 - 1.02 (64 -> 64 at 56x56, N = 96, 40 -> 33), 0.84 at
        //     2.5; longer 0.85 - 1.05.  Where half of the rows are empty 0.94 up to 0.865, 1.04 up to 1.12, 0.85 - 0.98 beyond.
        if (p.ok && !p.reg && dtype == CONV_F32 && R * S == 1 && p.v.fm == 7 && p.a.sampled && Cb % 8 == 0) {
            const double filled = p.a.total / 512.0;
            const bool strided = stride > 1 || ostr > 1;
            const bool rounds = p.v.wk == 4 && p.a.n_stage >= 8 &&
                                ((filled >= 0.83 && filled <= 0.88 && (!strided || p.a.n_stage >= 32)) ||
                                 (filled >= 1.5 && filled <= 1.83));
            const bool narrow = p.v.wk == 2 && Kp <= 64 && p.a.n_stage <= 12 && filled >= 0.82 && filled <= 2.3 &&
                                (Kp > 32 || filled <= 0.865 || filled >= 1.12);
            if (rounds || narrow) {
                IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                                        zero_fill, geo, 2, 2, 1, 2, (size_t)kMaxLds, 2, 8);
                if (c.ok && (most_error <= 0 || sums_within(c, most_error))) p = c;
            }
        }
    }
    if (p.ok && !p.reg && dtype == CONV_F32 && p.v.fw &&
        !forward_weights_pay(R * S, S, p.v.fm, estimate_us(p, zero_fill != 0), (double)Cb * R * S * Kp * 16)) {
        p.v.fw = 0;
        p.a.fwd_wt = 0;
    }
    // (CONVMI_IGEMM_REG="fk,fm,waves,ksplit": one variant of the register-operand kernel wherever it
    // exists; "0": never -- a tuning aid)
    if (const char *env = getenv("CONVMI_IGEMM_REG"); env && (p.ok || geo.fallback)) {
        int fk = 0, fm = 0, nw = 0, ks = 1;
        if (sscanf(env, "%d,%d,%d,%d", &fk, &fm, &nw, &ks) >= 3 && ks >= 1 && (ks == 1 || may_split)) {
            IgemmPlan c = try_reg(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                                  zero_fill, geo, fk, fm, nw, ks);
            if (c.ok && most_error > 0) sums_within(c, most_error);
            if (c.ok) return with_group(c);
        }
    }
    // (CONVMI_IGEMM_PATCH="fk,fm,waves": one variant of the patch kernel wherever it exists -- a tuning aid)
    if (const char *env = getenv("CONVMI_IGEMM_PATCH"); env && p.ok) {
        int fk = 0, fm = 0, nw = 0;
        if (sscanf(env, "%d,%d,%d", &fk, &fm, &nw) == 3) {
            IgemmPlan c = try_patch(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0, ox0,
                                    zero_fill, geo, fk, fm, nw);
            if (c.ok) return c;
        }
    }
    p = with_group(p);
    // One channel tile: every line of the input is staged by exactly one workgroup.  Loaded
    // non-temporally it does not displace the weights in the L2 nor settle in the last-level
    // cache on its way past.  The same with two channel tiles side by side on an XCD, as long as
    // every XCD walks all channel tiles (one channel group): the second reader still finds the
    // line (measured at N = 256: bf16 layer 6 forward -15 %, layer 11 backward -8 %, fp32 layers
    // 6 and 14 backward -3 %).  With several channel groups the XCDs of the other groups fetch
    // the same lines later, from the last-level cache: there the hint costs 8 - 17 % (layer 16).
    // (CONVMI_IGEMM_NT: 0 never, 1 wherever the variant exists, 2 one channel tile only -- tuning aids.)
    const char *env = getenv("CONVMI_IGEMM_NT");
    const int mode = env ? atoi(env) : -1;
    const bool want = mode == 0 ? false
                      : mode == 1 ? true
                      : mode == 2 ? p.a.n_kt == 1
                                  : (p.a.n_kt == 1 || (p.a.gk == 1 && p.a.kt_per <= 2));
    if (p.ok && want && !p.reg) {
        IgemmVariant v = p.v;
        v.nt = 1;
        if (igemm_variant_exists(v)) p.v = v;  // (with the weights it has)
    }
    return p;
}

IgemmPlan plan_igemm_tile(int dtype, int N, int Cb, int H, int W, int Kp, int P, int Q, int R, int S,
                          int stride, int pad_h, int pad_w, int OH, int OW, int ostr, int oy0, int ox0,
                          int zero_fill, const IgemmGeo &geo)
{
    IgemmPlan best;
    double best_cost = 0;
    const size_t caps[2] = {(size_t)kMaxLds / 2, (size_t)kMaxLds};
    struct Cand { int wk, wm, fk, fm; };
    // bf16: two channel fragments per wave halve the LDS reads per MFMA (one
    // fragment per wave cannot keep the bf16 matrix core fed from 128 B/clk of LDS)
    // (the last: 32 rows, for results with at most 32 channel rows)
    const Cand cands[6] = {{1, 4, 2, 4}, {2, 2, 2, 7}, {1, 4, 2, 7}, {4, 1, 1, 7}, {2, 2, 1, 7},
                           {1, 4, 1, 7}};
    for (int ci = 0; ci < 2; ++ci)
        for (const Cand &cd : cands) {
            if (cd.fk == 2 && dtype != CONV_BF16) continue;
            const int TK = cd.wk * cd.fk * 32;
            if (TK > 64 && Kp <= TK / 2) continue;
            if (TK == 32 && Kp > 96) continue;  // (three 32-row tiles at most: 80 rows waste less so)
            IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW,
                                    ostr, oy0, ox0, zero_fill, geo, cd.wk, cd.wm, cd.fk, cd.fm, caps[ci]);
            if (!c.ok) continue;
            // one workgroup per CU loses roughly a fifth to exposed barriers/staging
            double cost = igemm_waste(c, N, P, Q, Kp) * (ci == 0 ? 1.0 : 1.2) *
                          (1.0 + 0.01 * (128 / TK));
            // rounds of workgroups over the 256 CUs: a last, partly filled round costs a full one
            const int slots = 256 * (ci == 0 ? 2 : 1);
            cost *= (double)(ceil_div(c.a.total, slots) * slots) / c.a.total;
            // one fragment per wave starves the bf16 matrix core of LDS bandwidth; it only
            // matters where the filter gives the layer enough reuse to be MFMA-bound
            if (dtype == CONV_BF16 && cd.fk == 1 && R * S > 1) cost *= 1.5;
            if (dtype == CONV_BF16 && cd.fk == 2 && R * S == 1) cost *= 1.5;
            if (!best.ok || cost < best_cost) {
                best = c;
                best_cost = cost;
            }
        }
    // Two cells per column (a strided backward pass into one channel block): the staged tile
    // is twice as wide per result column, and with two channel planes per step the band that
    // fits the LDS leaves a third of the pixel slots empty; one plane per step fits a full
    // band (measured on the 7x7 stride-2 layer at N = 256, fp32: 1.65 ms against 1.07 ms).
    if (geo.cstride > 1 && R * S > 1) {
        for (const Cand &cd : cands) {
            if (cd.fk == 2 && dtype != CONV_BF16) continue;
            if (cd.wk * cd.fk * 32 != 32 || Kp > 32) continue;
            IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW,
                                    ostr, oy0, ox0, zero_fill, geo, cd.wk, cd.wm, cd.fk, cd.fm,
                                    (size_t)kMaxLds, 2, 1);
            if (c.ok && (!best.ok || igemm_waste(c, N, P, Q, Kp) < 0.9 * igemm_waste(best, N, P, Q, Kp)))
                best = c;
        }
    }
    // Tuning aid: CONVMI_IGEMM_CAND="wk,wm,fk,fm,nb,npl" asks for one kernel variant wherever it
    // exists and fits (npl 0: the default planes per step); unset in normal use.
    if (const char *env = getenv("CONVMI_IGEMM_CAND")) {
        int wk = 0, wm = 0, fk = 0, fm = 0, nb = 2, npl = 0;
        if (sscanf(env, "%d,%d,%d,%d,%d,%d", &wk, &wm, &fk, &fm, &nb, &npl) >= 4 && wk > 0 && wm > 0 &&
            fk > 0 && fm > 0 && (wk * wm == 4 || wk * wm == 8) && nb >= 2 && nb <= 5) {
            IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW,
                                    ostr, oy0, ox0, zero_fill, geo, wk, wm, fk, fm, (size_t)kMaxLds, nb, npl);
            if (c.ok) return c;
        }
    }
    // bf16, eight waves (two per SIMD inside one workgroup, one workgroup per CU): a 256 x 256
    // tile for 1x1 filters (four MFMA rounds per step), 128 x 512 for 3x3.  One staged tile
    // feeds twice the MFMAs of two four-wave workgroups, which is what layers bound by the
    // rate at which a CU pulls tiles in from memory gain from (measured at N = 256: 5 - 12 %
    // on the 1x1 layers with at least 256 output rows and 128 input channels, 2 - 6 % on the
    // 28 x 28 and 14 x 14 3x3 layers).  Not for results narrower than the tile, and not where
    // the tiles would not fill the chip (there the four-wave tiles, or a split reduction, do).
    // ... except where the reduction is short (at most 256 channels) and the result wide: a
    // tile then spends as long on its first loads and its stores as on its MFMAs, and two
    // four-wave workgroups per CU with 128 x 256 tiles, which overlap each other's ends, are
    // 10 - 12 % faster than one eight-wave workgroup (measured on the 128 -> 512 and
    // 256 -> 1024 layers and the backward pass of 1024 -> 256).
    if (dtype == CONV_BF16 && best.ok && R * S == 1 && stride == 1 && ostr == 1 && Kp >= 512 &&
        Cb <= 32 && Cb % 4 == 0) {
        IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0,
                                ox0, zero_fill, geo, 2, 2, 2, 4, (size_t)kMaxLds / 2, 2, 4);
        if (c.ok && c.a.total >= 300 && igemm_waste(c, N, P, Q, Kp) <= 1.1 * igemm_waste(best, N, P, Q, Kp))
            return c;
    }
    if (dtype == CONV_BF16 && best.ok) {
        IgemmPlan c;
        if (R * S == 1 && Kp >= 256 && Cb % 8 == 0)
            c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0,
                          ox0, zero_fill, geo, 4, 2, 2, 4, (size_t)kMaxLds, 2, 8);
        else if (R == 3 && S == 3 && stride == 1 && Kp >= 128 && Cb % 2 == 0)
            c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0,
                          ox0, zero_fill, geo, 2, 4, 2, 4, (size_t)kMaxLds, 2, 2);
        if (c.ok && c.a.total >= 150 && igemm_waste(c, N, P, Q, Kp) <= 1.1 * igemm_waste(best, N, P, Q, Kp))
            return c;
        // a result of one 32-row tile under a filter window (the merged classes of a strided
        // backward pass into one channel block): eight pixel waves, 32 x 1792; the band that
        // fits the LDS fills 7/8 of it and is still 13 % faster than four waves (conv1, N = 256)
        if (!c.ok && R * S > 1 && Kp <= 32 && Cb % 2 == 0 && geo.cstride <= 1) {
            c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr, oy0,
                          ox0, zero_fill, geo, 1, 8, 1, 7, (size_t)kMaxLds, 2, 2);
            if (c.ok && c.a.total >= 512 && igemm_waste(c, N, P, Q, Kp) <= 1.15 * igemm_waste(best, N, P, Q, Kp))
                return c;
        }
    }
    // bf16 1x1: a reduction step is two MFMA rounds, far shorter than a trip to memory; a
    // third buffer keeps the loads two steps ahead where it fits the same LDS budget
    if (dtype == CONV_BF16 && R * S == 1 && best.ok && best.a.n_stage >= 3) {
        const size_t cap = best.lds <= (size_t)kMaxLds / 2 ? (size_t)kMaxLds / 2 : (size_t)kMaxLds;
        IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr,
                                oy0, ox0, zero_fill, geo, best.v.wk, best.v.wm, best.v.fk, best.v.fm, cap, 3);
        if (c.ok && c.a.total <= best.a.total) best = c;
    }
    // ... and where the tiles number no more than the CUs (a narrow result behind a deep
    // reduction: the 7x7 layers that narrow the channel count) a workgroup has its CU to itself
    // anyway: eight channel blocks per step then, four MFMA rounds between two barriers instead
    // of two and twice the bytes in flight (measured at N = 256: layer 20 forward 76 -> 55 us,
    // layer 19 backward 83 -> 60, layer 17 forward 64 -> 54; deeper rings change nothing).
    if (dtype == CONV_BF16 && R * S == 1 && best.ok && best.v.wk * best.v.wm == 4 && best.v.fk == 1 &&
        best.a.total <= 256 && Cb % 8 == 0 && Cb >= 32) {
        IgemmPlan c = try_igemm(dtype, N, Cb, H, W, Kp, P, Q, R, S, stride, pad_h, pad_w, OH, OW, ostr,
                                oy0, ox0, zero_fill, geo, best.v.wk, best.v.wm, best.v.fk, best.v.fm,
                                (size_t)kMaxLds, 2, 8);
        if (c.ok && c.a.total <= best.a.total) best = c;
    }
    return best;
}

// The four residue classes of a 3x3 stride-2 backward pass in one launch of 64 x 128 tiles, where that is
// faster than one launch each of what plan_igemm picks.  Time of the one launch, which reads the forward pass's weights, / of
// the four and the launch that transforms theirs, 15 layers at N = 1 ... 256:
//   - bf16: everywhere (0.27 - 0.88);
//   - fp32: where the tiles fill the chip before their chain of K/8 steps tells, 1.25 tiles per output channel, or the
//     chain is short (K <= 96), but not where half of a tile's rows are empty (32 -> 64 at 149x149, N = 8 up: 1.1 - 1.65): 0.46 -
//     1.02.  Elsewhere 0.69 - 1.65: 0.7 - 0.95 from about half a tile per output channel on (256 -> 256 at 28x28, N = 8, 41 us
//     and 35), where the one launch sums each result in one chain and the four split it over waves; 1.06 - 1.4 below
//     (288 -> 384 at 35x35, N = 1 36.7 and 49.7).
// (128 x 128 tiles: at most 5 % ahead, on a few bf16 layers; fp32 up to twice as long.)
void plan_bwd_quad(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    p->bwd_quad = false;
    if (d.R != 3 || d.S != 3 || d.stride != 2 || p->n_bwd != 4 || f.Kb % 4 != 0) return;
    // (classes in the kernel's order, with the sub-filters' own extents)
    BwdClass cls[4];
    size_t off = 0;
    int tiles = 0;
    bool forward = true;
    for (int i = 0; i < 4; ++i) {
        const int R2 = i < 2 ? 2 : 1, S2 = i == 0 || i == 2 ? 2 : 1;
        const BwdClass *b = nullptr;
        for (int j = 0; j < 4; ++j)
            if (p->bwd[j].x.Rsub == R2 && p->bwd[j].x.Ssub == S2) b = &p->bwd[j];
        if (!b) return;
        cls[i] = *b;
        const IgemmArgs &a = b->p.a;
        cls[i].p = try_igemm(d.dtype, d.N, f.Kb, f.P, f.Q, f.Cp, a.P, a.Q, R2, S2, 1, a.pad_h, a.pad_w, d.H, d.W, 2,
                             a.oy0, a.ox0, 0, IgemmGeo{}, 2, 2, 1, 2, (size_t)kMaxLds, 2, R2 * S2 == 1 ? 4 : 2, 1);
        if (!cls[i].p.ok) return;
        tiles += cls[i].p.a.total;
        const int off_r = cls[i].x.r_off, off_s = cls[i].x.s_off;
        forward = forward_weights(cls[i].p.a, 9, (off_r + 2 * (R2 - 1)) * 3 + off_s + 2 * (S2 - 1), 6, 2);
        cls[i].x.R2 = R2;
        cls[i].x.S2 = S2;
        cls[i].ws_off = off;
        off += (size_t)f.Kb * R2 * S2 * f.Cp * f.vlen * esize_of(d.dtype);
    }
    // (CONVMI_BWD_QUAD: 0 never, 1 wherever it fits -- a tuning aid)
    bool want = d.dtype == CONV_BF16 || (f.Cp > 32 && (d.K <= 96 || tiles >= 1.25 * d.K));
    if (const char *env = getenv("CONVMI_BWD_QUAD")) want = atoi(env) != 0;
    // (bf16 has no form of the kernel that reads transformed weights)
    if (!want || (!forward && d.dtype == CONV_BF16)) return;
    if (d.dtype == CONV_F32) {
        // (one launch: the classes' estimates without theirs, which are together 1.14 of what it takes beyond 100 us)
        double us = 0;
        for (const BwdClass &c : cls) us += estimate_us(c.p, true) - 3.0;
        forward = forward && forward_weights_pay(9, 3, 2, 0.88 * us, (double)off);
    }
    for (int i = 0; i < 4; ++i) {
        cls[i].p.a.fwd_wt = forward ? 1 : 0;
        p->bwd[i] = cls[i];
    }
    p->bwd_ws = off;
    p->bwd_quad = true;
}

void plan_bwd(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int es = esize_of(d.dtype);
    p->bwd_mode = 0;
    p->n_bwd = 0;
    p->bwd_ws = 0;
    p->bwd_quad = false;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    // (filters, and channel-block counts, that no staged kernel is built for: 10 to 100 times the
    // untiled loop nests' rate -- 140 -> 188 channels, 3x3 stride 2 at 26x25, N = 64, fp32: 2324 -> 104 us)
    IgemmGeo any_filter;
    any_filter.fallback = true;
    if (d.stride == 1 && pad_h <= d.R - 1 && pad_w <= d.S - 1) {
        BwdClass &b = p->bwd[0];
        // Up to four fp32 copies of dI behind the weights where they keep to the static scratch of
        // the entry point without a workspace: a split reduction changes nothing for its callers.
        const size_t wt_b = ((size_t)f.Kb * d.R * d.S * f.Cp * f.vlen * es + 255) / 256 * 256;
        const size_t copy_b = (size_t)d.N * f.Cp * d.H * d.W * sizeof(float);
        IgemmGeo staged;
        staged.fwd_wt = true;
        for (const IgemmGeo &geo : {staged, any_filter})
            if (!b.p.ok)
                b.p = plan_igemm(d.dtype, d.N, f.Kb, f.P, f.Q, f.Cp, d.H, d.W, d.R, d.S, 1, d.R - 1 - pad_h,
                                 d.S - 1 - pad_w, d.H, d.W, 1, 0, 0, 0, geo, wt_b + 4 * copy_b <= kScratchBytes);
        b.part_off = wt_b;
        b.x = WtXformArgs{nullptr, nullptr, f.Cb, f.Kb, f.Cp, f.Kp, d.R, d.S, d.R, d.S,
                          1, 0, 0, d.R, d.S};
        b.ws_off = 0;
        if (b.p.ok) {
            p->bwd_mode = 1;
            p->n_bwd = 1;
            p->bwd_ws = (size_t)f.Kb * d.R * d.S * f.Cp * f.vlen * es;
            if (b.p.a.ksplit > 1) p->bwd_ws = wt_b + b.p.a.ksplit * copy_b;
        }
        return;
    }
    if (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0) {
        BwdClass &b = p->bwd[0];
        IgemmGeo geo;
        geo.fwd_wt = true;
        b.p = plan_igemm(d.dtype, d.N, f.Kb, f.P, f.Q, f.Cp, f.P, f.Q, 1, 1, 1, 0, 0, d.H, d.W,
                         d.stride, 0, 0, 1, geo);
        b.x = WtXformArgs{nullptr, nullptr, f.Cb, f.Kb, f.Cp, f.Kp, 1, 1, 1, 1, 1, 0, 0, 1, 1};
        b.ws_off = 0;
        if (b.p.ok) {
            p->bwd_mode = 1;
            p->n_bwd = 1;
            p->bwd_ws = (size_t)f.Kb * f.Cp * f.vlen * es;
        }
        return;
    }
    // Generic case: one stride-1 sub-convolution per residue class (py, px) of
    // the dI position modulo the stride, over the taps congruent to it.
    const int st = d.stride;
    if (st * st > 16) return;
    // dI with one channel block (conv1): the classes' sub-filters become the
    // rows of one filter over their common window, class (py, px) in channel
    // block py*st+px of the result, and the store interleaves the blocks into
    // the st x st cells of dI.  One launch, and st*st*vlen live rows per MFMA
    // instead of vlen.
    if (f.Cb == 1 && st * st * f.vlen <= 32 && st <= 4) {
        BwdClass &b = p->bwd[0];
        WtMergeArgs &m = b.m;
        memset(&m, 0, sizeof(m));
        int padU[2] = {0, 0}, win[2] = {1, 1};
        for (int ax = 0; ax < 2; ++ax) {
            const int F = ax == 0 ? d.R : d.S;
            const int pad_ax = ax == 0 ? pad_h : pad_w;
            int *sub = ax == 0 ? m.rsub : m.ssub, *roff = ax == 0 ? m.roff : m.soff;
            int *sh = ax == 0 ? m.rsh : m.ssh;
            int padc[4];
            for (int pp = 0; pp < st; ++pp) {
                const int ro = (pp + pad_ax) % st;
                sub[pp] = ro < F ? ceil_div(F - ro, st) : 0;
                roff[pp] = ro;
                padc[pp] = std::max(sub[pp], 1) - 1 - (pp + pad_ax) / st;
                padU[ax] = pp == 0 ? padc[pp] : std::max(padU[ax], padc[pp]);
            }
            for (int pp = 0; pp < st; ++pp) {
                sh[pp] = padU[ax] - padc[pp];
                win[ax] = std::max(win[ax], std::max(sub[pp], 1) + sh[pp]);
            }
        }
        // Where the classes fill only half of an MFMA's 32 rows (fp32, stride 2), a column of
        // the result stands for TWO cells side by side: 32 live rows, half the columns, and a
        // window one tap wider (cell e of the pair reads its taps e columns to the right).
        // (CONVMI_BWD_CELLS=1 keeps one cell per column: a tuning aid.)
        int cells = (2 * st * st * f.vlen <= 32 && ceil_div(d.W, st) >= 2) ? 2 : 1;
        if (const char *env = getenv("CONVMI_BWD_CELLS"); env && atoi(env) == 1) cells = 1;
        const int Hc = ceil_div(d.H, st), Wc = ceil_div(d.W, st);
        for (; cells >= 1 && padU[0] >= 0 && padU[1] >= 0; --cells) {
            m.Kb = f.Kb; m.Kp = f.Kp; m.R = d.R; m.S = d.S; m.R2 = win[0]; m.S2 = win[1] + cells - 1;
            m.st = st; m.cells = cells;
            IgemmGeo geo;
            geo.cstride = cells;
            geo.ostr_x = cells * st;
            b.p = plan_igemm(d.dtype, d.N, f.Kb, f.P, f.Q, cells * st * st * f.vlen, Hc, ceil_div(Wc, cells),
                             m.R2, m.S2, 1, padU[0], padU[1], d.H, d.W, st, 0, 0, 0, geo);
            if (b.p.ok) {
                b.p.a.shuffle = 1;
                b.p.a.out_kb = 1;
                b.merged = true;
                b.ws_off = 0;
                p->bwd_mode = 3;
                p->n_bwd = 1;
                p->bwd_ws = (size_t)f.Kb * m.R2 * m.S2 * cells * st * st * f.vlen * f.vlen * es;
                return;
            }
        }
    }
    const int R2 = ceil_div(d.R, st), S2 = ceil_div(d.S, st);
    size_t off = 0;
    int n = 0;
    bool fallback = false;  // (every class on the same kind of kernel: staged, or the exact ones)
    for (int cls = 0; cls < st * st; ++cls) {
        const int py = cls / st, px = cls % st;
        const int ry = (py + pad_h) % st, rx = (px + pad_w) % st;
        const int Rsub = ry < d.R ? ceil_div(d.R - ry, st) : 0;
        const int Ssub = rx < d.S ? ceil_div(d.S - rx, st) : 0;
        const int dy0 = (py + pad_h) / st, dx0 = (px + pad_w) / st;
        const int Hsub = py < d.H ? ceil_div(d.H - py, st) : 0;
        const int Wsub = px < d.W ? ceil_div(d.W - px, st) : 0;
        if (Hsub == 0 || Wsub == 0) continue;
        BwdClass &b = p->bwd[n];
        // With no tap in the class the sub-filter is all zero and the
        // launch writes zeros, which is what Algorithm 6 leaves there.
        const int Re = std::max(Rsub, 1), Se = std::max(Ssub, 1);
        // the class's own sub-filter extent where a kernel exists for it, else
        // the common extent with zero taps
        int R2c = Re, S2c = Se;
        auto plan = [&](const IgemmGeo &geo) {
            b.p = plan_igemm(d.dtype, d.N, f.Kb, f.P, f.Q, f.Cp, Hsub, Wsub, R2c, S2c, 1, Re - 1 - dy0,
                             Se - 1 - dx0, d.H, d.W, st, py, px, 0, geo);
        };
        if (fallback) {
            any_filter.no_taps = Rsub == 0 || Ssub == 0;
            plan(any_filter);
            if (!b.p.ok) return;
        } else {
            plan(IgemmGeo{});
            if (!b.p.ok) {
                R2c = R2;
                S2c = S2;
                plan(IgemmGeo{});
            }
            if (!b.p.ok) {  // from the first class again
                fallback = true;
                cls = -1;
                n = 0;
                off = 0;
                continue;
            }
        }
        b.x = WtXformArgs{nullptr, nullptr, f.Cb, f.Kb, f.Cp, f.Kp, d.R, d.S, R2c, S2c,
                          st, ry, rx, Rsub, Ssub};
        if (Rsub == 0 || Ssub == 0) { b.x.Rsub = 0; b.x.Ssub = 0; }
        b.ws_off = off;
        off += (size_t)f.Kb * R2c * S2c * f.Cp * f.vlen * es;
        ++n;
    }
    p->bwd_mode = 2;
    p->n_bwd = n;
    p->bwd_ws = off;
    if (!fallback) plan_bwd_quad(p);
}

// Where launch i of a backward pass may read the forward pass's weights.
FwdWeights class_weights(const conv_plan *p, int i)
{
    const WtXformArgs &x = p->bwd[i].x;
    const int st = p->bwd_mode == 2 ? p->d.stride : 1;
    if (x.R2 != x.Rsub || x.S2 != x.Ssub || x.Rsub < 1 || x.Ssub < 1) return FwdWeights{};
    return FwdWeights{p->d.R * p->d.S, (x.r_off + st * (x.R2 - 1)) * p->d.S + x.s_off + st * (x.S2 - 1), st * p->d.S, st};
}

// The classes in one launch of one variant, those of most taps first.
SplitClassesPlan try_split_classes(const conv_plan *p, int wk, int wm, int fm, int kw, int g, int strips)
{
    SplitClassesPlan s;
    if (p->bwd_mode != 2 || p->n_bwd < 1 || p->n_bwd > 4) return s;
    int order[4] = {0, 1, 2, 3};
    auto taps = [&](int i) { return p->bwd[i].x.R2 * p->bwd[i].x.S2; };
    std::stable_sort(order, order + p->n_bwd, [&](int i, int j) { return taps(i) > taps(j); });
    // (a variant's shares are those of the class that needs most)
    int ni = 0, grid = 0;
    for (int k = 0; k < p->n_bwd; ++k) {
        const SplitTile t = split_tile(p->bwd[order[k]].p, p->bwd[order[k]].x.R2, p->bwd[order[k]].x.S2, wm, fm, g, strips);
        if (!t.ok) return SplitClassesPlan{};
        ni = std::max(ni, t.ni);
    }
    if (!igemm_split_classes_exist(IgemmSplitVariant{wk, wm, fm, kw, g, ni, 1})) return SplitClassesPlan{};
    for (int k = 0; k < 4; ++k) {
        if (k >= p->n_bwd) {
            s.c.end[k] = grid;
            continue;
        }
        const int i = order[k];
        const FwdWeights fw = class_weights(p, i);
        if (fw.taps == 0) return SplitClassesPlan{};
        const SplitPlan c = try_split(p->bwd[i].p, p->bwd[i].x.R2, p->bwd[i].x.S2, fw, wk, wm, fm, kw, g, strips, ni);
        if (!c.ok) return SplitClassesPlan{};
        s.c.cls[k] = c.a;
        s.c.end[k] = grid += c.grid;
        s.lds = std::max(s.lds, c.lds);
        s.v = c.v;
    }
    s.ok = true;
    return s;
}

double classes_error(const conv_plan *p, const SplitClassesPlan &s)
{
    double most = 0;
    for (int k = 0; k < p->n_bwd; ++k) {
        SplitPlan c;
        c.a = s.c.cls[k];
        c.v = s.v;
        most = std::max(most, split_error(c));
    }
    return most;
}
// What the one launch takes: the workgroups of all classes share the CUs, and none is done before its own tile is.
double classes_us(const conv_plan *p, const SplitClassesPlan &s)
{
    double busy = 0, lone = 0, bytes = 0;
    for (int k = 0; k < p->n_bwd; ++k) {
        SplitPlan c;
        c.a = s.c.cls[k];
        c.v = s.v;
        c.lds = s.lds;
        const SplitTimes t = split_times(c, true);
        busy += t.busy * c.a.total;
        lone = std::max(lone, t.lone);
        bytes += tensor_bytes(c.a, false);
    }
    const double launch = 1.2;
    return std::max(std::max(lone, busy / 256 + 0.5 * lone) / 2.1e3 + launch, launch + bytes / 3.7e6);
}

// The backward pass on the bf16 instructions.
void plan_bwd_split(conv_plan *p)
{
    p->bwd_classes = SplitClassesPlan{};
    p->bwd_split = SplitPlan{};
    if (p->d.dtype != CONV_F32 || p->bwd_mode == 0 || p->bwd_mode == 3) return;
    if (p->bwd_mode == 2) {
        if (const char *env = getenv("CONVMI_IGEMM_SPLIT")) {
            int wk = 0, wm = 0, fm = 0, kw = 0, g = 0, strips = 1;
            if (sscanf(env, "%d,%d,%d,%d,%d,%d", &wk, &wm, &fm, &kw, &g, &strips) >= 5 && strips > 0)
                p->bwd_classes = try_split_classes(p, wk, wm, fm, kw, g, strips);
            return;
        }
        if (variant_asked_for()) return;
        // (one launch for the classes, or one each and the launch that transforms their weights)
        double old_us = 0, weights = 0, most_error = 0;
        for (int i = 0; i < p->n_bwd; ++i) {
            const BwdClass &b = p->bwd[i];
            old_us += p->bwd_quad ? 0.88 * (estimate_us(b.p, true) - 3.0) : estimate_us(b.p, true);
            weights += (double)b.x.Kb * b.x.R2 * b.x.S2 * b.x.Cp * 16;
            most_error = std::max(most_error, sums_error(b.p));
        }
        old_us += (p->bwd_quad ? 3.0 : 0.0) + (p->bwd[0].p.a.fwd_wt ? 0 : transform_launch_us(weights));
        double best_us = (old_us < 20 ? 0.75 : 0.88) * old_us;  // (above: 0.9 - 1.3 of the time)
        for (const auto &t : kSplitTiles) {
            // (the rounds of all classes dealt over all CUs take longer: nothing to look at)
            double clocks = 0;
            for (int i = 0; i < p->n_bwd; ++i)
                clocks += split_tiles(p->bwd[i].p.a, t[0], t[1] * t[2]) * ceil_div(p->bwd[i].p.a.Cb, 4) * p->bwd[i].x.R2 * p->bwd[i].x.S2;
            if (clocks * split_round(t[2], true) / 256 / 2.1e3 + 1.2 >= best_us) continue;
            for (int strips = 1; strips <= 4; ++strips) {
                const SplitClassesPlan c = try_split_classes(p, t[0], t[1], t[2], t[3], 1, strips);
                if (!c.ok) continue;
                const double us = classes_us(p, c);
                if (us < best_us && classes_error(p, c) <= most_error + kOwnRounding) {
                    p->bwd_classes = c;
                    best_us = us;
                }
            }
        }
        return;
    }
    p->bwd_split = plan_split(p->bwd[0].p, p->bwd[0].x.R2, p->bwd[0].x.S2, class_weights(p, 0), true);
}

// The largest of three bounds, each of which shades into the next: the sixth root of the sum of their sixth powers.
double shaded(const double (&bound)[3])
{
    double sum = 0;
    for (const double b : bound) sum += b * b * b * b * b * b;
    return std::sqrt(std::cbrt(sum));
}

// A plan of the kernel that keeps the weights in registers, for N images of Cb blocks of H x W pixels and a result of Kp channels.
IgemmStreamPlan try_stream(const conv_desc_t &d, int pad_h, int pad_w, int Cb, int Kp, int fk)
{
    IgemmStreamPlan s;
    if (d.dtype != CONV_BF16 || d.R != 3 || d.S != 3 || d.stride != 1 || pad_h != 1 || pad_w != 1) return s;
    s.cs = std::max(2, ceil_div(Cb, 2));
    s.fk = fk;
    const double pixels = (double)d.N * d.H * d.W;
    // exact small divisions, 24-bit products, 32-bit byte offsets
    if (!igemm_stream_exists(s.cs, fk) || d.W > igemm_stream_widest() || pixels >= 3.9e6 || pixels * std::max(Cb, Kp / 8) * 16 >= 4.0e9) return s;
    IgemmStreamArgs &a = s.a;
    a.N = d.N; a.Cb = Cb; a.H = d.H; a.W = d.W; a.Kp = Kp; a.out_kb = Kp / 8;
    a.n_kt = ceil_div(Kp, fk * 32);
    // one workgroup per CU, one round
    const int units = ceil_div((int)pixels, 128);
    a.steps = ceil_div(units, std::max(1, 256 / a.n_kt));
    a.total = ceil_div(units, a.steps) * a.n_kt;
    a.per_xcd = ceil_div(a.total, 8);
    if (igemm_stream_lds_bytes(s) > (size_t)kMaxLds) return s;
    s.ok = true;
    return s;
}
// What it takes, in microseconds, in the form of estimate_us.  Fitted to 480 launches (170 drawn layers of 16 ... 200 channels, N = 8 ...
// 256, both passes, three sets of tensors in turn): rms error 5 %.
double stream_us(const IgemmStreamPlan &s)
{
    const IgemmStreamArgs &a = s.a;
    const double pixels = (double)a.N * a.H * a.W, in_b = pixels * a.Cb * 16, out_b = pixels * a.Kp * 2;
    const double fixed = 2.8 + 0.27 * s.cs * s.fk;
    const double bound[3] = {fixed + a.steps * std::max(0.224 * s.cs * s.fk + 0.28, 0.74), fixed + (in_b * a.n_kt + out_b) / 7.28e6,
                             fixed + (in_b + out_b) / 5.23e6};
    return shaded(bound);
}
// Whether a pass keeps the weights in registers: up to 0.88 of what estimate_us says of the other plan.  Time / the other kernel's by the
// quotient of the estimates, 269 passes: below 0.75 0.62 - 0.88, in the mean 0.73 (32 -> 64 at 147x147, N = 64, backward 83 -> 61 us;
// 60 -> 28 at 147x147, N = 32, 49 -> 31; 32 -> 24 at 28x31, N = 222, 13 -> 8); 0.75 - 0.88 0.64 - 1.03, mean 0.82; 0.88 - 1 0.76 - 1.16,
// mean 0.97; beyond 0.78 - 1.53, mean 1.07 (64 -> 64 at 56x56, N = 70, 18.4 -> 21.0; N = 256 61 and 61, where both wait for memory).
// (CONVMI_STREAM: 0 never, 1 or 2: with so many groups of 32 result channels wherever it fits -- a tuning aid, as are those that
// ask for another kernel)
void plan_stream(conv_plan *p)
{
    p->fwd_stream = p->bwd_stream = IgemmStreamPlan{};
    const conv_info_t &f = p->info;
    const char *env = getenv("CONVMI_STREAM");
    if (p->d.dtype != CONV_BF16 || (env ? atoi(env) == 0 : variant_asked_for())) return;
    auto plan = [&](const IgemmPlan &other, int Cb, int Kp, double transform) {
        if (env) return try_stream(p->d, p->pad_h, p->pad_w, Cb, Kp, atoi(env));
        IgemmStreamPlan best;
        const double other_us = estimate_us(other, false) + transform;
        double best_us = 0.88 * other_us;
        for (int fk = 1; fk <= 2; ++fk) {
            const IgemmStreamPlan c = try_stream(p->d, p->pad_h, p->pad_w, Cb, Kp, fk);
            const double us = c.ok ? stream_us(c) : 0;
            // (several tiles of result channels read the input that often: up to 1.09 between 0.8 and 0.88)
            if (!c.ok || us >= best_us || (c.a.n_kt > 1 && us >= 0.8 * other_us)) continue;
            best = c;
            best_us = us;
        }
        return best;
    };
    if (p->fwd.ok && !p->fwd.fallback && p->fwd.a.ksplit == 1) p->fwd_stream = plan(p->fwd, f.Cb, f.Kp, 0);
    if (p->bwd_mode == 1 && !p->bwd[0].p.fallback) {
        const IgemmPlan &b = p->bwd[0].p;
        p->bwd_stream = plan(b, f.Kb, f.Cp, b.a.fwd_wt ? 0 : transform_launch_us((double)f.Kb * 9 * f.Cp * 16));
        p->bwd_stream.a.fwd_wt = 1;
    }
}

// Weight update, bf16, at most 4 input channels: (tap, channel) rows on the bf16 MFMA.
bool plan_upd_c4_bf16(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool bf16 = d.dtype == CONV_BF16;
    if (bf16 && d.C <= 4 && upd_c4_bf16_exists(d.R, d.S)) {
        // one input channel block, bf16: (tap, channel) rows on the bf16 MFMA, eight waves,
        // two LDS buffers holding the bands as they sit in HBM
        auto plan_c4_bf16 = [&]() -> bool {
            const int NPO = f.Kp <= 32 ? 4 : 8;  // planes of 8 output channels
            const int NP = d.N * f.P;
            UpdArgs &a = p->ua;
            memset(&a, 0, sizeof(a));
            a.N = d.N; a.Cb = 1; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
            a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = pad_h; a.pad_w = pad_w;
            a.tap0 = 0; a.ntaps_all = d.R * d.S;
            a.q0 = 0; a.Qpitch = f.Q; a.copy0 = 0;
            a.runs = ceil_div(f.Q, 8);
            const int RP = a.runs * 8;
            a.Hs = (f.P - 1) * d.stride + d.R;
            // a lane addresses up to 7 pixels past the first pixel of its run's last window
            a.LW = std::max(d.W + 2 * pad_w, d.stride * (RP - 1) + 8);
            int TR = std::min(NP, 16);
            for (;; --TR) {
                if (TR < 1) return false;
                const int LR = max_band_rows(d.N, f.P, TR, a.Hs, d.stride, d.R);
                a.LRW = LR * a.LW;
                a.PLS_in = ceil_div(a.LRW, 64) * 64;
                // (+4 pixels: the two planes a 16-lane transposing read touches start 64
                // bytes apart in the 256-byte bank row)
                a.PLS_out = ceil_div(TR * RP + 8, 64) * 64 + 4;
                p->upd_lds = 2 * ((size_t)a.PLS_in + (size_t)NPO * a.PLS_out) * 16;
                if (p->upd_lds <= (size_t)kMaxLds) break;
            }
            p->upd_lds = std::max(p->upd_lds, (size_t)16 * 1024);  // the accumulator exchange
            a.TR = TR;
            a.n_ct = 1;
            a.n_kt = ceil_div(f.Kp, 64);
            int splits = std::max(1, 256 / a.n_kt);  // one workgroup per CU, one round
            splits = std::max(splits, ceil_div(NP * f.Q, 1 << 17));
            int rps = ceil_div(ceil_div(NP, splits), TR) * TR;
            splits = ceil_div(NP, rps);
            a.rows_per_split = rps;
            a.splits = splits;
            a.sampled = 0;
            a.total = a.n_kt * splits;
            a.per_xcd = ceil_div(a.total, 8);
            if ((double)(d.N + 1) * std::max(a.Hs, std::max(d.H, f.P * f.Kb)) >= 4.0e6 ||
                a.LRW >= (1 << 22) || TR * RP + 8 >= (1 << 22) || (double)d.N * d.H * d.W * 16 >= 4.0e9 ||
                (double)d.N * f.Kp * f.P * f.Q * 2 >= 4.0e9)
                return false;
            p->upd_grid = a.per_xcd * 8;
            p->upd_copies = splits;
            p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
            p->upd_c4_bf16 = true;
            p->upd_ok = true;
            return true;
        };
        if (plan_c4_bf16()) return true;
    }
    return false;
}

// Weight update, at most 4 input channels, fp32 MFMA (fp32 tensors, or bf16 widened into LDS).
bool plan_upd_c4(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool bf16 = d.dtype == CONV_BF16;
    const bool square_pad = pad_h == pad_w;  // the filter-specific kernels take one pad
    if (d.C <= 4 && square_pad && ((d.R == 7 && d.S == 7) || (d.R == 3 && d.S == 3))) {
        // (a plan that does not fit leaves the layer to the general kernels)
        auto plan_c4 = [&]() -> bool {
            // one input channel block: filter-row formulation, eight waves, two LDS buffers
            const int NPO = f.Kp <= 32 ? 8 : 16;  // planes of 4 output channels
            const int Qp = (f.Q + 1) & ~1;
            const int NP = d.N * f.P;
            UpdArgs &a = p->ua;
            memset(&a, 0, sizeof(a));
            a.N = d.N; a.Cb = 1; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
            a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = pad_h; a.pad_w = pad_w;
            a.tap0 = 0; a.ntaps_all = d.R * d.S;
            a.live_ch = d.C;
            int TR = std::min(NP, std::max(1, 256 / Qp));
            for (;; --TR) {
                if (TR < 1) return false;
                a.Hs = (f.P - 1) * d.stride + d.R;
                // a lane reads up to 8 pixels (32 floats) past the pair's first pixel
                a.LW = std::max((Qp - 1) * d.stride + 8, d.W + 2 * pad_w);
                const int LR = max_band_rows(d.N, f.P, TR, a.Hs, d.stride, d.R);
                a.LRW = LR * a.LW;
                // whole wave-level loads of 64 positions; the dO plane pitch is 1 (mod 8) pixels
                a.PLS_in = ceil_div(a.LRW, 64) * 64 + 8;
                a.PLS_out = ceil_div(TR * Qp, 64) * 64 + 1;
                p->upd_lds = 2 * ((size_t)a.PLS_in + (size_t)NPO * a.PLS_out) * 16;
                if (p->upd_lds <= (size_t)kMaxLds) break;
            }
            a.TR = TR;
            a.n_ct = 1;
            a.n_kt = ceil_div(f.Kp, 64);  // 64 output channels per workgroup
            // (bf16 tensors: the staged band must fit the kernel's register staging)
            if (bf16 && (a.PLS_in - 8 > 8 * 512 || 8 * TR * Qp > 4 * 512)) return false;
            // one workgroup per CU, one round
            int splits = std::max(1, 256 / a.n_kt);
            splits = std::max(splits, ceil_div(NP * f.Q, 1 << 17));  // chains of at most 2^15 pixels
            int rps = ceil_div(ceil_div(NP, splits), TR) * TR;
            splits = ceil_div(NP, rps);
            a.rows_per_split = rps;
            a.splits = splits;
            a.sampled = 0;
            a.total = a.n_kt * splits;
            a.per_xcd = ceil_div(a.total, 8);
            if ((double)(d.N + 1) * std::max(a.Hs, std::max(d.H, f.P * f.Kb)) >= 8.0e6 ||
                a.LRW >= (1 << 22) || 8 * TR * Qp >= (1 << 22) || (double)d.N * d.H * d.W * 16 >= 4.0e9 ||
                (double)d.N * f.Kp * f.P * f.Q * 4 >= 4.0e9)
                return false;
            p->upd_grid = a.per_xcd * 8;
            p->upd_copies = splits;
            p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
            p->upd_c4 = true;
            p->upd_ok = true;
            return true;
        };
        if (plan_c4()) return true;
    }
    return false;
}

// Weight update, fp32 1x1 without padding: flat pixel list, eight waves.
bool plan_upd_flat_f32(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool sampled = (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0);
    const bool bf16 = d.dtype == CONV_BF16;
    if (!bf16 && sampled) {
        // fp32 1x1: 256 channels of the wider tensor x up to 256 of the other per workgroup,
        // the pixel list split so that one round of workgroups fills the chip
        // (the wider side, but the input wherever it has 256 channels: partial dW keeps 4
        // input channels together, which the rows of an accumulator tile store as 16 bytes)
        const bool a_is_in = f.Cp >= f.Kp || f.Cp >= 256;
        const int chA = a_is_in ? f.Cp : f.Kp, chB = a_is_in ? f.Kp : f.Cp;
        const double npix = (double)d.N * f.P * f.Q;
        const int plA = a_is_in ? f.Cb : f.Kb, plB = a_is_in ? f.Kb : f.Cb;
        if (chA >= 256 && chB >= 32 && npix < 4.0e6 &&
            (double)(d.N + 1) * std::max(f.Cb, f.Kb) < 8.0e6 && (double)d.H * d.W < 8.0e6 &&
            (double)d.N * f.Cp * d.H * d.W * 4 < 4.0e9 && (double)d.N * f.Kp * f.P * f.Q * 4 < 4.0e9) {
            const int wb = chB >= 192 ? 4 : chB >= 96 ? 2 : 1, wp = 4 / wb, BP = 32;
            UpdArgs &a = p->ua;
            memset(&a, 0, sizeof(a));
            a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
            a.R = 1; a.S = 1; a.stride = d.stride; a.pad = 0; a.pad_w = 0; a.tap0 = 0; a.ntaps_all = 1;
            const int n_at = ceil_div(plA, 64), n_bt = ceil_div(plB, 16 * wb);
            a.n_ct = a_is_in ? n_at : n_bt;
            a.n_kt = a_is_in ? n_bt : n_at;
            const int tiles = n_at * n_bt;
            const int np = (int)npix;
            int splits = std::max(1, 256 / tiles);
            splits = std::max(splits, ceil_div(np, 1 << 16));
            const int pps = ceil_div(ceil_div(np, splits), BP) * BP;
            splits = ceil_div(np, pps);
            a.rows_per_split = pps;
            a.splits = splits;
            a.sampled = 1;
            a.total = tiles * splits;
            a.per_xcd = ceil_div(a.total, 8);
            p->upd_wb = wb;
            p->upd_a_is_in = a_is_in;
            p->upd_lds = upd_f32_1x1_lds_bytes(wb);
            p->upd_grid = a.per_xcd * 8;
            p->upd_copies = splits;
            p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
            p->upd_flat = true;
            (void)wp;
            p->upd_ok = true;
            return true;
        }
    }
    return false;
}

// Weight update, bf16 1x1 without padding: flat pixel list.
bool plan_upd_flat_bf16(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool sampled = (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0);
    const bool bf16 = d.dtype == CONV_BF16;
    if (bf16 && sampled && (double)d.N * f.P * f.Q < 4.0e6 &&
        (double)(d.N + 1) * std::max(f.Cb, f.Kb) < 8.0e6 && (double)d.H * d.W < 8.0e6 &&
        (double)d.N * f.Cp * d.H * d.W * 2 < 4.0e9 && (double)d.N * f.Kp * f.P * f.Q * 2 < 4.0e9) {
        // bf16 1x1: the dW block that moves the fewest bytes.  The input is staged once per
        // output-channel block and dO once per input-channel block (re-reads that the L2
        // mostly serves: weight 1/2; with stride 2 only every other pixel of a fetched line
        // is used), and the pixel list is split so that one round of workgroups fills the
        // chip, each split writing a partial dW that the reduce kernel reads back (HBM both
        // ways).  Fitted to the update times of the 14x14 and 7x7 layers at N = 256 under every
        // block shape: a 128 x 256 block there beats 256 x 256 by 5 - 12 % (half the partial
        // copies), except where dW itself is the largest tensor (1024 -> 2048).
        static const UpdRowsVariant kFlat[9] = {
            {1, 1, 4, 2, 1, 2, 4}, {1, 1, 2, 2, 2, 2, 4}, {1, 1, 1, 2, 4, 2, 4},
            {1, 1, 4, 1, 2, 2, 4}, {1, 1, 2, 1, 4, 2, 4}, {1, 1, 2, 2, 2, 1, 2},
            {1, 1, 4, 1, 2, 2, 2}, {1, 1, 2, 1, 4, 2, 2}, {1, 1, 2, 2, 2, 1, 1}};
        UpdRowsVariant rv{};
        bool have = false;
        double best = 0;
        for (const UpdRowsVariant &c : kFlat) {
            if (!upd_bf16_1x1_variant_exists(c)) continue;
            const int TC = c.wc * c.fc * 32, TK = c.wk * c.fk * 32;
            const int n_ct = ceil_div(f.Cp, TC), n_kt = ceil_div(f.Kp, TK);
            const double staged = (double)f.in_bytes / d.stride * n_kt + (double)f.out_bytes * n_ct;
            const double copies = 2.0 * std::max(1, 256 / (n_ct * n_kt)) * (double)f.dwt_bytes;
            const double cost = (0.5 * staged + copies) * (1.0 + 1e-4 * (TC + TK));
            if (!have || cost < best) { rv = c; best = cost; have = true; }
        }
        // (a tuning aid: CONVMI_UPD_FLAT="wc,wk,wp,fc,fk" asks for one variant)
        if (const char *env = getenv("CONVMI_UPD_FLAT")) {
            UpdRowsVariant c{1, 1, 0, 0, 0, 0, 0};
            if (sscanf(env, "%d,%d,%d,%d,%d", &c.wc, &c.wk, &c.wp, &c.fc, &c.fk) == 5 &&
                upd_bf16_1x1_variant_exists(c)) {
                rv = c;
                have = true;
            }
        }
        if (have) {
            const int TC = rv.wc * rv.fc * 32, TK = rv.wk * rv.fk * 32, BP = 64;
            UpdArgs &a = p->ua;
            memset(&a, 0, sizeof(a));
            a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
            a.R = 1; a.S = 1; a.stride = d.stride; a.pad = 0; a.pad_w = 0; a.tap0 = 0; a.ntaps_all = 1;
            a.n_ct = ceil_div(f.Cp, TC);
            a.n_kt = ceil_div(f.Kp, TK);
            const int tiles = a.n_ct * a.n_kt;
            const int np = d.N * f.P * f.Q;
            int splits = std::max(1, 256 / tiles);
            splits = std::max(splits, ceil_div(np, 1 << 16));
            const int pps = ceil_div(ceil_div(np, splits), BP) * BP;
            splits = ceil_div(np, pps);
            a.rows_per_split = pps;
            a.splits = splits;
            a.sampled = 1;
            a.total = tiles * splits;
            a.per_xcd = ceil_div(a.total, 8);
            p->urv = rv;
            p->upd_lds = upd_bf16_1x1_lds_bytes(rv);
            p->upd_grid = a.per_xcd * 8;
            p->upd_copies = splits;
            p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
            p->upd_flat_bf16 = true;
            p->upd_ok = true;
            return true;
        }
    }
    return false;
}

// Weight update, bf16 row kernel (8-pixel runs).
bool plan_upd_rows(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool sampled = (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0);
    const bool bf16 = d.dtype == CONV_BF16;
    // (this kernel takes the two pads separately)
    const bool rows_strided = d.stride > 1 && d.R == 3 && d.S == 3;
    const bool rows_5x5 = d.stride == 1 && d.R == 5 && d.S == 5;  // one launch per filter row
    const bool rows_rs = !sampled && (rows_strided || rows_5x5 ||
                         (d.stride == 1 &&
                          ((d.R == 3 && d.S == 3) || (d.R == 1 && (d.S == 3 || d.S == 7)) ||
                           (d.S == 1 && (d.R == 3 || d.R == 7)))));
    const int rows_R = rows_5x5 ? 1 : d.R;  // filter rows a launch of the row kernel serves
    if (bf16 && (rows_rs || sampled)) {
        // bf16 row kernel: 8-pixel runs, filter-column shifts in registers.
        // 3x3: all nine taps in the wave (144 accumulators).  1x1: the layer is bound by
        // HBM, so take the channel tile that re-reads the least (input is read once per
        // output-channel tile, dO once per input-channel tile), then the smaller tile.
        static const UpdRowsVariant k1x1[7] = {{1, 1, 2, 2, 2, 1, 1}, {1, 1, 2, 4, 1, 1, 1},
                                               {1, 1, 4, 2, 1, 1, 1}, {1, 1, 2, 4, 1, 1, 2},
                                               {1, 1, 4, 2, 1, 2, 1}, {1, 1, 2, 4, 1, 2, 2},
                                               {1, 1, 4, 2, 1, 2, 2}};
        UpdRowsVariant rv{};
        bool have = false;
        if (rows_rs) {
            // 64 x 128 channels, or 64 x 64 with two wave groups along the pixels
            rv = f.Kp <= 64 ? UpdRowsVariant{rows_R, d.S, 2, 2, 2, 1, 1, 0} : UpdRowsVariant{rows_R, d.S, 2, 4, 1, 1, 1, 0};
            rv.strided = rows_strided ? 1 : 0;
            have = upd_rows_variant_exists(rv);
        } else {
            double best = 0;
            for (const UpdRowsVariant &c : k1x1) {
                if (!upd_rows_variant_exists(c)) continue;
                const int TC = c.wc * c.fc * 32, TK = c.wk * c.fk * 32;
                const double bytes = (double)f.in_bytes * ceil_div(f.Kp, TK) +
                                     (double)f.out_bytes * ceil_div(f.Cp, TC);
                const double cost = bytes * (1.0 + 1e-4 * (TC + TK));
                if (!have || cost < best) { rv = c; best = cost; have = true; }
            }
        }
        if (have) {
            const int TC = rv.wc * rv.fc * 32, TK = rv.wk * rv.fk * 32, NPI = TC / 8, NPO = TK / 8;
            const int NP = d.N * f.P;
            UpdArgs &a = p->ua;
            memset(&a, 0, sizeof(a));
            a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
            a.R = rows_R; a.S = d.S; a.stride = d.stride; a.pad = pad_h; a.pad_w = pad_w;
            a.tap0 = 0; a.ntaps_all = d.R * d.S;
            a.q0 = 0; a.Qpitch = f.Q; a.copy0 = 0;
            a.sampled = sampled ? 1 : 0;
            const int lst = rows_strided ? d.stride : 1;  // input pixels per output pixel in a band
            a.Hs = sampled ? f.P : (f.P - 1) * lst + rows_R;
            // a lane reads a window of whole 4-pixel groups covering a run and its S-1 shifts
            const int win = (8 + d.S - 1 + 3) / 4 * 4;
            // Rows too wide for two bands in the LDS are cut into up to four strips of whole
            // 8-pixel runs, one launch per strip; beyond that the general kernel takes over.
            int TR = 0, Qs = f.Q;
            for (int ns = 1; ns <= 4 && TR < 1; ++ns) {
                Qs = ns == 1 ? f.Q : ceil_div(ceil_div(f.Q, ns), 8) * 8;
                if (ns > 1 && (sampled || Qs * (ns - 1) >= f.Q)) continue;
                a.runs = ceil_div(Qs, 8);
                const int RP = a.runs * 8;
                a.LW = sampled ? RP : std::max(ns == 1 ? d.W + 2 * pad_w : 0, RP + win - 8);
                if (rows_strided) a.LW = std::max(ns == 1 ? d.W + 2 * pad_w : 0, lst * (RP - 1) + d.S);
                for (TR = std::min(NP, 64); TR >= 1; --TR) {
                    const int LR = sampled ? TR : max_band_rows(d.N, f.P, TR, a.Hs, lst, rows_R);
                    a.LRW = LR * a.LW;
                    a.PLS_in = ceil_div(a.LRW, 64) * 64 + 4;
                    a.PLS_out = ceil_div(TR * RP + 8, 64) * 64 + 4;
                    p->upd_lds = 2 * ((size_t)NPI * a.PLS_in + (size_t)NPO * a.PLS_out) * 16;
                    if (p->upd_lds <= (size_t)kMaxLds) break;
                }
            }
            const int n_strips = ceil_div(f.Q, Qs);
            a.Q = Qs;
            if (TR >= 1) {
                a.TR = TR;
                a.n_ct = ceil_div(f.Cb, NPI);
                a.n_kt = ceil_div(f.Kb, NPO);
                const int tiles = a.n_ct * a.n_kt;
                // one workgroup per CU
                int splits = std::max(1, 256 / tiles);
                splits = std::max(splits, ceil_div(NP * f.Q, 1 << 15));
                int rps = ceil_div(ceil_div(NP, splits), TR) * TR;
                splits = ceil_div(NP, rps);
                a.rows_per_split = rps;
                a.splits = splits;
                a.total = tiles * splits;
                a.per_xcd = ceil_div(a.total, 8);
                if ((double)(d.N + 1) * std::max(a.Hs, f.P) < 4.0e6 &&
                    (double)d.N * f.Cp * d.H * d.W * 2 < 4.0e9 &&
                    (double)d.N * f.Kp * f.P * f.Q * 2 < 4.0e9) {
                    p->urv = rv;
                    p->upd_grid = a.per_xcd * 8;
                    p->upd_copies = splits * rv.wp * n_strips;
                    p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
                    p->upd_strips = n_strips;
                    p->upd_strip_w = Qs;
                    p->upd_row_launches = rows_R == d.R ? 1 : d.R;
                    p->upd_rows = true;
                    p->upd_ok = true;
                    return true;
                }
            }
        }
    }
    return false;
}

// Weight update, fp32 band kernel.
bool plan_upd_bands(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool sampled = (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0);
    const bool bf16 = d.dtype == CONV_BF16;
    // (this kernel takes the two pads separately)
    // (stride > 1: its odd-row path only, which addresses every pixel on its own)
    if (!bf16 && !sampled && upd_f32_bands_exists(d.R, d.S)) {
        // fp32 band kernel: 64 x 64 channel tile, one workgroup per CU, the LDS holds two
        // bands; the pixel range is split so that one round of workgroups fills the chip.
        // Layers with at most 32 channels on the input side (and on both) take 32 x 64
        // (32 x 32) blocks of dW with four (eight) pixel groups where every strip has odd rows.
        // (65 to 96 input channels: three 32-channel blocks waste less than two of 64)
        const int want = f.Cp <= 32 ? (f.Kp <= 32 ? 2 : 1) : (f.Cp > 64 && f.Cp <= 96 ? 1 : 0);
        int layout = upd_f32_bands_layout_exists(d.R, d.S, want, true) ? want : 0;
        const int NP = d.N * f.P;
        UpdArgs &a = p->ua;
        memset(&a, 0, sizeof(a));
        a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
        a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = pad_h; a.pad_w = pad_w;
        a.tap0 = 0; a.ntaps_all = d.R * d.S;
        a.Hs = (f.P - 1) * d.stride + d.R;
        a.q0 = 0; a.Qpitch = f.Q; a.copy0 = 0;
        size_t lds = 0;
        // Rows too wide for two bands in the LDS are cut into up to four strips of output
        // columns, one launch per strip; beyond that the general kernel takes over.
        int TR = 0, Qs = f.Q, n_strips = 1, NPI = 16, NPO = 16;
        for (int attempt = 0; attempt < 2 && TR < 1; ++attempt) {
        if (attempt == 1) {
            if (layout == 0) break;
            layout = 0;  // no odd strips: the 64 x 64 layout
        }
        NPI = layout == 0 ? 16 : 8;
        NPO = layout == 2 ? 8 : 16;
        for (n_strips = 1; n_strips <= 4; ++n_strips) {
            Qs = ceil_div(f.Q, n_strips);
            if (ceil_div(f.Q, Qs) != n_strips) continue;
            const int q_last = f.Q - (n_strips - 1) * Qs;
            if ((layout != 0 || d.stride > 1) && ((Qs & 1) == 0 || (q_last & 1) == 0)) continue;
            a.LW = (Qs - 1) * d.stride + d.S;
            if (n_strips == 1) a.LW = std::max(a.LW, d.W + 2 * pad_w);
            // (rows with an odd number of pixel pairs are shared out whole: even bands)
            auto rows_whole = [](int q) { return (q % 2 == 0) && ((q / 2) % 2 == 1); };
            const bool by_rows = rows_whole(Qs) || rows_whole(q_last);
            for (TR = std::min(NP, 64); TR >= 1; --TR) {
                if (by_rows && TR > 1 && (TR & 1)) continue;
                const int LR = max_band_rows(d.N, f.P, TR, a.Hs, d.stride, d.R);
                a.LRW = LR * a.LW;
                a.PLS_in = ceil_div(a.LRW, 64) * 64 + 1;
                a.PLS_out = ceil_div(TR * Qs + 1, 64) * 64 + 1;  // the band and one zero pixel
                lds = 2 * ((size_t)NPI * a.PLS_in + (size_t)NPO * a.PLS_out) * 16;
                if (lds <= (size_t)kMaxLds) break;
            }
            if (TR >= 1) break;
        }
        }
        // (strided: bands of a single output row lose to the four-wave kernel)
        if (d.stride > 1 && TR < 2) TR = 0;
        const size_t xch = upd_f32_bands_exchange_bytes(d.R, d.S, layout);
        a.Q = Qs;
        // (the band kernel addresses both tensors with 32-bit byte offsets)
        if (TR >= 1 && (double)(d.N + 1) * a.Hs < 4.0e6 && a.LRW < (1 << 22) &&
            (double)f.in_bytes < 4.0e9 && (double)f.out_bytes < 4.0e9) {
            a.TR = TR;
            a.n_ct = ceil_div(f.Cb, NPI);
            a.n_kt = ceil_div(f.Kb, NPO);
            const int tiles = a.n_ct * a.n_kt;
            int splits = std::max(1, 256 / tiles);
            splits = std::max(splits, ceil_div(NP * f.Q, 1 << 16));  // chains of at most 2^15 pixels
            int rps = ceil_div(ceil_div(NP, splits), TR) * TR;
            splits = ceil_div(NP, rps);
            a.rows_per_split = rps;
            a.splits = splits;
            a.sampled = 0;
            a.total = tiles * splits;
            a.per_xcd = ceil_div(a.total, 8);
            p->upd_lds = std::max(lds, xch);
            p->upd_grid = a.per_xcd * 8;
            p->upd_copies = splits * n_strips;
            p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;
            p->upd_strips = n_strips;
            p->upd_strip_w = Qs;
            p->upd_bands_layout = layout;
            p->upd_bands = true;
            p->upd_ok = true;
            return true;
        }
    }
    return false;
}

// Weight update, general four-wave kernels (any remaining filter the kernels cover).
void plan_upd_general(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const int pad_h = p->pad_h, pad_w = p->pad_w;
    const bool sampled = (d.R == 1 && d.S == 1 && pad_h == 0 && pad_w == 0);
    const bool bf16 = d.dtype == CONV_BF16;
    // General kernels.  3x3 and 1x1 in one launch; any other filter with S in {1, 3, 5, 7} as
    // one launch of the 1 x S kernel per filter row r (run with pad_h - r rows of padding,
    // writing taps [r*S, (r+1)*S) of the partial copies).
    // filter rows one launch serves: all of them for 3x3 and the one-column filters
    const bool whole = (d.R == 3 && d.S == 3) || (d.S == 1 && (d.R == 3 || d.R == 7));
    const int kR = whole ? d.R : 1;
    UpdVariant v{};
    if (d.R == 1 && d.S == 1)
        v = bf16 ? UpdVariant{CONV_BF16, 1, 1, 2, 2, 2, 2, 8, 8}
                 : UpdVariant{CONV_F32, 1, 1, 2, 2, f.Cp > 64 ? 2 : 1, f.Kp > 64 ? 2 : 1, 4, 4};
    else if (whole || d.S == 1 || d.S == 3 || d.S == 5 || d.S == 7)
        v = bf16 ? UpdVariant{CONV_BF16, kR, d.S, 2, 2, 1, 2, 8, 8}
                 : UpdVariant{CONV_F32, kR, d.S, 2, 2, 1, 1, 1, 4};
    else
        return;
    if (kR == 1 && d.S == 1 && d.R > 1)  // (other one-column filters: the 1x1 kernel per row)
        v = bf16 ? UpdVariant{CONV_BF16, 1, 1, 2, 2, 2, 2, 8, 8}
                 : UpdVariant{CONV_F32, 1, 1, 2, 2, f.Cp > 64 ? 2 : 1, f.Kp > 64 ? 2 : 1, 4, 4};
    if (!upd_variant_exists(v)) return;
    p->upd_row_launches = kR == d.R ? 1 : d.R;
    const int V = f.vlen;
    const int TC = v.wc * v.fc * 32, TK = v.wk * v.fk * 32, NPI = TC / V, NPO = TK / V, NT = 256;
    // fp32 pairs pixels along a row (row pitch rounded up to even, zero padded);
    // bf16 walks the band's pixels linearly in steps of 16.
    // (1x1 without padding: both bands are flat pixel lists, no row padding needed,
    // but a band must hold an even number of pixels)
    // A row wider than a band can hold is cut into strips of Qs output columns, one launch
    // (and one set of partial copies) per strip.
    int Qs = f.Q, Qp = 0, n_strips = 1;
    const int NP = d.N * f.P;
    // staged pixels a band may hold (see the staging maps of the two kernels)
    const int max_px_in = bf16 ? v.ppt_in * NT / NPI : NT / v.ppt_in;
    const int max_px_out = bf16 ? v.ppt_out * NT / NPO : NT / v.ppt_out;
    // fp32 tiles are kept below half of the LDS so that two workgroups share a CU
    const size_t lds_cap = bf16 ? (size_t)kMaxLds : (size_t)kMaxLds / 2;
    int TR = 0, Hs = 0, LW = 0, LR = 0, npxO = 0;
    for (n_strips = 1; TR < 1; ++n_strips) {
        if (n_strips > f.Q) return;
        Qs = ceil_div(f.Q, n_strips);
        if (ceil_div(f.Q, Qs) != n_strips) continue;
        const int q_last = f.Q - (n_strips - 1) * Qs;  // width of the last strip
        Qp = (bf16 || sampled) ? Qs : ((Qs + 1) & ~1);
        for (TR = std::min(NP, std::max(1, max_px_out / Qp)); TR >= 1; --TR) {
            if (sampled) { Hs = f.P; LW = Qp; LR = TR; }
            else {
                Hs = (f.P - 1) * d.stride + kR;
                LW = (Qp - 1) * d.stride + d.S;
                if (n_strips == 1) LW = std::max(LW, d.W + 2 * pad_w);
                LR = max_band_rows(d.N, f.P, TR, Hs, d.stride, kR);
            }
            if (!bf16 && sampled && TR > 1 && ((TR * Qp) % 2 != 0 || (TR * q_last) % 2 != 0)) continue;
            npxO = bf16 ? ceil_div(TR * Qp, 16) * 16 : TR * Qp;
            const size_t lds_est = ((size_t)NPI * (LR * LW + 16) + (size_t)NPO * (npxO + 16)) * 16;
            if (LR * LW <= max_px_in && npxO <= max_px_out && lds_est <= lds_cap) break;
        }
        if (TR >= 1) break;
    }
    p->upd_strips = n_strips;
    p->upd_strip_w = Qs;
    UpdArgs &a = p->ua;
    memset(&a, 0, sizeof(a));
    a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = Qs;
    a.R = kR; a.S = d.S; a.stride = d.stride; a.pad = pad_h; a.pad_w = pad_w;
    a.tap0 = 0; a.ntaps_all = d.R * d.S;
    a.q0 = 0; a.Qpitch = f.Q; a.copy0 = 0;
    a.TR = TR;
    a.n_ct = ceil_div(f.Cb, NPI);
    a.n_kt = ceil_div(f.Kb, NPO);
    const int tiles = a.n_ct * a.n_kt;
    // two rounds of two workgroups per CU (measured better than one round: the tail is
    // shorter), and no accumulation
    // chain longer than about 2^15 pixels
    const int target = 1024;
    int splits = std::max(1, (target + tiles / 2) / tiles);
    splits = std::max(splits, ceil_div(NP * f.Q, 1 << 15));
    int rps = ceil_div(ceil_div(NP, splits), TR) * TR;
    splits = ceil_div(NP, rps);
    a.rows_per_split = rps;
    a.splits = splits;
    a.Hs = Hs; a.LW = LW; a.LRW = LR * LW; a.Qp = Qp;
    if (bf16) {
        // plane pitch = 8 (mod 16) pixels: the two channel planes a 16-lane
        // transposing read touches sit half an LDS row apart
        a.PLS_in = ((a.LRW + 15) / 16) * 16 + 8;
        a.PLS_out = ((npxO + 15) / 16) * 16 + 8;
    } else {
        // plane pitch = 1 (mod 8) pixels: the 8 channel blocks a 32-lane group
        // reads land in different LDS banks
        a.PLS_in = ((a.LRW + 7) / 8) * 8 + 1;
        a.PLS_out = ((npxO + 7) / 8) * 8 + 1;
    }
    a.sampled = sampled ? 1 : 0;
    a.total = tiles * splits;
    a.per_xcd = ceil_div(a.total, 8);
    p->uv = v;
    p->upd_lds = ((size_t)NPI * a.PLS_in + (size_t)NPO * a.PLS_out) * 16;
    if (p->upd_lds > (size_t)kMaxLds) return;
    // the kernels divide linear row indices through a float reciprocal, exact below 2^22
    if ((double)(d.N + 1) * std::max(a.Hs, f.P) >= 4.0e6) return;
    p->upd_grid = a.per_xcd * 8;
    p->upd_copies = splits * n_strips;
    p->upd_ws = (size_t)splits * n_strips * f.dwt_bytes;
    p->upd_ok = true;
}

// Weight update with small blocks of dW: fc x fk fragments x one filter row per workgroup, nw waves
// with a ring of `depth` stages each, the pixel list in `splits` parts.
struct RingCand {
    int fc, fk, nw, depth, splits;
    int sum;  // the kernel's summation
    bool window = false;  // one window of the input for all taps of a filter row
};
bool ring_exists(const conv_plan *p, const RingCand &c, int sum)
{
    const conv_desc_t &d = p->d;
    if (c.window)
        return d.dtype == CONV_BF16 && p->pad_w <= 4 && upd_window_exists(d.S, d.stride, c.fc, c.fk, c.nw, c.depth, sum);
    return upd_ring_exists(d.dtype, d.S, c.fc, c.fk, c.nw, c.depth, sum);
}
int window_pitch(const conv_plan *p);
size_t ring_lds_bytes(const conv_plan *p, const RingCand &c)
{
    return c.window ? upd_window_lds_bytes() : upd_ring_lds_bytes(p->d.S, c.fc, c.fk, c.nw, c.depth);
}
// Error of the sums of the update that is planned, its partial copies added in eight chains, ascending.
double planned_upd_error(const conv_plan *p)
{
    const UpdArgs &a = p->ua;
    double pixels, waves = 1;
    if (p->upd_flat || p->upd_flat_bf16) {
        pixels = a.rows_per_split;
        waves = p->upd_flat ? 4 / p->upd_wb : p->urv.wp;
    } else {
        pixels = (double)a.rows_per_split * std::min(p->info.Q, p->upd_strips > 1 ? p->upd_strip_w : p->info.Q);
        if (p->upd_rows) waves = p->urv.wp;
        if (p->upd_bands) waves = p->upd_bands_layout == 0 ? 2 : p->upd_bands_layout == 1 ? 4 : 8;
    }
    pixels = std::min(pixels, (double)p->d.N * p->info.P * p->info.Q) / waves;
    const int c = p->upd_copies;
    return chain_error(pixels / (p->d.dtype == CONV_BF16 ? 16 : 1), 0) + (p->upd_rows || waves == 1 ? 0 : waves / 2) +
           (c > 1 ? ceil_div(c, 8) / 2.0 + std::min(8, c) / 2.0 : 0);
}
// ... and of the ring kernel's, in the summation c.sum; sets its group.
double ring_error(const conv_plan *p, const RingCand &c, UpdArgs &a, double most)
{
    const bool bf16 = p->d.dtype == CONV_BF16;
    const int chains = upd_reduce_chains(p->info.dwt_bytes / sizeof(float), a.splits);
    const double n = (double)ceil_div(a.rows_per_split, c.nw) / (bf16 ? 16 : 1), unit = c.depth * (bf16 ? 1.0 : 8.0);
    // (waves without a pixel add zeros)
    const int waves = std::min(c.nw, ceil_div(std::min(a.rows_per_split, p->d.N * a.P * a.Q), bf16 ? 16 : 8));
    const double rest = std::log2((double)waves) / 2 +
                        (a.splits > 1 ? ceil_div(a.splits, chains) / 2.0 + std::log2((double)chains) / 2 : 0);
    a.group = c.sum == 1 ? std::max(1, group_within(n, unit, kErrorMargin * most - rest)) : 0;
    return rest + chain_error(n, c.sum == 0 ? 0 : c.sum == 1 ? a.group * unit : 8);
}
bool plan_ring(const conv_plan *p, const RingCand &c, UpdArgs &a)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    if (!ring_exists(p, c, c.sum)) return false;
    // (a window's list: rows of as many slots as the input columns that a row reads need)
    const int pitch = c.window ? window_pitch(p) : f.Q;
    const double npix = (double)d.N * f.P * pitch;
    // exact small divisions, 24-bit products, 32-bit byte offsets
    if (npix >= 3.9e6 || (double)(d.N + 1) * std::max(f.Cb, f.Kb) >= 8.0e6 || (double)d.H * d.W >= 8.0e6 ||
        (double)f.in_bytes + ((double)p->pad_h + d.R) * d.W * 16 >= 4.0e9 || (double)f.out_bytes >= 4.0e9)
        return false;
    const int stage = c.nw * (d.dtype == CONV_BF16 ? 16 : 8);  // pixels of a workgroup's stage
    const int np = (int)npix;
    memset(&a, 0, sizeof(a));
    a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
    a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = p->pad_h; a.pad_w = p->pad_w;
    a.Qpitch = pitch;
    a.n_ct = ceil_div(f.Cp, c.fc * 32);
    a.n_kt = ceil_div(f.Kp, c.fk * 32);
    // (a wave's chain of additions is an nw-th of a split: at most 2^13 pixels)
    const int splits = std::max(c.splits, ceil_div(np, c.nw << 13));
    a.rows_per_split = ceil_div(ceil_div(np, splits), stage) * stage;
    a.splits = ceil_div(np, a.rows_per_split);
    const double total = (double)a.n_ct * a.n_kt * d.R * a.splits;
    if (total >= 1.0e8) return false;
    a.total = a.n_ct * a.n_kt * d.R * a.splits;
    a.per_xcd = ceil_div(a.total, 8);
    return true;
}

// What such an update takes, in microseconds, as far as the choice of its block and splits goes: as
// estimate_us, with the exchange of the waves' sums, the bytes that the blocks of a pixel range
// re-read, and the reduce launch.  Fitted to 5 000 launches (38 layers x N = 8 ... 256, three sets of
// tensors in turn, rms error 2 - 11 %); the choice is on average 2 % behind the best of what was tried.
double ring_estimate_us(const conv_plan *p, const RingCand &c, const UpdArgs &a)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const bool bf16 = d.dtype == CONV_BF16;
    struct Fit { double launch, fixed, stage, c_mfma, c_load, per_op, exch, reduce, copy_tb, hbm_tb, l2_tb; };
    static const Fit fits[2][3] = {{{6.0, 0, 590, 1.18, 1.5, 8, 14, 1.7, 3.1, 3.9, 10.9},
                                    {5.2, 0, 950, 1.12, 1.5, 0, 128, 3.9, 16.5, 4.0, 11.0},
                                    {2.4, 1510, 800, 1.2, 1.5, 20, 108, 3.0, 3.2, 4.0, 12.0}},
                                   {{3.6, 0, 340, 2.58, 1.64, 33, 103, 1.7, 4.4, 4.4, 16.7},
                                    {2.7, 520, 576, 0.54, 1.38, 19, 144, 1.8, 4.1, 2.5, 14.2},
                                    {2.4, 890, 1160, 0.0, 1.07, 0, 98, 2.3, 2.9, 4.0, 12.0}}};
    const Fit &q = fits[bf16 ? 1 : 0][d.S == 1 ? 0 : d.S == 3 ? 1 : 2];
    const int tiles = d.S * c.fc * c.fk, ops = d.S * c.fc + c.fk;
    const double mfma = tiles * (bf16 ? 32.0 : 256.0);
    const double stages = ceil_div(ceil_div(a.rows_per_split, c.nw * (bf16 ? 16 : 8)), c.depth) * c.depth;
    const double shared = std::max(mfma * q.c_mfma * c.nw / 4, ops * c.nw * 16 * q.c_load) *
                          (c.sum == 0 ? 1.0 : c.sum == 1 ? 1.03 : 1.18);
    // (a run of four pixels of a strided 1x1 layer is two lines)
    const double lines = bf16 && d.R * d.S == 1 && d.stride > 1 ? 1.7 : 1.0;
    const double lone = q.fixed + lines * stages * std::max(shared, mfma * q.c_mfma + q.stage + ops * q.per_op) + q.exch * tiles * c.nw;
    const double busy = stages * shared + q.exch * tiles * c.nw;
    // workgroups a CU holds: LDS, and registers (16 per tile, and what the operands take)
    int regs = 16 * tiles + (bf16 ? 4 : 3) * ops + 40;
    if (c.sum > 0) regs += c.sum == 1 ? 16 * tiles : tiles > 1 && tiles <= 8 ? 32 : 16;
    if (c.sum == 1 && tiles <= 3) regs = std::min(regs, 128);  // (launch bounds)
    const int resident = std::max(1, std::min((int)(kMaxLds / ring_lds_bytes(p, c)),
                                              std::min(8, 512 / regs) * 4 / c.nw));
    const int per_cu = ceil_div(a.per_xcd * 8, 256), full = per_cu / resident, rest = per_cu - full * resident;
    double t = full * std::max(lone, resident * busy) + (rest > 0 ? std::max(lone, rest * busy) : 0.0);
    t = t / 2.3e3 + q.launch;
    const double es = bf16 ? 2.0 : 4.0, out_b = (double)f.out_bytes;
    const double in_b = d.R * d.S > 1 ? (double)f.in_bytes
                                      : (double)d.N * f.Cp * f.P * f.Q * (d.stride > 1 ? 2 : 1) * es;
    // (which of the three bounds it is shades into the next: 160 -> 160 7x1 at 17x17 in 32 x 32 blocks, 196 us by the first
    // and 190 by the last, takes 230)
    const double bound[3] = {t, q.launch + (in_b + out_b) / (q.hbm_tb * 1e6),
                             q.launch + (in_b * a.n_kt + out_b * a.n_ct) * d.R / (q.l2_tb * 1e6)};
    t = shaded(bound);
    if (a.splits > 1) t += q.reduce + a.splits * (double)f.dwt_bytes * 2 / (q.copy_tb * 1e6);
    return t;
}

// Slots of an output row of a window's list: as many as the input columns that the row reads need.
int window_pitch(const conv_plan *p)
{
    const conv_desc_t &d = p->d;
    return std::max(p->info.Q, ceil_div(std::min(d.W, d.stride * (p->info.Q - 1) - p->pad_w + d.S), d.stride));
}
// Whether a strided 3x3 layer's update may run with one window of the input for all taps, and whether it does beside what
// the ring kernel would run as: time of the window / of the ring kernel, 569 layers of 7e9 ... 5e10 operations, three sets
// of tensors in turn (beyond 5e10 operations the ring kernel's lines leave a layer to the row kernel and it stays there;
// measured there too, 0.65 - 0.81 of that kernel's time):
//   - where the ring kernel takes the window's 64 x 64 blocks: from 1e10 operations 0.71 - 1.11, in the mean 0.92 (400 -> 400
//     at 20x20, N = 62, 61 -> 45 us; 128 -> 308 at 30x33, N = 121, 33 -> 37); 7e9 - 1e10 0.88 - 1.10;
//   - where it takes half a block, for fewer splits or none, what counts is how full the last round of workgroups is.  The
//     window's grid at least a tenth fuller: from 1e10 0.67 - 1.09, in the mean 0.92 (440 -> 256 at 13x14, N = 172, 168 half
//     blocks or three splits of 84, 50 -> 33 us); below 0.70 - 1.32;
//   - ... and not: 0.86 - 1.53, in the mean 1.10 (512 -> 320 at 55x54, N = 5, 240 or 120, 21 -> 31 us; 672 -> 232 at 39x38,
//     N = 20, 252 or 396, 34 -> 51), below 1e10 1.00 - 1.61;
//   - 64 and 96 channels 1.08 - 1.3; one slot in nine dead (192 -> 320 at 17x17) 1.05 and more.  With stride 1, where a tap's
//     pixels are neighbours, the ring kernel's own loads share their cache lines and the addresses cost more than they
//     save: 1.00 - 1.28, but 0.92 - 0.98 for 512 -> 512 at 7x7.
// Over all of them this costs 1.010 of the better kernel's time, the window from 1e10 on 1.015, never 1.07.
bool ring_applies(const conv_plan *p);
bool window_applies(const conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const double flops = 2.0 * d.N * d.K * d.C * d.R * d.S * (double)p->info.P * p->info.Q;
    return d.dtype == CONV_BF16 && d.stride == 2 && d.S == 3 && std::min(d.C, d.K) > 96 && flops >= 1.0e10 &&
           ring_applies(p) && 16 * window_pitch(p) <= 17 * p->info.Q;
}
bool window_beats(const RingCand &ring, const UpdArgs &ring_a, const UpdArgs &window_a)
{
    auto filled = [](const UpdArgs &a) { return (double)a.total / (ceil_div(a.total, 256) * 256); };
    return ring.fc * ring.fk >= 4 || filled(window_a) >= 1.1 * filled(ring_a);
}
// What such an update takes, in microseconds, as far as the choice of its splits goes.
double window_us(const conv_plan *p, const RingCand &c, const UpdArgs &a)
{
    const double stages = (double)a.rows_per_split / (c.nw * 16);
    return ceil_div(a.total, 256) * (0.62 * stages + 4) + (a.splits > 1 ? 3.5 + a.splits * (double)p->info.dwt_bytes * 2 / 4.0e6 : 0);
}

// Whether the ring kernel is the better one: lines between its time / the other kernel's, both measured with two
// sets of tensors in turn over 64 layers x N = 1 ... 256.
//   - 1x1, bf16 (three sets of tensors), by what is read, half of a strided layer's input, and by what the channel
//     tiles read again: up to 82 MB read 0.4 - 1.04 (stride 2: 512 -> 256 at 28x28, N = 160, 80 MB, 0.91; but 512 ->
//     1024 at 28x28, N = 96, 1.02 - 1.10 from run to run); up to 140 MB where the channel tiles ask for 260 MB at most
//     (64 -> 64 at 56x56, N = 160, 128 MB, 0.91; 288 -> 64 at 35x35, N = 160, 138 and 238 MB, 0.94; but 768 -> 192 at
//     17x17, N = 160, 89 and 355 MB, 1.16; 128 -> 512 at 28x28, N = 128, 128 and 411 MB, 1.14); beyond 140 MB mostly
//     slower (128 -> 512, 161 MB 1.07, 64 -> 80 at 73x73, 147 MB 1.17).  By operations: up to 2.3e10 (2.2e10 0.92;
//     2.6e10 0.98 - 1.07; 5.3e10 1.30), between two narrow sides (below 128 channels) 5e9 (4.4e9 1.04, 6.6e9 1.12).
//   - 1x1, fp32: with 256 channels on a side, where the other kernel has eight waves and 256 channels, up to 3e10
//     (1.3e10 0.63 - 0.98, 2.6e10 0.91 - 0.99, 3.3e10 0.96 - 1.0, 5.3e10 1.02 - 1.05); else everywhere (0.2 - 0.73).
//   - wider filters, fp32: everywhere (0.19 - 0.97; full 64 x 64 blocks beyond 5e10 operations 0.82 - 0.97).
//   - wider filters, bf16: everywhere (0.14 - 1.03), except stride 2 beyond 5e10 (288 -> 384 at 35x35, 2.8e10 0.91, 5.5e10 1.06,
//     9.2e10 1.02, 1.5e11 1.07), seven columns beyond 140 MB of tensors (40 -> 268 at 38x38, 114 MB 0.92, 142 MB 1.07, 171 MB
//     1.13) and one column beyond 82 MB (36 -> 760 7x1 at 20x21, 64 MB 0.98, 86 MB 1.07, 128 MB 1.15).
bool ring_applies(const conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const double flops = 2.0 * d.N * d.K * d.C * d.R * d.S * (double)f.P * f.Q;
    const int wide = std::max(d.C, d.K), narrow = std::min(d.C, d.K);
    if (d.R * d.S == 1) {
        if (d.dtype == CONV_F32) return !(wide >= 256 && narrow >= 32) || flops <= 3.0e10;
        return flops <= 2.3e10 && (flops <= 5.0e9 || wide >= 128);
    }
    if (d.dtype == CONV_F32) return true;
    const double tensors = (double)f.in_bytes + (double)f.out_bytes;
    if ((d.S == 7 && tensors > 1.4e8) || (d.S == 1 && tensors > 8.2e7)) return false;
    return !(d.stride > 1 && flops > 5.0e10);
}
// ... and for the chosen blocks of a bf16 1x1 layer, whether what they read allows it.
bool ring_reads_apply(const conv_plan *p, const UpdArgs &a)
{
    const double in = (double)p->info.in_bytes / (p->d.stride > 1 ? 2 : 1), out = (double)p->info.out_bytes;
    return in + out <= 8.2e7 || (in + out <= 1.4e8 && in * a.n_kt + out * a.n_ct <= 2.6e8);
}

bool plan_upd_ring(conv_plan *p)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    static const int kBlocks[][4] = {{1, 1, 8, 4}, {2, 2, 8, 2}, {2, 4, 8, 2}, {1, 1, 8, 2}, {1, 2, 8, 2}, {2, 2, 4, 4}};
    RingCand best{};
    UpdArgs best_a{};
    double best_us = 0;
    bool have = false;
    const double most_error = planned_upd_error(p);
    int force = -1, group = 0;
    auto consider = [&](RingCand c) {
        UpdArgs a;
        c.sum = std::max(0, force);
        if (!plan_ring(p, c, a)) return;
        double error = ring_error(p, c, a, most_error);
        if (force < 0) {
            // one chain where it is exact enough (summing apart costs 1 - 5 % in groups, 6 - 18 % by the stage)
            const int apart = ring_exists(p, c, 1) ? 1 : ring_exists(p, c, 2) ? 2 : 0;
            if (apart > 0 && error > (apart == 1 ? kErrorMargin : 0.9) * most_error + kOwnRounding) {
                c.sum = apart;
                error = ring_error(p, c, a, most_error);
            }
            if (error > most_error + kOwnRounding) return;
        }
        if (group > 0) a.group = group;
        const double us = c.window ? window_us(p, c, a) : ring_estimate_us(p, c, a);
        if (!have || us < best_us) {
            best = c;
            best_a = a;
            best_us = us;
            have = true;
        }
    };
    // (CONVMI_UPD_RING="fc,fk,waves,depth,splits[,sum[,group]]": one variant wherever it exists, in one chain unless
    // another summation is asked for; "0": never; "any": the planner's choice wherever there is one -- a tuning aid)
    const char *env = getenv("CONVMI_UPD_RING"), *window_env = getenv("CONVMI_UPD_WINDOW");
    const bool any = env && strcmp(env, "any") == 0;
    if ((env && !any) || window_env) {
        RingCand c{};
        if (window_env) {
            env = window_env;
            c.window = true;
        }
        force = 0;
        if (sscanf(env, "%d,%d,%d,%d,%d,%d,%d", &c.fc, &c.fk, &c.nw, &c.depth, &c.splits, &force, &group) < 5) return false;
        consider(c);
    } else if (any || ring_applies(p)) {
        for (const auto &k : kBlocks) {
            const int tiles = ceil_div(f.Cp, k[0] * 32) * ceil_div(f.Kp, k[1] * 32) * d.R;
            // (32 x 32 blocks of a 1x1 filter re-read both tensors once per 32 channels: for small ones)
            if (d.R * d.S == 1 && k[0] == 1 &&
                (double)f.in_bytes + (double)f.out_bytes > (d.dtype == CONV_BF16 ? 64.0e6 : 100.0e6))
                continue;
            // (a range that one split's chains do not hold is cut for all CUs, not into as few parts as that takes)
            if (tiles >= 256 || (double)d.N * f.P * f.Q <= (double)(k[2] << 13)) consider({k[0], k[1], k[2], k[3], 1, 0});
            consider({k[0], k[1], k[2], k[3], std::max(1, 256 / tiles), 0});
            if (d.S == 3 || d.dtype == CONV_F32) consider({k[0], k[1], k[2], k[3], std::max(1, 512 / tiles), 0});
        }
        if (!any && window_applies(p)) {
            const RingCand ring = best;
            const UpdArgs ring_a = best_a;
            const bool have_ring = have;
            const int tiles = ceil_div(f.Cp, 64) * ceil_div(f.Kp, 64) * d.R;
            have = false;
            for (const int splits : {1, std::max(1, 256 / tiles), std::max(1, 512 / tiles)}) consider({2, 2, 8, 3, splits, 0, true});
            if (have_ring && !(have && window_beats(ring, ring_a, best_a))) {
                best = ring;
                best_a = ring_a;
                have = true;
            }
        }
    }
    if (have && !env && d.dtype == CONV_BF16 && d.R * d.S == 1 && !ring_reads_apply(p, best_a)) return false;
    if (!have || (double)best_a.splits * f.dwt_bytes > std::max(2.0 * ((double)f.in_bytes + (double)f.out_bytes), 8.0e9))
        return false;
    p->upd_ring_us = best_us;
    p->ua = best_a;
    p->urv = UpdRowsVariant{d.R, d.S, 1, best.depth, best.nw, best.fc, best.fk, best.sum};
    p->upd_lds = ring_lds_bytes(p, best);
    p->upd_grid = best_a.per_xcd * 8;
    p->upd_copies = best_a.splits;
    p->upd_ws = (size_t)p->upd_copies * f.dwt_bytes;  // (one split writes dW itself; the caller brings it all the same)
    p->upd_flat = p->upd_flat_bf16 = p->upd_rows = p->upd_bands = false;
    p->upd_row_launches = p->upd_strips = 1;
    p->upd_ring = true;
    p->upd_window = best.window;
    p->upd_ok = true;
    return true;
}

// Whether a variant of the update on the bf16 instructions serves the layer.
bool upd_split_fits(const conv_plan *p, const UpdSplitVariant &v)
{
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    if (v.t == 1 ? v.pi != v.sp : false) return false;
    const double npix = (double)d.N * f.P * f.Q;
    // exact small divisions, 24-bit products, 32-bit byte offsets
    if (npix >= 3.9e6 || (double)(d.N + 1) * f.P >= 3.9e6 || (double)d.H * d.W >= 8.0e6 || (double)f.in_bytes >= 4.0e9 ||
        (double)f.out_bytes >= 4.0e9 || (double)f.dwt_bytes >= 4.0e9)
        return false;
    if (v.t > 1) {  // the positions under a stage
        const long long crossings = (v.sp - 2) / f.Q + 1, gap = std::max(0, v.t - d.stride);
        if ((v.sp - 1LL) * d.stride + v.t + crossings * gap > v.pi) return false;
    }
    return true;
}
// ... and its plan with `splits` ranges of pixels.
UpdSplitPlan try_upd_split(const conv_plan *p, const UpdSplitVariant &v, int splits)
{
    UpdSplitPlan s;
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    const double npix = (double)d.N * f.P * f.Q;
    UpdArgs &a = s.a;
    memset(&a, 0, sizeof(a));
    const int np = (int)npix;
    a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
    a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = p->pad_h; a.pad_w = p->pad_w;
    a.n_ct = ceil_div(f.Cp, v.wc * v.fc * 32);
    a.n_kt = ceil_div(f.Kp, v.wk * v.fk * 32);
    // (a wave's chain of additions, one for 16 pixels: at most 2^16 pixels)
    splits = std::max(splits, ceil_div(np, 1 << 16));
    a.rows_per_split = ceil_div(ceil_div(np, splits), v.sp) * v.sp;
    a.splits = ceil_div(np, a.rows_per_split);
    const double total = (double)a.n_ct * a.n_kt * d.R * ceil_div(d.S, v.t) * a.splits;
    if (total >= 1.0e8 || (double)a.splits * f.dwt_bytes > std::max(2.0 * ((double)f.in_bytes + (double)f.out_bytes), 8.0e9)) return s;
    a.total = (int)total;
    a.per_xcd = ceil_div(a.total, 8);
    s.v = v;
    s.grid = a.per_xcd * 8;
    s.ok = true;
    return s;
}

// Error of its sums in the units of planned_upd_error: an MFMA rounds the sum of the large products once for sixteen pixels, and what
// is left out.
double upd_split_error(const conv_plan *p, const UpdArgs &a)
{
    const int chains = upd_reduce_chains(p->info.dwt_bytes / sizeof(float), a.splits);
    return std::min((double)a.rows_per_split, (double)p->d.N * a.P * a.Q) / 32 + 0.5 + kLeftOut +
           (a.splits > 1 ? ceil_div(a.splits, chains) / 2.0 + std::log2((double)chains) / 2 : 0);
}

// Clocks of a CU's matrix cores, LDS and vector units that a stage takes.
double upd_split_stage(const UpdSplitVariant &v)
{
    const int waves = v.wc * v.wk, frags = v.t * v.fc * v.fk, q = v.sp / 16;
    const double mfma = q * frags * 192.0, reads = q * (v.t * v.fc + v.fk) * 6.0;
    const double items = ceil_div(v.wc * v.fc * 4 * v.pi, waves * 64) + ceil_div(v.wk * v.fk * 4 * v.sp, waves * 64);
    return (0.25 * mfma + 116 * items + 8.35 * reads + 47) * (waves / 4.0);
}
// What such an update takes, in microseconds, the reduce launch included: the form of ring_estimate_us.  Fitted to 14 700 launches
// (250 drawn layers, every variant, 192 ... 1024 workgroups; three sets of tensors in turn): rms error 10 %, the choice 2 % behind the
// fastest.  (From `limit` on, any bound beyond it will do.)
double upd_split_us(const conv_plan *p, const UpdSplitPlan &s, double limit)
{
    const UpdSplitVariant &v = s.v;
    const UpdArgs &a = s.a;
    const conv_info_t &f = p->info;
    const int waves = v.wc * v.wk, frags = v.t * v.fc * v.fk, q = v.sp / 16;
    const double simd = waves / 4.0, mfma = q * frags * 192.0, reads = q * (v.t * v.fc + v.fk) * 6.0;
    const double stages = ceil_div(a.rows_per_split, v.sp);
    const double shared = upd_split_stage(v);
    const double busy = stages * shared + 399.0 * frags * simd;
    const double lone = std::max(busy, 4056 + 262.0 * frags + stages * std::max(0.94 * mfma + 23.8 * reads + 806, shared));
    // (waves per SIMD that the registers leave room for)
    const int occ = v.t > 1 || frags == 4 ? 2 : frags == 1 && v.sp == 32 ? 4 : 3;
    const int resident = std::max(1, std::min((int)(kMaxLds / upd_split_lds_bytes(v)), occ * 4 / waves));
    const int per_cu = ceil_div(s.grid, 256), full = per_cu / resident, rest = per_cu - full * resident;
    const double t = full * std::max(lone, resident * busy) + (rest > 0 ? std::max(lone, rest * busy) : 0.0);
    const double out_b = (double)f.out_bytes, in_b = p->d.R * p->d.S > 1 ? (double)f.in_bytes : (double)p->d.N * f.Cp * f.P * f.Q * 4;
    const double again = p->d.R * ceil_div(p->d.S, v.t), launch = 2.8;
    const double bound[3] = {t / 2.1e3 + launch, launch + (in_b * a.n_kt + out_b * a.n_ct) * again / 14.6e6, launch + (in_b + out_b) / 4.0e6};
    const double reduce = a.splits > 1 ? 2.9 + a.splits * (double)f.dwt_bytes * 2 / 4.84e6 : 0;
    const double least = std::max(std::max(bound[0], bound[1]), bound[2]) + reduce;
    return least >= limit ? least : shaded(bound) + reduce;
}

// Whether the update runs on the bf16 instructions: where the estimate says that this is at least 8 % faster than `fp32_us`, and the
// sums are no less exact.  (Above that line 0.99 - 1.09 of the time, 11 of 161 drawn layers: 32 -> 64 3x3 at 147x147, N = 31, 216 -> 235 us.)
// (CONVMI_UPD_SPLIT="t,fc,fk,wc,wk,sp,pi,splits": one variant wherever it fits; 0: never -- a tuning aid, as are those that ask for
// a variant on the fp32 instructions)
void plan_upd_split(conv_plan *p, double fp32_us)
{
    p->upd_split = UpdSplitPlan{};
    if (p->d.dtype != CONV_F32) return;
    if (const char *env = getenv("CONVMI_UPD_SPLIT")) {
        UpdSplitVariant v{};
        int splits = 1;
        if (sscanf(env, "%d,%d,%d,%d,%d,%d,%d,%d", &v.t, &v.fc, &v.fk, &v.wc, &v.wk, &v.sp, &v.pi, &splits) < 7) return;
        if (splits >= 1 && upd_split_exists(v) && upd_split_fits(p, v)) p->upd_split = try_upd_split(p, v, splits);
    } else if (!getenv("CONVMI_UPD_RING") && !getenv("CONVMI_UPD_WINDOW")) {
        const double most_error = planned_upd_error(p) + kOwnRounding;
        // (and by 1.5 us: below 20 us the estimates are as far apart as that)
        double best_us = 0.92 * fp32_us - 1.5;
        for (int i = 0; const UpdSplitVariant *e = upd_split_variant(i); ++i) {
            const UpdSplitVariant &v = *e;
            const int blocks = ceil_div(p->info.Cp, v.wc * v.fc * 32) * ceil_div(p->info.Kp, v.wk * v.fk * 32) * p->d.R * ceil_div(p->d.S, v.t);
            // (a launch whose stages are dealt over all CUs, or of one workgroup, takes longer: nothing to look at)
            const double clocks = std::max(blocks * ((double)p->d.N * p->info.P * p->info.Q / v.sp) * upd_split_stage(v) / 256, 4056.0);
            if (clocks / 2.1e3 + 2.8 >= best_us || !upd_split_fits(p, v)) continue;
            int last = 0;
            for (const int target : {192, 256, 384, 512, 768, 1024}) {
                const int splits = std::max(1, target / blocks);
                if (splits == last) continue;
                last = splits;
                const UpdSplitPlan c = try_upd_split(p, v, splits);
                if (!c.ok) continue;
                const double us = upd_split_us(p, c, best_us);
                if (us < best_us && upd_split_error(p, c.a) <= most_error) {
                    p->upd_split = c;
                    best_us = us;
                }
            }
        }
    }
    if (p->upd_split.ok) {
        p->upd_copies = p->upd_split.a.splits;
        p->upd_ws = (size_t)p->upd_copies * p->info.dwt_bytes;  // (one split writes dW itself; the caller brings it all the same)
    }
}

// A plan of the update with both operands staged for all waves, `splits` ranges of pixels.
UpdSharedPlan try_upd_shared(const conv_plan *p, const UpdSharedVariant &v, int splits)
{
    UpdSharedPlan s;
    const conv_desc_t &d = p->d;
    const conv_info_t &f = p->info;
    if (!upd_shared_exists(v) || splits < 1 || upd_shared_lds_bytes(v) > (size_t)kMaxLds) return s;
    if (v.t > 1 && v.st != d.stride) return s;
    const double npix = (double)d.N * f.P * f.Q;
    // exact small divisions, 24-bit products, 32-bit byte offsets
    if (npix >= 3.9e6 || (double)(d.N + 1) * f.P >= 3.9e6 || (double)d.H * d.W >= 8.0e6 || (double)f.in_bytes >= 4.0e9 ||
        (double)f.out_bytes >= 4.0e9 || (double)f.dwt_bytes >= 4.0e9)
        return s;
    if (v.t > 1) {  // the positions under a stage (stride 2: of each parity)
        const long long crossings = (v.sp - 2) / f.Q + 1;
        const long long most = v.st == 1 ? v.sp - 1LL + v.t + crossings * (v.t - 1) : v.sp - 1LL + (v.t + 1) / 2 + crossings * ((v.t + 1) / 2 - 1);
        if (most > (v.st == 1 ? v.pi : v.pi / 2)) return s;
    }
    UpdArgs &a = s.a;
    memset(&a, 0, sizeof(a));
    const int np = (int)npix;
    a.N = d.N; a.Cb = f.Cb; a.H = d.H; a.W = d.W; a.Kb = f.Kb; a.Kp = f.Kp; a.P = f.P; a.Q = f.Q;
    a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad = p->pad_h; a.pad_w = p->pad_w;
    a.n_ct = ceil_div(f.Cp, v.wc * v.fc * 32);
    a.n_kt = ceil_div(f.Kp, v.wk * v.fk * 32);
    // (a wave's chain of additions, one for 16 pixels: at most 2^14 pixels)
    splits = std::max(splits, ceil_div(np, v.wp << 14));
    a.rows_per_split = ceil_div(ceil_div(np, splits), v.sp) * v.sp;
    a.splits = ceil_div(np, a.rows_per_split);
    const double total = (double)a.n_ct * a.n_kt * d.R * ceil_div(d.S, v.t) * a.splits;
    if (total >= 1.0e8 || (double)a.splits * f.dwt_bytes > std::max(2.0 * ((double)f.in_bytes + (double)f.out_bytes), 8.0e9)) return s;
    a.total = (int)total;
    a.per_xcd = ceil_div(a.total, 8);
    s.v = v;
    s.grid = a.per_xcd * 8;
    s.ok = true;
    return s;
}

// Error of its sums in the units of planned_upd_error: an addition for sixteen pixels.
double upd_shared_error(const conv_plan *p, const UpdSharedPlan &s)
{
    const UpdArgs &a = s.a;
    const int chains = upd_reduce_chains(p->info.dwt_bytes / sizeof(float), a.splits);
    return std::min((double)a.rows_per_split, (double)p->d.N * a.P * a.Q) / s.v.wp / 32 + std::log2((double)s.v.wp) / 2 +
           (a.splits > 1 ? ceil_div(a.splits, chains) / 2.0 + std::log2((double)chains) / 2 : 0);
}

// What such an update takes, in microseconds, the reduce launch included: the form of ring_estimate_us.  Fitted to 12 000 launches
// (220 drawn layers, every variant, 128 ... 768 workgroups; three sets of tensors in turn): rms error 9 %, the choice 1.3 % behind
// the fastest.
double upd_shared_us(const conv_plan *p, const UpdSharedPlan &s)
{
    const UpdSharedVariant &v = s.v;
    const UpdArgs &a = s.a;
    const conv_info_t &f = p->info;
    const int waves = v.wc * v.wk * v.wp, frags = v.t * v.fc * v.fk, q = v.sp / 16 / v.wp, po = ceil_div(v.sp, 64) * 64;
    const double simd = waves / 4.0, mfma = q * frags * 32.0, loads = (v.wc * v.fc * 4 * v.pi + v.wk * v.fk * 4 * po) / 64.0;
    const double stages = (double)a.rows_per_split / v.sp;
    const double shared = (0.83 * mfma + 27.5 * q + 60) * simd + 12.5 * loads, exch = 413.0 * frags * simd * (v.wp > 1 ? 1.0 : 0.38);
    const double busy = stages * shared + exch;
    const double lone = std::max(busy, 1600 + exch + stages * std::max(shared, 521 + 0.12 * mfma + 27.0 * 2 * q * (v.t * v.fc + v.fk)));
    // (waves per SIMD that the registers leave room for)
    const int regs = ceil_div(16 * frags + 8 * (v.fc + v.fk) + 30, 8) * 8;
    const int resident = std::max(1, std::min((int)(kMaxLds / upd_shared_lds_bytes(v)), std::min(8, 512 / regs) * 4 / waves));
    const int per_cu = ceil_div(s.grid, 256), full = per_cu / resident, rest = per_cu - full * resident;
    const double t = full * std::max(lone, resident * busy) + (rest > 0 ? std::max(lone, rest * busy) : 0.0);
    // (a run of four pixels of a strided 1x1 layer is two lines)
    const double out_b = (double)f.out_bytes, in_b = (double)f.in_bytes / (p->d.R * p->d.S == 1 ? p->d.stride : 1);
    const double again = p->d.R * ceil_div(p->d.S, v.t), launch = 2.85;
    const double bound[3] = {t / 2.1e3 + launch, launch + (in_b * a.n_kt + out_b * a.n_ct) * again / 18.0e6, launch + (in_b + out_b) / 5.84e6};
    double us = shaded(bound);
    if (a.splits > 1) us += 2.4 + a.splits * (double)f.dwt_bytes * 2 / 5.24e6;
    return us;
}

// What the row kernel takes for seven rows, in microseconds: a band's start, its pairs of runs, the chunks of 64 channels' rows and the halo
// around them, and the partial copies.  Fitted to 482 drawn layers: rms error 4 %, with two groups of pixels 6.
double row_update_us(const conv_plan *p)
{
    const UpdArgs &a = p->ua;
    const UpdRowsVariant &v = p->urv;
    const bool groups = v.wp > 1;
    const double bands = (double)ceil_div(a.rows_per_split, a.TR) * ceil_div(p->upd_grid, 256) * p->upd_strips;
    const double pairs = ceil_div(ceil_div(a.TR * a.runs, 2), v.wp), width = (double)p->d.W / p->upd_strips;
    const double chunks = 4.0e-3 * (v.wc * (a.TR + p->d.R - 1) + v.wk * a.TR) * width;
    const double copies = (double)a.splits * p->upd_strips * p->info.dwt_bytes * 2 / 5.0e6;
    return groups ? bands * (0.956 + 0.114 * pairs + 0.238 * chunks) + 2.38 * copies : bands * (0.594 + 0.280 * pairs + 0.0944 * chunks) + 1.09 * copies;
}

// Whether both operands are staged for all waves, and up to which estimate: lines between its time / the other kernel's, both
// measured in turn over 500 drawn layers and 500 of these families (C, K = 96 ... 720, N = 16 ... 256, three sets of tensors):
//   - seven columns: in the row kernel's place everywhere (205 layers, 0.59 - 0.92, in the mean 0.80; 504 -> 284 1x7 at 23x21, N = 27,
//     57 -> 41 us); in the ring kernel's place up to 0.87 of its estimate (60 layers, 0.55 - 0.93);
//   - seven rows: in the row kernel's place up to 0.94 of row_update_us (482 layers: 0.41 - 1.14, in the mean 0.75, nine above 1.04; beyond,
//     0.98 - 1.53: 140 -> 48 at 46x48, N = 139, 90 -> 136, 624 -> 52 at 58x56, N = 87, 277 -> 385); in the ring kernel's up to 0.83 of its
//     estimate (0.44 - 1.13, in the mean 0.82; beyond, 0.93 - 1.16);
//   - 3x3 with stride 2 from 1e10 operations (below, 0.8 - 1.6 whatever the estimates say): up to 1.15 times the window kernel's
//     estimate (0.81 - 1.01, in the mean 0.91, 288 -> 384 at 35x35, N = 32, 42 -> 36; beyond, 0.92 - 1.22); up to 0.74 times the ring
//     kernel's for 64 x 64 blocks (0.65 - 1.09, in the mean 0.84; beyond, 0.77 - 1.27), 0.70 times with at most 64 channels in (0.85 - 1.1, in the
//     mean 0.96; beyond, 1.02), never with at most 64 out, half of a block (50 layers, 1.02 - 1.29: 332 -> 52 at 60x63, N = 166, 151 -> 182); and in the row kernel's place where its runs of eight pixels
//     fill a row badly, or the row is long (0.66 - 0.98, in the mean 0.84; 288 -> 384 at 35x35, N = 92, 113 -> 89; else 0.9 - 1.16);
//   - other filters: 1x1 0.85 - 1.19, 3x3 with stride 1 0.9 - 1.5, 5x5 1.15: not built for them.
double shared_line_us(const conv_plan *p, double ring_us)
{
    const conv_desc_t &d = p->d;
    const double everywhere = 1.0e9;
    if (d.R * d.S == 7 && p->upd_ring) return (d.R == 7 ? 0.83 : 0.87) * ring_us;
    if (d.R * d.S == 7 && p->upd_rows) return d.R == 7 ? 0.94 * row_update_us(p) : everywhere;
    if (d.R * d.S == 7) return 0;
    const double flops = 2.0 * d.N * d.K * d.C * d.R * d.S * (double)p->info.P * p->info.Q;
    if (d.R != 3 || d.S != 3 || d.stride != 2 || flops < 1.0e10) return 0;
    if (p->upd_ring && p->upd_window) return 1.15 * ring_us;
    if (p->upd_ring) return p->urv.fc * p->urv.fk < 4 || d.K <= 64 ? 0 : (d.C <= 64 ? 0.70 : 0.74) * ring_us;
    const int Q = p->info.Q;
    return p->upd_rows && (Q >= 29 || ceil_div(Q, 8) * 8 >= 1.14 * Q) ? everywhere : 0;
}
// (CONVMI_UPD_SHARED="t,st,fc,fk,wc,wk,wp,sp,pi,nb,splits": one variant wherever it fits; 0: never -- a tuning aid, as are those that
// ask for another kernel)
void plan_upd_shared(conv_plan *p, double ring_us)
{
    p->upd_shared = UpdSharedPlan{};
    if (p->d.dtype != CONV_BF16) return;
    if (const char *env = getenv("CONVMI_UPD_SHARED")) {
        UpdSharedVariant v{};
        int splits = 1;
        if (sscanf(env, "%d,%d,%d,%d,%d,%d,%d,%d,%d,%d,%d", &v.t, &v.st, &v.fc, &v.fk, &v.wc, &v.wk, &v.wp, &v.sp, &v.pi, &v.nb, &splits) < 10) return;
        p->upd_shared = try_upd_shared(p, v, splits);
    } else if (!getenv("CONVMI_UPD_RING") && !getenv("CONVMI_UPD_WINDOW")) {
        const double most_error = planned_upd_error(p) + kOwnRounding;
        double best_us = shared_line_us(p, ring_us);
        if (best_us <= 0) return;
        for (int i = 0; const UpdSharedVariant *v = upd_shared_variant(i); ++i) {
            if ((v->t == 1) != (p->d.S == 1)) continue;
            const int blocks = ceil_div(p->info.Cp, v->wc * v->fc * 32) * ceil_div(p->info.Kp, v->wk * v->fk * 32) * p->d.R * ceil_div(p->d.S, v->t);
            int last = 0;
            for (const int target : {128, 192, 256, 384, 512, 768}) {
                const int splits = std::max(1, target / blocks);
                if (splits == last) continue;
                last = splits;
                const UpdSharedPlan c = try_upd_shared(p, *v, splits);
                if (!c.ok) continue;
                const double us = upd_shared_us(p, c);
                if (us < best_us && upd_shared_error(p, c) <= most_error) {
                    p->upd_shared = c;
                    best_us = us;
                }
            }
        }
    }
    if (p->upd_shared.ok) {
        p->upd_copies = p->upd_shared.a.splits;
        p->upd_ws = (size_t)p->upd_copies * p->info.dwt_bytes;  // (one split writes dW itself; the caller brings it all the same)
    }
}

void plan_upd(conv_plan *p)
{
    p->upd_ok = false;
    p->upd_ws = 0;
    p->upd_row_launches = 1;
    p->upd_strips = 1;
    p->upd_c4 = false;
    p->upd_c4_bf16 = false;
    p->upd_flat = false;
    p->upd_flat_bf16 = false;
    p->upd_rows = false;
    p->upd_bands = false;
    p->upd_ring = false;
    p->upd_window = false;
    // the kernels written for a family of layers first, each declining what it does not fit
    const bool few = plan_upd_c4_bf16(p) || plan_upd_c4(p);
    if (!(few || plan_upd_flat_f32(p) || plan_upd_flat_bf16(p) || plan_upd_rows(p) || plan_upd_bands(p)))
        plan_upd_general(p);
    // Partial copies that dwarf the tensors themselves (very wide rows cut into many strips,
    // under a filter with thousands of channels): no tiled plan; the direct kernel needs no
    // workspace.
    const double cap = std::max(2.0 * ((double)p->info.in_bytes + (double)p->info.out_bytes), 8.0e9);
    if (p->upd_ok && (double)p->upd_ws > cap) {
        p->upd_ok = false;
        p->upd_ws = 0;
    }
    // ... and over all but a first layer's, the ring kernel where it is the better one.  (Not where the
    // update is left to the untiled loop: that leaves the taps outside the image out, where the tiled
    // kernels multiply dO by zero, and an infinite dO would make the difference a NaN.)
    const bool ring = !few && p->upd_ok && plan_upd_ring(p);
    // ... and on the bf16 instructions, with the same exception
    // (the kernels of eight waves with 256 channels, beyond the ring kernel's line: 110 - 135 TFLOP/s)
    if (!few && p->upd_ok) {
        const double flops = 2.0 * p->d.N * p->d.K * p->d.C * p->d.R * p->d.S * (double)p->info.P * p->info.Q;
        plan_upd_split(p, ring ? p->upd_ring_us : flops / 1.35e8);
        plan_upd_shared(p, p->upd_ring_us);
    }
}

bool aligned16(const void *p) { return (reinterpret_cast<uintptr_t>(p) & 15u) == 0; }

}  // namespace

extern "C" {

const char *conv_status_str(conv_status_t s)
{
    switch (s) {
        case CONV_OK: return "ok";
        case CONV_EINVAL: return "invalid argument";
        case CONV_EUNSUPPORTED: return "unsupported problem";
        case CONV_EWORKSPACE: return "workspace missing or too small";
        case CONV_ELAUNCH: return "kernel launch failed";
        case CONV_ESCRATCH: return "problem needs more scratch than the library's static buffer holds";
    }
    return "unknown status";
}

conv_status_t conv_create(const conv_desc_t *desc, conv_handle_t *out)
{
    if (!desc) return CONV_EINVAL;
    return conv_create_rect(desc, desc->pad, desc->pad, out);
}

namespace {
// Whether every pass has a kernel of its own; `staged`: without the register-operand kernel in the untiled
// loops' place.
bool all_tiled(const conv_plan *q, bool staged)
{
    return q->fwd.ok && q->bwd_mode != 0 && q->upd_ok && !(staged && (q->fwd.fallback || q->bwd_ws_optional));
}
conv_status_t create_plan(const conv_desc_t *desc, int32_t pad_h, int32_t pad_w, int32_t max_images,
                          conv_handle_t *out);
}  // namespace

conv_status_t conv_create_rect(const conv_desc_t *desc, int32_t pad_h, int32_t pad_w, conv_handle_t *out)
{
    return create_plan(desc, pad_h, pad_w, 0, out);
}

conv_status_t conv_create_chunked(const conv_desc_t *desc, int32_t pad_h, int32_t pad_w,
                                  int32_t max_images, conv_handle_t *out)
{
    if (max_images < 1) return CONV_EINVAL;
    return create_plan(desc, pad_h, pad_w, max_images, out);
}

namespace {
// max_images: > 0: no launch covers more images; 0: chunks only where the tensors need them;
// < 0: never (the plan of a chunk)
conv_status_t create_plan(const conv_desc_t *desc, int32_t pad_h, int32_t pad_w, int32_t max_images,
                          conv_handle_t *out)
{
    if (!desc || !out) return CONV_EINVAL;
    *out = nullptr;
    const conv_desc_t &d = *desc;
    if (d.N < 1 || d.C < 1 || d.K < 1 || d.H < 1 || d.W < 1 || d.R < 1 || d.S < 1 || d.stride < 1 ||
        pad_h < 0 || pad_w < 0)
        return CONV_EINVAL;
    if (d.dtype != CONV_F32 && d.dtype != CONV_BF16) return CONV_EINVAL;
    // Everything below this point is computed in int; the extents are bounded here, in
    // 64-bit, so that no later product or sum can leave the range.
    const long long Hp = (long long)d.H + 2LL * pad_h, Wp = (long long)d.W + 2LL * pad_w;
    if (Hp < d.R || Wp < d.S) return CONV_EINVAL;
    const int kMaxExtent = 1 << 24, kMaxSmall = 1 << 16;
    if (d.N > kMaxExtent || d.C > kMaxExtent || d.K > kMaxExtent || d.H > kMaxExtent ||
        d.W > kMaxExtent || d.R > kMaxSmall || d.S > kMaxSmall || d.stride > kMaxSmall ||
        pad_h > kMaxSmall || pad_w > kMaxSmall)
        return CONV_EUNSUPPORTED;
    {
        const int V = vlen_of(d.dtype);
        const double Cp = (double)ceil_div(d.C, V) * V, Kp = (double)ceil_div(d.K, V) * V;
        const double P = (double)((Hp - d.R) / d.stride + 1), Q = (double)((Wp - d.S) / d.stride + 1);
        const double kMaxElems = 549755813888.0;  // 2^39 elements per activation tensor
        if ((double)d.N * Cp * d.H * d.W > kMaxElems || (double)d.N * Kp * P * Q > kMaxElems ||
            Cp * Kp * d.R * d.S > 2147483647.0)
            return CONV_EUNSUPPORTED;
    }

    conv_plan *p = new (std::nothrow) conv_plan();
    if (!p) return CONV_EINVAL;
    p->d = d;
    p->d.pad = pad_h;
    p->pad_h = pad_h;
    p->pad_w = pad_w;
    conv_info_t &f = p->info;
    memset(&f, 0, sizeof(f));
    f.P = (d.H + 2 * pad_h - d.R) / d.stride + 1;
    f.Q = (d.W + 2 * pad_w - d.S) / d.stride + 1;
    f.vlen = vlen_of(d.dtype);
    f.Cb = ceil_div(d.C, f.vlen);
    f.Kb = ceil_div(d.K, f.vlen);
    f.Cp = f.Cb * f.vlen;
    f.Kp = f.Kb * f.vlen;
    const size_t es = esize_of(d.dtype);
    f.in_bytes = (size_t)d.N * f.Cp * d.H * d.W * es;
    f.out_bytes = (size_t)d.N * f.Kp * f.P * f.Q * es;
    f.wt_bytes = (size_t)f.Cp * d.R * d.S * f.Kp * es;
    f.dwt_bytes = (size_t)f.Cp * d.R * d.S * f.Kp * sizeof(float);

    // The tiled planners index rows, staged tiles and channel blocks with int products; they
    // are only asked where those stay far inside the range (the kernels' own limits -- exact
    // float reciprocals below 2^22, 24-bit multiplies -- are tighter still and checked by each
    // planner).  Anything else runs on the untiled kernels, or in chunks of the minibatch.
    const bool tiled_domain = (long long)(d.N + 1) * std::max<long long>(Hp, f.P) < (1LL << 24) &&
                              Wp < (1 << 15) && f.Cp < (1 << 20) && f.Kp < (1 << 20) &&
                              d.R <= 64 && d.S <= 64 && d.stride <= 64;
    p->fwd_ws = 0;
    if (tiled_domain) {
        // Few tiles and a long reduction (small minibatch, inference): the reduction may be split
        // over workgroups too, fp32 partial results in the workspace, summed in a fixed order.
        const IgemmPlan base = plan_igemm_tile(d.dtype, d.N, f.Cb, d.H, d.W, f.Kp, f.P, f.Q, d.R, d.S, d.stride,
                                               pad_h, pad_w, f.P, f.Q, 1, 0, 0, 0, IgemmGeo{});
        const bool few_tiles = base.ok && base.a.total <= 128 && base.a.n_stage >= 4;
        // (what that sum's error is in the large tiles, split for 512 workgroups)
        double most_error = 0;
        if (few_tiles && d.dtype == CONV_F32) {
            const int per = ceil_div(base.a.n_stage, std::min(base.a.n_stage / 2, 512 / base.a.total));
            most_error = chain_error(4.0 * base.v.npl * d.R * d.S * per, 0) + ceil_div(base.a.n_stage, per) / 2.0;
        }
        p->fwd = plan_igemm(d.dtype, d.N, f.Cb, d.H, d.W, f.Kp, f.P, f.Q, d.R, d.S, d.stride, pad_h,
                            pad_w, f.P, f.Q, 1, 0, 0, 0, IgemmGeo{}, few_tiles, most_error);
        // (a filter without a staged kernel: the register-operand kernel, 0.16 - 0.85 of the untiled loops' time, the
        // same where both are a launch: 8 -> 8 channels, 1x5 at 9x9, 4.1 us)
        if (!p->fwd.ok) {
            IgemmGeo any_filter;
            any_filter.fallback = true;
            p->fwd = plan_igemm(d.dtype, d.N, f.Cb, d.H, d.W, f.Kp, f.P, f.Q, d.R, d.S, d.stride, pad_h,
                                pad_w, f.P, f.Q, 1, 0, 0, 0, any_filter);
        }
        if (p->fwd.ok && p->fwd.a.ksplit > 1)
            p->fwd_ws = (size_t)p->fwd.a.ksplit * d.N * f.Kp * f.P * f.Q * sizeof(float);
        // A first layer (one channel block in, one reduction step, one channel tile): resident
        // workgroups that keep the filter in LDS and prefetch the next input tile.
        // (CONVMI_STEM=0 keeps one workgroup per tile: a tuning aid.)
        p->fwd.a.live_ch = f.Cb == 1 ? std::min(d.C, vlen_of(d.dtype)) : vlen_of(d.dtype);
        p->fwd_stem_lds = 0;
        if (p->fwd.ok && !p->fwd.reg) {
            const char *env = getenv("CONVMI_STEM");
            const size_t need = igemm_stem_lds(p->fwd.v, p->fwd.a);
            if (need > 0 && need <= (size_t)kMaxLds && !(env && atoi(env) == 0)) p->fwd_stem_lds = need;
            // (CONVMI_STEM_WG=n: at most n workgroups per XCD, so that small inputs too give a
            // workgroup several tiles to walk: for tests of that path)
            if (const char *cap = getenv("CONVMI_STEM_WG"); cap && atoi(cap) > 0) p->fwd.a.jstep = atoi(cap);
        }
        if (p->fwd_stem_lds == 0) p->fwd_split = plan_split(p->fwd, d.R, d.S, FwdWeights{}, false);
        plan_bwd(p);
        plan_bwd_split(p);
        plan_stream(p);
        p->bwd_ws_optional = p->bwd_mode != 0 && p->bwd[0].p.fallback;
        plan_upd(p);
    }
    // A pass without a tiled plan falls to the direct kernels (any filter, stride and pad).
    if (direct_fits(d.dtype, d.N, f.Cb, f.Kb, d.H, d.W, f.P, f.Q, d.R, d.S)) {
        p->fwd_direct = !p->fwd.ok;
        p->bwd_direct = p->bwd_mode == 0;
        p->upd_direct = !p->upd_ok;
        DirectArgs &a = p->da;
        a = DirectArgs{};
        a.N = d.N; a.Cb = f.Cb; a.Kb = f.Kb; a.H = d.H; a.W = d.W; a.P = f.P; a.Q = f.Q;
        a.R = d.R; a.S = d.S; a.stride = d.stride; a.pad_h = pad_h; a.pad_w = pad_w;
        if (p->fwd_direct) p->fwd_ws = 0;
        if (p->bwd_direct) p->bwd_ws = 0;
        if (p->upd_direct) {
            p->upd_ws = 0;
            p->upd_copies = 1;  // dW is written once, by the kernel itself
        }
    }
    f.upd_splits = (p->upd_ok || p->upd_direct) ? p->upd_copies : 0;
    f.workspace_bytes = std::max(std::max(p->bwd_ws, p->upd_ws), p->fwd_ws);

    // Chunks of the minibatch.  On request: every pass.  Otherwise only for tensors of 4 GB
    // and more, which the tiled kernels' 32-bit byte offsets do not reach, or minibatches
    // whose linear row indices pass the kernels' exact-division range: the fewest equal
    // chunks whose plans are all tiled, for the passes that would else run untiled.
    // `staged`: those plans do without the register-operand kernel in the untiled loops' place.  If there
    // are none, chunks serve only the passes that this kernel takes (`exact`): the others, the
    // update above all, stay on the untiled loops, with their treatment of infinities and no workspace.
    int nc = 0;
    const bool forced = max_images > 0;
    bool exact = false;
    if (forced) {
        if (max_images < d.N) nc = max_images;
    } else if (max_images == 0 && d.N >= 2 && !all_tiled(p, true) &&
               ((double)std::max(f.in_bytes, f.out_bytes) >= 4.0e9 ||
                (double)(d.N + 1) * std::max(d.H + 2 * pad_h, f.P) * std::max(f.Cb, f.Kb) >= 4.0e6)) {
        for (const bool staged : {true, false}) {
            // (if one image alone has no tiled plan, no chunk has)
            conv_desc_t d1 = d;
            d1.N = 1;
            conv_handle_t q1 = nullptr;
            const bool any = create_plan(&d1, pad_h, pad_w, -1, &q1) == CONV_OK && (!staged || all_tiled(q1, true));
            delete q1;
            for (int k = 2; any && k <= 64 && k <= d.N && nc == 0; ++k) {
                conv_desc_t dd = d;
                dd.N = ceil_div(d.N, k);
                conv_handle_t q = nullptr;
                if (create_plan(&dd, pad_h, pad_w, -1, &q) != CONV_OK) break;
                if (all_tiled(q, staged)) nc = dd.N;
                delete q;
            }
            exact = nc > 0 && !staged;
            if (nc > 0) break;
        }
    }
    if (nc > 0) {
        conv_desc_t dd = d;
        dd.N = nc;
        const int n_chunks = ceil_div(d.N, nc), rest = d.N - (n_chunks - 1) * nc;
        conv_status_t st = create_plan(&dd, pad_h, pad_w, -1, &p->chunk);
        if (st == CONV_OK && rest != nc) {
            dd.N = rest;
            st = create_plan(&dd, pad_h, pad_w, -1, &p->tail);
        }
        if (st != CONV_OK) {
            delete p;
            return st;
        }
        p->n_chunks = n_chunks;
        p->chunk_n = nc;
        auto all = [&](auto &&f) { return f(p->chunk) && (!p->tail || f(p->tail)); };
        p->fwd_chunked = forced || (exact ? !p->fwd.ok && all([](const conv_plan *q) { return q->fwd.fallback || q->fwd_direct; })
                                          : !p->fwd.ok || p->fwd.fallback);
        p->bwd_chunked = forced || (exact ? p->bwd_mode == 0 && all([](const conv_plan *q) { return q->bwd_ws_optional || q->bwd_direct; })
                                          : p->bwd_mode == 0 || p->bwd_ws_optional);
        p->upd_chunked = forced || (!exact && !p->upd_ok);
        if (p->fwd_chunked) p->fwd_direct = false, p->fwd_ws = 0;
        if (p->bwd_chunked) p->bwd_direct = false, p->bwd_ws = 0;
        if (p->upd_chunked) p->upd_direct = false, p->upd_ws = 0;
        const size_t sub = std::max(p->chunk->info.workspace_bytes,
                                    p->tail ? p->tail->info.workspace_bytes : (size_t)0);
        p->chunk_ws = (sub + 255) / 256 * 256;
        const size_t need = p->chunk_ws + (p->upd_chunked ? (size_t)n_chunks * f.dwt_bytes : 0);
        if (p->upd_chunked) f.upd_splits = n_chunks;  // one dW per chunk, summed in chunk order
        f.workspace_bytes = std::max(f.workspace_bytes, need);
    }
    *out = p;
    return CONV_OK;
}
}  // namespace

conv_status_t conv_destroy(conv_handle_t h)
{
    if (!h) return CONV_EINVAL;
    delete h;
    return CONV_OK;
}

conv_status_t conv_query(conv_handle_t h, conv_info_t *info)
{
    if (!h || !info) return CONV_EINVAL;
    *info = h->info;
    return CONV_OK;
}

conv_status_t conv_fwd_fused(conv_handle_t h, const void *in, const void *wt, void *out,
                             const float *bias, const void *residual, int32_t relu, void *ws,
                             void *stream)
{
    return conv_fwd_fused_norm(h, in, wt, out, nullptr, bias, residual, relu, ws, stream);
}

conv_status_t conv_fwd_fused_norm(conv_handle_t h, const void *in, const void *wt, void *out,
                                  const float *scale, const float *bias, const void *residual,
                                  int32_t relu, void *ws, void *stream)
{
    if (!h || !in || !wt || !out) return CONV_EINVAL;
    if (!aligned16(in) || !aligned16(wt) || !aligned16(out) || !aligned16(ws) || !aligned16(bias) ||
        !aligned16(residual) || !aligned16(scale))
        return CONV_EINVAL;
    if (h->fwd_chunked) {
        const size_t in_img = h->info.in_bytes / h->d.N, out_img = h->info.out_bytes / h->d.N;
        for (int c = 0; c < h->n_chunks; ++c) {
            conv_plan *q = (c == h->n_chunks - 1 && h->tail) ? h->tail : h->chunk;
            const size_t n0 = (size_t)c * h->chunk_n;
            const conv_status_t st = conv_fwd_fused_norm(
                q, static_cast<const char *>(in) + n0 * in_img, wt, static_cast<char *>(out) + n0 * out_img,
                scale, bias, residual ? static_cast<const char *>(residual) + n0 * out_img : nullptr, relu,
                ws, stream);
            if (st != CONV_OK) return st;
        }
        return CONV_OK;
    }
    if (h->fwd_direct) {
        DirectArgs a = h->da;
        a.x = in;
        a.wt = wt;
        a.y = out;
        a.scale = scale;
        a.bias = bias;
        a.resid = residual;
        a.relu = relu != 0;
        return launch_direct_fwd(h->d.dtype, a, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    if (!h->fwd.ok) return CONV_EUNSUPPORTED;
    IgemmArgs a = h->fwd.a;
    // (a workspace is asked for by the plan on the fp32 instructions, whatever runs in its place)
    if (a.ksplit > 1 && !ws) return CONV_EWORKSPACE;
    const bool split = a.ksplit > 1 && (!h->fwd_split.ok || h->fwd_split.a.ksplit > 1);
    a.in = in;
    a.wt = wt;
    a.out = split ? ws : out;
    // a split reduction applies the operators where the partial results are summed
    a.scale = split ? nullptr : scale;
    a.bias = split ? nullptr : bias;
    a.resid = split ? nullptr : residual;
    a.relu = split ? 0 : (relu != 0);
    hipError_t e;
    if (h->fwd_stream.ok && !(scale || bias || residual || relu)) {
        IgemmStreamArgs b = h->fwd_stream.a;
        b.in = in;
        b.wt = wt;
        b.out = out;
        return launch_igemm_stream(h->fwd_stream, b, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    // (bf16 with fused operators: the resident-filter kernel's phases are a few microseconds
    // long there, and the residual's round trips do not fit into them -- 0.49 ms against 0.38
    // on the general kernel for layer 1 of Table I; in fp32 it is 0.64 against 0.89)
    const bool fused_ops = scale || bias || residual || relu;
    if (h->fwd_stem_lds && !h->fwd_split.ok && !(fused_ops && h->d.dtype == CONV_BF16))
        e = launch_igemm_stem(h->fwd.v, a, h->fwd_stem_lds, (hipStream_t)stream);
    else
        e = launch_plan(h->fwd, h->fwd_split, a, (hipStream_t)stream);
    if (e == hipSuccess && split)
        e = launch_split_reduce(h->d.dtype, static_cast<const float *>(ws), out,
                                (size_t)h->d.N * h->info.Kp * h->info.P * h->info.Q, a.ksplit, scale,
                                bias, residual, relu != 0, h->info.P * h->info.Q, h->info.Kb,
                                (hipStream_t)stream);
    return e == hipSuccess ? CONV_OK : CONV_ELAUNCH;
}

conv_status_t conv_fwd(conv_handle_t h, const void *in, const void *wt, void *out, void *ws,
                       void *stream)
{
    return conv_fwd_fused(h, in, wt, out, nullptr, nullptr, 0, ws, stream);
}

conv_status_t conv_bwd_data(conv_handle_t h, const void *dout, const void *wt, void *din, void *ws,
                            void *stream)
{
    if (!h || !dout || !wt || !din) return CONV_EINVAL;
    if (!aligned16(dout) || !aligned16(wt) || !aligned16(din) || !aligned16(ws)) return CONV_EINVAL;
    if (h->bwd_chunked) {
        const size_t in_img = h->info.in_bytes / h->d.N, out_img = h->info.out_bytes / h->d.N;
        for (int c = 0; c < h->n_chunks; ++c) {
            conv_plan *q = (c == h->n_chunks - 1 && h->tail) ? h->tail : h->chunk;
            const size_t n0 = (size_t)c * h->chunk_n;
            const conv_status_t st =
                conv_bwd_data(q, static_cast<const char *>(dout) + n0 * out_img, wt,
                              static_cast<char *>(din) + n0 * in_img, ws, stream);
            if (st != CONV_OK) return st;
        }
        return CONV_OK;
    }
    if (h->bwd_direct || (h->bwd_ws_optional && !ws)) {
        DirectArgs a = h->da;
        a.x = dout;
        a.wt = wt;
        a.y = din;
        return launch_direct_bwd(h->d.dtype, a, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    if (h->bwd_mode == 0) return CONV_EUNSUPPORTED;
    if (!ws) return CONV_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    if (h->bwd_classes.ok) {
        IgemmSplitClasses c = h->bwd_classes.c;
        for (IgemmArgs &a : c.cls) {
            a.in = dout;
            a.wt = wt;
            a.out = din;
        }
        return launch_igemm_split_classes(h->bwd_classes.v, c, h->bwd_classes.lds, s) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    if (h->bwd_stream.ok) {
        IgemmStreamArgs b = h->bwd_stream.a;
        b.in = dout;
        b.wt = wt;
        b.out = din;
        return launch_igemm_stream(h->bwd_stream, b, s) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    // the transformed weights of all classes, up to four to a launch (none where the kernel reads the forward pass's)
    const bool forward = (h->bwd_split.ok ? h->bwd_split.a : h->bwd[0].p.a).fwd_wt != 0;
    for (int i = 0; i < h->n_bwd && !forward;) {
        if (h->bwd[i].merged) {
            WtMergeArgs m = h->bwd[i].m;
            m.src = wt;
            m.dst = static_cast<char *>(ws) + h->bwd[i].ws_off;
            if (launch_wt_merge(h->d.dtype, m, s) != hipSuccess) return CONV_ELAUNCH;
            ++i;
            continue;
        }
        WtXformSet set{};
        for (set.n = 0; set.n < 4 && i < h->n_bwd; ++set.n, ++i) {
            set.x[set.n] = h->bwd[i].x;
            set.x[set.n].src = wt;
            set.x[set.n].dst = static_cast<char *>(ws) + h->bwd[i].ws_off;
        }
        if (launch_wt_xform(h->d.dtype, set, s) != hipSuccess) return CONV_ELAUNCH;
    }
    if (h->bwd_quad) {
        IgemmQuadArgs q;
        int grid = 0;
        size_t lds = 0;
        for (int i = 0; i < 4; ++i) {
            const BwdClass &b = h->bwd[i];
            q.cls[i] = b.p.a;
            q.cls[i].in = dout;
            q.cls[i].wt = b.p.a.fwd_wt ? wt : static_cast<char *>(ws) + b.ws_off;
            q.cls[i].out = din;
            q.end[i] = grid += b.p.grid;
            lds = std::max(lds, b.p.lds);
        }
        return launch_igemm_quad(h->d.dtype, q, lds, s) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    for (int i = 0; i < h->n_bwd; ++i) {
        const BwdClass &b = h->bwd[i];
        const void *wt2 = forward ? wt : static_cast<char *>(ws) + b.ws_off;
        IgemmArgs a = b.p.a;
        a.in = dout;
        a.wt = wt2;
        void *part = a.ksplit > 1 && (!h->bwd_split.ok || h->bwd_split.a.ksplit > 1) ? static_cast<char *>(ws) + b.part_off : nullptr;
        a.out = part ? part : din;
        if (launch_plan(b.p, h->bwd_split, a, s) != hipSuccess) return CONV_ELAUNCH;
        if (part && launch_split_reduce(h->d.dtype, static_cast<const float *>(part), din,
                                        (size_t)h->d.N * h->info.Cp * h->d.H * h->d.W, a.ksplit, nullptr, nullptr,
                                        nullptr, 0, h->d.H * h->d.W, h->info.Cb, s) != hipSuccess)
            return CONV_ELAUNCH;
    }
    return CONV_OK;
}

conv_status_t conv_upd(conv_handle_t h, const void *in, const void *dout, void *dwt, void *ws,
                       void *stream)
{
    if (!h || !in || !dout || !dwt) return CONV_EINVAL;
    if (!aligned16(in) || !aligned16(dout) || !aligned16(dwt) || !aligned16(ws)) return CONV_EINVAL;
    if (h->upd_chunked) {
        // dW of chunk c goes to slot c behind the chunks' own workspace; the slots are then
        // summed in chunk order
        if (!ws) return CONV_EWORKSPACE;
        const size_t in_img = h->info.in_bytes / h->d.N, out_img = h->info.out_bytes / h->d.N;
        char *slots = static_cast<char *>(ws) + h->chunk_ws;
        for (int c = 0; c < h->n_chunks; ++c) {
            conv_plan *q = (c == h->n_chunks - 1 && h->tail) ? h->tail : h->chunk;
            const size_t n0 = (size_t)c * h->chunk_n;
            const conv_status_t st =
                conv_upd(q, static_cast<const char *>(in) + n0 * in_img,
                         static_cast<const char *>(dout) + n0 * out_img,
                         slots + (size_t)c * h->info.dwt_bytes, ws, stream);
            if (st != CONV_OK) return st;
        }
        if (launch_upd_reduce(reinterpret_cast<const float *>(slots), static_cast<float *>(dwt),
                              h->info.dwt_bytes / sizeof(float), h->n_chunks, false,
                              (hipStream_t)stream) != hipSuccess)
            return CONV_ELAUNCH;
        return CONV_OK;
    }
    if (h->upd_direct) {
        DirectArgs a = h->da;
        a.x = in;
        a.wt = dout;
        a.y = dwt;
        return launch_direct_upd(h->d.dtype, a, (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    }
    if (!h->upd_ok) return CONV_EUNSUPPORTED;
    if (!ws) return CONV_EWORKSPACE;
    hipStream_t s = (hipStream_t)stream;
    UpdArgs a = h->ua;
    a.in = in;
    a.dout = dout;
    a.partial = static_cast<float *>(ws);
    hipError_t e = hipSuccess;
    if (h->upd_split.ok) {
        UpdArgs b = h->upd_split.a;
        b.in = in;
        b.dout = dout;
        b.partial = b.splits == 1 ? static_cast<float *>(dwt) : static_cast<float *>(ws);
        e = launch_upd_split(h->upd_split.v, b, h->upd_split.grid, s);
        if (b.splits == 1) return e == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    } else if (h->upd_shared.ok) {
        UpdArgs b = h->upd_shared.a;
        b.in = in;
        b.dout = dout;
        b.partial = b.splits == 1 ? static_cast<float *>(dwt) : static_cast<float *>(ws);
        e = launch_upd_shared(h->upd_shared.v, b, h->upd_shared.grid, s);
        if (b.splits == 1) return e == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    } else if (h->upd_ring) {
        if (a.splits == 1) a.partial = static_cast<float *>(dwt);
        e = h->upd_window ? launch_upd_window(a, h->upd_grid, s)
                          : launch_upd_ring(h->d.dtype, h->urv.fc, h->urv.fk, h->urv.wp, h->urv.wk, h->urv.strided, a,
                                            h->upd_grid, s);
        if (a.splits == 1) return e == hipSuccess ? CONV_OK : CONV_ELAUNCH;
    } else if (h->upd_flat_bf16)
        e = launch_upd_bf16_1x1(h->urv, a, h->upd_grid, s);
    else if (h->upd_flat)
        e = launch_upd_f32_1x1(h->upd_wb, h->upd_a_is_in, a, h->upd_grid, s);
    else if (h->upd_c4_bf16)
        e = launch_upd_c4_bf16(h->d.R, h->d.S, a, h->upd_lds, h->upd_grid, s);
    else if (h->upd_c4)
        e = launch_upd_c4(h->d.dtype, h->d.R, h->d.S, a, h->upd_lds, h->upd_grid, s);
    else if (h->upd_rows)
        for (int st = 0; st < h->upd_strips && e == hipSuccess; ++st) {
            a.q0 = st * h->upd_strip_w;
            a.Q = std::min(h->upd_strip_w, h->info.Q - a.q0);
            a.copy0 = st * a.splits * h->urv.wp;
            for (int r = 0; r < h->upd_row_launches && e == hipSuccess; ++r) {
                // (one launch, or filter row r of a taller filter: its taps, its share of
                // the padding)
                a.pad = h->pad_h - r;
                a.tap0 = r * h->d.S * (h->upd_row_launches > 1 ? 1 : 0);
                e = launch_upd_rows(h->urv, a, h->upd_lds, h->upd_grid, s);
            }
        }
    else if (h->upd_bands)
        for (int st = 0; st < h->upd_strips && e == hipSuccess; ++st) {
            a.q0 = st * h->upd_strip_w;
            a.Q = std::min(h->upd_strip_w, h->info.Q - a.q0);
            a.copy0 = st * a.splits;
            e = launch_upd_f32_bands(h->d.R, h->d.S, h->upd_bands_layout, a, h->upd_lds, h->upd_grid, s);
        }
    else
        for (int st = 0; st < h->upd_strips && e == hipSuccess; ++st) {
            // strip st of the output columns; a narrower last strip of a flat (unpadded
            // 1x1) band is its own row pitch
            a.q0 = st * h->upd_strip_w;
            a.Q = std::min(h->upd_strip_w, h->info.Q - a.q0);
            a.copy0 = st * a.splits;
            if (a.sampled) {
                a.Qp = a.Q;
                a.LW = a.Q;
                a.LRW = a.TR * a.Q;
            }
            for (int r = 0; r < h->upd_row_launches && e == hipSuccess; ++r) {
                // (one launch, or filter row r of a taller filter: its taps, its share of
                // the padding)
                a.pad = h->pad_h - r;
                a.tap0 = r * h->d.S * (h->upd_row_launches > 1 ? 1 : 0);
                e = launch_upd(h->uv, a, h->upd_lds, h->upd_grid, s);
            }
        }
    if (e != hipSuccess) return CONV_ELAUNCH;
    if (launch_upd_reduce(a.partial, static_cast<float *>(dwt), h->info.dwt_bytes / sizeof(float),
                          h->upd_copies, h->upd_c4_bf16, s) != hipSuccess)
        return CONV_ELAUNCH;
    return CONV_OK;
}

namespace {
// bytes of workspace a pass of this plan reads or writes
static size_t pass_ws_bytes(const conv_plan *h, int pass)
{
    const bool chunked = pass == 0 ? h->fwd_chunked : pass == 1 ? h->bwd_chunked : h->upd_chunked;
    if (chunked) {
        size_t need = h->chunk ? pass_ws_bytes(h->chunk, pass) : 0;
        if (h->tail) need = std::max(need, pass_ws_bytes(h->tail, pass));
        if (pass == 2) need = h->chunk_ws + (size_t)h->n_chunks * h->info.dwt_bytes;
        return need;
    }
    return pass == 0 ? h->fwd_ws : pass == 1 ? h->bwd_ws : h->upd_ws;
}
// whether the backward pass runs without one too, on the untiled kernel
static bool bwd_ws_optional(const conv_plan *h)
{
    if (h->bwd_chunked) return bwd_ws_optional(h->chunk) && (!h->tail || bwd_ws_optional(h->tail));
    return h->bwd_direct || h->bwd_ws_optional;
}
}  // namespace

conv_status_t conv_fwd_ws(conv_handle_t h, const void *in, const void *wt, void *out, void *ws,
                          size_t ws_bytes, void *stream)
{
    if (!h) return CONV_EINVAL;
    if (ws_bytes < pass_ws_bytes(h, 0)) return CONV_EWORKSPACE;
    return conv_fwd(h, in, wt, out, ws, stream);
}

conv_status_t conv_bwd_data_ws(conv_handle_t h, const void *dout, const void *wt, void *din,
                               void *ws, size_t ws_bytes, void *stream)
{
    if (!h) return CONV_EINVAL;
    if (ws_bytes < pass_ws_bytes(h, 1)) {
        if (!bwd_ws_optional(h)) return CONV_EWORKSPACE;
        ws = nullptr;
    }
    return conv_bwd_data(h, dout, wt, din, ws, stream);
}

conv_status_t conv_upd_ws(conv_handle_t h, const void *in, const void *dout, void *dwt, void *ws,
                          size_t ws_bytes, void *stream)
{
    if (!h) return CONV_EINVAL;
    if (ws_bytes < pass_ws_bytes(h, 2)) return CONV_EWORKSPACE;
    return conv_upd(h, in, dout, dwt, ws, stream);
}

// ---------------------------------------------------------------------------
// Backward by data for callers that cannot allocate: the transformed weights live in a
// file-scope device array instead of a caller-provided workspace.
// ---------------------------------------------------------------------------
namespace {
constexpr int kMaxDevices = 64;
}  // namespace
// Every GPU the library runs on holds its own copy of this array, at its own address, until
// the process ends.  In host code the name is only a handle for hipGetSymbolAddress.
static __device__ __align__(256) unsigned char scratch[kScratchBytes];

namespace {
// Device address of `scratch` on the current device (looked up once per device), or null.
static void *scratch_of_current_device()
{
    static std::mutex mu;
    static void *ptr_of[kMaxDevices] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= kMaxDevices) return nullptr;
    std::lock_guard<std::mutex> lock(mu);
    if (!ptr_of[dev]) {
        void *ptr = nullptr;
        if (hipGetSymbolAddress(&ptr, HIP_SYMBOL(scratch)) != hipSuccess) return nullptr;
        ptr_of[dev] = ptr;
    }
    return ptr_of[dev];
}
}  // namespace

conv_status_t conv_bwd_data_noalloc(conv_handle_t h, const void *dout, const void *wt, void *din,
                                    void *stream)
{
    if (!h || !dout || !wt || !din) return CONV_EINVAL;
    if (pass_ws_bytes(h, 1) > kScratchBytes)
        return bwd_ws_optional(h) ? conv_bwd_data(h, dout, wt, din, nullptr, stream) : CONV_ESCRATCH;
    void *ptr = scratch_of_current_device();
    if (!ptr) return CONV_ELAUNCH;
    return conv_bwd_data(h, dout, wt, din, ptr, stream);
}

size_t conv_noalloc_scratch_bytes(void) { return kScratchBytes; }

#define CHECK_PACK_ARGS(h, a, b)                                  \
    if (!(h) || !(a) || !(b)) return CONV_EINVAL;                 \
    if (!aligned16(a) || !aligned16(b)) return CONV_EINVAL;

conv_status_t conv_pack_in(conv_handle_t h, const void *nchw, void *blk, void *stream)
{
    CHECK_PACK_ARGS(h, nchw, blk);
    const conv_desc_t &d = h->d;
    return launch_pack_act(d.dtype, nchw, blk, d.N, d.C, d.H, d.W, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_pack_out(conv_handle_t h, const void *nkpq, void *blk, void *stream)
{
    CHECK_PACK_ARGS(h, nkpq, blk);
    const conv_desc_t &d = h->d;
    return launch_pack_act(d.dtype, nkpq, blk, d.N, d.K, h->info.P, h->info.Q,
                           (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_pack_wt(conv_handle_t h, const void *kcrs, void *blk, void *stream)
{
    CHECK_PACK_ARGS(h, kcrs, blk);
    const conv_desc_t &d = h->d;
    return launch_pack_wt(d.dtype, kcrs, blk, d.K, d.C, d.R, d.S, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_unpack_in(conv_handle_t h, const void *blk, void *nchw, void *stream)
{
    CHECK_PACK_ARGS(h, blk, nchw);
    const conv_desc_t &d = h->d;
    return launch_unpack_act(d.dtype, blk, nchw, d.N, d.C, d.H, d.W, (hipStream_t)stream) == hipSuccess
               ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_unpack_out(conv_handle_t h, const void *blk, void *nkpq, void *stream)
{
    CHECK_PACK_ARGS(h, blk, nkpq);
    const conv_desc_t &d = h->d;
    return launch_unpack_act(d.dtype, blk, nkpq, d.N, d.K, h->info.P, h->info.Q,
                             (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_unpack_wt(conv_handle_t h, const void *blk, void *kcrs, void *stream)
{
    CHECK_PACK_ARGS(h, blk, kcrs);
    const conv_desc_t &d = h->d;
    return launch_unpack_wt(d.dtype, blk, kcrs, d.K, d.C, d.R, d.S, h->info.vlen,
                            (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
}
conv_status_t conv_unpack_dwt(conv_handle_t h, const void *blk_f32, void *kcrs_f32, void *stream)
{
    CHECK_PACK_ARGS(h, blk_f32, kcrs_f32);
    const conv_desc_t &d = h->d;
    return launch_unpack_wt(CONV_F32, blk_f32, kcrs_f32, d.K, d.C, d.R, d.S, h->info.vlen,
                            (hipStream_t)stream) == hipSuccess ? CONV_OK : CONV_ELAUNCH;
}

// What runs in the place of the plan on the fp32 instructions that stands before it.
static void describe_stream(const IgemmStreamPlan &p, char *buf, size_t buflen)
{
    if (!p.ok) return;
    const size_t n = strlen(buf);
    snprintf(buf + n, buflen - n, " instead=igemm_stream,channels%d,rows%d,steps%d,workgroups%d,lds%zu", p.cs * 16, p.fk * 32, p.a.steps, p.a.total,
             igemm_stream_lds_bytes(p));
}
void describe_split(const SplitPlan &s, char *buf, size_t buflen)
{
    if (!s.ok) return;
    const size_t n = strlen(buf);
    if (s.nw > 0)
        snprintf(buf + n, buflen - n, " on_bf16x3=igemm_reg_split,%dx%d,waves%d,fw%d,tiles%d,lds%zu", s.fk, s.fm,
                 s.nw, s.a.fwd_wt, s.a.total, s.lds);
    else
        snprintf(buf + n, buflen - n, " on_bf16x3=igemm_split,%dx%d,fm%d,sets%d,groups%d,shares%d,strips%d,fw%d,tiles%d,lds%zu",
                 s.v.wk, s.v.wm, s.v.fm, s.v.kw, s.v.g, s.v.ni, s.a.n_qt, s.a.fwd_wt, s.a.total, s.lds);
}
static void describe_classes(const SplitClassesPlan &s, char *buf, size_t buflen)
{
    if (!s.ok) return;
    const size_t n = strlen(buf);
    snprintf(buf + n, buflen - n, " on_bf16x3=igemm_split_classes,%dx%d,fm%d,sets%d,groups%d,shares%d,strips%d,workgroups%d,lds%zu", s.v.wk, s.v.wm,
             s.v.fm, s.v.kw, s.v.g, s.v.ni, s.c.cls[0].n_qt, s.c.end[3], s.lds);
}
static conv_status_t describe_update(conv_handle_t h, char *buf, size_t buflen)
{
    if (h->upd_ring) {
        snprintf(buf, buflen,
                 "upd_ring dt=%d RS=%dx%d waves=1x1x%d ring=%d frags=%dx%d sum=%d group=%d pixels/split=%d splits=%d tiles=%dx%dx%d "
                 "grid=%d lds=%zu launches=1 window=%d",
                 (int)h->d.dtype, h->d.R, h->d.S, h->urv.wp,
                 h->urv.wk, h->urv.fc, h->urv.fk, h->urv.strided, h->ua.group, h->ua.rows_per_split, h->ua.splits,
                 h->ua.n_ct, h->ua.n_kt, h->d.R, h->upd_grid, h->upd_lds, h->upd_window ? h->ua.Qpitch : 0);
        return CONV_OK;
    }
    if (h->upd_flat_bf16) {
        snprintf(buf, buflen,
                 "upd_1x1 dt=1 waves=%dx%dx%d frags=%dx%d pixels/split=%d splits=%d tiles=%dx%d "
                 "grid=%d lds=%zu",
                 h->urv.wc, h->urv.wk, h->urv.wp, h->urv.fc, h->urv.fk, h->ua.rows_per_split,
                 h->ua.splits, h->ua.n_ct, h->ua.n_kt, h->upd_grid, h->upd_lds);
        return CONV_OK;
    }
    if (h->upd_flat) {
        snprintf(buf, buflen,
                 "upd_1x1 dt=0 waves=2x%dx%d tile=256x%d (%s) pixels/split=%d splits=%d tiles=%dx%d "
                 "grid=%d lds=%zu",
                 h->upd_wb, 4 / h->upd_wb, 64 * h->upd_wb, h->upd_a_is_in ? "in x out" : "out x in",
                 h->ua.rows_per_split, h->ua.splits, h->ua.n_ct, h->ua.n_kt, h->upd_grid,
                 h->upd_lds);
        return CONV_OK;
    }
    if (h->upd_c4 || h->upd_c4_bf16) {
        snprintf(buf, buflen,
                 "upd_c4 dt=%d mfma=%s RS=%dx%d waves=%s TR=%d splits=%d rows/split=%d ktiles=%d grid=%d lds=%zu",
                 (int)h->d.dtype, h->upd_c4_bf16 ? "bf16" : "f32", h->d.R, h->d.S,
                 h->info.Kp <= 32 ? "1x8" : "2x4", h->ua.TR, h->ua.splits, h->ua.rows_per_split, h->ua.n_kt,
                 h->upd_grid, h->upd_lds);
        return CONV_OK;
    }
    if (h->upd_rows) {
        snprintf(buf, buflen,
                 "upd_rows dt=1 RS=%dx%d waves=%dx%dx%d frags=%dx%d TR=%d runs=%d splits=%d "
                 "rows/split=%d tiles=%dx%d grid=%d lds=%zu launches=%d",
                 h->d.R, h->d.S, h->urv.wc, h->urv.wk, h->urv.wp, h->urv.fc, h->urv.fk, h->ua.TR,
                 h->ua.runs, h->ua.splits, h->ua.rows_per_split, h->ua.n_ct, h->ua.n_kt,
                 h->upd_grid, h->upd_lds, h->upd_strips * h->upd_row_launches);
        return CONV_OK;
    }
    if (h->upd_bands) {
        snprintf(buf, buflen,
                 "upd_bands dt=0 RS=%dx%d waves=%s frags=1x1 TR=%d splits=%d rows/split=%d "
                 "tiles=%dx%d grid=%d lds=%zu launches=%d",
                 h->d.R, h->d.S,
                 h->upd_bands_layout == 0 ? "2x2x2" : h->upd_bands_layout == 1 ? "1x2x4" : "1x1x8",
                 h->ua.TR, h->ua.splits, h->ua.rows_per_split, h->ua.n_ct,
                 h->ua.n_kt, h->upd_grid, h->upd_lds, h->upd_strips);
        return CONV_OK;
    }
    snprintf(buf, buflen,
             "upd dt=%d RS=%dx%d waves=%dx%d frags=%dx%d TR=%d splits=%d rows/split=%d "
             "tiles=%dx%d grid=%d lds=%zu launches=%d",
             h->uv.dtype, h->uv.r, h->uv.s, h->uv.wc, h->uv.wk, h->uv.fc, h->uv.fk, h->ua.TR,
             h->ua.splits, h->ua.rows_per_split, h->ua.n_ct, h->ua.n_kt, h->upd_grid,
             h->upd_lds, h->upd_row_launches * h->upd_strips);
    return CONV_OK;
}
conv_status_t conv_describe(conv_handle_t h, int32_t pass, char *buf, size_t buflen)
{
    if (!h || !buf || buflen == 0) return CONV_EINVAL;
    buf[0] = 0;
    if ((pass == 0 && h->fwd_chunked) || (pass == 1 && h->bwd_chunked) || (pass == 2 && h->upd_chunked)) {
        const int n = snprintf(buf, buflen, "chunks=%d images=%d: ", h->n_chunks, h->chunk_n);
        if (n < 0 || (size_t)n >= buflen) return CONV_EINVAL;
        const conv_status_t st = conv_describe(h->chunk, pass, buf + n, buflen - n);
        if (st == CONV_OK && pass == 2) {
            const size_t end = strlen(buf);
            snprintf(buf + end, buflen - end, " chunk_chains=%d",
                     upd_reduce_chains(h->info.dwt_bytes / sizeof(float), h->n_chunks));
        }
        return st;
    }
    if ((pass == 0 && h->fwd_direct) || (pass == 1 && h->bwd_direct) || (pass == 2 && h->upd_direct)) {
        const DirectArgs &a = h->da;
        const int V = h->info.vlen;
        // (the kernels stride over what a capped grid of 2^22 workgroups does not reach)
        const size_t grid = std::min<size_t>(
            pass == 0   ? ((size_t)a.N * a.Kb * a.P * a.Q * V + 255) / 256
            : pass == 1 ? ((size_t)a.N * a.Cb * a.H * a.W * V + 255) / 256
                        : (size_t)a.Cb * a.R * a.S * a.Kb,
            (size_t)1 << 22);
        snprintf(buf, buflen, "direct dt=%d RS=%dx%d stride=%d threads=256 grid=%zu lds=%d launches=1",
                 (int)h->d.dtype, a.R, a.S, a.stride, grid, pass == 2 ? 4 * V * V * 4 : 0);
        return CONV_OK;
    }
    if (pass == 0 || pass == 1) {
        const IgemmPlan *p = pass == 0 ? &h->fwd : &h->bwd[0].p;
        if (pass == 1 && h->bwd_mode == 0) return CONV_EUNSUPPORTED;
        if (!p->ok) return CONV_EUNSUPPORTED;
        if (p->reg) {
            snprintf(buf, buflen,
                     "%s dt=%d waves=%d frags=%dx%d RS=%dx%d tiles=%d (m=%d k=%d) xcd_kgroups=%d grid=%d lds=%zu "
                     "steps=%d group=%d ksplit=%d launches=%d",
                     p->patch ? "igemm_patch" : "igemm_reg", p->v.dtype, p->v.wk, p->v.fk, p->v.fm, p->v.r, p->v.s,
                     p->a.total, p->a.n_mt, p->a.n_kt,
                     p->a.gk, p->grid, p->lds, p->a.n_stage, p->a.group, p->a.ksplit, pass == 0 || h->bwd_quad ? 1 : h->n_bwd);
            if (p->a.fwd_wt) strncat(buf, " forward_weights=1", buflen - strlen(buf) - 1);
            describe_split(pass == 0 ? h->fwd_split : h->bwd_split, buf, buflen);
            describe_stream(pass == 0 ? h->fwd_stream : h->bwd_stream, buf, buflen);
            if (pass == 1) describe_classes(h->bwd_classes, buf, buflen);
            return CONV_OK;
        }
        snprintf(buf, buflen,
                 "igemm dt=%d waves=%dx%d frags=%dx%d npl=%d nt=%d RS=%dx%d ppt=%d TR=%d TQ=%d tiles=%d "
                 "(m=%d q=%d k=%d) xcd_kgroups=%d grid=%d lds=%zu stages=%d group=%d ksplit=%d launches=%d",
                 p->v.dtype, p->v.wk, p->v.wm, p->v.fk, p->v.fm, p->v.npl, p->v.nt, p->v.r, p->v.s, p->v.ppt,
                 p->a.TR, p->a.TQ, p->a.total, p->a.n_mt, p->a.n_qt, p->a.n_kt, p->a.gk, p->grid, p->lds,
                 p->a.n_stage, p->a.group, p->a.ksplit, pass == 0 || h->bwd_quad ? 1 : h->n_bwd);
        if (p->a.fwd_wt) strncat(buf, " forward_weights=1", buflen - strlen(buf) - 1);
        if (pass == 0 && h->fwd_stem_lds) {
            const size_t n = strlen(buf);
            snprintf(buf + n, buflen - n, " resident_filter_lds=%zu", h->fwd_stem_lds);
        }
        describe_split(pass == 0 ? h->fwd_split : h->bwd_split, buf, buflen);
        describe_stream(pass == 0 ? h->fwd_stream : h->bwd_stream, buf, buflen);
        if (pass == 1) describe_classes(h->bwd_classes, buf, buflen);
        return CONV_OK;
    }
    if (pass == 2 && h->upd_split.ok) {
        // (the plan on the fp32 instructions, then what runs in its place)
        describe_update(h, buf, buflen);
        const UpdSplitVariant &v = h->upd_split.v;
        const size_t n = strlen(buf);
        snprintf(buf + n, buflen - n, " on_bf16x3=upd_split,taps%d,%dx%d,waves_%dx%d,stage%d,positions%d,copies%d,workgroups%d", v.t, v.fc, v.fk,
                 v.wc, v.wk, v.sp, v.pi, h->upd_split.a.splits, h->upd_split.a.total);
        return CONV_OK;
    }
    if (pass == 2 && h->upd_shared.ok) {
        // (the plan without the kernel that stages for all waves, then that kernel's)
        describe_update(h, buf, buflen);
        const UpdSharedVariant &v = h->upd_shared.v;
        const size_t n = strlen(buf);
        snprintf(buf + n, buflen - n, " instead=upd_shared,taps%d,stride%d,%dx%d,waves_%dx%dx%d,stage%d,positions%d,buffers%d,copies%d,workgroups%d",
                 v.t, v.st, v.fc, v.fk, v.wc, v.wk, v.wp, v.sp, v.pi, v.nb, h->upd_shared.a.splits, h->upd_shared.a.total);
        return CONV_OK;
    }
    if (pass == 2) {
        if (!h->upd_ok) return CONV_EUNSUPPORTED;
        return describe_update(h, buf, buflen);
    }
    return CONV_EINVAL;
}

}  // extern "C"
