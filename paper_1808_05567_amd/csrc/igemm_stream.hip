// bf16 3x3 convolutions of few channels over many pixels, stride 1, the result as large as the input: forward, and backward by data
// through duality.  The weights stay in registers and the pixels stream by.
//
// A workgroup is resident for the whole launch.  It owns FK*32 result channels over a contiguous range of the flat pixel list
// (n, y, x).  Each of its four waves holds all weights of those channels, 9 * CS * FK operands of 16 channels in up to 288 registers,
// and takes every fourth group of 32 pixels.  The input goes through LDS once: a ring of 16 chunks of 64 pixels, filled three
// steps of 128 pixels ahead by loads that write straight into LDS.  Since the result is as large as the input, a tap is a
// constant offset in the pixel list; lanes whose tap falls outside the image read zeros.
//
// The staged kernel (igemm_kernel.h) reads three operands from LDS for two MFMAs, brings the rows above and below each tile again
// and waits for a tile's first step; here an operand serves FK MFMAs and nothing is brought twice.
//
// What bounds it: from about 20 steps a workgroup on, memory (32 -> 32 at 147x147, N = 64, 178 MB: 40 us, 4.5 TB/s; 50 - 52 on the
// staged kernel; 32 -> 64 forward 83 -> 66, backward 83 -> 61); on fewer the weights' way into the registers, 4 us of a launch
// (64 -> 64 at 56x56, N = 8, 6.2 us, 5.4 on the staged kernel).  Three steps ahead: loads that bypass the L2 cost up to 20 %, two
// workgroups a CU 5 - 30 %.
#include <algorithm>

#include "igemm_kernel.h"

namespace convmi {

constexpr int kStreamChunks = 16, kStreamAhead = 3;  // chunks of the ring, steps that the loads run ahead
constexpr int stream_weight_bytes(int cs, int fk) { return 9 * cs * fk * 1024; }

// CS: groups of 16 channels of the input.  FW: the weights as the forward pass has them (IgemmArgs::fwd_wt).
template <int CS, int FK, bool FW>
__global__ __launch_bounds__(256, 1) void igemm_stream_kernel(const IgemmStreamArgs a)
{
    typedef Elem<CONV_BF16> E_;
    constexpr int NPL = 2 * CS;           // planes of eight channels
    constexpr int CH = NPL * 1024;        // bytes of a chunk
    constexpr int NL = 2 * NPL / 4;       // loads of a wave per step (two chunks)
    constexpr int NS = 4 * FK;            // stores
    constexpr int RING = kStreamChunks * CH;
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];

    const int tid = threadIdx.x, lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5, l32 = lane & 31;

    const int bid = blockIdx.x;
    const int lin = (bid & 7) * a.per_xcd + (bid >> 3);
    if (lin >= a.total) return;
    const int kt = lin % a.n_kt, k0 = kt * FK * 32;
    const int HW = a.H * a.W, M = a.N * HW;
    const int m_first = lin / a.n_kt * a.steps * 128;
    const int steps = min(a.steps, (M - m_first + 127) / 128);
    const int halo = (a.W + 64) / 64;  // chunks before the range's first pixel: a row and a pixel
    const float inv_HW = 1.0f / (float)HW, inv_W = 1.0f / (float)a.W;
    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);

    // the weights, into LDS behind the chunks of the first steps
    const int first_chunks = 2 * (kStreamAhead + halo);
    unsigned char *const wb = lds + first_chunks * CH;
    {
        constexpr int NW = 9 * CS * FK;  // wave-level loads
        const rsrc_t rsrc_wt = make_rsrc(a.wt, 0, (size_t)a.Cb * 9 * a.Kp * 16);
#pragma unroll
        for (int i = 0; i < (NW + 3) / 4; ++i) {
            const int at = min(4 * i + wave, NW - 1) * 64 + lane;
            unsigned off;
            if constexpr (FW) {  // [block of the result's channels][tap][channel of the input]
                const int c = at % (CS * 16), tap = at / (CS * 16) % 9, blk = at / (CS * 16) / 9;
                off = c < a.Cb * 8 && k0 / 8 + blk < a.Kp / 8 ? (unsigned)(((k0 / 8 + blk) * 9 + tap) * (a.Cb * 8) + c) * 16u : kOutOfRange;
            } else {  // [block of the input's channels][tap][channel of the result]
                const int k = at % (FK * 32), tap = at / (FK * 32) % 9, blk = at / (FK * 32) / 9;
                off = blk < a.Cb && k0 + k < a.Kp ? (unsigned)((blk * 9 + tap) * a.Kp + k0 + k) * 16u : kOutOfRange;
            }
            load_to_lds_16(rsrc_wt, off, 0u, wb + min(4 * i + wave, NW - 1) * 1024);
        }
    }
    // Chunk c of the ring: pixels m_first + 64 * (c - halo) on.  A wave takes planes of both chunks of a step.
    auto load_chunks = [&](int c) {
        unsigned off[2];
#pragma unroll
        for (int b = 0; b < 2; ++b) {
            const int m = m_first + 64 * (c + b - halo) + lane, n = fast_div(max(m, 0), inv_HW);
            off[b] = m >= 0 && m < M ? ((unsigned)n * (unsigned)(a.Cb - 1) * (unsigned)HW + (unsigned)m) * 16u : kOutOfRange;
        }
#pragma unroll
        for (int i = 0; i < NL; ++i) {
            const int u = 4 * i + wave, b = u / NPL, plane = u - b * NPL;
            load_to_lds_16(rsrc_in, plane < a.Cb ? (b ? off[1] : off[0]) : kOutOfRange, (unsigned)plane * (unsigned)HW * 16u,
                           lds + ((c + b) & (kStreamChunks - 1)) * CH + plane * 1024);
        }
    };
    for (int c = 0; c < first_chunks; c += 2) load_chunks(c);
    wait_all_memory();
    __syncthreads();

    constexpr int NACC = 60;
    u32x4 A[9][CS][FK];
#pragma unroll
    for (int t = 0; t < 9; ++t)
#pragma unroll
        for (int c = 0; c < CS; ++c)
#pragma unroll
            for (int j = 0; j < FK; ++j) {
                if constexpr (FW) {
                    // lanes 4*i + q of a group of 16 address rows 4q .. 4q + 3 of the group's 16 for channel i of four
                    const int q = lane & 3, rows = (lane >> 4) & 1, ch = 16 * c + 8 * h + ((lane >> 2) & 3);
                    typedef short s16x4 __attribute__((ext_vector_type(4)));
                    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
                    unsigned char *const p = wb + (((4 * j + 2 * rows + (q >> 1)) * 9 + 8 - t) * (CS * 16) + ch) * 16 + (q & 1) * 8;
                    const u32x2 x = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)p));
                    const u32x2 y = __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)(p + 64)));
                    A[t][c][j] = u32x4{x[0], x[1], y[0], y[1]};
                } else {
                    A[t][c][j] = *reinterpret_cast<const u32x4 *>(wb + (((2 * c + h) * 9 + t) * (FK * 32) + 32 * j + l32) * 16);
                }
                // (in accumulation registers, where an MFMA reads them as well; left to itself the compiler moves each one out first)
                if ((t * CS + c) * FK + j < NACC) asm volatile("" : "+a"(A[t][c][j]));
            }
    __syncthreads();
    // zeros behind the ring
    unsigned char *const zeros = lds + RING;
    for (int i = tid * 16; i < CH; i += 256 * 16) *reinterpret_cast<u32x4 *>(zeros + i) = u32x4{0, 0, 0, 0};
    __syncthreads();

    const size_t oplane = (size_t)HW * 16;
    const rsrc_t ro = make_rsrc(a.out, 0, (size_t)a.N * a.out_kb * oplane);
    const int lane_at = h * 1024;
    struct Place {
        int m, n, x, y, p0;  // the lane's pixel; ring position of tap (0, 0)
    };
    auto place = [&](int st) {
        Place c;
        c.m = m_first + st * 128 + wave * 32 + l32;
        c.n = fast_div(c.m, inv_HW);
        const int pix = c.m - c.n * HW;
        c.y = fast_div(pix, inv_W);
        c.x = pix - mul24(c.y, a.W);
        c.p0 = 64 * halo + st * 128 + wave * 32 + l32 - a.W - 1;
        return c;
    };
    auto read_tap = [&](const Place &c, int t, u32x4(&b)[CS]) {
        const int r = t / 3, q = t % 3;
        const bool in = (r == 0 ? c.y > 0 : r == 2 ? c.y + 1 < a.H : true) && (q == 0 ? c.x > 0 : q == 2 ? c.x + 1 < a.W : true);
        const unsigned p = (unsigned)(c.p0 + r * a.W + q);
        const unsigned at = (p >> 6 & (kStreamChunks - 1)) * CH + (p & 63) * 16;
        const unsigned char *const from = lds + ((t == 4 || in) ? at : RING) + lane_at;
#pragma unroll
        for (int i = 0; i < CS; ++i) b[i] = *reinterpret_cast<const u32x4 *>(from + i * 2048);
    };
    auto store = [&](const Place &c, const f32x16(&v)[FK], int i) {
        const int j = i >> 2, q = i & 3, row = k0 + 32 * j + 8 * q;
        const unsigned at = c.m < M ? ((unsigned)c.n * (unsigned)(a.out_kb - 1) * (unsigned)HW + (unsigned)c.m) * 16u + (unsigned)h * 8u : kOutOfRange;
        E_::template store4<CONVMI_OUT_POLICY>(ro, row < a.Kp ? at : kOutOfRange, (unsigned)(row / 8) * (unsigned)oplane, v[j][4 * q], v[j][4 * q + 1],
                                               v[j][4 * q + 2], v[j][4 * q + 3]);
    };

    // One wave to a SIMD: what is not an MFMA stands between them.  A step's results are stored while the next one multiplies, and
    // its first tap is read while the step before ends.
    u32x4 B[2][CS];
    f32x16 acc[2][FK];
    Place at[2];
    at[0] = place(0);
    read_tap(at[0], 0, B[0]);
    auto step = [&](auto pc, int st) {
        constexpr int P = decltype(pc)::value;  // st mod 2
        static_for<0, 9>([&](auto tc) {
            constexpr int t = decltype(tc)::value;
            __builtin_amdgcn_sched_barrier(0);
            // (the next tap is read while this one multiplies)
            if constexpr (t + 1 < 9) read_tap(at[P], t + 1, B[(P + t + 1) & 1]);
            if constexpr (t < NS) {
                if (st > 0) store(at[1 - P], acc[1 - P], t);
            }
            if constexpr (t == 8) {
                // The next step's chunks have landed (later ones may be on their way, and results), and all waves are done with the step
                // before this one, whose chunks the new ones replace.
                at[1 - P] = place(st + 1);
                __builtin_amdgcn_sched_barrier(0);
                asm volatile("s_waitcnt vmcnt(%0)" ::"n"((kStreamAhead - 1) * NS + (kStreamAhead - 2) * NL) : "memory");
                __builtin_amdgcn_s_barrier();
                asm volatile("" ::: "memory");
                __builtin_amdgcn_sched_barrier(0);
                read_tap(at[1 - P], 0, B[(P + 9) & 1]);
                load_chunks(2 * (st + kStreamAhead + halo));
            }
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int c = 0; c < CS; ++c)
#pragma unroll
                for (int j = 0; j < FK; ++j) {
                    if constexpr (t == 0) {
                        if (c == 0) acc[P][j] = f32x16{};
                    }
                    E_::template mma<8>(A[t][c][j], B[(P + t) & 1][c], acc[P][j]);
                }
        });
    };
    int st = 0;
    for (; st + 2 <= steps; st += 2) {
        step(std::integral_constant<int, 0>{}, st);
        step(std::integral_constant<int, 1>{}, st + 1);
    }
    if (st < steps) {
        step(std::integral_constant<int, 0>{}, st);
#pragma unroll
        for (int i = 0; i < NS; ++i) store(at[0], acc[0], i);
    } else {
#pragma unroll
        for (int i = 0; i < NS; ++i) store(at[1], acc[1], i);
    }
    wait_all_memory();  // (the last steps' loads still write into the ring)
}

typedef void (*stream_fn_t)(const IgemmStreamArgs);
static stream_fn_t find(int cs, int fk, bool fw)
{
#define STREAM_ENTRY(CS, FK) \
    if (cs == CS && fk == FK) return fw ? igemm_stream_kernel<CS, FK, true> : igemm_stream_kernel<CS, FK, false>
    STREAM_ENTRY(2, 1);
    STREAM_ENTRY(2, 2);
    STREAM_ENTRY(3, 1);
    STREAM_ENTRY(3, 2);
    STREAM_ENTRY(4, 1);
    STREAM_ENTRY(4, 2);
    return nullptr;
}
bool igemm_stream_exists(int cs, int fk) { return find(cs, fk, false) != nullptr; }

size_t igemm_stream_lds_bytes(const IgemmStreamPlan &p)
{
    const size_t chunk = (size_t)p.cs * 2048;
    return std::max((kStreamChunks + 1) * chunk, 2 * (kStreamAhead + ((size_t)p.a.W + 64) / 64) * chunk + stream_weight_bytes(p.cs, p.fk));
}
// Rows that the ring holds beside the steps that are on their way.
int igemm_stream_widest() { return 64 * ((kStreamChunks - 2 * kStreamAhead - 2) / 2) - 1; }

hipError_t launch_igemm_stream(const IgemmStreamPlan &p, const IgemmStreamArgs &a, hipStream_t stream)
{
    const stream_fn_t fn = find(p.cs, p.fk, a.fwd_wt != 0);
    if (!fn) return hipErrorInvalidDeviceFunction;
    const size_t lds = igemm_stream_lds_bytes(p);
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(fn), lds); err != hipSuccess) return err;
    hipLaunchKernelGGL(fn, dim3(8 * a.per_xcd), dim3(256), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
