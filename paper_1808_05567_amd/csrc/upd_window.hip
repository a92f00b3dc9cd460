// Weight-gradient update in bf16 of large 3x3 layers with stride 2: the ring kernel (upd_ring.hip: small blocks of dW, one
// filter row per workgroup, the waves split the pixels, no barrier in the main loop) with ONE window of the
// input for all taps of the filter row.
//
// The ring kernel loads 1 KiB per stage for every tap, and with a stride of two a run of four pixels is two lines, of which
// every tap uses half: a 2 x 2 block asks for 14 units of the load path's 64 B/clk per 12 MFMAs.  Here a wave walks
// a run of consecutive pixel slots; each chunk of 16 slots brings 32 input positions of every channel block,
// whole lines, and 16 pixels of dO into the wave's ring (6 units), and a tap is an offset into the ring: the
// transposing LDS reads take any position.  A chunk's window ends in the next chunk, so a stage waits for
// one chunk more than it multiplies.
//
// Slots: the output rows one after the other, each Lp slots long, Lp = Q or as many as the input columns that
// the row reads need (slots past Q are dead: dO arrives as zero there).  Slot c of a row stands at the
// row's input position stride * c; tap s reads position stride * c + s - pad_w, which lies in the
// same row wherever its column is inside the image.  Lanes whose tap falls outside the image, and those of
// dead slots, read from a patch of zeros instead: outside the image the input counts as zero, whatever
// the neighbouring row holds (it may be infinite).
//
// The pixels of a read lie two positions apart and would use half of the LDS banks: the positions of every other
// quad are stored with neighbours swapped.
//
// What bounds it now: vector instructions, 138 a stage (addresses of the next chunk and of the taps) next to 12 MFMAs, 45 of
// the 85 thousand clocks that a CU is busy; MFMAs 29.  288 -> 384 at 35x35, no padding, N = 37 / 70: 50 -> 47 /
// 87 -> 79 us with the reduce launch, 512 -> 512 at 14x14, N = 61: 33 -> 28.  (The same kernel for stride 1 and for 5 and
// 7 columns was built and measured: the lines at window_applies.)
#include <algorithm>

#include "igemm_kernel.h"

namespace convmi {

// The one form that is built: S taps of a filter row, stride ST, FC x FK accumulator tiles per tap, NW waves, a ring
// of NS chunks each, one chain of sums per wave.
constexpr int S = 3, ST = 2, FC = 2, FK = 2, NW = 8, NS = 3;

__global__ __launch_bounds__(NW * 64, 2) void upd_window_kernel(const UpdArgs a)
{
    constexpr int V = 8, NB = 4;              // channels of a block, blocks of a fragment
    constexpr int AHEAD = 4;                  // a chunk's positions start that many before its first slot's
    constexpr int NF = S * FC * FK;           // accumulator tiles
    constexpr int NO = ST * FC + FK;          // loads per chunk
    constexpr int G = NW / 4;                 // tiles summed per round (a thread per chunk)
    constexpr int CH = ST * 1024;             // bytes of a chunk, per input fragment
    constexpr int RING = NS * CH;             // ... of its ring
    constexpr int OUT0 = FC * RING;           // the dO rings follow
    constexpr int WAVE = OUT0 + FK * NS * 1024;
    static_assert(NS >= 3, "two chunks are read, one is on its way");

    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    f32x4 *const xch = reinterpret_cast<f32x4 *>(lds);

    const int tid = threadIdx.x;
    const int lane = tid & 63;
    const int wave = __builtin_amdgcn_readfirstlane(tid >> 6);
    const int h = lane >> 5;
    const int l32 = lane & 31;

    // (the patch of zeros behind the rings: as long as a fragment's rings, since the same offsets are added)
    unsigned char *const zeros = lds + NW * WAVE;
    for (int i = tid * 16; i < FC * RING; i += NW * 64 * 16) *reinterpret_cast<u32x4 *>(zeros + i) = u32x4{0, 0, 0, 0};

    // split slowest: the blocks of a range of slots run side by side and share its lines in the L2
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

    const int PQ = a.P * a.Q, HW = a.H * a.W, Lp = a.Qpitch;
    const int rows = a.N * a.P, slots = rows * Lp;
    const float inv_Lp = 1.0f / (float)Lp, inv_P = 1.0f / (float)a.P;
    // this wave's run of slots, a whole number of stages
    const int share = a.rows_per_split / NW;
    const int t0 = split * a.rows_per_split + wave * share;
    const int steps = (min(slots - t0, share) + 15) / 16;

    const rsrc_t rsrc_in = make_rsrc(a.in, 0, (size_t)a.N * a.Cb * HW * 16);
    const rsrc_t rsrc_out = make_rsrc(a.dout, 0, (size_t)a.N * a.Kb * PQ * 16);
    // Lane -> (quad of 4 positions, channel block, position of the quad), in the order of the LDS.
    const int lquad = lane >> 4, lblk = (lane >> 2) % NB, lpx = lane & 3;
    const unsigned in_ch = (unsigned)(c0 / V + lblk) * (unsigned)HW * 16u;  // channel part of the lane's offsets
    const unsigned out_ch = (unsigned)(k0 / V + lblk) * (unsigned)PQ * 16u;  // (fragment i: 4 i blocks on)
    const int in_blocks = a.Cb - c0 / V, out_blocks = a.Kb - k0 / V;

    unsigned char *const ring = lds + wave * WAVE;
    int tl = t0;  // first slot of the next chunk to load
    auto load = [&](int slot) {
        // input: position ST * tl - AHEAD + (the lane's) of the row list
#pragma unroll
        for (int l = 0; l < ST; ++l) {
            const int quad = 4 * l + lquad;
            const int off = 4 * quad + (lpx ^ (quad & 1)) - AHEAD;
            // (counted from a row before the first: the dividend is not negative)
            const int t = tl + (off >> 1) + Lp;  // slot, and which of its two positions
            const int row1 = fast_div(t, inv_Lp);
            const int row = row1 - 1;
            const int x = ST * (t - mul24(row1, Lp)) + (off & 1);
            const int n = fast_div(max(row, 0), inv_P);
            const int y = ST * (row - mul24(n, a.P)) + r - a.pad;
            const bool in = (unsigned)row < (unsigned)rows && (unsigned)y < (unsigned)a.H && x < a.W;
            const unsigned pix = (unsigned)(mul24(mul24(n, a.Cb), HW) + mul24(y, a.W) + x) * 16u;
#pragma unroll
            for (int i = 0; i < FC; ++i)
                load_to_lds_16(rsrc_in, in && lblk < in_blocks - NB * i ? in_ch + pix : kOutOfRange, (unsigned)(NB * i * HW) * 16u,
                               ring + i * RING + slot * CH + l * 1024);
        }
        const int t = tl + 4 * lquad + lpx;
        const int row = fast_div(t, inv_Lp);
        const int c = t - mul24(row, Lp);
        const int n = fast_div(row, inv_P);
        const bool live = row < rows && c < a.Q;
        const unsigned pix = (unsigned)(mul24(mul24(n, a.Kb), PQ) + mul24(row - mul24(n, a.P), a.Q) + c) * 16u;
#pragma unroll
        for (int i = 0; i < FK; ++i)
            load_to_lds_16(rsrc_out, live && lblk < out_blocks - NB * i ? out_ch + pix : kOutOfRange, (unsigned)(NB * i * PQ) * 16u,
                           ring + OUT0 + i * (NS * 1024) + slot * 1024);
        tl += 16;
    };

    f32x16 acc[NF];
#pragma unroll
    for (int f = 0; f < NF; ++f)
#pragma unroll
        for (int t = 0; t < 16; ++t) acc[f][t] = 0.0f;

    // Operand reads, transposing: lanes 4*j + q of a group of 16 address 4 channels of slot j and receive
    // slots 0..3 of their own channel; two reads (i) make the 8 slots of a lane half.
    const int q4 = lane & 3, j4 = (lane >> 2) & 3;
    const int part = (2 * ((lane >> 4) & 1) + (q4 >> 1)) * 64 + (q4 & 1) * 8;  // channel block and half
    const unsigned ring_addr = lds_address(ring);
    const unsigned zero_addr = lds_address(zeros) + (unsigned)part;
    const unsigned out_addr = ring_addr + (unsigned)(OUT0 + 2 * h * 256 + j4 * 16 + part);
    // window address of tap s (first read; the second is ST quads on), and whether it lies in the next chunk
    // (bit 2 s + read): in the ring's last chunk those lanes start over
    unsigned in_addr[S], wraps = 0;
#pragma unroll
    for (int s = 0; s < S; ++s) {
        const int p = ST * (8 * h + j4) + s - a.pad_w + AHEAD;
        const int quad = p >> 2;
        in_addr[s] = ring_addr + (unsigned)(quad * 256 + ((p & 3) ^ (quad & 1)) * 16 + part);
        wraps |= (quad >= 4 * ST ? 1u : 0u) << (2 * s) | (quad + ST >= 4 * ST ? 2u : 0u) << (2 * s);
    }
    // Column of the lane's two slots, and its window's first column; a tap outside [0, W) reads zeros.
    const int inc = 16 % Lp;
    int col[2];
#pragma unroll
    for (int i = 0; i < 2; ++i) {
        const int t = t0 + 8 * h + 4 * i + j4;
        col[i] = t - mul24(fast_div(t, inv_Lp), Lp);
    }

    if (steps > 0) {
#pragma unroll
        for (int d = 0; d < NS; ++d) load(d);
    }
    __syncthreads();  // (the zeros are written)
    auto stage = [&](auto dc) {
        constexpr int d = decltype(dc)::value;
        // this chunk's loads and the next one's have landed; the NS - 2 later ones may be on their way
        __builtin_amdgcn_sched_barrier(0);
        asm volatile("s_waitcnt vmcnt(%0)" ::"n"((NS - 2) * NO) : "memory");
        __builtin_amdgcn_sched_barrier(0);
        lds_u32x2 to[2 * FK], ti[2][2 * FC];
        static_for<0, FK>([&](auto ic) {
            constexpr int i = decltype(ic)::value;
            to[2 * i] = lds_read_tr16_b64_untracked<i * (NS * 1024) + d * 1024>(out_addr);
            to[2 * i + 1] = lds_read_tr16_b64_untracked<i * (NS * 1024) + d * 1024 + 256>(out_addr);
        });
        int x0[2];
#pragma unroll
        for (int i = 0; i < 2; ++i) {
            x0[i] = col[i] < a.Q ? ST * col[i] - a.pad_w : -0x10000;
            col[i] = min((unsigned)(col[i] + inc), (unsigned)(col[i] + inc - Lp));
        }
        auto read_tap = [&](auto sc) {
            constexpr int s = decltype(sc)::value;
            unsigned ad[2];
#pragma unroll
            for (int i = 0; i < 2; ++i) {
                const unsigned at = d == NS - 1 ? in_addr[s] - (wraps >> (2 * s + i) & 1) * (unsigned)RING : in_addr[s];
                ad[i] = (unsigned)(x0[i] + s) < (unsigned)a.W ? at : zero_addr;
            }
            static_for<0, FC>([&](auto ic) {
                constexpr int i = decltype(ic)::value;
                ti[s & 1][2 * i] = lds_read_tr16_b64_untracked<i * RING + d * CH>(ad[0]);
                ti[s & 1][2 * i + 1] = lds_read_tr16_b64_untracked<i * RING + d * CH + ST * 256>(ad[1]);
            });
        };
        auto operand = [&](const lds_u32x2 &x, const lds_u32x2 &y) {
            const u32x4 v = {x[0], x[1], y[0], y[1]};
            return __builtin_bit_cast(bf16x8, v);
        };
        // (the next tap's reads are on their way while a tap's MFMAs issue)
        read_tap(std::integral_constant<int, 0>{});
        static_for<0, S>([&](auto sc) {
            constexpr int s = decltype(sc)::value;
            if constexpr (s + 1 < S) read_tap(std::integral_constant<int, s + 1>{});
            __builtin_amdgcn_sched_barrier(0);
            lds_reads_pending<(s + 1 < S ? 2 * FC : 0)>();
            if (s == 0) {
#pragma unroll
                for (int o = 0; o < 2 * FK; ++o) lds_read_landed(to[o]);
            }
#pragma unroll
            for (int o = 0; o < 2 * FC; ++o) lds_read_landed(ti[s & 1][o]);
            __builtin_amdgcn_sched_barrier(0);
            if constexpr (s == S - 1) load(d);  // (the chunk has been read: the one NS further on takes its place)
#pragma unroll
            for (int i = 0; i < FC; ++i)
#pragma unroll
                for (int j = 0; j < FK; ++j)
                    acc[(s * FC + i) * FK + j] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(
                        operand(ti[s & 1][2 * i], ti[s & 1][2 * i + 1]), operand(to[2 * j], to[2 * j + 1]),
                        acc[(s * FC + i) * FK + j], 0, 0, 0);
        });
    };
    int u = 0;
    for (; u + NS <= steps; u += NS) static_for<0, NS>(stage);
    // (the last stages of the run)
    static_for<0, NS - 1>([&](auto dc) {
        if (u + decltype(dc)::value < steps) stage(dc);
    });
    wait_all_memory();  // (the last chunks' loads still write into the ring)

    // The waves' sums, G tiles per round, pairwise.  Rows of a tile are input channels: a
    // chunk of four consecutive ones is 16 bytes of dW.
    const int RS = a.R * S;
    float *const dst = a.partial + (size_t)split * ((size_t)a.Cb * RS * a.Kp * V);
#pragma unroll
    for (int f0 = 0; f0 < NF; f0 += G) {
        __syncthreads();  // (the rings, or the last round, are done with)
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

bool upd_window_exists(int s, int stride, int fc, int fk, int nw, int depth, int sum)
{
    return s == S && stride == ST && fc == FC && fk == FK && nw == NW && depth == NS && sum == 0;
}

size_t upd_window_lds_bytes()
{
    // (the exchange holds NW/4 tiles of every wave)
    return std::max((size_t)NW / 4 * NW * 4096, ((size_t)NW * (ST * FC + FK) + ST * FC) * NS * 1024);
}

hipError_t launch_upd_window(const UpdArgs &a, int grid, hipStream_t stream)
{
    const size_t lds = upd_window_lds_bytes();
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(upd_window_kernel), lds); err != hipSuccess)
        return err;
    hipLaunchKernelGGL(upd_window_kernel, dim3(grid), dim3(NW * 64), lds, stream, a);
    return hipGetLastError();
}

}  // namespace convmi
