// fp32 operands as sums of three bf16 numbers, for products of fp32 tensors on the bf16 matrix instructions.
//
// (The decomposition: G. Henry, P. T. P. Tang and A. Heinecke, "Leveraging the bfloat16 Artificial Intelligence Datatype For
// Higher-Precision Computations", ARITH 2019.)  x = h + m + l: h is x rounded to 8 significant bits, m is x - h rounded to 8, l what is
// left, at most 6 bits, so the sum is exact; |m| <= 2^-8 and |l| <= 2^-17 of the power of two below |x|.  Of the nine products of
// two such numbers six are formed, h*h, h*m, m*h, m*m, h*l, l*h.  The other three are together at most 2^-24 (1 + 2^-9) of the
// product, what rounding it to fp32 may cost, and zero where the product has 24 bits or fewer (m is zero up to 8 bits of an operand, l up to 16).
// Six bf16 MFMAs of 16 reduction indices take 192 clocks where fp32 ones take 512.  An fp32 MFMA rounds the sum once per product, a bf16
// one once per 16 (at most), and the five small products go into a sum of their own.
// Measured against 64 bits, one chain of n products, uniform * normal values, error of the fp32 MFMAs / of this: n = 16 7.4e-8 / 3.1e-8,
// 256 2.9e-7 / 8.6e-8, 4608 1.2e-6 / 4.1e-7, 36864 3.5e-6 / 1.2e-6 (all six in one sum: 3.3e-8, 2.3e-7, 1.1e-6, 3.2e-6).  Sums whose
// products all leave out the same (constant tensors), n = 4 3.2e-8 / 2.4e-8, 16 1.0e-7 / 3.5e-8, 256 2.4e-7 / 3.5e-8; sums of a single
// product other than zero 2.47e-8 / 2.51e-8, at most 1.0 / 1.42 times 2^-24 (mantissas just above one, which leave out the most:
// 3.40e-8 / 3.57e-8).  (m cut off instead of rounded: 2.7e-8, at most 2.25.  m*l and l*m formed too: 2.47e-8, and 28 images 3x3 128 ->
// 128 at 28x28 123 -> 145 us, 256 of 512 -> 1024 1x1 stride 2 at 28x28 1 010 -> 1 156.)
//
// What three bf16 numbers do not hold: infinities (x - h is NaN), values that round to infinity, and the last bits of values
// below 2^-109.  All of the first two make a sum infinite or NaN.  So do the last: a wave that finds bits which no l holds makes l NaN
// in operands that it converts for others, and its sums at the end where the operands are its own.  A wave with such sums forms its own
// again on the fp32 instructions.  (The look at the operands takes four to six of
// 50 instructions for eight values: 28 images 3x3 128 -> 128 at 28x28 123.5 -> 126 us, 256 of 512 -> 1024 1x1 stride 2 1 027 -> 1 055.
// A guard on the results alone misses operands of 2^-120 that meet 2^50, 1e-4 off.)  Tiny sums need none: the instructions keep denormal
// products and sums.  576 products an output, error of the fp32 MFMAs / of this: sums of 2^-124 2.1e-7 / 1.8e-7, of 2^-132 5.2e-5 / 3.2e-5.
#pragma once
#include "igemm_exchange.h"

namespace convmi {

struct Bf16x3 {
    u32x4 h, m, l;  // eight numbers
};

// Eight numbers, in eight pieces of five or six instructions that stand between MFMAs: pieces 2*p and 2*p + 1 make pair p, the
// first of it in the lower half of h, m, l.  `rest` carries x - h from one to the other.  `lost` collects the bits that no l holds, in
// its lower half.  SHARED: the last piece makes the last pair's l NaN if the eight have any (one pair: whoever multiplies it
// forms all its sums again).
constexpr int kSplitPieces = 8;
template <int I, bool SHARED>
static __device__ __forceinline__ void split_piece(const u32x4 (&raw)[2], Bf16x3 &s, float (&rest)[2], unsigned &lost)
{
    constexpr int p = I / 2;
    if constexpr (I % 2 == 0) {
        const float a = __uint_as_float(raw[p / 2][p % 2 * 2]), b = __uint_as_float(raw[p / 2][p % 2 * 2 + 1]);
        unsigned h = pack_bf16x2(a, b);
        asm volatile("" : "+v"(h));  // (else the halves are rounded again one by one)
        rest[0] = a - __uint_as_float(h << 16);
        rest[1] = b - __uint_as_float(h & 0xFFFF0000u);
        asm volatile("" : "+v"(rest[0]), "+v"(rest[1]));  // (here, not where it is used)
        s.h[p] = h;
    } else {
        unsigned m = pack_bf16x2(rest[0], rest[1]);
        asm volatile("" : "+v"(m));
        const unsigned la = __float_as_uint(rest[0] - __uint_as_float(m << 16)), lb = __float_as_uint(rest[1] - __uint_as_float(m & 0xFFFF0000u));
        unsigned l = __builtin_amdgcn_perm(lb, la, 0x07060302);
        lost = SHARED && p == 0 ? la | lb : lost | la | lb;
        if constexpr (SHARED && p == 3) l = (unsigned short)lost != 0 ? 0x7FC07FC0u : l;
        asm volatile("" : "+v"(l), "+v"(lost));
        s.m[p] = m;
        s.l[p] = l;
    }
}
template <bool SHARED>
static __device__ __forceinline__ Bf16x3 split8(const u32x4 (&raw)[2], unsigned &lost)
{
    Bf16x3 s;
    float rest[2];
    static_for<0, kSplitPieces>([&](auto i) { split_piece<decltype(i)::value, SHARED>(raw, s, rest, lost); });
    return s;
}
static __device__ __forceinline__ void mma_bf16(const u32x4 &a, const u32x4 &b, f32x16 &c)
{
    c = __builtin_amdgcn_mfma_f32_32x32x16_bf16(__builtin_bit_cast(bf16x8, a), __builtin_bit_cast(bf16x8, b), c, 0, 0, 0);
}
// big += h*h, small += the five others: product I of the six
constexpr int kSplitProducts = 6;
template <int I>
static __device__ __forceinline__ void mma_split(const Bf16x3 &a, const Bf16x3 &b, f32x16 &big, f32x16 &small)
{
    if constexpr (I == 0) mma_bf16(a.l, b.h, small);
    if constexpr (I == 1) mma_bf16(a.h, b.h, big);
    if constexpr (I == 2) mma_bf16(a.h, b.l, small);
    if constexpr (I == 3) mma_bf16(a.m, b.m, small);
    if constexpr (I == 4) mma_bf16(a.m, b.h, small);
    if constexpr (I == 5) mma_bf16(a.h, b.m, small);
}

// The weights of a backward pass as the forward pass has them, [channel block of dI][tap][channel of dO][4]: 32 channels of dI by
// 16 of dO are 128 chunks of 4 channels of dI, lane's chunk i (of two) in channel block 4*i + wt_block(lane) and channel
// wt_channel(lane) of dO.  Converted, they go to a wave's own 3 KiB of LDS, from where transposing reads bring each lane
// eight channels of dO of its own channel of dI.
constexpr int kWtBytes = 3072;
static __device__ __forceinline__ int wt_block(int lane) { return (lane >> 2) & 3; }
static __device__ __forceinline__ int wt_channel(int lane) { return (lane >> 4) * 4 + (lane & 3); }
static __device__ __forceinline__ void put_weights(unsigned char *area, int lane, const Bf16x3 &s)
{
    unsigned char *const at = area + (wt_channel(lane) * 8 + wt_block(lane)) * 8;
    *reinterpret_cast<u32x2 *>(at) = u32x2{s.h[0], s.h[1]};
    *reinterpret_cast<u32x2 *>(at + 32) = u32x2{s.h[2], s.h[3]};
    *reinterpret_cast<u32x2 *>(at + 1024) = u32x2{s.m[0], s.m[1]};
    *reinterpret_cast<u32x2 *>(at + 1056) = u32x2{s.m[2], s.m[3]};
    *reinterpret_cast<u32x2 *>(at + 2048) = u32x2{s.l[0], s.l[1]};
    *reinterpret_cast<u32x2 *>(at + 2080) = u32x2{s.l[2], s.l[3]};
}
// Four of the eight channels of dO of piece P (h, m, l), the first or second half.
template <int P, int HALF>
static __device__ __forceinline__ u32x2 get_weights(const unsigned char *area, int lane)
{
    typedef short s16x4 __attribute__((ext_vector_type(4)));
    typedef __attribute__((address_space(3))) s16x4 *lds_s16x4;
    // lanes 4*j + q of a group of 16 address 4 channels of dI, block q of the group's four, of channel j of dO
    const int q = lane & 3, rows = (lane >> 4) & 1, h = lane >> 5;
    const unsigned char *const at = area + P * 1024 + ((8 * h + 4 * HALF + ((lane & 15) >> 2)) * 8 + 4 * rows + q) * 8;
    return __builtin_bit_cast(u32x2, __builtin_amdgcn_ds_read_tr16_b64_v4i16((lds_s16x4)const_cast<unsigned char *>(at)));
}

static __device__ __forceinline__ Bf16x3 get_weights(const unsigned char *area, int lane)
{
    const u32x2 h0 = get_weights<0, 0>(area, lane), h1 = get_weights<0, 1>(area, lane), m0 = get_weights<1, 0>(area, lane),
                m1 = get_weights<1, 1>(area, lane), l0 = get_weights<2, 0>(area, lane), l1 = get_weights<2, 1>(area, lane);
    return Bf16x3{u32x4{h0[0], h0[1], h1[0], h1[1]}, u32x4{m0[0], m0[1], m1[0], m1[1]}, u32x4{l0[0], l0[1], l1[0], l1[1]}};
}

// Largest magnitude, NaN if one is.
static __device__ __forceinline__ float max_magnitude(float t, const f32x16 &v)
{
#pragma unroll
    for (int i = 0; i < 16; i += 2)
        t = __builtin_elementwise_maximum(__builtin_elementwise_maximum(t, __builtin_fabsf(v[i])), __builtin_fabsf(v[i + 1]));
    return t;
}
// Whether a wave whose lanes' largest results are t forms them again: one is infinite or NaN.
static __device__ __forceinline__ bool sums_need_fp32(float t) { return __any(!(t < __builtin_inff())) != 0; }
// The sums of a wave that lost bits of its own operands are NaN from here on.
template <int N>
static __device__ __forceinline__ void mark_if_lost(unsigned lost, f32x16 (&sums)[N])
{
    if (__builtin_expect(__any((unsigned short)lost != 0) != 0, 0))
#pragma unroll
        for (int j = 0; j < N; ++j) sums[j][0] = __builtin_nanf("");
}

// Barrier of the workgroup behind which the waves' LDS operations are done; loads into registers stay in flight.
static __device__ __forceinline__ void lds_barrier()
{
    asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");
    __builtin_amdgcn_s_barrier();
    asm volatile("" ::: "memory");
}

}  // namespace convmi
