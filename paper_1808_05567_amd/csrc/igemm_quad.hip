// Backward by data of a 3x3 filter under stride 2: its four residue classes (Section II-I: one
// stride-1 convolution per class of the dI position modulo the stride, with 2x2, 2x1, 1x2 and 1x1
// taps) in ONE launch.
//
// The classes are independent and write different pixels of dI.  One launch each, they drained the
// chip four times, each with a quarter of the tiles and a quarter to four ninths of the work.  Here the tiles
// of all classes are in one grid, the class with the most taps first, so that the short ones fill
// in behind it.  A workgroup finds its class from its index and runs that class's body of the
// staged kernel: 64 x 128 tiles, four waves.
//
// Bound by the operand reads from LDS in bf16 (three reads to two MFMAs), by the MFMAs in fp32.  Measured against
// one launch per class and per transform of its weights: 288 -> 384 at 35x35, N = 32, bf16 58 -> 39 us
// (fp32 202 -> 176); 64 -> 64 at 56x56, N = 8, 19 -> 8 (24 -> 15); 512 -> 512 at 14x14, N = 128, 81 -> 51
// (293 -> 233).  All classes read the forward pass's weights (FWD_WT in igemm_kernel.h), which leaves out the launch that
// transformed them: 288 -> 384 at 35x35, N = 32, bf16 40 -> 36; 42 passes at N = 2 ... 192, 0.80 of the time in bf16 (0.61 ... 1.04),
// 0.96 in fp32 (0.87 ... 1.03).
#include "igemm_kernel.h"

namespace convmi {

template <int DT, bool FWD_WT, int NPL, int R, int S, int PPT>
static __device__ __forceinline__ void quad_tile(const IgemmArgs &a, int bid, unsigned char *lds)
{
    igemm_tile<DT, 2, 2, 1, 2, NPL, R, S, PPT, 2, 0, false, FWD_WT>(a, bid, lds);
}

template <int DT, bool FWD_WT>
__global__ __launch_bounds__(256, 2) void igemm_quad_kernel(const IgemmQuadArgs q)
{
    extern __shared__ __attribute__((aligned(16))) unsigned char lds[];
    const int bid = blockIdx.x;  // (every class's grid is a multiple of 8: its XCDs stay bid mod 8)
    if (bid < q.end[0])
        quad_tile<DT, FWD_WT, 2, 2, 2, 1>(q.cls[0], bid, lds);
    else if (bid < q.end[1])
        quad_tile<DT, FWD_WT, 2, 2, 1, 1>(q.cls[1], bid - q.end[0], lds);
    else if (bid < q.end[2])
        quad_tile<DT, FWD_WT, 2, 1, 2, 1>(q.cls[2], bid - q.end[1], lds);
    else if (q.cls[3].PLS <= 128)
        quad_tile<DT, FWD_WT, 4, 1, 1, 0>(q.cls[3], bid - q.end[2], lds);
    else
        quad_tile<DT, FWD_WT, 4, 1, 1, 1>(q.cls[3], bid - q.end[2], lds);
}

hipError_t launch_igemm_quad(int dtype, const IgemmQuadArgs &q, size_t lds_bytes, hipStream_t stream)
{
    void (*const fn)(const IgemmQuadArgs) = dtype == CONV_BF16    ? igemm_quad_kernel<CONV_BF16, true>
                                            : q.cls[0].fwd_wt ? igemm_quad_kernel<CONV_F32, true>
                                                              : igemm_quad_kernel<CONV_F32, false>;
    if (hipError_t err = ensure_dynamic_lds(reinterpret_cast<const void *>(fn), lds_bytes); err != hipSuccess)
        return err;
    hipLaunchKernelGGL(fn, dim3(q.end[3]), dim3(256), lds_bytes, stream, q);
    return hipGetLastError();
}

}  // namespace convmi
