// Where the lanes of the split kernel (igemm_split.h) find their two chunks of a round's weights: an offset per lane that stays as it
// is, and one that all lanes share.  Plain arithmetic, for the host as well.
//
// The range check compares the lane's offset with what the shared one leaves of the tensor.  So the shared offset lies inside the
// tensor wherever a lane asks for anything, and lanes that never have a chunk carry kNoChunk, which is out of any range.
#pragma once

#ifdef __HIP__
#define CONVMI_HOST_DEVICE __host__ __device__ __forceinline__
#else
#define CONVMI_HOST_DEVICE inline
#endif

namespace convmi {

constexpr unsigned kNoChunk = 0xFFFFFFFFu;

// Weights as the kernel's launch has them, [block][tap][Kp][4], a round is one tap of blocks cb .. cb + 3: the lane half h holds
// blocks cb + 2*h and the next (b = 0, 1) of row k.  (Blocks beyond the last one are beyond the tensor's end.)
static CONVMI_HOST_DEVICE unsigned weight_lane(int k, int h, int b, int Cb, int RS, int Kp)
{
    return k < Kp && 2 * h + b < Cb ? (unsigned)(2 * h + b) * (unsigned)RS * (unsigned)Kp * 16u + (unsigned)k * 16u : kNoChunk;
}
static CONVMI_HOST_DEVICE unsigned weight_shared(int cb, int tap, int RS, int Kp)
{
    return ((unsigned)cb * (unsigned)RS + (unsigned)tap) * (unsigned)Kp * 16u;
}

// As the forward pass has them, [block of rows][tap][Cb * 4 channels][4 rows]: chunk of the block `blk` of rows and channel
// cb * 4 + channel.  (Channels beyond the last one would be the next tap's: the caller leaves them out.)
static CONVMI_HOST_DEVICE unsigned weight_lane_fwd(int blk, int channel, int Cb, int taps, int Kp)
{
    return blk < Kp / 4 ? (unsigned)blk * (unsigned)taps * (unsigned)Cb * 64u + (unsigned)channel * 16u : kNoChunk;
}
static CONVMI_HOST_DEVICE unsigned weight_shared_fwd(int cb, int tap, int Cb) { return ((unsigned)tap * (unsigned)Cb + (unsigned)cb) * 64u; }

}  // namespace convmi
