// fsr_plain.hip -- one-image FSR at S = 32: one workgroup of one wavefront
// per block.  Supports 8, 16 and 24 are in fsr_plain_sg.hip.
#include "fsr_block.h"

namespace fsr {

template <int kDft, int kArgmax>
__global__ __launch_bounds__(64, kDft == kDftSplitBf16 ? 4 : 2) void fsr_plain_s32(PlainLaunch p) {
    __shared__ __align__(16) float lds[kLdsFloats + (kArgmax == kArgmaxLds ? kArgmaxLdsFloats : 0)];
    const int64_t blk = xcd_runs(blockIdx.x, p.n_blocks);
    reconstruct_block<kDft, kArgmax, false>(plain_job(p, blk), p.block, p.border, p.gamma, p.tab, lds,
                                     reinterpret_cast<uint2*>(lds + kLdsFloats));
}

// One wavefront per block for the smallest images too.  Four (the routine of
// the sequential variant, fsr_block_split4.h) take a 64 x 64 frame alone from
// 47.1 to 36.2 us, but such a workgroup needs slots on all four SIMDs of a
// compute unit and 51 KiB of its LDS at one time, which another stream's large
// launch does not leave until its last blocks run, while workgroups of one
// wavefront take single slots as they come free: sent while a 1080p frame of
// 10.9 ms runs on another stream, the frame is done after 9.9 ms with four and
// after 0.28 ms with one.  Which streams overlap cannot be told from the call's
// own: the null stream too runs beside non-blocking ones.
hipError_t launch_plain(const PlainLaunch& p, hipStream_t stream) {
    if (p.n_blocks <= 0) return hipSuccess;
    const dim3 grid((unsigned)p.n_blocks), block(64);
    if (p.support != kS) return launch_plain_sg(p, stream);
    if (p.lds_argmax) {
        if (p.dft != kDftFft32) return hipErrorInvalidValue;   // rejected by the host API first
        hipLaunchKernelGGL((fsr_plain_s32<kDftFft32, kArgmaxLds>), grid, block, 0, stream, p);
    } else if (p.dft == kDftSplitBf16) {
        hipLaunchKernelGGL((fsr_plain_s32<kDftSplitBf16, kArgmaxWave>), grid, block, 0, stream, p);
    } else {
        hipLaunchKernelGGL((fsr_plain_s32<kDftFft32, kArgmaxWave>), grid, block, 0, stream, p);
    }
    return hipGetLastError();
}

}  // namespace fsr
