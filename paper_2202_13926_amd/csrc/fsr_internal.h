// fsr_internal.h -- declarations shared by the host runtime and the kernels.
#pragma once

#include <hip/hip_runtime.h>
#include <stdint.h>

namespace fsr {

constexpr int kS = 32;            // support edge handled by these kernels
constexpr int kBins = kS * kS;    // 1024 frequency bins per block

// Device tables for one (S, rho) pair: the spatial weight rho^dist (Eq. 5
// before masking) and the frequency weight w_f (Eq. 9), both S x S,
// row-major, float32, and the DFT operands of the support size.
struct BlockTables {
    const float* rho_pow;   // [m * S + n]
    const float* freq_w;    // [k * S + l]
    // S < 32: F[m][k] = exp(-j 2 pi m k / S), S x S float2, exactly
    // conjugate-symmetric in k
    const float2* dft_sg;
    // DFT-matrix operands of the split-bf16 matrix-core transform in MFMA
    // lane order, bf16 bit patterns [part 2][q 2][term kMfmaMaxTerms][lane 64][8]
    const uint16_t* mfma_dft;
};

constexpr int kMfmaMaxTerms = 3;
constexpr int kMfmaDftElems = 2 * 2 * kMfmaMaxTerms * 64 * 8;

// One image of a reconstruction call.
struct ImageDesc {
    const float* image;
    const uint8_t* mask;
    float* out;
    uint16_t* argmax_log;   // nullable: n_blocks x iterations
    int32_t height, width;
    int64_t stride;
    int32_t iterations;
    int32_t nbx;            // blocks per row, ceil(width / B)
    int64_t block_begin;    // first global block id of this image (batched path)
};

// Blocks per wavefront of a call (or batch) of n_blocks blocks at these
// parameters: 8 at S = 8 with B <= 4 (fsr_block_multi.h), else 1, and 1 for
// calls whose blocks all find a wavefront slot of their own: eighteen
// wavefronts on each of the 256 compute units.  Such a call is bound by the
// latency of an iteration, which is longer when each lane holds eight bins.
// Measured at I = 100, us a call with 1 and 8 blocks per wavefront: 256 blocks
// 18.7 and 35.5, 2025 21.5 and 35.7, 4096 27.7 and 36.2, 5184 34.8 and 36.5,
// 8100 41.9 and 37.1; with B = 2, 256 blocks 18.6 and 32.2, 4096 27.8 and 33.4,
// 5184 34.8 and 33.3.  Calls side by side share the slots, and near the line
// four streams at once are then better served by eight: us a call on 1 / 2 / 4
// streams of 1024 blocks 20.6 / 10.4 / 7.5 and 36.9 / 20.4 / 12.2, of 2116 24.1 /
// 14.1 / 9.0 and 37.7 / 21.0 / 13.0, of 4096 28.0 / 17.4 / 15.9 and 38.1 / 21.3 /
// 13.4.
constexpr int64_t kOnePerWaveMaxBlocks = 18 * 256;

inline int32_t blocks_per_wave(int32_t support, int32_t block, int64_t n_blocks) {
    return support == 8 && block * block <= 16 && n_blocks > kOnePerWaveMaxBlocks ? 8 : 1;
}

struct PlainLaunch {
    ImageDesc img;
    int32_t block, border;  // B, L
    int32_t support;        // S = B + 2L: 32, or 8, 16, 24 (fsr_block_sg.h)
    float gamma;
    BlockTables tab;
    int64_t n_blocks;
    int32_t dft;            // 0: FP32 FFTs, 1: split-bf16 matrix products
    int32_t lds_argmax;     // 1: argmax reduced through an LDS tree (FP32 FFTs only)
};

hipError_t launch_plain(const PlainLaunch& p, hipStream_t stream);
// The reuse variant at S = 32 (fsr_reuse.hip) over n_frames frames of p.img's
// size, frame_stride elements apart.  may_allocate: device memory may be
// taken from the stream's pool for the call (not under stream capture).
hipError_t launch_reuse(const PlainLaunch& p, float delta, int32_t n_frames, int64_t frame_stride,
                        bool may_allocate, hipStream_t stream);
int64_t reuse_steps(int32_t height, int32_t width, int32_t block, int32_t border);
hipError_t launch_plain_sg(const PlainLaunch& p, hipStream_t stream);   // S = 8, 16, 24

}  // namespace fsr
