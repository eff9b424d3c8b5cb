// fsr_reuse.hip -- the sequential variant that reuses reconstructed pixels
// (the original FSR that Sec. II departs from), at S = 32.
//
// The variant is defined by raster order: block (by, bx) sees the
// reconstructions of every earlier block whose target meets its support.
// With r = ceil(L / B) those are the blocks of rows by - r .. by - 1 and
// columns bx - r .. bx + r, and those of row by and columns bx - r .. bx - 1.
// Giving block (by, bx) the step t = bx + (r + 1) by puts every such block
// at a smaller step, and two blocks of one step lie at least r + 1 block
// columns apart, so that neither's target meets the other's support.  One
// launch per step (a wavefront schedule) therefore gives exactly the raster
// result, with the stream's order between launches as the only
// synchronisation.  Frames of one size are independent: one launch per step
// takes that step's blocks of every frame.
#include <algorithm>

#include "fsr_block.h"
#include "fsr_block_split4.h"

namespace fsr {

// Blocks (by, step - slope * by) for by = by_lo + blockIdx.x of frame
// blockIdx.y; the host sizes the grid so that every bx lies in [0, nbx).
// Frame f's image, mask and output start f * frame_stride elements after
// frame 0's, its argmax log (if any) f * log_stride entries after.
__global__ __launch_bounds__(64, 4) void fsr_reuse_s32(PlainLaunch p, float delta, int32_t step,
                                                    int32_t by_lo, int32_t slope, int64_t frame_stride,
                                                    int64_t log_stride) {
    __shared__ __align__(16) float lds[kLdsFloats];
    const int by = by_lo + (int)blockIdx.x;
    const int bx = step - slope * by;
    const int64_t f = blockIdx.y;
    BlockJob jb = plain_job(p, (int64_t)by * p.img.nbx + bx);
    jb.image += f * frame_stride;
    jb.mask += f * frame_stride;
    jb.out += f * frame_stride;
    if (jb.log != nullptr) jb.log += f * log_stride;
    jb.delta = delta;
    reconstruct_block<kDftFft32, kArgmaxWave, false, true>(jb, p.block, p.border, p.gamma, p.tab, lds);
}

// The same blocks with four wavefronts each, for steps of at most
// kSplitMaxBlocks blocks over all frames; bitwise the same result.
__global__ __launch_bounds__(64 * kSplitWaves) void fsr_reuse_split4_s32(PlainLaunch p, float delta, int32_t step,
                                                            int32_t by_lo, int32_t slope, int64_t frame_stride,
                                                            int64_t log_stride) {
    __shared__ __align__(16) SplitLds sh;
    const int by = by_lo + (int)blockIdx.x;
    const int bx = step - slope * by;
    const int64_t f = blockIdx.y;
    BlockJob jb = plain_job(p, (int64_t)by * p.img.nbx + bx);
    jb.image += f * frame_stride;
    jb.mask += f * frame_stride;
    jb.out += f * frame_stride;
    if (jb.log != nullptr) jb.log += f * log_stride;
    jb.delta = delta;
    reconstruct_block_split(jb, p.block, p.border, p.gamma, p.tab, sh);
}

// ---- All blocks in one launch: a workgroup takes a block row of a frame and
// reconstructs its blocks one after another, each as soon as the row above
// has finished the blocks it reuses (r + 1 block columns ahead), which it
// reads from a progress counter per row.  Compared with one launch per step
// there is no gap between a block and the next, and a row waits for the row
// above alone, not for every block of a step.
//
// Order and progress.  Rows are handed out by a ticket counter in the order
// (block row, frame), so the row a workgroup waits for was always taken by a
// workgroup that is already running: row 0 waits for nobody, and by induction
// every wait ends, however few workgroups are resident.  Waiting for row
// by - 1 at column bx + r covers the rows further up: they were that far when
// row by - 1 reconstructed there.
//
// Visibility.  Outputs are written and reused pixels read by agent-scope
// accesses (fsr_block_split4.h), which go through the caches to the point
// where all compute units meet.  Wavefront 0 waits for its stores before it
// stores the row's counter, and a workgroup loads reused pixels only after a
// barrier behind the counter's load; within the workgroup the barrier at the
// head of each block orders wavefront 0's stores before the others' loads.
// So no cache has to be written back or invalidated per block: with release
// and acquire fences instead, a block's set-up and hand-over took 4.8 us
// instead of 4.1 (they also drop the image and the tables from the caches).
struct RowQueue {
    int32_t ticket;
    int32_t pad[63];   // the counters on lines of their own
};

__global__ __launch_bounds__(256) void fsr_reuse_rows_reset(int32_t* words, int32_t n) {
    const int i = blockIdx.x * 256 + threadIdx.x;
    if (i < n) words[i] = 0;
}

__global__ __launch_bounds__(64 * kSplitWaves) void fsr_reuse_rows_s32(PlainLaunch p, float delta, int32_t n_frames,
                                                                       int32_t nby, int32_t ahead,
                                                                       int64_t frame_stride, int64_t log_stride,
                                                                       RowQueue* queue) {
    __shared__ __align__(16) SplitLds sh;
    __shared__ int32_t from_first;   // a value of thread 0 for the workgroup
    const int32_t nbx = p.img.nbx, rows = nby * n_frames;
    int32_t* progress = reinterpret_cast<int32_t*>(queue + 1);   // by frame and block row
    for (;;) {
        __syncthreads();   // from_first has been read
        if (threadIdx.x == 0) from_first = atomicAdd(&queue->ticket, 1);
        __syncthreads();
        const int32_t t = __builtin_amdgcn_readfirstlane(from_first);
        if (t >= rows) return;
        const int32_t by = t / n_frames, f = t - by * n_frames;
        int32_t* mine = progress + (int64_t)f * nby + by;
        int32_t seen = by > 0 ? 0 : nbx;   // blocks of the row above known to be finished
        for (int32_t bx = 0; bx < nbx; ++bx) {
            const int32_t need = bx + ahead < nbx ? bx + ahead : nbx;
            if (seen < need) {
                __syncthreads();   // from_first has been read
                if (threadIdx.x == 0) {
                    int32_t v;
                    while ((v = __hip_atomic_load(mine - 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT)) < need)
                        __builtin_amdgcn_s_sleep(4);
                    from_first = v;
                }
                __syncthreads();
                seen = __builtin_amdgcn_readfirstlane(from_first);
            } else {
                __syncthreads();   // the previous block's outputs, before this one's loads
            }
            BlockJob jb = plain_job(p, (int64_t)by * nbx + bx);
            jb.image += f * frame_stride;
            jb.mask += f * frame_stride;
            jb.out += f * frame_stride;
            if (jb.log != nullptr) jb.log += f * log_stride;
            jb.delta = delta;
            reconstruct_block_split(jb, p.block, p.border, p.gamma, p.tab, sh);
            if (threadIdx.x < 64) {
                asm volatile("s_waitcnt vmcnt(0)" ::: "memory");   // the outputs have arrived
                if (threadIdx.x == 0) __hip_atomic_store(mine, bx + 1, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            }
        }
    }
}

// Rows of a call that the queue takes (4 MiB of counters).
constexpr int64_t kMaxQueueRows = int64_t(1) << 20;

// Calls of fewer steps than this go out as one launch per step: the queue's
// counters, their reset and the second launch take some 20 us before the first
// block.  us a call at I = 0 / 25 / 100, one launch per step and rows: 1 block
// 20.4 / 28.0 / 51.5 and 41 / 43.3 / 62.1, a row of 4 33.5 / 64.3 / 157.9 and
// 44.5 / 73.8 / 165.5, of 6 42.4 / 88.5 / 228.8 and 48.9 / 95.9 / 233.3, of 8
// 74.7 / 116.9 / 303.0 and 55.5 / 115.5 / 301.7.
constexpr int64_t kMinRowSteps = 8;

// At most `widest` rows can make progress at one time; a workgroup that ends
// its row takes the next.  So the grid holds that many: a workgroup per row
// would hold LDS and wavefront slots for rows that cannot start yet, on every
// compute unit where a call has many frames, and keep other streams' kernels
// out.  us a call with a workgroup per row and with `widest`: 12 frames of
// 352 x 288, I = 50, 9158 and 8737; 32 of 320 x 240, I = 20, 4404 and 4259
// (one row per frame more: 8742 and 4528).
//
// hipErrorOutOfMemory when the counters cannot be allocated (nothing is
// enqueued then).
static hipError_t launch_reuse_rows(const PlainLaunch& p, float delta, int32_t n_frames, int32_t nby, int32_t ahead,
                                    int32_t widest, int64_t frame_stride, int64_t log_stride, hipStream_t stream) {
    const int32_t rows = nby * n_frames;
    const int32_t words = (int32_t)(sizeof(RowQueue) / sizeof(int32_t)) + rows;
    void* ws = nullptr;
    if (hipMallocAsync(&ws, (size_t)words * sizeof(int32_t), stream) != hipSuccess) {
        (void)hipGetLastError();   // handled: the caller launches per step
        return hipErrorOutOfMemory;
    }
    hipLaunchKernelGGL(fsr_reuse_rows_reset, dim3((words + 255) / 256), dim3(256), 0, stream,
                       static_cast<int32_t*>(ws), words);
    hipError_t e = hipGetLastError();
    if (e == hipSuccess) {
        const int32_t groups = std::min(rows, widest);
        hipLaunchKernelGGL(fsr_reuse_rows_s32, dim3(groups), dim3(64 * kSplitWaves), 0, stream, p, delta, n_frames, nby,
                           ahead, frame_stride, log_stride, static_cast<RowQueue*>(ws));
        e = hipGetLastError();
    }
    const hipError_t freed = hipFreeAsync(ws, stream);
    return e != hipSuccess ? e : freed;
}

int64_t reuse_steps(int32_t height, int32_t width, int32_t block, int32_t border) {
    const int64_t nby = (height + block - 1) / block, nbx = (width + block - 1) / block;
    const int64_t slope = (border + block - 1) / block + 1;
    return (nbx - 1) + slope * (nby - 1) + 1;
}

hipError_t launch_reuse(const PlainLaunch& p, float delta, int32_t n_frames, int64_t frame_stride,
                        bool may_allocate, hipStream_t stream) {
    const int32_t B = p.block;
    const int64_t nbx = p.img.nbx, nby = (p.img.height + B - 1) / B;
    const int64_t slope = (p.border + B - 1) / B + 1;
    const int64_t steps = reuse_steps(p.img.height, p.img.width, B, p.border);
    const int64_t log_stride = p.n_blocks * (int64_t)p.img.iterations;
    const int64_t widest = std::min(nby, (nbx + slope - 1) / slope) * n_frames;
    const int64_t launches = std::min(steps, nbx * nby);   // steps that hold a block
    if (may_allocate && launches >= kMinRowSteps && widest <= kSplitMaxBlocks && nby * n_frames <= kMaxQueueRows) {
        const hipError_t e = launch_reuse_rows(p, delta, n_frames, (int32_t)nby, (int32_t)slope,
                                               (int32_t)widest, frame_stride, log_stride, stream);
        if (e != hipErrorOutOfMemory) return e;
    }
    for (int64_t t = 0; t < steps; ++t) {
        // by in [ceil((t - (nbx - 1)) / slope), floor(t / slope)] within [0, nby)
        const int64_t over = t - (nbx - 1);
        const int64_t lo = over > 0 ? (over + slope - 1) / slope : 0;
        const int64_t hi = std::min<int64_t>(nby - 1, t / slope);
        if (hi < lo) continue;   // no block at this step (possible when slope > nbx)
        const dim3 grid((unsigned)(hi - lo + 1), (unsigned)n_frames);
        if ((hi - lo + 1) * (int64_t)n_frames <= kSplitMaxBlocks)
            hipLaunchKernelGGL(fsr_reuse_split4_s32, grid, dim3(64 * kSplitWaves), 0, stream, p, delta, (int32_t)t,
                               (int32_t)lo, (int32_t)slope, frame_stride, log_stride);
        else
            hipLaunchKernelGGL(fsr_reuse_s32, grid, dim3(64), 0, stream, p, delta, (int32_t)t, (int32_t)lo,
                               (int32_t)slope, frame_stride, log_stride);
        const hipError_t e = hipGetLastError();
        if (e != hipSuccess) return e;
    }
    return hipSuccess;
}

}  // namespace fsr
