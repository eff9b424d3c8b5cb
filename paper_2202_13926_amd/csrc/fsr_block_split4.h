// fsr_block_split4.h -- one S = 32 support block of the sequential variant
// (the original FSR that Sec. II departs from) on a workgroup of four
// wavefronts.  Its blocks depend on one another, so that at one time there
// are too few to fill the device, and a call is bound by the latency of a
// block, i.e. by the chain of its iterations.
//
// Wavefront q keeps the bins of slots NS q .. NS q + NS - 1 (bins (2s + h, c),
// NS = 4) in registers and a copy of R_w in LDS; W lies in LDS with every row
// repeated (one offset per iteration; residency does not matter here).  Per
// iteration each lane puts its largest key (the same keys and tie codes
// 15 - s as in fsr_block.h) into LDS, and behind one workgroup barrier (keys
// and R_w are double-buffered, so one suffices) every wavefront reduces all
// four wavefronts' keys itself: over the wavefronts per lane, then over the
// lanes.  That is one cross-lane reduction on the chain; reducing per
// wavefront first and then over the four candidates has two.  R_w at the
// winner is read with the W rows, in the same LDS wait.  The set-up is spread
// over the wavefronts too: each gathers four of the sixteen row pairs, all
// loads at once, and takes one radix-4 column of the FFT passes.
//
// Every value is computed by the same operations in the same order as in
// fsr_block.h (kDftFft32), so the result is bitwise that of the
// one-wavefront routine.
//
// Measured with a launch of 256 independent blocks at I = 100: 36.2 us against
// 47.1 with one wavefront per block (270 against 385 ns an iteration).  What is
// left of an iteration is mostly three LDS round trips (keys out, keys in, W
// and R_w) and the six steps of the reduction; a lone wavefront also pays some
// 4.5 cycles for every instruction, scalar ones included, and waits out each
// result that the next instruction needs.  Hence the iterations in pairs
// (constant buffers), the addresses taken from the bin index, and the
// objective step by step over the slots with the model's twiddle from a table
// in LDS: these two took that launch from 40.5 to 36.2 us, and the VGA frame of
// the sequential variant from 30.0 to 26.5 ms.  Before them, with a two-stage
// reduction 43.8 us instead of 42.2, with eight wavefronts per block 44.5.
// Keys by lane (one 16-byte read each) 37.3.  A step of the sequential variant
// at VGA, I = 0: 4.1 us against 6.4 with one wavefront per block.
#pragma once

#include "fsr_block.h"
#include "fsr_block_sg.h"

namespace fsr {

constexpr int kSplitWaves = 4;
constexpr int kSplitSlots = kSlots / kSplitWaves;   // slots per wavefront

// Steps of at most this many blocks, two per compute unit, take this routine.
// Measured at I = 100, us a launch of 256 / 272 / 512 / 528 / 768 / 1024
// independent blocks: here 36.3 / 40.6 / 41.2 / 47.7 / 48.0 / 73.7, one
// wavefront per block 47.1 / 47.5 / 47.9 / 47.9 / 47.7 / 48.0 (a third
// workgroup on a compute unit costs what the latency saves: every wavefront
// repeats the reduction).  1080p frames (at most 96 blocks per step and frame)
// in one launch per step, ms a call of 1 / 4 / 5 / 6 / 8 frames: four
// wavefronts for every step 66.0 / 71.7 / 72.5 / 79.4 / 81.8, one 87.0 / 91.3 /
// 92.1 / 92.5 / 90.2, four up to this line 66.0 / 71.7 / 72.5 / 83.4 / 83.3.
constexpr int64_t kSplitMaxBlocks = 512;

// LDS of a workgroup: the W table with its rows repeated (row r at r and
// r + 32); the transpose planes, before them the gathered tile; the exchange
// area of the FFT passes; two buffers of R_w by slot and of the lanes' keys;
// flags.
struct SplitLds {
    float2 w[2 * kS * kS];
    union {
        float planes[2 * kS * Planes::kPitch];
        float2 tile[kSlots * 64];   // (f~, w) of slot s, lane
    };
    float2 ex[16 * 64];
    float2 tw[kS];   // exp(-j 2 pi i / 32), read by the model
    float2 r[2][kBins];
    uint32_t key[2][kSplitWaves][64];
    int known[kSplitWaves];
};

// One 32-point DFT pass of dft32_lane_pair on four wavefronts: z[j] of
// wavefront q holds slot q + 4 j on entry (element s = 4 j + q of the lane's
// sequence) and output k' = q + 4 j on return (bin k' + 16 h of the pass).
// The radix-4 x 4 transform's first stage takes the column s2 = q, its second
// the row k1 = q; the 16 values meet in ex in between.
__device__ __forceinline__ void split_dft32_pass(float (&re)[4], float (&im)[4], float2* ex, int q, int lane) {
    const int h = lane >> 5;
    dft4_slots(re, im);
    if (q != 0) {
#pragma unroll
        for (int k1 = 1; k1 < 4; ++k1) cmul(re[k1], im[k1], kTw.re[(2 * k1 * q) & 31], kTw.im[(2 * k1 * q) & 31]);
    }
#pragma unroll
    for (int k1 = 0; k1 < 4; ++k1) ex[(4 * k1 + q) * 64 + lane] = make_float2(re[k1], im[k1]);
    __syncthreads();
#pragma unroll
    for (int s2 = 0; s2 < 4; ++s2) {
        const float2 v = ex[(4 * q + s2) * 64 + lane];
        re[s2] = v.x;
        im[s2] = v.y;
    }
    dft4_slots(re, im);
    const float sgn = h ? -1.0f : 1.0f;
#pragma unroll
    for (int k2 = 0; k2 < 4; ++k2) {
        const int k = q + 4 * k2;
        float er, ei, orr, oi;
        split_halves(re[k2], er, orr);
        split_halves(im[k2], ei, oi);
        cmul(orr, oi, kTw.re[k], kTw.im[k]);
        re[k2] = fmaf(sgn, orr, er);
        im[k2] = fmaf(sgn, oi, ei);
    }
}

// Outputs are stored, and reused pixels loaded, by agent-scope accesses
// (another workgroup of the same launch may read, or have written, them).
__device__ __forceinline__ void reconstruct_block_split(const BlockJob& jb, int B, int L, float gamma,
                                                        const BlockTables& tab, SplitLds& sh) {
    constexpr int NS = kSplitSlots;
    const int lane = (int)(threadIdx.x & 63);
    const int q = __builtin_amdgcn_readfirstlane((int)(threadIdx.x >> 6));   // wavefront of the block
    const int c = lane & 31, h = lane >> 5;
    const int ti = lane_div(lane, B), tj = lane - ti * B;
    const int tm = L + ti, tn = L + tj;

    // ---- gather and weighting, pixel (m, n) = (2s + h, c) of slots
    // 4q .. 4q + 3; all loads go out together (an address that holds nothing
    // of use reads pixel 0)
    // the target pixel of the lane: written at the end, loaded here
    const int ty = jb.by * B + ti, tx = jb.bx * B + tj;
    const bool writes = q == 0 && lane < B * B && ty < jb.height && tx < jb.width;
    const int64_t toff = writes ? (int64_t)ty * jb.stride + tx : 0;
    const uint8_t tknown = jb.mask[toff];
    const float tvalue = jb.image[toff];
    {
        const int y0 = jb.by * B - L, x0 = jb.bx * B - L;
        const int x = x0 + c;
        const bool xin = (unsigned)x < (unsigned)jb.width;
        uint8_t kraw[NS];
        float fraw[NS], rp[NS], old[NS];
        bool in[NS], earlier[NS];
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const int m = 2 * (NS * q + j) + h, y = y0 + m;
            in[j] = xin && (unsigned)y < (unsigned)jb.height;
            const int64_t off = in[j] ? (int64_t)y * jb.stride + x : 0;
            kraw[j] = jb.mask[off];
            fraw[j] = jb.image[off];
            rp[j] = global_ptr(tab.rho_pow)[m * kS + c];
            earlier[j] = in[j] && (m < L || (m < L + B && c < L));
            old[j] = __hip_atomic_load(jb.out + (earlier[j] ? off : 0), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
        }
        uint64_t any = 0;
#pragma unroll
        for (int j = 0; j < NS; ++j) {
            const uint8_t k = in[j] ? kraw[j] : (uint8_t)0;
            const bool reused = earlier[j] && !k && jb.delta > 0.0f;
            const float f = k ? fraw[j] : reused ? old[j] : 0.0f;
            const float w = k ? rp[j] : reused ? jb.delta * rp[j] : 0.0f;
            any |= ballot(k != 0 || reused);
            sh.tile[(NS * q + j) * 64 + lane] = make_float2(f, w);
        }
        if (lane == 0) sh.known[q] = any != 0;
    }
    __syncthreads();
    const bool any_known = (sh.known[0] | sh.known[1] | sh.known[2] | sh.known[3]) != 0;

    float acc = 0.0f;
    const int iters = jb.iterations;
    if (any_known) {
        // ---- R_w = mu W + DFT2((f~ - mu) w) and W, both real tiles in one
        // complex FFT, as in fsr_block.h; every wavefront forms the sums and
        // the scale itself
        float zr[4], zi[4], mu, scale, xmax;
        {
            float xr[16], wr[16];
            float sx = 0.0f, sw = 0.0f;
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                const float2 v = sh.tile[64 * s + lane];
                xr[s] = v.x;
                wr[s] = v.y;
            }
#pragma unroll
            for (int s = 0; s < 16; ++s) {
                sx = fmaf(xr[s], wr[s], sx);
                sw += wr[s];
            }
            sx = wave_sum_f32(sx);
            sw = wave_sum_f32(sw);
            mu = sw > 0.0f ? sx / sw : 0.0f;
#pragma unroll
            for (int s = 0; s < 16; ++s) xr[s] = (xr[s] - mu) * wr[s];
            xmax = max_abs_and_scale(xr, scale);
        }
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const float2 v = sh.tile[64 * (q + 4 * j) + lane];
            zr[j] = (v.x - mu) * v.y;
            zi[j] = v.y * scale;
        }
        float* pr = Planes::re(sh.planes);
        float* pi = Planes::im(sh.planes);
        split_dft32_pass(zr, zi, sh.ex, q, lane);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pr[Planes::idx(q + 4 * j + 16 * h, c)] = zr[j];
            pi[Planes::idx(q + 4 * j + 16 * h, c)] = zi[j];
        }
        __syncthreads();
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            zr[j] = pr[Planes::idx(c, 2 * (q + 4 * j) + h)];
            zi[j] = pi[Planes::idx(c, 2 * (q + 4 * j) + h)];
        }
        split_dft32_pass(zr, zi, sh.ex, q, lane);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            pr[Planes::idx(c, q + 4 * j + 16 * h)] = zr[j];
            pi[Planes::idx(c, q + 4 * j + 16 * h)] = zi[j];
        }
        __syncthreads();
        // ---- the two spectra of this wavefront's slots; W into the table
        float vr[NS], vi[NS], wf[NS];
        const float half_inv_s = 0.5f / scale;
#pragma unroll
        for (int s = 0; s < NS; ++s) {
            const int k = 2 * (NS * q + s) + h, km = (kS - k) & 31, lm = (kS - c) & 31;
            const float ar = pr[Planes::idx(k, c)], ai = pi[Planes::idx(k, c)];
            const float br = pr[Planes::idx(km, lm)], bi = pi[Planes::idx(km, lm)];
            const float xr = xmax == 0.0f ? 0.0f : 0.5f * (ar + br);
            const float xi = xmax == 0.0f ? 0.0f : 0.5f * (ai - bi);
            const float wr = (ai + bi) * half_inv_s, wi = (br - ar) * half_inv_s;
            vr[s] = fmaf(mu, wr, xr);
            vi[s] = fmaf(mu, wi, xi);
            wf[s] = global_ptr(tab.freq_w)[k * kS + c];
            sh.w[k * kS + c] = make_float2(wr, wi);
            sh.w[(k + kS) * kS + c] = make_float2(wr, wi);
        }
        if (q == 0 && h == 0) sh.tw[c] = make_float2(kTw.re[c], kTw.im[c]);
        const int tmn8 = opaque((8 * tm) | ((8 * tn) << 16));
        // byte offset of the lane's entry (h, c) in W, plus this wavefront's
        // first slot (512 bytes per slot): the low byte stays 8 c
        const int hc8 = opaque(256 * h + 8 * c + 512 * NS * q);
        const uint32_t code0 = 15u - (uint32_t)(NS * q);
        __syncthreads();
        const float w00 = sh.w[0].x;
        const float gi = w00 > 0.0f ? gamma / w00 : 0.0f;

        // R_w of this wavefront's slots, for the wavefronts that need the winner's
#pragma unroll
        for (int s = 0; s < NS; ++s) sh.r[0][64 * (NS * q + s) + lane] = make_float2(vr[s], vi[s]);

        // one iteration on buffer kBuf; returns the bin
        const auto iterate = [&](auto buffer) {
            constexpr int kBuf = decltype(buffer)::value;
            // this wavefront's largest key of each lane (Eq. 16, the same keys
            // as the one-wavefront routine)
            // -- step by step over the slots, so that no instruction waits
            // for the one before it
            float e[NS];
            uint32_t lmax = 0;
#pragma unroll
            for (int s = 0; s < NS; ++s) e[s] = vi[s] * vi[s];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < NS; ++s) e[s] = fmaf(vr[s], vr[s], e[s]);
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < NS; ++s) e[s] *= wf[s];
            __builtin_amdgcn_sched_barrier(0);
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                const uint32_t key = (__float_as_uint(e[s]) & 0xFFFFFFF0u) | (code0 - (uint32_t)s);
                lmax = umax(lmax, key);
            }
            sh.key[kBuf][q][lane] = lmax;
            __syncthreads();
            // every wavefront reduces all keys: over the wavefronts, then the
            // lanes; equal keys go to the lower lane
#pragma unroll
            for (int w = 0; w < kSplitWaves; ++w) lmax = umax(lmax, sh.key[kBuf][w][lane]);
            const uint32_t mx = wave_max_u32(lmax);
            const int ln = (int)__builtin_ctzll(ballot(lmax == mx));
            const int idx = 64 * (15 - (int)(mx & 15u)) + ln;   // 32 u + v
            // A lone wavefront pays for every scalar instruction too, so the
            // addresses come from 8 idx = 256 u + 8 v and the phase from idx
            // itself (32 u n vanishes mod 32)
            const int idx8 = 8 * idx;
            const float2 rw = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(sh.r[kBuf]) + idx8);
            // residual (Eqs. 12, 14-15) on this wavefront's slots, as in
            // fsr_block.h.  The reads go out first; the model's lane exchange
            // is used after the update
            const int woff = sub_low_byte(hc8 + 8192 - (idx8 & ~255), idx8);
            const float2* wrow = reinterpret_cast<const float2*>(reinterpret_cast<const char*>(sh.w) + woff);
            float2 w[NS];
#pragma unroll
            for (int s = 0; s < NS; ++s) w[s] = wrow[64 * s];
            __builtin_amdgcn_sched_barrier(0);
            // model: g += gamma p exp(+j 2 pi (u m + v n) / S) on the target;
            // every wavefront computes it (no branch in the loop's chain),
            // wavefront 0's is the one written
            const int q8 = dot2_u16((idx >> 5) | (idx << 16), tmn8) & (8 * kS - 8);
            const float2 tw = *reinterpret_cast<const float2*>(reinterpret_cast<const char*>(sh.tw) + q8);
            const float cr = gi * rw.x, ci = gi * rw.y;    // gamma * p (Eqs. 10-11)
#pragma unroll
            for (int s = 0; s < NS; ++s) {
                vr[s] = fmaf(-cr, w[s].x, vr[s]);
                vr[s] = fmaf(ci, w[s].y, vr[s]);
                vi[s] = fmaf(-cr, w[s].y, vi[s]);
                vi[s] = fmaf(-ci, w[s].x, vi[s]);
                sh.r[kBuf ^ 1][64 * (NS * q + s) + lane] = make_float2(vr[s], vi[s]);
            }
            __builtin_amdgcn_sched_barrier(0);
            acc = fmaf(cr, tw.x, acc);
            acc = fmaf(ci, tw.y, acc);
            return idx;
        };
        constexpr std::integral_constant<int, 0> first{};
        constexpr std::integral_constant<int, 1> second{};
        // pairs of iterations, in two copies, with and without the log
        const auto run = [&](auto with_log) {
            const auto logged = [&](int it, int idx) {
                if constexpr (decltype(with_log)::value) {
                    if (q == 0 && lane == 0) jb.log[it] = (uint16_t)idx;
                }
            };
            int it = 0;
            for (; it + 1 < iters; it += 2) {
                logged(it, iterate(first));
                logged(it + 1, iterate(second));
            }
            if (it < iters) logged(it, iterate(first));
        };
        if (jb.log != nullptr) run(std::true_type{});
        else run(std::false_type{});
    } else if (q == 0 && jb.log != nullptr) {
        for (int it = lane; it < iters; it += 64) jb.log[it] = (uint16_t)0xFFFF;
    }

    // ---- compose (Sec. II): known pixels copied, unknown pixels Re g
    if (writes)
        __hip_atomic_store(jb.out + toff, tknown ? tvalue : acc, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
}

}  // namespace fsr
