// Degree-pair buckets and tile shapes, shared by the pipeline and the small-graph path (device code).
#pragma once

#include "common.h"
#include "internal.h"
#include "isect.h"
#include "mlp.h"

namespace tcx {

__device__ __forceinline__ uint32_t bucket_of(uint32_t din, uint32_t dout) {
    if (din == 0 || dout == 0) return BUCKET_NONE;
    const uint32_t li = min(14, floor_log2(din));
    const uint32_t lo = min(15, floor_log2(dout));
    return 16u * li + lo;
}

// A block's statistics per bucket, added to the control block at the end.
struct BucketSums {
    uint32_t nv[NBUCKET];
    unsigned long long in[NBUCKET], out[NBUCKET], work[NBUCKET], win[NBUCKET];
    __device__ void clear(int threads) {
        for (int b = threadIdx.x; b < NBUCKET; b += threads) {
            nv[b] = 0;
            in[b] = out[b] = work[b] = win[b] = 0;
        }
    }
    // One middle vertex; lo, hi: the first and last rank of its list (read only when it has work).
    __device__ void add(uint32_t din, uint32_t dout, uint32_t lo, uint32_t hi) {
        const uint32_t b = bucket_of(din, dout);
        if (b == (uint32_t)BUCKET_NONE) return;
        atomicAdd(&nv[b], 1u);
        atomicAdd(&in[b], (unsigned long long)din);
        atomicAdd(&out[b], (unsigned long long)dout);
        atomicAdd(&work[b], (unsigned long long)din * dout);
        // windows the bitmap strategy walks for this middle list (first one
        // aligned down to a word)
        atomicAdd(&win[b], (unsigned long long)(((hi - (lo & ~31u)) >> BM_WINDOW_LOG2) + 1u));
    }
    __device__ void flush(Ctrl* ctrl, int threads) {
        for (int b = threadIdx.x; b < NBUCKET; b += threads) {
            if (!nv[b]) continue;
            atomicAdd(&ctrl->bucket_nv[b], nv[b]);
            atomicAdd((unsigned long long*)&ctrl->bucket_in[b], in[b]);
            atomicAdd((unsigned long long*)&ctrl->bucket_out[b], out[b]);
            atomicAdd((unsigned long long*)&ctrl->bucket_work[b], work[b]);
            atomicAdd((unsigned long long*)&ctrl->bucket_win[b], win[b]);
        }
    }
};

// Bucket features (6 floats): the bucket's two degree classes and the log
// sizes of its work, from the statistics gathered by the pipeline: the
// LDS-bitmap windows its middle lists span (the bitmap strategy's set-up
// count, which grows with the rank range a list covers and so with the
// graph's size), in-edges, out-neighbours, and in-edges x out-degree.
__device__ __forceinline__ void bucket_features(const Ctrl* ctrl, int b, float (&f)[MLP_IN]) {
    f[0] = (float)(b >> 4) / 14.f;
    f[1] = (float)(b & 15) / 15.f;
    f[2] = log2f(1.f + (float)ctrl->bucket_win[b]) / 32.f;
    f[3] = log2f(1.f + (float)ctrl->bucket_in[b]) / 32.f;
    f[4] = log2f(1.f + (float)ctrl->bucket_out[b]) / 32.f;
    f[5] = log2f(1.f + (float)ctrl->bucket_work[b]) / 48.f;
}

// Vertices per multi-vertex tile for bucket b (1 = chunks of single vertices).
__device__ __forceinline__ uint32_t tile_group(const Ctrl* ctrl, uint32_t b) {
    const uint32_t li = b >> 4;
    if (li >= 14) return 1u;
    const uint32_t maxin = 2u << li;   // in-degrees of the bucket are below this
    const uint32_t K = ctrl->chunk[b];
    if (2u * maxin > K) return 1u;
    const uint32_t g = K / maxin;
    // the edge-centric kernels stage the tile's lists in LDS when they fit:
    // no more vertices than STAGE_MAX list elements at the bucket's longest
    const uint32_t lo = b & 15u;
    const uint32_t stage_cap = lo >= 12 ? 1u : (uint32_t)STAGE_MAX / (2u << lo);
    const uint32_t cap = ctrl->choice[b] == KER_BITMAP ? (uint32_t)SEG_MAX_BITMAP
                                                       : (stage_cap < (uint32_t)SEG_MAX ? stage_cap : (uint32_t)SEG_MAX);
    return g > cap ? cap : (g > 1u ? g : 1u);
}

}  // namespace tcx
