// The counting pipeline on one stream: edge-list generation and filtering,
// CSR construction, degree-pair bucketing, kernel selection and intersection.
//
// Stages (Algorithm 2; Section 4.2 for the filter, the induced subgraph and
// dynamic grouping):
//   degree    validate ids, count input pairs per vertex (self-loops dropped)
//   rank      sort vertices by (degree, id): rank = position
//   orient    each pair as (rank lo, rank hi); loops / bad ids -> sentinel
//   sort      radix sort of the oriented pairs -> rows contiguous, ascending
//   csr       drop repeats and sentinels, emit col/src, row offsets
//   csc       in-edges (u -> v) with a non-empty tail of row u, grouped by v
//             (stable radix sort on v), in-offsets from the group boundaries
//             (the other formulations instead group all in-edges and build the
//             symmetric adjacency beside the filtered CSR)
//   bucket    per middle vertex v: (in-edges with work, |N+(v)|) -> bucket
//   select    choose the intersection strategy and tile shape per bucket
//   group     order vertices by (strategy, bucket); emit tiles (and, for counts of large
//             graphs, the hub kernels' tile ranges and 16-bit columns)
//   isect     the three intersection kernels, each over its tile range
//   finish    map per-vertex / per-edge outputs back to original ids
// Compaction and grouping go through sorts and scans. Where many threads add to one
// address (degrees of hubs, bucket statistics, per-vertex counts of the top ranks), a block
// adds in LDS and once to memory at its end. All of these are integer sums, so the
// outputs do not depend on the order. The
// kernels that write the keys of a sort also take the per-tile digit counts of
// its first pass (one read of the keys less per sort).
#include <math.h>
#include <string.h>

#include "common.h"
#include "internal.h"
#include "isect.h"
#include "mlp.h"
#include "pipeline.h"

#include <algorithm>
#include "tiles.h"

namespace tcx {

constexpr int NT = 256;

static unsigned grid_for(size_t n, unsigned cap = 16384) {
    size_t g = (n + NT - 1) / NT;
    if (g < 1) g = 1;
    if (g > cap) g = cap;
    return (unsigned)g;
}

// Blocks for a kernel whose own work is `blocks` blocks and which also clears a word per vertex: one for
// each 8192 vertices at least, as a few pairs may come with many vertices (with one block, three
// pairs on 2^24 vertices took 4.2 ms in all, now 0.96).
static unsigned clearing_grid(unsigned blocks, int32_t n, unsigned cap) {
    const unsigned clear = ((unsigned)n + 8191u) / 8192u;
    return std::min(std::max(blocks, clear), cap);
}

// ------------------------------------------------------------------ degree
// Input degree = loop-free valid pairs per vertex. Device-wide atomics would
// serialise on hub vertices, so the 2E endpoints are first partitioned by
// their high bits (one radix pass for ids of up to 25 bits, two up to 27), and
// each bucket of 2^bw vertices is then counted in an LDS histogram of up to
// 2^15 counters (128 KB); a wider bucket is counted in parts, each block
// reading the whole bucket and counting the ids of its own part. Endpoints
// of loops and invalid pairs are written as `sentinel`; with sentinel = n - 1
// each block also records how many it wrote, and they are taken off vertex
// n - 1 at the end. Wider ids fall back to a full sort of the endpoints
// (sentinel n, which sorts last) and run boundaries.
constexpr int DEG_MAX_BW = 14;        // buckets of 2^14 vertices beyond 25-bit ids (two passes)
constexpr int DEG_MAX_CW = 15;        // LDS histogram of at most 2^15 counters (128 KB)
constexpr int DEG_MAX_BUCKET_BITS = 13;   // up to 8192 buckets (ids below 2^27)
constexpr unsigned DEG_EP_BLOCKS = 1024;

// FOLD: the orientation's digits are the upper bits of the endpoint sort's, so its counts
// are sums of those of the first and of the second ids, counted apart: two LDS
// adds per pair instead of four (a batch of 148 million pairs 1.42 -> 0.79 ms; R-MAT 24,
// whose ids spread over the counters, 0.72 ms either way).
// The pairs counted as sentinels are corrected one by one.
template <int D, bool FOLD>
__global__ __launch_bounds__(NT) void k_endpoints(const int2* __restrict__ edges, uint64_t E, int32_t n,
                                                  uint32_t sentinel, uint32_t* __restrict__ keys, Ctrl* ctrl,
                                                  uint32_t* __restrict__ nsent, uint32_t* __restrict__ counts,
                                                  uint32_t ntiles, uint32_t tile_keys, RadixDigit dg,
                                                  uint32_t* __restrict__ pcounts, uint32_t pf, RadixDigit pdg,
                                                  uint32_t* __restrict__ p2tot, uint32_t* __restrict__ deg) {
    // deg: zeroed on the way, for the counts to come (null: a sort counts)
    // tile t = endpoints [t * tile_keys, (t + 1) * tile_keys) = pairs [t * EPT, (t + 1) * EPT),
    // in rounds of NT * PER pairs; with counts set, the first digit of the endpoint sort is
    // counted per tile. With pcounts set, the digit pdg of the first id is counted too, per
    // tile of pf endpoint tiles: the first pass of the orientation's pair partition, whose
    // tiles hold pf * EPT pairs. With p2tot set, the same digit of the second id is counted
    // over all pairs (added into p2tot[256]): the digit totals of that partition's second
    // pass, which then takes its offsets by look-back.
    static_assert(NT == 256, "a thread per digit of the orientation's pass");
    constexpr uint32_t PER = 4;
    const uint32_t EPT = tile_keys / 2;
    const uint32_t pntiles = (ntiles + pf - 1) / pf;
    __shared__ uint32_t red[NT / WAVE];
    __shared__ TileCountsT<D> tc;
    __shared__ TileCountsT<FOLD ? D : 256> tp;   // FOLD: of the second ids
    __shared__ TileCountsT<FOLD ? 1 : 256> tq;
    __shared__ uint32_t s_p[FOLD ? 256 : 1], s_q[FOLD ? 256 : 1];
    tc.clear();
    if (FOLD || pcounts) tp.clear();
    if (!FOLD && p2tot) tq.clear();
    if (FOLD) s_p[threadIdx.x] = s_q[threadIdx.x] = 0;
    const int up = FOLD ? pdg.shift - dg.shift : 0;
    __syncthreads();
    if (deg)
        for (int64_t v = (int64_t)blockIdx.x * NT + threadIdx.x; v < n; v += (int64_t)gridDim.x * NT) deg[v] = 0;
    bool bad = false;
    uint32_t sent = 0;
    for (uint32_t pt = blockIdx.x; pt < pntiles; pt += gridDim.x) {
     for (uint32_t tile = pt * pf; tile < (pt + 1) * pf && tile < ntiles; ++tile) {
      for (uint32_t r = 0; r < EPT; r += PER * NT) {
        int2 ed[PER];
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint64_t i = (uint64_t)tile * EPT + r + k * NT + threadIdx.x;
            ed[k] = i < E ? edges[i] : make_int2(0, 0);
        }
#pragma unroll
        for (uint32_t k = 0; k < PER; ++k) {
            const uint64_t i = (uint64_t)tile * EPT + r + k * NT + threadIdx.x;
            if (i >= E) continue;
            const int2 e = ed[k];
            const bool in_range = e.x >= 0 && e.x < n && e.y >= 0 && e.y < n;
            bad |= !in_range;
            const bool ok = in_range && e.x != e.y;
            const uint32_t a = ok ? (uint32_t)e.x : sentinel, b = ok ? (uint32_t)e.y : sentinel;
            if (keys) ((uint2*)keys)[i] = make_uint2(a, b);
            sent += ok ? 0u : 2u;
            if (FOLD) {
                tc.add_shared((a >> dg.shift) & dg.mask);
                tp.add_shared((b >> dg.shift) & dg.mask);
                if (!ok) {
                    const uint32_t ds = (sentinel >> pdg.shift) & pdg.mask;
                    atomicAdd(&s_p[((uint32_t)e.x >> pdg.shift) & pdg.mask], 1u);
                    atomicSub(&s_p[ds], 1u);
                    atomicAdd(&s_q[((uint32_t)e.y >> pdg.shift) & pdg.mask], 1u);
                    atomicSub(&s_q[ds], 1u);
                }
                continue;
            }
            if (counts) {
                tc.add_shared((a >> dg.shift) & dg.mask);
                tc.add_shared((b >> dg.shift) & dg.mask);
            }
            if (pcounts) tp.add_shared(((uint32_t)e.x >> pdg.shift) & pdg.mask);
            if (p2tot) tq.add_shared(((uint32_t)e.y >> pdg.shift) & pdg.mask);
        }
      }
        if (FOLD) {
            __syncthreads();
            for (uint32_t d = threadIdx.x; d < (uint32_t)D; d += NT) {
                const uint32_t x = tc.sum(d), y = tp.sum(d);
                counts[(size_t)d * ntiles + tile] = x + y;
                if (x) atomicAdd(&s_p[d >> up], x);
                if (y) atomicAdd(&s_q[d >> up], y);
                tc.reset(d);
                tp.reset(d);
            }
            __syncthreads();
        } else if (counts) {
            tc.flush(counts, ntiles, tile);
        }
     }
        if (FOLD) {
            pcounts[(size_t)threadIdx.x * pntiles + pt] = s_p[threadIdx.x];
            s_p[threadIdx.x] = 0;
            __syncthreads();
        } else if (pcounts) {
            tp.flush(pcounts, pntiles, pt);
        }
    }
    if (p2tot) {
        __syncthreads();
        const uint32_t t = FOLD ? s_q[threadIdx.x] : tq.sum(FOLD ? 0 : threadIdx.x);
        if (t) atomicAdd(&p2tot[threadIdx.x], t);
    }
    if (__ballot(bad) && lane_id() == 0) atomicOr(&ctrl->err, 1u);
    sent = wave_sum(sent);
    if (lane_id() == 0) red[wave_id()] = sent;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint32_t t = 0;
        for (int k = 0; k < NT / WAVE; ++k) t += red[k];
        nsent[blockIdx.x] = t;
    }
}

// tot[b] = endpoints of bucket b (ids >> bw == b), which the partition left
// ordered by bucket; for partitions of several passes (one pass leaves its digit totals).
__global__ __launch_bounds__(NT) void k_bucket_sizes(const uint32_t* __restrict__ ep, uint32_t len, int bw,
                                                     uint32_t nb, uint32_t* __restrict__ tot) {
    for (uint32_t b = blockIdx.x * NT + threadIdx.x; b < nb; b += gridDim.x * NT) {
        uint32_t at[2];
        for (uint32_t q = 0; q < 2; ++q) {   // first positions of buckets b and b + 1
            uint32_t lo = 0, hi = len;
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if ((ep[mid] >> bw) < b + q) lo = mid + 1;
                else hi = mid;
            }
            at[q] = b + q == nb ? len : lo;
        }
        tot[b] = at[1] - at[0];
    }
}

// A block counts, in LDS, the ids of part pt (ids whose bits [cw, bw) equal pt,
// cw = min(bw, CW)) among one stretch of at most `chunk` endpoints of a bucket
// b: bucket b has ceil(size / chunk) stretches, blocks take them in bucket order (blocks past
// the last one leave). tot: endpoints per bucket (null: one bucket of len_all). A bucket of one
// stretch stores its counts; the others add them to the degree array, which starts at zero. A hub makes its bucket
// several times the mean, and its adds go to one LDS counter, a lane at a time,
// so one block per bucket left the end of the kernel to that block (degree stage, one
// stretch per bucket -> these: R-MAT 20 0.31 -> 0.28 ms, Chung-Lu of 6 million pairs
// 0.35 -> 0.13 ms, of 148 million 6.15 -> 2.78 ms). Taking a wave's lanes that share
// an id as one add instead was slower everywhere but in the last. The
// 2^15-counter histogram leaves room for one block per CU, so that size runs 1024 threads.
template <typename EP, int CW, int NTB>
__global__ __launch_bounds__(NTB) void k_bucket_count(const EP* __restrict__ ep,
                                                      const uint32_t* __restrict__ tot, uint32_t len_all, int bw,
                                                      uint32_t parts, uint32_t nb, uint32_t chunk, int32_t n,
                                                      uint32_t* __restrict__ deg) {
    __shared__ uint32_t h[1u << CW];
    __shared__ uint32_t s_bucket, s_start, s_size, s_stretch, s_stretches, scratch[NTB / WAVE];
    const int cw = bw < CW ? bw : CW;
    const uint32_t nh = 1u << cw, hmask = nh - 1u, bmask = (1u << bw) - 1u;
    const uint32_t slot = blockIdx.x / parts, pt = blockIdx.x % parts;
    {   // the slot's bucket: a scan over the buckets' stretches, and over their sizes for its start
        const uint32_t per = (nb + NTB - 1u) / NTB, q0 = threadIdx.x * per;
        uint32_t cnt = 0, size = 0, total;
        for (uint32_t q = q0; q < q0 + per && q < nb; ++q) {
            const uint32_t c = tot ? tot[q] : len_all;
            cnt += stretches(c, chunk);
            size += c;
        }
        uint32_t at = block_exclusive_scan<NTB>(cnt, scratch, &total);
        uint32_t pos = block_exclusive_scan<NTB>(size, scratch);
        if (slot >= total) return;   // the same for the whole block
        if (slot >= at && slot < at + cnt)
            for (uint32_t q = q0;; ++q) {
                const uint32_t sz = tot ? tot[q] : len_all, c = stretches(sz, chunk);
                if (slot < at + c) {
                    s_bucket = q;
                    s_start = pos;
                    s_size = sz;
                    s_stretch = slot - at;
                    s_stretches = c;
                    break;
                }
                at += c;
                pos += sz;
            }
    }
    for (uint32_t j = threadIdx.x; j < nh; j += NTB) h[j] = 0;
    __syncthreads();
    const uint32_t b = s_bucket, s0 = s_start, len = s_size;
    const uint32_t a0 = s0 + (uint32_t)(((uint64_t)len * s_stretch) / s_stretches);
    const uint32_t a1 = s0 + (uint32_t)(((uint64_t)len * (s_stretch + 1u)) / s_stretches);
    // 16-byte chunks of the stretch, PER ids each, U loads in flight together
    constexpr uint32_t PER = 16 / sizeof(EP), U = 2;
    const uint32_t c1 = (a1 + PER - 1u) / PER;
    for (uint32_t c0 = a0 / PER + threadIdx.x; c0 < c1; c0 += NTB * U) {
        uint4 x[U];
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) x[k] = ((const uint4*)ep)[c0 + k * NTB < c1 ? c0 + k * NTB : c0];
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) {
            const uint32_t at = (c0 + k * NTB) * PER;
            const uint32_t w[4] = {x[k].x, x[k].y, x[k].z, x[k].w};
#pragma unroll
            for (uint32_t q = 0; q < PER; ++q) {
                const uint32_t id = sizeof(EP) == 2 ? (w[q / 2] >> (16 * (q & 1))) & 0xFFFFu : w[q % 4];
                const uint32_t loc = id & bmask;
                if (at + q >= a0 && at + q < a1 && (loc >> cw) == pt) atomicAdd(&h[loc & hmask], 1u);
            }
        }
    }
    __syncthreads();
    const uint64_t v0 = ((uint64_t)b << bw) + ((uint64_t)pt << cw);
    for (uint32_t j = threadIdx.x; j < nh; j += NTB) {
        const uint64_t v = v0 + j;
        if (v >= (uint64_t)n) break;
        if (s_stretches == 1) deg[v] = h[j];
        else if (h[j]) atomicAdd(&deg[v], h[j]);
    }
}

// Endpoints per stretch: one and a half times the mean of 256 buckets (or of the buckets, where
// they are more), so that ordinary buckets are one stretch and few buckets
// still give enough blocks; at least 8192.
template <typename EP>
static void launch_bucket_count(const EP* ep, const uint32_t* tot, int bw, uint32_t nb, uint64_t len, int32_t n,
                                uint32_t* deg, hipStream_t s) {
    const int cw = bw < DEG_MAX_CW ? bw : DEG_MAX_CW;
    const uint32_t parts = 1u << (bw - cw);
    const uint64_t want = 3 * len / (2 * (uint64_t)(nb > 256u ? nb : 256u));
    const uint32_t chunk = (uint32_t)(want > 8192 ? want : 8192);
    const dim3 grid((unsigned)(parts * (nb + len / chunk + 1)));   // at least the stretches
    auto go = [&](auto kernel, int threads) {
        hipLaunchKernelGGL(kernel, grid, dim3(threads), 0, s, ep, tot, (uint32_t)len, bw, parts, nb, chunk, n, deg);
    };
    if (cw <= 12) go(k_bucket_count<EP, 12, NT>, NT);
    else if (cw == 13) go(k_bucket_count<EP, 13, NT>, NT);
    else if (cw == 14) go(k_bucket_count<EP, 14, 1024>, 1024);   // 2^14 counters (64 KB): 8 blocks ran 2 waves per SIMD
    else go(k_bucket_count<EP, DEG_MAX_CW, 1024>, 1024);
}

// dend[v] = one past the last occurrence of v among the sorted endpoints.
__global__ __launch_bounds__(NT) void k_endpoint_bounds(const uint32_t* __restrict__ keys, uint64_t len, int32_t n,
                                                        uint32_t* __restrict__ dend) {
    for (uint64_t i = (uint64_t)blockIdx.x * NT + threadIdx.x; i < len; i += (uint64_t)gridDim.x * NT) {
        const uint32_t v = keys[i];
        if (v < (uint32_t)n && (i + 1 == len || keys[i + 1] != v)) dend[v] = (uint32_t)(i + 1);
    }
}

// Key (min(degree, RANK_CAP), id), sorted on its upper half: two passes. The
// vertices of degree RANK_CAP or more (at most 2E / RANK_CAP) share the last
// place there and are ordered by k_rank. (Sorting whole degrees took three or four
// passes, for bits that a handful of hubs have; the rank stage with two, and with the first
// digit counted here: R-MAT 20 85 -> 54 us, R-MAT 24 0.61 -> 0.43 ms.) OFFSETS: deg holds degree offsets
// [n + 1], else counts [n], where vertex n - 1 still counts the sentinel
// endpoints of nsent[0..nblocks): they are taken off here.
constexpr uint32_t RANK_CAP = 0xFFFFu;
constexpr int RANK_BITS = 16;

template <bool OFFSETS>
__device__ __forceinline__ uint32_t degree_at(const uint32_t* __restrict__ deg, uint32_t v) {
    return OFFSETS ? deg[v + 1] - deg[v] : deg[v];
}

template <bool OFFSETS, bool ALIKE>
__global__ __launch_bounds__(NT) void k_vertex_keys(uint32_t* __restrict__ deg, int32_t n,
                                                    const uint32_t* __restrict__ nsent, uint32_t nblocks,
                                                    uint64_t* __restrict__ keys, uint32_t* __restrict__ counts,
                                                    uint32_t ntiles, uint32_t tile_keys, RadixDigit dg) {
    __shared__ TileCounts tc;
    __shared__ uint32_t s_sent;
    tc.clear();
    if (threadIdx.x == 0) s_sent = 0;
    __syncthreads();
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        if (!OFFSETS && tile == ntiles - 1) {   // the tile of vertex n - 1
            uint32_t t = 0;
            for (uint32_t i = threadIdx.x; i < nblocks; i += NT) t += nsent[i];
            t = wave_sum(t);
            if (lane_id() == 0) atomicAdd(&s_sent, t);
            __syncthreads();
        }
        for (uint32_t r = threadIdx.x; r < tile_keys; r += NT) {
            const uint64_t v = (uint64_t)tile * tile_keys + r;
            if (v >= (uint64_t)n) break;
            uint32_t d = degree_at<OFFSETS>(deg, (uint32_t)v);
            if (!OFFSETS && v == (uint64_t)n - 1) {
                d -= s_sent;
                deg[v] = d;
            }
            const uint64_t key = ((uint64_t)(d < RANK_CAP ? d : RANK_CAP) << 32) | (uint32_t)v;
            keys[v] = key;
            const uint32_t digit = (uint32_t)(key >> dg.shift) & dg.mask;
            if (ALIKE) tc.add_shared(digit);   // most keys are those of isolated vertices
            else tc.add(digit);
        }
        tc.flush(counts, ntiles, tile);
    }
}

// rank[v] = position of v; inv its inverse. Vertices of degree RANK_CAP or more stand
// last, by id: each finds its place by comparing (degree, id) with all of them, which the
// block passes through LDS 256 at a time. They are few in a simple graph with hubs, but up to
// 2E / RANK_CAP where pairs repeat: one thread gathering their degrees one by one took
// the rank stage of 3,000, 8,000 and 30,000 vertices that are all of them (2^27, 3e8 and 1e9 pairs,
// CSR in 11, 27 and 98 ms) 0.24, 0.58 and 2.08 ms, this takes 0.07, 0.13 and 0.37; sorting whole
// degrees would take 0.06, and 0.18 ms more at R-MAT 24. Also clears rowend[0..n) and
// part[0..npart) for the stages to come.
template <bool OFFSETS>
__global__ __launch_bounds__(NT) void k_rank(const uint64_t* __restrict__ sorted, int32_t n,
                                             const uint32_t* __restrict__ deg, uint32_t* __restrict__ rank,
                                             uint32_t* __restrict__ inv, uint32_t* __restrict__ rowend,
                                             uint32_t* __restrict__ part, uint32_t npart) {
    __shared__ uint64_t s_key[NT];
    for (uint32_t i = blockIdx.x * NT + threadIdx.x; i < npart; i += gridDim.x * NT) part[i] = 0;
    for (int64_t i0 = (int64_t)blockIdx.x * NT; i0 < n; i0 += (int64_t)gridDim.x * NT) {
        const int64_t i = i0 + threadIdx.x;
        const uint32_t last = (uint32_t)(i0 + NT < n ? i0 + NT : n) - 1u;
        const uint64_t key = sorted[i < n ? i : last];
        const uint32_t v = (uint32_t)key;
        uint32_t pos = (uint32_t)i;
        if ((uint32_t)(sorted[last] >> 32) == RANK_CAP) {   // the same for the whole block
            uint32_t lo = 0, hi = last;   // first of the capped keys
            while (lo < hi) {
                const uint32_t mid = lo + (hi - lo) / 2;
                if ((uint32_t)(sorted[mid] >> 32) < RANK_CAP) lo = mid + 1;
                else hi = mid;
            }
            const bool capped = (uint32_t)(key >> 32) == RANK_CAP;
            const uint64_t me = capped ? ((uint64_t)degree_at<OFFSETS>(deg, v) << 32) | v : 0ull;
            // a step's degrees and the ids after it are in flight while the step before is compared
            auto id_at = [&](uint32_t j) -> uint32_t { return j < (uint32_t)n ? (uint32_t)sorted[j] : ~0u; };
            auto key_of = [&](uint32_t u) -> uint64_t {
                return u != ~0u ? ((uint64_t)degree_at<OFFSETS>(deg, u) << 32) | u : ~0ull;
            };
            uint32_t before = 0, u = id_at(lo + NT + threadIdx.x);
            uint64_t other = key_of(id_at(lo + threadIdx.x));
            for (uint32_t j0 = lo; j0 < (uint32_t)n; j0 += NT) {
                __syncthreads();   // the keys before have been compared
                s_key[threadIdx.x] = other;
                __syncthreads();
                other = key_of(u);
                u = id_at(j0 + 2 * NT + threadIdx.x);
#pragma unroll 16
                for (int q = 0; q < NT; ++q) before += s_key[q] < me ? 1u : 0u;
            }
            if (capped) pos = lo + before;
        }
        if (i < n) {
            rank[v] = pos;
            inv[pos] = v;
            rowend[i] = 0;
        }
    }
}

// ------------------------------------------------------------------ orient (filter by degree order)
// Pair -> (lo rank << nb) | hi rank. Loops and invalid ids become the all-ones
// sentinel on 2*nb bits, which exceeds every valid key (lo rank <= n - 2).
// Eight pairs per thread per step, all loads issued before any is used: the
// rank lookups are random gathers, so the kernel lives on memory-level
// parallelism.
constexpr int OR_U = 8;
// sort tiles (radix_tile_keys) are whole multiples of one round, OR_U * NT keys
// U pairs per thread per step: 16 where the tile is a multiple of 16 * NT
// (4096- and 8192-key tiles; 0.21 -> 0.20 ms at R-MAT 20, no change at larger
// sizes, where the gathers' line traffic bounds the kernel), else OR_U.
template <int U>
__global__ __launch_bounds__(NT) void k_orient(const int2* __restrict__ edges, uint64_t E, int32_t n,
                                               const uint32_t* __restrict__ rank, int nb, uint64_t sentinel,
                                               uint64_t* __restrict__ keys, uint32_t* __restrict__ counts,
                                               uint32_t ntiles, uint32_t tile_keys, RadixDigit dg) {
    // block step = one tile of the pair sort; its first digit is counted as the keys are made
    __shared__ TileCounts tc;
    tc.clear();
    __syncthreads();
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
      for (uint32_t r = 0; r < tile_keys; r += U * NT) {
        const uint64_t i0 = (uint64_t)tile * tile_keys + r + threadIdx.x;
        int2 ed[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint64_t i = i0 + (uint64_t)k * NT;
            ed[k] = i < E ? edges[i] : make_int2(-1, -1);
        }
        uint32_t ra[U], rb[U];
        bool ok[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            ok[k] = ed[k].x >= 0 && ed[k].x < n && ed[k].y >= 0 && ed[k].y < n && ed[k].x != ed[k].y;
            ra[k] = rank[ok[k] ? ed[k].x : 0];
            rb[k] = rank[ok[k] ? ed[k].y : 0];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const uint64_t i = i0 + (uint64_t)k * NT;
            if (i < E) {
                const uint32_t lo = ra[k] < rb[k] ? ra[k] : rb[k], hi = ra[k] < rb[k] ? rb[k] : ra[k];
                const uint64_t key = ok[k] ? (((uint64_t)lo << nb) | hi) : sentinel;
                keys[i] = key;
                if (counts) tc.add((uint32_t)(key >> dg.shift) & dg.mask);
            }
        }
      }
        if (counts) tc.flush(counts, ntiles, tile);
    }
}

// Orientation past 2^21 vertices. There the rank table (4 bytes per vertex)
// outgrows an XCD's 4 MB L2, and two random rank gathers per pair cost two cache
// lines from beyond it. Instead the pairs pass through two stable radix passes
// (radix_pass_u64): one on the high bits of the first id, one on the high bits of
// the second that also replaces the first id by its rank as the pair moves. The
// first pass of the pair sort then reads (second id << 32 | rank of the first
// id), grouped by the second id's high bits, looks up the second rank and forms
// the oriented key as it loads each pair (RX_ORIENT, in its histogram and its
// scatter alike). The blocks of each pass look up ranks in a few
// 2^(vbits - 8)-id ranges at a time, which stay in L2.
constexpr int ORIENT_PART_MIN_BITS = 21;
constexpr int ORIENT_PART_BITS = 8;   // digit of each partition pass

// ------------------------------------------------------------------ unique + CSR
// The sorted pair keys in runs of equal keys: the first of each run is kept,
// sentinel keys (loops, invalid ids; they sort last) are dropped. Each block
// owns a chunk of whole 2048-key tiles, whose kept keys the row sort has
// counted; in a tile, thread t takes the UQ_ITEMS consecutive keys from
// t * UQ_ITEMS (four 16-byte loads, in flight together), so a block scans once
// per tile rather than once per 256 keys; the kept keys are compacted in LDS
// and written out in contiguous runs.
constexpr int UQ_MAX_BLOCKS = 1024;
constexpr int UQ_ITEMS = 8;
constexpr uint32_t UQ_TILE = NT * UQ_ITEMS;

struct Chunking {
    uint32_t nblk, chunk;
};

static Chunking chunking(uint64_t len) {
    uint32_t nblk = (uint32_t)((len + 8191) / 8192);
    if (nblk > (uint32_t)UQ_MAX_BLOCKS) nblk = UQ_MAX_BLOCKS;
    if (nblk < 1) nblk = 1;
    uint64_t chunk = (len + nblk - 1) / nblk;
    chunk = (chunk + UQ_TILE - 1) / UQ_TILE * UQ_TILE;
    if (chunk == 0) chunk = UQ_TILE;
    nblk = (uint32_t)((len + chunk - 1) / chunk);
    if (nblk < 1) nblk = 1;
    return {nblk, (uint32_t)chunk};
}

struct alignas(16) U64x2 {
    uint64_t a, b;
};

// Keys i0 .. i0 + UQ_ITEMS - 1 (i0 a multiple of UQ_ITEMS); `fill` past E.
__device__ __forceinline__ void uq_load(const uint64_t* __restrict__ keys, uint64_t i0, uint64_t E, uint64_t fill,
                                        uint64_t (&k)[UQ_ITEMS]) {
    if (i0 + UQ_ITEMS <= E) {
        const U64x2* p = (const U64x2*)(keys + i0);   // 64-byte aligned
#pragma unroll
        for (int q = 0; q < UQ_ITEMS / 2; ++q) {
            const U64x2 v = p[q];
            k[2 * q] = v.a;
            k[2 * q + 1] = v.b;
        }
    } else {
#pragma unroll
        for (int j = 0; j < UQ_ITEMS; ++j) k[j] = i0 + j < E ? keys[i0 + j] : fill;
    }
}

// Bit j: key i0 + j is the first of its run and not the sentinel.
__device__ __forceinline__ uint32_t uq_keep(const uint64_t* __restrict__ keys, uint64_t i0, uint64_t sentinel,
                                            const uint64_t (&k)[UQ_ITEMS]) {
    uint64_t prev = i0 > 0 ? keys[i0 - 1] : ~k[0];
    uint32_t keep = 0;
#pragma unroll
    for (int j = 0; j < UQ_ITEMS; ++j) {
        keep |= (k[j] != sentinel && k[j] != prev) ? 1u << j : 0u;
        prev = k[j];
    }
    return keep;
}

// Keeps the first of every run of equal keys; rowend[s] = number of kept keys
// up to and including the last key of row s.
__global__ __launch_bounds__(NT) void k_unique_write(const uint64_t* __restrict__ keys, uint64_t E, uint64_t sentinel,
                                                     Ctrl* ctrl, uint32_t chunk, const uint32_t* __restrict__ partial,
                                                     uint32_t nblk, int nb, uint32_t* __restrict__ col,
                                                     uint32_t* __restrict__ src, uint32_t* __restrict__ rowend) {
    __shared__ uint32_t scratch[NT / WAVE];
    __shared__ uint32_t s_col[UQ_TILE], s_src[UQ_TILE];   // the tile's kept keys, compacted
    const uint64_t b0 = (uint64_t)blockIdx.x * chunk;
    const uint64_t b1 = b0 + chunk < E ? b0 + chunk : E;
    const uint64_t lowmask = (1ull << nb) - 1ull;
    uint32_t carry = partial[blockIdx.x];
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->m = partial[nblk];
    for (uint64_t t0 = b0; t0 < b1; t0 += UQ_TILE) {   // the same trip count in every thread
        const uint64_t i0 = t0 + (uint64_t)threadIdx.x * UQ_ITEMS;
        uint64_t k[UQ_ITEMS];
        uint32_t keep = 0;
        uint64_t next = sentinel;   // the key after this thread's last one
        if (i0 < b1) {
            uq_load(keys, i0, E, sentinel, k);
            keep = uq_keep(keys, i0, sentinel, k);
            if (i0 + UQ_ITEMS < E) next = keys[i0 + UQ_ITEMS];
        }
        uint32_t total;
        const uint32_t ex = block_exclusive_scan<NT>((uint32_t)__popc(keep), scratch, &total);
        uint32_t pos = carry + ex, lp = ex;
        if (i0 < b1) {
#pragma unroll
            for (int j = 0; j < UQ_ITEMS; ++j) {
                if (k[j] == sentinel) break;   // the sentinels (and the fill past E) come last
                const uint32_t s = (uint32_t)(k[j] >> nb);
                const uint32_t kp = (keep >> j) & 1u;
                if (kp) {
                    s_col[lp] = (uint32_t)(k[j] & lowmask);
                    s_src[lp] = s;
                }
                pos += kp;
                lp += kp;
                // the sentinel's row differs from every valid row
                const uint64_t nx = j + 1 < UQ_ITEMS ? k[j + 1] : next;
                if ((uint32_t)(nx >> nb) != s) rowend[s] = pos;
            }
        }
        // the kept keys leave in contiguous runs (a thread's own ones are up to
        // eight scattered 4-byte stores per lane otherwise)
        __syncthreads();
        for (uint32_t q = threadIdx.x; q < total; q += NT) {
            col[carry + q] = s_col[q];
            src[carry + q] = s_src[q];
        }
        __syncthreads();
        carry += total;
    }
}

// ------------------------------------------------------------------ CSC (in-edges grouped by v)
// Key of an in-edge e = (u -> v) with a non-empty tail: v in the bits above
// sh, then e, and (packed form, lbits > 0) the tail length in the low lbits
// bits; others get v = n - 1 and sort last: the top-ranked vertex has no
// out-neighbours, so none of its in-edges has work, and ids then need
// bits_for(n) bits, not bits_for(n + 1) (one pass less when n is a power of
// two). In-edges of other vertices without out-neighbours keep their group:
// such a vertex gets no bucket and no tile, so they are never read (testing
// d+(v) here would cost a random gather per edge). A length that does not fit
// the packed field is stored as all ones, and the row end of u is gathered for
// that entry later. Packing saves that gather for the others. FOLLOWS: a bit between
// e and the length says that the row's entry before e is in v's group of the
// GRP_N-vertex groups from gfirst on.
template <bool FOLLOWS>
__global__ __launch_bounds__(NT) void k_csc_keys(const uint32_t* __restrict__ col, const uint32_t* __restrict__ src,
                                                 const uint32_t* __restrict__ off, Ctrl* ctrl, int32_t n,
                                                 uint64_t* __restrict__ keys, int sh, int lbits, uint32_t gfirst,
                                                 uint32_t* __restrict__ counts, uint32_t ntiles, uint32_t tile_keys,
                                                 RadixDigit dg, uint32_t* __restrict__ inend) {
    // inend[0..n): cleared on the way, for k_csc_finish
    for (int64_t v = (int64_t)blockIdx.x * NT + threadIdx.x; v < n; v += (int64_t)gridDim.x * NT) inend[v] = 0;
    __shared__ TileCounts tc;
    tc.clear();
    __syncthreads();
    const uint32_t m = ctrl->m;
    const uint64_t esc = (1ull << lbits) - 1ull;   // escape: length gathered at expansion
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
      for (uint32_t r = 0; r < tile_keys; r += OR_U * NT) {
        const uint64_t e0 = (uint64_t)tile * tile_keys + r + threadIdx.x;
        uint32_t v[OR_U], u[OR_U];
#pragma unroll
        for (int k = 0; k < OR_U; ++k) {   // loads of all OR_U edges in flight together
            const uint64_t e = e0 + (uint64_t)k * NT;
            v[k] = e < m ? col[e] : 0u;
            u[k] = e < m ? src[e] : 0u;
        }
        uint32_t vp[FOLLOWS ? OR_U : 1], up[FOLLOWS ? OR_U : 1];   // the edge before
        if (FOLLOWS) {
#pragma unroll
            for (int k = 0; k < OR_U; ++k) {
                const uint64_t e = e0 + (uint64_t)k * NT;
                vp[k] = e > 0 && e < m ? col[e - 1] : 0u;
                up[k] = e > 0 && e < m ? src[e - 1] : ~0u;
            }
        }
        uint32_t end[OR_U];
#pragma unroll
        for (int k = 0; k < OR_U; ++k) end[k] = off[u[k] + 1];   // rows ascend with e: near-sequential
#pragma unroll
        for (int k = 0; k < OR_U; ++k) {
            const uint64_t e = e0 + (uint64_t)k * NT;
            if (e >= m) continue;
            const bool work = e + 1 < end[k];   // a non-empty tail
            uint64_t low = e;
            if (lbits > 0) {
                const uint64_t len = work ? end[k] - (e + 1) : 0u;
                if (FOLLOWS)
                    low = low << 1 | (up[k] == u[k] && vp[k] >= gfirst && (vp[k] - gfirst) / GRP_N == (v[k] - gfirst) / GRP_N
                                          ? 1u : 0u);
                low = (low << lbits) | (len < esc ? len : esc);
            }
            const uint64_t key = ((uint64_t)(work ? v[k] : (uint32_t)(n - 1)) << sh) | low;
            keys[e] = key;
            if (counts) tc.add((uint32_t)(key >> dg.shift) & dg.mask);
        }
      }
        if (counts) tc.flush(counts, ntiles, tile);
    }
}

// One pass over the sorted in-edge keys: inend[v] = one past the last in-edge
// of v and m_active from the group boundaries, and each key with work written
// to out (the other buffer: neighbours' keys are still being read) as the tail
// range of its edge e, start (e + 1) | end << 32, so a kernel reads it in one
// load. Packed keys carry the length; otherwise the row end of u is gathered.
// Thread t takes keys 2t and 2t + 1 (16-byte loads and stores, coalesced
// across the wave) and reads the key after them.
__device__ __forceinline__ uint64_t csc_range(uint64_t key, uint64_t emask, uint64_t lmask, int lbits, int fbit,
                                              const uint32_t* __restrict__ src, const uint32_t* __restrict__ off) {
    uint32_t e, end;
    uint64_t follows = 0;
    if (lbits > 0) {
        if (fbit) follows = (key >> lbits) << 63;
        e = (uint32_t)((key >> (lbits + fbit)) & emask);
        const uint64_t len = key & lmask;
        end = len != lmask ? e + 1u + (uint32_t)len : off[src[e] + 1];
    } else {
        e = (uint32_t)key;
        end = off[src[e] + 1];
    }
    return (uint64_t)(e + 1u) | ((uint64_t)end << 32) | follows;
}

__global__ __launch_bounds__(NT) void k_csc_finish(const uint64_t* __restrict__ keys, uint64_t* __restrict__ out,
                                                   Ctrl* ctrl, int32_t n, uint32_t* __restrict__ inend, int sh,
                                                   const uint32_t* __restrict__ src,
                                                   const uint32_t* __restrict__ off, int ebits, int lbits, int fbit) {
    const uint32_t m = ctrl->m;
    const uint32_t last = (uint32_t)(n - 1);   // the group of in-edges without work
    const uint64_t emask = (1ull << ebits) - 1ull, lmask = (1ull << lbits) - 1ull;
    const uint64_t none = (uint64_t)last << sh;
    for (uint64_t i0 = ((uint64_t)blockIdx.x * NT + threadIdx.x) * 2; i0 < m; i0 += (uint64_t)gridDim.x * NT * 2) {
        uint64_t k0, k1;
        if (i0 + 2 <= m) {
            const U64x2 v = *(const U64x2*)(keys + i0);   // 16-byte aligned
            k0 = v.a;
            k1 = v.b;
        } else {
            k0 = keys[i0];
            k1 = none;
        }
        const uint64_t k2 = i0 + 2 < m ? keys[i0 + 2] : none;
        const uint32_t v0 = (uint32_t)(k0 >> sh), v1 = (uint32_t)(k1 >> sh), v2 = (uint32_t)(k2 >> sh);
        if (v0 < last && v1 != v0) {
            inend[v0] = (uint32_t)(i0 + 1);
            if (v1 == last) ctrl->m_active = (uint32_t)(i0 + 1);
        }
        if (i0 + 1 < m && v1 < last && v2 != v1) {
            inend[v1] = (uint32_t)(i0 + 2);
            if (v2 == last) ctrl->m_active = (uint32_t)(i0 + 2);
        }
        const uint64_t r0 = v0 < last ? csc_range(k0, emask, lmask, lbits, fbit, src, off) : 0ull;
        const uint64_t r1 = v1 < last ? csc_range(k1, emask, lmask, lbits, fbit, src, off) : 0ull;
        if (i0 + 2 <= m) {
            U64x2 w;
            w.a = r0;
            w.b = r1;
            *(U64x2*)(out + i0) = w;
        } else {
            out[i0] = r0;
        }
    }
}

// ------------------------------------------------------------------ the other formulations
// All in-edges, grouped by v and, inside a group, in CSR order (so by u): key
// v << sh | e, sorted on the v bits only (the sort is stable).
__global__ __launch_bounds__(NT) void k_sym_keys(const uint32_t* __restrict__ col, const Ctrl* ctrl,
                                                 uint64_t* __restrict__ keys, int sh) {
    const uint32_t m = ctrl->m;
    for (uint64_t e = (uint64_t)blockIdx.x * NT + threadIdx.x; e < m; e += (uint64_t)gridDim.x * NT)
        keys[e] = ((uint64_t)col[e] << sh) | e;
}

// inend[v] = one past the last in-edge of v in the sorted order.
__global__ __launch_bounds__(NT) void k_sym_bounds(const uint64_t* __restrict__ keys, const Ctrl* ctrl,
                                                   uint32_t* __restrict__ inend, int sh) {
    const uint32_t m = ctrl->m;
    for (uint64_t i = (uint64_t)blockIdx.x * NT + threadIdx.x; i < m; i += (uint64_t)gridDim.x * NT) {
        const uint64_t v = keys[i] >> sh;
        if (i + 1 == m || (keys[i + 1] >> sh) != v) inend[v] = (uint32_t)(i + 1);
    }
}

// Row offsets of the symmetric adjacency: row v holds N-(v) (in-neighbours,
// all ranked below v) and then N+(v), so fo[v] = inoff[v] + off[v].
__global__ __launch_bounds__(NT) void k_sym_rows(const uint32_t* __restrict__ inoff, const uint32_t* __restrict__ off,
                                                 int32_t n, uint32_t* __restrict__ fo) {
    for (int64_t v = (int64_t)blockIdx.x * NT + threadIdx.x; v <= n; v += (int64_t)gridDim.x * NT)
        fo[v] = inoff[v] + off[v];
}

// Per sorted in-edge i = (u -> v), edge e: (full rows) the two copies of the
// edge in the symmetric adjacency, u at position i - inoff[v] of row v's lower
// part (fo[v] + i - inoff[v] = off[v] + i) and v at position e - off[u] of row
// u's upper part (fo[u] + indeg(u) + e - off[u] = inoff[u + 1] + e); then the
// key becomes the range that the edge streams, start | end << 32.
__global__ __launch_bounds__(NT) void k_sym_build(uint64_t* __restrict__ keys, const Ctrl* ctrl,
                                                  const uint32_t* __restrict__ src, const uint32_t* __restrict__ col,
                                                  const uint32_t* __restrict__ off, const uint32_t* __restrict__ inoff,
                                                  uint32_t* __restrict__ fcol, int sh, int form) {
    const uint32_t m = ctrl->m;
    const uint64_t emask = (1ull << sh) - 1ull;
    for (uint64_t i = (uint64_t)blockIdx.x * NT + threadIdx.x; i < m; i += (uint64_t)gridDim.x * NT) {
        const uint64_t key = keys[i];
        const uint32_t v = (uint32_t)(key >> sh), e = (uint32_t)(key & emask);
        const uint32_t u = src[e];
        const uint32_t ua = off[u], ub = off[u + 1];
        uint32_t st = ua, en = ub;   // MATRIX_UPPER: N+(u) in the oriented columns
        if (form != FORM_MATRIX_UPPER) {
            const uint32_t i0 = inoff[u], i1 = inoff[u + 1];
            fcol[off[v] + (uint32_t)i] = u;
            fcol[i1 + e] = v;
            st = form == FORM_FULL ? i0 + ua : i1 + ua;   // whole row of u, or its upper part
            en = i1 + ub;
        }
        keys[i] = (uint64_t)st | ((uint64_t)en << 32);
    }
}

// ------------------------------------------------------------------ buckets
// Each block adds its sums to the same few words, about 20 ns after one another, so
// there are few and large blocks, and four vertices per thread are in flight for the
// gathers of the lists' ends (2048 blocks of 256, one vertex at a time: 35 us for a million
// vertices of a uniform graph and 27 at R-MAT 20, now 18 and 14). Small graphs, whose
// blocks are few anyway, take small ones (R-MAT 16: the call 428 us with large ones, 424).
constexpr int VB_NT = 1024, VB_BLOCKS = 512, VB_SMALL = 1 << 19;
__global__ __launch_bounds__(VB_NT) void k_vbucket(const uint32_t* __restrict__ off, const uint32_t* __restrict__ col,
                                                const uint32_t* __restrict__ inoff, int32_t n,
                                                uint8_t* __restrict__ vbucket, Ctrl* ctrl) {
    __shared__ BucketSums S;
    const int nt = (int)blockDim.x;
    S.clear(nt);
    __syncthreads();
    constexpr int U = 4;   // vertices in flight per thread
    for (int64_t v0 = (int64_t)blockIdx.x * nt + threadIdx.x; v0 < n; v0 += (int64_t)gridDim.x * nt * U) {
        uint32_t din[U], o0[U], o1[U], lo[U], hi[U];
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t v = v0 + (int64_t)k * gridDim.x * nt, w = v < n ? v : v0;
            din[k] = inoff[w + 1] - inoff[w];
            o0[k] = off[w];
            o1[k] = off[w + 1];
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const bool work = din[k] > 0 && o1[k] > o0[k];
            lo[k] = work ? col[o0[k]] : 0u;
            hi[k] = work ? col[o1[k] - 1u] : 0u;
        }
#pragma unroll
        for (int k = 0; k < U; ++k) {
            const int64_t v = v0 + (int64_t)k * gridDim.x * nt;
            if (v >= n) break;
            const uint32_t b = bucket_of(din[k], o1[k] - o0[k]);
            vbucket[v] = (uint8_t)b;
            if (b != BUCKET_NONE) S.add(din[k], o1[k] - o0[k], lo[k], hi[k]);
        }
    }
    __syncthreads();
    S.flush(ctrl, nt);
}

// ------------------------------------------------------------------ selection
// One thread per bucket. The heuristic follows the paper's dynamic grouping:
// fixed degree thresholds decide between the cooperative (staged) and the
// per-pair strategies. Here the staged LDS bitmap takes middle vertices with
// at least 64 in-edges, or at least 16 in-edges and 64 out-neighbours (the
// bitmap's set-up is then amortised), binary search takes lists of at least
// 16 out-neighbours, and merge-path the rest. The thresholds were chosen from
// per-bucket timings of all three kernels on R-MAT and Chung-Lu graphs of
// 2^17 to 2^22 vertices and on a batch of 4096 small Chung-Lu graphs.
__device__ int heuristic_choice(int b) {
    const int li = b >> 4, lo = b & 15;   // floor log2 of in-degree and out-degree
    if (li >= 6 || (li >= 4 && lo >= 6)) return KER_BITMAP;
    if (lo >= 4) return KER_BSEARCH;
    return KER_MERGE;
}

constexpr uint32_t EDGE_CHUNK_MAX = 2048;   // in-edges per tile of the edge-centric kernels
constexpr unsigned long long EDGE_TILES = 512;

__global__ __launch_bounds__(NBUCKET) void k_select(Ctrl* ctrl, int mode, const uint8_t* __restrict__ learned,
                                                    const uint8_t* __restrict__ learned_tile,
                                                    const uint16_t* __restrict__ chunk_override,
                                                    const uint8_t* __restrict__ group_override, int whole_rows,
                                                    int features, HubTab* __restrict__ hub) {
    __shared__ __align__(16) uint32_t s_key[NBUCKET], s_nv[NBUCKET];
    const int b = threadIdx.x;
    s_nv[b] = b == BUCKET_NONE ? 0u : ctrl->bucket_nv[b];
    if (features) {   // the selector networks write them otherwise
        float f[MLP_IN];
        bucket_features(ctrl, b, f);
        for (int i = 0; i < MLP_IN; ++i) ctrl->features[b][i] = f[i];
    }
    if (hub) hub->first[b] = hub->grp[b] = ~0u;   // set by k_emit_tiles
    int ch;
    if (mode == SEL_FORCE_MERGE) ch = KER_MERGE;
    else if (mode == SEL_FORCE_BSEARCH) ch = KER_BSEARCH;
    else if (mode == SEL_FORCE_BITMAP) ch = KER_BITMAP;
    else if (mode == SEL_LEARNED && learned) ch = learned[b] < NKERNEL ? learned[b] : heuristic_choice(b);
    else ch = heuristic_choice(b);
    const int lo = b & 15, li = b >> 4;
    // tile shape: in-edges per tile and lanes per in-edge.
    // Bitmap tiles of vertices with at least 256 in-edges, and of whole-row tails
    // (cut per bitmap window), take the largest chunk: a tile's set-up (entry
    // table, bitmap of the middle list, dependent loads of its descriptors) is
    // then spread over the most in-edges (measured at R-MAT 20: bitmap kernel
    // 1.24 -> 1.08 ms against 256 in-edges everywhere).
    // The edge-centric kernels' tiles of vertices with short lists (fewer than
    // 64 out-neighbours) grow with the bucket's in-edges, to about EDGE_TILES
    // tiles per bucket, between 256 and 2048 in-edges: their per-tile set-up is
    // a chain of dependent loads that the short lists do not hide (measured: a
    // random geometric graph of 2^23 vertices, merge 6.9 -> 4.4 ms and binary
    // search 5.6 -> 4.2 ms; R-MAT 20, whose edge-kernel buckets are small,
    // keeps 256; longer lists gained nothing and lost at R-MAT 24). The shape
    // depends on the bucket alone, so a bucket timed alone (selector training)
    // has the tiles that it has among the others.
    uint32_t chunk = (ch == KER_BITMAP && (whole_rows || li >= 8)) ? (uint32_t)CHUNK_MAX : 256u;
    if (ch != KER_BITMAP && lo <= 5) {
        const unsigned long long per = ctrl->bucket_in[b] / EDGE_TILES;
        chunk = per < 256ull ? 256u : (per > (unsigned long long)EDGE_CHUNK_MAX ? EDGE_CHUNK_MAX : (uint32_t)per);
    }
    uint32_t group = lo >= 9 ? 64u : (lo >= 3 ? (1u << (lo - 3)) : 1u);
    // the tile network scales the rule's tile size by 1/2, 1 or 2
    if (learned_tile && learned_tile[b] == 0) chunk = chunk / 2u;
    else if (learned_tile && learned_tile[b] == 2) chunk = chunk * 2u;
    if (chunk_override && chunk_override[b]) chunk = chunk_override[b];
    if (group_override && group_override[b]) group = group_override[b];
    const uint32_t cmax = ch == KER_BITMAP ? (uint32_t)CHUNK_MAX : EDGE_CHUNK_MAX;
    if (chunk > cmax) chunk = cmax;
    if (chunk < 16u) chunk = 16u;
    if (group > 64u || (group & (group - 1u))) group = 64u;
    if (group < 1u) group = 1u;
    ctrl->choice[b] = (uint8_t)ch;
    ctrl->chunk[b] = (uint16_t)chunk;
    ctrl->group[b] = (uint8_t)group;
    // slot order: (kernel, heavier tiles first); the empty bucket last
    const uint32_t key = (b == BUCKET_NONE) ? 0xFFFFFFFFu : ((uint32_t)ch << 16) | (uint32_t)(255 - (16 * lo + li));
    s_key[b] = key;
    __syncthreads();
    uint32_t r = 0, at = 0;   // buckets before this one, and their vertices
#pragma unroll 8
    for (int q = 0; q < NBUCKET; q += 4) {   // keys are distinct but for the empty bucket's, the highest
        const uint4 k = *(const uint4*)&s_key[q], c = *(const uint4*)&s_nv[q];
        r += (k.x < key ? 1u : 0u) + (k.y < key ? 1u : 0u) + (k.z < key ? 1u : 0u) + (k.w < key ? 1u : 0u);
        at += (k.x < key ? c.x : 0u) + (k.y < key ? c.y : 0u) + (k.z < key ? c.z : 0u) + (k.w < key ? c.w : 0u);
    }
    ctrl->slot[b] = (uint8_t)r;
    ctrl->bstart[b] = at;
    ctrl->bend[b] = at + s_nv[b];
}

template <bool ALIKE>
__global__ __launch_bounds__(NT) void k_vkeys_slot(const uint8_t* __restrict__ vbucket, int32_t n, const Ctrl* ctrl,
                                                   uint64_t* __restrict__ keys, uint32_t* __restrict__ counts,
                                                   uint32_t ntiles, uint32_t tile_keys, RadixDigit dg) {
    __shared__ TileCounts tc;
    __shared__ uint8_t s_slot[NBUCKET];
    tc.clear();
    s_slot[threadIdx.x] = ctrl->slot[threadIdx.x];
    __syncthreads();
    static_assert(NT == NBUCKET, "a slot per thread");
    for (uint32_t tile = blockIdx.x; tile < ntiles; tile += gridDim.x) {
        for (uint32_t r = threadIdx.x; r < tile_keys; r += NT) {
            const uint64_t v = (uint64_t)tile * tile_keys + r;
            if (v >= (uint64_t)n) break;
            const uint64_t key = ((uint64_t)s_slot[vbucket[v]] << 32) | (uint32_t)v;
            keys[v] = key;
            const uint32_t digit = (uint32_t)(key >> dg.shift) & dg.mask;
            if (ALIKE) tc.add_shared(digit);   // most keys are those of isolated vertices
            else tc.add(digit);
        }
        tc.flush(counts, ntiles, tile);
    }
}

// The vertex list and the tiles that start at each of its positions.
__global__ __launch_bounds__(NT) void k_ntiles(const uint64_t* __restrict__ sorted, uint32_t* __restrict__ vlist,
                                               const uint8_t* __restrict__ vbucket,
                                               const uint32_t* __restrict__ inoff, int32_t n, const Ctrl* ctrl,
                                               uint32_t* __restrict__ ntile) {
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const uint32_t v = (uint32_t)sorted[i];
        vlist[i] = v;
        const uint32_t b = vbucket[v];
        uint32_t t = 0;
        if (b != BUCKET_NONE) {
            const uint32_t g = tile_group(ctrl, b);
            if (g > 1) {
                t = ((uint32_t)i - ctrl->bstart[b]) % g == 0 ? 1u : 0u;
            } else {
                const uint32_t din = inoff[v + 1] - inoff[v];
                const uint32_t K = ctrl->chunk[b];
                t = (din + K - 1) / K;
            }
        }
        ntile[i] = t;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ntile[n] = 0;
}

__global__ __launch_bounds__(NT) void k_emit_tiles(const uint32_t* __restrict__ vlist,
                                                   const uint8_t* __restrict__ vbucket,
                                                   const uint32_t* __restrict__ inoff,
                                                   const uint32_t* __restrict__ tstart, int32_t n, Ctrl* ctrl,
                                                   uint4* __restrict__ tiles, uint64_t tile_cap,
                                                   HubTab* __restrict__ hub, uint32_t gfirst) {
    for (int64_t i = (int64_t)blockIdx.x * NT + threadIdx.x; i < n; i += (int64_t)gridDim.x * NT) {
        const uint32_t b = vbucket[vlist[i]];
        const int kk = b == BUCKET_NONE ? NKERNEL : ctrl->choice[b];
        int kprev = -1;
        if (i > 0) {
            const uint32_t bp = vbucket[vlist[i - 1]];
            kprev = bp == BUCKET_NONE ? NKERNEL : ctrl->choice[bp];
        }
        const uint32_t t0 = tstart[i], t1 = tstart[i + 1];
        if (t1 > t0 && b != BUCKET_NONE) {
            const uint32_t g = tile_group(ctrl, b);
            if (g > 1) {
                const uint32_t cnt = min(g, ctrl->bend[b] - (uint32_t)i);
                if (t0 < tile_cap) tiles[t0] = make_uint4((uint32_t)i, cnt, 0u, TILE_MULTI);
            } else {
                const uint32_t v = vlist[i];
                const uint32_t K = ctrl->chunk[b];
                const uint32_t e_beg = inoff[v], e_end = inoff[v + 1];
                // ranks ascend within a bucket, so its hub tiles are a suffix of its tiles
                if (hub && kk == KER_BITMAP && v >= hub_first((uint32_t)n) &&
                    ((uint32_t)i == ctrl->bstart[b] || vlist[i - 1] < hub_first((uint32_t)n)))
                    hub->first[b] = t0;
                if (hub && kk == KER_BITMAP && v >= gfirst && ((uint32_t)i == ctrl->bstart[b] || vlist[i - 1] < gfirst))
                    hub->grp[b] = t0;   // and the group kernel's a suffix of these
                for (uint32_t t = t0; t < t1 && t < tile_cap; ++t) {
                    const uint32_t e0 = e_beg + (t - t0) * K;
                    tiles[t] = make_uint4(v, e0, (e0 + K < e_end ? e0 + K : e_end) - e0, 0u);
                }
            }
        }
        for (int k = kprev + 1; k <= kk; ++k) ctrl->tile_begin[k] = t0;
        if (i == n - 1) {
            for (int k = kk + 1; k <= NKERNEL; ++k) ctrl->tile_begin[k] = tstart[n];
            ctrl->ntiles = tstart[n];
        }
    }
}

// Tile ranges of the bitmap kernel and of the hub kernel, per bucket in slot
// order (one thread per slot), and the group kernel's tiles. The hub kernel gets tiles on graphs with about
// HUB_MIN_TAILS tail elements or more: its columns, its launch and its longer
// set-up per tile cost 50 us and more, which it makes up for around there (R-MAT
// 20, 1.2e9 tail elements: 2.69 -> 2.66 ms; R-MAT 21, 3e9: 5.52 -> 5.27 ms; Chung-Lu of 40
// million pairs, 0.5e9: 6.99 ms without, 7.02 ms with it).
constexpr uint64_t HUB_MIN_TAILS = 1ull << 30;
// The wave kernel takes the buckets of in-degree class WAVE_LI and below that have no
// hub tile (its comment has the figures).
constexpr uint32_t WAVE_LI = 9;
// In-edges per tile of the group kernel: GRP_TILES tiles per block, within limits (6 and 24 tiles
// per block: R-MAT 24 43.4 and 43.1 ms against 43.1; R-MAT 20 with tiles of 4000, 2000 and 1000
// in-edges 2433, 2432 and 2480 us, and with shorter set-ups 2085 us from 4096, 2103 from 2048).
constexpr uint32_t GRP_TILES = 12, GRP_EDGES_MIN = 4096, GRP_EDGES_MAX = 16384;
static_assert(GRP_COUNT % NBUCKET == 0, "whole groups per thread");
__global__ __launch_bounds__(NBUCKET) void k_hub_ranges(const Ctrl* ctrl, const uint32_t* __restrict__ tstart,
                                                        const uint8_t* __restrict__ vbucket,
                                                        const uint32_t* __restrict__ inoff, uint32_t gfirst,
                                                        uint32_t group_blocks, int waves, HubTab* __restrict__ hub) {
    __shared__ uint32_t s_bucket[NBUCKET];
    __shared__ uint32_t scratch[NBUCKET / WAVE];
    const uint32_t r = threadIdx.x;
    __shared__ uint8_t s_single[NBUCKET];   // single-vertex tiles of the bitmap strategy
    s_bucket[ctrl->slot[r]] = r;
    s_single[r] = r != (uint32_t)BUCKET_NONE && ctrl->choice[r] == KER_BITMAP && tile_group(ctrl, r) == 1u;
    __syncthreads();
    const uint32_t b = s_bucket[r];
    // tail elements of the graph, about: sum over u of d+(u)^2 / 2 from the buckets' means
    const uint64_t nv = b != (uint32_t)BUCKET_NONE ? ctrl->bucket_nv[b] : 0u;
    const double out = nv ? (double)ctrl->bucket_out[b] : 0.0;
    __shared__ uint64_t scratch64[NBUCKET / WAVE];
    uint64_t tails;
    (void)block_exclusive_scan<NBUCKET>((uint64_t)(nv ? 0.5 * out * out / (double)nv : 0.0), scratch64, &tails);
    const bool use = tails >= HUB_MIN_TAILS;   // the same in every thread
    uint32_t t0 = 0, t1 = 0, h = 0;
    uint32_t nwv = 0;   // vertices for the wave kernel
    if (nv && ctrl->choice[b] == KER_BITMAP) {
        t0 = tstart[ctrl->bstart[b]];
        t1 = tstart[ctrl->bend[b]];
        if (use && group_blocks && hub->grp[b] != ~0u) t1 = hub->grp[b];
        const bool has = use && hub->first[b] != ~0u;
        h = has ? hub->first[b] : t1;
        if (waves && (b >> 4) <= WAVE_LI && !has) {
            nwv = (uint32_t)nv;
            h = t1 = t0;
        }
    }
    uint32_t nwave;
    const uint32_t pw = block_exclusive_scan<NBUCKET>(nwv, scratch, &nwave);
    hub->wave_pos[r] = ctrl->bstart[b];
    hub->wave_pref[r] = pw;
    uint32_t rest, hubs;
    const uint32_t pr = block_exclusive_scan<NBUCKET>(h - t0, scratch, &rest);
    const uint32_t ph = block_exclusive_scan<NBUCKET>(t1 - h, scratch, &hubs);
    hub->rest_tile[r] = t0;
    hub->rest_pref[r] = pr;
    hub->hub_tile[r] = h;
    hub->hub_pref[r] = ph;
    // the group kernel: two groups per thread
    constexpr uint32_t GPT = GRP_COUNT / NBUCKET;
    uint32_t inc[GPT], edges[GPT], mine = 0, total, tiles, nt[GPT], sum = 0;
    for (uint32_t k = 0; k < GPT; ++k) {
        inc[k] = edges[k] = 0;
        if (!use || !group_blocks) continue;
        const uint32_t v0 = gfirst + (r * GPT + k) * GRP_N;
        uint32_t w[GRP_N / 4];   // the group's buckets, at any alignment
        __builtin_memcpy(w, vbucket + v0, GRP_N);
#pragma unroll
        for (uint32_t q = 0; q < GRP_N; ++q)
            inc[k] |= s_single[(w[q / 4] >> (8 * (q & 3))) & 0xFFu] ? 1u << q : 0u;
        edges[k] = inc[k] ? inoff[v0 + GRP_N] - inoff[v0] : 0u;
        mine += edges[k];
    }
    (void)block_exclusive_scan<NBUCKET>(mine, scratch, &total);
    uint32_t per = group_blocks ? total / (group_blocks * GRP_TILES) : 0u;
    per = per < GRP_EDGES_MIN ? GRP_EDGES_MIN : (per > GRP_EDGES_MAX ? GRP_EDGES_MAX : per);
    for (uint32_t k = 0; k < GPT; ++k) sum += nt[k] = (edges[k] + per - 1u) / per;
    uint32_t pg = block_exclusive_scan<NBUCKET>(sum, scratch, &tiles);
    for (uint32_t k = 0; k < GPT; ++k) {
        hub->grp_inc[r * GPT + k] = inc[k];
        hub->grp_pref[r * GPT + k] = pg;
        pg += nt[k];
    }
    if (r == 0) {
        hub->rest_pref[NBUCKET] = rest;
        hub->hub_pref[NBUCKET] = hubs;
        hub->grp_pref[GRP_COUNT] = tiles;
        hub->grp_edges = per;
        hub->wave_pref[NBUCKET] = nwave;
        hub->used = hubs + tiles + nwave;
    }
}

// The hub kernel's 16-bit columns; left alone when there is no hub tile.
// Eight columns per thread: two 16-byte loads, one 16-byte store (m is below
// the capacity by at least the last group's padding: see hub_usable).
__global__ __launch_bounds__(NT) void k_col16(const uint32_t* __restrict__ col, const Ctrl* ctrl, uint32_t base,
                                              const HubTab* __restrict__ hub, uint16_t* __restrict__ out) {
    if (hub->hub_pref[NBUCKET] == 0 && hub->grp_pref[GRP_COUNT] == 0) return;
    const uint64_t m = ctrl->m;
    for (uint64_t i = ((uint64_t)blockIdx.x * NT + threadIdx.x) * 8; i < m; i += (uint64_t)gridDim.x * NT * 8) {
        uint32_t x[8];
        if (i + 8 <= m) {
            const uint4 p = *(const uint4*)(col + i), q = *(const uint4*)(col + i + 4);
            x[0] = p.x; x[1] = p.y; x[2] = p.z; x[3] = p.w;
            x[4] = q.x; x[5] = q.y; x[6] = q.z; x[7] = q.w;
        } else {
            for (int k = 0; k < 8; ++k) x[k] = i + k < m ? col[i + k] : 0u;
        }
        uint32_t y[8];
#pragma unroll
        for (int k = 0; k < 8; ++k) y[k] = x[k] >= base ? x[k] - base : HUB_NONE;
        *(uint4*)(out + i) = make_uint4(y[0] | y[1] << 16, y[2] | y[3] << 16, y[4] | y[5] << 16, y[6] | y[7] << 16);
    }
}

// ------------------------------------------------------------------ outputs
__global__ __launch_bounds__(NT) void k_map_pv(const uint64_t* __restrict__ pv, const uint32_t* __restrict__ inv,
                                               int32_t n, uint64_t* __restrict__ out) {
    for (int64_t r = (int64_t)blockIdx.x * NT + threadIdx.x; r < n; r += (int64_t)gridDim.x * NT) out[inv[r]] = pv[r];
}

// ------------------------------------------------------------------ clustering epilogue
// Local clustering coefficient C(v) = t[v] / C(d(v), 2) (zero when d(v) < 2)
// and the number of wedges (paths of length two) sum_v C(d(v), 2), which with
// T gives the transitivity 3T / wedges. d(v) is the simple-graph degree: the
// out-degree of v's CSR row plus its in-degree over the kept edges: the grouped in-edges
// (those with a non-empty tail) and the rows that end in v.
constexpr unsigned CL_MAX_BLOCKS = 4096;   // block partials live in the intersection partials

// last[v] += rows whose highest neighbour is v: the in-edges that the in-edge
// grouping leaves out. Most rows end in a few hubs, so the top LAST_N ranks
// are counted in LDS (one atomic per kept edge into the in-degrees took 689 us at
// R-MAT 18; this takes 6). From LAST_FEW vertices on four times the blocks, for the rows
// themselves (2^24 vertices, few pairs: 66 -> 22 us).
constexpr uint32_t LAST_N = 8192;
constexpr unsigned LAST_NT = 1024;
constexpr int32_t LAST_FEW = 1 << 22;
__global__ __launch_bounds__(LAST_NT) void k_row_last(const uint32_t* __restrict__ off,
                                                      const uint32_t* __restrict__ col, int32_t n,
                                                      uint32_t* __restrict__ last) {
    __shared__ uint32_t s_cnt[LAST_N];
    const uint32_t first = (uint32_t)n > LAST_N ? (uint32_t)n - LAST_N : 0u;
    for (uint32_t i = threadIdx.x; i < LAST_N; i += LAST_NT) s_cnt[i] = 0;
    __syncthreads();
    for (int64_t u = (int64_t)blockIdx.x * LAST_NT + threadIdx.x; u < n; u += (int64_t)gridDim.x * LAST_NT) {
        const uint32_t a = off[u], b = off[u + 1];
        if (a == b) continue;
        const uint32_t v = col[b - 1];
        if (v >= first) atomicAdd(&s_cnt[v - first], 1u);
        else atomicAdd(&last[v], 1u);
    }
    __syncthreads();
    for (uint32_t i = threadIdx.x; i < LAST_N; i += LAST_NT) {
        const uint32_t q = (i + blockIdx.x * 64u) % LAST_N;
        if (s_cnt[q]) atomicAdd(&last[first + q], s_cnt[q]);
    }
}

__global__ __launch_bounds__(NT) void k_clustering(const uint64_t* __restrict__ t, const uint32_t* __restrict__ inv,
                                                   const uint32_t* __restrict__ off,
                                                   const uint32_t* __restrict__ inoff,
                                                   const uint32_t* __restrict__ last, int32_t n,
                                                   double* __restrict__ coeff, uint64_t* __restrict__ partials) {
    __shared__ uint64_t red[NT / WAVE];
    uint64_t acc = 0;
    for (int64_t r = (int64_t)blockIdx.x * NT + threadIdx.x; r < n; r += (int64_t)gridDim.x * NT) {
        const uint64_t d = (uint64_t)(off[r + 1] - off[r]) + (inoff[r + 1] - inoff[r]) + last[r];
        const uint64_t w = d < 2 ? 0ull : d * (d - 1) / 2;
        acc += w;
        coeff[inv[r]] = w ? (double)t[r] / (double)w : 0.0;
    }
    acc = wave_sum_u64(acc);
    if (lane_id() == 0) red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int i = 0; i < NT / WAVE; ++i) s += red[i];
        partials[blockIdx.x] = s;
    }
}

__global__ __launch_bounds__(NT) void k_sum_wedges(const uint64_t* __restrict__ partials, unsigned count, Ctrl* ctrl) {
    __shared__ uint64_t red[NT / WAVE];
    uint64_t acc = 0;
    for (unsigned i = threadIdx.x; i < count; i += NT) acc += partials[i];
    acc = wave_sum_u64(acc);
    if (lane_id() == 0) red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int i = 0; i < NT / WAVE; ++i) s += red[i];
        ctrl->wedges = s;
    }
}

__global__ __launch_bounds__(NT) void k_map_edges(const uint32_t* __restrict__ col, const uint32_t* __restrict__ src,
                                                  const uint32_t* __restrict__ inv, const Ctrl* ctrl,
                                                  int2* __restrict__ out) {
    const uint32_t m = ctrl->m;
    for (uint64_t e = (uint64_t)blockIdx.x * NT + threadIdx.x; e < m; e += (uint64_t)gridDim.x * NT)
        out[e] = make_int2((int)inv[src[e]], (int)inv[col[e]]);
}

__global__ __launch_bounds__(NT) void k_export_csr(const uint32_t* __restrict__ rank, const uint32_t* __restrict__ off,
                                                   const uint32_t* __restrict__ col, const Ctrl* ctrl, int32_t n,
                                                   int32_t* __restrict__ o_rank, int64_t* __restrict__ o_off,
                                                   int32_t* __restrict__ o_col) {
    const uint32_t m = ctrl->m;
    const uint64_t stride = (uint64_t)gridDim.x * NT;
    for (uint64_t i = (uint64_t)blockIdx.x * NT + threadIdx.x; i < (uint64_t)n + 1; i += stride) {
        if (i < (uint64_t)n) o_rank[i] = (int32_t)rank[i];
        o_off[i] = (int64_t)off[i];
    }
    for (uint64_t e = (uint64_t)blockIdx.x * NT + threadIdx.x; e < m; e += stride) o_col[e] = (int32_t)col[e];
}

__global__ void k_set_tile_range(Ctrl* ctrl, int ker, uint32_t t0, uint32_t t1) {
    if (threadIdx.x == 0) {
        ctrl->tile_begin[ker] = t0;
        ctrl->tile_begin[ker + 1] = t1;
        ctrl->tile_next[ker] = 0;
    }
}

// The intersection kernels' shared tile counters, zeroed before a relaunch.
static void reset_tile_counters(Ctrl* ctrl, hipStream_t s) {
    fill_u32(ctrl->tile_next, 0u, NKERNEL + 2, s);
}

// Packed in-edge keys: v, e, and the tail length in the bits left over (at
// most what the bound d+(u) <= sqrt(2E) needs; lengths that do not fit are
// escaped). Without room for at least 6 length bits, e alone is kept.
// follows: a bit above the length for CSC_FOLLOWS (fbit 1; 0 without room).
struct CscPacking {
    int sh, ebits, lbits, fbit;
};

static CscPacking csc_packing(int64_t E, int32_t n, bool follows) {
    const uint64_t twoE = 2ull * (uint64_t)E;
    uint64_t r = (uint64_t)sqrt((double)twoE);   // floor(sqrt(2E)), the bound on d+(u)
    while (r * r > twoE) --r;
    while ((r + 1) * (r + 1) <= twoE) ++r;
    const int eb = bits_for((uint64_t)E), vb = bits_for((uint64_t)n);
    int lb = bits_for(r + 2);   // lengths below r + 1, plus the escape value
    const int room = 64 - vb - eb;
    if (follows && room >= 7) {
        if (lb > room - 1) lb = room - 1;
        return {eb + 1 + lb, eb, lb, 1};
    }
    if (lb > room) lb = room;
    if (lb >= 6) return {eb + lb, eb, lb, 0};
    return {32, 32, 0, 0};
}

// ------------------------------------------------------------------ workspace layout
Layout make_layout(int64_t E, int32_t n) {
    Layout L;
    const size_t A = 256;
    const size_t nn = (size_t)n, ee = (size_t)E;
    const size_t kcap = ee > nn ? ee : nn;
    size_t o = 0;
    auto take = [&](size_t bytes) { size_t r = o; o = align_up(o + (bytes ? bytes : 1), A); return r; };
    L.ctrl = take(sizeof(Ctrl));
    L.deg = take(4 * (nn + 1));
    L.rank = take(4 * nn);
    L.inv = take(4 * nn);
    L.vbucket = take(nn);
    L.vlist = take(4 * nn);
    L.tstart = take(4 * (nn + 1));
    L.off = take(4 * (nn + 1));
    L.inoff = take(4 * (nn + 1));
    L.rowend = take(4 * nn);
    L.pv = take(8 * nn);
    L.vkeysA = take(8 * nn);
    L.vkeysB = take(8 * nn);
    L.keysA = take(8 * kcap);
    L.keysB = take(8 * kcap);
    L.col = take(4 * ee);
    L.src = take(4 * ee);
    L.tile_cap = ee / 16 + nn + 1;
    L.tiles = take(16 * L.tile_cap);
    L.partial = take(4 * (UQ_MAX_BLOCKS + 1));
    L.bstart = take(4 * ((1u << DEG_MAX_BUCKET_BITS) + 4));
    L.isect_partials = take(isect_partials_bytes());
    L.scan_tmp = take(scan_temp_bytes());
    L.lb_aux = take(4 * 256);
    L.radix_tmp = take(radix_temp_bytes(2 * ee > nn ? 2 * ee : nn));
    L.total = o;
    return L;
}

// ------------------------------------------------------------------ the pipeline
int stage_count() { return NSTAGE; }
const char* stage_name(int s) {
    static const char* names[NSTAGE] = {"degree", "rank", "orient", "sort", "csr", "csc", "bucket",
                                        "group", "isect_merge", "isect_bsearch", "isect_bitmap", "finish"};
    return (s >= 0 && s < NSTAGE) ? names[s] : "";
}

// The symmetric adjacency of the other formulations, after the pipeline's own workspace.
static uint32_t* sym_off(const RunArgs& r, const Layout& L) { return (uint32_t*)((char*)r.ws + L.total); }
static uint32_t* sym_col(const RunArgs& r, const Layout& L) {
    return (uint32_t*)((char*)r.ws + L.total + align_up(4 * ((size_t)r.n + 1), 256));
}

static IsectArgs isect_args(const RunArgs& r, const Layout& L, uint64_t* csc) {
    char* ws = (char*)r.ws;
    const bool sym = r.formulation == FORM_FULL || r.formulation == FORM_MATRIX;
    IsectArgs ia;
    ia.ctrl = (Ctrl*)(ws + L.ctrl);
    ia.off = sym ? sym_off(r, L) : (const uint32_t*)(ws + L.off);
    ia.col = sym ? sym_col(r, L) : (const uint32_t*)(ws + L.col);
    ia.src = (const uint32_t*)(ws + L.src);
    ia.csc = csc;
    ia.inoff = (const uint32_t*)(ws + L.inoff);
    ia.vlist = (const uint32_t*)(ws + L.vlist);
    ia.vbucket = (const uint8_t*)(ws + L.vbucket);
    ia.tiles = (const uint4*)(ws + L.tiles);
    ia.per_edge = r.per_edge_counts;
    ia.per_vertex = (r.per_vertex || r.clustering) ? (uint64_t*)(ws + L.pv) : nullptr;
    ia.hot_first = isect_hot_first((uint32_t)r.n);
    ia.per_middle = r.per_middle ? (uint64_t*)(ws + L.pv) : nullptr;
    ia.support = r.support;
    ia.list_off = r.list_off;
    ia.list_cur = r.list_cur;
    ia.list_out = r.list_out;
    ia.list_cap = r.list_cap;
    ia.inv = (const uint32_t*)(ws + L.inv);
    ia.col_narrow = (sym ? 2 * r.E : r.E) < ((int64_t)1 << 30) ? 1u : 0u;   // m <= E
    ia.clip = r.formulation != FORM_FILTERED ? 1u : 0u;
    ia.col16 = nullptr;
    ia.hub = nullptr;
    ia.groups = ia.waves = false;
    ia.first_rank = 0;
    return ia;
}

// Where the CSC array ended up (it depends on the parity of the sort passes;
// the filtered form's tail ranges are written to the buffer its sort left free).
static uint64_t* csc_of(const RunArgs& r, const Layout& L) {
    char* ws = (char*)r.ws;
    const int nb = bits_for((uint64_t)r.n) > 0 ? bits_for((uint64_t)r.n) : 1;
    const int p1 = (nb + 7) / 8;                       // radix passes of the pair sort (on the row)
    const int p2 = (bits_for((uint64_t)r.n) + 7) / 8;   // passes of the CSC sort
    uint64_t* sorted = (p1 & 1) ? (uint64_t*)(ws + L.keysB) : (uint64_t*)(ws + L.keysA);
    uint64_t* other = (p1 & 1) ? (uint64_t*)(ws + L.keysA) : (uint64_t*)(ws + L.keysB);
    const bool keys_in_sorted = (p2 & 1) != 0;
    return keys_in_sorted == (r.formulation == FORM_FILTERED) ? other : sorted;
}

// The hub kernel counts (in all, or per middle vertex) on the filtered graph.
// Its 16-bit columns take the key buffer that the in-edge sort left free, 8 bytes
// per pair against 2 and a last group of eight. From HUB_MIN_PAIRS on, about where
// the preparing kernels and the extra launches (with the group and the wave kernel) pay on
// graphs of ordinary density. Queued counts without and with them: R-MAT 15, 16, 17, 18 and 19 (16 pairs per
// vertex) 306 and 377, 368 and 402, 504 and 541, 692 and 700, 1219 and 1202 us; Chung-Lu of 6 million
// pairs 924 and 963; uniform of 10 million 1210 and 1233; random geometric of 8.4 million 1083
// and 1099. Denser graphs gain earlier (R-MAT 17 with 12 million pairs: 1733 and 1450).
constexpr int64_t HUB_MIN_PAIRS = 1 << 24;
static bool hub_usable(const RunArgs& r) {
    return r.formulation == FORM_FILTERED && r.E >= HUB_MIN_PAIRS && !r.per_vertex && !r.clustering &&
           !r.per_edge_counts && !r.support && !r.list_out;
}

// The group kernel takes part where only the count is asked for, all HUB_SPAN columns
// exist, and the packed in-edge keys have room for its mark.
static bool groups_wanted(const RunArgs& r) {
    return hub_usable(r) && !r.per_middle && r.n >= (int32_t)HUB_SPAN && r.E < (1ll << 31);
}
static bool groups_usable(const RunArgs& r) { return groups_wanted(r) && csc_packing(r.E, r.n, true).fbit; }

// Its tables take the degree count's bucket starts, dead since the degree stage.
static HubTab* hub_tab(const RunArgs& r, const Layout& L) {
    static_assert(sizeof(HubTab) <= 4 * ((1u << DEG_MAX_BUCKET_BITS) + 4), "hub tables fit the bucket starts");
    return hub_usable(r) ? (HubTab*)((char*)r.ws + L.bstart) : nullptr;
}

// Fills the tables and the columns (after the tiles) and points ia at them.
static void prepare_hub(const RunArgs& r, const Layout& L, const uint64_t* csc, IsectArgs& ia) {
    HubTab* hub = hub_tab(r, L);
    if (!hub) return;
    char* ws = (char*)r.ws;
    uint16_t* col16 = (uint16_t*)(csc == (const uint64_t*)(ws + L.keysA) ? ws + L.keysB : ws + L.keysA);
    ia.groups = groups_usable(r);
    ia.waves = (uint32_t)r.n <= WV_RANKS;
    ia.first_rank = ia.groups ? grp_first((uint32_t)r.n) : 0u;
    hipLaunchKernelGGL(k_hub_ranges, dim3(1), dim3(NBUCKET), 0, r.stream, ia.ctrl, (const uint32_t*)(ws + L.tstart),
                       (const uint8_t*)(ws + L.vbucket), ia.inoff, ia.first_rank,
                       ia.groups ? (uint32_t)isect_group_blocks() : 0u, ia.waves ? 1 : 0, hub);
    hipLaunchKernelGGL(k_col16, dim3(grid_for((size_t)r.E / 8 + 1)), dim3(NT), 0, r.stream, ia.col, ia.ctrl,
                       hub_first((uint32_t)r.n), hub, col16);
    ia.col16 = col16;
    ia.hub = hub;
}

hipError_t launch_isect_stage(const RunArgs& r, hipEvent_t* ev) {
    const Layout L = make_layout(r.E, r.n);
    uint64_t* csc = csc_of(r, L);
    IsectArgs ia = isect_args(r, L, csc);
    prepare_hub(r, L, csc, ia);
    uint64_t* partials = (uint64_t*)((char*)r.ws + L.isect_partials);
    const int order[NKERNEL] = {KER_MERGE, KER_BSEARCH, KER_BITMAP};
    reset_tile_counters(ia.ctrl, r.stream);
    IsectParts parts;
    if (ev) (void)hipEventRecord(ev[0], r.stream);
    for (int q = 0; q < NKERNEL; ++q) {
        const int k = order[q];
        launch_isect(k, ia, r.grid_override ? r.grid_override[k] : 0, partials, r.stream, &parts);
        if (ev) (void)hipEventRecord(ev[1 + q], r.stream);
    }
    launch_reduce_total(partials, parts, ia.ctrl, nullptr, 0, 0, r.stream);
    return hipGetLastError();
}

hipError_t run_list_pass(const RunArgs& r) {
    const Layout L = make_layout(r.E, r.n);
    const IsectArgs ia = isect_args(r, L, csc_of(r, L));
    uint64_t* partials = (uint64_t*)((char*)r.ws + L.isect_partials);
    reset_tile_counters(ia.ctrl, r.stream);
    for (int k = 0; k < NKERNEL; ++k) launch_isect(k, ia, r.grid_override ? r.grid_override[k] : 0, partials, r.stream);
    return hipGetLastError();
}

__global__ __launch_bounds__(NT) void k_widen(const uint32_t* __restrict__ in, uint64_t* __restrict__ out,
                                              const Ctrl* ctrl) {
    const uint32_t m = ctrl->m;
    for (uint64_t i = (uint64_t)blockIdx.x * NT + threadIdx.x; i < m; i += (uint64_t)gridDim.x * NT) out[i] = in[i];
}

void widen_u32_u64(const uint32_t* in, uint64_t* out, const Ctrl* ctrl, size_t cap, hipStream_t s) {
    hipLaunchKernelGGL(k_widen, dim3(grid_for(cap)), dim3(NT), 0, s, in, out, ctrl);
}

size_t sym_extra_bytes(int64_t E, int32_t n) {
    return align_up(4 * ((size_t)n + 1), 256) + align_up(8 * ((size_t)E > 0 ? (size_t)E : 1), 256);
}

size_t list_extra_bytes(int64_t E) {
    return align_up(8 * ((size_t)E + 1), 256) + align_up(4 * ((size_t)E > 0 ? (size_t)E : 1), 256);
}

hipError_t launch_isect_range(const RunArgs& r, int ker, uint32_t t0, uint32_t t1) {
    const Layout L = make_layout(r.E, r.n);
    IsectArgs ia = isect_args(r, L, csc_of(r, L));
    hipLaunchKernelGGL(k_set_tile_range, dim3(1), dim3(64), 0, r.stream, ia.ctrl, ker, t0, t1);   // zeroes the counter
    launch_isect(ker, ia, r.grid_override ? r.grid_override[ker] : 0, (uint64_t*)((char*)r.ws + L.isect_partials),
                 r.stream);
    return hipGetLastError();
}

void select_buckets(const RunArgs& r, Ctrl* ctrl, HubTab* hub) {
    hipStream_t s = r.stream;
    const bool learned = !r.given && r.select == SEL_LEARNED && r.mlp && r.learned;
    const bool learned_tile = learned && r.mlp_tile && r.learned_tile;
    if (learned) mlp_select((const MlpCompute*)r.mlp, ctrl, r.learned, s);
    if (learned_tile) mlp_select((const MlpCompute*)r.mlp_tile, ctrl, r.learned_tile, s);
    hipLaunchKernelGGL(k_select, dim3(1), dim3(NBUCKET), 0, s, ctrl, r.given ? (int)SEL_LEARNED : r.select,
                       r.given ? r.given : (learned ? r.learned : nullptr), learned_tile ? r.learned_tile : nullptr,
                       r.chunk_override, r.group_override, r.formulation != FORM_FILTERED ? 1 : 0, learned ? 0 : 1, hub);
}

hipError_t run_pipeline(const RunArgs& r, RunResult* out) {
    hipStream_t s = r.stream;
    char* ws = (char*)r.ws;
    const Layout L = make_layout(r.E, r.n);
    const int64_t E = r.E;
    const int32_t n = r.n;
    Ctrl* ctrl = (Ctrl*)(ws + L.ctrl);
    uint32_t* deg = (uint32_t*)(ws + L.deg);
    uint32_t* rank = (uint32_t*)(ws + L.rank);
    uint32_t* inv = (uint32_t*)(ws + L.inv);
    uint8_t* vbucket = (uint8_t*)(ws + L.vbucket);
    uint32_t* vlist = (uint32_t*)(ws + L.vlist);
    uint32_t* tstart = (uint32_t*)(ws + L.tstart);
    uint32_t* off = (uint32_t*)(ws + L.off);
    uint32_t* inoff = (uint32_t*)(ws + L.inoff);
    uint32_t* rowend = (uint32_t*)(ws + L.rowend);
    uint64_t* pv = (uint64_t*)(ws + L.pv);
    uint64_t* vkeysA = (uint64_t*)(ws + L.vkeysA);
    uint64_t* vkeysB = (uint64_t*)(ws + L.vkeysB);
    uint64_t* keysA = (uint64_t*)(ws + L.keysA);
    uint64_t* keysB = (uint64_t*)(ws + L.keysB);
    uint32_t* col = (uint32_t*)(ws + L.col);
    uint32_t* src = (uint32_t*)(ws + L.src);
    uint4* tiles = (uint4*)(ws + L.tiles);
    uint32_t* partial = (uint32_t*)(ws + L.partial);
    void* scan_tmp = ws + L.scan_tmp;
    void* radix_tmp = ws + L.radix_tmp;
    const int2* edges = (const int2*)r.edges;
    const size_t kcap = (size_t)(E > n ? E : n);

    auto mark = [&](int stage) {
        if (r.events) (void)hipEventRecord(r.events[stage], s);
    };
    mark(0);
    // ---- degree: input pairs per vertex, from the sorted endpoints
    fill_u32((uint32_t*)ctrl, 0u, sizeof(Ctrl) / 4, s);
    // bucket width: one partition pass of at most 8 bits up to 25-bit ids (buckets
    // of 2^17 vertices counted in four parts at 25 bits), two (buckets of 2^14) up to 27 bits
    const int vbits = bits_for((uint64_t)n);               // vertex ids fit in vbits bits
    const bool orient_part = vbits >= ORIENT_PART_MIN_BITS;
    uint32_t* p1_counts = nullptr;   // the orientation's first partition pass, counted by k_endpoints
    uint32_t p1_f = 1;
    // and the digit totals of its second pass, which with 8192-key tiles (2^25 pairs or more)
    // then looks back instead of running a histogram pass
    uint32_t* p2_tot =
        orient_part && radix_tile_keys((size_t)E, 8) == 8192u ? (uint32_t*)(ws + L.lb_aux) : nullptr;
    const int bw = vbits <= 20 ? (vbits < 12 ? vbits : 12) : (vbits <= 24 ? vbits - 8 : (vbits == 25 ? 16 : DEG_MAX_BW));
    const bool bucketed = vbits - bw <= DEG_MAX_BUCKET_BITS;
    uint32_t nsent_blocks = 0;   // blocks of k_endpoints that recorded sentinel endpoints
    {
        uint32_t* ep = (uint32_t*)keysA;       // 2E uint32 fit in E uint64
        uint32_t* ep_alt = (uint32_t*)keysB;
        // the endpoint sort's first digit is counted by k_endpoints as it writes the keys
        // one partition pass is enough for most: it then reads the pairs itself and
        // k_endpoints only counts. Ids of 25 bits take 512 groups, so that the low half of an id
        // is enough there too (degree stage with 256 groups and whole ids against it: Chung-Lu of
        // 148 million pairs 2.37 and 1.93 ms, R-MAT of 160 million 2.19 and 1.84)
        const bool direct = bucketed && vbits > bw && vbits - bw <= 9;
        const uint32_t ep_digits = 1u << (vbits - bw);
        const uint32_t ep_tile = direct ? endpoint_tile((size_t)(2 * E), ep_digits) : radix_tile_keys((size_t)(2 * E), 4);
        const uint32_t ep_tiles = (uint32_t)(((uint64_t)(2 * E) + ep_tile - 1) / ep_tile);
        const bool ep_sort = !bucketed || vbits > bw;
        const RadixDigit ep_dg = direct ? RadixDigit{bw, ep_digits - 1u} : bucketed ? radix_first_digit(bw, vbits) : radix_first_digit(0, bits_for((uint64_t)n + 1));
        // past 2^21 vertices the orientation's first partition pass (pairs by the high bits
        // of the first id) takes its digit counts from here too, kept in the column array
        // until then; its tiles hold one or two endpoint tiles' pairs
        const uint32_t pt_pairs = radix_tile_keys((size_t)E, 8);
        const uint64_t pt_tiles = ((uint64_t)E + pt_pairs - 1) / pt_pairs;
        if (orient_part && pt_pairs % (ep_tile / 2) == 0 && pt_pairs / (ep_tile / 2) <= 2 &&
            256u * (pt_tiles + 1) <= (uint64_t)E) {   // the count table fits the column array
            p1_counts = col;
            p1_f = pt_pairs / (ep_tile / 2);
        }
        const uint32_t p1_tiles = (ep_tiles + p1_f - 1) / p1_f;
        const unsigned eg = clearing_grid(p1_tiles, bucketed ? n : 0, DEG_EP_BLOCKS);
        if (p2_tot) fill_u32(p2_tot, 0u, 256, s);
        const bool fold = direct && p1_counts;
        hipLaunchKernelGGL((ep_digits > 256u && direct ? (fold ? k_endpoints<512, true> : k_endpoints<512, false>)
                                                       : (fold ? k_endpoints<256, true> : k_endpoints<256, false>)),
                           dim3(eg), dim3(NT), 0, s,
                           edges, (uint64_t)E, n,
                           bucketed ? (uint32_t)(n - 1) : (uint32_t)n, direct ? nullptr : ep, ctrl, partial,
                           ep_sort ? radix_first_counts(radix_tmp) : nullptr, ep_tiles, ep_tile, ep_dg, p1_counts,
                           p1_f, RadixDigit{vbits - ORIENT_PART_BITS, (1u << ORIENT_PART_BITS) - 1u}, p2_tot,
                           bucketed ? deg : nullptr);
        if (direct) {
            const uint32_t* tot = partition_endpoints(edges, (size_t)E, n, (uint32_t)(n - 1), ep_dg, (uint16_t*)ep,
                                                      radix_tmp, s);
            launch_bucket_count((const uint16_t*)ep, tot, bw, ep_digits, (uint64_t)(2 * E), n, deg, s);
            nsent_blocks = eg;
        } else if (bucketed) {
            // partition by bits [bw, vbits), then count per bucket
            const uint32_t nb = 1u << (vbits - bw);
            int a0 = 0;
            if (vbits > bw)
                a0 = radix_sort_u32(ep, ep_alt, nullptr, nullptr, nullptr, (size_t)(2 * E), bw, vbits, radix_tmp, s,
                                    true, true, &ctrl->err);   // a grouping: the order inside a bucket is free
            const uint32_t* tot = nullptr;   // one bucket: no partition
            if (vbits - bw > 8) {
                uint32_t* sizes = (uint32_t*)(ws + L.bstart);
                hipLaunchKernelGGL(k_bucket_sizes, dim3(grid_for((size_t)nb)), dim3(NT), 0, s, a0 ? ep_alt : ep,
                                   (uint32_t)(2 * E), bw, nb, sizes);
                tot = sizes;
            }
            launch_bucket_count(a0 ? ep_alt : ep, tot, bw, nb, (uint64_t)(2 * E), n, deg, s);
            nsent_blocks = eg;
        } else {
            const int a0 = radix_sort_u32(ep, ep_alt, nullptr, nullptr, nullptr, (size_t)(2 * E), 0,
                                          bits_for((uint64_t)n + 1), radix_tmp, s, true, true,
                                          &ctrl->err);   // whole keys
            fill_u32(rowend, 0u, (size_t)n, s);
            hipLaunchKernelGGL(k_endpoint_bounds, dim3(grid_for((size_t)(2 * E))), dim3(NT), 0, s, a0 ? ep_alt : ep,
                               (uint64_t)(2 * E), n, rowend);
            scan_offsets_max_u32(rowend, deg, (size_t)n, scan_tmp, s);   // deg[] holds degree offsets
        }
    }
    mark(1);
    // Few pairs on many vertices: the digits of most vertex keys are alike, and a wave's adds to one counter
    // take a turn each (3 pairs on 2^24 vertices: 20 us in each of the two kernels that count them). Otherwise
    // looking for that costs more than it saves (R-MAT 16 with t[v] 427 -> 429 us).
    const bool alike = 2 * E < (int64_t)n;
    // ---- rank: sort (degree, id); degrees are below 2E + 1
    const Chunking uc = chunking((uint64_t)E);   // of the unique pass, whose counts k_rank clears
    {
        const uint32_t v_tile = radix_tile_keys((size_t)n, 8);
        const uint32_t v_tiles = (uint32_t)(((uint64_t)n + v_tile - 1) / v_tile);
        const dim3 vg(v_tiles < 16384u ? v_tiles : 16384u);
        int dbits = bits_for((uint64_t)2 * (uint64_t)E + 1);
        if (dbits > RANK_BITS) dbits = RANK_BITS;
        const RadixDigit v_dg = radix_first_digit(32, 32 + dbits);
        uint32_t* v_counts = radix_first_counts(radix_tmp);
        if (bucketed)
            hipLaunchKernelGGL((alike ? k_vertex_keys<false, true> : k_vertex_keys<false, false>), vg, dim3(NT), 0, s,
                               deg, n, partial, nsent_blocks, vkeysA, v_counts, v_tiles, v_tile, v_dg);
        else
            hipLaunchKernelGGL((alike ? k_vertex_keys<true, true> : k_vertex_keys<true, false>), vg, dim3(NT), 0, s,
                               deg, n, partial, 0u, vkeysA, v_counts, v_tiles, v_tile, v_dg);
        const int alt = radix_sort_u64(vkeysA, vkeysB, nullptr, nullptr, nullptr, (size_t)n, 32, 32 + dbits,
                                       radix_tmp, s, true, false, &ctrl->err);
        const dim3 rg(grid_for((size_t)n));
        if (bucketed)
            hipLaunchKernelGGL(k_rank<false>, rg, dim3(NT), 0, s, alt ? vkeysB : vkeysA, n, deg, rank, inv, rowend,
                               partial, uc.nblk + 1);
        else
            hipLaunchKernelGGL(k_rank<true>, rg, dim3(NT), 0, s, alt ? vkeysB : vkeysA, n, deg, rank, inv, rowend,
                               partial, uc.nblk + 1);
    }
    mark(2);
    // ---- orient
    const int nb = bits_for((uint64_t)n) > 0 ? bits_for((uint64_t)n) : 1;
    const uint64_t sentinel = (2 * nb >= 64) ? ~0ull : ((1ull << (2 * nb)) - 1ull);
    const uint32_t e_tile = radix_tile_keys((size_t)E, 8);
    const uint32_t e_tiles = (uint32_t)(((uint64_t)E + e_tile - 1) / e_tile);
    const bool part = orient_part;
    if (part) {
        // pairs by their first id's high bits, then by their second's (first id -> rank);
        // both passes only group the pairs for locality of the rank lookups
        const int ob = ORIENT_PART_BITS;
        radix_pass_u64((const uint64_t*)edges, keysB, (size_t)E, vbits - ob, ob, RadixXf{RX_NONE, nullptr, n, 0, 0},
                       radix_tmp, s, p1_counts, false);
        radix_pass_u64(keysB, keysA, (size_t)E, 32 + vbits - ob, ob, RadixXf{RX_RANK_LOW, rank, n, 0, 0}, radix_tmp,
                       s, nullptr, false, MoreTot{nullptr, 0, 0, 0, 0}, p2_tot, &ctrl->err);
    } else if (e_tile % (16 * NT) == 0)
        hipLaunchKernelGGL(k_orient<16>, dim3(e_tiles < 16384u ? e_tiles : 16384u), dim3(NT), 0, s, edges,
                           (uint64_t)E, n, rank, nb, sentinel, keysA, radix_first_counts(radix_tmp), e_tiles, e_tile,
                           radix_first_digit(nb, 2 * nb));
    else
        hipLaunchKernelGGL(k_orient<OR_U>, dim3(e_tiles < 16384u ? e_tiles : 16384u), dim3(NT), 0, s, edges,
                           (uint64_t)E, n, rank, nb, sentinel, keysA, radix_first_counts(radix_tmp), e_tiles, e_tile,
                           radix_first_digit(nb, 2 * nb));
    mark(3);
    // ---- sort oriented pairs: a radix sort on the lower rank (the row; its first
    // digit counted by k_orient or, past 2^21 vertices, taken by a first pass that
    // orients each pair as it loads it), then every row sorted on chip by the
    // higher rank. The row sort fixes the order inside a row, so the first pass
    // only partitions; the later ones are stable.
    int alt;
    if (part) {
        // the orienting pass's histogram also counts the digits of the passes after
        // it, so that those look back with no histogram pass of their own
        const int w0 = radix_digit_width(nb);
        const MoreTot rest = radix_sort_totals(radix_tmp, (size_t)E, 8, nb + w0, 2 * nb);
        radix_pass_u64(keysA, keysB, (size_t)E, nb, w0, RadixXf{RX_ORIENT, rank, n, nb, sentinel}, radix_tmp, s,
                       nullptr, false, rest);
        alt = 1 - radix_sort_u64(keysB, keysA, nullptr, nullptr, nullptr, (size_t)E, nb + w0, 2 * nb, radix_tmp, s,
                                 false, false, &ctrl->err, rest.n > 0);
    } else {
        alt = radix_sort_u64(keysA, keysB, nullptr, nullptr, nullptr, (size_t)E, nb, 2 * nb, radix_tmp, s, true,
                             true, &ctrl->err);
    }
    uint64_t* sorted = alt ? keysB : keysA;
    uint64_t* other = alt ? keysA : keysB;
    // the row sort also counts the kept (first of equal) keys per chunk of the unique pass
    sort_runs_u64(sorted, other, (size_t)E, nb, true, sentinel, partial, uc.chunk, s);
    mark(4);
    // ---- unique + CSR
    {
        const Chunking c = uc;
        scan_exclusive_sum_u32(partial, partial, (size_t)c.nblk + 1, scan_tmp, s);
        hipLaunchKernelGGL(k_unique_write, dim3(c.nblk), dim3(NT), 0, s, sorted, (uint64_t)E, sentinel, ctrl, c.chunk,
                           partial, c.nblk, nb, col, src, rowend);
        scan_offsets_max_u32(rowend, off, (size_t)n, scan_tmp, s);
    }
    mark(5);
    if (r.csr_rank) {   // CSR export only: stop after the induced subgraph
        hipLaunchKernelGGL(k_export_csr, dim3(grid_for(kcap)), dim3(NT), 0, s, rank, off, col, ctrl, n, r.csr_rank,
                           r.csr_off, r.csr_col);
        out->ctrl_dev = ctrl;
        return hipGetLastError();
    }
    const int nbv = bits_for((uint64_t)n);
    uint64_t* csc;
    const uint32_t* moff = off;   // offsets of the middle lists
    if (r.formulation == FORM_FILTERED) {
        // ---- CSC: in-edges with work grouped by v (the sorted pair keys are free now);
        // in-edge groups: ids 0 .. n - 1 (n - 1 = no work). Each in-edge carries its
        // own edge index and tail, so the order inside a group is free: the
        // sort's first pass only partitions.
        const CscPacking pk = csc_packing(E, n, groups_wanted(r));
        auto csc_keys = pk.fbit ? k_csc_keys<true> : k_csc_keys<false>;
        hipLaunchKernelGGL(csc_keys, dim3(clearing_grid(e_tiles, n, 16384u)), dim3(NT), 0, s, col, src, off,
                           ctrl, n, other, pk.sh, pk.lbits, pk.fbit ? grp_first((uint32_t)n) : 0u,
                           radix_first_counts(radix_tmp), e_tiles, e_tile, radix_first_digit(pk.sh, pk.sh + nbv),
                           rowend);
        const int alt2 = radix_sort_u64(other, sorted, nullptr, nullptr, &ctrl->m, (size_t)E, pk.sh, pk.sh + nbv,
                                        radix_tmp, s, true, true, &ctrl->err);
        // bounds and tail ranges in one pass, into the buffer the sort left free
        const uint64_t* ckeys = alt2 ? sorted : other;
        csc = alt2 ? other : sorted;
        hipLaunchKernelGGL(k_csc_finish, dim3(grid_for(((size_t)E + 1) / 2)), dim3(NT), 0, s, ckeys,
                           csc, ctrl, n, rowend, pk.sh, src, off, pk.ebits, pk.lbits, pk.fbit);
        scan_offsets_max_u32(rowend, inoff, (size_t)n, scan_tmp, s);
    } else {
        // ---- all in-edges grouped by v; the symmetric adjacency; the streamed ranges
        const int sh = bits_for((uint64_t)E) > 0 ? bits_for((uint64_t)E) : 1;
        hipLaunchKernelGGL(k_sym_keys, dim3(grid_for((size_t)E)), dim3(NT), 0, s, col, ctrl, other, sh);
        const int alt2 =
            radix_sort_u64(other, sorted, nullptr, nullptr, &ctrl->m, (size_t)E, sh, sh + nbv, radix_tmp, s, false,
                           false, &ctrl->err);
        csc = alt2 ? sorted : other;
        fill_u32(rowend, 0u, (size_t)n, s);
        hipLaunchKernelGGL(k_sym_bounds, dim3(grid_for((size_t)E)), dim3(NT), 0, s, csc, ctrl, rowend, sh);
        scan_offsets_max_u32(rowend, inoff, (size_t)n, scan_tmp, s);
        uint32_t* fo = sym_off(r, L);
        if (r.formulation != FORM_MATRIX_UPPER) {
            hipLaunchKernelGGL(k_sym_rows, dim3(grid_for((size_t)n + 1)), dim3(NT), 0, s, inoff, off, n, fo);
            moff = fo;
        }
        hipLaunchKernelGGL(k_sym_build, dim3(grid_for((size_t)E)), dim3(NT), 0, s, csc, ctrl, src, col, off, inoff,
                           sym_col(r, L), sh, r.formulation);
    }
    mark(6);
    // ---- buckets + selection
    const uint32_t* mcol = (r.formulation == FORM_FULL || r.formulation == FORM_MATRIX) ? sym_col(r, L) : col;
    hipLaunchKernelGGL(k_vbucket,
                       dim3(n < VB_SMALL ? grid_for((size_t)n)
                                         : (unsigned)std::min<int64_t>(((int64_t)n + VB_NT - 1) / VB_NT, VB_BLOCKS)),
                       dim3(n < VB_SMALL ? NT : VB_NT), 0, s, moff, mcol, inoff, n, vbucket,
                       ctrl);
    select_buckets(r, ctrl, hub_tab(r, L));
    mark(7);
    // ---- group: order vertices by (kernel, bucket); tiles
    {
        const uint32_t v_tile = radix_tile_keys((size_t)n, 8);
        const uint32_t v_tiles = (uint32_t)(((uint64_t)n + v_tile - 1) / v_tile);
        hipLaunchKernelGGL((alike ? k_vkeys_slot<true> : k_vkeys_slot<false>), dim3(v_tiles < 16384u ? v_tiles : 16384u),
                           dim3(NT), 0, s, vbucket, n, ctrl, vkeysA, radix_first_counts(radix_tmp), v_tiles, v_tile,
                           radix_first_digit(32, 40));
        const int a3 = radix_sort_u64(vkeysA, vkeysB, nullptr, nullptr, nullptr, (size_t)n, 32, 40, radix_tmp, s,
                                      true, false, &ctrl->err);
        hipLaunchKernelGGL(k_ntiles, dim3(grid_for((size_t)n)), dim3(NT), 0, s, a3 ? vkeysB : vkeysA, vlist, vbucket,
                           inoff, n, ctrl, tstart);
    }
    scan_exclusive_sum_u32(tstart, tstart, (size_t)n + 1, scan_tmp, s);
    hipLaunchKernelGGL(k_emit_tiles, dim3(grid_for((size_t)n)), dim3(NT), 0, s, vlist, vbucket, inoff, tstart, n,
                       ctrl, tiles, (uint64_t)L.tile_cap, hub_tab(r, L),
                       groups_usable(r) ? grp_first((uint32_t)n) : ~0u);
    if (r.per_edge_counts) fill_u32(r.per_edge_counts, 0u, (size_t)E, s);
    if (r.support) fill_u32(r.support, 0u, (size_t)E, s);
    if (r.per_vertex || r.per_middle || r.clustering) fill_u64(pv, 0ull, (size_t)n, s);
    IsectArgs ia = isect_args(r, L, csc);
    if (!r.stop_before_isect) prepare_hub(r, L, csc, ia);
    mark(8);
    if (r.stop_before_isect) {
        out->ctrl_dev = ctrl;
        return hipGetLastError();
    }
    // ---- intersections
    uint64_t* partials = (uint64_t*)(ws + L.isect_partials);
    const int order[NKERNEL] = {KER_MERGE, KER_BSEARCH, KER_BITMAP};
    IsectParts parts;
    for (int q = 0; q < NKERNEL; ++q) {
        const int k = order[q];
        launch_isect(k, ia, r.grid_override ? r.grid_override[k] : 0, partials, s, &parts);
        mark(9 + q);
    }
    launch_reduce_total(partials, parts, ctrl, r.result, r.range_status, r.internal_status, s);
    // ---- finish
    if (r.per_vertex)
        hipLaunchKernelGGL(k_map_pv, dim3(grid_for((size_t)n)), dim3(NT), 0, s, pv, inv, n, r.per_vertex);
    else if (r.per_middle)
        hipLaunchKernelGGL(k_map_pv, dim3(grid_for((size_t)n)), dim3(NT), 0, s, pv, inv, n, r.per_middle);
    if (r.clustering) {   // the degree offsets are dead by now: reuse them
        fill_u32(deg, 0u, (size_t)n, s);
        hipLaunchKernelGGL(k_row_last, dim3(n < LAST_FEW ? 128 : 512), dim3(LAST_NT), 0, s, off, col, n, deg);
        const unsigned g = grid_for((size_t)n, CL_MAX_BLOCKS);
        hipLaunchKernelGGL(k_clustering, dim3(g), dim3(NT), 0, s, pv, inv, off, inoff, deg, n, r.clustering,
                           partials);
        hipLaunchKernelGGL(k_sum_wedges, dim3(1), dim3(NT), 0, s, partials, g, ctrl);
    }
    if (r.per_edge_pairs)
        hipLaunchKernelGGL(k_map_edges, dim3(grid_for((size_t)E)), dim3(NT), 0, s, col, src, inv, ctrl,
                           (int2*)r.per_edge_pairs);
    mark(NSTAGE);
    out->ctrl_dev = ctrl;
    return hipGetLastError();
}

}  // namespace tcx
