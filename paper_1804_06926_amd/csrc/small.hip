// Counting small graphs on a bit matrix.
//
// The general pipeline is about 70 kernels; on a graph of a few thousand edges
// each lasts a few microseconds whatever its work, so a call is 300 us of launches. Up
// to SMALL_MAX_N vertices the adjacency matrix has 32 MB of bits at most, and
// no sort is needed at all:
//   build   each block owns a range of matrix rows: it reads the whole edge
//           list, sets the bits of its rows in LDS (repeated pairs and both
//           directions fall together) and writes the rows and, per row, the
//           list of its neighbours (v << 16 | u), at a place that the input degrees below the
//           range bound, so blocks need nothing from each other
//   count   waves take 32 consecutive neighbour pairs (v, u); |N(v) and N(u)| of the
//           edge is the set bits of row v AND row u, and its sum over a vertex's edges is
//           2 t[v]. The pairs of one v follow each other, so its sums gather in a
//           register. Wide rows are read once per edge, for u before v in (degree, id) order,
//           and count for u too: the end of lower degree, so no counter is hot
//   finish  t[v], T = sum t[v] / 3, clustering coefficients
// A synchronising call also reports statistics (tc_last_stats): the degree order by
// comparing every two vertices, the oriented degrees from the neighbour lists, then the
// pipeline's own bucket selection. A queued call has no use for them.
// Bound: latency (three launches queued, seven to nine with statistics, one wave's chain of loads each); at the largest
// sizes the rows read (0.5 GB for 16384 vertices and 131072 pairs, 48 us). Measured against
// the pipeline, queued / synchronous: Erdos-Renyi 4096 vertices, 32768 pairs 299 -> 28 /
// 335 -> 90 us; Chung-Lu 125 and 1000 171 -> 17 / 246 -> 80 us; uniform 16384 and
// 131072 324 -> 90 / 366 -> 189 us.
#include "common.h"
#include "internal.h"
#include "mlp.h"
#include "pipeline.h"
#include "tiles.h"

namespace tcx {

constexpr int SB_NT = 1024;            // build: threads per block
constexpr int SM_BLOCKS = 256;         // build: blocks, at most (16 * K rows each)
constexpr uint32_t SM_CHUNK = 32;      // count: neighbour pairs per wave and step
constexpr int SM_ID_BITS = 14;         // order key: input degree << 14 | id, in 32 bits
static_assert(SMALL_MAX_N <= 1 << SM_ID_BITS && SMALL_MAX_PAIRS < 1 << (32 - SM_ID_BITS), "order keys fit 32 bits");
constexpr int SF_NT = 1024;            // finish: threads (and vertices) per block
constexpr int SC_NT = 256;             // count: threads per block
constexpr int SR_V = 64;               // rank: vertices per block of SB_NT threads

// Matrix words (uint64) per row: a multiple of the wave, K per lane.
static int row_k(int32_t n) { return n <= 4096 ? 1 : (n <= 8192 ? 2 : 4); }

struct SmallLayout {
    size_t bits, pairs, seg, key, dsim, t2, rank, lo, hi, dplus, din, tiles, total;
};

static SmallLayout small_layout(int64_t E, int32_t n) {
    SmallLayout L;
    size_t o = align_up(sizeof(Ctrl), 256);   // the control block comes first, as in make_layout
    auto take = [&](size_t bytes) { size_t r = o; o = align_up(o + (bytes ? bytes : 1), 256); return r; };
    const size_t nn = (size_t)n;
    L.bits = take(nn * (size_t)row_k(n) * 512);
    L.pairs = take(8 * (size_t)E);
    L.seg = take(sizeof(uint2) * SM_BLOCKS);
    L.key = take(4 * nn);
    L.dsim = take(4 * nn);
    L.t2 = take(4 * nn);
    L.rank = take(4 * nn);
    L.lo = take(4 * nn);
    L.hi = take(4 * nn);
    L.dplus = take(4 * nn);
    L.din = take(4 * nn);
    L.tiles = take(4 * NBUCKET);
    L.total = o;
    return L;
}

// The matrix wins at every size measured up to these limits (the slowest, Chung-Lu
// of 16384 vertices and 131072 pairs, 96 us queued and 232 us with statistics against
// 354 and 399 us by the pipeline), so they are no crossover but what the layout holds: an order key
// of degree and id fits 32 bits up to 2^18 pairs, twice the vertices would take 128 MB of
// matrix, and every build block reads the whole edge list, 45 us at 131072 pairs.
bool small_graph(int64_t E, int32_t n) {
    return n >= 1 && n <= SMALL_MAX_N && E >= 1 && E <= SMALL_MAX_PAIRS;
}
size_t small_workspace(int64_t E, int32_t n) { return small_graph(E, n) ? small_layout(E, n).total : 0; }

// ------------------------------------------------------------------ build
// Block b owns rows [16 K b, 16 K (b + 1)). seg[b] = {first pair, pairs} of its
// neighbour lists. Block 0 clears the control block and reports bad ids.
template <int K>
__global__ __launch_bounds__(SB_NT) void k_small_build(const int2* __restrict__ edges, uint32_t E, int32_t n,
                                                       uint64_t* __restrict__ bits, uint32_t* __restrict__ pairs,
                                                       uint2* __restrict__ seg, uint32_t* __restrict__ key,
                                                       uint32_t* __restrict__ dsim, uint32_t* __restrict__ t2,
                                                       uint32_t* __restrict__ tiles, Ctrl* ctrl) {
    constexpr uint32_t R = 16u * K, W = 64u * K;   // rows, words per row
    __shared__ uint64_t s_row[R * W];
    __shared__ uint32_t s_deg[R], s_sim[R], s_at[R], s_below, s_bad;
    const uint32_t r0 = blockIdx.x * R;
    for (uint32_t i = threadIdx.x; i < R * W; i += SB_NT) s_row[i] = 0;
    if (threadIdx.x < R) s_deg[threadIdx.x] = 0;
    if (threadIdx.x == 0) { s_below = 0; s_bad = 0; }
    if (blockIdx.x == 0) {
        for (uint32_t i = threadIdx.x; i < sizeof(Ctrl) / 4; i += SB_NT) ((uint32_t*)ctrl)[i] = 0;
        if (threadIdx.x < NBUCKET) tiles[threadIdx.x] = 0;
    }
    __syncthreads();
    uint32_t below = 0;   // endpoints before this block's rows (of loops and bad pairs too: a bound on its place)
    uint32_t top = 0;     // highest id (negative ones wrap past every n)
    auto take = [&](uint32_t x, uint32_t y) {
        const uint32_t dx = x - r0, dy = y - r0;
        below += (x < r0 ? 1u : 0u) + (y < r0 ? 1u : 0u);
        top = max(top, max(x, y));
        if (min(dx, dy) < R && max(x, y) < (uint32_t)n && x != y) {
            if (dx < R) {
                atomicOr((uint32_t*)s_row + dx * (2u * W) + (y >> 5), 1u << (y & 31u));
                atomicAdd(&s_deg[dx], 1u);
            }
            if (dy < R) {
                atomicOr((uint32_t*)s_row + dy * (2u * W) + (x >> 5), 1u << (x & 31u));
                atomicAdd(&s_deg[dy], 1u);
            }
        }
    };
    constexpr uint32_t U = 8;
    uint32_t i0 = 0;
    for (; i0 + SB_NT * U <= E; i0 += SB_NT * U) {   // whole rounds, a round's loads in flight together
        int2 ed[U];
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) ed[k] = edges[i0 + k * SB_NT + threadIdx.x];
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) take((uint32_t)ed[k].x, (uint32_t)ed[k].y);
    }
    {
        int2 ed[U];
#pragma unroll
        for (uint32_t k = 0; k < U; ++k) {
            const uint32_t i = i0 + k * SB_NT + threadIdx.x;
            ed[k] = edges[i < E ? i : E - 1u];
        }
#pragma unroll
        for (uint32_t k = 0; k < U; ++k)
            if (i0 + k * SB_NT + threadIdx.x < E) take((uint32_t)ed[k].x, (uint32_t)ed[k].y);
    }
    const bool bad = top >= (uint32_t)n;
    below = wave_sum(below);
    if (lane_id() == 0 && below) atomicAdd(&s_below, below);
    if (__ballot(bad) && lane_id() == 0) s_bad = 1;
    __syncthreads();
    const uint32_t wv = (uint32_t)wave_id(), ln = (uint32_t)lane_id();
    for (uint32_t r = wv; r < R; r += SB_NT / WAVE) {
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            const uint64_t w = s_row[r * W + k * WAVE + ln];
            if (r0 + r < (uint32_t)n) bits[(size_t)(r0 + r) * W + k * WAVE + ln] = w;
            c += (uint32_t)__popcll(w);
        }
        c = wave_sum(c);
        if (ln == 0) s_sim[r] = c;
    }
    __syncthreads();
    if (wv == 0) {   // R <= 64 rows: one wave scans their sizes
        const uint32_t c = ln < R ? s_sim[ln] : 0u;
        const uint32_t inc = wave_inclusive_scan(c);
        if (ln < R) s_at[ln] = s_below + inc - c;
        if (ln == WAVE - 1) seg[blockIdx.x] = make_uint2(s_below, inc);
    }
    if (threadIdx.x < R && r0 + threadIdx.x < (uint32_t)n) {
        key[r0 + threadIdx.x] = s_deg[threadIdx.x] << SM_ID_BITS | (r0 + threadIdx.x);
        dsim[r0 + threadIdx.x] = s_sim[threadIdx.x];
        t2[r0 + threadIdx.x] = 0;
    }
    if (blockIdx.x == 0 && threadIdx.x == 0) ctrl->err = s_bad;
    __syncthreads();
    for (uint32_t r = wv; r < R; r += SB_NT / WAVE) {
        uint64_t w[K];
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            w[k] = s_row[r * W + k * WAVE + ln];
            c += (uint32_t)__popcll(w[k]);
        }
        uint32_t at = s_at[r] + wave_inclusive_scan(c) - c;
#pragma unroll
        for (int k = 0; k < K; ++k)
            while (w[k]) {
                const uint32_t b = (uint32_t)__ffsll((unsigned long long)w[k]) - 1u;
                w[k] &= w[k] - 1ull;
                pairs[at++] = (r0 + r) << 16 | (k * WAVE + ln) * 64u + b;
            }
    }
}

// ------------------------------------------------------------------ count
// Per edge (v, u), u before v: c = |N(v) and N(u)| added to t2[v] and t2[u].
template <int K>
__global__ __launch_bounds__(SC_NT) void k_small_count(const uint64_t* __restrict__ bits,
                                                       const uint32_t* __restrict__ pairs,
                                                       const uint2* __restrict__ seg, uint32_t nseg,
                                                       const uint32_t* __restrict__ key, uint32_t* __restrict__ t2) {
    static_assert(SM_BLOCKS <= SC_NT && SM_CHUNK <= WAVE, "one segment per thread, at most one pair per lane");
    constexpr uint32_t W = 64u * K;
    constexpr int U = K == 4 ? 4 : 8;   // edges whose rows are in flight together
    // Rows of 512 bytes are cheap to read twice, so there both (v, u) and (u, v) count for
    // their first vertex alone and no sum per edge is needed (4096 vertices, 32768 pairs: 9.9 against
    // 12.4 us); wider rows are read once per edge (16384 vertices, 131072 pairs: 48 against 79 us).
    constexpr bool ONCE = K > 1;
    __shared__ uint32_t s_pref[SM_BLOCKS + 1], scratch[SC_NT / WAVE];
    __shared__ uint2 s_seg[SM_BLOCKS];
    const uint2 sg = threadIdx.x < nseg ? seg[threadIdx.x] : make_uint2(0, 0);
    uint32_t chunks;
    const uint32_t ex = block_exclusive_scan<SC_NT>((sg.y + SM_CHUNK - 1) / SM_CHUNK, scratch, &chunks);
    s_seg[threadIdx.x] = sg;
    s_pref[threadIdx.x] = ex;
    __syncthreads();
    const uint32_t ln = (uint32_t)lane_id();
    for (uint32_t c = blockIdx.x * (SC_NT / WAVE) + (uint32_t)wave_id(); c < chunks; c += gridDim.x * (SC_NT / WAVE)) {
        uint32_t s = 0;   // the last segment whose first chunk is at most c
#pragma unroll
        for (uint32_t step = SM_BLOCKS / 2; step > 0; step >>= 1)
            if (s_pref[s + step] <= c) s += step;
        const uint32_t p = (c - s_pref[s]) * SM_CHUNK;
        const bool on = ln < SM_CHUNK && p + ln < s_seg[s].y;
        const uint32_t mine = on ? pairs[s_seg[s].x + p + ln] : 0u;
        const bool keep = on && (!ONCE || key[mine & 0xFFFFu] < key[mine >> 16]);
        uint64_t M = __ballot(keep);   // uniform: scalar from here on
        uint32_t v = 0, acc = 0;       // this lane's part of the sum of v's edges so far
        while (M) {
            uint32_t q[U], x[U], got = 0;
            uint64_t a[U][K], b[U][K];
#pragma unroll
            for (int j = 0; j < U; ++j) {   // past the last one: its rows again, dropped below
                if (M) {
                    q[j] = __builtin_amdgcn_readlane(mine, __ffsll((unsigned long long)M) - 1);
                    M &= M - 1ull;
                    ++got;
                } else {
                    q[j] = q[j > 0 ? j - 1 : 0];
                }
#pragma unroll
                for (int i = 0; i < K; ++i) {
                    a[j][i] = bits[(size_t)(q[j] >> 16) * W + i * WAVE + ln];
                    b[j][i] = bits[(size_t)(q[j] & 0xFFFFu) * W + i * WAVE + ln];
                }
            }
            uint32_t any = 0;
#pragma unroll
            for (int j = 0; j < U; ++j) {
                x[j] = 0;
#pragma unroll
                for (int i = 0; i < K; ++i) x[j] += (uint32_t)__popcll(a[j][i] & b[j][i]);
                if ((uint32_t)j >= got) x[j] = 0;
                any |= x[j];
            }
            if (!__ballot(any != 0)) continue;   // no triangle on any of these edges
#pragma unroll
            for (int j = 0; j < U; ++j) {
                if (q[j] >> 16 != v) {   // v's list ends here
                    acc = wave_sum(acc);
                    if (ln == 0 && acc) atomicAdd(&t2[v], acc);
                    v = q[j] >> 16;
                    acc = 0;
                }
                acc += x[j];
            }
            if (!ONCE) continue;
            // the U sums over the wave at once: each step halves the values a lane holds, so that
            // lane group g (of WAVE / U lanes) ends up with the sum of edge g
            uint32_t mu = 0;   // this group's u
#pragma unroll
            for (int j = 0; j < U; ++j)
                if (ln / (WAVE / U) == (uint32_t)j) mu = q[j] & 0xFFFFu;
#pragma unroll
            for (int h = U / 2, o = WAVE / 2; h > 0; h >>= 1, o >>= 1) {
                const bool up = (ln & (uint32_t)o) != 0;
#pragma unroll
                for (int i = 0; i < h; ++i) {
                    const uint32_t send = up ? x[i] : x[i + h];
                    x[i] = (up ? x[i + h] : x[i]) + __shfl_xor(send, o, WAVE);
                }
            }
#pragma unroll
            for (int o = WAVE / U / 2; o > 0; o >>= 1) x[0] += __shfl_xor(x[0], o, WAVE);
            if (ln % (WAVE / U) == 0 && x[0]) atomicAdd(&t2[mu], x[0]);
        }
        acc = wave_sum(acc);
        if (ln == 0 && acc) atomicAdd(&t2[v], acc);
    }
}

// ------------------------------------------------------------------ statistics
// rank[v] = vertices before v in (input degree, id) order. Thread: one vertex
// against 1/16 of all of them (a wave shares its range, so the keys come by scalar loads).
__global__ __launch_bounds__(SB_NT) void k_small_rank(const uint32_t* __restrict__ key, uint32_t n,
                                                      uint32_t* __restrict__ rank) {
    __shared__ uint32_t s_cnt[SR_V];
    if (threadIdx.x < SR_V) s_cnt[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t v = blockIdx.x * SR_V + (uint32_t)lane_id(), parts = SB_NT / WAVE, part = (uint32_t)wave_id();
    const uint32_t kv = v < n ? key[v] : 0u;
    const uint32_t u0 = n * part / parts, u1 = n * (part + 1u) / parts;
    uint32_t c = 0;
#pragma unroll 16
    for (uint32_t u = u0; u < u1; ++u) c += key[u] < kv ? 1u : 0u;
    atomicAdd(&s_cnt[lane_id()], c);
    __syncthreads();
    if (threadIdx.x < SR_V && v < n) rank[v] = s_cnt[threadIdx.x];
}

// Per vertex v: out-degree, lowest and highest rank among the neighbours after v. One wave per vertex.
template <int K>
__global__ __launch_bounds__(256) void k_small_orient(const uint64_t* __restrict__ bits,
                                                      const uint32_t* __restrict__ rank, uint32_t n,
                                                      uint32_t* __restrict__ dplus, uint32_t* __restrict__ lo,
                                                      uint32_t* __restrict__ hi) {
    const uint32_t v = blockIdx.x * 4u + (uint32_t)wave_id(), ln = (uint32_t)lane_id();
    if (v >= n) return;
    const uint32_t rv = rank[v];
    uint32_t c = 0, l = ~0u, h = 0;
#pragma unroll
    for (int k = 0; k < K; ++k) {
        uint64_t w = bits[(size_t)v * (64u * K) + k * WAVE + ln];
        while (w) {
            const uint32_t u = (k * WAVE + ln) * 64u + (uint32_t)__ffsll((unsigned long long)w) - 1u;
            w &= w - 1ull;
            const uint32_t ru = rank[u];
            if (ru > rv) {
                ++c;
                l = ru < l ? ru : l;
                h = ru > h ? ru : h;
            }
        }
    }
    c = wave_sum(c);
#pragma unroll
    for (int o = WAVE / 2; o > 0; o >>= 1) {
        const uint32_t l2 = __shfl_xor(l, o, WAVE), h2 = __shfl_xor(h, o, WAVE);
        l = l2 < l ? l2 : l;
        h = h2 > h ? h2 : h;
    }
    if (ln == 0) {
        dplus[v] = c;
        lo[v] = l;
        hi[v] = h;
    }
}

// Per vertex v: in-edges with work (v is not the last of the row), its bucket's statistics.
template <int K>
__global__ __launch_bounds__(SB_NT) void k_small_buckets(const uint64_t* __restrict__ bits,
                                                         const uint32_t* __restrict__ rank,
                                                         const uint32_t* __restrict__ dplus,
                                                         const uint32_t* __restrict__ lo,
                                                         const uint32_t* __restrict__ hi, uint32_t n,
                                                         uint32_t* __restrict__ din, Ctrl* ctrl) {
    __shared__ BucketSums S;
    S.clear(SB_NT);
    __syncthreads();
    const uint32_t ln = (uint32_t)lane_id(), waves = SB_NT / WAVE;
    for (uint32_t v = blockIdx.x * waves + (uint32_t)wave_id(); v < n; v += gridDim.x * waves) {
        const uint32_t rv = rank[v];
        uint32_t c = 0;
#pragma unroll
        for (int k = 0; k < K; ++k) {
            uint64_t w = bits[(size_t)v * (64u * K) + k * WAVE + ln];
            while (w) {
                const uint32_t u = (k * WAVE + ln) * 64u + (uint32_t)__ffsll((unsigned long long)w) - 1u;
                w &= w - 1ull;
                c += (rank[u] < rv && hi[u] != rv) ? 1u : 0u;
            }
        }
        c = wave_sum(c);
        if (ln == 0) {
            din[v] = c;
            S.add(c, dplus[v], lo[v], hi[v]);
        }
    }
    __syncthreads();
    S.flush(ctrl, SB_NT);
}

// ------------------------------------------------------------------ finish
// T, m, and the optional outputs; with stats, the tiles the selection stands
// for (the same counts as the tile layout gives). A vertex per thread; blocks
// add their sums to the control block (cleared by the build), and the
// last one to do so (a ticket; nobody waits) writes the results.
__global__ __launch_bounds__(SF_NT) void k_small_finish(const uint32_t* __restrict__ t2,
                                                        const uint32_t* __restrict__ dsim,
                                                        const uint2* __restrict__ seg, uint32_t nseg, uint32_t n,
                                                        const uint32_t* __restrict__ din,
                                                        const uint32_t* __restrict__ dplus, int stats,
                                                        uint64_t* __restrict__ per_vertex, double* __restrict__ coeff,
                                                        uint64_t* __restrict__ result, uint64_t range_status,
                                                        uint32_t* __restrict__ tiles, Ctrl* ctrl) {
    __shared__ uint64_t s_t[SF_NT / WAVE], s_w[SF_NT / WAVE];
    __shared__ uint32_t s_m, s_tiles[NBUCKET], s_ker[NKERNEL], s_last;
    if (threadIdx.x == 0) s_m = 0;
    if (threadIdx.x < NBUCKET) s_tiles[threadIdx.x] = 0;
    if (threadIdx.x < NKERNEL) s_ker[threadIdx.x] = 0;
    __syncthreads();
    const uint32_t v = blockIdx.x * SF_NT + threadIdx.x;
    uint64_t t = 0, w = 0;
    if (v < n) {
        t = t2[v] / 2u;
        if (per_vertex) per_vertex[v] = t;
        if (coeff) {
            const uint64_t d = dsim[v];
            w = d < 2 ? 0ull : d * (d - 1) / 2;
            coeff[v] = w ? (double)t / (double)w : 0.0;
        }
        if (stats) {
            const uint32_t b = bucket_of(din[v], dplus[v]);
            if (b != (uint32_t)BUCKET_NONE && tile_group(ctrl, b) == 1u)
                atomicAdd(&s_tiles[b], (din[v] + ctrl->chunk[b] - 1u) / ctrl->chunk[b]);
        }
    }
    t = wave_sum_u64(t);
    w = wave_sum_u64(w);
    if (lane_id() == 0) {
        s_t[wave_id()] = t;
        s_w[wave_id()] = w;
    }
    __syncthreads();
    // tiles: of the single-vertex buckets (cleared by the build)
    // The sums meet in device-scope atomics alone, and each is complete (its old value has come
    // back) before the barrier ahead of the ticket, so no cache has to be written back.
    uint32_t seen = 0;
    if (stats && threadIdx.x < NBUCKET && s_tiles[threadIdx.x])
        seen |= atomicAdd(&tiles[threadIdx.x], s_tiles[threadIdx.x]);
    if (threadIdx.x == 0) {
        uint64_t T = 0, Wd = 0;
        for (int i = 0; i < SF_NT / WAVE; ++i) {
            T += s_t[i];
            Wd += s_w[i];
        }
        // 3T until the end
        if (T) seen |= (uint32_t)atomicAdd((unsigned long long*)&ctrl->total, (unsigned long long)T);
        if (Wd) seen |= (uint32_t)atomicAdd((unsigned long long*)&ctrl->wedges, (unsigned long long)Wd);
    }
    if (threadIdx.x < NBUCKET) s_tiles[threadIdx.x] = seen;   // waits for the old values
    __syncthreads();
    if (threadIdx.x == 0) s_last = atomicAdd(&ctrl->pad0, 1u) == gridDim.x - 1u ? 1u : 0u;
    __syncthreads();
    if (!s_last) return;
    if (threadIdx.x < nseg) atomicAdd(&s_m, seg[threadIdx.x].y);
    if (stats && threadIdx.x < (unsigned)BUCKET_NONE && ctrl->bucket_nv[threadIdx.x]) {
        const uint32_t b = threadIdx.x, g = tile_group(ctrl, b);
        atomicAdd(&s_ker[ctrl->choice[b]],
                  g == 1u ? atomicAdd(&tiles[b], 0u) : (ctrl->bucket_nv[b] + g - 1u) / g);
    }
    __syncthreads();
    if (threadIdx.x == 0) {
        const uint64_t T = atomicAdd((unsigned long long*)&ctrl->total, 0ull) / 3ull;
        ctrl->total = T;
        ctrl->m = s_m / 2u;
        if (result) {
            result[0] = T;
            result[1] = ctrl->err ? range_status : 0ull;
        }
        uint32_t at = 0;
        for (int k = 0; k < NKERNEL; ++k) {
            ctrl->tile_begin[k] = at;
            at += s_ker[k];
        }
        ctrl->tile_begin[NKERNEL] = at;
        ctrl->ntiles = at;
    }
}

// ------------------------------------------------------------------ launcher
template <int K>
static void run_k(const RunArgs& r, const SmallLayout& L) {
    const bool stats = !r.result;   // a queued call has no use for them
    char* ws = (char*)r.ws;
    hipStream_t s = r.stream;
    Ctrl* ctrl = (Ctrl*)ws;
    uint64_t* bits = (uint64_t*)(ws + L.bits);
    uint32_t* pairs = (uint32_t*)(ws + L.pairs);
    uint2* seg = (uint2*)(ws + L.seg);
    uint32_t *key = (uint32_t*)(ws + L.key), *dsim = (uint32_t*)(ws + L.dsim), *t2 = (uint32_t*)(ws + L.t2),
             *rank = (uint32_t*)(ws + L.rank), *lo = (uint32_t*)(ws + L.lo), *hi = (uint32_t*)(ws + L.hi),
             *dplus = (uint32_t*)(ws + L.dplus), *din = (uint32_t*)(ws + L.din), *tiles = (uint32_t*)(ws + L.tiles);
    const uint32_t n = (uint32_t)r.n, nblk = (n + 16u * K - 1) / (16u * K);
    static_assert(SMALL_MAX_N / (16 * 4) <= SM_BLOCKS && 8192 / (16 * 2) <= SM_BLOCKS && 4096 / 16 <= SM_BLOCKS,
                  "a segment per build block");
    hipLaunchKernelGGL(k_small_build<K>, dim3(nblk), dim3(SB_NT), 0, s, (const int2*)r.edges, (uint32_t)r.E, r.n, bits,
                       pairs, seg, key, dsim, t2, tiles, ctrl);
    // at most 2E pairs, and one short chunk per segment
    const uint64_t chunks = 2ull * (uint64_t)r.E / SM_CHUNK + nblk;
    const unsigned grid = (unsigned)((chunks + SC_NT / WAVE - 1) / (SC_NT / WAVE));
    hipLaunchKernelGGL(k_small_count<K>, dim3(grid < 2048u ? grid : 2048u), dim3(SC_NT), 0, s, bits, pairs, seg, nblk,
                       key, t2);
    if (stats) {
        hipLaunchKernelGGL(k_small_rank, dim3((n + SR_V - 1) / SR_V), dim3(SB_NT), 0, s, key, n, rank);
        hipLaunchKernelGGL(k_small_orient<K>, dim3((n + 3) / 4), dim3(256), 0, s, bits, rank, n, dplus, lo, hi);
        hipLaunchKernelGGL(k_small_buckets<K>, dim3(n < 4096u ? (n + 15) / 16 : 256u), dim3(SB_NT), 0, s, bits, rank,
                           dplus, lo, hi, n, din, ctrl);
        select_buckets(r, ctrl, nullptr);
    }
    hipLaunchKernelGGL(k_small_finish, dim3((n + SF_NT - 1) / SF_NT), dim3(SF_NT), 0, s, t2, dsim, seg, nblk, n, din, dplus, stats ? 1 : 0,
                       r.per_vertex, r.clustering, r.result, r.range_status, tiles, ctrl);
}

hipError_t run_small(const RunArgs& r, RunResult* out) {
    const SmallLayout L = small_layout(r.E, r.n);
    switch (row_k(r.n)) {
        case 1: run_k<1>(r, L); break;
        case 2: run_k<2>(r, L); break;
        default: run_k<4>(r, L); break;
    }
    out->ctrl_dev = (Ctrl*)r.ws;
    return hipGetLastError();
}

}  // namespace tcx
