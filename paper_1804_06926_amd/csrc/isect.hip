// Per-edge intersection kernels (Section 3.2, Algorithm 2 "Compute_Intersection";
// Section 4.2, dynamic grouping and the large/small neighbour-list kernels).
//
// The graph is the degree-ordered CSR over ranks: row u holds N+(u), the
// neighbours ranked above u, ascending. For a kept edge e = (u -> v) at
// position p of row u, a common neighbour w of N+(u) and N+(v) must rank above
// v, so only the tail of row u after p can match:
//     c_e = | row_u[p+1 ..] intersected with N+(v) |  =  | N+(u) intersected with N+(v) |.
// Work is grouped by the middle vertex v. A tile is either one vertex v with a
// chunk of its in-edges, or several vertices of one bucket with all their
// in-edges. Three interchangeable strategies compute the same c_e for every
// in-edge of a tile:
//   merge   : merge-path split of (tail, N+(v)) across a group of lanes
//   bsearch : binary search of each element of the shorter list in the other
//   bitmap  : N+(v) staged once per vertex as an LDS bitmap; all tails of the
//             tile streamed through it as one flat, coalesced item range
// Each hit adds 1 to the exact 64-bit triangle count; optional outputs are
// the per-edge counts c_e, the per-vertex counts t[u], t[v], t[w] and the
// edge support (triangles per edge: a hit w adds 1 to edges uv, uw and vw;
// uw is the tail element's own CSR position, vw the position of w in N+(v)).
// Block b starts with tile b; after that the blocks take tiles in order from a
// shared counter (one atomic per tile), so a block that drew light tiles takes
// more: tiles are ordered heaviest bucket first, which makes this a
// longest-first schedule. Blocks without a first tile exit at once (small
// graphs). The counter is zeroed before each launch (launch_isect callers).
// Each block writes its partial count and one reduction adds them in a fixed
// order; T does not depend on which block counted which tile (integer sums).
// A second pass of the same kernels writes the triangles themselves (listing).
// The same kernels serve the paper's other formulations (whole neighbour
// lists; the matrix formulation of Section 3.3): an entry's range is then a
// whole row that may reach below and above the middle list, and the bitmap
// kernel cuts it to each window it tests (clipped mode, counts only).
#include "common.h"
#include "internal.h"
#include "isect.h"

namespace tcx {

constexpr int IS_NT = 256;
constexpr int BM_WORDS = 4096;            // 131072-bit window (16 KiB)
constexpr uint32_t BM_BITS = BM_WORDS * 32u;
// The selector's window feature counts windows of this size from the lowest element up; the modes
// that only count take somewhat shorter ones, from the highest down.
static_assert(BM_BITS == (1u << BM_WINDOW_LOG2), "the selector's window feature counts windows of this size");
constexpr int UNROLL = 8;                 // bitmap kernel: tail loads in flight per lane
constexpr uint32_t WT_MAX = 1024;         // bitmap kernel: 64-item windows per chunk of the item range
constexpr uint32_t LONG_TAIL = 64;        // bitmap kernel: tails of at least one window are walked directly
constexpr int NV_MAX = 2048;              // bitmap kernel, support mode: longest N+(v) whose hits are gathered in LDS
constexpr int PARTIALS_PER_KERNEL = 4096; // max blocks per intersection launch

template <int N>
struct SegsT {
    uint32_t v[N];
    uint32_t e0[N];
    uint32_t pref[N + 1];
    uint32_t scratch[IS_NT / WAVE];
};
using Segs = SegsT<SEG_MAX>;

// The next tile for this block after its first (static) one: t0 + the shared
// counter ker, which is zero when the launch starts. Called by the
// whole block (barriers); the value is the same in every thread.
constexpr int HUB_COUNTER = NKERNEL, GRP_COUNTER = NKERNEL + 1;   // the hub and the group kernel's
__device__ __forceinline__ uint32_t grab_tile(Ctrl* ctrl, int ker, uint32_t t0, uint32_t* s_tile) {
    __syncthreads();   // every thread has read the previous value
    if (threadIdx.x == 0) *s_tile = t0 + atomicAdd(&ctrl->tile_next[ker], 1u);
    __syncthreads();
    return *s_tile;
}

// Tile i of a launch whose tiles are not contiguous: ranges of tiles (tile,
// pref of HubTab), i < pref[NBUCKET].
struct TileRanges {   // a copy in LDS, for the hub kernel
    uint32_t tile[NBUCKET], pref[NBUCKET + 1];
    // Whole block; a barrier follows before use.
    __device__ void load(const uint32_t* g_tile, const uint32_t* g_pref) {
        for (uint32_t i = threadIdx.x; i < (uint32_t)NBUCKET; i += blockDim.x) tile[i] = g_tile[i];
        for (uint32_t i = threadIdx.x; i <= (uint32_t)NBUCKET; i += blockDim.x) pref[i] = g_pref[i];
    }
    __device__ uint32_t at(uint32_t i) const {
        uint32_t r = 0;   // the last range whose prefix is at most i
#pragma unroll
        for (uint32_t step = NBUCKET / 2; step > 0; step >>= 1)
            if (pref[r + step] <= i) r += step;
        return tile[r] + (i - pref[r]);
    }
};
// The same in global memory, by a whole wave (four prefixes per lane): the bitmap
// kernel has no LDS left for a copy at six blocks per CU.
__device__ __forceinline__ uint32_t range_tile(const uint32_t* __restrict__ tile, const uint32_t* __restrict__ pref,
                                               uint32_t i) {
    static_assert(NBUCKET == 4 * WAVE, "four prefixes per lane");
    uint32_t r = 0;   // prefixes at most i (pref[0] = 0 is one)
#pragma unroll
    for (int k = 0; k < 4; ++k) r += (uint32_t)__popcll(__ballot(pref[k * WAVE + lane_id()] <= i));
    return tile[r - 1u] + (i - pref[r - 1u]);
}

// Decode tile t into segments (v, first in-edge, count); returns the count.
// Called by the whole block; contains barriers.
template <int N>
__device__ uint32_t load_tile(const IsectArgs& a, uint32_t t, SegsT<N>& S) {
    const uint4 d = a.tiles[t];
    uint32_t nseg, cnt = 0;
    if (d.w & TILE_MULTI) {
        nseg = d.y;
        if (nseg > (uint32_t)N) nseg = N;   // the tile layout never makes more
        if (threadIdx.x < nseg) {
            const uint32_t v = a.vlist[d.x + threadIdx.x];
            S.v[threadIdx.x] = v;
            S.e0[threadIdx.x] = a.inoff[v];
            cnt = a.inoff[v + 1] - a.inoff[v];
        }
    } else {   // one vertex: no scan needed
        if (threadIdx.x == 0) {
            S.v[0] = d.x;
            S.e0[0] = d.y;
            S.pref[0] = 0;
            S.pref[1] = d.z;
        }
        __syncthreads();
        return 1;
    }
    uint32_t total;
    const uint32_t excl = block_exclusive_scan<IS_NT>(cnt, S.scratch, &total);
    if (threadIdx.x < nseg) S.pref[threadIdx.x] = excl;
    if (threadIdx.x == 0) S.pref[nseg] = total;
    __syncthreads();
    return nseg;
}

// Per-vertex counts. Most triangles' highest vertex is one of a few hubs, and
// device-wide atomics on one address serialise (about 23 ns each), so a block of
// the bitmap or binary-search kernel counts the HOT_N top-ranked vertices in
// LDS and adds them up once, at its end. (Merge path serves short lists, which
// end in hubs less often, and lives on its occupancy: with these counters it
// ran four blocks per CU instead of seven, and a uniform graph of 10
// million pairs took 1577 us instead of 1501.) Measured per call with t[v]: R-MAT 16 994 -> 565 us; R-MAT 18
// with clustering coefficients 2796 -> 1110 us (1024, 4096 and 8192 counters: 1151,
// 1202 and 1380 us).
constexpr uint32_t HOT_N = 2048;
struct Hot {
    uint32_t* cnt;    // LDS [HOT_N], or null: no vertex is counted in LDS
    uint32_t first;   // rank of cnt[0]
    __device__ void add(const IsectArgs& a, uint32_t x, uint32_t c) const {
        if (cnt && x >= first) atomicAdd(&cnt[x - first], c);
        else atomicAdd((unsigned long long*)&a.per_vertex[x], (unsigned long long)c);
    }
    // Whole block, before the first and after the last tile; barriers around are the caller's.
    __device__ void clear() const {
        for (uint32_t i = threadIdx.x; i < HOT_N; i += blockDim.x) cnt[i] = 0;
    }
    __device__ void flush(const IsectArgs& a) const {
        for (uint32_t i = threadIdx.x; i < HOT_N; i += blockDim.x) {
            const uint32_t q = (i + blockIdx.x * 64u) % HOT_N;   // blocks start at different counters
            const uint32_t c = cnt[q];
            if (c) atomicAdd((unsigned long long*)&a.per_vertex[first + q], (unsigned long long)c);
        }
    }
};

__device__ __forceinline__ void edge_done(const IsectArgs& a, const Hot& hot, uint32_t e, uint32_t v, uint32_t c) {
    if (a.per_edge) a.per_edge[e] = c;
    if (a.support && c) atomicAdd(&a.support[e], c);
    if (a.per_middle && c) atomicAdd((unsigned long long*)&a.per_middle[v], (unsigned long long)c);
    if (a.per_vertex && c) {
        hot.add(a, a.src[e], c);
        hot.add(a, v, c);
    }
}

// Triangle (u, v, w) of in-edge e = (u -> v) at list slot pos, original ids.
__device__ __forceinline__ void list_write(const IsectArgs& a, uint64_t pos, uint32_t e, uint32_t w) {
    if (pos >= a.list_cap) {   // only if the two passes disagree
        atomicOr(&a.ctrl->err, 8u);
        return;
    }
    int32_t* o = a.list_out + 3 * pos;
    o[0] = (int32_t)a.inv[a.src[e]];
    o[1] = (int32_t)a.inv[a.col[e]];
    o[2] = (int32_t)a.inv[w];
}

// A hit w = col[ea] = col[eb] for in-edge ein: ea is the edge (u, w) of the
// tail, eb the edge (v, w).
__device__ __forceinline__ void hit(const IsectArgs& a, const Hot& hot, uint32_t w, uint32_t ea, uint32_t eb,
                                    uint32_t ein) {
    if (a.per_vertex) hot.add(a, w, 1u);
    if (a.support) {
        atomicAdd(&a.support[ea], 1u);
        atomicAdd(&a.support[eb], 1u);
    }
    if (a.list_out) list_write(a, a.list_off[ein] + atomicAdd(&a.list_cur[ein], 1u), ein, w);
}

// Position of x in the ascending list L[0..n), or n when absent.
__device__ __forceinline__ uint32_t find_pos(const uint32_t* L, uint32_t n, uint32_t x) {
    uint32_t lo = 0, hi = n;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (L[mid] < x) lo = mid + 1u;
        else hi = mid;
    }
    return (lo < n && L[lo] == x) ? lo : n;
}

__device__ __forceinline__ void block_partial(uint64_t acc, uint64_t* partials) {
    __shared__ uint64_t red[IS_NT / WAVE];
    acc = wave_sum_u64(acc);
    if (lane_id() == 0) red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int i = 0; i < IS_NT / WAVE; ++i) s += red[i];
        partials[blockIdx.x] = s;
    }
}

// ------------------------------------------------------------------ LDS bitmap
// Element i of col. NARROW: the array is below 4 GiB, so a 32-bit byte offset
// from the (scalar) base addresses it and no 64-bit address math is needed.
template <bool NARROW>
__device__ __forceinline__ uint32_t col_at(const uint32_t* col, uint32_t i) {
    if (NARROW) return *(const uint32_t*)((const char*)col + (uint32_t)(i << 2));
    return col[i];
}

// Outputs of a bitmap launch: T only; also per middle vertex (one sum per vertex
// and tile); also per in-edge counts (per-edge outputs); per-vertex counts (t[w] in LDS counters
// for the top ranks, gathered per element of N+(v) for others where they are many); edge support (the hits per element of N+(v), the support of
// edge vw, are gathered in LDS; an element's position in the list is the
// position of its bitmap word's first element plus the bits before it);
// or the triangle list (the per-entry count is the cursor of the entry's
// slots). Each mode sizes its LDS to what it uses.
// BM_CLIP counts only, for tails that are whole rows: each tail and the middle
// list are cut to the window being tested, and windows holding no element of
// the middle list are skipped.
enum { BM_COUNT = 0, BM_ENTRY = 1, BM_VERTEX = 2, BM_LIST = 3, BM_CLIP = 4, BM_MIDDLE = 5, BM_SUPPORT = 6, BM_NMODE = 7 };

constexpr int EH = CHUNK_MAX / IS_NT;   // entries of a vertex per thread

// First position p in [p, e) of the ascending col whose value is at least x (e if none).
template <bool NARROW>
__device__ __forceinline__ uint32_t first_at_least(const uint32_t* col, uint32_t p, uint32_t e, uint64_t x) {
    while (p < e) {
        const uint32_t mid = p + ((e - p) >> 1);
        if ((uint64_t)col_at<NARROW>(col, mid) < x) p = mid + 1u;
        else e = mid;
    }
    return p;
}

// The same search by a whole wave, the same result in every lane: 64 probes
// per step narrow the range 64-fold, so a list of d elements costs about
// log64(d) dependent loads instead of log2(d).
template <bool NARROW>
__device__ __forceinline__ uint32_t wave_first_at_least(const uint32_t* col, uint32_t p, uint32_t e, uint64_t x) {
    const uint32_t ln = (uint32_t)lane_id();
    while (e - p > (uint32_t)WAVE) {
        const uint32_t step = (e - p + WAVE - 1) / WAVE;
        const uint32_t q = p + (ln + 1u) * step - 1u;   // last element of the lane's step
        const bool below = q < e && (uint64_t)col_at<NARROW>(col, q) < x;
        const uint32_t c = (uint32_t)__popcll(__ballot(below));   // steps wholly below x
        const uint32_t np = p + c * step;
        e = np + step < e ? np + step : e;
        p = np;
    }
    const uint32_t q = p + ln;
    const bool below = q < e && (uint64_t)col_at<NARROW>(col, q) < x;
    return p + (uint32_t)__popcll(__ballot(below));
}

// Entry table of one vertex's in-edges in a tile, in LDS: entry k streams
// items [s_pref[k], s_pref[k + 1]) of a flat item range, item q at
// col[s_base[k] + q] (s_base = start - s_pref, modular). Tails of at least
// LONG_TAIL items come first, then the shorter non-empty ones; empty tails are
// left out, so s_pref is strictly increasing. Thread t holds entries EH * t ..
// EH * t + EH - 1 (start st_h, length len_h; length 0 past the vertex's
// entries) and later owns the table slots with the same indexes, so each
// phase needs one block scan. Returns the entries kept; nl = long entries,
// L = total items. Whole block; contains barriers.
template <int NTB, int EPT, bool CNT>
__device__ __forceinline__ uint32_t entry_table(const uint32_t (&st_h)[EPT], const uint32_t (&len_h)[EPT],
                                                uint32_t* s_pref, uint32_t* s_base, uint32_t* s_cnt,
                                                uint32_t* scratch, uint32_t& nl, uint32_t& L) {
    uint32_t f = 0;   // long entries in the high half, non-empty short ones in the low half
#pragma unroll
    for (int h = 0; h < EPT; ++h) f += len_h[h] >= LONG_TAIL ? 0x10000u : (len_h[h] ? 1u : 0u);
    uint32_t total;
    const uint32_t ex = block_exclusive_scan<NTB>(f, scratch, &total);
    const uint32_t cl = total >> 16, cs = total & 0xFFFFu;
    uint32_t pl = ex >> 16, ps = cl + (ex & 0xFFFFu);
#pragma unroll
    for (int h = 0; h < EPT; ++h) {   // lengths and starts in table order
        if (!len_h[h]) continue;
        const uint32_t pos = len_h[h] >= LONG_TAIL ? pl++ : ps++;
        s_pref[pos] = len_h[h];
        s_base[pos] = st_h[h];
        if (CNT) s_cnt[pos] = 0;
    }
    __syncthreads();
    const uint32_t nt = cl + cs;
    uint32_t len[EPT], st[EPT], sum = 0;
#pragma unroll
    for (int h = 0; h < EPT; ++h) {   // this thread's slots, rewritten in place below
        const uint32_t k = EPT * threadIdx.x + (uint32_t)h;
        len[h] = k < nt ? s_pref[k] : 0u;
        st[h] = k < nt ? s_base[k] : 0u;
        sum += len[h];
    }
    uint32_t items;
    uint32_t run = block_exclusive_scan<NTB>(sum, scratch, &items);
#pragma unroll
    for (int h = 0; h < EPT; ++h) {
        const uint32_t k = EPT * threadIdx.x + (uint32_t)h;
        if (k < nt) {
            s_pref[k] = run;
            s_base[k] = st[h] - run;
        }
        run += len[h];
    }
    if (threadIdx.x == 0) s_pref[nt] = items;
    nl = cl;
    L = items;
    return nt;
}

// Six blocks of four waves fit a CU by LDS in every mode but the per-vertex (40 KB:
// four) and the support one (44 KB: three); the register budget is held to the same occupancy (80 VGPRs).
template <int MODE, bool NARROW>
__global__ __launch_bounds__(IS_NT, MODE == BM_VERTEX ? 4 : (MODE == BM_SUPPORT ? 3 : 6)) void k_isect_bitmap(
    IsectArgs a, uint64_t* partials) {
    constexpr bool VERTEX = MODE == BM_VERTEX, SUPPORT = MODE == BM_SUPPORT;
    constexpr bool CLIP = MODE == BM_CLIP;
    // Counts alone take the windows from the top of the middle list down, each as far as its
    // highest element not yet in one, and after each keep of every tail only what lies
    // below the window (s_cut). Ranks ascend with the degree, so nearly all of a tail lies in the
    // first window; walking whole tails once per window read R-MAT 24's remaining 6.9e9 tail
    // elements 12.2e9 times (with it, beside the wave kernel, 39.0 -> 38.5 ms).
    constexpr bool SHRINK = MODE == BM_COUNT || MODE == BM_MIDDLE;
    constexpr int WORDS = SHRINK ? BM_WORDS - CHUNK_MAX : BM_WORDS;   // the same LDS with s_cut
    constexpr uint32_t BITS = (uint32_t)WORDS * 32u;
    constexpr bool need_cnt = MODE != BM_COUNT && MODE != BM_MIDDLE && !CLIP;
    __shared__ uint32_t s_hot[VERTEX ? HOT_N : 1];
    // Hits per element of N+(v). In the per-vertex mode of those that have no counter in s_hot ("cold"), two
    // to a word (a tile has at most CHUNK_MAX in-edges of v), in a tile that follows one of at least
    // COLD_HITS cold hits per element of its lists in this block: where triangles are dense and not held by a few
    // vertices, one device-wide add per cold hit is what bounds the kernel (t[v] of 300 cliques of 500 vertices
    // 105 ms, now 21; of a geometric graph of 2^20 vertices and degree 100 56 ms, now 37.5; R-MAT 22 20.5 and
    // 17.4), elsewhere the set-up costs more than it saves (R-MAT 18 with coefficients 0.99 ms, with it
    // everywhere 1.05). COLD_HITS 2: R-MAT 22 18.0 ms, the others alike.
    constexpr uint32_t COLD_HITS = 1;
    static_assert(CHUNK_MAX < 65536, "a tile's hits of an element fit 16 bits");
    __shared__ uint32_t s_wc[SUPPORT ? NV_MAX : (VERTEX ? NV_MAX / 2 : 1)];
    __shared__ uint32_t s_cold;            // cold hits of the block's last tile
    uint32_t cold = 0, cold_nb = 0;        // this thread's; the elements of the tile's lists
    // position in N+(v) of the first element of a word, or (per-vertex mode: all that four
    // blocks per CU leave) of eight
    constexpr int FIRST_LOG2 = SUPPORT ? 5 : 8;
    __shared__ uint16_t s_first[SUPPORT ? WORDS : (VERTEX ? WORDS / 8 : 1)];
    const Hot hot = {VERTEX ? s_hot : nullptr, a.hot_first};
    if (VERTEX) hot.clear();
    __shared__ __align__(16) uint32_t bm[WORDS + 1];   // + one always-zero word for out-of-window positions
    __shared__ uint16_t s_wst[WT_MAX];           // entry holding the first item of each window of a chunk
    __shared__ uint32_t s_pref[CHUNK_MAX + 1];
    __shared__ uint32_t s_cnt[need_cnt ? CHUNK_MAX : 1];
    __shared__ uint32_t s_cut[SHRINK ? CHUNK_MAX : 1];   // one past an entry's last item below the window, or 0
    __shared__ uint32_t s_base[CHUNK_MAX + 1];   // entry nt is read (unused) by lanes past the end
    __shared__ uint8_t s_flag[IS_NT / WAVE][UNROLL][WAVE];    // entry-start marks, one slot per item offset
    __shared__ SegsT<SEG_MAX_BITMAP> S;
    for (int i = threadIdx.x; i <= WORDS; i += IS_NT) bm[i] = 0;
    for (int i = threadIdx.x; i < (IS_NT / WAVE) * UNROLL * WAVE; i += IS_NT) (&s_flag[0][0][0])[i] = 0;
    uint64_t acc = 0;
    __shared__ uint32_t s_tile;
    const uint32_t t_begin = a.ctrl->tile_begin[KER_BITMAP];
    uint32_t ntile = a.ctrl->tile_begin[KER_BITMAP + 1] - t_begin;
    // with the hub kernel beside it, this one takes the tiles that are left
    constexpr bool RANGES = MODE == BM_COUNT || MODE == BM_MIDDLE;
    const bool ranges = RANGES && a.hub && a.hub->used != 0;
    if (ranges) ntile = a.hub->rest_pref[NBUCKET];
    for (uint32_t i = blockIdx.x; i < ntile; i = grab_tile(a.ctrl, KER_BITMAP, gridDim.x, &s_tile)) {
        const bool dense = VERTEX && cold_nb != 0 && s_cold >= COLD_HITS * cold_nb;   // grab_tile's barriers are between
        const uint32_t nseg = load_tile(a, ranges ? range_tile(a.hub->rest_tile, a.hub->rest_pref, i) : t_begin + i, S);
        if (VERTEX && threadIdx.x == 0) s_cold = 0;   // read by all before load_tile's barrier
        cold_nb = 0;
        for (uint32_t sg = 0; sg < nseg; ++sg) {
            const uint32_t v = S.v[sg];
            const uint32_t e0 = S.e0[sg];
            const uint32_t ne = S.pref[sg + 1] - S.pref[sg];
            const uint32_t b0 = a.off[v], b1 = a.off[v + 1];
            const uint32_t nb = b1 - b0;
            uint32_t seg_sum = 0;   // BM_MIDDLE: this thread's hits for v (below 2^32: a tile's tail elements)
            // the vertex's entries (ne <= CHUNK_MAX = EH * IS_NT: EH consecutive ones per thread)
            uint32_t st_h[EH], len_h[EH];
#pragma unroll
            for (int h = 0; h < EH; ++h) {
                const uint32_t k = EH * threadIdx.x + (uint32_t)h;
                st_h[h] = len_h[h] = 0;
                if (k < ne) {
                    const uint64_t ent = a.csc[e0 + k];   // tail start | tail end << 32
                    st_h[h] = tail_start(ent);
                    len_h[h] = tail_end(ent, CLIP) - st_h[h];
                }
            }
            // the table: once per vertex, or per window when the tails are clipped
            uint32_t nt = 0, nl = 0, L = 0;
            if (!CLIP) nt = entry_table<IS_NT, EH, need_cnt>(st_h, len_h, s_pref, s_base, s_cnt, S.scratch, nl, L);
            const uint32_t lo = a.col[b0], hi = a.col[b1 - 1];
            const uint32_t base = lo & ~31u;
            const uint32_t nwin = (hi - base) / BITS + 1;
            const bool gather = nb <= (uint32_t)NV_MAX &&
                                (SUPPORT || (dense && lo < a.hot_first));
            if (gather)
                for (uint32_t j = threadIdx.x; j < (SUPPORT ? nb : (nb + 1u) / 2u); j += IS_NT) s_wc[j] = 0u;
            __syncthreads();
            // clipped tails: each entry keeps a cursor (st_h, with len_h left) and the
            // value under it, so a window that holds none of its elements costs no load
            uint64_t cv_h[EH];
            if (CLIP) {
#pragma unroll
                for (int h = 0; h < EH; ++h)
                    cv_h[h] = len_h[h] ? (uint64_t)col_at<NARROW>(a.col, st_h[h]) : ~0ull;
            }
            uint32_t mnext = 0;   // clipped: first element of the middle list not yet in a window
            uint32_t left = nb;   // SHRINK: elements of the middle list in no window yet
            for (uint32_t win = 0; SHRINK || win < nwin; ++win) {
                uint32_t wlo = base + win * BITS;
                uint32_t j0 = 0, j1 = nb;   // elements of the middle list set in this window
                bool more = false;          // SHRINK: a window follows
                if (SHRINK) {
                    const uint32_t top = win ? a.col[b0 + left - 1u] : hi;
                    wlo = top >= BITS ? top - (BITS - 1u) : 0u;
                    j1 = left;
                    if (lo < wlo) j0 = wave_first_at_least<NARROW>(a.col, b0, b0 + left, wlo) - b0;
                    more = j0 > 0;
                    if (more)
                        for (uint32_t k = threadIdx.x; k < nt; k += IS_NT) s_cut[k] = 0;
                }
                if (CLIP) {
                    const uint64_t whi = (uint64_t)wlo + BITS;
                    j0 = mnext;
                    j1 = wave_first_at_least<NARROW>(a.col, b0 + j0, b1, whi) - b0;
                    mnext = j1;
                    if (j1 == j0) continue;   // same for the whole block: nothing to match here
                    // each tail cut to [wlo, whi); what lies above stays for the next windows
                    uint32_t cs_h[EH], cl_h[EH];
#pragma unroll
                    for (int h = 0; h < EH; ++h) {
                        uint32_t p = st_h[h];
                        const uint32_t e = p + len_h[h];
                        uint32_t e2 = p;
                        if (cv_h[h] < whi) {
                            // elements below wlo belong to windows without middle elements
                            if (cv_h[h] < wlo) p = first_at_least<NARROW>(a.col, p, e, wlo);
                            e2 = first_at_least<NARROW>(a.col, p, e, whi);
                            cv_h[h] = e2 < e ? (uint64_t)col_at<NARROW>(a.col, e2) : ~0ull;
                        }
                        cs_h[h] = p;
                        cl_h[h] = e2 - p;
                        st_h[h] = e2;
                        len_h[h] = e - e2;
                    }
                    nt = entry_table<IS_NT, EH, false>(cs_h, cl_h, s_pref, s_base, s_cnt, S.scratch, nl, L);
                }
                for (uint32_t j = j0 + threadIdx.x; j < j1; j += IS_NT) {
                    const uint32_t x = a.col[b0 + j] - wlo;
                    if (x < BITS) {
                        atomicOr(&bm[x >> 5], 1u << (x & 31u));
                        if (gather && (j == 0 || (a.col[b0 + j - 1] - wlo) >> FIRST_LOG2 != x >> FIRST_LOG2))
                            s_first[x >> FIRST_LOG2] = (uint16_t)j;
                    }
                }
                __syncthreads();
                // All tails of the tile form one flat item range [0, L); item q of
                // entry k lives at col[base[k] + q]. The range is cut into 64-item
                // windows, taken in chunks of WT_MAX windows: per chunk a table gives
                // the entry holding each window's first item, and wave w walks a
                // contiguous, 64-aligned quarter of the chunk in rounds of UNROLL
                // windows (one item per lane per window). A round runs in phases,
                // each over all UNROLL windows: read the windows' first entries from
                // the table; mark the entry starts inside each window (lane ln looks
                // at entry first + 1 + ln and marks its start offset in a per-wave
                // slot array); read the slots back as a ballot mask, so that a lane's
                // entry is first + (starts at or before its offset); issue the tail
                // loads, unconditional (lanes past the end read a valid address);
                // test the bitmap. Rounds that lie inside the long tails (placed
                // first) skip the marks: there an entry spans at least one window,
                // so one compare with the next entry's start gives a lane's entry.
                const uint32_t wv = (uint32_t)wave_id(), ln = (uint32_t)lane_id();
                const uint32_t Llong = s_pref[nl];   // items of the long tails: [0, Llong)
                for (uint32_t c0 = 0; c0 < L; c0 += WT_MAX * WAVE) {
                    const uint32_t c1 = L - c0 < WT_MAX * WAVE ? L : c0 + WT_MAX * WAVE;
                    const uint32_t nwc = (c1 - c0 + WAVE - 1) / WAVE;   // windows in this chunk
                    // window table: entry k covers items [pref[k], pref[k+1])
                    for (uint32_t k = threadIdx.x; k < nt; k += IS_NT) {
                        const uint32_t p0 = s_pref[k] > c0 ? s_pref[k] : c0;
                        const uint32_t p1 = s_pref[k + 1] < c1 ? s_pref[k + 1] : c1;
                        for (uint32_t w = (p0 - c0 + WAVE - 1) / WAVE; p0 < p1 && w * WAVE + c0 < p1; ++w)
                            s_wst[w] = (uint16_t)k;
                    }
                    __syncthreads();
                    const uint32_t span = (c1 - c0 + WAVE - 1) / WAVE;   // windows, split over the waves
                    const uint32_t q0 = c0 + WAVE * ((span * wv) / (IS_NT / WAVE));
                    const uint32_t qe = c0 + WAVE * ((span * (wv + 1)) / (IS_NT / WAVE));
                    const uint32_t q1 = qe < c1 ? qe : c1;
                    const uint32_t lim = Llong < q1 ? Llong : q1;   // rounds below lim see long tails only
                    for (uint32_t W = q0; W < q1; W += WAVE * UNROLL) {
                        uint32_t xs[UNROLL], ks[UNROLL], kj[UNROLL];
#pragma unroll
                        for (int j = 0; j < UNROLL; ++j) {   // same address in all lanes: broadcast
                            const uint32_t wi = (W - c0) / WAVE + (uint32_t)j;
                            kj[j] = s_wst[wi < nwc ? wi : nwc - 1u];
                        }
                        if (W + WAVE * UNROLL <= lim) {
                            // long tails only: an entry spans at least one window, so at most
                            // one entry starts inside a window; a lane's entry is the window's
                            // first entry, plus one at or after the next start
#pragma unroll
                            for (int j = 0; j < UNROLL; ++j) {
                                const uint32_t nx = s_pref[kj[j] + 1u];
                                ks[j] = kj[j] + (W + j * WAVE + ln >= nx ? 1u : 0u);
                            }
                            uint32_t ad[UNROLL];
#pragma unroll
                            for (int j = 0; j < UNROLL; ++j) ad[j] = s_base[ks[j]] + W + j * WAVE + ln;
#pragma unroll
                            for (int j = 0; j < UNROLL; ++j) xs[j] = col_at<NARROW>(a.col, ad[j]) - wlo;
                        } else {
                            // mark the starts (pref is strictly increasing, so the marked offsets
                            // are distinct and at least 1). Entries past the last one read
                            // pref[nt] = L: a start at or after item L moves only lanes whose
                            // items lie beyond q1 (unused).
                            uint32_t o[UNROLL];
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) {
                                const uint32_t kk = kj[j] + 1u + ln;
                                o[j] = s_pref[kk < nt ? kk : nt] - (W + j * WAVE);
                            }
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j)
                                if (o[j] < 64u) s_flag[wv][j][o[j]] = 1;
                            // the lanes of the wave exchange marks through LDS: keep the
                            // mark / read / clear phases in program order
                            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
                            uint32_t f[UNROLL];
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) f[j] = s_flag[wv][j][ln];
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) s_flag[wv][j][ln] = 0;   // each lane clears its own slot
                            __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront");
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) {
                                const uint64_t M = __ballot(f[j] != 0u);
                                const uint32_t below = __builtin_amdgcn_mbcnt_hi(
                                    (uint32_t)(M >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)M, 0u));
                                ks[j] = kj[j] + below + (f[j] != 0u ? 1u : 0u);
                            }
                            uint32_t ad[UNROLL];
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) {
                                const uint32_t q = W + j * WAVE + ln;
                                const uint32_t sb = s_base[ks[j]];
                                ad[j] = q < q1 ? sb + q : b0;
                            }
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j) xs[j] = col_at<NARROW>(a.col, ad[j]);
    #pragma unroll
                            for (int j = 0; j < UNROLL; ++j)
                                xs[j] = (W + j * WAVE + ln < q1) ? xs[j] - wlo : 0x7FFFFFFFu;
                        }
                        // membership: bit positions past the window map to the spare
                        // always-zero word bm[WORDS]
                        uint32_t wd[UNROLL];
#pragma unroll
                        for (int j = 0; j < UNROLL; ++j) wd[j] = bm[(xs[j] < BITS ? xs[j] : BITS) >> 5];
                        uint32_t hits = 0;
#pragma unroll
                        for (int j = 0; j < UNROLL; ++j) hits += __builtin_amdgcn_ubfe(wd[j], xs[j], 1u);
                        acc += hits;
                        if (MODE == BM_MIDDLE) seg_sum += hits;
                        if (SHRINK && more) {
                            // an entry's items below the window are its first ones: the last of
                            // them in this wave's 64 items marks the cut
#pragma unroll
                            for (int j = 0; j < UNROLL; ++j) {
                                const bool below = (int32_t)xs[j] < 0;
                                const uint64_t B = __ballot(below);
                                if (!B) continue;
                                const uint32_t kn = (uint32_t)__shfl_down((int)ks[j], 1, WAVE);
                                const bool next = ((B >> 1) >> ln) & 1ull;   // never for lane 63
                                if (below && !(next && kn == ks[j]))
                                    atomicMax(&s_cut[ks[j]], W + (uint32_t)j * WAVE + ln + 1u);
                            }
                        }
                        if (!need_cnt) continue;
                        // long tails only, and enough hits that a count per window is cheaper than an add per
                        // hit (per-edge counts with adds alone: R-MAT 17 of 30 million pairs 18.0 ms, now 8.7; with
                        // counts alone: 60 million uniform pairs on 300,000 vertices 16.7 ms, now 13.6)
                        const bool by_window = MODE != BM_LIST && W + WAVE * UNROLL <= lim &&
                                               __popcll(__ballot(hits != 0)) >= 8;
                        uint32_t colds = 0;   // windows in which this lane has a cold hit
#pragma unroll
                        for (int j = 0; j < UNROLL; ++j) {
                            const uint32_t x = xs[j];
                            const bool is = (wd[j] >> (x & 31u)) & 1u;
                            if (by_window) {   // at most two entries in the window
                                const uint64_t H = __ballot(is);
                                const uint32_t at = s_pref[kj[j] + 1u] - (W + (uint32_t)j * WAVE);
                                const uint64_t A = at < (uint32_t)WAVE ? (1ull << at) - 1ull : ~0ull;
                                const uint32_t c = (uint32_t)__popcll(ln == 0 ? H & A : H & ~A);
                                if (ln < 2 && c) atomicAdd(&s_cnt[kj[j] + ln], c);
                            }
                            if (is) {
                                if (MODE == BM_LIST) {
                                    const uint32_t slot = atomicAdd(&s_cnt[ks[j]], 1u);
                                    const uint32_t e = s_base[ks[j]] + s_pref[ks[j]] - 1u;
                                    list_write(a, a.list_off[e] + slot, e, x + wlo);
                                } else if (!by_window) {
                                    atomicAdd(&s_cnt[ks[j]], 1u);
                                }
                                if (VERTEX) {
                                    if (x + wlo >= a.hot_first) {
                                        atomicAdd(&s_hot[x + wlo - a.hot_first], 1u);
                                    } else {
                                        colds |= 1u << j;
                                    }
                                }
                                if (SUPPORT) {   // edge (u, w): the tail element's own position
                                    atomicAdd(&a.support[s_base[ks[j]] + W + (uint32_t)j * WAVE + ln], 1u);
                                    if (gather)   // w's place in N+(v), flushed per vertex
                                        atomicAdd(&s_wc[s_first[x >> 5] + __popc(wd[j] & ((1u << (x & 31u)) - 1u))], 1u);
                                    else
                                        atomicAdd(&a.support[b0 + find_pos(a.col + b0, nb, x + wlo)], 1u);
                                }
                            }
                        }
                        while (VERTEX && __ballot(colds != 0)) {   // one per lane and step
                            if (colds != 0) {
                                const uint32_t jj = (uint32_t)__ffs((int)colds) - 1u;
                                colds &= colds - 1u;
                                ++cold;
                                uint32_t x = xs[0];
#pragma unroll
                                for (int j = 1; j < UNROLL; ++j) x = jj == (uint32_t)j ? xs[j] : x;
                                if (gather) {
                                    // x's place in N+(v): elements before its eight words, in those before its own,
                                    // and below it there
                                    const uint32_t w = (x >> 5) & 7u, below = (1u << (x & 31u)) - 1u;
                                    const uint4* eight = (const uint4*)&bm[(x >> 8) * 8u];
                                    const uint4 p = eight[0], q = eight[1];
                                    const uint32_t word[8] = {p.x, p.y, p.z, p.w, q.x, q.y, q.z, q.w};
                                    uint32_t at = s_first[x >> FIRST_LOG2];
#pragma unroll
                                    for (uint32_t i = 0; i < 8; ++i)
                                        at += (uint32_t)__popc(word[i] & (i < w ? ~0u : (i == w ? below : 0u)));
                                    atomicAdd(&s_wc[at >> 1], 1u << (16u * (at & 1u)));
                                } else {
                                    atomicAdd((unsigned long long*)&a.per_vertex[x + wlo], 1ull);
                                }
                            }
                        }
                    }
                    __syncthreads();   // the table is rebuilt for the next chunk
                }
                __syncthreads();
                for (uint32_t j = j0 + threadIdx.x; j < j1; j += IS_NT) {
                    const uint32_t x = a.col[b0 + j] - wlo;
                    if (x < BITS) bm[x >> 5] = 0u;
                }
                __syncthreads();
                if (SHRINK) {
                    if (!more) break;
                    left = j0;
                    uint32_t cs_h[EH], cl_h[EH];
#pragma unroll
                    for (int h = 0; h < EH; ++h) {
                        const uint32_t k = EH * threadIdx.x + (uint32_t)h;
                        cs_h[h] = cl_h[h] = 0;
                        if (k < nt && s_cut[k] > s_pref[k]) {
                            cl_h[h] = s_cut[k] - s_pref[k];
                            cs_h[h] = s_base[k] + s_pref[k];
                        }
                    }
                    nt = entry_table<IS_NT, EH, false>(cs_h, cl_h, s_pref, s_base, s_cnt, S.scratch, nl, L);
                    if (L == 0) break;   // the same for the whole block
                }
            }
            if (gather) {
                for (uint32_t j = threadIdx.x; j < nb; j += IS_NT) {
                    const uint32_t c = SUPPORT ? s_wc[j] : (s_wc[j >> 1] >> (16u * (j & 1u))) & 0xFFFFu;
                    if (!c) continue;
                    if (SUPPORT) atomicAdd(&a.support[b0 + j], c);
                    else atomicAdd((unsigned long long*)&a.per_vertex[a.col[b0 + j]], (unsigned long long)c);
                }
            }
            if (VERTEX) {   // t[u] per in-edge, t[v] once per wave
                uint32_t mine = 0;
                for (uint32_t k = threadIdx.x; k < nt; k += IS_NT) {
                    const uint32_t c = s_cnt[k];
                    if (c) hot.add(a, a.src[s_base[k] + s_pref[k] - 1u], c);
                    mine += c;
                }
                mine = wave_sum(mine);
                if (lane_id() == 0 && mine) hot.add(a, v, mine);
                cold_nb += nb;
            } else if (need_cnt) {
                for (uint32_t k = threadIdx.x; k < nt; k += IS_NT)
                    edge_done(a, hot, s_base[k] + s_pref[k] - 1u, v, s_cnt[k]);
            }
            if (MODE == BM_MIDDLE) {   // one update per vertex and tile
                uint32_t total;
                (void)block_exclusive_scan<IS_NT>(seg_sum, S.scratch, &total);
                if (threadIdx.x == 0 && total)
                    atomicAdd((unsigned long long*)&a.per_middle[v], (unsigned long long)total);
            }
            __syncthreads();
        }
        if (VERTEX && __ballot(cold != 0)) {
            cold = wave_sum(cold);
            if (lane_id() == 0) atomicAdd(&s_cold, cold);
            cold = 0;
        }
    }
    if (VERTEX) {
        __syncthreads();
        hot.flush(a);
    }
    block_partial(acc, partials);
}

// ------------------------------------------------------------------ hub kernel
// The bitmap strategy for single-vertex tiles whose middle vertex is one of the
// HUB_SPAN top-ranked ones (counts in all, or per middle vertex), where a skewed
// graph has most of its work (R-MAT 24: 84% of the tail elements). The tail of
// an in-edge (u -> v) holds only ranks above v, so here it lies inside those
// ranks: it is read from 16-bit columns, half the bytes, and N+(v) is a byte
// per rank in LDS (64 KB), so that an element costs a field extract, an LDS byte and
// half an add instead of a word address, a bit test and an add.
// A wave takes a share of the tile's in-edges, one per lane, orders them by
// length, and eight lanes walk one tail together, a 16-byte chunk per lane and
// step: eight tails of similar length per wave, HB_D steps of loads in flight,
// and no item table, scan or barrier between the tile's set-up and its end. What a
// first or last chunk holds beside the tail is turned into HUB_NONE by mask
// words from an LDS table. The next tile's descriptor and in-edges are loaded
// while the current one is walked. Bound: the line traffic of the tails beyond
// L2: 91 GB of counted traffic at R-MAT 24 with all its ranks (counts in all leave
// the highest to the group kernel below), 7.4 TB/s. Measured so: this
// kernel and the bitmap kernel for the remaining tiles 12.2 + 9.5 ms, the bitmap kernel
// alone 30.1 ms; R-MAT 20 (tiles too short for the set-up to vanish) 0.65 + 0.19
// against 0.89 ms. Steps in flight: 3 and 4 alike, 6 and 8 slower (23.2, 36.5 ms with the
// bitmap kernel against 22.6: registers); 1024 threads with two steps 1% faster at
// R-MAT 24 and 1% slower on a batch of Chung-Lu graphs.
constexpr int HB_NT = 512;                // two blocks fit a CU by LDS
constexpr int HB_W = HB_NT / WAVE;
constexpr int HB_D = 3;                   // steps in flight
constexpr uint32_t HB_L = 8;              // lanes per tail
constexpr uint32_t HB_R = WAVE / HB_L;    // tails walked together by a wave
constexpr uint32_t HB_E = 8;              // elements per chunk
// partial slots of the bitmap kernel's share from here on: the wave, the hub and the group kernel's
constexpr int WV_PARTIAL0 = 1536, HB_PARTIAL0 = 3072, HB_PARTIAL1 = 3584;
static_assert(CHUNK_MAX <= HB_NT, "one in-edge per lane");

// Order of magnitude of a step count: 0, 1, 2, 3, then two classes per doubling, at most HB_CLS - 1.
constexpr int HB_CLS = 12;
__device__ __forceinline__ uint32_t step_class(uint32_t steps) {
    if (steps < 4u) return steps;
    const uint32_t l = (uint32_t)floor_log2(steps);
    const uint32_t c = 2u * l + ((steps >> (l - 1u)) & 1u);
    return c < (uint32_t)HB_CLS ? c : (uint32_t)HB_CLS - 1u;
}

struct HubMasks {   // k first / last elements of a chunk set to ones
    uint4 head[HB_E + 1], tail[HB_E + 1];
    // Whole block; a barrier follows before use.
    __device__ void fill() {
        if (threadIdx.x > HB_E) return;
        const uint32_t k = threadIdx.x;
        uint32_t h[4], t[4];
        for (uint32_t q = 0; q < 4; ++q) {
            h[q] = (2 * q < k ? 0xFFFFu : 0u) | (2 * q + 1 < k ? 0xFFFF0000u : 0u);
            t[q] = (2 * q + k >= HB_E ? 0xFFFFu : 0u) | (2 * q + 1 + k >= HB_E ? 0xFFFF0000u : 0u);
        }
        head[k] = make_uint4(h[0], h[1], h[2], h[3]);
        tail[k] = make_uint4(t[0], t[1], t[2], t[3]);
    }
};

constexpr uint32_t GRP_OFF = HUB_SPAN - GRP_SPAN;   // the group kernel's ranks as 16-bit columns start here

typedef unsigned short Half2 __attribute__((ext_vector_type(2)));

// The word of column x in the group kernel's map. The lowest rank is in no
// N+ of these vertices, so its word stays zero, and HUB_NONE has the same.
__device__ __forceinline__ uint32_t grp_word(uint32_t x) { return x % GRP_SPAN; }
static_assert(GRP_OFF % GRP_SPAN == HUB_NONE % GRP_SPAN && GRP_SPAN * 4 == 65536, "16-bit byte addresses");

// Or over the eight lanes of a tail.
__device__ __forceinline__ uint32_t or8(uint32_t x) {
    static_assert(HB_L == 8, "eight lanes per tail");
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0xB1, 0xF, 0xF, true);    // lane ^ 1
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x4E, 0xF, 0xF, true);    // lane ^ 2
    x |= (uint32_t)__builtin_amdgcn_mov_dpp((int)x, 0x141, 0xF, 0xF, true);   // lane -> 7 - lane
    return x;
}

// Elements of this wave's tails that the map holds: S, E = start and end of
// the lane's tail in the 16-bit columns (empty: S >= E).
// GROUP: the map is a word per rank of the group kernel, with a bit per member of
// group g that has the rank as an out-neighbour; a tail starts at its row's first member,
// and an element counts the members that are in the row and have it. The row's members are its
// first elements, at most GRP_N, all in the tail's first step.
template <bool GROUP>
__device__ __forceinline__ uint32_t walk_tails(const uint4* __restrict__ chunks, uint32_t S, uint32_t E,
                                               const void* map, const HubMasks& M, uint32_t g) {
    static_assert(GRP_N + HB_E - 1 <= HB_L * HB_E, "a group's members lie in the first step");
    const uint32_t ln = (uint32_t)lane_id(), gl = ln % HB_L, gi = ln / HB_L;
    // tails in order of length (descending classes), empty ones last
    const uint32_t nch = S < E ? (E - 1u) / HB_E + 1u - S / HB_E : 0u;
    const uint32_t cls = step_class((nch + HB_L - 1) / HB_L);
    uint32_t pos = 0, base = 0, live = 0;
#pragma unroll
    for (int c = HB_CLS - 1; c >= 0; --c) {
        const uint64_t B = __ballot(cls == (uint32_t)c);
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(B >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)B, 0u));
        if (cls == (uint32_t)c) pos = base + below;
        if (c == 0) live = base;
        base += (uint32_t)__popcll(B);
    }
    S = (uint32_t)__builtin_amdgcn_ds_permute((int)(pos * 4u), (int)S);
    E = (uint32_t)__builtin_amdgcn_ds_permute((int)(pos * 4u), (int)E);
    const uint32_t rounds = (live + HB_R - 1) / HB_R;
    // one cursor per lane over (round, chunk); all lanes advance together
    uint32_t r = 0, s = 0, e = 0, c = 0, c1 = 0, issued = 0, hits = 0, own = 0;
    bool fresh = true;   // the cursor is at its tails' first step
    auto fetch = [&]() {
        const int from = (int)(((r * HB_R + gi) & (WAVE - 1)) * 4u);
        s = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)S);
        e = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)E);
        c = s / HB_E + gl;
        c1 = (r < rounds && s < e) ? (e - 1u) / HB_E + 1u : 0u;
    };
    uint4 x[HB_D];
    uint32_t hk[HB_D], tk[HB_D];
    bool fs[HB_D];
    auto issue = [&](int q) {
        const bool on = c < c1;
        x[q] = chunks[on ? c : 0u];   // unconditional: lanes without a chunk read a valid one
        const int h = (int)(s - c * HB_E), t = (int)(c * HB_E + HB_E - e);
        hk[q] = on ? (uint32_t)(h < 0 ? 0 : h) : HB_E;
        tk[q] = on ? (uint32_t)(t < 0 ? 0 : t) : 0u;
        fs[q] = fresh;
        if (r < rounds) ++issued;
        fresh = !__ballot(c + HB_L < c1);
        if (!fresh) c += HB_L;
        else { ++r; fetch(); }
    };
    fetch();
#pragma unroll
    for (int q = 0; q < HB_D; ++q) issue(q);
    for (uint32_t done = 0; done < issued; done += HB_D) {
#pragma unroll
        for (int q = 0; q < HB_D; ++q) {
            const uint4 h = M.head[hk[q]], t = M.tail[tk[q]];
            const uint32_t w[4] = {x[q].x | h.x | t.x, x[q].y | h.y | t.y, x[q].z | h.z | t.z, x[q].w | h.w | t.w};
            if (GROUP) {
                if (fs[q]) {   // the row's members of the group
                    const uint32_t g0 = GRP_OFF + g * GRP_N;
                    uint32_t b = 0;
#pragma unroll
                    for (int k = 0; k < 4; ++k) {
                        const uint32_t lo = (w[k] & 0xFFFFu) - g0, hi = (w[k] >> 16) - g0;
                        b |= (lo < GRP_N ? 1u : 0u) << (lo % GRP_N);
                        b |= (hi < GRP_N ? 1u : 0u) << (hi % GRP_N);
                    }
                    own = or8(b);
                }
#pragma unroll
                for (int k = 0; k < 4; ++k) {
                    // byte addresses of two words at once; the count adds in the bit count itself
                    const uint32_t at = __builtin_bit_cast(uint32_t, __builtin_bit_cast(Half2, w[k]) << (Half2)2);
                    const uint32_t m0 = *(const uint32_t*)((const char*)map + (at & 0xFFFFu)) & own;
                    const uint32_t m1 = *(const uint32_t*)((const char*)map + (at >> 16)) & own;
                    asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(hits) : "v"(m0));
                    asm("v_bcnt_u32_b32 %0, %1, %0" : "+v"(hits) : "v"(m1));
                }
            } else {
                const uint8_t* bytes = (const uint8_t*)map;
#pragma unroll
                for (int k = 0; k < 4; ++k) hits += (uint32_t)bytes[w[k] & 0xFFFFu] + (uint32_t)bytes[w[k] >> 16];
            }
            issue(q);
        }
    }
    return hits;
}

template <bool MIDDLE>
__global__ __launch_bounds__(HB_NT, 2 * HB_W / 4) void k_isect_hub(IsectArgs a, uint64_t* partials) {
    __shared__ __align__(16) uint8_t map[HUB_SPAN + 1];   // map[HUB_NONE] stays zero
    __shared__ HubMasks M;
    __shared__ TileRanges R;
    __shared__ uint32_t s_tile;
    __shared__ uint64_t red[HB_W];
    if (a.hub->hub_pref[NBUCKET] == 0) {   // no tile: not worth the set-up
        if (threadIdx.x == 0) partials[blockIdx.x] = 0;
        return;
    }
    R.load(a.hub->hub_tile, a.hub->hub_pref);
    for (uint32_t i = threadIdx.x; i < (HUB_SPAN + 1) / 16; i += HB_NT) ((uint4*)map)[i] = make_uint4(0, 0, 0, 0);
    M.fill();
    __syncthreads();
    const uint32_t wv = (uint32_t)wave_id(), ln = (uint32_t)lane_id();
    const uint32_t ntile = R.pref[NBUCKET];
    uint64_t acc = 0;
    // this lane's in-edge of tile d: the wave's share is a contiguous range
    auto entry_of = [&](const uint4& d) -> uint64_t {
        const uint32_t lo = d.z * wv / HB_W, hi = d.z * (wv + 1u) / HB_W;
        return lo + ln < hi ? a.csc[d.y + lo + ln] : 0ull;   // tail start | tail end << 32; an empty tail
    };
    uint32_t i = blockIdx.x;
    uint4 d = make_uint4(0, 0, 0, 0);
    uint32_t b0 = 0, b1 = 0;
    uint64_t ent = 0;
    if (i < ntile) {
        d = a.tiles[R.at(i)];   // {v, first in-edge, in-edges, 0}
        ent = entry_of(d);
        b0 = a.off[d.x];
        b1 = a.off[d.x + 1];
    }
    while (i < ntile) {
        for (uint32_t j = b0 + threadIdx.x; j < b1; j += HB_NT) map[a.col16[j]] = 1;
        // the next tile, in flight during this one
        const uint32_t inext = grab_tile(a.ctrl, HUB_COUNTER, gridDim.x, &s_tile);   // barriers: the map is complete
        uint4 dn = d;
        uint64_t ent_n = 0;
        uint32_t b0n = 0, b1n = 0;
        if (inext < ntile) {
            dn = a.tiles[R.at(inext)];
            ent_n = entry_of(dn);
            b0n = a.off[dn.x];
            b1n = a.off[dn.x + 1];
        }
        const uint32_t hits = walk_tails<false>((const uint4*)a.col16, tail_start(ent), tail_end(ent), map, M, 0u);
        acc += hits;
        if (MIDDLE) {   // one update per tile
            const uint64_t t = wave_sum_u64(hits);
            if (ln == 0) red[wv] = t;
        }
        __syncthreads();   // the map has been read
        for (uint32_t j = b0 + threadIdx.x; j < b1; j += HB_NT) map[a.col16[j]] = 0;
        __syncthreads();   // cleared before the next list is set
        if (MIDDLE && threadIdx.x == 0) {
            uint64_t t = 0;
            for (int q = 0; q < HB_W; ++q) t += red[q];
            if (t) atomicAdd((unsigned long long*)&a.per_middle[d.x], (unsigned long long)t);
        }
        i = inext;
        d = dn;
        ent = ent_n;
        b0 = b0n;
        b1 = b1n;
    }
    acc = wave_sum_u64(acc);
    __syncthreads();
    if (ln == 0) red[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int q = 0; q < HB_W; ++q) t += red[q];
        partials[blockIdx.x] = t;
    }
}

// ------------------------------------------------------------------ hub group kernel
// The hub kernel's work (counts in all) for the GRP_SPAN top-ranked vertices, GRP_N consecutive
// ones at a time: a row that holds several members of a group is read once, from its
// first member on, for all of them, instead of once per member (R-MAT 24: 0.49 of the
// elements, 32.6 of 60.0 GB in lines). The map is a word per rank: bit k, where the
// group's k-th vertex has the rank as an out-neighbour. The in-edges of a group are
// contiguous, as its vertices are; those whose row has an earlier member are
// marked (CSC_FOLLOWS) and skipped. A tile is a stretch of grp_edges of them, long
// enough that setting the words of 32 rows (10^4 to 10^5 elements) is small beside it; a wave
// takes 64 in-edges at a time, with no barrier between a tile's set-up and its end.
// Measured with the hub kernel for the ranks below: R-MAT 24 4.9 + 4.6 ms against 12.2 ms of the
// hub kernel alone, R-MAT 20 0.44 + 0.07 against 0.64. Bound at R-MAT 24: line traffic
// beyond L2, 33.5 GB at 6.9 TB/s (the hub kernel: 32.8 GB at 7.1); at R-MAT 20 the
// set-up of many short tiles (rows set one step of loads at a time, tiles from 2048 in-edges: 0.46). Bit counts that add to their accumulator and byte
// addresses made two at a time took it from 5.5 to 5.0 ms.
__global__ __launch_bounds__(HB_NT, 2 * HB_W / 4) void k_isect_group(IsectArgs a, uint64_t* partials) {
    __shared__ __align__(16) uint32_t words[GRP_SPAN];
    __shared__ HubMasks M;
    __shared__ uint32_t s_pref[GRP_COUNT + 1], s_off[GRP_N + 1], s_tile;
    __shared__ uint64_t red[HB_W];
    const uint32_t ntile = a.hub->grp_pref[GRP_COUNT];
    if (blockIdx.x >= ntile) {
        if (threadIdx.x == 0) partials[blockIdx.x] = 0;
        return;
    }
    for (uint32_t i = threadIdx.x; i <= GRP_COUNT; i += HB_NT) s_pref[i] = a.hub->grp_pref[i];
    for (uint32_t i = threadIdx.x; i < GRP_SPAN / 4; i += HB_NT) ((uint4*)words)[i] = make_uint4(0, 0, 0, 0);
    M.fill();
    const uint32_t per = a.hub->grp_edges, first = a.first_rank;
    const uint32_t wv = (uint32_t)wave_id(), ln = (uint32_t)lane_id();
    uint64_t acc = 0;
    __syncthreads();
    for (uint32_t i = blockIdx.x; i < ntile;) {
        uint32_t g = 0;   // the last group whose prefix is at most i
#pragma unroll
        for (uint32_t step = GRP_COUNT / 2; step > 0; step >>= 1)
            if (s_pref[g + step] <= i) g += step;
        const uint32_t v0 = first + g * GRP_N;
        if (threadIdx.x <= GRP_N) s_off[threadIdx.x] = a.off[v0 + threadIdx.x];
        const uint32_t e0 = a.inoff[v0] + (i - s_pref[g]) * per, ee = a.inoff[v0 + GRP_N];
        const uint32_t e1 = ee - e0 < per ? ee : e0 + per, inc = a.hub->grp_inc[g];
        auto entry_at = [&](uint32_t q) -> uint64_t { return q < e1 ? a.csc[q] : CSC_FOLLOWS; };
        uint32_t q = e0 + wv * WAVE + ln;
        uint64_t ent = entry_at(q);
        __syncthreads();
        // the words: eight elements per thread and step, two steps in flight
        const uint32_t b0 = s_off[0], b1 = s_off[GRP_N];
        const uint32_t c1 = (b1 + HB_E - 1u) / HB_E;
        for (uint32_t c = b0 / HB_E + threadIdx.x; c < c1; c += 2 * HB_NT) {
            uint4 x[2];
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) x[u] = ((const uint4*)a.col16)[c + u * HB_NT < c1 ? c + u * HB_NT : c];
#pragma unroll
            for (uint32_t u = 0; u < 2; ++u) {
                const uint32_t j = (c + u * HB_NT) * HB_E;
                if (j >= b1) break;
                const uint32_t w[4] = {x[u].x, x[u].y, x[u].z, x[u].w};
                uint32_t row = 0;   // the last row that starts at or before j
#pragma unroll
                for (uint32_t step = GRP_N / 2; step > 0; step >>= 1)
                    if (s_off[row + step] <= j) row += step;
                uint32_t end = s_off[row + 1];
#pragma unroll
                for (uint32_t k = 0; k < HB_E; ++k) {
                    const uint32_t at = j + k;
                    if (at < b0 || at >= b1) continue;
                    while (end <= at) end = s_off[++row + 1];
                    const uint32_t y = (w[k / 2] >> (16 * (k & 1))) & 0xFFFFu;
                    if ((inc >> row) & 1u) atomicOr(&words[grp_word(y)], 1u << row);
                }
            }
        }
        const uint32_t inext = grab_tile(a.ctrl, GRP_COUNTER, gridDim.x, &s_tile);   // barriers: the words are complete
        while (__ballot(q < e1)) {
            const uint64_t now = ent;
            q += HB_NT;
            ent = entry_at(q);
            const bool lead = !(now & CSC_FOLLOWS);
            acc += walk_tails<true>((const uint4*)a.col16, lead ? tail_start(now) - 1u : 0u,
                                    lead ? tail_end(now) : 0u, words, M, g);
        }
        __syncthreads();   // the words have been read
        for (uint32_t k = threadIdx.x; k < GRP_SPAN / 4; k += HB_NT) ((uint4*)words)[k] = make_uint4(0, 0, 0, 0);
        i = inext;
        // the next tile's barrier stands between these stores and its own
    }
    acc = wave_sum_u64(acc);
    if (ln == 0) red[wv] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t t = 0;
        for (int k = 0; k < HB_W; ++k) t += red[k];
        partials[blockIdx.x] = t;
    }
}

// ------------------------------------------------------------------ wave kernel
// The bitmap strategy for vertices of few in-edges (several of them to a tile of the
// bitmap kernel; counts in all or per middle vertex): a wave per vertex and no barrier, as
// there a block's time goes to the chain of set-up loads, barriers and windows
// of one vertex after the other. N+(v) is a table of 15-bit tags (rank / WV_SLOTS) at
// slot rank % WV_SLOTS, so that one probe answers for ranks of any distance and there
// are no windows. A rank whose slot is taken goes to a small open table of whole
// ranks, and the slot's top bit says so: a probe that meets another tag with that
// bit set looks there. N+(v) is taken in parts where that table would fill up.
// Eight lanes walk a tail together, a 16-byte chunk per lane and step.
// R-MAT 24: the bitmap kernel's remaining 9.6 ms -> 3.6 ms for it and 1.7 here (11.5 GB at
// 6.5 TB/s; the bitmap kernel now 26 GB at 7.2, the traffic limit); a batch of
// Chung-Lu graphs 3.0 -> 1.4 + 0.6 ms. Which vertices: those of fewer than 1024 in-edges in
// buckets without a hub tile (fewer than 128, 256, 512, 1024, 2048, 8192: R-MAT 24 38.6,
// 38.5, 38.4, 38.4, 38.4, 38.5 ms, the batch 22.6, 22.2, 22.2, 22.0, 21.9, 22.0). The part
// of such a bucket below the hub ranks was slower here (38.8 ms): middle lists of
// up to 1000 elements, in several parts.
constexpr int WV_NT = 256, WV_W = WV_NT / WAVE, WV_D = 3;
constexpr uint32_t WV_OVF = 256, WV_E = 4;   // whole ranks; elements per chunk
constexpr uint32_t WV_FLAG = 0x8000u;

struct WaveSet {
    uint16_t tag[WV_SLOTS];
    uint32_t ovf[WV_OVF];
};
__device__ __forceinline__ void wave_order() { __builtin_amdgcn_fence(__ATOMIC_SEQ_CST, "wavefront"); }
__device__ __forceinline__ uint32_t ovf_slot(uint32_t x) { return (x / WV_SLOTS * 37u + x) % WV_OVF; }

// Elements of this wave's tails that the set holds; S, E as in walk_tails, in the columns.
__device__ __forceinline__ uint32_t walk_set(const uint4* __restrict__ chunks, uint32_t S, uint32_t E,
                                             const WaveSet& set) {
    const uint32_t ln = (uint32_t)lane_id(), gl = ln % HB_L, gi = ln / HB_L;
    const uint32_t nch = S < E ? (E - 1u) / WV_E + 1u - S / WV_E : 0u;
    const uint32_t cls = step_class((nch + HB_L - 1) / HB_L);
    uint32_t pos = 0, base = 0, live = 0;
#pragma unroll
    for (int c = HB_CLS - 1; c >= 0; --c) {
        const uint64_t B = __ballot(cls == (uint32_t)c);
        const uint32_t below =
            __builtin_amdgcn_mbcnt_hi((uint32_t)(B >> 32), __builtin_amdgcn_mbcnt_lo((uint32_t)B, 0u));
        if (cls == (uint32_t)c) pos = base + below;
        if (c == 0) live = base;
        base += (uint32_t)__popcll(B);
    }
    S = (uint32_t)__builtin_amdgcn_ds_permute((int)(pos * 4u), (int)S);
    E = (uint32_t)__builtin_amdgcn_ds_permute((int)(pos * 4u), (int)E);
    const uint32_t rounds = (live + HB_R - 1) / HB_R;
    uint32_t r = 0, s = 0, e = 0, c = 0, c1 = 0, issued = 0, hits = 0;
    auto fetch = [&]() {
        const int from = (int)(((r * HB_R + gi) & (WAVE - 1)) * 4u);
        s = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)S);
        e = (uint32_t)__builtin_amdgcn_ds_bpermute(from, (int)E);
        c = s / WV_E + gl;
        c1 = (r < rounds && s < e) ? (e - 1u) / WV_E + 1u : 0u;
    };
    uint4 x[WV_D];
    uint32_t at[WV_D], len[WV_D];   // of the chunk's first element in the tail (modular); the tail's length
    auto issue = [&](int q) {
        const bool on = c < c1;
        x[q] = chunks[on ? c : 0u];   // unconditional: lanes without a chunk read a valid one
        at[q] = c * WV_E - s;
        len[q] = on ? e - s : 0u;
        if (r < rounds) ++issued;
        if (__ballot(c + HB_L < c1)) c += HB_L;
        else { ++r; fetch(); }
    };
    fetch();
#pragma unroll
    for (int q = 0; q < WV_D; ++q) issue(q);
    for (uint32_t done = 0; done < issued; done += WV_D) {
#pragma unroll
        for (int q = 0; q < WV_D; ++q) {
            const uint32_t w[WV_E] = {x[q].x, x[q].y, x[q].z, x[q].w};
            uint32_t y[WV_E];
#pragma unroll
            for (uint32_t k = 0; k < WV_E; ++k) y[k] = set.tag[w[k] % WV_SLOTS];
            bool other = false;
#pragma unroll
            for (uint32_t k = 0; k < WV_E; ++k) {
                const bool in = at[q] + k < len[q];
                y[k] = in ? y[k] ^ (w[k] / WV_SLOTS) : 1u;
                hits += (y[k] & WV_TAG) == 0u ? 1u : 0u;
                other |= y[k] > WV_FLAG;   // another tag, and the slot has overflowed
            }
            if (__ballot(other)) {
#pragma unroll
                for (uint32_t k = 0; k < WV_E; ++k) {
                    if (y[k] <= WV_FLAG) continue;
                    uint32_t h = ovf_slot(w[k]), o;
                    while ((o = set.ovf[h]) != ~0u && o != w[k]) h = (h + 1u) % WV_OVF;
                    hits += o == w[k] ? 1u : 0u;
                }
            }
            issue(q);
        }
    }
    return hits;
}

template <bool MIDDLE>
__global__ __launch_bounds__(WV_NT, 6) void k_isect_wave(IsectArgs a, uint64_t* partials) {
    __shared__ __align__(16) WaveSet sets[WV_W];
    __shared__ uint32_t s_pos[NBUCKET], s_pref[NBUCKET + 1];
    const uint32_t total = a.hub->wave_pref[NBUCKET];
    for (uint32_t i = threadIdx.x; i < (uint32_t)NBUCKET; i += WV_NT) s_pos[i] = a.hub->wave_pos[i];
    for (uint32_t i = threadIdx.x; i <= (uint32_t)NBUCKET; i += WV_NT) s_pref[i] = a.hub->wave_pref[i];
    __syncthreads();
    const uint32_t ln = (uint32_t)lane_id();
    WaveSet& set = sets[wave_id()];
    const uint32_t stride = gridDim.x * WV_W;
    uint32_t i = (uint32_t)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * WV_W + (uint32_t)wave_id()));
    auto vertex = [&](uint32_t q) -> uint32_t {   // of place q of the ranges
        if (q >= total) return 0u;
        uint32_t r = 0;
#pragma unroll
        for (int k = 0; k < NBUCKET / WAVE; ++k) r += (uint32_t)__popcll(__ballot(s_pref[k * WAVE + ln] <= q));
        return a.vlist[s_pos[r - 1u] + (q - s_pref[r - 1u])];
    };
    for (uint32_t k = ln; k < WV_OVF; k += WAVE) set.ovf[k] = ~0u;
    uint64_t acc = 0;
    uint32_t v = vertex(i), vn = vertex(i + stride);
    uint32_t b0 = a.off[v], b1 = a.off[v + 1], e0 = a.inoff[v], e1 = a.inoff[v + 1];
    for (; i < total; i += stride) {
        // the next vertex's bounds and the one after it, in flight during this one
        const uint32_t nb0 = a.off[vn], nb1 = a.off[vn + 1], ne0 = a.inoff[vn], ne1 = a.inoff[vn + 1];
        const uint32_t vnn = vertex(i + 2u * stride);
        uint64_t ent = e0 + ln < e1 ? a.csc[e0 + ln] : 0ull;
        uint32_t hits = 0;
        for (uint32_t b = b0; b < b1;) {   // parts of N+(v)
            for (uint32_t k = ln; k < WV_SLOTS * 2 / 16; k += WAVE)
                ((uint4*)set.tag)[k] = make_uint4(0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu, 0x7FFF7FFFu);
            uint32_t over = 0;
            do {
                const uint32_t x = b + ln < b1 ? a.col[b + ln] : ~0u;
                const bool on = x != ~0u;
                const uint32_t sl = x % WV_SLOTS, tg = x / WV_SLOTS;
                wave_order();
                const bool free = on && set.tag[sl] == WV_TAG;
                wave_order();
                if (free) set.tag[sl] = (uint16_t)tg;
                wave_order();
                const uint32_t now = set.tag[sl];
                const bool lost = on && !(free && now == tg);   // ranks are distinct: one lane per slot has its tag there
                wave_order();
                if (lost) {
                    set.tag[sl] = (uint16_t)(now | WV_FLAG);
                    uint32_t h = ovf_slot(x);
                    while (atomicCAS(&set.ovf[h], ~0u, x) != ~0u) h = (h + 1u) % WV_OVF;
                }
                over += (uint32_t)__popcll(__ballot(lost));
                b += WAVE;
            } while (b < b1 && over <= WV_OVF / 2);   // a step adds at most 64
            wave_order();
            for (uint32_t q = e0;;) {
                hits += walk_set((const uint4*)a.col, tail_start(ent), tail_end(ent), set);
                if (e1 - e0 <= (uint32_t)WAVE) break;
                q += WAVE;
                if (q >= e1) {
                    ent = a.csc[e0 + ln];
                    break;
                }
                ent = q + ln < e1 ? a.csc[q + ln] : 0ull;
            }
            if (over) {
                wave_order();
                for (uint32_t k = ln; k < WV_OVF; k += WAVE) set.ovf[k] = ~0u;
            }
            wave_order();
        }
        acc += hits;
        if (MIDDLE) {
            const uint64_t t = wave_sum_u64(hits);
            if (ln == 0 && t) a.per_middle[v] += t;   // this wave has all of v
        }
        v = vn;
        vn = vnn;
        b0 = nb0;
        b1 = nb1;
        e0 = ne0;
        e1 = ne1;
    }
    block_partial(acc, partials);
}

// ------------------------------------------------------------------ shared helpers for edge-centric kernels
// Outputs of a launch: none that is written per triangle (T, per edge, per middle
// vertex); any; t[v] through LDS counters; none on whole-row ranges (a kernel of its own, as an
// end that may or may not carry the group mark cost the merge kernel of the random
// geometric graph of 2^23 vertices its schedule: the call 14.64 -> 14.76 ms).
enum { EM_COUNT = 0, EM_ANY = 1, EM_VERTEX = 2, EM_WHOLE = 3 };
constexpr bool em_counts(int mode) { return mode == EM_COUNT || mode == EM_WHOLE; }
// A tail of up to this many times N+(v) is searched in N+(v), which is mostly in
// LDS; where every in-edge took the shorter of its two lists, a wave ran both searches
// one after the other (1, 2, 4, 8: random geometric graph of 2^23 vertices 16.1, 14.7, 14.6,
// 14.6 ms; R-MAT 24 36.0, 35.7, 35.6, 35.6; a batch 19.9, 19.5, 19.5, 19.5).
constexpr uint32_t SEARCH_LONGER = 4;
// Number of elements of A taken in the first d outputs of the merge of A and
// B, A first on ties (merge-path split, Green et al. / Odeh et al.).
__device__ __forceinline__ uint32_t merge_split(const uint32_t* A, uint32_t na, const uint32_t* B, uint32_t nb,
                                                uint32_t d) {
    uint32_t lo = d > nb ? d - nb : 0u;
    uint32_t hi = d < na ? d : na;
    while (lo < hi) {
        const uint32_t mid = (lo + hi) >> 1;
        if (A[mid] <= B[d - 1u - mid]) lo = mid + 1u;
        else hi = mid;
    }
    return lo;
}

// Segment holding flattened in-edge q (largest sg with pref[sg] <= q).
__device__ __forceinline__ uint32_t find_seg(const Segs& S, uint32_t nseg, uint32_t q) {
    uint32_t lo = 0, hi = nseg - 1;
    while (lo < hi) {
        const uint32_t mid = (lo + hi + 1) >> 1;
        if (S.pref[mid] <= q) lo = mid;
        else hi = mid - 1;
    }
    return lo;
}

// Elements X[q] (q = gl, gl + g, ...) of one list searched in the ascending
// list Y (ny > 0) by a group of g lanes: four elements per lane at a time, as
// four interleaved branch-free searches for the last element not above (halving the range
// each step), so that every step issues four independent loads. Returns the matches; a
// match at X[q] = Y[p] is edge ex0 + q and edge ey0 + p. Bound by its instructions:
// without the outputs' branches, with one read after the search instead of two, the geometric
// graph's call went from 16.9 to 16.1 ms.
template <int MODE>
__device__ __forceinline__ uint32_t search_list(const IsectArgs& a, const Hot& hot, const uint32_t* X, uint32_t nx,
                                                const uint32_t* Y, uint32_t ny, uint32_t g, uint32_t gl,
                                                uint32_t ex0, uint32_t ey0, uint32_t ein) {
    uint32_t c = 0;
    if (ny == 0) return 0;
    for (uint32_t q0 = gl; q0 < nx; q0 += 4u * g) {
        uint32_t xv[4], bs[4];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t q = q0 + (uint32_t)u * g;
            xv[u] = X[q < nx ? q : nx - 1u];
            bs[u] = 0;
        }
        for (uint32_t len = ny; len > 1;) {
            const uint32_t half = len >> 1;
            uint32_t yv[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) yv[u] = Y[bs[u] + half];
#pragma unroll
            for (int u = 0; u < 4; ++u) bs[u] = yv[u] <= xv[u] ? bs[u] + half : bs[u];
            len -= half;
        }
        uint32_t y0[4];   // bs = last position not above x, or 0
#pragma unroll
        for (int u = 0; u < 4; ++u) y0[u] = Y[bs[u]];
#pragma unroll
        for (int u = 0; u < 4; ++u) {
            const uint32_t q = q0 + (uint32_t)u * g;
            const bool is = q < nx && y0[u] == xv[u];
            if (em_counts(MODE)) {
                c += is ? 1u : 0u;
            } else if (is) {
                ++c;
                hit(a, hot, xv[u], ex0 + q, ey0 + bs[u], ein);
            }
        }
    }
    return c;
}

// One in-edge by a group of g lanes: merge path (MERGE) or binary search.
// ea0, eb0: CSR positions of A[0] (the tail) and B[0] (N+(v)); the in-edge
// itself sits just before its tail, at ea0 - 1.
template <bool MERGE, int MODE>
__device__ __forceinline__ uint32_t isect_edge(const IsectArgs& a, const Hot& hot, const uint32_t* A, uint32_t na, const uint32_t* B,
                                               uint32_t nb, uint32_t g, uint32_t gl, uint32_t ea0, uint32_t eb0) {
    uint32_t c = 0;
    if (MERGE) {
        // The lane's diagonal range [d0, d1) of the merge path consumes the A
        // elements [i0, i1); each A element is consumed by exactly one lane and
        // counts when it equals the B head at that point, which (B ascending)
        // is the first B element not below it. So the lane walks its A
        // elements, four loaded at a time, with a monotone cursor into B that
        // starts at the diagonal's B position d0 - i0.
        const uint32_t tot = na + nb;
        const uint32_t d0 = (uint32_t)(((uint64_t)tot * gl) / g);
        const uint32_t d1 = (uint32_t)(((uint64_t)tot * (gl + 1u)) / g);
        const uint32_t i0 = merge_split(A, na, B, nb, d0);
        const uint32_t i1 = merge_split(A, na, B, nb, d1);
        uint32_t j = d0 - i0;
        for (uint32_t i = i0; i < i1; i += 4u) {
            uint32_t av[4];
#pragma unroll
            for (int u = 0; u < 4; ++u) av[u] = A[i + u < i1 ? i + u : i1 - 1u];
#pragma unroll
            for (int u = 0; u < 4; ++u) {
                if (i + u >= i1) break;
                while (j < nb && B[j] < av[u]) ++j;
                if (j < nb && B[j] == av[u]) {
                    ++c;
                    if (!em_counts(MODE)) hit(a, hot, av[u], ea0 + i + u, eb0 + j, ea0 - 1u);
                }
            }
        }
    } else if (na <= SEARCH_LONGER * nb) {
        c = search_list<MODE>(a, hot, A, na, B, nb, g, gl, ea0, eb0, ea0 - 1u);   // tail elements searched in N+(v)
    } else {
        c = search_list<MODE>(a, hot, B, nb, A, na, g, gl, eb0, ea0, ea0 - 1u);   // N+(v) searched in the tail
    }
    return c;
}

template <bool MERGE, int MODE>
__global__ __launch_bounds__(IS_NT, MODE == EM_VERTEX ? 4 : (MERGE ? 7 : 6)) void k_isect_edges(IsectArgs a,
                                                                                              uint64_t* partials) {
    constexpr bool VERTEX = MODE == EM_VERTEX;
    __shared__ uint32_t s_hot[VERTEX ? HOT_N : 1];
    const Hot hot = {VERTEX ? s_hot : nullptr, a.hot_first};
    if (VERTEX) hot.clear();   // the first tile's barriers follow
    __shared__ uint32_t sb[STAGE_MAX];
    __shared__ uint32_t s_boff[SEG_MAX + 1];
    __shared__ Segs S;
    constexpr int KER = MERGE ? KER_MERGE : KER_BSEARCH;
    uint64_t acc = 0;
    __shared__ uint32_t s_tile;
    const uint32_t t_begin = a.ctrl->tile_begin[KER], t_end = a.ctrl->tile_begin[KER + 1];
    for (uint32_t t = t_begin + blockIdx.x; t < t_end; t = grab_tile(a.ctrl, KER, t_begin + gridDim.x, &s_tile)) {
        const uint32_t nseg = load_tile(a, t, S);
        const uint32_t v0 = S.v[0];
        // stage the N+(v) lists of all the tile's vertices back to back when they fit
        uint32_t dl = 0;
        if (threadIdx.x < nseg) dl = a.off[S.v[threadIdx.x] + 1] - a.off[S.v[threadIdx.x]];
        uint32_t TB;
        const uint32_t bex = block_exclusive_scan<IS_NT>(dl, S.scratch, &TB);
        if (threadIdx.x < nseg) s_boff[threadIdx.x] = bex;
        if (threadIdx.x == 0) s_boff[nseg] = TB;
        __syncthreads();
        const bool staged = TB <= (uint32_t)STAGE_MAX;
        if (staged) {
            for (uint32_t j = threadIdx.x; j < TB; j += IS_NT) {
                uint32_t lo2 = 0, hi2 = nseg - 1;   // segment holding list position j
                while (lo2 < hi2) {
                    const uint32_t mid = (lo2 + hi2 + 1) >> 1;
                    if (s_boff[mid] <= j) lo2 = mid;
                    else hi2 = mid - 1;
                }
                sb[j] = a.col[a.off[S.v[lo2]] + (j - s_boff[lo2])];
            }
        }
        __syncthreads();
        const uint32_t g = a.ctrl->group[a.vbucket[v0]];            // lanes per in-edge (power of 2)
        const uint32_t gi = threadIdx.x / g, gl = threadIdx.x % g;  // group index, lane in group
        const uint32_t ngroups = IS_NT / g;
        const uint32_t ne = S.pref[nseg];
        const uint32_t rounds = (ne + ngroups - 1) / ngroups;
        // each round's in-edge entry (tail start | end << 32) is loaded one round ahead,
        // so that its latency overlaps the intersection before it
        uint32_t sg_next = 0;
        uint64_t ent_next = 0;
        if (gi < ne) {
            sg_next = nseg == 1 ? 0u : find_seg(S, nseg, gi);
            ent_next = a.csc[S.e0[sg_next] + (gi - S.pref[sg_next])];
        }
        for (uint32_t r = 0; r < rounds; ++r) {
            const uint32_t q = r * ngroups + gi;
            const uint32_t sg = sg_next;
            const uint64_t ent = ent_next;
            const uint32_t qn = q + ngroups;
            if (qn < ne) {
                sg_next = nseg == 1 ? 0u : find_seg(S, nseg, qn);
                ent_next = a.csc[S.e0[sg_next] + (qn - S.pref[sg_next])];
            }
            uint32_t c = 0, e = 0, v = 0;
            if (q < ne) {
                v = S.v[sg];
                const uint32_t s = tail_start(ent), end = tail_end(ent, MODE == EM_WHOLE);
                e = s - 1u;
                const uint32_t nb = s_boff[sg + 1] - s_boff[sg];
                const uint32_t bo = a.off[v];
                // two call sites, so that each knows whether N+(v) is in LDS or in global memory
                if (staged) c = isect_edge<MERGE, MODE>(a, hot, a.col + s, end - s, sb + s_boff[sg], nb, g, gl, s, bo);
                else c = isect_edge<MERGE, MODE>(a, hot, a.col + s, end - s, a.col + bo, nb, g, gl, s, bo);
            }
            // reduce within the group of g lanes (g divides the wave)
            for (uint32_t o = g >> 1; o > 0; o >>= 1) c += __shfl_xor(c, (int)o, WAVE);
            if (q < ne && gl == 0) {
                acc += c;
                if (!em_counts(MODE) || a.per_edge || a.per_middle) edge_done(a, hot, e, v, c);
            }
        }
        __syncthreads();
    }
    if (VERTEX) {
        __syncthreads();
        hot.flush(a);
    }
    block_partial(acc, partials);
}

// Sum of the per-block partial counts of the stage's kernels, in a fixed order.
constexpr int RED_NT = 1024;
__global__ __launch_bounds__(RED_NT) void k_reduce_total(const uint64_t* __restrict__ partials, IsectParts parts,
                                                         Ctrl* ctrl, uint64_t* result, uint64_t range_status,
                                                         uint64_t internal_status) {
    __shared__ uint64_t red[RED_NT / WAVE];
    uint64_t acc = 0;
    for (int q = 0; q < parts.launches; ++q)
        for (uint32_t i = threadIdx.x; i < parts.n[q]; i += RED_NT) acc += partials[parts.first[q] + i];
    acc = wave_sum_u64(acc);
    if (lane_id() == 0) red[wave_id()] = acc;
    __syncthreads();
    if (threadIdx.x == 0) {
        uint64_t s = 0;
        for (int i = 0; i < RED_NT / WAVE; ++i) s += red[i];
        ctrl->total = s;
        if (result) {
            result[0] = s;
            result[1] = (ctrl->err & 1u) ? range_status : (ctrl->err ? internal_status : 0ull);
        }
    }
}

// ------------------------------------------------------------------ launchers
static int g_num_cu = 0;

static int num_cu() {
    if (!g_num_cu) {
        int dev = 0;
        (void)hipGetDevice(&dev);
        hipDeviceProp_t p;
        if (hipGetDeviceProperties(&p, dev) == hipSuccess) g_num_cu = p.multiProcessorCount;
        if (g_num_cu <= 0) g_num_cu = 256;
    }
    return g_num_cu;
}

// Persistent grids: as many blocks as the CUs hold at once (LDS and registers
// decide), so that no block starts late and stretches the tail.
static int resident_blocks(const void* fn, int threads = IS_NT) {
    int b = 0;
    if (hipOccupancyMaxActiveBlocksPerMultiprocessor(&b, fn, threads, 0) != hipSuccess || b <= 0) b = 1;
    return b;
}

static int bitmap_mode(const IsectArgs& a) {
    if (a.clip) return BM_CLIP;   // whole-row tails: counts only
    if (a.list_out) return BM_LIST;
    if (a.support) return BM_SUPPORT;   // never with per-vertex counts
    if (a.per_vertex) return BM_VERTEX;
    if (a.per_edge) return BM_ENTRY;
    if (a.per_middle) return BM_MIDDLE;
    return BM_COUNT;
}

static const void* bitmap_fn(int mode, bool narrow) {
    switch (mode) {
        case BM_LIST: return narrow ? (const void*)k_isect_bitmap<BM_LIST, true>
                                    : (const void*)k_isect_bitmap<BM_LIST, false>;
        case BM_VERTEX: return narrow ? (const void*)k_isect_bitmap<BM_VERTEX, true>
                                      : (const void*)k_isect_bitmap<BM_VERTEX, false>;
        case BM_SUPPORT: return narrow ? (const void*)k_isect_bitmap<BM_SUPPORT, true>
                                       : (const void*)k_isect_bitmap<BM_SUPPORT, false>;
        case BM_ENTRY: return narrow ? (const void*)k_isect_bitmap<BM_ENTRY, true>
                                     : (const void*)k_isect_bitmap<BM_ENTRY, false>;
        case BM_MIDDLE: return narrow ? (const void*)k_isect_bitmap<BM_MIDDLE, true>
                                      : (const void*)k_isect_bitmap<BM_MIDDLE, false>;
        case BM_CLIP: return narrow ? (const void*)k_isect_bitmap<BM_CLIP, true>
                                    : (const void*)k_isect_bitmap<BM_CLIP, false>;
        default: return narrow ? (const void*)k_isect_bitmap<BM_COUNT, true>
                               : (const void*)k_isect_bitmap<BM_COUNT, false>;
    }
}

int isect_blocks_per_cu(int ker, int mode) {
    static int cache[NKERNEL][BM_NMODE] = {};
    int& c = cache[ker][mode];
    if (!c) {
        const bool vertex = mode == BM_VERTEX;
        const void* fn = ker == KER_MERGE ? (const void*)k_isect_edges<true, EM_ANY>
                         : ker == KER_BSEARCH ? (vertex ? (const void*)k_isect_edges<false, EM_VERTEX>
                                                        : (const void*)k_isect_edges<false, EM_ANY>)
                                              : bitmap_fn(mode, true);
        c = resident_blocks(fn);
    }
    return c;
}

uint32_t isect_hot_first(uint32_t n) { return n > HOT_N ? n - HOT_N : 0u; }

int isect_group_blocks() {
    static int blocks = 0;
    if (!blocks) {
        const int b = num_cu() * resident_blocks((const void*)k_isect_group, HB_NT);
        blocks = b < PARTIALS_PER_KERNEL - HB_PARTIAL1 ? b : PARTIALS_PER_KERNEL - HB_PARTIAL1;
    }
    return blocks;
}

size_t isect_partials_bytes() { return sizeof(uint64_t) * NKERNEL * PARTIALS_PER_KERNEL; }

void launch_isect(int ker, const IsectArgs& a, int grid, uint64_t* partials, hipStream_t s, IsectParts* parts) {
    const int mode = ker == KER_BITMAP ? bitmap_mode(a) : (a.per_vertex ? BM_VERTEX : BM_COUNT);
    if (grid <= 0) grid = num_cu() * isect_blocks_per_cu(ker, mode);
    const bool hub = ker == KER_BITMAP && a.hub;
    const int cap = hub ? WV_PARTIAL0 : PARTIALS_PER_KERNEL;
    if (grid > cap) grid = cap;
    uint64_t* p = partials + (size_t)ker * PARTIALS_PER_KERNEL;
    const bool plain = !a.support && !a.per_vertex && !a.list_out;
    auto note = [&](uint32_t first, int n) {   // every block of a launch writes its partial
        if (!parts) return;
        parts->first[parts->launches] = (uint32_t)(p - partials) + first;
        parts->n[parts->launches++] = (uint32_t)n;
    };
    note(0, grid);
    if (hub) {
        static int per_cu = 0;
        if (!per_cu) per_cu = resident_blocks((const void*)k_isect_hub<false>, HB_NT);
        int hg = num_cu() * per_cu;
        if (hg > HB_PARTIAL1 - HB_PARTIAL0) hg = HB_PARTIAL1 - HB_PARTIAL0;
        note(HB_PARTIAL0, hg);
        if (a.per_middle)
            hipLaunchKernelGGL(k_isect_hub<true>, dim3(hg), dim3(HB_NT), 0, s, a, p + HB_PARTIAL0);
        else
            hipLaunchKernelGGL(k_isect_hub<false>, dim3(hg), dim3(HB_NT), 0, s, a, p + HB_PARTIAL0);
        if (a.waves) {
            static int wave_cu[2] = {0, 0};
            const int md = a.per_middle ? 1 : 0;
            if (!wave_cu[md])
                wave_cu[md] = resident_blocks(md ? (const void*)k_isect_wave<true> : (const void*)k_isect_wave<false>, WV_NT);
            int wg = num_cu() * wave_cu[md];
            if (wg > HB_PARTIAL0 - WV_PARTIAL0) wg = HB_PARTIAL0 - WV_PARTIAL0;
            note(WV_PARTIAL0, wg);
            if (md) hipLaunchKernelGGL(k_isect_wave<true>, dim3(wg), dim3(WV_NT), 0, s, a, p + WV_PARTIAL0);
            else hipLaunchKernelGGL(k_isect_wave<false>, dim3(wg), dim3(WV_NT), 0, s, a, p + WV_PARTIAL0);
        }
        if (a.groups) {
            const int gg = isect_group_blocks();
            note(HB_PARTIAL1, gg);
            hipLaunchKernelGGL(k_isect_group, dim3(gg), dim3(HB_NT), 0, s, a, p + HB_PARTIAL1);
        }
    }
    switch (ker) {
        case KER_MERGE:
            if (a.clip) hipLaunchKernelGGL((k_isect_edges<true, EM_WHOLE>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            else if (plain) hipLaunchKernelGGL((k_isect_edges<true, EM_COUNT>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            else hipLaunchKernelGGL((k_isect_edges<true, EM_ANY>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            break;
        case KER_BSEARCH:
            if (a.clip) hipLaunchKernelGGL((k_isect_edges<false, EM_WHOLE>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            else if (plain) hipLaunchKernelGGL((k_isect_edges<false, EM_COUNT>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            else if (a.per_vertex) hipLaunchKernelGGL((k_isect_edges<false, EM_VERTEX>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            else hipLaunchKernelGGL((k_isect_edges<false, EM_ANY>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            break;
        default: {
            const bool nw = a.col_narrow != 0;
            if (mode == BM_LIST) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_LIST, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_LIST, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else if (mode == BM_VERTEX) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_VERTEX, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_VERTEX, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else if (mode == BM_SUPPORT) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_SUPPORT, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_SUPPORT, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else if (mode == BM_CLIP) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_CLIP, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_CLIP, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else if (mode == BM_MIDDLE) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_MIDDLE, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_MIDDLE, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else if (mode == BM_ENTRY) {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_ENTRY, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_ENTRY, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            } else {
                if (nw) hipLaunchKernelGGL((k_isect_bitmap<BM_COUNT, true>), dim3(grid), dim3(IS_NT), 0, s, a, p);
                else hipLaunchKernelGGL((k_isect_bitmap<BM_COUNT, false>), dim3(grid), dim3(IS_NT), 0, s, a, p);
            }
            break;
        }
    }
}

void launch_reduce_total(const uint64_t* partials, const IsectParts& parts, Ctrl* ctrl, uint64_t* result,
                         uint64_t range_status, uint64_t internal_status, hipStream_t s) {
    hipLaunchKernelGGL(k_reduce_total, dim3(1), dim3(RED_NT), 0, s, partials, parts, ctrl, result, range_status,
                       internal_status);
}

}  // namespace tcx
