// tgl_mfg.hip -- one hop's sampled slots as a message-flow-graph block in
// compressed sparse column form (Algorithm 1 of TGL ends every layer with
// "generate DGL MFGs"; the sampler breakdown of Section 4 counts that step as
// "Oth.").
//
// The block is a relabelling of the slot arrays: destinations are the hop's
// groups, edges its valid slots, sources the destinations followed by one
// temporal node per edge.  Its one non-local quantity is each group's first
// edge, the exclusive scan of the per-group valid counts, so the export is
// three passes that never leave the device: per-group valid counts, scanned
// within tiles of groups (with the destination nodes and the tile totals),
// the scan of the tile totals, and a copy of the valid slots, which also
// writes each group's first edge (indptr).  A group's valid slots are a
// prefix of its k slots (tgl_sample fills a group newest-first or
// all-or-nothing); slots after a group's first PAD are not exported.
#include "tgl_internal.hpp"

namespace tgl {
namespace {

// G = min(count * windows, cap), from the device count
__device__ __forceinline__ int64_t mfg_groups(const int64_t *count, int64_t windows, int64_t cap) {
    int64_t c = *count;
    c = c < 0 ? 0 : c;
    return c > cap / windows ? cap : c * windows;
}

// Groups per tile of the count pass: 1024, or 256 for hops of at most 2^20
// groups, whose tile totals are few enough for one block to scan.  18,000
// groups of 10 slots take 6 us on 256 (16 us on 9 blocks with 2048); 3.9M of a
// capacity of 7.7M take 95 us on 512 plus 28 for the totals' scan, 90 plus 11
// on 1024, 104 plus 5 on 2048.
constexpr int kTileMost = 4 * kBlock;
constexpr int kTileLeast = kBlock;
constexpr int64_t kSmallGroups = int64_t(1) << 20;

int tile_groups(int64_t groups_cap) { return groups_cap <= kSmallGroups ? kTileLeast : kTileMost; }

// A group as the scatter reads it: its first edge within the tile (below
// kTileMost * TGL_MAX_FANOUT = 2^20) and its valid slots (at most 2^10).
constexpr int kCountBits = 11;
static_assert(TGL_MAX_FANOUT < (1 << kCountBits) &&
                  int64_t(kTileMost) * TGL_MAX_FANOUT <= int64_t(1) << (32 - kCountBits),
              "offset and count share 32 bits");

// floor(v / k) with recip = floor(2^64 / k) + 1 (k > 1), exact for v < 2^54
__device__ __forceinline__ int64_t group_of(int64_t v, int32_t k, uint64_t recip) {
    return k == 1 ? v : static_cast<int64_t>(__umul64hi(static_cast<uint64_t>(v), recip));
}

// Pass 1, one tile of GPT * kBlock groups per block.  (A lane per group, eight
// slots at a time, took 82 us, and the offsets another pass of 36 us: the
// blocks of both hops of a 768,000-root citation step 477 -> 439 us, of a
// 1,800-root batch 50 -> 27 us.)  The tile's slots are
// read in order, neighbouring lanes neighbouring slots, kCountUnroll rounds in
// flight; a PAD slot whose predecessor in the group is valid (or that comes
// first) bounds the group's prefix.  Then thread t owns groups GPT t ... of
// the tile: their counts, scanned over the tile, and the tile's edge total.
// Last, the destination nodes (hop 1: the group's root; later hops: the
// previous hop's slot it came from).
constexpr int kCountUnroll = 8;
template <int GPT>
__global__ __launch_bounds__(kBlock) void mfg_count_kernel(const int32_t *__restrict__ nbr, int32_t k, uint64_t recip,
                                                           const int32_t *__restrict__ roots,
                                                           const float *__restrict__ root_ts, int32_t windows,
                                                           const int32_t *__restrict__ prev_nbr,
                                                           const float *__restrict__ prev_ts,
                                                           const int64_t *__restrict__ parent,
                                                           const int64_t *__restrict__ count, int64_t cap,
                                                           int64_t *__restrict__ sizes, uint32_t *__restrict__ packed,
                                                           int64_t *__restrict__ partials,
                                                           int32_t *__restrict__ src_nid, float *__restrict__ src_ts) {
    constexpr int kTile = GPT * kBlock;
    __shared__ uint32_t lds[kBlock / kWave];
    __shared__ int32_t s_cnt[kTile];
    const int64_t G = mfg_groups(count, windows, cap);
    if (blockIdx.x == 0 && threadIdx.x == 0) sizes[0] = G;
    const int64_t tile0 = static_cast<int64_t>(blockIdx.x) * kTile;
    const int ng = G <= tile0 ? 0 : (G - tile0 < kTile ? static_cast<int>(G - tile0) : kTile);
    if (ng == 0) {                                  // block-uniform: past the groups
        if (threadIdx.x == 0) partials[blockIdx.x] = 0;
        return;
    }
#pragma unroll
    for (int i = 0; i < GPT; i++) s_cnt[i * kBlock + threadIdx.x] = k;
    __syncthreads();
    const int32_t *const sl = nbr + tile0 * k;
    const int n = ng * k;                           // at most 2^20
    for (int i0 = 0; i0 < n; i0 += kCountUnroll * kBlock) {
        int32_t v[kCountUnroll], before[kCountUnroll];
#pragma unroll
        for (int u = 0; u < kCountUnroll; u++) {
            const int i = i0 + u * kBlock + static_cast<int>(threadIdx.x);
            v[u] = sl[i < n ? i : n - 1];           // clamped: loads issue together
        }
        // a wavefront's first lane reads its predecessor itself
#pragma unroll
        for (int u = 0; u < kCountUnroll; u++) {
            const int i = i0 + u * kBlock + static_cast<int>(threadIdx.x);
            before[u] = __shfl_up(v[u], 1, kWave);
            if (lane_id() == 0) before[u] = sl[i > 0 && i < n ? i - 1 : 0];
        }
#pragma unroll
        for (int u = 0; u < kCountUnroll; u++) {
            const int i = i0 + u * kBlock + static_cast<int>(threadIdx.x);
            if (i >= n || v[u] >= 0) continue;
            const int g = static_cast<int>(group_of(i, k, recip));
            const int j = i - g * k;
            if (j == 0 || before[u] >= 0) atomicMin(&s_cnt[g], j);
        }
    }
    __syncthreads();
    uint32_t c[GPT], sum = 0;
#pragma unroll
    for (int i = 0; i < GPT; i++) {
        const int g = static_cast<int>(threadIdx.x) * GPT + i;
        c[i] = g < ng ? static_cast<uint32_t>(s_cnt[g]) : 0u;
        sum += c[i];
    }
    uint32_t total;
    uint32_t run = block_exclusive_sum<uint32_t>(sum, lds, &total);
    if (threadIdx.x == 0) partials[blockIdx.x] = total;
#pragma unroll
    for (int i = 0; i < GPT; i++) {
        s_cnt[threadIdx.x * GPT + i] = static_cast<int32_t>((run << kCountBits) | c[i]);
        run += c[i];
    }
    __syncthreads();
#pragma unroll
    for (int i = 0; i < GPT; i++) {
        const int gi = i * kBlock + static_cast<int>(threadIdx.x);
        if (gi >= ng) continue;
        const int64_t g = tile0 + gi;
        packed[g] = static_cast<uint32_t>(s_cnt[gi]);
        if (prev_nbr) {
            const int64_t p = parent[g];
            src_nid[g] = prev_nbr[p];
            src_ts[g] = prev_ts[p];
        } else if (roots) {
            const int64_t r = g / windows;
            src_nid[g] = roots[r];
            src_ts[g] = root_ts[r];
        } else {                                    // no roots given for a positive count: PAD-like
            src_nid[g] = -1;
            src_ts[g] = -1.0f;
        }
    }
}

// Slots per lane and round of the scatter: their loads are issued together.
constexpr int kScatterUnroll = 4;

// Pass 3, slots i = g * k + j of the G groups, kScatterUnroll per lane and
// round: valid slot j < count of g becomes edge first(g) + j and source node
// G + that edge; slot 0 also writes first(g) to indptr.  The groups' offsets
// and counts of a lane's slots are loaded together, then their fields; a slot
// past its group's prefix reads slot 0 (one cached line) and stores nothing,
// rather than each load waiting behind a branch of its own.  Bound by its
// bytes: 3.9M groups, 21M edges, 1.43 GB in 285 us = 5.0 TB/s (2 or 8 slots
// per lane and round the same; nontemporal stores 355 us).  tile_shift:
// log2 of the groups per tile.  Also closes indptr with indptr[G] = E.
__global__ __launch_bounds__(kBlock) void mfg_scatter_kernel(const int32_t *__restrict__ nbr,
                                                             const int64_t *__restrict__ eid,
                                                             const float *__restrict__ ts,
                                                             const float *__restrict__ dt, int32_t k, uint64_t recip,
                                                             const int64_t *__restrict__ sizes,
                                                             const uint32_t *__restrict__ packed,
                                                             const int64_t *__restrict__ tile_off, int tile_shift,
                                                             int64_t *__restrict__ indptr,
                                                             int64_t *__restrict__ edge_dst,
                                                             int64_t *__restrict__ edge_eid,
                                                             float *__restrict__ edge_dt, int32_t *__restrict__ src_nid,
                                                             float *__restrict__ src_ts) {
    constexpr int U = kScatterUnroll;
    const int64_t G = sizes[0];
    if (blockIdx.x == 0 && threadIdx.x == 0) indptr[G] = sizes[1];
    const int64_t total = G * k;
    const int64_t stride = static_cast<int64_t>(gridDim.x) * kBlock * U;
    for (int64_t i0 = static_cast<int64_t>(blockIdx.x) * kBlock * U + threadIdx.x; i0 < total; i0 += stride) {
        int64_t g[U], first[U];
        int32_t j[U];
        uint32_t pc[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = i0 + u * kBlock;
            const int64_t ic = i < total ? i : total - 1;
            g[u] = group_of(ic, k, recip);
            j[u] = static_cast<int32_t>(ic - g[u] * k);
            pc[u] = packed[g[u]];
            first[u] = tile_off[g[u] >> tile_shift];
        }
        int64_t at[U];
        bool ok[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t i = i0 + u * kBlock;
            ok[u] = i < total && static_cast<uint32_t>(j[u]) < (pc[u] & ((1u << kCountBits) - 1));
            at[u] = ok[u] ? i : 0;
        }
        int64_t ve[U];
        float vd[U], vt[U];
        int32_t vn[U];
#pragma unroll
        for (int u = 0; u < U; u++) {
            ve[u] = eid[at[u]];
            vd[u] = dt[at[u]];
            vn[u] = nbr[at[u]];
            vt[u] = ts[at[u]];
        }
#pragma unroll
        for (int u = 0; u < U; u++) {
            const int64_t e0 = first[u] + (pc[u] >> kCountBits);
            if (j[u] == 0 && i0 + u * kBlock < total) indptr[g[u]] = e0;
            if (!ok[u]) continue;
            const int64_t e = e0 + j[u];
            if (edge_dst) edge_dst[e] = g[u];
            edge_eid[e] = ve[u];
            edge_dt[e] = vd[u];
            src_nid[G + e] = vn[u];
            src_ts[G + e] = vt[u];
        }
    }
}

unsigned grid_of(int64_t n) {
    int64_t b = (n + kBlock - 1) / kBlock;
    if (b < 1) b = 1;
    if (b > (1 << 16)) b = 1 << 16;
    return static_cast<unsigned>(b);
}

struct MfgWs {
    uint32_t *packed = nullptr;
    int64_t *partials = nullptr;
    int64_t tiles = 0;
    size_t bytes = 0;
};

MfgWs carve_mfg_ws(void *base, int64_t groups_cap) {
    MfgWs w;
    Carver cv(base);
    const int tile = tile_groups(groups_cap);
    w.tiles = groups_cap > 0 ? (groups_cap + tile - 1) / tile : 1;
    w.packed = cv.take<uint32_t>(static_cast<size_t>(groups_cap > 0 ? groups_cap : 1));
    // a capacity above kSmallGroups has fewer tiles than that one; room for as
    // many, so that a workspace for some capacity serves every smaller one
    const int64_t small_tiles = kSmallGroups / kTileLeast;
    w.partials = cv.take<int64_t>(static_cast<size_t>(
        (groups_cap > kSmallGroups && w.tiles < small_tiles ? small_tiles : w.tiles) + 1));
    w.bytes = cv.size();
    return w;
}

}  // namespace
}  // namespace tgl

using namespace tgl;

extern "C" {

size_t tgl_mfg_workspace(int64_t groups_cap) {
    if (groups_cap < 0) return 0;
    return carve_mfg_ws(nullptr, groups_cap).bytes;
}

tgl_status tgl_mfg_export(const tgl_hop_out *hop, const tgl_hop_out *prev, const int32_t *roots,
                          const float *root_ts, const int64_t *count, int32_t windows, int32_t k,
                          int64_t groups_cap, const tgl_mfg *out, void *workspace, size_t workspace_bytes,
                          void *stream) {
    if (!hop || !out || !count) return TGL_EINVAL;
    if (windows < 1 || windows > TGL_MAX_SNAPSHOTS || k < 1 || k > TGL_MAX_FANOUT) return TGL_EINVAL;
    if (groups_cap < 0 || groups_cap > (int64_t(1) << 62) / (k + 1)) return TGL_EINVAL;
    if (!out->indptr || !out->sizes) return TGL_EINVAL;
    if (groups_cap > 0) {
        if (!hop->nbr || !hop->eid || !hop->ts || !hop->dt) return TGL_EINVAL;
        if (!out->edge_eid || !out->edge_dt || !out->src_nid || !out->src_ts) return TGL_EINVAL;
        // roots are read only for groups below count * windows, a device value:
        // they may be NULL when the call had no roots
        if (prev && (!prev->nbr || !prev->ts || !hop->parent)) return TGL_EINVAL;
        if (!prev && (!roots) != (!root_ts)) return TGL_EINVAL;
    }
    if (prev && windows != 1) return TGL_EINVAL;
    const MfgWs need = carve_mfg_ws(nullptr, groups_cap);
    if (!workspace || workspace_bytes < need.bytes) return TGL_ENOSPACE;
    const MfgWs ws = carve_mfg_ws(workspace, groups_cap);

    hipStream_t st = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    ScopedTimer tm(TGL_TIMER_MFG, st);
    const int tile = tile_groups(groups_cap);
    const uint64_t recip = k > 1 ? ~0ull / static_cast<uint64_t>(k) + 1 : 0;   // floor(2^64 / k) + 1, or 2^64 / k exactly
    const auto count_tiles = tile == kTileLeast ? mfg_count_kernel<kTileLeast / kBlock> : mfg_count_kernel<kTileMost / kBlock>;
    count_tiles<<<static_cast<unsigned>(ws.tiles), kBlock, 0, st>>>(
        hop->nbr, k, recip, roots, root_ts, windows, prev ? prev->nbr : nullptr, prev ? prev->ts : nullptr,
        prev ? hop->parent : nullptr, count, groups_cap, out->sizes, ws.packed, ws.partials, out->src_nid, out->src_ts);
    launch_scan_partials(ws.partials, ws.tiles, out->sizes + 1, st);
    const int64_t slots = groups_cap * k;
    mfg_scatter_kernel<<<grid_of((slots + kScatterUnroll - 1) / kScatterUnroll), kBlock, 0, st>>>(
        hop->nbr, hop->eid, hop->ts, hop->dt, k, recip, out->sizes, ws.packed, ws.partials, __builtin_ctz(tile),
        out->indptr, out->edge_dst, out->edge_eid, out->edge_dt, out->src_nid, out->src_ts);
    return launch_status();
}

}  // extern "C"
