// tgl_search.hpp -- positions below a threshold in the time-sorted runs of a
// T-CSR, found by the lanes of one group of a wavefront.  Shared by the
// sampler, which locates window edges with it, and the T-CSR build, which
// locates every entry's neighbour history.
#pragma once

#include "tgl_cells.hpp"
#include "tgl_internal.hpp"

namespace tgl {

// Four floats loaded at once from an address that is a multiple of 4 bytes: the
// timestamps tgl_tcsr_nodes is given need no other alignment.
using f32x4 = float __attribute__((ext_vector_type(4), aligned(4)));

// ts[p4 .. p4+3] for p4 a multiple of 4; entries at or past M read as +inf
// (they are never inside a window).
__device__ __forceinline__ float4 load_ts4(const float *__restrict__ tsa, uint32_t p4, uint32_t M) {
    if (static_cast<uint64_t>(p4) + 3 < M) {
        const f32x4 v = *reinterpret_cast<const f32x4 *>(tsa + p4);
        return make_float4(v.x, v.y, v.z, v.w);
    }
    const float inf = __builtin_inff();
    float4 r = make_float4(inf, inf, inf, inf);
    if (p4 < M) r.x = tsa[p4];
    if (static_cast<uint64_t>(p4) + 1 < M) r.y = tsa[p4 + 1];
    if (static_cast<uint64_t>(p4) + 2 < M) r.z = tsa[p4 + 2];
    return r;
}

// A stretch of a time-sorted run held in the registers of one G-lane group:
// lane gl holds the H timestamps p0 .. p0 + H - 1, p0 = (lo & ~3) + H * gl,
// loaded as H / 4 aligned float4.  One load covers any [lo, hi) of at most
// `span` entries.
template <int G>
struct HeldRun {
    static constexpr int NV = G >= 16 ? 1 : 16 / G;     // float4 per lane
    static constexpr uint32_t H = 4 * NV;               // timestamps per lane
    static constexpr uint32_t span = H * G - 3;
    float4 v[NV];
    uint32_t p0;
};

template <int G>
__device__ __forceinline__ HeldRun<G> load_run(const float *__restrict__ tsa, uint32_t lo, uint32_t hi,
                                               uint32_t M, int gl) {
    HeldRun<G> r;
    r.p0 = (lo & ~3u) + HeldRun<G>::H * static_cast<uint32_t>(gl);
    const float inf = __builtin_inff();
#pragma unroll
    for (int m = 0; m < HeldRun<G>::NV; m++) {
        const uint32_t p4 = r.p0 + 4 * m;
        r.v[m] = p4 < hi && lo < hi ? load_ts4(tsa, p4, M) : make_float4(inf, inf, inf, inf);
    }
    return r;
}

// The run [a, b), b - a <= TGL_NODE_INLINE, held from the inline timestamps
// of its node record rec (16-byte words 1..7): position a + i is inline
// timestamp i, so the stretch starts at a and count_in applies unchanged.
template <int G>
__device__ __forceinline__ HeldRun<G> load_inline(const int4 *__restrict__ rec, uint32_t a, int gl) {
    constexpr int kWords = TGL_NODE_INLINE / 4;
    static_assert(HeldRun<G>::H * G >= TGL_NODE_INLINE, "held stretch covers the inline timestamps");
    HeldRun<G> r;
    r.p0 = a + HeldRun<G>::H * static_cast<uint32_t>(gl);
    const float inf = __builtin_inff();
#pragma unroll
    for (int m = 0; m < HeldRun<G>::NV; m++) {
        const int q = HeldRun<G>::NV * gl + m;
        if (q < kWords) {
            const int4 w = rec[1 + q];
            r.v[m] = make_float4(__int_as_float(w.x), __int_as_float(w.y), __int_as_float(w.z), __int_as_float(w.w));
        } else {
            r.v[m] = make_float4(inf, inf, inf, inf);
        }
    }
    return r;
}

// Sum over the G lanes of the calling lane's group.
template <int G>
__device__ __forceinline__ int group_sum(int c) {
#pragma unroll
    for (int off = G / 2; off >= 1; off >>= 1) c += __shfl_xor(c, off, kWave);
    return c;
}

// lo + #{p in [lo, hi): ts[p] < v} for [lo, hi) inside the held stretch.
template <int G>
__device__ __forceinline__ uint32_t count_in(const HeldRun<G> &r, uint32_t lo, uint32_t hi, float v) {
    int c = 0;
#pragma unroll
    for (int m = 0; m < HeldRun<G>::NV; m++) {
        const uint32_t p = r.p0 + 4 * m;
        c += (p >= lo && p < hi && r.v[m].x < v);
        c += (p + 1 >= lo && p + 1 < hi && r.v[m].y < v);
        c += (p + 2 >= lo && p + 2 < hi && r.v[m].z < v);
        c += (p + 3 >= lo && p + 3 < hi && r.v[m].w < v);
    }
    return lo + static_cast<uint32_t>(group_sum<G>(c));
}

// For each i: lo[i] += #{p in [lo[i], hi[i]): arr[p] < v[i]}, over a sorted
// stretch of arr (n_arr elements), found by the G lanes of one group together.
// While a range is longer than one held stretch, each round probes G evenly
// spaced positions of it; the probes below v[i] form a prefix, whose length
// narrows the range to one gap; the last range is loaded whole and counted.
// The NE searches advance together, so the probes of one round, and the final
// loads, of all of them are in flight at the same time: the chain of dependent
// loads is that of one search.
template <int G, int NE>
__device__ __forceinline__ void search_n(const float *__restrict__ arr, uint32_t n_arr, uint32_t (&lo)[NE],
                                         uint32_t (&hi)[NE], const float (&v)[NE], int gl) {
    for (;;) {
        bool any = false;
#pragma unroll
        for (int i = 0; i < NE; i++) any |= hi[i] - lo[i] > HeldRun<G>::span;
        if (!any) break;                            // group-uniform
        // probes at lo + j * step, j = 1..G, step = len / (G + 1) >= 1: all
        // inside (lo, hi), strictly increasing
        float probe[NE];
#pragma unroll
        for (int i = 0; i < NE; i++) {
            probe[i] = 0.0f;
            const uint32_t len = hi[i] - lo[i];
            if (len > HeldRun<G>::span)
                probe[i] = arr[lo[i] + static_cast<uint32_t>(gl + 1) * (len / (G + 1))];
        }
#pragma unroll
        for (int i = 0; i < NE; i++) {
            const uint32_t len = hi[i] - lo[i];
            if (len > HeldRun<G>::span) {           // group-uniform
                const uint32_t step = len / (G + 1);
                const uint32_t c = static_cast<uint32_t>(__popcll(group_ballot<G>(probe[i] < v[i])));
                // probes 1..c are below v[i], probe c+1 (if any) is not
                const uint32_t nlo = c > 0 ? lo[i] + c * step + 1 : lo[i];
                if (c < G) hi[i] = lo[i] + (c + 1) * step;
                lo[i] = nlo;
            }
        }
    }
    bool open = false;
#pragma unroll
    for (int i = 0; i < NE; i++) open |= hi[i] > lo[i];
    if (!open) return;                              // group-uniform: every answer is known
    HeldRun<G> r[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) r[i] = load_run<G>(arr, lo[i], hi[i], n_arr, gl);
#pragma unroll
    for (int i = 0; i < NE; i++) lo[i] = count_in<G>(r[i], lo[i], hi[i], v[i]);
}

// A node's run [a, b) and its first and last timestamps: where a threshold
// falls in it is estimated by linear interpolation between them.
struct RunShape {
    uint32_t a, b;
    float first, last;
};

// Estimated position of threshold v in the run (lower bound: the count of
// timestamps below v, plus a), and the spread of that estimate: if the
// run's timestamps were independent draws between first and last, the count
// below v would be binomial, with standard deviation at most sqrt(b - a) / 2.
__device__ __forceinline__ void run_estimate(const RunShape &rs, float v, uint32_t &pos, uint32_t &spread) {
    const float n = static_cast<float>(rs.b - rs.a);
    float f = (v - rs.first) / (rs.last - rs.first);
    if (!(f >= 0.0f)) f = f < 0.0f ? 0.0f : 0.5f;                 // below the run, or NaN
    if (f > 1.0f) f = 1.0f;
    const float o = f * n;                                         // <= n
    pos = rs.a + (o < n ? static_cast<uint32_t>(o) : rs.b - rs.a);
    spread = static_cast<uint32_t>(0.5f * __builtin_sqrtf(n)) + 1u;
}

// Probe g of a guided round: c + (g - G/2) d + d/2, clamped into [lo, hi).
// Non-decreasing in g.
template <int G>
__device__ __forceinline__ uint32_t guided_pos(uint32_t lo, uint32_t hi, uint32_t c, uint32_t d, int g) {
    const int64_t q = static_cast<int64_t>(c) + (static_cast<int64_t>(g) - G / 2) * static_cast<int64_t>(d) +
                      static_cast<int64_t>(d / 2);
    const int64_t last = static_cast<int64_t>(hi) - 1;
    return static_cast<uint32_t>(q < static_cast<int64_t>(lo) ? static_cast<int64_t>(lo) : (q > last ? last : q));
}

// One round of the search of a sorted stretch of arr, guided by estimates:
// for each i whose range [lo[i], hi[i]) is longer than a held stretch, the G
// lanes probe positions d[i] apart around c[i].  The probes below v[i] form
// a prefix (arr is sorted and the positions do not decrease), so the answer
// lies after the last of them and at or before the next: the range shrinks
// to about d[i] when the estimate is off by less than G/2 spacings, and
// never grows.  lo[i] + #{p in [lo[i], hi[i]): arr[p] < v[i]} is unchanged.
template <int G, int NE>
__device__ __forceinline__ void guided_round(const float *__restrict__ arr, uint32_t (&lo)[NE], uint32_t (&hi)[NE],
                                             const float (&v)[NE], const uint32_t (&c)[NE], const uint32_t (&d)[NE],
                                             int gl) {
    float probe[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) {
        probe[i] = 0.0f;
        if (hi[i] - lo[i] > HeldRun<G>::span) probe[i] = arr[guided_pos<G>(lo[i], hi[i], c[i], d[i], gl)];
    }
#pragma unroll
    for (int i = 0; i < NE; i++) {
        if (hi[i] - lo[i] > HeldRun<G>::span) {     // group-uniform
            const int n = __popcll(group_ballot<G>(probe[i] < v[i]));
            const uint32_t nlo = n > 0 ? guided_pos<G>(lo[i], hi[i], c[i], d[i], n - 1) + 1 : lo[i];
            if (n < G) hi[i] = guided_pos<G>(lo[i], hi[i], c[i], d[i], n);
            lo[i] = nlo;
        }
    }
}

// Positions below NE thresholds, each in a range of its own: out[i] = lo0[i]
// + #{p in [lo0[i], hi0[i]): ts[p] < v[i]} for each i with act[i] (lo0[i] otherwise),
// each range a stretch of one sorted run.  Ranges longer than one probe round
// are narrowed on the search index first when there is one.
template <int G, int NE>
__device__ __forceinline__ void count_below_ranges(const float *__restrict__ tsa, uint32_t M,
                                                   const float *__restrict__ tsx, uint32_t nx,
                                                   const uint32_t (&lo0)[NE], const uint32_t (&hi0)[NE],
                                                   const float (&v)[NE], const bool (&act)[NE],
                                                   uint32_t (&out)[NE], int gl) {
    constexpr uint32_t X = TGL_INDEX_STRIDE;
    uint32_t lo[NE], hi[NE];
    bool any_index = false;
#pragma unroll
    for (int i = 0; i < NE; i++) {
        const bool use = act[i] && tsx && hi0[i] - lo0[i] > HeldRun<G>::span * (G + 1);
        const uint32_t ja = lo0[i] / X + (lo0[i] % X != 0);
        const uint32_t jb = hi0[i] / X + (hi0[i] % X != 0);
        lo[i] = use ? ja : lo0[i];
        hi[i] = use ? jb : lo0[i];
        any_index |= use;
    }
    if (any_index) {                                // group-uniform
        search_n<G, NE>(tsx, nx, lo, hi, v, gl);
#pragma unroll
        for (int i = 0; i < NE; i++) {
            const bool use = act[i] && tsx && hi0[i] - lo0[i] > HeldRun<G>::span * (G + 1);
            const uint32_t ja = lo0[i] / X + (lo0[i] % X != 0);
            const uint32_t jb = hi0[i] / X + (hi0[i] % X != 0);
            const uint32_t r = lo[i];
            lo[i] = use ? (r > ja ? (r - 1) * X + 1 : lo0[i]) : lo0[i];   // ts[(r-1) X] < v[i]
            hi[i] = use ? (r < jb ? r * X : hi0[i]) : (act[i] ? hi0[i] : lo0[i]);   // ts[r X] >= v[i]
        }
    } else {
#pragma unroll
        for (int i = 0; i < NE; i++) {
            lo[i] = lo0[i];
            hi[i] = act[i] ? hi0[i] : lo0[i];
        }
    }
    search_n<G, NE>(tsa, M, lo, hi, v, gl);
#pragma unroll
    for (int i = 0; i < NE; i++) out[i] = act[i] ? lo[i] : lo0[i];
}

// Positions below NE thresholds in [lo0, hi0), a range of the run [rs.a,
// rs.b), from the run's time directory (tgl_cell per search-index slot; the
// run owns K >= 1 cells), as count_below_n returns them: threshold i falls in cell
// k = cell(v[i]), whose first position pos and timestamp, and the next
// cell's pos (rs.b after the last cell), are read with one round of loads.
// The run's count below v[i] is pos when v[i] <= ts[pos], else it lies in
// [pos + 1, next pos], a stretch of about TGL_INDEX_STRIDE entries when the
// run's timestamps are spread evenly, which count_below_ranges searches
// (with the index when it is long).  Clamping the stretch into [lo0, hi0)
// gives the count within that range.  Every position read from the
// directory is clamped into the run.
template <int G, int NE>
__device__ __forceinline__ void count_below_dir(const float *__restrict__ tsa, uint32_t M,
                                                const float *__restrict__ tsx, uint32_t nx,
                                                const uint2 *__restrict__ dir, uint32_t lo0, uint32_t hi0,
                                                const RunShape &rs, const float (&v)[NE], const bool (&act)[NE],
                                                uint32_t (&out)[NE], int gl) {
    constexpr uint32_t X = TGL_INDEX_STRIDE;
    const uint32_t ja = rs.a / X + (rs.a % X != 0);
    const uint32_t K = rs.b / X + (rs.b % X != 0) - ja;
    const float sc = dir_scale(rs.first, rs.last, K);
    uint2 c0[NE];
    uint32_t c1[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) {
        c0[i] = make_uint2(rs.a, 0u);
        c1[i] = rs.b;
        if (act[i]) {                               // group-uniform
            const uint32_t kc = dir_cell(v[i], rs.first, rs.last, sc, K);
            c0[i] = dir[ja + kc];
            if (kc + 1 < K) c1[i] = dir[ja + kc + 1].x;
        }
    }
    uint32_t lo[NE], hi[NE];
    bool open[NE];
#pragma unroll
    for (int i = 0; i < NE; i++) {
        const uint32_t pos = c0[i].x < rs.a ? rs.a : (c0[i].x > rs.b ? rs.b : c0[i].x);
        const uint32_t nxt = c1[i] < pos ? pos : (c1[i] > rs.b ? rs.b : c1[i]);
        const bool past = v[i] > __uint_as_float(c0[i].y) && pos < nxt;
        uint32_t l = past ? pos + 1 : pos;
        uint32_t h = past ? nxt : l;
        l = l < lo0 ? lo0 : (l > hi0 ? hi0 : l);
        h = h < l ? l : (h > hi0 ? hi0 : h);
        lo[i] = act[i] ? l : lo0;
        hi[i] = act[i] ? h : lo0;
        open[i] = act[i] && h > l;
    }
    count_below_ranges<G, NE>(tsa, M, tsx, nx, lo, hi, v, open, out, gl);
}

// Positions below NE thresholds in the time-sorted run [lo0, hi0) of the
// timestamp array (M entries): out[i] = lo0 + #{p in [lo0, hi0): ts[p] < v[i]}
// for each i with act[i] (out[i] = lo0 otherwise).  rec, when not null, is the
// record of a node whose whole run (lo0 onwards) is inline in it: the run is
// then read from there.  A run of at most one held stretch is loaded once and
// serves every threshold.  A longer range starts from the time directory dir
// of its run rs when there is one (count_below_dir).  Otherwise a range long
// enough to need more than one probe round is first narrowed on the search
// index tsx (nx samples, tsx[j] = ts[j * TGL_INDEX_STRIDE]) when there is
// one, starting with a round guided by the run shape rs (the run that holds
// the stretch, lo0 its start): with r the samples inside the run below v[i],
// the answer lies after sample r - 1 and at or before sample r, fewer than
// TGL_INDEX_STRIDE timestamps.
template <int G, int NE, bool DIR>
__device__ __forceinline__ void count_below_n(const float *__restrict__ tsa, uint32_t M,
                                              const float *__restrict__ tsx, uint32_t nx,
                                              const uint2 *__restrict__ dir,
                                              const int4 *__restrict__ rec, uint32_t lo0, uint32_t hi0,
                                              const RunShape &rs, const float (&v)[NE], const bool (&act)[NE],
                                              uint32_t (&out)[NE], int gl) {
    constexpr uint32_t X = TGL_INDEX_STRIDE;
    if (rec || hi0 - lo0 <= HeldRun<G>::span) {    // group-uniform: one load serves every bound
        const HeldRun<G> r = rec ? load_inline<G>(rec, lo0, gl) : load_run<G>(tsa, lo0, hi0, M, gl);
#pragma unroll
        for (int i = 0; i < NE; i++) out[i] = act[i] ? count_in<G>(r, lo0, hi0, v[i]) : lo0;
        return;
    }
    if constexpr (DIR) {
        // the range is longer than one held stretch, so its run owns a cell
        count_below_dir<G, NE>(tsa, M, tsx, nx, dir, lo0, hi0, rs, v, act, out, gl);
#pragma unroll
        for (int i = 0; i < NE; i++)
            if (!act[i]) out[i] = lo0;
        return;
    }
    uint32_t lo[NE], hi[NE];
    if (tsx && hi0 - lo0 > HeldRun<G>::span * (G + 1)) {   // group-uniform
        // samples j in [ja, jb) are the positions j * X inside [lo0, hi0)
        const uint32_t ja = lo0 / X + (lo0 % X != 0);
        const uint32_t jb = hi0 / X + (hi0 % X != 0);
        uint32_t gc[NE], gd[NE];
#pragma unroll
        for (int i = 0; i < NE; i++) {
            lo[i] = ja;
            hi[i] = act[i] ? jb : ja;
            uint32_t pos, spread;
            run_estimate(rs, v[i], pos, spread);
            gc[i] = pos / X;
            gd[i] = spread / X > 0 ? spread / X : 1u;
        }
        guided_round<G, NE>(tsx, lo, hi, v, gc, gd, gl);
        search_n<G, NE>(tsx, nx, lo, hi, v, gl);
#pragma unroll
        for (int i = 0; i < NE; i++) {
            const uint32_t r = lo[i];
            lo[i] = r > ja ? (r - 1) * X + 1 : lo0;  // ts[(r-1) X] < v[i]
            hi[i] = r < jb ? r * X : hi0;            // ts[r X] >= v[i]
            if (!act[i]) hi[i] = lo[i];
        }
    } else {
#pragma unroll
        for (int i = 0; i < NE; i++) {
            lo[i] = lo0;
            hi[i] = act[i] ? hi0 : lo0;
        }
    }
    search_n<G, NE>(tsa, M, lo, hi, v, gl);
#pragma unroll
    for (int i = 0; i < NE; i++) out[i] = act[i] ? lo[i] : lo0;
}

}  // namespace tgl
