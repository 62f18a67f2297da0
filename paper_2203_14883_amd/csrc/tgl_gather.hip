// tgl_gather.hip -- lookup of per-node and per-edge rows for sampled slots
// (Figure 2 of TGL, steps 2 and 3: node features, node memory and mailbox rows
// by neighbour id, edge features by edge id; Table 3 gives the row widths of
// the paper's datasets: 172-dim edge features on Wikipedia, 413 / 186 on
// GDELT, 768-dim node features on MAG).
//
// Every output word is independent, so the kernel is a plain HBM-bound gather
// by words: a wavefront writes kFlat KB of consecutive output at a time, lane
// l its 16-byte words l, l + 64, ..., whichever rows they fall in, so that
// every lane works and every store instruction writes whole lines whatever
// the row's width.  All keys of a lane's words are loaded together, then all
// the words; outputs are written with nontemporal stores (they are consumed
// by the next stage, not re-read here).  Tables are a dimension of the grid.
//
// A wavefront per eight rows, its lanes striding over one row after another,
// left lanes idle at every row's end and wrote lines in parts.  Same inputs,
// rows then words (write rate): node memory, mailbox and edge features (100 +
// 372 + 172 float32) of 180,000 slots from small tables 145 -> 113 us (4.1
// TB/s), of 2M slots from 1M to 3M rows 2.38 -> 1.72 ms; 172 float32 of 2M
// slots 493 -> 373 us; 4 float32 172 -> 26 us; 768 bf16 of 4M slots, half of
// them PAD, 1.78 -> 1.60 ms (3.8 TB/s written, 1.9 read).
#include "tgl_internal.hpp"

namespace tgl {
namespace {

using i32x4 = int __attribute__((ext_vector_type(4)));

// 16-byte words per lane whose loads are in flight together.  768 bf16 of 4M
// slots: 2 words 1.62 ms, 4 words 1.59, 6 words 1.74, 8 words 1.70; the 180,000
// slots above 119, 113, 112 and 111 us.  Nontemporal loads of the rows lose
// what caches hold (112 -> 154 us), plain stores too (137 us).
constexpr int kFlat = 4;

struct GatherTable {
    const i32x4 *rows;
    i32x4 *out;
    int64_t num_rows;
    int32_t words;         // 16-byte words per row
    int32_t key;           // TGL_KEY_NODE / TGL_KEY_EDGE
    uint32_t recip;        // ceil(2^32 / words), words > 1
};

struct GatherArgs {
    const int32_t *nbr;
    const int64_t *eid;
    int64_t n;
    const int64_t *count;  // or null
    int64_t per;
    int64_t whole;         // n / per
    GatherTable t[TGL_MAX_TABLES];
};

__global__ __launch_bounds__(kBlock) void gather_kernel(const GatherArgs a) {
    const GatherTable T = a.t[blockIdx.y];
    const int lane = lane_id();
    constexpr int kWaves = kBlock / kWave;
    constexpr int kSpan = kFlat * kWave;
    const int64_t waves = static_cast<int64_t>(gridDim.x) * kWaves;
    const int64_t wave = __builtin_amdgcn_readfirstlane(static_cast<int>(blockIdx.x * kWaves + threadIdx.x / kWave));
    int64_t n = a.n;
    if (a.count) {
        // valid prefix: min(n, count * per), without overflowing the product
        const int64_t c = *a.count;
        const int64_t lim = c <= 0 ? 0 : (c > a.whole ? n : c * a.per);
        n = lim < n ? lim : n;
    }
    const i32x4 zero = {0, 0, 0, 0};
    const uint32_t W = static_cast<uint32_t>(T.words);
    const int64_t total = n * W;
    const int64_t step = waves * kSpan;
    if (wave * kSpan >= total) return;
    // the span's first word as (row0, off0), advanced without dividing
    const int64_t step_q = step / W;
    const uint32_t step_r = static_cast<uint32_t>(step - step_q * W);
    int64_t w0 = wave * kSpan;
    int64_t row0 = w0 / W;
    uint32_t off0 = static_cast<uint32_t>(w0 - row0 * W);
    for (; w0 < total; w0 += step) {
        int64_t src[kFlat];
#pragma unroll
        for (int u = 0; u < kFlat; u++) {
            // r < W + kSpan <= 4352, so r / W is exactly r * recip >> 32
            const uint32_t r = off0 + static_cast<uint32_t>(u * kWave + lane);
            const uint32_t q = W == 1 ? r : __umulhi(r, T.recip);
            const int64_t row = row0 + q < n ? row0 + q : n - 1;    // clamped: loads issue together
            const int64_t k = T.key == TGL_KEY_NODE ? static_cast<int64_t>(a.nbr[row]) : a.eid[row];
            src[u] = k >= 0 && k < T.num_rows && w0 + u * kWave + lane < total ? k * W + (r - q * W) : -1;
        }
        i32x4 v[kFlat];
#pragma unroll
        for (int u = 0; u < kFlat; u++) v[u] = src[u] >= 0 ? T.rows[src[u]] : zero;
#pragma unroll
        for (int u = 0; u < kFlat; u++) {
            const int64_t i = w0 + u * kWave + lane;
            if (i < total) __builtin_nontemporal_store(v[u], T.out + i);
        }
        row0 += step_q;
        off0 += step_r;
        if (off0 >= W) {
            off0 -= W;
            row0++;
        }
    }
}

}  // namespace
}  // namespace tgl

using namespace tgl;

extern "C" {

tgl_status tgl_gather(const int32_t *nbr, const int64_t *eid, int64_t n, const int64_t *count,
                      int64_t per_count, const tgl_table *tables, int32_t num_tables, void *stream) {
    if (n < 0 || per_count < 1 || !tables || num_tables < 1 || num_tables > TGL_MAX_TABLES) return TGL_EINVAL;
    GatherArgs a{};
    a.nbr = nbr;
    a.eid = eid;
    a.n = n;
    a.count = count;
    a.per = per_count;
    a.whole = n / per_count;
    int64_t most = 0;                           // words of the widest row
    for (int i = 0; i < num_tables; i++) {
        const tgl_table &t = tables[i];
        if (t.row_bytes < 16 || t.row_bytes > TGL_MAX_ROW_BYTES || t.row_bytes % 16 != 0) return TGL_EINVAL;
        if (t.num_rows < 0 || t.num_rows > INT64_MAX / t.row_bytes) return TGL_EINVAL;
        if (t.key != TGL_KEY_NODE && t.key != TGL_KEY_EDGE) return TGL_EINVAL;
        if (n > 0 && !t.out) return TGL_EINVAL;
        if (t.num_rows > 0 && !t.rows) return TGL_EINVAL;
        if ((reinterpret_cast<uintptr_t>(t.rows) & 15u) != 0 || (reinterpret_cast<uintptr_t>(t.out) & 15u) != 0)
            return TGL_EINVAL;
        if (n > 0 && t.key == TGL_KEY_NODE && !nbr) return TGL_EINVAL;
        if (n > 0 && t.key == TGL_KEY_EDGE && !eid) return TGL_EINVAL;
        a.t[i].rows = static_cast<const i32x4 *>(t.rows);
        a.t[i].out = static_cast<i32x4 *>(t.out);
        a.t[i].num_rows = t.num_rows;
        a.t[i].words = t.row_bytes / 16;
        a.t[i].key = t.key;
        const uint32_t W = static_cast<uint32_t>(t.row_bytes / 16);
        a.t[i].recip = W > 1 ? static_cast<uint32_t>(((uint64_t(1) << 32) + W - 1) / W) : 0;
        most = a.t[i].words > most ? a.t[i].words : most;
    }
    if (n == 0) return TGL_OK;
    hipStream_t st = static_cast<hipStream_t>(stream);
    (void)hipGetLastError();
    constexpr int64_t kPerBlock = static_cast<int64_t>(kBlock) * kFlat;      // words
    // blocks for the widest table, n * most words (without overflow), capped
    // (fewer, longer blocks are slower: 4M slots of 768 bf16 1.79 / 1.74 / 1.66 /
    // 1.58 ms on 4 Ki, 16 Ki, 64 Ki and a block per 16 KB).  With a count, which
    // may be far below n, a call for a hop's capacity would wait for blocks with
    // nothing to do: 5.2M slots of three tables, 2,000 of them counted, 303 us on
    // a block per 16 KB, 23 on 96 Ki in all, 12 on 48 Ki and below; all counted 3480,
    // 3437 and 3458 us (3490 on 12 Ki).
    constexpr int64_t kCountedBlocks = 48 << 10;
    const int64_t max_blocks = count ? kCountedBlocks / num_tables : 1 << 22;
    int64_t blocks = n > max_blocks * kPerBlock / most ? max_blocks : (n * most + kPerBlock - 1) / kPerBlock;
    {
        ScopedTimer tm(TGL_TIMER_GATHER, st);
        gather_kernel<<<dim3(static_cast<unsigned>(blocks), static_cast<unsigned>(num_tables)), kBlock, 0, st>>>(a);
    }
    return launch_status();
}

}  // extern "C"
