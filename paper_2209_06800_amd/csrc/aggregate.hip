// Host side of the neighbour aggregation (launch geometry, column slabs, scratch for partial sums) and
// the fix-up kernel that combines the partial sums of rows cut into several work items.  The
// aggregation kernels themselves live in aggregate_kernels.h.
#include <hip/hip_runtime.h>

#include <algorithm>
#include <mutex>
#include <vector>

#include "aggregate_kernels.h"

namespace mgg {

namespace {

constexpr int kWavesPerBlock = 4;                   // fix-up kernel
constexpr int kBlock = kWave * kWavesPerBlock;

// Rows cut into several items: one wavefront per such row adds its partial sums slot by slot, front
// to back (a fixed order: results do not depend on scheduling), adds the self term and the row
// factor, and writes the row.  Scratch rows start on 32-byte boundaries, so every lane takes four
// consecutive columns with one 16-byte load per slot, several slots in flight; no LDS, no barrier.
template <bool BF16>
__global__ __launch_bounds__(kBlock) void fixup_kernel(const SplitRow *split_rows, int32_t n_split, int32_t dim, const float *scratch,
                                                       int64_t scratch_ld, const void *x_local, int64_t ld_x,
                                                       const float *dinv_own, int32_t gcn, float self_w, void *out_v, int32_t out_bf16,
                                                       int64_t ld_out, int32_t phase, const float *bias, int32_t relu,
                                                       int32_t no_self)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int r_id = static_cast<int>(blockIdx.x) * kWavesPerBlock + static_cast<int>(threadIdx.x / kWave);
    if (r_id >= n_split) return;
    const SplitRow sr = split_rows[r_id];
    const float dv = gcn ? dinv_own[sr.row] : 1.f;
    const float ws = gcn ? dv : self_w;
    const float *base = scratch + static_cast<int64_t>(sr.first_slot) * scratch_ld;
    for (int k = 4 * lane; k < dim; k += 4 * kWave) {
        float4 sum = make_float4(0.f, 0.f, 0.f, 0.f);
        const float *src = base + k;                 // columns k .. k+3 exist in scratch (its rows are padded to 8)
        int i = 0;
        for (; i + 3 < sr.n_slots; i += 4) {
            const float4 v0 = *reinterpret_cast<const float4 *>(src + static_cast<int64_t>(i) * scratch_ld);
            const float4 v1 = *reinterpret_cast<const float4 *>(src + static_cast<int64_t>(i + 1) * scratch_ld);
            const float4 v2 = *reinterpret_cast<const float4 *>(src + static_cast<int64_t>(i + 2) * scratch_ld);
            const float4 v3 = *reinterpret_cast<const float4 *>(src + static_cast<int64_t>(i + 3) * scratch_ld);
            sum.x = (((sum.x + v0.x) + v1.x) + v2.x) + v3.x; sum.y = (((sum.y + v0.y) + v1.y) + v2.y) + v3.y;
            sum.z = (((sum.z + v0.z) + v1.z) + v2.z) + v3.z; sum.w = (((sum.w + v0.w) + v1.w) + v2.w) + v3.w;
        }
        for (; i < sr.n_slots; ++i) {
            const float4 v = *reinterpret_cast<const float4 *>(src + static_cast<int64_t>(i) * scratch_ld);
            sum.x += v.x; sum.y += v.y; sum.z += v.z; sum.w += v.w;
        }
        const float total[4] = {sum.x, sum.y, sum.z, sum.w};
        float *o = static_cast<float *>(out_v) + static_cast<int64_t>(sr.row) * ld_out + k;
        uint16_t *ob = static_cast<uint16_t *>(out_v) + static_cast<int64_t>(sr.row) * ld_out + k;
        const bool whole = k + 3 < dim;
        float r[4], xv[4] = {0.f, 0.f, 0.f, 0.f};
        if (!no_self) {
            const int64_t at = static_cast<int64_t>(sr.row) * ld_x + k;
            if constexpr (BF16) {
                const uint16_t *x = static_cast<const uint16_t *>(x_local) + at;
#pragma unroll
                for (int e = 0; e < 4; ++e)
                    if (k + e < dim) xv[e] = __uint_as_float(static_cast<uint32_t>(x[e]) << 16);
            } else {
                const float *x = static_cast<const float *>(x_local) + at;
                if (whole) {
                    const float4 q = load_loose<float4>(x);
                    xv[0] = q.x; xv[1] = q.y; xv[2] = q.z; xv[3] = q.w;
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (k + e < dim) xv[e] = x[e];
                }
            }
        }
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            r[e] = 0.f;
            if (k + e < dim) {
                r[e] = phase == 2 ? o[e] + dv * total[e] : dv * (total[e] + ws * xv[e]);
                if (phase != 1) {
                    if (bias) r[e] += bias[k + e];
                    if (relu) r[e] = fmaxf(r[e], 0.f);
                }
            }
        }
        if (whole) {
            if (out_bf16) store_vec_bf16<4>(ob, r);
            else store_vec<4>(o, r);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (k + e < dim) {
                    if (out_bf16) ob[e] = to_bf16(r[e]);
                    else o[e] = r[e];
                }
        }
    }
}

inline bool aligned(const void *p, size_t a) { return (reinterpret_cast<uintptr_t>(p) % a) == 0; }

// Measurement aid: rows of row_bytes gathered by pre-drawn random ids from a table of table_rows rows, 16-byte
// loads, eight in flight per lane, nothing but an add per element -- the rate at which the memory hierarchy
// delivers gathered rows to the CUs when the kernel around the gathers costs nothing.
template <int LPR>
__global__ __launch_bounds__(256) void probe_gather_kernel(const float4 *__restrict__ table, const int32_t *__restrict__ idx, int per_wave, float *sink)
{
    constexpr int NPW = kWave / LPR;
    const int lane = threadIdx.x & (kWave - 1), sub = lane / LPR, lis = lane % LPR;
    const int64_t wave = static_cast<int64_t>(blockIdx.x) * (blockDim.x / kWave) + threadIdx.x / kWave;
    const int32_t *my = idx + wave * per_wave;
    float4 acc = make_float4(0.f, 0.f, 0.f, 0.f);
    int ids = my[lane];
    for (int g = 0; g < per_wave; g += kWave) {
        const int nxt = g + kWave < per_wave ? my[g + kWave + lane] : 0;
#pragma unroll
        for (int t0 = 0; t0 < kWave / NPW; t0 += 8) {
            float4 r[8];
#pragma unroll
            for (int u = 0; u < 8; ++u) {
                const int j = (t0 + u) * NPW + sub;
                const int id = NPW == 1 ? __builtin_amdgcn_readlane(ids, j) : __shfl(ids, j);
                r[u] = table[static_cast<int64_t>(id) * LPR + lis];
            }
#pragma unroll
            for (int u = 0; u < 8; ++u) { acc.x += r[u].x; acc.y += r[u].y; acc.z += r[u].z; acc.w += r[u].w; }
        }
        ids = nxt;
    }
    if (acc.x + acc.y + acc.z + acc.w == 12345.678f) sink[0] = acc.x;     // keeps the loads alive
}

}  // namespace

// A fixed scratch array for callers that must not allocate (mgg_aggregate_static).  Each GPU the
// library runs on holds its own copy; its device address is looked up once per device.
constexpr size_t kStaticScratchBytes = static_cast<size_t>(64) << 20;
static __device__ __align__(256) float g_static_scratch[kStaticScratchBytes / sizeof(float)];
constexpr int kMaxDevices = 64;
static float *g_static_scratch_ptr[kMaxDevices];      // per device; written once, under the mutex
static std::mutex g_static_scratch_mutex;

float *static_scratch(size_t *bytes)
{
    int dev = -1;
    hipError_t e = hipGetDevice(&dev);
    if (e != hipSuccess) { hip_fail(e, "hipGetDevice"); return nullptr; }
    if (dev < 0 || dev >= kMaxDevices) { fail(MGG_ERR_UNSUPPORTED, "device %d beyond the %d the static scratch is kept for", dev, kMaxDevices); return nullptr; }
    std::lock_guard<std::mutex> lock(g_static_scratch_mutex);
    if (!g_static_scratch_ptr[dev]) {
        float *ptr = nullptr;
        e = hipGetSymbolAddress(reinterpret_cast<void **>(&ptr), HIP_SYMBOL(g_static_scratch));
        if (e != hipSuccess || !ptr) { hip_fail(e, "hipGetSymbolAddress(static scratch)"); return nullptr; }
        g_static_scratch_ptr[dev] = ptr;
    }
    if (bytes) *bytes = kStaticScratchBytes;
    return g_static_scratch_ptr[dev];
}

mgg_status_t probe_gather(int64_t table_bytes, int32_t row_bytes, int64_t n_gathers, int32_t iters, uint64_t seed, double *gbs)
{
    if (row_bytes != 128 && row_bytes != 256 && row_bytes != 512 && row_bytes != 1024)
        return fail(MGG_ERR_INVALID_ARG, "row_bytes must be 128, 256, 512 or 1024");
    constexpr int per_wave = 512, wpb = 4;
    if (table_bytes < row_bytes || table_bytes > (static_cast<int64_t>(8) << 30) || n_gathers < per_wave * wpb || n_gathers > (static_cast<int64_t>(1) << 28) ||
        iters < 1 || !gbs)
        return fail(MGG_ERR_INVALID_ARG, "probe sizes out of range");
    const int64_t rows = table_bytes / row_bytes;
    const int64_t waves = n_gathers / per_wave / wpb * wpb;
    n_gathers = waves * per_wave;
    float4 *table = nullptr;
    int32_t *idx = nullptr;
    float *sink = nullptr;
    hipEvent_t e0 = nullptr, e1 = nullptr;
    std::vector<int32_t> h(static_cast<size_t>(n_gathers));
    uint64_t x = seed * 0x9E3779B97F4A7C15ull + 1;
    for (auto &v : h) {                                   // splitmix64
        x += 0x9E3779B97F4A7C15ull;
        uint64_t z = x;
        z = (z ^ (z >> 30)) * 0xBF58476D1CE4E5B9ull; z = (z ^ (z >> 27)) * 0x94D049BB133111EBull; z ^= z >> 31;
        v = static_cast<int32_t>(z % static_cast<uint64_t>(rows));
    }
    mgg_status_t st = MGG_OK;
    hipError_t e = hipMalloc(reinterpret_cast<void **>(&table), static_cast<size_t>(rows) * row_bytes);
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&idx), h.size() * sizeof(int32_t));
    if (e == hipSuccess) e = hipMalloc(reinterpret_cast<void **>(&sink), sizeof(float));
    if (e != hipSuccess) st = alloc_fail(e, static_cast<size_t>(rows) * row_bytes + h.size() * sizeof(int32_t), " of probe buffers");
    if (st == MGG_OK) {
        e = hipMemset(table, 0, static_cast<size_t>(rows) * row_bytes);
        if (e == hipSuccess) e = hipMemcpy(idx, h.data(), h.size() * sizeof(int32_t), hipMemcpyHostToDevice);
        if (e == hipSuccess) e = hipEventCreate(&e0);
        if (e == hipSuccess) e = hipEventCreate(&e1);
        const dim3 grid(static_cast<unsigned>(waves / wpb)), block(kWave * wpb);
        for (int it = -2; it < iters && e == hipSuccess; ++it) {           // two untimed launches first
            if (it == 0) e = hipEventRecord(e0, nullptr);
            if (row_bytes == 128) hipLaunchKernelGGL(probe_gather_kernel<8>, grid, block, 0, nullptr, table, idx, per_wave, sink);
            else if (row_bytes == 256) hipLaunchKernelGGL(probe_gather_kernel<16>, grid, block, 0, nullptr, table, idx, per_wave, sink);
            else if (row_bytes == 512) hipLaunchKernelGGL(probe_gather_kernel<32>, grid, block, 0, nullptr, table, idx, per_wave, sink);
            else hipLaunchKernelGGL(probe_gather_kernel<64>, grid, block, 0, nullptr, table, idx, per_wave, sink);
            if (e == hipSuccess) e = hipGetLastError();
        }
        float ms = 0.f;
        if (e == hipSuccess) e = hipEventRecord(e1, nullptr);
        if (e == hipSuccess) e = hipEventSynchronize(e1);
        if (e == hipSuccess) e = hipEventElapsedTime(&ms, e0, e1);
        if (e != hipSuccess) st = hip_fail(e, "gather probe");
        else *gbs = static_cast<double>(n_gathers) * row_bytes * iters / (ms * 1e-3) / 1e9;
    }
    if (e0) (void)hipEventDestroy(e0);
    if (e1) (void)hipEventDestroy(e1);
    (void)hipFree(table); (void)hipFree(idx); (void)hipFree(sink);
    return st;
}

namespace {

// the ablation of interleaving: the local lists first, the remote lists in a second launch that adds to the result
bool two_launches(const mgg_partition *p) { return p->opt_split_phases != 0 && !p->halo_gid.empty(); }

// What one aggregation launches, decided by plan_aggregate: arithmetic on the host alone.
struct Plan {
    int vec, nvec;               // elements of a vector, vectors of a row
    int32_t last_col;            // first column of the last vector
    int slab_vecs, n_slabs;      // vectors of a column slab
    int64_t n_chunks;            // chunks of the work that go through all slabs one after the other
    int lpr, ch;                 // lanes of a table row, vectors a lane takes of it
    bool lds, team, fine;        // halo rows through LDS; a workgroup takes one item; the fine schedule
    int wpb;                     // wavefronts per workgroup
    int32_t n_items, items_per_wave, short_per_wave, n_item_blocks;
    int grid_x, chunk_x;         // workgroups of a slab, of a slab and chunk
};

// `bases`: the addresses of the two tables, or-ed; scratch_rows: rows of partial sums there is room for
mgg_status_t plan_aggregate(const mgg_partition *p, mgg_agg_t mode, bool bf16, int32_t dim, int64_t ld_x, uint64_t bases, int64_t scratch_rows, Plan *out)
{
    Plan pl{};
    const size_t esz = bf16 ? 2 : 4;
    // 16 bytes per lane whatever the layout.  Where the padding between dim and ld_x completes the last
    // vector (and rows and bases are aligned) the padding is read; its values only reach output columns
    // that do not exist.  Elsewhere -- a plain contiguous tensor of an odd width -- the last vector is
    // moved back to end with the row, so that nothing past the table is read, and stores only the columns
    // that are its own.  Such loads and stores are aligned to an element only, which global memory takes at
    // full width (260 k-node R-MAT, half share, 75 contiguous fp32 columns: 226 us element by element, 167 us).
    // Rows shorter than a vector go element by element.
    int vec = bf16 ? 8 : 4;
    const bool rows_aligned = ld_x % vec == 0 && bases % 16 == 0;
    {
        const int64_t padded = (static_cast<int64_t>(dim) + vec - 1) / vec * vec;
        if (rows_aligned && padded <= ld_x) {
            dim = static_cast<int32_t>(padded);
        } else if (dim < vec) {
            vec = 1;
        }
        pl.last_col = dim - vec;
    }
    const int nvec = (dim + vec - 1) / vec;
    // Column slabs: when one XCD's share of the table rows does not fit its L2 at full width, the
    // launch walks the feature dimension slab by slab (grid.y), all work items of slab 0 first,
    // so that what stays in L2 between two uses of a table row is a slab of it, not the whole
    // row.  Costs one more pass over the ids per slab; output columns of different slabs are
    // disjoint, so nothing has to be combined.
    int slab_vecs = nvec;
    int64_t n_chunks = 1;
    {
        const int64_t opt = p->opt_col_slab_bytes;
        const int64_t vec_bytes = static_cast<int64_t>(vec) * static_cast<int64_t>(esz);
        int64_t slab_bytes = 0;
        if (opt == 0) {
            // automatic: measured on MI355X, slabs pay (1.05-1.6x) when rows are at least 1 KB wide: what has to
            // survive in L2 between two uses of a table row is then a slab of it.  512-byte slabs, except that
            // 256-byte slabs are taken when they bring one XCD's share of the table rows within twice its 4 MB
            // L2 and 512-byte slabs do not (the 233 k x 2.4 KB table of the configs: 18.7 ms against 20.5 with
            // 512 and 20.4 with 128).  On tables far beyond the caches (2 M rows of 1 KB: 4.70 ms against 4.92
            // without slabs) the gain is small but still there; narrower rows lose to the extra passes.
            const int64_t table_rows = p->n_local_rows + static_cast<int64_t>(p->halo_gid.size());
            const int64_t class_rows = (p->xcd_min_deg > 0 ? table_rows / kXcd : table_rows) + 1;
            // Bags of a few tens of lookups have no classes: every L2 sees the whole table.  256-byte slabs from where 512-byte ones
            // of it do not fit an L2 up to where their own do not fit the Infinity Cache (200 k bags of 26 lookups in rows of 1 KB, 512
            // against 256: 2 k to 4 k table rows 7 to 9 % less time, 8 k the same, 16 k 0.62 of the time with 256, 50 k 0.638 and 0.528 ms,
            // 200 k 0.738 and 0.703, 1 M the same, 3 M 5 % less to 9 % more).
            const bool no_classes = p->bags && 2 * p->n_classed < static_cast<int64_t>(p->local_col.size()) + static_cast<int64_t>(p->remote_col.size());
            // Where 256-byte slabs of a class fit one L2 the gathers hit, and what is left to wait for is the id stream: read
            // once per slab, from HBM if it does not stay in the Infinity Cache (bare gathers out of L2: 28.8 TB/s with ids
            // from there, 22.4 from HBM).  Chunks of the work then go through all slabs one after the other, their ids some
            // 36 MB (120 k rows of 1 KB, 46 M neighbours: 2.70 ms with 512-byte slabs, 2.57 so, 2.83 with 256-byte slabs in
            // one chunk; of 2 KB 5.36 -> 5.21; from 16 k rows on also where 512-byte slabs fit: 60 k rows of 1 KB, 25 M neighbours,
            // 1.75 with 512, 1.56 so, 30 k 1.07 and 1.02).  Rows off line boundaries pay a line more per slab: 512 (1200-byte rows:
            // 4.14 against 4.17 ms).  So do small classes whose ids and factors stay in the Infinity Cache from slab to slab in any
            // case (8 k rows, 17.4 M neighbours: 0.578 ms with 512, 0.619 so; 12 k, 17.7 M: 0.637, 0.667; but 16 k, 21 M: 0.886,
            // 0.848, and 8 k, 40 M, 319 MB: 1.67, 1.57; sums, 4 bytes a neighbour: 12 k, 55 M 2.11, 1.96).
            const int64_t id_bytes = (static_cast<int64_t>(p->local_col.size()) + static_cast<int64_t>(p->remote_col.size())) * (mode == MGG_AGG_GCN_SYM ? 8 : 4);
            const bool on_lines = ld_x * static_cast<int64_t>(esz) % 128 == 0 && bases % 128 == 0;
            if (static_cast<int64_t>(dim) * static_cast<int64_t>(esz) >= 1024 && no_classes) {
                slab_bytes = table_rows * 512 > (4 << 20) && table_rows * 256 <= (static_cast<int64_t>(256) << 20) ? 256 : 512;
            } else if (static_cast<int64_t>(dim) * static_cast<int64_t>(esz) >= 1024) {
                const bool ids_stay = mode == MGG_AGG_GCN_SYM && class_rows * 512 <= (800 << 10) && id_bytes <= (static_cast<int64_t>(256) << 20);
                if (class_rows * 256 <= (4 << 20) && id_bytes >= (static_cast<int64_t>(128) << 20) && on_lines && !ids_stay) {
                    slab_bytes = 256;
                    n_chunks = (id_bytes + (36 << 20) - 1) / (36 << 20);
                } else if (class_rows * 512 > (8 << 20) && class_rows * 256 <= (8 << 20)) slab_bytes = 256;
                else slab_bytes = 512;
            }
        } else if (opt >= 64) {
            slab_bytes = opt;
        }
        if (slab_bytes > 0 && slab_bytes % vec_bytes == 0 && slab_bytes / vec_bytes < nvec) slab_vecs = static_cast<int>(slab_bytes / vec_bytes);
    }
    // a lane holds at most 4 chunks of a row: wider rows are always walked in slabs of 256 vectors
    if (slab_vecs > 64 * 4) slab_vecs = 64 * 4;
    const int n_slabs = (nvec + slab_vecs - 1) / slab_vecs;
    if (n_slabs > 65535) return fail(MGG_ERR_UNSUPPORTED, "dim %d too wide (at most %d)", dim, 65535 * 64 * 4 * vec);
    int lpr = vec == 1 && bf16 ? 8 : 4;            // (rows shorter than a vector have one kernel per element type)
    while (lpr < slab_vecs && lpr < 64) lpr <<= 1;
    const int ch = (slab_vecs + 63) / 64;

    // 16-byte loads from memory into LDS want aligned addresses, unlike those into registers, and are given 32-bit row offsets
    const int64_t most_rows = std::max<int64_t>(p->n_local_rows, static_cast<int64_t>(p->halo_gid.size()));
    const bool lds = p->opt_lds_halo != 0 && !p->halo_gid.empty() && rows_aligned && ch == 1 && p->wpb <= kStageWpb &&
                     static_cast<uint64_t>(most_rows) * static_cast<uint64_t>(ld_x) * esz < (1ull << 32);
    // The fine schedule where its partial sums have room and rows are wide enough to pay for them: what a gather from L2 saves
    // goes by the row's bytes, an item and its partial sum of 4 bytes a column cost the same whatever those are.  Time with it
    // over time without, nine shares of 10 to 44 M neighbours: fp32 of up to 32 columns 1.01 to 1.28, 48 and 64 columns 0.90 to
    // 1.01, 100 to 256 columns 0.87 to 0.99; bf16 of up to 64 columns 1.03 to 1.32, 216 and 256 columns 0.93 to 1.01; 16 lanes of
    // bf16 (128 columns, or 256-byte slabs) 0.95 to 0.98 on tables of 400 k rows and more with 20 M neighbours and more, 0.99 to
    // 1.13 on smaller ones.
    const int64_t all_rows = p->n_local_rows + static_cast<int64_t>(p->halo_gid.size());
    const int64_t nnz = static_cast<int64_t>(p->local_col.size()) + static_cast<int64_t>(p->remote_col.size());
    const bool pays = lpr >= (bf16 ? 32 : 16) || (lpr == 16 && all_rows >= (3 << 17) && nnz >= 20000000);
    // Not with halo rows through LDS, which are staged 8 KB at a time however few a piece has (17.8 M neighbours at 64 columns
    // 0.721 ms with it, 0.609 without; 28 M at 128 in bf16 1.43 and 1.16), nor in two launches, which walk every piece twice and
    // add up its partial sums twice (0.449 and 0.406; 1.01 and 0.88).
    pl.fine = pays && !lds && !two_launches(p) && p->n_fine_sums > 0 && scratch_rows >= p->n_split_items + p->n_fine_sums;
    pl.n_items = static_cast<int32_t>(pl.fine ? p->fine_items.size() : p->items.size());
    const int32_t n_short = static_cast<int32_t>(p->short_rows.size());
    // Few items: a team of wavefronts takes each of them together (aggregate_team_kernel), 8 or 4 to an item up to 4096
    // wavefronts in all, 2 up to 8192, where the chain of loads behind the longest item is what the launch waits for: each
    // member of its team has a batch of 8 loads at least, and not less than the launch's loads come to on each of the 5120
    // wavefronts that are resident (1.5 times that for teams of 4, 3 times for 8; an item or a group of short rows counts as a
    // batch more).  Without that second half, launches that other rows keep busy or whose items are all short were up to 28 %
    // slower with a team than without (3,100 rows of 22 neighbours at 128 columns; 300 rows of 2,000 beside 100,000 short ones at
    // 128 columns: 96 us, 85 without).  Over 632 launches, four team sizes each, the rule is 1.4 % off the best on average, no team
    // 6.6 %, the rule without the second half 3.8 %.  A caller who says how many wavefronts a workgroup or how many items a
    // wavefront takes gets just that.
    bool team = false;
    int wpb = p->wpb;
    const int npw = 64 / lpr;
    const int64_t short_groups = (n_short + npw - 1) / npw;
    if (ch == 1 && !lds && p->opt_items_per_wave == 0 && !p->wpb_given) {
        const int64_t item_waves = p->n_work_items * n_slabs, loads = (nnz / npw + 8 * (short_groups + p->n_work_items)) * n_slabs;
        for (int t = kMaxTeam; t >= 2 && !team; t /= 2)
            if (item_waves * t <= (t == 2 ? 8192 : 4096) && p->longest_item / (t * npw) >= std::max<int64_t>(8, (t == 2 ? 2 : t == 4 ? 3 : 6) * loads / (2 * 5120))) { team = true; wpb = t; }
    }
    const int64_t n_groups = team ? pl.n_items : (pl.n_items + wpb - 1) / wpb;
    // Work per wavefront: M items one after the other, pipelined.  More per wavefront amortises its start-up latencies; fewer
    // leaves more workgroups for the hardware to balance.  Automatic: 2 where the launch still has about 8192 workgroups
    // (0.3-2.5 % faster than 1 and than 8 on every workload tried), else 1.  Groups of short rows: the same for rows of a graph
    // whose ids fit their 16 lanes or more, all requested with the group before (260 k-node R-MAT, half, 75 columns 140.3 -> 137.2
    // us; 28 M neighbours at 75 columns 1.034 -> 1.024 ms, at 128 1.497 -> 1.488); one where a row takes fewer lanes (16 columns 46.2
    // -> 49.8 us with 2) and in bags, whose longer lists are requested ahead in the group itself (26 lookups of 64 columns 241 ->
    // 245 us with 2).
    if (team) pl.items_per_wave = 1;
    else if (p->opt_items_per_wave > 0) pl.items_per_wave = p->opt_items_per_wave;
    else pl.items_per_wave = static_cast<int32_t>(std::min<int64_t>(2, std::max<int64_t>(1, n_groups * n_slabs / 8192)));
    if (p->opt_short_per_wave > 0) pl.short_per_wave = p->opt_short_per_wave;
    else if (p->bags || lpr < 16) pl.short_per_wave = 1;
    else pl.short_per_wave = static_cast<int32_t>(std::min<int64_t>(2, std::max<int64_t>(1, (short_groups + wpb - 1) / wpb * n_slabs / 8192)));
    pl.n_item_blocks = team ? team_blocks(pl.n_items) : static_cast<int32_t>((n_groups + static_cast<int64_t>(kXcd) * pl.items_per_wave - 1) / (static_cast<int64_t>(kXcd) * pl.items_per_wave) * kXcd);
    const int64_t short_waves = (short_groups + pl.short_per_wave - 1) / pl.short_per_wave;
    pl.grid_x = pl.n_item_blocks + static_cast<int>((short_waves + wpb - 1) / wpb);
    if (n_slabs > 1) pl.grid_x = (pl.grid_x + kXcd - 1) / kXcd * kXcd;   // keeps workgroup x on XCD x mod 8 in every slab
    pl.n_chunks = std::max<int64_t>(1, std::min<int64_t>({n_chunks, pl.grid_x / kXcd, 65535 / n_slabs}));
    pl.chunk_x = pl.n_chunks == 1 ? pl.grid_x : static_cast<int>((pl.grid_x + pl.n_chunks * kXcd - 1) / (pl.n_chunks * kXcd) * kXcd);
    if (pl.chunk_x > 0) pl.n_chunks = (pl.grid_x + pl.chunk_x - 1) / pl.chunk_x;
    pl.vec = vec; pl.nvec = nvec; pl.slab_vecs = slab_vecs; pl.n_slabs = n_slabs; pl.lpr = lpr; pl.ch = ch;
    pl.lds = lds; pl.team = team; pl.wpb = wpb;
    *out = pl;
    return MGG_OK;
}

}  // namespace

mgg_status_t launch_aggregate(const mgg_partition *p, mgg_agg_t mode, float eps, mgg_dtype_t x_dtype,
                              const void *x_local, const void *x_halo, int32_t dim, int64_t ld_x, void *out,
                              int64_t ld_out, hipStream_t stream, const float *bias, mgg_act_t act, int32_t out_dim,
                              mgg_dtype_t out_dtype, float *scratch, size_t scratch_bytes)
{
    const bool bf16 = x_dtype == MGG_BF16;
    const void *xh = x_halo ? x_halo : x_local;   // never dereferenced when there is no halo
    if (out_dim <= 0) out_dim = dim;
    // scratch rows for the partial sums of split rows: the caller's buffer, else the partition's own;
    // nothing is allocated here
    int64_t scratch_ld = scratch_ld_for(dim), scratch_rows = p->d.scratch_rows;
    if (scratch) scratch_rows = static_cast<int64_t>(scratch_bytes / (static_cast<size_t>(scratch_ld) * sizeof(float)));
    Plan pl;
    mgg_status_t s = plan_aggregate(p, mode, bf16, dim, ld_x, reinterpret_cast<uint64_t>(x_local) | reinterpret_cast<uint64_t>(xh), scratch_rows, &pl);
    if (s != MGG_OK) return s;
    if (p->n_split_items > 0) {
        const size_t need = static_cast<size_t>(p->n_split_items) * static_cast<size_t>(scratch_ld) * sizeof(float);
        if (scratch) {
            if (scratch_bytes < need) return fail(MGG_ERR_INVALID_ARG, "scratch of %zu bytes given, width %d needs %zu", scratch_bytes, dim, need);
            if (!aligned(scratch, 32)) return fail(MGG_ERR_INVALID_ARG, "scratch must be 32-byte aligned");
        } else {
            if (p->d.scratch_ld < scratch_ld)
                return fail(MGG_ERR_INVALID_ARG, "no scratch for width %d: call mgg_partition_reserve(p, %d) first (reserved: %lld columns)", dim, dim,
                            (long long)p->d.scratch_ld);
            scratch = p->d.scratch;
            scratch_ld = p->d.scratch_ld;
        }
    }

    AggArgs a{};
    a.cols = p->d.cols; a.wts = p->d.wts;
    a.dinv_own = p->d.dinv_own;
    a.short_desc = p->d.short_desc; a.items = pl.fine ? p->d.fine_items : p->d.items;
    a.x_local = x_local; a.x_halo = xh;
    a.out = out; a.scratch = scratch;
    a.ld_x = ld_x; a.ld_out = ld_out; a.scratch_ld = scratch_ld;
    a.nvec = pl.nvec; a.last_col = pl.last_col; a.slab_vecs = pl.slab_vecs; a.n_slabs = pl.n_slabs;
    a.n_items = pl.n_items; a.n_item_blocks = pl.n_item_blocks; a.items_per_wave = pl.items_per_wave;
    a.n_short = static_cast<int32_t>(p->short_rows.size()); a.short_per_wave = pl.short_per_wave;
    const dim3 grid(static_cast<unsigned>(pl.chunk_x), static_cast<unsigned>(pl.n_slabs * pl.n_chunks));
    a.ps = p->ps;
    const bool gcn = mode == MGG_AGG_GCN_SYM;
    a.self_w = p->bags ? 0.f : 1.f + eps;
    a.no_self = p->bags ? 1 : 0;
    a.bias = bias;
    a.out_dim = out_dim;
    a.relu = act == MGG_ACT_RELU;
    a.out_bf16 = out_dtype == MGG_BF16;
    // one launch for both neighbour lists, or two
    const bool two_phases = two_launches(p) && out_dtype != MGG_BF16;   // phase 2 reads `out` back
    for (int phase = two_phases ? 1 : 0; phase <= (two_phases ? 2 : 0); ++phase) {
        a.phase = phase;
        if (pl.grid_x > 0) {
            hipError_t e;
            if (bf16) e = launch_aggregate_bf16(a, gcn, pl.vec, grid, pl.wpb, stream, pl.lpr, pl.ch, pl.lds, pl.team);
            else e = launch_aggregate_f32(a, gcn, pl.vec, grid, pl.wpb, stream, pl.lpr, pl.ch, pl.lds, pl.team);
            if (e != hipSuccess) return hip_fail(e, "aggregate kernel launch");
        }
        const int32_t n_split = static_cast<int32_t>(p->split_rows.size() + (pl.fine ? p->fine_split_rows.size() : 0));
        if (n_split > 0) {
            const dim3 fgrid(static_cast<unsigned>((n_split + kWavesPerBlock - 1) / kWavesPerBlock));
            if (bf16)
                hipLaunchKernelGGL(fixup_kernel<true>, fgrid, dim3(kBlock), 0, stream, p->d.split_rows, n_split, out_dim, scratch,
                                   scratch_ld, x_local, ld_x, p->d.dinv_own, gcn ? 1 : 0, a.self_w, out, a.out_bf16, ld_out, a.phase, bias, a.relu, a.no_self);
            else
                hipLaunchKernelGGL(fixup_kernel<false>, fgrid, dim3(kBlock), 0, stream, p->d.split_rows, n_split, out_dim, scratch,
                                   scratch_ld, x_local, ld_x, p->d.dinv_own, gcn ? 1 : 0, a.self_w, out, a.out_bf16, ld_out, a.phase, bias, a.relu, a.no_self);
            hipError_t e = hipGetLastError();
            if (e != hipSuccess) return hip_fail(e, "fix-up kernel launch");
        }
    }
    return MGG_OK;
}

// what plan_aggregate decides, for mgg_aggregate_plan
mgg_status_t describe_plan(const mgg_partition *p, mgg_agg_t mode, mgg_dtype_t x_dtype, int32_t dim, int64_t ld_x, int32_t base_align, size_t scratch_bytes,
                           mgg_aggregate_plan_t *o)
{
    const bool bf16 = x_dtype == MGG_BF16;
    const int64_t rows = static_cast<int64_t>(std::min<size_t>(scratch_bytes / (static_cast<size_t>(scratch_ld_for(dim)) * sizeof(float)), INT64_MAX));
    Plan pl;
    const mgg_status_t s = plan_aggregate(p, mode, bf16, dim, ld_x, static_cast<uint64_t>(base_align), rows, &pl);
    if (s != MGG_OK) return s;
    o->lanes_per_row = pl.lpr; o->vectors_per_lane = pl.ch;
    o->slab_bytes = static_cast<int32_t>(static_cast<size_t>(pl.slab_vecs) * pl.vec * (bf16 ? 2 : 4));
    o->n_slabs = pl.n_slabs; o->n_chunks = static_cast<int32_t>(pl.n_chunks);
    o->team = pl.team ? pl.wpb : 1; o->wpb = pl.wpb;
    o->items_per_wave = pl.items_per_wave; o->short_per_wave = pl.short_per_wave;
    o->fine = pl.fine; o->lds_halo = pl.lds;
    o->n_workgroups = static_cast<int64_t>(pl.chunk_x) * pl.n_slabs * pl.n_chunks;
    return MGG_OK;
}

}  // namespace mgg
