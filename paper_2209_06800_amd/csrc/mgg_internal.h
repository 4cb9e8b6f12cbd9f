// Internal declarations shared by the translation units of libmgg (not installed).
#pragma once

#include <hip/hip_runtime_api.h>
#include <hip/hip_vector_types.h>

#include <cstdarg>
#include <cstdint>
#include <memory>
#include <vector>

#include "mgg.h"

namespace mgg {

// One wavefront work item: a run of neighbour partitions of one owned row, from the local list and from the remote list
// (section 5.1: a warp handles pairs of local / remote partitions; the kernel walks the local ones first).  slot < 0: the item covers the whole row and writes the final value;
// slot >= 0: it writes a raw partial sum into scratch row `slot`.  row < 0: padding, nothing to do.
struct WorkItem {
    int32_t row;
    int32_t lbeg, lend;   // range in local_col
    int32_t rbeg, rend;   // range in remote_col
    int32_t slot;
    int32_t pad0, pad1;
};

// The same on the device, where an item's neighbours lie in one run of `cols`: the local ones, then the remote ones.
// (Pieces of rows that are whole items in the other schedule leave the remote ones where they are: `rbeg`.)
struct DeviceItem {
    int32_t row, beg, n_local, n, slot, rbeg;
    int32_t pad[2];
};
static_assert(sizeof(DeviceItem) == 32, "a wavefront reads an item as eight dwords");

// A row that was cut into several items: its partial sums sit in scratch rows
// [first_slot, first_slot + n_slots) and are combined in that order.
struct SplitRow {
    int32_t row;
    int32_t first_slot;
    int32_t n_slots;
    int32_t pad;
};

constexpr int kXcd = 8;             // accelerator complex dies of an MI355X, each with its own L2
constexpr int kDefaultWpb = 2;      // work items (wavefronts) per workgroup of the aggregation kernel
constexpr int kDefaultXcdMinDeg = 256;

// Item of workgroup b where a workgroup takes one item: items lie in groups of kDefaultWpb per XCD queue (the only group
// size there are teams for), and workgroup b runs on XCD b mod kXcd, so that queue x stays on XCD x.
constexpr int team_item(int b) { return ((b / kXcd / kDefaultWpb) * kXcd + b % kXcd) * kDefaultWpb + b / kXcd % kDefaultWpb; }
static_assert(team_item(0) == 0 && team_item(1) == 2 && team_item(kXcd) == 1 && team_item(kXcd + 7) == 15 && team_item(2 * kXcd) == 16, "items 0, 1, 16, 17 are queue 0");
constexpr int team_blocks(int n_items) { return (n_items + kXcd * kDefaultWpb - 1) / (kXcd * kDefaultWpb) * (kXcd * kDefaultWpb); }
constexpr int kFineXcdMinDeg = 128;         // rows regrouped in the fine schedule too
constexpr int64_t kFineMinNeighbours = 8 << 20;   // shares of fewer neighbours have none
constexpr int kFineMinDim = 32;             // up to this width it is never taken (plan_aggregate)
constexpr int kDefaultHotPhases = 0;        // automatic choice between hash classes and popularity phases
constexpr int kAutoHotPhases = 4;           // phases when the automatic choice takes popularity classes
constexpr int kMaxHotPhases = 31;           // class index phase * 8 + XCD has to stay below kColdClass
constexpr int kDefaultMinPiece = 16;        // a class with fewer neighbours in a row joins the row's cold piece
constexpr int kDefaultHotMinCount = 8;      // table rows gathered fewer times than this are never hot
constexpr int kColdClass = 255;
constexpr int64_t kHotBytesPerXcd = 3 << 20;   // of the 4 MB L2 of one XCD, what the hot rows of a phase may fill

struct DeviceArrays {
    uint32_t *cols = nullptr;          // table rows of the neighbours in the order of the work (bit 31 set: row of the halo table)
    float *wts = nullptr;              // 1/sqrt(deg+1) of the neighbour, per entry of cols
    float *dinv_own = nullptr;
    int4 *short_desc = nullptr;        // per short row: row, start in cols, local neighbours, all neighbours
    DeviceItem *items = nullptr;
    DeviceItem *fine_items = nullptr;
    SplitRow *split_rows = nullptr;    // those of the fine schedule alone follow the others
    float *scratch = nullptr;          // [scratch_rows x scratch_ld] partial sums
    int64_t scratch_ld = 0, scratch_rows = 0;
};

// What the device arrays are filled with, laid out on the host (lay_out_device).
struct DeviceLayout {
    size_t nnz = 0;
    std::unique_ptr<uint32_t[]> cols;
    std::unique_ptr<float[]> wts;      // empty for bags: plain sums only
    std::vector<int4> short_desc;
    std::vector<DeviceItem> items, fine_items;
    std::vector<SplitRow> split_rows;
};

}  // namespace mgg

struct mgg_partition {
    int64_t num_nodes = 0, lb = 0, ub = 0, n_own = 0;
    int64_t n_local_rows = 0;         // rows of the local table: n_own for a graph partition, the local slice for bags
    bool bags = false;                // built by mgg_build_bags: owned rows are bags, no self term, plain sums
    int32_t num_parts = 1, part_id = 0;
    int32_t ps = 64, dist = 8, short_max = 16, xcd_min_deg = -1, wpb = 4;
    bool wpb_given = false;           // by the caller: every launch keeps to it
    int32_t hot_rows = 0, hot_phases = 0, n_phases = 0, min_piece = 0, hot_min_count = 0;
    int32_t class_mode = 0;           // 0: no source classes, 1: by hash, 2: by popularity
    std::vector<uint8_t> src_class;   // class of every table row (local rows, then halo slots); empty: no classes
    int device = -1;  // HIP device the arrays live on; -1 = host only
    std::vector<int32_t> local_row_ptr, local_col, remote_row_ptr, remote_col;
    std::vector<int32_t> sched_local_col, sched_remote_col;   // rows in the order they are walked, regrouped ones by source class (empty: same as above)
    std::vector<int32_t> halo_gid, deg_own, deg_halo;
    std::vector<int64_t> halo_peer_ptr;
    std::vector<float> dinv_own, dinv_halo;
    std::vector<int32_t> short_rows;
    std::vector<mgg::WorkItem> items;
    std::vector<mgg::SplitRow> split_rows;
    int64_t n_split_items = 0;
    // The fine schedule (empty: none): rows of kFineXcdMinDeg to 255 neighbours are pieces by source class, too.  It is taken
    // where the scratch at hand holds its partial sums, which are at most three times as many.
    std::vector<mgg::WorkItem> fine_items;
    std::vector<mgg::SplitRow> fine_split_rows;      // of those rows; their partial sums follow the others
    int64_t n_fine_sums = 0;
    int64_t n_work_items = 0;         // items without the padding of the XCD queues
    int32_t longest_item = 0;         // neighbours of the longest one
    int64_t n_classed = 0;            // neighbours in rows that are cut by source class
    // run-time switches of this partition's aggregations: the process-wide defaults at build time, then mgg_partition_set_option
    int32_t opt_lds_halo = 0, opt_col_slab_bytes = 0, opt_split_phases = 0, opt_items_per_wave = 0, opt_short_per_wave = 0;
    int32_t reserved_dim = 0;         // widest aggregation the partition's own scratch buffer was sized for
    int64_t n_groups_local = 0, n_groups_remote = 0;
    mgg::DeviceArrays d;          // device copies; d.scratch is sized by mgg_partition_reserve (or at build)
};

namespace mgg {

mgg_status_t fail(mgg_status_t code, const char *fmt, ...) __attribute__((format(printf, 2, 3)));
mgg_status_t hip_fail(hipError_t e, const char *what);
mgg_status_t alloc_fail(hipError_t e, size_t bytes, const char *what);

#define MGG_HIP_TRY(expr)                                    \
    do {                                                     \
        hipError_t _e = (expr);                              \
        if (_e != hipSuccess) return ::mgg::hip_fail(_e, #expr); \
    } while (0)

int32_t option_lds_halo();
int32_t option_col_slab_bytes();
int32_t option_split_phases();
int32_t option_update_stream();
int32_t option_items_per_wave();
void take_default_options(mgg_partition *p);      // copies the four process-wide defaults above into a new partition
mgg_status_t check_option(const char *key, int32_t value);   // range check shared by both setters

// kernels (aggregate.hip / update.hip)
mgg_status_t launch_aggregate(const mgg_partition *p, mgg_agg_t mode, float eps, mgg_dtype_t x_dtype,
                              const void *x_local, const void *x_halo, int32_t dim, int64_t ld_x,
                              void *out, int64_t ld_out, hipStream_t stream, const float *bias = nullptr,
                              mgg_act_t act = MGG_ACT_NONE, int32_t out_dim = 0, mgg_dtype_t out_dtype = MGG_F32,
                              float *scratch = nullptr, size_t scratch_bytes = 0);
// bias / act: optional epilogue of the final value.  out_dim (0 = dim): columns of `out` that exist
// when the tables carry padding columns beyond them (dim counts the padded width).  out_dtype BF16: the
// rows are rounded to bf16 (nearest even) on the way out -- what the bf16 MFMA would do on the way in.
// scratch / scratch_bytes: where the partial sums of rows cut into several items go; NULL = the partition's
// own buffer (mgg_partition_reserve).  The launch allocates nothing: too small a buffer is an error.
inline int64_t scratch_ld_for(int32_t dim) { return (static_cast<int64_t>(dim) + 7) / 8 * 8; }   // rows of partial sums start on 32-byte boundaries
// (the least an aggregation can do with, and what it has a use for)
inline int64_t scratch_rows_wanted(const mgg_partition *p, int32_t dim) { return p->n_split_items + (dim > kFineMinDim ? p->n_fine_sums : 0); }
inline size_t scratch_bytes_wanted(const mgg_partition *p, int32_t dim) { return static_cast<size_t>(scratch_rows_wanted(p, dim)) * static_cast<size_t>(scratch_ld_for(dim)) * sizeof(float); }
inline size_t scratch_bytes_for(const mgg_partition *p, int32_t dim) { return static_cast<size_t>(p->n_split_items) * static_cast<size_t>(scratch_ld_for(dim)) * sizeof(float); }
// what launch_aggregate would launch (host arithmetic, host-only partitions too)
mgg_status_t describe_plan(const mgg_partition *p, mgg_agg_t mode, mgg_dtype_t x_dtype, int32_t dim, int64_t ld_x, int32_t base_align, size_t scratch_bytes,
                           mgg_aggregate_plan_t *o);
// the library's fixed scratch array on the current device (aggregate.hip); NULL + error set on failure
float *static_scratch(size_t *bytes);
mgg_status_t launch_update(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, int32_t d_in,
                           mgg_dtype_t w_dtype, const void *w, const float *bias, int32_t d_out,
                           mgg_act_t act, mgg_dtype_t out_dtype, void *out, int64_t ld_out,
                           hipStream_t stream);

// Two chained Updates; one kernel when the shape is covered, otherwise two launches through `hidden`
// ([n_rows x dims[1]], bf16 with bf16 weights, else fp32).
mgg_status_t launch_update_mlp(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, const int32_t dims[3],
                               mgg_dtype_t w_dtype, const void *w1, const float *b1, mgg_act_t act1, const void *w2, const float *b2,
                               mgg_act_t act2, void *hidden, int64_t ld_hidden, mgg_dtype_t out_dtype, void *out, int64_t ld_out,
                               hipStream_t stream);
mgg_status_t probe_gather(int64_t table_bytes, int32_t row_bytes, int64_t n_gathers, int32_t iters, uint64_t seed, double *gbs);
// in place: x[i][:] = softmax(x[i][:]) for every row (update.hip)
mgg_status_t launch_row_softmax(int64_t n_rows, int32_t d, mgg_dtype_t dtype, void *x, int64_t ld, hipStream_t stream);

}  // namespace mgg
