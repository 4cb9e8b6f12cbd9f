// Device code of the neighbour aggregation for gfx950 (section 1 "GNN" equation; section 4.1 LR / LL /
// AC stages; section 5.1 warp-per-partition mapping with local and remote work interleaved; section 5.2
// asynchronous remote access staged through shared memory).  Included by the translation units that
// instantiate the kernels for one element type each.
//
// Mapping, per 64-lane wavefront:
//   - a row of an embedding table is spread over LPR lanes (LPR = 4..64, a power of two), each lane
//     owning VEC contiguous elements per chunk (16-byte loads, at any element boundary), so one load
//     instruction fetches NPW = 64/LPR neighbour rows;
//   - a work item is a run of neighbours of ONE owned row, its local partitions followed by its remote ones,
//     taken ps (<= 64) at a time, so every wavefront mixes both kinds;
//   - the ids are loaded one per lane; the lane that holds an id turns it into the
//     address of its table row once, and the addresses (and GCN factors) reach the lanes that gather
//     through DPP row broadcasts, which cost no LDS access and no wait;
//   - the NPW sub-wave accumulators are combined with lane swaps at the end;
//   - short rows are handled one per sub-wave (several rows per wavefront);
//   - rows cut into several items leave raw partial sums in scratch rows, and a second small kernel
//     adds them in a fixed order (results do not depend on scheduling).
// Bound by the memory hierarchy (about 0.5 flop per byte): no MFMA here.  A bare gather loop of this form delivers
// 28.8 TB/s of 256-byte rows out of L2 (2 MB table, ids from the Infinity Cache), 22.4 with ids from HBM, 13.5 from an
// 8 MB table and 7.6 from 64 MB; one dword per lane and row, ids in scalar registers, stays at 18.5 TB/s out of L2.
#pragma once

#include <hip/hip_runtime.h>

#include <type_traits>

#include "mgg_internal.h"

namespace mgg {

#ifndef MGG_AGG_INFLIGHT
#define MGG_AGG_INFLIGHT 8          // loads a lane keeps in flight per batch
#endif
constexpr int kWave = 64;
constexpr int kMaxWpb = 16;         // wavefronts per workgroup of the aggregation kernel
constexpr int kMaxTeam = 8;         // wavefronts that take one item together in a small launch
constexpr int kStageSlots = 8;      // LDS-staged variant: load instructions (1 KB each) per wavefront stage
constexpr int kStageWpb = 8;        // LDS-staged variant: most wavefronts per workgroup (a wavefront owns 2 stages of 8 KB)

struct AggArgs {
    const uint32_t *cols;                // table rows of the neighbours in the order of the work (bit 31 set: halo table)
    const float *wts;                    // GCN: factor of the neighbour, one per entry of cols
    const float *dinv_own;               // 1/sqrt(deg+1) of the owned rows (the row factor of GCN)
    const DeviceItem *items;
    const void *x_local, *x_halo;
    void *out;               // fp32, or bf16 when out_bf16 (rounded to nearest even)
    float *scratch;
    int64_t ld_x, ld_out, scratch_ld;
    int32_t nvec;            // vectors of VEC elements per row (dim / VEC)
    int32_t slab_vecs;       // vectors per column slab (= nvec: one slab)
    int32_t n_slabs;         // blockIdx.y counts the slabs of one chunk of the work (gridDim.x workgroups), then those of the next
    int32_t n_items, n_item_blocks, n_short;
    int32_t items_per_wave;  // work items a wavefront takes one after the other (M)
    int32_t short_per_wave;  // groups of 64/LPR short rows a wavefront takes one after the other
    const int4 *short_desc;  // per short row: row, start in cols, local neighbours, all neighbours
    int32_t ps;
    float self_w;            // GIN: 1 + eps
    int32_t out_bf16;
    int32_t no_self;         // bags: the owned row has no embedding of its own, x_local is only a table
    int32_t last_col;        // first column of the last vector: (nvec - 1) * VEC, or less when that vector is moved back to end
                             // with the row (it then gathers some columns of its neighbour and drops them)
    int32_t out_dim;         // columns of `out` that exist (<= nvec * VEC; the rest of the last vector is padding of the tables)
    int32_t phase;           // 0: local and remote lists in one launch; 1: local lists (+ self term) only;
                             // 2: remote lists only, added to what phase 1 left in out
    const float *bias;       // optional epilogue of the final value: + bias[column], then ReLU if relu != 0
    int32_t relu;            // (used when the Update's matrix product was applied before the aggregation)
};

// ---- element access ---------------------------------------------------------------------
template <bool BF16, int VEC> struct Raw;
template <> struct Raw<false, 4> { using type = float4; };
template <> struct Raw<false, 1> { using type = float; };
template <> struct Raw<true, 8> { using type = uint4; };
template <> struct Raw<true, 1> { using type = uint16_t; };

// Loads and stores of a vector that is only as aligned as its elements (global memory takes 16-byte
// accesses at any element boundary; the code only must not promise more).
template <class T, int ALIGN = 4>
__device__ __forceinline__ T load_loose(const void *p)
{
    T v;
    __builtin_memcpy(&v, __builtin_assume_aligned(p, ALIGN), sizeof v);
    return v;
}
template <class T, int ALIGN = 4>
__device__ __forceinline__ void store_loose(void *p, const T &v) { __builtin_memcpy(__builtin_assume_aligned(p, ALIGN), &v, sizeof v); }

__device__ __forceinline__ float bf16_lo(uint32_t d) { return __uint_as_float(d << 16); }
__device__ __forceinline__ float bf16_hi(uint32_t d) { return __uint_as_float(d & 0xffff0000u); }

template <bool BF16, int VEC>
__device__ __forceinline__ void unpack(const typename Raw<BF16, VEC>::type &r, float (&f)[VEC])
{
    if constexpr (!BF16) {
        if constexpr (VEC == 4) { f[0] = r.x; f[1] = r.y; f[2] = r.z; f[3] = r.w; }
        else { f[0] = r; }
    } else {
        if constexpr (VEC == 8) {
            f[0] = bf16_lo(r.x); f[1] = bf16_hi(r.x); f[2] = bf16_lo(r.y); f[3] = bf16_hi(r.y);
            f[4] = bf16_lo(r.z); f[5] = bf16_hi(r.z); f[6] = bf16_lo(r.w); f[7] = bf16_hi(r.w);
        } else { f[0] = __uint_as_float(static_cast<uint32_t>(r) << 16); }
    }
}

template <int VEC>
__device__ __forceinline__ void store_vec(float *dst, const float (&v)[VEC])
{
    if constexpr (VEC == 8) {
        store_loose<float4>(dst, make_float4(v[0], v[1], v[2], v[3]));
        store_loose<float4>(dst + 4, make_float4(v[4], v[5], v[6], v[7]));
    } else if constexpr (VEC == 4) {
        store_loose<float4>(dst, make_float4(v[0], v[1], v[2], v[3]));
    } else {
        dst[0] = v[0];
    }
}

// To bf16 bits, nearest even, a NaN to a NaN, in one instruction for one value or two.  (Rounding in integers takes nine for a
// pair and carries a NaN whose low bits are set over into -0.)
__device__ __forceinline__ uint32_t pack_bf16(float lo, float hi)
{
    typedef float f32x2 __attribute__((ext_vector_type(2)));
    typedef __bf16 bf16x2 __attribute__((ext_vector_type(2)));
    const f32x2 f = {lo, hi};
    union { bf16x2 b; uint32_t u; } r;
    r.b = __builtin_convertvector(f, bf16x2);
    return r.u;
}
__device__ __forceinline__ uint16_t to_bf16(float f) { return static_cast<uint16_t>(pack_bf16(f, 0.f)); }

// bf16 output: the same VEC values, rounded, as one 2*VEC-byte store
template <int VEC>
__device__ __forceinline__ void store_vec_bf16(uint16_t *dst, const float (&v)[VEC])
{
    if constexpr (VEC >= 2) {
        uint32_t pk[VEC / 2];
#pragma unroll
        for (int e = 0; e < VEC / 2; ++e) pk[e] = pack_bf16(v[2 * e], v[2 * e + 1]);
        if constexpr (VEC == 8) store_loose<uint4, 2>(dst, make_uint4(pk[0], pk[1], pk[2], pk[3]));
        else store_loose<uint2, 2>(dst, make_uint2(pk[0], pk[1]));
    } else {
        dst[0] = to_bf16(v[0]);
    }
}

// ---- one kernel configuration --------------------------------------------------------------
template <bool BF16_, int VEC_, int LPR_, int CH_>
struct Cfg {
    static constexpr bool BF16 = BF16_;
    static constexpr int VEC = VEC_, LPR = LPR_, CH = CH_;
    static constexpr int NPW = kWave / LPR;                 // neighbour rows per load instruction
    static constexpr int U = MGG_AGG_INFLIGHT / CH < LPR ? MGG_AGG_INFLIGHT / CH : LPR;   // neighbour rows in flight per lane
    static_assert(U > 0 && LPR % U == 0, "batches have to divide the slots of a sub-wave");
    // Wavefronts per SIMD the register allocation must allow.  The workgroup limit (16 wavefronts) gives 4; the
    // 256-byte fp32 variant is held to 5.  More spills or starves the batches: 602 columns, 116 M neighbours, 17.58 ms
    // so, 17.7 at 6, 19.2 at 7, 18.5 at 8 with batches of 4 loads, 18.7 at 4 with batches of 16.
    static constexpr int MIN_WAVES = (!BF16_ && VEC_ == 4 && LPR_ == 16 && CH_ == 1) ? 5 : 4;
    using elem = typename std::conditional<BF16, uint16_t, float>::type;
    using raw = typename Raw<BF16, VEC>::type;
};

template <class K>
struct Acc {
    float v[K::CH][K::VEC];
    __device__ __forceinline__ void clear()
    {
#pragma unroll
        for (int c = 0; c < K::CH; ++c)
#pragma unroll
            for (int e = 0; e < K::VEC; ++e) v[c][e] = 0.f;
    }
    __device__ __forceinline__ void add(int c, const typename K::raw &r, float w)
    {
        float f[K::VEC];
        unpack<K::BF16, K::VEC>(r, f);
#pragma unroll
        for (int e = 0; e < K::VEC; ++e) v[c][e] = fmaf(w, f[e], v[c][e]);
    }
    __device__ __forceinline__ void add(int c, const typename K::raw &r)      // weight 1
    {
        float f[K::VEC];
        unpack<K::BF16, K::VEC>(r, f);
#pragma unroll
        for (int e = 0; e < K::VEC; ++e) v[c][e] += f[e];
    }
};

// Where the lanes of a wavefront sit in a table row: the byte offset of each chunk this lane gathers.
// A lane whose columns lie beyond the end of the slab gathers the slab's last vector instead (valid
// memory, never written back), so that no load of the inner loop needs a predicate.
template <class K>
struct Lanes {
    int sub, slot;              // which neighbour row of a load instruction; the lane's place in its sub-wave
    int lis;                    // first vector of the row this lane owns
    int vend;                   // end of the column slab (in vectors)
    int block;                  // workgroup of its slab
    uint32_t col_off[K::CH];    // byte offset of each chunk in a table row
    __device__ __forceinline__ void init(const AggArgs &a, int lane)
    {
        sub = lane / K::LPR;
        slot = lane % K::LPR;
        const int chunk = static_cast<int>(blockIdx.y) / a.n_slabs, slab = static_cast<int>(blockIdx.y) - chunk * a.n_slabs;
        block = chunk * static_cast<int>(gridDim.x) + static_cast<int>(blockIdx.x);      // (past the last one: no short row is left)
        lis = lane % K::LPR + slab * a.slab_vecs;
        vend = min(a.nvec, (slab + 1) * a.slab_vecs);
#pragma unroll
        for (int c = 0; c < K::CH; ++c) col_off[c] = static_cast<uint32_t>(min(min(c * K::LPR + lis, vend - 1) * K::VEC, a.last_col)) * static_cast<uint32_t>(sizeof(typename K::elem));
    }
};

// Loads from an address and an offset as global memory, aligned to an element only (an address that is the same in all
// lanes stays in scalar registers).
template <int ALIGN> struct Vec16;
template <> struct Vec16<4> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(4))); };
template <> struct Vec16<2> { typedef uint32_t type __attribute__((ext_vector_type(4), aligned(2))); };
template <class T, int ALIGN>
__device__ __forceinline__ T load_at(uint64_t addr, uint32_t off)
{
    T v;
    const auto at = reinterpret_cast<const __attribute__((address_space(1))) char *>(addr) + off;
    if constexpr (sizeof(T) == 16) {
        const auto q = *reinterpret_cast<const __attribute__((address_space(1))) typename Vec16<ALIGN>::type *>(at);
        __builtin_memcpy(&v, &q, sizeof v);
    } else {
        v = *reinterpret_cast<const __attribute__((address_space(1))) T *>(at);
    }
    return v;
}

// ---- neighbours of a sub-wave: one per slot ---------------------------------------------------
// Lane `slot` of a sub-wave holds one neighbour: the address of its table row and, for GCN, its factor.  Step T of
// the gather takes the neighbour in slot T of every sub-wave; its address reaches the lanes of the sub-wave through
// DPP row broadcasts (a DPP row is 16 lanes; a sub-wave of 8 or 4 lanes takes one masked broadcast per sub-wave of
// a row, one of 32 lanes keeps its upper 16 slots in a second register so that both its rows hold all of them), or
// through v_readlane where a row takes the whole wavefront.  Against handing offsets round with ds_bpermute this takes
// no LDS instruction and no wait for one: with the joint runs of both tables and the order of the ids it is worth 2.16
// against 2.30 ms on 37 M neighbours at 100 columns, 140 against 155 us on 3.2 M at 75, 0.352 against 0.374 ms on 17.8 M
// at 64.  A broadcast reads lanes that must be active: it is never placed under a lane mask.
template <class K>
struct Slots {
    static constexpr int NR = K::LPR == 32 ? 2 : 1;
    static constexpr int COUNT = K::LPR;
    uint32_t lo[NR], hi[NR], w[NR];
};

template <int N, int BANKS>
__device__ __forceinline__ uint32_t row_bcast(uint32_t old, uint32_t v)     // lane N of every DPP row, to the lanes of BANKS
{
    return static_cast<uint32_t>(__builtin_amdgcn_update_dpp(static_cast<int>(old), static_cast<int>(v), 0x150 + N, 0xf, BANKS, BANKS == 0xf));
}

// slot T of the lane's sub-wave (t0 + T where a row takes the whole wavefront; t0 is wave-uniform)
template <class K, int T>
__device__ __forceinline__ uint32_t from_slot(const uint32_t (&v)[Slots<K>::NR], int t0)
{
    if constexpr (K::LPR == 64) return static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(v[0]), t0 + T));
    else if constexpr (K::LPR == 32) return row_bcast<T % 16, 0xf>(0, v[T / 16]);
    else if constexpr (K::LPR == 16) return row_bcast<T, 0xf>(0, v[0]);
    else if constexpr (K::LPR == 8) return row_bcast<8 + T, 0xc>(row_bcast<T, 0x3>(0, v[0]), v[0]);
    else return row_bcast<12 + T, 0x8>(row_bcast<8 + T, 0x4>(row_bcast<4 + T, 0x2>(row_bcast<T, 0x1>(0, v[0]), v[0]), v[0]), v[0]);
}

// both rows of a 32-lane sub-wave: slots 0-15 in v[0], 16-31 in v[1]
template <class K>
__device__ __forceinline__ void spread(uint32_t (&v)[Slots<K>::NR])
{
    if constexpr (K::LPR == 32) {
        const auto r = __builtin_amdgcn_permlane16_swap(v[0], v[0], false, false);
        v[0] = r[0]; v[1] = r[1];
    }
}

// id of a neighbour (bit 31: halo table) -> address of its table row
template <class K>
__device__ __forceinline__ void set_slots(Slots<K> &s, uint32_t id, float w, const char *xl, const char *xh, uint64_t ldb)
{
    const uint64_t base = reinterpret_cast<uint64_t>(static_cast<int32_t>(id) < 0 ? xh : xl);
    id &= 0x7fffffffu;
    uint64_t addr = base + static_cast<uint64_t>(id) * static_cast<uint32_t>(ldb);
    if (ldb >> 32) addr += static_cast<uint64_t>(id * static_cast<uint32_t>(ldb >> 32)) << 32;
    s.lo[0] = static_cast<uint32_t>(addr); s.hi[0] = static_cast<uint32_t>(addr >> 32); s.w[0] = __float_as_uint(w);
    spread<K>(s.lo); spread<K>(s.hi); spread<K>(s.w);
}

template <class K, int T>
__device__ __forceinline__ void load_step(const Slots<K> &s, int t0, const Lanes<K> &ln, typename K::raw (&r)[K::CH])
{
    const uint64_t row = static_cast<uint64_t>(from_slot<K, T>(s.hi, t0)) << 32 | from_slot<K, T>(s.lo, t0);
#pragma unroll
    for (int c = 0; c < K::CH; ++c) {
        uint32_t off = ln.col_off[c];
        if constexpr (K::LPR == 64) asm("" : "+v"(off));      // stays 32 bits wide: one instruction adds it to the scalar address
        r[c] = load_at<typename K::raw, sizeof(typename K::elem)>(row, off);
    }
}

// MASKED: only sub-waves with more than T neighbours in this block (cnt) add theirs; the others add exactly nothing
template <class K, bool GCN, int T, bool MASKED>
__device__ __forceinline__ void add_step(Acc<K> &acc, const Slots<K> &s, int t0, const typename K::raw (&r)[K::CH], int cnt)
{
    const float w = GCN ? __uint_as_float(from_slot<K, T>(s.w, t0)) : 1.f;
#pragma unroll
    for (int c = 0; c < K::CH; ++c) {
        if constexpr (MASKED) {
            float f[K::VEC];
            unpack<K::BF16, K::VEC>(r[c], f);
#pragma unroll
            for (int e = 0; e < K::VEC; ++e) acc.v[c][e] = fmaf(w, t0 + T < cnt ? f[e] : 0.f, acc.v[c][e]);
        } else if constexpr (GCN) {
            acc.add(c, r[c], w);
        } else {
            acc.add(c, r[c]);
        }
    }
}

template <class K, int T0, int U>
__device__ __forceinline__ void load_steps(const Slots<K> &s, int t0, const Lanes<K> &ln, typename K::raw (&r)[K::U][K::CH])
{
    if constexpr (U > 0) {
        load_steps<K, T0, U - 1>(s, t0, ln, r);
        load_step<K, T0 + U - 1>(s, t0, ln, r[U - 1]);
    }
}
template <class K, bool GCN, int T0, int U, bool MASKED>
__device__ __forceinline__ void add_steps(Acc<K> &acc, const Slots<K> &s, int t0, const typename K::raw (&r)[K::U][K::CH], int cnt)
{
    if constexpr (U > 0) {
        add_steps<K, GCN, T0, U - 1, MASKED>(acc, s, t0, r, cnt);
        add_step<K, GCN, T0 + U - 1, MASKED>(acc, s, t0, r[U - 1], cnt);
    }
}

// Steps T0 .. T0 + n - 1 (n wave-uniform, 1 <= n): the loads of up to K::U of them first, then the sums.  No step that
// has nothing to gather is issued.
template <class K, int T0, int U, int I = 0>
__device__ __forceinline__ void load_some(const Slots<K> &s, int t0, int n, const Lanes<K> &ln, typename K::raw (&r)[K::U][K::CH])
{
    if constexpr (I < U) {
        if (I < n) {
            load_step<K, T0 + I>(s, t0, ln, r[I]);
        } else {
#pragma unroll
            for (int c = 0; c < K::CH; ++c) __builtin_memset(&r[I][c], 0, sizeof r[I][c]);
        }
        load_some<K, T0, U, I + 1>(s, t0, n, ln, r);
    }
}
template <class K, bool GCN, int T0, int U, bool MASKED, int I = 0>
__device__ __forceinline__ void add_some(Acc<K> &acc, const Slots<K> &s, int t0, int n, const typename K::raw (&r)[K::U][K::CH], int cnt)
{
    if constexpr (I < U) {
        if (I < n) add_step<K, GCN, T0 + I, MASKED>(acc, s, t0, r[I], cnt);
        add_some<K, GCN, T0, U, MASKED, I + 1>(acc, s, t0, n, r, cnt);
    }
}
template <class K, bool GCN, int T0, bool MASKED>
__device__ __forceinline__ void batch(Acc<K> &acc, const Slots<K> &s, int t0, int n, const Lanes<K> &ln, int cnt)
{
    typename K::raw r[K::U][K::CH];
    if (n >= K::U) {
        load_steps<K, T0, K::U>(s, t0, ln, r);
        __builtin_amdgcn_sched_barrier(0);          // every load is on its way before the first sum waits for one
        add_steps<K, GCN, T0, K::U, MASKED>(acc, s, t0, r, cnt);
    } else {
        load_some<K, T0, K::U - 1>(s, t0, n, ln, r);
        __builtin_amdgcn_sched_barrier(0);
        add_some<K, GCN, T0, K::U - 1, MASKED>(acc, s, t0, n, r, cnt);
    }
}

// n steps (n wave-uniform, 0 <= n <= COUNT) from slot T0 on, K::U at a time
template <class K, bool GCN, bool MASKED, int T0 = 0>
__device__ __forceinline__ void steps(Acc<K> &acc, const Slots<K> &s, int n, const Lanes<K> &ln, int cnt = 0)
{
    if constexpr (K::LPR == 64) {
        for (int t0 = 0; t0 < n; t0 += K::U) batch<K, GCN, 0, MASKED>(acc, s, t0, n - t0, ln, cnt);
    } else if constexpr (T0 < Slots<K>::COUNT) {
        if (n > T0) {
            batch<K, GCN, T0, MASKED>(acc, s, 0, n - T0, ln, cnt);
            steps<K, GCN, MASKED, T0 + K::U>(acc, s, n, ln, cnt);
        }
    }
}

// Accumulate one run of `len` (1 .. 64) neighbours of one row, neighbour i in lane i.  64 of them are taken as they
// lie, slot by slot of every sub-wave.  Fewer are first dealt round the sub-waves (slot i of sub-wave s: neighbour
// i NPW + s), so that all of them finish within a step of each other; what does not fill a step waits in the last
// slot and is added under a lane mask.
template <class K, bool GCN>
__device__ __forceinline__ void gather_run(Acc<K> &acc, uint32_t id, float w, int len, const char *xl, const char *xh, uint64_t ldb, const Lanes<K> &ln)
{
    Slots<K> s;
    if constexpr (K::NPW == 1) {
        set_slots<K>(s, id, w, xl, xh, ldb);
        steps<K, GCN, false>(acc, s, len, ln);
    } else {
        if (len == kWave) {
            set_slots<K>(s, id, w, xl, xh, ldb);
            steps<K, GCN, false>(acc, s, Slots<K>::COUNT, ln);
            return;
        }
        const int whole = len / K::NPW, left = len % K::NPW;
        const int from = ln.slot == K::LPR - 1 ? (ln.sub < left ? whole * K::NPW + ln.sub : 0) : ln.slot * K::NPW + ln.sub;
        id = static_cast<uint32_t>(__shfl(static_cast<int>(id), from));
        if constexpr (GCN) w = __shfl(w, from);
        set_slots<K>(s, id, w, xl, xh, ldb);
        typename K::raw last[K::CH];
        if (left) load_step<K, K::LPR - 1>(s, 0, ln, last);
        steps<K, GCN, false>(acc, s, whole, ln);
        if (left) {
            const float wl = GCN ? __uint_as_float(from_slot<K, K::LPR - 1>(s.w, 0)) : 1.f;
            if (ln.sub < left) {
#pragma unroll
                for (int c = 0; c < K::CH; ++c) acc.add(c, last[c], wl);
            }
        }
    }
}

struct ItemFields {
    int row, beg, n_l, n, slot, rbeg;      // local neighbours from beg on, the others from rbeg on
};

// Neighbour `lane` of the `len` (1 .. 64) from position `at` on.  Lanes beyond them read the first one again: what
// they hold is always a row of a table.  Both arrays are read as coalesced streams (the factors are stored per edge).
template <bool GCN>
__device__ __forceinline__ void load_run(const AggArgs &a, int at, int len, int lane, uint32_t &id, float &w)
{
    const int p = lane < len ? lane : 0;
    id = (a.cols + at)[p];
    if constexpr (GCN) w = (a.wts + at)[p];
}
// The same from position `pos` of an item on, whose remote neighbours may lie apart from its local ones.
template <bool GCN>
__device__ __forceinline__ void load_run(const AggArgs &a, const ItemFields &it, int pos, int len, int lane, uint32_t &id, float &w)
{
    const int p = pos + (lane < len ? lane : 0), at = p < it.n_l ? it.beg + p : it.rbeg + p - it.n_l;
    id = a.cols[at];
    if constexpr (GCN) w = a.wts[at];
}

// Final value of an owned row from its neighbour sum: adds the self term and the row factor.
template <class K>
__device__ __forceinline__ void write_final(const AggArgs &a, bool gcn, const Acc<K> &acc, const typename K::raw (&xs)[K::CH], int32_t row,
                                            const Lanes<K> &ln)
{
    float *o = static_cast<float *>(a.out) + static_cast<int64_t>(row) * a.ld_out;             // fp32 output
    uint16_t *ob = static_cast<uint16_t *>(a.out) + static_cast<int64_t>(row) * a.ld_out;     // bf16 output
    const float dv = gcn ? a.dinv_own[row] : 1.f;
    const float ws = gcn ? dv : a.self_w;     // GCN: dv * (sum + dv * x_v) = sum_u x_u/sqrt(du dv) + x_v/dv^2
#pragma unroll
    for (int c = 0; c < K::CH; ++c) {
        const int vi = c * K::LPR + ln.lis;
        if (vi < ln.vend) {
            const int col0 = static_cast<int>(ln.col_off[c] / sizeof(typename K::elem)), own0 = vi * K::VEC;   // own0 > col0: moved back
            float xv[K::VEC], r[K::VEC];
            if (a.no_self || a.phase == 2) {
#pragma unroll
                for (int e = 0; e < K::VEC; ++e) xv[e] = 0.f;
            } else {
                unpack<K::BF16, K::VEC>(xs[c], xv);         // requested when the item began
            }
            if (a.phase == 2) {                 // second of two launches: add to the first one's result
#pragma unroll
                for (int e = 0; e < K::VEC; ++e) r[e] = (col0 + e >= own0 && col0 + e < a.out_dim ? o[col0 + e] : 0.f) + dv * acc.v[c][e];
            } else {
#pragma unroll
                for (int e = 0; e < K::VEC; ++e) r[e] = dv * (acc.v[c][e] + ws * xv[e]);
            }
            if (a.phase != 1) {                 // the value is final: optional bias and ReLU
                if (a.bias) {
#pragma unroll
                    for (int e = 0; e < K::VEC; ++e)
                        if (col0 + e < a.out_dim) r[e] += a.bias[col0 + e];
                }
                if (a.relu) {
#pragma unroll
                    for (int e = 0; e < K::VEC; ++e) r[e] = fmaxf(r[e], 0.f);
                }
            }
            // a last vector that reaches into the padding stores what exists, one that was moved back what is its own
            const bool whole = col0 == own0 && col0 + K::VEC <= a.out_dim;
            if (whole) {
                if (a.out_bf16) store_vec_bf16<K::VEC>(ob + col0, r);     // (never combined with phase 2, which reads `out` back)
                else store_vec<K::VEC>(o + col0, r);
            } else {
#pragma unroll
                for (int e = 0; e < K::VEC; ++e)
                    if (col0 + e >= own0 && col0 + e < a.out_dim) {
                        if (a.out_bf16) ob[col0 + e] = to_bf16(r[e]);
                        else o[col0 + e] = r[e];
                    }
            }
        }
    }
}

template <class K>
__device__ __forceinline__ void write_partial(const AggArgs &a, const Acc<K> &acc, int32_t slot, const Lanes<K> &ln)
{
    float *o = a.scratch + static_cast<int64_t>(slot) * a.scratch_ld;
#pragma unroll
    for (int c = 0; c < K::CH; ++c) {
        const int vi = c * K::LPR + ln.lis;
        if (vi >= ln.vend) continue;
        const int col0 = static_cast<int>(ln.col_off[c] / sizeof(typename K::elem)), own0 = vi * K::VEC;
        if (col0 == own0) {                     // (scratch rows hold whole vectors)
            store_vec<K::VEC>(o + col0, acc.v[c]);
        } else {
#pragma unroll
            for (int e = 0; e < K::VEC; ++e)
                if (col0 + e >= own0) o[col0 + e] = acc.v[c][e];
        }
    }
}

// combine the sub-wave accumulators: lanes with equal `lis` hold the same columns
template <class K>
__device__ __forceinline__ float sum_subwaves(float v)
{
    if constexpr (K::LPR <= 8) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x128, 0xf, 0xf, true));    // row_ror:8
    if constexpr (K::LPR <= 4) v += __int_as_float(__builtin_amdgcn_update_dpp(0, __float_as_int(v), 0x124, 0xf, 0xf, true));    // row_ror:4
    if constexpr (K::LPR <= 16) {
        const auto r = __builtin_amdgcn_permlane16_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    if constexpr (K::LPR <= 32) {
        const auto r = __builtin_amdgcn_permlane32_swap(__float_as_uint(v), __float_as_uint(v), false, false);
        v = __uint_as_float(r[0]) + __uint_as_float(r[1]);
    }
    return v;
}

// ---- the kernel -----------------------------------------------------------------------------------
// One work item after the other, M (a.items_per_wave) per wavefront, as a software pipeline: while the
// rows of one run of neighbours are gathered, the ids of the next run -- of the same item or of the
// wavefront's next item -- are already on their way, the descriptor of the item after next has been
// requested, and the owned row's own embedding (needed only when the item is written out) was
// requested when the item began.  Nothing a wavefront needs next is first asked for when it is needed.
//
// Item descriptors travel as one dword per lane (lane f mod 8 holds field f of the 32-byte record)
// through the vector memory path, whose loads return in order behind the gathers already in flight.
__device__ __forceinline__ ItemFields item_fields(const AggArgs &a, int d)
{
    ItemFields f;
    f.row = __builtin_amdgcn_readlane(d, 0); f.beg = __builtin_amdgcn_readlane(d, 1); f.n_l = __builtin_amdgcn_readlane(d, 2);
    f.n = __builtin_amdgcn_readlane(d, 3); f.slot = __builtin_amdgcn_readlane(d, 4); f.rbeg = __builtin_amdgcn_readlane(d, 5);
    if (a.phase == 1) f.n = f.n_l;
    if (a.phase == 2) { f.n -= f.n_l; f.n_l = 0; }
    if (f.row < 0) f.n = 0;
    return f;
}

// Work items are taken M per wavefront.  Workgroup b runs on XCD b mod 8 and takes M consecutive groups (of wpb
// items) of that XCD's queue; groups are interleaved XCD by XCD in `items`.
struct ItemQueue {
    const int32_t *items32;
    int first, stride, M, n_items, lane;
    __device__ __forceinline__ void init(const AggArgs &a, int block, int wave, int wpb, int lane_)
    {
        M = a.items_per_wave;
        items32 = reinterpret_cast<const int32_t *>(a.items);
        const int qb = block / kXcd, xc = block % kXcd;
        first = (qb * M * kXcd + xc) * wpb + wave; stride = kXcd * wpb; n_items = a.n_items; lane = lane_;
    }
    __device__ __forceinline__ int load(int k) const
    {
        const int id = first + k * stride;                                  // wave-uniform
        if (k < M && id < n_items) return items32[static_cast<int64_t>(id) * 8 + (lane & 7)];
        return -1;                                                          // nothing there: reads as a padding item
    }
};

// the owned row's own embedding, requested ahead of its use in write_final
template <class K>
__device__ __forceinline__ void load_self_row(const AggArgs &a, int32_t row, const Lanes<K> &ln, typename K::raw (&xs)[K::CH])
{
    const char *base = static_cast<const char *>(a.x_local) + static_cast<int64_t>(row) * a.ld_x * static_cast<int64_t>(sizeof(typename K::elem));
#pragma unroll
    for (int c = 0; c < K::CH; ++c) xs[c] = load_loose<typename K::raw, sizeof(typename K::elem)>(base + ln.col_off[c]);
}

template <class K>
__device__ __forceinline__ void sum_subwaves(Acc<K> &acc)
{
    if constexpr (K::NPW > 1) {
#pragma unroll
        for (int c = 0; c < K::CH; ++c)
#pragma unroll
            for (int e = 0; e < K::VEC; ++e) acc.v[c][e] = sum_subwaves<K>(acc.v[c][e]);
    }
}

template <class K>
__device__ __forceinline__ void finish_item(const AggArgs &a, bool gcn, Acc<K> &acc, const typename K::raw (&xs)[K::CH], int row, int slot, const Lanes<K> &ln)
{
    sum_subwaves<K>(acc);
    if (ln.sub == 0) {
        if (slot < 0) write_final<K>(a, gcn, acc, xs, row, ln);
        else write_partial<K>(a, acc, slot, ln);
    }
}

// ---- short rows: one per sub-wave, a.short_per_wave groups of NPW rows per wavefront --------------
// A 16-byte record per short row (row, start of its two lists, their lengths) is requested two groups
// ahead, the first ids one group ahead.  A row's two lists are taken as one: the rows of a wavefront have
// about the same number of neighbours (they are sorted by it) while the split between the tables differs
// from row to row, so the wavefront runs that many steps instead of the longest local list plus the
// longest remote one (43,423 bags of 34 lookups, 16 bf16 columns: 44 -> 23 us).
template <class K, bool GCN>
__device__ __forceinline__ void short_rows(const AggArgs &a, int wave, int wpb, int lane, const Lanes<K> &ln, const char *xl, const char *xh, uint64_t ldb)
{
    const int Ms = a.short_per_wave;
    const int sw = (ln.block - a.n_item_blocks) * wpb + wave;
    Acc<K> acc;
    typename K::raw xs[K::CH];
    auto load_sd = [&](int k) -> int4 {
        const int64_t s_id = (static_cast<int64_t>(sw) * Ms + k) * K::NPW + ln.sub;
        int4 sd = make_int4(-1, 0, 0, 0);
        if (k < Ms && s_id < a.n_short) sd = a.short_desc[s_id];
        if (a.phase == 1) sd.w = sd.z;
        if (a.phase == 2) { sd.y += sd.z; sd.w -= sd.z; }
        return sd;
    };
    auto load_ids = [&](const int4 &sd, int b0, uint32_t &id, float &w) {
        id = 0; w = 0.f;
        const int p = b0 + ln.slot;
        if (p < sd.w) {
            id = a.cols[sd.y + p];
            if constexpr (GCN) w = a.wts[sd.y + p];
        }
    };
    int4 sd_cur = load_sd(0), sd_nxt = load_sd(1);
    uint32_t id;
    float w;
    load_ids(sd_cur, 0, id, w);
    for (int k = 0; k < Ms; ++k) {
        if ((static_cast<int64_t>(sw) * Ms + k) * K::NPW >= a.n_short) break;       // wave-uniform: nothing left
        const int4 sd_nn = load_sd(k + 2);
        uint32_t nid;
        float nw;
        load_ids(sd_nxt, 0, nid, nw);
        const bool have = sd_cur.x >= 0;
        const int32_t row = have ? sd_cur.x : 0;
        if (have && !a.no_self && a.phase != 2) load_self_row<K>(a, row, ln, xs);
        acc.clear();
        const int n = sd_cur.w;
        // longest and shortest list among the sub-waves of this wavefront (wave-uniform): the rows are sorted by what both
        // lists hold together, so the first and the last one have them
        int n_max = n, n_min = n;
        if (a.phase == 0) {
            n_max = __builtin_amdgcn_readfirstlane(n);
            n_min = __builtin_amdgcn_readlane(n, kWave - 1);
        } else {
#pragma unroll
            for (int off = K::LPR; off < kWave; off <<= 1) { n_max = max(n_max, __shfl_xor(n_max, off)); n_min = min(n_min, __shfl_xor(n_min, off)); }
            n_max = __builtin_amdgcn_readfirstlane(n_max);
            n_min = __builtin_amdgcn_readfirstlane(n_min);
        }
        for (int b0 = 0; b0 < n_max; b0 += K::LPR) {
            // lists longer than a sub-wave: one block of ids ahead (26-lookup bags, 64 columns: 152 -> 148 us)
            uint32_t bid = 0;
            float bw = 0.f;
            if (b0 + K::LPR < n_max) load_ids(sd_cur, b0 + K::LPR, bid, bw);
            // slots without a neighbour gather the row of one that exists, and drop it
            const bool mine = b0 + ln.slot < n;
            const int any = __builtin_ctzll(__ballot(mine));          // b0 < n_max: some lane has one
            id = mine ? id : static_cast<uint32_t>(__builtin_amdgcn_readlane(static_cast<int>(id), any));
            Slots<K> s;
            set_slots<K>(s, id, w, xl, xh, ldb);
            const int cnt_max = min(K::LPR, n_max - b0);
            if (n_min - b0 >= cnt_max) steps<K, GCN, false>(acc, s, cnt_max, ln);
            else steps<K, GCN, true>(acc, s, cnt_max, ln, n - b0);
            id = bid; w = bw;
        }
        if (have) write_final<K>(a, GCN, acc, xs, row, ln);
        sd_cur = sd_nxt; sd_nxt = sd_nn;
        id = nid; w = nw;
    }
}

template <class K, bool GCN>
__global__ __launch_bounds__(kWave * kMaxWpb) __attribute__((amdgpu_waves_per_eu(K::MIN_WAVES))) void aggregate_kernel(const AggArgs a)
{
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    const int wpb = static_cast<int>(blockDim.x) / kWave;   // wavefronts per workgroup
    Lanes<K> ln;
    ln.init(a, lane);
    const char *xl = static_cast<const char *>(a.x_local);
    const char *xh = static_cast<const char *>(a.x_halo);
    const uint64_t ldb = static_cast<uint64_t>(a.ld_x) * sizeof(typename K::elem);
    if (ln.block >= a.n_item_blocks) {
        short_rows<K, GCN>(a, wave, wpb, lane, ln, xl, xh, ldb);
        return;
    }
    const int ps = a.ps;
    Acc<K> acc;
    typename K::raw xs[K::CH];
    ItemQueue q;
    q.init(a, ln.block, wave, wpb, lane);
    int d_cur = q.load(0), d_nxt = q.load(1);
    bool ids_ready = false;
    uint32_t id = 0;
    float w = 0.f;
    for (int k = 0; k < q.M; ++k) {
        const int d_nn = q.load(k + 2);
        const ItemFields it = item_fields(a, d_cur);
        if (it.row >= 0) {
            const int n = it.n;
            if (!ids_ready && n > 0) load_run<GCN>(a, it, 0, min(ps, n), lane, id, w);
            const ItemFields nx = item_fields(a, d_nxt);
            if (it.slot < 0 && !a.no_self && a.phase != 2) load_self_row<K>(a, it.row, ln, xs);
            acc.clear();
            for (int pos = 0; pos < n; pos += ps) {
                // ids of the next run -- of this item, or the first one of the next
                uint32_t nid = 0;
                float nw = 0.f;
                if (pos + ps < n) load_run<GCN>(a, it, pos + ps, min(ps, n - pos - ps), lane, nid, nw);
                else if (nx.n > 0) load_run<GCN>(a, nx, 0, min(ps, nx.n), lane, nid, nw);
                gather_run<K, GCN>(acc, id, w, min(ps, n - pos), xl, xh, ldb, ln);
                id = nid; w = nw;
            }
            ids_ready = n > 0 && nx.n > 0;
            finish_item<K>(a, GCN, acc, xs, it.row, it.slot, ln);
        } else {
            ids_ready = false;
        }
        d_cur = d_nxt; d_nxt = d_nn;
    }
}

// Launches with too few items to fill the chip: all wavefronts of a workgroup take one item together, a share of its
// neighbours each, and the first one adds up what the others leave in LDS, in a fixed order.  What such a launch costs is
// the chain of loads behind its longest item (466 rows of up to 255 neighbours, 210 fp32 columns: 11.4 -> 4.8 us; 1,592
// rows, 192 columns: 16.7 -> 9.6 us with the fix-up; 2,125 rows, 139 bf16 columns: 12.1 -> 10.4).  The items of an XCD's queue
// stay on it (team_item): with item b on workgroup b half of the gathers of a regrouped row came out of another XCD's class (60 rows
// of 20,000 over 200 k rows of 64 columns 66.9 -> 51.6 us, of 128 columns 129.6 -> 108.7; 120 of 3,000 over 60 k rows of 256 columns
// 56.9 -> 46.2).
template <class K, bool GCN>
__global__ __launch_bounds__(kWave * kMaxTeam) void aggregate_team_kernel(const AggArgs a)
{
    __shared__ float sums[kMaxTeam - 1][K::LPR][K::VEC];
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    const int team = static_cast<int>(blockDim.x) / kWave;
    Lanes<K> ln;
    ln.init(a, lane);
    const char *xl = static_cast<const char *>(a.x_local);
    const char *xh = static_cast<const char *>(a.x_halo);
    const uint64_t ldb = static_cast<uint64_t>(a.ld_x) * sizeof(typename K::elem);
    if (ln.block >= a.n_item_blocks) {
        short_rows<K, GCN>(a, wave, team, lane, ln, xl, xh, ldb);
        return;
    }
    const int item = team_item(ln.block);
    if (item >= a.n_items) return;                           // a queue that ends early, padding: the whole workgroup leaves
    const ItemFields it = item_fields(a, reinterpret_cast<const int32_t *>(a.items)[static_cast<int64_t>(item) * 8 + (lane & 7)]);
    if (it.row < 0) return;
    const int ps = a.ps;
    const int share = (it.n + team * K::NPW - 1) / (team * K::NPW) * K::NPW;
    const int end = min(it.n, (wave + 1) * share);
    Acc<K> acc;
    typename K::raw xs[K::CH];
    if (wave == 0 && it.slot < 0 && !a.no_self && a.phase != 2) load_self_row<K>(a, it.row, ln, xs);
    acc.clear();
    uint32_t id = 0;
    float w = 0.f;
    int pos = wave * share;
    if (pos < end) load_run<GCN>(a, it, pos, min(ps, end - pos), lane, id, w);
    for (; pos < end; pos += ps) {
        uint32_t nid = 0;
        float nw = 0.f;
        if (pos + ps < end) load_run<GCN>(a, it, pos + ps, min(ps, end - pos - ps), lane, nid, nw);
        gather_run<K, GCN>(acc, id, w, min(ps, end - pos), xl, xh, ldb, ln);
        id = nid; w = nw;
    }
    sum_subwaves<K>(acc);
    if (wave > 0 && ln.sub == 0) {
#pragma unroll
        for (int e = 0; e < K::VEC; ++e) sums[wave - 1][ln.slot][e] = acc.v[0][e];
    }
    __syncthreads();
    if (wave > 0 || ln.sub > 0) return;
    for (int t = 0; t < team - 1; ++t)
#pragma unroll
        for (int e = 0; e < K::VEC; ++e) acc.v[0][e] += sums[t][ln.slot][e];
    if (it.slot < 0) write_final<K>(a, GCN, acc, xs, it.row, ln);
    else write_partial<K>(a, acc, it.slot, ln);
}

// ---- LDS staging of halo rows (section 5.2, "pipelined memory operation") -----------------------
// A wavefront owns two LDS stages of kStageSlots load instructions (1 KB each: NPW rows).  The rows of
// a remote partition are requested with global_load_lds -- memory to LDS, holding no registers while in
// flight -- one batch ahead: while batch k is being added from its stage, batch k + 1 is already on its
// way into the other stage, and the local partition of the pair is accumulated through registers in
// between.  Waits count outstanding loads (vmcnt(N)), so only the batch about to be consumed is waited
// for.  Only for 16-byte vectors and one chunk per lane.
typedef const __attribute__((address_space(1))) void *gptr_t;
typedef __attribute__((address_space(3))) void *lptr_t;

template <int N> __device__ __forceinline__ void wait_vmcnt()
{
    if constexpr (N <= 0) asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
    else if constexpr (N == 8) asm volatile("s_waitcnt vmcnt(8)" ::: "memory");
    else asm volatile("s_waitcnt vmcnt(0)" ::: "memory");
}

// requests (up to) kStageSlots load steps of a remote partition, starting at step t0, into `stage`; lane i holds the
// byte offset of the table row of neighbour i (the host takes this path for tables below 4 GB).
// Always issues exactly kStageSlots instructions so that outstanding loads can be counted
template <class K>
__device__ __forceinline__ void stage_halo_batch(uint4 (*stage)[kWave], const char *table, uint32_t row_off, int len, int t0, const Lanes<K> &ln)
{
#pragma unroll
    for (int u = 0; u < kStageSlots; ++u) {
        const int j = (t0 + u) * K::NPW + ln.sub;
        const uint32_t off = static_cast<uint32_t>(__shfl(static_cast<int>(row_off), j < len ? j : 0));   // neighbour 0 exists whenever a batch is staged
        const char *src = table + (off + ln.col_off[0]);
        __builtin_amdgcn_global_load_lds((gptr_t)(const void *)src, (lptr_t)(void *)&stage[u][0], 16, 0, 0);
    }
}

template <class K, bool GCN>
__device__ __forceinline__ void consume_stage(Acc<K> &acc, uint4 (*stage)[kWave], float my_w, int len, int t0, const Lanes<K> &ln, int lane)
{
#pragma unroll
    for (int u = 0; u < kStageSlots; ++u) {
        const int j = (t0 + u) * K::NPW + ln.sub;
        const bool ok = j < len;
        const float wj = GCN ? __shfl(my_w, ok ? j : 0) : 1.f;
        const uint4 q = stage[u][lane];
        typename K::raw r;
        __builtin_memcpy(&r, &q, sizeof r);
        float f[K::VEC];
        unpack<K::BF16, K::VEC>(r, f);
#pragma unroll
        for (int e = 0; e < K::VEC; ++e) acc.v[0][e] = fmaf(wj, ok ? f[e] : 0.f, acc.v[0][e]);
    }
}

// The items of aggregate_kernel with their halo rows through LDS (option lds_halo); local partitions through registers.
// The same pipeline over items, in pairs of a local and a remote partition.
template <class K, bool GCN>
__global__ __launch_bounds__(kWave * kMaxWpb) __attribute__((amdgpu_waves_per_eu(K::MIN_WAVES))) void aggregate_lds_kernel(const AggArgs a)
{
    extern __shared__ uint4 stage_all[];        // two stages of kStageSlots load instructions per wavefront
    const int lane = threadIdx.x & (kWave - 1);
    const int wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) / kWave);
    const int wpb = static_cast<int>(blockDim.x) / kWave;
    Lanes<K> ln;
    ln.init(a, lane);
    const char *xl = static_cast<const char *>(a.x_local);
    const char *xh = static_cast<const char *>(a.x_halo);
    const uint64_t ldb = static_cast<uint64_t>(a.ld_x) * sizeof(typename K::elem);
    if (ln.block >= a.n_item_blocks) {
        short_rows<K, GCN>(a, wave, wpb, lane, ln, xl, xh, ldb);
        return;
    }
    uint4 (*stage)[kStageSlots][kWave] = reinterpret_cast<uint4 (*)[kStageSlots][kWave]>(stage_all + static_cast<size_t>(wave) * 2 * kStageSlots * kWave);
    const int ps = a.ps;
    Acc<K> acc;
    typename K::raw xs[K::CH];
    ItemQueue q;
    q.init(a, ln.block, wave, wpb, lane);
    int d_cur = q.load(0), d_nxt = q.load(1);
    bool ids_ready = false;
    uint32_t id_l = 0, id_r = 0;
    float w_l = 0.f, w_r = 0.f;
    for (int k = 0; k < q.M; ++k) {
        const int d_nn = q.load(k + 2);
        const ItemFields it = item_fields(a, d_cur), nx = item_fields(a, d_nxt);
        d_cur = d_nxt; d_nxt = d_nn;
        if (it.row < 0) { ids_ready = false; continue; }
        const int n_l = it.n_l, n_r = it.n - it.n_l, n_pair = max(n_l, n_r);
        if (!ids_ready) {
            if (n_l > 0) load_run<GCN>(a, it.beg, min(ps, n_l), lane, id_l, w_l);
            if (n_r > 0) load_run<GCN>(a, it.rbeg, min(ps, n_r), lane, id_r, w_r);
        }
        if (it.slot < 0 && !a.no_self && a.phase != 2) load_self_row<K>(a, it.row, ln, xs);
        acc.clear();
        for (int pos = 0; pos < n_pair; pos += ps) {
            // ids of the next pair -- of this item, or the first one of the next
            const bool last = pos + ps >= n_pair;
            const int at = last ? 0 : pos + ps, nl = (last ? (nx.n > 0 ? nx.n_l : 0) : n_l) - at, nr = (last ? (nx.n > 0 ? nx.n - nx.n_l : 0) : n_r) - at;
            uint32_t nid_l = 0, nid_r = 0;
            float nw_l = 0.f, nw_r = 0.f;
            if (nl > 0) load_run<GCN>(a, (last ? nx.beg : it.beg) + at, min(ps, nl), lane, nid_l, nw_l);
            if (nr > 0) load_run<GCN>(a, (last ? nx.rbeg : it.rbeg) + at, min(ps, nr), lane, nid_r, nw_r);
            const int len_l = min(ps, n_l - pos), len_r = min(ps, n_r - pos);
            // remote rows travel into LDS one batch ahead of their accumulation; the local partition
            // of the pair is gathered through registers while the first batch is in flight
            const int steps_r = len_r > 0 ? (len_r + K::NPW - 1) / K::NPW : 0;
            const uint32_t off_r = (id_r & 0x7fffffffu) * static_cast<uint32_t>(ldb);
            if (steps_r > 0) stage_halo_batch<K>(stage[0], xh, off_r, len_r, 0, ln);
            if (len_l > 0) gather_run<K, GCN>(acc, id_l, w_l, len_l, xl, xh, ldb, ln);
            int buf = 0;
            for (int t0 = 0; t0 < steps_r; t0 += kStageSlots, buf ^= 1) {
                if (t0 + kStageSlots < steps_r) {
                    stage_halo_batch<K>(stage[buf ^ 1], xh, off_r, len_r, t0 + kStageSlots, ln);
                    wait_vmcnt<kStageSlots>();          // everything but the batch just requested has landed
                } else {
                    wait_vmcnt<0>();
                }
                consume_stage<K, GCN>(acc, stage[buf], w_r, len_r, t0, ln, lane);
                asm volatile("s_waitcnt lgkmcnt(0)" ::: "memory");   // this stage is free again
            }
            id_l = nid_l; w_l = nw_l; id_r = nid_r; w_r = nw_r;
        }
        ids_ready = n_pair > 0 && nx.n > 0;
        finish_item<K>(a, GCN, acc, xs, it.row, it.slot, ln);
    }
}

template <class K>
hipError_t launch_cfg(const AggArgs &a, bool gcn, dim3 grid, int wpb, hipStream_t stream, bool lds_halo, bool team)
{
    if constexpr (K::CH == 1) {
        if (team) {
            if (gcn) hipLaunchKernelGGL((aggregate_team_kernel<K, true>), grid, dim3(kWave * wpb), 0, stream, a);
            else hipLaunchKernelGGL((aggregate_team_kernel<K, false>), grid, dim3(kWave * wpb), 0, stream, a);
            return hipGetLastError();
        }
    }
    if constexpr (K::CH == 1 && sizeof(typename K::raw) == 16) {
        if (lds_halo) {
            const size_t lds = static_cast<size_t>(wpb) * 2 * kStageSlots * kWave * sizeof(uint4);     // 16 KB per wavefront
            if (gcn) hipLaunchKernelGGL((aggregate_lds_kernel<K, true>), grid, dim3(kWave * wpb), lds, stream, a);
            else hipLaunchKernelGGL((aggregate_lds_kernel<K, false>), grid, dim3(kWave * wpb), lds, stream, a);
            return hipGetLastError();
        }
    }
    if (gcn) hipLaunchKernelGGL((aggregate_kernel<K, true>), grid, dim3(kWave * wpb), 0, stream, a);
    else hipLaunchKernelGGL((aggregate_kernel<K, false>), grid, dim3(kWave * wpb), 0, stream, a);
    return hipGetLastError();
}

// LPR = smallest power of two >= the vectors of a slab (at least 4, at most 64); CH = chunks per lane.
template <bool BF16, int VEC>
hipError_t dispatch_shape(const AggArgs &a, bool gcn, dim3 grid, int wpb, hipStream_t stream, int lpr, int ch, bool lds, bool team)
{
    if (lpr == 4) return launch_cfg<Cfg<BF16, VEC, 4, 1>>(a, gcn, grid, wpb, stream, lds, team);
    if (lpr == 8) return launch_cfg<Cfg<BF16, VEC, 8, 1>>(a, gcn, grid, wpb, stream, lds, team);
    if (lpr == 16) return launch_cfg<Cfg<BF16, VEC, 16, 1>>(a, gcn, grid, wpb, stream, lds, team);
    if (lpr == 32) return launch_cfg<Cfg<BF16, VEC, 32, 1>>(a, gcn, grid, wpb, stream, lds, team);
    if (ch == 1) return launch_cfg<Cfg<BF16, VEC, 64, 1>>(a, gcn, grid, wpb, stream, lds, team);
    if (ch == 2) return launch_cfg<Cfg<BF16, VEC, 64, 2>>(a, gcn, grid, wpb, stream, lds, team);
    return launch_cfg<Cfg<BF16, VEC, 64, 4>>(a, gcn, grid, wpb, stream, lds, team);      // ch <= 4: the host cuts wider rows into slabs
}

// one translation unit per element type (aggregate_f32.hip, aggregate_bf16.hip)
hipError_t launch_aggregate_f32(const AggArgs &a, bool gcn, int vec, dim3 grid, int wpb, hipStream_t stream, int lpr, int ch, bool lds, bool team);
hipError_t launch_aggregate_bf16(const AggArgs &a, bool gcn, int vec, dim3 grid, int wpb, hipStream_t stream, int lpr, int ch, bool lds, bool team);

}  // namespace mgg
