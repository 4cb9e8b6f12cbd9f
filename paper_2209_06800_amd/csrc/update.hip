// Dense Update for gfx950 (section 1: Update is a fully-connected layer; section 7: X W with
// ReLU, and GIN's MLP): out = act(A . W + bias) on the matrix cores.
//
// Shape of the problem: A is tall (10^5..10^6 rows) and both d_in and d_out are small
// (16..602).  launch_update picks per shape:
//   - fp32 weights: the kernels of update_split.hip;
//   - bf16 weights: the whole-line kernels of update_stream.hip where they apply (HBM-bound shapes with whole K
//     slabs), else the kernels of this file -- weights resident in LDS with a grid sized to the chip, or
//     staged slab by slab; update_f32_kernel takes the fp32 shapes update_split.hip refuses (rows shorter than four
//     elements, leading dimensions or weight matrices beyond its 32-bit offsets).
// In this file a workgroup of four wavefronts covers a tile of (32*WM) rows x (NT*32*WN) columns, WM*WN = 4; each
// wavefront owns 32 rows x NT*32 columns (NT <= 4, so that three wavefronts fit a SIMD and the load phase
// of one overlaps the MFMA phase of another):
//   - A goes straight from HBM into registers in the MFMA operand layout, the fragment of the
//     next K slab being requested before the current slab is multiplied (no LDS round trip);
//   - W is staged in LDS and shared by the workgroup;
//   - fp32 weights use v_mfma_f32_32x32x2_f32, bf16 weights v_mfma_f32_32x32x16_bf16,
//     both with fp32 accumulators; bias, ReLU and the output rounding are fused.
// MFMA sums over k in any order, so a lane takes whichever k values are contiguous for it in
// memory as long as the A and W operands agree; that makes the direct loads of A full-width.
// Row softmax runs as a second pass over the output, unless update_split.hip has done it in the product's epilogue.
#include <hip/hip_runtime.h>

#include "update_common.h"

namespace mgg {

namespace {

using namespace upd;

// ---- fp32 weights: v_mfma_f32_32x32x2_f32 ---------------------------------------------------
// K slab of 32: lane (i, h) holds A[m0+i][k0 + 16h .. k0 + 16h + 15]; MFMA number c contracts
// the k pair {k0 + c, k0 + 16 + c}.  W slab in LDS as [32][NC] floats.
// arow always points at a valid row (rows past the end are clamped to the last one and never
// stored), so the only predicate is the wave-uniform "this slab is complete and aligned".
__device__ __forceinline__ void load_a_f32(const UpdArgs &p, const float *arow, int kb, int k_slab_end, float (&af)[16])
{
    if (p.a_vec_ok && k_slab_end <= p.d_in) {
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const float4 v = *reinterpret_cast<const float4 *>(arow + kb + 4 * q);
            af[4 * q] = v.x; af[4 * q + 1] = v.y; af[4 * q + 2] = v.z; af[4 * q + 3] = v.w;
        }
    } else if (p.a_vec_ok) {
        // the last, incomplete slab of aligned rows: whole 16-byte pieces as long as they start inside the
        // row (the leading dimension is a multiple of 4, so such a piece ends inside it too), then the
        // elements past d_in -- padding of the row -- are cleared
#pragma unroll
        for (int q = 0; q < 4; ++q) {
            const int k = kb + 4 * q;
            float4 v = make_float4(0.f, 0.f, 0.f, 0.f);
            if (k < p.d_in) v = *reinterpret_cast<const float4 *>(arow + k);
            af[4 * q] = v.x;
            af[4 * q + 1] = k + 1 < p.d_in ? v.y : 0.f;
            af[4 * q + 2] = k + 2 < p.d_in ? v.z : 0.f;
            af[4 * q + 3] = k + 3 < p.d_in ? v.w : 0.f;
        }
    } else {
#pragma unroll
        for (int e = 0; e < 16; ++e) af[e] = (kb + e < p.d_in) ? arow[kb + e] : 0.f;
    }
}

template <int NT, int WN>
__global__ __launch_bounds__(kThreads) void update_f32_kernel(const UpdArgs p)
{
    constexpr int BK = 32, NC = NT * 32 * WN, WM = kWaves / WN;
    __shared__ __attribute__((aligned(16))) float w_lds[BK * NC];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 31, h = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int64_t m0 = (static_cast<int64_t>(blockIdx.x) * WM + wm) * 32;
    const int nb = blockIdx.y * NC;                 // first column of the workgroup
    const int n0 = nb + wn * NT * 32;               // first column of this wavefront
    const float *W = static_cast<const float *>(p.w);
    const int64_t row = m0 + i < p.n_rows ? m0 + i : p.n_rows - 1;
    const float *arow = static_cast<const float *>(p.a) + row * p.ld_a;

    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

    float af[16], an[16];
    load_a_f32(p, arow, 16 * h, BK, af);
#pragma unroll 1
    for (int k0 = 0; k0 < p.d_in; k0 += BK) {
        if (k0 + BK < p.d_in) load_a_f32(p, arow, k0 + BK + 16 * h, k0 + 2 * BK, an);   // next slab's fragment
        __syncthreads();
        fill_w_f32<NC>(w_lds, W, k0, BK, nb, p);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 16; ++c) {
            const float *wrow = w_lds + (16 * h + c) * NC + wn * NT * 32 + i;
#pragma unroll
            for (int t = 0; t < NT; ++t)
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x2f32(wrow[t * 32], af[c], acc[t], 0, 0, 0);
        }
#pragma unroll
        for (int c = 0; c < 16; ++c) af[c] = an[c];
    }
    store_tiles<NT>(p, acc, m0, n0, lane);
}

// ---- bf16 weights: v_mfma_f32_32x32x16_bf16 -------------------------------------------------
// K slab of 64: lane (i, h) holds A[m0+i][k0 + 32h .. k0 + 32h + 31] as four 8-element
// operands; MFMA number c contracts k0 + 32h + 8c .. + 7 (both halves h at once).
// W slab in LDS transposed, [NC][64 + 8] bf16, so a lane's 8 k-values are contiguous.
union Frag8 { uint32_t u[4]; bf16x8 v; };

template <bool A_BF16>
__device__ __forceinline__ void load_a_bf16(const UpdArgs &p, const void *arow_v, int kb, int k_slab_end, Frag8 (&af)[4])
{
    const bool full = p.a_vec_ok && k_slab_end <= p.d_in;      // wave-uniform
    if constexpr (A_BF16) {
        const uint16_t *arow = static_cast<const uint16_t *>(arow_v);
        if (full) {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                const uint4 v = *reinterpret_cast<const uint4 *>(arow + kb + 8 * c);
                af[c].u[0] = v.x; af[c].u[1] = v.y; af[c].u[2] = v.z; af[c].u[3] = v.w;
            }
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c)
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = kb + 8 * c + 2 * e;
                    const uint32_t lo = k < p.d_in ? arow[k] : 0u;
                    const uint32_t hi = k + 1 < p.d_in ? arow[k + 1] : 0u;
                    af[c].u[e] = lo | (hi << 16);
                }
        }
    } else {
        const float *arow = static_cast<const float *>(arow_v);
#pragma unroll
        for (int c = 0; c < 4; ++c) {
            const int k = kb + 8 * c;
            float f[8];
            if (full) {
                const float4 v0 = *reinterpret_cast<const float4 *>(arow + k);
                const float4 v1 = *reinterpret_cast<const float4 *>(arow + k + 4);
                f[0] = v0.x; f[1] = v0.y; f[2] = v0.z; f[3] = v0.w; f[4] = v1.x; f[5] = v1.y; f[6] = v1.z; f[7] = v1.w;
            } else {
#pragma unroll
                for (int e = 0; e < 8; ++e) f[e] = k + e < p.d_in ? arow[k + e] : 0.f;
            }
#pragma unroll
            for (int e = 0; e < 4; ++e) af[c].u[e] = pack_bf16(f[2 * e], f[2 * e + 1]);
        }
    }
}

template <int NT, int WN, bool A_BF16>
__global__ __launch_bounds__(kThreads) void update_bf16_kernel(const UpdArgs p)
{
    constexpr int BK = 64, NC = NT * 32 * WN, LDW = BK + 8, WM = kWaves / WN;
    __shared__ __attribute__((aligned(16))) uint16_t w_lds[NC * LDW];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 31, h = lane >> 5;
    const int wm = wave / WN, wn = wave % WN;
    const int64_t m0 = (static_cast<int64_t>(blockIdx.x) * WM + wm) * 32;
    const int nb = blockIdx.y * NC;
    const int n0 = nb + wn * NT * 32;
    const uint16_t *W = static_cast<const uint16_t *>(p.w);
    const int64_t row = m0 + i < p.n_rows ? m0 + i : p.n_rows - 1;
    const void *arow = A_BF16 ? static_cast<const void *>(static_cast<const uint16_t *>(p.a) + row * p.ld_a)
                              : static_cast<const void *>(static_cast<const float *>(p.a) + row * p.ld_a);

    f32x16 acc[NT];
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;

    Frag8 af[4], an[4];
    load_a_bf16<A_BF16>(p, arow, 32 * h, BK, af);
#pragma unroll 1
    for (int k0 = 0; k0 < p.d_in; k0 += BK) {
        if (k0 + BK < p.d_in) load_a_bf16<A_BF16>(p, arow, k0 + BK + 32 * h, k0 + 2 * BK, an);
        __syncthreads();
        fill_w_bf16_t<NC>(w_lds, LDW, W, k0, BK, nb, p);
        __syncthreads();
#pragma unroll
        for (int c = 0; c < 4; ++c) {
#pragma unroll
            for (int t = 0; t < NT; ++t) {
                union { uint4 q; bf16x8 v; } bw;
                bw.q = *reinterpret_cast<const uint4 *>(&w_lds[(wn * NT * 32 + t * 32 + i) * LDW + 32 * h + 8 * c]);
                acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw.v, af[c].v, acc[t], 0, 0, 0);
            }
        }
#pragma unroll
        for (int c = 0; c < 4; ++c) af[c] = an[c];
    }
    store_tiles<NT>(p, acc, m0, n0, lane);
}


// ---- W resident in LDS (small d_in * d_out) ---------------------------------------------------
// When the whole weight matrix fits 64 KB of LDS it is staged once per workgroup, and every
// wavefront then walks over many 32-row tiles of A on its own: no barrier in the main loop.
// These shapes are bound by HBM, and what a wavefront can keep in flight is what its registers
// hold, so the raw K slabs of A are requested D slabs ahead -- across tile boundaries -- and a
// slab is turned into MFMA operands only when its turn comes.  Loads that are waited for are
// always older than the stores of the tile finished last, so (memory operations of a wavefront
// retire in order) no wait ever includes a store.  The grid is sized to the chip, not to the matrix.
extern __shared__ __attribute__((aligned(16))) unsigned char w_res[];

// Register budget: without a bound the compiler spends over 250 registers on the widest variant
// and one wavefront per SIMD is left; three (four for the narrow variants) run 1.2-1.3x faster.
#define MGG_UPD_WAVES(NT) ((NT) == 4 ? 3 : 4)
// bf16 path: raw slab = the lane's 32 consecutive k values, fp32 (8 x 16 bytes) or bf16 (4 x 16 bytes)
template <bool A_BF16> struct RawB16 { uint4 v[A_BF16 ? 4 : 8]; };

template <bool A_BF16>
__device__ __forceinline__ void load_raw_b16(const UpdArgs &p, const void *arow_v, int kb, int k_slab_end, RawB16<A_BF16> &r)
{
    const bool full = p.a_vec_ok && k_slab_end <= p.d_in;      // wave-uniform
    if constexpr (A_BF16) {
        const uint16_t *arow = static_cast<const uint16_t *>(arow_v);
        if (full) {
#pragma unroll
            for (int c = 0; c < 4; ++c) r.v[c] = *reinterpret_cast<const uint4 *>(arow + kb + 8 * c);
        } else {
#pragma unroll
            for (int c = 0; c < 4; ++c) {
                uint32_t u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) {
                    const int k = kb + 8 * c + 2 * e;
                    const uint32_t lo = k < p.d_in ? arow[k] : 0u;
                    const uint32_t hi = k + 1 < p.d_in ? arow[k + 1] : 0u;
                    u[e] = lo | (hi << 16);
                }
                r.v[c] = make_uint4(u[0], u[1], u[2], u[3]);
            }
        }
    } else {
        const float *arow = static_cast<const float *>(arow_v);
        if (full) {
#pragma unroll
            for (int c = 0; c < 8; ++c) r.v[c] = *reinterpret_cast<const uint4 *>(arow + kb + 4 * c);
        } else {
#pragma unroll
            for (int c = 0; c < 8; ++c) {
                uint32_t u[4];
#pragma unroll
                for (int e = 0; e < 4; ++e) u[e] = kb + 4 * c + e < p.d_in ? __float_as_uint(arow[kb + 4 * c + e]) : 0u;
                r.v[c] = make_uint4(u[0], u[1], u[2], u[3]);
            }
        }
    }
}

template <bool A_BF16>
__device__ __forceinline__ void raw_to_frags(const RawB16<A_BF16> &r, Frag8 (&af)[4])
{
#pragma unroll
    for (int c = 0; c < 4; ++c) {
        if constexpr (A_BF16) {
            af[c].u[0] = r.v[c].x; af[c].u[1] = r.v[c].y; af[c].u[2] = r.v[c].z; af[c].u[3] = r.v[c].w;
        } else {
            const uint4 lo = r.v[2 * c], hi = r.v[2 * c + 1];
            af[c].u[0] = pack_bf16(__uint_as_float(lo.x), __uint_as_float(lo.y));
            af[c].u[1] = pack_bf16(__uint_as_float(lo.z), __uint_as_float(lo.w));
            af[c].u[2] = pack_bf16(__uint_as_float(hi.x), __uint_as_float(hi.y));
            af[c].u[3] = pack_bf16(__uint_as_float(hi.z), __uint_as_float(hi.w));
        }
    }
}

template <int NT, bool A_BF16, int D>
__global__ __launch_bounds__(kThreads) __attribute__((amdgpu_waves_per_eu(MGG_UPD_WAVES(NT), MGG_UPD_WAVES(NT))))
void update_bf16_resident_kernel(const UpdArgs p)
{
    constexpr int BK = 64, NC = NT * 32;
    uint16_t *w_lds = reinterpret_cast<uint16_t *>(w_res);
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int i = lane & 31, h = lane >> 5;
    const int n_slabs = (p.d_in + BK - 1) / BK;
    const int ldw = n_slabs * BK + 8;                       // padded row of the transposed copy
    const uint16_t *W = static_cast<const uint16_t *>(p.w);
    fill_w_bf16_t<NC>(w_lds, ldw, W, 0, n_slabs * BK, 0, p);
    __syncthreads();

    const int64_t n_tiles = (p.n_rows + 31) / 32, stride = static_cast<int64_t>(gridDim.x) * kWaves;
    int64_t tile = static_cast<int64_t>(blockIdx.x) * kWaves + wave;
    if (tile >= n_tiles) return;
    auto row_ptr_of = [&](int64_t t) -> const void * {
        const int64_t r = t * 32 + i < p.n_rows ? t * 32 + i : p.n_rows - 1;
        if constexpr (A_BF16) return static_cast<const uint16_t *>(p.a) + r * p.ld_a;
        else return static_cast<const float *>(p.a) + r * p.ld_a;
    };
    int64_t itile = tile;
    int is = 0;
    const void *irow = row_ptr_of(itile);
    RawB16<A_BF16> q[D];
    auto issue = [&](RawB16<A_BF16> &dst) {
        if (itile < n_tiles) {
            load_raw_b16<A_BF16>(p, irow, is * BK + 32 * h, (is + 1) * BK, dst);
            if (++is == n_slabs) { is = 0; itile += stride; if (itile < n_tiles) irow = row_ptr_of(itile); }
        }
    };
#pragma unroll
    for (int d = 0; d < D; ++d) issue(q[d]);

    while (tile < n_tiles) {
        f32x16 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = 0.f;
#pragma unroll 1
        for (int s = 0; s < n_slabs; ++s) {
            Frag8 af[4];
            raw_to_frags<A_BF16>(q[0], af);
#pragma unroll
            for (int d = 0; d + 1 < D; ++d) q[d] = q[d + 1];
            issue(q[D - 1]);
#pragma unroll
            for (int c = 0; c < 4; ++c) {
#pragma unroll
                for (int t = 0; t < NT; ++t) {
                    union { uint4 q4; bf16x8 v; } bw;
                    bw.q4 = *reinterpret_cast<const uint4 *>(&w_lds[(t * 32 + i) * ldw + s * BK + 32 * h + 8 * c]);
                    acc[t] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(bw.v, af[c].v, acc[t], 0, 0, 0);
                }
            }
        }
        store_tiles<NT>(p, acc, tile * 32, 0, lane);
        tile += stride;
    }
}

// slabs requested ahead (the raw fp32 slab of the bf16 path is twice the size of the others)
#ifndef MGG_UPD_DEPTH_B16
#define MGG_UPD_DEPTH_B16 1
#endif

// ---- row softmax (section 7: the last step of the 2-layer GCN) ---------------------------------
// One wavefront per row, in place: the row is held in registers (lanes stride over the columns),
// maximum and sum are combined with cross-lane shuffles.  Bound by HBM: one read and one write.
template <bool BF16, int CPL>      // CPL: columns per lane
__global__ __launch_bounds__(kThreads) void row_softmax_kernel(void *x, int64_t n_rows, int32_t d, int64_t ld)
{
    const int lane = threadIdx.x & 63;
    const int64_t row = static_cast<int64_t>(blockIdx.x) * kWaves + (threadIdx.x >> 6);
    if (row >= n_rows) return;
    float v[CPL];
    float m = -INFINITY;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int col = c * kWave + lane;
        v[c] = -INFINITY;
        if (col < d) {
            if constexpr (BF16) v[c] = __uint_as_float(static_cast<uint32_t>(static_cast<const uint16_t *>(x)[row * ld + col]) << 16);
            else v[c] = static_cast<const float *>(x)[row * ld + col];
        }
        m = fmaxf(m, v[c]);
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) m = fmaxf(m, __shfl_xor(m, off));
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        v[c] = c * kWave + lane < d ? expf(v[c] - m) : 0.f;
        sum += v[c];
    }
#pragma unroll
    for (int off = 32; off >= 1; off >>= 1) sum += __shfl_xor(sum, off);
    const float inv = 1.f / sum;
#pragma unroll
    for (int c = 0; c < CPL; ++c) {
        const int col = c * kWave + lane;
        if (col < d) {
            if constexpr (BF16) static_cast<uint16_t *>(x)[row * ld + col] = to_bf16(v[c] * inv);
            else static_cast<float *>(x)[row * ld + col] = v[c] * inv;
        }
    }
}

inline bool aligned16(const void *q) { return (reinterpret_cast<uintptr_t>(q) & 15u) == 0; }

template <int NT>
hipError_t launch_resident(const UpdArgs &p, bool a_bf16, int blocks, size_t lds_bytes, hipStream_t s)
{
    if (a_bf16) hipLaunchKernelGGL((update_bf16_resident_kernel<NT, true, 2 * MGG_UPD_DEPTH_B16>), dim3(blocks), dim3(kThreads), lds_bytes, s, p);
    else hipLaunchKernelGGL((update_bf16_resident_kernel<NT, false, MGG_UPD_DEPTH_B16>), dim3(blocks), dim3(kThreads), lds_bytes, s, p);
    return hipGetLastError();
}

template <int NT, int WN>
hipError_t launch_shape(const UpdArgs &p, bool w_bf16, bool a_bf16, dim3 grid, hipStream_t s)
{
    if (!w_bf16) hipLaunchKernelGGL((update_f32_kernel<NT, WN>), grid, dim3(kThreads), 0, s, p);
    else if (a_bf16) hipLaunchKernelGGL((update_bf16_kernel<NT, WN, true>), grid, dim3(kThreads), 0, s, p);
    else hipLaunchKernelGGL((update_bf16_kernel<NT, WN, false>), grid, dim3(kThreads), 0, s, p);
    return hipGetLastError();
}

}  // namespace

mgg_status_t launch_row_softmax(int64_t n_rows, int32_t d, mgg_dtype_t dtype, void *x, int64_t ld, hipStream_t stream)
{
    if (n_rows == 0) return MGG_OK;
    if (d > 8 * kWave) return fail(MGG_ERR_UNSUPPORTED, "softmax over %d columns (at most %d)", d, 8 * kWave);
    const int64_t blocks = (n_rows + kWaves - 1) / kWaves;
    if (blocks > INT32_MAX) return fail(MGG_ERR_UNSUPPORTED, "too many rows for one launch");
    const dim3 grid(static_cast<unsigned>(blocks)), block(kThreads);
    const bool bf = dtype == MGG_BF16;
    const int cpl = (d + kWave - 1) / kWave;
#define MGG_SOFTMAX(C) do { if (bf) hipLaunchKernelGGL((row_softmax_kernel<true, C>), grid, block, 0, stream, x, n_rows, d, ld); \
                            else hipLaunchKernelGGL((row_softmax_kernel<false, C>), grid, block, 0, stream, x, n_rows, d, ld); } while (0)
    if (cpl <= 1) MGG_SOFTMAX(1);
    else if (cpl <= 2) MGG_SOFTMAX(2);
    else if (cpl <= 4) MGG_SOFTMAX(4);
    else MGG_SOFTMAX(8);
#undef MGG_SOFTMAX
    hipError_t e = hipGetLastError();
    if (e != hipSuccess) return hip_fail(e, "softmax kernel launch");
    return MGG_OK;
}

static mgg_status_t launch_update_gemm(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, int32_t d_in,
                                       mgg_dtype_t w_dtype, const void *w, const float *bias, int32_t d_out, mgg_act_t act,
                                       mgg_dtype_t out_dtype, void *out, int64_t ld_out, hipStream_t stream, bool *softmax);

mgg_status_t launch_update(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, int32_t d_in,
                           mgg_dtype_t w_dtype, const void *w, const float *bias, int32_t d_out, mgg_act_t act,
                           mgg_dtype_t out_dtype, void *out, int64_t ld_out, hipStream_t stream)
{
    // softmax couples the columns of a row: the product is written first and the rows are normalised in place, unless the
    // product's kernel holds whole rows and has done it
    bool softmax = act == MGG_ACT_SOFTMAX;
    if (softmax && d_out > 8 * kWave) return fail(MGG_ERR_UNSUPPORTED, "softmax over %d columns (at most %d)", d_out, 8 * kWave);
    mgg_status_t s = launch_update_gemm(n_rows, a_dtype, a, ld_a, d_in, w_dtype, w, bias, d_out, softmax ? MGG_ACT_NONE : act,
                                        out_dtype, out, ld_out, stream, &softmax);
    if (s != MGG_OK || !softmax) return s;
    return launch_row_softmax(n_rows, d_out, out_dtype, out, ld_out, stream);
}

mgg_status_t launch_update_mlp(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, const int32_t dims[3],
                               mgg_dtype_t w_dtype, const void *w1, const float *b1, mgg_act_t act1, const void *w2, const float *b2,
                               mgg_act_t act2, void *hidden, int64_t ld_hidden, mgg_dtype_t out_dtype, void *out, int64_t ld_out,
                               hipStream_t stream)
{
    if (n_rows == 0) return MGG_OK;
    if (w_dtype == MGG_BF16 && option_update_stream() != 0) {
        int dev = 0, cus = 256;
        if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
        hipError_t e = hipSuccess;
        if (launch_mlp_stream(n_rows, a_dtype, a, ld_a, dims[0], w1, b1, act1, dims[1], w2, b2, act2, dims[2], out_dtype, out, ld_out, cus,
                              stream, &e)) {
            if (e != hipSuccess) return hip_fail(e, "MLP kernel launch");
            return MGG_OK;
        }
    }
    if (!hidden) return fail(MGG_ERR_INVALID_ARG, "hidden buffer is NULL and the shape is not covered by the one-kernel MLP");
    const mgg_dtype_t hid_dtype = w_dtype == MGG_BF16 ? MGG_BF16 : MGG_F32;
    mgg_status_t s = launch_update(n_rows, a_dtype, a, ld_a, dims[0], w_dtype, w1, b1, dims[1], act1, hid_dtype, hidden, ld_hidden, stream);
    if (s != MGG_OK) return s;
    return launch_update(n_rows, hid_dtype, hidden, ld_hidden, dims[1], w_dtype, w2, b2, dims[2], act2, out_dtype, out, ld_out, stream);
}

static mgg_status_t launch_update_gemm(int64_t n_rows, mgg_dtype_t a_dtype, const void *a, int64_t ld_a, int32_t d_in,
                                       mgg_dtype_t w_dtype, const void *w, const float *bias, int32_t d_out, mgg_act_t act,
                                       mgg_dtype_t out_dtype, void *out, int64_t ld_out, hipStream_t stream, bool *softmax)
{
    if (n_rows == 0) return MGG_OK;
    const bool w_bf16 = w_dtype == MGG_BF16, a_bf16 = a_dtype == MGG_BF16;
    UpdArgs p{};
    p.a = a; p.w = w; p.bias = bias; p.out = out;
    p.n_rows = n_rows; p.ld_a = ld_a; p.ld_out = ld_out;
    p.d_in = d_in; p.d_out = d_out;
    p.relu = act == MGG_ACT_RELU;
    p.out_bf16 = out_dtype == MGG_BF16;
    p.a_vec_ok = aligned16(a) && (ld_a % (a_bf16 ? 8 : 4) == 0);
    p.out_vec_ok = (ld_out % 4 == 0) && (reinterpret_cast<uintptr_t>(out) % (out_dtype == MGG_BF16 ? 8 : 16) == 0);
    p.w_vec_ok = aligned16(w) && (d_out % (w_bf16 ? 8 : 4) == 0);

    // tiles of 32 columns per wavefront (1, 2 or 4) and wavefronts side by side (1 or 2);
    // outputs wider than 256 columns tile over grid.y
    int nt = 1, wn = 1;
    if (d_out > 128) { nt = 4; wn = 2; }
    else if (d_out > 64) nt = 4;
    else if (d_out > 32) nt = 2;
    int dev = 0, cus = 256;
    if (hipGetDevice(&dev) == hipSuccess) (void)hipDeviceGetAttribute(&cus, hipDeviceAttributeMultiprocessorCount, dev);
    if (!w_bf16) {
        hipError_t e = hipSuccess;
        if (launch_update_split(p, cus, stream, softmax, &e)) {
            if (e != hipSuccess) return hip_fail(e, "update kernel launch");
            return MGG_OK;
        }
    }
    // HBM-bound shapes with whole K slabs: the whole-line variant
    if (option_update_stream() != 0) {
        hipError_t e = hipSuccess;
        if (launch_update_stream(p, w_bf16, a_bf16, cus, stream, &e)) {
            if (e != hipSuccess) return hip_fail(e, "update kernel launch");
            return MGG_OK;
        }
    }
    // small weight matrices stay resident in LDS and the grid is sized to the chip
    if (w_bf16 && wn == 1) {
        const size_t k_pad = (static_cast<size_t>(d_in) + 63) / 64 * 64;
        const size_t lds_bytes = static_cast<size_t>(nt) * 32 * (k_pad + 8) * 2;
        if (lds_bytes <= 64 * 1024) {
            int per_cu = static_cast<int>((160 * 1024) / (lds_bytes + 512));
            per_cu = per_cu < 1 ? 1 : (per_cu > (nt == 4 ? 3 : 4) ? (nt == 4 ? 3 : 4) : per_cu);
            const int64_t n_tiles = (n_rows + 31) / 32;
            const int64_t want = (n_tiles + kWaves - 1) / kWaves;
            const int blocks = static_cast<int>(want < static_cast<int64_t>(cus) * per_cu ? want : static_cast<int64_t>(cus) * per_cu);
            hipError_t e;
            if (nt == 1) e = launch_resident<1>(p, a_bf16, blocks, lds_bytes, stream);
            else if (nt == 2) e = launch_resident<2>(p, a_bf16, blocks, lds_bytes, stream);
            else e = launch_resident<4>(p, a_bf16, blocks, lds_bytes, stream);
            if (e != hipSuccess) return hip_fail(e, "update kernel launch");
            return MGG_OK;
        }
    }
    const int nc = nt * 32 * wn, rows_per_block = 32 * (kWaves / wn);
    const int64_t gx = (n_rows + rows_per_block - 1) / rows_per_block;
    if (gx > INT32_MAX) return fail(MGG_ERR_UNSUPPORTED, "too many rows for one launch");
    dim3 grid(static_cast<unsigned>(gx), static_cast<unsigned>((d_out + nc - 1) / nc));
    hipError_t e;
    if (wn == 2) e = launch_shape<4, 2>(p, w_bf16, a_bf16, grid, stream);
    else if (nt == 1) e = launch_shape<1, 1>(p, w_bf16, a_bf16, grid, stream);
    else if (nt == 2) e = launch_shape<2, 1>(p, w_bf16, a_bf16, grid, stream);
    else e = launch_shape<4, 1>(p, w_bf16, a_bf16, grid, stream);
    if (e != hipSuccess) return hip_fail(e, "update kernel launch");
    return MGG_OK;
}

}  // namespace mgg
