// Dense Update with fp32 weights for gfx950 (section 1: Update is a fully-connected layer; section 7:
// X W with ReLU): out = act(A . W + bias), fp32 in and out, on the bf16 matrix instruction.
//
// v_mfma_f32_32x32x2_f32 runs at 1/16 of the bf16 rate (about 157 TFLOP/s), which bounded every fp32 shape
// wider than about 64 x 64.  An fp32 number is the exact sum of three bf16 numbers (24 = 8 + 8 + 8 bits of
// significand; each part is rounded to nearest, so the next one is at most 2^-8 of it and of either sign), and
// a product of two bf16 numbers is exact in fp32.  Of a w = (a1 + a2 + a3)(w1 + w2 + w3) all terms but a3 w3 are
// summed, which is at most 2^-32 |a w|.  (The six largest alone would leave out up to 2^-24 |a w| more, which shows
// where a row has a single non-zero: 1.0e-7 of the result instead of 6.0e-8.)
//
// Two accumulators: a1 w1 goes into one, the seven small terms into the other, which is 2^-8 of the first, and they are
// added at the end.  So 16 products round the large sum once; the fp32 instruction rounds it for every two products,
// and one chain of all terms would round it eight times per 16 columns of A however many of them are zero.  2-norm
// error against float64 at 602 columns: 4.4e-7 with the fp32 instruction, 1.4e-7 so; with one non-zero in 16
// 1.1e-7 with the fp32 instruction, 2.3e-7 with a chain of six terms, 0.5e-7 so.
//
// Range.  Both operands are multiplied by 2^24 on their way into the parts and the sums by 2^-48 at the end, all exact:
// the smallest fp32 number, 2^-149, has its last bit at 2^-125 then, so that no part of any element is denormal,
// however small the element is beside others of its row, and what is lost at the low end of the sums is below 2^-149
// after scaling back.  At the high end an element of 2^104, or sums of 2^80, overflow: the elements of the result
// that are not finite (infinities and NaN among the operands make such, too) are computed with the fp32 instruction
// from global memory and put in their place.  Their neighbours keep their bits: a row of the result depends on
// that row of A and on W alone.  Not met by data of ordinary scale, and slow: one column of W infinite, 232,965 x 602 ->
// 256 takes 1.06 ms instead of 0.49.
//
// What bounds it: HBM for narrow outputs, the matrix pipe and the operand traffic through LDS for wide ones.
// Against kernels on the fp32 instruction (us there -> here, one MI355X; fp32 rows end to end unless a leading
// dimension is given), and the 2-norm error against float64:
//   232,965 x 602 (ld 608) -> 256    676 -> 494     4.4e-7 -> 1.4e-7
//   400,000 x 250 -> 250             970 -> 405     2.8e-7 -> 0.9e-7
//   306,128 x 100 -> 256             232 -> 157     1.8e-7 -> 0.6e-7
//   1,771,062 x 256 -> 47            684 -> 504     2.9e-7 -> 0.9e-7
//   262,144 x 64 -> 64                38 ->  30     1.5e-7 -> 0.6e-7
//   2,000 x 602 -> 256               116 ->  17     4.4e-7 -> 1.4e-7
//   400,000 x 32 -> 16                20 ->  16     1.0e-7 -> 0.4e-7
// (Six terms would take 427 us on the first and 350 on the second.)
//
// Layout.  Eight wavefronts; a wavefront owns 32 rows x NT*32 columns, at most 128: the two accumulators take 128
// registers then.  A slab of 32 k values is read with 8
// lanes per row (one whole 128-byte line per row and instruction, at any alignment: 16-byte loads need only
// element alignment, and a vector that would pass the end of a ragged row is moved back to end with it), staged raw in a
// per-wavefront LDS buffer, read back in operand layout and split there: an element of A is split once per block of columns.
// W is split while it is staged: three planes of 16-byte pieces [k / 8][column], so that operand reads and
// staging writes are conflict-free and W needs no alignment.
//   - resident: all of W in LDS, split once per workgroup; wavefronts walk over their tiles without a barrier;
//   - slab: two slabs of W in LDS; the next one is loaded into registers, split between the MFMAs of the
//     current one and written to the other buffer; one barrier per slab;
//   - narrow: up to 32 columns, resident, on the 16 x 16 instruction.
#include <algorithm>
#include <utility>

#include "update_common.h"

namespace mgg {

namespace {

using namespace upd;

constexpr int kSWaves = 8, kSThreads = kWave * kSWaves;
constexpr int kLda = 36;                                    // row of the per-wavefront buffer, in floats
constexpr int kWaveBytes = 32 * kLda * 4;
constexpr int kLdsMax = 160 * 1024 - 1024;                  // (beside it: the bias)
constexpr float kScale = 0x1p24f, kUnscale = 0x1p-48f;       // of an operand; of a sum of products
constexpr int w_slab_bytes(int nc) { return 3 * 4 * nc * 16; }

union Frag { uint32_t u[4]; uint4 q; bf16x8 v; };

extern __shared__ __attribute__((aligned(16))) unsigned char lds_split[];

__device__ __forceinline__ void wave_sync_lds()
{
    // LDS traffic of one wavefront is executed in order; this only keeps the compiler from reordering it
    __builtin_amdgcn_fence(__ATOMIC_RELEASE, "wavefront");
    __builtin_amdgcn_wave_barrier();
    __builtin_amdgcn_fence(__ATOMIC_ACQUIRE, "wavefront");
}

// eight fp32 values -> three bf16 operands whose sum they are, times kScale
__device__ __forceinline__ void split8(const float (&f)[8], Frag (&o)[3])
{
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        float lo = f[2 * e] * kScale, hi = f[2 * e + 1] * kScale;
#pragma unroll
        for (int s = 0; s < 3; ++s) {
            const uint32_t pk = pack_bf16(lo, hi);
            o[s].u[e] = pk;
            if (s < 2) { lo -= __uint_as_float(pk << 16); hi -= __uint_as_float(pk & 0xffff0000u); }
        }
    }
}

typedef float f32x4 __attribute__((ext_vector_type(4)));
typedef f32x4 f32x4_loose __attribute__((aligned(4)));       // in memory, at any element
struct RawA { f32x4 v[4]; };

// f(integral_constant 0), f(1), ... f(N - 1): steps whose number decides at compile time what they hold
template <class F, int... X>
__device__ __forceinline__ void static_for(F &&f, std::integer_sequence<int, X...>) { (f(std::integral_constant<int, X>{}), ...); }

// 32 rows x 32 k values: instruction j takes rows 8 j + lane / 8.  Rows past the end are clamped to the last
// one (never stored).  A vector that would reach past the row ends with it instead: slab position 4 c + e then holds
// k = min(k0 + 4 c, d_in - 4) + e, and W is laid out to match (w_row).  m0 is wave-uniform: an address is a
// scalar base and a 32-bit offset per lane (the host checks the leading dimensions for it).
__device__ __forceinline__ void load_a(const UpdArgs &p, int64_t m0, int k0, int lane, RawA &r)
{
    const int64_t last = (p.n_rows - 1) / 32 * 32;
    m0 = m0 < last ? m0 : last;
    const int rows = static_cast<int>(p.n_rows - m0 < 32 ? p.n_rows - m0 : 32);
    const char *base = reinterpret_cast<const char *>(static_cast<const float *>(p.a) + m0 * p.ld_a);
    const uint32_t col = static_cast<uint32_t>(min(k0 + (lane & 7) * 4, p.d_in - 4));
#pragma unroll
    for (int j = 0; j < 4; ++j) {
        const uint32_t off = (static_cast<uint32_t>(min(j * 8 + (lane >> 3), rows - 1)) * static_cast<uint32_t>(p.ld_a) + col) * 4u;
        r.v[j] = *reinterpret_cast<const f32x4_loose *>(base + off);
    }
}

__device__ __forceinline__ void stage_a(const RawA &r, int lane, float *abuf)
{
#pragma unroll
    for (int j = 0; j < 4; ++j) *reinterpret_cast<f32x4 *>(abuf + (j * 8 + (lane >> 3)) * kLda + (lane & 7) * 4) = r.v[j];
}

// The row of W that meets slab position pos (counted from the first slab; pos & 3 = e in load_a).  Where load_a moved
// a vector back its first elements were met before: `again`, and their weight is zero.  (Zero times an infinity of A: the
// sum is not finite then, and computed again.)
__device__ __forceinline__ int w_row(int pos, int d_in, bool &again)
{
    const int first = pos & ~3, k = min(first, d_in - 4) + (pos & 3);
    again = k < first;
    return k;
}

// One unit of W: 8 consecutive slab positions of one column.  Unit id0 + lane (id0 wave-uniform, a multiple of 64) is
// (position / 8, column) = (id / NC, id % NC).  Columns past the edge read the last one and are never stored.
template <int NC>
__device__ __forceinline__ int unit_pos(int id0, int lane) { return NC >= kWave ? id0 / NC * 8 : (id0 + lane) / NC * 8; }      // (scalar if NC >= 64)

template <int NC>
__device__ __forceinline__ void load_w_unit(const UpdArgs &p, int k0, int id0, int n0, int lane, float (&f)[8])
{
    const int n = min(n0 + (NC >= kWave ? id0 % NC + lane : lane % NC), p.d_out - 1);
    const int pos = k0 + unit_pos<NC>(id0, lane);
    const char *base = static_cast<const char *>(p.w);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bool again;
        const uint32_t k = static_cast<uint32_t>(w_row(pos + e, p.d_in, again)), row = k * static_cast<uint32_t>(p.d_out) * 4u;   // (host: W below 2 GB)
        if constexpr (NC >= kWave) f[e] = *reinterpret_cast<const float *>(base + row + static_cast<uint32_t>(n) * 4u);
        else f[e] = *reinterpret_cast<const float *>(base + (row + static_cast<uint32_t>(n) * 4u));
    }
}

// plane s of unit (kg, n) of a slab -> w[s][kg][n]
template <int NC>
__device__ __forceinline__ void store_w_unit(const UpdArgs &p, int k0, int id0, int lane, float (&f)[8], uint4 *w)
{
    const int id = id0 + lane, pos = k0 + unit_pos<NC>(id0, lane);
#pragma unroll
    for (int e = 0; e < 8; ++e) {
        bool again;
        (void)w_row(pos + e, p.d_in, again);
        f[e] = again ? 0.f : f[e];
    }
    Frag o[3];
    split8(f, o);
#pragma unroll
    for (int s = 0; s < 3; ++s) w[s * 4 * NC + id % (4 * NC)] = o[s].q;
}

// all of W (resident forms), two units per thread on their way at a time
template <int NC>
__device__ __forceinline__ void stage_w(const UpdArgs &p, int n_slabs, int n0, int wave, int lane, uint4 *w)
{
    constexpr int B = 2, SLAB = w_slab_bytes(NC) / 16;
    const int units = n_slabs * 4 * NC;                      // (a multiple of a wavefront)
    for (int base = wave * kWave; base < units; base += B * kSThreads) {
        float f[B][8];
#pragma unroll
        for (int b = 0; b < B; ++b) load_w_unit<NC>(p, 0, base + b * kSThreads, n0, lane, f[b]);      // (past the end: the last row again, not kept)
#pragma unroll
        for (int b = 0; b < B; ++b) {
            const int id0 = base + b * kSThreads;
            if (id0 < units) store_w_unit<NC>(p, 0, id0, lane, f[b], w + id0 / (4 * NC) * SLAB);
        }
    }
}

// The A operands of a slab as the loop carries them: the first half (k 0..7 and 16..23 of the slab) split, the second raw.
struct SlabA {
    Frag a0[3];
    float raw1[8];
};

__device__ __forceinline__ void read_raw(const float *abuf, int lane, int c, float (&f)[8])
{
#pragma unroll
    for (int q = 0; q < 2; ++q) {
        const float4 x = *reinterpret_cast<const float4 *>(abuf + (lane & 31) * kLda + 16 * (lane >> 5) + 8 * c + 4 * q);
        f[4 * q] = x.x; f[4 * q + 1] = x.y; f[4 * q + 2] = x.z; f[4 * q + 3] = x.w;
    }
}

// Products of one K slab: hi + lo += A slab * W slab, in 2 NT steps of eight MFMAs.  The W operands of a step are read from LDS
// one step ahead; between(x), called after step x, holds everything else the wavefront has to do, spread over the steps,
// so that the matrix pipe is not left idle while a wavefront waits, converts or stores (the fences keep the compiler
// from gathering it at the end).  In it, the next slab replaces `sa`: its raw half is used up by step NT - 1.
template <int NT, class Between>
__device__ __forceinline__ void multiply_slab(f32x16 (&hi)[NT], f32x16 (&lo)[NT], SlabA &sa, const uint4 *w, int lane, Between between)
{
    constexpr int NC = NT * 32, S = 2 * NT;
    const uint4 *wl = w + 2 * (lane >> 5) * NC + (lane & 31);
    Frag b[2][3], a0[3], a1[3];
    auto load_b = [&](int x) __attribute__((always_inline)) {
#pragma unroll
        for (int s = 0; s < 3; ++s) b[x & 1][s].q = wl[s * 4 * NC + x / NT * NC + x % NT * 32];
    };
#pragma unroll
    for (int s = 0; s < 3; ++s) a0[s] = sa.a0[s];
    load_b(0);
    static_for([&](auto step) __attribute__((always_inline)) {
        constexpr int x = step;
        if constexpr (x + 1 < S) load_b(x + 1);
        __builtin_amdgcn_sched_barrier(0);
        if constexpr (x == NT - 1) split8(sa.raw1, a1);
        constexpr int wi[7] = {2, 1, 2, 0, 1, 1, 0}, ai[7] = {1, 2, 0, 2, 1, 0, 1};          // small terms: w3 a2, w2 a3, w3 a1, ...
#pragma unroll
        for (int y = 0; y < 7; ++y)
            lo[x % NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[x & 1][wi[y]].v, x < NT ? a0[ai[y]].v : a1[ai[y]].v, lo[x % NT], 0, 0, 0);
        hi[x % NT] = __builtin_amdgcn_mfma_f32_32x32x16_bf16(b[x & 1][0].v, x < NT ? a0[0].v : a1[0].v, hi[x % NT], 0, 0, 0);
        between(step);
        __builtin_amdgcn_sched_barrier(0);
    }, std::make_integer_sequence<int, S>{});
}

// The part of `between` that brings the next slab of A from registers through LDS into operands.  The slab after that is
// requested right behind the last piece of W: a wavefront waits for its loads in order, and those of A come from HBM.
template <int NT, int x, class Next>
__device__ __forceinline__ void next_a(RawA &q, int lane, float *abuf, SlabA &sa, float (&raw0)[8], Next &&issue)
{
    constexpr int S = 2 * NT, X0 = S / 2, X1 = S > 4 ? S - 2 : S / 2;
    if constexpr (x == X0) {
        wave_sync_lds();
        stage_a(q, lane, abuf);
        wave_sync_lds();
        issue();
    }
    if constexpr (x == X1) {
        read_raw(abuf, lane, 0, raw0);
        read_raw(abuf, lane, 1, sa.raw1);
    }
    if constexpr (x == S - 1) {
        split8(raw0, sa.a0);
        wave_sync_lds();                                    // the buffer is free for the epilogue
    }
}

// the same at once, for the first slab
__device__ __forceinline__ void first_a(RawA &q, int lane, float *abuf, SlabA &sa)
{
    float raw0[8];
    stage_a(q, lane, abuf);
    wave_sync_lds();
    read_raw(abuf, lane, 0, raw0);
    read_raw(abuf, lane, 1, sa.raw1);
    split8(raw0, sa.a0);
    wave_sync_lds();
}

// acc holds the transposed 32x32 tiles (register r of lane (m, h): row m, column 8*(r/4) + 4*h + r%4); each goes
// through the wavefront's LDS buffer and leaves with 8 lanes per row, a whole line per row where rows are aligned.
// PLAIN: as it is, without scale, bias and ReLU.
template <int NT, bool PLAIN>
__device__ __forceinline__ void store_lines(const UpdArgs &p, const f32x16 (&acc)[NT], const float *bias, float *cbuf, int64_t m0, int n0, int lane)
{
    const int m = lane & 31, h = lane >> 5, c = (lane & 7) * 4;
    const int rows = static_cast<int>(p.n_rows - m0 < 32 ? p.n_rows - m0 : 32);
    const int esz = p.out_bf16 ? 2 : 4;
    char *base = static_cast<char *>(p.out) + (m0 * p.ld_out + n0) * esz;
#pragma unroll
    for (int t = 0; t < NT; ++t) {
        if (n0 + t * 32 >= p.d_out) break;
#pragma unroll
        for (int q = 0; q < 4; ++q)
            *reinterpret_cast<float4 *>(cbuf + m * kLda + 8 * q + 4 * h) = make_float4(acc[t][4 * q], acc[t][4 * q + 1], acc[t][4 * q + 2], acc[t][4 * q + 3]);
        wave_sync_lds();
        const int col = n0 + t * 32 + c;
        const float4 b = *reinterpret_cast<const float4 *>(bias + t * 32 + c);
#pragma unroll
        for (int j = 0; j < 4; ++j) {
            const int r = j * 8 + (lane >> 3);
            const float4 x = *reinterpret_cast<const float4 *>(cbuf + r * kLda + c);
            float v[4] = {x.x, x.y, x.z, x.w};
            if (!PLAIN) {
                v[0] = fmaf(x.x, kUnscale, b.x); v[1] = fmaf(x.y, kUnscale, b.y); v[2] = fmaf(x.z, kUnscale, b.z); v[3] = fmaf(x.w, kUnscale, b.w);
                if (p.relu) {
#pragma unroll
                    for (int e = 0; e < 4; ++e) v[e] = v[e] > 0.f ? v[e] : 0.f;
                }
            }
            if (r >= rows || col >= p.d_out) continue;
            char *at = base + (static_cast<uint32_t>(r) * static_cast<uint32_t>(p.ld_out) + static_cast<uint32_t>(t * 32 + c)) * static_cast<uint32_t>(esz);
            if (p.out_bf16) {
                uint16_t *o = reinterpret_cast<uint16_t *>(at);
                if (col + 4 <= p.d_out) {
                    const uint32_t pk[2] = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
                    __builtin_memcpy(__builtin_assume_aligned(o, 2), pk, 8);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < p.d_out) o[e] = to_bf16(v[e]);
                }
            } else {
                float *o = reinterpret_cast<float *>(at);
                if (col + 4 <= p.d_out) {
                    __builtin_memcpy(__builtin_assume_aligned(o, 4), v, 16);
                } else {
#pragma unroll
                    for (int e = 0; e < 4; ++e)
                        if (col + e < p.d_out) o[e] = v[e];
                }
            }
        }
        wave_sync_lds();
    }
}

// Row softmax on the accumulators (scale and bias first), for outputs whose whole row one wavefront holds: row m lies in lanes m and
// m + 32, so maximum and sum need one exchange.  Saves the pass that would read and write every row again
// (row_softmax_kernel: 7 us of a 65 us two-layer GCN on 30 k nodes).
template <int NT>
__device__ __forceinline__ void softmax_rows(const UpdArgs &p, f32x16 (&acc)[NT], float scale, const float *bias, int lane)
{
    const int h = lane >> 5;
    float m = -INFINITY;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int col = t * 32 + 8 * (r / 4) + 4 * h + r % 4;
            if (col < p.d_out) {
                acc[t][r] = fmaf(acc[t][r], scale, bias[col]);
            } else {
                acc[t][r] = -INFINITY;
            }
            m = fmaxf(m, acc[t][r]);
        }
    m = fmaxf(m, __shfl_xor(m, 32));
    float sum = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            const int col = t * 32 + 8 * (r / 4) + 4 * h + r % 4;
            acc[t][r] = col < p.d_out ? expf(acc[t][r] - m) : 0.f;
            sum += acc[t][r];
        }
    sum += __shfl_xor(sum, 32);
    const float inv = 1.f / sum;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) acc[t][r] *= inv;
}

// The tile's sums, hi + lo (still scaled); true where one is not finite.
template <int NT>
__device__ __forceinline__ bool combine(f32x16 (&hi)[NT], const f32x16 (&lo)[NT])
{
    float z = 0.f;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r) {
            hi[t][r] += lo[t][r];
            z = fmaf(hi[t][r], 0.f, z);                      // NaN from the first infinity or NaN on
        }
    return __ballot(z != 0.f) != 0;
}

// Which elements of the tile those are: bit 16 t + r of a lane.  Rows and columns that do not exist are left out.
template <int NT>
__device__ __forceinline__ uint64_t not_finite(const UpdArgs &p, const f32x16 (&acc)[NT], int64_t m0, int n0, int lane)
{
    uint64_t bad = 0;
    if (m0 + (lane & 31) >= p.n_rows) return bad;
#pragma unroll
    for (int t = 0; t < NT; ++t)
#pragma unroll
        for (int r = 0; r < 16; ++r)
            if (n0 + t * 32 + 8 * (r / 4) + 4 * (lane >> 5) + r % 4 < p.d_out && !(fabsf(acc[t][r]) < INFINITY)) bad |= 1ull << (16 * t + r);
    return bad;
}

// A 32 x 32 block of sums with the fp32 instruction, operands straight from global memory.
__device__ __forceinline__ f32x16 exact_block(const UpdArgs &p, int64_t m0, int n0, int lane)
{
    const int i = lane & 31, h = lane >> 5;
    const int rows = static_cast<int>(p.n_rows - m0 < 32 ? p.n_rows - m0 : 32);
    const float *a = static_cast<const float *>(p.a) + (m0 + min(i, rows - 1)) * p.ld_a;
    const float *w = static_cast<const float *>(p.w) + min(n0 + i, p.d_out - 1);
    f32x16 acc;
#pragma unroll
    for (int r = 0; r < 16; ++r) acc[r] = 0.f;
#pragma unroll 1
    for (int k0 = 0; k0 < p.d_in; k0 += 16) {
        float af[8], wf[8];
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const int k = min(k0 + 2 * c + h, p.d_in - 1);
            af[c] = a[k];
            wf[c] = w[static_cast<int64_t>(k) * p.d_out];
        }
#pragma unroll
        for (int c = 0; c < 8; ++c) {
            const bool in = k0 + 2 * c + h < p.d_in;
            acc = __builtin_amdgcn_mfma_f32_32x32x2f32(in ? wf[c] : 0.f, in ? af[c] : 0.f, acc, 0, 0, 0);
        }
    }
    return acc;
}

// Puts the elements `bad` marks right, over what store_lines has written; with softmax, the whole rows they are in.
template <int NT, bool SOFTMAX>
__device__ __forceinline__ void repair(const UpdArgs &p, uint64_t bad, const float *bias, int64_t m0, int n0, int lane)
{
    const int h = lane >> 5;
    const int64_t at = (m0 + (lane & 31)) * p.ld_out;
    auto put = [&](int col, float v) __attribute__((always_inline)) {
        if (p.out_bf16) static_cast<uint16_t *>(p.out)[at + col] = to_bf16(v);
        else static_cast<float *>(p.out)[at + col] = v;
    };
    if (!__ballot(bad != 0)) return;                        // (only rows or columns that do not exist)
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // what other lanes stored there is there
    if constexpr (SOFTMAX) {
        f32x16 acc[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t) acc[t] = exact_block(p, m0, n0 + t * 32, lane);
        softmax_rows<NT>(p, acc, 1.f, bias, lane);
        const bool row_bad = (bad | __shfl_xor(static_cast<unsigned long long>(bad), 32)) != 0;
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                const int col = n0 + t * 32 + 8 * (r / 4) + 4 * h + r % 4;
                if (row_bad && col < p.d_out) put(col, acc[t][r]);
            }
    } else {
#pragma unroll 1
        for (int t = 0; t < NT; ++t, bad >>= 16) {
            if (!__ballot((bad & 0xffffu) != 0)) continue;
            const f32x16 acc = exact_block(p, m0, n0 + t * 32, lane);
#pragma unroll
            for (int r = 0; r < 16; ++r) {
                if (!(bad >> r & 1)) continue;
                const int col = n0 + t * 32 + 8 * (r / 4) + 4 * h + r % 4;
                float v = acc[r] + bias[col - n0];
                if (p.relu) v = v > 0.f ? v : 0.f;
                put(col, v);
            }
        }
    }
}

// What only depends on the arguments and the lane would be computed ahead of all loops and held in registers that
// the accumulators need; the epilogue works on a copy the compiler cannot see through.
__device__ __forceinline__ UpdArgs opaque(UpdArgs p)
{
    int64_t zero = 0;                                        // (the pointers themselves through asm would be flat ones)
    asm volatile("" : "+s"(zero), "+s"(p.d_out), "+s"(p.ld_out), "+s"(p.ld_a));
    p.out = static_cast<char *>(p.out) + zero;
    p.w = static_cast<const char *>(p.w) + zero;
    p.a = static_cast<const char *>(p.a) + zero;
    return p;
}

__device__ __forceinline__ int opaque(int lane)
{
    asm volatile("" : "+v"(lane));
    return lane;
}

struct Place {
    int col, group, groups;
};

// Column blocks of the same rows run at the same time on one XCD (workgroups b, b + 8, ...), so that A reaches its L2 once;
// side by side where there are too few rows for that.
__device__ __forceinline__ Place place(int n_cols)
{
    const int b = static_cast<int>(blockIdx.x), groups = static_cast<int>(gridDim.x) / n_cols;
    if (groups % 8) return {b % n_cols, b / n_cols, groups};
    return {(b >> 3) % n_cols, (b >> 3) / n_cols * 8 + (b & 7), groups};
}

// (wavefronts per SIMD the registers are cut for: two; four, two workgroups per CU, with accumulators of 32 registers)
template <int NT, bool SOFTMAX>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(NT >= 2 ? 2 : 4, NT >= 2 ? 2 : 4)))
void update_split_resident_kernel(const UpdArgs p, int n_cols)
{
    constexpr int NC = NT * 32, SLAB = w_slab_bytes(NC) / 16;
    __shared__ __attribute__((aligned(16))) float bias[NC];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const Place at = place(n_cols);
    const int n0 = at.col * NC;
    const int n_slabs = (p.d_in + 31) / 32;
    uint4 *w = reinterpret_cast<uint4 *>(lds_split);
    float *abuf = reinterpret_cast<float *>(lds_split + n_slabs * w_slab_bytes(NC) + wave * kWaveBytes);

    // tiles are dealt out workgroup by workgroup, so that a small call still spreads over the chip
    const int64_t n_tiles = (p.n_rows + 31) / 32, stride = static_cast<int64_t>(at.groups) * kSWaves;
    int64_t tile = static_cast<int64_t>(wave) * at.groups + at.group;

    RawA q[2];
    int64_t itile = tile;                                    // issue cursor: the slab requested next
    int is = 0;
    auto issue = [&](RawA &r) __attribute__((always_inline)) {
        load_a(p, itile * 32, is * 32, lane, r);             // (past the last tile: rows are clamped)
        if (++is == n_slabs) { is = 0; itile += stride; }
    };
    issue(q[0]);
    issue(q[1]);
    stage_bias<NC>(bias, p.bias ? p.bias + n0 : nullptr, p.d_out - n0);
    stage_w<NC>(p, n_slabs, n0, wave, lane, w);
    __syncthreads();

    if (tile >= n_tiles) return;
    SlabA sa;
    first_a(q[0], lane, abuf, sa);
    q[0] = q[1];
    issue(q[1]);
    do {
        f32x16 acc[NT], lo[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = lo[t][r] = 0.f;
        int s = 0;
#pragma unroll 1
        do {
            float raw0[8];
            multiply_slab<NT>(acc, lo, sa, w + s * SLAB, lane, [&](auto step) __attribute__((always_inline)) {
                next_a<NT, decltype(step)::value>(q[0], lane, abuf, sa, raw0, [&]() __attribute__((always_inline)) { q[0] = q[1]; issue(q[1]); });
            });
        } while (++s < n_slabs);
        const bool any = combine<NT>(acc, lo);
        uint64_t bad = 0;
        if constexpr (SOFTMAX) {
            if (any) bad = not_finite<NT>(opaque(p), acc, tile * 32, n0, opaque(lane));
            softmax_rows<NT>(opaque(p), acc, kUnscale, bias, opaque(lane));
        }
        store_lines<NT, SOFTMAX>(opaque(p), acc, bias, abuf, tile * 32, n0, opaque(lane));
        if (any) {
            if constexpr (!SOFTMAX) bad = not_finite<NT>(opaque(p), acc, tile * 32, n0, opaque(lane));
            repair<NT, SOFTMAX>(opaque(p), bad, bias, tile * 32, n0, opaque(lane));
        }
        tile += stride;
    } while (tile < n_tiles);
}

template <int NT>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(2, 2)))
void update_split_slab_kernel(const UpdArgs p, int64_t n_tiles, int n_cols)
{
    constexpr int NC = NT * 32, SLAB = w_slab_bytes(NC) / 16;
    constexpr int UNITS = (4 * NC + kSThreads - 1) / kSThreads;          // of a slab, per thread
    __shared__ __attribute__((aligned(16))) float bias[NC];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const Place at = place(n_cols);
    const int n0 = at.col * NC;
    const int n_slabs = (p.d_in + 31) / 32;
    uint4 *w = reinterpret_cast<uint4 *>(lds_split);                     // two slabs
    float *abuf = reinterpret_cast<float *>(lds_split + 2 * w_slab_bytes(NC) + wave * kWaveBytes);
    // (narrow slabs have fewer units than threads: some are staged twice, with the same values)
    auto unit0 = [&](int u) { return (u * kSThreads + wave * kWave) % (4 * NC); };
    auto load_w = [&](int ks, int u, float (&f)[8]) { load_w_unit<NC>(p, ks * 32, unit0(u), n0, lane, f); };
    auto store_w = [&](int buf, int ks, int u, float (&f)[8]) { store_w_unit<NC>(p, ks * 32, unit0(u), lane, f, w + buf * SLAB); };

    int64_t tile = at.group;                                             // the host launches at most n_tiles groups
    auto first_row = [&](int64_t t) { return (t * kSWaves + wave) * 32; };
    RawA q;
    SlabA sa;
    load_a(p, first_row(tile), 0, lane, q);
    {
        float wf[UNITS][8];
#pragma unroll
        for (int u = 0; u < UNITS; ++u) load_w(0, u, wf[u]);
        stage_bias<NC>(bias, p.bias ? p.bias + n0 : nullptr, p.d_out - n0);
#pragma unroll
        for (int u = 0; u < UNITS; ++u) store_w(0, 0, u, wf[u]);
    }
    first_a(q, lane, abuf, sa);
    // issue cursor of A: the slab after the one in `sa` (after the last tile: rows are clamped, and never used)
    int64_t itile = tile;
    int is = 0;
    auto issue = [&]() __attribute__((always_inline)) {
        if (++is == n_slabs) { is = 0; itile += at.groups; }
        load_a(p, first_row(itile), is * 32, lane, q);
    };
    issue();
    __syncthreads();
    int cur = 0;
#pragma unroll 1
    for (;;) {
        f32x16 acc[NT], lo[NT];
#pragma unroll
        for (int t = 0; t < NT; ++t)
#pragma unroll
            for (int r = 0; r < 16; ++r) acc[t][r] = lo[t][r] = 0.f;
        const int64_t ntile = tile + at.groups;
        int ks = 0;
#pragma unroll 1
        do {
            const int nks = ks + 1 == n_slabs ? 0 : ks + 1;            // the slab after this one
            float raw0[8], wf[8];
            multiply_slab<NT>(acc, lo, sa, w + cur * SLAB, lane, [&](auto step) __attribute__((always_inline)) {
                // W: one unit after the other through the same registers, half of the slab in flight each
                constexpr int S = 2 * NT, x = step;
#pragma unroll
                for (int u = 0; u < UNITS; ++u) {
                    if (x == u * 6 * S / 16) load_w(nks, u, wf);
                    if (x == u * 6 * S / 16 + S / 2) store_w(cur ^ 1, nks, u, wf);       // the other buffer: nobody reads it before the barrier
                }
                next_a<NT, x>(q, lane, abuf, sa, raw0, issue);
            });
            __syncthreads();
            cur ^= 1;
        } while (++ks < n_slabs);
        const bool any = combine<NT>(acc, lo);
        store_lines<NT, false>(opaque(p), acc, bias, abuf, first_row(tile), n0, opaque(lane));
        if (any) repair<NT, false>(opaque(p), not_finite<NT>(opaque(p), acc, first_row(tile), n0, opaque(lane)), bias, first_row(tile), n0, opaque(lane));
        if (ntile >= n_tiles) break;
        tile = ntile;
    }
}

// ---- up to 32 output columns: blocks of 16 --------------------------------------------------------
// v_mfma_f32_16x16x32_bf16 on C blocks of 16 columns: a block of 32 on the 32 x 32 instruction, its accumulators through LDS to
// whole lines, spent more on the epilogue than HBM leaves (400,000 x 32 -> 16: 21.3 us, 16.0 so; -> 8: 19.9, 15.0; 400,000 x 64 -> 8:
// 27.4, 23; 400,000 x 16 -> 32: 18.0, 16.4).  The accumulator of a 16 x 16 tile (register r of lane (m, g) =
// (lane % 16, lane / 16): row m, column 4 g + r) is stored as it stands: the four lanes of a row write consecutive columns.
// W is resident; two slabs of A on their way are all the pipelining there is, which four wavefronts per SIMD make up for.
template <int C>
struct Sums {
    f32x4 v[2][C];           // [rows 0..15 and 16..31 of the tile][block of columns]
};

template <int C>
__device__ __forceinline__ void softmax_narrow(const UpdArgs &p, f32x4 (&v)[C], int lane)
{
    float m = -INFINITY;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            if (16 * c + 4 * (lane >> 4) + e >= p.d_out) v[c][e] = -INFINITY;
            m = fmaxf(m, v[c][e]);
        }
    m = fmaxf(m, __shfl_xor(m, 16));
    m = fmaxf(m, __shfl_xor(m, 32));
    float sum = 0.f;
#pragma unroll
    for (int c = 0; c < C; ++c)
#pragma unroll
        for (int e = 0; e < 4; ++e) {
            v[c][e] = 16 * c + 4 * (lane >> 4) + e < p.d_out ? expf(v[c][e] - m) : 0.f;
            sum += v[c][e];
        }
    sum += __shfl_xor(sum, 16);
    sum += __shfl_xor(sum, 32);
    const float inv = 1.f / sum;
#pragma unroll
    for (int c = 0; c < C; ++c) v[c] *= inv;
}

__device__ __forceinline__ f32x4 activate(const UpdArgs &p, const f32x4 &sum, float scale, const f32x4 &b)
{
    f32x4 v;
#pragma unroll
    for (int e = 0; e < 4; ++e) {
        v[e] = fmaf(sum[e], scale, b[e]);
        if (p.relu) v[e] = v[e] > 0.f ? v[e] : 0.f;
    }
    return v;
}

// columns col .. col + 3 of a row: those that exist, and of these the ones whose bit in `which` is set
__device__ __forceinline__ void store4(const UpdArgs &p, const f32x4 &v, int64_t row, int col, int which)
{
    if (row >= p.n_rows || col >= p.d_out) return;
    const bool whole = which == 15 && col + 4 <= p.d_out;
    if (p.out_bf16) {
        uint16_t *o = static_cast<uint16_t *>(p.out) + row * p.ld_out + col;
        const uint32_t pk[2] = {pack_bf16(v[0], v[1]), pack_bf16(v[2], v[3])};
        if (whole) {
            __builtin_memcpy(__builtin_assume_aligned(o, 2), pk, 8);
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((which >> e & 1) && col + e < p.d_out) o[e] = static_cast<uint16_t>(pk[e / 2] >> (16 * (e & 1)));
        }
    } else {
        float *o = static_cast<float *>(p.out) + row * p.ld_out + col;
        if (whole) {
            *reinterpret_cast<f32x4_loose *>(o) = v;
        } else {
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if ((which >> e & 1) && col + e < p.d_out) o[e] = v[e];
        }
    }
}

// What `repair` does, for such a tile, 16 x 16 elements at a time.
template <int C, bool SOFTMAX>
__device__ __forceinline__ void repair_narrow(const UpdArgs &p, const Sums<C> &sum, const float *bias, int64_t m0, int lane)
{
    const int i = lane & 15, g = lane >> 4;
    asm volatile("s_waitcnt vmcnt(0)" ::: "memory");        // what was stored there is there
#pragma unroll
    for (int x = 0; x < 2; ++x) {
        const int64_t row = m0 + 16 * x + i;
        int bad[C], any = 0;
#pragma unroll
        for (int c = 0; c < C; ++c) {
            bad[c] = 0;
#pragma unroll
            for (int e = 0; e < 4; ++e)
                if (!(fabsf(sum.v[x][c][e]) < INFINITY) && row < p.n_rows && 16 * c + 4 * g + e < p.d_out) bad[c] |= 1 << e;
            any |= bad[c];
        }
        if (!__ballot(any != 0)) continue;
        if constexpr (SOFTMAX) {                             // a row as a whole
            any |= __shfl_xor(any, 16);
            any |= __shfl_xor(any, 32);
        }
        const float *a = static_cast<const float *>(p.a) + min(row, p.n_rows - 1) * p.ld_a;
        f32x4 v[C];
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const float *w = static_cast<const float *>(p.w) + min(16 * c + i, p.d_out - 1);
            f32x4 acc = {0.f, 0.f, 0.f, 0.f};
#pragma unroll 1
            for (int k0 = 0; k0 < p.d_in; k0 += 32) {
                float af[8], wf[8];
#pragma unroll
                for (int k8 = 0; k8 < 8; ++k8) {
                    const int k = min(k0 + 4 * k8 + g, p.d_in - 1);
                    af[k8] = a[k];
                    wf[k8] = w[static_cast<int64_t>(k) * p.d_out];
                }
#pragma unroll
                for (int k8 = 0; k8 < 8; ++k8) {
                    const bool in = k0 + 4 * k8 + g < p.d_in;
                    acc = __builtin_amdgcn_mfma_f32_16x16x4f32(in ? wf[k8] : 0.f, in ? af[k8] : 0.f, acc, 0, 0, 0);
                }
            }
            v[c] = activate(p, acc, 1.f, *reinterpret_cast<const f32x4 *>(bias + 16 * c + 4 * g));
        }
        if constexpr (SOFTMAX) softmax_narrow<C>(p, v, lane);
#pragma unroll
        for (int c = 0; c < C; ++c) {
            const int which = SOFTMAX ? (any ? 15 : 0) : bad[c];
            if (which) store4(p, v[c], row, 16 * c + 4 * g, which);
        }
    }
}

template <int C, bool SOFTMAX>
__global__ __launch_bounds__(kSThreads) __attribute__((amdgpu_waves_per_eu(4, 4)))
void update_split_narrow_kernel(const UpdArgs p)
{
    constexpr int NC = 16 * C, SLAB = w_slab_bytes(NC) / 16;
    __shared__ __attribute__((aligned(16))) float bias[NC];
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane(static_cast<int>(threadIdx.x) >> 6);
    const int i = lane & 15, g = lane >> 4;
    const int n_slabs = (p.d_in + 31) / 32;
    uint4 *w = reinterpret_cast<uint4 *>(lds_split);
    float *abuf = reinterpret_cast<float *>(lds_split + n_slabs * w_slab_bytes(NC) + wave * kWaveBytes);

    // tiles are dealt out workgroup by workgroup, so that a small call still spreads over the chip
    const int64_t n_tiles = (p.n_rows + 31) / 32, stride = static_cast<int64_t>(gridDim.x) * kSWaves;
    int64_t tile = static_cast<int64_t>(wave) * gridDim.x + blockIdx.x;
    RawA q[2];
    int64_t itile = tile;                                    // issue cursor: the slab requested next
    int is = 0;
    auto issue = [&](RawA &r) __attribute__((always_inline)) {
        load_a(p, itile * 32, is * 32, lane, r);             // (past the last tile: rows are clamped)
        if (++is == n_slabs) { is = 0; itile += stride; }
    };
    issue(q[0]);
    issue(q[1]);
    stage_bias<NC>(bias, p.bias, p.d_out);
    stage_w<NC>(p, n_slabs, 0, wave, lane, w);
    __syncthreads();

    for (; tile < n_tiles; tile += stride) {
        Sums<C> hi{}, lo{};
#pragma unroll 1
        for (int s = 0; s < n_slabs; ++s) {
            Frag a[2][3];
            stage_a(q[0], lane, abuf);
            wave_sync_lds();
            float raw[2][8];
#pragma unroll
            for (int x = 0; x < 2; ++x)
#pragma unroll
                for (int h = 0; h < 2; ++h) {
                    const f32x4 y = *reinterpret_cast<const f32x4 *>(abuf + (16 * x + i) * kLda + 8 * g + 4 * h);
#pragma unroll
                    for (int e = 0; e < 4; ++e) raw[x][4 * h + e] = y[e];
                }
            wave_sync_lds();                                 // the buffer is free for the next slab
            q[0] = q[1];
            issue(q[1]);
            split8(raw[0], a[0]);
            split8(raw[1], a[1]);
#pragma unroll
            for (int c = 0; c < C; ++c) {
                Frag wf[3];
#pragma unroll
                for (int t = 0; t < 3; ++t) wf[t].q = w[s * SLAB + t * 4 * NC + g * NC + 16 * c + i];
                constexpr int wi[7] = {2, 1, 2, 0, 1, 1, 0}, ai[7] = {1, 2, 0, 2, 1, 0, 1};          // (multiply_slab)
#pragma unroll
                for (int y = 0; y < 7; ++y)
#pragma unroll
                    for (int x = 0; x < 2; ++x) lo.v[x][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[wi[y]].v, a[x][ai[y]].v, lo.v[x][c], 0, 0, 0);
#pragma unroll
                for (int x = 0; x < 2; ++x) hi.v[x][c] = __builtin_amdgcn_mfma_f32_16x16x32_bf16(wf[0].v, a[x][0].v, hi.v[x][c], 0, 0, 0);
            }
        }
        float z = 0.f;
#pragma unroll
        for (int x = 0; x < 2; ++x) {
            f32x4 v[C];
#pragma unroll
            for (int c = 0; c < C; ++c) {
                hi.v[x][c] += lo.v[x][c];
#pragma unroll
                for (int e = 0; e < 4; ++e) z = fmaf(hi.v[x][c][e], 0.f, z);      // NaN from the first infinity or NaN on
                v[c] = activate(p, hi.v[x][c], kUnscale, *reinterpret_cast<const f32x4 *>(bias + 16 * c + 4 * g));
            }
            if constexpr (SOFTMAX) softmax_narrow<C>(p, v, lane);
#pragma unroll
            for (int c = 0; c < C; ++c) store4(p, v[c], tile * 32 + 16 * x + i, 16 * c + 4 * g, 15);
        }
        if (__ballot(z != 0.f)) repair_narrow<C, SOFTMAX>(p, hi, bias, tile * 32, lane);
    }
}

// Workgroups of a column block: as many as there are row tiles, or as fit the chip beside the other column blocks.
int groups_of(int64_t n_tiles, int64_t slots, int n_cols)
{
    int64_t g = std::min(n_tiles, std::max<int64_t>(1, slots / n_cols));
    if (n_cols > 1 && g > 8 && g < n_tiles) g = g / 8 * 8;                                  // (see place)
    return static_cast<int>(g);
}

template <int NT, bool SOFTMAX>
hipError_t launch_resident(const UpdArgs &p, int cus, hipStream_t s)
{
    const size_t lds = static_cast<size_t>((p.d_in + 31) / 32) * w_slab_bytes(NT * 32) + kSWaves * kWaveBytes;
    const int n_cols = (p.d_out + NT * 32 - 1) / (NT * 32);
    const int64_t n_tiles = (p.n_rows + 31) / 32;
    const int64_t slots = static_cast<int64_t>(cus) * (NT < 2 && 2 * lds <= kLdsMax ? 2 : 1);
    const dim3 grid(static_cast<unsigned>(groups_of(n_tiles, slots, n_cols)) * n_cols);
    if (lds > 48 * 1024)                                     // beyond what a launch may take unasked
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&update_split_resident_kernel<NT, SOFTMAX>), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    hipLaunchKernelGGL((update_split_resident_kernel<NT, SOFTMAX>), grid, dim3(kSThreads), lds, s, p, n_cols);
    return hipGetLastError();
}

template <int NT>
hipError_t launch_slab(const UpdArgs &p, int cus, hipStream_t s)
{
    constexpr int lds = 2 * w_slab_bytes(NT * 32) + kSWaves * kWaveBytes;
    const int n_cols = (p.d_out + NT * 32 - 1) / (NT * 32);
    const int64_t n_tiles = (p.n_rows + 32 * kSWaves - 1) / (32 * kSWaves);
    const dim3 grid(static_cast<unsigned>(groups_of(n_tiles, cus, n_cols)) * n_cols);
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&update_split_slab_kernel<NT>), hipFuncAttributeMaxDynamicSharedMemorySize, lds);
    hipLaunchKernelGGL((update_split_slab_kernel<NT>), grid, dim3(kSThreads), lds, s, p, n_tiles, n_cols);
    return hipGetLastError();
}

template <int C, bool SOFTMAX>
hipError_t launch_narrow(const UpdArgs &p, int cus, hipStream_t s)
{
    const size_t lds = static_cast<size_t>((p.d_in + 31) / 32) * w_slab_bytes(16 * C) + kSWaves * kWaveBytes;
    const int64_t n_tiles = (p.n_rows + 31) / 32, slots = static_cast<int64_t>(cus) * (2 * lds <= kLdsMax ? 2 : 1);
    const dim3 grid(static_cast<unsigned>(std::min(n_tiles, slots)));
    if (lds > 48 * 1024)
        (void)hipFuncSetAttribute(reinterpret_cast<const void *>(&update_split_narrow_kernel<C, SOFTMAX>), hipFuncAttributeMaxDynamicSharedMemorySize, static_cast<int>(lds));
    hipLaunchKernelGGL((update_split_narrow_kernel<C, SOFTMAX>), grid, dim3(kSThreads), lds, s, p);
    return hipGetLastError();
}

}  // namespace

bool launch_update_split(const upd::UpdArgs &p, int cus, hipStream_t stream, bool *softmax, hipError_t *err)
{
    // a row shorter than a 16-byte vector, or 32-bit offsets inside W or a 32-row tile of A or out that could overflow
    if (p.d_in < 4 || p.d_out > (1 << 20) || p.ld_a > (1 << 24) || p.ld_out > (1 << 24) || static_cast<int64_t>(p.d_in) * p.d_out > (1 << 29)) return false;
    const int64_t n_slabs = (p.d_in + 31) / 32;
    auto resident = [&](int cols) { return n_slabs * w_slab_bytes(cols) + kSWaves * kWaveBytes <= kLdsMax; };
    // The matrix instruction and the place of the softmax decide how a sum is rounded: they depend on d_in and d_out alone,
    // so that a row has the same bits in a call of any number of rows.  Up to 32 columns: the narrow form where W fits.
    if (p.d_out <= 32 && resident(p.d_out <= 16 ? 16 : 32)) {
        if (p.d_out <= 16) *err = *softmax ? launch_narrow<1, true>(p, cus, stream) : launch_narrow<1, false>(p, cus, stream);
        else *err = *softmax ? launch_narrow<2, true>(p, cus, stream) : launch_narrow<2, false>(p, cus, stream);
        *softmax = false;
        return true;
    }
    // Softmax in the epilogue where a wavefront holds whole rows in few registers; elsewhere it stays the caller's second pass.
    if (*softmax && p.d_out > 32 && p.d_out <= 64 && resident(64)) {
        *err = launch_resident<2, true>(p, cus, stream);
        *softmax = false;
        return true;
    }
    // As many columns per wavefront as there are (up to 128), so that A is read and split as seldom as the registers allow.  Few
    // rows: narrower column blocks side by side until the workgroups cover the chip (the rows are re-read out of the caches:
    // 2,000 x 602 -> 256 takes 16.7 us in 8 blocks of 32, 116 with the fp32 instruction in one block).
    int nt = p.d_out > 64 ? 4 : p.d_out > 32 ? 2 : 1;
    auto groups = [&](int t) { return (resident(32 * t) ? (p.n_rows + 31) / 32 : (p.n_rows + 255) / 256) * ((p.d_out + 32 * t - 1) / (32 * t)); };
    while (nt > 1 && groups(nt) < cus) nt /= 2;
    if (resident(32 * nt)) *err = nt == 4 ? launch_resident<4, false>(p, cus, stream) : nt == 2 ? launch_resident<2, false>(p, cus, stream) : launch_resident<1, false>(p, cus, stream);
    else *err = nt == 4 ? launch_slab<4>(p, cus, stream) : nt == 2 ? launch_slab<2>(p, cus, stream) : launch_slab<1>(p, cus, stream);
    return true;
}

}  // namespace mgg
