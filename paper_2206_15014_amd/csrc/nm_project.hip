// nm_project: the Z-update of the ADMM decomposition, Z = Pi(W + U) (Sec. 3.1, Eq. 3 applied to
// W + U), with the quantisation constraint solved after the sparsity constraint (Sec. 3.3.1,
// ADMM-Max scale per group of output neurons, Sec. 4) and the dual update U + W - Z, on gfx950.
//
// Purely HBM-bound: 4 (W) + 4 (U) bytes read and 4 (Z) + 4 (U') bytes written per weight, plus
// one more read of W and U for the scales where a scale group is too large for the wavefronts that
// hold its values (the second read mostly hits the last-level cache).  At these sizes a launch is a
// few microseconds, so what counts is loads in flight and the number of launches: every lane
// requests all it needs before its first use.  With one row per scale and up to 4096 columns there is one launch, and
// with scale groups of several rows one whose workgroups tell one another their maxima (project_parts_kernel).
// Otherwise - under stream capture, in place, very many small or a few very large scale groups - there are two, or three for large
// scale groups:
//  - row maxima, then the projection, which forms the scales.  The per-row scale array is the only scratch: it
//    first receives the rows' largest magnitudes, negated, and the projection replaces them by the scales
//    while it runs - a value with the sign bit set is a maximum, one without is a scale, and either tells a
//    reader what it needs;
//  - the scales, one workgroup or wavefront per scale group, then the projection (groups of up to 4096 values);
//  - row maxima, scales, projection.
// Every arithmetic step is one fp32 operation, in the order the declaration of nm_project states.
//
// Measurements stand at the rules of launch_project_m.  The 48 matrices of a BERT-base encoder (32 rows per scale, operands from
// HBM), against three launches a matrix with a load at a time per thread: 748 -> 598 us on two launches, 504 on one, of which moving every
// byte once takes about 250.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <type_traits>

#include "nm.h"
#include "nm_internal.h"

#include <atomic>

// Where the workgroups of project_parts_kernel tell one another their maxima: every GPU the library runs on holds its own copy. A
// call uses one region of the 64 in turn, a word per workgroup; should two calls in flight ever share one, words of the other call are
// seen for what they are by their number.
constexpr int MEET_REGIONS = 64, MEET_WORDS = 4096;
static_assert(MEET_REGIONS * MEET_WORDS * sizeof(unsigned long long) == NM_PROJECT_EXCHANGE_BYTES, "as the header says");
static __device__ unsigned long long meet_words[MEET_REGIONS * MEET_WORDS];

namespace nm {

namespace {

__device__ __forceinline__ float wave_max_f(float m)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    return m;
}

// max over the wavefront of 32-bit signed values
__device__ __forceinline__ int wave_max_i(int m)
{
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = max(m, __shfl_xor(m, d, 64));
    return m;
}

__device__ __forceinline__ float scale_of_max(float m, float qmax) { return (m == 0.0f) ? 1.0f : __fdiv_rn(m, qmax); }

// COUNT groups of F float4s of W + U: one test of U for all of them (a test per load would leave each to wait for the one
// before it), and, where TOGETHER, every load requested before the first sum.
template <int COUNT, int F, bool TOGETHER = true, typename At>
__device__ __forceinline__ void sums_at(const float* W, const float* U, At at, float4 (&x)[COUNT][F])
{
#pragma unroll
    for (int i = 0; i < COUNT; ++i)
#pragma unroll
        for (int f = 0; f < F; ++f) x[i][f] = *reinterpret_cast<const float4*>(W + at(i) + 4 * f);
    if (!U) return;
    float4 u[COUNT][F];
#pragma unroll
    for (int i = 0; i < COUNT; ++i)
#pragma unroll
        for (int f = 0; f < F; ++f) u[i][f] = *reinterpret_cast<const float4*>(U + at(i) + 4 * f);
    if constexpr (TOGETHER) __builtin_amdgcn_sched_barrier(0);
#pragma unroll
    for (int i = 0; i < COUNT; ++i)
#pragma unroll
        for (int f = 0; f < F; ++f) {
            x[i][f].x = __fadd_rn(x[i][f].x, u[i][f].x);
            x[i][f].y = __fadd_rn(x[i][f].y, u[i][f].y);
            x[i][f].z = __fadd_rn(x[i][f].z, u[i][f].z);
            x[i][f].w = __fadd_rn(x[i][f].w, u[i][f].w);
        }
}

// f(std::integral_constant<int, min(count, MOST)>): `count` (at least 1) is uniform over the wavefront, so a wavefront
// requests no more than the row has left for it, and still all of that at once.
template <int MOST, typename F>
__device__ __forceinline__ void with_count(int count, F f)
{
    if constexpr (MOST > 1) {
        if (count < MOST) return with_count<MOST - 1>(count, f);
    }
    f(std::integral_constant<int, MOST>{});
}

__device__ __forceinline__ float max4(float m, const float4& v)
{
    return fmaxf(m, fmaxf(fmaxf(fabsf(v.x), fabsf(v.y)), fmaxf(fabsf(v.z), fabsf(v.w))));
}

// max over aligned groups of LANES lanes
template <int LANES>
__device__ __forceinline__ float lanes_max_f(float m)
{
#pragma unroll
    for (int d = LANES / 2; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    return m;
}

// -(largest |W + U|) of every row: -0 for a row of zeros.  LANES lanes per row: 16 (16 rows per workgroup), a
// wavefront, or the whole workgroup; four or five 16-byte pieces of W and of U per lane in flight.
template <int LANES>
__global__ void __launch_bounds__(256)
project_amax_kernel(const float* __restrict__ W, const float* __restrict__ U, int rows, int cols, int ldw,
                    float* __restrict__ amax, int vec)         // vec: rows are whole, 16-byte aligned float4s
{
    __shared__ float part[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int row = (int)(blockIdx.x * (256 / LANES) + threadIdx.x / LANES), at = (int)threadIdx.x % LANES;
    if (row >= rows) return;                   // LANES = 256: one row per workgroup, none leaves before the barrier
    const size_t base = (size_t)row * ldw;
    float m = 0.0f;
    if (vec) {
        const int pieces = cols / 4;
        int i = LANES == 256 ? 64 * wave : 0;  // the wavefront's first piece (of each of its rows)
        while (i < pieces) {
            const int left = (pieces - i + LANES - 1) / LANES, take = left > 5 ? 4 : left;
            with_count<5>(take, [&](auto count) __attribute__((always_inline)) {
                constexpr int C = decltype(count)::value;
                float4 v[C][1];
                const int from = LANES == 256 ? i + (at & 63) : i + at;
                sums_at<C, 1>(W, U, [&](int k) __attribute__((always_inline)) { return base + 4 * (size_t)min(from + k * LANES, pieces - 1); }, v);    // (the last piece again past the end)
#pragma unroll
                for (int k = 0; k < C; ++k) m = max4(m, v[k][0]);
            });
            i += take * LANES;
        }
    } else {                                   // any alignment, any width: one float at a time
        for (int c = at; c < cols; c += LANES) {
            float v = W[base + c];
            if (U) v = __fadd_rn(v, U[base + c]);
            m = fmaxf(m, fabsf(v));
        }
    }
    m = lanes_max_f<LANES < 64 ? LANES : 64>(m);
    if constexpr (LANES == 256) {
        if (at % 64 == 0) part[wave] = m;
        __syncthreads();
        m = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    }
    if (at == 0) amax[row] = -m;
}

// Row maxima -> scales of the row groups, in place: one wavefront per group of rows_per_scale
// rows; s = largest magnitude / largest code (Sec. 3.3.1), 1 for an all-zero group.
__global__ void __launch_bounds__(256)
project_scale_kernel(float* __restrict__ s, int rows, int rows_per_scale, float qmax)
{
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const long long r0 = ((long long)blockIdx.x * 4 + wave) * rows_per_scale;
    if (r0 >= rows) return;
    const int r1 = (int)((r0 + rows_per_scale < rows) ? r0 + rows_per_scale : rows);
    float m = 0.0f;
    for (int r = (int)r0 + lane; r < r1; r += 64) m = fmaxf(m, fabsf(s[r]));
    m = wave_max_f(m);
    const float scale = scale_of_max(m, qmax);
    for (int r = (int)r0 + lane; r < r1; r += 64) s[r] = scale;
}

// Maxima and scales in one launch for scale groups of up to 16 values per lane, every value of the group in flight at
// once: LANES = 64, a wavefront per group (1024 values), or 256, a workgroup (4096).
template <int LANES>
__global__ void __launch_bounds__(256)
project_group_scale_kernel(const float* __restrict__ W, const float* __restrict__ U, int rows, int cols, int ldw, int rows_per_scale,
                           int groups, float qmax, float* __restrict__ s)
{
    __shared__ float part[4];
    const int wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6), lane = threadIdx.x & 63;
    const int group = LANES == 64 ? (int)blockIdx.x * 4 + wave : (int)blockIdx.x, at = LANES == 64 ? lane : (int)threadIdx.x;
    if (group >= groups) return;               // LANES = 256: none leaves before the barrier
    const int r0 = group * rows_per_scale, r1 = rows - r0 < rows_per_scale ? rows : r0 + rows_per_scale;
    const int width = cols / 4, pieces = (r1 - r0) * width, first = LANES == 64 ? 0 : 64 * wave;
    float m = 0.0f;
    if (first < pieces)
        with_count<4>((pieces - first + LANES - 1) / LANES, [&](auto count) __attribute__((always_inline)) {
            constexpr int C = decltype(count)::value;
            float4 v[C][1];
            sums_at<C, 1>(W, U, [&](int k) __attribute__((always_inline)) {
                const unsigned i = (unsigned)min(at + LANES * k, pieces - 1), r = i / (unsigned)width;
                return (size_t)(r0 + (int)r) * ldw + 4 * (size_t)(i - r * (unsigned)width);
            }, v);
#pragma unroll
            for (int k = 0; k < C; ++k) m = max4(m, v[k][0]);
        });
    m = wave_max_f(m);
    if constexpr (LANES == 256) {
        if (lane == 0) part[wave] = m;
        __syncthreads();
        m = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    }
    const float scale = scale_of_max(m, qmax);
    for (int r = r0 + at; r < r1; r += LANES) s[r] = scale;
}

// One group of M consecutive columns: z = Pi(v), the kept entries at scale s where bits > 0.
template <int M>
__device__ __forceinline__ void project_group(const float (&v)[M], int N, int bits, float s, float (&z)[M])
{
    const float qmax = (float)((1 << (bits ? bits - 1 : 7)) - 1);
    // Eq. 5 (offset 0), then Eq. 4: the value the integer code stands for (an integer code: its zero has no sign)
    auto requantised = [&](float x) {
        const int q = (int)fminf(fmaxf(rintf(__fdiv_rn(x, s)), -qmax), qmax);
        return __fmul_rn(s, (float)q);
    };
    if constexpr (M == 4) {
        if (N <= 2) {
            // Groups of four with one or two kept: the six pairwise comparisons decide every pair
            // (the lower column outranks on >=, the higher one otherwise), the keep flags follow
            // from them, and only the kept entries (the lowest and the highest kept column) are
            // quantised.
            const float a0 = fabsf(v[0]), a1 = fabsf(v[1]), a2 = fabsf(v[2]), a3 = fabsf(v[3]);
            const bool c01 = a0 >= a1, c02 = a0 >= a2, c03 = a0 >= a3, c12 = a1 >= a2, c13 = a1 >= a3, c23 = a2 >= a3;
            float z0, z1, z2, z3;
            if (N == 2) {
                auto under_two = [](bool p, bool q, bool r) { return !((p && q) || (p && r) || (q && r)); };
                const bool k0 = under_two(!c01, !c02, !c03), k1 = under_two(c01, !c12, !c13);
                const bool k2 = under_two(c02, c12, !c23), k3 = under_two(c03, c13, c23);
                float lo = k0 ? v[0] : (k1 ? v[1] : v[2]);
                float hi = k3 ? v[3] : (k2 ? v[2] : v[1]);
                if (bits) { lo = requantised(lo); hi = requantised(hi); }
                z0 = k0 ? lo : 0.0f;
                z1 = k1 ? (k0 ? hi : lo) : 0.0f;
                z2 = k2 ? (k3 ? lo : hi) : 0.0f;
                z3 = k3 ? hi : 0.0f;
            } else {
                const bool k0 = c01 && c02 && c03, k1 = !c01 && c12 && c13, k2 = !c02 && !c12 && c23;
                const bool k3 = !(k0 || k1 || k2);
                float kept = k0 ? v[0] : (k1 ? v[1] : (k2 ? v[2] : v[3]));
                if (bits) kept = requantised(kept);
                z0 = k0 ? kept : 0.0f; z1 = k1 ? kept : 0.0f; z2 = k2 ? kept : 0.0f; z3 = k3 ? kept : 0.0f;
            }
            z[0] = z0; z[1] = z1; z[2] = z2; z[3] = z3;
            return;
        }
    }
    // Eq. 3: an entry is kept when fewer than N entries outrank it; a larger magnitude outranks a
    // smaller one and, between equal magnitudes, the lower column the higher.
    float a[M];
#pragma unroll
    for (int c = 0; c < M; ++c) a[c] = fabsf(v[c]);
#pragma unroll
    for (int c = 0; c < M; ++c) {
        int outranked = 0;
#pragma unroll
        for (int d = 0; d < M; ++d) {
            if (d == c) continue;
            outranked += (d < c) ? (a[d] >= a[c]) : (a[d] > a[c]);
        }
        float kept_value = v[c];
        if (bits) kept_value = requantised(v[c]);
        z[c] = (outranked < N) ? kept_value : 0.0f;
    }
}

// P groups of M columns; at(i) is the place of the i-th.
template <int M, int P, bool TOGETHER = true, typename At>
__device__ __forceinline__ void load_groups(const float* W, const float* U, At at, float (&v)[P][M])
{
    float4 x[P][M / 4];
    sums_at<P, M / 4, TOGETHER>(W, U, at, x);
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int f = 0; f < M / 4; ++f) {
            v[i][4 * f + 0] = x[i][f].x; v[i][4 * f + 1] = x[i][f].y; v[i][4 * f + 2] = x[i][f].z; v[i][4 * f + 3] = x[i][f].w;
        }
}

template <int M>
__device__ __forceinline__ void store_group(const float (&v)[M], const float (&z)[M], float* Z, float* U_out, size_t at)
{
#pragma unroll
    for (int f = 0; f < M / 4; ++f) {
        *reinterpret_cast<float4*>(Z + at + 4 * f) = make_float4(z[4 * f + 0], z[4 * f + 1], z[4 * f + 2], z[4 * f + 3]);
        if (U_out)
            *reinterpret_cast<float4*>(U_out + at + 4 * f) =
                make_float4(__fsub_rn(v[4 * f + 0], z[4 * f + 0]), __fsub_rn(v[4 * f + 1], z[4 * f + 1]),
                            __fsub_rn(v[4 * f + 2], z[4 * f + 2]), __fsub_rn(v[4 * f + 3], z[4 * f + 3]));
    }
}

// In all three kernels U_out may be U (same leading dimension): no restrict on the two, and a lane reads
// every group it writes before it writes any.  (Lanes past a row's end load its last group and drop it.)

// One scale per row: WAVES wavefronts hold a row's values between its maximum and its projection, so W
// and U are read once.  16 columns per lane: rows of up to 1024 columns on one wavefront (four rows
// per workgroup), of up to 4096 on four.
template <int M, int WAVES>
__global__ void __launch_bounds__(256)
project_row_kernel(const float* __restrict__ W, const float* U, int rows, int cols, int ldw, int N, int bits,
                   float* __restrict__ scales, float* __restrict__ Z, float* U_out, int ldz)
{
    constexpr int P = 16 / M, STEP = 64 * WAVES;
    __shared__ float part[4];
    const int lane = threadIdx.x & 63, wave = threadIdx.x >> 6;
    const int row = WAVES == 1 ? blockIdx.x * 4 + wave : blockIdx.x;
    if (row >= rows) return;                   // WAVES > 1: one row per workgroup, none leaves before the barrier
    const int groups = cols / M, at = WAVES == 1 ? lane : (int)threadIdx.x;
    float v[P][M];
    load_groups<M, P>(W, U, [&](int i) __attribute__((always_inline)) { return (size_t)row * ldw + (size_t)min(at + i * STEP, groups - 1) * M; }, v);
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < P; ++i)
#pragma unroll
        for (int c = 0; c < M; ++c) m = fmaxf(m, fabsf(v[i][c]));
    m = wave_max_f(m);
    if constexpr (WAVES > 1) {
        if (lane == 0) part[wave] = m;
        __syncthreads();                       // (also: every lane of the row has its values before the first store)
        m = fmaxf(fmaxf(part[0], part[1]), fmaxf(part[2], part[3]));
    }
    const float s = scale_of_max(m, (float)((1 << (bits - 1)) - 1));
    if (at == 0) scales[row] = s;
#pragma unroll
    for (int i = 0; i < P; ++i) {
        if (at + i * STEP >= groups) break;
        float z[M];
        project_group<M>(v[i], N, bits, s, z);
        store_group<M>(v[i], z, Z, U_out, (size_t)row * ldz + (size_t)(at + i * STEP) * M);
    }
}

// One wavefront per PER * 64 groups of a row, `chunks` of them.  rows_per_scale > 0: scales[] holds the row maxima,
// negated, and this launch turns them into scales: the wavefront at a row's start writes the row's, while
// others still read.  A reader takes the largest of its group's values as signed integers: any scale (sign
// bit clear, and all rows of a group get the same one) is above every maximum, and among maxima (sign bit
// set) the larger magnitude is the larger integer.  So it ends with the scale itself or with the group's
// largest magnitude, whichever mixture it met.
// rows_per_scale = 0: scales[row] is final.
template <int M, int PER>
__global__ void __launch_bounds__(256)
project_wave_kernel(const float* __restrict__ W, const float* U, int rows, int cols, int ldw, int N, int bits, int rows_per_scale,
                    float* scales, float* __restrict__ Z, float* U_out, int ldz, int chunks)
{
    const int lane = threadIdx.x & 63;
    const unsigned id = (unsigned)__builtin_amdgcn_readfirstlane((int)(blockIdx.x * 4u + (threadIdx.x >> 6)));
    const int row = (int)(id / (unsigned)chunks), chunk = (int)(id - (unsigned)row * (unsigned)chunks);
    if (row >= rows) return;                   // no barrier below
    const int groups = cols / M, g0 = chunk * (64 * PER) + lane;
    float v[PER][M];
    load_groups<M, PER>(W, U, [&](int i) __attribute__((always_inline)) { return (size_t)row * ldw + (size_t)min(g0 + i * 64, groups - 1) * M; }, v);
    float s = 1.0f;
    if (bits && rows_per_scale > 0) {
        const int r0 = row / rows_per_scale * rows_per_scale, r1 = rows - r0 < rows_per_scale ? rows : r0 + rows_per_scale;
        int top = (int)0x80000000;             // the maximum of no row
        for (int r = r0 + lane; r < r1; r += 64)
            top = max(top, __hip_atomic_load(reinterpret_cast<int*>(scales) + r, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT));
        top = wave_max_i(top);
        s = __int_as_float(top);
        if (top < 0) s = scale_of_max(-s, (float)((1 << (bits - 1)) - 1));
        if (chunk == 0 && lane == 0)
            __hip_atomic_store(reinterpret_cast<int*>(scales) + row, __float_as_int(s), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
    } else if (bits) {
        s = scales[row];
    }
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        if (g0 + i * 64 >= groups) break;
        float z[M];
        project_group<M>(v[i], N, bits, s, z);
        store_group<M>(v[i], z, Z, U_out, (size_t)row * ldz + (size_t)(g0 + i * 64) * M);
    }
}

// One launch for scale groups of several rows: `parts` (up to 64) workgroups per scale group, each with its part of the group's
// values in registers (PER groups of M columns per thread), so W and U are read once.  The workgroups of a group tell one
// another their parts' maxima through a 64-bit word each: the call's number above, the maximum's bits below, so a word
// says by itself whether it belongs to this call, nothing has to be cleared and no order between two words matters.  They are neighbours
// on one XCD and start together; one that has waited `patience` turns for the others (a chip that is busy with something else)
// reads the rest of the group itself and waits no more.  So W and U must not change meanwhile: with several parts U_out is not U.
// magic = ceil(2^32 / (cols / 4)), which divides every number up to the group's 16-byte pieces exactly (the launcher's condition).
template <int M, int PER, int THREADS>
__global__ void __launch_bounds__(THREADS)
project_parts_kernel(const float* __restrict__ W, const float* U, int rows, int cols, int ldw, int N, int bits, int rows_per_scale,
                     int n_groups, int parts, uint32_t magic, float* __restrict__ scales, float* __restrict__ Z, float* U_out, int ldz,
                     uint32_t call, int patience)
{
    constexpr int F = M / 4;
    __shared__ float part_max[THREADS / 64];
    __shared__ float group_max;
    __shared__ int missing;
    const int tid = threadIdx.x, lane = tid & 63;
    const int total = n_groups * parts, per_xcd = (total + 7) >> 3;
    const int id = (int)(blockIdx.x & 7) * per_xcd + (int)(blockIdx.x >> 3);
    if (id >= total) return;                   // the whole workgroup
    const int group = id / parts, part = id - group * parts;
    const int r0 = group * rows_per_scale, n = rows - r0 < rows_per_scale ? rows - r0 : rows_per_scale;
    const int width = cols / 4, pieces = n * width;        // of 16 bytes
    const int own = (pieces / F + parts - 1) / parts * F;  // pieces of a part (the last ones may have fewer, or none)
    const int begin = min(part * own, pieces), end = min(begin + own, pieces);
    auto place = [&](int piece, int ld) __attribute__((always_inline)) {
        const int r = (int)__umulhi((uint32_t)piece, magic);
        return (size_t)(r0 + r) * ld + 4 * (size_t)(piece - r * width);
    };
    float v[PER][M];
    load_groups<M, PER>(W, U, [&](int i) __attribute__((always_inline)) { return place(min(begin + (tid + i * THREADS) * F, pieces - F), ldw); }, v);
    float m = 0.0f;
#pragma unroll
    for (int i = 0; i < PER; ++i)
#pragma unroll
        for (int c = 0; c < M; ++c) m = fmaxf(m, fabsf(v[i][c]));          // (a clamped place is one of the group's too)
    auto workgroup_max = [&]() __attribute__((always_inline)) {
        m = wave_max_f(m);
        if (lane == 0) part_max[tid >> 6] = m;
        __syncthreads();
        m = part_max[0];
#pragma unroll
        for (int w = 1; w < THREADS / 64; ++w) m = fmaxf(m, part_max[w]);
    };
    workgroup_max();
    if (parts > 1) {
        if (tid < 64) {
            unsigned long long* words = meet_words + (call % MEET_REGIONS) * MEET_WORDS + group * parts;
            if (lane == 0)
                __hip_atomic_store(words + part, ((unsigned long long)call << 32) | __float_as_uint(m), __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
            unsigned long long word = 0;
            bool here = lane >= parts;
            for (int turn = 0;; ++turn) {
                if (!here) {
                    word = __hip_atomic_load(words + lane, __ATOMIC_RELAXED, __HIP_MEMORY_SCOPE_AGENT);
                    here = (uint32_t)(word >> 32) == call;
                }
                if (__all(here) || turn >= patience) break;
                __builtin_amdgcn_s_sleep(1);
            }
            const float top = wave_max_f(fmaxf(here && lane < parts ? __uint_as_float((uint32_t)word) : 0.0f, m));
            const int all_here = __all(here);
            if (lane == 0) {
                group_max = top;
                missing = !all_here;
            }
        }
        __syncthreads();
        if (missing) {
            // from the end of this part round to its beginning
            const int rest = pieces - (end - begin);
            for (int i = tid; i < rest; i += 4 * THREADS) {
                float4 x[4][1];
                sums_at<4, 1>(W, U, [&](int k) __attribute__((always_inline)) {
                    const int q = min(i + k * THREADS, rest - 1) + end;
                    return place(q >= pieces ? q - pieces : q, ldw);
                }, x);
#pragma unroll
                for (int k = 0; k < 4; ++k) m = max4(m, x[k][0]);
            }
            workgroup_max();                   // (part_max: last read before the barrier above)
        } else {
            m = group_max;
        }
    }
    const float s = scale_of_max(m, (float)((1 << (bits - 1)) - 1));
    if (part == 0)
        for (int r = tid; r < n; r += THREADS) scales[r0 + r] = s;
#pragma unroll
    for (int i = 0; i < PER; ++i) {
        const int piece = begin + (tid + i * THREADS) * F;
        if (piece >= end) break;
        float z[M];
        project_group<M>(v[i], N, bits, s, z);
        store_group<M>(v[i], z, Z, U_out, place(piece, ldz));
    }
}

template <int M, int MOST, int THREADS, typename... Args>
void launch_project_parts_per(int per, unsigned blocks, hipStream_t st, Args... args)
{
    if constexpr (MOST > 1) {
        if (per < MOST) return launch_project_parts_per<M, MOST - 1, THREADS>(per, blocks, st, args...);
    }
    hipLaunchKernelGGL((project_parts_kernel<M, MOST, THREADS>), dim3(blocks), dim3(THREADS), 0, st, args...);
}

// A number for a call whose workgroups meet: 32 bits that no earlier call of this process had, 0 when there are none left (after
// 2^32 calls) or when the launch would be replayed with the number it has now (stream capture: such calls go by the other launches).
uint32_t meeting_call(hipStream_t st)
{
    static std::atomic<unsigned long long> calls{0};
    hipStreamCaptureStatus status = hipStreamCaptureStatusActive;
    if (hipStreamIsCapturing(st, &status) != hipSuccess) {
        (void)hipGetLastError();
        return 0;
    }
    if (status != hipStreamCaptureStatusNone) return 0;
    const unsigned long long call = 1 + calls.fetch_add(1, std::memory_order_relaxed);
    return call <= 0xFFFFFFFFull ? (uint32_t)call : 0;
}

// Whether project_parts_kernel takes the call, and its launch.  The lines, over 700 shapes (16 to 30522 rows, 8 to 8192 columns, 2 to
// 300 rows per scale, U given; launches one after the other, against the launches below): the mean is 0.72 of their time
// and none is slower by more than 6 % (0.6 us).  3072 x 768, 32 rows per scale 13.6 -> 12.3 us from HBM and 9.9 -> 8.4 from the last-level
// cache, 768 x 3072 15.7 -> 12.9 and 12.4 -> 9.2, 768 x 768 7.8 -> 6.6, 30522 x 768 106 -> 81; the 48 matrices of a BERT-base encoder 599 -> 504.
//  - 1024 threads where that still gives 128 workgroups, else 256 (768 x 768: 7.7 and 6.6; 30522 x 768: 81 and 106);
//  - up to 24 parts on 1024 threads, of which a CU holds two: an XCD then has room for all parts of a group at once (57 parts, 8192 x
//    3072 at 300 rows per scale, 104 -> 910 us); on 256 threads up to 64, and no more workgroups than the chip holds;
//  - many tiny groups leave most of a workgroup idle (15261 groups of 128 values 11.5 -> 15.0);
//  - above 20 million values in more than two parts the waiting workgroups' place is missed (8192 x 3072, 12 parts, 101 -> 106).
// The meeting does not suffer from a busy chip.  16 matrices of a BERT-base encoder, 32 rows per scale, against the launches below: beside a stream of
// large copies 350 -> 296 us, two streams projecting at once 295 -> 257, beside a stream of large products 7.6 ms (the wait for CUs)
// in both; patience of 4 to 4096 turns the same within 2 % but for two streams at 4 turns (276).
template <int M>
bool launch_project_parts(const float* W, const float* U, int rows, int cols, int ldw, int N, int bits, int rows_per_scale,
                          float* Z, float* U_out, int ldz, float* scales, hipStream_t st)
{
    constexpr int MOST = 16 / M;               // groups of M columns per thread
    const int span = rows_per_scale < rows ? rows_per_scale : rows, width = cols / 4;
    const long long n_groups = ((long long)rows + span - 1) / span, values = (long long)span * cols, elements = (long long)rows * cols;
    if (width < 2 || (values < 512 && n_groups > 2048) || values / 4 * width >= (1ll << 32) || n_groups > (1 << 20)) return false;
    long long parts = (values + 16 * 1024 - 1) / (16 * 1024);
    const bool wide = values > 16 * 256 && n_groups * parts >= 128;
    if (wide) {
        if (parts > 24 || (parts > 2 && elements > 20000000)) return false;
    } else {
        parts = (values + 16 * 256 - 1) / (16 * 256);
        if (parts > 64 || (parts > 1 && n_groups * parts > 2048)) return false;
    }
    if (parts > 1 && ((U_out == U && U) || n_groups * parts > MEET_WORDS)) return false;
    const uint32_t call = meeting_call(st);
    if (call == 0) return false;
    const int threads = wide ? 1024 : 256;
    const int per = (int)(((values / M + parts - 1) / parts + threads - 1) / threads);
    const unsigned blocks = (unsigned)(8 * ((n_groups * parts + 7) / 8));
    const uint32_t magic = (uint32_t)((0x100000000ull + width - 1) / width);
    const int patience = project_patience();
    if (wide)
        launch_project_parts_per<M, MOST, 1024>(per, blocks, st, W, U, rows, cols, ldw, N, bits, span, (int)n_groups, (int)parts, magic, scales, Z, U_out, ldz, call, patience);
    else
        launch_project_parts_per<M, MOST, 256>(per, blocks, st, W, U, rows, cols, ldw, N, bits, span, (int)n_groups, (int)parts, magic, scales, Z, U_out, ldz, call, patience);
    return true;
}

// `per` up to MOST
template <int M, int MOST, typename... Args>
void launch_project_wave(int per, unsigned blocks, hipStream_t st, Args... args)
{
    if constexpr (MOST > 1) {
        if (per < MOST) return launch_project_wave<M, MOST - 1>(per, blocks, st, args...);
    }
    hipLaunchKernelGGL((project_wave_kernel<M, MOST>), dim3(blocks), dim3(256), 0, st, args...);
}

// One thread per group of M consecutive columns, rows of any length one after the other; scales[row] is final.
// NARROW: the threads' numbers fit 32 bits.
template <int M, bool NARROW>
__global__ void __launch_bounds__(256)
project_kernel(const float* __restrict__ W, const float* U, int rows, int cols, int ldw,
               int N, int bits, const float* __restrict__ scales, float* __restrict__ Z, float* U_out, int ldz)
{
    const int groups = cols / M;
    const long long id = (long long)blockIdx.x * 256 + threadIdx.x, total = (long long)rows * groups;
    if (id >= total) return;
    uint32_t row, g;
    split_id(id, (uint32_t)groups, NARROW, row, g);
    const float s = bits ? scales[row] : 1.0f;
    float v[1][M], z[M];
    load_groups<M, 1, false>(W, U, [&](int) __attribute__((always_inline)) { return (size_t)row * ldw + (size_t)g * M; }, v);
    project_group<M>(v[0], N, bits, s, z);
    store_group<M>(v[0], z, Z, U_out, (size_t)row * ldz + (size_t)g * M);
}

// Lanes per row by the pieces a row has: a lane holds up to five, and fewer rows than fill the chip are better spread
// out.  30522 x 64: a wavefront per row 7.2 us, 16 lanes 3.6; 4096 x 768 maxima 5.8 -> 4.8 with all pieces in flight;
// 768 x 3072 on one wavefront per row is three rounds of loads one after the other on 768 wavefronts, 7.1 against 4.6.
void launch_row_maxima(const float* W, const float* U, int rows, int cols, int ldw, float* amax, int vec, hipStream_t st)
{
    if (cols <= 64 || (cols <= 256 && rows >= 8192))
        hipLaunchKernelGGL(project_amax_kernel<16>, dim3((rows + 15) / 16), dim3(256), 0, st, W, U, rows, cols, ldw, amax, vec);
    else if (cols <= 1280 || rows > (1 << 23))
        hipLaunchKernelGGL(project_amax_kernel<64>, dim3((rows + 3) / 4), dim3(256), 0, st, W, U, rows, cols, ldw, amax, vec);
    else
        hipLaunchKernelGGL(project_amax_kernel<256>, dim3(rows), dim3(256), 0, st, W, U, rows, cols, ldw, amax, vec);
}

void launch_max_to_scale(float* scales, int rows, int rows_per_scale, float qmax, hipStream_t st)
{
    const long long n_groups = ((long long)rows + rows_per_scale - 1) / rows_per_scale;
    hipLaunchKernelGGL(project_scale_kernel, dim3((unsigned)((n_groups + 3) / 4)), dim3(256), 0, st, scales, rows, rows_per_scale, qmax);
}

template <int M>
void launch_project_m(const float* W, const float* U, int rows, int cols, int ldw, int N, int bits, int rows_per_scale,
                      float* Z, float* U_out, int ldz, float* scales, hipStream_t st)
{
    const int groups = cols / M;
    const float qmax = (float)((1 << (bits ? bits - 1 : 7)) - 1);
    if (bits && rows_per_scale == 1 && cols <= 1024 && rows <= (1 << 25)) {
        hipLaunchKernelGGL((project_row_kernel<M, 1>), dim3((rows + 3) / 4), dim3(256), 0, st, W, U, rows, cols, ldw, N, bits, scales, Z, U_out, ldz);
        return;
    }
    if (bits && rows_per_scale == 1 && cols <= 4096 && cols > 1024 && rows <= (1 << 23)) {
        hipLaunchKernelGGL((project_row_kernel<M, 4>), dim3(rows), dim3(256), 0, st, W, U, rows, cols, ldw, N, bits, scales, Z, U_out, ldz);
        return;
    }
    if (bits && rows_per_scale > 1 &&
        launch_project_parts<M>(W, U, rows, cols, ldw, N, bits, rows_per_scale, Z, U_out, ldz, scales, st)) return;
    // Two ways to project.  project_wave_kernel has a row's groups in one or a few wavefronts, so it can form the
    // scales, and its loads are all in flight; project_kernel wastes no lane and needs no row of 64 groups.  Three ways to
    // the scales.  The lines below are where the measured times cross (16 to 30522 rows, 8 to 8192 columns, 1 to 300
    // rows per scale, U given; the first figure is maxima, scales and projection in three launches unless it says otherwise):
    //  - forming the scales in the projection saves a launch, which counts up to a few million values (4096 x 768, 2:4,
    //    32 rows per scale 17.0 -> 12.4 us; 768 x 4096 19.6 -> 12.9), while beyond, the second kernel is bound by its
    //    bytes and lanes without a group cost more (30522 x 776, 194 of 256 lanes used: 91.8 -> 95.8, so in three).  For
    //    M = 8 it stays ahead at any size (30522 x 640, 4:8: 82.2 -> 76.8): a thread of project_kernel has less in flight;
    //  - every wavefront reads its scale group's maxima: free up to 64 rows, later only with few wavefronts (256 rows per
    //    scale: 4096 x 768 17.9 -> 13.1, but 30522 x 768 93.7 -> 112, so in three);
    //  - small scale groups in a launch of their own (4096 x 128, 8 rows per scale 8.1 -> 5.5; 30522 x 8, 32 rows
    //    13.4 -> 4.5), except for wide rows of medium-sized matrices (4096 x 768, 2 rows per scale: 15.6, scales in the
    //    projection 12.4);
    //  - with final scales the wave kernel is ahead between 2 and 8 million values (4096 x 768, no scales 9.5 -> 8.1), for M =
    //    8 to 24 million.
    const int turns = (groups + 63) / 64;
    constexpr int P = 16 / M;                  // a lane holds 16 columns, 20 (M = 4) or 24 to save a nearly empty wavefront, one group in a small matrix
    const long long elements = (long long)rows * cols;
    const int by = (long long)rows * turns <= 2048 ? turns : (turns + (M == 4 ? 2 : 0)) / P;
    const int chunks = by > 0 ? by : 1, per = (turns + chunks - 1) / chunks;
    const long long waves = (long long)chunks * rows;
    const bool fits = groups >= 64 && waves <= (1 << 25);                          // (a launch holds fewer than 2^32 threads)
    const int used = (int)(groups * 100ll / (turns * 64ll));                       // percent of the lanes' loads that are the row's
    const int span = rows_per_scale < rows ? rows_per_scale : rows;                // rows of a full scale group
    const long long n_groups = ((long long)rows + rows_per_scale - 1) / rows_per_scale;
    const bool small_group = bits && (long long)span * cols <= 4096 && n_groups <= (1 << 23);
    const bool group_first = small_group && (elements <= (3 << 19) || (M == 4 ? cols <= 512 : used < 60 || elements >= (24 << 20)));
    const bool finish = bits && fits && (span <= 64 || (span <= 256 && waves <= 4096)) && !group_first &&
                        (M == 8 || elements < (1 << 20) || (used >= 60 && elements < (6 << 20)) || (used >= 90 && elements < (12 << 20)));
    if (bits && !finish && small_group) {
        // A wavefront per group where a workgroup would be mostly idle.  At 1024 values and above a workgroup's group is one
        // or more whole workgroups of project_kernel, which then finds W and U in its own XCD's L2 (30522 x 128, 8 rows
        // per scale 16.8 us, a wavefront per group 19.4).
        if ((long long)span * cols < 1024)
            hipLaunchKernelGGL(project_group_scale_kernel<64>, dim3((unsigned)((n_groups + 3) / 4)), dim3(256), 0, st, W, U, rows, cols, ldw,
                               rows_per_scale, (int)n_groups, qmax, scales);
        else
            hipLaunchKernelGGL(project_group_scale_kernel<256>, dim3((unsigned)n_groups), dim3(256), 0, st, W, U, rows, cols, ldw,
                               rows_per_scale, (int)n_groups, qmax, scales);
    } else if (bits) {
        launch_row_maxima(W, U, rows, cols, ldw, scales, 1, st);
        if (!finish) launch_max_to_scale(scales, rows, rows_per_scale, qmax, st);
    }
    if (finish || (fits && !small_group && used >= 60 && elements >= (2 << 20) && elements < (M == 4 ? 8 << 20 : 24 << 20)))
        launch_project_wave<M, M == 4 ? 5 : 3>(per, (unsigned)((waves + 3) / 4), st, W, U, rows, cols, ldw, N, bits, finish ? rows_per_scale : 0,
                                               scales, Z, U_out, ldz, chunks);
    else if ((long long)rows * groups <= 0xFFFFFFFFll)
        hipLaunchKernelGGL((project_kernel<M, true>), dim3((unsigned)(((long long)rows * groups + 255) / 256)), dim3(256), 0, st, W, U, rows, cols,
                           ldw, N, bits, scales, Z, U_out, ldz);
    else
        hipLaunchKernelGGL((project_kernel<M, false>), dim3((unsigned)(((long long)rows * groups + 255) / 256)), dim3(256), 0, st, W, U, rows, cols,
                           ldw, N, bits, scales, Z, U_out, ldz);
}

}  // namespace

// amax[row] <- -(largest |W|) of the row, any width and alignment.
void launch_row_maxima(const float* W, int rows, int cols, int ldw, float* amax, hipStream_t st)
{
    launch_row_maxima(W, nullptr, rows, cols, ldw, amax, ((uintptr_t)W % 16 == 0 && ldw % 4 == 0 && cols % 4 == 0) ? 1 : 0, st);
}

// scales[row] <- the scale of the row's group: largest |W| over the group's rows / qmax, 1 for an
// all-zero group.  Two launches, no workspace (scales[] first holds the rows' maxima, negated).
void launch_group_scales(const float* W, int rows, int cols, int ldw, int rows_per_scale, float qmax, float* scales,
                         hipStream_t st)
{
    launch_row_maxima(W, rows, cols, ldw, scales, st);
    launch_max_to_scale(scales, rows, rows_per_scale, qmax, st);
}

int launch_project(const float* W, const float* U, int rows, int cols, int ldw, int N, int M, int bits,
                   int rows_per_scale, float* Z, float* U_out, int ldz, float* scales, hipStream_t st)
{
    begin_launch();
    if (M == 4) launch_project_m<4>(W, U, rows, cols, ldw, N, bits, rows_per_scale, Z, U_out, ldz, scales, st);
    else launch_project_m<8>(W, U, rows, cols, ldw, N, bits, rows_per_scale, Z, U_out, ldz, scales, st);
    return launch_status();
}

}  // namespace nm
