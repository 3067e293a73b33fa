// nm_scale_search: the second scale rule of Sec. 3.3.1 ("ADMM-Dist") on gfx950 - per group of
// output neurons the scale that minimises the squared L2 distance between the kept parameters and
// their quantised values, searched over the candidate grid that the declaration in include/nm.h
// fixes (the paper states the criterion, not an algorithm).
//
// Three launches: the rows' largest magnitudes (into the scales array, negated), the error of every
// candidate per row (a workgroup or a wavefront per row, double precision, into the workspace), and per group
// the sum over its rows and the choice; the last two form the group's max-rule scale themselves.
// The per-row partial errors are the only scratch memory: [rows][candidates / 2 + 1] doubles.  Sums
// run in a fixed order (lane-strided partial sums, a fixed butterfly over the wavefront, then the
// rows of a group one after the other), so a call is deterministic; it is not the CPU's plain
// left-to-right order, so candidates whose errors agree to about 1e-15 relative can be ranked
// differently than there.
//
// The error launch is bound by arithmetic: about a dozen operations per kept weight and candidate, three
// of them in double.  The four wavefronts of a row share its candidates, not its columns, so a
// candidate's sum keeps its order and a matrix of 768 rows has 3072 wavefronts; the kept entries of a
// group are picked out first, so no lane idles on a column that is not kept; and the quotients come
// from the candidate's reciprocal (five operations, see nm_quantize.h) instead of a division.
// Measured against four wavefronts' rows per workgroup, every column tried under a mask, a division per quotient and
// the maxima turned into scales by a launch of their own (2:4 int8, 32 candidates, 32 rows per scale): the
// error launch 3072 x 768 41.1 -> 18.6 us, 768 x 3072 54.2 -> 22; the choice, which added 32 rows one load
// after the other, 11.6 -> 4.0; weights of a BERT-base layer to deployed ones 281 -> 146 us.
#include <hip/hip_runtime.h>
#include <stdint.h>

#include <mutex>

#include "nm.h"
#include "nm_internal.h"
#include "nm_quantize.h"

// Scratch of the entry point that allocates nothing (nm_scale_search_static): the rows' partial
// errors live in this array instead of a caller's workspace.  Every GPU the library runs on holds
// its own copy, at its own address, until the process ends.  In host code the name is only a handle
// for hipGetSymbolAddress - never a device address.
static __device__ __align__(256) unsigned char scratch[NM_SCALE_SEARCH_STATIC_MAX_BYTES];

namespace nm {

namespace {

__device__ __forceinline__ float candidate_scale(float smax, int c, int candidates)
{
    return __fdiv_rn(__fmul_rn(smax, (float)c), (float)candidates);
}

// The max-rule scale of rows r0 .. r1-1: from their maxima (negated) where `maxima`, else as it stands.
__device__ __forceinline__ float max_rule_scale(const float* scales, int r0, int r1, int maxima, float qmax, int lane)
{
    if (!maxima) return scales[r0];
    float m = 0.0f;
    for (int r = r0 + lane; r < r1; r += 64) m = fmaxf(m, fabsf(scales[r]));
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) m = fmaxf(m, __shfl_xor(m, d, 64));
    return (m == 0.0f) ? 1.0f : __fdiv_rn(m, qmax);
}

// CPW sums of one wavefront over a row: e[i] = sum over the kept entries of (w - s_i * q_i(w))^2, the
// candidates' scales in d[].  Columns in the order lane, lane + 64, ... (groups of M), kept entries of a group from
// the lowest column up.
template <int N, int M, int CPW, bool RECIP>
__device__ __forceinline__ void row_sums(const float* __restrict__ w, int groups, int lane, float qmax, const Divisor<RECIP> (&d)[CPW], double (&e)[CPW])
{
    double neg[CPW];
#pragma unroll
    for (int i = 0; i < CPW; ++i) {
        neg[i] = -(double)d[i].s;
        e[i] = 0.0;
    }
    float next[M];
    __builtin_memcpy(next, w + (size_t)min(lane, groups - 1) * M, 4 * M);
    for (int g = lane; g < groups; g += 64) {
        float v[M], a[M], kept[N];
#pragma unroll
        for (int c = 0; c < M; ++c) {
            v[c] = next[c];
            a[c] = fabsf(v[c]);
        }
        __builtin_memcpy(next, w + (size_t)min(g + 64, groups - 1) * M, 4 * M);
        if constexpr (N == M) {
#pragma unroll
            for (int c = 0; c < M; ++c) kept[c] = v[c];
        } else {
            bool nan = false;
#pragma unroll
            for (int c = 0; c < M; ++c) nan = nan || !(v[c] == v[c]);
            if constexpr (N == 2 && M == 4) {
                // the six comparisons decide every pair (the lower column outranks on >=); an entry is kept
                // when at most one outranks it
                const bool c01 = a[0] >= a[1], c02 = a[0] >= a[2], c03 = a[0] >= a[3], c12 = a[1] >= a[2], c13 = a[1] >= a[3], c23 = a[2] >= a[3];
                auto under_two = [](bool p, bool q, bool r) { return !((p && q) || (p && r) || (q && r)); };
                const bool k0 = under_two(!c01, !c02, !c03), k1 = under_two(c01, !c12, !c13);
                const bool k2 = under_two(c02, c12, !c23), k3 = under_two(c03, c13, c23);
                kept[0] = k0 ? v[0] : (k1 ? v[1] : v[2]);
                kept[1] = k3 ? v[3] : (k2 ? v[2] : v[1]);
            } else {
                int at = 0;
#pragma unroll
                for (int j = 0; j < N; ++j) kept[j] = 0.0f;
#pragma unroll
                for (int c = 0; c < M; ++c) {
                    // Eq. 3: kept when fewer than N entries outrank it (larger magnitude, or equal and a lower column)
                    int outranked = 0;
#pragma unroll
                    for (int k = 0; k < M; ++k) {
                        if (k == c) continue;
                        outranked += (k < c) ? (a[k] >= a[c]) : (a[k] > a[c]);
                    }
                    const bool keep = outranked < N;
#pragma unroll
                    for (int j = 0; j < N; ++j) kept[j] = (keep && at == j) ? v[c] : kept[j];
                    at += keep ? 1 : 0;
                }
            }
            // nothing outranks a NaN, so it is kept - maybe as one too many: it must reach the sum
            if (nan) kept[0] = __builtin_nanf("");
        }
#pragma unroll
        for (int j = 0; j < N; ++j) {
            const double x = (double)kept[j];
#pragma unroll
            for (int i = 0; i < CPW; ++i) {
                const float q = __builtin_amdgcn_fmed3f(rintf(d[i].quotient(kept[j])), -qmax, qmax);      // Eq. 5, offset 0 (of a NaN, r is one)
                const double r = __fma_rn(neg[i], (double)q, x);                               // (the product is exact: 31 bits)
                e[i] = __dadd_rn(e[i], __dmul_rn(r, r));
            }
        }
    }
}

// scales[]: the rows' maxima, negated (maxima != 0), or every row's max-rule scale.  err[row][k] = the row's
// sum for candidate k = c - candidates / 2.  WAVES = 4 wavefronts per row: wavefront w of the workgroup takes candidates
// w, w + 4, ...; WAVES = 1: a wavefront takes a row with all its candidates.
template <int N, int M, int WAVES, int CPW>
__global__ void __launch_bounds__(256)
row_errors_kernel(const float* __restrict__ W, int rows, int cols, int ldw, float qmax, int rows_per_scale, int maxima, int candidates,
                  const float* __restrict__ scales, double* __restrict__ err)
{
    const int lane = threadIdx.x & 63, wave = __builtin_amdgcn_readfirstlane((int)threadIdx.x >> 6);
    const int nc = candidates / 2 + 1;
    const int first = WAVES == 4 ? wave : 0;
    if (first >= nc) return;                   // no barrier below
    for (long long at = WAVES == 4 ? blockIdx.x : 4ll * blockIdx.x + wave; at < rows; at += (WAVES == 4 ? 1ll : 4ll) * gridDim.x) {
        const int row = (int)at;
        const int r0 = maxima ? row / rows_per_scale * rows_per_scale : row;
        const float smax = max_rule_scale(scales, r0, rows - r0 < rows_per_scale ? rows : r0 + rows_per_scale, maxima, qmax, lane);
        double e[CPW];
        float s[CPW];
#pragma unroll
        for (int i = 0; i < CPW; ++i) s[i] = candidate_scale(smax, candidates / 2 + min(first + WAVES * i, nc - 1), candidates);
        // The candidates lie between half of smax and smax, and |w| is at most 127 smax: within the range of the
        // reciprocal route, which holds up to |w| = 254 s as it does up to 127 s.
        if (smax >= 0x1p-59f && smax <= 0x1p60f) {
            Divisor<true> d[CPW];
#pragma unroll
            for (int i = 0; i < CPW; ++i) d[i] = Divisor<true>{s[i], __fdiv_rn(1.0f, s[i])};
            row_sums<N, M, CPW, true>(W + (size_t)row * ldw, cols / M, lane, qmax, d, e);
        } else {
            Divisor<false> d[CPW];
#pragma unroll
            for (int i = 0; i < CPW; ++i) d[i] = Divisor<false>{s[i], 0.0f};
            row_sums<N, M, CPW, false>(W + (size_t)row * ldw, cols / M, lane, qmax, d, e);
        }
#pragma unroll
        for (int i = 0; i < CPW; ++i) {
            double t = e[i];
#pragma unroll
            for (int d = 32; d >= 1; d >>= 1) t = __dadd_rn(t, __shfl_xor(t, d, 64));
            if (lane == 0 && first + WAVES * i < nc) err[(size_t)row * nc + first + WAVES * i] = t;
        }
    }
}

// One wavefront per scale group: lane k sums candidate k over the group's rows (sixteen loads in flight), then
// the least error wins, the larger scale between equal errors; every row of the group receives the scale.
__global__ void __launch_bounds__(64)
choose_scale_kernel(const double* __restrict__ err, int rows, int rows_per_scale, int maxima, float qmax, int candidates, float* scales)
{
    const int lane = threadIdx.x;
    const long long first = (long long)blockIdx.x * rows_per_scale;
    if (first >= rows) return;
    const int r0 = (int)first, r1 = rows - r0 < rows_per_scale ? rows : r0 + rows_per_scale;
    const int nc = candidates / 2 + 1;
    const double* mine = err + min(lane, nc - 1);
    double total = 0.0;
    for (int r = r0; r < r1; r += 16) {
        double t[16];
#pragma unroll
        for (int i = 0; i < 16; ++i) t[i] = mine[(size_t)min(r + i, r1 - 1) * nc];
#pragma unroll
        for (int i = 0; i < 16; ++i)
            if (r + i < r1) total = __dadd_rn(total, t[i]);
    }
    const float smax = max_rule_scale(scales, r0, r1, maxima, qmax, lane);       // read before any row of the group is overwritten (same wavefront)
    int best = lane < nc ? lane : -1;
    double best_err = total;
#pragma unroll
    for (int d = 32; d >= 1; d >>= 1) {
        const double oe = __shfl_xor(best_err, d, 64);
        const int ob = __shfl_xor(best, d, 64);
        const bool take = ob >= 0 && (best < 0 || oe < best_err || (oe == best_err && ob > best));
        best_err = take ? oe : best_err;
        best = take ? ob : best;
    }
    const float s = candidate_scale(smax, candidates / 2 + best, candidates);
    for (int r = r0 + lane; r < r1; r += 64) scales[r] = s;
}

template <int N, int M>
void launch_row_errors(const float* W, int rows, int cols, int ldw, float qmax, int rows_per_scale, int maxima, int candidates,
                       const float* scales, double* err, hipStream_t st)
{
    const int nc = candidates / 2 + 1;
    // Picking out the kept entries is work that every wavefront of a row repeats.  With few candidates it is most of the
    // work, and once the rows alone fill the chip a row is one wavefront's (7:8, 4096 x 3072, one row per scale: 2
    // candidates in the call, so 2 errors, 87 us on four wavefronts, 35.6 on one; 8, so 5, 87 and 49; 2:4, 4096 x 768, 32 rows
    // per scale, 2 candidates: 20.8 and 11.9).  The kernels are compiled for 2, 4 and 6 errors, and for 3, 5 and 9 on each of four wavefronts: 16, 32
    // and 64 candidates in the call need 9, 17 and 33; between them a few sums are formed in vain.
    const int wgs = nc <= 6 && rows >= 2048 ? (rows + 3) / 4 : rows;
    const dim3 grid((unsigned)(wgs < (1 << 20) ? wgs : (1 << 20))), wg(256);         // a launch holds fewer than 2^32 threads
#define NM_SHARE(w, n) hipLaunchKernelGGL((row_errors_kernel<N, M, w, n>), grid, wg, 0, st, W, rows, cols, ldw, qmax, rows_per_scale, maxima, candidates, scales, err)
    if (wgs != rows) {
        if (nc <= 2) NM_SHARE(1, 2);
        else if (nc <= 4) NM_SHARE(1, 4);
        else NM_SHARE(1, 6);
        return;
    }
    const int share = (nc + 3) / 4;            // candidates per wavefront: 1 .. 9
    if (share <= 3) NM_SHARE(4, 3);
    else if (share <= 5) NM_SHARE(4, 5);
    else NM_SHARE(4, 9);
#undef NM_SHARE
}

}  // namespace

int launch_scale_search(const float* W, int rows, int cols, int ldw, int N, int M, int bits, int rows_per_scale,
                        int candidates, float* scales, double* row_errors, hipStream_t st)
{
    begin_launch();
    const float qmax = (float)((1 << (bits - 1)) - 1);
    // Every workgroup of the second launch reads its group's maxima: cheaper than a launch that turns them
    // into scales up to a few hundred rows.
    const int maxima = rows_per_scale <= 256 ? 1 : 0;
    if (maxima) launch_row_maxima(W, rows, cols, ldw, scales, st);
    else launch_group_scales(W, rows, cols, ldw, rows_per_scale, qmax, scales, st);
#define NM_CASE(n, m) \
    if (N == n && M == m) launch_row_errors<n, m>(W, rows, cols, ldw, qmax, rows_per_scale, maxima, candidates, scales, row_errors, st)
    NM_CASE(1, 4); NM_CASE(2, 4); NM_CASE(3, 4); NM_CASE(4, 4);
    NM_CASE(1, 8); NM_CASE(2, 8); NM_CASE(3, 8); NM_CASE(4, 8); NM_CASE(5, 8); NM_CASE(6, 8); NM_CASE(7, 8); NM_CASE(8, 8);
#undef NM_CASE
    const long long n_groups = ((long long)rows + rows_per_scale - 1) / rows_per_scale;
    hipLaunchKernelGGL(choose_scale_kernel, dim3((unsigned)n_groups), dim3(64), 0, st, row_errors, rows, rows_per_scale, maxima, qmax, candidates, scales);
    return launch_status();
}

// The device address of `scratch` on the current device, looked up once per device (with that
// device current) and kept.  Returns 0, or NM_ERR_HIP.
static int static_scratch(void** out)
{
    constexpr int MAX_DEVICES = 64;
    static std::mutex lock;
    static void* address[MAX_DEVICES] = {};
    int dev = -1;
    if (hipGetDevice(&dev) != hipSuccess || dev < 0 || dev >= MAX_DEVICES) {
        fprintf(stderr, "libnm: nm_scale_search_static: no current device\n");
        return NM_ERR_HIP;
    }
    std::lock_guard<std::mutex> guard(lock);
    if (address[dev] == nullptr) {
        void* p = nullptr;
        const hipError_t e = hipGetSymbolAddress(&p, HIP_SYMBOL(scratch));
        if (e != hipSuccess || p == nullptr) {
            fprintf(stderr, "libnm: nm_scale_search_static: hipGetSymbolAddress failed on device %d: %s\n", dev, hipGetErrorString(e));
            return NM_ERR_HIP;
        }
        address[dev] = p;
    }
    *out = address[dev];
    return 0;
}

int launch_scale_search_static(const float* W, int rows, int cols, int ldw, int N, int M, int bits, int rows_per_scale,
                               int candidates, float* scales, hipStream_t st)
{
    void* p = nullptr;
    const int rc = static_scratch(&p);
    if (rc) return rc;
    // Nothing in the array has to start at zero: the second launch writes the partial errors of
    // every row and candidate of this call before the third reads exactly those.
    return launch_scale_search(W, rows, cols, ldw, N, M, bits, rows_per_scale, candidates, scales, static_cast<double*>(p), st);
}

}  // namespace nm
